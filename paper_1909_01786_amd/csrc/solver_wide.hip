// solver_wide.hip -- the search kernels for Deps of several words (W > 1).
//
// The same source as those for W = 1, a translation unit of its own so that the
// two compile side by side (a minute and a half each).
#define ASP_WIDE
#include "solver.hip"
