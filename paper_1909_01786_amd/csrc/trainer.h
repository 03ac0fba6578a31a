// trainer.h -- launch interface of the scorer's training kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace asp {

// Rows a backward kernel runs over.
enum { TR_NOGOODS = 0, TR_VARS = 1, TR_EMBED_NOGOODS = 2 };

// Partial sums of a backward kernel's team of waves: three matrices, a bias,
// the embedding's eight rows; at most kTrParts teams.
constexpr int kTrPart = 3 * 64 * 64 + 64 + 8 * 64;
constexpr int kTrParts = 768;

// Where the sums of a kernel's partials go: element i of segment k (src[k] +
// i of a partial) is added over the workgroups into dst[k][i].
struct TrSegs {
    int n = 0;
    int len[5];
    int64_t src[5];
    float* dst[5];
    void add(int64_t from, int count, float* to) {
        src[n] = from;
        len[n] = count;
        dst[n++] = to;
    }
};

// Row arrays come as float32 and, where a product reads them, as a bfloat16
// copy (uint16_t here).
hipError_t tr_embed_fwd(const float* X8, const float* E, const float* e, float* A, uint16_t* B,
                        int64_t rows, hipStream_t s);
hipError_t tr_layer_fwd(const int64_t* off, const int32_t* idx, const uint16_t* src,
                        const uint16_t* own, const float* scale, const float* W0, const float* W1,
                        const float* W2, const float* bias, float* A, uint16_t* B, int64_t rows,
                        hipStream_t s);
hipError_t tr_layer_bwd(int kind, const int64_t* off, const int32_t* idx, const float* g, float* own,
                        int has_own, const float* scale, const float* X1, const uint16_t* B1,
                        const uint16_t* B0, const float* X8, const float* Wa, const float* Wb,
                        const float* Wc, float* part, const TrSegs& sg, int64_t rows, hipStream_t s);
// Partials (2 * 64 + 2 floats each) that the readout's `part` takes.
int64_t tr_readout_waves(int64_t rows);
hipError_t tr_readout(const float* A, const float* y, const float* wo, const float* bo,
                      const float* scale, float* G, float* part, const TrSegs& sg, int64_t rows,
                      float inv_n, hipStream_t s);
hipError_t tr_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, int t,
                   const uint8_t* range, const float* lim, hipStream_t s);

}  // namespace asp
