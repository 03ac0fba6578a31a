// trainer.hip -- training kernels of the learned Decision's scorer (gfx950).
//
// The scorer of the score-driven Decision (a message-passing network over
// the bipartite graph of variables and static nogoods; the integer form in
// scorer.hip) is trained in its float form: activations a in [0, 1]
// (integer code / 256), matrices w in [-127/128, 127/128] (code / 128),
// biases b = code / 2^17, so that a layer
//     a' = clamp(u / 4 + b, 0, 1),   u = a S + norm(sum over edges of a_src P|N)
// is the integer layer act(z) = min(255, (z + 256) >> 9) divided by 256 up
// to its roundings.
//
// Every pass over the rows is one kernel: a tile of 64 rows gathers the sums
// of its neighbours' rows over its positive and over its negative edges (a
// product is linear, so multiplying the sums once by each sign's matrix is
// the sum of every edge's product), multiplies them and the tile's own rows
// by their matrices on the matrix cores, and applies the activation (or its
// mask) on the way out; the backward kernels also keep the tile's share of
// the weight gradients in accumulators over all their tiles.  The messages
// run along the two CSR orders of the literals (by nogood, by variable), so
// each direction and its gradient are gathers, never scattered atomics, and
// the weight gradients are added from one partial per workgroup: two runs
// give the same bits.
//
// What bounds them: the row arrays, 256 bytes of float32 a row and 128 of
// its bfloat16 copy, read and written once per kernel, and the gathers, a row
// per edge; the products are 64 wide, far from the matrix cores' rate.
// Precision: activations (rounded once, into the copy), matrices, and the
// backward edge sums enter the products as bfloat16, everything else is
// float32.  The forward sums of bfloat16 rows enter as three bfloat16 parts,
// all 24 bits, so a sum times a matrix is what the sum of its rows' products
// is, to float32 rounding.
// Measured on 64 programs (0.77M variable rows, 2.0M nogood rows, 4.6M edges):
// 63 ms a step with a kernel per product, edge sum and activation (75 of
// them, the column sums by atomics on 64 addresses), 10.6 ms so.
//
// Row arrays are [rows][64] float32, row-major.  Matrices are [in][out].
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "trainer.h"

namespace asp {
namespace {

#define DEV __device__ __forceinline__

constexpr int H = 64;
constexpr int NT = 256;          // threads per workgroup (four waves)
constexpr int TR = 64;           // rows per tile
constexpr int LDT = H + 8;       // LDS row stride of bf16 tiles (16-byte rows, bank offset)

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Element r of a 32x32 block held by `lane`: row (its column is lane % 32).
DEV int blk_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

typedef __bf16 Tile[TR * LDT];     // a 64x64 LDS operand

// acc += block (rb, cb), 32x32, of A B over K = 64: A's rows (stride LDT, k
// contiguous) and the rows of B's transpose.  Lane l supplies row / column
// l % 32 and k = 8 (l / 32) + 0..7 of each 16-wide k step.
DEV void mma(v16f& acc, const __bf16* A, int rb, const __bf16* BT, int cb, int lane) {
    const int kh = (lane >> 5) * 8;
    const int ia = (32 * rb + (lane & 31)) * LDT + kh, ib = (32 * cb + (lane & 31)) * LDT + kh;
#pragma unroll
    for (int k0 = 0; k0 < H; k0 += 16)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const v8bf*)(A + ia + k0),
                                                      *(const v8bf*)(BT + ib + k0), acc, 0, 0, 0);
}

// A weight matrix into LDS: BT[j][k] = W[k][j], or W[j][k] (trans).
DEV void stage_w(__bf16* T, const float* W, bool trans, int tid, int nt) {
    for (int i = tid; i < H * H; i += nt) {
        const int a = i >> 6, b = i & 63;
        T[trans ? a * LDT + b : b * LDT + a] = (__bf16)W[i];
    }
}

// A thread's share of a tile: row r, columns col_of(q, i), i < 16; four
// threads share a row.  Float32 rows: 16 t + 4 q + j, so that their loads
// read 64 contiguous bytes; bfloat16 rows: 32 t + 8 q + j, for the same.
DEV int col_f(int q, int i) { return 16 * (i >> 2) + 4 * q + (i & 3); }
DEV int col_b(int q, int i) { return 32 * (i >> 3) + 8 * q + (i & 7); }
DEV void load_row(float* v, const float* X, int64_t row, int q) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float4 x = *(const float4*)(X + row * H + 16 * t + 4 * q);
        v[4 * t] = x.x; v[4 * t + 1] = x.y; v[4 * t + 2] = x.z; v[4 * t + 3] = x.w;
    }
}
DEV void load_row(v8bf* v, const __bf16* X, int64_t row, int q) {
    v[0] = *(const v8bf*)(X + row * H + 8 * q);
    v[1] = *(const v8bf*)(X + row * H + 32 + 8 * q);
}
DEV void zero_row(float* v) {
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = 0.f;
}
DEV void zero_row(v8bf* v) { v[0] = v[1] = (v8bf)(0.f); }

// Row-major tiles: 16 floats rounded, or 16 bfloat16 as they are; and their
// transposes (tile row c holds column c, k = row).
DEV void stage(__bf16* T, const float* v, int r, int q) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        v4bf h;
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = (__bf16)v[4 * t + j];
        *(v4bf*)(T + r * LDT + 16 * t + 4 * q) = h;
    }
}
DEV void stage(__bf16* T, const v8bf* v, int r, int q) {
    *(v8bf*)(T + r * LDT + 8 * q) = v[0];
    *(v8bf*)(T + r * LDT + 32 + 8 * q) = v[1];
}
DEV void stage_t(__bf16* T, const float* v, int r, int q) {
#pragma unroll
    for (int i = 0; i < 16; ++i) T[col_f(q, i) * LDT + r] = (__bf16)v[i];
}
DEV void stage_t(__bf16* T, const v8bf* v, int r, int q) {
#pragma unroll
    for (int i = 0; i < 16; ++i) T[col_b(q, i) * LDT + r] = v[i >> 3][i & 7];
}
// 16 floats (bfloat16 columns) as three bfloat16 parts, x = T0 + T1 + T2.
DEV void stage3(Tile* T, const float* v, int r, int q) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        v8bf p0, p1, p2;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float x = v[8 * t + j];
            p0[j] = (__bf16)x;
            const float y = x - (float)p0[j];
            p1[j] = (__bf16)y;
            p2[j] = (__bf16)(y - (float)p1[j]);
        }
        const int at = r * LDT + 32 * t + 8 * q;
        *(v8bf*)(T[0] + at) = p0;
        *(v8bf*)(T[1] + at) = p1;
        *(v8bf*)(T[2] + at) = p2;
    }
}

// The sums of the edge sources' rows over a row's positive and negative
// edges (source idx >> 1, negative idx & 1), two edges in flight.
template <class X>
DEV void gather(float* sp, float* sn, const X* src, const int32_t* idx, int64_t e0, int64_t e1, int q) {
    zero_row(sp);
    zero_row(sn);
    for (int64_t e = e0; e < e1; e += 2) {
        const bool two = e + 1 < e1;
        const int32_t a = idx[e], b = two ? idx[e + 1] : a;
        float x[16], y[16];
        if constexpr (sizeof(X) == 2) {
            v8bf u[2], v[2];
            load_row(u, src, a >> 1, q);
            load_row(v, src, b >> 1, q);
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                x[t] = (float)u[t >> 3][t & 7];
                y[t] = (float)v[t >> 3][t & 7];
            }
        } else {
            load_row(x, src, a >> 1, q);
            load_row(y, src, b >> 1, q);
        }
        const bool na = a & 1, nb = b & 1;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            sp[t] += na ? 0.f : x[t];
            sn[t] += na ? x[t] : 0.f;
            sp[t] += two && !nb ? y[t] : 0.f;
            sn[t] += two && nb ? y[t] : 0.f;
        }
    }
}

// Tiles of one XCD (blockIdx % 8) are one stretch of the rows, taken by its
// workgroups side by side, so that the rows they gather -- those of the same
// programs -- are in that XCD's L2.  `at` is the first tile of a workgroup's
// first turn; its teams take at, at + 1, ...
struct Tiles {
    int64_t at, end, step;
};
DEV Tiles my_tiles(int64_t rows, int teams) {
    const int64_t nt = (rows + TR - 1) / TR;
    const int64_t x = blockIdx.x & 7, per = (nt + 7) / 8;
    Tiles t;
    t.at = x * per + (int64_t)(blockIdx.x >> 3) * teams;
    t.end = (x + 1) * per < nt ? (x + 1) * per : nt;
    t.step = (int64_t)(gridDim.x >> 3) * teams;
    return t;
}

// ------------------------------------------------------------ kernels
// Embedding: A[r] = clamp(X8[r] E / 4 + e, 0, 1) with 8 input features, and
// its bfloat16 copy B; four
// columns per thread, their entries of E in registers.
__global__ __launch_bounds__(NT) void k_embed_fwd(const float* X8, const float* E, const float* e,
                                                  float* A, __bf16* B, int64_t rows) {
    const int c = 4 * (threadIdx.x & 15);
    float4 w[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) w[f] = *(const float4*)(E + f * H + c);
    const float4 b = *(const float4*)(e + c);
    for (int64_t r = (int64_t)blockIdx.x * (NT / 16) + (threadIdx.x >> 4); r < rows;
         r += (int64_t)gridDim.x * (NT / 16)) {
        const float4 x0 = *(const float4*)(X8 + r * 8), x1 = *(const float4*)(X8 + r * 8 + 4);
        const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
        float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            z.x += x[f] * w[f].x;
            z.y += x[f] * w[f].y;
            z.z += x[f] * w[f].z;
            z.w += x[f] * w[f].w;
        }
        auto act = [](float u, float bias) {
            const float v = 0.25f * u + bias;
            return v <= 0.f ? 0.f : (v >= 1.f ? 1.f : v);
        };
        const float4 o = make_float4(act(z.x, b.x), act(z.y, b.y), act(z.z, b.z), act(z.w, b.w));
        *(float4*)(A + r * H + c) = o;
        *(v4bf*)(B + r * H + c) = (v4bf){(__bf16)o.x, (__bf16)o.y, (__bf16)o.z, (__bf16)o.w};
    }
}

// One layer's update of the rows: A = clamp((own W2 + scale (sum over
// positive edges of src W0 + over negative edges of src W1)) / 4 + b, 0, 1),
// and its bfloat16 copy B.  The teams (four waves, one tile each) share the
// matrices in LDS.
constexpr int kFwdTeams = 3;      // 110 KB of LDS, twelve waves per CU
__global__ __launch_bounds__(NT * kFwdTeams) void k_layer_fwd(const int64_t* off, const int32_t* idx,
                                                              const __bf16* src, const __bf16* own,
                                                              const float* scale, const float* W0,
                                                              const float* W1, const float* W2,
                                                              const float* bias, float* A, __bf16* B,
                                                              int64_t rows) {
    __shared__ __attribute__((aligned(16))) Tile sW[3];
    __shared__ __attribute__((aligned(16))) Tile sX[kFwdTeams][3];
    const int team = threadIdx.x / NT, tid = threadIdx.x % NT, w = tid >> 6, lane = tid & 63;
    const int r = 16 * w + (lane >> 2), q = lane & 3;
    const int rb = w & 1, cb = w >> 1;
    Tile* X = sX[team];
    stage_w(sW[0], W0, false, threadIdx.x, NT * kFwdTeams);
    stage_w(sW[1], W1, false, threadIdx.x, NT * kFwdTeams);
    stage_w(sW[2], W2, false, threadIdx.x, NT * kFwdTeams);
    const int col = 32 * cb + (lane & 31);
    const float bc = bias[col];
    const Tiles tl = my_tiles(rows, kFwdTeams);
    for (int64_t t0 = tl.at; t0 < tl.end; t0 += tl.step) {
        const int64_t t = t0 + team;
        const int64_t last = t < tl.end ? rows : 0;  // a team without a tile has no rows
        const int64_t row = t * TR + r;
        float sp[16], sn[16];
        v8bf o[2];
        zero_row(sp);
        zero_row(sn);
        zero_row(o);
        if (row < last) {
            load_row(o, own, row, q);
            gather(sp, sn, src, idx, off[row], off[row + 1], q);
            const float s = scale[row];              // a power of two
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                sp[i] *= s;
                sn[i] *= s;
            }
        }
        v16f acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            __syncthreads();
            stage3(X, p ? sn : sp, r, q);
            __syncthreads();
#pragma unroll
            for (int m = 2; m >= 0; --m) mma(acc, X[m], rb, sW[p], cb, lane);
        }
        __syncthreads();
        stage(X[0], o, r, q);
        __syncthreads();
        mma(acc, X[0], rb, sW[2], cb, lane);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t ro = t * TR + 32 * rb + blk_row(i, lane);
            float z = 0.25f * acc[i] + bc;
            z = z <= 0.f ? 0.f : (z >= 1.f ? 1.f : z);
            if (ro < last) {
                A[ro * H + col] = z;
                B[ro * H + col] = (__bf16)z;
            }
        }
    }
}

// The backward pass of one update.  The loss's derivative by the rows' new
// activations X1 is
//     dA = (sum over positive edges of g) Wa^T + (over negative ones) Wb^T + own Wc^T,
// g the neighbours' (scaled) derivatives, own the rows' own from the layer
// above; masked by 0 < X1 < 1 it gives the bias gradient, and over 4 the
// derivative G by the update's argument.  Weight gradients (of bfloat16
// copies B1, B0 of the activations): X1^T times each edge sum (the neighbours' update multiplied X1 by Wa and Wb).
//   kC: nogood rows; Wa, Wb = Q, R; own = G of the layer above (none at the
//       top), Wc = its S; and X0^T G, the gradient of this layer's S.
//   kV: variable rows; Wa, Wb = P, N; own = G of this layer's variable
//       update, Wc = T, with X1^T own, T's gradient.
//   kE: no edges (the nogood rows' embedding): own and Wc alone.
// `rows'` derivatives are kept scaled by the row's edge normaliser (a power
// of two), as the gathers need them; `own` and the result share the array.
// EMB: the rows come from the embedding: its gradient instead of a result.
// part: each team's [3][64][64] weight, [64] bias, [8][64] embedding
// gradients.
enum { kC = 0, kV = 1, kE = 2 };
constexpr int kBwdTeams = 3;      // 110 KB of LDS, twelve waves per CU
template <int KIND, bool EMB>
__global__ __launch_bounds__(NT * kBwdTeams) void k_layer_bwd(const int64_t* off, const int32_t* idx,
                                                              const float* g, float* own, int has_own,
                                                              const float* scale, const float* X1,
                                                              const __bf16* B1, const __bf16* B0,
                                                              const float* X8, const float* Wa,
                                                              const float* Wb, const float* Wc,
                                                              float* part, int64_t rows) {
    __shared__ __attribute__((aligned(16))) Tile sW[3];
    __shared__ __attribute__((aligned(16))) Tile sG[kBwdTeams];    // edge sums, or own: rows
    __shared__ __attribute__((aligned(16))) Tile sD[kBwdTeams];    // and transposed
    __shared__ __attribute__((aligned(16))) Tile sXT[kBwdTeams];   // B1, then B0, transposed
    const int team = threadIdx.x / NT, tid = threadIdx.x % NT, w = tid >> 6, lane = tid & 63;
    const int r = 16 * w + (lane >> 2), q = lane & 3;
    const int rb = w & 1, cb = w >> 1;
    __bf16 *G = sG[team], *D = sD[team], *XT = sXT[team];
    if (KIND != kE) {                                // B = W^T
        stage_w(sW[0], Wa, true, threadIdx.x, NT * kBwdTeams);
        stage_w(sW[1], Wb, true, threadIdx.x, NT * kBwdTeams);
    }
    if (has_own) stage_w(sW[2], Wc, true, threadIdx.x, NT * kBwdTeams);
    v16f dw[3];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int i = 0; i < 16; ++i) dw[m][i] = 0.f;
    float db = 0.f, de[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) de[f] = 0.f;
    const int col = 32 * cb + (lane & 31);
    const Tiles tl = my_tiles(rows, kBwdTeams);
    for (int64_t t0 = tl.at; t0 < tl.end; t0 += tl.step) {
        const int64_t t = t0 + team;
        const int64_t last = t < tl.end ? rows : 0;  // a team without a tile has no rows
        const int64_t row = t * TR + r;
        v16f acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        if (KIND != kE) {
            float sp[16], sn[16];
            v8bf x[2];
            zero_row(sp);
            zero_row(sn);
            zero_row(x);
            if (row < last) {
                load_row(x, B1, row, q);
                gather(sp, sn, g, idx, off[row], off[row + 1], q);
            }
            __syncthreads();
            stage_t(XT, x, r, q);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if (p) __syncthreads();
                stage(G, p ? sn : sp, r, q);
                stage_t(D, p ? sn : sp, r, q);
                __syncthreads();
                mma(acc, G, rb, sW[p], cb, lane);
                mma(dw[p], XT, rb, D, cb, lane);
            }
        }
        if (has_own) {
            float o[16];
            zero_row(o);
            if (row < last) {
                load_row(o, own, row, q);
                const float s = 1.f / scale[row];    // exact: a power of two
#pragma unroll
                for (int i = 0; i < 16; ++i) o[i] *= s;
            }
            __syncthreads();
            stage(G, o, r, q);
            if (KIND == kV) stage_t(D, o, r, q);
            __syncthreads();
            mma(acc, G, rb, sW[2], cb, lane);
            if (KIND == kV) mma(dw[2], XT, rb, D, cb, lane);
        }
        v8bf x0[2];
        zero_row(x0);
        if (KIND == kC && row < last) load_row(x0, B0, row, q);
        __syncthreads();
        if (KIND == kC) stage_t(XT, x0, r, q);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v4bf h;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = 4 * u + j;
                const int64_t ro = t * TR + 32 * rb + blk_row(i, lane);
                float d = 0.f;
                if (ro < last) {
                    const float a = X1[ro * H + col];
                    d = a > 0.f && a < 1.f ? acc[i] : 0.f;
                }
                db += d;
                d *= 0.25f;
                if (EMB) {
                    if (ro < last) {
                        const float4 f0 = *(const float4*)(X8 + ro * 8), f1 = *(const float4*)(X8 + ro * 8 + 4);
                        de[0] += d * f0.x; de[1] += d * f0.y; de[2] += d * f0.z; de[3] += d * f0.w;
                        de[4] += d * f1.x; de[5] += d * f1.y; de[6] += d * f1.z; de[7] += d * f1.w;
                    }
                } else if (ro < last) {
                    own[ro * H + col] = d * scale[ro];
                }
                h[j] = (__bf16)d;
            }
            if (KIND == kC)                          // rows 8 u + 4 (lane / 32) + 0..3 of column col
                *(v4bf*)(D + col * LDT + 32 * rb + 8 * u + 4 * (lane >> 5)) = h;
        }
        if (KIND == kC) {
            __syncthreads();
            mma(dw[2], XT, rb, D, cb, lane);
        }
    }
    // this team's partial sums
    float* P = part + (size_t)(blockIdx.x * kBwdTeams + team) * kTrPart;
    if (KIND != kE) {
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int i = 0; i < 16; ++i) P[m * H * H + (32 * rb + blk_row(i, lane)) * H + col] = dw[m][i];
    }
    // column sums: lanes l and l + 32 of the two waves of a column half
    __syncthreads();
    float* red = (float*)G;                          // [9][2][2][64]
#pragma unroll
    for (int f = 0; f < 9; ++f) red[((f * 2 + rb) * 2 + (lane >> 5)) * H + col] = f ? de[f - 1] : db;
    __syncthreads();
    for (int i = tid; i < 9 * H; i += NT) {
        const int f = i >> 6, c = i & 63;
        const float* p = red + f * 4 * H + c;
        P[3 * H * H + i] = (p[0] + p[H]) + (p[2 * H] + p[3 * H]);
    }
}

// G[dst + i] (or loss) = sum over the workgroups' partials of element i of
// each segment; 64 elements per workgroup, four threads each.
__global__ __launch_bounds__(NT) void k_sum_parts(const float* part, int64_t stride, int n, TrSegs sg) {
    __shared__ float red[4][H];
    const int c = threadIdx.x & 63, k = threadIdx.x >> 6;
    int i = (int)blockIdx.x * H + c, seg = 0;
    while (seg < sg.n && i >= sg.len[seg]) i -= sg.len[seg++];
    float s = 0.f;
    if (seg < sg.n) {
        const float* p = part + sg.src[seg] + i;
        for (int j = k; j < n; j += 4) s += p[(size_t)j * stride];
    }
    red[k][c] = s;
    __syncthreads();
    if (k == 0 && seg < sg.n) sg.dst[seg][i] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

// Readout and loss: for each labelled row (y >= 0), z = A wo + bo; the loss
// adds softplus(z) - y z (binary cross-entropy with logits) / n_lab; the
// derivative by the row's activations, (sigmoid(z) - y) / n_lab wo, is
// masked and scaled as the backward kernels' results are.  One wave per
// row, about sixteen rows a wave.  part, a wave each: [64] by wo, [64] by the
// last bias, by bo, the loss.
constexpr int kReadout = 2 * H + 2;
__global__ __launch_bounds__(NT) void k_readout(const float* A, const float* y, const float* wo,
                                                const float* bo, const float* scale, float* G,
                                                float* part, int64_t rows, float inv_n) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t waves = (int64_t)gridDim.x * (NT / 64);
    float gw = 0.f, db = 0.f, gb = 0.f, ls = 0.f;
    const float w = wo[lane], b0 = bo[0];
    for (int64_t r = (int64_t)blockIdx.x * (NT / 64) + wv; r < rows; r += waves) {
        const float lab = y[r];
        if (lab < 0.f) {
            G[r * H + lane] = 0.f;
            continue;
        }
        const float a = A[r * H + lane];
        float z = a * w;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) z += __shfl_xor(z, d, 64);
        z += b0;
        const float p = 1.f / (1.f + __expf(-z));
        const float g = (p - lab) * inv_n;
        const float d = a > 0.f && a < 1.f ? g * w : 0.f;
        G[r * H + lane] = 0.25f * d * scale[r];
        gw += g * a;
        db += d;
        if (lane == 0) {
            gb += g;
            ls += (fmaxf(z, 0.f) - z * lab + log1pf(__expf(-fabsf(z)))) * inv_n;
        }
    }
    float* o = part + ((size_t)blockIdx.x * (NT / 64) + wv) * kReadout;
    o[lane] = gw;
    o[H + lane] = db;
    if (lane == 0) {
        o[2 * H] = gb;
        o[2 * H + 1] = ls;
    }
}

// The readout's sums: each column one float32 running sum over the waves'
// partials, in their order, so that two runs give the same bits.  A running
// sum this long rounds: at 0.8M rows the loss and the last bias's gradient are
// 1e-5 to 4e-5 from a sum over a tree, which is nearer to the exact value and
// has no serial chain.  It is kept because these sums were running ones before
// (atomics, in the order of arrival): losses and Adam steps stay within
// rounding of those of earlier training runs, and a tree moved them by more.
// One workgroup: a thread per column adds a chunk in LDS while all threads
// load the next.  The chain of additions bounds it (48 thousand partials on
// 64 programs; their loads alone would take 5 us).
constexpr int kRunRows = 128, kRunT = 1024;
__global__ __launch_bounds__(kRunT) void k_running_sums(const float* part, int64_t n, TrSegs sg) {
    __shared__ __attribute__((aligned(16))) float buf[2][kRunRows * kReadout];
    constexpr int N4 = kRunRows * kReadout / 4, PER = (N4 + kRunT - 1) / kRunT;
    const int tid = threadIdx.x;
    const int64_t all = n * kReadout;
    float4 x[PER];
    auto load = [&](int64_t row) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = tid + k * kRunT;
            const int64_t at = row * kReadout + 4 * (int64_t)i;
            x[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i >= N4) continue;
            if (at + 4 <= all) {
                x[k] = *(const float4*)(part + at);
            } else {
                if (at < all) x[k].x = part[at];
                if (at + 1 < all) x[k].y = part[at + 1];
                if (at + 2 < all) x[k].z = part[at + 2];
            }
        }
    };
    auto keep = [&](float* b) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (tid + k * kRunT < N4) ((float4*)b)[tid + k * kRunT] = x[k];
    };
    float s = 0.f;
    load(0);
    keep(buf[0]);
    __syncthreads();
    int cur = 0;
    for (int64_t r = 0; r < n; r += kRunRows) {
        load(r + kRunRows);
        if (tid < kReadout) {
            const float* b = buf[cur] + tid;
#pragma unroll 32
            for (int i = 0; i < kRunRows; ++i) s += b[i * kReadout];
        }
        keep(buf[cur ^ 1]);
        __syncthreads();
        cur ^= 1;
    }
    if (tid >= kReadout) return;
    for (int k = 0; k < sg.n; ++k)
        if (tid >= sg.src[k] && tid < sg.src[k] + sg.len[k]) sg.dst[k][tid - sg.src[k]] = s;
}

// Adam (beta1 0.9, beta2 0.999, eps 1e-8) on n parameters at step t (1-based);
// then each parameter is clipped to [-lim[k], lim[k]] of its range k
// (matrices: the weight codes' range; biases: the bias codes' range).
__global__ __launch_bounds__(NT) void k_adam(float* p, const float* g, float* m, float* v,
                                             int64_t n, float lr, float bc1, float bc2,
                                             const uint8_t* range, const float* lim) {
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const float gi = g[i];
        const float mi = 0.9f * m[i] + 0.1f * gi;
        const float vi = 0.999f * v[i] + 0.001f * gi * gi;
        m[i] = mi;
        v[i] = vi;
        float x = p[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + 1e-8f);
        const float L = lim[range[i]];
        p[i] = x < -L ? -L : (x > L ? L : x);
    }
}

}  // namespace

// ------------------------------------------------------------ launchers
static int grid_for(int64_t work, int per_wg) {
    int64_t g = (work + per_wg - 1) / per_wg;
    if (g < 1) g = 1;
    return g > 65536 ? 65536 : (int)g;
}

// Workgroups of a kernel over row tiles: a multiple of eight (one share per
// XCD), no more than its tiles need, at most one per CU (which its LDS fills).
static int tile_grid(int64_t rows, int teams) {
    const int64_t g = ((rows + TR - 1) / TR + 8 * teams - 1) / (8 * teams) * 8;
    return (int)(g < 256 ? g : 256);
}

hipError_t tr_embed_fwd(const float* X8, const float* E, const float* e, float* A, uint16_t* B,
                        int64_t rows, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int g = grid_for(rows, NT / 16);
    hipLaunchKernelGGL(k_embed_fwd, dim3(g < 2048 ? g : 2048), dim3(NT), 0, s, X8, E, e, A,
                       (__bf16*)B, rows);
    return hipGetLastError();
}

hipError_t tr_layer_fwd(const int64_t* off, const int32_t* idx, const uint16_t* src,
                        const uint16_t* own, const float* scale, const float* W0, const float* W1,
                        const float* W2, const float* bias, float* A, uint16_t* B, int64_t rows,
                        hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_layer_fwd, dim3(tile_grid(rows, kFwdTeams)), dim3(NT * kFwdTeams), 0, s, off, idx,
                       (const __bf16*)src, (const __bf16*)own, scale, W0, W1, W2, bias, A, (__bf16*)B, rows);
    return hipGetLastError();
}

static hipError_t sum_parts(const float* part, int64_t stride, int n, const TrSegs& sg, hipStream_t s) {
    int tot = 0;
    for (int i = 0; i < sg.n; ++i) tot += sg.len[i];
    hipLaunchKernelGGL(k_sum_parts, dim3((tot + H - 1) / H), dim3(NT), 0, s, part, stride, n, sg);
    return hipGetLastError();
}

hipError_t tr_layer_bwd(int kind, const int64_t* off, const int32_t* idx, const float* g, float* own,
                        int has_own, const float* scale, const float* X1, const uint16_t* B1,
                        const uint16_t* B0, const float* X8, const float* Wa, const float* Wb, const float* Wc,
                        float* part, const TrSegs& sg, int64_t rows, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int grid = tile_grid(rows, kBwdTeams);
#define ASP_BWD(K, EMB)                                                                            \
    hipLaunchKernelGGL((k_layer_bwd<K, EMB>), dim3(grid), dim3(NT * kBwdTeams), 0, s, off, idx, g, own, has_own, \
                       scale, X1, (const __bf16*)B1, (const __bf16*)B0, X8, Wa, Wb, Wc, part, rows)
    if (kind == TR_NOGOODS) ASP_BWD(kC, false);
    else if (kind == TR_VARS && X8) ASP_BWD(kV, true);
    else if (kind == TR_VARS) ASP_BWD(kV, false);
    else ASP_BWD(kE, true);
#undef ASP_BWD
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return sum_parts(part, kTrPart, grid * kBwdTeams, sg, s);
}

int64_t tr_readout_waves(int64_t rows) {
    return (int64_t)grid_for(rows, (NT / 64) * 16) * (NT / 64);
}

hipError_t tr_readout(const float* A, const float* y, const float* wo, const float* bo,
                      const float* scale, float* G, float* part, const TrSegs& sg, int64_t rows,
                      float inv_n, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int grid = tr_readout_waves(rows) / (NT / 64);
    hipLaunchKernelGGL(k_readout, dim3(grid), dim3(NT), 0, s, A, y, wo, bo, scale, G, part, rows, inv_n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_running_sums, dim3(1), dim3(kRunT), 0, s, part, (int64_t)grid * (NT / 64), sg);
    return hipGetLastError();
}

hipError_t tr_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, int t,
                   const uint8_t* range, const float* lim, hipStream_t s) {
    const float bc1 = 1.f - powf(0.9f, (float)t), bc2 = 1.f - powf(0.999f, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n, NT)), dim3(NT), 0, s, p, g, m, v, n, lr, bc1, bc2,
                       range, lim);
    return hipGetLastError();
}

}  // namespace asp
