// Learned subgraph scorer: a three-layer MLP (kScorerIn -> 256 -> 256 -> 1,
// ReLU) with BF16 weights and activations and FP32 accumulation.  The two
// wide layers and their gradients run on the matrix cores
// (v_mfma_f32_32x32x16_bf16); the 256 -> 1 head, the loss, the bias sums
// and the Adam update are plain FP32 vector code.  A training step is two
// launches: everything that is local to a block of 32 batch rows (forward,
// loss, the gradients of the activations), then everything summed over the
// batch (the weights' gradients, each with its Adam update).  It scores candidate
// unions of UnionDP's partition phase (Section 4.2) and is trained on plans
// the exact DP produces (mpdp_scorer.h).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "mpdp.h"
#include "mpdp_scorer.h"

namespace {

constexpr int kIn = MPDP_SCORER_IN;
constexpr int kHid = MPDP_SCORER_HIDDEN;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(uint16_t)))) uint16_t u16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round to nearest even; NaN stays NaN
__device__ __forceinline__ uint16_t f2bf(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Device parameter block: FP32 master values, BF16 working copies,
// gradients and Adam moments, all in one allocation (offsets: scorer_layout).
struct Params {
    float *w1, *b1, *w2, *b2, *w3, *b3;           // master
    uint16_t *w1h, *w2h, *w3h;                     // bf16 copies used by the forward pass
    float *g;                                      // gradients, same order as the master values
    float *m, *v;                                  // Adam moments
};

constexpr size_t kN1 = (size_t)kIn * kHid, kN2 = (size_t)kHid * kHid, kN3 = kHid;
constexpr size_t kNParams = kN1 + kHid + kN2 + kHid + kN3 + 1;

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
    size_t master, bf, grad, m, v, total;
};

Layout scorer_layout() {
    Layout L{};
    size_t o = 0;
    L.master = o; o = up256(o + 4 * kNParams);
    L.bf = o;     o = up256(o + 2 * (kN1 + kN2 + kN3));
    L.grad = o;   o = up256(o + 4 * kNParams);
    L.m = o;      o = up256(o + 4 * kNParams);
    L.v = o;      o = up256(o + 4 * kNParams);
    L.total = o;
    return L;
}

Params params_at(void *base) {
    const Layout L = scorer_layout();
    char *b = static_cast<char *>(base);
    Params p;
    float *mst = reinterpret_cast<float *>(b + L.master);
    p.w1 = mst;
    p.b1 = p.w1 + kN1;
    p.w2 = p.b1 + kHid;
    p.b2 = p.w2 + kN2;
    p.w3 = p.b2 + kHid;
    p.b3 = p.w3 + kN3;
    uint16_t *h = reinterpret_cast<uint16_t *>(b + L.bf);
    p.w1h = h;
    p.w2h = h + kN1;
    p.w3h = h + kN1 + kN2;
    p.g = reinterpret_cast<float *>(b + L.grad);
    p.m = reinterpret_cast<float *>(b + L.m);
    p.v = reinterpret_cast<float *>(b + L.v);
    return p;
}

// Work buffer of one batch: activations and their gradients.
struct Work {
    uint16_t *h1, *h2, *dz2, *dz1;  // batch x 256 bf16
    float *row_loss, *dlogit;       // batch
    float *loss;                    // 1 (sum over the batch)
};

size_t work_bytes(uint32_t batch) {
    return up256(2 * (size_t)batch * kHid) * 4 + up256(4 * (size_t)batch) * 2 + 256;
}

Work work_at(void *base, uint32_t batch) {
    char *b = static_cast<char *>(base);
    const size_t a = up256(2 * (size_t)batch * kHid), f = up256(4 * (size_t)batch);
    Work w;
    w.h1 = reinterpret_cast<uint16_t *>(b);
    w.h2 = reinterpret_cast<uint16_t *>(b + a);
    w.dz2 = reinterpret_cast<uint16_t *>(b + 2 * a);
    w.dz1 = reinterpret_cast<uint16_t *>(b + 3 * a);
    w.row_loss = reinterpret_cast<float *>(b + 4 * a);
    w.dlogit = reinterpret_cast<float *>(b + 4 * a + f);
    w.loss = reinterpret_cast<float *>(b + 4 * a + 2 * f);
    return w;
}

// ---------------------------------------------------------------- matrix cores
//
// v_mfma_f32_32x32x16_bf16, C (32 x 32) += A (32 x 16) B (16 x 32): lane l
// supplies A(i, k) for i = l % 32 and k = 8 (l / 32) + 0..7, and B(k, j) for
// j = l % 32 and the same k; it holds C(i, j) for j = l % 32 and
// i = 8 (r / 4) + 4 (l / 32) + r % 4, r = 0..15.

__device__ __forceinline__ floatx16 mfma(const u16x8 &a, const u16x8 &b, const floatx16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

__device__ __forceinline__ int c_row(int lane, int r) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Eight values M(k, j), k = k0 .. k0 + 7, of a row-major matrix: one column.
__device__ __forceinline__ u16x8 column8(const uint16_t *__restrict__ m, int ld, int k0, int j) {
    u16x8 v;
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = m[(size_t)(k0 + t) * ld + j];
    return v;
}

// The same where rows from `rows` on count as zero.
__device__ __forceinline__ u16x8 column8_below(const uint16_t *__restrict__ m, int ld, uint32_t k0, int j,
                                               uint32_t rows) {
    u16x8 v;
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = k0 + (uint32_t)t < rows ? m[(size_t)(k0 + t) * ld + j] : (uint16_t)0;
    return v;
}

// Eight consecutive values, as one 16-byte access where the caller's buffers
// are aligned for it (`vec`, uniform), else one by one.
__device__ __forceinline__ u16x8 load8(const uint16_t *__restrict__ p, bool vec) {
    if (vec) return *reinterpret_cast<const u16x8 *>(p);
    u16x8 v;
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = p[t];
    return v;
}

__device__ __forceinline__ void store8(uint16_t *__restrict__ p, const u16x8 &v, bool vec) {
    if (vec) {
        *reinterpret_cast<u16x8 *>(p) = v;
    } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) p[t] = v[t];
    }
}

// ---------------------------------------------------------------- rows

constexpr int kRowBlock = 32;                 // batch rows of a workgroup
constexpr int kRowThreads = 512;              // eight waves, 32 of the 256 columns each
constexpr int kLd = kHid + 8;                 // LDS row stride: 16-byte reads of 32 rows spread over the banks
constexpr int kMfmaK = 16;

// Everything of a batch row but the weights' gradients, 32 rows to a
// workgroup, so that the activations pass from layer to layer through LDS:
// h1, h2, the logits (j ascending, FP32, then b3) and, for training, the
// loss of each row (max(l, 0) - l y + log1p(exp(-|l|))), dlogit =
// (sigmoid(l) - y) / batch, dz2 = bf16(h2 > 0 ? dlogit w3 : 0) and
// dz1 = bf16(h1 > 0 ? dz2 w2^T : 0).  The K steps of every product run in
// ascending order in one accumulator, whatever the batch.  Bound by latency:
// 512 rows occupy 16 CUs (16.7 us); each wave reads its 32 columns of w2 (16
// KB) once for each direction.
template <bool kTrain>
__global__ __launch_bounds__(kRowThreads) void k_rows(const uint16_t *__restrict__ x, const float *__restrict__ y,
                                                      uint32_t batch, const uint16_t *__restrict__ w1h,
                                                      const float *__restrict__ b1, const uint16_t *__restrict__ w2h,
                                                      const float *__restrict__ b2, const uint16_t *__restrict__ w3h,
                                                      const float *__restrict__ b3, float *__restrict__ logits,
                                                      Work w, bool vec) {
    __shared__ __align__(16) uint16_t h1[kRowBlock][kLd];
    __shared__ __align__(16) uint16_t h2[kRowBlock][kLd];
    __shared__ __align__(16) uint16_t dz[kRowBlock][kLd];
    __shared__ float w3[kHid], dl[kRowBlock];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    const int i = lane & 31, kq = 8 * (lane >> 5), j = 32 * wave + (lane & 31);
    const uint32_t row0 = blockIdx.x * kRowBlock;
    const bool have = row0 + (uint32_t)i < batch;
    if (t < kHid) w3[t] = bf2f(w3h[t]);

    floatx16 acc = {};
#pragma unroll
    for (int k0 = 0; k0 < kIn; k0 += kMfmaK) {
        u16x8 a = {};
        if (have) a = load8(x + (size_t)(row0 + i) * kIn + k0 + kq, vec);
        acc = mfma(a, column8(w1h, kHid, k0 + kq, j), acc);
    }
    {
        const float bias = b1[j];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float z = acc[r] + bias;
            h1[c_row(lane, r)][j] = f2bf(z > 0.f ? z : 0.f);
        }
    }
    __syncthreads();

    acc = floatx16{};
#pragma unroll 8
    for (int k0 = 0; k0 < kHid; k0 += kMfmaK)
        acc = mfma(*reinterpret_cast<const u16x8 *>(&h1[i][k0 + kq]), column8(w2h, kHid, k0 + kq, j), acc);
    {
        const float bias = b2[j];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float z = acc[r] + bias;
            h2[c_row(lane, r)][j] = f2bf(z > 0.f ? z : 0.f);
        }
    }
    __syncthreads();

    if (t < kRowBlock) {
        float sum = 0.f;
#pragma unroll 4
        for (int c = 0; c < kHid; c += 8) {
            const u16x8 h = *reinterpret_cast<const u16x8 *>(&h2[t][c]);
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += bf2f(h[u]) * w3[c + u];
        }
        const float l = sum + b3[0];
        const uint32_t row = row0 + (uint32_t)t;
        float d = 0.f;
        if (row < batch) {
            if (!kTrain) {
                logits[row] = l;
            } else {
                const float label = y[row];
                const float p = 1.f / (1.f + expf(-l));
                d = (p - label) / (float)batch;
                w.dlogit[row] = d;
                w.row_loss[row] = fmaxf(l, 0.f) - l * label + log1pf(expf(-fabsf(l)));
            }
        }
        dl[t] = d;
    }
    if (!kTrain) return;
    __syncthreads();

    // dz2, and the rows' activations out to memory for the sums over the
    // batch: thread t, 16 columns of row t / 16
    {
        const int r = t >> 4, c0 = (t & 15) * 16;
        const uint32_t row = row0 + (uint32_t)r;
        const float d = dl[r];
#pragma unroll
        for (int c = c0; c < c0 + 16; c += 8) {
            const u16x8 a1 = *reinterpret_cast<const u16x8 *>(&h1[r][c]), a2 = *reinterpret_cast<const u16x8 *>(&h2[r][c]);
            u16x8 z;
#pragma unroll
            for (int u = 0; u < 8; ++u) z[u] = a2[u] != 0 ? f2bf(d * w3[c + u]) : (uint16_t)0;
            *reinterpret_cast<u16x8 *>(&dz[r][c]) = z;
            if (row < batch) {
                store8(w.h1 + (size_t)row * kHid + c, a1, vec);
                store8(w.h2 + (size_t)row * kHid + c, a2, vec);
                store8(w.dz2 + (size_t)row * kHid + c, z, vec);
            }
        }
    }
    __syncthreads();

    acc = floatx16{};
#pragma unroll 8
    for (int k0 = 0; k0 < kHid; k0 += kMfmaK)
        acc = mfma(*reinterpret_cast<const u16x8 *>(&dz[i][k0 + kq]),
                   *reinterpret_cast<const u16x8 *>(w2h + (size_t)j * kHid + k0 + kq), acc);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = c_row(lane, r);
        if (row0 + (uint32_t)row < batch)
            w.dz1[(size_t)(row0 + row) * kHid + j] = h1[row][j] != 0 ? f2bf(acc[r]) : (uint16_t)0;
    }
}

// ---------------------------------------------------------------- sums over the batch

// Adam (Kingma & Ba): m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g^2;
// w -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps); then the BF16 copy.
struct AdamStep {
    float *w, *m, *v;   // master values and moments, in parameter order
    uint16_t *wh;       // BF16 copies (w1, w2, w3)
    float lr, c1, c2;
};

__device__ __forceinline__ void adam(const AdamStep &s, size_t at, float g, long bf_at) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mi = b1 * s.m[at] + (1.f - b1) * g;
    const float vi = b2 * s.v[at] + (1.f - b2) * g * g;
    s.m[at] = mi;
    s.v[at] = vi;
    const float w = s.w[at] - s.lr * (mi / s.c1) / (sqrtf(vi / s.c2) + eps);
    s.w[at] = w;
    if (bf_at >= 0) s.wh[bf_at] = f2bf(w);
}

constexpr int kSumThreads = 512;
constexpr int kSumWaves = kSumThreads / 64;
constexpr int kTiles2 = (kHid / 32) * (kHid / 32), kTiles1 = kHid / 32;
constexpr int kSumBlocks = kTiles2 + kTiles1 + kHid / 32;
constexpr int kStepsEach = 4;                        // MFMA steps whose operands a wave fetches at a time
constexpr int kStepsAll = kStepsEach * kSumWaves;    // of the workgroup: 512 batch rows
constexpr int kSumRows = 256;                        // batch rows of a column sum fetched at a time

struct SumTile {
    u16x8 a[kStepsAll][64], b[kStepsAll][64];        // operands as the lanes take them
};
struct SumColumns {
    uint16_t v[3][kSumRows][32];                     // dz1, dz2, h2
    float d[kSumRows];
};

// Gradients of the parameters: a 32 x 32 tile of dW2 = h1^T dz2 or
// dW1 = x^T dz1 per workgroup, or 32 columns of db1, db2 and dw3.  Every sum
// over the batch runs in ascending row order in one accumulator, so the
// gradients do not depend on how the work is laid out; what the eight waves
// share is the fetching: operands go to LDS 512 rows at a time, the next
// ones on their way while one wave multiplies.  kAdam: the update of each
// parameter follows at once.  512 rows: 25 us a tile product and 110 us a
// column sum when each step waited for its own reads, 13.6 us for all of them
// here; a step of training took 449 us in 18 launches and takes 30.
template <bool kAdam>
__global__ __launch_bounds__(kSumThreads) void k_sums(const uint16_t *__restrict__ x, uint32_t batch, Work w,
                                                      float *__restrict__ grad, AdamStep step) {
    __shared__ __align__(16) unsigned char lds[sizeof(SumTile) > sizeof(SumColumns) ? sizeof(SumTile)
                                                                                     : sizeof(SumColumns)];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6, b = (int)blockIdx.x;
    constexpr size_t oB1 = kN1, oW2 = oB1 + kHid, oB2 = oW2 + kN2, oW3 = oB2 + kHid, oB3 = oW3 + kN3;
    if (b < kTiles2 + kTiles1) {
        SumTile &T = *reinterpret_cast<SumTile *>(lds);
        const bool second = b < kTiles2;
        const int i0 = second ? 32 * (b >> 3) : 0, j0 = second ? 32 * (b & 7) : 32 * (b - kTiles2);
        const uint16_t *A = second ? w.h1 : x, *B = second ? w.dz2 : w.dz1;
        const int lda = second ? kHid : kIn, c = lane & 31;
        const uint32_t kq = 8u * (uint32_t)(lane >> 5);
        const uint32_t steps = batch / kMfmaK + (batch % kMfmaK != 0 ? 1u : 0u);
        u16x8 ra[kStepsEach], rb[kStepsEach];
        auto fetch = [&](uint32_t s0) {
#pragma unroll
            for (int u = 0; u < kStepsEach; ++u) {
                const uint32_t k0 = (s0 + (uint32_t)(wave * kStepsEach + u)) * kMfmaK + kq;
                ra[u] = column8_below(A, lda, k0, i0 + c, batch);
                rb[u] = column8_below(B, kHid, k0, j0 + c, batch);
            }
        };
        floatx16 acc = {};
        fetch(0);
        for (uint32_t s0 = 0; s0 < steps; s0 += kStepsAll) {
#pragma unroll
            for (int u = 0; u < kStepsEach; ++u) {
                T.a[wave * kStepsEach + u][lane] = ra[u];
                T.b[wave * kStepsEach + u][lane] = rb[u];
            }
            __syncthreads();
            if (s0 + kStepsAll < steps) fetch(s0 + kStepsAll);
            if (wave == 0) {
                const uint32_t ns = steps - s0 < (uint32_t)kStepsAll ? steps - s0 : (uint32_t)kStepsAll;
#pragma unroll 4
                for (uint32_t u = 0; u < ns; ++u) acc = mfma(T.a[u][lane], T.b[u][lane], acc);
            }
            __syncthreads();
        }
        float *out = reinterpret_cast<float *>(lds);
        if (wave == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) out[c_row(lane, r) * 32 + c] = acc[r];
        }
        __syncthreads();
        for (int e = t; e < 32 * 32; e += kSumThreads) {
            const float g = out[e];
            const size_t in = (size_t)(i0 + e / 32) * kHid + j0 + e % 32;
            const size_t at = (second ? oW2 : 0) + in;
            grad[at] = g;
            if (kAdam) adam(step, at, g, (long)((second ? kN1 : 0) + in));
        }
        return;
    }
    // 32 columns: waves 0, 1, 2 sum dz1, dz2 and h2 dlogit, wave 3 (of the
    // first such workgroup) dlogit; wave 4 the losses
    SumColumns &C = *reinterpret_cast<SumColumns *>(lds);
    const int cg = b - kTiles2 - kTiles1, c = t & 31, j = 32 * cg + c;
    const uint16_t *src[3] = {w.dz1, w.dz2, w.h2};
    constexpr int kEach = 3 * kSumRows * 32 / kSumThreads;
    uint16_t rv[kEach];
    float rd = 0.f;
    auto fetch = [&](uint32_t r0) {
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
            const uint32_t row = r0 + (uint32_t)((u % (kEach / 3)) * (kSumThreads / 32) + (t >> 5));
            rv[u] = row < batch ? src[u / (kEach / 3)][(size_t)row * kHid + j] : (uint16_t)0;
        }
        if (t < kSumRows) rd = r0 + (uint32_t)t < batch ? w.dlogit[r0 + (uint32_t)t] : 0.f;
    };
    float g = 0.f;
    fetch(0);
    for (uint32_t r0 = 0; r0 < batch; r0 += kSumRows) {
#pragma unroll
        for (int u = 0; u < kEach; ++u)
            C.v[u / (kEach / 3)][(u % (kEach / 3)) * (kSumThreads / 32) + (t >> 5)][c] = rv[u];
        if (t < kSumRows) C.d[t] = rd;
        __syncthreads();
        if (batch - r0 > (uint32_t)kSumRows) fetch(r0 + kSumRows);
        const int rows = batch - r0 < (uint32_t)kSumRows ? (int)(batch - r0) : kSumRows;
        if (wave < 2) {
#pragma unroll 16
            for (int i = 0; i < rows; ++i) g += bf2f(C.v[wave][i][c]);
        } else if (wave == 2) {
#pragma unroll 16
            for (int i = 0; i < rows; ++i) g += bf2f(C.v[2][i][c]) * C.d[i];
        } else if (wave == 3) {
#pragma unroll 16
            for (int i = 0; i < rows; ++i) g += C.d[i];
        }
        __syncthreads();
    }
    if (wave == 4 && cg == 0) {
        float l = 0.f;
        for (uint32_t i = (uint32_t)lane; i < batch; i += 64u) l += w.row_loss[i];
        for (int off = 32; off >= 1; off >>= 1) l += __shfl_xor(l, off);
        if (lane == 0) w.loss[0] = l;
    }
    if (wave > 3 || lane >= 32 || (wave == 3 && (cg != 0 || c != 0))) return;
    const size_t at = wave == 0 ? oB1 + j : wave == 1 ? oB2 + j : wave == 2 ? oW3 + j : oB3;
    grad[at] = g;
    if (kAdam) adam(step, at, g, wave == 2 ? (long)(kN1 + kN2 + j) : -1l);
}

__global__ void k_to_bf16(const float *__restrict__ x, uint16_t *__restrict__ y, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i]);
}

#define HIPCHK(expr)                                   \
    do {                                               \
        if ((expr) != hipSuccess) return MPDP_EDEVICE; \
    } while (0)

hipError_t refresh_bf16(const Params &p, hipStream_t s) {
    hipLaunchKernelGGL(k_to_bf16, dim3(64), dim3(256), 0, s, p.w1, p.w1h, kN1);
    hipLaunchKernelGGL(k_to_bf16, dim3(256), dim3(256), 0, s, p.w2, p.w2h, kN2);
    hipLaunchKernelGGL(k_to_bf16, dim3(1), dim3(256), 0, s, p.w3, p.w3h, kN3);
    return hipGetLastError();
}

template <bool kTrain>
hipError_t rows(const Params &p, const uint16_t *x, const float *y, uint32_t batch, const Work &w, float *logits,
                hipStream_t s) {
    const bool vec = ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w.h1)) & 15u) == 0;
    const uint32_t blocks = batch / kRowBlock + (batch % kRowBlock != 0 ? 1u : 0u);
    hipLaunchKernelGGL(k_rows<kTrain>, dim3(blocks), dim3(kRowThreads), 0, s, x, y, batch, p.w1h, p.b1, p.w2h, p.b2,
                       p.w3h, p.b3, logits, w, vec);
    return hipGetLastError();
}

template <bool kAdam>
hipError_t sums(const Params &p, const uint16_t *x, uint32_t batch, const Work &w, const AdamStep &step,
                hipStream_t s) {
    hipLaunchKernelGGL(k_sums<kAdam>, dim3(kSumBlocks), dim3(kSumThreads), 0, s, x, batch, w, p.g, step);
    return hipGetLastError();
}

// Mean loss of the last batch (waits for the stream).
mpdp_status read_loss(const Work &w, uint32_t batch, hipStream_t s, float *loss_out) {
    float l = 0.f;
    HIPCHK(hipMemcpyAsync(&l, w.loss, sizeof(float), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    *loss_out = l / (float)batch;
    return MPDP_OK;
}

}  // namespace

extern "C" {

size_t mpdp_scorer_param_bytes(void) { return scorer_layout().total; }

size_t mpdp_scorer_work_bytes(uint32_t batch) { return batch ? work_bytes(batch) : 0; }

mpdp_status mpdp_scorer_load(void *d_params, const float *w1, const float *b1, const float *w2, const float *b2,
                             const float *w3, const float *b3, void *hip_stream) {
    if (!d_params || !w1 || !b1 || !w2 || !b2 || !w3 || !b3) return MPDP_EINVAL;
    if (reinterpret_cast<uintptr_t>(d_params) % 256) return MPDP_EINVAL;
    std::vector<float> host(kNParams);
    size_t o = 0;
    auto put = [&](const float *src, size_t n) {
        std::memcpy(host.data() + o, src, 4 * n);
        o += n;
    };
    put(w1, kN1); put(b1, kHid); put(w2, kN2); put(b2, kHid); put(w3, kN3); put(b3, 1);
    for (float x : host)
        if (!std::isfinite(x)) return MPDP_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const Layout L = scorer_layout();
    const Params p = params_at(d_params);
    char *base = static_cast<char *>(d_params);
    HIPCHK(hipMemcpyAsync(base + L.master, host.data(), 4 * kNParams, hipMemcpyHostToDevice, s));
    HIPCHK(hipMemsetAsync(base + L.m, 0, 4 * kNParams, s));
    HIPCHK(hipMemsetAsync(base + L.v, 0, 4 * kNParams, s));
    HIPCHK(hipMemsetAsync(base + L.grad, 0, 4 * kNParams, s));
    HIPCHK(refresh_bf16(p, s));
    HIPCHK(hipStreamSynchronize(s));
    return MPDP_OK;
}

mpdp_status mpdp_scorer_layout(size_t *off_master, size_t *off_bf16, size_t *off_grad) {
    if (!off_master || !off_bf16 || !off_grad) return MPDP_EINVAL;
    const Layout L = scorer_layout();
    *off_master = L.master;
    *off_bf16 = L.bf;
    *off_grad = L.grad;
    return MPDP_OK;
}

mpdp_status mpdp_scorer_forward(const void *d_params, const uint16_t *d_x, uint32_t batch, float *d_logits,
                                void *d_work, size_t work_size, void *hip_stream) {
    if (!d_params || !d_x || !d_logits || !d_work || batch == 0) return MPDP_EINVAL;
    if (work_size < work_bytes(batch)) return MPDP_ENOMEM;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const Params p = params_at(const_cast<void *>(d_params));
    const Work w = work_at(d_work, batch);
    HIPCHK(rows<false>(p, d_x, nullptr, batch, w, d_logits, s));
    return MPDP_OK;
}

mpdp_status mpdp_scorer_grad(void *d_params, const uint16_t *d_x, const float *d_y, uint32_t batch, void *d_work,
                             size_t work_size, void *hip_stream, float *loss_out) {
    if (!d_params || !d_x || !d_y || !d_work || batch == 0) return MPDP_EINVAL;
    if (work_size < work_bytes(batch)) return MPDP_ENOMEM;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const Params p = params_at(d_params);
    const Work w = work_at(d_work, batch);
    HIPCHK(rows<true>(p, d_x, d_y, batch, w, nullptr, s));
    HIPCHK(sums<false>(p, d_x, batch, w, AdamStep{}, s));
    return loss_out ? read_loss(w, batch, s, loss_out) : MPDP_OK;
}

mpdp_status mpdp_scorer_train_step(void *d_params, const uint16_t *d_x, const float *d_y, uint32_t batch, float lr,
                                   uint32_t step, void *d_work, size_t work_size, void *hip_stream, float *loss_out) {
    if (step == 0 || !(lr > 0.f)) return MPDP_EINVAL;
    if (!d_params || !d_x || !d_y || !d_work || batch == 0) return MPDP_EINVAL;
    if (work_size < work_bytes(batch)) return MPDP_ENOMEM;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const Params p = params_at(d_params);
    const Work w = work_at(d_work, batch);
    const AdamStep adam{p.w1, p.m, p.v, p.w1h, lr, 1.f - powf(0.9f, (float)step), 1.f - powf(0.999f, (float)step)};
    HIPCHK(rows<true>(p, d_x, d_y, batch, w, nullptr, s));
    HIPCHK(sums<true>(p, d_x, batch, w, adam, s));
    return loss_out ? read_loss(w, batch, s, loss_out) : MPDP_OK;
}

}  // extern "C"
