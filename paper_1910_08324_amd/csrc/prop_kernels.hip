// Learned tile proposal on gfx950 (declared in include/spd_proposal.h): GPU tile generator,
// DIT-level features, and the forward / backward / Adam kernels of a three-layer 5-tap
// convolutional network in bfloat16 on MFMA (v_mfma_f32_32x32x16_bf16) with FP32 accumulation.
//
// Activations are stored channel-last and padded: act[row][pos'][32] with pos' = pos + 2 and
// zero positions 0, 1, 258..261, so the 5 taps of output position p read the contiguous
// 5 x C_in values starting at act[row][p][0].  A convolution is then, per row, the GEMM
//     D[co][p] = sum_k W[co][k] B[k][p],   B[k][p] = act_flat[row][p C_in + k],  k = t C_in + ci,
// one 32 (channels) x 32 (positions) MFMA tile per wave and 16 values of k per instruction.
// The weight gradient is the same product with positions as the reduction index.
#include <hip/hip_runtime.h>

#include <algorithm>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "spd.h"
#include "spd_proposal.h"

namespace spdp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int ROWS = SPD_PROP_TILE_ROWS;
constexpr int LEN = SPD_PROP_TILE_LEN;
constexpr int POS = SPD_PROP_POS;
constexpr int RP = SPD_PROP_ROW_POS;
constexpr int FCH = SPD_PROP_FEAT_CH;
constexpr int CH = SPD_PROP_CH;
constexpr int TAPS = SPD_PROP_TAPS;
constexpr int KW1 = 48;                 // padded k of layer 1 (5 taps x 8 channels = 40)
constexpr int KW = TAPS * CH;           // 160
constexpr int MAX_PARTS = 256;          // work-groups of the backward pass (one per CU)

// bfloat16: the upper half of an IEEE binary32, rounded to nearest even
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Work-group barrier that orders LDS only: global loads stay in flight across it (__syncthreads()
// waits for them too, which put the latency of every row's prefetch into the row).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// two values rounded to nearest even, the first in the lower half (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}
__device__ __forceinline__ float low_bf16(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float high_bf16(uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); }
// v where the half of m (an activation, never negative) is not zero, else zero
__device__ __forceinline__ uint32_t where_bf16(uint32_t v, uint32_t m) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 on = __builtin_elementwise_min(__builtin_bit_cast(u16x2, m), u16x2{1, 1});
    return v & __builtin_bit_cast(uint32_t, (u16x2)(u16x2{0, 0} - on));
}

__device__ __forceinline__ bf16x8 load8(const uint16_t *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}

// ---------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC 2011): ten rounds of two 32x32 -> 64-bit
// products, with the key bumped by the Weyl constants between rounds.
// ---------------------------------------------------------------------------------------
struct Words {
    uint32_t a0, a1, a2, a3;
};

__device__ __forceinline__ Words philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return {c0, c1, c2, c3};
}

__device__ __forceinline__ void box_muller(uint32_t a, uint32_t b, float &z0, float &z1) {
    float u = ((float)a + 1.0f) * 0x1p-32f;
    u = fminf(u, 1.0f);
    const float v = (float)b * 0x1p-32f;
    const float rad = sqrtf(-2.0f * logf(u));
    const float ang = 6.28318530717958647692f * v;
    z0 = rad * cosf(ang);
    z1 = rad * sinf(ang);
}

struct TileArgs {
    float *x;
    uint64_t seed;
    int64_t first_tile;
    int32_t n_tiles;
};

// one work-group per row; 256 threads x 4 blocks of 4 samples
__global__ __launch_bounds__(256) void tiles_kernel(const TileArgs A) {
    const int i = blockIdx.x / ROWS;
    const int r = blockIdx.x - i * ROWS;
    if (i >= A.n_tiles) return;
    const int64_t t = A.first_tile + i;
    const uint32_t tlo = (uint32_t)t, thi = (uint32_t)((uint64_t)t >> 32);
    const uint32_t k0 = (uint32_t)A.seed, k1 = (uint32_t)(A.seed >> 32);
    // pulse parameters of the tile (the same in every thread)
    const Words h = philox(0u, 0xFFFFFFFFu, tlo, thi, k0, k1);
    const int n_p = (int)(((uint64_t)h.a0 * 3u) >> 32);
    int prow[2] = {-1, -1}, pst[2] = {0, 0}, pw[2] = {0, 0};
    float pamp[2] = {0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (j < n_p) {
            const Words q = philox((uint32_t)(j + 1), 0xFFFFFFFFu, tlo, thi, k0, k1);
            prow[j] = (int)(((uint64_t)q.a0 * ROWS) >> 32);
            const int S = 1 + (int)(((uint64_t)q.a1 * 64u) >> 32);
            const float u = (float)((double)q.a2 * 0x1p-32);
            const float snr = (float)(6.0 + 24.0 * (double)u);
            pw[j] = S;
            pst[j] = (int)(((uint64_t)q.a3 * (uint64_t)(LEN - S + 1)) >> 32);
            pamp[j] = (float)((double)snr / sqrt((double)S));
        }
    }
    float *xr = A.x + (int64_t)blockIdx.x * LEN;
    for (int b = threadIdx.x; b < LEN / 4; b += 256) {
        const Words w = philox((uint32_t)b, (uint32_t)r, tlo, thi, k0, k1);
        float z[4];
        box_muller(w.a0, w.a1, z[0], z[1]);
        box_muller(w.a2, w.a3, z[2], z[3]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (prow[j] == r) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int s = 4 * b + q;
                    if (s >= pst[j] && s < pst[j] + pw[j]) z[q] += pamp[j];
                }
            }
        }
        *reinterpret_cast<float4 *>(xr + 4 * b) = make_float4(z[0], z[1], z[2], z[3]);
    }
}

// ---------------------------------------------------------------------------------------
// Features: thread p of a row's work-group sums level-4 unit p (16 samples); coarser levels
// are pairwise sums across lanes (butterflies of 2, 4, 8, 16 lanes, inside one wave).  Bound by
// reading the samples; a block's columns of 4096 samples go in one launch, as a column of a small
// block is done in less time than a launch takes (16 columns of 512 rows: 16 launches of 5 us
// each, 40 us as one; the gated search 492 -> 469 us).
// ---------------------------------------------------------------------------------------
struct FeatArgs {
    const float *x;
    int64_t ld;
    const float *mean;
    const float *sigma;
    uint16_t *feat;
    int32_t n_dm, n_rows;      // rows of a column, and of all columns
};

__global__ __launch_bounds__(256) void features_kernel(const FeatArgs A) {
    const int r = blockIdx.x;
    const int p = threadIdx.x;
    if (r >= A.n_rows) return;
    const int c = r / A.n_dm, d = r - c * A.n_dm;
    const float *xr = A.x + (int64_t)d * A.ld + (int64_t)c * LEN + 16 * p;
    const float mu = A.mean[d];
    const float inv = 1.0f / A.sigma[d];
    float y4 = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4 *>(xr + 4 * q);
        y4 += (v.x - mu) * inv;
        y4 += (v.y - mu) * inv;
        y4 += (v.z - mu) * inv;
        y4 += (v.w - mu) * inv;
    }
    const float y5 = y4 + __shfl_xor(y4, 1);
    const float y6 = y5 + __shfl_xor(y5, 2);
    const float y7 = y6 + __shfl_xor(y6, 4);
    const float y8 = y7 + __shfl_xor(y7, 8);
    // unit variance under white noise: divide level k by 2^(k/2)
    const uint16_t c0 = to_bf16(y4 * 0.25f);
    const uint16_t c1 = to_bf16(y5 * 0.17677669529663688f);
    const uint16_t c2 = to_bf16(y6 * 0.125f);
    const uint16_t c3 = to_bf16(y7 * 0.088388347648318441f);
    const uint16_t c4 = to_bf16(y8 * 0.0625f);
    uint16_t *fr = A.feat + (int64_t)r * RP * FCH;
    *reinterpret_cast<uint4 *>(fr + (p + 2) * FCH) =
        make_uint4((uint32_t)c0 | ((uint32_t)c1 << 16), (uint32_t)c2 | ((uint32_t)c3 << 16),
                   (uint32_t)c4, 0u);
    if (p < RP - POS) {
        const int pad = p < 2 ? p : POS + p;          // positions 0, 1, 258 .. 261
        *reinterpret_cast<uint4 *>(fr + pad * FCH) = make_uint4(0u, 0u, 0u, 0u);
    }
}

// ---------------------------------------------------------------------------------------
// Weights in bfloat16 for the MFMA operands: forward rows W[co][t C_in + ci] (layer 1 padded
// to k = 48), and for the input gradient the flipped transpose Wt[ci][t' 32 + co] =
// W[co][4 - t'][ci].
// ---------------------------------------------------------------------------------------
struct WB {
    uint16_t *w1, *w2, *w3, *w2t, *w3t;
};

__global__ void prep_weights_kernel(const float *params, WB o) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < CH * KW1) {
        const int co = i / KW1, k = i - co * KW1;
        o.w1[i] = k < TAPS * FCH ? to_bf16(params[SPD_PROP_OFF_W1 + co * TAPS * FCH + k]) : 0;
    }
    if (i < CH * KW) {
        o.w2[i] = to_bf16(params[SPD_PROP_OFF_W2 + i]);
        o.w3[i] = to_bf16(params[SPD_PROP_OFF_W3 + i]);
        const int ci = i / KW, k = i - ci * KW;
        const int tp = k / CH, co = k - tp * CH;
        const int src = co * KW + (TAPS - 1 - tp) * CH + ci;
        o.w2t[i] = to_bf16(params[SPD_PROP_OFF_W2 + src]);
        o.w3t[i] = to_bf16(params[SPD_PROP_OFF_W3 + src]);
    }
}

__device__ __forceinline__ float block_max(float v, float *sh) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    lds_barrier();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    lds_barrier();
    return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

__device__ __forceinline__ float block_sum(float v, float *sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    lds_barrier();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    lds_barrier();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

__device__ __forceinline__ void load_act(const uint16_t *p, float a[CH]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint4 v = *reinterpret_cast<const uint4 *>(p + 8 * q);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[8 * q + 2 * e] = __uint_as_float(w[e] << 16);
            a[8 * q + 2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Fixed-order reduction of the partials into the gradient vector, and the mean loss.
// ---------------------------------------------------------------------------------------
struct RedArgs {
    const float *part1, *part2, *part3, *hpart, *loss_t;
    float *grads;
    float *loss;
    int32_t n_parts, n_tiles;
};

// Sum of src[w * stride] over w in [w0, w1), in increasing w, with 8 loads in flight.
__device__ __forceinline__ float ordered_sum(const float *src, int64_t stride, int w0, int w1) {
    float g = 0.0f;
    int w = w0;
    for (; w + 8 <= w1; w += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = src[(int64_t)(w + q) * stride];
#pragma unroll
        for (int q = 0; q < 8; ++q) g += v[q];
    }
    for (; w < w1; ++w) g += src[(int64_t)w * stride];
    return g;
}

// A work-group takes RED_PARAMS gradient entries; each entry's partials are cut into RED_CHUNKS
// consecutive ranges summed in order by separate threads, and the range sums are added in order.
constexpr int RED_PARAMS = 8;
constexpr int RED_CHUNKS = 32;

__global__ __launch_bounds__(256) void reduce_kernel(const RedArgs A) {
    __shared__ float part[RED_CHUNKS][RED_PARAMS];
    __shared__ float lsum[256];
    const int j = threadIdx.x % RED_PARAMS;
    const int c = threadIdx.x / RED_PARAMS;
    const int i = blockIdx.x * RED_PARAMS + j;
    const float *src = nullptr;
    int stride = 0, idx = 0;
    if (i < SPD_PROP_OFF_B1) {
        src = A.part1; stride = CH * 40 + CH; idx = i;
    } else if (i < SPD_PROP_OFF_W2) {
        src = A.part1; stride = CH * 40 + CH; idx = CH * 40 + (i - SPD_PROP_OFF_B1);
    } else if (i < SPD_PROP_OFF_B2) {
        src = A.part2; stride = CH * KW + CH; idx = i - SPD_PROP_OFF_W2;
    } else if (i < SPD_PROP_OFF_W3) {
        src = A.part2; stride = CH * KW + CH; idx = CH * KW + (i - SPD_PROP_OFF_B2);
    } else if (i < SPD_PROP_OFF_B3) {
        src = A.part3; stride = CH * KW + CH; idx = i - SPD_PROP_OFF_W3;
    } else if (i < SPD_PROP_OFF_WH) {
        src = A.part3; stride = CH * KW + CH; idx = CH * KW + (i - SPD_PROP_OFF_B3);
    } else if (i <= SPD_PROP_OFF_BH) {
        src = A.hpart; stride = CH + 1; idx = i - SPD_PROP_OFF_WH;
    }
    const int w0 = (int)((int64_t)c * A.n_parts / RED_CHUNKS);
    const int w1 = (int)((int64_t)(c + 1) * A.n_parts / RED_CHUNKS);
    part[c][j] = src ? ordered_sum(src + idx, stride, w0, w1) : 0.0f;
    __syncthreads();
    if (c == 0 && i < SPD_PROP_NPARAMS) {
        float g = 0.0f;
        for (int q = 0; q < RED_CHUNKS; ++q) g += part[q][j];
        A.grads[i] = g;
    }
    if (blockIdx.x == 0) {
        // mean loss: 256 ordered ranges of the tiles, then the range sums in order
        const int t0 = (int)((int64_t)threadIdx.x * A.n_tiles / 256);
        const int t1 = (int)((int64_t)(threadIdx.x + 1) * A.n_tiles / 256);
        lsum[threadIdx.x] = ordered_sum(A.loss_t, 1, t0, t1);
        __syncthreads();
        if (threadIdx.x == 0) {
            float L = 0.0f;
            for (int q = 0; q < 256; ++q) L += lsum[q];
            A.loss[0] = L / (float)A.n_tiles;
        }
    }
}

struct AdamArgs {
    float *p;
    const float *g;
    float *m, *v;
    float lr, c1, c2;          // c1 = 1 / (1 - beta1^step), c2 = 1 / (1 - beta2^step)
};

__global__ void adam_kernel(const AdamArgs A) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= SPD_PROP_NPARAMS) return;
    const float g = A.g[i];
    const float m = 0.9f * A.m[i] + 0.1f * g;
    const float v = 0.999f * A.v[i] + 0.001f * g * g;
    A.m[i] = m;
    A.v[i] = v;
    A.p[i] -= A.lr * (m * A.c1) / (sqrtf(v * A.c2) + 1e-8f);
}

// ---------------------------------------------------------------------------------------
// Per-tile maximum over a search's planes, and labels.
// ---------------------------------------------------------------------------------------
struct TileMaxArgs {
    const float *snr;
    float *out;
    int64_t off[SPD_MAX_LEVELS];
    int64_t pitch[SPD_MAX_LEVELS];
    int64_t slots[SPD_MAX_LEVELS];
    int32_t n_levels, rows_per_tile, n_tiles;
};

// A float (never NaN here) as a signed integer of the same order: non-negative floats keep their
// bits, negative ones have the 31 magnitude bits inverted.  The map is its own inverse.
__device__ __forceinline__ int32_t order_key(int32_t bits) { return bits >= 0 ? bits : bits ^ 0x7FFFFFFF; }

__global__ void tile_init_kernel(int32_t *key, int32_t n_tiles) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_tiles) key[t] = order_key(__float_as_int(-__builtin_huge_valf()));
}

// one work-group per DM row: the row's maximum over every level, merged into its tile's entry
// with an integer atomic maximum on the order key.  Bound by the planes it reads.  The waves take
// runs of 1024 slots in turn, over the levels' ends (most levels are shorter than what a work-group
// reads at once), and a run's four loads per lane are issued together: 536 MB of IG(1) planes of 16,384
// rows 147 -> 138 us (3.9 TB/s), 268 MB of exhaustive planes 73 -> 66 us.
__global__ __launch_bounds__(256) void tile_max_kernel(const TileMaxArgs A, int32_t *key) {
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ float sh[4];
    const int d = blockIdx.x;
    if (d >= A.n_tiles * A.rows_per_tile) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float mx = -__builtin_huge_valf();
    int64_t run = wave;                                 // the wave's next run, from the level's first
    for (int lv = 0; lv < A.n_levels; ++lv) {
        const float *Y = A.snr + A.off[lv] + (int64_t)d * A.pitch[lv];
        const int64_t n = A.slots[lv], n4 = n >> 2, runs = (n4 + 255) >> 8;
        for (; run < runs; run += 4) {
            v4f v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {               // (past the end the last four slots again)
                const int64_t q = run * 256 + 64 * u + lane;
                v[u] = reinterpret_cast<const v4f *>(Y)[q < n4 ? q : n4 - 1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) mx = fmaxf(mx, fmaxf(fmaxf(v[u].x, v[u].y), fmaxf(v[u].z, v[u].w)));
        }
        run -= runs;
        if (wave == (lv & 3) && 4 * n4 + lane < n) mx = fmaxf(mx, Y[4 * n4 + lane]);
    }
    mx = block_max(mx, sh);
    if (threadIdx.x == 0) atomicMax(key + d / A.rows_per_tile, order_key(__float_as_int(mx)));
}

__global__ void tile_fin_kernel(int32_t *key, int32_t n_tiles) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_tiles) reinterpret_cast<float *>(key)[t] = __int_as_float(order_key(key[t]));
}

__global__ void labels_kernel(const float *e, const float *l, int32_t n, float thr, float m,
                              float *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float prod = m * l[i];
    out[i] = (e[i] > thr && e[i] > prod) ? 1.0f : 0.0f;
}

// tile (r, c) of an n_row x n_col grid: logits in column order (c n_row + r, as the features of
// one column of tiles after another give them), flags in row order (r n_col + c)
__global__ void flags_kernel(const float *logits, int32_t n_row, int32_t n_col, float thr,
                             uint8_t *flags) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n_row * n_col) return;
    const int64_t r = i / n_col, c = i - r * n_col;
    flags[i] = logits[c * n_row + r] > thr ? 1 : 0;
}

// ---------------------------------------------------------------------------------------
// Fused inference: one work-group per row runs the three convolutions with the activations in
// LDS (features 4.2 KB, two activation buffers of 21 KB), then the read-out; only the
// features come from HBM.  Each row leaves its read-out maximum and sum of exp(s - max); a
// second kernel combines a tile's 64 rows into the logit.  Training runs this
// launch too, and the backward launch forms the same activations again by the same MFMA sequence.
// ---------------------------------------------------------------------------------------
struct InferArgs {
    const uint16_t *feat;
    WB wb;
    const float *params;
    float *row_max;            // [rows]
    float *row_sum;            // [rows]
    int32_t rows;
};

// Activation rows in LDS: padded position pp keeps its 32 channels (four 16-byte chunks) in a
// row of 40 bf16 (80 bytes).  16-byte loads of one chunk by any 8 or 16 consecutive positions
// (the MFMA operand and the read-out) then fall in distinct LDS banks, with 32 or 64 banks;
// a 64-byte stride puts four positions on the same banks.
constexpr int ACT_LD = CH + 8;
__device__ __forceinline__ int act_at(int pp, int c) { return pp * ACT_LD + (c << 3); }

// The weights of one layer as this lane feeds them to the MFMA (A operand: output channel n =
// lane % 32, k = 16 s + 8 (lane / 32) .. + 7), held in registers across the rows of a launch.
template <int CI>
struct LayerW {
    static constexpr int KS = (TAPS * CI + 15) / 16;
    bf16x8 w[KS];
    __device__ __forceinline__ void load(const uint16_t *wg, int l) {
        const int h = l >> 5, n = l & 31;
#pragma unroll
        for (int s = 0; s < KS; ++s) w[s] = load8(wg + n * (KS * 16) + 16 * s + 8 * h);
    }
};

// one layer of a row held in LDS: out = relu(W in + b), 2 tiles of 32 positions per wave, their
// two accumulation chains interleaved so that consecutive MFMAs are independent.  The layer-1
// input (8 features per position, 16 bytes) is a plain row; wider inputs are padded.  bias: the
// layer's 32 biases in LDS.
template <int CI>
__device__ __forceinline__ void conv_lds(const uint16_t *in, const LayerW<CI> &W, const float *bias,
                                         uint16_t *out, int wave, int l) {
    constexpr int KS = LayerW<CI>::KS;
    static_assert(CI == FCH || CI == CH, "layer inputs are the features or an activation row");
    const int h = l >> 5;
    const int n = l & 31;
    f32x16 acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // k = 16 s + 8 h: tap s / 2, channels 16 (s % 2) + 8 h .. + 7 of position p0 + n + tap
            const int p0 = wave * 64 + t * 32;
            const uint16_t *src = CI == CH ? in + act_at(p0 + n + (s >> 1), 2 * (s & 1) + h)
                                           : in + (p0 + n) * CI + 16 * s + 8 * h;
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(W.w[s], load8(src), acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int po = wave * 64 + t * 32 + n + 2;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 bv = *reinterpret_cast<const float4 *>(bias + 8 * g + 4 * h);
            const float bb[4] = {bv.x, bv.y, bv.z, bv.w};
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = fmaxf(acc[t][4 * g + j] + bb[j], 0.0f);
            *reinterpret_cast<uint2 *>(out + act_at(po, g) + 4 * h) =
                make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        }
    }
}

// Persistent: each work-group takes rows blockIdx.x, + gridDim.x, ... with the weights in
// registers for the whole launch, and fetches the next row's features while it computes the
// current one.
__global__ __launch_bounds__(256) void infer_kernel(const InferArgs A) {
    constexpr int NF = RP * FCH / 8;                 // 16-byte pieces of a row's features
    static_assert(NF > 256 && NF <= 512, "a row's features take one or two pieces per thread");
    __shared__ __attribute__((aligned(16))) uint16_t f[RP * FCH];
    __shared__ __attribute__((aligned(16))) uint16_t a[RP * ACT_LD];
    __shared__ __attribute__((aligned(16))) uint16_t b[RP * ACT_LD];
    __shared__ __attribute__((aligned(16))) float bias[3 * CH];
    __shared__ float red[8];
    if ((int)blockIdx.x >= A.rows) return;
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int l = tid & 63;
    LayerW<FCH> W1;
    LayerW<CH> W2, W3;
    W1.load(A.wb.w1, l);
    W2.load(A.wb.w2, l);
    W3.load(A.wb.w3, l);
    if (tid < 3 * CH) {
        const int j = tid / CH, c = tid - j * CH;
        const int off = j == 0 ? SPD_PROP_OFF_B1 : (j == 1 ? SPD_PROP_OFF_B2 : SPD_PROP_OFF_B3);
        bias[tid] = A.params[off + c];
    }
    // zero pads of the activation buffers (positions 0, 1, 258 .. 261); the layers never write them
    for (int i = tid; i < 6 * CH / 8; i += 256) {
        const int pos = i / (CH / 8), part = i - pos * (CH / 8);
        const int pp = pos < 2 ? pos : POS + pos;
        *reinterpret_cast<uint4 *>(a + act_at(pp, part)) = make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4 *>(b + act_at(pp, part)) = make_uint4(0u, 0u, 0u, 0u);
    }
    const float *wh = A.params + SPD_PROP_OFF_WH;
    const float bh = A.params[SPD_PROP_OFF_BH];
    uint4 fp0 = make_uint4(0u, 0u, 0u, 0u), fp1 = fp0;
    auto fetch = [&](int r) {
        const uint4 *src = reinterpret_cast<const uint4 *>(A.feat + (int64_t)r * RP * FCH);
        fp0 = src[tid];
        if (tid + 256 < NF) fp1 = src[tid + 256];
    };
    fetch(blockIdx.x);
    for (int r = blockIdx.x; r < A.rows; r += gridDim.x) {
        reinterpret_cast<uint4 *>(f)[tid] = fp0;
        if (tid + 256 < NF) reinterpret_cast<uint4 *>(f)[tid + 256] = fp1;
        lds_barrier();
        if (r + (int)gridDim.x < A.rows) fetch(r + gridDim.x);
        conv_lds<FCH>(f, W1, bias, a, wave, l);
        lds_barrier();
        conv_lds<CH>(a, W2, bias + CH, b, wave, l);
        lds_barrier();
        conv_lds<CH>(b, W3, bias + 2 * CH, a, wave, l);
        lds_barrier();
        // read-out of position tid, then the row's max and sum of exp(s - max)
        float act[CH];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = *reinterpret_cast<const uint4 *>(a + act_at(tid + 2, q));
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                act[8 * q + 2 * e] = __uint_as_float(w[e] << 16);
                act[8 * q + 2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
            }
        }
        float sv = 0.0f;
#pragma unroll
        for (int c = 0; c < CH; ++c) sv += wh[c] * act[c];
        sv += bh;
        const float mx = block_max(sv, red);
        const float se = block_sum(expf(sv - mx), red + 4);
        if (tid == 0) {
            A.row_max[r] = mx;
            A.row_sum[r] = se;
        }
        lds_barrier();                    // f and a are rewritten for the next row
    }
}

// A tile's logit from its rows' maxima and sums and, training (labels not null), its loss and what
// the backward pass needs of it.  One wave per tile, a lane per row.
struct CombineArgs {
    const float *row_max, *row_sum;
    const float *labels;
    float *logits;             // may be null when training
    float *loss_t, *lse, *dlogit;
    int32_t n_tiles;
};

__global__ __launch_bounds__(256) void combine_kernel(const CombineArgs A) {
    static_assert(ROWS == 64, "a lane per row");
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (t >= A.n_tiles) return;
    const float m = A.row_max[(int64_t)t * ROWS + lane];
    float M = m;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    float Z = A.row_sum[(int64_t)t * ROWS + lane] * expf(m - M);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) Z += __shfl_xor(Z, o);
    if (lane) return;
    const float lse = M + logf(Z);
    const float logit = lse - 9.70406052783923f;               // log(64 * 256)
    if (A.logits) A.logits[t] = logit;
    if (!A.labels) return;
    const float y = A.labels[t];
    const float sig = 1.0f / (1.0f + expf(-logit));
    A.lse[t] = lse;
    A.dlogit[t] = (sig - y) / (float)A.n_tiles;
    A.loss_t[t] = fmaxf(logit, 0.0f) + log1pf(expf(-fabsf(logit))) - y * logit;
}

// ---------------------------------------------------------------------------------------
// Training: forward and backward of a row in one work-group, with every activation and gradient in
// LDS.  The forward launch (infer_kernel) gives each tile's logit; this one forms the row's
// activations again (bitwise the same) and runs the backward pass on them, so that neither
// activations nor gradients go through HBM.
//
// An MFMA tile of a convolution is formed twice from the same operands, once with the weights and
// once with the positions as rows: a lane then holds four consecutive channels of one position
// (stored channel-last, the layout the next convolution reads 16 bytes at a time) and four
// consecutive positions of one channel (stored channel by channel, the layout in which the weight
// gradient, whose reduction index is the position, reads 16 bytes at a time).  The five taps of a
// channel are five shifts of 12 consecutive positions, so two 16-byte loads and eight register
// funnel shifts feed five MFMAs.
//
// One work-group of 8 waves per CU (150,688 bytes of LDS), persistent over rows.  A wave convolves its 32
// positions; the weight gradients of a row, 12 MFMA tiles summed over 256 positions, are 24
// half-tiles, three per wave, whose accumulators are kept over the rows.  The weights of layer 3 and of
// the input gradients come from the cache for each row.  All of it needs more than the 256 registers of
// a lane with two waves per SIMD: the compiler keeps 44 values in scratch (180 bytes a lane).
// FP32 chains stay short whatever the number of tiles: every kBwdFlush rows the accumulators are added
// to the work-group's partial (the halves of a tile in turn) and the lanes' sums to their totals in
// LDS.  An accumulator then takes 256 MFMAs in a row, a bias gradient 512 additions and the
// read-out's 16 a row and 32 rows.  One chain over all rows of a work-group lost accuracy with the
// tiles of a call: 1024 tiles alike, read-out gradient 4e-5 off.
// Measured, 16,384 rows (256 tiles): 0.91 ms, and 0.14 ms for the forward launch, where separate
// launches per convolution, weight gradient and read-out, bound by 3.3 GB of activations and by
// 2-byte gathers, took 2.35 ms together.  Bound by latency: a row's MFMAs need 6.4k of its 30k cycles.
// ---------------------------------------------------------------------------------------
struct BwdArgs {
    const uint16_t *feat;
    WB wb;
    const float *params;
    const float *lse;          // [n_tiles] log of the sum of exp(s) over the tile
    const float *dlogit;       // [n_tiles] gradient of the loss at the tile's logit
    float *part1, *part2, *part3, *hpart;   // [gridDim.x] partial gradients
    int32_t rows;
};

constexpr int T_LD = 264;                      // positions per channel row: 16-byte rows, 4 banks apart
constexpr int T_ELEMS = CH * T_LD;
constexpr int ACT_ELEMS = RP * ACT_LD;
constexpr int BWD_ELEMS = RP * FCH + 3 * ACT_ELEMS + 4 * T_ELEMS + FCH * T_LD;
constexpr int P1 = CH * TAPS * FCH + CH, P2 = CH * KW + CH;   // floats of a partial of layer 1; 2, 3

// both forms of one 32-position tile at p0: n (weights as rows), t (positions as rows)
template <int CI, bool N>
__device__ __forceinline__ void conv_both(const uint16_t *in, const LayerW<CI> &W, int p0, int l,
                                          f32x16 &an, f32x16 &at) {
    const int h = l >> 5, n = l & 31;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (N) an[i] = 0.0f;
        at[i] = 0.0f;
    }
#pragma unroll
    for (int s = 0; s < LayerW<CI>::KS; ++s) {
        const bf16x8 b = load8(CI == CH ? in + act_at(p0 + n + (s >> 1), 2 * (s & 1) + h)
                                        : in + (p0 + n) * CI + 16 * s + 8 * h);
        if (N) an = __builtin_amdgcn_mfma_f32_32x32x16_bf16(W.w[s], b, an, 0, 0, 0);
        at = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, W.w[s], at, 0, 0, 0);
    }
}

constexpr int kBwdThreads = 512;
constexpr int kBwdFlush = 32;                  // rows between additions to the partial

// acc[co][column] += sum over 128 positions from p of dz[pos][co] in[pos + T][channel], the channel
// (lane n's column) chosen by the row `in` points to.  T < 0 (layer 1, columns 8 t + ci): lane n takes
// tap n / 8 of channel n % 8.
template <int T>
__device__ __forceinline__ void wgrad_half(const uint16_t *dz, const uint16_t *in, f32x16 &acc, int n) {
    const bool second = (n >> 4) & 1;
    const uint32_t odd = ((n >> 3) & 1) * 16;
#pragma unroll
    for (int ps = 0; ps < 8; ++ps) {
        const bf16x8 a = load8(dz + 16 * ps);
        const uint4 lo = *reinterpret_cast<const uint4 *>(in + 16 * ps);
        uint4 w = lo;
        if constexpr (T != 0) {
            const uint4 hi = *reinterpret_cast<const uint4 *>(in + 16 * ps + 8);
            const uint32_t d[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            if constexpr (T < 0) {
                uint32_t e[5];
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const uint32_t x = d[i + 1], y = d[i];   // (values: a choice of elements would put d in memory)
                    e[i] = second ? x : y;
                }
                w = make_uint4(__builtin_amdgcn_alignbit(e[1], e[0], odd), __builtin_amdgcn_alignbit(e[2], e[1], odd),
                               __builtin_amdgcn_alignbit(e[3], e[2], odd), __builtin_amdgcn_alignbit(e[4], e[3], odd));
            } else {
                constexpr int o = T >> 1;
                w = (T & 1) ? make_uint4(__builtin_amdgcn_alignbit(d[o + 1], d[o], 16),
                                         __builtin_amdgcn_alignbit(d[o + 2], d[o + 1], 16),
                                         __builtin_amdgcn_alignbit(d[o + 3], d[o + 2], 16),
                                         __builtin_amdgcn_alignbit(d[o + 4], d[o + 3], 16))
                            : make_uint4(d[o], d[o + 1], d[o + 2], d[o + 3]);
            }
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, w), acc, 0, 0, 0);
    }
}

__global__ __launch_bounds__(kBwdThreads, 2) void backward_kernel(const BwdArgs A) {
    constexpr int NF = RP * FCH / 8;
    static_assert(NF <= kBwdThreads, "a row's features take one piece per thread");
    __shared__ __attribute__((aligned(16))) uint16_t smem[BWD_ELEMS];
    __shared__ __attribute__((aligned(16))) float bias[4 * CH];   // the layers' biases, the read-out's weights
    __shared__ __attribute__((aligned(16))) float dsv[POS];
    __shared__ float red[8];
    __shared__ float tot[5][kBwdThreads];      // each lane's b1, b2, b3, gw, gb up to the last flush
    uint16_t *f = smem;
    uint16_t *c1 = f + RP * FCH, *c2 = c1 + ACT_ELEMS, *c3 = c2 + ACT_ELEMS;      // channel-last
    uint16_t *t1 = c3 + ACT_ELEMS, *t2 = t1 + T_ELEMS, *z1 = t2 + T_ELEMS, *z2 = z1 + T_ELEMS;
    uint16_t *ft = z2 + T_ELEMS;                                                  // channel by channel
    uint16_t *z3 = c1;                          // (layer 1's activations are not read after layer 2)
    static_assert(T_ELEMS <= ACT_ELEMS, "z3 fits in c1");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63;
    const int h = l >> 5, n = l & 31;
    const int p0 = wave * 32;                   // this wave's positions
    LayerW<FCH> W1;
    LayerW<CH> W2;
    W1.load(A.wb.w1, l);
    W2.load(A.wb.w2, l);
    if (tid < 4 * CH) {
        const int j = tid / CH, c = tid - j * CH;
        const int off = j == 0 ? SPD_PROP_OFF_B1 : j == 1 ? SPD_PROP_OFF_B2 : j == 2 ? SPD_PROP_OFF_B3 : SPD_PROP_OFF_WH;
        bias[tid] = A.params[off + c];
    }
    // the pads (positions 0, 1, 258 ..) are zero and, but for c1's, never written
    for (int i = tid; i < BWD_ELEMS / 8; i += kBwdThreads)
        reinterpret_cast<uint4 *>(smem)[i] = make_uint4(0u, 0u, 0u, 0u);
    static_assert(BWD_ELEMS % 8 == 0, "cleared in 16-byte pieces");
    const float *wh = bias + 3 * CH;
    const float bh = A.params[SPD_PROP_OFF_BH];
    const float whn = A.params[SPD_PROP_OFF_WH + n];
    f32x16 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0.0f;
    float b1 = 0.0f, b2 = 0.0f, b3 = 0.0f, gw = 0.0f, gb = 0.0f;
#pragma unroll
    for (int i = 0; i < 5; ++i) tot[i][tid] = 0.0f;
    const int64_t b = blockIdx.x;
    uint4 fp = make_uint4(0u, 0u, 0u, 0u);
    auto fetch = [&](int r) {
        if (tid < NF) fp = reinterpret_cast<const uint4 *>(A.feat + (int64_t)r * RP * FCH)[tid];
    };
    // the layer's activations of the wave's tile in both layouts; packed: the second one's values
    auto relu_both = [&](auto store_t, const f32x16 &an, const f32x16 &at, const float *bs, uint16_t *c,
                         uint16_t *t, uint32_t packed[8]) {
        const float bn = bs[n];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 bv = *reinterpret_cast<const float4 *>(bs + 8 * g + 4 * h);
            const float bb[4] = {bv.x, bv.y, bv.z, bv.w};
            float u[4], w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                u[j] = fmaxf(an[4 * g + j] + bb[j], 0.0f);
                w[j] = fmaxf(at[4 * g + j] + bn, 0.0f);
            }
            *reinterpret_cast<uint2 *>(c + act_at(p0 + n + 2, g) + 4 * h) =
                make_uint2(pack_bf16(u[0], u[1]), pack_bf16(u[2], u[3]));
            packed[2 * g] = pack_bf16(w[0], w[1]);
            packed[2 * g + 1] = pack_bf16(w[2], w[3]);
            if constexpr (decltype(store_t)::value) {
                uint32_t *q = reinterpret_cast<uint32_t *>(t + n * T_LD + p0 + 8 * g + 4 * h + 2);
                q[0] = packed[2 * g];
                q[1] = packed[2 * g + 1];
            }
        }
    };
    // the input gradient of the wave's tile, masked by the layer's activations prev (same layout),
    // to z; returns the lane's sum of the rounded values
    auto grad_t = [&](const f32x16 &at, const uint16_t *prev, uint16_t *z) {
        float sum = 0.0f;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t *q = reinterpret_cast<const uint32_t *>(prev + n * T_LD + p0 + 8 * g + 4 * h + 2);
            const uint32_t u0 = where_bf16(pack_bf16(at[4 * g], at[4 * g + 1]), q[0]);
            const uint32_t u1 = where_bf16(pack_bf16(at[4 * g + 2], at[4 * g + 3]), q[1]);
            sum += low_bf16(u0);
            sum += high_bf16(u0);
            sum += low_bf16(u1);
            sum += high_bf16(u1);
            *reinterpret_cast<uint2 *>(z + n * T_LD + p0 + 8 * g + 4 * h) = make_uint2(u0, u1);
        }
        return sum;
    };
    fetch(blockIdx.x);
    lds_barrier();
    int since = 0;                              // rows since the last flush
    bool flushed = false;
    for (int r = blockIdx.x; r < A.rows; r += gridDim.x) {
        const float lse = A.lse[r / ROWS], dlogit = A.dlogit[r / ROWS];
        if (tid < NF) {
            reinterpret_cast<uint4 *>(f)[tid] = fp;
            // (all eight channels: the caller's features may fill those spd_prop_features leaves zero)
            const uint32_t w[4] = {fp.x, fp.y, fp.z, fp.w};
#pragma unroll
            for (int c = 0; c < FCH; ++c) ft[c * T_LD + tid] = (uint16_t)(w[c / 2] >> (16 * (c & 1)));
        } else if (tid < NF + 6 * (ACT_LD / 8)) {
            // c1's pads, where z3 was
            const int i = tid - NF, p = i / (ACT_LD / 8), q = i - p * (ACT_LD / 8);
            *reinterpret_cast<uint4 *>(c1 + (p < 2 ? p : POS + p) * ACT_LD + 8 * q) = make_uint4(0u, 0u, 0u, 0u);
        }
        lds_barrier();
        if (r + (int)gridDim.x < A.rows) fetch(r + gridDim.x);
        uint32_t a3[8];
        f32x16 an, at;
        LayerW<CH> V;                           // weights loaded for each row, ahead of their use
        auto load_w = [&](const uint16_t *p) {
            asm volatile("" : "+s"(p));         // (here, not once for all rows)
            V.load(p, l);
        };
        load_w(A.wb.w3);
        // ---- forward
        conv_both<FCH, true>(f, W1, p0, l, an, at);
        relu_both(std::true_type{}, an, at, bias, c1, t1, a3);
        lds_barrier();
        conv_both<CH, true>(c1, W2, p0, l, an, at);
        relu_both(std::true_type{}, an, at, bias + CH, c2, t2, a3);
        lds_barrier();
        conv_both<CH, true>(c2, V, p0, l, an, at);
        relu_both(std::false_type{}, an, at, bias + 2 * CH, c3, t1, a3);
        load_w(A.wb.w3t);
        lds_barrier();
        // ---- read-out of position tid % 256 and half of the gradient at layer 3's output, in place
        {
            const int pos = tid & (POS - 1);
            const bool upper = tid >= POS;      // (uniform over the wave)
            float a[CH];
            uint16_t *p = c3 + act_at(pos + 2, 0);
            load_act(p, a);
            float s = 0.0f;
#pragma unroll
            for (int c = 0; c < CH; c += 4) {
                const float4 w = *reinterpret_cast<const float4 *>(wh + c);
                s += w.x * a[c];
                s += w.y * a[c + 1];
                s += w.z * a[c + 2];
                s += w.w * a[c + 3];
            }
            s += bh;
            const float ds = expf(s - lse) * dlogit;
            if (!upper) {
                gb += ds;
                dsv[pos] = ds;
            }
            lds_barrier();                    // both halves have read the position's activations
            // channels 16 upper .. + 15
            const float *w0 = wh + (upper ? CH / 2 : 0);
            uint4 *out = reinterpret_cast<uint4 *>(p + (upper ? CH / 2 : 0));
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float2 w = *reinterpret_cast<const float2 *>(w0 + 8 * q + 2 * i);
                    const float x = a[8 * q + 2 * i], x1 = a[8 * q + 2 * i + 1];
                    const float y = a[CH / 2 + 8 * q + 2 * i], y1 = a[CH / 2 + 8 * q + 2 * i + 1];
                    const float dx = ds * w.x, dy = ds * w.y;
                    v[i] = pack_bf16((upper ? y : x) > 0.0f ? dx : 0.0f, (upper ? y1 : x1) > 0.0f ? dy : 0.0f);
                }
                out[q] = make_uint4(v[0], v[1], v[2], v[3]);
            }
        }
        // (dsv is complete since the barrier above)
        float gr = 0.0f;                      // the row's
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 d4 = *reinterpret_cast<const float4 *>(dsv + p0 + 8 * g + 4 * h);
            const float ds[4] = {d4.x, d4.y, d4.z, d4.w};
            uint32_t u[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float x = low_bf16(a3[2 * g + i]), y = high_bf16(a3[2 * g + i]);
                gr += ds[2 * i] * x;
                gr += ds[2 * i + 1] * y;
                u[i] = pack_bf16(x > 0.0f ? ds[2 * i] * whn : 0.0f, y > 0.0f ? ds[2 * i + 1] * whn : 0.0f);
                b3 += low_bf16(u[i]);
                b3 += high_bf16(u[i]);
            }
            *reinterpret_cast<uint2 *>(z3 + n * T_LD + p0 + 8 * g + 4 * h) = make_uint2(u[0], u[1]);
        }
        gw += gr;
        lds_barrier();
        // ---- the gradient at layer 2's output, over its activations c2
        conv_both<CH, true>(c3, V, p0, l, an, at);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint2 *q = reinterpret_cast<uint2 *>(c2 + act_at(p0 + n + 2, g) + 4 * h);
            const uint2 m = *q;
            *q = make_uint2(where_bf16(pack_bf16(an[4 * g], an[4 * g + 1]), m.x),
                            where_bf16(pack_bf16(an[4 * g + 2], an[4 * g + 3]), m.y));
        }
        b2 += grad_t(at, t2, z2);
        load_w(A.wb.w2t);
        lds_barrier();
        // ---- the gradient at layer 1's output (none at the features)
        conv_both<CH, false>(c2, V, p0, l, an, at);
        b1 += grad_t(at, t1, z1);
        lds_barrier();
        // ---- weights: half-tile 3 wave + q: tiles 0..4 layer 3, 5..9 layer 2, 10, 11 layer 1
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int job = (3 * wave + q) >> 1, p = ((3 * wave + q) & 1) * 128 + 8 * h;
            const uint16_t *dz = (job < 5 ? z3 : job < 10 ? z2 : z1) + n * T_LD + p;
            const uint16_t *in = (job < 5 ? t2 : job < 10 ? t1 : ft) + (job < 10 ? n : (n & 7)) * T_LD + p;
            switch (job < 10 ? (job < 5 ? job : job - 5) : job - 5) {
                case 0: wgrad_half<0>(dz, in, acc[q], n); break;
                case 1: wgrad_half<1>(dz, in, acc[q], n); break;
                case 2: wgrad_half<2>(dz, in, acc[q], n); break;
                case 3: wgrad_half<3>(dz, in, acc[q], n); break;
                case 5: wgrad_half<-1>(dz, in, acc[q], n); break;
                default: wgrad_half<4>(dz, in, acc[q], n); break;
            }
        }
        if (++since == kBwdFlush || r + (int)gridDim.x >= A.rows) {
            // ---- to the partial: the two halves of each tile in turn (the lane's place in a tile is
            // formed here: kept over the rows, its addresses would push the accumulators out)
            int place = l;
            asm volatile("" : "+v"(place));
            const int pn = place & 31, ph = place >> 5;
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if (((3 * wave + q) & 1) != half) continue;
                    const int job = (3 * wave + q) >> 1;
                    const int k = (job < 5 ? job : job < 10 ? job - 5 : job - 10) * CH + pn;
                    const int ld = job < 10 ? KW : TAPS * FCH;
                    float *p = (job < 5 ? A.part3 + b * P2 : job < 10 ? A.part2 + b * P2 : A.part1 + b * P1) + k;
                    if (job < 11 || pn < 8) {
                        p += 4 * ph * ld;
                        float v[16];
#pragma unroll
                        for (int i = 0; i < 16; ++i) v[i] = 0.0f;
                        if (half || flushed) {
#pragma unroll
                            for (int i = 0; i < 16; ++i) v[i] = p[(8 * (i / 4) + (i % 4)) * ld];
                        }
#pragma unroll
                        for (int i = 0; i < 16; ++i) p[(8 * (i / 4) + (i % 4)) * ld] = v[i] + acc[q][i];
                    }
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[q][i] = 0.0f;
                }
                __syncthreads();
            }
            tot[0][tid] += b1;
            tot[1][tid] += b2;
            tot[2][tid] += b3;
            tot[3][tid] += gw;
            tot[4][tid] += gb;
            b1 = b2 = b3 = gw = gb = 0.0f;
            since = 0;
            flushed = true;
        }
        lds_barrier();                        // everything is rewritten for the next row
    }
    // ---- the lanes' totals: bias and read-out gradients of channel c over the waves in order
    if (tid < 4 * CH) {
        const int i = tid / CH, c = tid - i * CH;
        float v = 0.0f;
        for (int w = 0; w < kBwdThreads / 64; ++w) v += tot[i][64 * w + c] + tot[i][64 * w + 32 + c];
        float *p = i == 0 ? A.part1 + b * P1 + CH * TAPS * FCH : i == 1 ? A.part2 + b * P2 + CH * KW
                   : i == 2 ? A.part3 + b * P2 + CH * KW : A.hpart + b * (CH + 1);
        p[c] = v;
    }
    gb = tot[4][tid];
    for (int o = 32; o > 0; o >>= 1) gb += __shfl_xor(gb, o);
    if (l == 0) red[wave] = gb;
    __syncthreads();
    if (tid == 0) A.hpart[b * (CH + 1) + CH] = (red[0] + red[1]) + (red[2] + red[3]);   // (positions: waves 0..3)
}

// ---------------------------------------------------------------------------------------
// Workspace layout for n_tiles tiles.
// ---------------------------------------------------------------------------------------
struct Layout {
    int64_t wb, row_max, row_sum, lse, dlogit, loss_t, hpart, part1, part2, part3, total;
    int n_parts;
};

inline int64_t up256(int64_t v) { return (v + 255) & ~(int64_t)255; }

Layout layout(int32_t n_tiles) {
    Layout L;
    const int64_t rows = (int64_t)n_tiles * ROWS;
    L.n_parts = (int)(rows < MAX_PARTS ? rows : MAX_PARTS);
    int64_t o = 0;
    auto take = [&](int64_t b) { const int64_t at = o; o += up256(b); return at; };
    L.wb = take((int64_t)(CH * KW1 + 4 * CH * KW) * 2);
    L.row_max = take(rows * 4);
    L.row_sum = take(rows * 4);
    L.lse = take((int64_t)n_tiles * 4);
    L.dlogit = take((int64_t)n_tiles * 4);
    L.loss_t = take((int64_t)n_tiles * 4);
    L.hpart = take((int64_t)L.n_parts * (CH + 1) * 4);
    L.part1 = take((int64_t)L.n_parts * P1 * 4);
    L.part2 = take((int64_t)L.n_parts * P2 * 4);
    L.part3 = take((int64_t)L.n_parts * P2 * 4);
    L.total = o;
    return L;
}

struct Bufs {
    WB wb;
    float *row_max, *row_sum, *lse, *dlogit, *loss_t, *hpart, *part1, *part2, *part3;
};

Bufs bufs(const Layout &L, void *ws) {
    char *b = static_cast<char *>(ws);
    Bufs B;
    uint16_t *w = reinterpret_cast<uint16_t *>(b + L.wb);
    B.wb.w1 = w;
    B.wb.w2 = w + CH * KW1;
    B.wb.w3 = B.wb.w2 + CH * KW;
    B.wb.w2t = B.wb.w3 + CH * KW;
    B.wb.w3t = B.wb.w2t + CH * KW;
    auto at = [&](int64_t o) { return reinterpret_cast<float *>(b + o); };
    B.row_max = at(L.row_max);
    B.row_sum = at(L.row_sum);
    B.lse = at(L.lse);
    B.dlogit = at(L.dlogit);
    B.loss_t = at(L.loss_t);
    B.hpart = at(L.hpart);
    B.part1 = at(L.part1);
    B.part2 = at(L.part2);
    B.part3 = at(L.part3);
    return B;
}

thread_local char g_err[160];

int fail(hipError_t e) {
    snprintf(g_err, sizeof(g_err), "HIP launch failed: %s", hipGetErrorString(e));
    return SPD_EHIP;
}

#define SPDP_LAUNCH(...)                                   \
    do {                                                   \
        hipLaunchKernelGGL(__VA_ARGS__);                   \
        const hipError_t e_ = hipGetLastError();           \
        if (e_ != hipSuccess) return fail(e_);             \
    } while (0)

int check_ws(int32_t n_tiles, const void *ws, int64_t ws_bytes, Layout *L) {
    if (n_tiles < 1 || n_tiles > (1 << 20)) return SPD_EINVAL;
    *L = layout(n_tiles);
    if (!ws || ws_bytes < L->total) return SPD_EWORKSPACE;
    if ((uintptr_t)ws & 255) return SPD_EALIGN;
    return SPD_OK;
}

// Tile logits (labels not null: and losses and what the backward pass needs).
int run_forward(const float *params, const uint16_t *feat, int32_t n_tiles, const float *labels,
                float *logits, const Bufs &B, hipStream_t st) {
    const int rows = n_tiles * ROWS;
    SPDP_LAUNCH(prep_weights_kernel, dim3((CH * KW + 255) / 256), dim3(256), 0, st, params, B.wb);
    InferArgs a;
    a.feat = feat;
    a.wb = B.wb;
    a.params = params;
    a.row_max = B.row_max;
    a.row_sum = B.row_sum;
    a.rows = rows;
    // persistent grid: as many work-groups as the device keeps resident at once, at most one per row
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, infer_kernel, 256, 0) != hipSuccess)
        return fail(hipGetLastError());
    const int grid = std::max(1, std::min(rows, cus * std::max(1, per_cu)));
    SPDP_LAUNCH(infer_kernel, dim3(grid), dim3(256), 0, st, a);
    const CombineArgs c{B.row_max, B.row_sum, labels, logits, B.loss_t, B.lse, B.dlogit, n_tiles};
    SPDP_LAUNCH(combine_kernel, dim3((n_tiles + 3) / 4), dim3(256), 0, st, c);
    return SPD_OK;
}

}  // namespace spdp

using namespace spdp;

extern "C" {

int spd_tiles_generate(uint64_t seed, int64_t first_tile, int32_t n_tiles, float *x,
                       void *hip_stream) {
    if (n_tiles < 1 || n_tiles > (1 << 24) || first_tile < 0 || !x) return SPD_EINVAL;
    TileArgs a{x, seed, first_tile, n_tiles};
    SPDP_LAUNCH(tiles_kernel, dim3((unsigned)n_tiles * ROWS), dim3(256), 0,
                static_cast<hipStream_t>(hip_stream), a);
    return SPD_OK;
}

int spd_prop_features(const float *x, int64_t ld, int32_t n_rows, const float *mean,
                      const float *sigma, uint16_t *feat, void *hip_stream) {
    if (!x || !mean || !sigma || !feat || n_rows < 1 || ld < LEN || (ld & 3)) return SPD_EINVAL;
    if (((uintptr_t)x & 15) || ((uintptr_t)feat & 15)) return SPD_EALIGN;
    FeatArgs a{x, ld, mean, sigma, feat, n_rows, n_rows};
    SPDP_LAUNCH(features_kernel, dim3(n_rows), dim3(256), 0, static_cast<hipStream_t>(hip_stream), a);
    return SPD_OK;
}

int spd_prop_features_block(const float *x, int64_t ld, int32_t n_dm, int32_t n_col, const float *mean,
                            const float *sigma, uint16_t *feat, void *hip_stream) {
    if (!x || !mean || !sigma || !feat || n_dm < 1 || n_col < 1 || ld < (int64_t)n_col * LEN || (ld & 3) ||
        (int64_t)n_dm * n_col > INT32_MAX)
        return SPD_EINVAL;
    if (((uintptr_t)x & 15) || ((uintptr_t)feat & 15)) return SPD_EALIGN;
    FeatArgs a{x, ld, mean, sigma, feat, n_dm, n_dm * n_col};
    SPDP_LAUNCH(features_kernel, dim3(n_dm * n_col), dim3(256), 0, static_cast<hipStream_t>(hip_stream), a);
    return SPD_OK;
}

int spd_prop_workspace(int32_t n_tiles, int64_t *bytes) {
    if (!bytes || n_tiles < 1 || n_tiles > (1 << 20)) return SPD_EINVAL;
    *bytes = layout(n_tiles).total;
    return SPD_OK;
}

int spd_prop_forward(const float *params, const uint16_t *feat, int32_t n_tiles, float *logits,
                     void *workspace, int64_t workspace_bytes, void *hip_stream) {
    Layout L;
    const int st = check_ws(n_tiles, workspace, workspace_bytes, &L);
    if (st != SPD_OK) return st;
    if (!params || !feat || !logits) return SPD_EINVAL;
    if ((uintptr_t)feat & 15) return SPD_EALIGN;
    return run_forward(params, feat, n_tiles, nullptr, logits, bufs(L, workspace),
                       static_cast<hipStream_t>(hip_stream));
}

int spd_prop_backward(const float *params, const uint16_t *feat, const float *labels,
                      int32_t n_tiles, float *logits, float *grads, float *loss,
                      void *workspace, int64_t workspace_bytes, void *hip_stream) {
    Layout L;
    int st = check_ws(n_tiles, workspace, workspace_bytes, &L);
    if (st != SPD_OK) return st;
    if (!params || !feat || !labels || !grads || !loss) return SPD_EINVAL;
    const Bufs B = bufs(L, workspace);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    st = run_forward(params, feat, n_tiles, labels, logits, B, s);
    if (st != SPD_OK) return st;
    const BwdArgs w{feat, B.wb, params, B.lse, B.dlogit, B.part1, B.part2, B.part3, B.hpart, n_tiles * ROWS};
    SPDP_LAUNCH(backward_kernel, dim3(L.n_parts), dim3(kBwdThreads), 0, s, w);
    const RedArgs r{B.part1, B.part2, B.part3, B.hpart, B.loss_t, grads, loss, L.n_parts, n_tiles};
    SPDP_LAUNCH(reduce_kernel, dim3((SPD_PROP_NPARAMS + RED_PARAMS - 1) / RED_PARAMS), dim3(256), 0, s, r);
    return SPD_OK;
}

int spd_prop_adam(float *params, const float *grads, float *m, float *v, int32_t step, float lr,
                  void *hip_stream) {
    if (!params || !grads || !m || !v || step < 1) return SPD_EINVAL;
    AdamArgs a;
    a.p = params;
    a.g = grads;
    a.m = m;
    a.v = v;
    a.lr = lr;
    a.c1 = (float)(1.0 / (1.0 - pow(0.9, step)));
    a.c2 = (float)(1.0 / (1.0 - pow(0.999, step)));
    SPDP_LAUNCH(adam_kernel, dim3((SPD_PROP_NPARAMS + 255) / 256), dim3(256), 0,
                static_cast<hipStream_t>(hip_stream), a);
    return SPD_OK;
}

int spd_tile_max(const float *snr, const spd_plan_info *info, int32_t n_dm, int32_t rows_per_tile,
                 float *tile_max, void *hip_stream) {
    if (!snr || !info || !tile_max || rows_per_tile < 1 || n_dm < rows_per_tile ||
        n_dm % rows_per_tile || info->n_levels < 1 || info->n_levels > SPD_MAX_LEVELS)
        return SPD_EINVAL;
    TileMaxArgs a;
    memset(&a, 0, sizeof(a));
    a.snr = snr;
    a.out = tile_max;
    a.n_levels = info->n_levels;
    a.rows_per_tile = rows_per_tile;
    a.n_tiles = n_dm / rows_per_tile;
    for (int i = 0; i < info->n_levels; ++i) {
        a.off[i] = info->plane_offset[i];
        a.pitch[i] = info->plane_pitch[i];
        a.slots[i] = info->plane_slots[i];
    }
    // the output holds the order keys until the last pass turns them back into floats
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int32_t *key = reinterpret_cast<int32_t *>(tile_max);
    const dim3 tg((a.n_tiles + 255) / 256);
    SPDP_LAUNCH(tile_init_kernel, tg, dim3(256), 0, st, key, a.n_tiles);
    SPDP_LAUNCH(tile_max_kernel, dim3(n_dm), dim3(256), 0, st, a, key);
    SPDP_LAUNCH(tile_fin_kernel, tg, dim3(256), 0, st, key, a.n_tiles);
    return SPD_OK;
}

int spd_prop_labels(const float *exh_max, const float *lossy_max, int32_t n_tiles,
                    float threshold, float margin, float *labels, void *hip_stream) {
    if (!exh_max || !lossy_max || !labels || n_tiles < 1) return SPD_EINVAL;
    const float m = (float)(1.0 + (double)margin);
    SPDP_LAUNCH(labels_kernel, dim3((n_tiles + 255) / 256), dim3(256), 0,
                static_cast<hipStream_t>(hip_stream), exh_max, lossy_max, n_tiles, threshold, m,
                labels);
    return SPD_OK;
}

int spd_prop_flags(const float *logits, int32_t n_row_tiles, int32_t n_col_tiles,
                   float logit_threshold, uint8_t *flags, void *hip_stream) {
    if (!logits || !flags || n_row_tiles < 1 || n_col_tiles < 1 ||
        (int64_t)n_row_tiles * n_col_tiles > INT32_MAX)
        return SPD_EINVAL;
    const int64_t n = (int64_t)n_row_tiles * n_col_tiles;
    SPDP_LAUNCH(flags_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                static_cast<hipStream_t>(hip_stream), logits, n_row_tiles, n_col_tiles,
                logit_threshold, flags);
    return SPD_OK;
}

}  // extern "C"
