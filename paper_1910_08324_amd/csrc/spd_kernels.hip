// Boxcar single-pulse search kernels for gfx950 (CDNA4, wave64).
//
// step_kernel        BoxDIT and IGRID: one launch per step of up to six separation levels.
//                    A work-group takes one tile of a DM row into LDS, forms the decimated
//                    levels on chip and evaluates every level's width set; only the planes and
//                    the last level (1/64 of the input) go back to HBM.
// exh_kernel         exhaustive search (every width 1..L_end): one wave per 256 output slots,
//                    4 consecutive starts per lane, the input window streamed through an LDS ring.
// peak_* kernels     thresholded 3x3 peak finding over the per-level planes, with output in
//                    (level, dm, start) order: count -> scatter.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "spd_internal.h"

namespace spd {

#define SPD_NEG_INF (-__builtin_huge_valf())

// Work-group barrier that orders LDS only: global loads and stores stay in flight across it
// (a full __syncthreads() also waits for every outstanding global access of the wave).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ uint64_t lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// four consecutive floats at any address (global loads need no more than 4-byte alignment)
__device__ __forceinline__ float4 load_f4(const float *p) {
    typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));
    const v4u v = *reinterpret_cast<const v4u *>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

// ----------------------------------------------------------------------------------------
// 1/sqrt(L) table of the exhaustive search.  Computed in FP64 and rounded once to FP32, so
// every kernel scales a boxcar sum by the correctly rounded 1/sqrt(L) (white-noise scaling,
// Section 2.1).  The cascade kernel builds its own small table in LDS the same way.
// ----------------------------------------------------------------------------------------
// rho_d(L) of a measured standard-deviation table (Section 4.6): linear in log2 L between the
// values at adjacent powers of two, held at the last level above it.
__device__ __forceinline__ double rho_of_width(const float *rho_row, int n_rho, double L) {
    const double a = log2(L);
    int k = (int)floor(a + 1e-12);
    if (k >= n_rho - 1) return (double)rho_row[n_rho - 1];
    if (k < 0) k = 0;
    const double f = a - k;
    return (1.0 - f) * (double)rho_row[k] + f * (double)rho_row[k + 1];
}

__global__ void scales_kernel(const ScaleArgs A) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int d = blockIdx.y;
    if (t >= A.n) return;
    if (!A.rho) {
        A.scale[t] = (float)(1.0 / sqrt((double)(t + 1)));
        return;
    }
    const double L = (double)(t + 1);
    const double r = rho_of_width(A.rho + (int64_t)d * A.ld_rho, A.n_rho, L);
    A.scale[(int64_t)d * A.row_ld + t] = (float)(1.0 / (sqrt(L) * r));
}

__global__ void evalmask_kernel(const MaskArgs A) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < A.n_words) A.evalmask[t] = A.bits[t];
}

// ----------------------------------------------------------------------------------------
// BoxDIT / IGRID cascade: one launch per step of up to kStepMaxLevels levels.
//
// Work-group = (DM row d, tile t) of NTH threads (256; 128 for short IG(1) tiles).  The tile
// covers T units of the step's input series (the normalised samples in the first step, the
// decimated series y_{k0} afterwards) plus the halo its widest boxcars reach.  The whole tile
// lives in LDS:
//   1. load the window (coalesced float4), normalising z = (x - mu) / sigma in the first step;
//   2. form the decimated levels in place, one pass and one barrier per level;
//   3. evaluate every level's width set at every slot of the tile, 4 consecutive slots per
//      thread from a register window, writing the SNR/width planes (BoxDIT adds the carried
//      prefix and hands each level's longest boxcar on as the next level's prefix);
//   4. hand the last formed level (and its prefixes) to the next step through HBM.
// A bit per chunk of 256 slots says whether any of them is above the threshold (what the peak
// finder has to look at); candidates-only launches also leave the values and widths of those slots.
//
// The width sets of the paper's configurations are compiled in (FAM selects one): the unit
// counts of a level are then constants, so the bank is straight-line code with 4 VALU
// operations per (slot, width) plus one add per (slot, unit).  Other width sets, and groups
// near the end of the data where some widths do not fit, take the generic path.
// ----------------------------------------------------------------------------------------

// unit-count bitmask (bit U-1) of IGRID IG(d) with P layers: level 0 and level >= 1
__host__ __device__ constexpr uint64_t ig_mask_l0(int P, int d) {
    uint64_t m = 0;
    for (int W = 1; W <= P; W <<= 1) {
        const int inc = (W >> d) > 1 ? (W >> d) : 1;
        for (int q = 0; q < (1 << d); ++q)
            if (W + q * inc < 2 * W) m |= 1ull << (W + q * inc - 1);
    }
    return m;
}
__host__ __device__ constexpr uint64_t ig_mask_lk(int P, int d) {
    uint64_t m = 0;
    for (int q = 0; q < (1 << d); ++q) m |= 1ull << (P + q * (P >> d) - 1);
    return m;
}
__host__ __device__ constexpr uint64_t run_mask(int L) { return L >= 64 ? ~0ull : ((1ull << L) - 1); }

// Compiled-in width patterns of each family: (UMAX, MASK) for pattern 1 and pattern 2, and the
// waves per SIMD the kernel is compiled for (register budget: 8 waves leave 64 VGPRs and 96
// SGPRs per lane; IG(3)'s 30-unit window needs a few more VGPRs than that).
template <int FAM> struct Fam;
template <> struct Fam<0> { static constexpr int U1 = 1, U2 = 1, WAVES = 7;
                            static constexpr uint64_t M1 = 1, M2 = 1; };
template <> struct Fam<1> { static constexpr int U1 = 6, U2 = 6, WAVES = 8;
                            static constexpr uint64_t M1 = ig_mask_l0(4, 1), M2 = ig_mask_lk(4, 1); };
template <> struct Fam<2> { static constexpr int U1 = 14, U2 = 14, WAVES = 8;
                            static constexpr uint64_t M1 = ig_mask_l0(8, 2), M2 = ig_mask_lk(8, 2); };
template <> struct Fam<3> { static constexpr int U1 = 30, U2 = 30, WAVES = 7;
                            static constexpr uint64_t M1 = ig_mask_l0(16, 3), M2 = ig_mask_lk(16, 3); };
template <> struct Fam<4> { static constexpr int U1 = 8, U2 = 8, WAVES = 8;
                            static constexpr uint64_t M1 = run_mask(8), M2 = run_mask(8); };
template <> struct Fam<5> { static constexpr int U1 = 16, U2 = 16, WAVES = 8;
                            static constexpr uint64_t M1 = run_mask(16), M2 = run_mask(16); };
template <> struct Fam<6> { static constexpr int U1 = 32, U2 = 32, WAVES = 7;
                            static constexpr uint64_t M1 = run_mask(32), M2 = run_mask(32); };
template <> struct Fam<7> { static constexpr int U1 = 1, U2 = 1, WAVES = 8;
                            static constexpr uint64_t M1 = 1, M2 = 1; };

template <int NW>
__device__ __forceinline__ void window_load(const float *y, float w[4 * NW]) {
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const float4 v = *reinterpret_cast<const float4 *>(y + 4 * q);
        w[4 * q + 0] = v.x;
        w[4 * q + 1] = v.y;
        w[4 * q + 2] = v.z;
        w[4 * q + 3] = v.w;
    }
}

// All widths of the group fit: straight-line evaluation of a compiled-in width pattern on the
// group's window w (units m0 .. of the level).
// X enters holding the carried prefixes and leaves holding the sum over UMAX units.
// W: bu receives the unit count of the best width (0 if none); without W only the maximum is
// kept (the same value: the largest of the same products).
template <int UMAX, uint64_t MASK, bool W>
__device__ __forceinline__ void bank_fixed(const float *w, const float *rt, float X[kGroup],
                                           float best[kGroup], int bu[kGroup]) {
#pragma unroll
    for (int u = 0; u < UMAX; ++u) {
#pragma unroll
        for (int q = 0; q < kGroup; ++q) X[q] += w[q + u];
        if (((MASK >> u) & 1ull) != 0) {        // folded after unrolling
            const float r = rt[u];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const float v = X[q] * r;
                if (W) {
                    const bool gt = v > best[q];
                    best[q] = gt ? v : best[q];
                    bu[q] = gt ? (u + 1) : bu[q];
                } else {
                    best[q] = fmaxf(best[q], v);
                }
            }
        }
    }
}

// Any width set, with the valid-only check per slot.  Xc receives the sum over `ufull` units
// (the carry handed to the next BoxDIT level).  room: the most units a boxcar of the first slot
// may have inside the data (one less per further slot).  W as for bank_fixed.
template <bool W>
__device__ __forceinline__ void bank_generic(const float *y, const float *rt, int umax,
                                             uint64_t emask, int ufull, int room,
                                             float X[kGroup], float Xc[kGroup],
                                             float best[kGroup], int bu[kGroup]) {
    float4 wa = *reinterpret_cast<const float4 *>(y);
    for (int u4 = 0; u4 < umax; u4 += 4) {
        const float4 wb = *reinterpret_cast<const float4 *>(y + u4 + 4);
        const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int u = u4 + t;
            if (u >= umax) break;
#pragma unroll
            for (int q = 0; q < kGroup; ++q) X[q] += w[q + t];
            if ((emask >> u) & 1ull) {
                const float r = rt[u];
#pragma unroll
                for (int q = 0; q < kGroup; ++q) {
                    float v = X[q] * r;
                    if (u + 1 + q > room) v = SPD_NEG_INF;
                    if (W) {
                        const bool gt = v > best[q];
                        best[q] = gt ? v : best[q];
                        bu[q] = gt ? (u + 1) : bu[q];
                    } else {
                        best[q] = fmaxf(best[q], v);
                    }
                }
            }
            if (u + 1 == ufull) {
#pragma unroll
                for (int q = 0; q < kGroup; ++q) Xc[q] = X[q];
            }
        }
        wa = wb;
    }
}

// The same maxima and widths once more for the few chunks that get a record (candidates only),
// one unit after another: few registers, so that the launch keeps its occupancy.
template <class ScalePtr>
__device__ __forceinline__ void bank_record(const float *y, ScalePtr rt, int umax, uint64_t emask,
                                            int room, float X[kGroup], float best[kGroup],
                                            int bu[kGroup]) {
    float w[kGroup];
#pragma unroll
    for (int q = 1; q < kGroup; ++q) w[q] = y[q - 1];
#pragma unroll 1
    for (int u = 0; u < umax; ++u) {
#pragma unroll
        for (int q = 1; q < kGroup; ++q) w[q - 1] = w[q];
        w[kGroup - 1] = y[u + kGroup - 1];
#pragma unroll
        for (int q = 0; q < kGroup; ++q) X[q] += w[q];
        if ((emask >> u) & 1ull) {
            const float r = rt[u];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const float v = X[q] * r;
                const bool gt = u + 1 + q <= room && v > best[q];
                best[q] = gt ? v : best[q];
                bu[q] = gt ? (u + 1) : bu[q];
            }
        }
    }
}

// Where a tile finds its beam's buffers and sizes: in the launch arguments (one beam per
// launch) or in a table in device memory (many beams per launch).  Both are read-only during a
// launch and the same for every lane of a work-group, so they are addressed in the constant
// address space: their fields load as scalar (SMEM) reads.
// opaque(): the same view behind pointers the compiler cannot see through, so that what is read
// and computed from it stays where it is used.
typedef __attribute__((address_space(4))) const StepArgs *ConstArgsPtr;
typedef __attribute__((address_space(4))) const StepLevel *ConstLevelPtr;
typedef __attribute__((address_space(4))) const BeamView *ConstBeamPtr;
typedef __attribute__((address_space(4))) const int64_t *ConstI64Ptr;
typedef __attribute__((address_space(4))) const float *ConstFloatPtr;

// the launch arguments (StepArgs is the first argument of either kernel, or its first member)
__device__ __forceinline__ ConstArgsPtr launch_args() {
    return (ConstArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
}

struct ArgGeom {
    ConstArgsPtr P;
    __device__ ConstArgsPtr args() const { return P; }
    __device__ ArgGeom opaque() const {
        ConstArgsPtr p = P;
        asm volatile("" : "+s"(p));
        return ArgGeom{p};
    }
    __device__ const float *in() const { return P->in; }
    __device__ const float *cin() const { return P->cin; }
    __device__ float *out() const { return P->out; }
    __device__ float *cout() const { return P->cout; }
    __device__ const float *mean() const { return P->mean; }
    __device__ const float *sigma() const { return P->sigma; }
    __device__ float *Y() const { return P->Y; }
    __device__ uint16_t *W() const { return P->W; }
    __device__ uint32_t *above() const { return P->above; }
    __device__ uint8_t *edge() const { return P->edge; }
    __device__ int n_dm() const { return P->n_dm; }
    __device__ int64_t ld_in() const { return P->ld_in; }
    __device__ int64_t ld_cin() const { return P->ld_cin; }
    __device__ int64_t ld_out() const { return P->ld_out; }
    __device__ int n_in() const { return P->n_in; }
    __device__ int in_len() const { return P->in_len; }
    __device__ int n_tiles() const { return P->n_tiles; }
    __device__ RecStep *rec() const { return P->rec; }
    __device__ uint32_t *dir() const { return P->dir; }
    __device__ uint64_t *pool() const { return P->pool; }
    __device__ unsigned long long *pool_used() const { return P->pool_used; }
    __device__ uint32_t pool_units() const { return P->pool_units; }
    __device__ uint32_t pool_mask() const { return P->pool_mask; }
    __device__ int carry_end() const { return P->carry_end; }
    __device__ int64_t plane_off(int j) const { return P->lv[j].plane_off; }
    __device__ int64_t pitch(int j) const { return P->lv[j].pitch; }
    __device__ int slots(int j) const { return P->lv[j].slots; }
    __device__ int64_t dir_off(int j) const { return P->lv[j].dir_off; }
    __device__ int64_t cnt_off(int j) const { return P->lv[j].cnt_off; }
};

struct TabGeom {
    ConstArgsPtr P;
    ConstBeamPtr V;
    __device__ ConstArgsPtr args() const { return P; }
    __device__ TabGeom opaque() const {
        ConstArgsPtr p = P;
        ConstBeamPtr v = V;
        asm volatile("" : "+s"(p), "+s"(v));
        return TabGeom{p, v};
    }
    __device__ const float *in() const { return V->in; }
    __device__ const float *cin() const { return V->cin; }
    __device__ float *out() const { return V->out; }
    __device__ float *cout() const { return V->cout; }
    __device__ const float *mean() const { return V->mean; }
    __device__ const float *sigma() const { return V->sigma; }
    __device__ float *Y() const { return V->Y; }
    __device__ uint16_t *W() const { return V->W; }
    __device__ uint32_t *above() const { return V->above; }
    __device__ uint8_t *edge() const { return V->edge; }
    __device__ int n_dm() const { return V->n_dm; }
    __device__ int64_t ld_in() const { return V->ld_in; }
    __device__ int64_t ld_cin() const { return V->ld_cin; }
    __device__ int64_t ld_out() const { return V->ld_out; }
    __device__ int n_in() const { return V->n_in; }
    __device__ int in_len() const { return V->in_len; }
    __device__ int n_tiles() const { return V->n_tiles; }
    __device__ RecStep *rec() const { return V->rec; }
    __device__ uint32_t *dir() const { return V->dir; }
    __device__ uint64_t *pool() const { return V->pool; }
    __device__ unsigned long long *pool_used() const { return V->pool_used; }
    __device__ uint32_t pool_units() const { return V->pool_units; }
    __device__ uint32_t pool_mask() const { return V->pool_mask; }
    __device__ int carry_end() const { return V->carry_end; }
    __device__ int64_t plane_off(int j) const { return V->plane_off[j]; }
    __device__ int64_t pitch(int j) const { return V->pitch[j]; }
    __device__ int slots(int j) const { return V->slots[j]; }
    __device__ int64_t dir_off(int j) const { return V->dir_off[j]; }
    __device__ int64_t cnt_off(int j) const { return V->cnt_off[j]; }
};

// Candidates only: the record of a wave's chunk (its 64 groups of kGroup slots): the chunk's slots
// above the threshold with their SNRs and widths, so that the peak finder reads values instead of
// forming them again.  `left`: plane slots from this lane's first one on; `write`: the chunk exists
// in the tile.  Records take their room from part `part` of the beam's pool, `units` long; a chunk that
// finds none is marked and the peak finder forms its slots again.  Returns whether any slot is above.
__device__ __forceinline__ bool put_record(uint64_t *pool, unsigned long long *used, uint32_t part, uint32_t units,
                                           uint32_t *dir, bool write, int lane, int left, float threshold,
                                           const float best[kGroup], const int bu[kGroup], int k,
                                           int base) {
    uint32_t nib = 0;
    uint32_t total = 0;
    int pos = 0;
    const uint64_t below = lanes_below(lane);
#pragma unroll
    for (int q = 0; q < kGroup; ++q) {
        const bool on = q < left && best[q] > threshold;
        const uint64_t b = __ballot(on);
        nib |= on ? 1u << q : 0u;
        pos += __popcll(b & below);
        total += (uint32_t)__popcll(b);
    }
    uint32_t off = kEmptyChunk;
    if (total) {
        const uint32_t need = kChunk / 64 + total;
        if (lane == 0) {
            // (64 bits: every chunk of a search may ask, also when the pool is full)
            const unsigned long long at = atomicAdd(used + part * (kPoolCounterWords / 2), (unsigned long long)need);
            off = at + need <= units ? part * units + (uint32_t)at : kNoRecord;
        }
        off = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
        if (off != kNoRecord) {
            const uint32_t up = (uint32_t)__shfl_down((int)nib, 1);
            uint8_t *bits = reinterpret_cast<uint8_t *>(pool + off);
            if ((lane & 1) == 0) bits[lane >> 1] = (uint8_t)(nib | (up << 4));
            uint2 *ent = reinterpret_cast<uint2 *>(pool + off + kChunk / 64);
#pragma unroll
            for (int q = 0; q < kGroup; ++q)
                if ((nib >> q) & 1u)
                    ent[pos++] = make_uint2(__float_as_uint(best[q]),
                                            bu[q] ? (uint32_t)(base + (bu[q] << k)) : 0u);
        }
    }
    if (lane == 0 && write) *dir = off;
    return total != 0;
}

// The step's record for the peak finder (candidates only): pointers, sizes and level constants,
// exactly those the tiles of this launch use.  Written by one work-group.
template <int NTH, class G>
__device__ __forceinline__ void write_rec(const StepArgs &A, const G &V, RecStep *R) {
    const int tid = threadIdx.x;
    for (int i = tid; i < A.J * kMaxLevelWidths; i += NTH) {
        const int j = i / kMaxLevelWidths, u = i - j * kMaxLevelWidths;
        R->lv[j].rt[u] = A.rtab[j][u];
    }
    if (tid < A.J) {
        const StepLevel &L = A.lv[tid];
        RecLevel &r = R->lv[tid];
        r.k = L.k;
        r.cshift = L.cshift;
        r.umax = L.umax;
        r.ufull = L.ufull;
        r.base = L.base;
        r.slots = V.slots(tid);
        r.evalmask = L.evalmask;
    }
    if (tid == 0) {
        R->in = V.in();
        R->cin = V.cin();
        R->mean = V.mean();
        R->sigma = V.sigma();
        R->rho = A.rho;
        R->ld_in = V.ld_in();
        R->ld_cin = V.ld_cin();
        R->ld_rho = A.ld_rho;
        R->n_rho = A.n_rho;
        R->in_len = V.in_len();
        R->n_in = V.n_in();
        R->normalise = A.normalise;
        R->carry = A.carry;
        R->J = A.J;
    }
}

// Candidates only: what the peak finder gets of one chunk (a wave's 64 groups from gw on) of level j:
// its bit in the tile's word and its record.  Runs for the few chunks with a slot above the threshold,
// and evaluates them once more from the windows in LDS, so that the width sets' registers need not live
// across it.  V hides where its fields come from (see opaque()), so that none of its loads and address
// arithmetic moves into the tile's main path.
template <bool RHO, class G>
__device__ __forceinline__ void step_chunk(const G V, int j, int d, int tile, int gw, bool any,
                                           float *lds, uint32_t *st_cnt) {
    const ConstArgsPtr A = V.args();
    ConstLevelPtr L = A->lv + j;
    const int lane = threadIdx.x & 63;
    const int Sj = A->T >> j;
    const int ngroups = Sj / kGroup;
    const int g = gw + lane;
    const int chunk = gw >> 6;
    const int m0 = min(g, ngroups - 1) * kGroup;
    const int slots = V.slots(j);
    const int ma = tile * Sj + m0;
    float best[kGroup];
    int bu[kGroup];
#pragma unroll
    for (int q = 0; q < kGroup; ++q) {
        best[q] = SPD_NEG_INF;
        bu[q] = 0;
    }
    if (any && g < ngroups && ma < slots) {
        const bool has_carry = A->carry && (j > 0 || V.cin() != nullptr);
        const float *c = lds + A->lv[0].lds_c + m0;
        float X[kGroup];
#pragma unroll
        for (int q = 0; q < kGroup; ++q) X[q] = has_carry ? c[q] : 0.0f;
        const int room = (int)(((int64_t)V.n_in() - L->base) >> L->k) - ma;
        if constexpr (RHO)
            bank_record(lds + A->lv[0].lds_y + m0, (const float *)(lds + A->lds_sc + j * kMaxLevelWidths), L->umax,
                        L->evalmask, room, X, best, bu);
        else
            bank_record(lds + A->lv[0].lds_y + m0, (ConstFloatPtr)A->rtab[j], L->umax, L->evalmask, room, X, best, bu);
    }
    const int item = d * V.n_tiles() + tile;
    const int64_t di = V.dir_off(j) + (int64_t)item * L->cpt + chunk;
    const bool set = put_record(V.pool(), V.pool_used(), (uint32_t)item & V.pool_mask(), V.pool_units(), V.dir() + di,
                                chunk < L->cpt, lane, slots - ma, A->threshold, best, bu, L->k, L->base);
    if (set && lane == 0) atomicOr(&st_cnt[j], 1u << (chunk >> L->bit_shift));
}

// One tile (DM row d, tile `tile`) of a cascade launch.  A holds what every beam of the launch
// shares (levels, width patterns, tile length); G the beam's buffers and sizes.  W: the planes
// are stored (A.write_planes), so the banks also track the best width; candidates-only
// launches keep the maxima only.
template <bool FIRST, int FAM, bool RHO, int NTH, bool W, class G>
__device__ __forceinline__ void step_tile(const StepArgs &A, const G &V, const int d,
                                          const int tile, float *lds, uint32_t *st_cnt) {
    const int tid = threadIdx.x;
    const int T = A.T;
    if (RHO) {
        // this row's 1/sigma(L) relative to 1/(sqrt(L) sigma): scale[j][u-1] = rtab[j][u-1] / rho(L)
        const float *rr = A.rho + (int64_t)d * A.ld_rho;
        float *sc = lds + A.lds_sc;
        for (int i = tid; i < A.J * kMaxLevelWidths; i += NTH) {
            const int j = i / kMaxLevelWidths, u = i - j * kMaxLevelWidths + 1;
            if (u <= A.lv[j].umax) {
                const double L = (double)A.lv[j].base + ldexp((double)u, A.lv[j].k);
                sc[i] = (float)((double)A.rtab[j][u - 1] / rho_of_width(rr, A.n_rho, L));
            }
        }
    }
    // carried prefixes: BoxDIT families always, IGRID families never (known at compile time, so
    // their code and branches vanish), the generic kernel as the launch says
    constexpr int kCarry = (FAM >= 4 && FAM <= 6) ? 1 : (FAM == 0 ? -1 : 0);
    const bool carry = kCarry < 0 ? (A.carry != 0) : (kCarry == 1);
    const int64_t u0 = (int64_t)tile * T;
    if (tid < kStepMaxLevels) st_cnt[tid] = 0;
    if (d == 0 && tile == 0 && V.rec()) write_rec<NTH>(A, V, V.rec());

    // ---- 1. window of the input series (normalised in the first step) and carried prefixes
    {
        const float *inr = V.in() + (int64_t)d * V.ld_in();
        float mu = 0.0f, inv = 1.0f;
        if (FIRST) {
            mu = V.mean()[d];
            inv = 1.0f / V.sigma()[d];
        }
        const int N0 = A.lv[0].n_units;
        float *y0 = lds + A.lv[0].lds_y;
        const int64_t len = V.in_len();
        // up to kLoadBatch float4 loads per thread are issued before any of them is used, so a
        // tile's window costs about one memory round trip rather than one per float4 (rows need
        // no more than their 4-byte alignment)
        constexpr int kLoadBatch = 8;
        auto norm = [&](float4 w) {
            if (FIRST) {
                w.x = (w.x - mu) * inv;
                w.y = (w.y - mu) * inv;
                w.z = (w.z - mu) * inv;
                w.w = (w.w - mu) * inv;
            }
            return w;
        };
        const float *src = inr + u0;
        if (u0 + N0 <= len) {                           // the whole window is in the data
            for (int i0 = 4 * tid; i0 - 4 * tid < N0; i0 += 4 * NTH * kLoadBatch) {
                float4 v[kLoadBatch];
#pragma unroll
                for (int b = 0; b < kLoadBatch; ++b) {
                    if (i0 - 4 * tid + 4 * NTH * b >= N0) break;
                    v[b] = load_f4(src + min(i0 + 4 * NTH * b, N0 - 4));
                }
#pragma unroll
                for (int b = 0; b < kLoadBatch; ++b) {
                    if (i0 - 4 * tid + 4 * NTH * b >= N0) break;
                    // (lanes past the window hold its last float4 and write it again)
                    *reinterpret_cast<float4 *>(y0 + min(i0 + 4 * NTH * b, N0 - 4)) = norm(v[b]);
                }
            }
        } else {
            // the row's end: float4 up to it, then one sample at a time, then zeros
            const int rest = (int)max((int64_t)0, len - u0);
            for (int i0 = 4 * tid; i0 < N0; i0 += 4 * NTH * kLoadBatch) {
                float4 v[kLoadBatch];
#pragma unroll
                for (int b = 0; b < kLoadBatch; ++b) {
                    const int i = i0 + 4 * NTH * b;
                    if (i + 4 <= rest) v[b] = load_f4(src + i);
                }
#pragma unroll
                for (int b = 0; b < kLoadBatch; ++b) {
                    const int i = i0 + 4 * NTH * b;
                    if (i >= N0) break;
                    float4 w = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (i + 4 <= rest) {
                        w = norm(v[b]);
                    } else if (i < rest) {
                        w.x = FIRST ? (src[i] - mu) * inv : src[i];
                        if (i + 1 < rest) w.y = FIRST ? (src[i + 1] - mu) * inv : src[i + 1];
                        if (i + 2 < rest) w.z = FIRST ? (src[i + 2] - mu) * inv : src[i + 2];
                    }
                    *reinterpret_cast<float4 *>(y0 + i) = w;
                }
            }
        }
        if (!FIRST && carry && V.cin()) {
            const float *cr = V.cin() + (int64_t)d * V.ld_cin();
            float *c0 = lds + A.lv[0].lds_c;
            const int64_t cend = max((int64_t)V.slots(0), min((int64_t)V.carry_end() + 1, len));
            for (int i = tid; i < T; i += NTH) {
                const int64_t m = u0 + i;
                c0[i] = (m < cend) ? cr[m] : 0.0f;
            }
        }
    }
    lds_barrier();

    // ---- 2+3. cascade fused with the width sets.  Level j is evaluated in batches of NTH groups,
    // one per thread; each group also forms its two units of level j+1 (and, for BoxDIT, its two
    // carried prefixes) in registers.  After a barrier that ends the batch's reads they are
    // written in place: unit n of level j+1 goes to index n of the same buffer, below every
    // unit of level j a later batch still reads (and likewise for the carries).  The units of
    // level j+1 past the tile's slots (its halo) are formed after the last batch.
    // A wave whose groups lie in the plane and, at every width, in the data (one scalar comparison)
    // runs a compiled-in bank with no test per lane; the others the generic one.
    // What is needed only where a chunk has a slot above the threshold stays in step_chunk, out of
    // this loop's registers: the scalar unit, one for the whole CU, bounds the light width sets (eight
    // uneven beams, IG(1) candidates only: 919 scalar instructions per wave of a tile of 4096 when
    // tests per lane and the candidates' addresses were here, 654 now, 0.74 a clock).  Before -> after,
    // at equal tiles: those beams 2741 -> 2135 us, 1024 x 131072 BD-16 909 -> 793, 500 x 100003 IG(1)
    // (rows of any alignment take float4 loads) 241 -> 200; and 2000 -> 1925, 683 -> 676 and 197 -> 192
    // since launches with planes set their chunk bits here and the maxima at a row's end are left to
    // the peak finder.
    // Reading a window ahead of the barrier, which paid while LDS was the bound, and several
    // batches per barrier are slower now (batch 2245 and 2630 us).
    constexpr int kNW = (kGroup + Fam<FAM>::U1 - 1 + 3) / 4;
    constexpr bool kOnePattern = FAM == 0 || (Fam<FAM>::M1 == Fam<FAM>::M2 && Fam<FAM>::U1 == Fam<FAM>::U2);
    // A wave that reaches past the plane with every width in the data (look-ahead samples) runs the
    // compiled-in bank too in the densest sets, whose generic bank is what a small launch waits for
    // (16 x 16384 samples, planes: BD-32 65 -> 55 us, IG(3) 52 -> 47; with BD-16 also 49 -> 46, but 1024 x
    // 131072 samples then take 676 -> 680, and IG(1)'s beam 3304 -> 3314).
    constexpr bool kPastEnd = Fam<FAM>::U1 >= 30;
    const int jtop = A.has_out ? A.J : A.J - 1;
    float *ybuf = lds + A.lv[0].lds_y;
    float *cbuf = lds + A.lv[0].lds_c;
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    for (int j = 0; j < A.J; ++j) {
        const bool form_next = j + 1 <= jtop;
        const StepLevel &L = A.lv[j];
        const int Sj = T >> j;
        const int ms0 = tile * Sj;                         // absolute slot of tile slot 0
        const int ngroups = Sj / kGroup;
        const int slots = V.slots(j);
        const bool has_carry = carry && (j > 0 || V.cin() != nullptr);
        const bool to_lds = carry && (j + 1 < A.J);
        const bool to_glb = carry && (j + 1 == A.J) && A.has_out;
        float *cg = to_glb ? V.cout() + (int64_t)d * V.ld_out() + (int64_t)tile * (T >> A.J) : nullptr;
        const bool sync_batches = form_next || to_lds;   // a batch writes into the live buffers
        const int k = L.k;
        const int umax = L.umax;
        const int base = L.base;
        const float *rt = RHO ? lds + A.lds_sc + j * kMaxLevelWidths : A.rtab[j];
        float *rowY = nullptr;
        uint16_t *rowW = nullptr;
        if (W) {
            const int64_t o = V.plane_off(j) + (int64_t)d * V.pitch(j) + ms0;
            rowY = V.Y() + o;
            rowW = V.W() + o;
        }
        // U units from slot m end inside the data when m + U is at most this
        const int ends = (int)(((int64_t)V.n_in() - base) >> k);
        // groups below this have every width of every slot inside the data and lie in the plane
        const int inner = (FAM != 0 && L.pattern != 0)
                              ? min(ngroups, (min(ends - umax + 1, slots) - ms0) >> 2) : 0;
        static_assert(kGroup == 4, "groups of four slots");
        for (int gb = 0; gb < ngroups; gb += NTH) {
            const int gw = gb + wave0;                   // the wave's first group
            const int g = gb + tid;
            float nu0 = 0.0f, nu1 = 0.0f, xc0 = 0.0f, xc1 = 0.0f;
            if (gw < ngroups) {
                float best[kGroup], X[kGroup];
                int bu[kGroup];
#pragma unroll
                for (int q = 0; q < kGroup; ++q) {
                    best[q] = SPD_NEG_INF;
                    bu[q] = 0;
                    X[q] = 0.0f;
                }
                bool any;
                const int m0 = min(g, ngroups - 1) * kGroup;   // (lanes past the tile repeat its last group)
                const float *y = ybuf + m0;
                if (FAM != 0 && min(gw + 64, ngroups) <= inner) {
                    if (has_carry) {
                        const float4 c = *reinterpret_cast<const float4 *>(cbuf + m0);
                        X[0] = c.x;
                        X[1] = c.y;
                        X[2] = c.z;
                        X[3] = c.w;
                    }
                    float w[4 * kNW];
                    window_load<kNW>(y, w);
                    // y_{j+1}[n] = y_j[2n + cshift] + y_j[2n + cshift + 1] for 2n + cshift = m0, m0 + 2
                    nu0 = w[0] + w[1];
                    nu1 = w[2] + w[3];
                    if (kOnePattern || (FIRST && j == 0))
                        bank_fixed<Fam<FAM>::U1, Fam<FAM>::M1, W>(w, rt, X, best, bu);
                    else
                        bank_fixed<Fam<FAM>::U2, Fam<FAM>::M2, W>(w, rt, X, best, bu);
                    xc0 = X[0];
                    xc1 = X[2];
                    // (the maxima are formed here: sunk below the branches that follow, they would keep
                    // every partial sum of the bank in registers)
                    asm volatile("" : "+v"(best[0]), "+v"(best[1]), "+v"(best[2]), "+v"(best[3]));
                    if (W) asm volatile("" : "+v"(bu[0]), "+v"(bu[1]), "+v"(bu[2]), "+v"(bu[3]));
                    if (W) {
                        uint32_t bw[kGroup];
#pragma unroll
                        for (int q = 0; q < kGroup; ++q)
                            bw[q] = (kCarry == 0 || bu[q]) ? (uint32_t)(base + (bu[q] << k)) : 0u;   // (IGRID: base 0)
                        *reinterpret_cast<float4 *>(rowY + m0) = make_float4(best[0], best[1], best[2], best[3]);
                        *reinterpret_cast<uint2 *>(rowW + m0) = make_uint2(bw[0] | (bw[1] << 16), bw[2] | (bw[3] << 16));
                    }
                    if (cg) *reinterpret_cast<float2 *>(cg + (m0 >> 1)) = make_float2(xc0, xc1);
                    any = __ballot(fmaxf(fmaxf(best[0], best[1]), fmaxf(best[2], best[3])) > A.threshold) != 0;
                } else {
                    const int ma = ms0 + m0;
                    const float4 w0 = *reinterpret_cast<const float4 *>(y);
                    nu0 = w0.x + w0.y;
                    nu1 = w0.z + w0.w;
                    const bool act = g < ngroups && ma < slots;
                    if (act || (carry && g < ngroups && ma <= V.carry_end() >> j)) {   // (for the carry alone)
                        if (has_carry) {
#pragma unroll
                            for (int q = 0; q < kGroup; ++q) X[q] = cbuf[m0 + q];
                        }
                        float Xc[kGroup] = {0.0f, 0.0f, 0.0f, 0.0f};
                        if (kPastEnd && L.pattern != 0 &&
                            min(gw + 64, ngroups) <= ((ends - umax + 1 - ms0) >> 2)) {
                            float w[4 * kNW];
                            window_load<kNW>(y, w);
                            if (kOnePattern || (FIRST && j == 0))
                                bank_fixed<Fam<FAM>::U1, Fam<FAM>::M1, W>(w, rt, X, best, bu);
                            else
                                bank_fixed<Fam<FAM>::U2, Fam<FAM>::M2, W>(w, rt, X, best, bu);
#pragma unroll
                            for (int q = 0; q < kGroup; ++q) Xc[q] = X[q];
                        } else {
                            bank_generic<W>(y, rt, umax, L.evalmask, L.ufull, ends - ma, X, Xc, best, bu);
                        }
                        xc0 = Xc[0];
                        xc1 = Xc[2];
                        if (W) {
#pragma unroll
                            for (int q = 0; q < kGroup; ++q)
                                if (ma + q < slots) {
                                    rowY[m0 + q] = best[q];
                                    rowW[m0 + q] = (uint16_t)(bu[q] ? base + (bu[q] << k) : 0);
                                }
                        }
                        if (A.want_cand && act && ma + kGroup > slots && V.edge()) {
                            // the row's last slot against the evaluated slot after it
                            bool below = false;
#pragma unroll
                            for (int q = 0; q + 1 < kGroup; ++q)
                                if (ma + q + 1 == slots) below = !(best[q] >= best[q + 1]);
                            V.edge()[(int64_t)k * V.n_dm() + d] = below;
                        }
                        if (cg) {
                            // the last level's longest boxcar is the next step's carried prefix
                            cg[(m0 >> 1) + 0] = xc0;
                            cg[(m0 >> 1) + 1] = xc1;
                        }
                    }
                    any = __ballot(act && fmaxf(fmaxf(best[0], best[1]), fmaxf(best[2], best[3])) > A.threshold) != 0;
                }
                if constexpr (W) {
                    if (A.want_cand && any && tid == wave0) atomicOr(&st_cnt[j], 1u << ((gw >> 6) >> L.bit_shift));
                } else {
                    if (A.want_cand && (any || L.bit_shift))
                        step_chunk<RHO>(V.opaque(), j, d, tile, gw, any, lds, st_cnt);
                }
            }
            if (sync_batches) {
                lds_barrier();                   // the batch's reads of level j are done
                if (g < ngroups) {
                    if (kCarry == 0) {           // (IGRID: no shift, so the pair is one aligned float2)
                        *reinterpret_cast<float2 *>(ybuf + 2 * g) = make_float2(nu0, nu1);
                    } else {
                        const int n_next = form_next ? A.lv[j + 1].n_units : 0;
                        const int n0 = form_next ? (g * kGroup - A.lv[j + 1].cshift) >> 1 : -2;
                        if (n0 >= 0 && n0 < n_next) ybuf[n0] = nu0;
                        if (n0 + 1 >= 0 && n0 + 1 < n_next) ybuf[n0 + 1] = nu1;
                        // this level's longest boxcar is the next level's carried prefix (zero where
                        // it is not formed)
                        if (to_lds)
                            *reinterpret_cast<float2 *>(cbuf + 2 * g) = make_float2(xc0, xc1);
                    }
                }
            }
        }
        if (form_next) {
            // halo units of level j+1: read at index >= S_j, written below it
            const int cs1 = A.lv[j + 1].cshift, n_next = A.lv[j + 1].n_units;
            for (int n = max(0, (Sj - cs1) >> 1) + tid; n < n_next; n += NTH) {
                const float2 p = *reinterpret_cast<const float2 *>(ybuf + 2 * n + cs1);
                ybuf[n] = p.x + p.y;
            }
        }
        lds_barrier();                       // level j+1 is complete
    }

    // ---- 4. hand on the last formed level
    if (A.has_out) {
        const float *yJ = lds + A.lv[0].lds_y;
        float *o = V.out() + (int64_t)d * V.ld_out() + (int64_t)tile * (T >> A.J);
        for (int n = tid; n < (T >> A.J); n += NTH) o[n] = yJ[n];
    }
    if (A.want_cand) {
        lds_barrier();
        // the tile's chunk bits of all its levels side by side (one short write per work-group)
        if (tid < A.J)
            V.above()[V.cnt_off(tid) + ((int64_t)d * V.n_tiles() + tile) * A.J] = st_cnt[tid];
    }
}


// The tile of work-group i of n.  Consecutive work-groups go to the 8 XCDs in turn; here each XCD
// takes runs of kXcdRun consecutive tiles instead.  A tile's halo is then in its XCD's L2, and an
// XCD's requests no longer step by 8 tiles, which with tiles of a power of two kept them on few
// channels: tiles of 4096, 1024 x 131072, 4 levels a launch: BD-16 782 -> 669 us, IG(2) 510 -> 453;
// 4096 x 262144 IG(1) 3507 -> 3292, candidates only 1622 -> 1495.  (Runs of 4 and 16 gain less, of
// 1024 the same; tiles of 3072 and 6144 gain 0-3%.)
constexpr int kXcds = 8, kXcdRun = 64;
__device__ __forceinline__ int64_t xcd_order(int64_t i, int64_t n) {
    constexpr int kSpan = kXcds * kXcdRun;
    const int64_t first = i / kSpan * kSpan;
    if (first + kSpan > n) return i;                   // the last, partial span in order
    const int r = (int)(i - first);
    return first + (r % kXcds) * kXcdRun + r / kXcds;
}

// One launch for one beam: work-group = (DM row, tile) of NTH threads.
template <bool FIRST, int FAM, bool RHO, int NTH, bool W>
__global__ __launch_bounds__(NTH, (Fam<FAM>::WAVES)) void step_kernel(const StepArgs A) {
    // (16-byte alignment matters: with the buffer right behind st_cnt, at 8 bytes past a multiple
    // of 16, every float4 access of a tile was misaligned, and LDS, busy 95% of the cycles, bounded
    // every width set; now 15%: 1024 x 131072 BD-16 1000 -> 909 us, IG(2) with a sigma table 696 -> 553)
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ uint32_t st_cnt[kStepMaxLevels];
    const int i = (int)xcd_order(blockIdx.x, (int64_t)A.n_dm * A.n_tiles);
    const int d = i / A.n_tiles;
    const int tile = i - d * A.n_tiles;
    if (d >= A.n_dm) return;
    step_tile<FIRST, FAM, RHO, NTH, W>(A, ArgGeom{launch_args()}, d, tile, lds, st_cnt);
}

// One launch for many beams (same levels and tile length, any sizes): a persistent grid walks
// the work items (beam, DM row, tile) in order; item i belongs to the beam b with
// item_base[b] <= i < item_base[b + 1].  (The beam's fields and the loop cost registers: candidates
// only, the compiled-in families' first steps keep 2 to 7 VGPRs and 54 to 106 SGPRs a wave in spill
// slots, a single beam's none and 1 to 36; with planes none but IG(3), 4 VGPRs.)
template <bool FIRST, int FAM, bool W>
__global__ __launch_bounds__(kStepThreads, (Fam<FAM>::WAVES)) void step_kernel_batch(const StepBatchArgs B) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ uint32_t st_cnt[kStepMaxLevels];
    const ConstBeamPtr beams = (ConstBeamPtr)B.beams;
    const ConstI64Ptr base = (ConstI64Ptr)B.item_base;
    int b = -1;
    for (int64_t i = blockIdx.x; i < B.n_items; i += gridDim.x) {
        // (a smaller persistent grid keeps the items in order: they must not go backwards)
        const int64_t item = gridDim.x >= B.n_items ? xcd_order(i, B.n_items) : i;
        if (b < 0) {
            // the first item's beam by halving: each step is a scalar load that the next waits for
            // (32 beams of 512..4096 rows: 49.1 ms walking from the first beam, 44.6 halving)
            b = 0;
            for (int hi = B.n_beams - 1; b < hi;) {
                const int mid = (b + hi + 1) >> 1;
                if (base[mid] <= item) b = mid;
                else hi = mid - 1;
            }
        }
        while (b + 1 < B.n_beams && base[b + 1] <= item) ++b;
        const TabGeom V{launch_args(), beams + b};
        const int64_t local = item - base[b];
        const int d = (int)(local / V.n_tiles());
        const int tile = (int)(local - (int64_t)d * V.n_tiles());
        if (i != (int64_t)blockIdx.x) lds_barrier();   // the previous item is done with LDS
        step_tile<FIRST, FAM, false, kStepThreads, W>(B.s, V, d, tile, lds, st_cnt);
    }
}

// ----------------------------------------------------------------------------------------
// Exhaustive search kernel.
//
// Work item = (row d, 256 output slots starting at s0).  Lane l owns the 4 consecutive starts
// s0 + 4l + v.  Widths are visited in increasing order with one running sum per start, in
// groups of 16: inside a group only the maximum is tracked (add, multiply, max per start and
// width); after the group the best group, and the running sum entering it, are kept.  The
// winning width inside the winning group is recovered at the end by replaying that group's steps
// with the same FP32 operations, so it is the smallest width attaining the maximum, exactly as a
// per-width argmax would give.
// The input window z[s0 .. s0 + 256 + L_end) streams through a 1024-float LDS ring, 512 new
// samples per block of 512 widths.  The ring's first 18 float4 are mirrored after its end, so a
// group reads its consecutive float4 at immediate offsets from one base address.
//
// Long width sets (PRUNE) are bound by the vector issue rate: 2.5 instructions per (start, width)
// and the groups' bookkeeping.  Most groups of 64 widths at large L raise no start's best, and an
// upper bound that shows it needs little more than the running sums themselves (exh_bound): 1.3
// instructions per pair, and the group is then skipped.  Only where the bound does not rule a new best out
// for every start of the wave is the group evaluated; a group that did raise one is followed by
// plain evaluation, since such groups come in runs.  On white noise about one group in six is
// evaluated up to L_end 8192, half of those below 1024, so bounds start at width 257.  Measured:
// 128 x 131072 at L_end 8192 7.63 -> 5.78 ms (2.0 instead of 2.9 vector instructions per pair, 85% of
// the issue rate; 6 VGPRs spill at 6 waves per SIMD); 64 x 65536 at L_end 256, where the replay's
// fetches one after another cost as much as the widths, 137 -> 111 us.  Rows on which bounds are paid
// and fail are no slower than without them: 32 x 65536 samples, 18 kinds of rows (trends, steps of 64
// to 4096, offsets, sines, red noise, spikes, constants) take 0.66 to 0.88 of the time at L_end 1000
// and 4096.
__device__ __forceinline__ float load_z(const float *xr, int r, int n_in, float mu, float inv) {
    return r < n_in ? (xr[r] - mu) * inv : 0.0f;
}

// The width scales of a row are read-only during the launch and indexed by the group's widths,
// which every lane shares: addressed in the constant address space (ConstFloatPtr) they load as
// scalar reads.

constexpr int kRing4 = 256;        // float4 slots of the ring (1024 samples)
constexpr int kGuard4 = 18;        // mirrored slots after the ring's end

__device__ __forceinline__ void ring_put(float4 *ring4, int i, float4 v) {   // 0 <= i < kRing4
    ring4[i] = v;
    if (i < kGuard4) ring4[kRing4 + i] = v;
}

// G widths L0 .. L0+G-1 at the lane's 4 starts: running sums X, group maxima gm.  The window
// z[s0 + 4 lane + L0 - 1 ..] is read from the LDS ring one float4 per 4 widths.
template <bool CHECK, bool DENSE, int G>
__device__ __forceinline__ void exh_group(const float4 *ring4, int jb4, int L0, ConstFloatPtr scale,
                                          const uint32_t *evalmask, int Lw, const int room[4],
                                          float X[4], float gm[4]) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f *win = reinterpret_cast<const v4f *>(ring4 + (jb4 & (kRing4 - 1)));
    v4f wa = win[0];
#pragma unroll 4
    for (int t = 0; t < G / 4; ++t) {
        const v4f wb = win[t + 1];
        const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
        const int L = L0 + 4 * t;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const float r = scale[L - 1 + tt];
            bool on = true;
            if (!DENSE) on = (evalmask[(L - 1 + tt) >> 5] >> ((L - 1 + tt) & 31)) & 1u;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                X[v] += w[v + tt];
                float snr = X[v] * r;
                if (CHECK) {
                    const bool ok = (L + tt <= Lw) && (L + tt <= room[v]);
                    snr = ok ? snr : SPD_NEG_INF;
                }
                if (!DENSE) snr = on ? snr : SPD_NEG_INF;
                gm[v] = fmaxf(gm[v], snr);
            }
        }
        wa = wb;
    }
}

// Upper bound of each start's SNR over the kExhGroup widths from L0, and the running sums past
// them.  Only start 0's sums are followed by a running maximum, over three widths more than the
// group's; the group's sums of start v are, but for rounding, start 0's v widths later, shifted by a
// constant:  X_v(L) = X_0(L + v) + (Xs_v - Xs_0) - (the first v samples start 0 adds).
// Both sides are chains of at most kExhGroup + 3 additions of samples no larger than zmax, so
// every partial sum is at most A = |Xs_0| + |Xs_v| + 70 zmax and their roundings together stay
// below 145 2^-24 A < 1e-5 A.  The scale falls with the width, so r_first bounds a sum above zero
// and r_last one below.  (A sum or sample that is not finite makes the bound fail its comparison.)
__device__ __forceinline__ void exh_bound(const float4 *ring4, int jb4, float zmax, float r_first,
                                          float r_last, float X[4], float ub[4]) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f *win = reinterpret_cast<const v4f *>(ring4 + (jb4 & (kRing4 - 1)));
    v4f wa = win[0];
    const float d[4] = {0.0f, wa.x, wa.x + wa.y, (wa.x + wa.y) + wa.z};
    float xs[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) xs[v] = X[v];
    float m = SPD_NEG_INF;
#pragma unroll 4
    for (int t = 0; t < kExhGroup / 4; ++t) {
        const v4f wb = win[t + 1];
        const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
            for (int v = 0; v < 4; ++v) X[v] += w[v + tt];
            m = fmaxf(m, X[0]);
        }
        wa = wb;
    }
    const float x1 = X[0] + wa.x, x2 = x1 + wa.y, x3 = x2 + wa.z;
    m = fmaxf(m, fmaxf(x1, fmaxf(x2, x3)));
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float A = fabsf(xs[0]) + fabsf(xs[v]) + 70.0f * zmax;
        const float top = (m + (xs[v] - xs[0])) - d[v] + 1e-5f * A;
        ub[v] = fmaxf(top * r_first, top * r_last);
        if (!(fabsf(top) < __builtin_huge_valf())) ub[v] = __builtin_huge_valf();
    }
}

template <bool DENSE, bool MULTI, bool PRUNE>
__global__ __launch_bounds__(64, 6) void exh_kernel(const ExhArgs A) {
    static_assert(!PRUNE || (DENSE && !MULTI), "bounds are for long dense width sets");
    constexpr int G = kExhGroup / 4;
    __shared__ float4 ring4[kRing4 + kGuard4];

    // A wave takes `per` consecutive work items of a row (MULTI: several, when every width fits
    // one block of the ring, so each further item needs only 256 new samples, loaded while the
    // previous item computes).  Ring position 0 holds sample `base`.
    const int lane = threadIdx.x;
    const int per = MULTI ? A.segs_per_wave : 1;
    const int waves_per_row = (A.n_seg + per - 1) / per;
    const int d = blockIdx.x / waves_per_row;
    const int g0 = (blockIdx.x - d * waves_per_row) * per;
    if (d >= A.n_dm) return;
    const int g_end = min(g0 + per, A.n_seg);
    if (A.tile_flag) {
        // tile-gated: a wave's items lie in one tile (tile_len is a multiple of 1024 samples)
        const int64_t t = (int64_t)(d / A.tile_rows) * A.n_col_tiles + (g0 * kExhSlots) / A.tile_len;
        if (!A.tile_flag[t]) {
            if (A.want_cand && lane == 0)
                for (int g = g0; g < g_end; ++g) A.above[(int64_t)d * A.n_seg + g] = 0;
            return;
        }
    }
    const int base = g0 * kExhSlots;
    const float *xr = A.x + (int64_t)d * A.ld;
    const float *srow = A.scale + (int64_t)d * A.scale_ld;     // this row's 1/sigma(L) factors
    const float mu = A.mean[d];
    const float inv = 1.0f / A.sigma[d];
    const int Lw = A.l_end;
    const int n_in = A.n_in;

    float zmax = 0.0f;                           // PRUNE: largest |z| this lane has loaded
    auto load4 = [&](int r) -> float4 {          // z[r .. r + 3]
        float4 v;
        if (r + 3 < n_in) {
            v = load_f4(xr + r);
            v.x = (v.x - mu) * inv;
            v.y = (v.y - mu) * inv;
            v.z = (v.z - mu) * inv;
            v.w = (v.w - mu) * inv;
        } else {
            v.x = load_z(xr, r + 0, n_in, mu, inv);
            v.y = load_z(xr, r + 1, n_in, mu, inv);
            v.z = load_z(xr, r + 2, n_in, mu, inv);
            v.w = load_z(xr, r + 3, n_in, mu, inv);
        }
        return v;
    };
    auto note = [&](const float4 &v) {
        // (a maximum ignores NaN; a NaN sample shows in the running sums instead)
        if (PRUNE) zmax = fmaxf(zmax, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    };

#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = q * 256 + lane * 4;
        const float4 v = load4(base + j);
        note(v);
        ring_put(ring4, j >> 2, v);
    }
    int loaded_to = base + 1024;
    __syncthreads();

    const int nblk = (Lw + kExhBlock - 1) / kExhBlock;
    for (int g = g0; g < g_end; ++g) {
    const int s0 = g * kExhSlots;
    const int ro4 = (s0 - base) >> 2;              // ring offset (float4) of this item's window
    // the next item's window reaches 256 samples further: fetch them now, store after this item
    const bool fetch = MULTI && (g + 1 < g_end) && (s0 + kExhSlots + 768 > loaded_to);
    float4 nx = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (fetch) nx = load4(loaded_to + lane * 4);

    float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float best[4] = {SPD_NEG_INF, SPD_NEG_INF, SPD_NEG_INF, SPD_NEG_INF};
    float bx[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int bg[4] = {0, 0, 0, 0};
    int room[4];                                    // widest valid width per start
#pragma unroll
    for (int v = 0; v < 4; ++v) room[v] = n_in - (s0 + 4 * lane + v);
    // (a sigma table's scales need not fall with the width)
    const bool may_bound = PRUNE && A.scale_ld == 0;
    bool bounds = may_bound;                        // the last group raised no start's best

    for (int b = 0; b < nblk; ++b) {
        const bool refill = (b + 1 < nblk);
        float4 pf0, pf1;
        const int jn = b * kExhBlock + 1024;
        if (refill) {
            pf0 = load4(s0 + jn + lane * 4);
            pf1 = load4(s0 + jn + 256 + lane * 4);
        }
        float zm = 0.0f;                            // largest |z| of the ring, over the wave
        if (PRUNE) {
            zm = zmax;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) zm = fmaxf(zm, __shfl_xor(zm, o));
        }
        for (int gi = 0; gi < kExhBlock / kExhGroup; ++gi) {
            const int L0 = b * kExhBlock + gi * kExhGroup + 1;
            if (L0 > Lw) break;
            if (PRUNE && bounds && L0 > kExhBoundFrom && L0 + kExhGroup - 1 <= Lw &&
                (int64_t)s0 + kExhSlots - 1 + L0 + kExhGroup - 1 <= n_in) {
                float xs[4], ub[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) xs[v] = X[v];
                exh_bound(ring4, ro4 + lane + ((L0 - 1) >> 2), zm, ((ConstFloatPtr)srow)[L0 - 1],
                          ((ConstFloatPtr)srow)[L0 + kExhGroup - 2], X, ub);
                const bool may = !(ub[0] <= best[0] && ub[1] <= best[1] && ub[2] <= best[2] && ub[3] <= best[3]);
                if (!__ballot(may)) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) X[v] = xs[v];
            }
            bool raised = false;
            for (int L1 = L0; L1 < L0 + kExhGroup && L1 <= Lw; L1 += G) {
                // wave-uniform: every width of the group fits at every start of the work item
                const bool fast = (L1 + G - 1 <= Lw) && ((int64_t)s0 + kExhSlots - 1 + L1 + G - 1 <= n_in);
                float Xs[4], gm[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    Xs[v] = X[v];
                    gm[v] = SPD_NEG_INF;
                }
                const int jb4 = ro4 + lane + ((L1 - 1) >> 2);
                if (fast)
                    exh_group<false, DENSE, G>(ring4, jb4, L1, (ConstFloatPtr)srow, A.evalmask, Lw, room, X, gm);
                else
                    exh_group<true, DENSE, G>(ring4, jb4, L1, (ConstFloatPtr)srow, A.evalmask, Lw, room, X, gm);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (gm[v] > best[v]) {
                        best[v] = gm[v];
                        bg[v] = (L1 - 1) / G;
                        bx[v] = Xs[v];
                        raised = true;
                    }
                }
            }
            if (PRUNE) bounds = may_bound && !__ballot(raised);
        }
        if (refill) {
            __syncthreads();
            note(pf0);
            note(pf1);
            ring_put(ring4, ((jn >> 2) + lane) & (kRing4 - 1), pf0);
            ring_put(ring4, ((jn >> 2) + 64 + lane) & (kRing4 - 1), pf1);
            __syncthreads();
        }
    }

    // ---- recover the smallest width attaining the maximum inside the winning group.  With a
    // single block of widths the ring still holds the whole window (it was never refilled), so
    // the replay reads the same values from LDS; otherwise it loads them again.  The group's
    // samples and scales are fetched together: one at a time, their latency would cost a short
    // width set as much as its whole width loop.
    int bw[4] = {0, 0, 0, 0};
    const float *ring = reinterpret_cast<const float *>(ring4);
#pragma unroll 1
    for (int v = 0; v < 4; ++v) {                  // one start at a time: few registers
        const int Lb = bg[0] * G + 1;
        float z[G], r[G];
        if (nblk == 1) {
            const float *p = ring + (((ro4 + lane + (Lb - 1) / 4) & (kRing4 - 1)) * 4 + v);
#pragma unroll
            for (int t = 0; t < G; ++t) z[t] = p[t];
        } else {
#pragma unroll
            for (int i = 0; i < G / 4; ++i) {
                const float4 f = load4(s0 + 4 * lane + v + Lb - 1 + 4 * i);
                z[4 * i + 0] = f.x;
                z[4 * i + 1] = f.y;
                z[4 * i + 2] = f.z;
                z[4 * i + 3] = f.w;
            }
        }
#pragma unroll
        for (int i = 0; i < G / 4; ++i) {
            const float4 f = load_f4(srow + Lb - 1 + 4 * i);   // (the tables hold kExhGroup more)
            r[4 * i + 0] = f.x;
            r[4 * i + 1] = f.y;
            r[4 * i + 2] = f.z;
            r[4 * i + 3] = f.w;
        }
        const uint32_t on = DENSE ? 0xffffu : A.evalmask[(Lb - 1) >> 5] >> ((Lb - 1) & 31);
        const int fit = min(Lw, room[0] - v);
        float Xr = bx[0], bm = SPD_NEG_INF;
        int w = 0;
#pragma unroll
        for (int t = 0; t < G; ++t) {
            Xr += z[t];
            const float snr = Xr * r[t];
            const bool ok = Lb + t <= fit && (DENSE || ((on >> t) & 1u));
            if (ok && snr > bm) {
                bm = snr;
                w = Lb + t;
            }
        }
        // the next start's group and sum to the front, this one's width to the back
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            bg[q] = bg[q + 1];
            bx[q] = bx[q + 1];
            bw[q] = bw[q + 1];
        }
        bw[3] = w;
    }

    // ---- outputs
    const int m0 = s0 + 4 * lane;
    float *Yr = A.Y + (int64_t)d * A.pitch;
    uint16_t *Wr = A.W + (int64_t)d * A.pitch;
    if (m0 + 3 < A.n_out) {
        *reinterpret_cast<float4 *>(Yr + m0) = make_float4(best[0], best[1], best[2], best[3]);
        const uint32_t lo = (uint32_t)bw[0] | ((uint32_t)bw[1] << 16);
        const uint32_t hi = (uint32_t)bw[2] | ((uint32_t)bw[3] << 16);
        *reinterpret_cast<uint2 *>(Wr + m0) = make_uint2(lo, hi);
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (m0 + v < A.n_out) {
                Yr[m0 + v] = best[v];
                Wr[m0 + v] = (uint16_t)bw[v];
            }
        }
    }
    if (A.want_cand) {
        bool on = false;
#pragma unroll
        for (int v = 0; v < 4; ++v) on = on || (m0 + v < A.n_out && best[v] > A.threshold);
        const bool any = __ballot(on) != 0;
        if (lane == 0) A.above[(int64_t)d * A.n_seg + g] = any ? 1u : 0u;
        if (A.edge && g + 1 == A.n_seg && A.n_out % kExhSlots) {
            // the row's last slot against the evaluated slot after it (not in lane 63's last)
            const float right = __shfl_down(best[0], 1);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (m0 + v + 1 == A.n_out) A.edge[d] = !(best[v] >= (v < 3 ? best[v + 1] : right));
        }
    }
    if (fetch) {
        ring_put(ring4, (((loaded_to - base) >> 2) + lane) & (kRing4 - 1), nx);
        loaded_to += 256;
    }
    __syncthreads();
    }
}

// ----------------------------------------------------------------------------------------
// Peak finding (candidate selection).  A slot is a candidate iff its SNR is above the
// threshold and it passes the 3x3 neighbour test (strict against neighbours earlier in
// row-major order, non-strict against later ones; a neighbour at or below the threshold can
// never block one above it).
//
// The search left one bit per chunk of 256 slots that holds a slot above the threshold.  A
// work-group takes a run of (level, row, tile) slabs, deals the set bits out to its waves, and a
// wave tests a whole chunk at once, four slots per lane: its own values and those of the rows on
// either side (loaded only where their bits are set), time neighbours from the adjacent lanes.
// Two passes keep the output in (level, dm, start) order without a sort or a scan kernel: the
// first counts the candidates of each group of slabs, the second adds up the totals of the
// groups before its own, tests again (where there is anything to write) and writes the list.
// What bounds it is the latency of the chain word -> neighbours' words -> values, hence many
// small groups: a bright pulse sets a run of chunks, and a wave that takes a long range of slabs
// spends its time on that run alone.  Both passes together, against lists of 64 candidates a slab
// with dense rescans of the slabs that overflowed them, a scan kernel between: 500 x 95908 slots
// IG(1) 162 -> 21 us; 1024 x 131072 BD-16 269 -> 30 us; 4096 x 262144 IG(1) 253 -> 95 us;
// 512 x 131072 BD-32 candidates only (its rescans formed every slot of a tile again) 4290 -> 33 us.
//
// Values come from the planes or, candidates only, from the records the cascade left of every
// such chunk.  A chunk that found no room for its record has its slots formed again from the step's
// record (form_slots): the units of the level as pairwise sums of the step's input series, level by
// level as the cascade forms them, the BoxDIT carried prefix through the levels below, and the
// level's widths in increasing order with the same FP32 operations as step_tile, so value and width
// are bitwise those the planes would hold.
// ----------------------------------------------------------------------------------------
constexpr int kPeakThreads = 256;
constexpr int kPeakGroupWaves = kPeakThreads / 64;

// Slots m .. m + n - 1 (n <= 256) of level j of a step, row d, formed again by one wave: buf[i] receives
// the SNR and buf[256 + i] the width of slot m + i.  As many slots at a time as the row's window of
// the step's input has room for in buf (`units` floats, enough for one slot of any level): the window
// is loaded once and goes down the levels in place, as in step_tile, each lane adding the carried
// prefixes of its slots on the way.  A wave forms a chunk in the time that a lane on its own needs for a
// slot, whose units it would have to form from 2^j samples each.  Both passes of the peak finder, 256 x
// 131072 samples of noise with candidates only, where the records' room does not last, against slots
// formed by the lanes that needed them: IG(1) at a threshold of 3 1821 -> 584 us.
typedef __attribute__((address_space(4))) const RecStep *ConstRecPtr;
typedef __attribute__((address_space(3))) float *LdsFloatPtr;

__device__ __forceinline__ void wave_lds_order() {        // (a wave's LDS accesses are performed in order)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

__device__ __noinline__ void form_slots(const RecStep *rec, int d_, int j_, int m_, int n_, LdsFloatPtr buf_, int units_) {
    // (the arguments are the same in every lane)
    const int d = __builtin_amdgcn_readfirstlane(d_), j = __builtin_amdgcn_readfirstlane(j_);
    const int m = __builtin_amdgcn_readfirstlane(m_), n = __builtin_amdgcn_readfirstlane(n_);
    const int units = __builtin_amdgcn_readfirstlane(units_);
    const LdsFloatPtr buf = (LdsFloatPtr)(uintptr_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)buf_);
    const uint64_t rp = (uint64_t)rec;
    const ConstRecPtr R = (ConstRecPtr)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(rp >> 32)) << 32) |
                                        (uint32_t)__builtin_amdgcn_readfirstlane((int)rp));
    const int lane = threadIdx.x & 63;
    const float *inr = R->in + (int64_t)d * R->ld_in;
    const int64_t in_len = R->in_len;
    const bool norm = R->normalise != 0;
    float mu = 0.0f, inv = 1.0f;
    if (norm) {
        mu = R->mean[d];
        inv = 1.0f / R->sigma[d];
    }
    const auto *L = R->lv + j;
    const int umax = L->umax, k = L->k, base = L->base;
    const uint64_t emask = L->evalmask;
    const bool carry = R->carry && (j > 0 || R->cin != nullptr);
    int cs[kStepMaxLevels], uf[kStepMaxLevels], len[kStepMaxLevels];
#pragma unroll
    for (int i = 0; i < kStepMaxLevels; ++i) {
        cs[i] = i > 0 && i <= j ? R->lv[i].cshift : 0;
        uf[i] = i < j && carry ? R->lv[i].ufull : 0;
    }
    // units of level i that F slots of level j take; F: the most slots whose window fits
    int F = 2 * kChunk;
    do {
        F >>= 1;
        int l = F + umax - 1;
#pragma unroll
        for (int i = kStepMaxLevels - 1; i >= 0; --i) {
            if (i < j) l = max(2 * l + cs[i + 1 < kStepMaxLevels ? i + 1 : i], ((F - 1) << (j - i)) + uf[i]);
            len[i] = l;
        }
    } while (F > 1 && (len[0] > units || F >= 2 * n));
    // this level's scales, one a lane
    float rt = 0.0f;
    if (lane < umax) {
        rt = L->rt[lane];
        if (R->rho) {
            const double W = (double)base + ldexp((double)(lane + 1), k);
            rt = (float)((double)rt / rho_of_width(R->rho + (int64_t)d * R->ld_rho, R->n_rho, W));
        }
    }
    const int ends = (int)(((int64_t)R->n_in - base) >> k);   // U units from slot m fit: m + U <= ends
    float best[kGroup];                                       // slots 64 p + lane
    int bu[kGroup];
#pragma unroll
    for (int p = 0; p < kGroup; ++p) {
        best[p] = SPD_NEG_INF;
        bu[p] = 0;
    }
    for (int f = 0; f < n; f += F) {
        const int64_t r0 = (int64_t)(m + f) << j;             // the window's first input unit
        for (int i0 = lane; i0 - lane < len[0]; i0 += 4 * 64) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t r = r0 + i0 + 64 * q;
                v[q] = 0.0f;
                if (i0 + 64 * q < len[0] && r < in_len) v[q] = inr[r];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)                       // (zero past the data)
                if (i0 + 64 * q < len[0])
                    buf[i0 + 64 * q] = norm && r0 + i0 + 64 * q < in_len ? (v[q] - mu) * inv : v[q];
        }
        float X[kGroup];
        int at[kGroup];                                       // the lane's slots in the window (0: none)
        bool on[kGroup];
#pragma unroll
        for (int p = 0; p < kGroup; ++p) {
            const int i = 64 * p + lane - f;
            on[p] = i >= 0 && i < F && f + i < n;
            at[p] = on[p] ? i : 0;
            X[p] = 0.0f;
            const int64_t c = (int64_t)(m + f + at[p]) << j;
            if (carry && R->cin && on[p] && c < R->lv[0].slots) X[p] = R->cin[(int64_t)d * R->ld_cin + c];
        }
        wave_lds_order();
#pragma unroll
        for (int i = 0; i + 1 < kStepMaxLevels; ++i) {
            if (i >= j) continue;
            for (int u = 0; u < uf[i]; ++u)
#pragma unroll
                for (int p = 0; p < kGroup; ++p) X[p] += buf[(at[p] << (j - i)) + u];
            wave_lds_order();
            for (int x = lane; x - lane < len[i + 1]; x += 64) {
                float v = 0.0f;
                if (x < len[i + 1]) v = buf[2 * x + cs[i + 1]] + buf[2 * x + cs[i + 1] + 1];
                wave_lds_order();
                if (x < len[i + 1]) buf[x] = v;
                wave_lds_order();
            }
        }
        for (int u = 0; u < umax; ++u) {
#pragma unroll
            for (int p = 0; p < kGroup; ++p) X[p] += buf[at[p] + u];
            if ((emask >> u) & 1ull) {
                const float r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(rt), u));
#pragma unroll
                for (int p = 0; p < kGroup; ++p) {
                    const float v = X[p] * r;
                    const bool gt = on[p] && m + f + at[p] + u + 1 <= ends && v > best[p];
                    best[p] = gt ? v : best[p];
                    bu[p] = gt ? u + 1 : bu[p];
                }
            }
        }
        wave_lds_order();
    }
#pragma unroll
    for (int p = 0; p < kGroup; ++p) {
        buf[64 * p + lane] = best[p];
        buf[kChunk + 64 * p + lane] = __int_as_float(bu[p] ? base + (bu[p] << k) : 0);
    }
    wave_lds_order();
}

// The helpers take the arguments, of the launch (one beam) or of a beam in a batch's table, in the
// constant address space.
typedef __attribute__((address_space(4))) const PeakArgs CPeakArgs;

// the chunk bits of tile t of level k in row d
__device__ __forceinline__ uint32_t slab_word(CPeakArgs &A, int k, int d, int t) {
    return A.above[A.cnt_off[k] + ((int64_t)d * A.tiles_per_row[k] + t) * A.cnt_stride[k]];
}

// where the record of chunk c of tile t of level k in row d is (or kNoRecord, kEmptyChunk)
__device__ __forceinline__ uint32_t chunk_record(CPeakArgs &A, int k, int d, int t, int c) {
    return A.dir[A.dir_off[k] + ((int64_t)d * A.tiles_per_row[k] + t) * A.cpt[k] + c];
}

// SNRs (and widths, if w is not null) of slots m0 .. m0 + 3 of level k in row d, slots m0 + 4 lane
// of chunk c of tile t whose bit is set; slots past m_end are -inf.  From records, so are the
// slots at or below the threshold; true if the chunk has no record (nothing is set then).
template <bool REC>
__device__ __forceinline__ bool chunk_values(CPeakArgs &A, int k, int d, int t, int c, int lane, int m0,
                                             int m_end, float y[kGroup], int *w) {
#pragma unroll
    for (int q = 0; q < kGroup; ++q) y[q] = SPD_NEG_INF;
    if constexpr (!REC) {
        const int64_t i = A.level_off[k] + (int64_t)d * A.level_pitch[k] + m0;
        if (m0 + kGroup <= m_end) {
            const float4 v = *reinterpret_cast<const float4 *>(A.Y + i);
            y[0] = v.x;
            y[1] = v.y;
            y[2] = v.z;
            y[3] = v.w;
        } else {
#pragma unroll
            for (int q = 0; q < kGroup; ++q)
                if (m0 + q < m_end) y[q] = A.Y[i + q];
        }
        (void)w;                                   // (the scatter pass reads the widths it needs)
    } else {
        const uint32_t off = (uint32_t)__builtin_amdgcn_readfirstlane((int)chunk_record(A, k, d, t, c));
        if (off == kEmptyChunk) return false;
        if (off == kNoRecord) return true;
        const uint64_t *r = A.pool + off;
        const int word = lane >> 4, bit = (lane & 15) * kGroup;
        int pos = 0;
        uint64_t own = 0;
#pragma unroll
        for (int i = 0; i < kChunk / 64; ++i) {
            const uint64_t b = r[i];
            if (i < word) pos += __popcll(b);
            if (i == word) own = b;
        }
        pos += __popcll(own & ((1ull << bit) - 1));
        const uint2 *ent = reinterpret_cast<const uint2 *>(r + kChunk / 64);
        const uint32_t nib = (uint32_t)(own >> bit) & 15u;
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            if ((nib >> q) & 1u) {
                const uint2 e = ent[pos++];
                y[q] = __uint_as_float(e.x);
                if (w) w[q] = (int)e.y;
            }
        }
    }
    return false;
}

// SNR of slot m of level k in row d, -inf if its chunk's bit is clear (one lane on its own: the
// slots beside a chunk); missing: its chunk has no record
template <bool REC>
__device__ __forceinline__ float slot_value(CPeakArgs &A, int k, int d, int m, bool &missing) {
    const int ts = A.tile_slots[k];
    const int t = m / ts;
    const int i = m - t * ts;
    const int c = i / kChunk;
    if (!((slab_word(A, k, d, t) >> (c >> A.bit_shift[k])) & 1u)) return SPD_NEG_INF;
    if constexpr (!REC) {
        return A.Y[A.level_off[k] + (int64_t)d * A.level_pitch[k] + m];
    } else {
        const uint32_t off = chunk_record(A, k, d, t, c);
        if (off == kEmptyChunk) return SPD_NEG_INF;
        if (off == kNoRecord) {
            missing = true;
            return SPD_NEG_INF;
        }
        const uint64_t *r = A.pool + off;
        const int b = i - c * kChunk;
        int pos = 0;
        uint64_t own = 0;
#pragma unroll
        for (int q = 0; q < kChunk / 64; ++q) {
            const uint64_t v = r[q];
            if (q < (b >> 6)) pos += __popcll(v);
            if (q == (b >> 6)) own = v;
        }
        if (!((own >> (b & 63)) & 1ull)) return SPD_NEG_INF;
        pos += __popcll(own & ((1ull << (b & 63)) - 1));
        return __uint_as_float(reinterpret_cast<const uint2 *>(r + kChunk / 64)[pos].x);
    }
}

// form_slots for slots of level k
__device__ __forceinline__ void form_chunk(CPeakArgs &A, int k, int d, int m, int n, LdsFloatPtr form) {
    form_slots(A.rec + A.level_step[k], d, A.level_j[k], m, n, form, A.form_units);
}

// tile gating of the candidates (flag_mode): may slot m of level k in row d be a candidate?
__device__ __forceinline__ bool slot_kept(CPeakArgs &A, int k, int d, int m) {
    if (A.flag_mode == 0) return true;
    const int64_t s = (int64_t)m << A.level_shift[k];
    const bool f = A.tile_flag[(int64_t)(d / A.tile_rows) * A.n_col_tiles + s / A.tile_len] != 0;
    return A.flag_mode == 2 ? f : !f;
}

// Local maxima in time above the threshold in tile t of level k in row d, but for the row's last slot: a
// chunk on its own, with nothing on either side of it (see PeakArgs::edge).
template <bool REC, bool FORM>
__device__ __forceinline__ int tile_maxima(CPeakArgs &A, int k, int d, int t, int lane, LdsFloatPtr form,
                                           bool &missing) {
    const int slots = A.level_slots[k], ts = A.tile_slots[k], sh = A.bit_shift[k];
    const int m_end = min((t + 1) * ts, slots);
    const uint32_t word = slab_word(A, k, d, t);
    int n = 0;
    for (int c = 0; c < A.cpt[k] && n <= A.edge_maxima; ++c) {
        if (!((word >> (c >> sh)) & 1u)) continue;
        const int mc = t * ts + c * kChunk, m0 = mc + kGroup * lane;
        float y[kGroup];
        if (chunk_values<REC>(A, k, d, t, c, lane, m0, m_end, y, nullptr)) {
            if constexpr (FORM) {
                form_chunk(A, k, d, mc, min(kChunk, m_end - mc), form);
#pragma unroll
                for (int q = 0; q < kGroup; ++q) y[q] = form[kGroup * lane + q];
                wave_lds_order();
            } else {
                missing = true;
                return 0;
            }
        }
        const float left = __shfl_up(y[kGroup - 1], 1), right = __shfl_down(y[0], 1);
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            const float l = q > 0 ? y[q - 1] : lane ? left : SPD_NEG_INF;
            const float r = q + 1 < kGroup ? y[q + 1] : lane < 63 ? right : SPD_NEG_INF;
            n += __popcll(__ballot(y[q] > A.threshold && y[q] > l && y[q] >= r && m0 + q + 1 != slots));
        }
    }
    return n;
}

// The candidates of chunk c of tile t of level k in row d, whose bit is set: bit q of the result
// for slot m0 + q of this lane.  y receives the slots' SNRs and, from records, w their widths.  Chunks
// without a record, here or beside, are formed again (FORM) or end the test with `missing` set.
template <bool REC, bool FORM>
__device__ __forceinline__ uint32_t chunk_test(CPeakArgs &A, int k, int d, int t, int c, int lane, int &m0,
                                               float y[kGroup], int w[kGroup], LdsFloatPtr form, bool &missing) {
    const int ts = A.tile_slots[k];
    const int slots = A.level_slots[k];
    const int m_end = min((t + 1) * ts, slots);
    const int mc = t * ts + c * kChunk;                   // the chunk's first slot
    m0 = mc + kGroup * lane;
    const int bit = c >> A.bit_shift[k];
    const bool up = d > 0 && ((slab_word(A, k, d - 1, t) >> bit) & 1u);
    const bool down = d + 1 < A.n_dm && ((slab_word(A, k, d + 1, t) >> bit) & 1u);
    int rows = chunk_values<REC>(A, k, d, t, c, lane, m0, m_end, y, w) ? 1 : 0;   // of d, d - 1, d + 1 without a record
    float yn[2][kGroup];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int q = 0; q < kGroup; ++q) yn[a][q] = SPD_NEG_INF;
    if (up && chunk_values<REC>(A, k, d - 1, t, c, lane, m0, m_end, yn[0], nullptr)) rows |= 2;
    if (down && chunk_values<REC>(A, k, d + 1, t, c, lane, m0, m_end, yn[1], nullptr)) rows |= 4;
    if constexpr (REC && !FORM) {
        if (rows) {
            missing = true;
            return 0;
        }
    }
    if constexpr (FORM) {
#pragma unroll 1
        for (int a = 0; a < 3; ++a) {
            if (!((rows >> a) & 1)) continue;
            form_chunk(A, k, a == 0 ? d : a == 1 ? d - 1 : d + 1, mc, min(kChunk, m_end - mc), form);
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {                // (-inf past m_end)
                const float v = form[kGroup * lane + q];
                y[q] = a == 0 ? v : y[q];
                yn[0][q] = a == 1 ? v : yn[0][q];
                yn[1][q] = a == 2 ? v : yn[1][q];
                if (a == 0) w[q] = __float_as_int(form[kChunk + kGroup * lane + q]);
            }
            wave_lds_order();
        }
    }

    // time neighbours outside this lane's four slots: the adjacent lanes', or the adjacent
    // chunks' at either end (looked up only where the slot there passes the test without them)
    float l[3], r[3];
    l[0] = __shfl_up(yn[0][kGroup - 1], 1);
    l[1] = __shfl_up(y[kGroup - 1], 1);
    l[2] = __shfl_up(yn[1][kGroup - 1], 1);
    r[0] = __shfl_down(yn[0][0], 1);
    r[1] = __shfl_down(y[0], 1);
    r[2] = __shfl_down(yn[1][0], 1);
    const int last = min(mc + kChunk, (t + 1) * ts) - kGroup;   // first slot of the chunk's last lane
    if (lane == 0) l[0] = l[1] = l[2] = SPD_NEG_INF;
    if (m0 == last) r[0] = r[1] = r[2] = SPD_NEG_INF;
    uint32_t hit = 0;
#pragma unroll
    for (int q = 0; q < kGroup; ++q) {
        const float v = y[q];
        const float ul = q > 0 ? yn[0][q - 1] : l[0], ur = q + 1 < kGroup ? yn[0][q + 1] : r[0];
        const float sl = q > 0 ? y[q - 1] : l[1], sr = q + 1 < kGroup ? y[q + 1] : r[1];
        const float dl = q > 0 ? yn[1][q - 1] : l[2], dr = q + 1 < kGroup ? yn[1][q + 1] : r[2];
        const bool ok = v > A.threshold && v > ul && v > yn[0][q] && v > ur && v > sl && v >= sr &&
                        v >= dl && v >= yn[1][q] && v >= dr;
        if (ok && slot_kept(A, k, d, m0 + q)) hit |= 1u << q;
    }
    const bool at_left = __ballot(lane == 0 && (hit & 1u)) != 0 && mc > 0;
    const bool at_right = __ballot(m0 == last && (hit >> (kGroup - 1))) != 0 && last + kGroup < slots;
    if (at_left || at_right) {
        // lanes 0 .. 2 look up the left ones in rows d - 1 .. d + 1, lanes 3 .. 5 the right ones
        const int dn = d + (lane < 3 ? lane : lane - 3) - 1;
        const int mn = lane < 3 ? mc - 1 : last + kGroup;
        float v = SPD_NEG_INF;
        bool none = false;
        if (lane < 6 && (lane < 3 ? at_left : at_right) && dn >= 0 && dn < A.n_dm) v = slot_value<REC>(A, k, dn, mn, none);
        if constexpr (REC && !FORM) {
            if (__ballot(none)) {
                missing = true;
                return 0;
            }
        }
        if constexpr (FORM) {
#pragma unroll 1
            for (uint64_t b = __ballot(none); b; b &= b - 1) {
                const int i = __ffsll((unsigned long long)b) - 1;
                form_chunk(A, k, d + (i < 3 ? i : i - 3) - 1, i < 3 ? mc - 1 : last + kGroup, 1, form);
                if (lane == i) v = form[0];
                wave_lds_order();
            }
        }
        const float ul = __shfl(v, 0), sl = __shfl(v, 1), dl = __shfl(v, 2);
        const float ur = __shfl(v, 3), sr = __shfl(v, 4), dr = __shfl(v, 5);
        if (lane == 0 && !(y[0] > ul && y[0] > sl && y[0] >= dl)) hit &= ~1u;
        if (m0 == last && !(y[kGroup - 1] > ur && y[kGroup - 1] >= sr && y[kGroup - 1] >= dr)) hit &= ~(1u << (kGroup - 1));
    }
    if (A.edge_on[k]) {
        const int q = slots - 1 - m0;                     // the row's last slot in this lane
        const bool ends = q >= 0 && q < kGroup && ((hit >> q) & 1u) && A.edge[(int64_t)k * A.n_dm + d];
        if (__ballot(ends)) {
            const bool many = tile_maxima<REC, FORM>(A, k, d, t, lane, form, missing) > A.edge_maxima;
            if (ends && !many) hit &= ~(1u << q);
        }
    }
    return hit;
}

// level of slab s
__device__ __forceinline__ int slab_level(CPeakArgs &A, int64_t s) {
    int k = 0;
    while (k + 1 < A.n_levels && s >= A.slab_base[k + 1]) ++k;
    return k;
}

// The slabs [sbeg, send) of a group.  SCATTER false: `total` receives this wave's candidates; true: they
// are written from entry `run` on.  Without FORM the count ends, returning true, at the first chunk
// whose record is needed and missing.
template <bool REC, bool SCATTER, bool FORM>
__device__ __forceinline__ bool peak_items(CPeakArgs &A, int64_t sbeg, int64_t send, int64_t run, uint32_t &total,
                                           uint32_t (*cnt)[kPeakGroupWaves], LdsFloatPtr form) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    total = 0;
    int turn = 0;
    for (int64_t sb = sbeg; sb < send; sb += 64) {
        const int64_t s = sb + lane;
        uint32_t word = 0;
        int shift = 0;
        if (s < send) {
            const int k = slab_level(A, s);
            word = A.above[A.cnt_off[k] + (s - A.slab_base[k]) * A.cnt_stride[k]];
            shift = A.bit_shift[k];
        }
        if (!__ballot(word != 0)) continue;
        // the chunks of the 64 slabs in order: inclusive prefix of their numbers over the lanes
        int incl = __popc(word) << shift;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        const int items = __builtin_amdgcn_readlane(incl, 63);
        for (int i0 = 0; i0 < items; i0 += kPeakGroupWaves) {
            const int it = i0 + wave;
            uint32_t hit = 0;
            int k = 0, d = 0, m0 = 0;
            float y[kGroup];
            int w[kGroup];
            if (it < items) {
                const int l = __ffsll((unsigned long long)__ballot(incl > it)) - 1;
                uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)word, l);
                k = slab_level(A, sb + l);
                const int sh = A.bit_shift[k];
                const int r = it - (__builtin_amdgcn_readlane(incl, l) - (__popc(bits) << sh));
                for (int i = r >> sh; i > 0; --i) bits &= bits - 1;
                const int c = ((__ffs((int)bits) - 1) << sh) + (r & ((1 << sh) - 1));
                const uint32_t rs = (uint32_t)(sb + l - A.slab_base[k]);   // (rows x tiles fits 31 bits)
                d = (int)(rs / (uint32_t)A.tiles_per_row[k]);
                const int t = (int)(rs - (uint32_t)d * (uint32_t)A.tiles_per_row[k]);
                bool missing = false;
                if (c < A.cpt[k]) hit = chunk_test<REC, FORM>(A, k, d, t, c, lane, m0, y, w, form, missing);
                if (!SCATTER && missing) return true;
            }
            uint32_t n = 0;
            int pos = 0;
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const uint64_t b = __ballot((hit >> q) & 1u);
                n += (uint32_t)__popcll(b);
                if (SCATTER) pos += __popcll(b & lanes_below(lane));
            }
            if constexpr (!SCATTER) {
                total += n;
            } else {
                if (lane == 0) cnt[turn][wave] = n;
                __syncthreads();
                int64_t at = run + pos;
#pragma unroll
                for (int i = 0; i < kPeakGroupWaves; ++i) {
                    if (i < wave) at += cnt[turn][i];
                    run += cnt[turn][i];
                }
                turn ^= 1;
#pragma unroll
                for (int q = 0; q < kGroup; ++q) {
                    if (!((hit >> q) & 1u)) continue;
                    if (at < A.cand_cap) {
                        spd_candidate o;
                        o.start = A.t0 + ((int64_t)(m0 + q) << A.level_shift[k]);
                        o.dm = d;
                        o.width = REC ? w[q] : A.W[A.level_off[k] + (int64_t)d * A.level_pitch[k] + m0 + q];
                        o.level = k;
                        o.snr = y[q];
                        A.cand[at] = o;
                    }
                    ++at;
                }
            }
        }
    }
    return false;
}

// One group of slabs of a pass.  SCATTER false: count its candidates; true: write them.  A group that
// needs a record that is missing (kGroupForms in its total) runs again in a loop of its own, so that the
// registers for forming slots again are not taken from the usual one.
constexpr uint32_t kGroupForms = 1u << 31;
template <bool REC, bool SCATTER>
__device__ __forceinline__ void peak_group(CPeakArgs &A, int g) {
    __shared__ int64_t part[kPeakGroupWaves];
    __shared__ uint32_t cnt[2][kPeakGroupWaves];
    extern __shared__ float form_lds[];  // REC: each wave's window of form_slots
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t sbeg = (int64_t)g * A.slabs_per_group;
    const int64_t send = min(sbeg + A.slabs_per_group, A.n_slabs);
    int64_t run = 0;                     // SCATTER: where the next candidate goes
    uint32_t total = 0;                  // SCATTER false: this wave's candidates
    bool again = false;                  // (the same in the whole work-group)
    if constexpr (SCATTER) {
        const uint32_t mine = A.group_tot[g];
        const bool last = g + 1 == A.n_groups;
        if ((mine & ~kGroupForms) == 0 && !last) return;
        int64_t sum = 0;
        for (int i = threadIdx.x; i < g; i += kPeakThreads) sum += A.group_tot[i] & ~kGroupForms;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) part[wave] = sum;
        __syncthreads();
        run = *A.base_copy;
#pragma unroll
        for (int i = 0; i < kPeakGroupWaves; ++i) run += part[i];
        if (last && threadIdx.x == 0) *A.cand_count = run + (mine & ~kGroupForms);
        if ((mine & ~kGroupForms) == 0) return;
        again = REC && (mine & kGroupForms) != 0;
        if (!again) peak_items<REC, true, false>(A, sbeg, send, run, total, cnt, nullptr);
    } else {
        // candidates already in the list (the scatter pass may overwrite the same count)
        if (g == 0 && threadIdx.x == 0) *A.base_copy = A.base_count ? *A.base_count : 0;
        const bool missing = peak_items<REC, false, false>(A, sbeg, send, 0, total, cnt, nullptr);
        if constexpr (REC) again = __syncthreads_or(missing) != 0;
    }
    if constexpr (REC) {
        if (again) {
            // (behind a pointer that hides where the arguments come from: see above)
            CPeakArgs *P = &A;
            asm volatile("" : "+s"(P));
            const LdsFloatPtr form = (LdsFloatPtr)form_lds + wave * P->form_units;
            peak_items<true, SCATTER, true>(*P, sbeg, send, run, total, cnt, form);
        }
    }
    if constexpr (!SCATTER) {
        if (lane == 0) cnt[0][wave] = total;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t sum = again ? kGroupForms : 0u;
#pragma unroll
            for (int i = 0; i < kPeakGroupWaves; ++i) sum += cnt[0][i];
            A.group_tot[g] = sum;
        }
    }
}

template <bool REC, bool SCATTER>
__global__ __launch_bounds__(kPeakThreads) void peak_kernel(const PeakArgs A) {
    (void)A;                             // (read from the kernel arguments' address)
    peak_group<REC, SCATTER>(*(CPeakArgs *)__builtin_amdgcn_kernarg_segment_ptr(), blockIdx.x);
}

// Batched: the peak-finder arguments of every beam in a table in the constant address space
// (read with scalar loads), the groups of all beams in one index space: group i belongs to beam b
// with group_base[b] <= i < group_base[b + 1].  One launch per pass for the whole batch.
template <bool REC, bool SCATTER>
__global__ __launch_bounds__(kPeakThreads) void peak_batch_kernel(const PeakBatchArgs B) {
    const ConstI64Ptr base = (ConstI64Ptr)B.group_base;
    int lo = 0, hi = B.n_beams - 1;                     // last b with base[b] <= this group
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (base[mid] <= (int64_t)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    CPeakArgs &A = ((CPeakArgs *)B.tab)[lo];
    peak_group<REC, SCATTER>(A, (int)((int64_t)blockIdx.x - base[lo]));
}

// ----------------------------------------------------------------------------------------
// Launchers
// ----------------------------------------------------------------------------------------
int launch_scales(const ScaleArgs &a, void *stream) {
    if (a.n <= 0) return 0;
    const unsigned rows = a.rho ? (unsigned)a.n_rows : 1u;
    hipLaunchKernelGGL(scales_kernel, dim3((a.n + 255) / 256, rows), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_evalmask(const MaskArgs &a, void *stream) {
    hipLaunchKernelGGL(evalmask_kernel, dim3((a.n_words + 255) / 256), dim3(256), 0,
                       (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// IG(1) tiles of at most kSmallTileMax units run on work-groups of kSmallStepThreads (the
// planner sets StepArgs::nth): its light width sets leave the launch bound by the plane writes,
// which go faster from more, smaller work-groups (3.77 ms against 3.91 ms at the best tile of
// either size on the 4096 x 262144 beam; the denser sets are faster on 256 threads).  Results do
// not depend on the work-group size.
template <bool FIRST, int FAM, int NTH>
static void launch_nth(const StepArgs &a, int lds_bytes, hipStream_t st) {
    const dim3 grid((unsigned)((int64_t)a.n_dm * a.n_tiles));
    if (a.rho && a.write_planes)
        hipLaunchKernelGGL((step_kernel<FIRST, FAM, true, NTH, true>), grid, dim3(NTH), lds_bytes, st, a);
    else if (a.rho)
        hipLaunchKernelGGL((step_kernel<FIRST, FAM, true, NTH, false>), grid, dim3(NTH), lds_bytes, st, a);
    else if (a.write_planes)
        hipLaunchKernelGGL((step_kernel<FIRST, FAM, false, NTH, true>), grid, dim3(NTH), lds_bytes, st, a);
    else
        hipLaunchKernelGGL((step_kernel<FIRST, FAM, false, NTH, false>), grid, dim3(NTH), lds_bytes, st, a);
}

// The work-group size is the planner's (StepArgs::nth): 128 threads only for IG(1).
template <bool FIRST, int FAM>
static int launch_one(const StepArgs &a, int lds_bytes, hipStream_t st) {
    if (a.nth == kSmallStepThreads) {
        if (FAM != 1) return (int)hipErrorInvalidValue;
        launch_nth<FIRST, 1, kSmallStepThreads>(a, lds_bytes, st);
    } else if (a.nth == kStepThreads) {
        launch_nth<FIRST, FAM, kStepThreads>(a, lds_bytes, st);
    } else {
        return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

template <bool FIRST>
static int launch_step_fam(const StepArgs &a, int fam, int lds_bytes, hipStream_t st) {
    switch (fam) {
        case 1: return launch_one<FIRST, 1>(a, lds_bytes, st);
        case 2: return launch_one<FIRST, 2>(a, lds_bytes, st);
        case 3: return launch_one<FIRST, 3>(a, lds_bytes, st);
        case 4: return launch_one<FIRST, 4>(a, lds_bytes, st);
        case 5: return launch_one<FIRST, 5>(a, lds_bytes, st);
        case 6: return launch_one<FIRST, 6>(a, lds_bytes, st);
        case 7: return launch_one<FIRST, 7>(a, lds_bytes, st);
        default: return launch_one<FIRST, 0>(a, lds_bytes, st);
    }
}

template <bool FIRST, int FAM>
static int launch_batch(const StepBatchArgs &a, int lds_bytes, int grid, hipStream_t st) {
    if (a.s.write_planes)
        hipLaunchKernelGGL((step_kernel_batch<FIRST, FAM, true>), dim3((unsigned)grid),
                           dim3(kStepThreads), lds_bytes, st, a);
    else
        hipLaunchKernelGGL((step_kernel_batch<FIRST, FAM, false>), dim3((unsigned)grid),
                           dim3(kStepThreads), lds_bytes, st, a);
    return (int)hipGetLastError();
}

template <bool FIRST>
static int launch_batch_fam(const StepBatchArgs &a, int fam, int lds_bytes, int grid, hipStream_t st) {
    switch (fam) {
        case 1: return launch_batch<FIRST, 1>(a, lds_bytes, grid, st);
        case 2: return launch_batch<FIRST, 2>(a, lds_bytes, grid, st);
        case 3: return launch_batch<FIRST, 3>(a, lds_bytes, grid, st);
        case 4: return launch_batch<FIRST, 4>(a, lds_bytes, grid, st);
        case 5: return launch_batch<FIRST, 5>(a, lds_bytes, grid, st);
        case 6: return launch_batch<FIRST, 6>(a, lds_bytes, grid, st);
        case 7: return launch_batch<FIRST, 7>(a, lds_bytes, grid, st);
        default: return launch_batch<FIRST, 0>(a, lds_bytes, grid, st);
    }
}

int launch_step_batch(const StepBatchArgs &a, int fam, int lds_bytes, int grid, void *stream) {
    if (a.s.normalise) return launch_batch_fam<true>(a, fam, lds_bytes, grid, (hipStream_t)stream);
    return launch_batch_fam<false>(a, fam, lds_bytes, grid, (hipStream_t)stream);
}

int launch_step(const StepArgs &a, int fam, int lds_bytes, void *stream) {
    // the first step (raw samples, normalised on load) and the later steps (decimated series)
    // are separate instantiations, so profiles tell them apart
    if (a.normalise) return launch_step_fam<true>(a, fam, lds_bytes, (hipStream_t)stream);
    return launch_step_fam<false>(a, fam, lds_bytes, (hipStream_t)stream);
}

uint64_t family_mask(int fam, int pattern) {
    switch (fam) {
        case 1: return pattern == 1 ? Fam<1>::M1 : Fam<1>::M2;
        case 2: return pattern == 1 ? Fam<2>::M1 : Fam<2>::M2;
        case 3: return pattern == 1 ? Fam<3>::M1 : Fam<3>::M2;
        case 4: return Fam<4>::M1;
        case 5: return Fam<5>::M1;
        case 6: return Fam<6>::M1;
        case 7: return Fam<7>::M1;
        default: return 0;
    }
}

int launch_exhaustive(const ExhArgs &a, bool dense, void *stream) {
    const int64_t per_row = (a.n_seg + a.segs_per_wave - 1) / a.segs_per_wave;
    const dim3 grid((unsigned)((int64_t)a.n_dm * per_row));
    const bool multi = a.segs_per_wave > 1;
    // bounds pay once a width set goes past one ring window (shorter ones raise a best in most groups)
    const bool prune = dense && a.l_end > kExhBlock;
    hipStream_t st = (hipStream_t)stream;
    if (multi) {
        if (dense)
            hipLaunchKernelGGL((exh_kernel<true, true, false>), grid, dim3(64), 0, st, a);
        else
            hipLaunchKernelGGL((exh_kernel<false, true, false>), grid, dim3(64), 0, st, a);
    } else if (prune) {
        hipLaunchKernelGGL((exh_kernel<true, false, true>), grid, dim3(64), 0, st, a);
    } else {
        if (dense)
            hipLaunchKernelGGL((exh_kernel<true, false, false>), grid, dim3(64), 0, st, a);
        else
            hipLaunchKernelGGL((exh_kernel<false, false, false>), grid, dim3(64), 0, st, a);
    }
    return (int)hipGetLastError();
}

__global__ void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

int launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, void *stream) {
    if (n <= 0) return 0;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       p, n, v);
    return (int)hipGetLastError();
}

template <bool SCATTER>
static int launch_peak_pass(const PeakArgs &a, hipStream_t st) {
    const dim3 grid((unsigned)a.n_groups);
    if (a.dir)
        hipLaunchKernelGGL((peak_kernel<true, SCATTER>), grid, dim3(kPeakThreads),
                           kPeakGroupWaves * a.form_units * 4, st, a);
    else
        hipLaunchKernelGGL((peak_kernel<false, SCATTER>), grid, dim3(kPeakThreads), 0, st, a);
    return (int)hipGetLastError();
}

int launch_peaks(const PeakArgs &a, void *stream) {
    const int err = launch_peak_pass<false>(a, (hipStream_t)stream);
    return err ? err : launch_peak_pass<true>(a, (hipStream_t)stream);
}

template <bool SCATTER>
static int launch_peak_batch_pass(const PeakBatchArgs &a, hipStream_t st) {
    const dim3 grid((unsigned)a.n_groups);
    if (a.records)
        hipLaunchKernelGGL((peak_batch_kernel<true, SCATTER>), grid, dim3(kPeakThreads),
                           kPeakGroupWaves * a.form_units * 4, st, a);
    else
        hipLaunchKernelGGL((peak_batch_kernel<false, SCATTER>), grid, dim3(kPeakThreads), 0, st, a);
    return (int)hipGetLastError();
}

int launch_peaks_batch(const PeakBatchArgs &a, void *stream) {
    if (a.n_groups <= 0) return 0;
    const int err = launch_peak_batch_pass<false>(a, (hipStream_t)stream);
    return err ? err : launch_peak_batch_pass<true>(a, (hipStream_t)stream);
}

const char *hip_error_text(int err) { return hipGetErrorString((hipError_t)err); }

}  // namespace spd
