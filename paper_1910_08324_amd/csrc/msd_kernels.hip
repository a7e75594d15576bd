// Noise statistics per DM trial (declared in include/spd_msd.h): robust mean and standard
// deviation with iterative outlier rejection, for the samples and for every power-of-two
// decimation of them.  One work-group per row, FP64 throughout.
//
// A read of the row serves every level at once.  The row streams through in tiles of 1024
// samples, one float4 per thread; inside a tile the decimated values of levels 1..8 are formed
// in registers (levels 1, 2 within a thread, 3..8 by a butterfly across lanes, DPP and row swaps).  Levels 0..5 are accumulated as they stream
// by: per level, each thread keeps a count and the sums of (value - shift) and of its square,
// the shift being the level's current mean estimate; levels 0..2, which every lane serves, count
// their kept values per wave and total their lanes' sums directly, levels 3..5 merge per-lane
// partials (count, mean, sum of squared deviations) with Chan, Golub & LeVeque's formula in a
// fixed order.  Levels 6 and up (at most 1/32 of the values) are stored whole in the workspace by
// the first read and taken from there in every pass.  Levels converge independently; the row's
// passes stop when every level has.
//
// Most passes need not read the row.  Before the first read a pre-estimate (mean and sd of 8
// tiles spread over the row) centres a band for each level 0..5; the first read (the estimate
// that keeps every value) lists, per level and wave, every value outside the band and keeps the
// count and sums of the values it did not list.  While the limit of a later pass still covers
// the whole band (|value - list centre| <= band half-width implies |value - mean| <= limit,
// checked with a margin for rounding), every unlisted value is kept, so the pass needs only the
// listed values: it tests them exactly as a full read would and adds the unlisted statistics;
// such a pass runs its levels side by side, one wave per level.  The kept sets, hence the counts,
// pass counts and stopping decisions, are those of full reads; only the order of the FP64 sums
// differs (and is fixed).  When the band is no longer covered, or a list overflowed its room, the
// pass reads the row again and lists anew around its own estimate (0.8 of its limit).
//
// What bounds it is the issue of the first read's FP64 and list instructions, then the reductions
// and list passes of a row, one after another.  One loop per kind of read (one loop for all moved
// 250 scalar registers per tile at its joins), the first without the tests that always hold, two
// tiles' loads in flight, no barrier in a tile (levels 9.. are formed after the read), no pass
// through LDS for the levels, and the listed values gathered there: 4096 x 262144 samples,
// 14 levels, 3.49 -> 1.89 ms (2.3 TB/s of samples), the results bit for bit the same.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "spd.h"
#include "spd_msd.h"

namespace spdm {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kTile = 4 * kThreads;   // samples per tile
constexpr int kRegLevels = 9;          // levels 0..8 formed in registers
constexpr int kListLevels = 6;         // levels 0..5 are summed as the row streams by
constexpr int kArrFirst = 6;           // levels 6.. are stored whole by the first pass
constexpr double kListFrac = 0.8;      // a rebuild lists values beyond 0.8 of the limit
constexpr int kProbeTiles = 8;         // tiles of the pre-estimate, spread over the row

// Per row, the workspace holds the values of levels 6.. (level 6 first, then 7, ...; fewer than
// n / 32 in all), then for each level k < 6 one list per wave with room for 1/16 of the wave's
// values of the level, plus 16.
__host__ __device__ inline int64_t arr_offset(int n, int k) {   // of level k >= 6
    int64_t o = 0;
    for (int i = kArrFirst; i < k; ++i) o += (int64_t)(n >> i);
    return o;
}
__host__ __device__ constexpr int list_room(int n, int k) { return ((n >> k) >> 6) + 16; }
__host__ __device__ inline int64_t list_offset(int n, int k) {   // of level k's first list
    int64_t o = (int64_t)(n >> 5) + 8;
    for (int i = 0; i < k; ++i) o += (int64_t)kWaves * list_room(n, i);
    return o;
}
__host__ __device__ inline int64_t ws_row_doubles(int n) { return list_offset(n, kListLevels); }

struct Part {
    double n, mean, m2;
};

__device__ __forceinline__ Part merge(Part a, Part b) {
    if (a.n == 0.0) return b;
    if (b.n == 0.0) return a;
    const double n = a.n + b.n;
    const double d = b.mean - a.mean;
    Part r;
    r.n = n;
    r.mean = a.mean + d * (b.n / n);
    r.m2 = a.m2 + b.m2 + d * d * (a.n * b.n / n);
    return r;
}

// merge the 256 threads' partials: butterflies inside each wave, then the four waves in order
__device__ Part block_merge(Part p, Part *sh) {
    for (int o = 1; o < 64; o <<= 1) {
        Part q;
        q.n = __shfl_xor(p.n, o);
        q.mean = __shfl_xor(p.mean, o);
        q.m2 = __shfl_xor(p.m2, o);
        // both lanes of a pair combine (lower, upper) in the same order, so they agree
        const bool upper = (threadIdx.x & o) != 0;
        p = upper ? merge(q, p) : merge(p, q);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = p;
    __syncthreads();
    return merge(merge(sh[0], sh[1]), merge(sh[2], sh[3]));
}

// totals over the work-group of per-thread (count, sum, sum of squares) in a fixed order:
// butterflies inside each wave (a + b == b + a, so the lanes agree), then the four waves in order
__device__ Part block_sums(Part p, Part *sh) {
    for (int o = 1; o < 64; o <<= 1) {
        p.n += __shfl_xor(p.n, o);
        p.mean += __shfl_xor(p.mean, o);
        p.m2 += __shfl_xor(p.m2, o);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = p;
    __syncthreads();
    Part t;
    t.n = (sh[0].n + sh[1].n) + (sh[2].n + sh[3].n);
    t.mean = (sh[0].mean + sh[1].mean) + (sh[2].mean + sh[3].mean);
    t.m2 = (sh[0].m2 + sh[1].m2) + (sh[2].m2 + sh[3].m2);
    return t;
}

// the same two reductions over one wave only (every lane receives the result)
__device__ __forceinline__ Part wave_merge(Part p) {
    for (int o = 1; o < 64; o <<= 1) {
        Part q;
        q.n = __shfl_xor(p.n, o);
        q.mean = __shfl_xor(p.mean, o);
        q.m2 = __shfl_xor(p.m2, o);
        const bool upper = (threadIdx.x & o) != 0;
        p = upper ? merge(q, p) : merge(p, q);
    }
    return p;
}

__device__ __forceinline__ Part wave_sums(Part p) {
    for (int o = 1; o < 64; o <<= 1) {
        p.n += __shfl_xor(p.n, o);
        p.mean += __shfl_xor(p.mean, o);
        p.m2 += __shfl_xor(p.m2, o);
    }
    return p;
}

// a thread's running sums of one level: count, sum and sum of squares of (value - shift)
struct Acc {
    int n;
    double s1, s2;
};

__device__ __forceinline__ void acc_reset(Acc &a) {
    a.n = 0;
    a.s1 = a.s2 = 0.0;
}

__device__ __forceinline__ Part acc_part(const Acc &a, double shift) {
    Part p = {0.0, 0.0, 0.0};
    if (a.n > 0) {
        p.n = (double)a.n;
        p.mean = shift + a.s1 / p.n;
        p.m2 = fmax(0.0, a.s2 - a.s1 * (a.s1 / p.n));
    }
    return p;
}

// the estimate of one level, shared by the work-group
struct Level {
    double shift;       // subtracted before summing
    double m, lim;      // a value is kept in a rejection pass if |value - m| <= lim
    double sd, kept;
    double lc, lt;      // last full read: values with |value - lc| > lt are listed
    double nn, ns1, ns2;  // the unlisted values: count and sums of (value - lc) and its square
    int active;         // still being refined
    int iters;          // rejection passes that changed the estimate
    int listed;         // the lists hold every value beyond lt (none overflowed)
};

// every unlisted value is kept by a pass with this level's current mean and limit: the band
// |v - lc| <= lt lies inside |v - m| <= lim with room for the rounding of both differences
__device__ __forceinline__ bool band_covered(const Level &L) {
    const double slack = 1e-12 * (L.lim + L.lt + fabs(L.lc) + fabs(L.m));
    return L.listed && L.lt + fabs(L.lc - L.m) + slack <= L.lim;
}

struct MsdArgs {
    const float *x;
    int64_t ld;
    double *ws;          // per row: the values of levels 6.., then the lists of levels 0..5
    int64_t ws_row;      // doubles per row
    float *mean, *sigma, *rho, *level_sd;
    int32_t *passes;
    int32_t n_dm, n_in, levels, max_iter;
    double tau;
};

// a level's estimate after a pass with statistics u (one thread)
__device__ __forceinline__ void update_level(Level &S, const Part &u, bool probe, bool first,
                                             const MsdArgs &A) {
    if (probe) {
        // centre and band of the first pass's lists: 0.9 of the limit the pre-estimate gives,
        // less by three standard errors of its sd
        const double sd = u.n > 1.0 ? sqrt(u.m2 / (u.n - 1.0)) : 0.0;
        const double frac = 0.9 / (1.0 + 3.0 / sqrt(fmax(2.0 * u.n, 1.0)));
        S.shift = u.n > 0.0 ? u.mean : S.shift;
        S.lc = S.shift;
        S.lt = frac * A.tau * sd;
        return;
    }
    if (first) {
        S.m = u.mean;
        S.sd = u.n > 1.0 ? sqrt(u.m2 / (u.n - 1.0)) : 0.0;
        S.kept = u.n;
        S.active = A.max_iter > 0;
    } else if (u.n == S.kept || u.n < 2.0) {
        S.active = 0;
    } else {
        S.kept = u.n;
        S.m = u.mean;
        S.sd = sqrt(u.m2 / (u.n - 1.0));
        S.iters += 1;
        if (S.iters >= A.max_iter) S.active = 0;
    }
    S.lim = A.tau * S.sd;
    S.shift = S.m;
}

// take value v of a level (valid or not) into the thread's sums.  After the first pass the
// shift is the level's mean, so one difference serves the test and the sums.
__device__ __forceinline__ void take(Acc &a, const Level &L, bool first, bool valid, double v) {
    const double d = v - L.shift;
    const bool ok = valid && (first || fabs(d) <= L.lim);
    const double e = ok ? d : 0.0;           // (d may be NaN for a value past the data)
    a.n += ok ? 1 : 0;
    a.s1 += e;
    a.s2 = fma(e, e, a.s2);
}

// Level K from level K-1: a butterfly, after which every lane of a run of 2^(K-2) holds the sum of the
// run's two halves (a + b == b + a, so the lanes agree).  Within a row of 16 lanes DPP moves the
// other half's value: it is the same in every lane of that half, so mirrors serve as exchanges.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

template <int K>
__device__ __forceinline__ double level_step(double v) {
    if constexpr (K == 3) return v + dpp_f64<0xb1>(v);       // quad_perm 1 0 3 2
    else if constexpr (K == 4) return v + dpp_f64<0x4e>(v);  // quad_perm 2 3 0 1
    else if constexpr (K == 5) return v + dpp_f64<0x141>(v); // row_half_mirror
    else if constexpr (K == 6) return v + dpp_f64<0x140>(v); // row_mirror
    else {
        // rows 0 | 1 and 2 | 3 (level 7), lanes 0..31 | 32..63 (level 8)
        const long long b = __double_as_longlong(v);
        const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
        double x[2];
        if constexpr (K == 7) {
            const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
#pragma unroll
            for (int i = 0; i < 2; ++i) x[i] = __longlong_as_double(((long long)h[i] << 32) | l[i]);
        } else {
            const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
#pragma unroll
            for (int i = 0; i < 2; ++i) x[i] = __longlong_as_double(((long long)h[i] << 32) | l[i]);
        }
        return x[0] + x[1];
    }
}

// how many of the lanes below this one have their bit set in b (mbcnt)
__device__ __forceinline__ int count_below(uint64_t b) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
}

// A wave's list of one level being built: entry i waits in LDS at stage[i & 127], and each run of 64
// goes to memory in one store.  (A store per append kept the tile loop waiting: the compiler has to
// assume that a conditional store was not made when it counts what may be outstanding before a
// load, so a wait for the load became a wait for the store: 4096 x 262144 samples 2.15 ms, so 1.89.)
constexpr int kStage = 128;

__device__ __forceinline__ void list_flush(const double *stage, double *list, int first, int end, int lane) {
    __builtin_amdgcn_wave_barrier();         // the wave's LDS accesses are performed in order
    const int i = first + lane;
    const double v = stage[i & (kStage - 1)];
    if (i < end) list[i] = v;
    __builtin_amdgcn_wave_barrier();
}

// append the values of the lanes whose `far` is set to the wave's list, in lane order after the
// values appended before (a full list still counts them, which marks the overflow)
__device__ __forceinline__ void list_append(bool far, uint64_t b, double v, double *stage, double *list,
                                            int &cnt, int room, int lane) {
    if (b) {
        const int i = cnt + count_below(b);
        if (far) stage[i & (kStage - 1)] = v;
        const int was = cnt;
        cnt += __popcll(b);
        if ((cnt ^ was) & 64) list_flush(stage, list, was & ~63, min(room, (was & ~63) + 64), lane);
    }
}

// take for a level every lane of the wave serves: the count of kept values is kept per wave
// (a ballot's population count, on the scalar unit) instead of per lane.  LIST: values beyond
// the list threshold also go to the wave's list of the level.
// FIRST: every valid value is kept.  FULL: every value is valid.
template <bool FULL, bool FIRST, bool LIST>
__device__ __forceinline__ void take_w(Acc &a, uint32_t &nw, const Level &L, bool valid, double v,
                                       double *stage, double *list, int &cnt, int room, int lane) {
    const double d = v - L.shift;
    const bool ok = (FULL || valid) && (FIRST || fabs(d) <= L.lim);
    const double e = ok ? d : 0.0;           // (d may be NaN for a value past the data)
    nw += FULL && FIRST ? 64u : (uint32_t)__popcll(__ballot(ok));
    a.s1 += e;
    a.s2 = fma(e, e, a.s2);
    if (LIST) {
        const bool far = (FULL || valid) && !(fabs(d) <= L.lt);   // lc == shift
        list_append(far, __ballot(far), v, stage, list, cnt, room, lane);
    }
}

// statistics of a level all of whose values share one shift: the work-group's totals of the
// lanes' sums and the waves' counts give the mean and the sum of squared deviations (`tot`
// receives the totals: count and the sums of (value - shift) and its square)
__device__ __forceinline__ Part wave_counted_part(const Acc &a, uint32_t nw, double shift, Part *sh,
                                                  Part *tot = nullptr) {
    Part p = {(threadIdx.x & 63) == 0 ? (double)nw : 0.0, a.s1, a.s2};
    const Part t = block_sums(p, sh);
    if (tot) *tot = t;
    Part u = {0.0, 0.0, 0.0};
    if (t.n > 0.0) {
        u.n = t.n;
        u.mean = shift + t.mean / t.n;
        u.m2 = fmax(0.0, t.m2 - t.mean * (t.mean / t.n));
    }
    return u;
}

__global__ __launch_bounds__(kThreads, 4) void msd_kernel(const MsdArgs A) {
    __shared__ Part sh[4];
    __shared__ Level lv[SPD_MAX_LEVELS];
    __shared__ double stages[kWaves][kListLevels][kStage];
    __shared__ int list_cnt[kWaves][kListLevels];  // values each wave listed in the last full read
    __shared__ int any_active, pass_mode;
    const int d = blockIdx.x;
    if (d >= A.n_dm) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform over the wave
    const int n = A.n_in;
    const int K = A.levels;
    const int klist = min(K, kListLevels);
    const float *xr = A.x + (int64_t)d * A.ld;
    double *wr = A.ws + (int64_t)d * A.ws_row;
    const int n_tiles = (n + kTile - 1) / kTile;
    // a tile gives each wave 32 + 16 + 8 + 4 + 2 + 1 values of levels 3..8.  After step k a run of
    // 2^(k-2) lanes holds one value of level k; the run's middle lane takes it: the odd lanes level 3,
    // lanes 2, 6, 10.. level 4, ..., lane 32 level 8 (lane 0 none)
    const int my_k = lane ? 3 + __builtin_ctz(lane) : kRegLevels;
    double (*stage)[kStage] = stages[wave];
    // this wave's list of level k
    auto list_of = [&](int k) { return wr + list_offset(n, k) + (int64_t)wave * list_room(n, k); };

    if (tid < K) {
        Level &L = lv[tid];
        L.shift = (double)xr[0] * (double)(1 << tid);   // pre-estimate: a value of the right size
        L.m = 0.0;
        L.lim = 0.0;
        L.sd = 0.0;
        L.kept = 0.0;
        L.lc = L.shift;
        L.lt = 0.0;
        L.nn = L.ns1 = L.ns2 = 0.0;
        L.active = 1;
        L.iters = 0;
        L.listed = 0;
    }
    __syncthreads();

    // Kinds of pass: the pre-estimate (mean and sd of a few tiles spread over the row, which
    // centre the first pass's lists and set their band), a full read (the first estimate, or a
    // rejection pass, both listing the values beyond the band), a list pass (the listed values
    // only).  The pre-estimate counts as no pass.
    enum { kProbe = 0, kRead = 1, kList = 2 };
    const int n_probe = min(n_tiles, kProbeTiles);
    int pass = -1;
    for (; pass <= A.max_iter; ++pass) {
        const bool probe = pass < 0;
        const bool first = pass <= 0;            // every valid value is kept
        if (tid == 0) {
            int a = 0;
            bool lists = pass > 0;
            for (int k = 0; k < K; ++k) a |= lv[k].active;
            for (int k = 0; k < klist; ++k)
                if (lv[k].active) lists = lists && band_covered(lv[k]);
            const int mode = probe ? kProbe : lists ? kList : kRead;
            if (mode == kRead && pass > 0) {
                for (int k = 0; k < klist; ++k) {
                    Level &L = lv[k];
                    L.lc = L.shift;                 // the current mean
                    L.lt = kListFrac * L.lim;
                }
            }
            any_active = pass <= 0 ? 1 : a;
            pass_mode = mode;
        }
        __syncthreads();
        if (!any_active) break;
        const int mode = pass_mode;
        const bool build = mode == kRead;
        // the samples are read again only while a level of 0..5 is open and its listed values do
        // not suffice (levels 6.. come from the workspace after the first pass)
        bool read_row = first;
        for (int k = 0; k < klist; ++k) read_row = read_row || lv[k].active;
        read_row = read_row && mode != kList;
        Acc a0, a1, a2, am;                      // levels 0, 1, 2 and this lane's level of 3..8
        uint32_t n0w = 0, n1w = 0, n2w = 0;      // the wave's kept counts of levels 0, 1, 2
        int lc_[kListLevels];                    // the wave's listed counts (full read)
#pragma unroll
        for (int k = 0; k < kListLevels; ++k) lc_[k] = 0;
        acc_reset(a0);
        acc_reset(a1);
        acc_reset(a2);
        acc_reset(am);
        const Level L0 = lv[0];
        const Level L1 = lv[min(1, K - 1)];
        const Level L2 = lv[min(2, K - 1)];
        const Level Lm = lv[min(my_k, K - 1)];
        const bool on0 = first || L0.active;
        const bool on1 = K > 1 && (first || L1.active);
        const bool on2 = K > 2 && (first || L2.active);
        const bool onm = my_k < klist && (first || Lm.active);   // lanes of levels 3..5
        const bool arr = pass == 0 && my_k >= kArrFirst && my_k < K;   // lanes of 6..8

        auto fetch = [&](int tile) {                   // a tile all inside the data
            // streamed once per full read: keep the cache for the lists being written
            typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
            return __builtin_nontemporal_load(reinterpret_cast<const v4f *>(xr + tile * kTile + 4 * tid));
        };
        // where this lane's value of levels 6..8 of the next tile goes (first pass): a byte offset in
        // the row's values, past their end for the lanes that have none, whose stores are dropped
        // (every lane stores, so that the loads' waits can count the store)
        const auto arr_buf = __builtin_amdgcn_make_buffer_rsrc(wr, 0, (int)(((n >> 5) + 8) * 8), 0x00027000);
        uint32_t arr_at = 0x80000000u, arr_step = 0;
        if (arr) {
            arr_at = (uint32_t)(arr_offset(n, my_k) + wave * (256 >> my_k) + (lane >> (my_k - 2))) * 8u;
            arr_step = (uint32_t)(kTile >> my_k) * 8u;
        }
        // one tile; FULL: every sample of the tile is inside the data (all tiles but the last),
        // so the per-value validity tests fold away; FIRST: every valid value is kept; LIST: the
        // values beyond the band are listed
        auto tile_body = [&](auto full_tag, auto first_tag, auto list_tag, int tile, float c0, float c1,
                             float c2, float c3) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(full_tag)::value;
            constexpr bool FIRST = decltype(first_tag)::value;
            constexpr bool LIST = decltype(list_tag)::value;
            const int s = FULL ? 0 : tile * kTile + 4 * tid;     // first sample of this thread
            const double v0[4] = {(double)c0, (double)c1, (double)c2, (double)c3};
            if (FIRST || on0)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    take_w<FULL, FIRST, LIST>(a0, n0w, L0, FULL || s + q < n, v0[q], stage[0], list_of(0), lc_[0],
                                              list_room(n, 0), lane);
            // levels 1, 2 within the thread
            const double v1a = v0[0] + v0[1], v1b = v0[2] + v0[3];
            if (on1) {
                take_w<FULL, FIRST, LIST>(a1, n1w, L1, FULL || s + 2 <= n, v1a, stage[1], list_of(1), lc_[1],
                                          list_room(n, 1), lane);
                take_w<FULL, FIRST, LIST>(a1, n1w, L1, FULL || s + 4 <= n, v1b, stage[1], list_of(1), lc_[1],
                                          list_room(n, 1), lane);
            }
            double v = v1a + v1b;
            if (on2)
                take_w<FULL, FIRST, LIST>(a2, n2w, L2, FULL || s + 4 <= n, v, stage[2], list_of(2), lc_[2],
                                          list_room(n, 2), lane);
            // levels 3..8 across lanes; every lane keeps the one value of its own level
            double mv = v = level_step<3>(v);
            v = level_step<4>(v);
            mv = my_k == 4 ? v : mv;
            v = level_step<5>(v);
            mv = my_k == 5 ? v : mv;
            if (FIRST && LIST) {                               // levels 6.. are stored once
                v = level_step<6>(v);
                mv = my_k == 6 ? v : mv;
                v = level_step<7>(v);
                mv = my_k == 7 ? v : mv;
                v = level_step<8>(v);
                mv = my_k == 8 ? v : mv;
            }
            bool far = false;
            if (onm) {
                bool valid = true;
                if (!FULL) {
                    const int run = 1 << (my_k - 2);           // lanes that share the value
                    const int s0 = tile * kTile + 4 * (tid & -run);
                    valid = s0 + (1 << my_k) <= n && !__builtin_isnan(mv);
                }
                const double dm = mv - Lm.shift;
                const bool ok = valid && (FIRST || fabs(dm) <= Lm.lim);
                const double e = ok ? dm : 0.0;
                am.n += ok ? 1 : 0;
                am.s1 += e;
                am.s2 = fma(e, e, am.s2);
                if (LIST) far = valid && !(fabs(dm) <= Lm.lt);   // lc == shift
            }
            if (FIRST && LIST) {
                // the first pass stores levels 6..8 whole: level k's values of a tile in wave,
                // then lane order
                uint32_t at = arr_at;
                if (!FULL && arr) {
                    const int64_t i = (int64_t)tile * (kTile >> my_k) + wave * (256 >> my_k) + (lane >> (my_k - 2));
                    if (i >= (n >> my_k)) at = 0x80000000u;
                }
                typedef unsigned v2u __attribute__((ext_vector_type(2)));
                const long long w = __double_as_longlong(mv);
                __builtin_amdgcn_raw_buffer_store_b64(v2u{(unsigned)w, (unsigned)(w >> 32)}, arr_buf, (int)at, 0, 0);
                arr_at += arr_step;
            }
            if (LIST) {
                // append level by level (the ballot and the counts stay in uniform control flow)
                const uint64_t b = __ballot(far);
                if (b) {
#pragma unroll
                    for (int k = 3; k < kListLevels; ++k) {
                        const uint64_t lanes = k == 3 ? 0xaaaaaaaaaaaaaaaaull : k == 4 ? 0x4444444444444444ull
                                                                              : 0x1010101010101010ull;
                        list_append(far && my_k == k, b & lanes, mv, stage[k], list_of(k), lc_[k],
                                    list_room(n, k), lane);
                    }
                }
            }
        };
        // the pre-estimate reads tiles (i n_tiles) / n_probe, a full read every tile.  The loads of
        // two tiles are in flight while one is taken.
        auto read_tiles = [&](auto first_tag, auto list_tag) __attribute__((always_inline)) {
            constexpr bool kAll = decltype(list_tag)::value;
            const int n_read = kAll ? n_tiles : n_probe;
            auto tile_at = [&](int i) { return kAll ? i : (int)(((int64_t)i * n_tiles) / n_probe); };
            const int n_full = n_read - (tile_at(n_read - 1) * kTile + kTile > n ? 1 : 0);
            if (n_full > 0) {
                auto f0 = fetch(tile_at(0));
                auto f1 = fetch(tile_at(min(1, n_full - 1)));
                for (int i = 0; i < n_full; i += 2) {
                    const auto c0 = f0;
                    f0 = fetch(tile_at(min(i + 2, n_full - 1)));
                    tile_body(std::true_type{}, first_tag, list_tag, tile_at(i), c0.x, c0.y, c0.z, c0.w);
                    if (i + 1 >= n_full) break;
                    const auto c1 = f1;
                    f1 = fetch(tile_at(min(i + 3, n_full - 1)));
                    tile_body(std::true_type{}, first_tag, list_tag, tile_at(i + 1), c1.x, c1.y, c1.z, c1.w);
                }
            }
            if (n_full < n_read) {
                const int tile = tile_at(n_full), s = tile * kTile + 4 * tid;
                tile_body(std::false_type{}, first_tag, list_tag, tile, s + 0 < n ? xr[s + 0] : 0.0f,
                          s + 1 < n ? xr[s + 1] : 0.0f, s + 2 < n ? xr[s + 2] : 0.0f,
                          s + 3 < n ? xr[s + 3] : 0.0f);
            }
        };
        if (read_row) {
            if (probe) read_tiles(std::true_type{}, std::false_type{});
            else if (first) read_tiles(std::true_type{}, std::true_type{});
            else read_tiles(std::false_type{}, std::true_type{});
        }
        if (build) {
#pragma unroll
            for (int k = 0; k < kListLevels; ++k) {
                if (k >= klist) break;
                if (lc_[k] & 63)
                    list_flush(stage[k], list_of(k), lc_[k] & ~63, min(list_room(n, k), lc_[k]), lane);
                if (lane == 0) list_cnt[wave][k] = lc_[k];
            }
        }
        if (pass == 0 && K > 9) {
            // levels 9.. from pairs of the level below, all in the workspace
            __syncthreads();
            int64_t off_prev = arr_offset(n, 8), off = arr_offset(n, 9);
            for (int k = 9; k < K; ++k) {
                const int64_t cnt = (int64_t)(n >> k);
                for (int64_t i = tid; i < cnt; i += kThreads) wr[off + i] = wr[off_prev + 2 * i] + wr[off_prev + 2 * i + 1];
                off_prev = off;
                off += cnt;
                __syncthreads();
            }
        }
        __syncthreads();                          // list counts (and workspace levels) visible

        // merge the pass's statistics and update every level still being refined (the decision
        // to skip a level is uniform across the work-group)
        auto update_merged = [&](int k, const Part u) {
            if (tid == 0) update_level(lv[k], u, probe, first, A);
        };
        // the listed values of level k kept by the current estimate (every one in the first
        // pass): totals of the count and of the sums of (value - centre) and its square, in a
        // fixed order (the waves' lists in turn)
        auto list_sums = [&](int k, double centre) {
            const Level L = lv[k];
            const int room = list_room(n, k);
            Acc a;
            acc_reset(a);
            // the waves' lists one after another: entry j of the concatenation
            const double *l = wr + list_offset(n, k);
            const int c0 = min(list_cnt[0][k], room), c1 = min(list_cnt[1][k], room);
            const int c2 = min(list_cnt[2][k], room), c3 = min(list_cnt[3][k], room);
            const int p1 = c0, p2 = p1 + c1, p3 = p2 + c2, c = p3 + c3;
            for (int j0 = 0; j0 < c; j0 += 4 * kThreads) {
                double v[4];                     // four loads in flight, then their sums in order
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u * kThreads + tid;
                    const int w = (j >= p1) + (j >= p2) + (j >= p3);
                    const int base = w == 0 ? 0 : w == 1 ? p1 : w == 2 ? p2 : p3;
                    v[u] = j < c ? l[(int64_t)w * room + (j - base)] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool ok = j0 + u * kThreads + tid < c &&
                                    (first || fabs(v[u] - L.shift) <= L.lim);
                    const double e = ok ? v[u] - centre : 0.0;
                    a.n += ok ? 1 : 0;
                    a.s1 += e;
                    a.s2 = fma(e, e, a.s2);
                }
            }
            Part p = {(double)a.n, a.s1, a.s2};
            return block_sums(p, sh);
        };
        // full read: the unlisted values' statistics are the kept totals less the listed kept
        // values (all around the list centre)
        auto keep_unlisted = [&](int k, const Part &tot) {
            bool full = true;
            for (int w = 0; w < kWaves; ++w) full = full && list_cnt[w][k] <= list_room(n, k);
            Part ls = {0.0, 0.0, 0.0};
            if (full) ls = list_sums(k, lv[k].lc);
            if (tid == 0) {
                Level &S = lv[k];
                S.listed = full;
                S.nn = tot.n - ls.n;
                S.ns1 = tot.mean - ls.mean;
                S.ns2 = tot.m2 - ls.m2;
            }
        };
        if (mode == kList) {
            // a list pass: each wave takes levels wave, wave + 4, ... on its own (wave-only
            // reductions, the wave's lane 0 updates the level), one barrier at the end
            for (int k = wave; k < K; k += kWaves) {
                const Level L = lv[k];
                if (!L.active) continue;
                Part u = {0.0, 0.0, 0.0};
                if (k < klist) {
                    // the listed values: the four waves' lists one after another
                    const double *l = wr + list_offset(n, k);
                    const int room = list_room(n, k);
                    const int c0 = min(list_cnt[0][k], room), c1 = min(list_cnt[1][k], room);
                    const int c2 = min(list_cnt[2][k], room), c3 = min(list_cnt[3][k], room);
                    const int p1 = c0, p2 = p1 + c1, p3 = p2 + c2, c = p3 + c3;
                    Acc a;
                    acc_reset(a);
                    for (int j0 = 0; j0 < c; j0 += 4 * 64) {
                        double v[4];             // four loads in flight, then their sums in order
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int j = j0 + q * 64 + lane;
                            const int w = (j >= p1) + (j >= p2) + (j >= p3);
                            const int base = w == 0 ? 0 : w == 1 ? p1 : w == 2 ? p2 : p3;
                            v[q] = j < c ? l[(int64_t)w * room + (j - base)] : 0.0;
                        }
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const bool ok = j0 + q * 64 + lane < c && fabs(v[q] - L.shift) <= L.lim;
                            const double e = ok ? v[q] - L.lc : 0.0;
                            a.n += ok ? 1 : 0;
                            a.s1 += e;
                            a.s2 = fma(e, e, a.s2);
                        }
                    }
                    const Part t = wave_sums(Part{(double)a.n, a.s1, a.s2});
                    const double cnt = L.nn + t.n;
                    if (cnt > 0.0) {
                        const double s1 = L.ns1 + t.mean, s2 = L.ns2 + t.m2;
                        u.n = cnt;
                        u.mean = L.lc + s1 / cnt;
                        u.m2 = fmax(0.0, s2 - s1 * (s1 / cnt));
                    }
                } else {
                    // a level stored whole in the workspace
                    const int64_t cnt = (int64_t)(n >> k);
                    const double *vals = wr + arr_offset(n, k);
                    Acc a;
                    acc_reset(a);
                    for (int64_t i0 = 0; i0 < cnt; i0 += 4 * 64) {
                        double v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int64_t i = i0 + q * 64 + lane;
                            v[q] = i < cnt ? vals[i] : 0.0;
                        }
#pragma unroll
                        for (int q = 0; q < 4; ++q) take(a, L, false, i0 + q * 64 + lane < cnt, v[q]);
                    }
                    u = wave_merge(acc_part(a, L.shift));
                }
                if (lane == 0) update_level(lv[k], u, false, false, A);
            }
            __syncthreads();
            continue;
        }
        for (int k = 0; k < klist; ++k) {
            if (!(first || lv[k].active)) continue;
            if (k < 3) {
                const Acc &a = k == 0 ? a0 : k == 1 ? a1 : a2;
                const uint32_t nw = k == 0 ? n0w : k == 1 ? n1w : n2w;
                Part tot;
                const Part u = wave_counted_part(a, nw, lv[k].shift, sh, &tot);
                if (build) keep_unlisted(k, tot);
                update_merged(k, u);
            } else {
                Part p = {0.0, 0.0, 0.0};
                if (my_k == k) p = acc_part(am, lv[k].shift);
                const Part u = block_merge(p, sh);
                if (build) {
                    Part q = {0.0, 0.0, 0.0};
                    if (my_k == k) q = Part{(double)am.n, am.s1, am.s2};
                    keep_unlisted(k, block_sums(q, sh));
                }
                update_merged(k, u);
            }
            __syncthreads();
        }
        if (probe) continue;
        int64_t off = 0;
        for (int k = kArrFirst; k < K; ++k) {
            const int64_t cnt = (int64_t)(n >> k);
            const Level Lk = lv[k];
            if (first || Lk.active) {
                Acc a;
                acc_reset(a);
                for (int64_t i0 = 0; i0 < cnt; i0 += 4 * kThreads) {
                    double v[4];                 // four loads in flight, then their sums in order
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int64_t i = i0 + u * kThreads + tid;
                        v[u] = i < cnt ? wr[off + i] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) take(a, Lk, first, i0 + u * kThreads + tid < cnt, v[u]);
                }
                update_merged(k, block_merge(acc_part(a, Lk.shift), sh));
                __syncthreads();
            }
            off += cnt;
        }
    }

    if (tid < K) {
        const double sd0 = lv[0].sd;
        const double sd = lv[tid].sd;
        if (tid == 0) {
            A.mean[d] = (float)lv[0].m;
            A.sigma[d] = (float)sd0;
            if (A.passes) A.passes[d] = pass;
        }
        if (A.rho) A.rho[(int64_t)d * K + tid] = (float)(sd / (sqrt((double)(1 << tid)) * sd0));
        if (A.level_sd) A.level_sd[(int64_t)d * K + tid] = (float)sd;
    }
}

}  // namespace spdm

extern "C" {

int spd_msd_workspace(int32_t n_dm, int32_t n_in, int32_t levels, int64_t *bytes) {
    if (!bytes || n_dm < 1 || n_in < 2 || n_in > INT32_MAX - 4096 || levels < 1 ||
        levels > SPD_MAX_LEVELS || ((int64_t)n_in >> (levels - 1)) < 2)
        return SPD_EINVAL;
    // levels 6.. of every row (fewer than n_in / 32 values) and the lists of levels 0..5
    *bytes = (int64_t)n_dm * spdm::ws_row_doubles(n_in) * 8 + 256;
    return SPD_OK;
}

int spd_msd(const float *x, int64_t ld, int32_t n_dm, int32_t n_in, int32_t levels, float tau,
            int32_t max_iter, float *mean, float *sigma, float *rho, float *level_sd,
            int32_t *passes, void *workspace, int64_t workspace_bytes, void *hip_stream) {
    int64_t need = 0;
    const int st = spd_msd_workspace(n_dm, n_in, levels, &need);
    if (st != SPD_OK) return st;
    if (!x || ld < n_in || !mean || !sigma || !(tau > 0.0f) || max_iter < 0) return SPD_EINVAL;
    if (!workspace || workspace_bytes < need) return SPD_EWORKSPACE;
    if ((uintptr_t)workspace & 255) return SPD_EALIGN;
    spdm::MsdArgs a;
    a.x = x;
    a.ld = ld;
    a.ws = static_cast<double *>(workspace);
    a.ws_row = spdm::ws_row_doubles(n_in);
    a.mean = mean;
    a.sigma = sigma;
    a.rho = rho;
    a.level_sd = level_sd;
    a.passes = passes;
    a.n_dm = n_dm;
    a.n_in = n_in;
    a.levels = levels;
    a.max_iter = max_iter;
    a.tau = (double)tau;
    hipLaunchKernelGGL(spdm::msd_kernel, dim3(n_dm), dim3(spdm::kThreads), 0,
                       static_cast<hipStream_t>(hip_stream), a);
    return hipGetLastError() == hipSuccess ? SPD_OK : SPD_EHIP;
}

}  // extern "C"
