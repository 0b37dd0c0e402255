// Neighbour-list path of the KSG estimator (gfx950).
//
// Every estimate of a job shares the rows of Y and Z; only X is permuted.  A
// row's k-th neighbour distance eps and its three strict counts below eps
// only involve rows that are close to it in the (Y,Z) subspace (for the k-NN
// radius and n_yz) or in the Z subspace (n_z and n_xz, since both need
// d_z < eps).  So, once per (Y,Z) sample:
//
//   build    for each row i, the other rows bucketed by d_yz(i,j) and by
//            d_z(i,j) (12-bit keys of the float encoding), keeping the
//            smallest buckets that fit the list capacity, in bucket order,
//            then sentinels with a lower bound of every distance left out;
//
// and then, a wave per row and group of estimates, a lane per estimate:
//
//   scan     k-NN over list 1 in bucket order, max(d_x, d_yz) with the
//            estimate's permuted X; it stops at the first bucket whose floor
//            reaches the current k-th distance (nothing later can enter).  The
//            radius is exact when it stopped that way or when the k-th
//            distance is at most the list's bound.  n_yz counts the entries of
//            list 1 below eps, n_z and n_xz scan list 2 until its bucket floor
//            reaches eps, exact when it stopped that way or eps <= its bound;
//   counts   with one Z column and one Y column n_z and n_xz are ranges of
//            ranks of z instead: rows of a range counted one by one (rank
//            counts), or, with one X column and no window, two-dimensional
//            ranges in a wavelet matrix per estimate.  Such jobs with several
//            X columns and no window exchange the sides: lists over X, the
//            permuted columns are Y and Z;
//   walk     without Z, with one X and one Y column, no lists: radii from the
//            neighbouring ranks of y, counts from the sorted columns;
//   fallback the pairs the lists cannot decide (rare) are queued and redone
//            over all rows (a block per pair, or a wave when they are many);
//   reduce   the digamma sum per estimate in the same fixed order as the
//            all-pairs kernel (64-row butterfly, then chunks in index order),
//            so both paths return the same bits.
//
// The results are the definitions' exact values: every distance is the same
// fl32 subtraction, |.| and max as in the all-pairs kernel, and the lists only
// skip rows whose distances provably cannot change the outcome.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>

#include "engine.h"
#include "ksg_device.h"

namespace mte {

namespace {

using dev::absdiff;
using dev::find_job;
using dev::fmax_;
using dev::inf_f;
using dev::topk_insert;
using dev::Unroll;

constexpr uint32_t kKeyMask = kKeyBins - 1;
constexpr uint32_t kFloorMask = ~((1u << kKeyShift) - 1u);

// Work-item and work-group indices straight from the hardware registers (the
// group index is a scalar value, so it stays wave-uniform).
__device__ __forceinline__ int tid_x() { return (int)__builtin_amdgcn_workitem_id_x(); }
__device__ __forceinline__ int64_t bid_x() { return (int64_t)__builtin_amdgcn_workgroup_id_x(); }

// Read-only memory addressed through the constant address space: a load from
// a wave-uniform address is then a scalar load.
template <class T>
using Const = const __attribute__((address_space(4))) T;
template <class T>
__device__ __forceinline__ Const<T> *as_const(const T *p) { return (Const<T> *)p; }

// Load through a global-address-space pointer: a generic (flat) load would
// count against both the vector-memory and the LDS counters, and the wait for
// the gathers would then also wait for the next step's entries loaded ahead.
__device__ __forceinline__ float gload(const float *p, uint32_t off) {
    return ((const __attribute__((address_space(1))) float *)p)[off];
}

// List entries stored through global-address-space pointers: a generic
// (flat) store counts against the LDS counter too, so the next wait for an
// LDS atomic's return would also wait for the store to reach memory.
__device__ __forceinline__ void gstore(LEnt *p, uint32_t idx, const LEnt &v) {
    auto *q = (__attribute__((address_space(1))) uint32_t *)(p + idx);
    q[0] = __float_as_uint(v.d);
    q[1] = (uint32_t)v.j;
}

// The same with a byte offset: the address is then a uniform base plus one
// 32-bit register, the form the global loads take without address arithmetic.
__device__ __forceinline__ float gload_b(const float *p, uint32_t byte_off) {
    return *(const __attribute__((address_space(1))) float *)((const __attribute__((address_space(1))) char *)p +
                                                              byte_off);
}

constexpr uint64_t kRankNone = 0xbf800000u;   // radius -1: the pair is in the redo queue

// Bucket key of a distance d >= 0 (+inf included): its exponent and top
// mantissa bits.  The sign bit is clear, so a plain shift (which gfx950
// issues at twice the rate of a bit-field extract) gives the 12-bit field.
__device__ __forceinline__ uint32_t key_of(float d) {
    return __float_as_uint(d) >> kKeyShift;
}

// Smallest value of d's bucket (d >= 0).
__device__ __forceinline__ float bucket_floor(float d) {
    return __uint_as_float(__float_as_uint(d) & kFloorMask);
}

__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = __builtin_fminf(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The build shares the CUs with the surrogate permutation (a second stream),
// and both are bound by instruction issue; the scan needs both.  The build's
// waves take the issue arbiter's highest priority, so that the permutation,
// held to a few blocks per CU, runs in the build's idle issue cycles instead
// of stretching it: at N = 10^4 with 201 estimates the pair finishes
// together in 0.25 ms instead of 0.28.
constexpr int kBuildPrio = 3;

// Threads per build block: 8 waves, so that the 4 blocks whose histograms fit
// in LDS keep 8 waves on every SIMD (the kernel waits mostly on LDS atomics
// and L2 loads, and needs the waves to hide them).
constexpr int kBT = 512;
constexpr int kBW = kBT / 64;

// Inclusive scan over the kBT threads of a build block; returns the block total.
template <int NW = kBW>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t &incl, uint32_t *wtot) {
    const int lane = tid_x() & 63, wave = tid_x() >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(v, off, 64);
        if (lane >= off) v += u;
    }
    if (lane == 63) wtot[wave] = v;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        before += w < wave ? wtot[w] : 0u;
        total += wtot[w];
    }
    incl = before + v;
    __syncthreads();
    return total;
}

// ------------------------------------------------------------------ build
// One block per (list set, QB consecutive rows).  Pass 1 histograms the keys
// of d_yz and d_z over the other rows; for each row and list the largest key
// prefix that fits the capacity is kept and the histogram becomes the bucket
// write cursors; pass 2 recomputes the same distances and writes the kept
// rows bucket by bucket.  Each reference row is loaded once for the QB rows of
// the block.  The histogram of a row has C copies, lane l counting into copy
// l mod C, so that lanes with equal keys mostly update different words (the
// cursors of a bucket's copies follow each other, keeping bucket order).
// PACK: both lists' counts of a bucket share one 32-bit word, 16 bits each
// (counts stay below 2^16 when N <= 2^16).
template <int QB>
constexpr int row_batch() { return QB == 1 ? 8 : 4; }   // reference rows per thread per step

// The selection gives each thread kPer consecutive buckets (read and written
// as 16-byte words).  Bucket b of a histogram is word b: the passes over the
// pairs then take a bucket's address straight from the distance's bits.
constexpr int kPer = kKeyBins / kBT;
constexpr int kHistWords = kKeyBins;

__device__ __forceinline__ uint32_t hist_slot(uint32_t key) { return key; }

template <int QB, int C, bool PACK>
struct BuildSmem {
    static constexpr int kCopy = PACK ? kHistWords : 2 * kHistWords;   // words of one copy
    alignas(16) uint32_t h[QB][C][kCopy];
    float q[QB][kMaxDy + kMaxDz];
    uint32_t wtot[kBW];
    uint32_t red[2][kBW];
    uint32_t kept_bins[QB][2], kept_rows[QB][2];
    int set;
};

template <bool PACK>
__device__ __forceinline__ uint32_t *bin_word(uint32_t *h, int w, uint32_t key) {
    return PACK ? h + hist_slot(key) : h + w * kHistWords + hist_slot(key);
}

template <bool PACK>
__device__ __forceinline__ uint32_t bin_inc(int w) {
    return PACK ? (1u << (16 * w)) : 1u;
}

template <bool PACK>
__device__ __forceinline__ uint32_t bin_get(uint32_t word, int w) {
    return PACK ? (word >> (16 * w)) & 0xffffu : word;
}

template <bool PACK>
__device__ __forceinline__ void bin_set(uint32_t *wd, int w, uint32_t v) {
    if (PACK) *wd = (*wd & ~(0xffffu << (16 * w))) | (v << (16 * w));
    else *wd = v;
}

// Max-norm over coordinates [c_lo, c_hi) of the contiguous column copy
// (column c at zy + c * n) into acc[r][u] for the block rows r and the
// reference rows whose byte offsets within a column are boff[u]; the loads of
// up to kColChunk coordinates are issued together before they are used.
constexpr int kColChunk = 4;

template <int QB, int R>
__device__ __forceinline__ void acc_cols(const float *zy, int n, const float (*q)[kMaxDy + kMaxDz], int c_lo,
                                         int c_hi, const uint32_t (&boff)[R], float (&acc)[QB][R]) {
    for (int c0 = c_lo; c0 < c_hi; c0 += kColChunk) {
        float v[kColChunk][R];
#pragma unroll
        for (int cc = 0; cc < kColChunk; ++cc) {
            if (c0 + cc < c_hi) {
                const float *col = zy + (size_t)(c0 + cc) * n;
#pragma unroll
                for (int u = 0; u < R; ++u) v[cc][u] = gload_b(col, boff[u]);
            }
        }
#pragma unroll
        for (int cc = 0; cc < kColChunk; ++cc) {
            if (c0 + cc < c_hi) {
#pragma unroll
                for (int r = 0; r < QB; ++r) {
                    const float qc = q[r][c0 + cc];
#pragma unroll
                    for (int u = 0; u < R; ++u) acc[r][u] = fmax_(acc[r][u], absdiff(qc, v[cc][u]));
                }
            }
        }
    }
}

// Geometry of one list set, held in registers for the whole block.
struct BuildGeo {
    const float *zy;
    int n, dy, dz, w;
};

// Calls f(r, j, d_z, d_yz) for every block row r (valid rows only) and every
// row j outside its Theiler window (|j - i| > w; j != i when w = 0),
// row_batch<QB>() reference rows per thread at a time.
template <int QB, class F>
__device__ __forceinline__ void for_each_pair(const BuildGeo &G, const float (*q)[kMaxDy + kMaxDz], int i0,
                                              int nq, int tid, F &&f) {
    constexpr int kRowBatch = row_batch<QB>();
    const int n = G.n, D = G.dy + G.dz;
    // |j - i| > w  <=>  (unsigned)(j - i + w) > 2w
    const uint32_t w2 = 2u * (uint32_t)G.w;
    for (int j0 = tid; j0 < n; j0 += kBT * kRowBatch) {
        float a[QB][kRowBatch], b[QB][kRowBatch];
        uint32_t boff[kRowBatch];
#pragma unroll
        for (int u = 0; u < kRowBatch; ++u) {
            const int j = j0 + u * kBT;
            boff[u] = (uint32_t)(j < n ? j : i0) * 4u;
        }
#pragma unroll
        for (int r = 0; r < QB; ++r)
#pragma unroll
            for (int u = 0; u < kRowBatch; ++u) a[r][u] = 0.f;
        acc_cols<QB, kRowBatch>(G.zy, n, q, 0, G.dz, boff, a);
#pragma unroll
        for (int r = 0; r < QB; ++r)
#pragma unroll
            for (int u = 0; u < kRowBatch; ++u) b[r][u] = a[r][u];
        acc_cols<QB, kRowBatch>(G.zy, n, q, G.dz, D, boff, b);
#pragma unroll
        for (int u = 0; u < kRowBatch; ++u) {
            const int j = j0 + u * kBT;
            if (j >= n) continue;
#pragma unroll
            for (int r = 0; r < QB; ++r)
                if (r < nq && (uint32_t)(j + (G.w - i0 - r)) > w2) f(r, j, a[r][u], b[r][u]);
        }
    }
}

template <int QB, int C, bool PACK>
__global__ __launch_bounds__(kBT) void list_build_kernel(const ListSet *__restrict__ sets, int n_sets,
                                                           const int64_t *__restrict__ blk_off) {
    using Sm = BuildSmem<QB, C, PACK>;
    __shared__ Sm sm;
    __builtin_amdgcn_s_setprio(kBuildPrio);
    const int tid = tid_x();
    const int copy = tid & (C - 1);
    const int64_t b = bid_x() + blk_off[0];
    if (tid == 0) sm.set = find_job(blk_off, n_sets, b);
    for (int x = tid; x < QB * C * Sm::kCopy; x += kBT) (&sm.h[0][0][0])[x] = 0u;
    __syncthreads();
    const ListSet &S = sets[sm.set];
    const BuildGeo G{S.zy, S.n, S.dy, S.dz, S.theiler};
    const int n = G.n;
    const int i0 = (int)(b - blk_off[sm.set]) * QB;
    const int nq = min(QB, n - i0);
    for (int x = tid; x < QB * (G.dy + G.dz); x += kBT) {
        const int r = x / (G.dy + G.dz), c = x - r * (G.dy + G.dz);
        sm.q[r][c] = G.zy[(size_t)c * n + min(i0 + r, n - 1)];
    }
    __syncthreads();

    for_each_pair<QB>(G, sm.q, i0, nq, tid, [&](int r, int, float a, float c) {
        const uint32_t k1 = key_of(c), k2 = key_of(a);
        if (PACK) {
            // d_yz and d_z often share a bucket (when d_y <= d_z): one atomic
            // then counts both lists
            atomicAdd(bin_word<PACK>(sm.h[r][copy], 0, k1),
                      k1 == k2 ? bin_inc<PACK>(0) + bin_inc<PACK>(1) : bin_inc<PACK>(0));
            if (k1 != k2) atomicAdd(bin_word<PACK>(sm.h[r][copy], 1, k2), bin_inc<PACK>(1));
        } else {
            atomicAdd(bin_word<PACK>(sm.h[r][copy], 0, k1), bin_inc<PACK>(0));
            atomicAdd(bin_word<PACK>(sm.h[r][copy], 1, k2), bin_inc<PACK>(1));
        }
    });
    __syncthreads();

    // per row and list: keep the largest bucket prefix with at most m entries
    // (bucket keys below kept_bins are listed: the prefix is contiguous
    // because the cumulative counts grow with the key)
#pragma unroll
    for (int r = 0; r < QB; ++r) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const uint32_t cap = (uint32_t)(w == 0 ? S.m1 : S.m2);
            uint32_t local = 0;
#pragma unroll
            for (int x = 0; x < kPer; ++x)
#pragma unroll
                for (int cp = 0; cp < C; ++cp)
                    local += bin_get<PACK>(*bin_word<PACK>(sm.h[r][cp], w, tid * kPer + x), w);
            uint32_t incl;
            block_scan(local, incl, sm.wtot);
            uint32_t run = incl - local, nb = 0, nr = 0;
#pragma unroll
            for (int x = 0; x < kPer; ++x) {
                uint32_t cnt = 0;
#pragma unroll
                for (int cp = 0; cp < C; ++cp) {
                    // exclusive start of (bucket, copy) = write cursor
                    uint32_t *wd = bin_word<PACK>(sm.h[r][cp], w, tid * kPer + x);
                    const uint32_t v = bin_get<PACK>(*wd, w);
                    bin_set<PACK>(wd, w, run + cnt);
                    cnt += v;
                }
                run += cnt;
                if (run <= cap) { ++nb; nr += cnt; }
            }
            nb = (uint32_t)wave_sum((int)nb);
            nr = (uint32_t)wave_sum((int)nr);
            if ((tid & 63) == 0) { sm.red[0][tid >> 6] = nb; sm.red[1][tid >> 6] = nr; }
            __syncthreads();
            if (tid == 0) {
                uint32_t kb = 0, kr = 0;
                for (int v = 0; v < kBW; ++v) { kb += sm.red[0][v]; kr += sm.red[1][v]; }
                sm.kept_bins[r][w] = kb;
                sm.kept_rows[r][w] = kr;
            }
            __syncthreads();
        }
    }
    // pass 2 with the kept prefixes and the rows' list bases in registers
    uint32_t keep[QB][2];
    LEnt *out1[QB];
    LEnt *out2[QB];
#pragma unroll
    for (int r = 0; r < QB; ++r) {
        keep[r][0] = sm.kept_bins[r][0];
        keep[r][1] = sm.kept_bins[r][1];
        const int64_t i = min(i0 + r, n - 1);
        out1[r] = S.l1 + i * S.s1;
        out2[r] = S.l2 + i * S.s2;
    }
    const uint32_t m1 = (uint32_t)S.m1, m2 = (uint32_t)S.m2;
    for_each_pair<QB>(G, sm.q, i0, nq, tid, [&](int r, int j, float a, float c) {
        const uint32_t k1 = key_of(c), k2 = key_of(a);
        if (k1 < keep[r][0]) {
            const uint32_t pos =
                bin_get<PACK>(atomicAdd(bin_word<PACK>(sm.h[r][copy], 0, k1), bin_inc<PACK>(0)), 0);
            if (pos < m1) gstore(out1[r], pos, LEnt{c, j});
        }
        if (k2 < keep[r][1]) {
            const uint32_t pos =
                bin_get<PACK>(atomicAdd(bin_word<PACK>(sm.h[r][copy], 1, k2), bin_inc<PACK>(1)), 1);
            if (pos < m2) gstore(out2[r], pos, LEnt{a, j});
        }
    });
    // lengths and the sentinels after each list.  A list is whole
    // when it holds every row outside the window, or when the first bucket
    // left out is the +inf bucket (every row at a finite distance fitted and
    // the others' differences overflow): a row at +inf can enter neither a
    // radius (every listed distance is at most +inf) nor a strict count below
    // any radius, so leaving it out changes nothing.  Whole lists get +inf
    // sentinels; the bound + 1 ulp would be a NaN there.
    for (int x = tid; x < QB * 2 * kListPad; x += kBT) {
        const int r = x / (2 * kListPad), w = (x / kListPad) & 1, u = x % kListPad;
        if (r >= nq) continue;
        const int64_t i = i0 + r;
        const int tw = S.theiler;   // rows outside the window
        const uint32_t total = (uint32_t)(n - 1 - min((int)i, tw) - min(n - 1 - (int)i, tw));
        const uint32_t kb = sm.kept_bins[r][w], kr = sm.kept_rows[r][w];
        const bool whole = kr == total || (kb << kKeyShift) >= __float_as_uint(inf_f());
        const float sent = whole ? inf_f() : __uint_as_float((kb << kKeyShift) + 1u);
        if (w == 0) S.l1[i * S.s1 + kr + u] = LEnt{sent, (int32_t)i};
        else S.l2[i * S.s2 + kr + u] = LEnt{sent, (int32_t)i};
        if (u == 0) S.len[2 * i + w] = (int32_t)kr;
    }
}

// ------------------------------------------------------------------ build, compiled dimensions
// list_build_kernel for sets with DZ Z columns and one Y column, N < 2^16,
// QB rows per block: two passes over the pairs as there, with straight-line
// distance code and a counting pass without branches.  The counting pass
// counts every row j < N, the query row itself included (its distances are
// exactly 0, so it adds one to bin 0 of both lists), and sends the lanes past
// the last row to bin 4095, the bin of NaN encodings, which no distance
// reaches; afterwards the query row and the rows of its Theiler window are
// taken out again and bin 4095 is cleared.  The selection takes both lists
// of every row in one block scan: a bin's word holds both lists' counts, 16
// bits each, and their sums stay below 2^16, so one packed prefix is both
// lists' write cursors.  The write pass checks the window per pair.
constexpr int kLR = 4;                  // reference rows per thread per step

template <int DZ, int QB, int R>
__device__ __forceinline__ void lean_dists(const float *zy, int n, const float (&q)[QB][DZ + 1],
                                           const uint32_t (&boff)[R], float (&az)[QB][R], float (&ayz)[QB][R]) {
    float v[DZ + 1][R];
#pragma unroll
    for (int c = 0; c < DZ + 1; ++c)
#pragma unroll
        for (int u = 0; u < R; ++u) v[c][u] = gload_b(zy + (size_t)c * n, boff[u]);
#pragma unroll
    for (int r = 0; r < QB; ++r)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            float a = absdiff(q[r][0], v[0][u]);
#pragma unroll
            for (int c = 1; c < DZ; ++c) a = fmax_(a, absdiff(q[r][c], v[c][u]));
            az[r][u] = a;
            ayz[r][u] = fmax_(a, absdiff(q[r][DZ], v[DZ][u]));
        }
}

template <int QB>
struct LeanSmem {
    alignas(16) uint32_t h[QB][kKeyBins];   // list 1 count | list 2 count << 16, then cursors
    float q[QB][kBuildFixedDz + 1];
    uint32_t wtot[QB][kBW];
    uint32_t red[2 * QB][kBW];
    int set;
};

template <int DZ, int QB>
__global__ __launch_bounds__(kBT) void list_build_dz_kernel(const ListSet *__restrict__ sets, int n_sets,
                                                            const int64_t *__restrict__ blk_off) {
    __shared__ LeanSmem<QB> sm;
    __builtin_amdgcn_s_setprio(kBuildPrio);
    const int tid = tid_x(), lane = tid & 63, wave = tid >> 6;
    const int64_t b = bid_x() + blk_off[0];
    if (tid == 0) sm.set = find_job(blk_off, n_sets, b);
    for (int x = tid; x < QB * kKeyBins; x += kBT) (&sm.h[0][0])[x] = 0u;
    __syncthreads();
    const ListSet &S = sets[sm.set];
    const float *zy = S.zy;
    const int n = S.n, tw = S.theiler;
    const int i0 = (int)(b - blk_off[sm.set]) * QB;
    const int nq = min(QB, n - i0);
    for (int x = tid; x < QB * (DZ + 1); x += kBT) {
        const int r = x / (DZ + 1), c = x - r * (DZ + 1);
        sm.q[r][c] = zy[(size_t)c * n + min(i0 + r, n - 1)];
    }
    __syncthreads();
    float q[QB][DZ + 1];
#pragma unroll
    for (int r = 0; r < QB; ++r)
#pragma unroll
        for (int c = 0; c < DZ + 1; ++c) q[r][c] = sm.q[r][c];
    constexpr uint32_t kInc1 = 1u, kInc2 = 1u << 16, kSink = (uint32_t)kKeyBins - 1u;
    const int step = kBT * kLR;
    const int full = n / step * step;

    // pass 1: counts of every row j < n
    auto count_step = [&](int j0, bool tail) {
        uint32_t boff[kLR], sink[kLR];
#pragma unroll
        for (int u = 0; u < kLR; ++u) {
            const int j = j0 + u * kBT;
            const bool in = !tail || j < n;
            boff[u] = (uint32_t)(in ? j : i0) * 4u;
            sink[u] = in ? 0u : kSink;
        }
        float az[QB][kLR], ayz[QB][kLR];
        lean_dists<DZ, QB, kLR>(zy, n, q, boff, az, ayz);
#pragma unroll
        for (int r = 0; r < QB; ++r)
#pragma unroll
            for (int u = 0; u < kLR; ++u) {
                const uint32_t k1 = key_of(ayz[r][u]) | sink[u], k2 = key_of(az[r][u]) | sink[u];
                // one compare: the increment is chosen in the branch that
                // takes the second key's atomic
                uint32_t inc = kInc1 + kInc2;
                if (k1 != k2) {
                    inc = kInc1;
                    atomicAdd(&sm.h[r][k2], kInc2);
                }
                atomicAdd(&sm.h[r][k1], inc);
            }
    };
    int j0 = tid;
    for (; j0 < full; j0 += step) count_step(j0, false);
    if (j0 < n) count_step(j0, true);
    __syncthreads();
    // take out the query rows and their windows (counted above), clear the sink
    const int wn = 2 * tw + 1;
    for (int x = tid; x < QB * wn; x += kBT) {
        const int r = x / wn, j = i0 + r + (x % wn) - tw;
        if (r >= nq || j < 0 || j >= n) continue;
        float a = 0.f;
#pragma unroll
        for (int c = 0; c < DZ; ++c) a = fmax_(a, absdiff(sm.q[r][c], zy[(size_t)c * n + j]));
        const float cyz = fmax_(a, absdiff(sm.q[r][DZ], zy[(size_t)DZ * n + j]));
        atomicSub(&sm.h[r][key_of(cyz)], kInc1);
        atomicSub(&sm.h[r][key_of(a)], kInc2);
    }
    __syncthreads();
    if (tid < QB) sm.h[tid][kSink] = 0u;
    __syncthreads();

    // selection: per row, the packed exclusive prefix over the bins (thread t
    // owns bins t*kPer .. t*kPer+kPer-1) becomes the cursors; a list keeps
    // the bins whose inclusive count fits its capacity (a prefix, since the
    // counts only grow)
    const uint32_t m1 = (uint32_t)S.m1, m2 = (uint32_t)S.m2;
    uint32_t kb[QB][2], kr[QB][2];
    {
        uint32_t loc[QB], run[QB];
#pragma unroll
        for (int r = 0; r < QB; ++r) {
            loc[r] = 0;
#pragma unroll
            for (int x = 0; x < kPer; ++x) loc[r] += sm.h[r][tid * kPer + x];
            run[r] = loc[r];
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1)
#pragma unroll
            for (int r = 0; r < QB; ++r) {
                const uint32_t t = __shfl_up(run[r], off, 64);
                if (lane >= off) run[r] += t;
            }
        if (lane == 63)
#pragma unroll
            for (int r = 0; r < QB; ++r) sm.wtot[r][wave] = run[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < QB; ++r) {
            uint32_t before = 0;
#pragma unroll
            for (int w = 0; w < kBW; ++w) before += w < wave ? sm.wtot[r][w] : 0u;
            run[r] += before - loc[r];         // exclusive start of this thread's bins
            uint32_t nb = 0, nr = 0;
#pragma unroll
            for (int x = 0; x < kPer; ++x) {
                uint32_t *wd = &sm.h[r][tid * kPer + x];
                const uint32_t v = *wd;
                *wd = run[r];
                run[r] += v;
                // bins kept by list 1 (low half) and list 2 (high half)
                if ((run[r] & 0xffffu) <= m1) { nb += 1u; nr += v & 0xffffu; }
                if ((run[r] >> 16) <= m2) { nb += 1u << 16; nr += v & 0xffff0000u; }
            }
            nb = (uint32_t)wave_sum((int)nb);
            nr = (uint32_t)wave_sum((int)nr);
            if (lane == 0) {
                sm.red[2 * r][wave] = nb;
                sm.red[2 * r + 1][wave] = nr;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < QB; ++r) {
            uint32_t nb = 0, nr = 0;
#pragma unroll
            for (int w = 0; w < kBW; ++w) {
                nb += sm.red[2 * r][w];
                nr += sm.red[2 * r + 1][w];
            }
            kb[r][0] = nb & 0xffffu;
            kb[r][1] = nb >> 16;
            kr[r][0] = nr & 0xffffu;
            kr[r][1] = nr >> 16;
        }
    }

    // pass 2: write the kept rows (bin 4095 never holds a row: kept bins are
    // taken below it)
    uint32_t keep1[QB], keep2[QB];
    LEnt *out1[QB];
    LEnt *out2[QB];
#pragma unroll
    for (int r = 0; r < QB; ++r) {
        keep1[r] = min(kb[r][0], kSink);
        keep2[r] = min(kb[r][1], kSink);
        const int64_t i = min(i0 + r, n - 1);
        out1[r] = S.l1 + i * S.s1;
        out2[r] = S.l2 + i * S.s2;
    }
    const uint32_t w2 = 2u * (uint32_t)tw;
    auto write_step = [&](int jb, bool tail) {
        uint32_t boff[kLR];
        int jj[kLR];
#pragma unroll
        for (int u = 0; u < kLR; ++u) {
            jj[u] = jb + u * kBT;
            boff[u] = (uint32_t)(!tail || jj[u] < n ? jj[u] : i0) * 4u;
        }
        float az[QB][kLR], ayz[QB][kLR];
        lean_dists<DZ, QB, kLR>(zy, n, q, boff, az, ayz);
#pragma unroll
        for (int r = 0; r < QB; ++r)
#pragma unroll
            for (int u = 0; u < kLR; ++u) {
                const int j = jj[u];
                const bool ok = r < nq && (!tail || j < n) && (uint32_t)(j + (tw - i0 - r)) > w2;
                const uint32_t k1 = key_of(ayz[r][u]), k2 = key_of(az[r][u]);
                if (ok && k1 < keep1[r]) {
                    const uint32_t pos = atomicAdd(&sm.h[r][k1], kInc1) & 0xffffu;
                    if (pos < m1) gstore(out1[r], pos, LEnt{ayz[r][u], j});
                }
                if (ok && k2 < keep2[r]) {
                    const uint32_t pos = atomicAdd(&sm.h[r][k2], kInc2) >> 16;
                    if (pos < m2) gstore(out2[r], pos, LEnt{az[r][u], j});
                }
            }
    };
    j0 = tid;
    for (; j0 < full; j0 += step) write_step(j0, false);
    if (j0 < n) write_step(j0, true);
    // lengths and the sentinels (as in list_build_kernel; they lie
    // past the kept entries, so no barrier is needed before them)
    for (int x = tid; x < QB * 2 * kListPad; x += kBT) {
        const int r = x / (2 * kListPad), w = (x / kListPad) & 1, u = x % kListPad;
        if (r >= nq) continue;
        const int64_t i = i0 + r;
        const uint32_t total = (uint32_t)(n - 1 - min((int)i, tw) - min(n - 1 - (int)i, tw));
        // the row's kept bins and rows, summed again from the waves' shares
        // in LDS (a register array indexed by r would go to scratch memory)
        uint32_t nb = 0, nr = 0;
#pragma unroll
        for (int v2 = 0; v2 < kBW; ++v2) {
            nb += sm.red[2 * r][v2];
            nr += sm.red[2 * r + 1][v2];
        }
        const uint32_t kbw = w == 0 ? nb & 0xffffu : nb >> 16, krw = w == 0 ? nr & 0xffffu : nr >> 16;
        const bool whole = krw == total || (kbw << kKeyShift) >= __float_as_uint(inf_f());
        const float sent = whole ? inf_f() : __uint_as_float((kbw << kKeyShift) + 1u);
        if (w == 0) S.l1[i * S.s1 + krw + u] = LEnt{sent, (int32_t)i};
        else S.l2[i * S.s2 + krw + u] = LEnt{sent, (int32_t)i};
        if (u == 0) S.len[2 * i + w] = (int32_t)krw;
    }
}

// ------------------------------------------------------------------ columns
// One thread per (set, row): the row's Z then Y coordinates into the set's
// contiguous column copy, so that the build addresses every column from one
// base pointer; the first threads also clear the launch's counters.
__global__ __launch_bounds__(kBlock) void list_zy_kernel(const ListLaunch L) {
    const int64_t g = bid_x() * kBlock + tid_x();
    // the launch's counters are cleared here too (a kernel launch fewer; the
    // grid covers at least kListCounterWords threads)
    if (g < kListCounterWords) L.counters[g] = 0u;
    if (g >= L.rows) return;
    const int t = find_job(L.row_off, L.n_sets, g);
    const ListSet &S = L.sets[t];
    const int64_t j = g - L.row_off[t], n = S.n;
    const int dy = S.dy, dz = S.dz;
    for (int c = 0; c < dz; ++c) S.zy[c * n + j] = S.cols[dy + c][j];
    for (int c = 0; c < dy; ++c) S.zy[(dz + c) * n + j] = S.cols[c][j];
}

// ------------------------------------------------------------------ ranks
// Columns ranked by value, ties by row index (the z column of a set counted
// by ranks, the X column of a job without Z or counted in a wavelet matrix).
// Every row's smaller rows are counted, n compares per row, split into
// kRankParts ranges of rows so that one column fills the chip: a wave takes 64
// rows and one range, whose values come 16 at a time through the scalar
// cache.  A second kernel adds the ranges' counts and scatters.  Beside the
// build at n = 10^4 the two take 75 us for two columns; one block's bitonic
// sort of one in LDS took 208 us, the same compares on 157 blocks 171 us.
constexpr int kRankThreads = 256;

__global__ __launch_bounds__(kRankThreads) void list_rank_part_kernel(const ListLaunch L) {
    const RankCol *C = L.rank_cols + __builtin_amdgcn_workgroup_id_z();
    Const<RankCol> *R = as_const(C);
    const int n = R->n;
    const int i0 = (int)bid_x() * kRankThreads;
    if (i0 >= n) return;
    __builtin_amdgcn_s_setprio(kBuildPrio);   // short, and the permutation waits for it beside the build
    const int part = (int)__builtin_amdgcn_workgroup_id_y();
    const int i = i0 + tid_x();
    const float *col = R->col;
    const float vi = gload(col, (uint32_t)min(i, n - 1));
    const int j0 = (int)((int64_t)n * part / kRankParts), j1 = (int)((int64_t)n * (part + 1) / kRankParts);
    Const<float> *v = as_const(col);
    int r = 0;
    // rows before the block's count with <=, rows after it with <; the rows
    // of the block itself by their index too
    const int a = max(j0, min(j1, i0)), b = max(a, min(j1, i0 + kRankThreads));
    constexpr int RU = 16;
    int j = j0;
    for (; j + RU <= a; j += RU) {
#pragma unroll
        for (int u = 0; u < RU; ++u) r += v[j + u] <= vi;
    }
    for (; j < a; ++j) r += v[j] <= vi;
    for (; j < b; ++j) r += (int)(v[j] < vi) | ((int)(v[j] == vi) & (int)(j < i));
    for (; j + RU <= j1; j += RU) {
#pragma unroll
        for (int u = 0; u < RU; ++u) r += v[j + u] < vi;
    }
    for (; j < j1; ++j) r += v[j] < vi;
    if (i < n) R->part[(int64_t)part * n + i] = r;
}

__global__ __launch_bounds__(kRankThreads) void list_rank_place_kernel(const ListLaunch L) {
    const RankCol &C = L.rank_cols[__builtin_amdgcn_workgroup_id_y()];
    const int n = C.n;
    const int i = (int)bid_x() * kRankThreads + tid_x();
    if (i >= n) return;
    int r = 0;
#pragma unroll
    for (int p = 0; p < kRankParts; ++p) r += C.part[(int64_t)p * n + i];
    // (columns that are not finite, which device calls do not check, may
    // repeat a rank, and then another names no row: readers of ord clamp what
    // they find, and the sums the word of a row that nobody counted)
    r = min(r, n - 1);
    if (C.rank) C.rank[i] = r;
    if (C.ord) C.ord[r] = i;
    C.sorted[r] = C.col[i];
    if (i < C.pad) {
        C.sorted[-1 - i] = -inf_f();
        C.sorted[n + i] = inf_f();
    }
    // (fewer rows than pads: the last thread writes the rest)
    if (i == n - 1)
        for (int q = n; q < C.pad; ++q) {
            C.sorted[-1 - q] = -inf_f();
            C.sorted[n + q] = inf_f();
        }
}

// ------------------------------------------------------------------ row order
// One block per list set with an order array: its rows grouped by Morton
// (Z-curve) cell of their first D <= 6 coordinates in the contiguous copy (Z
// columns, then Y).  Each coordinate is cut into 2^(12/D) equal steps between
// the column's minimum and maximum and the step indices' bits are interleaved
// from the top into a cell code below 2^12; a counting sort over the codes in
// LDS (histogram, block scan, scatter) then lists the rows cell by cell.  The
// cell codes stay in registers (a thread takes rows tid + u * 1024) and the
// block takes 17 KB of LDS, so it finds room beside the build's blocks.
// Rows next to each other in this order are near in (Y,Z) and share list
// entries.  The order of the rows within a cell follows the scatter's LDS
// atomics and may differ between launches: only the order in which the scan
// visits rows depends on it, not any result.
constexpr int kSortThreads = 1024;
constexpr int kOrderDims = 6;
constexpr int kOrderBits = 12;
constexpr int kOrderCells = 1 << kOrderBits;

__global__ __launch_bounds__(kSortThreads) void list_order_kernel(const ListLaunch L) {
    constexpr int NW = kSortThreads / 64, PER = kOrderCells / kSortThreads;
    constexpr int ROWS = kNoZSortMax / kSortThreads;   // rows per thread
    __shared__ uint32_t h[kOrderCells];
    __shared__ float red[2][kOrderDims][NW];
    __shared__ uint32_t wtot[NW];
    const ListSet &S = L.sets[bid_x()];
    const int n = S.n;
    if (!S.order || n > kNoZSortMax) return;    // the host sets no order array then
    const int tid = tid_x(), lane = tid & 63, w = tid >> 6;
    const int D = min(kOrderDims, S.dy + S.dz);
    const int bpd = kOrderBits / D;
    for (int c = tid; c < kOrderCells; c += kSortThreads) h[c] = 0;
    // column ranges
    float lo[kOrderDims], hi[kOrderDims];
#pragma unroll
    for (int q = 0; q < kOrderDims; ++q) {
        lo[q] = inf_f();
        hi[q] = -inf_f();
        if (q < D)
            for (int x = tid; x < n; x += kSortThreads) {
                const float c = S.zy[(int64_t)q * n + x];
                lo[q] = __builtin_fminf(lo[q], c);
                hi[q] = __builtin_fmaxf(hi[q], c);
            }
        lo[q] = wave_min(lo[q]);
        hi[q] = -wave_min(-hi[q]);
        if (lane == 0) {
            red[0][q][w] = lo[q];
            red[1][q][w] = hi[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kOrderDims; ++q) {
        lo[q] = red[0][q][0];
        hi[q] = red[1][q][0];
        for (int u = 1; u < NW; ++u) {
            lo[q] = __builtin_fminf(lo[q], red[0][q][u]);
            hi[q] = __builtin_fmaxf(hi[q], red[1][q][u]);
        }
    }
    // the steps are cut on halved values: differences of halved finite
    // floats cannot overflow, so no step of the cell code meets inf / inf
    const float steps = (float)(1 << bpd);
#pragma unroll
    for (int q = 0; q < kOrderDims; ++q) {
        lo[q] *= 0.5f;
        hi[q] *= 0.5f;
    }
    uint32_t code[ROWS];                        // each row's cell, computed once
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int x = tid + u * kSortThreads;
        code[u] = 0;
        if (x >= n) continue;
        uint32_t cell[kOrderDims];
#pragma unroll
        for (int q = 0; q < kOrderDims; ++q) {
            cell[q] = 0;
            if (q < D && hi[q] > lo[q]) {
                const float t = (0.5f * S.zy[(int64_t)q * n + x] - lo[q]) / (hi[q] - lo[q]) * steps;
                cell[q] = t >= 1.0f ? (t < steps ? (uint32_t)t : (uint32_t)steps - 1u) : 0u;
            }
        }
        uint32_t c = 0;
        for (int bit = bpd - 1; bit >= 0; --bit)
            for (int q = 0; q < D; ++q) c = c << 1 | ((cell[q] >> bit) & 1u);
        code[u] = c;              // < 2^(D * bpd) <= kOrderCells
        atomicAdd(&h[c], 1u);
    }
    __syncthreads();
    // exclusive offsets: each thread owns PER consecutive cells
    uint32_t loc[PER], sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        loc[u] = h[tid * PER + u];
        sum += loc[u];
    }
    uint32_t incl;
    block_scan<NW>(sum, incl, wtot);
    uint32_t run = incl - sum;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        h[tid * PER + u] = run;
        run += loc[u];
    }
    __syncthreads();
    // the counts add up to n, so every position is below n
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int x = tid + u * kSortThreads;
        if (x < n) S.order[atomicAdd(&h[code[u]], 1u)] = x;
    }
}

// ------------------------------------------------------------------ scan
// Each list row is followed by kListPad sentinel entries (row = self) whose
// key distance lies in the bucket that starts at the row's bound: the bound
// plus one unit in the last place (+inf for a whole list: nothing left out,
// or only rows at +inf).
// A step of kU entries that starts at or before the list's end, and the step
// after it, whose X values are loaded ahead, then need no bounds checks, and
// the last step of a list always ends on a sentinel, whose bucket-floor test
// (floor = bound >= radius) is exactly the
// condition under which the list decides the pair.  A sentinel that enters
// the k-NN list (bound + 1 ulp < k-th distance) leaves a radius above the
// bound, i.e. an undecided pair, as it should.
constexpr int kU = 8;   // the largest step
static_assert(2 * kU <= kListPad, "a step and the next must stay within the sentinels");

// A step's entries (distance, row) in scalar registers.
template <int NU>
struct Step {
    float d[NU];
    uint32_t j[NU];
};

template <int NU>
__device__ __forceinline__ void load_step(Const<uint32_t> *l, Step<NU> &s) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        s.d[u] = __uint_as_float(l[2 * u]);
        s.j[u] = l[2 * u + 1];
    }
}

// The step's values are needed here: keeps the compiler from sinking a step's
// load to the end of the loop that loads it ahead.
template <int NU>
__device__ __forceinline__ void pin_step(const Step<NU> &s) {
#pragma unroll
    for (int u = 0; u < NU; u += 4)
        asm volatile("" ::"s"(s.d[u]), "s"(s.j[u]), "s"(s.d[u + 1]), "s"(s.j[u + 1]), "s"(s.d[u + 2]), "s"(s.j[u + 2]),
                     "s"(s.d[u + 3]), "s"(s.j[u + 3]));
}

// Queue pair (i, e) of job jb, whose E estimates make n * E pairs, for the redo.
__device__ __forceinline__ void push_failed(const ListLaunch &L, int jb, int64_t i, int E, int e) {
    const uint32_t pos = atomicAdd(&L.counters[0], 1u);
    const int64_t at = L.fail_off[jb] + i * E + e;
    if (L.fail_wide) static_cast<uint64_t *>(L.failq)[pos] = (uint64_t)at;
    else static_cast<uint32_t *>(L.failq)[pos] = (uint32_t)at;
}

// The job of each lane's estimate, the t-th of the unit's class (lanes may
// belong to different jobs of one set).
struct LaneJob {
    int job, e;
};
__device__ __forceinline__ LaneJob lane_job(const ListLaunch &L, Const<ScanUnit> *U, int t) {
    const ClassJob *c = L.class_jobs + U->first;
    int lo = 0, hi = U->n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (c[mid].t0 <= t) lo = mid; else hi = mid - 1;
    }
    return LaneJob{c[lo].job, t - c[lo].t0};
}

// Wave-uniform helpers.
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
// The lane mask of one compare as the compare writes it (no round trip of the
// predicate through a vector register); masks are combined by the scalar unit.
__device__ __forceinline__ uint64_t cmp_mask(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int lowest(uint64_t m) { return __builtin_amdgcn_readfirstlane(__builtin_ctzll(m)); }
__device__ __forceinline__ float bcast(float v, int o) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), o));
}
__device__ __forceinline__ int bcast(int v, int o) { return __builtin_amdgcn_readlane(v, o); }
__device__ __forceinline__ const float *bcast(const float *v, int o) {
    const uint64_t a = (uint64_t)v;
    return (const float *)((uint64_t)(uint32_t)bcast((int)(a >> 32), o) << 32 | (uint32_t)bcast((int)a, o));
}

// A wave takes one row and one scan group of a class, a lane per estimate, so
// that a step's list entries are the same for all lanes: they come through
// the scalar cache into scalar registers, and the only vector loads are the
// X gathers, up to 256 adjacent bytes per entry (xt holds a group's estimates
// of one row in adjacent words) at a uniform base.  With the entries loaded per
// lane the broadcast loads (64 or 96 bytes a lane and step) took two thirds of
// the vector memory path's cycles, and the kernel held 79 vector registers
// instead of 36 (one X column, k <= 4, 8 entries a step; its 106 scalar
// registers are all there are, so the forms for many columns spill some).  Whole
// tests, before and after: N = 10^4, dz = 5, 201 estimates 662 -> 560 us;
// N = 30011, dz = 4, 101 estimates 3.00 -> 2.75 ms; 32 served requests
// 11.4 -> 9.8 ms; network of 8 targets, T = 3000 101 -> 86 ms; without Z
// (n_y was counted entry by entry in each lane) 3.07 -> 1.50 ms.
//
// A block is one wave: the waves of a block give their slots back together,
// and the slowest of four kept 4.6 of the 7 waves a SIMD could hold (5.6 with
// one).  The next step's X values and the entries of the step after it are
// loaded while a step is worked on.  The scan alone at N = 10^4, 201
// estimates: 299 -> 262 us, N = 30011 915 -> 783 us, the served mix 1.53 ->
// 1.30 ms a launch; a third of the cycles are vector instructions, the rest
// X gathers, and about 70 us at the end belong to the few longest waves.
//
// The 64 lanes stop at very different list positions (a few estimates of a
// row have radii far above the others).  Each phase runs with all lanes while
// more than `coop` of them still need entries (a lane past its own stop reads
// on without effect: no later entry is below its radius), then finishes the
// remaining lanes together, 64 list entries per step, one per lane, for each
// of them in turn.  Entries, distances and tests are the same, so the results
// are too.
//
// Phases: the k-NN radius over list 1; n_yz, the entries of list 1 below the
// radius (every such entry precedes the stop, so no X is gathered); n_z and
// n_xz over list 2.  Jobs counted by ranks leave after n_yz, jobs without Z
// take n_x from the sorted X column.
template <int KMAX, int DXM, int KU>
__global__ __launch_bounds__(kScanLanes) void list_scan_kernel(const ListLaunch L) {
    static_assert(KU <= kU, "two steps must stay within the sentinels");
    const int lane = tid_x();
    // XCD x's k-th block: the last of x's units whose first block is <= k
    const int64_t b = bid_x();
    const int x = (int)(b % kXcds);
    const int64_t k = b / kXcds;
    Const<int64_t> *xo = as_const(L.xcd_off) + (int64_t)x * (L.unit_t + 1);
    if (k >= xo[L.unit_t]) return;            // past x's blocks (no barrier in this kernel)
    int lo = 0, hi = L.unit_t - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (xo[mid] <= k) lo = mid; else hi = mid - 1;
    }
    Const<ScanUnit> *U = as_const(L.units) + (x + lo * kXcds);
    const int at = (int)(k - xo[lo]);
    const int jb = U->job, grp = U->group, il = U->row0 + at;
    const bool one_job = U->n_jobs == 1;
    Const<Job> *J = as_const(L.jobs) + jb;
    Const<ListSet> *S = as_const(L.sets) + J->set;
    const int n = J->n, E = J->T, dx = J->sdx;
    const bool swap = J->swap;
    const int i = S->order ? as_const(S->order)[il] : il;
    const int e0 = scan_group_first(grp, E), ne = scan_group_first(grp + 1, E) - e0;
    const bool live = lane < ne;
    const uint64_t livem = ballot(live);
    const int coop = L.coop_lanes;
    const LEnt *l1 = S->l1 + (int64_t)i * S->s1, *l2 = S->l2 + (int64_t)i * S->s2;

    // X of row j under this lane's estimate: group column + xtw j + lane
    const int64_t cs = (int64_t)scan_groups(E) * n * J->xtw;
    const float *xg = J->xt + (int64_t)grp * n * J->xtw;
    // (row4 in a vector register: the offset is then one multiply-add of 24 bits)
    const uint32_t loff = (uint32_t)min(lane, ne - 1) * 4u;
    uint32_t row4 = (uint32_t)J->xtw * 4u;
    asm volatile("" : "+v"(row4));
    auto xval = [&](int c, uint32_t j, uint32_t off) {
        return gload_b(xg + c * cs, (j & 0xffffffu) * (row4 & 0xffffffu) + off);
    };
    float xq[DXM];
    Unroll<0, DXM>::upto(dx, [&](auto cc) {
        constexpr int c = decltype(cc)::value;
        xq[c] = xval(c, (uint32_t)i, loff);
    });
    // the X values of a step's rows (all loads issued before any is used; the
    // first column of the next step is loaded while this one is worked on)
    auto gather = [&](const Step<KU> &s, float (&v)[KU]) {
#pragma unroll
        for (int u = 0; u < KU; ++u) v[u] = xval(0, s.j[u], loff);
    };
    // max-norm over the X columns between the lane's row and a step's rows
    // (the first cd of them)
    auto xdist = [&](const Step<KU> &s, const float (&v0)[KU], float (&d)[KU], int cd) {
#pragma unroll
        for (int u = 0; u < KU; ++u) d[u] = absdiff(xq[0], v0[u]);
        Unroll<1, DXM>::upto(cd, [&](auto cc) {
            constexpr int c = decltype(cc)::value;
            float v[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) v[u] = xval(c, s.j[u], loff);
#pragma unroll
            for (int u = 0; u < KU; ++u) d[u] = fmax_(d[u], absdiff(xq[c], v[u]));
        });
    };
    // the same between row i and one row per lane under lane o's estimate
    auto coop_xdist = [&](int o, uint32_t j, int cd) {
        const uint32_t oo = (uint32_t)o * 4u;
        float d = absdiff(bcast(xq[0], o), xval(0, j, oo));
        Unroll<1, DXM>::upto(cd, [&](auto cc) {
            constexpr int c = decltype(cc)::value;
            d = fmax_(d, absdiff(bcast(xq[c], o), xval(c, j, oo)));
        });
        return d;
    };

    // k-NN radius over list 1
    float top[KMAX];
    const int pad_front = KMAX - J->k;
#pragma unroll
    for (int m = 0; m < KMAX; ++m) top[m] = m < pad_front ? -inf_f() : inf_f();
    const int len1 = as_const(S->len)[2 * (int64_t)i];
    uint64_t open = livem;        // lanes whose radius needs later entries
    int64_t seen1 = 0, seen2 = 0; // list entries read by the pairs (statistics)
    int m1 = 0;
    {
        Const<uint32_t> *p = as_const(reinterpret_cast<const uint32_t *>(l1));
        Step<KU> cur, nxt;
        float v[KU];
        load_step(p, cur);
        load_step(p + 2 * KU, nxt);
        gather(cur, v);
        for (;;) {
            float vn[KU];
            Step<KU> nxt2;
            gather(nxt, vn);
            load_step(p + 2 * (m1 + 2 * KU), nxt2);
            __builtin_amdgcn_sched_barrier(0);
            float d[KU];
            xdist(cur, v, d, dx);
            float dmin = inf_f();
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                d[u] = fmax_(d[u], cur.d[u]);
                dmin = __builtin_fminf(dmin, d[u]);
            }
            // a distance not below the k-th leaves a lane's list as it is
            if (cmp_mask(dmin < top[KMAX - 1])) {
#pragma unroll
                for (int u = 0; u < KU; ++u) topk_insert<KMAX>(top, d[u]);
            }
            seen1 += (int64_t)__builtin_popcountll(open) * KU;
            open = livem & ~cmp_mask(bucket_floor(cur.d[KU - 1]) >= top[KMAX - 1]);
            m1 += KU;
            pin_step(nxt2);
            if (__builtin_popcountll(open) <= coop || m1 > len1) break;
            cur = nxt;
            nxt = nxt2;
#pragma unroll
            for (int u = 0; u < KU; ++u) v[u] = vn[u];
        }
    }
    uint64_t dec = livem & ~open; // decided lanes
    if (open && m1 <= len1) {     // (else the list is exhausted: the open lanes are undecided)
        const int end = len1 + kListPad;
        // the lanes share each chunk's entries; the next chunk's are loaded ahead
        LEnt nxt = l1[min(m1 + lane, end - 1)];
        for (int p = m1; open && p < end; p += 64) {
            const LEnt en = nxt;
            nxt = l1[min(p + 64 + lane, end - 1)];
            const float stop = bucket_floor(bcast(en.d, 63));
            for (uint64_t rest = open; rest; rest &= rest - 1) {
                const int o = lowest(rest);
                float d = fmax_(coop_xdist(o, (uint32_t)en.j, dx), en.d);
                if (p + lane >= end) d = inf_f();
                // +inf leaves the other lanes' lists as they are
                for (uint64_t cand = cmp_mask(d < bcast(top[KMAX - 1], o)); cand; cand &= cand - 1) {
                    const float dv = bcast(d, lowest(cand));
                    topk_insert<KMAX>(top, lane == o ? dv : inf_f());
                }
                seen1 += min(64, end - p);
            }
            const uint64_t done = open & cmp_mask(stop >= top[KMAX - 1]);
            dec |= done;
            open &= ~done;
        }
    }
    const float eps = top[KMAX - 1];

    // n_yz: list 1 below eps
    int cxz = 0, cyz = 0, cz = 0;
    if (!swap) {
        Const<uint32_t> *p = as_const(reinterpret_cast<const uint32_t *>(l1));
        open = dec;
        int m = 0;
        Step<KU> cur;
        load_step(p, cur);
        while (__builtin_popcountll(open) > coop && m <= len1) {
            Step<KU> nxt;
            load_step(p + 2 * (m + KU), nxt);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < KU; ++u) cyz += cur.d[u] < eps;
            open = dec & ~cmp_mask(bucket_floor(cur.d[KU - 1]) >= eps);
            m += KU;
            pin_step(nxt);
            cur = nxt;
        }
        const int end = len1 + kListPad;
        float nd = open ? l1[min(m + lane, end - 1)].d : 0.f;
        for (int c = m; open && c < end; c += 64) {
            const float d = nd;
            nd = l1[min(c + 64 + lane, end - 1)].d;
            const float stop = bucket_floor(bcast(d, 63));
            const uint64_t in = cmp_mask(c + lane < end);
            for (uint64_t rest = open; rest; rest &= rest - 1) {
                const int o = lowest(rest);
                const int q = __builtin_popcountll(in & cmp_mask(d < bcast(eps, o)));
                cyz += lane == o ? q : 0;
            }
            open &= ~cmp_mask(stop >= eps);
        }
    }

    // n_z and n_xz from list 2 below eps (every row with d_z < eps is listed
    // when eps <= its bound); a job of a set counted by ranks takes them from
    // the rank-count kernel.  A swapped job counts n_xz on its X list, with the
    // Z column alone
    const bool noz = J->dz == 0, ranked = J->er != nullptr;
    const int cd = swap ? 1 : dx;
    if (swap || (!noz && !ranked)) {
        const LEnt *lc = swap ? l1 : l2;
        const int len2 = swap ? len1 : as_const(S->len)[2 * (int64_t)i + 1];
        Const<uint32_t> *p = as_const(reinterpret_cast<const uint32_t *>(lc));
        const uint64_t want = dec;
        open = want;
        int m2 = 0;
        Step<KU> cur, nxt;
        float v[KU];
        load_step(p, cur);
        load_step(p + 2 * KU, nxt);
        gather(cur, v);
        while (__builtin_popcountll(open) > coop && m2 <= len2) {
            float vn[KU];
            Step<KU> nxt2;
            gather(nxt, vn);
            load_step(p + 2 * (m2 + 2 * KU), nxt2);
            __builtin_amdgcn_sched_barrier(0);
            float d[KU];
            xdist(cur, v, d, cd);
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                cz += cur.d[u] < eps;
                cxz += fmax_(d[u], cur.d[u]) < eps;
            }
            seen2 += (int64_t)__builtin_popcountll(open) * KU;
            open = want & ~cmp_mask(bucket_floor(cur.d[KU - 1]) >= eps);
            m2 += KU;
            pin_step(nxt2);
            cur = nxt;
            nxt = nxt2;
#pragma unroll
            for (int u = 0; u < KU; ++u) v[u] = vn[u];
        }
        dec = want & ~open;
        if (open && m2 <= len2) {
            const int end = len2 + kListPad;
            LEnt nx = lc[min(m2 + lane, end - 1)];
            for (int c = m2; open && c < end; c += 64) {
                const LEnt en = nx;
                nx = lc[min(c + 64 + lane, end - 1)];
                const float stop = bucket_floor(bcast(en.d, 63));
                const uint64_t in = cmp_mask(c + lane < end);
                for (uint64_t rest = open; rest; rest &= rest - 1) {
                    const int o = lowest(rest);
                    const float pe = bcast(eps, o);
                    const float dv = coop_xdist(o, (uint32_t)en.j, cd);
                    const int qz = __builtin_popcountll(in & cmp_mask(en.d < pe));
                    const int qxz = __builtin_popcountll(in & cmp_mask(fmax_(dv, en.d) < pe));
                    cz += lane == o ? qz : 0;
                    cxz += lane == o ? qxz : 0;
                    seen2 += min(64, end - c);
                }
                const uint64_t done = open & cmp_mask(stop >= eps);
                dec |= done;
                open &= ~done;
            }
        }
    }
    const bool decided = (dec >> lane) & 1u;
    // the lane's own job Jl, number jl, and its estimate e there
    auto finish = [&](auto *Jl, int jl, int e) {
        if (noz && decided) {
            // Without Z: n_z is the number of rows outside the window; n_x counts
            // the rows j != i with |x_j - x_i| < eps.  The permuted values x_j run
            // over the job's X column, so that count is the range of the sorted
            // column around x_i: the s with -eps < fl(xs[s] - x_i) < eps
            // (fl(. - x_i) is monotone), less row i itself and the rows of its
            // Theiler window.
            const int w = J->theiler;
            cz = n - 1 - min(i, w) - min(n - 1 - i, w);
            const float xv = xq[0];
            const float *xs = Jl->xs;
            int lo2 = 0, hi2 = n;
            while (lo2 < hi2) {
                const int mid = (lo2 + hi2) >> 1;
                if (gload(xs, mid) - xv > -eps) hi2 = mid; else lo2 = mid + 1;
            }
            const int first = lo2;
            hi2 = n;
            while (lo2 < hi2) {
                const int mid = (lo2 + hi2) >> 1;
                if (gload(xs, mid) - xv >= eps) hi2 = mid; else lo2 = mid + 1;
            }
            cxz = lo2 - first - (0.f < eps ? 1 : 0);
            for (int j = max(0, i - w); j <= min(n - 1, i + w); ++j)
                if (j != i && absdiff(xv, xval(0, (uint32_t)j, loff)) < eps) --cxz;
        }
        const int64_t at_e = (int64_t)e * n + i;
        // a ranked pair hands its radius and n_yz over, by the rank of its row;
        // a swapped one its radius and n_xz, by the row it stands at (its
        // count kernel queues it for the redo)
        if (ranked)
            Jl->er[(int64_t)e * n + (swap ? i : as_const(J->zrank)[i])] =
                decided ? ((uint64_t)(uint32_t)(swap ? cxz : cyz) << 32) | __float_as_uint(eps) : kRankNone;
        if (!decided && !swap) {
            push_failed(L, jl, i, Jl->n_est, e);
        } else if (decided && !ranked) {
            Jl->pk[at_e] = pack_counts(cxz, cyz, cz);
            if (Jl->eps) Jl->eps[at_e] = eps;
            if (Jl->cnt) {
                Jl->cnt[((int64_t)e * 3 + 0) * n + i] = cxz;
                Jl->cnt[((int64_t)e * 3 + 1) * n + i] = cyz;
                Jl->cnt[((int64_t)e * 3 + 2) * n + i] = cz;
            }
        }
    };
    if (live) {
        if (one_job) {
            finish(J, jb, e0 + lane);
        } else {
            const LaneJob lj = lane_job(L, U, e0 + lane);
            finish(L.jobs + lj.job, lj.job, lj.e);
        }
        if (L.stats && lane == 0) {
            const int slot = (int)(b & (kListStatSlots - 1));
            unsigned long long *st =
                reinterpret_cast<unsigned long long *>(L.counters + kListStatWord + slot * kListStatStride);
            atomicAdd(&st[0], (unsigned long long)seen1);
            atomicAdd(&st[1], (unsigned long long)seen2);
        }
    }
}

// ------------------------------------------------------------------ walk
// Jobs without Z, with one X and one Y column: the rows nearest to row i in y
// are the ranks next to its own, so the k-NN radius needs no lists.  As in the
// scan a wave takes one row (by rank in y) and one scan group of estimates; it
// walks outwards, kWalkU ranks at a time on the side whose next rank is nearer
// in y, until that distance reaches the k-th (for all but kWalkFew lanes; those
// go on one after the other, 64 ranks per step).  xt's rows are in rank order,
// so a step's X values are adjacent rows, and neighbouring waves read the same
// ones; for the last lanes xr holds an estimate's X by rank.  Every pair is
// decided.  n_x and n_y are two binary searches each, on the sorted columns in
// LDS (one or two blocks per estimate).  At N = 9995, 201 estimates the lists of every
// row (800 MB) took 0.53 ms to build and 0.62 ms to scan (1.22 ms for
// the whole test, 0.51 this way): the walk takes 0.33 ms, bound by the waves'
// chains of dependent loads, the counts 43 us.
constexpr int kWalkU = 8;
constexpr int kWalkFew = 16;
static_assert(2 * kWalkU <= kWalkPad, "a step past the end stays within the pads");

// MANY: some unit's lanes belong to several jobs (an instance of its own: with
// both cases in one the kernel held 76 registers instead of 66, 6 waves per
// SIMD instead of 7, and took 5% longer).
template <int KMAX, bool WIN, bool MANY>
__global__ __launch_bounds__(kScanLanes) void list_walk_kernel(const ListLaunch L) {
    const int lane = tid_x();
    const int64_t b = bid_x();
    const int x = (int)(b % kXcds);
    const int64_t k = b / kXcds;
    Const<int64_t> *xo = as_const(L.walk_xcd_off) + (int64_t)x * (L.walk_unit_t + 1);
    if (k >= xo[L.walk_unit_t]) return;
    int lo = 0, hi = L.walk_unit_t - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (xo[mid] <= k) lo = mid; else hi = mid - 1;
    }
    Const<ScanUnit> *U = as_const(L.walk_units) + (x + lo * kXcds);
    const int r = U->row0 + (int)(k - xo[lo]), grp = U->group;
    Const<Job> *J = as_const(L.jobs) + U->job;
    Const<ListSet> *S = as_const(L.sets) + J->rset;
    const int n = J->n, E = J->T, w = J->theiler;
    const float *ysg = S->ys;
    Const<float> *ys = as_const(ysg);
    Const<int32_t> *yord = as_const(S->yord);
    const int i = min(max(yord[r], 0), n - 1);
    const int e0 = scan_group_first(grp, E), ne = scan_group_first(grp + 1, E) - e0;
    const bool live = lane < ne;
    const uint64_t livem = ballot(live);
    // rank q's row of the group, q from -kWalkPad to n + kWalkPad - 1 (the pads
    // hold 0 and are +inf away in y)
    const float *xg = J->xt + ((int64_t)grp * (n + 2 * kWalkPad) + kWalkPad) * kScanLanes;
    const uint32_t loff = (uint32_t)min(lane, ne - 1) * 4u;
    const float xq = gload_b(xg + (int64_t)r * kScanLanes, loff), yq = ys[r];
    float top[KMAX];
    const int pad_front = KMAX - J->k;
#pragma unroll
    for (int m = 0; m < KMAX; ++m) top[m] = m < pad_front ? -inf_f() : inf_f();

    // ranks a .. a+kWalkU-1: y, X and, with a window, the rows
    struct Blk {
        float y[kWalkU], v[kWalkU];
        int j[kWalkU];
    };
    auto fetch = [&](int a, Blk &B) {
        const float *xa = xg + (int64_t)a * kScanLanes;
#pragma unroll
        for (int u = 0; u < kWalkU; ++u) {
            B.y[u] = ys[a + u];
            B.v[u] = gload_b(xa, loff + u * (kScanLanes * 4u));
            if (WIN) B.j[u] = yord[min(max(a + u, 0), n - 1)];
        }
    };
    auto use = [&](const Blk &B) {
        float d[kWalkU], dmin = inf_f();
#pragma unroll
        for (int u = 0; u < kWalkU; ++u) {
            d[u] = fmax_(absdiff(xq, B.v[u]), absdiff(B.y[u], yq));
            if (WIN && abs(B.j[u] - i) <= w) d[u] = inf_f();
            dmin = __builtin_fminf(dmin, d[u]);
        }
        if (cmp_mask(dmin < top[KMAX - 1])) {
#pragma unroll
            for (int u = 0; u < kWalkU; ++u) topk_insert<KMAX>(top, d[u]);
        }
    };
    // the next ranks: lt - 1 downwards, rt upwards
    int lt = r, rt = r + 1;
    uint64_t open = livem, seen = 0;
    {
        Blk bl, br;
        fetch(lt - kWalkU, bl);
        fetch(rt, br);
        for (;;) {
            const float dl = absdiff(bl.y[kWalkU - 1], yq), dr = absdiff(br.y[0], yq);
            const float dn = __builtin_fminf(dl, dr);
            open = livem & ~cmp_mask(dn >= top[KMAX - 1]);
            // (no rank is left: every radius stands.  The steps go by the
            // indices, so that values that are not finite end the walk too)
            if (lt <= 0 && rt >= n) open = 0;
            if (__builtin_popcountll(open) <= kWalkFew) break;
            seen += (uint64_t)__builtin_popcountll(open) * kWalkU;
            Blk cur;
            if (lt > 0 && (rt >= n || cmp_mask(dl <= dr))) {
                cur = bl;
                lt -= kWalkU;
                fetch(lt - kWalkU, bl);
            } else {
                cur = br;
                rt += kWalkU;
                fetch(rt, br);
            }
            use(cur);
        }
    }
    // X by rank of the lane's estimate, and its radii
    const float *xrow = nullptr;
    float *rad = nullptr;
    if constexpr (MANY) {
        const LaneJob lj = lane_job(L, U, e0 + min(lane, ne - 1));
        xrow = L.jobs[lj.job].xr + (int64_t)lj.e * n;
        rad = L.jobs[lj.job].rad + (int64_t)lj.e * n;
    }
    while (open && (lt > 0 || rt < n)) {
        const float dl = lt > 0 ? absdiff(ys[lt - 1], yq) : inf_f(), dr = rt < n ? absdiff(ys[rt], yq) : inf_f();
        const float dn = __builtin_fminf(dl, dr);
        open &= ~cmp_mask(dn >= top[KMAX - 1]);
        if (!open) break;
        const bool left = lt > 0 && (rt >= n || cmp_mask(dl <= dr) != 0);
        const int q = left ? lt - 1 - lane : rt + lane, qc = min(max(q, 0), n - 1);
        float dy = absdiff(gload(ysg, (uint32_t)qc), yq);
        if (q < 0 || q >= n) dy = inf_f();
        if (WIN && abs(S->yord[qc] - i) <= w) dy = inf_f();
        if (left) lt -= 64; else rt += 64;
        for (uint64_t rest = open; rest; rest &= rest - 1) {
            const int o = lowest(rest);
            const float *xr = MANY ? bcast(xrow, o) : J->xr + (int64_t)(e0 + o) * n;
            const float d = fmax_(absdiff(bcast(xq, o), gload(xr, (uint32_t)qc)), dy);
            // +inf leaves the other lanes' lists as they are
            for (uint64_t cand = cmp_mask(d < bcast(top[KMAX - 1], o)); cand; cand &= cand - 1) {
                const float dv = bcast(d, lowest(cand));
                topk_insert<KMAX>(top, lane == o ? dv : inf_f());
            }
            seen += 64;
        }
    }
    if (!MANY) rad = J->rad + (int64_t)(e0 + lane) * n;
    if (live) rad[i] = top[KMAX - 1];
    if (L.stats && lane == 0) {
        const int slot = (int)(b & (kListStatSlots - 1));
        unsigned long long *st =
            reinterpret_cast<unsigned long long *>(L.counters + kListStatWord + slot * kListStatStride);
        atomicAdd(&st[0], (unsigned long long)seen);
    }
}

__global__ __launch_bounds__(kRowThreads) void list_walk_count_kernel(const ListLaunch L) {
    extern __shared__ uint64_t wv_lds[];
    const int64_t g = bid_x();
    const int cut = (int)__builtin_amdgcn_workgroup_id_y();
    const int jb = __builtin_amdgcn_readfirstlane(find_job(L.est_off, L.n_jobs, g));
    Const<Job> *J = as_const(L.jobs) + jb;
    if (!J->walk) return;
    Const<ListSet> *S = as_const(L.sets) + J->rset;
    const int n = J->n, w = J->theiler, tid = tid_x();
    const int64_t e = g - as_const(L.est_off)[jb];
    float *xs = reinterpret_cast<float *>(wv_lds), *ys = xs + n;
    const float *xsg = J->xs, *ysg = S->ys, *yc = J->cols[1], *xe = J->xp + e * n;
    for (int q = tid; q < n; q += L.walk_threads) {
        xs[q] = gload(xsg, (uint32_t)q);
        ys[q] = gload(ysg, (uint32_t)q);
    }
    __syncthreads();
    // rows of a sorted column within eps of v: (s - v) > -eps and < eps
    auto range = [&](const float *s, float v, float eps) {
        int p = 0, q = n;
        while (p < q) {
            const int m = (p + q) >> 1;
            if (s[m] - v > -eps) q = m; else p = m + 1;
        }
        const int first = p;
        q = n;
        while (p < q) {
            const int m = (p + q) >> 1;
            if (s[m] - v >= eps) q = m; else p = m + 1;
        }
        return p - first;
    };
    const int c0 = (int)((int64_t)n * cut / L.est_cuts), c1 = (int)((int64_t)n * (cut + 1) / L.est_cuts);
    for (int i = c0 + tid; i < c1; i += L.walk_threads) {
        const float eps = J->rad[e * n + i], xq = gload(xe, (uint32_t)i), yq = gload(yc, (uint32_t)i);
        // the row itself is in both ranges exactly when eps > 0
        const int own = 0.f < eps ? 1 : 0;
        int nx = range(xs, xq, eps) - own, ny = range(ys, yq, eps) - own;
        for (int j = max(0, i - w); j <= min(n - 1, i + w); ++j) {
            if (j == i) continue;
            nx -= absdiff(xq, gload(xe, (uint32_t)j)) < eps;
            ny -= absdiff(yq, gload(yc, (uint32_t)j)) < eps;
        }
        const int nz = n - 1 - min(i, w) - min(n - 1 - i, w);
        J->pk[e * n + i] = pack_counts(nx, ny, nz);
        if (J->eps) J->eps[e * n + i] = eps;
        if (J->cnt) {
            J->cnt[(e * 3 + 0) * n + i] = nx;
            J->cnt[(e * 3 + 1) * n + i] = ny;
            J->cnt[(e * 3 + 2) * n + i] = nz;
        }
    }
}

// ------------------------------------------------------------------ rank counts
// Counts of the pairs of a set with one Z column.  The rows within the
// radius of row i in z are the ranks [lo, hi) with fl(zs[r] - z_i) > -eps
// and fl(zs[r] - z_i) < eps (two binary searches), so n_z = hi - lo, and
// n_yz, n_xz are the rows of that range within eps in y, in x: a wave takes
// 64 pairs (64 ranks, one estimate), finds their ranges lane by lane, then
// counts each pair in turn with all lanes, 64 ranks per step (coalesced
// loads of y and of the estimate's permuted x in rank order, ballot counts).
// The pair's own row and the rows of its Theiler window are taken out
// afterwards.  Same tests as the definition, so the same counts, and every
// pair is decided.
template <int DXM>
__global__ __launch_bounds__(kRankThreads) void list_rank_count_kernel(const ListLaunch L) {
    const int lane = tid_x() & 63;
    const int64_t w = (int64_t)bid_x() * (kRankThreads / 64) +
                      (int)__builtin_amdgcn_readfirstlane((uint32_t)tid_x() >> 6);
    if (w >= L.rank_waves) return;
    const int jb = find_job(L.rank_off, L.n_jobs, w);
    const Job &J = L.jobs[jb];
    const ListSet &S = L.sets[J.rset];
    const int n = J.n, dx = J.dx;
    const int nt = (n + 63) / 64;
    const int64_t loc = w - L.rank_off[jb];
    const int e = (int)(loc / nt);
    const int r = (int)(loc - (int64_t)e * nt) * 64 + lane;
    const int rr = min(r, n - 1);
    // (ranks and rows are clamped to the set: with inputs that are not finite,
    // which device calls do not check, a rank may name no row)
    const int i = min(max(S.zord[rr], 0), n - 1);
    const uint64_t word = J.er[(int64_t)e * n + rr];
    const float eps = __uint_as_float((uint32_t)word);
    const bool ok = r < n && eps >= 0.f;      // -1: the pair is in the redo queue
    const float *zs = S.zs;
    const float *xr = J.xr + (int64_t)e * dx * n;
    const float zq = zs[rr];
    float xq[DXM];
#pragma unroll
    for (int c = 0; c < DXM; ++c) xq[c] = c < dx ? xr[(int64_t)c * n + rr] : 0.f;
    int lo = 0, hi = n;
    {
        int a = 0, b = n;
        while (a < b) {
            const int m = (a + b) >> 1;
            if (zs[m] - zq > -eps) b = m; else a = m + 1;
        }
        lo = a;
        b = n;
        while (a < b) {
            const int m = (a + b) >> 1;
            if (zs[m] - zq >= eps) b = m; else a = m + 1;
        }
        hi = a;
    }
    int mx = 0, mz = 0;
    int64_t ent = 0;
    for (uint64_t todo = ballot(ok); todo; todo &= todo - 1) {
        const int o = lowest(todo);
        const int plo = bcast(lo, o), phi = bcast(hi, o), pi = bcast(i, o);
        const float pe = bcast(eps, o);
        float px[DXM];
#pragma unroll
        for (int c = 0; c < DXM; ++c) px[c] = bcast(xq[c], o);
        int cx = 0;
        // kRankU steps per iteration, their loads issued together (a pair's
        // steps would otherwise wait for their loads one after another): the
        // network-inference workload ran 3% faster than with one step per
        // iteration; buffer loads over the range (no clamp, a lane mask
        // instead) were 6% slower than either
        constexpr int kRankU = DXM == 1 ? 4 : 1;
        for (int q = plo; q < phi; q += 64 * kRankU) {
            bool in[kRankU];
            uint32_t bo[kRankU];
            float x0[kRankU];
#pragma unroll
            for (int u = 0; u < kRankU; ++u) {
                const int m = q + 64 * u + lane;
                in[u] = m < phi;
                // byte offsets from the wave-uniform bases: the loads take
                // no 64-bit address arithmetic
                bo[u] = (uint32_t)(in[u] ? m : phi - 1) * 4u;
                x0[u] = gload_b(xr, bo[u]);
            }
#pragma unroll
            for (int u = 0; u < kRankU; ++u) {
                float d = absdiff(x0[u], px[0]);
                Unroll<1, DXM>::upto(dx, [&](auto cc) {
                    constexpr int c = decltype(cc)::value;
                    d = fmax_(d, absdiff(gload_b(xr + (int64_t)c * n, bo[u]), px[c]));
                });
                // the masks of single compares, combined by the scalar unit
                const uint64_t inm = cmp_mask(in[u]);
                cx += __builtin_popcountll(inm & cmp_mask(d < pe));
            }
        }
        int cz = phi - plo;
        // without a Theiler window only the pair's own row is taken out: it
        // is in the range and within eps in y and x exactly when eps > 0
        // (its differences are all 0), else the range is empty
        const int w0 = max(0, pi - J.theiler), w1 = min(n - 1, pi + J.theiler);
        if (J.theiler == 0) {
            const int own = pe > 0.f ? 1 : 0;
            cz -= own;
            cx -= own;
        } else {
            for (int j = w0 + lane; j - lane <= w1; j += 64) {
                const bool inw = j <= w1;
                const int rj = min(max(S.zrank[inw ? j : w1], 0), n - 1);
                const bool inr = inw && rj >= plo && rj < phi;
                float d = absdiff(xr[rj], px[0]);
                Unroll<1, DXM>::upto(dx, [&](auto cc) {
                    constexpr int c = decltype(cc)::value;
                    d = fmax_(d, absdiff(xr[(int64_t)c * n + rj], px[c]));
                });
                cz -= __builtin_popcountll(ballot(inr));
                cx -= __builtin_popcountll(ballot(inr && d < pe));
            }
        }
        ent += phi - plo;
        if (lane == o) {
            mx = cx;
            mz = cz;
        }
    }
    if (ok) {
        const int my = (int)(word >> 32);     // n_yz, from the scan
        J.pk[(int64_t)e * n + i] = pack_counts(mx, my, mz);
        if (J.eps) J.eps[(int64_t)e * n + i] = eps;
        if (J.cnt) {
            J.cnt[((int64_t)e * 3 + 0) * n + i] = mx;
            J.cnt[((int64_t)e * 3 + 1) * n + i] = my;
            J.cnt[((int64_t)e * 3 + 2) * n + i] = mz;
        }
    }
    if (L.stats && lane == 0) {
        const int slot = (int)(w & (kListStatSlots - 1));
        unsigned long long *st =
            reinterpret_cast<unsigned long long *>(L.counters + kListStatWord + slot * kListStatStride);
        atomicAdd(&st[1], (unsigned long long)ent);
    }
}

// ------------------------------------------------------------------ wavelet counts
// n_xz of the pairs of a set with one Z column, one X column and no Theiler
// window: the rows of ranks [lo, hi) in z whose x lies within eps of x_i are,
// in ranks of x, those in [a, b) (two more binary searches, on the job's
// sorted X).  Of a swapped job the scan has counted n_xz, and the same
// structure over y (its sequence is the same for all estimates) gives n_yz.
// One block per estimate keeps the wavelet matrix of the sequence
// "rank of x by rank of z" in LDS: per bit of the rank, from the top, a bit
// vector with running counts, the sequence stably partitioned by that bit
// from level to level.  A pair's count then takes one walk over the levels
// for a and one for b, a lane per pair, instead of reading the hi - lo rows
// (on average 740 at N = 10^4) with all lanes over one pair after another:
// 423 -> 160 us at N = 9995, 201 estimates (the whole test 1.06 -> 0.71 ms).
constexpr int kWvWaves = kRowThreads / 64;
constexpr int kWvBits = 16;

struct WvNode {
    uint32_t bits, ones;                      // 32 elements' bits, ones before them
};

__device__ __forceinline__ int wv_bits(int n) { return 32 - __builtin_clz((unsigned)n); }   // n < 2^bits

__global__ __launch_bounds__(kRowThreads) void list_wavelet_kernel(const ListLaunch L) {
    extern __shared__ uint64_t wv_lds[];
    __shared__ int wtot[kWvWaves];
    __shared__ int zeros[kWvBits];
    const int64_t g = bid_x();
    const int jb = __builtin_amdgcn_readfirstlane(find_job(L.est_off, L.n_jobs, g));
    Const<Job> *J = as_const(L.jobs) + jb;
    if (!J->xw) return;                       // counted elsewhere (uniform in the block)
    Const<ListSet> *S = as_const(L.sets) + J->rset;
    const bool swap = J->swap;
    const int n = J->n, e = (int)(g - as_const(L.est_off)[jb]);
    const int tid = tid_x(), lane = tid & 63, nt = L.wavelet_threads, waves = nt / 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (n + 63) / 64, per = (nblk + waves - 1) / waves;
    if (tid < kWvWaves) wtot[tid] = 0;        // (of the waves that a small block lacks)
    const int nb = wv_bits(n), stride = 2 * nblk + 1;
    WvNode *node = reinterpret_cast<WvNode *>(wv_lds);
    // the sequence, from one buffer into the other level by level
    uint16_t *sa = reinterpret_cast<uint16_t *>(node + nb * stride), *sb = sa + n;
    float *xs = reinterpret_cast<float *>(sa);
    // source row of each row and rank of each source row, then the sequence
    const uint16_t *src = J->xw + (int64_t)e * n;
    uint16_t *xw = J->xw + (int64_t)(J->n_est + e) * n;
    const int32_t *xrank = swap ? S->yrank : J->xrank;
    for (int q = tid; q < n; q += nt) {
        sa[q] = src[q];
        sb[q] = (uint16_t)xrank[q];
    }
    __syncthreads();
    const int32_t *zord = S->zord;
    const int blk0 = wave * per, blk1 = min(nblk, blk0 + per);
    for (int blk = blk0; blk < blk1; ++blk) {
        const int p = blk * 64 + lane;
        if (p < n) {
            const int i = min(max(zord[p], 0), n - 1);
            xw[p] = sb[swap ? i : min((int)sa[i], n - 1)];
        }
    }
    __syncthreads();
    for (int blk = blk0; blk < blk1; ++blk) {
        const int p = blk * 64 + lane;
        if (p < n) sa[p] = xw[p];
    }
    __syncthreads();
    for (int lev = 0; lev < nb; ++lev) {
        const int sh = nb - 1 - lev;
        WvNode *nd = node + lev * stride;
        int run = 0;
        for (int blk = blk0; blk < blk1; ++blk) {
            const int p = blk * 64 + lane;
            run += __builtin_popcountll(cmp_mask(p < n && ((sa[p] >> sh) & 1)));
        }
        if (lane == 0) wtot[wave] = run;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kWvWaves; ++w) {
            before += w < wave ? wtot[w] : 0;
            total += wtot[w];
        }
        const int z = n - total;
        if (tid == 0) {
            zeros[lev] = z;
            nd[2 * nblk] = WvNode{0u, (uint32_t)total};
        }
        for (int blk = blk0; blk < blk1; ++blk) {
            const int p = blk * 64 + lane;
            const uint32_t v = p < n ? sa[p] : 0u;
            const bool one = (v >> sh) & 1u;
            const uint64_t m = cmp_mask(one);
            const uint32_t mlo = (uint32_t)m, mhi = (uint32_t)(m >> 32);
            if (lane == 0) {
                nd[2 * blk] = WvNode{mlo, (uint32_t)before};
                nd[2 * blk + 1] = WvNode{mhi, (uint32_t)(before + __builtin_popcount(mlo))};
            }
            const int r1 = before + (int)__builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
            if (p < n) sb[one ? z + r1 : p - r1] = (uint16_t)v;
            before += __builtin_popcountll(m);
        }
        __syncthreads();
        uint16_t *t = sa;
        sa = sb;
        sb = t;
    }
    // the sorted X column takes the sequence's place
    const float *xsg = swap ? S->ys : J->xs;
    for (int q = tid; q < n; q += nt) xs[q] = gload(xsg, (uint32_t)q);
    __syncthreads();

    const float *zs = S->zs;
    const uint64_t *er = J->er + (int64_t)e * n;
    auto ones = [&](const WvNode *nd, int p) {
        const WvNode w = nd[p >> 5];
        return (int)w.ones + __builtin_popcount(w.bits & ((1u << (p & 31)) - 1u));
    };
    for (int r = tid; r < n; r += nt) {
        const int i = min(max(zord[r], 0), n - 1);
        const int m0 = swap ? min((int)src[i], n - 1) : r;
        const uint64_t word = er[m0];
        const float eps = __uint_as_float((uint32_t)word);
        const float zq = gload(zs, (uint32_t)r), xq = xs[min((int)xw[r], n - 1)];
        // ranks of z within eps, then ranks of x
        int lo, hi, a, b;
        {
            int p = 0, q = n;
            while (p < q) {
                const int m = (p + q) >> 1;
                if (gload(zs, (uint32_t)m) - zq > -eps) q = m; else p = m + 1;
            }
            lo = p;
            q = n;
            while (p < q) {
                const int m = (p + q) >> 1;
                if (gload(zs, (uint32_t)m) - zq >= eps) q = m; else p = m + 1;
            }
            hi = p;
            p = 0;
            q = n;
            while (p < q) {
                const int m = (p + q) >> 1;
                if (xs[m] - xq > -eps) q = m; else p = m + 1;
            }
            a = p;
            q = n;
            while (p < q) {
                const int m = (p + q) >> 1;
                if (xs[m] - xq >= eps) q = m; else p = m + 1;
            }
            b = p;
        }
        int la = lo, ra = hi, lb = lo, rb = hi, cnt = 0;
        for (int lev = 0; lev < nb; ++lev) {
            const WvNode *nd = node + lev * stride;
            const int z = zeros[lev], sh = nb - 1 - lev;
            const int la1 = ones(nd, la), ra1 = ones(nd, ra), lb1 = ones(nd, lb), rb1 = ones(nd, rb);
            if ((b >> sh) & 1) {
                cnt += (rb - rb1) - (lb - lb1);
                lb = z + lb1;
                rb = z + rb1;
            } else {
                lb -= lb1;
                rb -= rb1;
            }
            if ((a >> sh) & 1) {
                cnt -= (ra - ra1) - (la - la1);
                la = z + la1;
                ra = z + ra1;
            } else {
                la -= la1;
                ra -= ra1;
            }
        }
        if (!(eps >= 0.f)) {                  // in the redo queue, a swapped pair from here
            if (swap) {
                push_failed(L, jb, i, J->n_est, e);
            }
            continue;
        }
        // the pair's own row is in the range and within eps exactly when eps > 0
        const int own = eps > 0.f ? 1 : 0;
        const int other = (int)(word >> 32), ct = cnt - own;
        const int cxz = swap ? other : ct, cyz = swap ? ct : other;
        J->pk[(int64_t)e * n + i] = pack_counts(cxz, cyz, hi - lo - own);
        if (J->eps) J->eps[(int64_t)e * n + i] = eps;
        if (J->cnt) {
            J->cnt[((int64_t)e * 3 + 0) * n + i] = cxz;
            J->cnt[((int64_t)e * 3 + 1) * n + i] = cyz;
            J->cnt[((int64_t)e * 3 + 2) * n + i] = hi - lo - own;
        }
    }
}

// ------------------------------------------------------------------ fallback
// The undecided (row, estimate) pairs, over every other row as in the
// definition: each thread keeps the KMAX smallest distances of its rows, k
// pops of the minimum give the radius, then the threads count and a sum adds
// the counts.  Two shapes, chosen from the queue length (a scalar, so the
// choice is uniform): a few pairs (the usual case, e.g. 244 of 2 million on
// C2) take a whole 1024-thread block each, which keeps the latency of a pair
// short; many pairs (lists short for the data) take one wave each, with no
// block synchronisation, for throughput.
constexpr int kFbBatch = 12;
constexpr int kFbThreads = 1024;
constexpr int kFbWaves = kFbThreads / 64;
constexpr uint32_t kFbBlockModeMax = 2048;   // queue length up to which a pair gets a block

struct FbPair {
    const Job *J;
    int i, e, n, dx, dy, dz;
};

__device__ __forceinline__ FbPair fb_pair(const ListLaunch &L, uint32_t it) {
    const int64_t item = L.fail_wide ? (int64_t) static_cast<const uint64_t *>(L.failq)[it]
                                     : (int64_t) static_cast<const uint32_t *>(L.failq)[it];
    const int jb = find_job(L.fail_off, L.n_jobs, item);
    const int64_t r = item - L.fail_off[jb];
    FbPair p;
    p.J = &L.jobs[jb];
    const int E = p.J->n_est;
    p.i = (int)(r / E);
    p.e = (int)(r - (int64_t)p.i * E);
    p.n = p.J->n;
    p.dx = p.J->dx;
    p.dy = p.J->dy;
    p.dz = p.J->dz;
    return p;
}

// distances of rows j0, j0 + step, ... (kFbBatch of them; rows inside row i's
// Theiler window and rows past the end get +inf in every subspace)
__device__ __forceinline__ void fb_dists(const FbPair &p, int j0, int step, float (&ax)[kFbBatch],
                                         float (&ay)[kFbBatch], float (&az)[kFbBatch]) {
    const Job &J = *p.J;
    int jj[kFbBatch];
#pragma unroll
    for (int u = 0; u < kFbBatch; ++u) {
        const int j = j0 + u * step;
        jj[u] = j < p.n ? j : p.i;
        ax[u] = ay[u] = az[u] = 0.f;
    }
    for (int c = 0; c < p.dx; ++c) {
        // the estimate-major copy: consecutive rows are adjacent words (in the
        // transposed one they are n_est words apart, a page apart in big launches)
        const float *xe = J.xp + ((int64_t)p.e * p.dx + c) * p.n;
        const float q = gload(xe, (uint32_t)p.i);
        float v[kFbBatch];
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) v[u] = gload(xe, (uint32_t)jj[u]);
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) ax[u] = fmax_(ax[u], absdiff(q, v[u]));
    }
    const float *const *yc = J.cols + p.dx;
    for (int c = 0; c < p.dy; ++c) {
        const float q = gload(yc[c], (uint32_t)p.i);
        float v[kFbBatch];
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) v[u] = gload(yc[c], (uint32_t)jj[u]);
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) ay[u] = fmax_(ay[u], absdiff(q, v[u]));
    }
    const float *const *zc = J.cols + p.dx + p.dy;
    for (int c = 0; c < p.dz; ++c) {
        const float q = gload(zc[c], (uint32_t)p.i);
        float v[kFbBatch];
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) v[u] = gload(zc[c], (uint32_t)jj[u]);
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) az[u] = fmax_(az[u], absdiff(q, v[u]));
    }
#pragma unroll
    for (int u = 0; u < kFbBatch; ++u)
        if (abs(jj[u] - p.i) <= J.theiler) ax[u] = ay[u] = az[u] = inf_f();
}

// top-k of this thread's rows j0, j0 + step, ..., and the counts below eps
template <int KMAX>
__device__ __forceinline__ void fb_topk(const FbPair &p, int j0, int step, float (&top)[KMAX]) {
#pragma unroll
    for (int m = 0; m < KMAX; ++m) top[m] = inf_f();
    for (int j = j0; j < p.n; j += step * kFbBatch) {
        float ax[kFbBatch], ay[kFbBatch], az[kFbBatch];
        fb_dists(p, j, step, ax, ay, az);
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) topk_insert<KMAX>(top, fmax_(fmax_(ax[u], ay[u]), az[u]));
    }
}

__device__ __forceinline__ void fb_counts(const FbPair &p, int j0, int step, float eps, int (&c3)[3]) {
    c3[0] = c3[1] = c3[2] = 0;
    for (int j = j0; j < p.n; j += step * kFbBatch) {
        float ax[kFbBatch], ay[kFbBatch], az[kFbBatch];
        fb_dists(p, j, step, ax, ay, az);
#pragma unroll
        for (int u = 0; u < kFbBatch; ++u) {
            c3[0] += fmax_(ax[u], az[u]) < eps;
            c3[1] += fmax_(ay[u], az[u]) < eps;
            c3[2] += az[u] < eps;
        }
    }
}

__device__ __forceinline__ void fb_store(const FbPair &p, float eps, int (&c3)[3]) {
    const Job &J = *p.J;
    const int n = p.n, i = p.i, e = p.e;
    if (p.dz == 0) c3[2] = n - 1 - min(i, J.theiler) - min(n - 1 - i, J.theiler);
    J.pk[(int64_t)e * n + i] = pack_counts(c3[0], c3[1], c3[2]);
    if (J.eps) J.eps[(int64_t)e * n + i] = eps;
    if (J.cnt)
        for (int t = 0; t < 3; ++t) J.cnt[((int64_t)e * 3 + t) * n + i] = c3[t];
}

// k pops of the wave-wide minimum of the threads' sorted lists; the last
// popped value is the wave's k-th smallest
template <int KMAX>
__device__ __forceinline__ float wave_kth(float (&top)[KMAX], int k, float *popped) {
    const int lane = tid_x() & 63;
    float mn = inf_f();
    for (int t = 0; t < k; ++t) {
        mn = wave_min(top[0]);
        const uint64_t bal = __ballot(top[0] == mn);
        if (lane == __builtin_ctzll(bal)) {
#pragma unroll
            for (int m = 0; m < KMAX - 1; ++m) top[m] = top[m + 1];
            top[KMAX - 1] = inf_f();
        }
        if (popped && lane == 0) popped[t] = mn;
    }
    return mn;
}

template <int KMAX>
__global__ __launch_bounds__(kFbThreads) void list_fallback_kernel(const ListLaunch L) {
    __shared__ float wtop[kFbWaves][KMAX];
    __shared__ int wcnt[kFbWaves][3];
    __shared__ float s_eps;
    const int tid = tid_x();
    const int lane = tid & 63;
    // The item count, the wave index and the block index are scalar values,
    // so the item loops and everything derived from an item are uniform and
    // all lanes stay together through the cross-lane steps below.
    const uint32_t total = __builtin_amdgcn_readfirstlane(__atomic_load_n(&L.counters[0], __ATOMIC_RELAXED));
    const int wave = (int)__builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
    if (total <= kFbBlockModeMax) {
        for (uint32_t it = (uint32_t)bid_x(); it < total; it += (uint32_t)L.fb_grid) {
            const FbPair p = fb_pair(L, it);
            float top[KMAX];
            fb_topk<KMAX>(p, tid, kFbThreads, top);
            wave_kth<KMAX>(top, p.J->k, wtop[wave]);
            __syncthreads();
            if (tid == 0) {
                int pos[kFbWaves] = {};
                float kth = inf_f();
                for (int t = 0; t < p.J->k; ++t) {
                    int best = 0;
                    float bv = inf_f();
                    for (int w = 0; w < kFbWaves; ++w)
                        if (pos[w] < p.J->k && wtop[w][pos[w]] < bv) { bv = wtop[w][pos[w]]; best = w; }
                    ++pos[best];
                    kth = bv;
                }
                s_eps = kth;
            }
            __syncthreads();
            const float eps = s_eps;
            int c3[3];
            fb_counts(p, tid, kFbThreads, eps, c3);
            for (int t = 0; t < 3; ++t) c3[t] = wave_sum(c3[t]);
            if (lane == 0) { wcnt[wave][0] = c3[0]; wcnt[wave][1] = c3[1]; wcnt[wave][2] = c3[2]; }
            __syncthreads();
            if (tid == 0) {
                int s3[3] = {0, 0, 0};
                for (int w = 0; w < kFbWaves; ++w)
                    for (int t = 0; t < 3; ++t) s3[t] += wcnt[w][t];
                fb_store(p, eps, s3);
            }
            __syncthreads();
        }
    } else {
        const uint32_t first = (uint32_t)bid_x() * kFbWaves + (uint32_t)wave;
        const uint32_t n_waves = (uint32_t)L.fb_grid * kFbWaves;
        for (uint32_t it = first; it < total; it += n_waves) {
            const FbPair p = fb_pair(L, it);
            float top[KMAX];
            fb_topk<KMAX>(p, lane, 64, top);
            const float eps = wave_kth<KMAX>(top, p.J->k, nullptr);
            int c3[3];
            fb_counts(p, lane, 64, eps, c3);
            for (int t = 0; t < 3; ++t) c3[t] = wave_sum(c3[t]);
            if (lane == 0) fb_store(p, eps, c3);
        }
    }
}

// ------------------------------------------------------------------ reduce
// (H[n_xz] + H[n_yz]) - H[n_z] per row, summed in the all-pairs kernel's order
// so that both paths return the same bits: a 64-row butterfly per chunk, then
// the chunk sums added in index order.  Phase 1: one wave per (estimate,
// chunk), blocks of kWaves chunks of one estimate, sums stored [chunk][estimate];
// phase 2: one thread per estimate adds its chunk sums.
__global__ __launch_bounds__(kBlock) void list_chunk_kernel(const ListLaunch L, const double *__restrict__ harm) {
    const int64_t g = bid_x();
    const int jb = find_job(L.est_off, L.n_jobs, g);
    const Job &J = L.jobs[jb];
    const int e = (int)(g - L.est_off[jb]);
    const int n = J.n, lane = tid_x() & 63;
    const int wave = (int)__builtin_amdgcn_readfirstlane((uint32_t)tid_x() >> 6);
    const int c = (int)__builtin_amdgcn_workgroup_id_y() * kWaves + wave;
    const int nch = (n + kChunk - 1) / kChunk;
    if (c >= nch) return;
    const int i = c * kChunk + lane;
    double v = 0.0;
    if (i < n) {
        const Counts c3 = unpack_counts(J.pk[(int64_t)e * n + i], n);
        v = (harm[c3.xz] + harm[c3.yz]) - harm[c3.z];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = v + __shfl_xor(v, off, 64);
    if (lane == 0) J.chunk[(int64_t)c * J.n_est + e] = v;
}

__global__ __launch_bounds__(kBlock) void list_reduce_kernel(const ListLaunch L, const double *__restrict__ harm) {
    const int64_t g = bid_x() * kBlock + tid_x();
    if (g >= L.ests) return;
    const int jb = find_job(L.est_off, L.n_jobs, g);
    const Job &J = L.jobs[jb];
    const int e = (int)(g - L.est_off[jb]);
    const int n = J.n;
    const int nch = (n + kChunk - 1) / kChunk;
    // chunk sums are [chunk][estimate], so the threads of a wave (consecutive
    // estimates) load adjacent words; added in index order, the loads of 16
    // chunk sums issued before their adds
    const double *part = J.chunk + e;
    const int64_t st = J.n_est;
    constexpr int kU = 16;
    double acc = 0.0;
    int c = 0;
    for (; c + kU <= nch; c += kU) {
        double v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = part[(c + u) * st];
#pragma unroll
        for (int u = 0; u < kU; ++u) acc += v[u];
    }
    for (; c < nch; ++c) acc += part[c * st];
    J.out[e] = harm[J.k - 1] - acc / (double)n;
}

// Both phases in one launch for jobs of up to kSumChunks chunks: a block per
// estimate, its waves take the chunks in turn, the chunk sums stay in LDS and
// one thread adds them in index order.  A gather of 64 harmonic numbers costs a
// CU 64 cycles, so their first kSumHead (the neighbour counts of most rows) are
// read from LDS.  Bound by latency (a launch, two dependent loads, the last
// additions); the figures stand with the choice (sums_in_one).
constexpr int kSumHead = 2048;
constexpr int kSumU = 4;          // chunks of a wave in flight

__global__ __launch_bounds__(kRowThreads) void list_sum_kernel(const ListLaunch L, const double *__restrict__ harm) {
    __shared__ double head[kSumHead];
    __shared__ double part[kSumChunks];
    const int64_t g = bid_x();
    const int jb = find_job(L.est_off, L.n_jobs, g);
    const Job &J = L.jobs[jb];
    const int e = (int)(g - L.est_off[jb]);
    const int n = J.n, tid = tid_x(), lane = tid & 63;
    const int wave = (int)__builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
    const int nch = (n + kChunk - 1) / kChunk, nh = min(n, kSumHead);
    const int nt = row_threads(L.max_chunks * kChunk), waves = nt / 64;
    const uint64_t *pk = J.pk + (int64_t)e * n;
    for (int q = tid; q < nh; q += nt) head[q] = harm[q];
    __syncthreads();
    auto h = [&](uint32_t c) { return c < (uint32_t)kSumHead ? head[c] : harm[c]; };
    for (int c0 = wave; c0 < nch; c0 += waves * kSumU) {
        uint64_t w[kSumU];
        double v[kSumU];
#pragma unroll
        for (int u = 0; u < kSumU; ++u) w[u] = pk[min((c0 + u * waves) * kChunk + lane, n - 1)];
#pragma unroll
        for (int u = 0; u < kSumU; ++u) {
            const bool in = (c0 + u * waves) * kChunk + lane < n;
            const Counts c3 = unpack_counts(w[u], n);
            v[u] = in ? (h(c3.xz) + h(c3.yz)) - h(c3.z) : 0.0;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int u = 0; u < kSumU; ++u) v[u] = v[u] + __shfl_xor(v[u], off, 64);
#pragma unroll
        for (int u = 0; u < kSumU; ++u)
            if (lane == 0 && c0 + u * waves < nch) part[c0 + u * waves] = v[u];
    }
    __syncthreads();
    if (tid) return;
    double acc = 0.0;
    int c = 0;
    for (; c + 16 <= nch; c += 16)
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += part[c + u];
    for (; c < nch; ++c) acc += part[c];
    J.out[e] = harm[J.k - 1] - acc / (double)n;
}

template <int KMAX, int DXM>
void *scan_fn(int step) {
    return step == 4 ? reinterpret_cast<void *>(&list_scan_kernel<KMAX, DXM, 4>)
                     : reinterpret_cast<void *>(&list_scan_kernel<KMAX, DXM, 8>);
}

template <int KMAX>
void *walk_fn(bool win, bool many) {
    if (many)
        return win ? reinterpret_cast<void *>(&list_walk_kernel<KMAX, true, true>)
                   : reinterpret_cast<void *>(&list_walk_kernel<KMAX, false, true>);
    return win ? reinterpret_cast<void *>(&list_walk_kernel<KMAX, true, false>)
               : reinterpret_cast<void *>(&list_walk_kernel<KMAX, false, false>);
}

template <int KMAX>
void *scan_dx(int dxm, int step) {
    return dxm == 1 ? scan_fn<KMAX, 1>(step) : dxm == 2 ? scan_fn<KMAX, 2>(step) : scan_fn<KMAX, kMaxDx>(step);
}

}  // namespace

int launch_list_zy(const ListLaunch &L, void *stream) {
    const int64_t threads = L.rows > kListCounterWords ? L.rows : (int64_t)kListCounterWords;
    hipLaunchKernelGGL(list_zy_kernel, dim3((unsigned)((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       (hipStream_t)stream, L);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_list_order(const ListLaunch &L, void *stream) {
    if (!L.ordered) return 0;
    hipLaunchKernelGGL(list_order_kernel, dim3((unsigned)L.n_sets), dim3(kSortThreads), 0, (hipStream_t)stream, L);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int QB, int... D>
void *lean_fn(int dz, std::integer_sequence<int, D...>) {
    void *fns[] = {nullptr, reinterpret_cast<void *>(&list_build_dz_kernel<D + 1, QB>)...};
    return dz >= 0 && dz <= (int)sizeof...(D) ? fns[dz] : nullptr;
}

int launch_list_build(const ListLaunch &L, const BuildPart &P, void *stream) {
    if (P.blocks <= 0) return 0;
    // the part's sets and their block offsets (absolute: a kernel subtracts
    // the first)
    const ListSet *sets = L.sets + P.set0;
    int n_sets = P.set1 - P.set0;
    const int64_t *off = L.build_off + P.set0;
    const dim3 grid((unsigned)P.blocks), block(kBT);
    if (P.dz > 0) {
        void *fn = P.qb == 4 ? lean_fn<4>(P.dz, std::make_integer_sequence<int, kBuildFixedDz>{})
                             : lean_fn<kBuildRows>(P.dz, std::make_integer_sequence<int, kBuildFixedDz>{});
        if (!fn) return -1;
        void *args[] = {(void *)&sets, (void *)&n_sets, (void *)&off};
        return hipLaunchKernel(fn, grid, block, args, 0, (hipStream_t)stream) == hipSuccess ? 0 : -1;
    }
    if (P.pack && P.qb == kBuildRows)
        hipLaunchKernelGGL((list_build_kernel<kBuildRows, kBuildCopies, true>), grid, block, 0,
                           (hipStream_t)stream, sets, n_sets, off);
    else if (!P.pack && P.qb == 1)
        hipLaunchKernelGGL((list_build_kernel<1, 1, false>), grid, block, 0, (hipStream_t)stream, sets, n_sets, off);
    else
        return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_list_scan(const ListLaunch &L, void *stream) {
    if (L.scan_blocks <= 0) return 0;
    void *fn = nullptr;
    const int st = L.scan_step;
    if (L.kmax == 4) fn = scan_dx<4>(L.dxm, st);
    else if (L.kmax == 8) fn = scan_dx<8>(L.dxm, st);
    else if (L.kmax == 16) fn = scan_dx<16>(L.dxm, st);
    else return -1;
    ListLaunch arg = L;
    void *args[] = {(void *)&arg};
    return hipLaunchKernel(fn, dim3((unsigned)L.scan_blocks), dim3(kScanLanes), args, 0, (hipStream_t)stream) ==
                   hipSuccess
               ? 0
               : -1;
}

int launch_list_rank(const ListLaunch &L, void *stream) {
    if (L.n_rank_cols <= 0) return 0;
    const unsigned rows = (unsigned)((L.max_rank_n + kRankThreads - 1) / kRankThreads);
    hipLaunchKernelGGL(list_rank_part_kernel, dim3(rows, (unsigned)kRankParts, (unsigned)L.n_rank_cols),
                       dim3(kRankThreads), 0, (hipStream_t)stream, L);
    hipLaunchKernelGGL(list_rank_place_kernel, dim3(rows, (unsigned)L.n_rank_cols), dim3(kRankThreads), 0,
                       (hipStream_t)stream, L);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// LDS of a wavelet block of n rows: the nodes, then the sequence or the
// sorted X column; 0 when it does not fit.
size_t list_wavelet_lds(int n) {
    if (n >= 32768) return 0;
    int nb = 0;
    while ((int64_t(1) << nb) <= n) ++nb;
    const size_t b = sizeof(WvNode) * (size_t)nb * (2 * (((size_t)n + 63) / 64) + 1) + sizeof(float) * (size_t)n;
    return b <= 163840 - 1024 ? b : 0;
}

int launch_list_wavelet(const ListLaunch &L, void *stream) {
    if (L.wavelet_lds == 0) return 0;
    void *fn = reinterpret_cast<void *>(&list_wavelet_kernel);
    if (L.wavelet_lds > 65536 - 1024 &&
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 163840 - 1024) != hipSuccess)
        return -1;
    ListLaunch arg = L;
    void *args[] = {(void *)&arg};
    const dim3 grid((unsigned)L.ests), block((unsigned)L.wavelet_threads);
    return hipLaunchKernel(fn, grid, block, args, L.wavelet_lds, (hipStream_t)stream) == hipSuccess ? 0 : -1;
}

int launch_list_walk(const ListLaunch &L, void *stream) {
    if (L.walk_blocks <= 0) return 0;
    const bool win = L.walk_window != 0;
    void *fn = L.kmax == 4 ? walk_fn<4>(win, L.walk_many) : L.kmax == 8 ? walk_fn<8>(win, L.walk_many)
                                                                        : walk_fn<16>(win, L.walk_many);
    ListLaunch arg = L;
    void *args[] = {(void *)&arg};
    if (hipLaunchKernel(fn, dim3((unsigned)L.walk_blocks), dim3(kScanLanes), args, 0, (hipStream_t)stream) !=
        hipSuccess)
        return -1;
    void *cf = reinterpret_cast<void *>(&list_walk_count_kernel);
    static_assert(2 * sizeof(float) * kNoZSortMax <= 163840 - 1024, "two sorted columns in LDS");
    if (L.walk_lds > 65536 - 1024 &&
        hipFuncSetAttribute(cf, hipFuncAttributeMaxDynamicSharedMemorySize, 163840 - 1024) != hipSuccess)
        return -1;
    const dim3 cuts((unsigned)L.ests, (unsigned)L.est_cuts);
    return hipLaunchKernel(cf, cuts, dim3((unsigned)L.walk_threads), args, L.walk_lds, (hipStream_t)stream) == hipSuccess ? 0 : -1;
}

int launch_list_rank_count(const ListLaunch &L, void *stream) {
    if (L.rank_waves <= 0) return 0;
    const int64_t blocks = (L.rank_waves + kRankThreads / 64 - 1) / (kRankThreads / 64);
    if (L.rank_dxm > 1)
        hipLaunchKernelGGL(list_rank_count_kernel<kMaxDx>, dim3((unsigned)blocks), dim3(kRankThreads), 0,
                           (hipStream_t)stream, L);
    else
        hipLaunchKernelGGL(list_rank_count_kernel<1>, dim3((unsigned)blocks), dim3(kRankThreads), 0,
                           (hipStream_t)stream, L);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_list_fallback(const ListLaunch &L, void *stream) {
    if (L.fail_pairs <= 0) return 0;
    const dim3 grid((unsigned)L.fb_grid), block(kFbThreads);
    if (L.kmax == 4) hipLaunchKernelGGL(list_fallback_kernel<4>, grid, block, 0, (hipStream_t)stream, L);
    else if (L.kmax == 8) hipLaunchKernelGGL(list_fallback_kernel<8>, grid, block, 0, (hipStream_t)stream, L);
    else if (L.kmax == 16) hipLaunchKernelGGL(list_fallback_kernel<16>, grid, block, 0, (hipStream_t)stream, L);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_list_reduce(const ListLaunch &L, const double *harm, void *stream) {
    if (L.ests <= 0 || L.max_chunks <= 0) return 0;
    if (sums_in_one(L.max_chunks, L.ests)) {
        hipLaunchKernelGGL(list_sum_kernel, dim3((unsigned)L.ests), dim3((unsigned)row_threads(L.max_chunks * kChunk)),
                           0, (hipStream_t)stream, L, harm);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    const dim3 grid1((unsigned)L.ests, (unsigned)((L.max_chunks + kWaves - 1) / kWaves));
    hipLaunchKernelGGL(list_chunk_kernel, grid1, dim3(kBlock), 0, (hipStream_t)stream, L, harm);
    hipLaunchKernelGGL(list_reduce_kernel, dim3((unsigned)((L.ests + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       (hipStream_t)stream, L, harm);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace mte
