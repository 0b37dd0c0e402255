// Internal interface between the host runtime and the KSG kernels.
//
// A launch processes a list of jobs.  A job is a set of estimates of
// I(X;Y|Z) that share the rows of Y and Z and differ only in the permutation
// applied to the rows of X (the candidate's own estimate uses the identity,
// its surrogates the keyed shuffles).  Different jobs of one launch may have
// different N, column counts and k.
//
// Work is split into items (job, estimate group, query tile, reference split)
// pulled from one atomic counter by a persistent grid:
//   phase A: fused items (whole reference range: k-NN pass, then the count
//            pass, then the digamma partial sums) for jobs with one split, and
//            k-NN items (partial top-k over one reference range) for jobs with
//            several splits;
//   phase B: count items for jobs with several splits; they wait until the
//            last k-NN item of their (job, group, tile) has merged the radii.
// All phase-A items are handed out before any phase-B item, and waits only go
// from phase B to phase A, so every wait ends.
#pragma once

#include <cstdint>

namespace mte {

#ifdef __HIP__
#define MTE_HD __host__ __device__
#else
#define MTE_HD
#endif

constexpr int kMaxCols = 64;       // dx + dy + dz per job
constexpr int kMaxDx = 16;
constexpr int kMaxDy = 8;
constexpr int kMaxDz = 31;
constexpr int kMaxK = 16;
constexpr int kBlock = 256;        // threads per block (4 wave64)
constexpr int kWaves = kBlock / 64;
constexpr int kChunk = 64;         // rows per fixed-order partial sum
constexpr int kSumChunks = 512;    // chunks that one block sums

// Threads of a block that takes an estimate's n rows (its counts, its sums): a
// wave for every 64 rows up to 16.  With 16 always, launches of very many
// estimates of few rows ran mostly idle waves (a search round of 67,000
// candidates, 22 estimates each, N = 40: counts 14.2 ms, sums 10.7).
constexpr int kRowThreads = 1024;
MTE_HD inline int row_threads(int n) { return n >= kRowThreads ? kRowThreads : (n + 63) / 64 * 64; }

// One estimate's surrogate key (identity when `ident` != 0).
struct EstKey {
    uint64_t h;        // key hash of (seed, cand, s)
    uint32_t ident;
    uint32_t pad;
};

struct Job {
    const float *cols[kMaxCols];  // X columns, then Y, then Z; each N floats
    int n, dx, dy, dz, k;
    int n_est;                    // estimates
    int rs;                       // reference splits (1 = fused items)
    int split_len;                // references per split (multiple of 64)
    int n_tiles;                  // query tiles of the launch's tile size
    int n_groups;                 // estimate groups of the launch's group size
    int64_t a_off, b_off;         // first item index in phase A and phase B
    const EstKey *keys;           // [n_est]
    float *xp;                    // [n_est][dx][n] permuted X (scratch)
    double *chunk;                // partial sums per 64-row chunk (scratch): [n_est][ceil(n/64)],
                                  // list path [ceil(n/64)][n_est]
    float *part;                  // [rs][n_est][n][KMAX] partial top-k (rs > 1)
    float *eps;                   // [n_est][n] radii (rs > 1, or diagnostics)
    int32_t *cnt;                 // [rs][n_est][3][n] per-split counts (rs > 1)
    uint32_t *sync;               // counters, see SyncLayout
    double *out;                  // [n_est] results
    float *diag_eps;              // optional [n_est][n]
    int32_t *diag_cnt;            // optional [n_est][3][n] (n_xz, n_yz, n_z)
    // neighbour-list path only (see ListSet): list set index, and the
    // permuted X columns transposed so that the estimates of one row are
    // adjacent, in scan groups: the jobs of a set with the same k and dx (a scan
    // class) take their estimates together, this one's from place t0 of the
    // class's T on, and xt, the class's, is xt[c][g][i][l] = X_c[pi(i)] of the
    // l-th estimate of group g ([dx][groups][n][xtw], scan_groups and
    // scan_width of T) for the scan (xp holds the same values estimate-major
    // for the fallback).  The per-row counts go to pk; eps and cnt are the
    // caller's diagnostics ([n_est][n], [n_est][3][n]) or null.
    // A swapped job (swap) scans with the sides exchanged: set is a set over
    // its X columns, row m stands for the row i with pi_e(i) = m, and xt holds
    // that row's Z and Y (xt[0] the Z, xt[1] the Y column; sdx = 2 columns,
    // else sdx = dx).  rset is the set of its (Y, Z) sample (= set otherwise).
    int set, rset, swap, sdx;
    int t0, T, xtw;
    float *xt;
    int theiler;                  // Theiler window w: pairs with |i - j| <= w are left out
    int reps;                     // replications R (rows: R blocks of n/R, replication-major)
    int rep_shuffle;              // surrogates shuffle the replication order (else rows within each)
    // list path without Z (dz = 0, dx = 1) and jobs counted in a wavelet
    // matrix (xw): the job's X column sorted ascending (n floats); null
    // otherwise
    float *xs;
    // list path: each (row, estimate)'s counts in one word,
    // n_xz | n_yz << kPackBits | n_z << 2 kPackBits ([n_est][n])
    uint64_t *pk;
    // list path with one Z column (rank counts, see ListSet::zs): the set's
    // rank of each row, the permuted X in rank order, estimate-major
    // (xr[e][c][r] = X_c[pi_e(zord[r])], [n_est][dx][n]), or, with one X column
    // and no Theiler window, the rank of each row of the X column (xrank) and
    // each row's source row (xw[e][i] = pi_e(i), [n_est][n], followed by
    // [n_est][n] words for the ranks in rank order), and each pair's radius (low word, -1
    // for a pair left to the all-rows redo) and n_yz from the scan, by rank
    // (er[e][r]), of a swapped job n_xz, by row m (er[e][m]); null otherwise
    const int32_t *zrank;
    float *xr;
    const int32_t *xrank;
    uint16_t *xw;
    uint64_t *er;
    // A job without Z, one X and one Y column (walk) takes no lists: its rows
    // go by rank in y (zrank, xr and xt's rows), neighbours in y are
    // neighbouring ranks (xt has kWalkPad rows before and after each group's,
    // and xtw is kScanLanes: a step's rows are then constant offsets).
    // rad: radii by row ([n_est][n]; in the low halves of the count words the
    // counts read 8 bytes for 4, 0.5% of a test)
    int walk;
    float *rad;
};

// Counts of the list path are packed kPackBits to a field: N <= kListMaxN.
constexpr int kPackBits = 21;
constexpr int kListMaxN = 1 << kPackBits;
constexpr uint64_t kPackMask = (uint64_t(1) << kPackBits) - 1;

// A row's counts as that word, and back as places in the harmonic table, which
// holds n + 1 values.  Inputs that are not finite, which device calls do not
// check, can leave a range that lacks the row itself, so that the range less
// the row is -1 (0 here), and rows that no kernel wrote a word for: whatever a
// word holds, its three places lie inside the table.
MTE_HD inline uint64_t pack_counts(int cxz, int cyz, int cz) {
    return (uint64_t)(uint32_t)(cxz < 0 ? 0 : cxz) | ((uint64_t)(uint32_t)(cyz < 0 ? 0 : cyz) << kPackBits) |
           ((uint64_t)(uint32_t)(cz < 0 ? 0 : cz) << (2 * kPackBits));
}
struct Counts {
    uint32_t xz, yz, z;
};
MTE_HD inline Counts unpack_counts(uint64_t w, int n) {
    const uint32_t xz = (uint32_t)(w & kPackMask), yz = (uint32_t)((w >> kPackBits) & kPackMask),
                   z = (uint32_t)(w >> (2 * kPackBits)), m = (uint32_t)n;
    return Counts{xz < m ? xz : m, yz < m ? yz : m, z < m ? z : m};
}

// Largest N of a list-path job without Z (its two sorted columns lie in LDS).
constexpr int kNoZSortMax = 16384;

// Neighbour lists of one (Y, Z) sample, shared by every job of a launch whose
// Y and Z columns are the same.  For row i, list 1 holds the other rows j with
// the (Y,Z) max-norm distance d_yz(i,j) in the smallest key buckets that fit
// m1 entries, list 2 the same for the Z distance d_z(i,j) and m2.  A key is
// the top 12 bits of the distance's float encoding (8 exponent and 4
// mantissa bits), so a list is ordered by bucket, not fully sorted.  Its bound, the
// floor of the first bucket left out (+inf when nothing is), is a lower bound
// of every unlisted distance, so a radius up to it is decided by the list
// alone; the sentinels after the list carry it to the scan.
struct LEnt {
    float d;                      // d_yz in list 1, d_z in list 2 (the list key)
    int32_t j;                    // row
};

constexpr int kListPad = 16;                  // sentinel entries after each row's list: two steps

struct ListSet {
    const float *cols[kMaxDy + kMaxDz];   // Y columns, then Z columns
    float *zy;                    // [dz + dy][n] contiguous copy: Z columns, then Y (build input)
    int32_t *order;               // [n] the scan's row order in launches of several jobs: rows
                                  // grouped by Morton cell of their Z, Y coordinates; null: identity
    int n, dy, dz;
    int theiler;                  // Theiler window of the rows (|i - j| <= w left out)
    int m1, m2;                   // list capacities per row
    int s1, s2;                   // row strides: capacity + kListPad sentinels
    LEnt *l1;                     // [n][s1]  (Y,Z) list
    LEnt *l2;                     // [n][s2]  Z list
    int32_t *len;                 // [n][2]
    // One Z column and n <= kRankMaxN: the rows sorted by z, so that the rows
    // within a radius of a row's z are one range of ranks (float subtraction
    // is monotone in its first operand).  zs[r] the r-th smallest z, zord[r]
    // its row, zrank the inverse.  n_z and n_xz of such a set's jobs come
    // from these ranges, not from the Z list (whose capacity is then
    // kRankListCap).  Null otherwise.
    float *zs;
    int32_t *zord;
    int32_t *zrank;
    // for swapped and walk jobs (Job::swap, Job::walk): y sorted, each row's
    // rank in y and, for walk jobs, the row of each rank; ys then has kWalkPad
    // words of -inf before and +inf after it
    float *ys;
    int32_t *yrank, *yord;
};
constexpr int kWalkPad = 16;

// A run of list sets built by one kernel form: compiled dimensions (dz Z
// columns and one Y column) or, dz = 0, the generic form; qb rows per block;
// pack: 16-bit packed histograms (every set has N <= 2^16).
struct BuildPart {
    int set0 = 0, set1 = 0;
    int dz = 0, qb = 0, pack = 0;
    int64_t block0 = 0, blocks = 0;
};

constexpr int kCoopLanes = 4;                 // default cooperative-finish threshold of the scan
constexpr int kRankMaxN = 32768;              // rank counts: rows ranked by O(n^2) compares
constexpr int kRankListCap = 1;               // Z-list capacity of a set counted by ranks (nothing reads it)

constexpr int kBuildRows = 2;                // rows per build block when N <= 2^16
constexpr int kLeanRows = 2;                 // rows per block of the compiled-dimension build
// Compiled-dimension build: dz <= kBuildFixedDz Z columns and one Y column.
constexpr int kBuildFixedDz = 15;
constexpr int kXcds = 8;   // accelerator complex dies (one L2 each) of an MI355X
constexpr int kBuildCopies = 1;              // histogram copies per row (spread LDS atomics)
constexpr int kListStatWord = 16;
constexpr int kListStatSlots = 64;            // spread so that the atomics do not queue on one address
constexpr int kListStatStride = 16;           // words (64 bytes) per slot
constexpr int kListCounterWords = kListStatWord + kListStatSlots * kListStatStride;
constexpr int kKeyShift = 19;                 // 4096 key buckets
constexpr int kKeyBins = 1 << (32 - kKeyShift - 1);

// Scan groups of a class: its E estimates in G = ceil(E / 64) groups of nearly
// equal size, group g holding the estimates g*E/G .. (g+1)*E/G - 1, one lane
// each; a row of a group takes scan_width(E) words of xt: as many as there are
// estimates below 64, else the largest group's in whole 64-byte lines (130
// estimates, 43 a group, N = 9995, 3 X and 2 Z columns: 5.38 ms with 48 words,
// 5.42 with 43, 6.31 with 64; but 100 estimates at N = 4000 0.73 ms with 64
// words, 0.76 with 50).
constexpr int kScanLanes = 64;
MTE_HD inline int scan_groups(int n_est) { return (n_est + kScanLanes - 1) / kScanLanes; }
MTE_HD inline int scan_width(int n_est) {
    return n_est < kScanLanes ? n_est : ((n_est + scan_groups(n_est) - 1) / scan_groups(n_est) + 15) / 16 * 16;
}
MTE_HD inline int scan_group_first(int g, int n_est) { return (int)((int64_t)g * n_est / scan_groups(n_est)); }
MTE_HD inline int scan_group_of(int e, int n_est) {
    return (int)((((int64_t)e + 1) * scan_groups(n_est) - 1) / n_est);
}

// A range of rows (positions in the set's row order) of one scan group; `job`
// is the first job of its class, whose jobs are class_jobs[first .. first +
// n_jobs - 1] in order of their t0.
struct ScanUnit {
    int32_t job, group, row0, nrows, first, n_jobs;
};
struct ClassJob {
    int32_t t0, job;
};

// A column to be ranked by value: its rows' ranks, the row of each rank and
// the values in rank order (rank and ord may be null).  part: [kRankParts][n]
// scratch, which lies among the launch's count words (nothing else is written
// there before the ranks are placed).
constexpr int kRankParts = 16;
struct RankCol {
    const float *col;
    int n;
    int32_t *part, *rank, *ord;
    float *sorted;
    int pad;                      // words of -inf before and +inf after `sorted`
};

// One launch of the list path over `n_jobs` jobs.
struct ListLaunch {
    const Job *jobs;              // device
    const ListSet *sets;          // device
    const int64_t *fail_off;      // [n_jobs+1] prefix sums of the pairs that may be redone: n * n_est,
                                  // none of a walk job
    const int64_t *row_off;       // [n_sets+1] prefix sums of the sets' n
    const int64_t *build_off;     // [n_sets+1] prefix sums of the build blocks per set
    int64_t build_blocks;
    int stats;                    // non-zero: the scan accumulates its entry counts
    const int64_t *est_off;       // [n_jobs+1] prefix sums of n_est
    int n_jobs, n_sets;
    int64_t lanes, rows, ests;
    int64_t fail_pairs;           // pairs that may be redone (fail_off[n_jobs]); none: no redo launch
    int ordered;                  // some set has a row order
    void *failq;                  // undecided pairs, fail_off[job] + i * n_est + e each, in
    int fail_wide;                // uint64 words if the launch has 2^32 pairs or more, else uint32
    uint32_t *counters;           // [0] undecided pairs; from word kListStatWord,
                                  // kListStatSlots slots of kListStatStride words each
                                  // holding two uint64 totals of list entries read (k-NN
                                  // scan, Z-list scan); kListCounterWords words, zeroed
                                  // per launch
    int kmax, dxm;                // compile-time classes of the scan kernel
    int rank_dxm;                 // largest dx of the jobs counted over rank ranges
    int fb_grid;                  // blocks of the fallback kernel
    int max_chunks;               // largest ceil(n / kChunk) of the jobs (reduction grid)
    int coop_lanes;               // the scan finishes cooperatively once this many lanes remain
    // Scan units, dealt to the XCDs in turn (unit u on XCD u % kXcds, each XCD
    // taking its units one after another): xcd_off[x * (unit_t + 1) + t] is
    // the first block, counting XCD x's blocks alone, of x's t-th unit
    // (unit x + t * kXcds; the entry at t = unit_t, and past x's last unit,
    // is x's block count).
    const int64_t *xcd_off;
    const ScanUnit *units;
    const ClassJob *class_jobs;
    int unit_t;
    int64_t scan_blocks;          // grid of the scan
    // the same for the walk jobs
    const int64_t *walk_xcd_off;
    const ScanUnit *walk_units;
    int walk_unit_t, walk_window; // walk_window: some walk job has a Theiler window
    int walk_many;                // some walk unit's lanes belong to several jobs
    int64_t walk_blocks;
    size_t walk_lds;              // LDS bytes of their counts: two sorted columns
    int walk_threads, wavelet_threads;   // row_threads of the largest job of either form
    int scan_step;                // list entries per step of the scan's lane-by-lane loops (4, 8)
    const RankCol *rank_cols;     // the columns to rank
    int n_rank_cols;
    int est_cuts;                 // blocks per estimate of the walk counts
    size_t wavelet_lds;           // LDS bytes of a wavelet block (0: no job is counted there)
    int64_t rank_waves;           // rank-count waves: sum over those sets' jobs of
                                  // n_est * ceil(n / 64)
    const int64_t *rank_off;      // [n_jobs+1] prefix sums of each job's rank-count waves
    int max_rank_n;               // largest n of a ranked column
};

// Counter words of one job (all zero before a launch):
//   [0, G*T)        k-NN items done per (group, tile)
//   [G*T, 2*G*T)    radii ready per (group, tile)
//   [2GT, 3GT)      count items done per (group, tile)
//   [3GT, 3GT+G)    tiles finished per group
inline int64_t sync_words(int n_groups, int n_tiles) {
    return 3LL * n_groups * n_tiles + n_groups;
}

// Tile configurations compiled into the library.
struct TileCfg {
    int kmax;   // top-k register slots (k <= kmax)
    int g;      // estimates per lane
    int qp;     // queries per lane
    int dzm;    // Z column capacity
    int dym;    // Y column capacity
    int dxm;    // X column capacity
};

struct LaunchInfo {
    int64_t items_a, items_b;     // item counts of the two phases
    int grid;                     // persistent blocks
};

// Compiled configurations of the all-pairs kernel for jobs with few estimates
// (solo.hip): top-k capacity, Z, Y and X column capacities, estimates and
// query rows per wave.
struct SoloCfg {
    int kmax, dzm, dym, dxm, g, qp;
    int fz;                                  // >= 0: compiled dimensions (dz = fz, dy = dx = 1)
};
constexpr int kSoloMaxEstimates = 7;         // jobs with more take the persistent kernel
int solo_variant_count();
bool solo_variant(int i, SoloCfg *cfg);
// One wave per (job, estimate group, query tile); wave_off: [n_jobs+1] prefix
// sums of each job's waves.  Writes Job::pk (and the diagnostics).
int launch_solo(int variant, const Job *jobs_dev, int n_jobs, const int64_t *wave_off, int64_t total_waves,
                void *stream);

// Host-side launch helpers implemented in kernels.hip.
// jobs_dev: device copy of `n_jobs` Job records; work: 2 device words
// (queue head, error flag) cleared by `launch_reset`.
int kernel_variant_count();
bool kernel_variant(int i, TileCfg *cfg);
int variant_blocks_per_cu(int variant);
int launch_reset(uint32_t *words, int64_t n_words, void *stream);
// The same for jobs of at most kPermTableMax rows per replication, shuffled
// within replications: one block per (job, estimate, replication) (item_off:
// [n_jobs+1] prefix sums), `max_rows` the largest rows per replication.
constexpr int kPermTableMax = 16384;
int launch_permute_table(const Job *jobs_dev, int n_jobs, int64_t items, const int64_t *item_off, int max_rows,
                         void *stream);
// Permuted X columns: total_blocks work items (blk_off: [n_jobs+1] prefix
// sums of each job's items), on a grid of at most max_grid blocks (0: one
// block per item) that take the items in turn.
int launch_permute(const Job *jobs_dev, int n_jobs, int64_t total_blocks, const int64_t *blk_off,
                   void *stream, int64_t max_grid = 0);
int launch_main(int variant, const Job *jobs_dev, int n_jobs, const int64_t *a_off_dev,
                const int64_t *b_off_dev, const LaunchInfo &li, uint32_t *work,
                const double *harm, void *stream);

int launch_list_zy(const ListLaunch &L, void *stream);      // the sets' contiguous Y,Z copies; clears the counters
int launch_list_order(const ListLaunch &L, void *stream);  // the scan's row order (several jobs)
int launch_list_build(const ListLaunch &L, const BuildPart &P, void *stream);
int launch_list_scan(const ListLaunch &L, void *stream);
int launch_list_walk(const ListLaunch &L, void *stream);        // radii and counts of the walk jobs
int launch_list_rank(const ListLaunch &L, void *stream);        // ranks of the columns in rank_cols
int launch_list_rank_count(const ListLaunch &L, void *stream);  // counts of the ranked sets' jobs over rank ranges
int launch_list_wavelet(const ListLaunch &L, void *stream);     // the same in wavelet matrices
size_t list_wavelet_lds(int n);                                 // LDS of such a block, 0: does not fit
int launch_list_fallback(const ListLaunch &L, void *stream);
int launch_list_reduce(const ListLaunch &L, const double *harm, void *stream);
// The digamma sums take one launch where a block per estimate is enough, and
// then no Job::chunk: a few chunks each, or estimates for a quarter of the
// chip.  Kernel times, both launches and one: N = 1000, 1 estimate 8.5 and 4.2 us;
// N = 1003, 101 estimates 10.4 and 5.8; N = 10^4, 201 estimates 20.1 and 14.0;
// but 1 estimate 9.6 and 11.5.
constexpr int kSumFew = 64, kSumEsts = 64;
inline bool sums_in_one(int max_chunks, int64_t ests) {
    return max_chunks <= kSumFew || (max_chunks <= kSumChunks && ests >= kSumEsts);
}

// Host reference of the surrogate permutation (same definition as the device).
uint64_t mix64(uint64_t z);
uint64_t surrogate_key(uint64_t seed, uint32_t cand, uint32_t s);
void permutation_host(uint64_t h, int64_t n, uint32_t *out);
// Source rows of one surrogate over R replications of n/R rows (the device's
// definition; R = 1 without rep_shuffle is permutation_host).
void replication_source_rows_host(uint64_t h, int64_t n, int reps, int rep_shuffle, uint32_t *out);
// MTE_SHUFFLE_REPLICATIONS when R! >= S, else MTE_SHUFFLE_WITHIN.
int shuffle_mode(int reps, int S);
// Blocks of the permute kernel for one estimate of a job.
inline int64_t permute_blocks(int64_t n, int reps) { return (int64_t)reps * ((n / reps + 1023) / 1024); }

}  // namespace mte
