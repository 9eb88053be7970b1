// Internal declarations shared by the kernels and the host side of libfastcod.so.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace fc {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;               // 256-thread workgroups
constexpr int kBlock = kWave * kWavesPerBlock;
constexpr int kSetCap = 512;                    // LDS hash slots per wavefront (load <= 1/2)

// Exclusive upper bounds of t = fl32(q + 0.5) per axis: the smallest float >= the grid size,
// so that `t < bound` holds exactly when floor(t) < size, also for sizes above 2^24.
struct Grid {
    int32_t X, Y, Z;
    float Xf, Yf, Zf;
};

// Raster lookup straight from the caller's volumes.
struct RasterVol {
    const int32_t *roi;
    const int32_t *lab;
    int32_t X, XY;
    int32_t N, M;
};

// Compact lookup: occupancy bits in 16x8x8 super-bricks (32 words of 32 voxels each), every
// occupancy word paired with the position of its first code (its rank base), and one code per
// occupied voxel, those of one word in the order of its bits.
struct CompactVol {
    const uint2 *mb;          // [W] {occupancy word, rank base}
    const uint32_t *coarse;   // one bit per (2^cs)^3 block: any occupied voxel inside
    int32_t csx, csyz;        // log2 of the coarse block's x and y/z sides: 3,3 / 4,4 / 5,5 (cubes) or
                              // 4,3 (one 16x8x8 super-brick per block, coarse index = super-brick index)
    int32_t CBX, CBXY;        // coarse blocks along x, and per z-slab
    int32_t ncoarse_words;    // words of `coarse` (a multiple of 2)
    const uint32_t *codes;    // row | label << rbits; all ones in a field: none
    int32_t SBX, SBXY;        // super-bricks along x, and per z-slab
    int32_t rbits;            // bits of the row field in a code (at most 31)
    uint32_t rmask;           // (1 << rbits) - 1
    int32_t N, M;
    int64_t W;                // occupancy words
    int64_t ncodes;           // capacity of the code array (bounds of every code read)
    uint32_t codes_off;       // byte offset of the code array from mb (one allocation)
    uint32_t span;            // bytes from mb to the end of the code array (< 2^32 - 16)
};

// Per-wavefront slices of appended C updates (flat-stream kernel, plain path): wavefront w writes
// its entries to pairs[w * cap ...] and their number to counts[w]; cap 0 = every update is an atomic.
struct PairOut {
    uint32_t *pairs;
    uint32_t *counts;
    uint32_t cap;
};

// Histogram of the appended updates into C, tile by tile in LDS.
constexpr int kMaxPairTiles = 4096;                 // up to 2^26 entries of C take this path
constexpr int kMaxPairTileLog2 = 14;                // 16K counters (64 KB of LDS) per tile of C
constexpr int kMinPairTileLog2 = 11;
// Sorting workgroups (1024 threads): with up to 64 of the fallback beside them, two per CU of a 256-CU
// device, all resident at once.
constexpr int kPairBlocks = 448;
constexpr int kPairRound = 16 * 1024;              // updates a workgroup sorts at a time
struct PairTiles {
    int32_t log2 = 0, n = 0, blocks = 0;   // entries per tile, tiles, sorting workgroups
    int64_t hist_words = 0;                // round counts and run table
};
// The smallest tiles of which at most 512 cover C (one round of the tile pass), so that a small C is
// spread over the chip too: a C of 564,000 entries in 35 tiles of 2^14 took 20 us, mostly in 35
// workgroups' LDS atomics.
// Sorting workgroups for about four updates a streamline, half a round each: fewer of them leave longer
// runs to the tile pass.
inline PairTiles pair_tiles(int64_t NM, int64_t S, int64_t nwaves, int64_t cap) {
    PairTiles pt;
    pt.log2 = kMinPairTileLog2;
    while (pt.log2 < kMaxPairTileLog2 && ((NM + (int64_t(1) << pt.log2) - 1) >> pt.log2) > 512) ++pt.log2;
    pt.n = (int32_t)((NM + (int64_t(1) << pt.log2) - 1) >> pt.log2);
    int64_t blocks = (4 * S + kPairRound / 2 - 1) / (kPairRound / 2);
    if (blocks < (nwaves + 63) / 64) blocks = (nwaves + 63) / 64;   // at most 64 slices each
    pt.blocks = (int32_t)(blocks < kPairBlocks ? blocks : kPairBlocks);
    const int64_t most = (nwaves + pt.blocks - 1) / pt.blocks * cap;   // updates of one workgroup
    pt.hist_words = 2 * kPairBlocks + ((most + kPairRound - 1) / kPairRound * pt.blocks * (pt.n + 1) + 1) / 2;
    return pt;
}

// Streamlines whose distinct (row, label) keys outgrow the per-wave LDS set are handed to a
// fallback kernel through this queue of point indices (one point inside each such streamline).
struct Overflow {
    unsigned long long *count;
    int64_t *list;
    int64_t cap;
    unsigned long long *work;   // the range (work item) queues' counters (flat-stream and batched
                                // kernels), kQueueWords apart; zeroed per launch
};

// Point ranges (work items) are handed out by kRangeQueues counters, each in a 128-byte line of its
// own: wavefront w takes the ranges c, c + Q, c + 2Q, ... of queue c = w mod Q (Q = kRangeQueues, or
// fewer for a small grid), so that no counter is contended by more than a few dozen wavefronts
// (a single counter serialises every wavefront's fetch).  Counter block: one 128-byte line for the
// overflow count, then the queues.
constexpr int kRangeQueues = 64;
constexpr int kQueueWords = 16;                                   // 64-bit words per counter line
constexpr size_t kQueueBlockBytes = 128 * (size_t)kRangeQueues;  // one launch's queues
// bytes before the overflow list: count line + `launches` blocks of queues (256-aligned)
inline size_t overflow_header_bytes(int launches) {
    return (128 + kQueueBlockBytes * (size_t)launches + 255) & ~size_t(255);
}

// Per-workgroup scratch of the fallback kernel; bit maps are all-zero between launches.
struct FallbackScratch {
    uint32_t *words;      // [blocks][stride]: N-bit map, M-bit map, M-entry label list
    int64_t stride;
    int32_t blocks;
    int32_t nwordsN, nwordsM;
};

// C is addressed as C[i * si + m * sm]: row-major [N][M] (si = M, sm = 1) or the transposed
// accumulation layout [M][N] (si = 1, sm = N); N * M < 2^31.
// end_mode 0: every point's label counts (pass-through); 1: the label of each streamline's last point
// only; 2: the labels of its first and last points.
struct CountArgs {
    const float *pts;
    const int64_t *offsets;
    int64_t S;
    Grid g;
    float scale;
    int32_t *C;
    uint32_t si, sm;
    Overflow ovf;
    int32_t end_mode;
    int32_t up;   // upsampling factor: up - 1 points inserted between neighbouring points (1 = none)
};

// Everything the flat-stream kernels need about one subject (also the device-side descriptor of
// the batched form): streamlines [s_begin, S) of (pts, offsets) are counted into C.  s_begin > 0
// lets a caller count one streamline range of a larger set (offsets stay absolute).
struct StreamSubject {
    const float *pts;
    const int64_t *offsets;
    int64_t S;
    int64_t s_begin;
    Grid g;
    float scale;
    CompactVol cv;
    int32_t *C;
    uint32_t si, sm;
    int32_t end_mode;
    int32_t up;   // upsampling factor (1 = none)
};

// ---- launchers (kernels.hip); every launcher returns the hipError_t of its launch ----
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, int cus, hipStream_t st);
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, int cus, hipStream_t st);

// compact volume build: cv's layout and sizes, written through mb (W {word, base} pairs), codes and
// coarse (ncoarse_words, zero on entry); ncodes: the number of codes written (zero on entry); S: streamlines
// of the call that builds it (0: built to be kept)
hipError_t launch_compact_build(const int32_t *roi, const int32_t *lab, Grid g, CompactVol cv, uint2 *mb, uint32_t *codes,
                                uint32_t *coarse, uint32_t *ncodes, int64_t S, hipStream_t st);

// The 4 voxels x .. x + 3 of a row of X that one lane of the build reads: it loads elements xs .. xs + 3
// (kWide: rows of at least 4 voxels, the last 4 where x .. x + 3 pass the end), `mine` are those inside its
// 4 voxels and the row, and element d of the load is voxel x.  d <= 3 also in lanes past the end of the row,
// whose `mine` is empty: they shift by it all the same.
struct RowLane {
    int32_t xs;
    int d;
    uint32_t mine;
};
template <bool kWide>
__host__ __device__ inline RowLane row_lane(int32_t x, int32_t X) {
    RowLane r{x, 0, 0u};
    if (kWide) {
        if (r.xs > X - 4) r.xs = X - 4;
        r.d = x - r.xs < 3 ? x - r.xs : 3;
        if (x < X) r.mine = (0xFu << r.d) & 0xFu;
    } else {
        if (r.xs > X - 1) r.xs = X - 1;
        if (x < X) r.mine = 0xFu >> (x + 4 > X ? x + 4 - X : 0);
    }
    return r;
}

// Range that a streamline starting at point p belongs to: floor(n * h(p / P)), h the inverse of
// g(x) = 1.5 x - 0.5 x^2, so the ranges shrink linearly from 1.5x to 0.5x the mean in the order they
// are handed out and the last ones to start end close together.  p counts to 24 bits (exact as a
// float); each step, IEEE square root included, is monotone in p, as the table needs.
struct RangeOf {
    int sh;
    float inv_P, n;
    int64_t P;
    int32_t last;
    __host__ __device__ RangeOf(int64_t points, int64_t nparts) : n((float)nparts), last((int32_t)nparts - 1) {
        P = points > 0 ? points : 0;
        sh = P >> 24 ? 40 - __builtin_clzll((unsigned long long)P) : 0;
        inv_P = P > 0 ? 1.0f / (float)(uint32_t)(P >> sh) : 0.0f;
    }
    __host__ __device__ int32_t operator()(int64_t p) const {
        const float u = fminf((float)(uint32_t)((p < 0 ? 0 : (p > P ? P : p)) >> sh) * inv_P, 1.0f);
        const int32_t i = (int32_t)(n * (1.5f - sqrtf(2.25f - 2.0f * u)));
        return i < 0 ? 0 : (i > last ? last : i);
    }
    // the same for ranges of equal size
    __host__ __device__ int32_t equal(int64_t p) const {
        const int32_t i = (int32_t)(n * fminf((float)(uint32_t)((p < 0 ? 0 : (p > P ? P : p)) >> sh) * inv_P, 1.0f));
        return i < 0 ? 0 : (i > last ? last : i);
    }
};

// Per-call state zeroed by the partition launch, so that it needs no launches of its own: C when
// it is not accumulated into, a fixed scratch area's fallback bit maps, the coarse map of a volume built by
// the same call, the overflow and range counters.  Each range may be empty.
constexpr int kZeroRanges = 3;
struct ZeroRanges {
    int32_t *w32[kZeroRanges] = {};
    int64_t n32[kZeroRanges] = {};
    unsigned long long *w64 = nullptr;
    int64_t n64 = 0;
};
// nparts ranges of whole streamlines, their point counts falling linearly from 1.5x to 0.5x the mean
// in range order: first[nparts + 1] (nullptr: no ranges); also zeroes `z`
hipError_t launch_partition(const int64_t *offsets, int64_t S, int64_t nparts, int32_t *first, const ZeroRanges &z,
                            int cus, hipStream_t st);
// Streamline ranges of a flat-stream launch: a table of nparts ranges handed out by the queues, or
// (first == nullptr) one range per wavefront: `per` streamlines each and one more in the first `extra`, or
// (per == 0) ranges of about equally many points and streamlines that the wavefronts find themselves.
struct Ranges {
    const int32_t *first;
    int64_t nparts;
    uint32_t per, extra;
    double inv_nparts, inv_S;   // (per == 0)
};
// LDS of a workgroup's copy of a coarse map, stored 16 bytes at a time
inline size_t coarse_lds_bytes(int32_t words) { return 4 * (size_t)((words + 3) & ~3); }
// resident 256-thread workgroups per CU of the flat-stream kernel
int count_stream_blocks_per_cu(bool scaled, int batch, bool ends, int up, size_t dyn_lds);

hipError_t launch_count_wave(const CountArgs &a, const RasterVol &rv, int blocks, hipStream_t st);
// parcellation outputs of C [N][M]: label [N], frac [N][M], sums [N] (each may be null)
hipError_t launch_parcellate(const int32_t *C, int32_t N, int32_t M, int32_t *label, float *frac, int64_t *sums,
                             int cus, hipStream_t st);
// Alg. 1's count: C(row of the first point, label of the last point) += 1 for every streamline
hipError_t launch_count_seed_end(const CountArgs &a, const RasterVol *rv, const CompactVol *cv, int cus,
                                 hipStream_t st);
// batch: 64-point windows per pipelined batch (2 or 4)
hipError_t launch_count_stream(const CountArgs &a, const CompactVol &cv, const Ranges &rg, int blocks, int batch,
                               const PairOut &po, hipStream_t st);
// C[NM] += histogram of the updates in the slices (nwaves slices of po.cap entries, lengths in
// po.counts); before it, the overflow queue of `a` (as launch_fallback_compact).  pt: pair_tiles of the
// same sizes; hist: pt.hist_words words; sorted: nwaves * po.cap 16-bit entries.
hipError_t launch_pair_histogram(const PairOut &po, int32_t nwaves, const PairTiles &pt, const CountArgs &a,
                                 const CompactVol &cv, FallbackScratch fs, int32_t *C, int64_t NM, uint32_t *hist,
                                 uint32_t *sorted32, hipStream_t st);
hipError_t launch_fallback_raster(const CountArgs &a, const RasterVol &rv, FallbackScratch fs,
                                  hipStream_t st);
hipError_t launch_fallback_compact(const CountArgs &a, const CompactVol &cv, FallbackScratch fs,
                                   hipStream_t st);

// C[i][m] = CT[m][i] (or += with accumulate), C [N][M], CT [M][N]
hipError_t launch_transpose(const int32_t *CT, int32_t *C, int32_t N, int32_t M, bool accumulate, hipStream_t st);

// One transpose of a batch: C[i][m] = CT[m][i] over kTransposeTile^2 tiles, tiles numbered from
// first_tile (the running sum of ceil(N/kTransposeTile) * ceil(M/kTransposeTile) over the jobs before it)
constexpr int kTransposeTile = 64;
struct TransposeJob {
    const int32_t *CT;
    int32_t *C;
    int32_t N, M;
    int64_t first_tile;
};
// every job of `jobs` (device array of njobs, first_tile increasing from 0; ntiles tiles in all)
hipError_t launch_transpose_many(const TransposeJob *jobs, int32_t njobs, int64_t ntiles, int cus, hipStream_t st);

// batched form
// Workgroups of a preparation launch: `blocks` for every subject, or (table) `blocks` in all, subject k's from
// base[k] to base[k + 1].
struct PrepareGrid {
    int64_t blocks = 1;
    bool table = false;
};
// Up to 16 workgroups per CU in all, one thread per unit of work[k] at most: a unit zeroes four entries of C; a
// streamline, whose offset is waited for, counts as kPrepareStreamlineWork.  Equally many each while that gives the largest subject all it can use or half of its share of the
// work; in proportion otherwise, one at least where there is work (base: n + 1 entries, written then).
// (A plan of one subject of 3M streamlines and 255 of 100 takes 1054 us a launch, 1828 with equally many.)
constexpr int64_t kPrepareStreamlineWork = 4;
inline PrepareGrid prepare_grid(const int64_t *work, int32_t n, int64_t nzero, int cus, int64_t *base) {
    const int64_t cap = (int64_t)cus * 16;
    int64_t most = 0, sum = 0;
    for (int32_t k = 0; k < n; ++k) {
        most = most > work[k] ? most : work[k];
        sum += work[k];
    }
    auto blocks_of = [](int64_t w) { return (w + kBlock - 1) / kBlock; };
    PrepareGrid g;
    const int64_t all = blocks_of(most), each = cap / n > 1 ? cap / n : 1;
    g.table = each < all && most * n > 2 * sum;
    if (!g.table) {
        const int64_t want = blocks_of(most > nzero ? most : nzero);
        g.blocks = want < 1 ? 1 : (want < each ? want : each);
        return g;
    }
    base[0] = 0;
    for (int32_t k = 0; k < n; ++k) {
        int64_t b = (int64_t)((double)cap * ((double)work[k] / (double)sum));
        if (b < 1) b = 1;
        if (b > blocks_of(work[k])) b = blocks_of(work[k]);
        base[k + 1] = base[k] + b;
    }
    g.blocks = base[n];
    return g;
}
// zeroes every subject's C (sizes: entries; nullptr: none), writes the work items (items == nullptr: none)
// and zeroes zero[0 .. nzero) (the counting launches' overflow count and range queues);
// block_base: device copy of the grid's table (grid.table)
hipError_t launch_prepare_batched(const StreamSubject *subs, const int64_t *item_base, const int64_t *sizes, int32_t nsub,
                                  const PrepareGrid &grid, const int64_t *block_base, int2 *items, unsigned long long *zero,
                                  int64_t nzero, hipStream_t st);
// Points a work item holds at least, on average: smaller launches get fewer items, and with at most one
// per wavefront nothing is drawn from a queue.  (24 little subjects of 3.4M points in all: 45.1 us a
// launch at 512, 41.4 at 256, 58.6 at 1024, 58 with 28,672 items whatever the points.)
constexpr int64_t kMinItemPoints = 256;
// Kinds of subject of the batched form, each counted by its own launch (subjects of one kind are
// neighbours in the descriptor table): pass-through, endpoint modes 1/2,
// upsampled pass-through (u = 2, or u = 3..4), Alg. 1's seed-to-end count (no work items).
enum class BatchedKind : int { kPass = 0, kEnds = 1, kUp2 = 2, kUp4 = 3, kSeedEnd = 4 };
constexpr int kBatchedKinds = 5;
inline BatchedKind batched_kind(int mode, int up) {
    if (mode == 3) return BatchedKind::kSeedEnd;
    if (up > 2) return BatchedKind::kUp4;
    if (up == 2) return BatchedKind::kUp2;
    return mode == 1 || mode == 2 ? BatchedKind::kEnds : BatchedKind::kPass;
}
int count_batched_blocks_per_cu(int batch, int coarse_words, BatchedKind kind = BatchedKind::kPass);
// items[0, nitems) of subjects of one kind (kPass, kEnds, kUp2, kUp4) of the table's nsub entries
hipError_t launch_count_batched(const StreamSubject *subs, int32_t nsub, const int2 *items, int64_t nitems,
                                const Overflow &ovf, int32_t coarse_words, int blocks, int batch, BatchedKind kind, hipStream_t st);
// table entries [lo, lo + n): Alg. 1's count of their streamlines [s_begin, S)
hipError_t launch_count_seed_end_batched(const StreamSubject *subs, int32_t lo, int32_t n, int cus, hipStream_t st);
hipError_t launch_fallback_batched(const StreamSubject *subs, int32_t nsub, const Overflow &ovf, FallbackScratch fs,
                                   hipStream_t st);

// ceiling probes (measurement only): the read-only point stream, no-return atomics C[idx[k]] += 1,
// and the stream with the compact-volume lookups of every point; sink: one device word
hipError_t launch_probe_stream(const float *pts, int64_t P, int cus, uint32_t *sink, hipStream_t st);
hipError_t launch_probe_atomics(int32_t *C, int64_t n_words, const uint32_t *idx, int64_t n, int cus, hipStream_t st);
hipError_t launch_probe_lookup(const StreamSubject &sub, int64_t P, int cus, uint32_t *sink, hipStream_t st);

hipError_t launch_validate(const int64_t *offsets, int64_t S, const int32_t *roi, const int32_t *lab,
                           int64_t nvox, int32_t N, int32_t M, int32_t *flags, int cus, hipStream_t st);

}  // namespace fc
