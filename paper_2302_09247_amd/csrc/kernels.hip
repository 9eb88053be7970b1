// Device code of libfastcod.so (gfx950, wave64): pass-through connectivity counting.
//
// The operation is FastCod's Alg. 2 (Section 2, "Method"): for every streamline, the set of ROI
// rows it passes through (passthrough) and the set of target labels it passes through
// (loc2region applied to its points) are formed, and every (row, label) pair of the two sets adds
// one to C.  The stages here:
//   * compact volume build: one pass over both volumes -> occupancy bits + packed codes;
//   * partition: tapering ranges of whole streamlines (one pass over the offsets; smaller calls' wavefronts
//     find a range each themselves); the same launch zeroes the call's per-call state;
//   * count kernels (wave-per-streamline over raster volumes, or flat point stream over the
//     compact volume): voxelise each point, look it up, de-duplicate the hits of each streamline
//     in a per-wavefront LDS hash set, and emit its |I| x |M| pair updates: the flat-stream
//     kernel appends them to per-wavefront slices of a pair buffer, the others (and a full slice)
//     add them into C with global atomics;
//   * pair histogram: the appended updates sorted by tile of C, workgroup by workgroup, then one LDS
//     histogram per tile added into C;
//   * fallback: streamlines with more distinct keys than the LDS set holds, one workgroup each,
//     with global bit maps.
// Integer counting is exact and additions commute, so every variant gives the same C.
#include "internal.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

namespace fc {

constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr uint32_t kLabelTag = 0x80000000u;

__device__ __forceinline__ int64_t clamp64(int64_t v, int64_t lo, int64_t hi) {
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// number of set bits of m below this lane
__device__ __forceinline__ int mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// this lane's bit of a wave-uniform mask, which the hardware takes directly as a lane predicate
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Global-memory views of pointers the compiler cannot place by itself (pointers read from a table
// in memory rather than passed as kernel arguments).  It would access them with flat instructions,
// which also count against the LDS wait counter: every LDS wait after one would wait for it too.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T *gview(const T *p) {
    return (const __attribute__((address_space(1))) T *)p;
}
// C[k] += 1 as a device-scope atomic without return, in global memory
__device__ __forceinline__ void add_one(int32_t *p) {
    __hip_atomic_fetch_add((__attribute__((address_space(1))) int32_t *)p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t lanes_between(int lo, int hi) {  // bits [lo, hi)
    const uint64_t below_hi = hi >= 64 ? ~0ull : ((1ull << hi) - 1ull);
    return below_hi & ~((1ull << lo) - 1ull);
}

__device__ __forceinline__ float load_stream(const float *p) { return __builtin_nontemporal_load(p); }

// Voxel of one point: per axis t = fl32(fl32(p*s) + 0.5) and floor(t), inside iff 0 <= t < size.
// (floor(t) >= 0 iff t >= 0, and floor(t) < size iff t < size; NaN fails both.)  __fmul_rn /
// __fadd_rn are never contracted into an FMA.
template <bool SCALED>
__device__ __forceinline__ bool voxelise(float x, float y, float z, float s, const Grid &g, int &ix,
                                         int &iy, int &iz) {
    if (SCALED) {
        x = __fmul_rn(x, s);
        y = __fmul_rn(y, s);
        z = __fmul_rn(z, s);
    }
    const float tx = __fadd_rn(x, 0.5f), ty = __fadd_rn(y, 0.5f), tz = __fadd_rn(z, 0.5f);
    const bool in = (tx >= 0.0f) & (tx < g.Xf) & (ty >= 0.0f) & (ty < g.Yf) & (tz >= 0.0f) & (tz < g.Zf);
    ix = in ? (int)tx : 0;  // truncation == floor for t >= 0
    iy = in ? (int)ty : 0;
    iz = in ? (int)tz : 0;
    return in;
}

// ---------------------------------------------------------------------------------------------
// volume lookups
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ void raster_get(const RasterVol &v, int ix, int iy, int iz, int &r, int &m) {
    const int lin = ix + v.X * iy + v.XY * iz;
    const int rv = v.roi[lin], mv = v.lab[lin];
    r = (unsigned)rv < (unsigned)v.N ? rv : -1;
    m = (unsigned)mv < (unsigned)v.M ? mv : -1;
}

__device__ __forceinline__ uint32_t compact_word(const CompactVol &c, int ix, int iy, int iz, uint32_t &bit) {
    const uint32_t sb = (uint32_t)(ix >> 4) + (uint32_t)c.SBX * (uint32_t)(iy >> 3) +
                        (uint32_t)c.SBXY * (uint32_t)(iz >> 3);
    const uint32_t b = (uint32_t)(ix & 15) | ((uint32_t)(iy & 7) << 4) | ((uint32_t)(iz & 7) << 7);
    bit = b & 31u;
    return (sb << 5) | (b >> 5);
}

__device__ __forceinline__ void compact_get(const CompactVol &c, int ix, int iy, int iz, int &r, int &m) {
    uint32_t bit;
    const uint32_t w = compact_word(c, ix, iy, iz, bit);
    const uint2 e = c.mb[w];
    r = -1;
    m = -1;
    if (!((e.x >> bit) & 1u)) return;
    const uint32_t rank = e.y + __popc(e.x & ((1u << bit) - 1u));
    const uint32_t code = c.codes[rank];
    const uint32_t rv = code & c.rmask, mv = code >> c.rbits;
    r = rv < (uint32_t)c.N ? (int)rv : -1;
    m = mv < (uint32_t)c.M ? (int)mv : -1;
}

struct RasterLookup {
    RasterVol v;
    __device__ void get(int ix, int iy, int iz, int &r, int &m) const { raster_get(v, ix, iy, iz, r, m); }
};
struct CompactLookup {
    CompactVol v;
    __device__ void get(int ix, int iy, int iz, int &r, int &m) const { compact_get(v, ix, iy, iz, r, m); }
};

// Row and label of the point at p (-1: none).
template <typename Lookup, bool SCALED>
__device__ __forceinline__ void lookup_point(const float *p, float scale, const Grid &g, const Lookup &lk, int &r,
                                             int &m) {
    int ix, iy, iz;
    r = m = -1;
    if (voxelise<SCALED>(p[0], p[1], p[2], scale, g, ix, iy, iz)) lk.get(ix, iy, iz, r, m);
}

// ---------------------------------------------------------------------------------------------
// per-wavefront set of the open streamline's distinct keys (LDS, open addressing)
//   key = row for ROI hits, label | kLabelTag for target hits (rows and labels are < 2^31 - 1)
//   slots[0 .. nI) hold the table slots of rows, slots[CAP/2 - nM .. CAP/2) those of labels;
//   nI + nM <= CAP/2 keeps the table at most half full, so probing always ends.
// ---------------------------------------------------------------------------------------------

template <int CAP>
struct WaveSet {
    static constexpr int kLog2 = __builtin_ctz(CAP);
    static constexpr int kHalf = CAP / 2;
    uint32_t *tab;
    uint32_t *slots;
    int nI, nM;
    bool skip;  // the open streamline overflowed: its hits are ignored until it closes

    __device__ void init(uint32_t *t, uint32_t *s) {
        tab = t;
        slots = s;
        nI = nM = 0;
        skip = false;
        for (int k = lane_id(); k < CAP; k += kWave) tab[k] = kEmpty;
    }

    // Insert the keys of the lanes in `cand`; returns the lanes whose key was not yet present.
    // The lanes still probing are a wave-uniform mask; the outcome ballots count those lanes only
    // (a lane outside `cand` may hold any value, kEmpty included, as its key).
    __device__ uint64_t insert(uint64_t cand, uint32_t key, uint32_t &slot) {
        uint64_t act = cand, fresh = 0ull;
        uint32_t h = (__umul24(key ^ (key >> 20), 0x9E3779u) >> 12) & (CAP - 1);
        while (act) {
            uint32_t old = 0u;
            if (in_mask(act)) old = atomicCAS(&tab[h], kEmpty, key);
            const uint64_t got = __ballot(old == kEmpty) & act, dup = __ballot(old == key) & act;
            if (in_mask(got)) slot = h;
            fresh |= got;
            act &= ~(got | dup);
            h = (h + 1u) & (CAP - 1);
        }
        return fresh;
    }

    // Adds the candidate rows / labels; false when the set could outgrow its capacity.
    __device__ bool add(uint64_t candR, int r, uint64_t candM, int m) {
        if (nI + nM + __popcll(candR) + __popcll(candM) > kHalf) return false;
        uint32_t slotR = 0, slotM = 0;
        const uint64_t newR = candR ? insert(candR, (uint32_t)r, slotR) : 0ull;
        const uint64_t newM = candM ? insert(candM, (uint32_t)m | kLabelTag, slotM) : 0ull;
        if (in_mask(newR)) slots[nI + mbcnt(newR)] = slotR;
        if (in_mask(newM)) slots[kHalf - 1 - (nM + mbcnt(newM))] = slotM;
        nI += __popcll(newR);
        nM += __popcll(newM);
        return true;
    }

    __device__ void clear_entries() {
        for (int k = lane_id(); k < nI; k += kWave) tab[slots[k]] = kEmpty;
        for (int k = lane_id(); k < nM; k += kWave) tab[slots[kHalf - 1 - k]] = kEmpty;
        nI = nM = 0;
    }

    // The streamline ends: C(i, m) += 1 for all its rows i and labels m (through `sink`), then reset.
    template <typename Sink>
    __device__ void close(Sink &sink, uint32_t si, uint32_t sm) {
        if (!skip && nI > 0 && nM > 0) {
            for (int b = 0; b < nI; b += kWave) {
                const int k = b + lane_id();
                const uint64_t ok = __ballot(k < nI);
                const uint32_t i = in_mask(ok) ? tab[slots[k]] : 0u;
                const uint32_t row = i * si;   // N*M < 2^31
                for (int j = 0; j < nM; ++j) {
                    const uint32_t mk = __builtin_amdgcn_readfirstlane(tab[slots[kHalf - 1 - j]]) & ~kLabelTag;
                    sink.push_lanes(ok, row + mk * sm);
                }
            }
        }
        clear_entries();
        skip = false;
    }
};

// C updates straight to global memory (one atomic per pair).
struct DirectSink {
    int32_t *C;
    __device__ void push_lanes(uint64_t vm, uint32_t idx) {   // the lanes in vm (wave-uniform)
        if (in_mask(vm)) add_one(C + idx);
    }
    __device__ void push(bool valid, uint32_t idx) { push_lanes(__ballot(valid), idx); }
};

// C updates buffered per wavefront in LDS and issued 64 at a time: a wave-wide atomic
// instruction instead of one per closing streamline.  On this architecture every vector memory
// wait also waits for older atomics, so fewer, fuller atomic instructions stall the stream less.
struct BufferedSink {
    uint32_t *buf;  // [kWave] LDS
    int n;          // pending entries (wave-uniform)
    int32_t *C;
    __device__ void init(uint32_t *b, int32_t *c) {
        buf = b;
        n = 0;
        C = c;
    }
    __device__ void push(bool valid, uint32_t idx) { push_lanes(__ballot(valid), idx); }
    __device__ void push_lanes(uint64_t vm, uint32_t idx) {   // the lanes in vm (wave-uniform)
        if (!vm) return;
        const bool valid = in_mask(vm);
        const int pos = n + mbcnt(vm);
        if (valid && pos < kWave) buf[pos] = idx;
        const int cnt = __popcll(vm);
        if (n + cnt >= kWave) {
            add_one(C + buf[lane_id()]);
            if (valid && pos >= kWave) buf[pos - kWave] = idx;
            n = n + cnt - kWave;
        } else {
            n += cnt;
        }
    }
    __device__ void drain() {
        if (lane_id() < n) add_one(C + buf[lane_id()]);
        n = 0;
    }
};

// C updates appended to this wavefront's slice of a pair buffer for a later histogram pass,
// kSinkCap at a time: 16 bytes per lane per store instruction, one store per 256 updates.  On this
// architecture every later vector-memory wait also waits for older stores, so fewer, fuller
// stores stall the stream less (a cached store is acknowledged once the cache takes it; an atomic
// must first fetch its line of C).  Once the slice is full, updates go to C as atomics.
// (kSinkCap: 256 or 512, a multiple of 256; the LDS it takes limits the workgroups per CU.)
template <int kSinkCap>
struct AppendSink {
    static_assert(kSinkCap == 4 * kWave || kSinkCap == 8 * kWave, "one or two 16-byte stores per lane");
    uint32_t *buf;   // [kSinkCap] LDS, 16-byte aligned
    int n;           // pending entries (wave-uniform)
    uint32_t *out;   // next free entry of this wavefront's slice (16-byte aligned)
    uint32_t room;   // free entries left in the slice
    int32_t *C;
    __device__ void init(uint32_t *b, int32_t *c, const PairOut &po, uint32_t wave) {
        buf = b;
        n = 0;
        C = c;
        out = po.pairs + (size_t)wave * po.cap;   // (po.cap is a multiple of 8)
        room = po.cap;
    }
    __device__ void emit(int cnt) {   // the first cnt (<= kSinkCap) entries of buf
        const int lane = lane_id();
        if (cnt == kSinkCap && (uint32_t)cnt <= room) {
            const uint4 v = reinterpret_cast<const uint4 *>(buf)[lane];
            if constexpr (kSinkCap == 8 * kWave) {
                const uint4 v2 = reinterpret_cast<const uint4 *>(buf)[lane + kWave];
                reinterpret_cast<uint4 *>(out)[lane] = v;
                reinterpret_cast<uint4 *>(out)[lane + kWave] = v2;
            } else {
                reinterpret_cast<uint4 *>(out)[lane] = v;
            }
            out += kSinkCap;
            room -= (uint32_t)kSinkCap;
        } else if ((uint32_t)cnt <= room) {
            for (int k = lane; k < cnt; k += kWave) out[k] = buf[k];
            out += cnt;
            room -= (uint32_t)cnt;
        } else {
            for (int k = lane; k < cnt; k += kWave) add_one(C + buf[k]);
        }
    }
    __device__ void push(bool valid, uint32_t idx) { push_lanes(__ballot(valid), idx); }
    __device__ void push_lanes(uint64_t vm, uint32_t idx) {   // the lanes in vm (wave-uniform)
        if (!vm) return;
        const bool valid = in_mask(vm);
        const int pos = n + mbcnt(vm);
        if (valid && pos < kSinkCap) buf[pos] = idx;
        const int cnt = __popcll(vm);
        if (n + cnt >= kSinkCap) {
            emit(kSinkCap);
            if (valid && pos >= kSinkCap) buf[pos - kSinkCap] = idx;
            n = n + cnt - kSinkCap;
        } else {
            n += cnt;
        }
    }
    // flushes the pending entries and records the slice's length
    __device__ void drain(const PairOut &po, uint32_t wave) {
        if (n) emit(n);
        n = 0;
        if (lane_id() == 0) po.counts[wave] = po.cap - room;
    }
};

// Per-wavefront state of the flat-stream kernel's open streamline: raw candidate lists (hits
// that differ from the previous point's), de-duplicated only when the streamline closes and only
// if it has both rows and labels.  tab is an open-addressing set, empty between closes; it holds
// at most RCAP + LCAP <= TCAP/2 keys, so probing always ends.
template <int RCAP, int LCAP, int TCAP>
struct DeferredSet {
    static_assert(RCAP + LCAP <= TCAP / 2, "set must stay at most half full");
    uint32_t *rows;   // [RCAP] raw row candidates; at close: table slot of each new row, or kEmpty
    uint32_t *labs;   // [LCAP] raw label candidates; at close: table slot of each new label, or kEmpty
    uint32_t *ulab;   // [LCAP] distinct labels (at close)
    uint32_t *tab;    // [TCAP]
    int nR, nL;
    bool skip;        // the open streamline overflowed: its hits go to the fallback kernel

    __device__ void init(uint32_t *base) {
        rows = base;
        labs = rows + RCAP;
        ulab = labs + LCAP;
        tab = ulab + LCAP;
        nR = nL = 0;
        skip = false;
        for (int k = lane_id(); k < TCAP; k += kWave) tab[k] = kEmpty;
    }
    __device__ bool has_state() const { return (nR | nL) != 0 || skip; }

    // Endpoint modes: the open streamline's labels are its end labels (ml, mf; -1 = none) instead of
    // its points' labels (none were appended).  Nothing to do without rows.
    __device__ void add_end_labels(int ml, int mf) {
        if (skip || nR == 0) return;
        const int addl = ml >= 0 ? 1 : 0, addf = (mf >= 0 && mf != ml) ? 1 : 0;
        if (lane_id() == 0) {
            if (addl) labs[nL] = (uint32_t)ml;
            if (addf) labs[nL + addl] = (uint32_t)mf;
        }
        nL += addl + addf;
    }

    // Appends the candidates of the lanes in cR (rows) and cM (labels); false when a list is full.
    __device__ bool append(uint64_t cR, int r, uint64_t cM, int m) {
        const int addR = __popcll(cR), addM = __popcll(cM);
        if (nR + addR > RCAP || nL + addM > LCAP) return false;
        if (in_mask(cR)) rows[nR + mbcnt(cR)] = (uint32_t)r;
        if (in_mask(cM)) labs[nL + mbcnt(cM)] = (uint32_t)m;
        nR += addR;
        nL += addM;
        return true;
    }

    __device__ static uint32_t slot_of(uint32_t key) {
        return (key ^ (key >> 9) ^ (key >> 18) ^ (key >> 27)) & (TCAP - 1);
    }
    // Inserts the key of every lane in `cand`; returns the lanes whose key was new (slot set).
    // The lanes still probing are a wave-uniform mask; the outcome ballots count those lanes only
    // (a lane outside `cand` may hold any value as its key).  Each lane's slot ends where its key
    // was found or put.
    __device__ uint64_t insert(uint64_t cand, uint32_t key, uint32_t &slot) const {
        uint64_t act = cand, fresh = 0ull;
        uint32_t h = slot_of(key);
        while (act) {
            uint32_t old = 0u;
            if (in_mask(act)) {
                old = atomicCAS(&tab[h], kEmpty, key);
                slot = h;
            }
            const uint64_t got = __ballot(old == kEmpty) & act, dup = __ballot(old == key) & act;
            fresh |= got;
            act &= ~(got | dup);
            h = (h + 1u) & (TCAP - 1);
        }
        return fresh;
    }

    // The streamline ends: C(i, m) += 1 for each distinct row i and distinct label m, then reset.
    template <typename Sink>
    __device__ void close(Sink &sink, uint32_t si, uint32_t sm) {
        if (!skip && nR > 0 && nL > 0) {
            const int lane = lane_id();
            int nU = 0;
            // (lane conditions as wave-uniform masks throughout: no per-lane booleans carried
            // across loads and loops)
            for (int b = 0; b < nL; b += kWave) {
                const int k = b + lane;
                const uint64_t ok = __ballot(k < nL);
                const uint32_t m = in_mask(ok) ? labs[k] : 0u;
                uint32_t slot = 0;
                const uint64_t fresh = insert(ok, m | kLabelTag, slot);
                if (in_mask(fresh)) ulab[nU + mbcnt(fresh)] = m;
                if (in_mask(ok)) labs[k] = in_mask(fresh) ? slot : kEmpty;
                nU += __popcll(fresh);
            }
            const float rcp = 1.0f / (float)nU;
            for (int b = 0; b < nR; b += kWave) {
                const int k = b + lane;
                const uint64_t ok = __ballot(k < nR);
                const uint32_t i = in_mask(ok) ? rows[k] : 0u;
                uint32_t slot = 0;
                const uint64_t fresh = insert(ok, i, slot);
                if (in_mask(ok)) rows[k] = in_mask(fresh) ? slot : kEmpty;
                // the nF new rows x the nU distinct labels, 64 pairs per push.  The new rows move to
                // lanes 0 .. nF-1 (a permutation of all 64 lanes: the others fill nF .. 63); pair q is
                // row q / nU and label q % nU.  q < 4096, so the float quotient is at most one low,
                // and only at exact multiples of nU.
                const int nF = __popcll(fresh);
                if (nF == 0) continue;
                const int to = in_mask(fresh) ? mbcnt(fresh) : nF + mbcnt(~fresh);
                const int frow = __builtin_amdgcn_ds_permute(to << 2, (int)(i * si));   // N*M < 2^31
                const int tot = nF * nU;
                for (int q0 = 0; q0 < tot; q0 += kWave) {
                    const int q = q0 + lane;
                    const uint64_t live = __ballot(q < tot);
                    int rq = (int)((float)q * rcp);
                    rq += (rq + 1) * nU <= q ? 1 : 0;
                    const int uq = q - rq * nU;
                    const uint32_t row = (uint32_t)__builtin_amdgcn_ds_bpermute((in_mask(live) ? rq : 0) << 2, frow);
                    const uint32_t lab = ulab[in_mask(live) ? uq : 0];
                    sink.push_lanes(live, row + lab * sm);
                }
            }
            for (int k = lane; k < nL; k += kWave)
                if (labs[k] != kEmpty) tab[labs[k]] = kEmpty;
            for (int k = lane; k < nR; k += kWave)
                if (rows[k] != kEmpty) tab[rows[k]] = kEmpty;
        }
        nR = nL = 0;
        skip = false;
    }
};

// Queue entries: point index in bits 0..47, subject in bits 48..62.
constexpr int kSubjectShift = 48;
__device__ __forceinline__ void push_overflow(const Overflow &o, int64_t point_index, int32_t subject = 0) {
    if (lane_id() == 0) {
        const unsigned long long k = atomicAdd(o.count, 1ull);
        if ((int64_t)k < o.cap) o.list[k] = point_index | ((int64_t)subject << kSubjectShift);
    }
}

// ---------------------------------------------------------------------------------------------
// fills
// ---------------------------------------------------------------------------------------------

__global__ void k_fill_i32(int32_t *__restrict__ p, int64_t n, int32_t v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ void k_fill_u64(unsigned long long *__restrict__ p, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

static int fill_blocks(int64_t n, int cus) {
    int64_t b = (n + kBlock - 1) / kBlock;
    const int64_t cap = (int64_t)cus * 16;
    if (b > cap) b = cap;
    return (int)(b < 1 ? 1 : b);
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, int cus, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    k_fill_i32<<<fill_blocks(n, cus), kBlock, 0, st>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, int cus, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    k_fill_u64<<<fill_blocks(n, cus), kBlock, 0, st>>>(p, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// compact volume build
// ---------------------------------------------------------------------------------------------

// One pass over both volumes: each voxel is read once, and its occupancy bit, rank base and code are
// written from registers.  A workgroup takes 8 super-bricks along x; each of its 8 wavefronts takes 64
// voxels along x (4 super-bricks) of 8 rows and 2 slices: 4 steps of 4 rows, 4 voxels (16 bytes) per
// lane.  Lane 16 r + q holds voxels 4 q .. 4 q + 3 of row r; the 8 lanes of a row pair and super-brick
// (a group) share one occupancy word per step.  The workgroups' codes lie in the order in which they
// reserve room for them (only each word's base has to know it), a workgroup's super-brick by
// super-brick: the counting kernel's neighbouring lookups then share lines.
//
// Bound by the read of the volumes.  The five launches it replaces (zero fill, occupancy marks as
// atomics, popcounts, scan, codes with a second read of the occupied voxels) had taken 71 us on a
// 260x311x260 grid, 30 us on 145x174x145 and 18 us on 64^3.  A reservation and coarse bits of its own
// for every wavefront took 75, 27 and 11 us: atomics on one line are served one after another.
// kWide: rows of at least 4 voxels; a lane whose voxels pass the end of the row then takes its last 4
// (16-byte loads need only the 4-byte alignment of the elements).
// kNt: non-temporal loads, for more than kBuildCachedVoxels in a call of at least kBuildCachedStreamlines.
// Cached, 168 MB of volumes (260x311x260) displace the offsets and the zeroed C of a large call from the
// last-level cache: the build takes 36 instead of 42 us, but 5M streamlines of 220 points take 2609 instead
// of 2594 a call.  Smaller calls leave room for both: cached, 100,000 streamlines on that grid take 117 instead of
// 125 us, 1M 414 and 424, 3M 1052 and 1060, 5M of 150 points 1698 and 1702; 100,000 on 210x240x200 98 and 103.
// coarse[] and *ncodes are zero on entry.
constexpr int kBuildSteps = 4;                   // steps of a wavefront: two a slice
constexpr int kBuildParts = 16 / kBuildSteps;    // wavefronts per super-brick along z
constexpr int kBuildWaves = 2 * kBuildParts;     // two 64-voxel chunks along x
constexpr int64_t kBuildCachedVoxels = int64_t(1) << 23;   // 64 MB of volumes
constexpr int64_t kBuildCachedStreamlines = int64_t(1) << 22;
template <bool kWide, bool kNt>
__global__ void __launch_bounds__(kBuildWaves *kWave)
k_compact_build(const int32_t *__restrict__ roi, const int32_t *__restrict__ lab, Grid g, CompactVol cv, int32_t SBY,
                uint2 *__restrict__ mb, uint32_t *__restrict__ codes, uint32_t *__restrict__ coarse,
                uint32_t *__restrict__ ncodes) {
    __shared__ uint32_t s_cnt[8 * kBuildParts];   // codes of (super-brick, part)
    __shared__ uint32_t s_any[kBuildWaves];       // occupied 8-voxel halves of a wavefront's super-bricks
    __shared__ uint32_t s_base;
    constexpr int kSteps = kBuildSteps;
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int part = wv >> 1;
    const int32_t nxg = (cv.SBX + 7) >> 3;
    const int32_t xg = (int32_t)(blockIdx.x % (uint32_t)nxg), t = (int32_t)(blockIdx.x / (uint32_t)nxg);
    const int32_t sby = t % SBY, sbz = t / SBY;
    const int32_t xc = 2 * xg + (wv & 1);
    const int q = lane & 15, rr = lane >> 4;
    const int32_t x = xc * 64 + 4 * q;
    const RowLane rl = row_lane<kWide>(x, g.X);
    const int32_t xs = rl.xs;
    const int d = rl.d;
    const uint32_t mine = rl.mine;
    uint32_t code[kSteps][4];
    uint32_t word[kSteps];
    uint32_t occ = 0u;   // 4 bits a step: this lane's occupied elements
    const int at_bit = 4 * (q & 3) + 16 * (rr & 1);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        const int32_t y = sby * 8 + 4 * (st & 1) + rr, z = sbz * 8 + part * (kSteps / 2) + (st >> 1);
        // (rows past the grid are read at its last row, and not occupied)
        const int32_t row = g.X * (min(y, g.Y - 1) + g.Y * min(z, g.Z - 1));
        int32_t r[4], m[4];
        if (kWide) {
            typedef int32_t v4i __attribute__((ext_vector_type(4), aligned(4)));
            const v4i *pr = reinterpret_cast<const v4i *>(roi + (row + xs)), *pm = reinterpret_cast<const v4i *>(lab + (row + xs));
            const v4i r4 = kNt ? __builtin_nontemporal_load(pr) : *pr, m4 = kNt ? __builtin_nontemporal_load(pm) : *pm;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                r[i] = r4[i];
                m[i] = m4[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int32_t xi = min(xs + i, g.X - 1);
                r[i] = roi[row + xi];
                m[i] = lab[row + xi];
            }
        }
        uint32_t o = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool rv = (unsigned)r[i] < (unsigned)cv.N, mv = (unsigned)m[i] < (unsigned)cv.M;
            // (all ones: neither a row nor a label, as both fields hold a value that is none)
            code[st][i] = (rv ? (uint32_t)r[i] : cv.rmask) |
                          ((mv ? (uint32_t)m[i] : (0xFFFFFFFFu >> cv.rbits)) << cv.rbits);
            o |= min(~code[st][i], 1u) << i;
        }
        o &= (y < g.Y && z < g.Z) ? mine : 0u;
        occ |= o << (4 * st);
        uint32_t w = (o >> d) << at_bit;
        w |= (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
        w |= (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
        w |= (uint32_t)__builtin_amdgcn_ds_swizzle((int)w, 0x401F);              // lane ^ 16
        word[st] = w;
    }
    // codes of this part of each super-brick: its two groups' (rows 0, 1 and rows 2, 3 of a step)
    uint32_t cnt = 0u, any = 0u;
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        cnt += (uint32_t)__popc(word[st]);
        any |= word[st];
    }
    const uint32_t other = (uint32_t)__shfl_xor((int)cnt, 32);
    const int sb = 4 * (wv & 1) + (q >> 2);   // super-brick within the workgroup
    const uint64_t lo = __ballot((any & 0x00FF00FFu) != 0u), hi = __ballot((any & 0xFF00FF00u) != 0u);
    if (rr == 0 && (q & 3) == 0) s_cnt[sb * kBuildParts + part] = cnt + other;
    if (lane == 0) {
        uint32_t halves = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // lanes 4 k (rows 0, 1) and 4 k + 32 (rows 2, 3) are super-brick k's
            halves |= (uint32_t)(((lo | lo >> 32) >> (4 * k)) & 1ull) << (2 * k);
            halves |= (uint32_t)(((hi | hi >> 32) >> (4 * k)) & 1ull) << (2 * k + 1);
        }
        s_any[wv] = halves;
    }
    __syncthreads();
    uint32_t incl = lane < 8 * kBuildParts ? s_cnt[lane] : 0u;
    const uint32_t own = incl;
#pragma unroll
    for (int k = 1; k < 8 * kBuildParts; k <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)incl, k);
        if (lane >= k) incl += u;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 8 * kBuildParts - 1);
    uint32_t base = (uint32_t)__shfl((int)(incl - own), sb * kBuildParts + part) + (rr >= 2 ? other : 0u);
    if (total) {   // (uniform over the workgroup)
        if (threadIdx.x == 0) {
            s_base = atomicAdd(ncodes, total);
            // coarse bits of the 16 halves: blocks of 8 << (csx - 3) voxels along x, one run of bits
            uint32_t halves = 0u, bits = 0u;
            for (int w = 0; w < kBuildWaves; ++w) halves |= s_any[w] << (8 * (w & 1));
            for (int h = 0; h < 16; ++h) bits |= ((halves >> h) & 1u) << (h >> (cv.csx - 3));
            const uint32_t cb = (uint32_t)((xg * 128) >> cv.csx) + (uint32_t)cv.CBX * (uint32_t)((sby * 8) >> cv.csyz) +
                                (uint32_t)cv.CBXY * (uint32_t)((sbz * 8) >> cv.csyz);
            const uint64_t run = (uint64_t)bits << (cb & 31u);
            if ((uint32_t)run) atomicOr(&coarse[cb >> 5], (uint32_t)run);
            if (run >> 32) atomicOr(&coarse[(cb >> 5) + 1], (uint32_t)(run >> 32));
        }
        __syncthreads();
        base += s_base;
    }
    // each lane of a group writes the {word, base} pair of one step
    const int32_t sbx = xc * 4 + (q >> 2);
    const int sel = (q & 3) + 4 * (rr & 1);
    uint32_t bases[kSteps];
    uint2 pair = make_uint2(0u, 0u);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        bases[st] = base;
        base += (uint32_t)__popc(word[st]);
        if (sel == st) pair = make_uint2(word[st], bases[st]);
    }
    if (sbx < cv.SBX && sel < kSteps)
        mb[(((int64_t)sbx + (int64_t)cv.SBX * sby + (int64_t)cv.SBXY * sbz) << 5) + part * (2 * kSteps) +
           2 * sel + (rr >> 1)] = pair;
    if (!total) return;
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        const uint32_t o = (occ >> (4 * st)) & 0xFu;
        if (!o) continue;
        uint32_t at = bases[st] + (uint32_t)__popc(word[st] & ((1u << at_bit) - 1u));
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if ((o >> i) & 1u) codes[at++] = code[st][i];
    }
}

hipError_t launch_compact_build(const int32_t *roi, const int32_t *lab, Grid g, CompactVol cv, uint2 *mb, uint32_t *codes,
                                uint32_t *coarse, uint32_t *ncodes, int64_t S, hipStream_t st) {
    const int32_t SBY = cv.SBXY / cv.SBX;
    const int64_t SBZ = cv.W / 32 / cv.SBXY;
    const unsigned blocks = (unsigned)((int64_t)((cv.SBX + 7) / 8) * SBY * SBZ);
    const bool wide = g.X >= 4;
    const bool nt = S >= kBuildCachedStreamlines && (int64_t)g.X * g.Y * g.Z > kBuildCachedVoxels;
#define FC_BUILD(W_, T_) \
    k_compact_build<W_, T_><<<blocks, kBuildWaves * kWave, 0, st>>>(roi, lab, g, cv, SBY, mb, codes, coarse, ncodes)
    if (wide && nt) FC_BUILD(true, true);
    else if (wide) FC_BUILD(true, false);
    else FC_BUILD(false, false);
#undef FC_BUILD
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// partition: first[i] = first streamline of point range i (i < nparts), first[nparts] = S, with
// P = offsets[S] read on the device (launches stay asynchronous)
// ---------------------------------------------------------------------------------------------

// Streamlines from which a thread of the partition launch takes four of them: up to there one each makes no
// more wavefronts than the device holds at once, and a wavefront's ranges are written sooner.
constexpr int64_t kPartitionUnrollFrom = int64_t(1) << 20;

// p[0 .. n) = 0 by the whole grid, 16 bytes a store
__device__ __forceinline__ void grid_zero(int32_t *p, int64_t n, int64_t t0, int64_t stride) {
    const int64_t head = min(n, (int64_t)((0u - (uint32_t)(reinterpret_cast<uintptr_t>(p) >> 2)) & 3u));
    const int64_t n4 = (n - head) >> 2;
    int4 *p4 = reinterpret_cast<int4 *>(p + head);
    for (int64_t i = t0; i < n4; i += stride) p4[i] = make_int4(0, 0, 0, 0);
    if (t0 < head) p[t0] = 0;
    if (t0 < n - head - 4 * n4) p[head + 4 * n4 + t0] = 0;
}

// Bound by latency (and by the zero fill of C on large ones), so the offsets are read once, in order:
// the thread of streamline s knows the ranges that begin with it, those in (range(s - 1), range(s)].
// A binary search per range, 13 to 20 dependent loads, took 6.4 us on 1k-10k streamlines and 12 us on
// 1M.  Streamlines that begin up to kOwn ranges write them side by side, one that begins more (a giant one
// before it) has its whole wavefront write them: with a whole wavefront for every streamline that begins more
// than two, one after another, and four streamlines a thread, long streamlines in a row held a few wavefronts
// up (57,400 streamlines, 4000 of them ten times as long, took 75 us a call, now 56, the search 59; 33,000
// ordinary ones 49, now 38, the search 40).  first == nullptr: only the zero fills.
template <int kUnroll>
__global__ void k_partition(const int64_t *__restrict__ offsets, int64_t S, int64_t nparts, int32_t *__restrict__ first,
                            ZeroRanges z) {
    constexpr int kShort = 2, kOwn = 8;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = lane_id();
    const RangeOf range_of(first ? offsets[S] : 0, nparts);
    for (int64_t b0 = first ? kUnroll * (t0 - lane) : S + 1; b0 <= S; b0 += kUnroll * stride) {   // (uniform over the wavefront)
        int64_t off[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) off[j] = offsets[min(b0 + j * kWave + lane, S)];
        int32_t before = b0 > 0 ? range_of(offsets[b0 - 1]) : -1;   // range of the streamline before the wavefront's
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            const int64_t s = b0 + j * kWave + lane;
            const int32_t hi = s < S ? range_of(off[j]) : (int32_t)nparts;
            const int32_t lo = __builtin_amdgcn_update_dpp(before, hi, 0x138, 0xF, 0xF, false) + 1;   // wave_shr:1
            before = __builtin_amdgcn_readlane(hi, kWave - 1);
            const bool mine = s <= S;
#pragma unroll
            for (int k = 0; k < kShort; ++k)
                if (mine && lo + k <= hi) first[lo + k] = (int32_t)s;
            if (!__ballot(mine && lo + kShort <= hi)) continue;
#pragma unroll 1
            for (int k = kShort; k < kOwn; ++k)
                if (mine && lo + k <= hi) first[lo + k] = (int32_t)s;
            uint64_t rest = __ballot(mine && lo + kOwn <= hi);
            while (rest) {
                const int k = __builtin_ctzll(rest);
                rest &= rest - 1ull;
                const int32_t l = __builtin_amdgcn_readlane(lo, k), h = __builtin_amdgcn_readlane(hi, k);
                for (int32_t i = l + kOwn + lane; i <= h; i += kWave) first[i] = (int32_t)(b0 + j * kWave + k);
            }
        }
    }
    // (the zero fills come last: a wait for a load also waits for the stores before it)
#pragma unroll
    for (int r = 0; r < kZeroRanges; ++r) grid_zero(z.w32[r], z.n32[r], t0, stride);
    for (int64_t i = t0; i < z.n64; i += stride) z.w64[i] = 0ull;
}

hipError_t launch_partition(const int64_t *offsets, int64_t S, int64_t nparts, int32_t *first, const ZeroRanges &z,
                            int cus, hipStream_t st) {
    const int unroll = S < kPartitionUnrollFrom ? 1 : 4;
    int64_t n = std::max(first ? (S + unroll) / unroll : int64_t(1), z.n64);
    for (int64_t k : z.n32) n = std::max(n, (k + 3) / 4);
    if (unroll == 1) k_partition<1><<<fill_blocks(n, cus), kBlock, 0, st>>>(offsets, S, nparts, first, z);
    else k_partition<4><<<fill_blocks(n, cus), kBlock, 0, st>>>(offsets, S, nparts, first, z);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// count, variant 1: one wavefront per streamline, raster lookups
// ---------------------------------------------------------------------------------------------

constexpr int kMaxUp = 4;   // largest upsampling factor

template <bool SCALED>
__global__ void __launch_bounds__(kBlock) k_count_wave(CountArgs a, RasterVol rv) {
    __shared__ uint32_t s_tab[kWavesPerBlock * kSetCap];
    __shared__ uint32_t s_slots[kWavesPerBlock * (kSetCap / 2)];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    WaveSet<kSetCap> set;
    set.init(s_tab + wv * kSetCap, s_slots + wv * (kSetCap / 2));
    DirectSink sink{a.C};
    const int64_t Ptot = a.offsets[a.S] > 0 ? a.offsets[a.S] : 0;
    const int64_t nw = (int64_t)gridDim.x * kWavesPerBlock;
    const bool endmode = a.end_mode != 0;   // endpoint modes: the labels are looked up at the close
    const int up = a.up < 1 ? 1 : (a.up > kMaxUp ? kMaxUp : a.up);   // upsampling factor
    for (int64_t s = (int64_t)blockIdx.x * kWavesPerBlock + wv; s < a.S; s += nw) {
        const int64_t b0 = clamp64(a.offsets[s], 0, Ptot);
        const int64_t b1 = clamp64(a.offsets[s + 1], b0, Ptot);
        int last_r = -1, last_m = -1;
        for (int64_t w0 = b0; w0 < b1; w0 += kWave) {
            const int64_t p = w0 + lane;
            const bool here = p < b1, next = p + 1 < b1;
            // the lane's scaled point and (upsampling) the step to the next one
            float qx = 0.f, qy = 0.f, qz = 0.f, dx = 0.f, dy = 0.f, dz = 0.f;
            if (here) {
                qx = load_stream(a.pts + 3 * p);
                qy = load_stream(a.pts + 3 * p + 1);
                qz = load_stream(a.pts + 3 * p + 2);
                if (SCALED) {
                    qx = __fmul_rn(qx, a.scale);
                    qy = __fmul_rn(qy, a.scale);
                    qz = __fmul_rn(qz, a.scale);
                }
                if (up > 1 && next) {
                    float ux = a.pts[3 * p + 3], uy = a.pts[3 * p + 4], uz = a.pts[3 * p + 5];
                    if (SCALED) {
                        ux = __fmul_rn(ux, a.scale);
                        uy = __fmul_rn(uy, a.scale);
                        uz = __fmul_rn(uz, a.scale);
                    }
                    dx = __fsub_rn(ux, qx);
                    dy = __fsub_rn(uy, qy);
                    dz = __fsub_rn(uz, qz);
                }
            }
            // sub-point t: the point itself (t = 0) or a_t of the way to the next one
            int rr[kMaxUp], mm[kMaxUp];
#pragma unroll
            for (int t = 0; t < kMaxUp; ++t) {
                rr[t] = mm[t] = -1;
                if (t < up && here && (t == 0 || next)) {
                    float x = qx, y = qy, z = qz;
                    if (t > 0) {
                        const float at = (float)((double)t / (double)up);
                        x = __fadd_rn(qx, __fmul_rn(at, dx));
                        y = __fadd_rn(qy, __fmul_rn(at, dy));
                        z = __fadd_rn(qz, __fmul_rn(at, dz));
                    }
                    int ix, iy, iz, r, m;
                    if (voxelise<false>(x, y, z, 1.0f, a.g, ix, iy, iz)) {
                        raster_get(rv, ix, iy, iz, r, m);
                        rr[t] = r;
                        mm[t] = endmode ? -1 : m;
                    }
                }
            }
            int rl = rr[0], ml = mm[0];   // the lane's last sub-point
#pragma unroll
            for (int t = 1; t < kMaxUp; ++t)
                if (t == up - 1) {
                    rl = rr[t];
                    ml = mm[t];
                }
            // drop a hit equal to the hit before it in streamline order, then the LDS set
            int rp = __shfl_up(rl, 1), mp = __shfl_up(ml, 1);
            if (lane == 0) {
                rp = last_r;
                mp = last_m;
            }
            last_r = __shfl(rl, kWave - 1);
            last_m = __shfl(ml, kWave - 1);
#pragma unroll
            for (int t = 0; t < kMaxUp; ++t) {
                if (t >= up) break;
                const int pr = t == 0 ? rp : rr[t > 0 ? t - 1 : 0], pm = t == 0 ? mp : mm[t > 0 ? t - 1 : 0];
                const uint64_t candR = __ballot(rr[t] >= 0 && rr[t] != pr);
                const uint64_t candM = __ballot(mm[t] >= 0 && mm[t] != pm);
                if ((candR | candM) == 0ull || set.skip) continue;
                if (!set.add(candR, rr[t], candM, mm[t])) {
                    push_overflow(a.ovf, b0);
                    set.clear_entries();
                    set.skip = true;
                }
            }
        }
        if (endmode && !set.skip && set.nI > 0) {
            // (rows were found, so the streamline has points)
            int r, ml, mf = -1;
            const RasterLookup lk{rv};
            lookup_point<RasterLookup, SCALED>(a.pts + 3 * (b1 - 1), a.scale, a.g, lk, r, ml);
            if (a.end_mode == 2) lookup_point<RasterLookup, SCALED>(a.pts + 3 * b0, a.scale, a.g, lk, r, mf);
            const uint64_t cand = __ballot((lane == 0 && ml >= 0) || (lane == 1 && mf >= 0 && mf != ml));
            if (cand && !set.add(0ull, 0, cand, lane == 0 ? ml : mf)) {
                push_overflow(a.ovf, b0);
                set.clear_entries();
                set.skip = true;
            }
        }
        set.close(sink, a.si, a.sm);
    }
}

hipError_t launch_count_wave(const CountArgs &a, const RasterVol &rv, int blocks, hipStream_t st) {
    if (a.scale != 1.0f) k_count_wave<true><<<blocks, kBlock, 0, st>>>(a, rv);
    else k_count_wave<false><<<blocks, kBlock, 0, st>>>(a, rv);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// count, variant 2: flat point stream over ranges of whole streamlines
// ---------------------------------------------------------------------------------------------
//
// A wavefront takes contiguous ranges of whole streamlines, from the table or one of its own.  It walks a
// range in batches of kBatch 64-point windows regardless of streamline boundaries.  Per batch: voxelise, occupancy-bit gathers (a 2-3 MB structure that stays in L2),
// and for the few flagged lanes the rank and code gathers; only then are the next batch's
// streaming loads issued (vector loads return in issue order, so no gather wait of this batch
// covers them), and the windows are folded into the open streamline's LDS set while they are in
// flight.  The streamline starts inside a window come from a block of 64 offsets held one per
// lane; each start closes the open streamline.
//
// All global reads go through buffer resources: out-of-range offsets read zero instead of
// faulting, so the point stream needs no per-lane clamping (lanes past the range are masked by
// their index) and a lane's load offset is one constant register plus a scalar batch offset.

constexpr uint32_t kRsrcWord3 = 0x00020000u;   // raw 32-bit buffer, gfx9-family descriptor
constexpr int kAuxStream = 2;                  // non-temporal: points are read once
constexpr int kAuxCached = 0;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint64_t bytes) {
    const uint32_t n = bytes > 0xFFFFFFF0ull ? 0xFFFFFFF0u : (uint32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)n, (int)kRsrcWord3);
}

__device__ __forceinline__ uint32_t fbits(float f) { return __float_as_uint(f); }

// wave-uniform copies (the values are uniform already; this tells the compiler)
__device__ __forceinline__ int uniform32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t readlane64(int64_t v, int k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), k);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Next point range (work item) of wavefront `wave`: queue c = wave mod Q holds ranges c, c + Q,
// c + 2Q, ..., handed out in that order by its own counter (Q: kRangeQueues, or the largest power of
// two not above the grid's wavefronts, so that every queue has wavefronts).
__device__ __forceinline__ int64_t next_range(const Overflow &ovf, uint32_t wave) {
    const uint32_t nw = gridDim.x * (uint32_t)kWavesPerBlock;
    const uint32_t q = nw >= (uint32_t)kRangeQueues ? (uint32_t)kRangeQueues : (1u << (31 - __builtin_clz(nw)));
    const uint32_t c = wave & (q - 1u);
    // (the range index is formed in lane 0 and broadcast: forming it from the broadcast count
    // costs the surrounding loop about 20 vector registers)
    unsigned long long t = 0;
    if (lane_id() == 0) t = (unsigned long long)c + (unsigned long long)q * atomicAdd(ovf.work + (size_t)c * kQueueWords, 1ull);
    return uniform64((int64_t)t);
}

constexpr int kRCap = 192, kLCap = 64, kTCap = 512;   // per-wave candidate lists and set
constexpr int64_t kMaxRangePoints = int64_t(1) << 28;  // longest point range the flat-stream loop takes
constexpr int kSetWords = kRCap + 2 * kLCap + kTCap;
using StreamSet = DeferredSet<kRCap, kLCap, kTCap>;

// A streamline range and the offsets it needs, as loaded.
struct RangeBounds {
    int64_t s0, s1;          // streamlines
    int64_t P, p0, p1;       // offsets[S], offsets[s0], offsets[s1]
};
__device__ __forceinline__ RangeBounds range_bounds(const int64_t *offsets, int64_t S, int64_t s0, int64_t s1) {
    const auto offs = gview(offsets);
    return {s0, s1, offs[S], offs[s0], offs[s1]};
}

// Counts streamlines [s0, s1) of one subject (whole streamlines only) into sub.C through `sink`.
// `coarse` is the subject's coarse occupancy map in LDS.  kCodesFirst: a batch's codes are awaited before the
// next batch's pair gathers are issued (see the pipeline below).
template <bool SCALED, int kBatch, bool kEnds, int kUp, bool kBrick, bool kCodesFirst, typename Sink>
__device__ void stream_range(const StreamSubject &sub, const uint32_t *coarse, const RangeBounds &rb, int32_t subject,
                             const Overflow &ovf, StreamSet &set, Sink &sink) {
    constexpr int kV = kBatch * kUp;   // lookups per batch: kUp sub-points of each of kBatch windows
    const int lane = lane_id();
    const CompactVol &cv = sub.cv;
    const int64_t s0 = rb.s0, s1 = rb.s1;
    const auto offs = gview(sub.offsets);
    const int64_t Ptot = uniform64(rb.P > 0 ? rb.P : 0);
    // occupancy pairs and codes share one allocation and one resource (codes at cv.codes_off)
    const __amdgpu_buffer_rsrc_t rvol = make_rsrc(cv.mb, cv.span);
    const int codes_off = uniform32((int)cv.codes_off);
    const uint32_t lane12 = 12u * (uint32_t)lane;
    // the grid bounds live in VGPRs: as scalars they crowd out the loop's lane masks
    uint32_t bX = fbits(sub.g.Xf), bY = fbits(sub.g.Yf), bZ = fbits(sub.g.Zf);
    asm volatile("" : "+v"(bX), "+v"(bY), "+v"(bZ));
    const uint32_t SBX = (uint32_t)cv.SBX, SBXY = (uint32_t)cv.SBXY;
    const uint32_t csx = (uint32_t)cv.csx, csyz = (uint32_t)cv.csyz, CBX = (uint32_t)cv.CBX, CBXY = (uint32_t)cv.CBXY;
    constexpr uint32_t kOutOfRange = 0xFFFFFFF8u;   // buffer offset past every resource: reads 0, no traffic
    const int64_t P0 = uniform64(clamp64(rb.p0, 0, Ptot));
    const int64_t P1 = uniform64(clamp64(rb.p1, P0, Ptot));
    if (P0 >= P1) return;
    if (P1 - P0 > kMaxRangePoints) {
        // positions below are 32-bit offsets from P0: a range this long (a few giant streamlines
        // make one) goes to the fallback kernel, one entry per non-empty streamline
        for (int64_t s = s0; s < s1; ++s) {
            const int64_t b = uniform64(clamp64(offs[s], P0, P1));
            const int64_t e = uniform64(clamp64(offs[s + 1], b, P1));
            if (e > b) push_overflow(ovf, b, subject);
        }
        return;
    }
    const uint32_t L = (uint32_t)(P1 - P0);   // points of the range; positions are relative to P0
    // endpoint modes (kEnds instantiations only): no point contributes its label but a streamline's
    // last (and, both_ends, its first); lab_prev is the label of the point before the window (or of
    // the batch's last window's end), lab_first that of the open streamline's first point
    const bool both_ends = kEnds && uniform32(sub.end_mode) == 2;
    int lab_prev = -1, lab_first = -1;
    // upsampling (kUp > 1 instantiations): sub-point t = 1 .. up-1 of a point lies a_t = fl32(t/up)
    // of the way to the next point of its streamline, in scaled coordinates
    const int up = kUp > 1 ? uniform32(sub.up) : 1;
    float at[kUp];
#pragma unroll
    for (int t = 0; t < kUp; ++t) at[t] = (float)((double)t / (double)up);
    // Starts of streamlines s0+1 .. s1-1 (relative to P0), 64 at a time, one per lane (L = "no
    // more starts"); k0 of them are consumed and `nxt` (uniform) is the next unconsumed start.
    int64_t vb = s0 + 1;
    uint32_t voff = 0, nxt = L;
    int k0 = 0;
    auto load_starts = [&]() {
        voff = (vb + lane < s1) ? (uint32_t)(clamp64(offs[vb + lane], P0, P1) - P0) : L;
        k0 = 0;
        nxt = (uint32_t)__builtin_amdgcn_readlane((int)voff, 0);
    };
    auto consumed = [&](uint64_t taken) {
        k0 += __popcll(taken);
        if (k0 >= kWave) {
            vb += kWave;
            load_starts();
        } else {
            nxt = (uint32_t)__builtin_amdgcn_readlane((int)voff, k0);
        }
    };
    // starts in [wb, wend) (wend <= wb + 64) as lane bits relative to wb; consumes them (empty
    // streamlines share a start)
    auto take_starts = [&](uint32_t wb, uint32_t wend) -> uint64_t {
        uint64_t starts = 0;
        while (nxt < wend) {
            const uint64_t inwin = __ballot(lane >= k0) & __ballot(voff < wend);
            const uint32_t qv = min(voff - wb, (uint32_t)(kWave - 1));   // lane of the start (in-window lanes)
            uint64_t it = inwin;
            while (it) {
                const int k = __builtin_ctzll(it);
                it &= it - 1ull;
                starts |= 1ull << __builtin_amdgcn_readlane((int)qv, k);
            }
            consumed(inwin);
        }
        return starts;
    };
    auto skip_starts = [&](uint32_t limit) {
        while (nxt < limit) consumed(__ballot(lane >= k0) & __ballot(voff < limit));
    };
    load_starts();
    // the open streamline ends; ml: the label of its last point (endpoint modes)
    auto close_open = [&](int ml) {
        if (kEnds) set.add_end_labels(ml, both_ends ? lab_first : -1);
        set.close(sink, sub.si, sub.sm);
    };
    int last_r = -1, last_m = -1;
    // points [P0, P1): loads at or past the range's end read zero without memory traffic, so the
    // next batch can always be issued
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(sub.pts + 3 * P0, 12ull * L);
    constexpr uint32_t BW = kWave * kBatch;   // points per batch

    // one register set of points: the lookup stage of a batch consumes it, and the points of the
    // batch after next are then loaded into it (see the pipeline below)
    // kUp > 1: each lane also holds the next point (the same load one point further on: it hits
    // the lines the window itself brings in)
    constexpr int kNext = kUp > 1 ? kBatch : 1;
    float ax[kBatch], ay[kBatch], az[kBatch], nx[kNext], ny[kNext], nz[kNext];
    auto load_batch = [&](uint32_t w) {
        const uint32_t so = 12u * w;
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b96(rp, lane12, so + 768u * b, kAuxStream);
            ax[b] = __uint_as_float(v[0]);
            ay[b] = __uint_as_float(v[1]);
            az[b] = __uint_as_float(v[2]);
        }
        if (kUp > 1) {
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b96(rp, lane12 + 12u, so + 768u * b, kAuxCached);
                nx[b] = __uint_as_float(v[0]);
                ny[b] = __uint_as_float(v[1]);
                nz[b] = __uint_as_float(v[2]);
            }
        }
    };
    // Lookup stage of the batch at w0 (its points are in ax.. / nx..): gather offsets and bit
    // indices.
    auto lookup = [&](uint32_t w0, uint32_t (&addr)[kV], uint32_t (&bix)[kV]) {
        const uint32_t left = w0 < L ? L - w0 : 0u;
        const int rem = left > BW ? (int)BW : (int)left;          // valid points in this batch
        const int remn = left > BW ? (int)BW + 1 : (int)left;     // lane + 1 < remn: a next point exists
        // voxelise and test the coarse occupancy bit in LDS; only lookups in occupied coarse
        // blocks gather their occupancy word and rank base (8 bytes): the others read past the
        // resource (zero, no traffic), so the gathered word alone decides the hit.  Lookup
        // v = b*kUp + t is sub-point t of window b.
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            float qx = ax[b], qy = ay[b], qz = az[b];
            if (SCALED) {
                qx = __fmul_rn(qx, sub.scale);
                qy = __fmul_rn(qy, sub.scale);
                qz = __fmul_rn(qz, sub.scale);
            }
            float dx = 0.f, dy = 0.f, dz = 0.f;
            if (kUp > 1) {
                float mx = nx[b], my = ny[b], mz = nz[b];
                if (SCALED) {
                    mx = __fmul_rn(mx, sub.scale);
                    my = __fmul_rn(my, sub.scale);
                    mz = __fmul_rn(mz, sub.scale);
                }
                dx = __fsub_rn(mx, qx);
                dy = __fsub_rn(my, qy);
                dz = __fsub_rn(mz, qz);
            }
#pragma unroll
            for (int t = 0; t < kUp; ++t) {
                const int v = b * kUp + t;
                float x = qx, y = qy, z = qz;
                if (t > 0) {
                    x = __fadd_rn(qx, __fmul_rn(at[t], dx));
                    y = __fadd_rn(qy, __fmul_rn(at[t], dy));
                    z = __fadd_rn(qz, __fmul_rn(at[t], dz));
                }
                const float tx = __fadd_rn(x, 0.5f), ty = __fadd_rn(y, 0.5f), tz = __fadd_rn(z, 0.5f);
                // 0 <= t < bound  <=>  bits(t) < bits(bound) as unsigned (t is never -0; NaN and
                // negative values compare above every finite positive bound)
                // (bitwise & throughout: no short-circuit branches)
                const int valid = t == 0 ? (int)(lane + b * kWave < rem) : (int)(t < up) & (int)(lane + b * kWave + 1 < remn);
                const bool ok = valid & (int)(fbits(tx) < bX) & (int)(fbits(ty) < bY) & (int)(fbits(tz) < bZ);
                const uint32_t ix = (uint32_t)(int)tx, iy = (uint32_t)(int)ty, iz = (uint32_t)(int)tz;
                uint32_t sb = __umul24(iz >> 3, SBXY) + __umul24(iy >> 3, SBX) + (ix >> 4);
                asm("" : "+v"(sb));   // keeps the 24-bit multiplies: (sb << 8) must not fold into them
                // coarse block: the super-brick itself (kBrick: the volume's map is per super-brick)
                // or a cube of 8, 16 or 32
                const uint32_t cb = kBrick ? sb : __umul24(iz >> csyz, CBXY) + __umul24(iy >> csyz, CBX) + (ix >> csx);
                const uint32_t cw = coarse[ok ? (cb >> 5) : 0u];
                const bool hit = (int)ok & (int)(__builtin_amdgcn_ubfe(cw, cb, 1) != 0u);   // bfe: offset mod 32
                // byte offset of the (word, base) pair: 32 words of 16x2x1 voxels per super-brick,
                // word (y/2 mod 4) + 4 (z mod 8), bit (x mod 16) + 16 (y mod 2)
                addr[v] = hit ? (sb << 8) | ((iy << 2) & 0x18u) | ((iz << 5) & 0xE0u) : kOutOfRange;
                bix[v] = (ix & 15u) | ((iy & 1u) << 4);
            }
        }
    };
    // (word, base) pairs of a batch's lookups.  Always issued: lanes that failed the coarse test
    // read past the resource (zero, no traffic), so every path through the loop issues the same
    // vector-memory sequence and each wait covers exactly what it needs.
    auto gather_pairs = [&](const uint32_t (&addr)[kV], uint32_t (&mw)[kV], uint32_t (&base)[kV]) {
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            const auto e = __builtin_amdgcn_raw_buffer_load_b64(rvol, addr[v], 0, kAuxCached);
            mw[v] = e[0];
            base[v] = e[1];
        }
    };
    // The rest of a batch once its codes are in: candidates, streamline starts and closes.
    auto tail = [&](uint32_t w0, const int (&r)[kV], const int (&m)[kV], const bool (&flag)[kV]) {
        uint64_t fl[kBatch];
        uint64_t fall = 0;
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            fl[b] = 0ull;
#pragma unroll
            for (int t = 0; t < kUp; ++t) fl[b] |= __ballot(flag[b * kUp + t]);
            fall |= fl[b];
        }
        if (fall == 0ull) {
            // nothing looked up: only a streamline start inside the batch matters (it closes the
            // open streamline, whose hits all came earlier)
            const uint32_t bend = (w0 + BW < L) ? w0 + BW : L;
            if (nxt < bend) {
                if (set.has_state()) close_open(nxt == w0 ? lab_prev : -1);
                skip_starts(bend);
                lab_first = -1;
            }
            last_r = last_m = lab_prev = -1;
            return;
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const uint32_t wb = w0 + (uint32_t)b * kWave;
            if (wb >= L) break;
            const uint32_t wend = (wb + kWave < L) ? wb + kWave : L;
            // streamline starts inside this window -> bit q of `starts` for lane q
            const uint64_t starts = (nxt < wend) ? take_starts(wb, wend) : 0ull;
            if (fl[b] == 0ull) {
                if (starts) {
                    if (set.has_state()) close_open((starts & 1ull) ? lab_prev : -1);
                    lab_first = -1;
                }
                last_r = last_m = lab_prev = -1;
                continue;
            }
            // sub-points t >= 1 exist only where the next point continues the lane's streamline:
            // not before a start, not at the range's end
            uint64_t nextok = ~0ull;
            if (kUp > 1) {
                uint64_t brk = starts >> 1;
                if (wb + kWave >= L || nxt == wb + kWave) brk |= 1ull << (kWave - 1);
                const uint32_t lastp = L - 1 - wb;   // lane of the range's last point
                if (lastp < (uint32_t)kWave) brk |= ~0ull << lastp;
                nextok = ~brk;
            }
            int rr[kUp], mm[kUp];
#pragma unroll
            for (int t = 0; t < kUp; ++t) {
                const bool ok = t == 0 || in_mask(nextok);
                rr[t] = ok ? r[b * kUp + t] : -1;
                mm[t] = (ok && !kEnds) ? m[b * kUp + t] : -1;
            }
            // each lane's last counted sub-point (t = up - 1) precedes the next lane's point
            int rl = rr[0], ml = mm[0];
#pragma unroll
            for (int t = 1; t < kUp; ++t)
                if (t == up - 1) {
                    rl = rr[t];
                    ml = mm[t];
                }
            // drop a hit equal to the hit just before it in streamline order: sub-point 0 against
            // the previous lane's last sub-point (lane 0: the previous window's), t >= 1 against t - 1
            int rp_ = __builtin_amdgcn_update_dpp(last_r, rl, 0x138, 0xF, 0xF, false);   // wave_shr:1
            int mp_ = __builtin_amdgcn_update_dpp(last_m, ml, 0x138, 0xF, 0xF, false);
            if (in_mask(starts)) rp_ = mp_ = -1;  // first point of a streamline
            uint64_t candR[kUp], candM[kUp];
            // (one ballot per comparison: each compare writes its lane mask directly)
            candR[0] = __ballot(rr[0] >= 0) & __ballot(rr[0] != rp_);
            candM[0] = __ballot(mm[0] >= 0) & __ballot(mm[0] != mp_);
#pragma unroll
            for (int t = 1; t < kUp; ++t) {
                candR[t] = __ballot(rr[t] >= 0) & __ballot(rr[t] != rr[t - 1]);
                candM[t] = __ballot(mm[t] >= 0) & __ballot(mm[t] != mm[t - 1]);
            }
            last_r = __builtin_amdgcn_readlane(rl, kWave - 1);
            last_m = __builtin_amdgcn_readlane(ml, kWave - 1);
            // the candidates of the lanes in `seg` into the open streamline's set
            auto add = [&](uint64_t seg, uint32_t at) {
#pragma unroll
                for (int t = 0; t < kUp; ++t) {
                    const uint64_t cR = candR[t] & seg, cM = candM[t] & seg;
                    if ((cR | cM) && !set.skip && !set.append(cR, rr[t], cM, mm[t])) {
                        push_overflow(ovf, P0 + (int64_t)at, subject);
                        set.nR = set.nL = 0;
                        set.skip = true;
                    }
                }
            };
            int lab_last = lab_prev;   // label of the closing streamline's last point
            if (kEnds) {
                const int ml_in = m[b * kUp];   // the lanes' labels
                lab_prev = __builtin_amdgcn_readlane(ml_in, (int)min(L - 1u - wb, (uint32_t)(kWave - 1)));
                if (wb == 0u) lab_first = __builtin_amdgcn_readlane(ml_in, 0);
            }
            if (!starts) {   // the whole window belongs to the open streamline
                add(~0ull, wb);
                continue;
            }
            int pos = 0;
            uint64_t st = starts;
            for (;;) {
                const int end = st ? __builtin_ctzll(st) : kWave;
                add(lanes_between(pos, end), wb + pos);
                if (!st) break;
                if (kEnds && end > 0) lab_last = __builtin_amdgcn_readlane(m[b * kUp], end - 1);
                close_open(lab_last);
                if (kEnds) lab_first = __builtin_amdgcn_readlane(m[b * kUp], end);
                pos = end;
                st &= st - 1ull;
            }
        }
    };
    // Software pipeline over batches k: the pair gathers of batch k + 1 are in flight while batch k's
    // codes return and its tail runs.  Vector-memory loads complete in issue order, so each
    // iteration issues: the codes of k, the pairs of k + 1, the points of k + 2; batch k's decode
    // then waits for its codes only, and the next iteration's flags for the pairs of k + 1 only.
    // kCodesFirst (the batched pass-through kernel) waits for the codes of k before the pairs of k + 1: its
    // updates are atomics, and where they are the bound it gains more from fewer loads beside them than
    // it loses by the wait.  A plan of 12 subjects of 200M points and 75M entries of C takes 1094 us a
    // launch with and 1112 without it, one of 4 subjects of 87M points and 14M entries 299 and 294.
    const uint32_t code_oob = kOutOfRange - (uint32_t)codes_off;   // with the code offset: past the resource
    uint32_t bix[kV], mw[kV], rank[kV];
    {
        uint32_t addr[kV];
        load_batch(0u);
        lookup(0u, addr, bix);
        __builtin_amdgcn_sched_barrier(0);
        gather_pairs(addr, mw, rank);
        __builtin_amdgcn_sched_barrier(0);
        load_batch(BW);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (uint32_t w0 = 0; w0 < L; w0 += BW) {
        // flags of batch k and its code gathers (unflagged lanes read past the resource)
        bool flag[kV];
#pragma unroll
        for (int v = 0; v < kV; ++v) flag[v] = __builtin_amdgcn_ubfe(mw[v], bix[v], 1) != 0u;
        uint32_t code[kV];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            const uint32_t at = rank[v] + __popc(__builtin_amdgcn_ubfe(mw[v], 0, bix[v]));
            code[v] = __builtin_amdgcn_raw_buffer_load_b32(rvol, flag[v] ? at << 2 : code_oob, codes_off, kAuxCached);
        }
        __builtin_amdgcn_sched_barrier(0);
        // lookups and pair gathers of batch k + 1 (its points arrived during the last iteration),
        // then the points of batch k + 2 into the registers the lookups just freed
        uint32_t bix2[kV], mw2[kV], rank2[kV];
        {
            uint32_t addr[kV];
            lookup(w0 + BW, addr, bix2);
            __builtin_amdgcn_sched_barrier(0);
            if (kCodesFirst) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
            gather_pairs(addr, mw2, rank2);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_batch(w0 + 2 * BW);
        __builtin_amdgcn_sched_barrier(0);
        // codes of batch k
        int r[kV], m[kV];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            const uint32_t rv = code[v] & cv.rmask, mv = code[v] >> cv.rbits;
            r[v] = (flag[v] && rv < (uint32_t)cv.N) ? (int)rv : -1;
            m[v] = (flag[v] && mv < (uint32_t)cv.M) ? (int)mv : -1;
        }
        tail(w0, r, m, flag);
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            bix[v] = bix2[v];
            mw[v] = mw2[v];
            rank[v] = rank2[v];
        }
    }
    close_open(lab_prev);
}

// A coarse map to LDS, 16 bytes a thread and step (by `threads` threads; the map is 16-byte aligned, and
// what follows its last word in its allocation may be read and stored: ncoarse_words rounded up to 4).
// Returns the first step's load; store it with put_coarse, so that other loads can fly beside it.
__device__ __forceinline__ uint4 get_coarse(const CompactVol &cv, int t) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (4 * t < cv.ncoarse_words) v = reinterpret_cast<const uint4 *>(cv.coarse)[t];
    return v;
}
__device__ __forceinline__ void put_coarse(const CompactVol &cv, uint32_t *lds, uint4 v, int t, int threads) {
    const int n4 = (cv.ncoarse_words + 3) >> 2;
    if (t < n4) reinterpret_cast<uint4 *>(lds)[t] = v;
    for (int k = t + threads; k < n4; k += threads)
        reinterpret_cast<uint4 *>(lds)[k] = reinterpret_cast<const uint4 *>(cv.coarse)[k];
}

// Ranges of about equally many points and streamlines, found by the wavefronts themselves.  Streamline s lies at
// offsets[s] + s * len, len the mean length (so that a wavefront gets at most twice the mean of either),
// and wavefront w takes those from t(w) up to t(w + 1), t(w) the w-th of nparts equal parts: its first
// one by a search of 64 offsets a round (three rounds for 256K streamlines), its last one from the 64
// offsets that follow, which hold it (twice the mean of at most 32 a wavefront) unless offsets decrease.
// (Ranges of equally many points give the wavefronts at the short end of streamlines sorted by length many
// more to close: 24,000 take 67 us a call, instead of 22.)
__device__ __forceinline__ RangeBounds range_by_points(const Ranges &rg, const StreamSubject &sub, uint32_t wave) {
    if ((int64_t)wave >= rg.nparts) return {0, 0, 0, 0, 0};
    const auto offs = gview(sub.offsets);
    const uint32_t lane = (uint32_t)lane_id(), S = (uint32_t)sub.S;   // (S <= INT32_MAX)
    const int64_t P = offs[S];
    int64_t len = 0;
    auto target = [&](uint32_t w) {   // (P is not needed before the first offsets are under way)
        const int64_t points = P > 0 ? P : 0;
        len = (int64_t)((double)points * rg.inv_S) + 1;
        return (int64_t)((double)(points + len * S) * ((double)w * rg.inv_nparts));
    };
    auto first_at = [&](uint32_t w) {   // (over any offsets: 0 .. S, and no later for a smaller w)
        uint32_t lo = 0u, hi = S;
        while (lo < hi) {
            const uint32_t step = (hi - lo + (uint32_t)kWave - 1u) / (uint32_t)kWave, at = lo + lane * step;
            int64_t v = 0;
            if (at < hi) v = offs[at];
            const int64_t t = target(w);
            const uint32_t n = (uint32_t)__popcll(__ballot(at < hi) & __ballot(v + len * at < t));
            hi = n ? min(hi, lo + n * step) : lo;
            if (n) lo += (n - 1u) * step + 1u;
        }
        return lo;
    };
    const uint32_t s0 = wave == 0u ? 0u : first_at(wave);
    int64_t v = 0;
    if (s0 + lane <= S) v = offs[s0 + lane];
    uint32_t s1 = S;
    if ((int64_t)wave + 1 < rg.nparts) {
        const int64_t t = target(wave + 1u);
        const uint32_t n = (uint32_t)__popcll(__ballot(s0 + lane < S) & __ballot(v + len * (s0 + lane) < t));
        s1 = n < (uint32_t)kWave ? s0 + n : max(s0, first_at(wave + 1u));
    }
    const int64_t p1 = s1 - s0 < (uint32_t)kWave ? readlane64(v, (int)(s1 - s0)) : offs[s1];
    return {s0, s1, P, readlane64(v, 0), p1};
}

// The streamline ranges of wavefront `wave`: ranges [first[i], first[i + 1]) from its queue, or (no table)
// one range, whose offsets first_range loads ahead of their use.  kSearch: rg.per may be 0.
template <bool kSearch>
__device__ __forceinline__ RangeBounds first_range(const Ranges &rg, const StreamSubject &sub, uint32_t wave) {
    if (rg.first) return {0, 0, 0, 0, 0};
    if (kSearch && rg.per == 0u) return range_by_points(rg, sub, wave);
    const int64_t s0 = min(sub.S, (int64_t)wave * rg.per + min(wave, rg.extra));
    return range_bounds(sub.offsets, sub.S, s0, min(sub.S, s0 + rg.per + (wave < rg.extra ? 1 : 0)));
}
// Calls f(bounds) for each of them.
template <typename F>
__device__ __forceinline__ void for_each_range(const Ranges &rg, const StreamSubject &sub, const Overflow &ovf, uint32_t wave,
                                               RangeBounds rb, F &&f) {
    const bool table = rg.first != nullptr;
    for (;;) {
        if (table) {
            const int64_t part = next_range(ovf, wave);
            if (part >= rg.nparts) break;
            const int64_t s0 = uniform64(clamp64(rg.first[part], 0, sub.S));
            const int64_t s1 = uniform64(clamp64(rg.first[part + 1], s0, sub.S));
            rb = range_bounds(sub.offsets, sub.S, s0, s1);
        }
        if (rb.s0 < rb.s1) f(rb);
        if (!table) break;
    }
}

// The flat-stream kernel's body: the wavefront's ranges, pair updates through its append sink.
template <bool SCALED, int kBatch, bool kEnds, bool kBrick, bool kSearch>
__device__ __forceinline__ void count_stream_body(const StreamSubject &sub, const Overflow &ovf,
                                                  const Ranges &rg, const PairOut &po) {
    // 4-window batches run 6 wavefronts per SIMD (their vector registers), so they can afford the LDS of 512
    // buffered updates; 2-window batches keep 8 per SIMD with 256
    constexpr int kSinkCap = kBatch == 4 ? 8 * kWave : 4 * kWave;
    __shared__ uint32_t s_set[kWavesPerBlock * kSetWords];
    __shared__ __align__(16) uint32_t s_pend[kWavesPerBlock * kSinkCap];
    extern __shared__ __align__(16) uint32_t s_coarse[];   // coarse occupancy bit map (coarse_lds_bytes)
    const int wv = uniform32(threadIdx.x >> 6);
    const uint32_t wave = blockIdx.x * kWavesPerBlock + wv;
    const RangeBounds rb = first_range<kSearch>(rg, sub, wave);
    const uint4 cmap = get_coarse(sub.cv, threadIdx.x);
    StreamSet set;
    set.init(s_set + wv * kSetWords);
    put_coarse(sub.cv, s_coarse, cmap, threadIdx.x, kBlock);
    __syncthreads();
    AppendSink<kSinkCap> sink;
    sink.init(s_pend + wv * kSinkCap, sub.C, po, wave);
    for_each_range(rg, sub, ovf, wave, rb, [&](const RangeBounds &r) {
        stream_range<SCALED, kBatch, kEnds, 1, kBrick, false>(sub, s_coarse, r, 0, ovf, set, sink);
    });
    sink.drain(po, wave);
}

// Two-window batches (the short-call schedule) need few vector registers; with at most 80 scalar
// registers a SIMD holds 8 of these wavefronts.  (Each wavefront's scalar allocation is its count
// rounded up to 16, plus 16 more: 800 / (96 + 16) = 7 wavefronts at 81..96 registers, 6 above that.)
template <bool SCALED, bool kEnds, bool kBrick>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_num_sgpr(80)))
k_count_stream2(StreamSubject sub, Overflow ovf, Ranges rg, PairOut po) {
    count_stream_body<SCALED, 2, kEnds, kBrick, true>(sub, ovf, rg, po);
}

// (kSearch: wavefronts find their ranges themselves.  Two instantiations: with the search before it the loop
// keeps other scalars in registers, and 5M streamlines, which come in a table, take 2613 instead of 2592 us.)
// Six wavefronts per SIMD (at most 80 vector registers): left to itself the compiler takes 81 to 84, which is
// five, and 5M streamlines of 150 points on a 210x240x200 grid take 1727 instead of 1616 us, on 145x174x145 1791
// instead of 1669, on 260x311x260 1702 instead of 1667; 5M of 220 points there take 2600 either way.
template <bool SCALED, bool kEnds, bool kBrick, bool kSearch>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6)))
k_count_stream4(StreamSubject sub, Overflow ovf, Ranges rg, PairOut po) {
    count_stream_body<SCALED, 4, kEnds, kBrick, kSearch>(sub, ovf, rg, po);
}

// Upsampled pass-through (up = 2 .. kUp): the scale is always applied (multiplying by 1.0f is
// exact), so two instantiations cover every case.  Six wavefronts per SIMD (at most 80 vector registers):
// left to itself the compiler takes 81 for kUp 2, which is five, and 300k streamlines upsampled by 2 take
// 217 instead of 212 us.
template <int kUp>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6)))
k_count_stream_up(StreamSubject sub, Overflow ovf, Ranges rg, PairOut po) {
    constexpr int kB = kUp == 2 ? 2 : 1;   // kB * kUp lookups per batch, as the plain kernel's 4
    constexpr int kSinkCap = 4 * kWave;
    __shared__ uint32_t s_set[kWavesPerBlock * kSetWords];
    __shared__ __align__(16) uint32_t s_pend[kWavesPerBlock * kSinkCap];
    extern __shared__ __align__(16) uint32_t s_coarse[];
    const int wv = uniform32(threadIdx.x >> 6);
    const uint32_t wave = blockIdx.x * kWavesPerBlock + wv;
    const RangeBounds rb = first_range<true>(rg, sub, wave);
    const uint4 cmap = get_coarse(sub.cv, threadIdx.x);
    StreamSet set;
    set.init(s_set + wv * kSetWords);
    put_coarse(sub.cv, s_coarse, cmap, threadIdx.x, kBlock);
    __syncthreads();
    AppendSink<kSinkCap> sink;
    sink.init(s_pend + wv * kSinkCap, sub.C, po, wave);
    for_each_range(rg, sub, ovf, wave, rb, [&](const RangeBounds &r) {
        stream_range<true, kB, false, kUp, false, false>(sub, s_coarse, r, 0, ovf, set, sink);
    });
    sink.drain(po, wave);
}

// Batched form: work items (subject, first streamline) from every subject, handed out by the
// queues; each wavefront keeps the coarse map of the subject it last worked on in its own LDS.
// The scale is always applied (multiplying by 1.0f is exact).
// One instantiation per kind of subject: pass-through (kEnds false, kUp 1), the endpoint modes
// (kEnds: end labels at each close), and upsampled pass-through (kUp 2 or 4, with
// sub.up <= kUp); a launch takes the items of subjects of one kind only.
template <int kBatch, bool kEnds, int kUp>
__global__ void __launch_bounds__(kBlock) k_count_batched(const StreamSubject *__restrict__ subs, int32_t nsub,
                                                          const int2 *__restrict__ items, int64_t nitems,
                                                          Overflow ovf, int32_t coarse_words) {
    __shared__ uint32_t s_set[kWavesPerBlock * kSetWords];
    __shared__ uint32_t s_pend[kWavesPerBlock * kWave];
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) uint32_t s_coarse[];   // kWavesPerBlock * coarse_words (at most 512, a multiple of 4)
    const int lane = lane_id(), wv = uniform32(threadIdx.x >> 6);
    uint32_t *coarse = s_coarse + wv * coarse_words;
    StreamSet set;
    set.init(s_set + wv * kSetWords);
    // updates go to C as atomics: with many hits per point, this form's cost is the hit processing
    BufferedSink sink;
    sink.init(s_pend + wv * kWave, nullptr);
    int loaded = -1;
    const uint32_t wave = blockIdx.x * kWavesPerBlock + wv;
    // one item per wavefront: no queue
    const bool queued = nitems > (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t turn = 0; queued || turn == 0; ++turn) {
        const int64_t item = queued ? next_range(ovf, wave) : (int64_t)wave;
        if (item >= nitems) break;
        const int2 it = items[item];
        // (offsets that decrease leave items unwritten: the result is undefined then, the accesses are not)
        const int subject = uniform32(min(max(it.x, 0), nsub - 1));
        const StreamSubject &sub = subs[subject];
        const int64_t s0 = uniform64(clamp64(it.y, 0, sub.S));
        int64_t s1 = sub.S;
        if (item + 1 < nitems) {
            const int2 nx = items[item + 1];
            if (nx.x == subject) s1 = nx.y;
        }
        s1 = uniform64(clamp64(s1, s0, sub.S));
        if (s0 >= s1) continue;
        const RangeBounds rb = range_bounds(sub.offsets, sub.S, s0, s1);
        if (subject != loaded) {
            // two 16-byte loads a lane, at most 512 words
            const auto src = reinterpret_cast<const __attribute__((address_space(1))) v4u *>(gview(sub.cv.coarse));
            const int n4 = (sub.cv.ncoarse_words + 3) >> 2;
            v4u c0 = {}, c1 = {};
            if (lane < n4) c0 = src[lane];
            if (lane + kWave < n4) c1 = src[lane + kWave];
            v4u *dst = reinterpret_cast<v4u *>(coarse);
            if (lane < n4) dst[lane] = c0;
            if (lane + kWave < n4) dst[lane + kWave] = c1;
            loaded = subject;
        }
        sink.C = sub.C;
        stream_range<true, kBatch, kEnds, kUp, false, kUp == 1 && !kEnds>(sub, coarse, rb, subject, ovf, set, sink);
        sink.drain();   // the next item may belong to another subject's C
    }
}

// Resident workgroups per CU of kernel fn (kBlock threads, dyn bytes of dynamic LDS) on the current device;
// asked of the runtime once per kernel and size.
static int resident_blocks(const void *fn, size_t dyn) {
    static std::mutex mu;
    static std::map<std::tuple<int, const void *, size_t>, int> known;
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> g(mu);
    const auto key = std::make_tuple(dev, fn, dyn);
    const auto it = known.find(key);
    if (it != known.end()) return it->second;
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kBlock, dyn);
    if (e != hipSuccess || n < 1) return 4;
    if (known.size() >= 4096) known.clear();   // (sizes follow the grids)
    known[key] = n;
    return n;
}

template <bool SCALED, int B, bool E>
static int blocks_per_cu_of(size_t dyn) {
    const void *fn = B == 2 ? reinterpret_cast<const void *>(&k_count_stream2<SCALED, E, true>)
                            : reinterpret_cast<const void *>(&k_count_stream4<SCALED, E, true, false>);
    return resident_blocks(fn, dyn);
}

template <int B, bool E>
static int blocks_per_cu_b(bool scaled, size_t dyn) {
    return scaled ? blocks_per_cu_of<true, B, E>(dyn) : blocks_per_cu_of<false, B, E>(dyn);
}

template <int U>
static int blocks_per_cu_up(size_t dyn) {
    return resident_blocks(reinterpret_cast<const void *>(&k_count_stream_up<U>), dyn);
}

int count_stream_blocks_per_cu(bool scaled, int batch, bool ends, int up, size_t dyn) {
    if (up > 1) return up == 2 ? blocks_per_cu_up<2>(dyn) : blocks_per_cu_up<4>(dyn);
    if (ends) return batch == 2 ? blocks_per_cu_b<2, true>(scaled, dyn) : blocks_per_cu_b<4, true>(scaled, dyn);
    return batch == 2 ? blocks_per_cu_b<2, false>(scaled, dyn) : blocks_per_cu_b<4, false>(scaled, dyn);
}

static StreamSubject stream_subject(const CountArgs &a, const CompactVol &cv) {
    StreamSubject s;
    s.pts = a.pts;
    s.offsets = a.offsets;
    s.S = a.S;
    s.s_begin = 0;
    s.g = a.g;
    s.scale = a.scale;
    s.cv = cv;
    s.C = a.C;
    s.si = a.si;
    s.sm = a.sm;
    s.end_mode = a.end_mode;
    s.up = a.up;
    return s;
}

template <int B, bool E, bool K>
static void launch_stream_bk(const CountArgs &a, const CompactVol &cv, const Ranges &rg, int blocks,
                             const PairOut &po, hipStream_t st) {
    const bool scaled = a.scale != 1.0f;
    const size_t dyn = coarse_lds_bytes(cv.ncoarse_words);
    const StreamSubject sub = stream_subject(a, cv);
    const bool search = !rg.first && rg.per == 0u;
#define FC_LAUNCH_STREAM(S_)                                                                           \
    do {                                                                                               \
        if (B == 2) k_count_stream2<S_, E, K><<<blocks, kBlock, dyn, st>>>(sub, a.ovf, rg, po);        \
        else if (search) k_count_stream4<S_, E, K, true><<<blocks, kBlock, dyn, st>>>(sub, a.ovf, rg, po); \
        else k_count_stream4<S_, E, K, false><<<blocks, kBlock, dyn, st>>>(sub, a.ovf, rg, po);        \
    } while (0)
    if (scaled) FC_LAUNCH_STREAM(true);
    else FC_LAUNCH_STREAM(false);
#undef FC_LAUNCH_STREAM
}

// the super-brick coarse map (csx 4, csyz 3) has its own instantiations
template <int B, bool E>
static void launch_stream_b(const CountArgs &a, const CompactVol &cv, const Ranges &rg, int blocks,
                            const PairOut &po, hipStream_t st) {
    if (cv.csx == 4 && cv.csyz == 3) launch_stream_bk<B, E, true>(a, cv, rg, blocks, po, st);
    else launch_stream_bk<B, E, false>(a, cv, rg, blocks, po, st);
}

hipError_t launch_count_stream(const CountArgs &a, const CompactVol &cv, const Ranges &rg, int blocks,
                               int batch, const PairOut &po, hipStream_t st) {
    if (a.up > 1) {
        const size_t dyn = coarse_lds_bytes(cv.ncoarse_words);
        const StreamSubject sub = stream_subject(a, cv);
        if (a.up == 2) k_count_stream_up<2><<<blocks, kBlock, dyn, st>>>(sub, a.ovf, rg, po);
        else k_count_stream_up<4><<<blocks, kBlock, dyn, st>>>(sub, a.ovf, rg, po);
        return hipGetLastError();
    }
    const bool ends = a.end_mode != 0;
    if (batch == 2) {
        if (ends) launch_stream_b<2, true>(a, cv, rg, blocks, po, st);
        else launch_stream_b<2, false>(a, cv, rg, blocks, po, st);
    } else {
        if (ends) launch_stream_b<4, true>(a, cv, rg, blocks, po, st);
        else launch_stream_b<4, false>(a, cv, rg, blocks, po, st);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// fallback for overflowed streamlines: one workgroup per queued streamline, global bit maps
// ---------------------------------------------------------------------------------------------

// One overflowed streamline (the one containing point p), counted by a whole workgroup with the
// workgroup's all-zero scratch: a bit map over rows, one over labels and a list of the labels.
// Sub-point k of the streamline [b0, b1) upsampled by `up` (0 <= k < (b1 - b0 - 1) * up + 1):
// point j = b0 + k / up itself when t = k % up is 0, else the point a_t = fl32(t / up) of the way to
// point j + 1, in scaled coordinates.  False when it has no voxel.
template <typename Lookup, bool SCALED>
__device__ bool sub_lookup(const float *__restrict__ pts, int64_t b0, int64_t k, int up, float scale, const Grid &g,
                           const Lookup &lk, int &r, int &m) {
    const int64_t j = b0 + k / up;
    const int t = (int)(k % up);
    float x = pts[3 * j], y = pts[3 * j + 1], z = pts[3 * j + 2];
    if (SCALED) {
        x = __fmul_rn(x, scale);
        y = __fmul_rn(y, scale);
        z = __fmul_rn(z, scale);
    }
    if (t > 0) {
        float ux = pts[3 * j + 3], uy = pts[3 * j + 4], uz = pts[3 * j + 5];
        if (SCALED) {
            ux = __fmul_rn(ux, scale);
            uy = __fmul_rn(uy, scale);
            uz = __fmul_rn(uz, scale);
        }
        const float a = (float)((double)t / (double)up);
        x = __fadd_rn(x, __fmul_rn(a, __fsub_rn(ux, x)));
        y = __fadd_rn(y, __fmul_rn(a, __fsub_rn(uy, y)));
        z = __fadd_rn(z, __fmul_rn(a, __fsub_rn(uz, z)));
    }
    int ix, iy, iz;
    if (!voxelise<false>(x, y, z, 1.0f, g, ix, iy, iz)) return false;
    lk.get(ix, iy, iz, r, m);
    return true;
}

constexpr int kFallbackCached = 4;   // sub-points per thread whose lookup is kept for the later passes

template <typename Lookup, bool SCALED>
__device__ void fallback_streamline(const float *__restrict__ pts, const int64_t *__restrict__ offsets, int64_t S,
                                    const Grid &g, float scale, const Lookup &lk, int32_t *__restrict__ C, uint32_t si,
                                    uint32_t sm, int64_t p, uint32_t *bmN, uint32_t *bmM, uint32_t *labels,
                                    int *s_nlab, int end_mode, int up) {
    const int64_t Ptot = offsets[S] > 0 ? offsets[S] : 0;
    // streamline containing point p: the last s with offsets[s] <= p.  The offsets never decrease,
    // so of blockDim.x evenly spaced candidates the ones at or below p are a prefix of the threads,
    // and their count narrows [lo, hi) blockDim.x-fold per round (3 rounds for 5M streamlines).
    int64_t lo = 0, hi = S;  // answer in [lo, hi)
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + blockDim.x - 1) / blockDim.x;
        const int64_t idx = lo + (int64_t)threadIdx.x * step;
        const int at_or_below = (threadIdx.x > 0 && idx < hi && offsets[idx] <= p) ? 1 : 0;
        lo += (int64_t)__syncthreads_count(at_or_below) * step;
        hi = min(hi, lo + step);
    }
    const int64_t b0 = clamp64(offsets[lo], 0, Ptot);
    const int64_t b1 = clamp64(offsets[lo + 1], b0, Ptot);
    const int64_t nsub = b1 > b0 ? (b1 - b0 - 1) * up + 1 : 0;   // points after upsampling
    if (threadIdx.x == 0) *s_nlab = 0;
    // each sub-point is looked up once: thread t's sub-points t + j * blockDim.x, j < kFallbackCached,
    // keep (r, m) in registers for the three passes; the rest (streamlines of more than
    // kFallbackCached * blockDim.x sub-points) are looked up again in each pass.  -1: none.
    int cr[kFallbackCached], cm[kFallbackCached];
#pragma unroll
    for (int j = 0; j < kFallbackCached; ++j) {
        const int64_t k = threadIdx.x + (int64_t)j * blockDim.x;
        int r = -1, m = -1;
        if (k >= nsub || !sub_lookup<Lookup, SCALED>(pts, b0, k, up, scale, g, lk, r, m)) r = m = -1;
        cr[j] = r;
        cm[j] = m;
    }
    const int64_t k_rest = threadIdx.x + (int64_t)kFallbackCached * blockDim.x;
    auto lookup_rest = [&](int64_t k, int &r, int &m) {
        if (!sub_lookup<Lookup, SCALED>(pts, b0, k, up, scale, g, lk, r, m)) r = m = -1;
    };
    __syncthreads();
    // endpoint modes: the labels are the streamline's end labels
    if (end_mode != 0 && threadIdx.x == 0 && nsub > 0) {
        int r, ml, mf = -1, n = 0;
        if (!sub_lookup<Lookup, SCALED>(pts, b0, nsub - 1, up, scale, g, lk, r, ml)) ml = -1;
        if (end_mode == 2 && !sub_lookup<Lookup, SCALED>(pts, b0, 0, up, scale, g, lk, r, mf)) mf = -1;
        if (ml >= 0) atomicExch(&labels[n++], (uint32_t)ml);
        if (mf >= 0 && mf != ml) atomicExch(&labels[n++], (uint32_t)mf);
        *s_nlab = n;
    }
    // distinct labels
    auto add_label = [&](int m) {
        if (m >= 0) {
            const uint32_t bitm = 1u << (m & 31);
            if (!(atomicOr(&bmM[m >> 5], bitm) & bitm)) {
                const int k = atomicAdd(s_nlab, 1);
                atomicExch(&labels[k], (uint32_t)m);
            }
        }
    };
    if (end_mode == 0) {
#pragma unroll
        for (int j = 0; j < kFallbackCached; ++j) add_label(cm[j]);
        for (int64_t k = k_rest; k < nsub; k += blockDim.x) {
            int r, m;
            lookup_rest(k, r, m);
            add_label(m);
        }
    }
    __syncthreads();
    const int nlab = *s_nlab;
    // distinct rows: the first claimant of each row adds its pairs
    auto add_row = [&](int r) {
        if (r >= 0) {
            const uint32_t bitr = 1u << (r & 31);
            if (!(atomicOr(&bmN[r >> 5], bitr) & bitr)) {
                int32_t *row = C + (uint32_t)r * si;
                for (int k = 0; k < nlab; ++k)
                    atomicAdd(row + __hip_atomic_load(&labels[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * sm, 1);
            }
        }
    };
    if (nlab > 0) {
#pragma unroll
        for (int j = 0; j < kFallbackCached; ++j) add_row(cr[j]);
        for (int64_t k = k_rest; k < nsub; k += blockDim.x) {
            int r, m;
            lookup_rest(k, r, m);
            add_row(r);
        }
    }
    __syncthreads();
    // restore the all-zero scratch (bit maps and label list)
    auto clear = [&](int r, int m) {
        if (r >= 0) atomicExch(&bmN[r >> 5], 0u);
        if (m >= 0) atomicExch(&bmM[m >> 5], 0u);
    };
#pragma unroll
    for (int j = 0; j < kFallbackCached; ++j) clear(cr[j], cm[j]);
    for (int64_t k = k_rest; k < nsub; k += blockDim.x) {
        int r, m;
        lookup_rest(k, r, m);
        clear(r, m);
    }
    for (int k = threadIdx.x; k < nlab; k += blockDim.x) atomicExch(&labels[k], 0u);
    __syncthreads();
}

constexpr int64_t kPointMask = (int64_t(1) << kSubjectShift) - 1;

// The overflow queue's streamlines, one per workgroup at a time (workgroups [0, fs.blocks)).
template <typename Lookup, bool SCALED>
__device__ __forceinline__ void fallback_queue(const CountArgs &a, const Lookup &lk, const FallbackScratch &fs, int *s_nlab) {
    uint32_t *bmN = fs.words + (int64_t)blockIdx.x * fs.stride;
    uint32_t *bmM = bmN + fs.nwordsN;
    uint32_t *labels = bmM + fs.nwordsM;
    const int64_t nq = (int64_t)*a.ovf.count;
    const int64_t nq_c = nq < a.ovf.cap ? nq : a.ovf.cap;
    for (int64_t q = blockIdx.x; q < nq_c; q += fs.blocks)
        fallback_streamline<Lookup, SCALED>(a.pts, a.offsets, a.S, a.g, a.scale, lk, a.C, a.si, a.sm,
                                            a.ovf.list[q] & kPointMask, bmN, bmM, labels, s_nlab, a.end_mode, a.up);
}

template <typename Lookup, bool SCALED>
__global__ void __launch_bounds__(kBlock) k_fallback(CountArgs a, Lookup lk, FallbackScratch fs) {
    __shared__ int s_nlab;
    fallback_queue<Lookup, SCALED>(a, lk, fs, &s_nlab);
}

// Batched fallback: the queue entry names its subject.
__global__ void __launch_bounds__(kBlock) k_fallback_batched(const StreamSubject *__restrict__ subs, int32_t nsub,
                                                             Overflow ovf, FallbackScratch fs) {
    __shared__ int s_nlab;
    uint32_t *bmN = fs.words + (int64_t)blockIdx.x * fs.stride;
    uint32_t *bmM = bmN + fs.nwordsN;
    uint32_t *labels = bmM + fs.nwordsM;
    const int64_t nq = (int64_t)*ovf.count;
    const int64_t nq_c = nq < ovf.cap ? nq : ovf.cap;
    for (int64_t q = blockIdx.x; q < nq_c; q += gridDim.x) {
        const int64_t e = ovf.list[q];
        int32_t subject = (int32_t)(e >> kSubjectShift);
        subject = subject < 0 ? 0 : (subject >= nsub ? nsub - 1 : subject);
        const StreamSubject &sub = subs[subject];
        fallback_streamline<CompactLookup, true>(sub.pts, sub.offsets, sub.S, sub.g, sub.scale, CompactLookup{sub.cv},
                                                 sub.C, sub.si, sub.sm, e & kPointMask, bmN, bmM, labels, &s_nlab,
                                                 sub.end_mode, sub.up);
    }
}

// ---------------------------------------------------------------------------------------------
// Alg. 1's seed-to-endpoint count
// ---------------------------------------------------------------------------------------------

// C(row of the first point, label of the last point) += 1 for streamlines [sb, S) (the seed is the first
// point).  A wavefront takes 63 streamlines at a time: lane k reads offset k of the 64 around them and
// the two points beside it, the last of one streamline and the first of the next (24 bytes, mostly of
// one line), and passes the last one to the lane before it; the label is looked up only where the row
// was found.  Bound by the scattered reads: one thread per streamline with both points and both lookups
// of its own took 46 us for a million streamlines.
template <typename Lookup, bool SCALED>
__device__ __forceinline__ void seed_end_streamlines(const float *__restrict__ pts, const int64_t *__restrict__ offsets,
                                                     int64_t sb, int64_t S, float scale, const Grid &g, const Lookup &lk,
                                                     int32_t *__restrict__ C, uint32_t si, uint32_t sm) {
    constexpr int kLines = kWave - 1;
    const int lane = lane_id();
    const auto offs = gview(offsets);
    const int64_t Ptot = offs[S] > 0 ? offs[S] : 0;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    const int64_t wave = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6);
    for (int64_t s0 = sb + wave * kLines; s0 < S; s0 += waves * kLines) {   // (uniform over the wavefront)
        const int64_t s = s0 + lane;
        const int64_t o = clamp64(offs[min(s, S)], 0, Ptot);
        // points o - 1 and o, where they exist
        float e[3] = {NAN, NAN, NAN}, f[3] = {NAN, NAN, NAN};
        const auto p = gview(pts) + 3 * o;
        if (o > 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) e[k] = p[k - 3];
        }
        if (o < Ptot) {
#pragma unroll
            for (int k = 0; k < 3; ++k) f[k] = p[k];
        }
        // streamline s = [o, next): its last point is the next lane's e
        const int64_t next = __shfl_down(o, 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) e[k] = __shfl_down(e[k], 1);
        int r = -1, m = -1, none;
        if (lane < kLines && s < S && next > o) lookup_point<Lookup, SCALED>(f, scale, g, lk, r, none);
        if (r >= 0) lookup_point<Lookup, SCALED>(e, scale, g, lk, none, m);
        if (m >= 0) add_one(C + ((uint32_t)r * si + (uint32_t)m * sm));
    }
}

template <typename Lookup, bool SCALED>
__global__ void k_count_seed_end(CountArgs a, Lookup lk) {
    seed_end_streamlines<Lookup, SCALED>(a.pts, a.offsets, 0, a.S, a.scale, a.g, lk, a.C, a.si, a.sm);
}

template <typename Lookup>
static void launch_seed_end_l(const CountArgs &a, const Lookup &lk, int cus, hipStream_t st) {
    const unsigned blocks = fill_blocks(a.S / (kWave - 1) * kWave + kWave, cus);
    if (a.scale != 1.0f) k_count_seed_end<Lookup, true><<<blocks, kBlock, 0, st>>>(a, lk);
    else k_count_seed_end<Lookup, false><<<blocks, kBlock, 0, st>>>(a, lk);
}

hipError_t launch_count_seed_end(const CountArgs &a, const RasterVol *rv, const CompactVol *cv, int cus,
                                 hipStream_t st) {
    if (a.S <= 0) return hipSuccess;
    if (rv) launch_seed_end_l(a, RasterLookup{*rv}, cus, st);
    else launch_seed_end_l(a, CompactLookup{*cv}, cus, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// parcellation outputs of C: one wavefront per row
// ---------------------------------------------------------------------------------------------

// label[i] = lowest m holding the row's maximum (-1 when no entry is positive), sums[i] = row sum,
// frac[i][m] = C[i][m] / sums[i] taken in double and rounded to float (0 when the sum is not
// positive).  Any output may be null.
//
// Bound by memory (8 bytes an entry), but each wavefront's rows are a serial chain of load, reduction and
// division: reduced with cross-lane moves of the vector unit and divided by one reciprocal a row, 45,808 x
// 180 takes 16.9 us (66.5 MB, 3.9 TB/s); a reduction through LDS permutes, 24 waits a row, and a division
// an entry took 20.4.
constexpr int kParcVals = 6;   // row entries per lane kept in registers (rows of up to 384 labels)

// One step of a reduction over the wavefront towards lane 63: the value `kCtrl` lanes lower (a DPP
// control), 0 where there is none.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, kCtrl, kRows, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), kCtrl, kRows, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}
template <typename Op>
__device__ __forceinline__ uint64_t wave_reduce64(uint64_t v, Op &&op) {   // (op(v, 0) == v)
    v = op(v, dpp64<0x111, 0xF>(v));   // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds its row's
    v = op(v, dpp64<0x112, 0xF>(v));
    v = op(v, dpp64<0x114, 0xF>(v));
    v = op(v, dpp64<0x118, 0xF>(v));
    v = op(v, dpp64<0x142, 0xA>(v));   // row_bcast 15 into rows 1 and 3
    v = op(v, dpp64<0x143, 0xC>(v));   // row_bcast 31 into rows 2 and 3
    return (uint64_t)readlane64((int64_t)v, kWave - 1);
}

__global__ void __launch_bounds__(kBlock) k_parcellate(const int32_t *__restrict__ C, int32_t N, int32_t M,
                                                       int32_t *__restrict__ label, float *__restrict__ frac,
                                                       int64_t *__restrict__ sums) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * kWavesPerBlock;
    // each lane keeps entries lane + 64 q (q < kParcVals) of its wavefront's row in registers, and
    // the next row's are loaded while this one is reduced; entries past kParcVals * 64 are read
    // from memory
    int v[kParcVals], vn[kParcVals];
    auto load_row = [&](int64_t i, int (&dst)[kParcVals]) {
#pragma unroll
        for (int q = 0; q < kParcVals; ++q) {
            const int m = lane + q * kWave;
            dst[q] = (i < N && m < M) ? C[i * (int64_t)M + m] : 0;
        }
    };
    int64_t i = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    load_row(i, v);
    for (; i < N; i += nw) {
        load_row(i + nw, vn);
        const int32_t *row = C + i * (int64_t)M;
        long long total = 0;
        int best = 0, bidx = -1;   // largest positive value seen and its lowest column
#pragma unroll
        for (int q = 0; q < kParcVals; ++q) {
            const int m = lane + q * kWave;
            total += v[q];
            if (m < M && v[q] > best) {
                best = v[q];
                bidx = m;
            }
        }
        for (int m = lane + kParcVals * kWave; m < M; m += kWave) {
            const int x = row[m];
            total += x;
            if (x > best) {
                best = x;
                bidx = m;
            }
        }
        total = (long long)wave_reduce64((uint64_t)total, [](uint64_t a, uint64_t b) { return a + b; });
        // the largest value, and of its columns the lowest (0: no positive value)
        const uint64_t key = best > 0 ? ((uint64_t)(uint32_t)best << 32) | (0xFFFFFFFFu - (uint32_t)bidx) : 0ull;
        const uint64_t top = wave_reduce64(key, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
        bidx = top ? (int)(0xFFFFFFFFu - (uint32_t)top) : -1;
        if (lane == 0) {
            if (label) label[i] = bidx;
            if (sums) sums[i] = total;
        }
        if (frac) {
            float *out = frac + i * (int64_t)M;
            const double d = (double)total, rcp = 1.0 / d;
            // x / d in double, correctly rounded: the quotient by the rounded reciprocal, corrected by its
            // exact remainder (Markstein).  That needs a divisor whose significand is not all ones, which
            // no whole number below 2^52 has.
            const bool by_rcp = total < (1ll << 52);
            auto fraction = [&](int x) {
                const double n = (double)x, q0 = n * rcp, r = __builtin_fma(-q0, d, n);
                return (float)(by_rcp ? __builtin_fma(r, rcp, q0) : n / d);
            };
            if (total > 0) {
#pragma unroll
                for (int q = 0; q < kParcVals; ++q) {
                    const int m = lane + q * kWave;
                    if (m < M) out[m] = fraction(v[q]);
                }
                for (int m = lane + kParcVals * kWave; m < M; m += kWave) out[m] = fraction(row[m]);
            } else {
                for (int m = lane; m < M; m += kWave) out[m] = 0.0f;
            }
        }
#pragma unroll
        for (int q = 0; q < kParcVals; ++q) v[q] = vn[q];
    }
}

hipError_t launch_parcellate(const int32_t *C, int32_t N, int32_t M, int32_t *label, float *frac, int64_t *sums,
                             int cus, hipStream_t st) {
    if (N <= 0) return hipSuccess;
    int64_t blocks = ((int64_t)N + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > (int64_t)cus * 8) blocks = (int64_t)cus * 8;
    k_parcellate<<<(unsigned)blocks, kBlock, 0, st>>>(C, N, M, label, frac, sums);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// batched form: work items, zero fill of every C, launchers
// ---------------------------------------------------------------------------------------------

// Prepares a launch; blockIdx.y is the subject, or (block_base) the one whose workgroups blockIdx.x falls
// into.  Its C is zeroed (sizes: entries of each subject's C;
// nullptr: not here), and its work items item_base[s] .. item_base[s + 1] are written: item j = (subject,
// first streamline of [s_begin, S) whose start lies in the j-th of the n_s equal parts of the points
// offsets[s_begin] .. offsets[S]).  The offsets are read once, in order, as in k_partition: a binary
// search per item took 8.5 us on little subjects and 16 us on large ones, after a launch for the zero
// fill of its own; with a small share of the workgroups for one large subject, its pass took 4 ms of 3M
// streamlines beside 999 of 100.  Also zeroes zero[0 .. nzero): the counting launches' overflow count and queues.
__global__ void k_prepare_batched(const StreamSubject *__restrict__ subs, const int64_t *__restrict__ item_base,
                                  const int64_t *__restrict__ sizes, int32_t nsub,
                                  const int64_t *__restrict__ block_base, int2 *__restrict__ items,
                                  unsigned long long *__restrict__ zero, int64_t nzero) {
    constexpr int kShort = 2, kOwn = 8;
    int32_t k = (int32_t)blockIdx.y;
    int64_t block = blockIdx.x, blocks = gridDim.x;
    if (block_base) {
        // the last subject whose base is at or below this workgroup: 64 bases a round
        int32_t lo = 0, hi = nsub;   // block_base[lo] <= block, and the answer in [lo, hi)
        while (hi - lo > 1) {
            const int32_t step = (hi - lo + kWave - 1) / kWave, at = lo + lane_id() * step;
            const uint64_t le = __ballot(at < hi && block_base[at < hi ? at : lo] <= block);
            lo += (__popcll(le) - 1) * step;   // (lane 0's is)
            hi = min(hi, lo + step);
        }
        k = lo;
        block -= block_base[k];
        blocks = block_base[k + 1] - block_base[k];
    }
    const int64_t stride = blocks * blockDim.x;
    const int64_t t0 = block * blockDim.x + threadIdx.x;
    const StreamSubject &sub = subs[k];
    const int64_t i0 = item_base[k], S = sub.S, sb = clamp64(sub.s_begin, 0, S);
    const int32_t ns = items ? (int32_t)(item_base[k + 1] - i0) : 0;
    const int lane = lane_id();
    const auto offs = gview(sub.offsets);
    const int64_t P0 = ns > 0 ? offs[sb] : 0;
    const RangeOf range_of(ns > 0 ? offs[S] - P0 : 0, ns);
    for (int64_t b0 = t0 - lane; b0 < (ns > 0 ? S - sb : 0); b0 += stride) {   // (uniform over the wavefront)
        const int64_t s = sb + b0 + lane;
        const bool mine = s < S;
        const int32_t before = b0 > 0 ? range_of.equal(offs[sb + b0 - 1] - P0) : -1;
        const int32_t in = range_of.equal(offs[mine ? s : S] - P0);
        const int32_t hi = s == S - 1 ? ns - 1 : in;   // (the last streamline takes the items left over)
        const int32_t lo = __builtin_amdgcn_update_dpp(before, in, 0x138, 0xF, 0xF, false) + 1;   // wave_shr:1
#pragma unroll
        for (int q = 0; q < kShort; ++q)
            if (mine && lo + q <= hi) items[i0 + lo + q] = make_int2(k, (int)(lo + q <= in ? s : S));
        if (!__ballot(mine && lo + kShort <= hi)) continue;
#pragma unroll 1
        for (int q = kShort; q < kOwn; ++q)
            if (mine && lo + q <= hi) items[i0 + lo + q] = make_int2(k, (int)(lo + q <= in ? s : S));
        uint64_t rest = __ballot(mine && lo + kOwn <= hi);
        while (rest) {
            const int q = __builtin_ctzll(rest);
            rest &= rest - 1ull;
            const int32_t l = __builtin_amdgcn_readlane(lo, q), h = __builtin_amdgcn_readlane(hi, q),
                          n = __builtin_amdgcn_readlane(in, q);
            const int64_t sq = sb + b0 + q;
            for (int32_t i = l + kOwn + lane; i <= h; i += kWave) items[i0 + i] = make_int2(k, (int)(i <= n ? sq : S));
        }
    }
    // (the zero fills come last: a wait for a load also waits for the stores before it)
    if (sizes) grid_zero(sub.C, sizes[k], t0, stride);
    if (block_base || k == 0) {
        const int64_t threads = (int64_t)gridDim.x * blockDim.x;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nzero; i += threads) zero[i] = 0ull;
    }
}

hipError_t launch_prepare_batched(const StreamSubject *subs, const int64_t *item_base, const int64_t *sizes, int32_t nsub,
                                  const PrepareGrid &grid, const int64_t *block_base, int2 *items, unsigned long long *zero,
                                  int64_t nzero, hipStream_t st) {
    k_prepare_batched<<<dim3((unsigned)grid.blocks, grid.table ? 1u : (unsigned)nsub), kBlock, 0, st>>>(
        subs, item_base, sizes, nsub, grid.table ? block_base : nullptr, items, zero, nzero);
    return hipGetLastError();
}

template <int B, bool E, int U>
static int batched_blocks_per_cu_of(size_t dyn) {
    return resident_blocks(reinterpret_cast<const void *>(&k_count_batched<B, E, U>), dyn);
}

int count_batched_blocks_per_cu(int batch, int coarse_words, BatchedKind kind) {
    const size_t dyn = 4 * (size_t)kWavesPerBlock * (size_t)coarse_words;
    switch (kind) {
        case BatchedKind::kEnds:
            return batch == 2 ? batched_blocks_per_cu_of<2, true, 1>(dyn) : batched_blocks_per_cu_of<4, true, 1>(dyn);
        case BatchedKind::kUp2: return batched_blocks_per_cu_of<2, false, 2>(dyn);
        case BatchedKind::kUp4: return batched_blocks_per_cu_of<1, false, 4>(dyn);
        default:
            return batch == 2 ? batched_blocks_per_cu_of<2, false, 1>(dyn) : batched_blocks_per_cu_of<4, false, 1>(dyn);
    }
}

hipError_t launch_count_batched(const StreamSubject *subs, int32_t nsub, const int2 *items, int64_t nitems,
                                const Overflow &ovf, int32_t coarse_words, int blocks, int batch, BatchedKind kind, hipStream_t st) {
    if (nitems <= 0) return hipSuccess;
    const size_t dyn = 4 * (size_t)kWavesPerBlock * (size_t)coarse_words;
    switch (kind) {
        case BatchedKind::kEnds:
            if (batch == 2) k_count_batched<2, true, 1><<<blocks, kBlock, dyn, st>>>(subs, nsub, items, nitems, ovf, coarse_words);
            else k_count_batched<4, true, 1><<<blocks, kBlock, dyn, st>>>(subs, nsub, items, nitems, ovf, coarse_words);
            break;
        case BatchedKind::kUp2:   // two windows of two lookups each per batch, as k_count_stream_up<2>
            k_count_batched<2, false, 2><<<blocks, kBlock, dyn, st>>>(subs, nsub, items, nitems, ovf, coarse_words);
            break;
        case BatchedKind::kUp4:
            k_count_batched<1, false, 4><<<blocks, kBlock, dyn, st>>>(subs, nsub, items, nitems, ovf, coarse_words);
            break;
        default:
            if (batch == 2) k_count_batched<2, false, 1><<<blocks, kBlock, dyn, st>>>(subs, nsub, items, nitems, ovf, coarse_words);
            else k_count_batched<4, false, 1><<<blocks, kBlock, dyn, st>>>(subs, nsub, items, nitems, ovf, coarse_words);
            break;
    }
    return hipGetLastError();
}

// Alg. 1's count for table entries [lo, lo + gridDim.y): streamlines [s_begin, S) of each.
__global__ void k_count_seed_end_batched(const StreamSubject *__restrict__ subs, int32_t lo) {
    const StreamSubject &sub = subs[lo + blockIdx.y];
    seed_end_streamlines<CompactLookup, true>(sub.pts, sub.offsets, clamp64(sub.s_begin, 0, sub.S), sub.S, sub.scale, sub.g,
                                              CompactLookup{sub.cv}, sub.C, sub.si, sub.sm);
}

hipError_t launch_count_seed_end_batched(const StreamSubject *subs, int32_t lo, int32_t n, int cus, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    k_count_seed_end_batched<<<dim3((unsigned)(cus > 0 ? cus : 64) * 2, (unsigned)n), kBlock, 0, st>>>(subs, lo);
    return hipGetLastError();
}

hipError_t launch_fallback_batched(const StreamSubject *subs, int32_t nsub, const Overflow &ovf, FallbackScratch fs,
                                   hipStream_t st) {
    k_fallback_batched<<<fs.blocks, kBlock, 0, st>>>(subs, nsub, ovf, fs);
    return hipGetLastError();
}

template <typename Lookup>
static hipError_t launch_fallback(const CountArgs &a, const Lookup &lk, FallbackScratch fs, hipStream_t st) {
    if (a.scale != 1.0f) k_fallback<Lookup, true><<<fs.blocks, kBlock, 0, st>>>(a, lk, fs);
    else k_fallback<Lookup, false><<<fs.blocks, kBlock, 0, st>>>(a, lk, fs);
    return hipGetLastError();
}

hipError_t launch_fallback_raster(const CountArgs &a, const RasterVol &rv, FallbackScratch fs, hipStream_t st) {
    return launch_fallback(a, RasterLookup{rv}, fs, st);
}

hipError_t launch_fallback_compact(const CountArgs &a, const CompactVol &cv, FallbackScratch fs, hipStream_t st) {
    return launch_fallback(a, CompactLookup{cv}, fs, st);
}

// ---------------------------------------------------------------------------------------------
// transpose of the accumulation layout: C[i][m] (+)= CT[m][i], 32x32 tiles through LDS
// ---------------------------------------------------------------------------------------------

template <bool ACC>
__global__ void __launch_bounds__(256) k_transpose(const int32_t *__restrict__ CT, int32_t *__restrict__ C, int32_t N,
                                                   int32_t M) {
    __shared__ int32_t tile[32][33];
    const int i0 = blockIdx.x * 32, m0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    int32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = m0 + ty + 8 * q, i = i0 + tx;
        v[q] = (m < M && i < N) ? CT[(int64_t)m * N + i] : 0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[ty + 8 * q][tx] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = ty + 8 * q, i = i0 + k, m = m0 + tx;
        if (i < N && m < M) {
            int32_t *dst = C + (int64_t)i * M + m;
            *dst = ACC ? *dst + tile[tx][k] : tile[tx][k];
        }
    }
}

hipError_t launch_transpose(const int32_t *CT, int32_t *C, int32_t N, int32_t M, bool accumulate, hipStream_t st) {
    const dim3 grid((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32));
    if (accumulate) k_transpose<true><<<grid, 256, 0, st>>>(CT, C, N, M);
    else k_transpose<false><<<grid, 256, 0, st>>>(CT, C, N, M);
    return hipGetLastError();
}

// Grid-stride over the tiles of all jobs; each tile finds its job by a binary search over
// first_tile (block-uniform, so the barriers stay uniform).  A 64x64 tile gives every thread 16
// loads in flight before its stores.
__global__ void __launch_bounds__(256) k_transpose_many(const TransposeJob *__restrict__ jobs, int32_t njobs,
                                                        int64_t ntiles) {
    constexpr int T = kTransposeTile;
    __shared__ int32_t tile[T][T + 1];
    const int tx = threadIdx.x & (T - 1), ty = threadIdx.x / T;   // T x (256 / T)
    constexpr int R = 256 / T;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int lo = 0, hi = njobs;   // jobs[lo].first_tile <= t, and t < jobs[hi].first_tile (or ntiles)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (jobs[mid].first_tile <= t) lo = mid;
            else hi = mid;
        }
        const TransposeJob j = jobs[lo];
        const int64_t local = t - j.first_tile;
        const int64_t tn = (j.N + T - 1) / T;
        const int i0 = (int)(local % tn) * T, m0 = (int)(local / tn) * T;
        int32_t v[T / R];   // (a fixed trip count, so that all the loads issue before the LDS stores)
#pragma unroll
        for (int q = 0; q < T / R; ++q) {
            const int m = m0 + ty + q * R, i = i0 + tx;
            v[q] = (m < j.M && i < j.N) ? j.CT[(int64_t)m * j.N + i] : 0;
        }
#pragma unroll
        for (int q = 0; q < T / R; ++q) tile[ty + q * R][tx] = v[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < T / R; ++q) {
            const int i = i0 + ty + q * R, m = m0 + tx;
            if (i < j.N && m < j.M) j.C[(int64_t)i * j.M + m] = tile[tx][ty + q * R];
        }
        __syncthreads();   // the tile is rewritten by the next iteration
    }
}

hipError_t launch_transpose_many(const TransposeJob *jobs, int32_t njobs, int64_t ntiles, int cus, hipStream_t st) {
    if (njobs <= 0 || ntiles <= 0) return hipSuccess;
    const int64_t cap = (int64_t)(cus > 0 ? cus : 64) * 16;
    const unsigned blocks = (unsigned)std::min<int64_t>(ntiles, cap);
    k_transpose_many<<<blocks, 256, 0, st>>>(jobs, njobs, ntiles);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// histogram of appended C updates: each workgroup sorts its own updates by tile of C, then one LDS
// histogram per tile over every workgroup's run of it
// ---------------------------------------------------------------------------------------------

constexpr uint32_t kNoEntry = 0xFFFFFFFFu;   // never an update (updates index C: < 2^31)

// Slices [w0, w1) of workgroup b out of nblk.
__device__ __forceinline__ void slice_range(int32_t nwaves, int b, int nblk, int32_t &w0, int32_t &w1) {
    w0 = (int32_t)((int64_t)nwaves * b / nblk);
    w1 = (int32_t)((int64_t)nwaves * (b + 1) / nblk);
}

constexpr int kMaxSlicesPerBlock = 64;   // nblk >= nwaves / 64 (checked by the launcher)

// Exclusive scan of c[0 .. n) in LDS (n <= kMaxPairTiles) by a 1024-thread workgroup; thread i
// owns entries 4i .. 4i+3.  wsum: 16 words of LDS.  Every 2^every_log2-th entry of the scan, and the
// total after them, also go to o[].
__device__ __forceinline__ uint32_t block_scan_tiles(uint32_t *c, int32_t n, uint32_t *wsum, uint16_t *__restrict__ o,
                                                     int every_log2) {
    static_assert(kMaxPairTiles == 4 * 1024, "four tiles per thread");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t s = 0u, own[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int t = 4 * tid + q;
        own[q] = t < n ? c[t] : 0u;
        s += own[q];
    }
    uint32_t x = s;   // inclusive scan over the wavefront
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    uint32_t before = 0u, total = 0u;
    for (int k = 0; k < 16; ++k) {
        const uint32_t w = wsum[k];
        before += k < wv ? w : 0u;
        total += w;
    }
    uint32_t run = before + x - s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int t = 4 * tid + q;
        if (t < n) {
            c[t] = run;
            if ((t & ((1 << every_log2) - 1)) == 0) o[t >> every_log2] = (uint16_t)run;
        }
        run += own[q];
    }
    if (tid == 0) o[n >> every_log2] = (uint16_t)total;
    return total;
}

// Workgroups [0, fs.blocks): the overflow queue (the fallback of a pair-buffer call; it adds to C
// atomically, and C is not touched otherwise before the tile pass).
// Workgroups fs.blocks + b, b < nblk: the updates of slices [w0, w1) in rounds of up to kPairRound,
// each round grouped by tile in LDS and written to sorted[] in that order, coalesced, as 16-bit indices
// within their tile.  Round j of workgroup b starts at sorted[blk[b].y + j * kPairRound] and is run table
// row j * nblk + b: off[row][t] = where its updates of tile t start in the round (off[row][ntiles]: its
// end); blk[b].x = its rounds.
//
// Bound by latency on a million updates, by memory and LDS atomics on ten million.  A sort of all
// updates at once (tile histograms and run reservations with an atomic per workgroup and tile, then a
// pass that stored each update into its tile's run) took 26 us for 2M updates after a fallback launch
// of 5 us, and 86 us after 12 us for 11M; here no workgroup waits for another, and the two passes over
// the updates take 14 and 44 us with the fallback beside them.  Two workgroups per CU: 64 VGPRs and
// 48.6 KB of LDS each.
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8), amdgpu_num_sgpr(80)))
k_pair_sort(PairOut po, int32_t nwaves, int32_t ntiles, int32_t tile_log2, int32_t nblk, uint2 *__restrict__ blk,
            uint16_t *__restrict__ off, uint16_t *__restrict__ sorted, CountArgs a, CompactLookup lk, FallbackScratch fs) {
    constexpr int kUnroll = 4;
    __shared__ uint32_t cnt[kMaxPairTiles];                      // the round's count per bin, then its offset in stage
    __shared__ __align__(16) uint16_t stage[kPairRound];         // the round's updates, grouped by tile
    __shared__ uint32_t pre[kMaxSlicesPerBlock + 1];
    __shared__ uint32_t wsum[16];
    __shared__ int s_nlab;
    if (blockIdx.x < (unsigned)fs.blocks) {
        fallback_queue<CompactLookup, true>(a, lk, fs, &s_nlab);
        return;
    }
    const int b = (int)blockIdx.x - fs.blocks;
    int32_t w0, w1;
    slice_range(nwaves, b, nblk, w0, w1);
    const int ns = w1 - w0;
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        uint32_t x = lane < ns ? min(po.counts[w0 + lane], po.cap) : 0u;   // (past ns: pre = the total)
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(x, d);
            if (lane >= d) x += y;
        }
        pre[lane + 1] = x;
        if (lane == 0) pre[0] = 0u;
    }
    __syncthreads();
    const uint32_t total = pre[ns];
    const uint32_t out0 = (uint32_t)w0 * po.cap;   // (nwaves * cap < 2^31, cap a multiple of 8)
    const uint32_t *src = po.pairs + (size_t)w0 * po.cap;   // (at most 64 slices: 32-bit offsets)
    // A tile has 2^copies_log2 neighbouring bins, a lane counts in the one of its number: neighbouring
    // updates mostly share a tile, and atomics on one LDS word are served one after another.
    const int copies_log2 = min(4, 31 - __clz(kMaxPairTiles / ntiles));
    const int32_t nbins = ntiles << copies_log2;
    const uint32_t copy = threadIdx.x & ((1u << copies_log2) - 1u);
    auto bin = [&](uint32_t e) { return ((e >> tile_log2) << copies_log2) | copy; };
    int row = b;
    for (uint32_t r0 = 0; r0 < total; r0 += kPairRound, row += nblk) {   // uniform over the workgroup
        for (int t = threadIdx.x; t < nbins; t += 1024) cnt[t] = 0u;
        const uint32_t r1 = min(total, r0 + (uint32_t)kPairRound);
        // f(update) for the round's updates, kUnroll loads in flight.  Both passes below load them (the
        // second time from the caches): held in registers, the code is unrolled for all of them, and
        // fetching it takes longer than running it.
        auto for_each = [&](auto &&f) {
#pragma unroll 1
            for (uint32_t k0 = r0 + threadIdx.x; k0 < r1; k0 += kUnroll * 1024u) {
                uint32_t v[kUnroll];
#pragma unroll
                for (int j = 0; j < kUnroll; ++j) {
                    const uint32_t k = k0 + j * 1024u;
                    int lo = 0;   // the slice holding flat index k: pre[lo] <= k < pre[lo + 1]
#pragma unroll
                    for (int d = kMaxSlicesPerBlock / 2; d > 0; d >>= 1) lo += pre[lo + d] <= k ? d : 0;
                    v[j] = kNoEntry;
                    if (k < r1) v[j] = src[(uint32_t)lo * po.cap + (k - pre[lo])];
                }
#pragma unroll
                for (int j = 0; j < kUnroll; ++j)
                    if ((v[j] >> tile_log2) < (uint32_t)ntiles) f(v[j]);   // (kNoEntry: no tile)
            }
        };
        __syncthreads();
        for_each([&](uint32_t e) { atomicAdd(&cnt[bin(e)], 1u); });
        __syncthreads();
        const uint32_t n = block_scan_tiles(cnt, nbins, wsum, off + (size_t)row * (ntiles + 1), copies_log2);
        __syncthreads();
        const uint32_t low = (1u << tile_log2) - 1u;
        for_each([&](uint32_t e) { stage[atomicAdd(&cnt[bin(e)], 1u)] = (uint16_t)(e & low); });
        __syncthreads();
        uint4 *dst = reinterpret_cast<uint4 *>(sorted + out0 + r0);   // (16-byte aligned: multiples of 8 entries)
        for (uint32_t i = threadIdx.x; i < (n + 7) / 8; i += 1024u) dst[i] = reinterpret_cast<const uint4 *>(stage)[i];
        __syncthreads();
    }
    if (threadIdx.x == 0) blk[b] = make_uint2((total + kPairRound - 1) / kPairRound, out0);
}

// One workgroup per tile of 2^kLog2 entries: C[tile] += the histogram of the tile's updates.  Eight
// lanes read a run together, kRuns runs of a group in flight.  C's entries are loaded behind the first
// updates: loads complete in order, so ahead of them they would hold the updates up.  (Reading whole
// tiles from one sorted array took 20 us for 2M updates in 35 tiles, 14 us for 1M in 503 and 19 us for
// 11M; this takes 11, 15 and 35 us, in exchange for the passes above.)  A wavefront one of whose runs has 72
// updates or more takes the long ones 64 at a time, equal neighbours added together: a small C, or one
// whose updates gather in a few tiles, is bound by the hot tile's LDS atomics.  Eight at a time, one
// tile of 2032 entries took 89 us for 1M streamlines' updates, now 47; four hot entries 250 us for 100k
// streamlines', now 88.
template <int kLog2>
__global__ void __launch_bounds__(512) k_pair_tile_add(const uint16_t *__restrict__ sorted, const uint16_t *__restrict__ off,
                                                       const uint2 *__restrict__ blk, int32_t nblk, int32_t ntiles,
                                                       int32_t *__restrict__ Cm, int64_t NM) {
    constexpr uint32_t kTile = 1u << kLog2;
    constexpr int kSteps = kTile / (4 * 512);
    constexpr int kRuns = kPairBlocks / 64;
    static_assert(kSteps >= 1 && kPairBlocks == 64 * kRuns, "512 threads: 64 groups of 8 lanes");
    __shared__ __align__(16) uint32_t h[kTile];
    const int64_t t0 = (int64_t)blockIdx.x << kLog2;
    int32_t *C = Cm + t0;   // the tile's entries of C
    const uint32_t len = (uint32_t)min((int64_t)kTile, NM - t0);
    const bool whole = len == kTile && (reinterpret_cast<uintptr_t>(C) & 15u) == 0;
    const int grp = threadIdx.x >> 3, l8 = threadIdx.x & 7;
    uint2 run[kRuns];
    uint32_t most = 0u;
#pragma unroll
    for (int k = 0; k < kRuns; ++k) {
        const int b = grp + 64 * k;
        run[k] = b < nblk ? blk[b] : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int j = 0; j < kSteps; ++j) reinterpret_cast<uint4 *>(h)[threadIdx.x + j * 512] = make_uint4(0u, 0u, 0u, 0u);
    uint32_t s[kRuns], e[kRuns], longest = 0u;
    auto bounds = [&](uint32_t j) {   // of the groups' runs in round j
        uint32_t a0[kRuns], a1[kRuns];
#pragma unroll
        for (int k = 0; k < kRuns; ++k) {
            const uint16_t *o = off + (size_t)(j * nblk + grp + 64 * k) * (ntiles + 1) + blockIdx.x;
            a0[k] = a1[k] = 0u;
            if (j < run[k].x) {
                a0[k] = o[0];
                a1[k] = o[1];
            }
        }
#pragma unroll
        for (int k = 0; k < kRuns; ++k) {
            const uint32_t at = run[k].y + j * (uint32_t)kPairRound;
            s[k] = at + a0[k] + l8;
            e[k] = at + a1[k];
            longest = max(longest, a1[k] - a0[k]);
        }
    };
    uint32_t v[kRuns];
    auto load = [&]() -> bool {   // the next updates of the groups' runs; true if there are more after them
        bool more = false;
#pragma unroll
        for (int k = 0; k < kRuns; ++k) {
            v[k] = kNoEntry;
            if (s[k] < e[k]) v[k] = sorted[s[k]];
            s[k] += 8u;
            more |= s[k] < e[k];
        }
        return __any(more);
    };
    auto add = [&]() {
#pragma unroll
        for (int k = 0; k < kRuns; ++k)
            if (v[k] != kNoEntry) atomicAdd(&h[v[k]], 1u);
    };
    // Runs with 64 updates or more to go (a tile that holds many of a workgroup's updates): 16 bytes a lane,
    // from the 16-byte boundary at or below the group's next update.  Such a step ends within the run.
    auto add_long = [&]() {
        for (;;) {
            uint4 w[kRuns];
            uint32_t from[kRuns];   // the group's next update, or kNoEntry
            bool any = false;
#pragma unroll
            for (int k = 0; k < kRuns; ++k) {
                from[k] = s[k] - l8;
                if (from[k] + 64u > e[k]) from[k] = kNoEntry;
                w[k] = make_uint4(0u, 0u, 0u, 0u);
                if (from[k] != kNoEntry) w[k] = reinterpret_cast<const uint4 *>(sorted)[(from[k] >> 3) + l8];
                any |= from[k] != kNoEntry;
            }
            if (!__any(any)) return;
#pragma unroll
            for (int k = 0; k < kRuns; ++k)
                if (from[k] != kNoEntry) {
                    const uint32_t at = (from[k] & ~7u) + 8u * l8;
                    const uint32_t q[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
                    uint32_t cnt = 0u;   // equal neighbours are added together
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t u = i & 1 ? q[i >> 1] >> 16 : q[i >> 1] & 0xFFFFu;
                        cnt += at + i >= from[k] ? 1u : 0u;
                        if (i == 7 || (i & 1 ? q[(i + 1) >> 1 & 3] & 0xFFFFu : q[i >> 1] >> 16) != u) {
                            if (cnt) atomicAdd(&h[u], cnt);
                            cnt = 0u;
                        }
                    }
                    s[k] = (from[k] & ~7u) + 64u + l8;
                }
        }
    };
    bounds(0u);
    bool more = load();
    __builtin_amdgcn_sched_barrier(0);
    const bool any_long = __any(longest >= 8u + 64u);   // (8 updates of each run are under way)
    int4 c[kSteps];
    auto load_c = [&]() {
#pragma unroll
        for (int j = 0; j < kSteps; ++j) c[j] = reinterpret_cast<const int4 *>(C)[threadIdx.x + j * 512];
    };
    if (whole && !any_long) load_c();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kRuns; ++k) most = max(most, run[k].x);
    __syncthreads();   // h is zero
    if (any_long) {
        // (a loop of its own: with the long steps inside the other one, a C of 14M entries took 2% longer a call)
        add();
        for (uint32_t j = 0;;) {
            add_long();
            do {
                more = load();
                add();
            } while (more);
            ++j;
            if (!__any(j < most)) break;
            bounds(j);
        }
        if (whole) load_c();
    } else {
        for (uint32_t j = 0;;) {
            add();
            if (more) {
                more = load();
                continue;
            }
            ++j;
            if (!__any(j < most)) break;
            bounds(j);
            more = load();
        }
    }
    __syncthreads();
    if (whole) {
        int4 *C4 = reinterpret_cast<int4 *>(C);
        const uint4 *h4 = reinterpret_cast<const uint4 *>(h);
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const uint4 d = h4[threadIdx.x + j * 512];
            c[j].x += (int)d.x;
            c[j].y += (int)d.y;
            c[j].z += (int)d.z;
            c[j].w += (int)d.w;
            C4[threadIdx.x + j * 512] = c[j];
        }
    } else {
        for (uint32_t k = threadIdx.x; k < len; k += blockDim.x) C[k] += (int32_t)h[k];
    }
}

hipError_t launch_pair_histogram(const PairOut &po, int32_t nwaves, const PairTiles &pt, const CountArgs &a,
                                 const CompactVol &cv, FallbackScratch fs, int32_t *C, int64_t NM, uint32_t *hist,
                                 uint32_t *sorted32, hipStream_t st) {
    if (pt.n < 1 || pt.n > kMaxPairTiles || nwaves < 1 || pt.blocks < 1) return hipErrorInvalidValue;
    if ((int64_t)pt.blocks * kMaxSlicesPerBlock < nwaves) return hipErrorInvalidValue;
    uint2 *blk = reinterpret_cast<uint2 *>(hist);
    uint16_t *off = reinterpret_cast<uint16_t *>(hist + 2 * kPairBlocks), *sorted = reinterpret_cast<uint16_t *>(sorted32);
    k_pair_sort<<<fs.blocks + pt.blocks, 1024, 0, st>>>(po, nwaves, pt.n, pt.log2, pt.blocks, blk, off, sorted, a,
                                                       CompactLookup{cv}, fs);
    switch (pt.log2) {
        case 11: k_pair_tile_add<11><<<pt.n, 512, 0, st>>>(sorted, off, blk, pt.blocks, pt.n, C, NM); break;
        case 12: k_pair_tile_add<12><<<pt.n, 512, 0, st>>>(sorted, off, blk, pt.blocks, pt.n, C, NM); break;
        case 13: k_pair_tile_add<13><<<pt.n, 512, 0, st>>>(sorted, off, blk, pt.blocks, pt.n, C, NM); break;
        default: k_pair_tile_add<14><<<pt.n, 512, 0, st>>>(sorted, off, blk, pt.blocks, pt.n, C, NM); break;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// ceiling probes: what the counting path can reach on this device at best
// ---------------------------------------------------------------------------------------------

constexpr uint32_t kProbeMagic = 0x9E3779B9u;   // a folded value that (practically) never occurs

// Points [P][3] streamed read-only with the counting kernel's access pattern: one contiguous range
// per wavefront, 64 x 12-byte non-temporal buffer loads, kBatch windows per step.  The loaded bits
// are folded into one word per lane, stored only if it equals kProbeMagic, so the loads stay.
template <int kBatch>
__global__ void __launch_bounds__(kBlock) k_probe_stream(const float *__restrict__ pts, int64_t P, int64_t nwaves,
                                                         uint32_t *__restrict__ sink) {
    const int lane = lane_id();
    // (the wave index through readfirstlane: a range derived from threadIdx would make the buffer
    // resource divergent and put every load in a loop over lanes)
    const int64_t wave = (int64_t)blockIdx.x * kWavesPerBlock + uniform32((int)(threadIdx.x >> 6));
    const int64_t per = (P + nwaves - 1) / nwaves;
    const int64_t p0 = min(P, wave * per), p1 = min(P, p0 + per);
    const uint32_t L = (uint32_t)(p1 - p0);
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(pts + 3 * p0, 12ull * L);
    const uint32_t lane12 = 12u * (uint32_t)lane;
    uint32_t acc = 0u;
    for (uint32_t w0 = 0; w0 < L; w0 += kBatch * kWave) {
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b96(rp, lane12, 12u * w0 + 768u * b, kAuxStream);
            acc ^= v[0] ^ (v[1] << 1) ^ (v[2] << 2);
        }
    }
    if (acc == kProbeMagic) sink[0] = acc;
}

// No-return int32 atomic adds C[idx[k]] += 1, k < n (indices >= n_words are skipped), four index
// loads in flight per thread before their atomics.
__global__ void __launch_bounds__(kBlock) k_probe_atomics(int32_t *__restrict__ C, int64_t n_words,
                                                          const uint32_t *__restrict__ idx, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k0 < n; k0 += 4 * stride) {
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t k = k0 + j * stride;
            v[j] = k < n ? idx[k] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((int64_t)v[j] < n_words) atomicAdd(C + v[j], 1);
    }
}

// The counting kernel's per-point lookups without its per-streamline work: the point stream of
// k_probe_stream, voxelisation, the coarse test in LDS, the (word, rank base) gather and, for
// occupied voxels, the code gather, in the counting kernel's software pipeline (each iteration
// issues batch k's code gathers, batch k+1's pair gathers and batch k+2's points, then decodes
// batch k).  The decoded rows and labels are folded like the stream probe.  No de-duplication,
// no pair updates: the stream-plus-lookup ceiling of the flat-stream kernel.
template <int kBatch, bool kBrick>
__global__ void __launch_bounds__(kBlock) k_probe_lookup(StreamSubject sub, int64_t P, int64_t nwaves,
                                                         uint32_t *__restrict__ sink) {
    extern __shared__ __align__(16) uint32_t s_coarse[];
    const CompactVol &cv = sub.cv;
    put_coarse(cv, s_coarse, get_coarse(cv, threadIdx.x), threadIdx.x, kBlock);
    __syncthreads();
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * kWavesPerBlock + uniform32((int)(threadIdx.x >> 6));
    const int64_t per = (P + nwaves - 1) / nwaves;
    const int64_t p0 = min(P, wave * per), p1 = min(P, p0 + per);
    const uint32_t L = (uint32_t)(p1 - p0);
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(sub.pts + 3 * p0, 12ull * L);
    const __amdgpu_buffer_rsrc_t rvol = make_rsrc(cv.mb, cv.span);
    const uint32_t lane12 = 12u * (uint32_t)lane;
    uint32_t bX = fbits(sub.g.Xf), bY = fbits(sub.g.Yf), bZ = fbits(sub.g.Zf);
    asm volatile("" : "+v"(bX), "+v"(bY), "+v"(bZ));
    const uint32_t SBX = (uint32_t)cv.SBX, SBXY = (uint32_t)cv.SBXY;
    const uint32_t csx = (uint32_t)cv.csx, csyz = (uint32_t)cv.csyz, CBX = (uint32_t)cv.CBX, CBXY = (uint32_t)cv.CBXY;
    const int codes_off = uniform32((int)cv.codes_off);
    constexpr uint32_t kOutOfRange = 0xFFFFFFF8u;
    const uint32_t code_oob = kOutOfRange - (uint32_t)codes_off;
    constexpr uint32_t BW = kWave * kBatch;
    float ax[kBatch], ay[kBatch], az[kBatch];
    auto load_batch = [&](uint32_t w) {
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b96(rp, lane12, 12u * w + 768u * b, kAuxStream);
            ax[b] = __uint_as_float(v[0]);
            ay[b] = __uint_as_float(v[1]);
            az[b] = __uint_as_float(v[2]);
        }
    };
    auto lookup = [&](uint32_t w0, uint32_t (&addr)[kBatch], uint32_t (&bix)[kBatch]) {
        const uint32_t left = w0 < L ? L - w0 : 0u;
        const int rem = left > BW ? (int)BW : (int)left;
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const float tx = __fadd_rn(__fmul_rn(ax[b], sub.scale), 0.5f);
            const float ty = __fadd_rn(__fmul_rn(ay[b], sub.scale), 0.5f);
            const float tz = __fadd_rn(__fmul_rn(az[b], sub.scale), 0.5f);
            const bool ok = (int)(lane + b * kWave < rem) & (int)(fbits(tx) < bX) & (int)(fbits(ty) < bY) &
                            (int)(fbits(tz) < bZ);
            const uint32_t ix = (uint32_t)(int)tx, iy = (uint32_t)(int)ty, iz = (uint32_t)(int)tz;
            uint32_t sb = __umul24(iz >> 3, SBXY) + __umul24(iy >> 3, SBX) + (ix >> 4);
            asm("" : "+v"(sb));
            const uint32_t cb = kBrick ? sb : __umul24(iz >> csyz, CBXY) + __umul24(iy >> csyz, CBX) + (ix >> csx);
            const uint32_t cw = s_coarse[ok ? (cb >> 5) : 0u];
            const bool hit = (int)ok & (int)(__builtin_amdgcn_ubfe(cw, cb, 1) != 0u);
            addr[b] = hit ? (sb << 8) | ((iy << 2) & 0x18u) | ((iz << 5) & 0xE0u) : kOutOfRange;
            bix[b] = (ix & 15u) | ((iy & 1u) << 4);
        }
    };
    auto gather_pairs = [&](const uint32_t (&addr)[kBatch], uint32_t (&mw)[kBatch], uint32_t (&base)[kBatch]) {
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const auto e = __builtin_amdgcn_raw_buffer_load_b64(rvol, addr[b], 0, kAuxCached);
            mw[b] = e[0];
            base[b] = e[1];
        }
    };
    uint32_t acc = 0u;
    uint32_t bix[kBatch], mw[kBatch], base[kBatch];
    {
        uint32_t addr[kBatch];
        load_batch(0u);
        lookup(0u, addr, bix);
        __builtin_amdgcn_sched_barrier(0);
        gather_pairs(addr, mw, base);
        __builtin_amdgcn_sched_barrier(0);
        load_batch(BW);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (uint32_t w0 = 0; w0 < L; w0 += BW) {
        bool flag[kBatch];
        uint32_t c[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            flag[b] = __builtin_amdgcn_ubfe(mw[b], bix[b], 1) != 0u;
            const uint32_t at = base[b] + __popc(__builtin_amdgcn_ubfe(mw[b], 0, bix[b]));
            const uint32_t off = flag[b] ? at << 2 : code_oob;
            c[b] = __builtin_amdgcn_raw_buffer_load_b32(rvol, off, codes_off, kAuxCached);
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t bix2[kBatch], mw2[kBatch], base2[kBatch];
        {
            uint32_t addr[kBatch];
            lookup(w0 + BW, addr, bix2);
            __builtin_amdgcn_sched_barrier(0);
            gather_pairs(addr, mw2, base2);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_batch(w0 + 2 * BW);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const uint32_t rv = c[b] & cv.rmask, mv = c[b] >> cv.rbits;
            acc += flag[b] ? (rv ^ (mv << 3)) : 0u;
            bix[b] = bix2[b];
            mw[b] = mw2[b];
            base[b] = base2[b];
        }
    }
    if (acc == kProbeMagic) sink[0] = acc;
}

hipError_t launch_probe_stream(const float *pts, int64_t P, int cus, uint32_t *sink, hipStream_t st) {
    if (P <= 0) return hipSuccess;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(&k_probe_stream<4>),
                                                     kBlock, 0) != hipSuccess || per_cu < 1)
        per_cu = 4;
    const int64_t blocks = (int64_t)cus * per_cu;
    k_probe_stream<4><<<(unsigned)blocks, kBlock, 0, st>>>(pts, P, blocks * kWavesPerBlock, sink);
    return hipGetLastError();
}

hipError_t launch_probe_atomics(int32_t *C, int64_t n_words, const uint32_t *idx, int64_t n, int cus, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + kBlock - 1) / kBlock, (int64_t)cus * 8);
    k_probe_atomics<<<(unsigned)blocks, kBlock, 0, st>>>(C, n_words, idx, n);
    return hipGetLastError();
}

hipError_t launch_probe_lookup(const StreamSubject &sub, int64_t P, int cus, uint32_t *sink, hipStream_t st) {
    if (P <= 0) return hipSuccess;
    const size_t dyn = coarse_lds_bytes(sub.cv.ncoarse_words);
    const bool brick = sub.cv.csx == 4 && sub.cv.csyz == 3;
    const void *fn = brick ? reinterpret_cast<const void *>(&k_probe_lookup<4, true>)
                           : reinterpret_cast<const void *>(&k_probe_lookup<4, false>);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, dyn) != hipSuccess || per_cu < 1) per_cu = 4;
    const int64_t blocks = (int64_t)cus * per_cu;
    if (brick) k_probe_lookup<4, true><<<(unsigned)blocks, kBlock, dyn, st>>>(sub, P, blocks * kWavesPerBlock, sink);
    else k_probe_lookup<4, false><<<(unsigned)blocks, kBlock, dyn, st>>>(sub, P, blocks * kWavesPerBlock, sink);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// validation
// ---------------------------------------------------------------------------------------------

__global__ void k_validate(const int64_t *__restrict__ offsets, int64_t S, const int32_t *__restrict__ roi,
                           const int32_t *__restrict__ lab, int64_t nvox, int32_t N, int32_t M, int32_t *flags) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int f = 0;
    if (t0 == 0 && offsets[0] != 0) f |= 1;
    for (int64_t s = t0; s < S; s += stride)
        if (offsets[s + 1] < offsets[s]) f |= 1;
    for (int64_t v = t0; v < nvox; v += stride) {
        if (roi[v] >= N) f |= 2;
        if (lab[v] >= M) f |= 4;
    }
    if (f) atomicOr(flags, f);
}

hipError_t launch_validate(const int64_t *offsets, int64_t S, const int32_t *roi, const int32_t *lab, int64_t nvox,
                           int32_t N, int32_t M, int32_t *flags, int cus, hipStream_t st) {
    k_fill_i32<<<1, kWave, 0, st>>>(flags, 1, 0);
    const int64_t n = S > nvox ? S : nvox;
    k_validate<<<fill_blocks(n, cus), kBlock, 0, st>>>(offsets, S, roi, lab, nvox, N, M, flags);
    return hipGetLastError();
}

}  // namespace fc
