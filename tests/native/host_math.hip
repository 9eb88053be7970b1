// Host build of the arithmetic that the kernels share with the host (csrc/internal.h), for
// tests/test_host_math.py.
#include "host.h"
#include "internal.h"

extern "C" {

// xs, d and mine of the lane at x in a row of X voxels
void row_lane(int wide, int32_t x, int32_t X, int32_t out[3]) {
    const fc::RowLane r = wide ? fc::row_lane<true>(x, X) : fc::row_lane<false>(x, X);
    out[0] = r.xs;
    out[1] = r.d;
    out[2] = (int32_t)r.mine;
}

// compact layout of a grid: 1 and {row bits, row mask, bytes, offset of the codes}, or 0 if it is refused
int layout(const int32_t dims[3], int32_t N, int32_t M, int64_t out[4]) {
    fch::CompactLayout L;
    if (!fch::compact_layout(dims, N, M, L, fch::kMaxCoarseWords, true)) return 0;
    const fc::CompactVol cv = fch::compact_view(nullptr, L, N, M);
    out[0] = cv.rbits;
    out[1] = cv.rmask;
    out[2] = (int64_t)L.bytes;
    out[3] = cv.codes_off;
    return 1;
}

// ranges of n point positions, of nparts tapering or (equal) equal ranges over P points
void range_of(int64_t P, int64_t nparts, int equal, const int64_t *p, int64_t n, int32_t *out) {
    const fc::RangeOf r(P, nparts);
    for (int64_t k = 0; k < n; ++k) out[k] = equal ? r.equal(p[k]) : r(p[k]);
}

// workgroups of a preparation launch: 1 with base[0 .. n] if they go by the table, else 0 and base[0] = those of each subject
int prepare_grid(const int64_t *work, int32_t n, int64_t nzero, int cus, int64_t *base) {
    const fc::PrepareGrid g = fc::prepare_grid(work, n, nzero, cus, base);
    if (!g.table) base[0] = g.blocks;
    return g.table && g.blocks == base[n] ? 1 : (g.table ? -1 : 0);
}

}
