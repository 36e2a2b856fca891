// Inner product of two sparse tensors with different patterns (the TIN
// statement with no free index, Sec. II-A): a = sum over the coordinates
// both store of B * C.  The co-iteration intersects the operands level by
// level (the paper's coordinate-tree iteration, Sec. IV-C): a coordinate of
// B's last-but-one level — a position of a CSR matrix, a fiber of a CSF
// tensor — is looked up in C's segment of the same parent by binary search;
// the entries of a fiber are then looked up in the matching C fiber.
//
// CSR (k_inner_matrix): a workgroup takes kUnitIters * 256 consecutive
// positions, a lane every 256th.  The parent of each comes from the parent
// pos entries of the workgroup's range, staged in LDS, and so do C's parent
// pos entries and the C coordinates that can match: positions are sorted by
// (parent, coordinate), so the matches of the range lie between the first
// position of C's first parent holding a coordinate at or past the range's
// first, and the last position of C's last parent holding one at or below
// the range's last.  The searches then run in LDS.  Those range bounds come
// from a pre-pass (k_inner_bounds, a lane per workgroup boundary, all
// searching at once) rather than from a serial search at the start of each
// workgroup.  When more than kParents parents or kCStage C coordinates fall
// in the range, each lane searches pos and crd in HBM instead.
//
// CSF (k_inner_fibers): see there.
//
// Products are summed in double: each lane, then a fixed tree over the
// workgroup into one partial per workgroup, then a fixed-order final pass
// (k_inner_final), so the result does not depend on timing.
#include "device.hpp"
#include "internal.hpp"

namespace spl {
namespace {

constexpr int kParents = 1024;   // parents staged per workgroup
constexpr int kCStage = 2560;    // C coordinates staged per workgroup
constexpr int kUnitIters = 8;    // units per lane

// Largest r in [lo, hi) with pos[r] <= u (the parent holding unit u); I is
// the index type (32-bit where the indices are LDS offsets, fewer VALU
// instructions a step).
template <typename I, typename P>
__device__ __forceinline__ I parent_of(const P &pos, I lo, I hi, I u) {
    while (hi - lo > 1) {
        const I mid = (lo + hi) >> 1;
        if (static_cast<I>(pos(mid)) <= u)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// First position in the sorted crd[lo, hi) whose coordinate is at least j
// (UPPER false) or above j (UPPER true).
template <bool UPPER>
__device__ __forceinline__ int64_t bound_sorted(const int32_t *__restrict__ crd, int64_t lo,
                                                int64_t hi, int32_t j) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (UPPER ? crd[mid] <= j : crd[mid] < j)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Position of coordinate j in the sorted crd[lo, hi), or -1.
template <typename I, typename C>
__device__ __forceinline__ I find_sorted(const C &crd, I lo, I hi, int32_t j) {
    while (lo < hi) {
        const I mid = (lo + hi) >> 1;
        const int32_t v = crd(mid);
        if (v == j) return mid;
        if (v < j)
            lo = mid + 1;
        else
            hi = mid;
    }
    return -1;
}

// Range bounds of every workgroup: for boundary b (unit u_b = b * span,
// capped at units), the parent of u_b and the first C position of that
// parent whose coordinate is at least u_b's (the start of workgroup b), and
// the parent of u_b - 1 and the first C position of that parent whose
// coordinate is above u_b - 1's (the end of workgroup b - 1).
__global__ __launch_bounds__(kBlock) void k_inner_bounds(int64_t n, int64_t units, int64_t span,
                                                         int64_t parts,
                                                         const int32_t *__restrict__ bpos,
                                                         const int32_t *__restrict__ bcrd,
                                                         const int32_t *__restrict__ cpos,
                                                         const int32_t *__restrict__ ccrd,
                                                         int64_t *__restrict__ bnd) {
    const int64_t b = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (b > parts) return;
    const int64_t ub = b * span < units ? b * span : units;
    auto gpos = [&](int64_t r) { return bpos[r]; };
    int64_t ra = 0, ca = 0, rb = 0, cb = 0;
    if (ub < units) {
        ra = parent_of<int64_t>(gpos, 0, n, ub);
        ca = bound_sorted<false>(ccrd, cpos[ra], cpos[ra + 1], bcrd[ub]);
    }
    if (ub > 0) {
        rb = parent_of<int64_t>(gpos, 0, n, ub - 1);
        cb = bound_sorted<true>(ccrd, cpos[rb], cpos[rb + 1], bcrd[ub - 1]);
    }
    bnd[4 * b] = ra;
    bnd[4 * b + 1] = ca;
    bnd[4 * b + 2] = rb;
    bnd[4 * b + 3] = cb;
}

template <typename V>
__global__ __launch_bounds__(kBlock) void k_inner_matrix(
    int64_t units, const int32_t *__restrict__ bpos, const int32_t *__restrict__ bcrd,
    const V *__restrict__ bv, const int32_t *__restrict__ cpos, const int32_t *__restrict__ ccrd,
    const V *__restrict__ cv, const int64_t *__restrict__ bnd, double *__restrict__ part) {
    __shared__ int32_t s_pos[kParents + 1];   // B's parent pos entries of the range
    __shared__ int32_t s_cpos[kParents + 1];  // C's
    __shared__ int32_t s_ccrd[kCStage];       // C's coordinates that can match
    __shared__ double s_sum[kBlock / kWave];
    static_assert(kBlock / kWave == 4, "four waves per workgroup");
    const int64_t u0 = static_cast<int64_t>(blockIdx.x) * (kBlock * kUnitIters);
    const int64_t u1 = u0 + kBlock * kUnitIters < units ? u0 + kBlock * kUnitIters : units;
    auto gpos = [&](int64_t r) { return bpos[r]; };
    const int64_t w = blockIdx.x;
    const int64_t r0 = bnd[4 * w], c0 = bnd[4 * w + 1];
    const int64_t cnt = bnd[4 * w + 6] - r0 + 1, c1 = bnd[4 * w + 7];
    const bool staged = cnt <= kParents && c1 - c0 <= kCStage;
    if (staged) {
        // every lane issues all its loads before any store (past a run: 0,
        // with no access), so the copy costs one round of loads, not one
        // per loop iteration
        constexpr int kPosPer = (kParents + 1 + kBlock - 1) / kBlock;
        constexpr int kCPer = (kCStage + kBlock - 1) / kBlock;
        const int np = static_cast<int>(cnt) + 1;
        const int nc = c1 > c0 ? static_cast<int>(c1 - c0) : 0;
        const __amdgpu_buffer_rsrc_t rp = span_rsrc(bpos + r0, 4u * np);
        const __amdgpu_buffer_rsrc_t rq = span_rsrc(cpos + r0, 4u * np);
        const __amdgpu_buffer_rsrc_t rc = span_rsrc(ccrd + c0, 4u * nc);
        uint32_t a[kPosPer], b[kPosPer], c[kCPer];
#pragma unroll
        for (int i = 0; i < kPosPer; ++i) {
            const int k = i * kBlock + threadIdx.x;
            a[i] = buf_u32(rp, k < np ? 4u * k : kBufOut);
            b[i] = buf_u32(rq, k < np ? 4u * k : kBufOut);
        }
#pragma unroll
        for (int i = 0; i < kCPer; ++i) {
            const int k = i * kBlock + threadIdx.x;
            c[i] = buf_u32(rc, k < nc ? 4u * k : kBufOut);
        }
#pragma unroll
        for (int i = 0; i < kPosPer; ++i) {
            const int k = i * kBlock + threadIdx.x;
            if (k < np) {
                s_pos[k] = static_cast<int32_t>(a[i]);
                s_cpos[k] = static_cast<int32_t>(b[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < kCPer; ++i) {
            const int k = i * kBlock + threadIdx.x;
            if (k < nc) s_ccrd[k] = static_cast<int32_t>(c[i]);
        }
    }
    __syncthreads();

    // Unit and position indices fit in 32 bits (they index arrays whose
    // sizes are int32 pos entries), and so do the staged LDS offsets.
    double acc = 0.0;
    int32_t jv[kUnitIters];  // the lane's coordinates, loaded together
    // (bounds compared in 64 bits: the last range may end past 2^31 - 1)
#pragma unroll
    for (int it = 0; it < kUnitIters; ++it) {
        const int64_t u = u0 + it * kBlock + threadIdx.x;
        jv[it] = u < u1 ? bcrd[u] : 0;
    }
    const int32_t cnt32 = static_cast<int32_t>(cnt);
    const int32_t c0s = static_cast<int32_t>(c0), c1s = static_cast<int32_t>(c1);
    int32_t rk = 0;  // staged parent index of the lane's previous unit (units ascend)
#pragma unroll
    for (int it = 0; it < kUnitIters; ++it) {
        const int64_t u64 = u0 + it * kBlock + threadIdx.x;
        if (u64 >= u1) break;
        const int32_t u = static_cast<int32_t>(u64);
        const int32_t j = jv[it];
        int32_t g;
        if (staged) {
            rk = parent_of<int32_t>([&](int32_t k) { return s_pos[k]; }, rk, cnt32, u);
            // C's positions of this parent, clipped to the staged range
            const int32_t lo = s_cpos[rk] > c0s ? s_cpos[rk] : c0s;
            const int32_t hi = s_cpos[rk + 1] < c1s ? s_cpos[rk + 1] : c1s;
            g = find_sorted<int32_t>([&](int32_t k) { return s_ccrd[k]; }, lo - c0s, hi - c0s, j);
            if (g >= 0) g += c0s;
        } else {
            const int64_t r = parent_of<int64_t>(gpos, r0, r0 + cnt, u);
            g = static_cast<int32_t>(
                find_sorted<int64_t>([&](int64_t k) { return ccrd[k]; }, cpos[r], cpos[r + 1], j));
        }
        if (g < 0) continue;
        acc += to_f64(bv[u]) * to_f64(cv[g]);
    }
    // fixed order: a butterfly in each wave, then the four wave sums in order
    acc = group_sum<kWave>(acc);
    if ((threadIdx.x & (kWave - 1)) == 0) s_sum[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((s_sum[0] + s_sum[1]) + s_sum[2]) + s_sum[3];
}

// ------------------------------------------------------------- CSF operands
constexpr int kFiberBlock = 256;               // lanes per workgroup
constexpr int kEntries = 4;                    // entries of B per lane
constexpr int kFiberTile = kFiberBlock * kEntries;  // entries of B per workgroup
constexpr int kTileParents = kFiberTile / 4;   // parents staged per workgroup
constexpr int kTileC = kFiberTile * 5 / 4;     // C fibers, and C entries, staged
constexpr int kProbe = 8;                     // lanes that search one bound together

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t vi32x4 __attribute__((ext_vector_type(4), aligned(4)));

// First index of [lo, hi) at which `before` does not hold (hi: it holds at
// all; it holds up to some index and at none past it), found by the kProbe
// lanes of an aligned group together: each step leaves an eighth.
template <typename Before>
__device__ __forceinline__ uint32_t split_point(uint32_t lo, uint32_t hi, const Before &before) {
    const uint32_t lane = threadIdx.x & (kProbe - 1);
    const int first = threadIdx.x & (kWave - kProbe);  // the group's first lane of its wave
    while (lo < hi) {
        const uint32_t step = (hi - lo + kProbe - 1) / kProbe;
        const uint32_t at = lo + step * lane + (step - 1);
        const bool b = at < hi && before(at);
        const uint32_t k = __popcll((__ballot(b) >> first) & ((1u << kProbe) - 1));
        lo += step * k;
        if (lo > hi) lo = hi;
        if (lo + (step - 1) < hi) hi = lo + (step - 1);
    }
    return lo;
}

// Bounds of every tile of kFiberTile entries of B: what precedes its first
// entry (the start, side 0) and what its last one reaches (the end, side 1),
// as (parent, fiber, C fiber, C entry): the parent and the fiber that hold
// the entry; the first C fiber of that parent at or past (start) or past
// (end) the fiber's coordinate; and where that fiber or its predecessor
// matches, the first of its entries at or past (past) the entry's
// coordinate, else that C fiber's first entry.  bnd[2 * b] is the start of
// tile b, bnd[2 * b + 1] the end of tile b - 1.
// The chain of dependent loads bounds this pass (four searches, one after
// another): kProbe lanes search together, which makes it a third as long as
// a binary search's (19 us for 20,000 tiles of a 2e7-entry tensor; 16 lanes
// 25).
__global__ __launch_bounds__(kBlock) void k_fiber_bounds(
    uint32_t n, uint32_t units, uint32_t nnzb, uint32_t parts, const int32_t *__restrict__ bpos,
    const int32_t *__restrict__ bcrd, const int32_t *__restrict__ bpos2,
    const int32_t *__restrict__ bcrd2, const int32_t *__restrict__ cpos,
    const int32_t *__restrict__ ccrd, const int32_t *__restrict__ cpos2,
    const int32_t *__restrict__ ccrd2, i32x4 *__restrict__ bnd) {
    const uint32_t t = (blockIdx.x * kBlock + threadIdx.x) / kProbe;
    const uint32_t b = t >> 1;
    const bool end = t & 1;
    if (b > parts || (end ? b == 0 : b == parts)) return;
    const uint32_t past = b * kFiberTile < nnzb ? b * kFiberTile : nnzb;
    const int32_t e = static_cast<int32_t>(end ? past - 1 : past);
    const uint32_t u =
        split_point(1, units, [&](uint32_t x) { return bpos2[x] <= e; }) - 1;
    const int32_t iu = static_cast<int32_t>(u);
    const uint32_t r = split_point(1, n, [&](uint32_t x) { return bpos[x] <= iu; }) - 1;
    const int32_t j = bcrd[u], k = bcrd2[e];
    const uint32_t lo = cpos[r], hi = cpos[r + 1];
    const uint32_t c =
        split_point(lo, hi, [&](uint32_t x) { return end ? ccrd[x] <= j : ccrd[x] < j; });
    uint32_t q;
    const uint32_t f = end ? c - 1 : c;  // the C fiber that may match
    if ((end ? c > lo : c < hi) && ccrd[f] == j)
        q = split_point(cpos2[f], cpos2[f + 1],
                        [&](uint32_t x) { return end ? ccrd2[x] <= k : ccrd2[x] < k; });
    else
        q = cpos2[c];
    if ((threadIdx.x & (kProbe - 1)) == 0) {
        const i32x4 v = {static_cast<int32_t>(r), iu, static_cast<int32_t>(c),
                         static_cast<int32_t>(q)};
        bnd[t] = v;
    }
}

// x[i]: the last index of [x[i], last[i]] whose read is at most key[i] (x[i]
// itself if none is), N searches side by side so that their reads overlap.
template <int N, typename Read>
__device__ __forceinline__ void last_at_most(const Read &read, const int32_t (&key)[N],
                                             int32_t (&x)[N], const int32_t (&last)[N]) {
    int32_t far = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) far = last[i] - x[i] > far ? last[i] - x[i] : far;
    for (int32_t step = far > 0 ? 1 << (31 - __clz(far)) : 0; step > 0; step >>= 1) {
        int32_t y[N], v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            y[i] = last[i] - x[i] > step ? x[i] + step : last[i];
            v[i] = read(y[i]);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = v[i] <= key[i] ? y[i] : x[i];
    }
}

// One workgroup per tile of kFiberTile consecutive entries of B (a fiber may
// lie in several tiles), kEntries consecutive ones per lane.  B's parents of
// the tile, and C's fibers and entries that can match (the tile's bounds are
// clipped at both levels), are staged in LDS.  Then
//  1. a lane per fiber of B finds the C fiber of its coordinate and notes it
//     where the fiber's first entry of the tile stands;
//  2. a running maximum over the tile's notes (they ascend) gives every
//     entry its C fiber;
//  3. every lane finds its entries' coordinates in their C fibers, and reads
//     the values of those that match.
// Everything but the matching values of C (whose lines neighbouring lanes
// share) is read once at consecutive addresses, whatever the lengths of the
// fibers; with a lane walking each pair of fibers in HBM the chain of
// dependent loads bounded the kernel: 273 -> 156 us on 2e7 entries a tensor
// in FP64, most fibers of one to five (0.7 GB, 4.5 TB/s of the 4.8 that a
// large copy reaches), the whole call 1.66 -> 1.37 ms on 1e8 entries and
// 33 -> 0.11 ms with 4,000 fibers of 2,200.  A lane's searches run side by
// side (last_at_most): one after another, with a three-way compare, 166.
// Tiles of 2,048 with 512 lanes or with 8 entries a lane: 179 and 190, though
// the bounds and the final sum then take half.
// What does not fit its stage (more parents than kTileParents; more C fibers
// or entries than kTileC, neither of which is staged then) is searched in
// HBM; a tile of more than 2 * kFiberTile fibers (most of them empty) finds
// each entry's fiber by a search instead of 1 and 2.
template <typename V>
__global__ __launch_bounds__(kFiberBlock) void k_inner_fibers(
    uint32_t nnzb, const int32_t *__restrict__ bpos, const int32_t *__restrict__ bcrd,
    const int32_t *__restrict__ bpos2, const int32_t *__restrict__ bcrd2,
    const V *__restrict__ bv, const int32_t *__restrict__ cpos, const int32_t *__restrict__ ccrd,
    const int32_t *__restrict__ cpos2, const int32_t *__restrict__ ccrd2,
    const V *__restrict__ cv, const i32x4 *__restrict__ bnd, double *__restrict__ part) {
    __shared__ int32_t s_pos[kTileParents + 1];   // B's parent pos entries of the tile
    __shared__ int32_t s_cpos[kTileParents + 1];  // C's
    __shared__ int32_t s_cf[kTileC];              // C's fibers that can match
    __shared__ uint16_t s_cq[kTileC + 1];         // their first entries, from the tile's first
    __shared__ int32_t s_ck[kTileC];              // C's entries that can match
    __shared__ __attribute__((aligned(16))) uint32_t s_note[kFiberTile];
    __shared__ uint32_t s_top[kFiberBlock / kWave];
    __shared__ double s_sum[kFiberBlock / kWave];
    static_assert(kEntries % 4 == 0, "whole vectors of B");
    const uint32_t p0 = blockIdx.x * kFiberTile;
    const int np = static_cast<int>(nnzb - p0 < kFiberTile ? nnzb - p0 : kFiberTile);
    const i32x4 a = bnd[2 * blockIdx.x], z = bnd[2 * blockIdx.x + 3];
    const int32_t r0 = a.x, nr = z.x - a.x + 1, u0 = a.y, nu = z.y - a.y + 1;
    const int32_t c0 = a.z, nc = z.z - a.z, q0 = a.w, nq = z.w - a.w;
    if (nc <= 0 || nq <= 0) {  // no entry of C in the tile's range
        if (threadIdx.x == 0) part[blockIdx.x] = 0.0;
        return;
    }
    const bool sp = nr <= kTileParents, sc = nc <= kTileC && nq <= kTileC;
    const bool by_fiber = nu <= 2 * kFiberTile;

    // the lane's entries of B, four at a time except in a ragged last tile
    const int e0 = threadIdx.x * kEntries;
    int32_t k[kEntries];
    V vb[kEntries];
    if (np == kFiberTile) {
#pragma unroll
        for (int i = 0; i < kEntries; i += 4) {
            const vi32x4 x = *reinterpret_cast<const vi32x4 *>(bcrd2 + p0 + e0 + i);
            k[i] = x.x, k[i + 1] = x.y, k[i + 2] = x.z, k[i + 3] = x.w;
        }
#pragma unroll
        for (int i = 0; i < kEntries; ++i)
            vb[i] = load_stream(bv + p0 + i * kFiberBlock + threadIdx.x);
    } else {
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            const int x = i * kFiberBlock + threadIdx.x;
            k[i] = e0 + i < np ? bcrd2[p0 + e0 + i] : 0;
            vb[i] = x < np ? bv[p0 + x] : V(0);
        }
    }
    if (sp)
        for (int i = threadIdx.x; i <= nr; i += kFiberBlock) {
            s_pos[i] = bpos[r0 + i];
            s_cpos[i] = cpos[r0 + i];
        }
    auto in_range = [&](int32_t q) {  // an entry of C from q0, clipped to the range
        return q < q0 ? 0 : q - q0 < nq ? q - q0 : nq;
    };
    if (sc) {
        // every lane issues all its loads before any store (past the range:
        // 0, with no access)
        constexpr int kPer = (kTileC + kFiberBlock) / kFiberBlock;
        const __amdgpu_buffer_rsrc_t rf = span_rsrc(ccrd + c0, 4u * nc);
        const __amdgpu_buffer_rsrc_t rq = span_rsrc(cpos2 + c0, 4u * (nc + 1));
        const __amdgpu_buffer_rsrc_t rk = span_rsrc(ccrd2 + q0, 4u * nq);
        uint32_t f[kPer], q[kPer], w[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int x = i * kFiberBlock + threadIdx.x;
            f[i] = buf_u32(rf, x < nc ? 4u * x : kBufOut);
            q[i] = buf_u32(rq, x <= nc ? 4u * x : kBufOut);
            w[i] = buf_u32(rk, x < nq ? 4u * x : kBufOut);
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int x = i * kFiberBlock + threadIdx.x;
            if (x < nc) s_cf[x] = static_cast<int32_t>(f[i]);
            if (x <= nc) s_cq[x] = static_cast<uint16_t>(in_range(static_cast<int32_t>(q[i])));
            if (x < nq) s_ck[x] = static_cast<int32_t>(w[i]);
        }
    }
    // Fibers b + i * 256 + lane of the tile: their coordinates, and the
    // tile's first entry of each (-1: it has none in the tile).
    int32_t u[kEntries], j[kEntries], first[kEntries];
    auto load_fibers = [&](int32_t b) {
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            const int32_t x = b + i * kFiberBlock + static_cast<int32_t>(threadIdx.x);
            u[i] = u0 + (x < nu ? x : nu - 1);
            j[i] = bcrd[u[i]];
            const int64_t f = static_cast<int64_t>(bpos2[u[i]]) - p0;
            const int64_t e = static_cast<int64_t>(bpos2[u[i] + 1]) - p0;
            const int32_t at = f > 0 ? static_cast<int32_t>(f) : 0;
            first[i] = x < nu && at < e && at < np ? at : -1;
        }
    };
    if (by_fiber) load_fibers(0);
#pragma unroll
    for (int i = 0; i < kEntries; ++i) s_note[e0 + i] = 0;
    __syncthreads();

    // The notes of fibers u of coordinates j: 2 * g + 1, g the first C fiber
    // of the parent, from c0, at or past j; one more if it matches.
    auto match = [&](const int32_t (&u)[kEntries], const int32_t (&j)[kEntries],
                     uint32_t (&out)[kEntries]) {
        int32_t r[kEntries], x[kEntries], last[kEntries];
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            r[i] = 0;
            last[i] = nr - 1;
        }
        if (sp)
            last_at_most([&](int32_t y) { return s_pos[y]; }, u, r, last);
        else
            last_at_most([&](int32_t y) { return bpos[r0 + y]; }, u, r, last);
        int32_t lo[kEntries];
        bool any[kEntries];  // C fibers of the parent in the range
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            lo[i] = sp ? s_cpos[r[i]] : cpos[r0 + r[i]];
            const int32_t hi = sp ? s_cpos[r[i] + 1] : cpos[r0 + r[i] + 1];
            lo[i] = lo[i] < c0 ? 0 : lo[i] - c0 < nc ? lo[i] - c0 : nc;
            last[i] = (hi < c0 ? 0 : hi - c0 < nc ? hi - c0 : nc) - 1;
            any[i] = last[i] >= lo[i];
            x[i] = any[i] ? lo[i] : 0;
            last[i] = any[i] ? last[i] : 0;
        }
        if (sc)
            last_at_most([&](int32_t y) { return s_cf[y]; }, j, x, last);
        else
            last_at_most([&](int32_t y) { return ccrd[c0 + y]; }, j, x, last);
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            const int32_t v = sc ? s_cf[x[i]] : ccrd[c0 + x[i]];
            const int32_t g = any[i] ? x[i] + (v < j[i] ? 1 : 0) : lo[i];
            out[i] = 2u * static_cast<uint32_t>(g) + 1u + (any[i] && v == j[i] ? 1u : 0u);
        }
    };
    uint32_t note[kEntries];
    if (by_fiber) {
        for (int32_t b = 0; b < nu; b += kFiberTile) {
            if (b > 0) load_fibers(b);
            uint32_t w[kEntries];
            match(u, j, w);
#pragma unroll
            for (int i = 0; i < kEntries; ++i)
                if (first[i] >= 0) s_note[first[i]] = w[i];
        }
        __syncthreads();
        // running maximum: in the lane, over the wave, over the waves
        uint32_t top = 0;
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            note[i] = s_note[e0 + i];
            top = note[i] > top ? note[i] : top;
        }
        const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t o = __shfl_up(top, off);
            top = lane >= off && o > top ? o : top;
        }
        if (lane == kWave - 1) s_top[threadIdx.x / kWave] = top;
        uint32_t run = __shfl_up(top, 1);
        if (lane == 0) run = 0;
        __syncthreads();
        for (int w = 0; w < static_cast<int>(threadIdx.x / kWave); ++w)
            run = s_top[w] > run ? s_top[w] : run;
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            run = note[i] > run ? note[i] : run;
            note[i] = run;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            // the last fiber that starts at or before the entry (past the
            // tile: any)
            const int32_t p = static_cast<int32_t>(p0 + (e0 + i < np ? e0 + i : np - 1));
            u[i] = u0 + parent_of<int32_t>([&](int32_t x) { return bpos2[u0 + x]; }, 0, nu, p);
            j[i] = bcrd[u[i]];
        }
        match(u, j, note);
    }

    // the entries' places in C from q0 (-1: none), handed through LDS to the
    // lanes that read the values, each wave consecutive ones
    int32_t x[kEntries], last[kEntries];
    bool any[kEntries];
#pragma unroll
    for (int i = 0; i < kEntries; ++i) {
        const uint32_t w = note[i] - 1u;
        any[i] = e0 + i < np && (w & 1u);
        const int32_t g = any[i] ? static_cast<int32_t>(w >> 1) : 0;
        x[i] = sc ? s_cq[g] : in_range(cpos2[c0 + g]);
        last[i] = (sc ? s_cq[g + 1] : in_range(cpos2[c0 + g + 1])) - 1;
        any[i] = any[i] && x[i] <= last[i];
        x[i] = any[i] ? x[i] : 0;
        last[i] = any[i] ? last[i] : 0;
    }
    if (sc)
        last_at_most([&](int32_t y) { return s_ck[y]; }, k, x, last);
    else
        last_at_most([&](int32_t y) { return ccrd2[q0 + y]; }, k, x, last);
#pragma unroll
    for (int i = 0; i < kEntries; ++i) {
        const int32_t v = sc ? s_ck[x[i]] : ccrd2[q0 + x[i]];
        s_note[e0 + i] = any[i] && v == k[i] ? static_cast<uint32_t>(x[i]) : ~0u;
    }
    __syncthreads();
    int32_t at[kEntries];
    V vc[kEntries];
#pragma unroll
    for (int i = 0; i < kEntries; ++i)
        at[i] = static_cast<int32_t>(s_note[i * kFiberBlock + threadIdx.x]);
#pragma unroll
    for (int i = 0; i < kEntries; ++i) vc[i] = cv[q0 + (at[i] >= 0 ? at[i] : 0)];
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < kEntries; ++i)
        if (at[i] >= 0) acc += to_f64(vb[i]) * to_f64(vc[i]);
    // fixed order: a butterfly in each wave, then the wave sums in order
    acc = group_sum<kWave>(acc);
    if ((threadIdx.x & (kWave - 1)) == 0) s_sum[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kFiberBlock / kWave; ++w) acc += s_sum[w];
        part[blockIdx.x] = acc;
    }
}

int64_t inner_parts(int order, int64_t nnz) {
    return ceil_div(nnz, order == 2 ? kBlock * kUnitIters : kFiberTile);
}
size_t part_bytes(int64_t parts) { return (static_cast<size_t>(parts) * 8 + 255) / 256 * 256; }

}  // namespace

size_t inner_general_ws(int order, int64_t nnz) {
    // the partials, then 32 bytes of bounds per workgroup boundary
    const int64_t parts = inner_parts(order, nnz > 0 ? nnz : 1);
    return part_bytes(parts) + static_cast<size_t>(parts + 1) * 32;
}

hipError_t launch_inner_general(int vtype, int order, int64_t n, int64_t units,
                                const int32_t *bpos, const int32_t *bcrd, const int32_t *bpos2,
                                const int32_t *bcrd2, const void *bv, const int32_t *cpos,
                                const int32_t *ccrd, const int32_t *cpos2, const int32_t *ccrd2,
                                const void *cv, int64_t nnzb, int64_t nnzc, int64_t cunits,
                                void *ws, double *out, hipStream_t s) {
    // Every entry of the first operand is read, and only the second's lines
    // that can match, so the sparser tensor goes first (products commute
    // exactly) unless the other one's fibers would no longer fit a tile's
    // stage for it: 8e6 entries against half, a quarter, a 64th of them 68,
    // 66, 59 us this way, 64, 52, 30 the other way, but against three
    // quarters of them 70 and 83.
    if (order == 3 && nnzb / 2 >= nnzc && nnzc > 0)
        return launch_inner_general(vtype, order, n, cunits, cpos, ccrd, cpos2, ccrd2, cv, bpos,
                                    bcrd, bpos2, bcrd2, bv, nnzc, nnzb, units, ws, out, s);
    const bool none = nnzb <= 0 || nnzc <= 0;
    const int64_t parts = none ? 0 : inner_parts(order, nnzb);
    double *part = static_cast<double *>(ws);
    char *bounds = static_cast<char *>(ws) + part_bytes(parts);
    if (!none) {
        const dim3 grid(static_cast<unsigned>(parts));
        auto go = [&](auto *b, auto *c) {
            using V = std::remove_const_t<std::remove_pointer_t<decltype(b)>>;
            if (order == 2) {
                int64_t *bnd = reinterpret_cast<int64_t *>(bounds);
                k_inner_bounds<<<dim3(static_cast<unsigned>(ceil_div(parts + 1, kBlock))), kBlock,
                                 0, s>>>(n, nnzb, kBlock * kUnitIters, parts, bpos, bcrd, cpos,
                                         ccrd, bnd);
                k_inner_matrix<V><<<grid, kBlock, 0, s>>>(nnzb, bpos, bcrd, b, cpos, ccrd, c, bnd,
                                                          part);
            } else {
                i32x4 *bnd = reinterpret_cast<i32x4 *>(bounds);
                const int64_t lanes = (parts + 1) * 2 * kProbe;
                k_fiber_bounds<<<dim3(static_cast<unsigned>(ceil_div(lanes, kBlock))), kBlock, 0,
                                 s>>>(static_cast<uint32_t>(n), static_cast<uint32_t>(units),
                                      static_cast<uint32_t>(nnzb), static_cast<uint32_t>(parts),
                                      bpos, bcrd, bpos2, bcrd2, cpos, ccrd, cpos2, ccrd2, bnd);
                k_inner_fibers<V><<<grid, kFiberBlock, 0, s>>>(static_cast<uint32_t>(nnzb), bpos, bcrd,
                                                          bpos2, bcrd2, b, cpos, ccrd, cpos2,
                                                          ccrd2, c, bnd, part);
            }
        };
        if (vtype == SPL_F64)
            go(static_cast<const double *>(bv), static_cast<const double *>(cv));
        else
            go(static_cast<const float *>(bv), static_cast<const float *>(cv));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_inner_final(parts, part, out, s);
}

}  // namespace spl
