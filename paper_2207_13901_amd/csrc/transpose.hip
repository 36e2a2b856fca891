// Transposition of a (Dense, Compressed) matrix: the CSR arrays of B^T from
// those of B.  The format language stores CSC as (Dense, Compressed) over
// the reversed dimension order (Sec. II-B), so a CSC matrix A is the CSR of
// A^T and this call turns it into A's CSR, on which every CSR leaf runs.
//
// Entries are read in B's order, sorted by (row, column), and stably sorted
// by column with an LSD radix sort: a stable sort by column of a row-major
// sequence is the column-major sequence, i.e. B^T's CSR with rows sorted.
// The column bits are split evenly over passes of at most 8 bits.  An entry
// travels as (column, row, value): the first pass expands the rows from B's
// pos, tile by tile, so that nothing is searched or gathered afterwards, and
// the last pass writes the rows and values straight into B^T's arrays (which
// also serve as one side of the passes' ping-pong).  Each pass cuts the
// sequence into tiles of 4,096 entries; k_radix_counts counts the tile's
// digits (LDS integer counters), k_radix_offsets scans every digit's counts
// over the tiles, and k_radix_scatter ranks every entry among the tile's
// entries of its digit in sequence order, puts the tile in digit order in
// LDS and writes it out, each digit's run to consecutive places.  Integer
// only, no order-dependent atomics: the result is deterministic and
// bit-exact.  k_transpose_pos then writes B^T's pos from the sorted columns.
//
// What bounds it: HBM, but for the first pass.  At 32e6 FP32 entries and 2e6
// columns (three passes of 7 bits) the later scatters take 169 us each, 24 bytes
// an entry at 4.5 TB/s (a plain copy: 4.76), the first 193, 20 bytes an entry at
// 3.3 TB/s: every tile looks up and marks its rows before it can scatter.  The
// counts take 32 us each, the offsets 6 each and pos 31: 0.66 ms a call.  Sorting (column, source
// position) pairs with scatters that stored each round directly, then finding
// every entry's row by a binary search in pos and gathering its value, took
// 4.26 ms (scatters 536 us each, the last step 2,441).
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace spl {
namespace {

constexpr int kRadixBits = 8;
constexpr int kDigits = 1 << kRadixBits;
constexpr int kRounds = 16;
constexpr int kRadixTile = kBlock * kRounds;  // 4,096 entries per tile
constexpr int kWaves = kBlock / kWave;
constexpr int kWaveTile = kRadixTile / kWaves;  // consecutive entries of one wave
static_assert(kBlock == kDigits, "a thread per digit");
// Up to this many tiles a scatter workgroup adds up the tiles' counts by
// itself; beyond, k_radix_offsets has done so (two passes over 32 tiles: 41.3 ->
// 37.0 us a call, over 62 tiles 44.4 -> 42.4, over 125 tiles 46.7 and 51.0).
constexpr int64_t kOwnOffsets = 64;

__device__ __forceinline__ int digit_of(int32_t key, int shift, int bits) {
    return static_cast<int>((static_cast<uint32_t>(key) >> shift) & ((1u << bits) - 1u));
}

// The tile a workgroup takes.  Workgroups go to the eight XCDs in turn, and
// neighbouring tiles' runs of a digit are neighbours in the output: every
// XCD takes one contiguous eighth of the tiles, so that the lines that two
// tiles share are completed in one L2.
__device__ __forceinline__ int64_t tile_of_block(int64_t ntiles) {
    const int64_t per = (ntiles + 7) / 8;
    return static_cast<int64_t>(blockIdx.x & 7) * per + (blockIdx.x >> 3);
}
unsigned tile_grid(int64_t ntiles) { return static_cast<unsigned>((ntiles + 7) / 8 * 8); }

// Number of entries of tile t with digit d, to counts[d * ntiles + t], where
// k_radix_offsets scans a digit's tiles, or (own) counts[t * kDigits + d],
// where a scatter workgroup's threads, one a digit, add up the tiles.
__global__ __launch_bounds__(kBlock) void k_radix_counts(int64_t n, const int32_t *__restrict__ keys,
                                                         int shift, int bits, int64_t ntiles,
                                                         bool own, int32_t *__restrict__ counts) {
    __shared__ int32_t s_cnt[kWaves][kDigits];
    const int tid = threadIdx.x, wave = tid / kWave;
    const int64_t tile = tile_of_block(ntiles);
    if (tile >= ntiles) return;
    const int64_t base = tile * kRadixTile;
    const int cnt = static_cast<int>(n - base < kRadixTile ? n - base : kRadixTile);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s_cnt[w][tid] = 0;
    // every load before the first count; past the end: 0, not counted
    const auto rk = span_rsrc(keys + base, 4u * static_cast<uint32_t>(cnt));
    int32_t k[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        k[r] = static_cast<int32_t>(buf_u32<0>(rk, 4u * static_cast<uint32_t>(r * kBlock + tid)));
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (r * kBlock + tid < cnt) atomicAdd(&s_cnt[wave][digit_of(k[r], shift, bits)], 1);
    __syncthreads();
    if (tid < 1 << bits) {
        int32_t c = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) c += s_cnt[w][tid];
        counts[own ? tile * kDigits + tid : static_cast<int64_t>(tid) * ntiles + tile] = c;
    }
}

// Exclusive sum of `v` over the workgroup's threads before this one.
__device__ __forceinline__ int32_t block_before(int32_t v, int32_t *s_tot) {
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int32_t inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t u = __shfl_up(inc, off);
        inc += lane >= off ? u : 0;
    }
    if (lane == kWave - 1) s_tot[wave] = inc;
    __syncthreads();
    int32_t before = inc - v;
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w) before += w < wave ? s_tot[w] : 0;
    __syncthreads();
    return before;
}

// Digit blockIdx.x: its counts over the tiles become exclusive sums in place,
// its total goes to totals.  The barriers and the loads' latency are what a
// step of 256 * kPer tiles costs: 7,813 tiles take 6.4 us, with 8 a lane 11.7,
// with 32 7.8.
__global__ __launch_bounds__(kBlock) void k_radix_offsets(int64_t ntiles, int32_t *__restrict__ counts,
                                                          int32_t *__restrict__ totals) {
    constexpr int kPer = 16;
    typedef int32_t vi32x4 __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ int32_t s_tot[kWaves], s_all;
    int32_t *c = counts + static_cast<int64_t>(blockIdx.x) * ntiles;
    int32_t carry = 0;
    for (int64_t t0 = 0; t0 < ntiles; t0 += kBlock * kPer) {
        const int64_t first = t0 + static_cast<int64_t>(threadIdx.x) * kPer;
        int32_t v[kPer], sum = 0;
        const bool whole = first + kPer <= ntiles;
        if (whole) {
#pragma unroll
            for (int j = 0; j < kPer; j += 4) {
                const vi32x4 x = *reinterpret_cast<const vi32x4 *>(c + first + j);
                v[j] = x.x, v[j + 1] = x.y, v[j + 2] = x.z, v[j + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) v[j] = first + j < ntiles ? c[first + j] : 0;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) sum += v[j];
        const int32_t before = block_before(sum, s_tot);
        if (threadIdx.x == kBlock - 1) s_all = before + sum;
        int32_t run = carry + before;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int32_t here = v[j];
            v[j] = run;
            run += here;
        }
        if (whole) {
#pragma unroll
            for (int j = 0; j < kPer; j += 4) {
                const vi32x4 x = {v[j], v[j + 1], v[j + 2], v[j + 3]};
                *reinterpret_cast<vi32x4 *>(c + first + j) = x;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (first + j < ntiles) c[first + j] = v[j];
        }
        __syncthreads();
        carry += s_all;
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Rows that a tile's entries span up to which the first pass marks every row's
// start; in a tile of more rows (nearly all of them empty) every entry finds
// its row by a search.  Marking takes one workgroup a step per 256 rows,
// whatever the entries; a search log2(rows) steps of 16 loads a lane (4e5
// entries in 4 / 8 / 64 / 256 times as many rows: marked 81 / 93 / 370 / 1,877
// us a call, searched 80 / 82 / 109 / 131; 4,000 entries in 8e6 rows 9,099
// and 157).
constexpr int64_t kMarkRows = 4 * kRadixTile;

// The row holding position p: the last i in [0, n) with pos[i] <= p, found by
// one wave 64 probes at a time.
__device__ __forceinline__ int64_t wave_row_of(const int32_t *__restrict__ pos, int64_t n, int64_t p) {
    const int lane = threadIdx.x % kWave;
    int64_t lo = 0, hi = n;  // pos[lo] <= p, and pos[hi] > p or hi == n
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t at = lo + (lane + 1) * step;
        const bool le = at < hi && pos[at] <= p;
        const int k = __popcll(__ballot(le));  // pos is non-decreasing: the first k lanes
        hi = lo + (k + 1) * step < hi ? lo + (k + 1) * step : hi;
        lo += k * step;
    }
    return lo;
}

__device__ __forceinline__ int32_t wave_inclusive_max(int32_t v) {
    auto step = [&](auto ctl, auto rows) {
        const int32_t u = __builtin_amdgcn_update_dpp(0, v, decltype(ctl)::value,
                                                      decltype(rows)::value, 0xf, false);
        v = u > v ? u : v;
    };
    step(std::integral_constant<int, 0x111>(), std::integral_constant<int, 0xf>());
    step(std::integral_constant<int, 0x112>(), std::integral_constant<int, 0xf>());
    step(std::integral_constant<int, 0x114>(), std::integral_constant<int, 0xf>());
    step(std::integral_constant<int, 0x118>(), std::integral_constant<int, 0xf>());
    step(std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xa>());
    step(std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xc>());
    return v;
}

template <typename V>
__device__ __forceinline__ V buf_elem(__amdgpu_buffer_rsrc_t r, uint32_t k) {
    if constexpr (sizeof(V) == 8) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, 8u * k, 0, 0);
        return (static_cast<uint64_t>(w[1]) << 32) | w[0];
    } else if constexpr (sizeof(V) == 4) {
        return __builtin_amdgcn_raw_buffer_load_b32(r, 4u * k, 0, 0);
    } else {
        return static_cast<V>(__builtin_amdgcn_raw_buffer_load_b16(r, 2u * k, 0, 0));
    }
}

// Stable scatter of one pass over the digit at `shift`.  Wave w of a tile
// takes its entries [w * 1024, (w + 1) * 1024) in 16 rounds of 64: the lanes
// of a round that hold one digit are found with a ballot per digit bit, and
// the wave's running count of the digit (s_cnt) gives each its rank.  With
// the waves' counts scanned, every entry knows its place in the tile sorted
// by digit; columns, rows and values go through one LDS buffer in turn into
// that order and from there to HBM, where a digit's entries are consecutive
// (32 of them on average at 7 bits: whole lines but for the ends, where
// storing each round directly touched about one line per entry).  V is an
// unsigned integer of the value's size.  FIRST: the rows come from B's pos.
template <typename V, bool FIRST>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    int64_t n, const int32_t *__restrict__ keys_in, const int32_t *__restrict__ rows_in,
    const V *__restrict__ vals_in, int64_t nrows, const int32_t *__restrict__ pos, int shift,
    int bits, int64_t ntiles, bool own, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ totals, int32_t *__restrict__ keys_out,
    int32_t *__restrict__ rows_out, V *__restrict__ vals_out) {
    constexpr size_t kElem = sizeof(V) > 4 ? sizeof(V) : 4;
    __shared__ __align__(16) char s_raw[kRadixTile * kElem];
    __shared__ int32_t s_cnt[kWaves][kDigits];  // running counts, then places in the sorted tile
    __shared__ int32_t s_goff[kDigits];         // output place of sorted entry i: s_goff[d] + i
    __shared__ int32_t s_tot[kWaves];
    __shared__ int64_t s_rows[2];
    int32_t *s_i32 = reinterpret_cast<int32_t *>(s_raw);
    V *s_val = reinterpret_cast<V *>(s_raw);
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int64_t tile = tile_of_block(ntiles);
    if (tile >= ntiles) return;
    const int64_t base = tile * kRadixTile;
    const int cnt = static_cast<int>(n - base < kRadixTile ? n - base : kRadixTile);
    const int e0 = wave * kWaveTile + lane;  // this lane's entry of round 0

    const auto rk = span_rsrc(keys_in + base, 4u * static_cast<uint32_t>(cnt));
    int32_t key[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        key[r] = static_cast<int32_t>(buf_u32<0>(rk, 4u * static_cast<uint32_t>(e0 + r * kWave)));

    // The rows: row starts marked at their first entry (the last of several
    // rows starting there wins, the others being empty), then a running
    // maximum over the entries.
    int32_t row[kRounds];
    if constexpr (FIRST) {
        if (wave < 2) {
            const int64_t r = wave_row_of(pos, nrows, wave == 0 ? base : base + cnt - 1);
            if (lane == 0) s_rows[wave] = r;
        }
#pragma unroll
        for (int r = 0; r < kRounds; ++r) s_i32[r * kBlock + tid] = 0;
        __syncthreads();
        const int64_t r0 = s_rows[0], r1 = s_rows[1];
        if (r1 - r0 <= kMarkRows) {
            for (int64_t q = r0 + 1 + tid; q <= r1; q += kBlock)
                atomicMax(&s_i32[pos[q] - base], static_cast<int32_t>(q - r0));
            __syncthreads();
            int32_t top = 0;
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                row[r] = s_i32[e0 + r * kWave];
                top = row[r] > top ? row[r] : top;
            }
            top = wave_inclusive_max(top);
            if (lane == kWave - 1) s_tot[wave] = top;
            __syncthreads();
            int32_t run = 0;
#pragma unroll
            for (int w = 0; w < kWaves - 1; ++w) run = w < wave && s_tot[w] > run ? s_tot[w] : run;
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int32_t m = wave_inclusive_max(row[r]);
                row[r] = static_cast<int32_t>(r0) + (m > run ? m : run);
                const int32_t last = __builtin_amdgcn_readlane(m, kWave - 1);
                run = last > run ? last : run;
            }
        } else {
            const uint32_t span = static_cast<uint32_t>(r1 - r0);
            const int32_t *first = pos + r0;
            uint32_t at[kRounds];  // the last row found to start at or before the entry, from r0
#pragma unroll
            for (int r = 0; r < kRounds; ++r) at[r] = 0;
            for (uint32_t step = 1u << (31 - __clz(span)); step > 0; step >>= 1) {
                int32_t v[kRounds];
#pragma unroll
                for (int r = 0; r < kRounds; ++r)
                    v[r] = first[step <= span - at[r] ? at[r] + step : span];
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    const int64_t p = base + (e0 + r * kWave < cnt ? e0 + r * kWave : cnt - 1);
                    at[r] += step <= span - at[r] && v[r] <= p ? step : 0;
                }
            }
#pragma unroll
            for (int r = 0; r < kRounds; ++r) row[r] = static_cast<int32_t>(r0 + at[r]);
        }
    } else {
        const auto rr = span_rsrc(rows_in + base, 4u * static_cast<uint32_t>(cnt));
#pragma unroll
        for (int r = 0; r < kRounds; ++r)
            row[r] = static_cast<int32_t>(buf_u32<0>(rr, 4u * static_cast<uint32_t>(e0 + r * kWave)));
    }

#pragma unroll
    for (int w = 0; w < kWaves; ++w) s_cnt[w][tid] = 0;
    __syncthreads();
    const uint64_t lt = (1ull << lane) - 1;  // lanes below this one
    int32_t place[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int d = digit_of(key[r], shift, bits);
        const bool valid = e0 + r * kWave < cnt;
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool one = (d >> b) & 1;
            const uint64_t ones = __ballot(one);
            same &= one ? ones : ~ones;
        }
        const int before = __popcll(same & lt);
        // (one wave's LDS accesses execute in order: the round's reads, then
        // one write per digit by its first lane)
        const int32_t old = s_cnt[wave][d];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid && before == 0) s_cnt[wave][d] = old + __popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        place[r] = old + before;
    }
    __syncthreads();
    {
        int32_t c[kWaves], sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            c[w] = s_cnt[w][tid];
            sum += c[w];
        }
        int32_t start = block_before(sum, s_tot);
        const int32_t first = start;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            s_cnt[w][tid] = start;
            start += c[w];
        }
        // output entries before this digit's run of this tile
        int32_t total = 0, prior = 0;
        if (tid < 1 << bits) {
            if (ntiles == 1) {
                total = sum;
            } else if (own) {
                for (int64_t t0 = 0; t0 < ntiles; t0 += 16) {
                    int32_t v[16];
#pragma unroll
                    for (int k = 0; k < 16; ++k) v[k] = t0 + k < ntiles ? offsets[(t0 + k) * kDigits + tid] : 0;
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        prior += t0 + k < tile ? v[k] : 0;
                        total += v[k];
                    }
                }
            } else {
                prior = offsets[tid * ntiles + tile];
                total = totals[tid];
            }
        }
        s_goff[tid] = block_before(total, s_tot) + prior - first;
    }
    __syncthreads();
    // the values in flight while the columns go through LDS
    const auto rv = span_rsrc(vals_in + base, static_cast<uint32_t>(sizeof(V)) * static_cast<uint32_t>(cnt));
    V val[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        val[r] = buf_elem<V>(rv, static_cast<uint32_t>(e0 + r * kWave));
        place[r] += s_cnt[wave][digit_of(key[r], shift, bits)];
        if (e0 + r * kWave < cnt) s_i32[place[r]] = key[r];
    }
    __syncthreads();
    int32_t dst[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int i = r * kBlock + tid;
        const int32_t k = s_i32[i];
        dst[r] = i < cnt ? s_goff[digit_of(k, shift, bits)] + i : 0;
        if (i < cnt) keys_out[dst[r]] = k;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (e0 + r * kWave < cnt) s_i32[place[r]] = row[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (r * kBlock + tid < cnt) rows_out[dst[r]] = s_i32[r * kBlock + tid];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (e0 + r * kWave < cnt) s_val[place[r]] = val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (r * kBlock + tid < cnt) vals_out[dst[r]] = s_val[r * kBlock + tid];
}

// B^T's pos from the sorted columns: pos[c] is the first output position of
// column c (columns without entries repeat the next one's).  A lane takes
// four consecutive positions with one 16-byte load (keys is 256-byte
// aligned workspace; a lane per position took 80 us at 32e6 entries); a gap
// of more than a wave's columns between two entries is written by the whole
// wave.
__global__ __launch_bounds__(kBlock) void k_transpose_pos(int64_t m, int64_t nnz,
                                                          const int32_t *__restrict__ keys,
                                                          int32_t *__restrict__ tpos) {
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    const int64_t q0 = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    const int lane = threadIdx.x % kWave;
    // position q (the end of the sequence at q == nnz) starts the columns
    // after its predecessor's up to its own, h[j + 1] for q = q0 + j
    int32_t h[5];
    h[0] = q0 > 0 && q0 <= nnz ? keys[q0 - 1] : -1;
    if (q0 + 4 <= nnz) {
        const i32x4 k = *reinterpret_cast<const i32x4 *>(keys + q0);
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j + 1] = k[j];
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t q = q0 + j;
            h[j + 1] = q < nnz ? keys[q] : q == nnz ? static_cast<int32_t>(m) : h[j];
        }
    }
    bool any = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool wide = h[j + 1] - h[j] > kWave;  // (-1 is followed by a key below m)
        any |= wide;
        if (!wide)
            for (int64_t c = static_cast<int64_t>(h[j]) + 1; c <= h[j + 1]; ++c)
                tpos[c] = static_cast<int32_t>(q0 + j);
    }
    for (uint64_t todo = __ballot(any); todo; todo &= todo - 1) {
        const int src = __ffsll(static_cast<unsigned long long>(todo)) - 1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t lo = __shfl(h[j], src), hi = __shfl(h[j + 1], src);
            const int32_t at = static_cast<int32_t>(__shfl(q0, src)) + j;
            if (hi - lo > kWave)
                for (int64_t c = static_cast<int64_t>(lo) + 1 + lane; c <= hi; c += kWave) tpos[c] = at;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_fill_zero(int64_t count, int32_t *__restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i < count) out[i] = 0;
}

size_t up256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }
size_t value_bytes(int vtype) { return vtype == SPL_F64 ? 8 : vtype == SPL_F32 ? 4 : 2; }

template <typename V>
hipError_t transpose_typed(int64_t n, int64_t m, int64_t nnz, const int32_t *pos,
                           const int32_t *crd, const V *vals, int32_t *tpos, int32_t *tcrd,
                           V *tvals, char *w, hipStream_t s) {
    const int64_t tiles = ceil_div(nnz, kRadixTile);
    auto take = [&](size_t bytes) {
        char *p = w;
        w += up256(bytes);
        return p;
    };
    int32_t *keys[2] = {reinterpret_cast<int32_t *>(take(static_cast<size_t>(nnz) * 4)),
                        reinterpret_cast<int32_t *>(take(static_cast<size_t>(nnz) * 4))};
    int32_t *rows = reinterpret_cast<int32_t *>(take(static_cast<size_t>(nnz) * 4));
    V *wvals = reinterpret_cast<V *>(take(static_cast<size_t>(nnz) * sizeof(V)));
    int32_t *counts = reinterpret_cast<int32_t *>(take(static_cast<size_t>(tiles) * kDigits * 4));
    int32_t *totals = reinterpret_cast<int32_t *>(take(kDigits * 4));

    const int total_bits = transpose_bits(m), passes = transpose_passes(m);
    const int bits = (total_bits + passes - 1) / passes;
    const bool own = tiles <= kOwnOffsets;
    const dim3 grid(tile_grid(tiles));
    const int32_t *kin = crd, *rin = nullptr;
    const V *vin = vals;
    hipError_t e;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pass * bits;
        // the last pass writes B^T's arrays, the one before it the workspace, and so on
        const bool out = (passes - 1 - pass) % 2 == 0;
        int32_t *ko = keys[pass & 1], *ro = out ? tcrd : rows;
        V *vo = out ? tvals : wvals;
        if (tiles > 1) {
            k_radix_counts<<<grid, kBlock, 0, s>>>(nnz, kin, shift, bits, tiles, own, counts);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (!own) {
            k_radix_offsets<<<dim3(1u << bits), kBlock, 0, s>>>(tiles, counts, totals);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (pass == 0)
            k_radix_scatter<V, true><<<grid, kBlock, 0, s>>>(nnz, kin, rin, vin, n, pos, shift, bits,
                                                            tiles, own, counts, totals, ko, ro, vo);
        else
            k_radix_scatter<V, false><<<grid, kBlock, 0, s>>>(nnz, kin, rin, vin, n, pos, shift, bits,
                                                             tiles, own, counts, totals, ko, ro, vo);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        kin = ko;
        rin = ro;
        vin = vo;
    }
    k_transpose_pos<<<dim3(static_cast<unsigned>(ceil_div(nnz + 1, 4 * kBlock))), kBlock, 0, s>>>(
        m, nnz, kin, tpos);
    return hipGetLastError();
}

}  // namespace

int transpose_bits(int64_t m) {
    int bits = 0;
    while (bits < 31 && (static_cast<int64_t>(1) << bits) < m) ++bits;
    return bits ? bits : 1;
}

int transpose_passes(int64_t m) { return (transpose_bits(m) + kRadixBits - 1) / kRadixBits; }

size_t transpose_ws_bytes(int vtype, int64_t nnz) {
    if (nnz == 0) return 0;
    const size_t z = static_cast<size_t>(nnz);
    const size_t cells = static_cast<size_t>(ceil_div(nnz, kRadixTile)) * kDigits;
    return 3 * up256(z * 4) + up256(z * value_bytes(vtype)) + up256(cells * 4) + up256(kDigits * 4);
}

hipError_t launch_transpose(int vtype, int64_t n, int64_t m, int64_t nnz, const int32_t *pos,
                            const int32_t *crd, const void *vals, int32_t *tpos, int32_t *tcrd,
                            void *tvals, void *ws, hipStream_t s) {
    if (nnz == 0) {
        k_fill_zero<<<dim3(static_cast<unsigned>(ceil_div(m + 1, kBlock))), kBlock, 0, s>>>(m + 1,
                                                                                          tpos);
        return hipGetLastError();
    }
    auto go = [&](auto bits_type) {
        using V = decltype(bits_type);  // the value's bits
        return transpose_typed<V>(n, m, nnz, pos, crd, static_cast<const V *>(vals), tpos, tcrd,
                                  static_cast<V *>(tvals), static_cast<char *>(ws), s);
    };
    if (vtype == SPL_F64) return go(uint64_t{});
    if (vtype == SPL_F32) return go(uint32_t{});
    return go(uint16_t{});
}

}  // namespace spl
