// SpAdd3 leaf  A(i,j) = B(i,j) + C(i,j) + D(i,j)  for CSR operands (paper
// Sec. VI-A), fused so no pairwise intermediate is built, with the output
// assembled in two phases (Sec. V-B): a symbolic phase counts the union of
// the three coordinate lists of every row and an exclusive scan turns the
// counts into A.pos; the numeric phase writes A.crd and A.vals at those
// positions with no synchronization between rows.  Row split only: the
// non-zero split does not apply to a sum of CSR operands (Sec. VI-A, CPU
// results).
//
// Values are summed in operand order B, C, D over the operands present (a
// cancellation to zero keeps its coordinate).  Both phases copy the
// workgroup's input coordinates to LDS with coalesced loads, and one lane per
// row merges the three sorted coordinate lists there.  The symbolic phase
// counts the union, leaving sums within workgroups and their totals, which one
// workgroup scans and a last kernel adds.  The numeric phase's default form
// notes which operands hold each coordinate of the union; with that, every
// lane finds its output entries' inputs by counting and reads and writes
// beside its neighbours (k_spadd3_bits).  The merge forms (one lane per row,
// output staged in LDS windows
// so that its stores are coalesced) remain as schedule variants: one lane
// per row reading or storing straight to HBM keeps far more partly used
// lines open than the caches hold, and a window is filled only by the lanes
// whose rows reach into it.
#include "device.hpp"
#include "group_scan.hpp"
#include "internal.hpp"

namespace spl {
namespace {

constexpr int kScanItems = 16;
constexpr int kScanTile = kBlock * kScanItems;

struct Csr3 {
    const int32_t *bp, *bc, *cp, *cc, *dp, *dc;
};

// Where a workgroup reads the three operands' coordinates from: the
// operands themselves, or an LDS copy of the workgroup's ranges (element q
// of operand X at x[q - ox]).
struct Crd3 {
    const int32_t *b, *c, *d;
    int32_t ob, oc, od;
};

// Where a workgroup reads the three operands' values from (as Crd3).
template <typename V>
struct Vals3 {
    const V *b, *c, *d;
    int32_t ob, oc, od;
};

// Three-way merge of one row's sorted coordinate lists, resumable: next()
// yields the union's coordinates in increasing order; with values, the sum
// over the operands present in operand order B, C, D.
struct Merge3 {
    static constexpr int32_t kInf = 0x7fffffff;
    int32_t a, ae, b, be, d, de, xa, xb, xd;

    __device__ __forceinline__ Merge3(const Csr3 &m, const Crd3 &x, int64_t i) {
        a = m.bp[i];
        ae = m.bp[i + 1];
        b = m.cp[i];
        be = m.cp[i + 1];
        d = m.dp[i];
        de = m.dp[i + 1];
        xa = a < ae ? x.b[a - x.ob] : kInf;
        xb = b < be ? x.c[b - x.oc] : kInf;
        xd = d < de ? x.d[d - x.od] : kInf;
    }

    __device__ __forceinline__ bool done() const { return min(xa, min(xb, xd)) == kInf; }

    // Advance past the smallest remaining coordinate c; returns c.  Values
    // of operand X at position q are read at vals.X[q - vals.oX].
    template <bool kValues, typename V>
    __device__ __forceinline__ int32_t next(const Crd3 &x, const Vals3<V> &v, V &sum) {
        const int32_t c = min(xa, min(xb, xd));
        V s = 0;
        if (xa == c) {
            if (kValues) s = v.b[a - v.ob];
            ++a;
            xa = a < ae ? x.b[a - x.ob] : kInf;
        }
        if (xb == c) {
            if (kValues) s = s + v.c[b - v.oc];
            ++b;
            xb = b < be ? x.c[b - x.oc] : kInf;
        }
        if (xd == c) {
            if (kValues) s = s + v.d[d - v.od];
            ++d;
            xd = d < de ? x.d[d - x.od] : kInf;
        }
        sum = s;
        return c;
    }
};

// Copies three runs of n3[X] <= PER * kBlock consecutive coordinates from
// src[X] to dst[X] in LDS.  Every lane issues all its loads before any store
// (past a run: 0, with no access), so the copy costs one memory round trip,
// not one per loop iteration.
template <int PER>
__device__ __forceinline__ void stage3(const int32_t *const *src, const int32_t *n3,
                                       int32_t *const *dst) {
    const int t = threadIdx.x;
    uint32_t v[3][PER];
#pragma unroll
    for (int X = 0; X < 3; ++X) {
        const __amdgpu_buffer_rsrc_t rc = span_rsrc(src[X], 4u * n3[X]);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int k = j * kBlock + t;
            v[X][j] = buf_u32(rc, k < n3[X] ? 4u * k : kBufOut);
        }
    }
#pragma unroll
    for (int X = 0; X < 3; ++X)
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int k = j * kBlock + t;
            if (k < n3[X]) dst[X][k] = static_cast<int32_t>(v[X][j]);
        }
}

// Coordinates of the workgroup's rows [r0, r1) per operand staged in LDS.
// One lane per row reading its row straight from HBM keeps a few lines per
// lane open at once, more than the L1 and L2 hold, so lines are fetched
// several times; the coalesced copy reads each once.  When an operand's run
// exceeds kStageCap the workgroup reads the operands directly.
constexpr int kStageCap = 2560;

// Stages the coordinate runs of rows [r0, r1) when each fits kStageCap and
// returns whether it did (then with the workgroup synchronized); first3
// gets the runs' first positions.
__device__ __forceinline__ bool stage_crd(const Csr3 &m, int64_t r0, int64_t r1,
                                          int32_t (*s_x)[kStageCap], int32_t *first3) {
    first3[0] = m.bp[r0];
    first3[1] = m.cp[r0];
    first3[2] = m.dp[r0];
    const int32_t n3[3] = {m.bp[r1] - first3[0], m.cp[r1] - first3[1], m.dp[r1] - first3[2]};
    if (n3[0] > kStageCap || n3[1] > kStageCap || n3[2] > kStageCap) return false;
    const int32_t *src[3] = {m.bc + first3[0], m.cc + first3[1], m.dc + first3[2]};
    int32_t *dst[3] = {s_x[0], s_x[1], s_x[2]};
    stage3<kStageCap / kBlock>(src, n3, dst);
    __syncthreads();
    return true;
}

// Union size of row i's coordinate lists read through x (HBM).
__device__ __forceinline__ int32_t union_count(const Csr3 &m, const Crd3 &x, int64_t i) {
    Merge3 mg(m, x, i);
    int32_t k = 0;
    float unused;
    const Vals3<float> none{nullptr, nullptr, nullptr, 0, 0, 0};
    while (!mg.done()) {
        mg.next<false, float>(x, none, unused);
        ++k;
    }
    return k;
}

// Numeric phase.  The 256 rows of a workgroup own one contiguous run of the
// output, [apos[r0], apos[r0 + 256]), written in windows of kFillCap
// entries: in each window every lane continues its row's merge from where
// it stopped, emitting into LDS the entries whose output index falls in the
// window, and the workgroup then writes the window with coalesced stores.
// Each row is merged once whatever its length; only one row's lane works
// in the windows a long row fills alone.  The inputs are read directly:
// staging them as well would halve the workgroups per CU, which costs more
// than the repeated line fetches it saves.
constexpr int kFillCap = 2048;

// The workgroup's rows [r0, r1) merged a lane per row into output windows
// of `win` entries in LDS (w_crd, w_val), each window written with coalesced
// stores.
template <typename V, int T = kBlock>
__device__ __forceinline__ void fill_windows(int64_t n, const Csr3 &m, const Crd3 &x,
                                             const Vals3<V> &vv, const int32_t *apos,
                                             int32_t *acrd, V *aval, int64_t r0, int64_t r1,
                                             int win, int32_t *w_crd, V *w_val) {
    const int64_t i = r0 + threadIdx.x;
    const int64_t base = apos[r0];
    const int64_t total = apos[r1] - base;
    const bool mine = i < r1;
    int64_t k = mine ? apos[i] - base : 0;
    const int64_t hi = mine ? apos[i + 1] - base : 0;
    Merge3 mg(m, x, mine ? i : r0);
    for (int64_t w = 0; w < total; w += win) {
        const int64_t we = w + win < total ? w + win : total;
        for (; k < hi && k < we; ++k) {
            V sum;
            const int32_t c = mg.next<true, V>(x, vv, sum);
            w_crd[k - w] = c;
            w_val[k - w] = sum;
        }
        __syncthreads();
        for (int64_t q = threadIdx.x; q < we - w; q += T) {
            store_stream(acrd + base + w + q, w_crd[q]);
            store_stream(aval + base + w + q, w_val[q]);
        }
        __syncthreads();
    }
}

// STAGE 0: inputs read directly; 1: the workgroup's coordinate runs staged
// in LDS (as the count phase does); 2: coordinates and values staged, with a
// smaller output window.  Runs longer than kStageCap fall back to direct
// reads for the whole workgroup.
template <typename V, int STAGE>
__global__ __launch_bounds__(kBlock) void k_spadd3_fill(int64_t n, Csr3 m, const V *bv,
                                                        const V *cv, const V *dv,
                                                        const int32_t *apos, int32_t *acrd,
                                                        V *aval) {
    constexpr int kWin = STAGE == 2 ? 1024 : kFillCap;
    __shared__ int32_t s_crd[kWin];
    __shared__ V s_val[kWin];
    __shared__ int32_t s_x[STAGE ? 3 : 1][STAGE ? kStageCap : 1];
    __shared__ V s_v[STAGE == 2 ? 3 : 1][STAGE == 2 ? kStageCap : 1];
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kBlock;
    const int64_t r1 = r0 + kBlock < n ? r0 + kBlock : n;
    if constexpr (STAGE > 0) {
        // the staged path is a copy of its own, so that it reads LDS directly
        int32_t f[3];
        if (stage_crd(m, r0, r1, s_x, f)) {
            const Crd3 x{s_x[0], s_x[1], s_x[2], f[0], f[1], f[2]};
            if constexpr (STAGE == 2) {
                const int32_t nv[3] = {m.bp[r1] - f[0], m.cp[r1] - f[1], m.dp[r1] - f[2]};
                const V *src[3] = {bv + f[0], cv + f[1], dv + f[2]};
#pragma unroll
                for (int X = 0; X < 3; ++X)
                    for (int k = threadIdx.x; k < nv[X]; k += kBlock) s_v[X][k] = src[X][k];
                __syncthreads();
                fill_windows<V>(n, m, x, Vals3<V>{s_v[0], s_v[1], s_v[2], f[0], f[1], f[2]}, apos,
                                acrd, aval, r0, r1, kWin, s_crd, s_val);
            } else {
                fill_windows<V>(n, m, x, Vals3<V>{bv, cv, dv, 0, 0, 0}, apos, acrd, aval, r0, r1,
                                kWin, s_crd, s_val);
            }
            return;
        }
    }
    fill_windows<V>(n, m, Crd3{m.bc, m.cc, m.dc, 0, 0, 0}, Vals3<V>{bv, cv, dv, 0, 0, 0}, apos,
                    acrd, aval, r0, r1, kWin, s_crd, s_val);
}

// ---- count and default fill: rows staged in dynamic LDS -------------------
//
// A workgroup of T lanes takes T rows and stages the three operands'
// coordinate runs, each with a spare entry behind it, so that a lane walks
// its row's three lists there without branches.  T and the LDS asked for
// follow the operands' mean row lengths (stage_rows); a workgroup whose runs
// do not fit walks them in HBM.

struct Runs {
    int32_t first[3], n[3];
};

__device__ __forceinline__ Runs runs_of(const Csr3 &m, int64_t r0, int64_t r1) {
    Runs R;
    R.first[0] = m.bp[r0];
    R.first[1] = m.cp[r0];
    R.first[2] = m.dp[r0];
    R.n[0] = m.bp[r1] - R.first[0];
    R.n[1] = m.cp[r1] - R.first[1];
    R.n[2] = m.dp[r1] - R.first[2];
    return R;
}
__device__ __forceinline__ int64_t runs_bytes(const Runs &R) {
    return 4 * (static_cast<int64_t>(R.n[0]) + R.n[1] + R.n[2] + 3);
}

// Copies the runs to x[0], x[1], x[2] (kStageDeep entries per lane and operand
// loaded before the first is stored) and synchronizes the workgroup.
constexpr int kStageDeep = 10;

template <int T>
__device__ __forceinline__ void stage_runs(const Csr3 &m, const Runs &R, int32_t *const (&x)[3]) {
    const int32_t *src[3] = {m.bc + R.first[0], m.cc + R.first[1], m.dc + R.first[2]};
    const int most = max(R.n[0], max(R.n[1], R.n[2]));
    for (int k0 = threadIdx.x; k0 - static_cast<int>(threadIdx.x) < most; k0 += kStageDeep * T) {
        uint32_t v[3][kStageDeep];
#pragma unroll
        for (int X = 0; X < 3; ++X) {
            const auto rc = span_rsrc(src[X], 4u * static_cast<uint32_t>(R.n[X]));
#pragma unroll
            for (int j = 0; j < kStageDeep; ++j)
                v[X][j] = buf_u32(rc, 4u * static_cast<uint32_t>(k0 + j * T));
        }
#pragma unroll
        for (int X = 0; X < 3; ++X)
#pragma unroll
            for (int j = 0; j < kStageDeep; ++j)
                if (k0 + j * T < R.n[X]) x[X][k0 + j * T] = static_cast<int32_t>(v[X][j]);
    }
    __syncthreads();
}

// Walks row i's staged lists: calls found(bits) for every coordinate of the
// union in order, bit X set when operand X holds it.
template <typename Found>
__device__ __forceinline__ void walk_staged(const Csr3 &m, const Runs &R, int32_t *const (&x)[3],
                                            int64_t i, Found found) {
    constexpr int32_t kInf = Merge3::kInf;
    int32_t p[3] = {m.bp[i] - R.first[0], m.cp[i] - R.first[1], m.dp[i] - R.first[2]};
    const int32_t e[3] = {m.bp[i + 1] - R.first[0], m.cp[i + 1] - R.first[1],
                          m.dp[i + 1] - R.first[2]};
    auto head = [&](int X) {
        const int32_t v = x[X][p[X]];  // p <= the run's length: at most its spare entry
        return p[X] < e[X] ? v : kInf;
    };
    int32_t h[3] = {head(0), head(1), head(2)};
    for (int32_t c = min(h[0], min(h[1], h[2])); c != kInf; c = min(h[0], min(h[1], h[2]))) {
        uint32_t bits = 0;
#pragma unroll
        for (int X = 0; X < 3; ++X) {
            const uint32_t has = h[X] == c ? 1u : 0u;
            p[X] += static_cast<int32_t>(has);
            bits |= has << X;
        }
#pragma unroll
        for (int X = 0; X < 3; ++X) h[X] = head(X);
        found(bits);
    }
}

// Symbolic phase (35 us on the operands described at k_spadd3_bits, whose
// coordinates are 0.11 GB: bound by the walks' vector-ALU work as much as by
// HBM): apos[i + 1] = entries of the workgroup's output rows up to
// row i, block_sum = all of them in 64 bits (k_block_bases and k_add_bases
// then make positions of them; a total past 32 bits is refused, and the
// positions, wrapped then, are not used).
template <int T>
__global__ __launch_bounds__(T) void k_spadd3_count(int64_t n, Csr3 m, int room, int32_t *apos,
                                                    int64_t *block_sum) {
    extern __shared__ __align__(16) int32_t s_pool[];
    __shared__ int64_t s_wave[T / kWave];
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * T;
    const int64_t r1 = r0 + T < n ? r0 + T : n;
    const int64_t i = r0 + threadIdx.x;
    const Runs R = runs_of(m, r0, r1);
    int32_t k = 0;
    if (runs_bytes(R) <= room) {
        int32_t *const x[3] = {s_pool, s_pool + R.n[0] + 1, s_pool + R.n[0] + R.n[1] + 2};
        stage_runs<T>(m, R, x);
        if (i < n) walk_staged(m, R, x, i, [&](uint32_t) { ++k; });
    } else if (i < n) {
        k = union_count(m, Crd3{m.bc, m.cc, m.dc, 0, 0, 0}, i);
    }
    int64_t all;
    const int64_t upto = group_inclusive<T>(k, s_wave, &all);
    if (i < n) apos[i + 1] = static_cast<int32_t>(upto);
    if (threadIdx.x == 0) block_sum[blockIdx.x] = all;
}

// One workgroup: block_sum[b] becomes the sum of block_sum[0 .. b - 1]; the
// total to *total (pinned host memory).  1,024 lanes, kBasePer consecutive
// blocks each a round.
constexpr int kBaseLanes = 1024, kBasePer = 8;

__global__ __launch_bounds__(kBaseLanes) void k_block_bases(int64_t blocks,
                                                            int64_t *__restrict__ block_sum,
                                                            int64_t *total) {
    __shared__ int64_t s_wave[kBaseLanes / kWave];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < blocks; b0 += kBaseLanes * kBasePer) {
        const int64_t b = b0 + static_cast<int64_t>(threadIdx.x) * kBasePer;
        int64_t v[kBasePer], sum = 0;
#pragma unroll
        for (int j = 0; j < kBasePer; ++j) v[j] = b + j < blocks ? block_sum[b + j] : 0;
#pragma unroll
        for (int j = 0; j < kBasePer; ++j) sum += v[j];
        int64_t inc = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int64_t u = __shfl_up(inc, off);
            inc += lane >= off ? u : 0;
        }
        if (lane == kWave - 1) s_wave[wave] = inc;
        __syncthreads();
        int64_t all = 0, run = carry + inc - sum;
        for (int w = 0; w < kBaseLanes / kWave; ++w) {
            run += w < wave ? s_wave[w] : 0;
            all += s_wave[w];
        }
#pragma unroll
        for (int j = 0; j < kBasePer; ++j) {
            if (b + j < blocks) block_sum[b + j] = run;
            run += v[j];
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// apos[i + 1] += base of row i's block of 2^log2rows rows; apos[0] = 0.
// A workgroup takes 1,024 rows.  OWN: it adds up the block sums before its own
// by itself, which costs less than another launch while they are few, and the
// last workgroup writes the total; else k_block_bases has made bases of them.
constexpr int kAddRows = 4;
constexpr int64_t kOwnBases = 16384;  // blocks up to which it does

template <bool OWN>
__global__ __launch_bounds__(kBlock) void k_add_bases(int64_t n, int log2rows, int64_t blocks,
                                                      const int64_t *__restrict__ block_sum,
                                                      int32_t *__restrict__ apos, int64_t *total) {
    __shared__ int64_t s_sum[kBlock / kWave];
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kBlock * kAddRows;
    int64_t before = 0;  // entries before the workgroup's first block
    if constexpr (OWN) {
        const int64_t fb = first >> log2rows;
#pragma unroll 8
        for (int64_t b = threadIdx.x; b < fb; b += kBlock) before += block_sum[b];
        before = group_sum<kWave>(before);
        if (threadIdx.x % kWave == 0) s_sum[threadIdx.x / kWave] = before;
        __syncthreads();
        before = 0;
#pragma unroll
        for (int w = 0; w < kBlock / kWave; ++w) before += s_sum[w];
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
            int64_t all = before;
            for (int64_t b = fb; b < blocks; ++b) all += block_sum[b];
            *total = all;
        }
    }
#pragma unroll
    for (int j = 0; j < kAddRows; ++j) {
        const int64_t i = first + threadIdx.x + j * kBlock;
        if (i >= n) continue;
        int64_t add = before;
        if constexpr (OWN)
            for (int64_t b = first >> log2rows; b < i >> log2rows; ++b) add += block_sum[b];
        else
            add = block_sum[i >> log2rows];
        apos[i + 1] += static_cast<int32_t>(add);
    }
    if (first + threadIdx.x == 0) apos[0] = 0;
}

// Value at byte offset `off` of a buffer (0 past its range, with no access).
__device__ __forceinline__ float buf_load(const float *, __amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2));
}
__device__ __forceinline__ double buf_load(const double *, __amdgpu_buffer_rsrc_t r,
                                           uint32_t off) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 2);
    return __hiloint2double(static_cast<int>(w[1]), static_cast<int>(w[0]));
}

// Numeric phase (default form): the lane of a row walks its staged lists and
// leaves one byte per output entry, which operands hold it.  The workgroup's
// output entries, like its input entries, are in row and coordinate order, so
// the position of operand X's entry behind output entry k is the number of
// entries before k whose bit X is set: a wave takes 64 consecutive output
// entries, finds those numbers with ballots and a running count, and reads
// coordinates (LDS) and values and writes the output with consecutive lanes
// on consecutive addresses.  Every wave takes one run of these words; a first
// pass counts its bits, so that the others know where theirs start.
//
// Three FP32 operands of 1e6 rows and 8 entries a row (24e6 in, 18.4e6 out; 0.35
// GB, 73 us at the rate of a copy) take 103 us, 138 when every input entry
// looked for its output slot by binary search in the other operands' rows
// (its counts of 64-bit masks and searches kept the vector ALUs busy).  Ten
// words in flight: 131 us with two, 119 with four, 111 with eight, 127 with 16.
constexpr int kFillWords = 10;   // words of 64 entries in flight per wave

template <typename V, int T>
__global__ __launch_bounds__(T) void k_spadd3_bits(int64_t n, Csr3 m, int room, const V *bv,
                                                   const V *cv, const V *dv, const int32_t *apos,
                                                   int32_t *acrd, V *aval) {
    constexpr int kWaves = T / kWave;
    extern __shared__ __align__(16) int32_t s_pool[];
    __shared__ int32_t s_bits[kWaves][3];
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * T;
    const int64_t r1 = r0 + T < n ? r0 + T : n;
    const int64_t i = r0 + threadIdx.x;
    const Runs R = runs_of(m, r0, r1);
    const int32_t out0 = apos[r0];
    const int count = apos[r1] - out0;
    if (runs_bytes(R) + count > room) {
        V *w_val = reinterpret_cast<V *>(s_pool);
        const int win = room / static_cast<int>(4 + sizeof(V));
        fill_windows<V, T>(n, m, Crd3{m.bc, m.cc, m.dc, 0, 0, 0}, Vals3<V>{bv, cv, dv, 0, 0, 0},
                           apos, acrd, aval, r0, r1, win, reinterpret_cast<int32_t *>(w_val + win),
                           w_val);
        return;
    }
    int32_t *const x[3] = {s_pool, s_pool + R.n[0] + 1, s_pool + R.n[0] + R.n[1] + 2};
    uint8_t *s_has = reinterpret_cast<uint8_t *>(x[2] + R.n[2] + 1);
    int q = i < r1 ? apos[i] - out0 : 0;
    stage_runs<T>(m, R, x);
    if (i < r1)
        walk_staged(m, R, x, i, [&](uint32_t bits) { s_has[q++] = static_cast<uint8_t>(bits); });
    __syncthreads();
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int words = (count + 63) >> 6, per = (words + kWaves - 1) / kWaves;
    const int w0 = wave * per, w1 = min(w0 + per, words);
    int32_t at[3] = {0, 0, 0};  // entries of each operand before the wave's next word
    for (int w = w0; w < w1; ++w) {
        const int k = w * 64 + lane;
        const uint32_t has = k < count ? s_has[k] : 0;
#pragma unroll
        for (int X = 0; X < 3; ++X) at[X] += __popcll(__ballot((has >> X) & 1));
    }
    if (lane == 0)
        for (int X = 0; X < 3; ++X) s_bits[wave][X] = at[X];
    __syncthreads();
#pragma unroll
    for (int X = 0; X < 3; ++X) {
        at[X] = 0;
        for (int w = 0; w < wave; ++w) at[X] += s_bits[w][X];
    }
    const V *vals[3] = {bv, cv, dv};
    __amdgpu_buffer_rsrc_t rv[3];
#pragma unroll
    for (int X = 0; X < 3; ++X)
        rv[X] = span_rsrc(vals[X] + R.first[X], static_cast<uint32_t>(sizeof(V)) * R.n[X]);
    const int b1 = R.n[0] + 1, b2 = R.n[0] + R.n[1] + 2;  // where x[1] and x[2] start
    for (int w = w0; w < w1; w += kFillWords) {
        uint32_t has[kFillWords];
        int32_t c[kFillWords];
        V v[kFillWords][3];
#pragma unroll
        for (int u = 0; u < kFillWords; ++u) {
            const int k = (w + u) * 64 + lane;
            has[u] = w + u < w1 && k < count ? s_has[k] : 0;
            int p[3];
#pragma unroll
            for (int X = 0; X < 3; ++X) {
                const bool on = (has[u] >> X) & 1;
                const uint64_t all = __ballot(on);
                // at[X] + set lanes below this one
                p[X] = __builtin_amdgcn_mbcnt_hi(
                    static_cast<uint32_t>(all >> 32),
                    __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(all), at[X]));
                at[X] += __popcll(all);
                v[u][X] = buf_load(vals[X], rv[X], on ? static_cast<uint32_t>(sizeof(V)) * p[X] : kBufOut);
            }
            // (an entry past the end reads a staged coordinate that goes nowhere)
            c[u] = s_pool[has[u] & 1 ? p[0] : has[u] & 2 ? b1 + p[1] : b2 + p[2]];
        }
#pragma unroll
        for (int u = 0; u < kFillWords; ++u) {
            if (!has[u]) continue;
            const int k = (w + u) * 64 + lane;
            // the merge's order: B's value, else 0, then + C's, then + D's
            V s = has[u] & 1 ? v[u][0] : V(0);
            if (has[u] & 2) s = s + v[u][1];
            if (has[u] & 4) s = s + v[u][2];
            store_stream(acrd + out0 + k, c[u]);
            store_stream(aval + out0 + k, s);
        }
    }
}

// Rows per workgroup (128 or 64; 0: not even 64 mean rows fit) and LDS bytes
// for rows of `per_row` bytes on average.  (On the operands above 64 rows take
// 5 us more in count and fill together; at half of kMost a CU still holds
// five workgroups of 128 rows.)  Rows of a power law do not average out over
// a workgroup, so that it gets at least `least` bytes, with which a CU still
// holds as many workgroups as its registers let it (in blocks of 1,280 of its
// 163,840 bytes, less the static part: 16 workgroups of the count, 10 of the
// FP32 fill and 8 of the FP64 one); a workgroup that walks in HBM all the same
// has the wider output windows of it.  Operands of 1e6 rows whose lengths
// are a power law of mean 4 up to 100, FP32: with mean rows' bytes alone 333
// us a call, 625 with the long rows the same in all operands, so 192 and 383;
// Poisson rows of mean 4 112 and 113.
struct StageShape {
    int rows;
    unsigned bytes;
};
constexpr unsigned kCountRoom = 8 * 1280 - 64;
template <typename V>
constexpr unsigned kFillRoom = (sizeof(V) == 8 ? 16 : 12) * 1280 - 64;

StageShape stage_rows(double per_row, unsigned least) {
    constexpr double kSpread = 1.07;  // Poisson runs of 64 and more rows vary less than their mean
    constexpr unsigned kSlack = 512, kMost = 65536;
    for (int rows : {128, 64}) {
        const double need = per_row * rows * kSpread + kSlack;
        if (need > (rows == 128 ? kMost / 2 : kMost)) continue;
        const unsigned b = (static_cast<unsigned>(need) + 255u) & ~255u;
        return {rows, b > least ? b : least};
    }
    return {0, least};
}

// Element i of the scanned sequence: x[i], or with window bounds the window
// length max(end[i] - begin[i], 0).
__device__ __forceinline__ int32_t scan_value(const int32_t *x, const int32_t *begin,
                                              const int32_t *end, int64_t i) {
    if (!begin) return x[i];
    const int32_t len = end[i] - begin[i];
    return len > 0 ? len : 0;
}

// Block sums of the sequence's elements [0, n) in tiles of kScanTile.
__global__ __launch_bounds__(kBlock) void k_scan_tile_sums(int64_t n, const int32_t *x,
                                                           const int32_t *begin,
                                                           const int32_t *end,
                                                           int64_t *tile_sum) {
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
    int64_t acc = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t i = base + j * kBlock + threadIdx.x;
        if (i < n) acc += scan_value(x, begin, end, i);
    }
    __shared__ int64_t s[kBlock];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = s[0];
}

// Exclusive scan of the tile sums by one workgroup; total to *total.
__global__ __launch_bounds__(kBlock) void k_scan_tile_prefix(int64_t ntiles, int64_t *tile_sum,
                                                             int64_t *total) {
    __shared__ int64_t s[kBlock];
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < ntiles; b0 += kBlock) {
        const int64_t i = b0 + threadIdx.x;
        const int64_t v = i < ntiles ? tile_sum[i] : 0;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < kBlock; off <<= 1) {
            const int64_t add = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
            __syncthreads();
            s[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < ntiles) tile_sum[i] = carry + s[threadIdx.x] - v;
        carry += s[kBlock - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// x[i] <- tile prefix + inclusive scan within the tile, i.e. with x =
// counts at apos + 1 this leaves apos[i+1] = sum of counts[0..i] (in place;
// with window bounds the values are the window lengths instead of x).  The
// tile goes through LDS so that the loads and stores are coalesced; each
// thread scans 16 consecutive elements there (padded: element e at
// e + e / 16, so the threads' runs fall in different banks).  `own`: the tile
// sums are as counted, and every workgroup adds up those before its own; the
// last one writes the total.
__global__ __launch_bounds__(kBlock) void k_scan_tile_apply(int64_t n, int32_t *x,
                                                            const int32_t *begin,
                                                            const int32_t *end,
                                                            const int64_t *tile_sum, bool own,
                                                            int64_t *total, int32_t *head) {
    if (head && blockIdx.x == 0 && threadIdx.x == 0) *head = 0;  // the leading 0 of a pos array
    constexpr int kPad = kScanTile + kScanTile / kScanItems;
    __shared__ int64_t s_v[kPad];
    __shared__ int64_t s[kBlock];
    __shared__ int64_t s_first[kBlock / kWave];
    if (own) {
        int64_t before = 0;
        for (int64_t t = threadIdx.x; t < blockIdx.x; t += kBlock) before += tile_sum[t];
        before = group_sum<kWave>(before);
        if (threadIdx.x % kWave == 0) s_first[threadIdx.x / kWave] = before;
    }
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int e = j * kBlock + threadIdx.x;
        const int64_t i = base + e;
        s_v[e + e / kScanItems] = i < n ? scan_value(x, begin, end, i) : 0;
    }
    __syncthreads();
    const int e0 = threadIdx.x * kScanItems;
    const int p0 = e0 + e0 / kScanItems;  // this thread's run, unpadded inside
    int64_t run = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        run += s_v[p0 + j];
        s_v[p0 + j] = run;
    }
    s[threadIdx.x] = run;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        const int64_t add = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t first = own ? 0 : tile_sum[blockIdx.x];
    for (int w = 0; own && w < kBlock / kWave; ++w) first += s_first[w];
    if (own && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = first + s[kBlock - 1];
    const int64_t before = first + s[threadIdx.x] - run;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) s_v[p0 + j] += before;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int e = j * kBlock + threadIdx.x;
        const int64_t i = base + e;
        if (i < n) x[i] = static_cast<int32_t>(s_v[e + e / kScanItems]);
    }
}

}  // namespace

int64_t spadd3_scan_tiles(int64_t n) { return ceil_div(n > 0 ? n : 1, kScanTile); }

// The inclusive scan of n values into out[1..n], out[0] = 0.  Up to kOwnTiles
// tiles the workgroups of the last step add up the sums before theirs by
// themselves (16 loads a lane at most): a launch of one workgroup and its
// gap less (1e6 values: 18 -> 14 us).
constexpr int64_t kOwnTiles = 16 * kBlock;

static hipError_t launch_scan(int64_t n, const int32_t *x, const int32_t *begin,
                              const int32_t *end, int32_t *out, int64_t *tile_sum,
                              int64_t *total, hipStream_t s) {
    const int64_t nt = spadd3_scan_tiles(n);
    const dim3 grid(static_cast<unsigned>(nt));
    const bool own = nt <= kOwnTiles;
    k_scan_tile_sums<<<grid, kBlock, 0, s>>>(n, x, begin, end, tile_sum);
    hipError_t e;
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (!own) {
        k_scan_tile_prefix<<<1, kBlock, 0, s>>>(nt, tile_sum, total);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    k_scan_tile_apply<<<grid, kBlock, 0, s>>>(n, out + 1, begin, end, tile_sum, own, total, out);
    return hipGetLastError();
}

hipError_t launch_window_offsets(int64_t n, const int32_t *begin, const int32_t *end,
                                 int32_t *vpos, int64_t *tile_sum, int64_t *total, hipStream_t s) {
    return launch_scan(n, nullptr, begin, end, vpos, tile_sum, total, s);
}

hipError_t launch_pos_scan(int64_t n, int32_t *apos, int64_t *tile_sum, int64_t *total,
                           hipStream_t s, hipEvent_t counted) {
    // apos[1..n] hold counts: scanned in place
    const hipError_t e = launch_scan(n, apos + 1, nullptr, nullptr, apos, tile_sum, total, s);
    if (e != hipSuccess) return e;
    return counted ? hipEventRecord(counted, s) : hipSuccess;
}

int64_t spadd3_blocks(int64_t n) { return ceil_div(n > 0 ? n : 1, 64); }

hipError_t launch_spadd3_symbolic(int64_t n, int64_t nnz_in, const int32_t *bp, const int32_t *bc,
                                  const int32_t *cp, const int32_t *cc, const int32_t *dp,
                                  const int32_t *dc, int32_t *apos, int64_t *block_sum,
                                  int64_t *total, hipEvent_t counted, hipStream_t s) {
    Csr3 m{bp, bc, cp, cc, dp, dc};
    const StageShape g = stage_rows(n ? 4.0 * static_cast<double>(nnz_in) / static_cast<double>(n) : 0,
                                    kCountRoom);
    const int rows = g.rows ? g.rows : 64;
    const int64_t blocks = ceil_div(n, rows);
    if (n > 0) {
        const dim3 grid(static_cast<unsigned>(blocks));
        const int room = static_cast<int>(g.bytes);
        if (rows == 128)
            k_spadd3_count<128><<<grid, 128, g.bytes, s>>>(n, m, room, apos, block_sum);
        else
            k_spadd3_count<64><<<grid, 64, g.bytes, s>>>(n, m, room, apos, block_sum);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 add_grid(static_cast<unsigned>(ceil_div(n > 0 ? n : 1, kAddRows * kBlock)));
    const int log2rows = rows == 128 ? 7 : 6;
    if (blocks <= kOwnBases) {
        k_add_bases<true><<<add_grid, kBlock, 0, s>>>(n, log2rows, blocks, block_sum, apos, total);
    } else {
        k_block_bases<<<1, kBaseLanes, 0, s>>>(blocks, block_sum, total);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_add_bases<false><<<add_grid, kBlock, 0, s>>>(n, log2rows, blocks, block_sum, apos, total);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return hipEventRecord(counted, s);
}

template <typename V>
hipError_t spadd3_fill(int stage, int64_t n, int64_t nnz_in, const Csr3 &m, const void *bv, const void *cv,
                       const void *dv, const int32_t *apos, int32_t *acrd, void *aval,
                       hipStream_t s) {
    dim3 grid(static_cast<unsigned>(ceil_div(n, kBlock)));
    auto go = [&](auto kern) {
        kern<<<grid, kBlock, 0, s>>>(n, m, static_cast<const V *>(bv), static_cast<const V *>(cv),
                                     static_cast<const V *>(dv), apos, acrd, static_cast<V *>(aval));
        return hipGetLastError();
    };
    if (stage == 3) {
        // coordinates in, and at most as many bytes out
        const StageShape g = stage_rows(5.0 * static_cast<double>(nnz_in) / static_cast<double>(n),
                                        kFillRoom<V>);
        const int room = static_cast<int>(g.bytes);
        auto bits = [&](auto kern, int rows) {
            kern<<<dim3(static_cast<unsigned>(ceil_div(n, rows))), rows, g.bytes, s>>>(
                n, m, room, static_cast<const V *>(bv), static_cast<const V *>(cv),
                static_cast<const V *>(dv), apos, acrd, static_cast<V *>(aval));
            return hipGetLastError();
        };
        if (g.rows == 128) return bits(k_spadd3_bits<V, 128>, 128);
        if (g.rows == 64) return bits(k_spadd3_bits<V, 64>, 64);
    }
    if (stage == 1) return go(k_spadd3_fill<V, 1>);
    if (stage == 2) return go(k_spadd3_fill<V, 2>);
    return go(k_spadd3_fill<V, 0>);
}

hipError_t launch_spadd3_numeric(int vtype, int64_t n, int64_t nnz_in, const int32_t *bp, const int32_t *bc,
                                 const void *bv, const int32_t *cp, const int32_t *cc,
                                 const void *cv, const int32_t *dp, const int32_t *dc,
                                 const void *dv, const int32_t *apos, int32_t *acrd, void *aval,
                                 int stage, hipStream_t s) {
    Csr3 m{bp, bc, cp, cc, dp, dc};
    if (n == 0) return hipSuccess;
    if (vtype == SPL_F64) return spadd3_fill<double>(stage, n, nnz_in, m, bv, cv, dv, apos, acrd, aval, s);
    return spadd3_fill<float>(stage, n, nnz_in, m, bv, cv, dv, apos, acrd, aval, s);
}

}  // namespace spl
