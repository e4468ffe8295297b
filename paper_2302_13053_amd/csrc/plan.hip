// Per-graph plan: degrees, GCN normalisers and the degree-ordered row schedule.
//
// deg[v] is the CSR row length.  dinv[v] = 1/sqrt(deg v) is what the
// symmetric normalisation D^-1/2 (A+I) D^-1/2 multiplies with on both sides; it
// is computed as a correctly rounded fp32 sqrt followed by a correctly rounded
// fp32 divide (never the hardware rsqrt approximation) so that it can be
// compared bit for bit with a CPU computation.
//
// Power-law graphs have a few very long rows.  The aggregation kernels give
// one wavefront to an ordinary row and a whole workgroup to a long one, and
// start the long rows first, so the plan keeps the row ids sorted by
// decreasing degree (stable: equal degrees stay in id order) and the number of
// rows at or above a few degree thresholds.
#include <cstring>
#include <new>

#include "common.hpp"
#include "report.hpp"

namespace {

constexpr int kThreads = 256;

// What the host reads back: written by one kernel, to a HostReport or to device memory.
struct Readback {
    int64_t counts[kPlanThresholdCount + 1];      // rows of at least kPlanThresholds[i] entries ... and the largest degree
    uint32_t bad;
    uint32_t pad;
};

// ---------------------------------------------------------------------------
// The schedule order: a stable counting sort of the degrees, largest first (equal degrees stay in id order), one
// digit of the degree at a time, lowest digit first.
//
// Bound by launches and latencies, not bytes (12 bytes per row): a general 32-bit radix sort took 3 to 19 dependent
// launches here, where a power-law graph's degrees have 15 significant bits and a citation graph's 8.  Stability
// inside a workgroup without a sort: every wave owns a consecutive piece of the rows and counters of its own, a row's
// rank among the 64 that the wave looks at is the number of lower lanes with the same digit (one ballot per bit),
// and the pieces' counters are made offsets in the order of the pieces.
// ---------------------------------------------------------------------------
constexpr int kOrderThreads = 1024;
constexpr int kOrderWaves = kOrderThreads / 64;

// lanes (of those with `have`) whose digit equals this lane's
template <int BITS>
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool have)
{
    uint64_t m = __ballot(have);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint64_t set = __ballot(have && ((d >> b) & 1u));
        m &= ((d >> b) & 1u) ? set : ~set;
    }
    return m;
}

// The lane's position behind counters[d] in the order of the lanes; the counter moves past all of them.  Called by whole
// waves, with counters of the wave's own; a wave's LDS operations keep their order, the fences hold the compiler to it.
template <int BITS, typename C>
__device__ __forceinline__ uint32_t take_position(C* counters, uint32_t d, bool have)
{
    const uint64_t m = same_digit<BITS>(d, have);
    const int lane = threadIdx.x & 63;
    const uint32_t below = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    uint32_t at = 0;
    if (have) at = counters[d];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (have && below == 0) counters[d] = (C)(at + (uint32_t)__popcll(m));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return at + below;
}

// inclusive prefix sum over the workgroup of kOrderThreads; sc: kOrderWaves words, free again on return
__device__ __forceinline__ uint32_t order_scan(uint32_t v, uint32_t* sc)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    if (lane == 63) sc[wave] = v;
    __syncthreads();
    for (int w = 0; w < wave; ++w) v += sc[w];
    __syncthreads();
    return v;
}

// degree of row v; what cannot be one counts as bad and as zero
__device__ __forceinline__ int32_t row_degree(int64_t v, int64_t N, int64_t nnz, const int64_t* __restrict__ row_ptr, bool& bad)
{
    const int64_t lo = row_ptr[v], hi = row_ptr[v + 1], d = hi - lo;
    if (d < 0 || d > 0x7fffffff || (v == 0 && lo != 0) || (v == N - 1 && hi != nnz)) {
        bad = true;
        return 0;
    }
    return (int32_t)d;
}

struct Thresholds { int t[kPlanThresholdCount]; };

// A workgroup's rows: counts at the thresholds, largest degree, and whether one was bad.
struct RowStats {
    uint32_t at_least[kPlanThresholdCount];
    uint32_t largest, bad;
    uint32_t top;                        // rows of kTopDegree entries and more (larger graphs only)
};
__device__ __forceinline__ void add_row(RowStats& st, int32_t d, const Thresholds& th)
{
#pragma unroll
    for (int i = 0; i < kPlanThresholdCount; ++i) st.at_least[i] += d >= th.t[i] ? 1u : 0u;
    st.largest = max(st.largest, (uint32_t)d);
}
// the threads' sums into `all` (LDS, zeroed before the last barrier); a barrier follows
__device__ __forceinline__ void gather_stats(const RowStats& st, RowStats* all)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < kPlanThresholdCount; ++i) {
        uint32_t c = st.at_least[i];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m, 64);
        if (lane == 0 && c) atomicAdd(&all->at_least[i], c);
    }
    uint32_t top = st.largest;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) top = max(top, __shfl_xor(top, m, 64));
    if (lane == 0) atomicMax(&all->largest, top);
    if (st.bad) atomicOr(&all->bad, 1u);
    if (st.top) atomicAdd(&all->top, st.top);
    __syncthreads();
}

// Small graphs, N <= kSmallRows: degrees, normalisers, order and counts in one launch by one workgroup, degrees and
// ids in LDS (40 KB), 8 bits of the degree per pass and no more passes than the largest degree has.  2,708 rows: 6 launches and
// 30 us of a plan's 85 before.  The line: whole plans this way and by the kernels for larger graphs in us, 5,000 rows of up to
// 200 entries 36.2 and 38.1, up to 1,000 44.5 and 38.0; 8,192 rows 41.5 and 40.6, 53.9 and 40.6; 16,384 55.8 and 40.8, 79.1 and
// 41.0 (4,096 here: 34.0 and 41.1).
constexpr int kSmallRows = 4096;
constexpr int kSmallSteps = kSmallRows / kOrderThreads;
struct SmallShared {
    uint32_t deg[kSmallRows];
    uint16_t ids[2][kSmallRows];
    uint16_t counters[kOrderWaves][256];         // (positions stay below 2^16)
    uint32_t sc[kOrderWaves];
    RowStats all;
};
__global__ __launch_bounds__(kOrderThreads) void small_order_kernel(
    int N, int64_t nnz, const int64_t* __restrict__ row_ptr, int32_t* __restrict__ deg, float* __restrict__ dinv,
    int32_t* __restrict__ order, Thresholds th, Readback* rb)
{
    __shared__ SmallShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < (int)(sizeof(RowStats) / 4)) reinterpret_cast<uint32_t*>(&sh.all)[tid] = 0u;
    __syncthreads();
    RowStats st = {};
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kSmallSteps; ++j) {
        const int v = j * kOrderThreads + tid;
        if (v < N) {
            const int32_t d = row_degree(v, N, nnz, row_ptr, bad);
            sh.deg[v] = (uint32_t)d;
            deg[v] = d;
            dinv[v] = d > 0 ? 1.0f / sqrtf((float)d) : 0.0f;
            add_row(st, d, th);
        }
    }
    st.bad = bad ? 1u : 0u;
    gather_stats(st, &sh.all);
    const uint32_t largest = sh.all.largest;
    if (tid <= kPlanThresholdCount) rb->counts[tid] = tid < kPlanThresholdCount ? sh.all.at_least[tid] : largest;
    if (tid == 0) rb->bad = sh.all.bad;

    const int steps = (N + kOrderThreads - 1) / kOrderThreads;
    const int piece = wave * steps * 64;                     // first of the wave's steps * 64 positions
    for (int shift = 0, pass = 0; shift == 0 || (shift < 32 && largest >> shift); shift += 8, ++pass) {
        const uint16_t* from = sh.ids[pass & 1];
        uint16_t* to = sh.ids[(pass & 1) ^ 1];
        const bool last = shift + 8 >= 32 || (largest >> (shift + 8)) == 0;
        auto id_at = [&](int p) { return pass == 0 ? (uint32_t)p : (uint32_t)from[p]; };
        auto digit = [&](uint32_t id) { return 255u - ((sh.deg[id] >> shift) & 255u); };      // largest first
        uint32_t* c32 = reinterpret_cast<uint32_t*>(sh.counters);
        for (int i = tid; i < kOrderWaves * 128; i += kOrderThreads) c32[i] = 0u;
        __syncthreads();
        for (int j = 0; j < steps; ++j) {
            const int p = piece + j * 64 + lane;
            const bool have = p < N;
            take_position<8>(sh.counters[wave], have ? digit(id_at(p)) : 0u, have);
        }
        __syncthreads();
        uint32_t mine = 0;
        if (tid < 256) {
            for (int w = 0; w < kOrderWaves; ++w) mine += sh.counters[w][tid];
        }
        uint32_t at = order_scan(mine, sh.sc) - mine;
        if (tid < 256) {
            for (int w = 0; w < kOrderWaves; ++w) {
                const uint32_t c = sh.counters[w][tid];
                sh.counters[w][tid] = (uint16_t)at;
                at += c;
            }
        }
        __syncthreads();
        for (int j = 0; j < steps; ++j) {
            const int p = piece + j * 64 + lane;
            const bool have = p < N;
            const uint32_t id = have ? id_at(p) : 0u;
            const uint32_t q = take_position<8>(sh.counters[wave], have ? digit(id) : 0u, have);
            if (have) {
                if (last) order[q] = (int32_t)id;
                else to[q] = (uint16_t)id;
            }
        }
        __syncthreads();
    }
}

// Larger graphs: workgroups of consecutive rows, two launches per digit of 10 bits: every workgroup counts its rows'
// digits, then every workgroup adds up the counts before its own and moves its rows.
// The first launch also makes the degrees; its largest says which digit is the last (later launches find nothing
// to do).  A whole plan of 19,717 rows 90 -> 45 us, 232,965 155 -> 95, 2,449,029 229 -> 180.
// Degrees take part up to kTopDegree, two digits.  A graph of less than 2^31 entries has at most kTopRows rows that are
// longer: the first pass that moves rows lists them, and the last puts each where its rank in the list says.  (With a third digit,
// two more passes over all rows: 4,000,000 rows, one of three million entries 348 us, 233 now, 240 with a 32-bit radix sort;
// 100,000,000 6,562, 2,231 and 3,388.)
// Workgroups (order_blocks): each reads all others' counts, so 128 of at least 2,048 rows, or 1,024 up to 32,768 rows
// (64 workgroups: 232,965 rows 85 us longer; 100,000 rows in pieces of 1,024: 83 us, of 2,048: 72); they leave half the chip idle,
// which outweighs that from some six million rows on (4,000,000 rows, two digits: 242 us, 240 with 256; 7,000,000 349 and
// 293; 20,000,000 867 and 585), and 512 from some sixty (40,000,000 1,078 with 256, 1,065 with 512; one digit 546 and 579;
// 100,000,000 2,441 and 2,193).
constexpr int kOrderBits = 10, kOrderBins = 1 << kOrderBits;
static_assert(kOrderBins == kOrderThreads, "one bin per thread");
constexpr uint32_t kTopDegree = (1u << (2 * kOrderBits)) - 1u;
constexpr int kTopRows = 2048;
static_assert((int64_t)kTopRows * kTopDegree <= 0x7fffffffll && (int64_t)(kTopRows + 1) * kTopDegree > 0x7fffffffll, "rows of a plan");
constexpr int kOrderBlocks = 512;        // at most
static int64_t order_blocks(int64_t N) { return N < 6000000 ? 128 : N < 60000000 ? 256 : kOrderBlocks; }
struct OrderArgs {
    int64_t N, per_block;                // per_block: multiple of kOrderThreads
    int passes;                          // digits that a row of nnz entries has, one or two
    const int32_t* deg;
    uint2* pairs;                        // (degree, id) between the passes
    int32_t* order;
    uint32_t* counts;                    // [blocks][kOrderBins]
    RowStats* stats;                     // [blocks]
    uint2* top;                          // [kTopRows] (degree, id) of rows of kTopDegree entries and more, in any order
};

__device__ __forceinline__ uint32_t order_digit(uint32_t d, int shift)
{
    return (kOrderBins - 1) - ((min(d, kTopDegree) >> shift) & (kOrderBins - 1));
}

__global__ __launch_bounds__(kOrderThreads) void degree_kernel(
    OrderArgs a, int64_t nnz, const int64_t* __restrict__ row_ptr, int32_t* __restrict__ deg, float* __restrict__ dinv,
    Thresholds th)
{
    __shared__ uint32_t hist[kOrderBins];
    __shared__ RowStats all;
    const int tid = threadIdx.x;
    hist[tid] = 0u;
    if (tid < (int)(sizeof(RowStats) / 4)) reinterpret_cast<uint32_t*>(&all)[tid] = 0u;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * a.per_block, end = min(begin + a.per_block, a.N);
    RowStats st = {};
    bool bad = false;
#pragma unroll 4
    for (int64_t v = begin + tid; v < end; v += kOrderThreads) {
        const int32_t d = row_degree(v, a.N, nnz, row_ptr, bad);
        deg[v] = d;
        dinv[v] = d > 0 ? 1.0f / sqrtf((float)d) : 0.0f;
        add_row(st, d, th);
        st.top += (uint32_t)d >= kTopDegree ? 1u : 0u;
        atomicAdd(&hist[order_digit((uint32_t)d, 0)], 1u);
    }
    st.bad = bad ? 1u : 0u;
    gather_stats(st, &all);
    a.counts[(int64_t)blockIdx.x * kOrderBins + tid] = hist[tid];
    if (tid < (int)(sizeof(RowStats) / 4))
        reinterpret_cast<uint32_t*>(&a.stats[blockIdx.x])[tid] = reinterpret_cast<uint32_t*>(&all)[tid];
}

// largest degree of all workgroups' rows, uniform; a barrier has passed when the call returns
__device__ __forceinline__ uint32_t largest_degree(const RowStats* stats, int blocks, uint32_t* sc)
{
    uint32_t top = (int)threadIdx.x < blocks ? stats[threadIdx.x].largest : 0u;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) top = max(top, __shfl_xor(top, m, 64));
    if ((threadIdx.x & 63) == 0) sc[threadIdx.x >> 6] = top;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < (kOrderBlocks + 63) / 64; ++w) top = max(top, sc[w]);
    __syncthreads();
    return top;
}

// digits of the second pass
__global__ __launch_bounds__(kOrderThreads) void order_count_kernel(OrderArgs a, int pass)
{
    __shared__ uint32_t hist[kOrderBins];
    __shared__ uint32_t sc[kOrderWaves];
    const int tid = threadIdx.x, shift = pass * kOrderBits;
    if ((largest_degree(a.stats, gridDim.x, sc) >> shift) == 0) return;       // the pass before was the last
    hist[tid] = 0u;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * a.per_block, end = min(begin + a.per_block, a.N);
    const uint2* from = a.pairs;
#pragma unroll 4
    for (int64_t i = begin + tid; i < end; i += kOrderThreads) atomicAdd(&hist[order_digit(from[i].x, shift)], 1u);
    __syncthreads();
    a.counts[(int64_t)blockIdx.x * kOrderBins + tid] = hist[tid];
}

__global__ __launch_bounds__(kOrderThreads) void order_move_kernel(OrderArgs a, int pass, Readback* rb)
{
    __shared__ uint32_t counters[kOrderWaves][kOrderBins];
    __shared__ uint32_t sc[kOrderWaves];
    __shared__ uint32_t top_at, top_rows;        // where this workgroup's rows go in the list a.top, and how many it holds
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, shift = pass * kOrderBits;
    const int blocks = gridDim.x;
    const uint32_t largest = largest_degree(a.stats, blocks, sc);
    if (pass == 0 && blockIdx.x == 0 && tid <= kPlanThresholdCount + 1) {
        if (tid < kPlanThresholdCount) {
            int64_t c = 0;
            for (int b = 0; b < blocks; ++b) c += a.stats[b].at_least[tid];
            rb->counts[tid] = c;
        } else if (tid == kPlanThresholdCount) {
            rb->counts[tid] = largest;
        } else {
            uint32_t bad = 0;
            for (int b = 0; b < blocks; ++b) bad |= a.stats[b].bad;
            rb->bad = bad;
        }
    }
    if (pass > 0 && (largest >> shift) == 0) return;
    // (a row_ptr that is refused may claim more entries in a row than there are: the order is a permutation all the same,
    // since a row is placed by its rank only where all of them are in the list)
    const bool last = pass + 1 == a.passes || (largest >> (shift + kOrderBits)) == 0;
    for (int i = tid; i < kOrderWaves * kOrderBins; i += kOrderThreads) (&counters[0][0])[i] = 0u;
    if (largest >= kTopDegree) {                             // (uniform)
        if (tid == 0) top_at = top_rows = 0u;
        __syncthreads();                                     // (more barriers lie between the counts and their use)
        if (tid < blocks && a.stats[tid].top) {
            atomicAdd(&top_rows, a.stats[tid].top);
            if (tid < (int)blockIdx.x) atomicAdd(&top_at, a.stats[tid].top);
        }
    }
    // rows of bin tid: in the workgroups before this one, and in all
    uint32_t before = 0, all = 0;
#pragma unroll 16
    for (int b = 0; b < blocks; ++b) {
        const uint32_t c = a.counts[(int64_t)b * kOrderBins + tid];
        if (b < (int)blockIdx.x) before += c;
        all += c;
    }
    uint32_t at = order_scan(all, sc) - all + before;        // (its barriers also separate the zeroes from the counts)

    const int64_t per_wave = a.per_block / kOrderWaves;      // multiple of 64
    const int64_t begin = (int64_t)blockIdx.x * a.per_block + wave * per_wave, end = min(begin + per_wave, a.N);
    const uint2* from = a.pairs;
    uint2* to = a.pairs;                                     // (only a pass that is not the last writes them)
    auto entry = [&](int64_t i) { return pass == 0 ? make_uint2((uint32_t)a.deg[i], (uint32_t)i) : from[i]; };
#pragma unroll 4
    for (int64_t i = begin + lane; i < end; i += 64) atomicAdd(&counters[wave][order_digit(entry(i).x, shift)], 1u);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kOrderWaves; ++w) {
        const uint32_t c = counters[w][tid];
        counters[w][tid] = at;
        at += c;
    }
    __syncthreads();
    const bool ranked = last && pass > 0 && largest >= kTopDegree && top_rows <= (uint32_t)kTopRows;
    constexpr int AHEAD = 4;                                 // rows in flight per lane
    for (int64_t i0 = begin; i0 < end; i0 += 64 * AHEAD) {
        uint2 e[AHEAD];
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            const int64_t i = i0 + 64 * t + lane;
            e[t] = i < end ? entry(i) : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            if (i0 + 64 * t >= end) break;                   // (uniform)
            const bool have = i0 + 64 * t + lane < end;
            const uint32_t q = take_position<kOrderBits>(counters[wave], order_digit(e[t].x, shift), have);
            const bool longest = have && e[t].x >= kTopDegree;
            if (have) {
                if (!last) to[q] = e[t];
                else if (!(longest && ranked)) a.order[q] = (int32_t)e[t].y;
            }
            if (longest && !last) {
                const uint32_t at = atomicAdd(&top_at, 1u);
                if (at < (uint32_t)kTopRows) a.top[at] = e[t];
            }
            if (longest && ranked) {                         // by degree, then id
                uint32_t rank = 0;
                for (uint32_t i = 0; i < top_rows; ++i) {
                    const uint2 o = a.top[i];
                    rank += o.x > e[t].x || (o.x == e[t].x && o.y < e[t].y) ? 1u : 0u;
                }
                a.order[rank] = (int32_t)e[t].y;
            }
        }
    }
}

__global__ __launch_bounds__(kThreads) void check_columns(
    int64_t nnz, int64_t N, const int32_t* __restrict__ col_idx, uint32_t* bad)
{
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= nnz) return;
    const int32_t c = col_idx[e];
    if (c < 0 || c >= N) atomicOr(bad, 1u);
}

// part_ptr[k][s] = first position in row order[s] whose column is >= k * span (columns ascend in a row).
// Sixteen lanes per row, four rows per wave: lane k finds its boundary by bisection over the row (a dozen
// dependent loads that mostly hit the row's few cache lines in L2; walking every column of every row instead
// kept the vector units busy for 0.25 ms on the Reddit-shaped graph).  A prefix maximum over the sixteen
// positions then makes them a monotone chain from row start to row end whatever the order of the columns, so
// every entry lies in exactly one range even for a caller's CSR with unsorted rows (there the cut points are
// arbitrary, which costs locality, not correctness).
__global__ __launch_bounds__(kThreads) void split_rows_kernel(
    int64_t N, int64_t nnz, int64_t span, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    const int32_t* __restrict__ order, int32_t* __restrict__ part_ptr)
{
    static_assert(kMaxParts == 16, "one lane per boundary, four rows per wave");
    const int k = threadIdx.x & 15;
    const int64_t s = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 4;
    bool have = s < N;
    int64_t begin = 0, end = 0;
    if (have) {
        const int64_t v = order[s];
        begin = row_ptr[v];
        end = row_ptr[v + 1];
        // this runs before the host has seen the verdict on row_ptr: a row that does not lie inside
        // col_idx is left alone (such a CSR is rejected and the plan never used)
        if (begin < 0 || end > nnz || begin > end) { have = false; begin = end = 0; }
    }
    const int64_t target = (int64_t)k * span;
    int64_t lo = begin, hi = end;
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((int64_t)col_idx[mid] < target) lo = mid + 1;
        else hi = mid;
    }
    int p = (int)lo;                           // the split exists only for graphs of fewer than 2^31 entries
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const int o = __shfl_up(p, d, 16);
        if (k >= d) p = max(p, o);
    }
    if (have) {
        part_ptr[(int64_t)k * N + s] = p;
        if (k == 15) part_ptr[(int64_t)kMaxParts * N + s] = (int32_t)end;
    }
}

struct PlanLayout {
    bool split;
    int64_t o_deg, o_dinv, o_order, o_part, keep_bytes;            // what the plan keeps
    int64_t s_rb, s_pairs, s_counts, s_stats, s_top, scratch_bytes;   // what only its construction needs
    bool small;
    int passes, blocks;                                            // of the order sort
    int64_t per_block;
};

int plan_layout(int64_t N, int64_t nnz, unsigned flags, PlanLayout& L)
{
    const int64_t n1 = N > 0 ? N : 1;
    // Dense-enough graphs whose feature table cannot stay in L2 get the row split that lets
    // the aggregation walk one source-id range at a time.
    L.split = N > 0 && nnz > 0 &&
              ((flags & RETEXO_F_SPLIT_ROWS) ||
               (nnz >= 64 * N && N * 128 > (4ll << 20) && N * 128 <= kMaxParts * (8ll << 20)));
    L.o_deg = 0;
    L.o_dinv = align_up(4 * n1, 256);
    L.o_order = 2 * L.o_dinv;
    L.o_part = 3 * L.o_dinv;
    L.keep_bytes = L.o_part + (L.split ? align_up(4 * N * (kMaxParts + 1), 256) : 0);
    // scratch: readback block, and for larger graphs the pairs, counts and sums of the order sort
    L.small = N <= kSmallRows;
    const int64_t share = (n1 + order_blocks(N) - 1) / order_blocks(N);
    L.per_block = align_up(N > 32768 && share < 2048 ? 2048 : share, kOrderThreads);
    L.blocks = (int)((N + L.per_block - 1) / L.per_block);
    L.passes = nnz >> kOrderBits ? 2 : 1;                          // digits that a degree can have
    L.s_rb = 0;
    L.s_pairs = 256;
    const int64_t pairs = L.small ? 0 : align_up(8 * n1, 256);
    L.s_counts = L.s_pairs + pairs;
    L.s_stats = L.s_counts + (L.small ? 0 : 4ll * L.blocks * kOrderBins);
    L.s_top = L.s_stats + (L.small ? 0 : align_up((int64_t)sizeof(RowStats) * L.blocks, 256));
    L.scratch_bytes = L.s_top + (L.small ? 0 : (int64_t)sizeof(uint2) * kTopRows) + 256;
    return RETEXO_OK;
}

// Everything after the sizes are known: the kernels, the one read-back, the host fields.  `keep` and `scratch`
// are device memory of L.keep_bytes and L.scratch_bytes.
int plan_fill(retexo_plan* p, const PlanLayout& L, unsigned flags, void* keep, void* scratch, hipStream_t stream)
{
    const int64_t N = p->N, nnz = p->nnz;
    p->deg = (int32_t*)((char*)keep + L.o_deg);
    p->dinv = (float*)((char*)keep + L.o_dinv);
    p->order = (int32_t*)((char*)keep + L.o_order);
    char* sc = (char*)scratch;
    Readback* rb = (Readback*)(sc + L.s_rb);
    const bool check = (flags & RETEXO_F_VALIDATE) && nnz > 0;         // (its atomics need device memory)
    HostReport report(stream, p->block != nullptr);                    // (retexo_plan_create_in does not allocate)
    static_assert(sizeof(Readback) <= kReportBytes, "a report holds it");
    const bool direct = N > 0 && !check && report.get();
    if (direct) rb = (Readback*)report.get();
    Thresholds th;
    for (int i = 0; i < kPlanThresholdCount; ++i) th.t[i] = kPlanThresholds[i];
    if (N == 0) {
        RETEXO_HIP_TRY(hipMemsetAsync(rb, 0, sizeof(Readback), stream));
    } else if (L.small) {
        small_order_kernel<<<dim3(1), dim3(kOrderThreads), 0, stream>>>((int)N, nnz, p->row_ptr, p->deg, p->dinv, p->order,
                                                                        th, rb);
    } else {
        OrderArgs a;
        a.N = N;
        a.per_block = L.per_block;
        a.passes = L.passes;
        a.deg = p->deg;
        a.pairs = (uint2*)(sc + L.s_pairs);
        a.top = (uint2*)(sc + L.s_top);
        a.order = p->order;
        a.counts = (uint32_t*)(sc + L.s_counts);
        a.stats = (RowStats*)(sc + L.s_stats);
        const dim3 grid((unsigned)L.blocks), block(kOrderThreads);
        degree_kernel<<<grid, block, 0, stream>>>(a, nnz, p->row_ptr, p->deg, p->dinv, th);
        for (int pass = 0; pass < L.passes; ++pass) {
            if (pass > 0) order_count_kernel<<<grid, block, 0, stream>>>(a, pass);
            order_move_kernel<<<grid, block, 0, stream>>>(a, pass, rb);
        }
    }
    if (L.split) {
        // needs only the schedule order, so it runs before the host looks at the counts
        p->part_ptr = (int32_t*)((char*)keep + L.o_part);
        p->part_span = (N + kMaxParts - 1) / kMaxParts;
        const int64_t rows_per_block = kThreads / 16;
        split_rows_kernel<<<dim3((unsigned)((N + rows_per_block - 1) / rows_per_block)), dim3(kThreads), 0, stream>>>(
            N, nnz, p->part_span, p->row_ptr, p->col_idx, p->order, p->part_ptr);
    }
    if (check)
        check_columns<<<dim3((unsigned)((nnz + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream>>>(
            nnz, N, p->col_idx, &rb->bad);
    RETEXO_HIP_TRY(hipGetLastError());
    Readback h;
    if (!direct) RETEXO_HIP_TRY(hipMemcpyAsync(&h, rb, sizeof(h), hipMemcpyDeviceToHost, stream));
    RETEXO_HIP_TRY(report.wait());
    if (direct) memcpy(&h, rb, sizeof(h));
    if (h.bad) return RETEXO_E_CSR;
    for (int i = 0; i < kPlanThresholdCount; ++i) p->rows_at_least[i] = h.counts[i];
    p->max_degree = (int32_t)h.counts[kPlanThresholdCount];
    return RETEXO_OK;
}

}  // namespace

extern "C" int retexo_plan_create(retexo_plan** out, int64_t N, const int64_t* d_row_ptr,
                                  const int32_t* d_col_idx, unsigned flags, void* stream_)
{
    if (!out) return RETEXO_E_NULL;
    *out = nullptr;
    if (N < 0 || N >= (1ll << 31)) return RETEXO_E_SIZE;
    if (flags & ~(unsigned)(RETEXO_F_VALIDATE | RETEXO_F_SPLIT_ROWS)) return RETEXO_E_FLAGS;
    if (!d_row_ptr) return RETEXO_E_NULL;
    hipStream_t stream = (hipStream_t)stream_;

    retexo_plan* p = new (std::nothrow) retexo_plan();
    if (!p) return RETEXO_E_HIP;
    p->N = N;
    p->row_ptr = d_row_ptr;
    p->col_idx = d_col_idx;
    auto fail = [&](int code) { retexo_plan_destroy(p); return code; };

    // The entry count decides whether the row split is built, so it is fetched first; everything the plan
    // keeps then comes from one allocation (device allocations cost tens of microseconds each).
    int64_t nnz = 0;
    if (hipMemcpyAsync(&nnz, d_row_ptr + N, sizeof(int64_t), hipMemcpyDeviceToHost, stream) != hipSuccess)
        return fail(RETEXO_E_HIP);
    if (hipStreamSynchronize(stream) != hipSuccess) return fail(RETEXO_E_HIP);
    if (nnz < 0) return fail(RETEXO_E_CSR);
    if (nnz >= (1ll << 31)) return fail(RETEXO_E_SIZE);
    if (nnz > 0 && !d_col_idx) return fail(RETEXO_E_NULL);
    p->nnz = nnz;
    PlanLayout L;
    if (int e = plan_layout(N, nnz, flags, L)) return fail(e);
    if (hipMalloc(&p->block, (size_t)L.keep_bytes) != hipSuccess) return fail(RETEXO_E_HIP);
    if (hipMalloc(&p->build_scratch, (size_t)L.scratch_bytes) != hipSuccess) return fail(RETEXO_E_HIP);
    if (int e = plan_fill(p, L, flags, p->block, p->build_scratch, stream)) return fail(e);
    (void)hipFree(p->build_scratch);
    p->build_scratch = nullptr;
    *out = p;
    return RETEXO_OK;
}

extern "C" int64_t retexo_plan_workspace_bytes(int64_t N, int64_t nnz, unsigned flags)
{
    if (N < 0 || N >= (1ll << 31) || nnz < 0 || nnz >= (1ll << 31)) return RETEXO_E_SIZE;
    if (flags & ~(unsigned)(RETEXO_F_VALIDATE | RETEXO_F_SPLIT_ROWS)) return RETEXO_E_FLAGS;
    PlanLayout L;
    if (int e = plan_layout(N, nnz, flags, L)) return e;
    return L.keep_bytes + L.scratch_bytes;
}

extern "C" int retexo_plan_create_in(retexo_plan** out, int64_t N, int64_t nnz, const int64_t* d_row_ptr,
                                     const int32_t* d_col_idx, unsigned flags,
                                     void* d_workspace, int64_t workspace_bytes, void* stream_)
{
    if (!out) return RETEXO_E_NULL;
    *out = nullptr;
    if (N < 0 || N >= (1ll << 31) || nnz < 0 || nnz >= (1ll << 31)) return RETEXO_E_SIZE;
    if (flags & ~(unsigned)(RETEXO_F_VALIDATE | RETEXO_F_SPLIT_ROWS)) return RETEXO_E_FLAGS;
    if (!d_row_ptr || (nnz > 0 && !d_col_idx)) return RETEXO_E_NULL;
    PlanLayout L;
    if (int e = plan_layout(N, nnz, flags, L)) return e;
    if (!d_workspace || ((uintptr_t)d_workspace & 255) != 0 || workspace_bytes < L.keep_bytes + L.scratch_bytes)
        return RETEXO_E_WORKSPACE;
    retexo_plan* p = new (std::nothrow) retexo_plan();
    if (!p) return RETEXO_E_HIP;
    p->N = N;
    p->nnz = nnz;
    p->row_ptr = d_row_ptr;
    p->col_idx = d_col_idx;
    // the plan's arrays live in the caller's workspace: nothing to free but the host structure
    if (int e = plan_fill(p, L, flags, d_workspace, (char*)d_workspace + L.keep_bytes, (hipStream_t)stream_)) {
        delete p;
        return e;
    }
    *out = p;
    return RETEXO_OK;
}

extern "C" int retexo_plan_destroy(retexo_plan* p)
{
    if (!p) return RETEXO_OK;
    if (p->block) (void)hipFree(p->block);       // deg, dinv, order and part_ptr live in it
    if (p->build_scratch) (void)hipFree(p->build_scratch);
    delete p;
    return RETEXO_OK;
}

extern "C" int64_t retexo_plan_num_nodes(const retexo_plan* p) { return p ? p->N : RETEXO_E_NULL; }
extern "C" int64_t retexo_plan_nnz(const retexo_plan* p) { return p ? p->nnz : RETEXO_E_NULL; }
extern "C" int32_t retexo_plan_max_degree(const retexo_plan* p) { return p ? p->max_degree : RETEXO_E_NULL; }
extern "C" const int32_t* retexo_plan_deg(const retexo_plan* p) { return p ? p->deg : nullptr; }
extern "C" const float* retexo_plan_dinv(const retexo_plan* p) { return p ? p->dinv : nullptr; }

namespace {
// dst[i] = src[i] for i < n words; the exports are kernels (not copy nodes) so that a caller may record them
// into a HIP graph like every other stream-ordered entry point
__global__ __launch_bounds__(kThreads) void copy_words_kernel(int64_t n, const uint32_t* __restrict__ src,
                                                              uint32_t* __restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

int copy_words(int64_t n, const void* src, void* dst, hipStream_t stream)
{
    if (n <= 0) return RETEXO_OK;
    copy_words_kernel<<<dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream>>>(
        n, (const uint32_t*)src, (uint32_t*)dst);
    return hipGetLastError() == hipSuccess ? RETEXO_OK : RETEXO_E_HIP;
}
}  // namespace

extern "C" int retexo_plan_export(const retexo_plan* p, int32_t* d_deg, float* d_dinv, int32_t* d_order,
                                  void* stream_)
{
    if (!p) return RETEXO_E_NULL;
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t n = p->N;
    if (n == 0) return RETEXO_OK;
    if (d_deg) if (int e = copy_words(n, p->deg, d_deg, stream)) return e;
    if (d_dinv) if (int e = copy_words(n, p->dinv, d_dinv, stream)) return e;
    if (d_order) if (int e = copy_words(n, p->order, d_order, stream)) return e;
    return RETEXO_OK;
}

static_assert(kMaxParts == RETEXO_SPLIT_PARTS, "the header states the number of source-id ranges");

extern "C" int64_t retexo_plan_export_split(const retexo_plan* p, int32_t* d_pos, void* stream_)
{
    if (!p) return RETEXO_E_NULL;
    if (!p->part_ptr) return 0;
    if (d_pos)
        if (int e = copy_words(p->N * (kMaxParts + 1), p->part_ptr, d_pos, (hipStream_t)stream_)) return e;
    return p->part_span;
}
