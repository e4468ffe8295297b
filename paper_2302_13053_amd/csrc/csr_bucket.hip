// CSR construction from raw undirected pairs by bucketing (the fast path of retexo_csr_from_coo).
//
// The paper's graphs are undirected (section "Edge-partitioned Distributed Setup"): each pair {u,v}
// becomes the entries (u,v) and (v,u), repeats are kept once, self pairs are dropped, and
// add_self_loops appends one entry (v,v) per node.  The result — rows in id order, columns
// ascending and unique — is a function of the pair set alone, so any order of evaluation gives
// the same bits.  That freedom is what this file uses: instead of sorting 64-bit (row, col) keys
// with a general radix sort (five to six passes over 16 bytes per entry), the entries are first
// moved into buckets of consecutive rows that fit the local data share, and each bucket is then
// sorted and cleaned there, by one workgroup, without touching memory in between.
//
//   hist     every workgroup counts its share of the entries per row range ("bin", 2^s rows) in LDS
//   colsum   adds the workgroups' counts
//   plan     one workgroup: prefix sums over the bins, buckets = runs of bins of about `target`
//            entries (never more than kRowSpan rows), groups = runs of 256 buckets
//   part1    entries -> their group   (skipped when there is only one group)
//   part2    entries -> their bucket, packed as (row - first row of the bucket) << cbits | col
//            (both moves stage a tile in LDS ordered by destination, reserve the destination ranges
//             with one atomic per destination and tile, and write runs)
//   sort     one workgroup per bucket: entries counted per row, every row given a number of column
//            bins proportional to its length (so that a bin holds 1 or 2 entries whatever the
//            degree), LDS counting split into those bins, rank by comparison inside a bin,
//            drop repeats, count the kept entries per row;
//            a bucket that does not fit LDS is marked in a bit map or worked through in key ranges, the ranges
//            split until each fits (a single long row, a clustered row range, many repeats: all end)
//   total    one workgroup: prefix sums over the buckets' entry counts -> nnz
//   emit     one workgroup per bucket: row offsets of its rows, columns to their final place
//            (nothing is written when an id was out of range or the capacity is too small)
//
// Integer arithmetic only.  The order in which atomics hand out positions inside a bucket is
// arbitrary, but the sorted, repeat-free result is not, so the output is bitwise reproducible.
#include <string.h>
#include <type_traits>

#include "common.hpp"
#include "csr_bucket.hpp"
#include "report.hpp"

namespace {

constexpr int kThreads = 1024;           // hist, plan, part1, part2, sort, total
constexpr int kWaves = kThreads / 64;
constexpr int kMaxBins = 32768;          // row ranges the histogram distinguishes
constexpr int kMaxHistBlocks = 256;
constexpr int kSmallBins = 4096;         // row ranges of a small graph, whose items one workgroup counts and plans
constexpr int64_t kSmallItems = 196608;  // 190,000 pairs: 103 us, 111 in several workgroups; 220,000: 108 and 106
constexpr int kFewBuckets = 1024;        // so many that every workgroup of emit adds up their counts by itself
constexpr int kItemsPerTile = 4096;      // pairs per part1 tile (two entries each)
constexpr int kTileEntries = 8192;       // entries per part2 tile
constexpr int kGroupBuckets = 256;       // buckets per group
constexpr int kMaxGroups = 768;           // (part1's tables and its tile fit a CU twice)
constexpr int kMaxBuckets = kGroupBuckets * kMaxGroups;
constexpr int64_t kMaxEntries = 447000000;   // more were never built this way: they take the sorted keys
constexpr int kBucketMax = 10240;        // entries a bucket can hold in LDS (10 per thread)
constexpr int kTargetMax = 7168;         // entries a bucket is filled to in a large graph
constexpr int kTargetMin = 1024;         // ... and in a small one
constexpr int kTargetBuckets = 160;      // buckets a graph is spread over before they are filled further
constexpr int kRowSpan = 1024;           // rows per bucket at most (one per thread of the sort)
constexpr int kSortBins = kBucketMax + kRowSpan;         // bins of the LDS split: a row of c entries gets max(1, c/2 to c)
constexpr int kStack = 400;              // key ranges waiting in an oversized bucket (6 levels x 63 + 1)

struct BucketHeader {       // start of the workspace
    uint32_t bad_id;        // an id was outside [0, N)
    uint32_t overflow;      // nnz exceeds the capacity of col_idx
    int64_t nnz;
    uint32_t n_buckets;
    uint32_t n_groups;
    uint32_t part2_tiles;
    uint32_t internal;      // a construction invariant failed (never expected)
    uint32_t one_word;      // the rows of every group are few enough: part1's entries take one word (plan)
};


// exclusive prefix sum over the workgroup (NW waves); `total` is the sum over all threads.
// sc: 2 * NW + 1 words of LDS scratch, free again when the call returns.
template <int NW>
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* sc, uint32_t& total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) sc[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        const uint32_t w = lane < NW ? sc[lane] : 0u;
        uint32_t wi = w;
#pragma unroll
        for (int d = 1; d < NW; d <<= 1) {
            const uint32_t t = __shfl_up(wi, d, 64);
            if (lane >= d) wi += t;
        }
        if (lane < NW) sc[NW + lane] = wi - w;
        if (lane == NW - 1) sc[2 * NW] = wi;
    }
    __syncthreads();
    const uint32_t excl = incl - v + sc[NW + wave];
    total = sc[2 * NW];
    __syncthreads();
    return excl;
}

// largest g in [0, n) with table[g] <= x (table ascending, table[0] <= x)
__device__ __forceinline__ int find_segment(const uint32_t* table, int n, uint32_t x)
{
    int lo = 0, hi = n;
    while (lo + 1 < hi) {
        const int mid = (lo + hi) >> 1;
        if (table[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// arr[idx] += one for every lane with `active` set.  When all of them name the same element (a long row, a
// clustered range) the wave adds their number once instead of queueing up on one LDS address.
// Call with the whole wave (the loop around it must be uniform per wave).
__device__ __forceinline__ void lds_count(uint32_t* arr, uint32_t idx, bool active, uint32_t one = 1u)
{
    const uint64_t act = __ballot(active);
    if (!act) return;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((unsigned long long)act) - 1;
    const uint32_t first = __shfl(idx, leader, 64);
    const uint64_t same = __ballot(active && idx == first);
    if (same == act) {
        if (lane == leader) atomicAdd(&arr[first], (uint32_t)__popcll(act) * one);
    } else if (active) {
        atomicAdd(&arr[idx], one);
    }
}

// Items i, i + kThreads, ... (COUNT of them, those below `end`): pair i for i < n_pairs, afterwards the self-loop of node
// i - n_pairs.  All loads are issued before the first is used.
template <int COUNT>
struct Items {
    uint32_t u[COUNT], v[COUNT];
    uint32_t entries;                                    // two bits per item: 0, 1 or 2 entries (u,v), (v,u)
    __device__ __forceinline__ void load(int64_t i0, int64_t end, int64_t n_pairs, const int32_t* __restrict__ src,
                                         const int32_t* __restrict__ dst)
    {
#pragma unroll
        for (int t = 0; t < COUNT; ++t) {
            const int64_t i = i0 + t * kThreads;
            const bool pair = i < end && i < n_pairs;
            u[t] = pair ? (uint32_t)src[i] : 0u;
            v[t] = pair ? (uint32_t)dst[i] : 0u;
        }
    }
    __device__ __forceinline__ void look(int64_t i0, int64_t end, int64_t n_pairs, int64_t N, bool& bad)
    {
        entries = 0u;
#pragma unroll
        for (int t = 0; t < COUNT; ++t) {
            const int64_t i = i0 + t * kThreads;
            if (i >= end) continue;
            if (i >= n_pairs) {
                u[t] = v[t] = (uint32_t)(i - n_pairs);
                entries |= 1u << (2 * t);
            } else if (u[t] >= (uint64_t)N || v[t] >= (uint64_t)N) {
                bad = true;
            } else if (u[t] != v[t]) {                   // self pairs are dropped
                entries |= 2u << (2 * t);
            }
        }
    }
    __device__ __forceinline__ bool first(int t) const { return (entries >> (2 * t)) & 3u; }
    __device__ __forceinline__ bool second(int t) const { return (entries >> (2 * t)) & 2u; }
};

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void hist_kernel(
    int64_t n_pairs, const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t N, int64_t n_items,
    int64_t items_per_block, int s, int nbins, uint32_t* __restrict__ counts, BucketHeader* hdr)
{
    __shared__ uint32_t hist[kMaxBins];
    for (int i = threadIdx.x; i < nbins; i += kThreads) hist[i] = 0u;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * items_per_block;
    const int64_t end = begin + items_per_block < n_items ? begin + items_per_block : n_items;
    bool bad = false;
    // (one workgroup per CU, so the pairs in flight are what hides the memory: one per thread 168 us on the Reddit-shaped
    // graph, eight 105)
    Items<8> it;
    for (int64_t i0 = begin + threadIdx.x; i0 < end; i0 += 8 * kThreads) {
        it.load(i0, end, n_pairs, src, dst);
        it.look(i0, end, n_pairs, N, bad);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (it.first(t)) atomicAdd(&hist[it.u[t] >> s], 1u);
            if (it.second(t)) atomicAdd(&hist[it.v[t] >> s], 1u);
        }
    }
    if (bad) atomicOr(&hdr->bad_id, 1u);
    __syncthreads();
    uint32_t* mine = counts + (size_t)blockIdx.x * nbins;
    for (int i = threadIdx.x; i < nbins; i += kThreads) mine[i] = hist[i];
}

// bin_count[b] += the counts of this block's slice of the histogram blocks (bin_count starts at zero)
constexpr int kColsumSlices = 8;
__global__ __launch_bounds__(256) void colsum_kernel(int nblocks, int nbins, const uint32_t* __restrict__ counts,
                                                     uint32_t* bin_count)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= nbins) return;
    const int per = (nblocks + kColsumSlices - 1) / kColsumSlices;
    const int w0 = blockIdx.y * per, w1 = w0 + per < nblocks ? w0 + per : nblocks;
    uint32_t s = 0;
    for (int w = w0; w < w1; ++w) s += counts[(size_t)w * nbins + b];
    if (s) atomicAdd(&bin_count[b], s);
}

struct PlanArrays {
    uint32_t* bucket_bin0;    // [n_buckets + 1] first bin of each bucket
    uint32_t* bucket_off;     // [n_buckets + 1] entries before each bucket
    uint32_t* bucket_cursor;  // [n_buckets] part2's write positions
    uint32_t* group_bin0;     // [n_groups + 1]
    uint32_t* group_off;      // [n_groups + 1]
    uint32_t* group_cursor;   // [n_groups] part1's write positions
    uint32_t* group_tile0;    // [n_groups + 1] first part2 tile of each group
    uint16_t* coarse_group;   // [kMaxBins / 16] per block of 16 bins: group of its first bin | (bin offset inside the
                              // block at which the next group starts, 16 = none) << 10
};

// A bin starts a bucket when the entries before it enter another window of about `target`, when it is the
// first bin of a window of `span_bins` bins (so that a bucket never holds more than kRowSpan rows
// and its rows pack into 32 - cbits bits), or when it does not fit behind the bins before it in its
// window: it then reaches over the window's end, the next bin lies in another one, and the bucket
// holds it alone.  So only a bin that does not fit by itself makes a bucket that does not (those are
// worked through in key ranges, which a graph of few buckets waits for: 169,343 nodes of skewed
// degrees, 1.2 million pairs, 212 us where a bin was only looked at with its neighbour, 172 so).
// per_entry = floor(2^32 / target): the windows are up to 7e-6 longer than `target`, and a bin's is one multiplication (the
// divisions took 4 us of a construction of 150: one workgroup goes through the bins).
constexpr int kLookBack = 8;                     // bins; where the window holds more before it, its start counts
__device__ __forceinline__ uint32_t window_of(uint32_t off, uint32_t per_entry) { return __umulhi(off, per_entry); }
__device__ __forceinline__ bool starts_bucket(int bin, uint32_t off, const uint32_t* cnts, int span_bins, uint32_t target,
                                              uint32_t per_entry)
{
    if (bin == 0 || bin % span_bins == 0) return true;
    const uint32_t w = window_of(off, per_entry), cnt = cnts[bin];
    if (w != window_of(off - cnts[bin - 1], per_entry)) return true;
    uint32_t first = w * target;                 // no later than the first bin of the window
    if (off - first + cnt <= (uint32_t)kBucketMax) return false;
    uint32_t o = off;
    for (int back = 1; back <= kLookBack; ++back) {
        const uint32_t before = bin >= back ? o - cnts[bin - back] : 0u;
        if (bin < back || window_of(before, per_entry) != w) {
            first = o;
            break;
        }
        o = before;
    }
    return off - first + cnt > (uint32_t)kBucketMax;
}

// COUNT: a small graph, counted here as well (hist, colsum, the clearing of the header and this kernel were four launches: a
// construction over 2,708 nodes and 5,429 pairs 80 -> 57 us, 19,717 and 44,338 106 -> 67); there is one group then, and no part1.
template <bool COUNT>
__global__ __launch_bounds__(kThreads) void plan_kernel(int nbins, int span_bins, int group_bins, uint32_t target, uint32_t per_entry,
                                                        const uint32_t* __restrict__ bin_count, int64_t n_pairs,
                                                        const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                        int64_t N, int64_t n_items, int s,
                                                        PlanArrays a, uint32_t bucket_capacity, BucketHeader* hdr)
{
    __shared__ uint32_t cnts[COUNT ? kSmallBins : kMaxBins];      // the bin counts, read three times
    __shared__ uint32_t sc[2 * kWaves + 1];
    if constexpr (COUNT) {
        for (int b = threadIdx.x; b < nbins; b += kThreads) cnts[b] = 0u;
        if (threadIdx.x == 0) *hdr = BucketHeader{};
        __syncthreads();
        bool bad = false;
        Items<8> it;
        for (int64_t i0 = threadIdx.x; i0 < n_items; i0 += 8 * kThreads) {
            it.load(i0, n_items, n_pairs, src, dst);
            it.look(i0, n_items, n_pairs, N, bad);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                if (it.first(t)) atomicAdd(&cnts[it.u[t] >> s], 1u);
                if (it.second(t)) atomicAdd(&cnts[it.v[t] >> s], 1u);
            }
        }
        if (__syncthreads_or(bad)) {
            if (threadIdx.x == 0) hdr->bad_id = 1u;
            return;
        }
    } else {
        if (hdr->bad_id) return;
        for (int b = threadIdx.x; b < nbins; b += kThreads) cnts[b] = bin_count[b];
        __syncthreads();
    }
    // (an odd number of bins per thread: neighbouring threads then read different LDS banks)
    const int per = ((nbins + kThreads - 1) / kThreads) | 1;
    const int b0 = (int)threadIdx.x * per < nbins ? (int)threadIdx.x * per : nbins, b1 = b0 + per < nbins ? b0 + per : nbins;
    uint32_t sum = 0;
    for (int b = b0; b < b1; ++b) sum += cnts[b];
    uint32_t total;
    uint32_t off = block_scan_excl<kWaves>(sum, sc, total);
    uint32_t starts = 0;
    uint64_t which = 0;                            // which of the thread's bins (at most 33) start a bucket
    {
        uint32_t o = off;
        for (int b = b0; b < b1; ++b) {
            const uint32_t cnt = cnts[b];
            if (starts_bucket(b, o, cnts, span_bins, target, per_entry)) {
                ++starts;
                which |= 1ull << (b - b0);
            }
            o += cnt;
        }
    }
    uint32_t n_buckets;
    uint32_t id = block_scan_excl<kWaves>(starts, sc, n_buckets);
    if (n_buckets > bucket_capacity) {             // cannot happen: the host sized the arrays for the worst case
        if (threadIdx.x == 0) { hdr->internal = 1u; hdr->n_buckets = 0u; hdr->n_groups = 0u; hdr->part2_tiles = 0u; }
        return;
    }
    {
        uint32_t o = off;
        for (int b = b0; b < b1; ++b) {
            if ((which >> (b - b0)) & 1u) {
                a.bucket_bin0[id] = (uint32_t)b;
                a.bucket_off[id] = o;
                a.bucket_cursor[id] = o;
                ++id;
            }
            o += cnts[b];
        }
    }
    const uint32_t n_groups = (n_buckets + kGroupBuckets - 1) / kGroupBuckets;
    if (threadIdx.x == 0) {
        a.bucket_bin0[n_buckets] = (uint32_t)nbins;
        a.bucket_off[n_buckets] = total;
        hdr->n_buckets = n_buckets;
        hdr->n_groups = n_groups;
    }
    if (COUNT) return;
    __syncthreads();                               // the bucket arrays are complete
    // one group per thread (n_groups <= kMaxGroups <= kThreads)
    const uint32_t g = threadIdx.x;
    uint32_t tiles = 0, bins_here = 0;
    if (g < n_groups) {
        const uint32_t first = g * kGroupBuckets;
        const uint32_t last = first + kGroupBuckets < n_buckets ? first + kGroupBuckets : n_buckets;
        const uint32_t lo = a.bucket_off[first], hi = a.bucket_off[last];
        a.group_bin0[g] = a.bucket_bin0[first];
        bins_here = a.bucket_bin0[last] - a.bucket_bin0[first];
        a.group_off[g] = lo;
        a.group_cursor[g] = lo;
        tiles = (hi - lo + kTileEntries - 1) / kTileEntries;
    }
    uint32_t n_tiles;
    const uint32_t t0 = block_scan_excl<kWaves>(tiles, sc, n_tiles);
    if (g < n_groups) a.group_tile0[g] = t0;
    const int wide = __syncthreads_or(bins_here > (uint32_t)group_bins);
    if (threadIdx.x == 0) {
        a.group_bin0[n_groups] = (uint32_t)nbins;
        a.group_off[n_groups] = total;
        a.group_tile0[n_groups] = n_tiles;
        hdr->part2_tiles = n_tiles;
        hdr->one_word = wide ? 0u : 1u;
    }
    __syncthreads();                               // the group arrays are complete
    // A group other than the last holds 256 buckets, i.e. at least 256 bins, so a block of 16 bins meets at most
    // one group boundary.
    for (int c = threadIdx.x; c < kMaxBins / 16; c += kThreads) {
        const uint32_t first_bin = (uint32_t)c << 4;
        uint32_t g = n_groups - 1, at = 16;
        if (first_bin < (uint32_t)nbins) {
            g = (uint32_t)find_segment(a.group_bin0, (int)n_groups, first_bin);
            if (g + 1 < n_groups && a.group_bin0[g + 1] - first_bin < 16u) at = a.group_bin0[g + 1] - first_bin;
        }
        a.coarse_group[c] = (uint16_t)(g | (at << 10));
    }
}

// ---------------------------------------------------------------------------
// part1: the entries of one tile of items go to their groups, as (row, col) pairs or, where every group spans few enough
// rows, as one word (row - first row of the group) << cbits | col.  Bound by its bytes and part2's, which reads them: the
// Reddit-shaped graph's 117 million entries 415 -> 296 us here and 462 -> 312 there (372 and 409 with two words: the rest
// is all loads of a tile issued before the first is used).
__global__ __launch_bounds__(kThreads) void part1_kernel(
    int64_t n_pairs, const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t N, int64_t n_items, int s,
    int cbits, const uint16_t* __restrict__ coarse_group, const uint32_t* __restrict__ group_bin0, uint32_t* group_cursor, uint32_t* __restrict__ rows_out,
    uint32_t* __restrict__ cols_out, const BucketHeader* hdr)
{
    constexpr int IPT = kItemsPerTile / kThreads;          // items per thread
    __shared__ uint32_t toff[kMaxGroups + 1];
    __shared__ uint32_t base[kMaxGroups];
    __shared__ uint32_t first_row[kMaxGroups];
    __shared__ uint32_t srow[2 * kItemsPerTile], scol[2 * kItemsPerTile];
    __shared__ uint32_t sc[2 * kWaves + 1];
    __shared__ uint16_t coarse[kMaxBins / 16];
    if (hdr->bad_id || hdr->internal) return;
    const int64_t i0 = (int64_t)blockIdx.x * kItemsPerTile + threadIdx.x;
    Items<IPT> it;
    it.load(i0, n_items, n_pairs, src, dst);
    const int G = (int)hdr->n_groups;
    const bool one_word = hdr->one_word != 0;
    for (int i = threadIdx.x; i <= G; i += kThreads) toff[i] = 0u;
    if ((int)threadIdx.x < G) first_row[threadIdx.x] = group_bin0[threadIdx.x] << s;
    for (int c = threadIdx.x; c < kMaxBins / 16; c += kThreads) coarse[c] = coarse_group[c];
    __syncthreads();
    // the group of a bin: that of its block's first bin, or the next one from the recorded offset on
    auto group_of = [&](uint32_t bin) {
        const uint32_t e = coarse[bin >> 4];
        return (int)((e & 0x3ffu) + ((bin & 15u) >= (e >> 10) ? 1u : 0u));
    };

    // slot 2k / 2k+1: the entries of the thread's k-th item; group kNone marks an unused slot
    constexpr uint32_t kNone = 0xffffffffu;
    uint32_t er[2 * IPT], ec[2 * IPT], erank[2 * IPT], eg[2 * IPT];
    bool bad = false;
    it.look(i0, n_items, n_pairs, N, bad);
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
        er[2 * k] = ec[2 * k + 1] = it.u[k];
        ec[2 * k] = er[2 * k + 1] = it.v[k];
        eg[2 * k] = eg[2 * k + 1] = kNone;
        erank[2 * k] = erank[2 * k + 1] = 0u;
        if (it.first(k)) {
            const int g = group_of(it.u[k] >> s);
            eg[2 * k] = (uint32_t)g;
            erank[2 * k] = atomicAdd(&toff[g], 1u);
        }
        if (it.second(k)) {
            const int g = group_of(it.v[k] >> s);
            eg[2 * k + 1] = (uint32_t)g;
            erank[2 * k + 1] = atomicAdd(&toff[g], 1u);
        }
    }
    __syncthreads();
    // counts -> offsets inside the tile; one reservation per group that received something
    const uint32_t mine = (int)threadIdx.x < G ? toff[threadIdx.x] : 0u;
    uint32_t total;
    const uint32_t excl = block_scan_excl<kWaves>(mine, sc, total);
    if ((int)threadIdx.x < G) {
        toff[threadIdx.x] = excl;
        base[threadIdx.x] = mine ? atomicAdd(&group_cursor[threadIdx.x], mine) : 0u;
    }
    if (threadIdx.x == 0) toff[G] = total;
    __syncthreads();
    if (one_word) {
        // a word holds the whole entry; its group (below 1024) goes to the write loop beside it
#pragma unroll
        for (int k = 0; k < 2 * IPT; ++k)
            if (eg[k] != kNone) {
                const uint32_t p = toff[eg[k]] + erank[k];
                srow[p] = (er[k] - first_row[eg[k]]) << cbits | ec[k];
                scol[p] = eg[k];
            }
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < total; j += kThreads) {
            const uint32_t g = scol[j];
            rows_out[base[g] + (j - toff[g])] = srow[j];
        }
        return;
    }
    // ids are below 2^23, so the nine high bits of a staged row and the high bit of a staged column are free:
    // they carry the entry's group (below 1024) to the write loop
#pragma unroll
    for (int k = 0; k < 2 * IPT; ++k)
        if (eg[k] != kNone) {
            const uint32_t p = toff[eg[k]] + erank[k];
            srow[p] = er[k] | ((eg[k] & 0x1ffu) << 23);
            scol[p] = ec[k] | ((eg[k] >> 9) << 23);
        }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < total; j += kThreads) {
        const uint32_t r = srow[j], c = scol[j];
        const uint32_t g = (r >> 23) | ((c >> 23) << 9);
        const uint32_t d = base[g] + (j - toff[g]);
        rows_out[d] = r & 0x7fffffu;
        cols_out[d] = c & 0x7fffffu;
    }
}

// part2: the entries of one tile go to their buckets, packed.  FROM_PAIRS: there is a single group and the
// tile is a tile of input items; otherwise the tile is a piece of one group's (row, col) run.
template <bool FROM_PAIRS>
__global__ __launch_bounds__(kThreads) void part2_kernel(
    int64_t n_pairs, const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t N, int64_t n_items, int s,
    int cbits, const uint32_t* __restrict__ rows_in, const uint32_t* __restrict__ cols_in,
    const uint32_t* __restrict__ group_off, const uint32_t* __restrict__ group_tile0,
    const uint32_t* __restrict__ bucket_bin0, uint32_t* bucket_cursor, uint32_t* __restrict__ packed_out,
    const BucketHeader* hdr)
{
    constexpr int EPT = kTileEntries / kThreads;           // entries per thread
    __shared__ uint32_t bb0[kGroupBuckets + 1];
    __shared__ uint32_t toff[kGroupBuckets + 1];
    __shared__ uint32_t base[kGroupBuckets];
    __shared__ uint32_t stage[kTileEntries];
    __shared__ uint8_t stage_lb[kTileEntries];             // local bucket of each staged entry
    __shared__ uint32_t sc[2 * kWaves + 1];
    if (hdr->bad_id || hdr->internal) return;
    const uint32_t n_buckets = hdr->n_buckets;
    uint32_t g = 0, e_begin = 0, e_end = 0;
    if constexpr (!FROM_PAIRS) {
        if (blockIdx.x >= hdr->part2_tiles) return;
        g = (uint32_t)find_segment(group_tile0, (int)hdr->n_groups, blockIdx.x);
        // groups without entries have no tiles and repeat a tile index: the largest g with tile0[g] <= tile holds it
        e_begin = group_off[g] + (blockIdx.x - group_tile0[g]) * kTileEntries;
        e_end = e_begin + kTileEntries < group_off[g + 1] ? e_begin + kTileEntries : group_off[g + 1];
    }
    const uint32_t first = g * kGroupBuckets;
    const int nb = (int)(first + kGroupBuckets < n_buckets ? kGroupBuckets : n_buckets - first);
    for (int i = threadIdx.x; i <= nb; i += kThreads) { bb0[i] = bucket_bin0[first + i]; toff[i] = 0u; }
    __syncthreads();
    // the group's bins -> local bucket, looked up directly when the group spans few enough bins
    constexpr int kDirect = 4096;
    __shared__ uint8_t bin_lb[kDirect];
    const uint32_t bin_first = bb0[0], bin_span = bb0[nb] - bb0[0];
    const bool direct = bin_span <= (uint32_t)kDirect;
    if (direct) {
        for (uint32_t i = threadIdx.x; i < bin_span; i += kThreads)
            bin_lb[i] = (uint8_t)find_segment(bb0, nb, bin_first + i);
        __syncthreads();
    }

    const bool one_word = hdr->one_word != 0;
    const uint32_t group_row = bin_first << s;
    // slot k: one entry (FROM_PAIRS: slots 2k / 2k+1 are the entries of the thread's k-th item); bucket kNone = unused
    constexpr uint32_t kNone = 0xffffffffu;
    uint32_t ev[EPT], erank[EPT], eb[EPT];
    auto take = [&](uint32_t r, uint32_t c, uint32_t& v, uint32_t& lb_out, uint32_t& rank) {
        const int lb = direct ? (int)bin_lb[(r >> s) - bin_first] : find_segment(bb0, nb, r >> s);
        v = ((r - (bb0[lb] << s)) << cbits) | c;
        lb_out = (uint32_t)lb;
        rank = atomicAdd(&toff[lb], 1u);
    };
#pragma unroll
    for (int k = 0; k < EPT; ++k) { ev[k] = 0u; erank[k] = 0u; eb[k] = kNone; }
    if constexpr (FROM_PAIRS) {
        const int64_t i0 = (int64_t)blockIdx.x * kItemsPerTile + threadIdx.x;
        bool bad = false;
        Items<EPT / 2> it;
        it.load(i0, n_items, n_pairs, src, dst);
        it.look(i0, n_items, n_pairs, N, bad);
#pragma unroll
        for (int k = 0; k < EPT / 2; ++k) {
            if (it.first(k)) take(it.u[k], it.v[k], ev[2 * k], eb[2 * k], erank[2 * k]);
            if (it.second(k)) take(it.v[k], it.u[k], ev[2 * k + 1], eb[2 * k + 1], erank[2 * k + 1]);
        }
    } else {
        uint32_t w[EPT], c[EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const uint32_t e = e_begin + k * kThreads + threadIdx.x;
            w[k] = e < e_end ? rows_in[e] : 0u;
            c[k] = !one_word && e < e_end ? cols_in[e] : 0u;
        }
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            if (e_begin + k * kThreads + threadIdx.x >= e_end) continue;
            if (one_word) take(group_row + (w[k] >> cbits), w[k] & ((1u << cbits) - 1u), ev[k], eb[k], erank[k]);
            else take(w[k], c[k], ev[k], eb[k], erank[k]);
        }
    }
    __syncthreads();
    const uint32_t mine = (int)threadIdx.x < nb ? toff[threadIdx.x] : 0u;
    uint32_t total;
    const uint32_t excl = block_scan_excl<kWaves>(mine, sc, total);
    if ((int)threadIdx.x < nb) {
        toff[threadIdx.x] = excl;
        base[threadIdx.x] = mine ? atomicAdd(&bucket_cursor[first + threadIdx.x], mine) : 0u;
    }
    if (threadIdx.x == 0) toff[nb] = total;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < EPT; ++k)
        if (eb[k] != kNone) {
            const uint32_t p = toff[eb[k]] + erank[k];
            stage[p] = ev[k];
            stage_lb[p] = (uint8_t)eb[k];
        }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < total; j += kThreads) {
        const uint32_t lb = stage_lb[j];
        packed_out[base[lb] + (j - toff[lb])] = stage[j];
    }
}

// ---------------------------------------------------------------------------
// sort: LDS state of one bucket
constexpr int kSortThreads = 1024;       // threads of the sort kernel (512 with twice the keys per thread measured 15 % slower)
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortKeys = kBucketMax / kSortThreads;     // keys per thread
constexpr uint32_t kMerged = 255u;       // "bits" of a key range that was put together from small pieces (never split)
constexpr int kBinWords = kSortBins / 2 + 1;             // two 16-bit counters per word, one past the last
constexpr int kMapBits = 19;             // bits of the map that a dense oversized bucket is marked in at a time
typedef uint16_t __attribute__((may_alias)) half_t;
struct SortShared {
    union {
        struct {
            uint32_t keys[kBucketMax + 4];   // (the rank loop looks at four keys at a time)
            uint32_t bins[kBinWords];
            uint32_t rowmeta[kRowSpan];      // entries of a row in the keys being sorted, then: its first bin | column shift << 16
        };
        uint32_t map[(1 << kMapBits) / 32];
    };
    uint32_t rowcnt[kRowSpan];           // entries kept per row so far
    uint32_t stk_lo[kStack], stk_hi[kStack], stk_bits[kStack], stk_cnt[kStack];
    uint32_t sc[2 * kSortWaves + 1];
    uint32_t kept[kSortKeys * kSortWaves];
    uint32_t n, sp;
};
static_assert(sizeof(SortShared) <= 81920, "two workgroups per CU");
static_assert(kRowSpan <= kSortThreads, "one row per thread");

// Sort the n <= kBucketMax keys load(0 .. n), drop repeats, append the columns to out[out_cursor ...) and add
// the kept entries to the per-row counts.  Returns the number of kept keys (uniform over the workgroup).
// On entry all threads have passed a barrier after the last write to `sh`; on return its keys are free.
//
// Bound by LDS operations (some fifteen per key) and the barriers between the phases, not by bytes.  A row of c
// entries gets 2^lg column bins, c/2 to c of them, so that a bin holds one or two keys when the columns are spread evenly and
// a key's rank inside its bin takes one look at four neighbours; two 16-bit counters share a word, which is what lets two
// workgroups fit a CU.  The keys come straight from memory into registers, and go straight out: repeats are left
// out by ballots over the sorted order.
// Reddit-shaped graph (16,000 buckets of 7,168, and the oversized ones below): 1,285 us with bins of four to eight keys,
// staged and compacted in LDS by a function of its own whose saved registers went through memory; now 820 (850 with bins
// of two to four).
template <typename Load>
__device__ __forceinline__ uint32_t sort_keys(SortShared& sh, Load load, uint32_t n, int nrows, int cbits,
                                              uint32_t* __restrict__ out, uint32_t out_cursor)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t cmask = (1u << cbits) - 1u;
    const half_t* bin_at = reinterpret_cast<const half_t*>(sh.bins);
    uint32_t k[kSortKeys];
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j) {                      // all in flight before the first is used
        const uint32_t i = tid + j * kSortThreads;
        k[j] = i < n ? load(i) : 0u;
    }
    // a row has at most max(1, its entries) bins
    const uint32_t words = (n + (uint32_t)nrows) / 2 + 1;
    for (uint32_t i = tid; i < words; i += kSortThreads) sh.bins[i] = 0u;
    if (tid < nrows) sh.rowmeta[tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j) {                      // (lds_count needs whole waves)
        if ((uint32_t)(j * kSortThreads) >= n) break;
        lds_count(sh.rowmeta, k[j] >> cbits, tid + j * kSortThreads < n);
    }
    __syncthreads();
    {
        uint32_t c = 0, lg = 0, nsub = 0;
        if (tid < nrows) {
            c = sh.rowmeta[tid];
            lg = c <= 2u ? 0u : (uint32_t)(32 - __clz(c - 1u)) - 1u;
            lg = lg > (uint32_t)cbits ? (uint32_t)cbits : lg;
            nsub = 1u << lg;
        }
        uint32_t nbins_total;                                  // <= n + nrows
        const uint32_t first = block_scan_excl<kSortWaves>(nsub, sh.sc, nbins_total);
        if (tid < nrows) {
            sh.rowmeta[tid] = first | (((uint32_t)cbits - lg) << 16);
            sh.rowcnt[tid] += c;                               // the repeats among them are taken off below
        }
    }
    __syncthreads();
    // counting split; the atomic's old value is the rank inside the bin
    auto bin_of = [&](uint32_t key) {
        const uint32_t meta = sh.rowmeta[key >> cbits];
        return (meta & 0xffffu) + ((key & cmask) >> (meta >> 16));
    };
    uint32_t at[kSortKeys];                                    // bin | rank inside it << 16
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j) {
        if (tid + j * kSortThreads < n) {
            const uint32_t b = bin_of(k[j]), shift = (b & 1u) * 16u;
            at[j] = b | ((atomicAdd(&sh.bins[b >> 1], 1u << shift) >> shift) << 16);
        }
    }
    __syncthreads();
    {
        constexpr int WPT = (kBinWords + kSortThreads - 1) / kSortThreads;
        const uint32_t per = (words + kSortThreads - 1) / kSortThreads, w0 = tid * per;
        uint32_t c[WPT], sum = 0;
#pragma unroll
        for (int j = 0; j < WPT; ++j) {
            c[j] = (uint32_t)j < per && w0 + j < words ? sh.bins[w0 + j] : 0u;
            sum += (c[j] & 0xffffu) + (c[j] >> 16);
        }
        uint32_t total;
        uint32_t o = block_scan_excl<kSortWaves>(sum, sh.sc, total);
#pragma unroll
        for (int j = 0; j < WPT; ++j) {
            const uint32_t mid = o + (c[j] & 0xffffu);
            if ((uint32_t)j < per && w0 + j < words) sh.bins[w0 + j] = o | (mid << 16);
            o = mid + (c[j] >> 16);
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j)
        if (tid + j * kSortThreads < n) sh.keys[bin_at[at[j] & 0xffffu] + (at[j] >> 16)] = k[j];
    __syncthreads();
    // rank inside the bin by comparison; equal keys keep their order of position
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j) {
        const uint32_t p = tid + j * kSortThreads;
        if (p < n) {
            const uint32_t key = sh.keys[p];
            const uint32_t d = bin_of(key);
            const uint32_t q0 = bin_at[d], q1 = bin_at[d + 1];
            uint32_t below = 0;
            for (uint32_t q = q0; q < q1; q += 4) {          // four independent reads per step (the array is padded)
                const uint32_t o0 = sh.keys[q], o1 = sh.keys[q + 1], o2 = sh.keys[q + 2], o3 = sh.keys[q + 3];
                below += (o0 < key || (o0 == key && q < p)) ? 1u : 0u;
                below += (q + 1 < q1 && (o1 < key || (o1 == key && q + 1 < p))) ? 1u : 0u;
                below += (q + 2 < q1 && (o2 < key || (o2 == key && q + 2 < p))) ? 1u : 0u;
                below += (q + 3 < q1 && (o3 < key || (o3 == key && q + 3 < p))) ? 1u : 0u;
            }
            k[j] = key;
            at[j] = q0 + below;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j)
        if (tid + j * kSortThreads < n) sh.keys[at[j]] = k[j];
    __syncthreads();
    // keep the first key of every run of equal keys; the pieces of 64 that the waves look at are numbered in key order
    uint32_t keep = 0, before[kSortKeys];
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j) {
        const uint32_t i = tid + j * kSortThreads;
        const bool have = i < n;
        k[j] = have ? sh.keys[i] : 0u;
        const bool first = have && (i == 0 || sh.keys[i - 1] != k[j]);
        const uint64_t m = __ballot(first);
        before[j] = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        keep |= first ? 1u << j : 0u;
        if (lane == 0) sh.kept[j * kSortWaves + wave] = (uint32_t)__popcll(m);
        lds_count(sh.rowcnt, k[j] >> cbits, have && !first, (uint32_t)-1);
    }
    __syncthreads();
    // every wave adds up all pieces' counts: three per lane
    constexpr int PIECES = kSortKeys * kSortWaves, PPL = (PIECES + 63) / 64;
    uint32_t c[PPL], sum = 0;
#pragma unroll
    for (int t = 0; t < PPL; ++t) {
        c[t] = lane * PPL + t < PIECES ? sh.kept[lane * PPL + t] : 0u;
        sum += c[t];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    uint32_t lead[PPL];                                        // kept keys before each of the lane's pieces
    lead[0] = incl - sum;
#pragma unroll
    for (int t = 1; t < PPL; ++t) lead[t] = lead[t - 1] + c[t - 1];
#pragma unroll
    for (int j = 0; j < kSortKeys; ++j) {
        const int piece = j * kSortWaves + wave, from = piece / PPL, which = piece % PPL;      // (uniform)
        uint32_t base = lead[0];
#pragma unroll
        for (int t = 1; t < PPL; ++t) base = which == t ? lead[t] : base;
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, from);
        if (keep & (1u << j)) out[out_cursor + base + before[j]] = k[j] & cmask;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    __syncthreads();
    return total;
}

// A bucket that does not fit, i.e. one bin whose rows alone hold more.
//
// Dense ones are marked in a map of 2^19 bits at a time, which drops the repeats and puts the rest in order by itself;
// every stretch of the map reads all entries again (from L2).  The others are worked through in key ranges [lo, hi], lowest first: a range that fits is gathered and sorted; one
// that does not is an aligned block of 2^bits keys, which is counted in 64 pieces by its next key bits; neighbouring
// pieces are put together into ranges that fit, and a piece that still does not fit is split again (or is a single
// repeated key).  Each level removes 6 key bits, so the stack stays below kStack.
// Out of line: its registers and the sort's copy in it are then no concern of the buckets that fit.
// Reddit-shaped graph, 667 such buckets of eight rows: the sort kernel 1,024 us with key ranges alone, 820 with the map.
//
// Key ranges read all entries for every range too, some E / 8,000 of them beside their sorts, so the line is a number of
// stretches in proportion to E: up to one per kStretchEntries.  Whole constructions in us, map and key ranges: 4 stretches of
// 12,000 entries (200 such buckets) 282 and 285, of 40,000 458 and 643; 16 of 17,000 508 and 330, of 40,000 686 and 635, of
// 65,000 (100) 676 and 819; 64 of 66,000 (100) 1,724 and 854, of 130,000 (50) 2,151 and 1,939, of 260,000 (20) 2,423 and 4,854;
// 256 of 270,000 (20) 11,263 and 5,003, of a million (two) 22,400 and 58,200; 1,024 of a million (two) 102,000 and 75,200,
// of four million (one) 370,000 and 727,000; 4,096 of 4.3 million (one) 1,610,000 and 914,000.
constexpr uint32_t kStretchEntries = kBucketMax / 4;
__device__ __noinline__ uint32_t sort_oversized(SortShared& sh, BucketHeader* hdr, const uint32_t* __restrict__ in, uint32_t E,
                                                int nrows, int cbits, uint32_t* __restrict__ out)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t out_cursor = 0;
    // the bits that the bucket's keys really use (its rows, then the columns)
    const uint32_t kb = (uint32_t)cbits + (nrows > 1 ? 32u - (uint32_t)__clz((uint32_t)(nrows - 1)) : 0u);
    const uint32_t stretches = kb > (uint32_t)kMapBits ? 1u << (kb - kMapBits) : 1u;
    if (cbits >= 5 && E / kStretchEntries >= stretches) {
        constexpr uint32_t WORDS = (1u << kMapBits) / 32, PER_WAVE = WORDS / kSortWaves;
        uint32_t* map = sh.map;                              // (over the keys, bins and rowmeta)
        constexpr int AHEAD = 8;
        for (uint32_t st = 0; st < stretches; ++st) {
            for (uint32_t i = tid; i < WORDS; i += kSortThreads) map[i] = 0u;
            __syncthreads();
            for (uint32_t i0 = tid; i0 < E; i0 += AHEAD * kSortThreads) {
                uint32_t key[AHEAD];
#pragma unroll
                for (int t = 0; t < AHEAD; ++t) {
                    const uint32_t i = i0 + t * kSortThreads;
                    key[t] = i < E ? in[i] : 0xffffffffu;
                }
#pragma unroll
                for (int t = 0; t < AHEAD; ++t)
                    if (i0 + t * kSortThreads < E && key[t] >> kMapBits == st)
                        atomicOr(&map[(key[t] & ((1u << kMapBits) - 1u)) >> 5], 1u << (key[t] & 31u));
            }
            __syncthreads();
            // a wave's words are consecutive; 64 of them at a time, one per lane
            uint32_t mine = 0;
            for (uint32_t w = lane; w < PER_WAVE; w += 64) mine += (uint32_t)__popc(map[wave * PER_WAVE + w]);
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
            if (lane == 0) sh.sc[wave] = mine;
            __syncthreads();
            uint32_t at = out_cursor, all = 0;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = sh.sc[w];
                at += w < wave ? c : 0u;
                all += c;
            }
            for (uint32_t w0 = 0; w0 < PER_WAVE; w0 += 64) {
                const uint32_t word = wave * PER_WAVE + w0 + lane;
                uint32_t bits = map[word];
                const uint32_t c = (uint32_t)__popc(bits);
                const uint32_t key0 = (st << kMapBits) + (word << 5);
                uint32_t incl = c;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const uint32_t t = __shfl_up(incl, d, 64);
                    if (lane >= d) incl += t;
                }
                const uint32_t step = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                if (cbits >= 11) {                           // the 2,048 keys of a step are of one row
                    if (lane == 0 && step) atomicAdd(&sh.rowcnt[key0 >> cbits], step);
                } else if (c) {
                    atomicAdd(&sh.rowcnt[key0 >> cbits], c);
                }
                for (uint32_t o = at + incl - c; bits; ++o, bits &= bits - 1u)
                    out[o] = (key0 + (uint32_t)__builtin_ctz(bits)) & ((1u << cbits) - 1u);
                at += step;
            }
            out_cursor += all;
            __syncthreads();
        }
        return out_cursor;
    }
    if (tid == 0) {
        sh.stk_lo[0] = 0u;
        sh.stk_hi[0] = kb >= 32u ? 0xffffffffu : (1u << kb) - 1u;
        sh.stk_bits[0] = kb >= 32u ? 32u : kb;
        sh.stk_cnt[0] = E;
        sh.sp = 1u;
    }
    __syncthreads();
    for (;;) {
        const uint32_t sp = sh.sp;
        if (sp == 0) break;
        const uint32_t lo = sh.stk_lo[sp - 1], hi = sh.stk_hi[sp - 1], bits = sh.stk_bits[sp - 1],
                       cnt = sh.stk_cnt[sp - 1];
        __syncthreads();
        if (tid == 0) { sh.sp = sp - 1; sh.n = 0u; }
        __syncthreads();
        if (cnt > (uint32_t)kBucketMax && bits == 0u) {
            // more than a bucketful of one and the same key: it is kept once
            if (tid == 0) {
                out[out_cursor] = lo & ((1u << cbits) - 1u);
                atomicAdd(&sh.rowcnt[lo >> cbits], 1u);
            }
            out_cursor += 1;
            __syncthreads();
            continue;
        }
        if (cnt > (uint32_t)kBucketMax) {
            const uint32_t cb = bits > 6u ? bits - 6u : 0u;
            const int nchild = 1 << (bits - cb);
            if (tid < 64) sh.bins[tid] = 0u;
            __syncthreads();
            for (uint32_t i0 = (uint32_t)(tid - lane); i0 < E; i0 += kSortThreads) {  // uniform per wave
                const uint32_t i = i0 + lane;
                const uint32_t key = i < E ? in[i] : 0u;
                const bool match = i < E && key >= lo && key <= hi;
                lds_count(sh.bins, match ? (key - lo) >> cb : 0u, match);
            }
            __syncthreads();
            if (tid == 0) {
                // highest keys first, so that the lowest range is on top of the stack
                uint32_t top = sh.sp;
                auto push = [&](int c0, int c1, uint32_t b_, uint32_t n_) {      // pieces c0..c1
                    if (top >= (uint32_t)kStack) { hdr->internal = 1u; return; }  // cannot happen (6 levels x 64)
                    sh.stk_lo[top] = lo + ((uint32_t)c0 << cb);
                    sh.stk_hi[top] = c1 == nchild - 1 ? hi : lo + ((uint32_t)(c1 + 1) << cb) - 1u;
                    sh.stk_bits[top] = b_;
                    sh.stk_cnt[top] = n_;
                    ++top;
                };
                int ch = nchild - 1;
                while (ch >= 0) {
                    if (sh.bins[ch] > (uint32_t)kBucketMax) { push(ch, ch, cb, sh.bins[ch]); --ch; continue; }
                    const int c1 = ch;
                    uint32_t sum = 0;
                    while (ch >= 0 && sum + sh.bins[ch] <= (uint32_t)kBucketMax) { sum += sh.bins[ch]; --ch; }
                    if (sum) push(ch + 1, c1, kMerged, sum);
                }
                sh.sp = top;
            }
            __syncthreads();
            continue;
        }
        // the range fits: gather its keys
        for (uint32_t i0 = (uint32_t)(tid - lane); i0 < E; i0 += kSortThreads) {      // uniform per wave
            const uint32_t i = i0 + lane;
            const uint32_t key = i < E ? in[i] : 0u;
            const bool match = i < E && key >= lo && key <= hi;
            const uint64_t mask = __ballot(match);
            if (mask) {
                const int leader = __ffsll((unsigned long long)mask) - 1;
                uint32_t at = 0;
                if (lane == leader) at = atomicAdd(&sh.n, (uint32_t)__popcll(mask));
                at = __shfl(at, leader, 64);
                if (match) sh.keys[at + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull))] = key;
            }
        }
        __syncthreads();
        const uint32_t n = sh.n;                               // == cnt
        out_cursor += sort_keys(sh, [&](uint32_t i) { return sh.keys[i]; }, n, nrows, cbits, out, out_cursor);
    }
    return out_cursor;
}

__global__ __launch_bounds__(kSortThreads, 8) void sort_kernel(
    BucketHeader* hdr, const uint32_t* __restrict__ bucket_off, const uint32_t* __restrict__ bucket_bin0,
    const uint32_t* __restrict__ packed, uint32_t* __restrict__ cols_tmp, int32_t* __restrict__ row_unique,
    uint32_t* __restrict__ bucket_total, int cbits, int s, int64_t N)
{
    __shared__ SortShared sh;
    if (hdr->bad_id || hdr->internal) return;
    const uint32_t b = blockIdx.x;
    if (b >= hdr->n_buckets) return;
    const int tid = threadIdx.x;
    const uint32_t e0 = bucket_off[b], E = bucket_off[b + 1] - e0;
    const int64_t row0 = (int64_t)bucket_bin0[b] << s;
    int64_t row1 = (int64_t)bucket_bin0[b + 1] << s;
    row1 = row1 < N ? row1 : N;
    const int nrows = (int)(row1 - row0);                    // <= kRowSpan
    if (tid < nrows) sh.rowcnt[tid] = 0u;
    const uint32_t* in = packed + e0;
    uint32_t* out = cols_tmp + e0;
    uint32_t kept = 0;
    __syncthreads();
    if (E > (uint32_t)kBucketMax) kept = sort_oversized(sh, hdr, in, E, nrows, cbits, out);
    else if (E > 0) kept = sort_keys(sh, [&](uint32_t i) { return in[i]; }, E, nrows, cbits, out, 0u);
    __syncthreads();
    if (tid < nrows) row_unique[row0 + tid] = (int32_t)sh.rowcnt[tid];
    if (tid == 0) bucket_total[b] = kept;
}

__global__ __launch_bounds__(kThreads) void total_kernel(BucketHeader* hdr, const uint32_t* __restrict__ bucket_total,
                                                         uint32_t* __restrict__ bucket_out, int64_t col_capacity)
{
    __shared__ uint32_t sc[2 * kWaves + 1];
    if (hdr->bad_id || hdr->internal) return;
    const uint32_t n = hdr->n_buckets;
    const uint32_t per = (n + kThreads - 1) / kThreads;
    const uint32_t b0 = threadIdx.x * per < n ? threadIdx.x * per : n;
    const uint32_t b1 = b0 + per < n ? b0 + per : n;
    uint32_t s = 0;
    for (uint32_t b = b0; b < b1; ++b) s += bucket_total[b];
    uint32_t total;
    uint32_t o = block_scan_excl<kWaves>(s, sc, total);
    for (uint32_t b = b0; b < b1; ++b) { bucket_out[b] = o; o += bucket_total[b]; }
    if (threadIdx.x == 0) {
        bucket_out[n] = total;
        hdr->nnz = (int64_t)total;
        hdr->overflow = (int64_t)total > col_capacity ? 1u : 0u;
    }
}

// SUM: few buckets, whose counts every workgroup adds up itself (total's launch took 5 us of a small graph's construction).
template <bool SUM>
__global__ __launch_bounds__(256) void emit_kernel(
    BucketHeader* hdr, const uint32_t* __restrict__ bucket_off, const uint32_t* __restrict__ bucket_bin0,
    const uint32_t* __restrict__ bucket_out, const uint32_t* __restrict__ cols_tmp, const int32_t* __restrict__ row_unique,
    const uint32_t* __restrict__ bucket_total, int64_t col_capacity,
    int s, int64_t N, int64_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx, BucketHeader* report)
{
    constexpr int RPT = kRowSpan / 256;                      // rows per thread
    __shared__ uint32_t sc[2 * 4 + 1];
    const bool reports = report && blockIdx.x == 0 && threadIdx.x == 0;
    if (hdr->bad_id || hdr->internal || (!SUM && hdr->overflow)) {
        if (reports) *report = *hdr;
        return;
    }
    const uint32_t b = blockIdx.x, n = hdr->n_buckets;
    if (b >= n) return;
    uint32_t out0, nnz;
    if constexpr (SUM) {
        uint32_t c[kFewBuckets / 256], before = 0, all = 0;
#pragma unroll
        for (int j = 0; j < kFewBuckets / 256; ++j) {
            const uint32_t i = threadIdx.x + j * 256;
            c[j] = i < n ? bucket_total[i] : 0u;
            before += i < b ? c[j] : 0u;
            all += c[j];
        }
        (void)block_scan_excl<4>(before, sc, out0);
        (void)block_scan_excl<4>(all, sc, nnz);
        if (b == 0 && threadIdx.x == 0) {
            hdr->nnz = (int64_t)nnz;
            hdr->overflow = (int64_t)nnz > col_capacity ? 1u : 0u;
            if (reports) *report = *hdr;
        }
        if ((int64_t)nnz > col_capacity) return;
    } else {
        if (reports) *report = *hdr;
        out0 = bucket_out[b];
        nnz = (uint32_t)hdr->nnz;
    }
    const int64_t row0 = (int64_t)bucket_bin0[b] << s;
    int64_t row1 = (int64_t)bucket_bin0[b + 1] << s;
    row1 = row1 < N ? row1 : N;
    const int nrows = (int)(row1 - row0);
    const uint32_t count = SUM ? bucket_total[b] : bucket_out[b + 1] - out0;
    uint32_t c[RPT], sum = 0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = threadIdx.x * RPT + j;
        c[j] = i < nrows ? (uint32_t)row_unique[row0 + i] : 0u;
        sum += c[j];
    }
    uint32_t total;
    uint32_t o = out0 + block_scan_excl<4>(sum, sc, total);
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = threadIdx.x * RPT + j;
        if (i < nrows) row_ptr[row0 + i] = (int64_t)o;
        o += c[j];
    }
    if (b == n - 1 && threadIdx.x == 0) row_ptr[N] = (int64_t)nnz;
    // sixteen bytes at a time where the destination allows them (the source is at any word)
    const uint32_t* from = cols_tmp + bucket_off[b];
    int32_t* to = col_idx + out0;
    const uint32_t odd = (uint32_t)(-(intptr_t)((uintptr_t)to >> 2) & 3), head = odd < count ? odd : count;
    if (threadIdx.x < head) to[threadIdx.x] = (int32_t)from[threadIdx.x];
    const uint32_t quads = (count - head) / 4;
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    typedef uint32_t words4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll 4
    for (uint32_t q = threadIdx.x; q < quads; q += 256)
        *reinterpret_cast<words4*>(to + head + 4 * q) = *reinterpret_cast<const words4_any*>(from + head + 4 * q);
    const uint32_t tail = head + 4 * quads + threadIdx.x;
    if (tail < count) to[tail] = (int32_t)from[tail];
}

// ---------------------------------------------------------------------------
// Graphs of up to kTinyItems pairs and loops over up to kTinyRows nodes: one workgroup, one launch.  Bound by latencies, not
// work: counting, moving, sorting and emitting in four dependent launches took 31 us of a construction of 42 over 2,708 nodes
// and 5,429 pairs, which takes 32 so.  The lines are what LDS holds; near them 8,049 nodes and 8,021 pairs took 64.2 and 58.9, 1,076
// and 8,025, whose rows are mostly long, 61.2 and 60.8.  Entries are counted per row in LDS, which also says where in its row each goes; a row of up to
// kTinyShort entries is sorted and cleaned in the registers of one thread, a longer one is marked in a bit map of the nodes by a
// wave, which drops its repeats and orders it.
constexpr int kTinyItems = 8192, kTinyRows = 8192;
constexpr int kTinyShort = 16;
constexpr int kTinyLong = 2 * kTinyItems / (kTinyShort + 1) + 1;       // rows that can be longer
struct TinyShared {
    uint32_t row[kTinyRows];                 // entries of a row, then: its start | entries << 16
    uint16_t cols[2 * kTinyItems];
    uint32_t map[kWaves][kTinyRows / 32];
    uint16_t longer[kTinyLong];              // rows that are
    uint32_t sc[2 * kWaves + 1];
    uint32_t n_longer;
};
static_assert(2 * kTinyItems < 1 << 15 && kTinyRows <= 0xffff && sizeof(TinyShared) <= 160 * 1024, "fields and LDS");

// the first W values in ascending order: a bitonic network
template <int W>
__device__ __forceinline__ void sort_registers(uint32_t (&k)[kTinyShort])
{
#pragma unroll
    for (int size = 2; size <= W; size <<= 1)
#pragma unroll
        for (int d = size >> 1; d > 0; d >>= 1)
#pragma unroll
            for (int i = 0; i < W; ++i)
                if ((i & d) == 0) {
                    const uint32_t lo = min(k[i], k[i | d]), hi = max(k[i], k[i | d]);
                    k[i] = (i & size) == 0 ? lo : hi;
                    k[i | d] = (i & size) == 0 ? hi : lo;
                }
}

__global__ __launch_bounds__(kThreads) void tiny_kernel(
    int64_t n_pairs, const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int N, int n_items,
    int64_t col_capacity, int64_t* row_ptr, int32_t* __restrict__ col_idx, BucketHeader* report)
{
    constexpr int IPT = kTinyItems / kThreads;
    __shared__ TinyShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Items<IPT> it;
    it.load(tid, n_items, n_pairs, src, dst);
    for (int r = tid; r < N; r += kThreads) sh.row[r] = 0u;
    if (tid == 0) sh.n_longer = 0u;
    bool bad = false;
    it.look(tid, n_items, n_pairs, N, bad);
    if (__syncthreads_or(bad)) {
        if (tid == 0) {
            BucketHeader h = {};
            h.bad_id = 1u;
            *report = h;
        }
        return;
    }
    uint32_t at[IPT];                        // positions of an item's two entries in their rows
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        at[t] = it.first(t) ? atomicAdd(&sh.row[it.u[t]], 1u) : 0u;
        if (it.second(t)) at[t] |= atomicAdd(&sh.row[it.v[t]], 1u) << 16;
    }
    __syncthreads();
    // the thread's rows in the two scans: all waves have some, and an odd number keeps neighbouring threads on other LDS banks
    const int rows = ((N + kThreads - 1) / kThreads) | 1, r0 = min(tid * rows, N), r1 = min(r0 + rows, N);
    uint32_t sum = 0, total;
    for (int r = r0; r < r1; ++r) sum += sh.row[r];
    uint32_t o = block_scan_excl<kWaves>(sum, sh.sc, total);
    for (int r = r0; r < r1; ++r) {
        const uint32_t c = sh.row[r];
        sh.row[r] = o | c << 16;
        o += c;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        if (it.first(t)) sh.cols[(sh.row[it.u[t]] & 0xffffu) + (at[t] & 0xffffu)] = (uint16_t)it.v[t];
        if (it.second(t)) sh.cols[(sh.row[it.v[t]] & 0xffffu) + (at[t] >> 16)] = (uint16_t)it.u[t];
    }
    __syncthreads();
    for (int r = tid; r < N; r += kThreads) {
        const uint32_t c = sh.row[r] >> 16, s = sh.row[r] & 0xffffu;
        if (c > (uint32_t)kTinyShort) {
            sh.longer[atomicAdd(&sh.n_longer, 1u)] = (uint16_t)r;
            continue;
        }
        if (c < 2u) continue;
        uint32_t k[kTinyShort];
#pragma unroll
        for (int i = 0; i < kTinyShort; ++i) k[i] = (uint32_t)i < c ? sh.cols[s + i] : 0xffffffffu;
        if (c <= 4u) sort_registers<4>(k);
        else if (c <= 8u) sort_registers<8>(k);
        else sort_registers<kTinyShort>(k);
        uint32_t kept = 0;
#pragma unroll
        for (int i = 0; i < kTinyShort; ++i)
            if ((uint32_t)i < c && (i == 0 || k[i] != k[i > 0 ? i - 1 : 0])) sh.cols[s + kept++] = (uint16_t)k[i];
        sh.row[r] = s | kept << 16;
    }
    __syncthreads();
    const int n_longer = (int)sh.n_longer, words = (N + 31) / 32;
    uint32_t* map = sh.map[wave];
    for (int i = wave; i < n_longer; i += kWaves) {           // (a wave's own rows and map: LDS operations keep their order)
        const uint32_t r = sh.longer[i], c = sh.row[r] >> 16, s = sh.row[r] & 0xffffu;
        for (int w = lane; w < words; w += 64) map[w] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t e = lane; e < c; e += 64) {
            const uint32_t v = sh.cols[s + e];
            atomicOr(&map[v >> 5], 1u << (v & 31u));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32_t kept = 0;
        for (int w0 = 0; w0 < words; w0 += 64) {
            uint32_t bits = w0 + lane < words ? map[w0 + lane] : 0u;
            const uint32_t mine = (uint32_t)__popc(bits);
            uint32_t incl = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t t = __shfl_up(incl, d, 64);
                if (lane >= d) incl += t;
            }
            for (uint32_t p = s + kept + incl - mine; bits; ++p, bits &= bits - 1u)
                sh.cols[p] = (uint16_t)(((w0 + lane) << 5) + __builtin_ctz(bits));
            kept += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        if (lane == 0) sh.row[r] = s | kept << 16;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    sum = 0;
    for (int r = r0; r < r1; ++r) sum += sh.row[r] >> 16;
    o = block_scan_excl<kWaves>(sum, sh.sc, total);
    const bool over = (int64_t)total > col_capacity;          // (uniform)
    if (tid == 0) {
        BucketHeader h = {};
        h.nnz = (int64_t)total;
        h.overflow = over ? 1u : 0u;
        *report = h;
        if (!over) row_ptr[N] = (int64_t)total;
    }
    if (over) return;
    for (int r = r0; r < r1; ++r) {
        const uint32_t c = sh.row[r] >> 16, s = sh.row[r] & 0xffffu;
        row_ptr[r] = (int64_t)o;
        if (c <= (uint32_t)kTinyShort)
            for (uint32_t e = 0; e < c; ++e) col_idx[o + e] = (int32_t)sh.cols[s + e];
        o += c;
    }
    __syncthreads();                                          // (row_ptr is written)
    for (int i = wave; i < n_longer; i += kWaves) {
        const uint32_t r = sh.longer[i], c = sh.row[r] >> 16, s = sh.row[r] & 0xffffu;
        if (c <= (uint32_t)kTinyShort) continue;
        int32_t* to = col_idx + row_ptr[r];
        for (uint32_t e = lane; e < c; e += 64) to[e] = (int32_t)sh.cols[s + e];
    }
}

int column_bits(int64_t N)
{
    int b = 1;
    while ((1ll << b) < N) ++b;
    return b;
}

static_assert(sizeof(BucketHeader) <= 256, "the header has 256 bytes of the workspace");

struct BucketLayout {
    int cbits, s, nbins, span_bins, target, hist_blocks;
    int64_t M, n_items, items_per_block, bucket_bound;
    bool two_level, small;
    int64_t header, counts, bin_count, bucket_bin0, bucket_off, bucket_cursor, bucket_total, bucket_out,
        group_bin0, group_off, group_cursor, group_tile0, coarse_group, buf_a, buf_b, buf_c, row_unique, total;
};

bool make_bucket_layout(int64_t n_pairs, int64_t N, int add_self_loops, BucketLayout& L)
{
    if (N < 1) return false;
    L.cbits = column_bits(N);
    if (L.cbits > 23) return false;                          // rows of a bucket must pack into 32 - cbits bits
    L.M = 2 * n_pairs + (add_self_loops ? N : 0);
    if (L.M > kMaxEntries) return false;
    L.n_items = n_pairs + (add_self_loops ? N : 0);
    // The sort of a bucket costs much the same half full as full (twenty barriers, its scans), so a large graph's are
    // filled to 0.7 of what fits: 57.5 million pairs over 233 thousand nodes 1410 us at half, 1315 at 0.7, 1360 at 0.8 (when
    // several bins could still overfill a bucket; 1290 at 0.7 since); whole constructions of 30 to 50 million pairs gain 8
    // to 10 %.  A small graph would then
    // leave CUs idle and wait for a full bucket's sort, so it is spread over kTargetBuckets first (as many as keep the
    // bound of a graph of 0.4 million entries within one group): 3 to 5 % from 7 thousand to 5 million entries.
    const int64_t spread = L.M / kTargetBuckets;
    L.target = spread > kTargetMax ? kTargetMax : spread < kTargetMin ? kTargetMin : (int)spread;
    // Row ranges ("bins") of 2^s rows: at most kMaxBins, or kSmallBins of a graph that one workgroup counts and plans, up to
    // where its counting takes as long as the launches that it saves.
    auto bins = [&](int most_bits) {
        L.s = L.cbits > most_bits ? L.cbits - most_bits : 0;
        L.nbins = (int)((N + (1ll << L.s) - 1) >> L.s);
        const int64_t span_rows = (1ll << (32 - L.cbits)) < kRowSpan ? (1ll << (32 - L.cbits)) : kRowSpan;
        L.span_bins = (int)(span_rows >> L.s);
        // worst case of starts_bucket: one start per window, one more for a bin that reaches over the end of its window (at
        // most one in each, of more than kBucketMax - 1 - target entries), one per row window
        const int64_t windows = L.M / L.target, reach = L.M / (kBucketMax - 1 - L.target);
        if (L.span_bins >= 1) L.bucket_bound = windows + (windows < reach ? windows : reach) + L.nbins / L.span_bins + 4;
        return L.span_bins >= 1;
    };
    static_assert(kMaxBins == 1 << 15 && kSmallBins == 1 << 12, "bits of the bins");
    L.small = L.n_items <= kSmallItems && bins(12) && L.bucket_bound <= kGroupBuckets;
    if (!L.small && (!bins(15) || L.nbins > kMaxBins)) return false;
    if (L.bucket_bound > kMaxBuckets) return false;
    L.two_level = L.bucket_bound > kGroupBuckets;
    int64_t hb = (L.n_items + 16383) / 16384;
    L.hist_blocks = (int)(hb < 1 ? 1 : hb > kMaxHistBlocks ? kMaxHistBlocks : hb);
    L.items_per_block = align_up((L.n_items + L.hist_blocks - 1) / L.hist_blocks, kThreads);
    if (L.items_per_block < kThreads) L.items_per_block = kThreads;
    int64_t off = 0;
    auto take = [&](int64_t bytes) { const int64_t at = off; off += align_up(bytes > 0 ? bytes : 4, 256); return at; };
    const int64_t m = L.M > 0 ? L.M : 1;
    L.header = take(256);
    L.bin_count = take(4ll * L.nbins);                       // (zeroed together with the header)
    L.counts = take(4ll * L.hist_blocks * L.nbins);
    L.bucket_bin0 = take(4 * (L.bucket_bound + 1));
    L.bucket_off = take(4 * (L.bucket_bound + 1));
    L.bucket_cursor = take(4 * L.bucket_bound);
    L.bucket_total = take(4 * L.bucket_bound);
    L.bucket_out = take(4 * (L.bucket_bound + 1));
    L.group_bin0 = take(4 * (kMaxGroups + 1));
    L.group_off = take(4 * (kMaxGroups + 1));
    L.group_cursor = take(4 * kMaxGroups);
    L.group_tile0 = take(4 * (kMaxGroups + 1));
    L.coarse_group = take(2 * (kMaxBins / 16));
    L.buf_a = take(4 * m);                                   // part1: rows; later the sorted columns of the buckets
    L.buf_b = L.two_level ? take(4 * m) : off;               // part1: columns
    L.buf_c = take(4 * m);                                   // part2: packed entries
    L.row_unique = take(4 * N);
    L.total = off + 256;
    return true;
}

}  // namespace

int64_t csr_bucketed_workspace_bytes(int64_t n_pairs, int64_t N, int add_self_loops)
{
    BucketLayout L;
    if (!make_bucket_layout(n_pairs, N, add_self_loops, L)) return -1;
    return L.total;
}

int csr_build_bucketed(int64_t n_pairs, const int32_t* d_src, const int32_t* d_dst, int64_t N, int add_self_loops,
                       int64_t* d_row_ptr, int32_t* d_col_idx, int64_t col_capacity, int64_t* h_nnz,
                       void* d_workspace, hipStream_t stream)
{
    BucketLayout L;
    if (!make_bucket_layout(n_pairs, N, add_self_loops, L)) return RETEXO_E_SIZE;
    char* ws = (char*)d_workspace;
    BucketHeader* hdr = (BucketHeader*)(ws + L.header);
    auto u32 = [&](int64_t at) { return (uint32_t*)(ws + at); };
    PlanArrays pa{u32(L.bucket_bin0), u32(L.bucket_off), u32(L.bucket_cursor),
                  u32(L.group_bin0), u32(L.group_off), u32(L.group_cursor), u32(L.group_tile0),
                  (uint16_t*)(ws + L.coarse_group)};

    HostReport report(stream);
    static_assert(sizeof(BucketHeader) <= kReportBytes, "a report holds it");
    auto finish = [&]() -> int {
        RETEXO_HIP_TRY(hipGetLastError());
        BucketHeader h;
        if (!report.get()) RETEXO_HIP_TRY(hipMemcpyAsync(&h, hdr, sizeof(h), hipMemcpyDeviceToHost, stream));
        RETEXO_HIP_TRY(report.wait());
        if (report.get()) memcpy(&h, report.get(), sizeof(h));
        if (h.bad_id) return RETEXO_E_CSR;
        if (h.internal) return RETEXO_E_HIP;
        if (h_nnz) *h_nnz = h.nnz;
        if (h.overflow) return RETEXO_E_CAPACITY;
        return RETEXO_OK;
    };
    if (L.n_items <= kTinyItems && N <= kTinyRows) {
        tiny_kernel<<<dim3(1), dim3(kThreads), 0, stream>>>(n_pairs, d_src, d_dst, (int)N, (int)L.n_items, col_capacity, d_row_ptr,
                                                            d_col_idx, report.get() ? (BucketHeader*)report.get() : hdr);
        return finish();
    }
    auto plan = [&](auto count) {
        plan_kernel<decltype(count)::value><<<dim3(1), dim3(kThreads), 0, stream>>>(
            L.nbins, L.span_bins, (int)((1ll << (32 - L.cbits)) >> L.s), (uint32_t)L.target,
            (uint32_t)((1ull << 32) / (uint64_t)L.target), u32(L.bin_count), n_pairs, d_src, d_dst, N, L.n_items, L.s, pa,
            (uint32_t)L.bucket_bound, hdr);
    };
    if (L.small) {
        plan(std::true_type{});
    } else {
        if (int e = launch_zero(hdr, (size_t)(L.counts - L.header), stream)) return e;      // header and bin counts
        hist_kernel<<<dim3((unsigned)L.hist_blocks), dim3(kThreads), 0, stream>>>(
            n_pairs, d_src, d_dst, N, L.n_items, L.items_per_block, L.s, L.nbins, u32(L.counts), hdr);
        colsum_kernel<<<dim3((unsigned)((L.nbins + 255) / 256), kColsumSlices), dim3(256), 0, stream>>>(
            L.hist_blocks, L.nbins, u32(L.counts), u32(L.bin_count));
        plan(std::false_type{});
    }
    const unsigned item_tiles = (unsigned)((L.n_items + kItemsPerTile - 1) / kItemsPerTile);
    if (L.M > 0) {
        if (L.two_level) {
            part1_kernel<<<dim3(item_tiles), dim3(kThreads), 0, stream>>>(
                n_pairs, d_src, d_dst, N, L.n_items, L.s, L.cbits, pa.coarse_group, pa.group_bin0, pa.group_cursor, u32(L.buf_a), u32(L.buf_b), hdr);
            const unsigned tiles = (unsigned)((L.M + kTileEntries - 1) / kTileEntries + kMaxGroups);
            part2_kernel<false><<<dim3(tiles), dim3(kThreads), 0, stream>>>(
                n_pairs, d_src, d_dst, N, L.n_items, L.s, L.cbits, u32(L.buf_a), u32(L.buf_b), pa.group_off,
                pa.group_tile0, pa.bucket_bin0, pa.bucket_cursor, u32(L.buf_c), hdr);
        } else {
            part2_kernel<true><<<dim3(item_tiles), dim3(kThreads), 0, stream>>>(
                n_pairs, d_src, d_dst, N, L.n_items, L.s, L.cbits, nullptr, nullptr, pa.group_off,
                pa.group_tile0, pa.bucket_bin0, pa.bucket_cursor, u32(L.buf_c), hdr);
        }
    }
    sort_kernel<<<dim3((unsigned)L.bucket_bound), dim3(kSortThreads), 0, stream>>>(
        hdr, pa.bucket_off, pa.bucket_bin0, u32(L.buf_c), u32(L.buf_a), (int32_t*)(ws + L.row_unique),
        u32(L.bucket_total), L.cbits, L.s, N);
    auto emit = [&](auto sum) {
        emit_kernel<decltype(sum)::value><<<dim3((unsigned)L.bucket_bound), dim3(256), 0, stream>>>(
            hdr, pa.bucket_off, pa.bucket_bin0, u32(L.bucket_out), u32(L.buf_a), (const int32_t*)(ws + L.row_unique),
            u32(L.bucket_total), col_capacity, L.s, N, d_row_ptr, d_col_idx, (BucketHeader*)report.get());
    };
    if (L.bucket_bound <= kFewBuckets) {
        emit(std::true_type{});
    } else {
        total_kernel<<<dim3(1), dim3(kThreads), 0, stream>>>(hdr, u32(L.bucket_total), u32(L.bucket_out), col_capacity);
        emit(std::false_type{});
    }
    return finish();
}
