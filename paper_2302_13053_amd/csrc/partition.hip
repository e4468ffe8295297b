// One worker's share of an edge-partitioned graph, and the pack / unpack of
// boundary rows around a message-passing round.
//
// Section "Edge-partitioned Distributed Setup": worker i holds its inner nodes
// V_i, the edges that touch an inner node and, as boundary nodes, the other
// endpoints of those edges; before a round it receives the boundary nodes'
// current representations from their owners (the embedding exchange of the
// implementation section).  Given the global CSR and a node -> worker map this
// file derives, on the device and with integer arithmetic only:
//
//   local numbering   [ inner nodes, ascending global id | boundary nodes, ascending global id ]
//   local CSR         an inner node's row = its global row renumbered, columns ascending;
//                     a boundary node's row is empty
//   global degrees    of all local nodes (gcn_sym normalises a boundary node by its true degree)
//   send / receive    per peer q: the inner nodes q needs / the boundary nodes q owns, as local
//   lists             ids ascending in global id, so that the list one worker packs and the list
//                     its peer unpacks line up element by element
//
// Both halves of the numbering are monotone in the global id, so a renumbered
// row is its inner entries (ascending) followed by its boundary entries
// (ascending): a stable two-way split inside each row, no per-row sort.  The
// lists are a stable split of the nodes by peer in the same way: blocks of 256
// nodes count their members of every list, a scan over (list, block) places
// them, and every block writes its own.
#include <cstring>
#include <type_traits>

#include <rocprim/device/device_scan.hpp>

#include <string.h>

#include "common.hpp"
#include "report.hpp"

namespace {

constexpr int kThreads = 256;
constexpr int kMaxWorkers = 64;       // one bit per worker in a 64-bit mask

struct ShareHeader {                  // start of the workspace; read by the host
    uint32_t bad_part;                // a partition id outside [0, n_parts)
    uint32_t pad;
    int64_t n_inner, n_halo, nnz_local, n_send;
    int64_t send_off[kMaxWorkers + 1];
    int64_t recv_off[kMaxWorkers + 1];
};

__device__ __forceinline__ uint64_t wave_or(uint64_t x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)x, m, 64), hi = __shfl_xor((uint32_t)(x >> 32), m, 64);
        x |= ((uint64_t)hi << 32) | lo;
    }
    return x;
}

__device__ __forceinline__ uint32_t wave_or(uint32_t x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x |= __shfl_xor(x, m, 64);
    return x;
}

// state of a node while its share is derived: its owner, and whether it was found to be a boundary node
constexpr uint32_t kBoundary = 0x80000000u;
constexpr uint32_t kNobody = 0xffffu;         // (no worker has that id)

// Graphs of up to some hundred thousand nodes keep what is looked up per entry in LDS, one workgroup per CU (mark_lds_kernel,
// columns_lds_kernel): the owners in a power of two of bits each beside one bit per boundary node, and later sixteen bytes per 32
// nodes that give a node's local id.  Gathering a word per entry from L2 instead is bound by the L2 requests, and is what
// larger graphs do (mark_kernel, columns_kernel).
constexpr int kLdsThreads = 1024;
constexpr int kLdsWaves = kLdsThreads / 64;
constexpr int kLdsBlocks = 256;               // one per CU
constexpr int kTableWords = 36864;            // 144 KB
constexpr int kListRows = 2560;               // rows of one workgroup
constexpr int64_t kTableNodes = 32 * (kTableWords / 4);          // 294,912: nodes of columns_lds_kernel
// Smaller graphs are bound by launches and latencies, which one workgroup per CU makes longer: both kernels 11 us over 2,000
// nodes and 20,000 pairs, 6 over 40,000 and 400,000, even at 100,000 nodes and a million pairs.
constexpr int64_t kMarkNodes = 65536;
constexpr int64_t kTableEntries = 1 << 20;    // (the entries are not known before the nodes are marked)
int owner_bits(int n_parts) { return n_parts <= 2 ? 1 : n_parts <= 4 ? 2 : n_parts <= 16 ? 4 : 8; }
bool owners_fit(int64_t N, int n_parts)
{
    const int64_t words = (N * owner_bits(n_parts) + 31) / 32 + (N + 31) / 32;
    return N >= kMarkNodes && words <= kTableWords && (N + kLdsBlocks - 1) / kLdsBlocks <= kListRows;
}

// `bits` != 0: also the owners packed that many bits each (a worker that does not exist as zero, the call then ends in an
// error), and the boundary bits cleared
__global__ __launch_bounds__(kThreads) void state_kernel(int64_t N, const int32_t* __restrict__ part, int n_parts,
                                                         uint32_t* __restrict__ state, int bits, uint32_t* __restrict__ owners,
                                                         uint32_t* __restrict__ boundary, ShareHeader* hdr)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int q = v < N ? part[v] : 0;
    const bool bad = q < 0 || q >= n_parts;
    if (bad) atomicOr(&hdr->bad_part, 1u);
    if (v < N) state[v] = bad ? 0xffffu : (uint32_t)q;       // (no worker has that id; the call ends in an error)
    if (bits) {
        const int per = 32 / bits;                           // nodes per word
        uint32_t w = (bad ? 0u : (uint32_t)q) << ((threadIdx.x % per) * bits);
        for (int m = 1; m < per; m <<= 1) w |= __shfl_xor(w, m, 64);
        if (v < N && threadIdx.x % per == 0) owners[v / per] = w;
        if (v < N && threadIdx.x % 32 == 0) boundary[v / 32] = 0u;
    }
}

// One wave per global row: an inner row marks the foreign endpoints of its entries as boundary nodes, collects the set of
// workers it touches and counts its inner entries (columns_kernel then needs one pass).
// Bound by the gathers of one word per entry, so owner and mark share that word (a node is marked by the first rows that
// meet it, after that the mark is only read: 21 million stores to the Reddit-shaped graph's 0.17 million nodes were most
// of this kernel's time), and four tiles of 64 entries are in flight per wave.  Worker 0 of 4 there: 415 -> 230 us
// (eight in flight: 209, sixteen: 199, but short rows then issue that many empty tiles).
constexpr int kAhead = 4;
__global__ __launch_bounds__(kThreads) void mark_kernel(
    int64_t N, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    int p, uint32_t* state, uint64_t* __restrict__ mask, uint32_t* __restrict__ inner_entries)
{
    const int lane = threadIdx.x & 63;
    const int64_t v = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (v >= N) return;
    uint64_t m = 0;
    uint32_t inner = 0;
    if ((state[v] & 0xffffu) == (uint32_t)p) {
        const int64_t lo = row_ptr[v], hi = row_ptr[v + 1];
        for (int64_t e0 = lo; e0 < hi; e0 += 64 * kAhead) {
            int32_t u[kAhead];
            uint32_t st[kAhead];
#pragma unroll
            for (int t = 0; t < kAhead; ++t) {
                const int64_t e = e0 + 64 * t + lane;
                u[t] = e < hi ? col_idx[e] : -1;
            }
#pragma unroll
            for (int t = 0; t < kAhead; ++t) st[t] = u[t] >= 0 ? state[u[t]] : 0xffffu;
#pragma unroll
            for (int t = 0; t < kAhead; ++t) {
                const uint32_t q = st[t] & 0xffffu;
                inner += (uint32_t)__popcll(__ballot(q == (uint32_t)p));
                if (q != (uint32_t)p && q != 0xffffu) {
                    m |= 1ull << q;
                    if (!(st[t] & kBoundary)) state[u[t]] = st[t] | kBoundary;      // every writer stores the same value
                }
            }
        }
        m = wave_or(m);
    }
    if (lane == 0) {
        mask[v] = m;
        inner_entries[v] = inner;
    }
}

// The rows that a workgroup of the LDS kernels works on: short ones are handed to its waves one by one, long ones (a wave would
// still be at work on one when all others are done) are shared by all waves afterwards.
constexpr int64_t kLongRow = 2048;
struct RowList {
    uint16_t rows[kListRows];                    // short rows from the front, long rows from the back
    uint32_t n_short, n_long, next;
};
__device__ __forceinline__ void list_rows(RowList& l, int64_t first, int64_t end, bool mine, int64_t at, int64_t length)
{
    // whole waves: at = the lane's row (or past the end)
    const int lane = threadIdx.x & 63;
    const bool have = at < end && mine;
    const uint64_t s = __ballot(have && length <= kLongRow), g = __ballot(have && length > kLongRow);
    uint32_t s0 = 0, g0 = 0;
    if (lane == 0) {
        if (s) s0 = atomicAdd(&l.n_short, (uint32_t)__popcll(s));
        if (g) g0 = atomicAdd(&l.n_long, (uint32_t)__popcll(g));
    }
    s0 = __shfl(s0, 0, 64);
    g0 = __shfl(g0, 0, 64);
    const uint64_t below = (1ull << lane) - 1;
    if ((s >> lane) & 1ull) l.rows[s0 + __popcll(s & below)] = (uint16_t)(at - first);
    if ((g >> lane) & 1ull) l.rows[kListRows - 1 - (g0 + __popcll(g & below))] = (uint16_t)(at - first);
}
__device__ __forceinline__ uint32_t next_row(RowList& l)
{
    uint32_t k = 0;
    if ((threadIdx.x & 63) == 0) k = atomicAdd(&l.next, 1u);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)__shfl(k, 0, 64));
}

// mark_kernel with the owners in LDS; a workgroup marks its rows' boundary nodes there too and adds them to all others' at
// the end.  Bound by reading the inner rows' columns.  Worker 0 of 4 of the Reddit-shaped graph: 231 -> 76 us.
constexpr int kLdsAhead = 8;
template <int BITS>
__global__ __launch_bounds__(kLdsThreads) void mark_lds_kernel(
    int64_t N, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int p,
    const uint32_t* __restrict__ owners, uint32_t* __restrict__ boundary, uint64_t* __restrict__ mask,
    uint32_t* __restrict__ inner_entries)
{
    constexpr int PER = 32 / BITS;
    __shared__ uint32_t table[kTableWords];
    __shared__ RowList list;
    __shared__ uint64_t all_mask;
    __shared__ uint32_t all_inner;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int words = (int)((N + PER - 1) / PER), marks = (int)((N + 31) / 32);
    uint32_t* marked = table + words;
    for (int i = tid; i < words; i += kLdsThreads) table[i] = owners[i];
    for (int i = tid; i < marks; i += kLdsThreads) marked[i] = 0u;
    if (tid == 0) list.n_short = list.n_long = list.next = 0u;
    __syncthreads();
    auto owner = [&](uint32_t u) { return (table[u / PER] >> (u % PER * BITS)) & ((1u << BITS) - 1u); };
    const int64_t per = (N + gridDim.x - 1) / gridDim.x, first = blockIdx.x * per, end = min(first + per, N);
    for (int64_t r0 = first + (tid - lane); r0 < end; r0 += kLdsThreads) {
        const int64_t v = r0 + lane;
        const bool mine = v < end && owner((uint32_t)v) == (uint32_t)p;
        list_rows(list, first, end, mine, v, mine ? row_ptr[v + 1] - row_ptr[v] : 0);
        if (v < end && !mine) {
            mask[v] = 0ull;
            inner_entries[v] = 0u;
        }
    }
    __syncthreads();
    // the entries [lo, hi) of one row, `step` waves taking batches in turn from batch k on
    typedef std::conditional_t<BITS == 8, uint64_t, uint32_t> mask_t;        // (up to 16 workers otherwise)
    mask_t m;
    uint32_t inner;
    auto batch = [&](int64_t e0, int64_t hi, auto tiles) {
        constexpr int T = decltype(tiles)::value;
        int32_t u[T];
        uint32_t q[T];
#pragma unroll
        for (int t = 0; t < T; ++t) u[t] = e0 + 64 * t + lane < hi ? col_idx[e0 + 64 * t + lane] : -1;
#pragma unroll
        for (int t = 0; t < T; ++t) q[t] = owner((uint32_t)max(u[t], 0));
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const bool out = u[t] >= 0 && q[t] != (uint32_t)p;
            inner += (uint32_t)__popcll(__ballot(u[t] >= 0 && !out));
            if (out) atomicOr(&marked[u[t] >> 5], 1u << (u[t] & 31));
            m |= out ? (mask_t)1 << q[t] : (mask_t)0;
        }
    };
    auto walk = [&](int64_t lo, int64_t hi, int k, int step) {
        m = 0;
        inner = 0;
        constexpr int SPAN = 64 * kLdsAhead;
        int64_t e0 = lo + (int64_t)SPAN * k;
        for (; hi - e0 > SPAN / 2; e0 += (int64_t)SPAN * step) batch(e0, hi, std::integral_constant<int, kLdsAhead>{});
        if (hi - e0 > 128) batch(e0, hi, std::integral_constant<int, kLdsAhead / 2>{});
        else if (hi > e0) batch(e0, hi, std::integral_constant<int, 2>{});
        m = wave_or(m);
    };
    const uint32_t n_short = list.n_short, n_long = list.n_long;
    // (the next row's place is looked up while the current one is walked through)
    auto ask = [&](uint32_t k, int64_t& v, int64_t& lo, int64_t& hi) {
        v = first + (k < n_short ? list.rows[k] : 0);
        lo = k < n_short ? row_ptr[v] : 0;
        hi = k < n_short ? row_ptr[v + 1] : 0;
    };
    int64_t v, lo, hi;
    uint32_t k = next_row(list);
    ask(k, v, lo, hi);
    while (k < n_short) {
        int64_t v2, lo2, hi2;
        k = next_row(list);
        ask(k, v2, lo2, hi2);
        walk(lo, hi, 0, 1);
        if (lane == 0) {
            mask[v] = m;
            inner_entries[v] = inner;
        }
        v = v2;
        lo = lo2;
        hi = hi2;
    }
    for (uint32_t l = 0; l < n_long; ++l) {
        v = first + list.rows[kListRows - 1 - l];
        __syncthreads();
        if (tid == 0) {
            all_mask = 0ull;
            all_inner = 0u;
        }
        __syncthreads();
        walk(row_ptr[v], row_ptr[v + 1], wave, kLdsWaves);
        if (lane == 0) {
            atomicOr((unsigned long long*)&all_mask, (unsigned long long)m);
            atomicAdd(&all_inner, inner);
        }
        __syncthreads();
        if (tid == 0) {
            mask[v] = all_mask;
            inner_entries[v] = all_inner;
        }
    }
    __syncthreads();
    for (int i = tid; i < marks; i += kLdsThreads)
        if (marked[i]) atomicOr(&boundary[i], marked[i]);
}

// The 2 * n_parts lists (list q: what peer q is sent, list n_parts + q: what it sends), the inner and the boundary nodes:
// members per block of kThreads nodes, counts[list * blocks + block].  A wave counts its 64 nodes with one ballot per
// list.  The inner rows' entries are added up per block beside them, so that one scan and one more pass over the nodes give all
// numbers and places (three scans and a sum over the nodes were ten launches, 45 us of the Reddit-shaped graph's share).
constexpr int kMaxLists = 2 * kMaxWorkers + 2;
__device__ __forceinline__ uint64_t list_members(int list, int n_parts, int p, uint64_t m, uint32_t st)
{
    // st of a lane without a node: kNobody
    if (list < n_parts) return __ballot((m >> list) & 1ull);
    if (list < 2 * n_parts) return __ballot((st & kBoundary) && (st & 0xffffu) == (uint32_t)(list - n_parts));
    return __ballot(list == 2 * n_parts ? (st & 0xffffu) == (uint32_t)p : (st & kBoundary) != 0u);
}
// `boundary`: the bits of mark_lds_kernel, which go into the states here; else NULL
__global__ __launch_bounds__(kThreads) void list_count_kernel(int64_t N, int n_parts, int p, const int64_t* __restrict__ row_ptr,
                                                              uint32_t* __restrict__ state,
                                                              const uint32_t* __restrict__ boundary,
                                                              const uint64_t* __restrict__ mask, int64_t blocks,
                                                              uint32_t* __restrict__ counts, int64_t* __restrict__ block_entries)
{
    __shared__ uint32_t sh[kThreads / 64][kMaxLists];
    __shared__ int64_t entries[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint64_t m = v < N ? mask[v] : 0ull;
    uint32_t st = v < N ? state[v] : kNobody;
    if (boundary && v < N) {
        if ((boundary[v >> 5] >> (v & 31)) & 1u) st |= kBoundary;
        state[v] = st;
    }
    for (int l = 0; l < 2 * n_parts + 2; ++l) {
        const uint32_t c = (uint32_t)__popcll(list_members(l, n_parts, p, m, st));
        if (lane == 0) sh[wave][l] = c;
    }
    int64_t e = v < N && (st & 0xffffu) == (uint32_t)p ? row_ptr[v + 1] - row_ptr[v] : 0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) e += __shfl_xor((long long)e, d, 64);
    if (lane == 0) entries[wave] = e;
    __syncthreads();
    for (int l = threadIdx.x; l < 2 * n_parts + 2; l += kThreads)
        counts[(int64_t)l * blocks + blockIdx.x] = (sh[0][l] + sh[1][l]) + (sh[2][l] + sh[3][l]);
    if (threadIdx.x == 0) block_entries[blockIdx.x] = (entries[0] + entries[1]) + (entries[2] + entries[3]);
}

// the header's sizes, N >= 1: a list's offset is its first block's position; block_entries becomes its exclusive prefix sum
__global__ __launch_bounds__(kLdsThreads) void totals_kernel(int n_parts, int64_t blocks, const uint32_t* __restrict__ list_at,
                                                             int64_t* __restrict__ block_entries, const ShareHeader* hdr,
                                                             ShareHeader* report)
{
    __shared__ int64_t sums[kLdsWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto at = [&](int l) { return list_at[(int64_t)l * blocks]; };         // (differences are exact modulo 2^32)
    for (int l = tid; l <= n_parts; l += kLdsThreads) {
        report->send_off[l] = at(l);
        report->recv_off[l] = (int64_t)(at(n_parts + l) - at(n_parts));
    }
    if (tid == 0) {
        report->n_inner = (int64_t)(at(2 * n_parts + 1) - at(2 * n_parts));
        report->n_halo = (int64_t)(at(2 * n_parts + 2) - at(2 * n_parts + 1));
        report->n_send = at(n_parts);
    }
    int64_t before = 0;
    for (int64_t b0 = 0; b0 < blocks; b0 += kLdsThreads) {
        const int64_t mine = b0 + tid < blocks ? block_entries[b0 + tid] : 0;
        int64_t incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t t = __shfl_up((long long)incl, d, 64);
            if (lane >= d) incl += t;
        }
        if (lane == 63) sums[wave] = incl;
        __syncthreads();
        int64_t all = 0;
        for (int w = 0; w < kLdsWaves; ++w) {
            if (w < wave) incl += sums[w];
            all += sums[w];
        }
        if (b0 + tid < blocks) block_entries[b0 + tid] = before + incl - mine;
        before += all;
        __syncthreads();
    }
    if (tid == 0) {
        report->nnz_local = before;
        report->bad_part = hdr->bad_part;
    }
}

// local numbering, global ids, degrees and row offsets of the local nodes, and the members of the lists: a wave's members of a
// list go behind those of the waves and blocks before it
__global__ __launch_bounds__(kThreads) void number_kernel(
    int64_t N, const int64_t* __restrict__ row_ptr, int p, int n_parts,
    const uint32_t* __restrict__ state, const uint64_t* __restrict__ mask,
    int64_t n_inner, int64_t n_local, int64_t nnz_local, int64_t n_send, int64_t blocks,
    const uint32_t* __restrict__ list_at, const int64_t* __restrict__ entries_before,
    int32_t* __restrict__ to_local, uint4* __restrict__ table,
    int32_t* __restrict__ local_ids, int64_t* __restrict__ local_row_ptr, int32_t* __restrict__ global_deg,
    int32_t* __restrict__ send_ids, int32_t* __restrict__ recv_ids)
{
    __shared__ uint32_t sh[kThreads / 64][kMaxLists];
    __shared__ int64_t entries[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint32_t st = v < N ? state[v] : kNobody;
    const uint64_t m = v < N ? mask[v] : 0ull;
    const bool inner = (st & 0xffffu) == (uint32_t)p, halo = (st & kBoundary) != 0u;
    for (int q = 0; q < 2 * n_parts + 2; ++q) {
        const uint32_t c = (uint32_t)__popcll(list_members(q, n_parts, p, m, st));
        if (lane == 0) sh[wave][q] = c;
    }
    const int64_t deg = v < N ? row_ptr[v + 1] - row_ptr[v] : 0;
    int64_t incl = inner ? deg : 0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t t = __shfl_up((long long)incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) entries[wave] = incl;
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1;
    // position of the lane among the members of a list
    auto place = [&](int q, uint64_t members) {
        uint32_t at = list_at[(int64_t)q * blocks + blockIdx.x] + (uint32_t)__popcll(members & below);
        for (int w = 0; w < wave; ++w) at += sh[w][q];
        return at;
    };
    const uint64_t ins = list_members(2 * n_parts, n_parts, p, m, st), outs = list_members(2 * n_parts + 1, n_parts, p, m, st);
    const uint32_t before_in = place(2 * n_parts, ins) - list_at[(int64_t)2 * n_parts * blocks];
    const int64_t before_out = n_inner + (int64_t)(place(2 * n_parts + 1, outs) - list_at[(int64_t)(2 * n_parts + 1) * blocks]);
    const int64_t l = inner ? (int64_t)before_in : halo ? before_out : -1;
    if (v < N) {
        if (!table) to_local[v] = (int32_t)l;
        if (l >= 0) {
            int64_t first = nnz_local;                       // (boundary rows are empty)
            if (inner) {
                first = entries_before[blockIdx.x] + incl - deg;
                for (int w = 0; w < wave; ++w) first += entries[w];
            }
            local_ids[l] = (int32_t)v;
            local_row_ptr[l] = first;
            global_deg[l] = (int32_t)deg;
        }
        // per 32 nodes: which are inner, inner ids before them, which are boundary nodes, boundary ids before them
        if (table && (lane & 31) == 0)
            table[v >> 5] = make_uint4((uint32_t)(ins >> lane), before_in, (uint32_t)(outs >> lane), (uint32_t)before_out);
    }
    if (v == 0) local_row_ptr[n_local] = nnz_local;
    for (int q = 0; q < 2 * n_parts; ++q) {
        const uint64_t members = list_members(q, n_parts, p, m, st);
        if (!((members >> lane) & 1ull)) continue;
        const int64_t at = place(q, members);
        if (q < n_parts) send_ids[at] = (int32_t)l;
        else recv_ids[at - n_send] = (int32_t)l;
    }
}

// One wave per inner local row: renumber the global row; inner entries first, then boundary entries, each group in its
// original (ascending) order.  Four tiles of 64 entries in flight, as in mark_kernel (worker 0 of 4 of the Reddit-shaped
// graph: 457 -> 192 us; half of it was a pass that counted the inner entries first).
__global__ __launch_bounds__(kThreads) void columns_kernel(
    int64_t n_inner, const int32_t* __restrict__ local_ids, const int64_t* __restrict__ row_ptr,
    const int32_t* __restrict__ col_idx, const int32_t* __restrict__ to_local, const uint32_t* __restrict__ inner_entries,
    const int64_t* __restrict__ local_row_ptr, int32_t* __restrict__ local_col)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (i >= n_inner) return;
    const int64_t v = local_ids[i];
    const int64_t lo = row_ptr[v], hi = row_ptr[v + 1], base = local_row_ptr[i];
    const uint64_t below = (1ull << lane) - 1;
    int64_t at_in = base, at_out = base + inner_entries[v];
    for (int64_t e0 = lo; e0 < hi; e0 += 64 * kAhead) {
        int32_t u[kAhead], l[kAhead];
#pragma unroll
        for (int t = 0; t < kAhead; ++t) {
            const int64_t e = e0 + 64 * t + lane;
            u[t] = e < hi ? col_idx[e] : -1;
        }
#pragma unroll
        for (int t = 0; t < kAhead; ++t) l[t] = u[t] >= 0 ? to_local[u[t]] : 0;
#pragma unroll
        for (int t = 0; t < kAhead; ++t) {
            const bool valid = u[t] >= 0, in = valid && l[t] < n_inner, out = valid && !in;
            const uint64_t bin = __ballot(in), bout = __ballot(out);
            if (in) local_col[at_in + __popcll(bin & below)] = l[t];
            if (out) local_col[at_out + __popcll(bout & below)] = l[t];
            at_in += __popcll(bin);
            at_out += __popcll(bout);
        }
    }
}

// columns_kernel with the numbering in LDS (number_kernel's table).  A long row is cut into one piece per wave, whose inner
// entries are counted first.  Worker 0 of 4 of the Reddit-shaped graph: 192 -> 87 us.
__global__ __launch_bounds__(kLdsThreads) void columns_lds_kernel(
    int64_t N, int64_t n_inner, const int32_t* __restrict__ local_ids, const int64_t* __restrict__ row_ptr,
    const int32_t* __restrict__ col_idx, const uint4* __restrict__ numbering, const uint32_t* __restrict__ inner_entries,
    const int64_t* __restrict__ local_row_ptr, int32_t* __restrict__ local_col)
{
    __shared__ uint4 table[kTableWords / 4];
    __shared__ RowList list;
    __shared__ uint32_t piece_inner[kLdsWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int words = (int)((N + 31) / 32);
    for (int i = tid; i < words; i += kLdsThreads) table[i] = numbering[i];
    if (tid == 0) list.n_short = list.n_long = list.next = 0u;
    __syncthreads();
    const int64_t per = (n_inner + gridDim.x - 1) / gridDim.x, first = blockIdx.x * per, end = min(first + per, n_inner);
    for (int64_t r0 = first + (tid - lane); r0 < end; r0 += kLdsThreads) {
        const int64_t i = r0 + lane;
        list_rows(list, first, end, true, i, i < end ? local_row_ptr[i + 1] - local_row_ptr[i] : 0);
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1;
    // the entries [lo, hi) of a row, up to kLdsAhead tiles of 64 in flight
    auto batch = [&](int64_t e0, int64_t hi, auto tiles, auto use) {
        constexpr int T = decltype(tiles)::value;
        int32_t u[T];
        uint4 w[T];
#pragma unroll
        for (int t = 0; t < T; ++t) u[t] = e0 + 64 * t + lane < hi ? col_idx[e0 + 64 * t + lane] : -1;
#pragma unroll
        for (int t = 0; t < T; ++t) w[t] = table[max(u[t], 0) >> 5];
#pragma unroll
        for (int t = 0; t < T; ++t) use(u[t], w[t]);
    };
    auto walk = [&](int64_t lo, int64_t hi, auto use) {
        constexpr int SPAN = 64 * kLdsAhead;
        int64_t e0 = lo;
        for (; hi - e0 > SPAN / 2; e0 += SPAN) batch(e0, hi, std::integral_constant<int, kLdsAhead>{}, use);
        if (hi - e0 > 128) batch(e0, hi, std::integral_constant<int, kLdsAhead / 2>{}, use);
        else if (hi > e0) batch(e0, hi, std::integral_constant<int, 2>{}, use);
    };
    auto place = [&](int64_t lo, int64_t hi, int64_t at_in, int64_t at_out) {
        walk(lo, hi, [&](int32_t u, const uint4& w) {
            const bool valid = u >= 0;
            const uint32_t bit = 1u << (u & 31);
            const bool in = valid && (w.x & bit), out = valid && !in;
            const uint64_t bin = __ballot(in), bout = __ballot(out);
            const uint32_t l = in ? w.y + __popc(w.x & (bit - 1)) : w.w + __popc(w.z & (bit - 1));
            const int64_t at = in ? at_in + __popcll(bin & below) : at_out + __popcll(bout & below);
            if (valid) local_col[at] = (int32_t)l;
            at_in += __popcll(bin);
            at_out += __popcll(bout);
        });
    };
    const uint32_t n_short = list.n_short, n_long = list.n_long;
    // (the next row's place is looked up while the current one is written)
    struct Row {
        int64_t lo, hi, base;
        uint32_t inner;
    };
    auto ask = [&](uint32_t k) {
        Row r = {0, 0, 0, 0u};
        if (k < n_short) {
            const int64_t i = first + list.rows[k], v = local_ids[i];
            r.base = local_row_ptr[i];
            r.lo = row_ptr[v];
            r.hi = row_ptr[v + 1];
            r.inner = inner_entries[v];
        }
        return r;
    };
    uint32_t k = next_row(list);
    Row row = ask(k);
    while (k < n_short) {
        k = next_row(list);
        const Row next = ask(k);
        place(row.lo, row.hi, row.base, row.base + row.inner);
        row = next;
    }
    for (uint32_t l = 0; l < n_long; ++l) {
        const int64_t i = first + list.rows[kListRows - 1 - l], v = local_ids[i], base = local_row_ptr[i];
        const int64_t lo = row_ptr[v], hi = row_ptr[v + 1];
        const int64_t piece = ((hi - lo + kLdsWaves - 1) / kLdsWaves + 63) / 64 * 64;
        const int64_t from = min(lo + piece * wave, hi), to = min(from + piece, hi);
        uint32_t inner = 0;
        walk(from, to, [&](int32_t u, const uint4& w) {
            inner += (uint32_t)__popcll(__ballot(u >= 0 && ((w.x >> (u & 31)) & 1u)));
        });
        __syncthreads();
        if (lane == 0) piece_inner[wave] = inner;
        __syncthreads();
        uint32_t before = 0;
        for (int w = 0; w < wave; ++w) before += piece_inner[w];
        place(from, to, base + before, base + inner_entries[v] + ((from - lo) - before));
    }
}

// rows of a table <-> a dense buffer; one thread per VEC floats
template <int VEC, bool SCATTER>
__global__ __launch_bounds__(kThreads) void rows_kernel(
    int64_t n, const int32_t* __restrict__ ids, int64_t table_rows, int64_t F,
    const float* __restrict__ src, int64_t lds, float* __restrict__ dst, int64_t ldd)
{
    const int64_t chunks = (F + VEC - 1) / VEC;
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= n * chunks) return;
    const int64_t i = t / chunks, c = (t % chunks) * VEC;
    const int64_t r = ids[i];
    if (r < 0 || r >= table_rows) return;                 // ids outside the table are ignored
    const float* s = SCATTER ? src + i * lds + c : src + r * lds + c;
    float* d = SCATTER ? dst + r * ldd + c : dst + i * ldd + c;
    if constexpr (VEC == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        if (c + 4 <= F) {
            *reinterpret_cast<f4*>(d) = *reinterpret_cast<const f4*>(s);
        } else {                                          // ragged last vector of a row
            for (int k = 0; k < (int)(F - c); ++k) d[k] = s[k];
        }
    } else {
        *d = *s;
    }
}

__global__ __launch_bounds__(kThreads) void set_degrees_kernel(int64_t N, const int32_t* __restrict__ d_in,
                                                               int32_t* __restrict__ deg, float* __restrict__ dinv)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= N) return;
    const int32_t d = d_in[v];
    deg[v] = d;
    dinv[v] = d > 0 ? 1.0f / sqrtf((float)d) : 0.0f;
}

struct Layout {
    bool lds_marks, lds_columns;
    int64_t owners, boundary, table;
    int64_t header, mask, state, block_entries, inner_entries, to_local, counts, list_at, tmp, blocks, total;
    size_t tmp_bytes;
};

int make_layout(int64_t N, int n_parts, Layout& L)
{
    const int64_t n = N > 0 ? N : 1;
    L.blocks = (n + kThreads - 1) / kThreads;
    const int64_t lists = (2 * (int64_t)n_parts + 2) * L.blocks + 1;
    L.tmp_bytes = 0;
    if (rocprim::exclusive_scan(nullptr, L.tmp_bytes, (uint32_t*)nullptr, (uint32_t*)nullptr, 0u, (size_t)lists, rocprim::plus<uint32_t>(),
                                (hipStream_t)0) != hipSuccess) return RETEXO_E_HIP;
    int64_t off = 0;
    L.header = off;    off += align_up((int64_t)sizeof(ShareHeader), 256);
    L.mask = off;      off += align_up(8 * n, 256);
    L.state = off;     off += align_up(4 * n, 256);
    L.block_entries = off; off += align_up(8 * L.blocks, 256);
    L.inner_entries = off; off += align_up(4 * n, 256);
    L.to_local = off;  off += align_up(4 * n, 256);
    L.counts = off;    off += align_up(4 * lists, 256);
    L.list_at = off;   off += align_up(4 * lists, 256);
    L.lds_marks = owners_fit(N, n_parts);
    L.lds_columns = N <= kTableNodes;
    L.owners = off;    off += L.lds_marks ? align_up(n, 256) : 0;                     // (at most eight bits each)
    L.boundary = off;  off += L.lds_marks ? align_up((n + 31) / 32 * 4, 256) : 0;
    L.table = off;     off += L.lds_columns ? align_up((n + 31) / 32 * 16, 256) : 0;
    L.tmp = off;       off += align_up((int64_t)L.tmp_bytes, 256);
    L.total = off;
    return RETEXO_OK;
}

template <bool SCATTER>
int launch_rows(int64_t n, const int32_t* ids, int64_t table_rows, int64_t F, const float* src, int64_t lds,
                float* dst, int64_t ldd, hipStream_t stream)
{
    if (n == 0 || F == 0) return RETEXO_OK;
    const bool v4 = lds % 4 == 0 && ldd % 4 == 0 && (uintptr_t)src % 16 == 0 && (uintptr_t)dst % 16 == 0;
    const int64_t threads = n * (v4 ? (F + 3) / 4 : F);
    const dim3 grid((unsigned)((threads + kThreads - 1) / kThreads));
    if (v4) rows_kernel<4, SCATTER><<<grid, dim3(kThreads), 0, stream>>>(n, ids, table_rows, F, src, lds, dst, ldd);
    else rows_kernel<1, SCATTER><<<grid, dim3(kThreads), 0, stream>>>(n, ids, table_rows, F, src, lds, dst, ldd);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}

}  // namespace

extern "C" int64_t retexo_partition_workspace_bytes(int64_t N, int n_parts, int64_t send_capacity)
{
    if (N < 0 || N >= (1ll << 31) || send_capacity < 0 || send_capacity >= (1ll << 31)) return RETEXO_E_SIZE;
    if (n_parts < 1 || n_parts > kMaxWorkers) return RETEXO_E_SIZE;
    if (N * (int64_t)(n_parts - 1) >= (1ll << 31)) return RETEXO_E_SIZE;     // 32-bit positions in the lists
    Layout L;
    if (int s = make_layout(N, n_parts, L)) return s;
    return L.total;
}

extern "C" int retexo_partition_share(int64_t N, const int64_t* d_row_ptr, const int32_t* d_col_idx,
                                      const int32_t* d_part, int n_parts, int part,
                                      int64_t local_capacity, int64_t col_capacity, int64_t send_capacity,
                                      int32_t* d_local_ids, int64_t* d_local_row_ptr, int32_t* d_local_col_idx,
                                      int32_t* d_global_deg, int32_t* d_send_ids, int32_t* d_recv_ids,
                                      int64_t* h_sizes, int64_t* h_send_offsets, int64_t* h_recv_offsets,
                                      void* d_workspace, int64_t workspace_bytes, void* stream_)
{
    if (N < 0 || N >= (1ll << 31)) return RETEXO_E_SIZE;
    if (n_parts < 1 || n_parts > kMaxWorkers || part < 0 || part >= n_parts) return RETEXO_E_SIZE;
    if (N * (int64_t)(n_parts - 1) >= (1ll << 31)) return RETEXO_E_SIZE;     // 32-bit positions in the lists
    if (local_capacity < 0 || col_capacity < 0 || send_capacity < 0 || send_capacity >= (1ll << 31)) return RETEXO_E_SIZE;
    if (!h_sizes) return RETEXO_E_NULL;
    if (N > 0 && (!d_row_ptr || !d_part)) return RETEXO_E_NULL;
    Layout L;
    if (int s = make_layout(N, n_parts, L)) return s;
    if (!d_workspace || ((uintptr_t)d_workspace & 255) || workspace_bytes < L.total) return RETEXO_E_WORKSPACE;

    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)d_workspace;
    ShareHeader* hdr = (ShareHeader*)(ws + L.header);
    uint64_t* mask = (uint64_t*)(ws + L.mask);
    uint32_t* state = (uint32_t*)(ws + L.state);
    int64_t* block_entries = (int64_t*)(ws + L.block_entries);
    uint32_t* inner_entries = (uint32_t*)(ws + L.inner_entries);
    int32_t* to_local = (int32_t*)(ws + L.to_local);
    uint32_t* counts = (uint32_t*)(ws + L.counts);
    uint32_t* list_at = (uint32_t*)(ws + L.list_at);
    void* tmp = ws + L.tmp;

    if (int e = launch_zero(hdr, sizeof(ShareHeader), stream)) return e;
    HostReport report(stream);
    static_assert(sizeof(ShareHeader) <= kReportBytes && sizeof(ShareHeader) % 4 == 0, "a report holds it");
    const bool direct = N > 0 && report.get();
    const dim3 node_grid((unsigned)L.blocks);
    if (N > 0) {
        uint32_t* owners = (uint32_t*)(ws + L.owners);
        uint32_t* boundary = L.lds_marks ? (uint32_t*)(ws + L.boundary) : nullptr;
        const int bits = owner_bits(n_parts);
        state_kernel<<<node_grid, dim3(kThreads), 0, stream>>>(N, d_part, n_parts, state, L.lds_marks ? bits : 0, owners, boundary,
                                                               hdr);
        if (L.lds_marks) {
            const dim3 grid((unsigned)((N + 15) / 16 < kLdsBlocks ? (N + 15) / 16 : kLdsBlocks));
            auto mark = [&](auto kernel) {
                kernel<<<grid, dim3(kLdsThreads), 0, stream>>>(N, d_row_ptr, d_col_idx, part, owners, boundary, mask, inner_entries);
            };
            if (bits == 1) mark(mark_lds_kernel<1>);
            else if (bits == 2) mark(mark_lds_kernel<2>);
            else if (bits == 4) mark(mark_lds_kernel<4>);
            else mark(mark_lds_kernel<8>);
        } else {
            const int rows_per_block = kThreads / 64;
            mark_kernel<<<dim3((unsigned)((N + rows_per_block - 1) / rows_per_block)), dim3(kThreads), 0, stream>>>(
                N, d_row_ptr, d_col_idx, part, state, mask, inner_entries);
        }
        list_count_kernel<<<node_grid, dim3(kThreads), 0, stream>>>(N, n_parts, part, d_row_ptr, state, boundary, mask, L.blocks,
                                                                    counts, block_entries);
        size_t tb = L.tmp_bytes;
        RETEXO_HIP_TRY(rocprim::exclusive_scan(tmp, tb, counts, list_at, 0u, (size_t)((2 * n_parts + 2) * L.blocks + 1),
                                               rocprim::plus<uint32_t>(), stream));
        totals_kernel<<<dim3(1), dim3(kLdsThreads), 0, stream>>>(n_parts, L.blocks, list_at, block_entries, hdr,
                                                               direct ? (ShareHeader*)report.get() : hdr);
    }
    ShareHeader h;
    if (!direct) RETEXO_HIP_TRY(hipMemcpyAsync(&h, hdr, sizeof(h), hipMemcpyDeviceToHost, stream));
    RETEXO_HIP_TRY(report.wait());
    if (direct) memcpy(&h, report.get(), sizeof(h));
    if (h.bad_part) return RETEXO_E_PARTITION;
    h_sizes[0] = h.n_inner;
    h_sizes[1] = h.n_halo;
    h_sizes[2] = h.nnz_local;
    h_sizes[3] = h.n_send;
    const int64_t n_local = h.n_inner + h.n_halo;
    // a missing row-pointer array counts as no capacity at all: the size query of an empty share
    if (!d_local_row_ptr || n_local > local_capacity || h.nnz_local > col_capacity || h.n_send > send_capacity)
        return RETEXO_E_CAPACITY;
    if (!h_send_offsets || !h_recv_offsets) return RETEXO_E_NULL;
    if (n_local > 0 && (!d_local_ids || !d_global_deg)) return RETEXO_E_NULL;
    if (h.nnz_local > 0 && !d_local_col_idx) return RETEXO_E_NULL;
    if ((h.n_send > 0 && !d_send_ids) || (h.n_halo > 0 && !d_recv_ids)) return RETEXO_E_NULL;

    uint4* table = L.lds_columns && h.nnz_local >= kTableEntries ? (uint4*)(ws + L.table) : nullptr;
    if (N > 0) {
        number_kernel<<<node_grid, dim3(kThreads), 0, stream>>>(
            N, d_row_ptr, part, n_parts, state, mask, h.n_inner, n_local, h.nnz_local, h.n_send, L.blocks, list_at, block_entries,
            to_local, table, d_local_ids, d_local_row_ptr, d_global_deg, d_send_ids, d_recv_ids);
    } else {
        RETEXO_HIP_TRY(hipMemsetAsync(d_local_row_ptr, 0, sizeof(int64_t), stream));
    }
    if (h.n_inner > 0 && table) {
        const int64_t blocks = (h.n_inner + 15) / 16;
        columns_lds_kernel<<<dim3((unsigned)(blocks < kLdsBlocks ? blocks : kLdsBlocks)), dim3(kLdsThreads), 0, stream>>>(
            N, h.n_inner, d_local_ids, d_row_ptr, d_col_idx, table, inner_entries, d_local_row_ptr, d_local_col_idx);
    } else if (h.n_inner > 0) {
        const int rows_per_block = kThreads / 64;
        columns_kernel<<<dim3((unsigned)((h.n_inner + rows_per_block - 1) / rows_per_block)), dim3(kThreads), 0, stream>>>(
            h.n_inner, d_local_ids, d_row_ptr, d_col_idx, to_local, inner_entries, d_local_row_ptr, d_local_col_idx);
    }
    RETEXO_HIP_TRY(hipGetLastError());
    RETEXO_HIP_TRY(hipStreamSynchronize(stream));
    for (int q = 0; q <= n_parts; ++q) {
        h_send_offsets[q] = h.send_off[q];
        h_recv_offsets[q] = h.recv_off[q];
    }
    return RETEXO_OK;
}

extern "C" int retexo_halo_pack(int64_t n, const int32_t* d_ids, int64_t table_rows, int64_t F,
                                const float* d_H, int64_t ldh, float* d_buf, int64_t ldb, void* stream)
{
    if (n < 0 || F < 0 || table_rows < 0) return RETEXO_E_SIZE;
    if (n > 0 && F > 0 && (!d_ids || !d_H || !d_buf)) return RETEXO_E_NULL;
    if (ldh < F || ldb < F) return RETEXO_E_LD;
    return launch_rows<false>(n, d_ids, table_rows, F, d_H, ldh, d_buf, ldb, (hipStream_t)stream);
}

extern "C" int retexo_halo_unpack(int64_t n, const int32_t* d_ids, int64_t table_rows, int64_t F,
                                  const float* d_buf, int64_t ldb, float* d_H, int64_t ldh, void* stream)
{
    if (n < 0 || F < 0 || table_rows < 0) return RETEXO_E_SIZE;
    if (n > 0 && F > 0 && (!d_ids || !d_H || !d_buf)) return RETEXO_E_NULL;
    if (ldh < F || ldb < F) return RETEXO_E_LD;
    return launch_rows<true>(n, d_ids, table_rows, F, d_buf, ldb, d_H, ldh, (hipStream_t)stream);
}

extern "C" int retexo_plan_set_degrees(retexo_plan* plan, const int32_t* d_deg, void* stream)
{
    if (!plan) return RETEXO_E_NULL;
    if (plan->N > 0 && !d_deg) return RETEXO_E_NULL;
    if (plan->N == 0) return RETEXO_OK;
    plan->degrees_set = true;
    set_degrees_kernel<<<dim3((unsigned)((plan->N + kThreads - 1) / kThreads)), dim3(kThreads), 0, (hipStream_t)stream>>>(
        plan->N, d_deg, plan->deg, plan->dinv);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
