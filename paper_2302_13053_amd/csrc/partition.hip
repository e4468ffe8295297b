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

#include <rocprim/device/device_reduce.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/iterator/counting_iterator.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include "common.hpp"

namespace {

constexpr int kThreads = 256;
constexpr int kMaxWorkers = 64;       // one bit per worker in a 64-bit mask

struct ShareHeader {                  // start of the workspace; copied to the host
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

// state of a node while its share is derived: its owner, and whether it was found to be a boundary node
constexpr uint32_t kBoundary = 0x80000000u;

__global__ __launch_bounds__(kThreads) void state_kernel(int64_t N, const int32_t* __restrict__ part, int n_parts,
                                                         uint32_t* __restrict__ state, ShareHeader* hdr)
{
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (v >= N) return;
    const int q = part[v];
    const bool bad = q < 0 || q >= n_parts;
    if (bad) atomicOr(&hdr->bad_part, 1u);
    state[v] = bad ? 0xffffu : (uint32_t)q;       // (no worker has that id; the call ends in an error)
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

struct IsInner {
    const int32_t* part;
    int p;
    __device__ uint32_t operator()(int64_t v) const { return part[v] == p ? 1u : 0u; }
};
struct InnerRowLength {
    const int32_t* part;
    const int64_t* row_ptr;
    int p;
    __device__ int64_t operator()(int64_t v) const { return part[v] == p ? row_ptr[v + 1] - row_ptr[v] : 0; }
};
struct IsBoundary {
    const uint32_t* state;
    __device__ uint32_t operator()(int64_t v) const { return state[v] >> 31; }
};
struct LocalRowLength {               // row length of local node i (0 for boundary nodes and for i == n_local)
    const int32_t* local_ids;
    const int64_t* row_ptr;
    int64_t n_inner;
    __device__ int64_t operator()(int64_t i) const
    {
        if (i >= n_inner) return 0;
        const int64_t v = local_ids[i];
        return row_ptr[v + 1] - row_ptr[v];
    }
};

// The 2 * n_parts lists (list q: what peer q is sent, list n_parts + q: what it sends): members per block of kThreads
// nodes, counts[list * blocks + block].  A wave counts its 64 nodes with one ballot per list.
__device__ __forceinline__ uint64_t list_members(int list, int n_parts, uint64_t m, uint32_t st)
{
    return __ballot(list < n_parts ? (m >> list) & 1ull : (st & kBoundary) && (st & 0xffffu) == (uint32_t)(list - n_parts));
}
__global__ __launch_bounds__(kThreads) void list_count_kernel(int64_t N, int n_parts, const uint32_t* __restrict__ state,
                                                              const uint64_t* __restrict__ mask, int64_t blocks,
                                                              uint32_t* __restrict__ counts)
{
    __shared__ uint32_t sh[kThreads / 64][2 * kMaxWorkers];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint64_t m = v < N ? mask[v] : 0ull;
    const uint32_t st = v < N ? state[v] : 0u;
    for (int l = 0; l < 2 * n_parts; ++l) {
        const uint32_t c = (uint32_t)__popcll(list_members(l, n_parts, m, st));
        if (lane == 0) sh[wave][l] = c;
    }
    __syncthreads();
    for (int l = threadIdx.x; l < 2 * n_parts; l += kThreads)
        counts[(int64_t)l * blocks + blockIdx.x] = (sh[0][l] + sh[1][l]) + (sh[2][l] + sh[3][l]);
}

// totals of the scans (last scan value + last element), N >= 1; the lists' offsets are their first blocks' positions
__global__ __launch_bounds__(kThreads) void totals_kernel(int64_t N, const int32_t* __restrict__ part, int p, int n_parts,
                                                          const uint32_t* __restrict__ rank_in, const uint32_t* __restrict__ state,
                                                          const uint32_t* __restrict__ rank_halo, int64_t blocks,
                                                          const uint32_t* __restrict__ list_at, ShareHeader* hdr)
{
    const int64_t n_halo = (int64_t)rank_halo[N - 1] + (int64_t)(state[N - 1] >> 31);
    const int64_t n_send = list_at[(int64_t)n_parts * blocks];
    for (int l = threadIdx.x; l <= n_parts; l += kThreads) {
        hdr->send_off[l] = list_at[(int64_t)l * blocks];
        hdr->recv_off[l] = l == n_parts ? n_halo : (int64_t)list_at[(int64_t)(n_parts + l) * blocks] - n_send;
    }
    if (threadIdx.x == 0) {
        hdr->n_inner = (int64_t)rank_in[N - 1] + (part[N - 1] == p ? 1 : 0);
        hdr->n_halo = n_halo;
        hdr->n_send = n_send;
    }
}

// local numbering, global ids and degrees of the local nodes, and the members of the lists: a wave's members of a list go
// behind those of the waves and blocks before it
__global__ __launch_bounds__(kThreads) void number_kernel(
    int64_t N, const int64_t* __restrict__ row_ptr, int p, int n_parts,
    const uint32_t* __restrict__ rank_in, const uint32_t* __restrict__ state, const uint64_t* __restrict__ mask,
    const uint32_t* __restrict__ rank_halo, int64_t n_inner, int64_t n_send, int64_t blocks,
    const uint32_t* __restrict__ list_at, int32_t* __restrict__ to_local,
    int32_t* __restrict__ local_ids, int32_t* __restrict__ global_deg, int32_t* __restrict__ send_ids,
    int32_t* __restrict__ recv_ids)
{
    __shared__ uint32_t sh[kThreads / 64][2 * kMaxWorkers];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint32_t st = v < N ? state[v] : 0u;
    const uint64_t m = v < N ? mask[v] : 0ull;
    int64_t l = -1;
    if (v < N) {
        if ((st & 0xffffu) == (uint32_t)p) l = rank_in[v];
        else if (st & kBoundary) l = n_inner + rank_halo[v];
        to_local[v] = (int32_t)l;
        if (l >= 0) {
            local_ids[l] = (int32_t)v;
            global_deg[l] = (int32_t)(row_ptr[v + 1] - row_ptr[v]);
        }
    }
    for (int q = 0; q < 2 * n_parts; ++q) {
        const uint32_t c = (uint32_t)__popcll(list_members(q, n_parts, m, st));
        if (lane == 0) sh[wave][q] = c;
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1;
    for (int q = 0; q < 2 * n_parts; ++q) {
        const uint64_t members = list_members(q, n_parts, m, st);
        if (!((members >> lane) & 1ull)) continue;
        int64_t at = (int64_t)list_at[(int64_t)q * blocks + blockIdx.x] + __popcll(members & below);
        for (int w = 0; w < wave; ++w) at += sh[w][q];
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
    int64_t header, mask, state, rank_in, rank_halo, inner_entries, to_local, counts, list_at, tmp, blocks, total;
    size_t tmp_bytes;
};

int make_layout(int64_t N, int n_parts, Layout& L)
{
    const int64_t n = N > 0 ? N : 1;
    L.blocks = (n + kThreads - 1) / kThreads;
    const int64_t lists = 2 * (int64_t)n_parts * L.blocks + 1;
    size_t a = 0, b = 0, c = 0, d = 0;
    auto it32 = rocprim::make_transform_iterator(rocprim::make_counting_iterator<int64_t>(0), IsInner{nullptr, 0});
    auto it64 = rocprim::make_transform_iterator(rocprim::make_counting_iterator<int64_t>(0),
                                                 InnerRowLength{nullptr, nullptr, 0});
    if (rocprim::exclusive_scan(nullptr, a, it32, (uint32_t*)nullptr, 0u, (size_t)n, rocprim::plus<uint32_t>(),
                                (hipStream_t)0) != hipSuccess) return RETEXO_E_HIP;
    if (rocprim::exclusive_scan(nullptr, b, it64, (int64_t*)nullptr, (int64_t)0, (size_t)(n + 1),
                                rocprim::plus<int64_t>(), (hipStream_t)0) != hipSuccess) return RETEXO_E_HIP;
    if (rocprim::reduce(nullptr, c, it64, (int64_t*)nullptr, (int64_t)0, (size_t)n, rocprim::plus<int64_t>(),
                        (hipStream_t)0) != hipSuccess) return RETEXO_E_HIP;
    if (rocprim::exclusive_scan(nullptr, d, (uint32_t*)nullptr, (uint32_t*)nullptr, 0u, (size_t)lists, rocprim::plus<uint32_t>(),
                                (hipStream_t)0) != hipSuccess) return RETEXO_E_HIP;
    L.tmp_bytes = a > b ? a : b;
    if (c > L.tmp_bytes) L.tmp_bytes = c;
    if (d > L.tmp_bytes) L.tmp_bytes = d;
    int64_t off = 0;
    L.header = off;    off += align_up((int64_t)sizeof(ShareHeader), 256);
    L.mask = off;      off += align_up(8 * n, 256);
    L.state = off;     off += align_up(4 * n, 256);
    L.rank_in = off;   off += align_up(4 * n, 256);
    L.rank_halo = off; off += align_up(4 * n, 256);
    L.inner_entries = off; off += align_up(4 * n, 256);
    L.to_local = off;  off += align_up(4 * n, 256);
    L.counts = off;    off += align_up(4 * lists, 256);
    L.list_at = off;   off += align_up(4 * lists, 256);
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
    uint32_t* rank_in = (uint32_t*)(ws + L.rank_in);
    uint32_t* rank_halo = (uint32_t*)(ws + L.rank_halo);
    uint32_t* inner_entries = (uint32_t*)(ws + L.inner_entries);
    int32_t* to_local = (int32_t*)(ws + L.to_local);
    uint32_t* counts = (uint32_t*)(ws + L.counts);
    uint32_t* list_at = (uint32_t*)(ws + L.list_at);
    void* tmp = ws + L.tmp;

    RETEXO_HIP_TRY(hipMemsetAsync(hdr, 0, sizeof(ShareHeader), stream));
    const dim3 node_grid((unsigned)L.blocks);
    if (N > 0) {
        state_kernel<<<node_grid, dim3(kThreads), 0, stream>>>(N, d_part, n_parts, state, hdr);
        const int rows_per_block = kThreads / 64;
        mark_kernel<<<dim3((unsigned)((N + rows_per_block - 1) / rows_per_block)), dim3(kThreads), 0, stream>>>(
            N, d_row_ptr, d_col_idx, part, state, mask, inner_entries);
        auto count = rocprim::make_counting_iterator<int64_t>(0);
        size_t tb = L.tmp_bytes;
        RETEXO_HIP_TRY(rocprim::exclusive_scan(tmp, tb, rocprim::make_transform_iterator(count, IsInner{d_part, part}),
                                               rank_in, 0u, (size_t)N, rocprim::plus<uint32_t>(), stream));
        tb = L.tmp_bytes;
        RETEXO_HIP_TRY(rocprim::exclusive_scan(tmp, tb, rocprim::make_transform_iterator(count, IsBoundary{state}), rank_halo,
                                               0u, (size_t)N, rocprim::plus<uint32_t>(), stream));
        list_count_kernel<<<node_grid, dim3(kThreads), 0, stream>>>(N, n_parts, state, mask, L.blocks, counts);
        tb = L.tmp_bytes;
        RETEXO_HIP_TRY(rocprim::exclusive_scan(tmp, tb, counts, list_at, 0u, (size_t)(2 * n_parts * L.blocks + 1),
                                               rocprim::plus<uint32_t>(), stream));
        tb = L.tmp_bytes;
        RETEXO_HIP_TRY(rocprim::reduce(tmp, tb, rocprim::make_transform_iterator(count, InnerRowLength{d_part, d_row_ptr, part}),
                                       &hdr->nnz_local, (int64_t)0, (size_t)N, rocprim::plus<int64_t>(), stream));
        totals_kernel<<<dim3(1), dim3(kThreads), 0, stream>>>(N, d_part, part, n_parts, rank_in, state, rank_halo, L.blocks,
                                                              list_at, hdr);
    }
    ShareHeader h;
    RETEXO_HIP_TRY(hipMemcpyAsync(&h, hdr, sizeof(h), hipMemcpyDeviceToHost, stream));
    RETEXO_HIP_TRY(hipStreamSynchronize(stream));
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

    if (N > 0) {
        number_kernel<<<node_grid, dim3(kThreads), 0, stream>>>(
            N, d_row_ptr, part, n_parts, rank_in, state, mask, rank_halo, h.n_inner, h.n_send, L.blocks, list_at, to_local,
            d_local_ids, d_global_deg, d_send_ids, d_recv_ids);
    }
    {
        auto len = rocprim::make_transform_iterator(rocprim::make_counting_iterator<int64_t>(0),
                                                    LocalRowLength{d_local_ids, d_row_ptr, h.n_inner});
        size_t tb = L.tmp_bytes;
        RETEXO_HIP_TRY(rocprim::exclusive_scan(tmp, tb, len, d_local_row_ptr, (int64_t)0, (size_t)(n_local + 1),
                                               rocprim::plus<int64_t>(), stream));
    }
    if (h.n_inner > 0) {
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
    set_degrees_kernel<<<dim3((unsigned)((plan->N + kThreads - 1) / kThreads)), dim3(kThreads), 0, (hipStream_t)stream>>>(
        plan->N, d_deg, plan->deg, plan->dinv);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
