// Neighbourhood aggregation over a CSR graph: the AGGR / COMBINE of Eq. 1 in
// the forms of the paper's three model families (GraphSAGE mean with
// self-concatenation, GCN symmetric normalisation, GAT edge softmax).
//
// The work is a sparse-times-dense product whose cost is the gather of one
// F-float row of Z per CSR entry: 4 bytes and one FMA per (edge, feature).
// It is bound by memory, not arithmetic, so the design is about the gather:
//
//  * One wavefront owns one (row, column-slab) pair.  Its 64 lanes each own
//    VEC consecutive columns (VEC = 4/2/1 floats depending on alignment) in
//    each of NC chunks, so one neighbour is fetched by NC fully coalesced
//    wave-wide loads of 64*VEC*4 bytes.
//  * Neighbour ids are read 64 at a time (one coalesced load), then broadcast
//    one by one with v_readlane, which leaves the id in a scalar register and
//    turns the row address into scalar arithmetic.  The broadcast loop is
//    unrolled so that several neighbours' loads are in flight per wave.
//  * Rows are scheduled longest first (plan order).  Rows at or above a degree
//    threshold get a whole workgroup: its waves take interleaved 64-edge tiles
//    and combine their partial sums through LDS in a fixed order.  Every
//    output element is written by exactly one wave and nothing is accumulated
//    with atomics, so results are bitwise reproducible.
//  * Edge softmax: per 64-edge tile the scores are computed one edge per lane,
//    the tile maximum and the sum of exponentials are wave reductions, and the
//    running (max, sum, accumulator) triple is rescaled once per tile (online
//    softmax at tile granularity) — one exp per edge and head instead of one
//    per edge and lane.
#include <type_traits>

#include "common.hpp"
#include "gather.hpp"

namespace {


enum { SCALE_SUM = 0, SCALE_MEAN = 1, SCALE_GCN = 2 };

struct AggArgs {
    const int64_t* row_ptr;
    const int32_t* col_idx;
    const int32_t* order;
    const int32_t* deg;
    const int32_t* set_deg;  // what a mean divides by where it is not the row's length (retexo_plan_set_degrees); else NULL: a load less
    const float* dinv;
    const float* wsrc;     // per-source weight of every gathered row, or NULL (all 1)
    const float* Z;
    int64_t ldz;
    float* out;
    int64_t ldo;
    int64_t ocol;          // first output column of the aggregate
    const float* el;       // <a_src, z_u> of node u, head h at el[u * el_stride + h]   (edge softmax only)
    int64_t el_stride;     // HP for the table in the workspace; ldz when the scores sit in Z's padding columns
    const float* er;       // [N, HP]  <a_dst, z_v>, or NULL:
    const float* er_from;  // a_dst [heads, Dh]; the kernel forms <a_dst, z_v> from row v itself (pipelined kernel, one slab)
    int64_t row_begin;     // range of plan order handled by this launch
    int64_t row_count;
    int64_t heavy_rows;    // rows at the head of the plan order with a workgroup each, and the workgroups of those
    int64_t heavy_items;   // rows (kernels whose one launch covers all rows)
    int64_t F;
    int nslab;
    int slab_major;
    int slab_cols;         // columns of a slab, and workgroups that it takes (edge softmax, several rows per wave)
    uint32_t slab_blocks;
    int scale;             // SCALE_*
    int levels;            // sums in levels (see BatchSums)
    int heads;
    int Dh;
    float slope;
    int copy_self;         // also write z_v into out[:, 0:F]
    int out_vec;           // aggregate slot of out is aligned for VEC-wide stores
    int out_half;          // ... or at least for 8-byte stores (float4 gathers only)
    int self_vec;          // self slot of out is aligned for VEC-wide stores
    // source-range walk (grouped kernel only): this launch covers the entries of each row whose
    // column lies in ranges [part_lo, part_hi) of the plan's split; NULL = whole rows
    const int32_t* part_ptr;
    int64_t n_rows;        // N (row pitch of part_ptr)
    int part_lo, part_hi;
    int first;             // first range of the walk: start from zero, write the self copy
    int last;              // last range: apply the mean / gcn scaling
    uint32_t table_bytes;  // Z up to the end of its last row's last vector (grouped kernels, below 4 GiB)
    // edge softmax, kept for the backward pass (TRAIN kernels only):
    f32x4* save_stats;     // [N, HP] {row maximum, 1/sum, share of the sum with p > 0, share with p <= 0}
    float* save_pos;       // [N, ld_pos] the part of the aggregate that comes from entries with p > 0
    float* save_neg;       // [N, ld_pos] ... and from entries with p <= 0 (the aggregate is their sum)
    int64_t ld_pos;
};

// ---------------------------------------------------------------------------
// sum / mean / gcn_sym, and (MAXOP) the element-wise maximum
//
// One launch covers both classes of rows: the first a.heavy_items workgroups share one (row, slab) item among their
// eight waves (interleaved 64-entry tiles, combined through LDS in wave order), the others hold eight independent
// items.  Long rows so start first and the short ones fill the chip beside them; two launches one after the other cost
// small graphs the longer of both times twice.
// Entries are fetched U at a time, the rest of a tile as one shorter batch (the count is the same for all lanes): a
// row of five entries waits for memory once, not once for four and once more.  Bound by memory latency on small graphs
// (19,717 rows, 108,393 entries, 256 columns: see long_rows) and by the gathers' bytes on large ones.
// ---------------------------------------------------------------------------
template <int VEC, int NC, bool MAXOP, bool LEVELS>
__global__ __launch_bounds__(64 * kHeavyWaves) void agg_linear_kernel(AggArgs a)
{
    constexpr int U = NC * VEC <= 8 ? 8 : 4;          // entries in flight per lane: up to 64 registers
    static_assert(!LEVELS || U == 8, "levels of 16 and 128 entries");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool heavy = blockIdx.x < a.heavy_items;    // uniform over the workgroup
    const int64_t rows = heavy ? a.heavy_rows : a.n_rows - a.heavy_rows;
    const int64_t item = heavy ? (int64_t)blockIdx.x : ((int64_t)blockIdx.x - a.heavy_items) * kHeavyWaves + wave;
    if (item >= rows * a.nslab) return;
    int64_t slot;
    int slab;
    if (a.slab_major) { slab = (int)(item / rows); slot = item % rows; }
    else              { slot = item / a.nslab; slab = (int)(item % a.nslab); }
    const int v = __builtin_amdgcn_readfirstlane(a.order[heavy ? slot : a.heavy_rows + slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);
    const int d = a.set_deg ? a.set_deg[v] : hi - lo;

    const int64_t col0 = (int64_t)slab * (64 * VEC * NC) + lane * VEC;
    bool act[NC];
    float acc[NC][VEC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        act[c] = col0 + c * 64 * VEC < a.F;
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc[c][k] = MAXOP ? -INFINITY : 0.0f;
    }
    float sum[NC][VEC], tile[NC][VEC];                // (LEVELS)
    int batches = 0;
    auto raise = [&](float (&from)[NC][VEC], float (&to)[NC][VEC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                to[c][k] += from[c][k];
                from[c][k] = 0.0f;
            }
    };
    if constexpr (LEVELS) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) sum[c][k] = tile[c][k] = 0.0f;
    }
    const float* zl = a.Z + col0;
    const bool weighted = a.wsrc != nullptr;

    const int first = heavy ? 64 * wave : 0, step = heavy ? 64 * kHeavyWaves : 64;
    for (int base = lo + first; base < hi; base += step) {
        const int e = base + lane;
        const int my_u = e < hi ? a.col_idx[e] : 0;
        const float my_w = weighted ? (e < hi ? a.wsrc[my_u] : 0.0f) : 1.0f;
        const int cnt = min(64, hi - base);
        auto batch = [&](int j, auto whole_tag) {
            constexpr bool WHOLE = decltype(whole_tag)::value;
            float z[U][NC][VEC];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                if (!WHOLE && j + t >= cnt) break;
                const int u = bcast_i(my_u, j + t);
                const float* zr = zl + (int64_t)u * a.ldz;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (act[c]) load_row<VEC>(zr + c * 64 * VEC, z[t][c]);
            }
#pragma unroll
            for (int t = 0; t < U; ++t) {
                if (!WHOLE && j + t >= cnt) break;
                const float w = bcast_f(my_w, j + t);
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (act[c]) {
#pragma unroll
                        for (int k = 0; k < VEC; ++k) {
                            float& x = LEVELS ? sum[c][k] : acc[c][k];
                            x = MAXOP ? fmaxf(x, z[t][c][k]) : fmaf(w, z[t][c][k], x);
                        }
                    }
            }
            if constexpr (LEVELS) {
                ++batches;                            // (uniform)
                if (batches % 2 == 0) raise(sum, tile);
                if (batches % 16 == 0) raise(tile, acc);
            }
        };
        int j = 0;
        for (; j + U <= cnt; j += U) batch(j, std::true_type{});
        if (j < cnt) batch(j, std::false_type{});
    }
    if constexpr (LEVELS) {
        raise(sum, tile);
        raise(tile, acc);
    }

    __shared__ float red[kHeavyWaves][NC * VEC][64];
    if (heavy) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) red[wave][c * VEC + k][lane] = acc[c][k];
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                float s = red[0][c * VEC + k][lane];
#pragma unroll
                for (int w = 1; w < kHeavyWaves; ++w)
                    s = MAXOP ? fmaxf(s, red[w][c * VEC + k][lane]) : s + red[w][c * VEC + k][lane];
                acc[c][k] = s;
            }
    }

    float* orow = a.out + (int64_t)v * a.ldo;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (!act[c]) continue;
        const int64_t col = col0 + c * 64 * VEC;
        const int valid = (int)min((int64_t)VEC, a.F - col);
        float r[VEC];
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            float x = acc[c][k];
            if (MAXOP) x = d > 0 ? x : 0.0f;                     // empty neighbourhood: zero
            else if (a.scale == SCALE_MEAN) x = d > 0 ? x / (float)d : 0.0f;
            else if (a.scale == SCALE_GCN) x = x * a.dinv[v];
            r[k] = x;
        }
        store_row<VEC>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
        if (a.copy_self) {
            float zs[VEC];
            load_row<VEC>(a.Z + (int64_t)v * a.ldz + col, zs);
            store_row<VEC>(orow + col, zs, valid, a.self_vec != 0);
        }
    }
}

// ---------------------------------------------------------------------------
// sum / mean / gcn_sym with narrow column slabs ("grouped gather").
//
// When one column slab of the whole table (N rows x SW columns) is small
// enough to stay in the last-level caches, walking the graph once per slab
// turns most gathers into cache hits instead of HBM reads.  A slab is
// SW = 4*LPG columns wide; a wave splits into G = 64/LPG groups of LPG lanes,
// each lane owning one float4 of the slab, and every wave-wide load fetches the
// slab of G different neighbours (G x SW x 4 = 1 KiB per instruction, as in the
// full-row kernel).  Neighbour ids are loaded 64 at a time and handed to the
// groups with a wave shuffle; the groups' partial sums are combined with
// xor-shuffles when the row is done.  Same ownership rules as above: one wave
// (or one workgroup for long rows) writes an output element, in a fixed order.
// ---------------------------------------------------------------------------
// One 64-edge tile of the grouped gather.  Each lane holds one neighbour: the byte offset of its row (kNoEntry past the
// end of a partial tile) or, for tables of 4 GiB and more, its id, and its gcn weight.  Step t hands entry t*G + g to
// group g with a wave shuffle.  All loads of a batch of up to 8 steps are issued before their FMAs, and nothing in the
// batch branches.
//   OFF32: every row offset fits 32 bits, so the table is a buffer and what does not exist fetches nothing (load_entry);
//   otherwise lanes past the end fetch a valid address (id 0) and have the loaded values replaced by zero, and lanes past
//   the row width fetch the last valid vector of the slab and never store
// Without weights the masked form of both, with one for whole tiles that tests nothing, takes 72 registers instead of 60 and
// so a workgroup less per CU: long rows of the Reddit-shaped graph 88.7 us per range and slab group so, 86.7 as offsets; where
// a wave has one or two tiles (100,000 nodes and 10 million entries, 256 columns) 35.2 so and 37.0.
template <int LPG, bool WEIGHTED, bool OFF32>
__device__ __forceinline__ void grouped_tile(const char* zbase, table_t table, uint32_t colbytes, int64_t rowbytes,
                                             uint32_t my_off, int my_u, float my_w, int cnt, int g,
                                             float (&acc)[4])
{
    constexpr int G = 64 / LPG;
    constexpr int STEPS = 64 / G;
    constexpr int U = STEPS < 8 ? STEPS : 8;
#pragma unroll
    for (int t0 = 0; t0 < STEPS; t0 += U) {
        if (t0 * G >= cnt) break;
        f32x4 z[U];
        float w[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int j = (t0 + t) * G + g;
            if constexpr (OFF32) {
                z[t] = __builtin_bit_cast(f32x4, load_entry(table, (uint32_t)__shfl((int)my_off, j, 64), colbytes));
            } else {
                const int u = __shfl(my_u, j, 64);
                z[t] = *reinterpret_cast<const f32x4*>(zbase + (int64_t)u * rowbytes + colbytes);
                const bool ok = j < cnt;
                z[t].x = ok ? z[t].x : 0.0f;
                z[t].y = ok ? z[t].y : 0.0f;
                z[t].z = ok ? z[t].z : 0.0f;
                z[t].w = ok ? z[t].w : 0.0f;
            }
            if constexpr (WEIGHTED) w[t] = __shfl(my_w, j, 64);
        }
#pragma unroll
        for (int t = 0; t < U; ++t) {
            if constexpr (WEIGHTED) {
                acc[0] = fmaf(w[t], z[t].x, acc[0]);
                acc[1] = fmaf(w[t], z[t].y, acc[1]);
                acc[2] = fmaf(w[t], z[t].z, acc[2]);
                acc[3] = fmaf(w[t], z[t].w, acc[3]);
            } else {
                acc[0] += z[t].x;
                acc[1] += z[t].y;
                acc[2] += z[t].z;
                acc[3] += z[t].w;
            }
        }
    }
}

// Long rows of the narrow-slab scheme: the NW waves of a workgroup share one
// (row, slab) item, take interleaved 64-edge tiles and combine through LDS.
template <int LPG, int NW, bool WEIGHTED, bool OFF32>
__global__ __launch_bounds__(64 * NW) void agg_grouped_kernel(AggArgs a)
{
    constexpr int SW = 4 * LPG;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t items = a.row_count * a.nslab;
    const int64_t item = (int64_t)blockIdx.x;
    if (item >= items) return;        // uniform over the workgroup
    int64_t slot;
    int slab;
    if (a.slab_major) { slab = (int)(item / a.row_count); slot = item % a.row_count; }
    else              { slot = item / a.nslab; slab = (int)(item % a.nslab); }
    const int v = __builtin_amdgcn_readfirstlane(a.order[a.row_begin + slot]);
    int lo, hi;
    if (a.part_ptr) {
        lo = __builtin_amdgcn_readfirstlane(a.part_ptr[(int64_t)a.part_lo * a.n_rows + a.row_begin + slot]);
        hi = __builtin_amdgcn_readfirstlane(a.part_ptr[(int64_t)a.part_hi * a.n_rows + a.row_begin + slot]);
    } else {
        lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
        hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);
    }

    const int li = lane % LPG, g = lane / LPG;
    const int64_t col = (int64_t)slab * SW + li * 4;
    const bool act = col < a.F;
    const bool writer = act && g == 0 && wave == 0;
    const int valid = (int)min((int64_t)4, a.F - col);
    const char* zbase = reinterpret_cast<const char*>(a.Z);
    const table_t table = buffer_table(a.Z, OFF32 ? a.table_bytes : 0u);
    const uint32_t colbytes = act ? (uint32_t)(col * 4) : OFF32 ? kNoEntry : (uint32_t)((a.F - 1) / 4 * 16);
    const int64_t rowbytes = a.ldz * 4;
    float* orow = a.out + (int64_t)v * a.ldo;

    // running sum over the source ranges walked so far (written by the previous launch)
    float prev[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!a.first && writer) {
        if ((a.out_vec || a.out_half) && valid >= 4) {
            const f32x2 t0 = *reinterpret_cast<const f32x2*>(orow + a.ocol + col);
            const f32x2 t1 = *reinterpret_cast<const f32x2*>(orow + a.ocol + col + 2);
            prev[0] = t0.x; prev[1] = t0.y; prev[2] = t1.x; prev[3] = t1.y;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < valid) prev[k] = orow[a.ocol + col + k];
        }
    }

    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    // the ids (and weights) of a wave's next tile are requested before the current tile's rows
    int nxt_u = lo + 64 * wave + lane < hi ? a.col_idx[lo + 64 * wave + lane] : 0;
    float nxt_w = WEIGHTED ? (lo + 64 * wave + lane < hi ? a.wsrc[nxt_u] : 0.0f) : 1.0f;
    for (int base = lo + 64 * wave; base < hi; base += 64 * NW) {
        const int my_u = nxt_u;
        const float my_w = nxt_w;
        {
            const int en = base + 64 * NW + lane;
            nxt_u = en < hi ? a.col_idx[en] : 0;
            nxt_w = WEIGHTED ? (en < hi ? a.wsrc[nxt_u] : 0.0f) : 1.0f;
        }
        const int cnt = min(64, hi - base);
        const uint32_t my_off = base + lane < hi ? (uint32_t)my_u * (uint32_t)rowbytes : kNoEntry;
        grouped_tile<LPG, WEIGHTED, OFF32>(zbase, table, colbytes, rowbytes, my_off, my_u, my_w, cnt, g, acc);
    }
    // combine the lane groups, then the waves (in wave order)
#pragma unroll
    for (int m = LPG; m < 64; m <<= 1)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += __shfl_xor(acc[k], m, 64);
    __shared__ float red[NW][4][LPG];
    if (g == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) red[wave][k][li] = acc[k];
    }
    __syncthreads();
    if (!writer) return;
    const int d = (a.last && a.scale == SCALE_MEAN) ? a.deg[v] : 0;      // only the mean's last range needs it
    float out_v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float x = red[0][k][li];
#pragma unroll
        for (int w = 1; w < NW; ++w) x += red[w][k][li];
        x += prev[k];
        if (a.last) {
            if (a.scale == SCALE_MEAN) x = d > 0 ? x / (float)d : 0.0f;
            else if (a.scale == SCALE_GCN) x = x * a.dinv[v];
        }
        out_v[k] = x;
    }
    store_row<4>(orow + a.ocol + col, out_v, valid, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self && a.first) {
        float zs[4];
        load_row<4>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_row<4>(orow + col, zs, valid, a.self_vec != 0);
    }
}

// ---------------------------------------------------------------------------
// Narrow slabs, ordinary rows: one ROW per lane group.
//
// The G = 64/LPG lane groups of a wave take G consecutive rows of the schedule
// (similar lengths, since the schedule is sorted by degree) and walk their
// neighbour lists in lock step: every wave-wide load fetches the slab of one
// neighbour for each of the G rows.  No cross-group reduction is needed, the
// running-sum read, the scaling and the store are one wave-wide operation for
// G rows, and the per-row bookkeeping is shared — which is what matters once a
// row's share of one source range is only a few dozen entries long.
// Neighbour ids are fetched 8 LPG at a time per group (eight per lane: whole
// cache lines of col_idx, a block ahead) and handed round inside the group
// with ds_bpermute.
// ---------------------------------------------------------------------------
template <int LPG, bool WEIGHTED, bool OFF32>
__global__ __launch_bounds__(64 * kLightWaves) void agg_rowgroup_kernel(AggArgs a)
{
    constexpr int G = 64 / LPG;
    constexpr int SW = 4 * LPG;
    constexpr int U = LPG < 8 ? LPG : 8;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t bundles = (a.row_count + G - 1) / G;
    const int64_t items = bundles * a.nslab;
    const int64_t item = (int64_t)blockIdx.x * kLightWaves + wave;
    if (item >= items) return;
    int64_t bundle;
    int slab;
    if (a.slab_major) { slab = (int)(item / bundles); bundle = item % bundles; }
    else              { bundle = item / a.nslab; slab = (int)(item % a.nslab); }

    const int li = lane % LPG, g = lane / LPG;
    const int64_t slot = bundle * G + g;
    const bool has_row = slot < a.row_count;
    int v = 0, lo = 0, hi = 0;
    if (has_row) {
        v = a.order[a.row_begin + slot];
        if (a.part_ptr) {
            lo = a.part_ptr[(int64_t)a.part_lo * a.n_rows + a.row_begin + slot];
            hi = a.part_ptr[(int64_t)a.part_hi * a.n_rows + a.row_begin + slot];
        } else {
            lo = (int)a.row_ptr[v];
            hi = (int)a.row_ptr[v + 1];
        }
    }
    const int len = hi - lo;
    int maxlen = len, minlen = len;
#pragma unroll
    for (int m = LPG; m < 64; m <<= 1) {
        maxlen = max(maxlen, __shfl_xor(maxlen, m, 64));
        minlen = min(minlen, __shfl_xor(minlen, m, 64));
    }
    maxlen = __builtin_amdgcn_readfirstlane(maxlen);
    minlen = __builtin_amdgcn_readfirstlane(minlen);

    const int64_t col = (int64_t)slab * SW + li * 4;
    const bool act = col < a.F;
    const bool writer = act && has_row;
    const int valid = (int)min((int64_t)4, a.F - col);
    const char* zbase = reinterpret_cast<const char*>(a.Z);
    constexpr bool BUFFER = OFF32 && WEIGHTED;
    const table_t table = buffer_table(a.Z, BUFFER ? a.table_bytes : 0u);
    const uint32_t colbytes = act ? (uint32_t)(col * 4) : BUFFER ? kNoEntry : 0u;
    const int64_t rowbytes = a.ldz * 4;
    float* orow = a.out + (int64_t)v * a.ldo;

    float prev[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!a.first && writer) {
        if (a.out_vec && valid >= 4) {
            const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(orow + a.ocol + col));
            prev[0] = t.x; prev[1] = t.y; prev[2] = t.z; prev[3] = t.w;
        } else if (a.out_half && valid >= 4) {
            const f32x2 t0 = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(orow + a.ocol + col));
            const f32x2 t1 = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(orow + a.ocol + col + 2));
            prev[0] = t0.x; prev[1] = t0.y; prev[2] = t1.x; prev[3] = t1.y;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < valid) prev[k] = orow[a.ocol + col + k];
        }
    }

    const int gaddr = (lane - li) * 4;      // ds_bpermute byte address of this group's lane 0
    // Neighbour ids: every lane of a group fetches eight consecutive ids at a time, so a group reads col_idx in
    // whole cache lines (8 LPG entries: two lines for LPG = 8; measured: 4 per lane 1.4 % slower, 16 per lane
    // 0.6 % slower) instead of one 32-byte piece per LPG entries — the id loads were one L2 request in nine of a
    // kernel that is bound by L2 requests.  Entry e of such a block sits in component e % 8 of the group's
    // lane e / 8.
    constexpr int IPL = 8;
    constexpr int BLOCK = IPL * LPG;
    typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));      // 4-byte aligned 16-byte load
    int nxt_u[IPL];
    float nxt_w[IPL];
    constexpr int NONE = BUFFER ? -1 : 0;   // the id past a row's end: becomes kNoEntry, or is masked
    auto fetch_ids = [&](int first) {       // entries first + IPL li .. of this group's row
        const int nb = first + IPL * li;
        if (nb + IPL <= len) {
#pragma unroll
            for (int k = 0; k < IPL; k += 4) {
                const i32x4u t = *reinterpret_cast<const i32x4u*>(a.col_idx + lo + nb + k);
                nxt_u[k] = t.x; nxt_u[k + 1] = t.y; nxt_u[k + 2] = t.z; nxt_u[k + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < IPL; ++k) nxt_u[k] = nb + k < len ? a.col_idx[lo + nb + k] : NONE;
        }
        if constexpr (WEIGHTED) {
#pragma unroll
            for (int k = 0; k < IPL; ++k) nxt_w[k] = nb + k < len ? a.wsrc[nxt_u[k]] : 0.0f;
        }
    };
    fetch_ids(0);
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0; s0 < maxlen; s0 += BLOCK) {
        int my_u[IPL];
        float my_w[IPL];
        uint32_t my_off[IPL];
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            my_u[k] = nxt_u[k];
            my_w[k] = WEIGHTED ? nxt_w[k] : 0.0f;
            my_off[k] = BUFFER && my_u[k] < 0 ? kNoEntry : OFF32 ? (uint32_t)my_u[k] * (uint32_t)rowbytes : 0u;
        }
        fetch_ids(s0 + BLOCK);              // the next block, a whole block ahead of its use
        // steps of U entries; the gathers of step st + 1 are issued before those of step st are added up, so a
        // wave has up to 2 U row pieces in flight (two register sets, picked by the parity of the unrolled step)
        constexpr int T = BLOCK / U;
        f32x4 z[2][U];
        float w[2][U];
        // e0: first entry of the step in the block, c0: the same counted from the start of the row's share.  What a
        // group does not have (a shorter row of the bundle, columns past the row width) is not fetched: the kernel keeps
        // the address units busy 96 % of its time, and a sixth of the gathers of a bundle would be such fillers.  With
        // weights, whose gathers and permutes fill the vector units too, it is an offset past the table's end (F = 256
        // gcn_sym on the Reddit-shaped graph 9.42 -> 8.84 ms); without, lanes that are switched off are the cheaper
        // (F = 602 mean 14.57 ms, 14.67 as offsets).
        auto issue = [&](int e0, int c0, f32x4 (&zz)[U], float (&ww)[U]) {
            const bool all = act && c0 + U <= minlen && has_row;       // no filler in this step for this lane
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int e = e0 + t;              // entry of the block: lane e / IPL, component e % IPL
                const int from = OFF32 ? (int)my_off[e % IPL] : my_u[e % IPL];
                const int at = __builtin_amdgcn_ds_bpermute(gaddr + 4 * (e / IPL), from);
                if constexpr (BUFFER) {
                    zz[t] = __builtin_bit_cast(f32x4, load_entry(table, (uint32_t)at, colbytes));
                } else {
                    const char* src = OFF32 ? zbase + ((uint32_t)at + colbytes) : zbase + (int64_t)at * rowbytes + colbytes;
                    zz[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    if (all || (act && c0 + t < len)) zz[t] = *reinterpret_cast<const f32x4*>(src);
                }
                if constexpr (WEIGHTED)
                    ww[t] = __int_as_float(__builtin_amdgcn_ds_bpermute(gaddr + 4 * (e / IPL), __float_as_int(my_w[e % IPL])));
            }
        };
        issue(0, s0, z[0], w[0]);
#pragma unroll
        for (int st = 0; st < T; ++st) {
            const int c0 = s0 + st * U;
            if (c0 >= maxlen) break;                   // (uniform)
            if (st + 1 < T && c0 + U < maxlen) issue((st + 1) * U, c0 + U, z[(st + 1) & 1], w[(st + 1) & 1]);
            f32x4 (&zc)[U] = z[st & 1];
            float (&wc)[U] = w[st & 1];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                if constexpr (WEIGHTED) {
                    acc[0] = fmaf(wc[t], zc[t].x, acc[0]);
                    acc[1] = fmaf(wc[t], zc[t].y, acc[1]);
                    acc[2] = fmaf(wc[t], zc[t].z, acc[2]);
                    acc[3] = fmaf(wc[t], zc[t].w, acc[3]);
                } else {
                    acc[0] += zc[t].x;
                    acc[1] += zc[t].y;
                    acc[2] += zc[t].z;
                    acc[3] += zc[t].w;
                }
            }
        }
    }
    if (!writer) return;
    const int d = (a.last && a.scale == SCALE_MEAN) ? a.deg[v] : 0;      // only the mean's last range needs it
    float out_v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float x = acc[k] + prev[k];
        if (a.last) {
            if (a.scale == SCALE_MEAN) x = d > 0 ? x / (float)d : 0.0f;
            else if (a.scale == SCALE_GCN) x = x * a.dinv[v];
        }
        out_v[k] = x;
    }
    if (a.out_vec && valid >= 4) {
        f32x4 t = {out_v[0], out_v[1], out_v[2], out_v[3]};
        __builtin_nontemporal_store(t, reinterpret_cast<f32x4*>(orow + a.ocol + col));
    } else if (a.out_half && valid >= 4) {
        __builtin_nontemporal_store(f32x2{out_v[0], out_v[1]}, reinterpret_cast<f32x2*>(orow + a.ocol + col));
        __builtin_nontemporal_store(f32x2{out_v[2], out_v[3]}, reinterpret_cast<f32x2*>(orow + a.ocol + col + 2));
    } else {
        store_row<4>(orow + a.ocol + col, out_v, valid, false);
    }
    if (a.copy_self && a.first) {
        float zs[4];
        load_row<4>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_row<4>(orow + col, zs, valid, a.self_vec != 0);
    }
}

// A lane's four columns from `col` on, moved back to end with the row where they would reach over its end: nothing past a row is
// read, at whatever pitch rows lie.  The lane then stores only those from `col` on (store_own).  Rows of fewer than four columns
// are read with their padding.
__device__ __forceinline__ int64_t own_columns(int64_t col, int64_t F) { return F >= 4 ? min(col, F - 4) : col; }

// ---------------------------------------------------------------------------
// sum / mean / gcn_sym of rows, or slabs, of 4 P columns: P = 8, 16 or 32 lanes of four floats hold a row, and the R = 64 / P
// groups of a wave walk R rows of the schedule, or shares of one long row, in lock step (EntryWalk).  Long rows first in every
// slab, one per workgroup, their shares added up over the groups and then over the waves in order; one launch for both classes.
// Bound by memory latency on small graphs, where R rows wait together, and by the gathered lines on large ones (2,449,029
// nodes of 50 entries, 32 columns 2,330 us, 6.7 TB/s of lines).  linear_route says where it is taken, and what it measures.
// ---------------------------------------------------------------------------
template <int P, bool WEIGHTED, bool LEVELS>
__global__ __launch_bounds__(64 * kHeavyWaves) void agg_rows_kernel(AggArgs a)
{
    constexpr int U = 8, R = 64 / P, NW = kHeavyWaves, PER = U / 4;    // entries and lanes of a batch
    const int lane = threadIdx.x & 63, li = lane % P, g = lane / P;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t slab = blockIdx.x / a.slab_blocks, block = blockIdx.x % a.slab_blocks;
    const bool heavy = block < a.heavy_rows;          // uniform over the workgroup
    const int64_t first = heavy ? (int64_t)block : a.heavy_rows + ((int64_t)(block - (uint32_t)a.heavy_rows) * NW + wave) * R;
    if (first >= a.n_rows) return;
    const int64_t slot = heavy ? first : first + g;
    const bool have = slot < a.n_rows;
    int v = 0, d = 0;
    uint32_t lo = 0, hi = 0;
    if (have) {
        v = a.order[slot];
        lo = (uint32_t)a.row_ptr[v];
        hi = (uint32_t)a.row_ptr[v + 1];
        if constexpr (!WEIGHTED) d = a.set_deg ? a.set_deg[v] : (int)(hi - lo);
    }
    typedef EntryWalk<P, WEIGHTED> Walk;
    Walk walk;
    const uint32_t rowbytes = (uint32_t)(a.ldz * 4);
    int batches = heavy ? walk.start(a.col_idx, lo + Walk::kTile * (wave * R + g), hi, Walk::kTile * NW * R, rowbytes)
                        : walk.start(a.col_idx, lo, hi, Walk::kTile, rowbytes);
    batches = (batches + PER - 1) / PER;
    // the weights of the current tile's entries, requested with its first gathers, and of the one before it
    float w_cur[WEIGHTED ? 4 : 1], w_prev[WEIGHTED ? 4 : 1];
    auto weights = [&]() {
        if constexpr (WEIGHTED) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w_prev[k] = w_cur[k];
                w_cur[k] = walk.id[k] != kNoEntry ? a.wsrc[walk.id[k]] : 0.0f;
            }
        }
    };
    if constexpr (WEIGHTED) {
#pragma unroll
        for (int k = 0; k < 4; ++k) w_cur[k] = 0.0f;
    }
    weights();

    const bool act = (int)slab * (4 * P) + li * 4 < a.F;
    const int col = (int)own_columns((int)slab * (4 * P) + li * 4, a.F);
    const int skip = (int)slab * (4 * P) + li * 4 - col, valid = min(4, (int)a.F);
    const table_t table = buffer_table(a.Z, a.table_bytes);
    const uint32_t colbytes = act ? (uint32_t)col * 4 : kNoEntry;      // (columns past the row width fetch nothing)
    BatchSums<4, LEVELS> sums;
    f32x4 z[2][U];
    constexpr int kBatches = P / PER;                                   // of a tile
    auto issue = [&](int k, f32x4 (&zz)[U]) {                           // batch k
        const int j = k % kBatches;
        if (j == 0 && k > 0) {
            walk.take();
            weights();
        }
#pragma unroll
        for (int t = 0; t < U; ++t)
            zz[t] = __builtin_bit_cast(f32x4, load_entry(table, walk.at(j * PER + t / 4, t % 4), colbytes));
    };
    auto consume = [&](int k, const f32x4 (&zz)[U], float (&sum)[4]) {  // sum of batch k
        if constexpr (WEIGHTED) {
            // (the next tile's weights have taken the place of this one's when its last batch is added up)
            const bool old = (k + 1) % kBatches == 0 && k + 1 < batches;
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const float w = __int_as_float(__builtin_amdgcn_ds_bpermute(walk.gaddr + 4 * (k % kBatches * PER + t / 4),
                                                                            __float_as_int(old ? w_prev[t % 4] : w_cur[t % 4])));
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] = t == 0 ? w * zz[t][c] : fmaf(w, zz[t][c], sum[c]);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                sum[c] = ((zz[0][c] + zz[1][c]) + (zz[2][c] + zz[3][c])) + ((zz[4][c] + zz[5][c]) + (zz[6][c] + zz[7][c]));
        }
    };
    float sum[4];
    if (batches > 0) issue(0, z[0]);
    for (int k = 0; k < batches; k += 2) {
        if (k + 1 < batches) issue(k + 1, z[1]);
        consume(k, z[0], sum);
        sums.even(sum);
        if (k + 1 >= batches) {
            sums.last_even();
            break;
        }
        if (k + 2 < batches) issue(k + 2, z[0]);
        consume(k + 1, z[1], sum);
        sums.odd(k, sum);
    }
    sums.flush();
    float (&acc)[4] = sums.all;

    if (heavy) {
#pragma unroll
        for (int b = P; b < 64; b <<= 1)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] += __shfl_xor(acc[k], b, 64);
        __shared__ float red[NW][4][P];
        if (g == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) red[wave][k][li] = acc[k];
        }
        __syncthreads();
        if (wave != 0 || g != 0) return;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            acc[k] = red[0][k][li];
#pragma unroll
            for (int w = 1; w < NW; ++w) acc[k] += red[w][k][li];
        }
    }
    if (!have || !act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    float r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float x = acc[k];
        if constexpr (WEIGHTED) x = x * a.dinv[v];
        else if (a.scale == SCALE_MEAN) x = d > 0 ? x / (float)d : 0.0f;
        r[k] = x;
    }
    store_own(orow + a.ocol + col, r, skip, valid, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self) {
        const f32x4u t = *reinterpret_cast<const f32x4u*>(a.Z + (int64_t)v * a.ldz + col);
        const float zs[4] = {t.x, t.y, t.z, t.w};
        store_own(orow + col, zs, skip, valid, a.self_vec != 0);
    }
}

// ---------------------------------------------------------------------------
// attention scores  el[v,h] = <a_src[h], z_v,h>,  er[v,h] = <a_dst[h], z_v,h>
// one wave per node; padded heads (h >= heads) get 0
// ---------------------------------------------------------------------------
template <int HP>
__global__ __launch_bounds__(256) void gat_scores_kernel(
    int64_t N, int64_t F, int heads, int Dh, const float* Z, int64_t ldz,
    const float* __restrict__ a_src, const float* __restrict__ a_dst,
    float* el, int64_t el_stride, float* __restrict__ er)
{
    const int lane = threadIdx.x & 63;
    const int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= N) return;
    float ps[HP], pd[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) { ps[h] = 0.0f; pd[h] = 0.0f; }
    for (int64_t c = lane; c < F; c += 64) {
        const float z = Z[v * ldz + c];
        const int h = (int)(c / Dh);
        const float s = z * a_src[c], t = z * a_dst[c];   // a_* are [heads, Dh] = flat [F]
#pragma unroll
        for (int i = 0; i < HP; ++i) {
            ps[i] += (h == i) ? s : 0.0f;
            pd[i] += (h == i) ? t : 0.0f;
        }
    }
#pragma unroll
    for (int h = 0; h < HP; ++h) {
        const float s = wave_sum(ps[h]), t = wave_sum(pd[h]);
        if (lane == 0) { el[v * el_stride + h] = s; er[v * HP + h] = t; }
    }
}

// The same scores with 16-byte loads: 16 lanes per node (four nodes per wave), each lane walks the row
// in float4 steps of 64 columns; the per-head partial sums are reduced over the 16 lanes of a node.
// Needs 16-byte aligned rows and F % 4 == 0.
template <int HP>
__global__ __launch_bounds__(256) void gat_scores_vec_kernel(
    int64_t N, int64_t F, int heads, int Dh, const float* Z, int64_t ldz,
    const float* __restrict__ a_src, const float* __restrict__ a_dst,
    float* el, int64_t el_stride, float* __restrict__ er)
{
    const int li = threadIdx.x & 15;
    const int64_t v = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const bool have = v < N;
    const int64_t vv = have ? v : N - 1;                 // idle groups repeat the last node (nothing stored)
    float ps[HP], pd[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) { ps[h] = 0.0f; pd[h] = 0.0f; }
    const bool whole = Dh % 4 == 0;
    // four row pieces are requested before the first is used (a row of up to 256 columns is one batch)
    for (int64_t c0 = li * 4; c0 < F; c0 += 256) {
        f32x4 zq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = c0 + 64 * q;
            zq[q] = c < F ? *reinterpret_cast<const f32x4*>(Z + vv * ldz + c) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = c0 + 64 * q;
            if (c >= F) break;
            const f32x4 z = zq[q];
            const f32x4 as = *reinterpret_cast<const f32x4*>(a_src + c);
            const f32x4 ad = *reinterpret_cast<const f32x4*>(a_dst + c);
            const float zs[4] = {z.x, z.y, z.z, z.w}, sa[4] = {as.x, as.y, as.z, as.w}, da[4] = {ad.x, ad.y, ad.z, ad.w};
            if (whole) {
                // the four columns lie in one head: one head index and one add per head for the piece
                const int h = (int)c / Dh;
                const float s = ((zs[0] * sa[0] + zs[1] * sa[1]) + zs[2] * sa[2]) + zs[3] * sa[3];
                const float t = ((zs[0] * da[0] + zs[1] * da[1]) + zs[2] * da[2]) + zs[3] * da[3];
#pragma unroll
                for (int i = 0; i < HP; ++i) {
                    ps[i] += (h == i) ? s : 0.0f;
                    pd[i] += (h == i) ? t : 0.0f;
                }
                continue;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int h = ((int)c + k) / Dh;
                const float s = zs[k] * sa[k], t = zs[k] * da[k];
#pragma unroll
                for (int i = 0; i < HP; ++i) {
                    ps[i] += (h == i) ? s : 0.0f;
                    pd[i] += (h == i) ? t : 0.0f;
                }
            }
        }
    }
#pragma unroll
    for (int h = 0; h < HP; ++h) {
#pragma unroll
        for (int m = 8; m >= 1; m >>= 1) {
            ps[h] += __shfl_xor(ps[h], m, 64);
            pd[h] += __shfl_xor(pd[h], m, 64);
        }
    }
    if (have && li == 0) {
#pragma unroll
        for (int h = 0; h < HP; ++h) { el[v * el_stride + h] = ps[h]; er[v * HP + h] = pd[h]; }
    }
}

// ---------------------------------------------------------------------------
// gat_softmax.  HU: every lane's VEC columns lie inside one head (Dh % VEC == 0)
// ---------------------------------------------------------------------------
template <int VEC, int NC, int NW, int HP, bool HU>
__global__ __launch_bounds__(64 * (NW == 1 ? kLightWaves : NW)) void agg_gat_kernel(AggArgs a)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t items = a.row_count * a.nslab;
    const int64_t item = (NW == 1) ? (int64_t)blockIdx.x * kLightWaves + wave : (int64_t)blockIdx.x;
    if (item >= items) return;
    int64_t slot;
    int slab;
    if (a.slab_major) { slab = (int)(item / a.row_count); slot = item % a.row_count; }
    else              { slot = item / a.nslab; slab = (int)(item % a.nslab); }
    const int v = __builtin_amdgcn_readfirstlane(a.order[a.row_begin + slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);

    const int64_t col0 = (int64_t)slab * (64 * VEC * NC) + lane * VEC;
    bool act[NC];
    int hc[NC][HU ? 1 : VEC];      // head of each owned column (clamped for padding columns)
    float acc[NC][VEC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t col = col0 + c * 64 * VEC;
        act[c] = col < a.F;
#pragma unroll
        for (int k = 0; k < (HU ? 1 : VEC); ++k) hc[c][k] = min((int)((col + k) / a.Dh), a.heads - 1);
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc[c][k] = 0.0f;
    }
    const float* zl = a.Z + col0;

    float m[HP], s[HP], erv[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) {
        m[h] = -INFINITY;
        s[h] = 0.0f;
        erv[h] = a.er[(int64_t)v * HP + h];
    }

    for (int base = lo + 64 * (NW == 1 ? 0 : wave); base < hi; base += 64 * NW) {
        const int e = base + lane;
        const bool valid = e < hi;
        const int my_u = valid ? a.col_idx[e] : 0;
        const int cnt = min(64, hi - base);
        float p[HP], scale[HP];
        {
            float elu[HP];
            if constexpr (HP == 4) {
                const f32x4 t = *reinterpret_cast<const f32x4*>(a.el + (int64_t)my_u * a.el_stride);
                elu[0] = t.x; elu[1] = t.y; elu[2] = t.z; elu[3] = t.w;
            } else {
#pragma unroll
                for (int h = 0; h < HP; ++h) elu[h] = a.el[(int64_t)my_u * a.el_stride + h];
            }
#pragma unroll
            for (int h = 0; h < HP; ++h) {
                const float x = elu[h] + erv[h];
                const float sc = valid ? (x > 0.0f ? x : a.slope * x) : -INFINITY;
                const float mn = fmaxf(m[h], wave_max(sc));      // finite: the tile has an edge
                scale[h] = expf(m[h] - mn);                      // exp(-inf) = 0 on the first tile
                p[h] = valid ? expf(sc - mn) : 0.0f;
                s[h] = s[h] * scale[h] + wave_sum(p[h]);
                m[h] = mn;
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) acc[c][k] *= select_head<HP>(scale, hc[c][HU ? 0 : k]);

        int j = 0;
        for (; j + kUnroll <= cnt; j += kUnroll) {
            float z[kUnroll][NC][VEC];
            float w[kUnroll][HP];
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) {
                const int u = bcast_i(my_u, j + t);
#pragma unroll
                for (int h = 0; h < HP; ++h) w[t][h] = bcast_f(p[h], j + t);
                const float* zr = zl + (int64_t)u * a.ldz;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (act[c]) load_row<VEC>(zr + c * 64 * VEC, z[t][c]);
            }
#pragma unroll
            for (int t = 0; t < kUnroll; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (act[c]) {
#pragma unroll
                        for (int k = 0; k < VEC; ++k)
                            acc[c][k] = fmaf(select_head<HP>(w[t], hc[c][HU ? 0 : k]), z[t][c][k], acc[c][k]);
                    }
        }
        for (; j < cnt; ++j) {
            const int u = bcast_i(my_u, j);
            float w[HP];
#pragma unroll
            for (int h = 0; h < HP; ++h) w[h] = bcast_f(p[h], j);
            const float* zr = zl + (int64_t)u * a.ldz;
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (act[c]) {
                    float z[VEC];
                    load_row<VEC>(zr + c * 64 * VEC, z);
#pragma unroll
                    for (int k = 0; k < VEC; ++k)
                        acc[c][k] = fmaf(select_head<HP>(w, hc[c][HU ? 0 : k]), z[k], acc[c][k]);
                }
        }
    }

    if constexpr (NW > 1) {
        // merge the waves' (max, sum, accumulator) triples in wave order
        __shared__ float red[NW][NC * VEC][64];
        __shared__ float mred[NW][HP], sred[NW][HP];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) red[wave][c * VEC + k][lane] = acc[c][k];
        if (lane == 0) {
#pragma unroll
            for (int h = 0; h < HP; ++h) { mred[wave][h] = m[h]; sred[wave][h] = s[h]; }
        }
        __syncthreads();
        if (wave != 0) return;
        float f[NW][HP];
#pragma unroll
        for (int h = 0; h < HP; ++h) {
            float mm = mred[0][h];
#pragma unroll
            for (int w = 1; w < NW; ++w) mm = fmaxf(mm, mred[w][h]);
            float ss = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                // a wave that saw no tile has max -inf and contributes nothing
                f[w][h] = (mred[w][h] == -INFINITY) ? 0.0f : expf(mred[w][h] - mm);
                ss += sred[w][h] * f[w][h];
            }
            s[h] = ss;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                float t = 0.0f;
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    t += red[w][c * VEC + k][lane] * select_head<HP>(f[w], hc[c][HU ? 0 : k]);
                acc[c][k] = t;
            }
    }

    float* orow = a.out + (int64_t)v * a.ldo;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (!act[c]) continue;
        const int64_t col = col0 + c * 64 * VEC;
        const int valid = (int)min((int64_t)VEC, a.F - col);
        float r[VEC];
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            const float den = select_head<HP>(s, hc[c][HU ? 0 : k]);
            r[k] = den > 0.0f ? acc[c][k] / den : 0.0f;
        }
        store_row<VEC>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
        if (a.copy_self) {
            float zs[VEC];
            load_row<VEC>(a.Z + (int64_t)v * a.ldz + col, zs);
            store_row<VEC>(orow + col, zs, valid, a.self_vec != 0);
        }
    }
}

// ---------------------------------------------------------------------------
// gat_softmax, float4 gathers with 32-bit row offsets, software-pipelined.
//
// Same arithmetic as agg_gat_kernel, arranged so that memory latency and the
// score arithmetic overlap: as soon as a tile's neighbour ids are known the
// first batch of feature rows is requested, and the scores, wave reductions and
// exponentials of the tile are computed while those rows are in flight.  The
// per-edge, per-head weights go through a wave-private LDS array, so that a
// lane picks up the weight of its own head with one ds_read whose address is
// an immediate offset (no readlane + select chain per neighbour).  Lanes past
// the end of a tile carry the tile's first neighbour with weight zero, so every
// gather address is valid and nothing in the loop branches per lane.
// One launch covers both classes of rows, as in agg_linear_kernel.
// ---------------------------------------------------------------------------
template <int NC, int NW, int HP, bool HU, bool TRAIN>
__global__ __launch_bounds__(64 * NW) void agg_gat_fast_kernel(AggArgs a)
{
    constexpr int U = 4;
    // TRAIN: the aggregate is accumulated in two parts, entries with a non-positive score (acc) and
    // with a positive score (accp), each with its own weight per edge (zero for the other kind); the
    // backward pass needs the two parts separately, each accurate relative to its own size
    constexpr int WSETS = TRAIN ? 2 : 1;
    // weights of the waves' tiles; in the end the sums of a long row's waves
    __shared__ float lds[NW * WSETS * 64 * (HP > NC * 4 ? HP : NC * 4)];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool heavy = blockIdx.x < a.heavy_items;    // uniform over the workgroup
    const int64_t rows = heavy ? a.heavy_rows : a.n_rows - a.heavy_rows;
    const int64_t item = heavy ? (int64_t)blockIdx.x : ((int64_t)blockIdx.x - a.heavy_items) * NW + wave;
    if (item >= rows * a.nslab) return;
    int64_t slot;
    int slab;
    if (a.slab_major) { slab = (int)(item / rows); slot = item % rows; }
    else              { slot = item / a.nslab; slab = (int)(item % a.nslab); }
    const int v = __builtin_amdgcn_readfirstlane(a.order[heavy ? slot : a.heavy_rows + slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);

    const int64_t col0 = (int64_t)slab * (256 * NC) + lane * 4;
    bool act[NC];
    uint32_t colbytes[NC];
    int hc[NC][HU ? 1 : 4];
    float acc[NC][4], accp[TRAIN ? NC : 1][4];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t col = col0 + c * 256;
        act[c] = col < a.F;
        // lanes past the row width gather the last valid vector instead (never stored)
        colbytes[c] = (uint32_t)((act[c] ? col : ((a.F - 1) / 4) * 4) * 4);
#pragma unroll
        for (int k = 0; k < (HU ? 1 : 4); ++k) hc[c][k] = min((int)((col + k) / a.Dh), a.heads - 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            acc[c][k] = 0.0f;
            if constexpr (TRAIN) accp[c][k] = 0.0f;
        }
    }
    const char* zbase = reinterpret_cast<const char*>(a.Z);
    const uint32_t rowbytes = (uint32_t)(a.ldz * 4);
    float* myw = lds + wave * (WSETS * HP * 64);
    float* mywp = myw + (WSETS - 1) * HP * 64;

    // sp, sn: the parts of s from entries with a positive / non-positive score (kept apart so that a
    // share that is structurally zero comes out as an exact zero)
    float m[HP], s[HP], sp[TRAIN ? HP : 1], sn[TRAIN ? HP : 1], erv[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) {
        m[h] = -INFINITY;
        s[h] = 0.0f;
        if constexpr (TRAIN) { sp[h] = 0.0f; sn[h] = 0.0f; }
        erv[h] = a.er ? a.er[(int64_t)v * HP + h] : 0.0f;
    }
    // no table of destination scores: this row's come from the row itself.  The row is requested here and
    // used in the first tile, behind that tile's gathers, so that its latency is not one more step of the chain.
    f32x4 zself[NC];
    if (!a.er) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            zself[c] = *reinterpret_cast<const f32x4*>(zbase + (uint32_t)v * rowbytes + colbytes[c]);
    }
    const int base0 = lo + (heavy ? 64 * wave : 0), step = heavy ? 64 * NW : 64;

    for (int base = base0; base < hi; base += step) {
        const int e = base + lane;
        const bool valid = e < hi;
        const int cnt = min(64, hi - base);
        int my_u = valid ? a.col_idx[e] : 0;
        my_u = valid ? my_u : bcast_i(my_u, 0);          // lane 0 is always valid
        const int my_off = (int)((uint32_t)my_u * rowbytes);

        // first batch of rows is requested before the scores are computed
        f32x4 zq[U][NC];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const uint32_t off = (uint32_t)bcast_i(my_off, t);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                zq[t][c] = *reinterpret_cast<const f32x4*>(zbase + off + colbytes[c]);
        }

        float elu[HP];
        if constexpr (HP == 4) {
            const f32x4 t = *reinterpret_cast<const f32x4*>(a.el + (int64_t)my_u * a.el_stride);
            elu[0] = t.x; elu[1] = t.y; elu[2] = t.z; elu[3] = t.w;
        } else {
#pragma unroll
            for (int h = 0; h < HP; ++h) elu[h] = a.el[(int64_t)my_u * a.el_stride + h];
        }
        if (!a.er && base == base0) {          // (uniform)
            float pd[HP];
#pragma unroll
            for (int h = 0; h < HP; ++h) pd[h] = 0.0f;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (!act[c]) continue;
                const f32x4 ad = *reinterpret_cast<const f32x4*>(a.er_from + col0 + c * 256);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float t = zself[c][k] * ad[k];
                    const int hk = hc[c][HU ? 0 : k];
#pragma unroll
                    for (int h = 0; h < HP; ++h) pd[h] += hk == h ? t : 0.0f;
                }
            }
            wave_sum(pd);
#pragma unroll
            for (int h = 0; h < HP; ++h) erv[h] = pd[h];
        }
        float scale[HP];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // earlier reads of wl are done
        // Four heads side by side: one after the other, a tile's reductions are a chain of up to 96 dependent moves through
        // LDS, in which a wave with few others beside it stands still, and how much of it the compiler interleaves changes
        // with the code around it (rounds of 188 columns: 3,000 nodes of 150 entries 61.2 -> 57.2 us, 7,687 of 194
        // 121 -> 115).  Eight side by side take one register too many for a fifth wave.
#pragma unroll
        for (int h0 = 0; h0 < HP; h0 += 4) {
            float x[4], top[4], pe[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[i] = elu[h0 + i] + erv[h0 + i];
                pe[i] = top[i] = valid ? (x[i] > 0.0f ? x[i] : a.slope * x[i]) : -INFINITY;
            }
            wave_max(top);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float mn = fmaxf(m[h0 + i], top[i]);
                scale[h0 + i] = expf(m[h0 + i] - mn);
                pe[i] = valid ? expf(pe[i] - mn) : 0.0f;
                m[h0 + i] = mn;
            }
            if constexpr (TRAIN) {
                float pp[4], pn[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pp[i] = x[i] > 0.0f ? pe[i] : 0.0f;
                    pn[i] = x[i] > 0.0f ? 0.0f : pe[i];
                    myw[(h0 + i) * 64 + lane] = pn[i];
                    mywp[(h0 + i) * 64 + lane] = pp[i];
                }
                wave_sum(pp);
                wave_sum(pn);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sp[h0 + i] = sp[h0 + i] * scale[h0 + i] + pp[i];
                    sn[h0 + i] = sn[h0 + i] * scale[h0 + i] + pn[i];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) myw[(h0 + i) * 64 + lane] = pe[i];
            }
            wave_sum(pe);
#pragma unroll
            for (int i = 0; i < 4; ++i) s[h0 + i] = s[h0 + i] * scale[h0 + i] + pe[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (base != base0) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float f = select_head<HP>(scale, hc[c][HU ? 0 : k]);
                    acc[c][k] *= f;
                    if constexpr (TRAIN) accp[c][k] *= f;
                }
        }

        for (int j = 0; j < cnt; j += U) {
            // request the next batch, then consume the current one
            f32x4 zn[U][NC];
            const bool more = j + U < cnt;
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t off = (uint32_t)bcast_i(my_off, (j + U + t) & 63);
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        zn[t][c] = *reinterpret_cast<const f32x4*>(zbase + off + colbytes[c]);
                }
            }
#pragma unroll
            for (int t = 0; t < U; ++t) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if constexpr (HU) {
                        const float w = myw[hc[c][0] * 64 + j + t];
                        acc[c][0] = fmaf(w, zq[t][c].x, acc[c][0]);
                        acc[c][1] = fmaf(w, zq[t][c].y, acc[c][1]);
                        acc[c][2] = fmaf(w, zq[t][c].z, acc[c][2]);
                        acc[c][3] = fmaf(w, zq[t][c].w, acc[c][3]);
                        if constexpr (TRAIN) {
                            const float wq = mywp[hc[c][0] * 64 + j + t];
                            accp[c][0] = fmaf(wq, zq[t][c].x, accp[c][0]);
                            accp[c][1] = fmaf(wq, zq[t][c].y, accp[c][1]);
                            accp[c][2] = fmaf(wq, zq[t][c].z, accp[c][2]);
                            accp[c][3] = fmaf(wq, zq[t][c].w, accp[c][3]);
                        }
                    } else {
                        acc[c][0] = fmaf(myw[hc[c][0] * 64 + j + t], zq[t][c].x, acc[c][0]);
                        acc[c][1] = fmaf(myw[hc[c][1] * 64 + j + t], zq[t][c].y, acc[c][1]);
                        acc[c][2] = fmaf(myw[hc[c][2] * 64 + j + t], zq[t][c].z, acc[c][2]);
                        acc[c][3] = fmaf(myw[hc[c][3] * 64 + j + t], zq[t][c].w, acc[c][3]);
                        if constexpr (TRAIN) {
                            accp[c][0] = fmaf(mywp[hc[c][0] * 64 + j + t], zq[t][c].x, accp[c][0]);
                            accp[c][1] = fmaf(mywp[hc[c][1] * 64 + j + t], zq[t][c].y, accp[c][1]);
                            accp[c][2] = fmaf(mywp[hc[c][2] * 64 + j + t], zq[t][c].z, accp[c][2]);
                            accp[c][3] = fmaf(mywp[hc[c][3] * 64 + j + t], zq[t][c].w, accp[c][3]);
                        }
                    }
                }
            }
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t)
#pragma unroll
                    for (int c = 0; c < NC; ++c) zq[t][c] = zn[t][c];
            }
        }
    }

    if (heavy) {
        typedef float sums_t[NC * 4 * WSETS][64];
        sums_t* red = reinterpret_cast<sums_t*>(lds);
        __syncthreads();                                 // every wave is done with its weights
        __shared__ float mred[NW][HP], sred[NW][HP], spred[NW][HP], snred[NW][HP], fred[NW][HP];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                red[wave][c * 4 + k][lane] = acc[c][k];
                if constexpr (TRAIN) red[wave][NC * 4 + c * 4 + k][lane] = accp[c][k];
            }
        if (lane == 0) {
#pragma unroll
            for (int h = 0; h < HP; ++h) {
                mred[wave][h] = m[h];
                sred[wave][h] = s[h];
                if constexpr (TRAIN) { spred[wave][h] = sp[h]; snred[wave][h] = sn[h]; }
            }
        }
        __syncthreads();
        if (wave != 0) return;
        // every wave's factor per head, through LDS: as a register array it took 144 bytes of scratch per lane, and the
        // registers of the save mode kernel from 116 to 142, also for the short rows
        if (lane < NW * HP) {
            const int w = lane / HP, h = lane % HP;
            float mm = mred[0][h];
#pragma unroll
            for (int o = 1; o < NW; ++o) mm = fmaxf(mm, mred[o][h]);
            fred[w][h] = (mred[w][h] == -INFINITY) ? 0.0f : expf(mred[w][h] - mm);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int h = 0; h < HP; ++h) {
            float mm = mred[0][h];
            float ss = 0.0f, pp = 0.0f, nn = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                mm = fmaxf(mm, mred[w][h]);
                ss += sred[w][h] * fred[w][h];
                if constexpr (TRAIN) { pp += spred[w][h] * fred[w][h]; nn += snred[w][h] * fred[w][h]; }
            }
            s[h] = ss;
            m[h] = mm;
            if constexpr (TRAIN) { sp[h] = pp; sn[h] = nn; }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float t = 0.0f, tp = 0.0f;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float fw = fred[w][hc[c][HU ? 0 : k]];
                    t += red[w][c * 4 + k][lane] * fw;
                    if constexpr (TRAIN) tp += red[w][NC * 4 + c * 4 + k][lane] * fw;
                }
                acc[c][k] = t;
                if constexpr (TRAIN) accp[c][k] = tp;
            }
    }

    float* orow = a.out + (int64_t)v * a.ldo;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (!act[c]) continue;
        const int64_t col = col0 + c * 256;
        const int valid = (int)min((int64_t)4, a.F - col);
        float r[4];
        if constexpr (TRAIN) {
            float rp[4], rn[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float den = select_head<HP>(s, hc[c][HU ? 0 : k]);
                r[k] = den > 0.0f ? (acc[c][k] + accp[c][k]) / den : 0.0f;
                rp[k] = den > 0.0f ? accp[c][k] / den : 0.0f;
                rn[k] = den > 0.0f ? acc[c][k] / den : 0.0f;
            }
            store_row<4>(a.save_pos + (int64_t)v * a.ld_pos + col, rp, valid, true);
            store_row<4>(a.save_neg + (int64_t)v * a.ld_pos + col, rn, valid, true);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float den = select_head<HP>(s, hc[c][HU ? 0 : k]);
                r[k] = den > 0.0f ? acc[c][k] / den : 0.0f;
            }
        }
        store_row<4>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
        if (a.copy_self) {
            float zs[4];
            load_row<4>(a.Z + (int64_t)v * a.ldz + col, zs);
            store_row<4>(orow + col, zs, valid, a.self_vec != 0);
        }
    }
    if constexpr (TRAIN) {
        if (lane == 0 && slab == 0) {
#pragma unroll
            for (int h = 0; h < HP; ++h) {
                const bool any = s[h] > 0.0f;
                const float rs = any ? 1.0f / s[h] : 0.0f;
                const f32x4 t = {any ? m[h] : 0.0f, rs, sp[h] * rs, sn[h] * rs};
                a.save_stats[(int64_t)v * HP + h] = t;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// one launch for long and short rows: the number of its workgroups
unsigned both_classes(AggArgs& a, int64_t n_heavy, int64_t N, int waves = kHeavyWaves)
{
    a.heavy_rows = n_heavy;
    a.heavy_items = n_heavy * a.nslab;
    return (unsigned)(a.heavy_items + ((N - n_heavy) * a.nslab + waves - 1) / waves);
}

template <int VEC, int NC, bool MAXOP>
void launch_linear(const AggArgs& base, int64_t n_heavy, int64_t N, hipStream_t stream)
{
    AggArgs a = base;
    const unsigned blocks = both_classes(a, n_heavy, N);
    if constexpr (!MAXOP && VEC == 4 && NC <= 2) {          // (the widest slabs have no registers for them)
        if (a.levels) {
            agg_linear_kernel<VEC, NC, MAXOP, true><<<dim3(blocks), dim3(64 * kHeavyWaves), 0, stream>>>(a);
            return;
        }
    }
    agg_linear_kernel<VEC, NC, MAXOP, false><<<dim3(blocks), dim3(64 * kHeavyWaves), 0, stream>>>(a);
}

template <int P>
void launch_rows(const AggArgs& base, int64_t n_heavy, int64_t N, hipStream_t stream)
{
    AggArgs a = base;
    const int64_t rows = kHeavyWaves * (64 / P);
    a.heavy_rows = n_heavy;
    a.nslab = (int)((a.F + 4 * P - 1) / (4 * P));
    a.slab_blocks = (uint32_t)(n_heavy + (N - n_heavy + rows - 1) / rows);
    const dim3 grid(a.slab_blocks * (unsigned)a.nslab), block(64 * kHeavyWaves);
    if (a.wsrc && a.levels) agg_rows_kernel<P, true, true><<<grid, block, 0, stream>>>(a);
    else if (a.wsrc)        agg_rows_kernel<P, true, false><<<grid, block, 0, stream>>>(a);
    else if (a.levels)      agg_rows_kernel<P, false, true><<<grid, block, 0, stream>>>(a);
    else                    agg_rows_kernel<P, false, false><<<grid, block, 0, stream>>>(a);
}

template <int LPG, bool WEIGHTED, bool OFF32>
void launch_grouped_pair(const AggArgs& base, int64_t n_heavy, int64_t N, hipStream_t stream)
{
    if (n_heavy > 0) {
        AggArgs a = base;
        a.row_begin = 0;
        a.row_count = n_heavy;
        const int64_t blocks = n_heavy * a.nslab;
        agg_grouped_kernel<LPG, kHeavyWaves, WEIGHTED, OFF32>
            <<<dim3((unsigned)blocks), dim3(64 * kHeavyWaves), 0, stream>>>(a);
    }
    if (N > n_heavy) {
        AggArgs a = base;
        a.row_begin = n_heavy;
        a.row_count = N - n_heavy;
        const int64_t bundles = (a.row_count + (64 / LPG) - 1) / (64 / LPG);
        const int64_t blocks = (bundles * a.nslab + kLightWaves - 1) / kLightWaves;
        agg_rowgroup_kernel<LPG, WEIGHTED, OFF32>
            <<<dim3((unsigned)blocks), dim3(64 * kLightWaves), 0, stream>>>(a);
    }
}

template <int LPG>
void dispatch_grouped(const AggArgs& a, int64_t n_heavy, int64_t N, bool weighted, bool off32, hipStream_t s)
{
    if (weighted) {
        if (off32) launch_grouped_pair<LPG, true, true>(a, n_heavy, N, s);
        else launch_grouped_pair<LPG, true, false>(a, n_heavy, N, s);
    } else {
        if (off32) launch_grouped_pair<LPG, false, true>(a, n_heavy, N, s);
        else launch_grouped_pair<LPG, false, false>(a, n_heavy, N, s);
    }
}

// ---------------------------------------------------------------------------
// gat_softmax when the whole row fits one wave (F <= 256, four floats per lane)
// and a head is a power-of-two group of lanes:
// the score of an entry is computed from the gathered source row itself.
//
// The kernels above fetch el[u] = <a_src, z_u> from a table, one 16-byte read
// per entry, which on a graph whose table misses L2 costs a whole extra cache
// line per entry next to the eight lines of the row.  Here every lane
// multiplies its four floats of z_u with its four floats of a_src, the lanes of
// a head add up over the group with DPP moves, and the softmax runs online over
// batches of four entries (running maximum m, sum s and weighted row acc per
// lane, all three rescaled when the maximum moves).  Scores are kept in units
// of log2(e) (LeakyReLU commutes with a positive factor) so that every
// exponential is one v_exp_f32.  The destination's own score <a_dst, z_v> is formed
// the same way from row v when `attn_dst` is given (the plain forward: no score
// kernel runs at all); with attn_dst == NULL it is read from the table (save mode).
// The first a.heavy_items workgroups hold one long row each, whose interleaved
// 64-entry tiles the eight waves share; they merge their (m, s, acc) triples
// through LDS in wave order.  The others hold eight rows.  One launch for both: a
// row of 17,500 entries keeps its workgroup busy for half a millisecond, in which a
// launch of long rows alone leaves the chip idle (2,449,029 nodes, 124 million
// entries, F = 256, save mode 21.5 + 0.65 ms, 22.0 now; plain, F = 128: 60,000 nodes
// and 3 million entries 262 us, 167 now, 20,000 and 200,000 57 and 27).
// ---------------------------------------------------------------------------
// TRAIN (save mode): the aggregate is accumulated in two parts, entries with a positive score (accp) and the
// others (acc), with the sums of their weights (sp, sn), and the row statistics are kept for the backward
// pass; scores then stay in natural units, because the stored row maximum is used as such.
template <int G, bool TRAIN, int NW>
__global__ __launch_bounds__(64 * NW) void agg_gat_flash_kernel(
    AggArgs a, const float* __restrict__ attn_src, const float* __restrict__ attn_dst, int er_stride)
{
    constexpr int U = 4;      // entries per batch of the online softmax (2 and 8 measure the same: the kernel waits for memory)
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr float kIn = TRAIN ? 1.0f : kLog2e;       // factor on the scores as they are formed
    constexpr float kEx = TRAIN ? kLog2e : 1.0f;       // factor inside the exponentials
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool heavy = blockIdx.x < a.heavy_items;    // uniform over the workgroup
    const int64_t slot = heavy ? (int64_t)blockIdx.x : a.heavy_rows + ((int64_t)blockIdx.x - a.heavy_items) * NW + wave;
    if (slot >= a.n_rows) return;
    const int v = __builtin_amdgcn_readfirstlane(a.order[slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);

    const int64_t col = lane * 4;
    const bool act = col < a.F;
    // lanes past the row width gather the last valid vector instead (never stored, weight vector zero)
    const uint32_t colbytes = (uint32_t)((act ? col : ((a.F - 1) / 4) * 4) * 4);
    const int h = min((int)(col / a.Dh), a.heads - 1);
    f32x4 as = {0.0f, 0.0f, 0.0f, 0.0f};
    float erv = 0.0f;
    const char* zbase = reinterpret_cast<const char*>(a.Z);
    const uint32_t rowbytes = (uint32_t)(a.ldz * 4);
    if (act) {
        as = *reinterpret_cast<const f32x4*>(attn_src + col);        // [heads, Dh] is F contiguous floats
        as.x *= kIn; as.y *= kIn; as.z *= kIn; as.w *= kIn;
        if (!attn_dst) erv = a.er[(int64_t)v * er_stride + h] * kIn;
    }
    if (attn_dst) {
        // (uniform branch) every lane takes part in the sums; lanes past the row width add zero
        f32x4 ad = {0.0f, 0.0f, 0.0f, 0.0f};
        if (act) ad = *reinterpret_cast<const f32x4*>(attn_dst + col);
        const f32x4 zv = *reinterpret_cast<const f32x4*>(zbase + (uint32_t)v * rowbytes + colbytes);
        float d = (ad.x * kIn) * zv.x;
        d = fmaf(ad.y * kIn, zv.y, d);
        d = fmaf(ad.z * kIn, zv.z, d);
        d = fmaf(ad.w * kIn, zv.w, d);
        erv = group_sum<G>(d);
    }

    float m = -INFINITY, s = 0.0f, sp = 0.0f, sn = 0.0f;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, accp = {0.0f, 0.0f, 0.0f, 0.0f};
    const int step = heavy ? 64 * NW : 64;
    for (int base = lo + (heavy ? 64 * wave : 0); base < hi; base += step) {
        const int e = base + lane;
        const bool valid = e < hi;
        const int cnt = min(64, hi - base);
        int my_u = valid ? a.col_idx[e] : 0;
        my_u = valid ? my_u : bcast_i(my_u, 0);          // lane 0 is always valid
        const int my_off = (int)((uint32_t)my_u * rowbytes);

        f32x4 zq[U];
#pragma unroll
        for (int t = 0; t < U; ++t)
            zq[t] = *reinterpret_cast<const f32x4*>(zbase + (uint32_t)bcast_i(my_off, t) + colbytes);

        for (int j = 0; j < cnt; j += U) {
            // request the next batch, then consume the current one
            f32x4 zn[U];
            const bool more = j + U < cnt;
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t)
                    zn[t] = *reinterpret_cast<const f32x4*>(zbase + (uint32_t)bcast_i(my_off, (j + U + t) & 63) + colbytes);
            }
            float x[U], sc[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                float d = as.x * zq[t].x;
                d = fmaf(as.y, zq[t].y, d);
                d = fmaf(as.z, zq[t].z, d);
                d = fmaf(as.w, zq[t].w, d);
                x[t] = group_sum<G>(d) + erv;
                sc[t] = (j + t < cnt) ? (x[t] > 0.0f ? x[t] : a.slope * x[t]) : -INFINITY;   // entries past the tile weigh nothing
            }
            float mn = m;
#pragma unroll
            for (int t = 0; t < U; ++t) mn = fmaxf(mn, sc[t]);                           // finite: entry j of the tile is real
            const float scale = __builtin_amdgcn_exp2f((m - mn) * kEx);
            float pw[U];
#pragma unroll
            for (int t = 0; t < U; ++t) pw[t] = __builtin_amdgcn_exp2f((sc[t] - mn) * kEx);
            float ps = 0.0f;
#pragma unroll
            for (int t = 0; t < U; ++t) ps += pw[t];
            s = s * scale + ps;
            acc.x *= scale; acc.y *= scale; acc.z *= scale; acc.w *= scale;
            if constexpr (TRAIN) {
                float pps = 0.0f, pns = 0.0f;
                accp.x *= scale; accp.y *= scale; accp.z *= scale; accp.w *= scale;
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const float pp = x[t] > 0.0f ? pw[t] : 0.0f, pn = x[t] > 0.0f ? 0.0f : pw[t];
                    pps += pp;
                    pns += pn;
                    accp.x = fmaf(pp, zq[t].x, accp.x);
                    accp.y = fmaf(pp, zq[t].y, accp.y);
                    accp.z = fmaf(pp, zq[t].z, accp.z);
                    accp.w = fmaf(pp, zq[t].w, accp.w);
                    acc.x = fmaf(pn, zq[t].x, acc.x);
                    acc.y = fmaf(pn, zq[t].y, acc.y);
                    acc.z = fmaf(pn, zq[t].z, acc.z);
                    acc.w = fmaf(pn, zq[t].w, acc.w);
                }
                sp = sp * scale + pps;
                sn = sn * scale + pns;
            } else {
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    acc.x = fmaf(pw[t], zq[t].x, acc.x);
                    acc.y = fmaf(pw[t], zq[t].y, acc.y);
                    acc.z = fmaf(pw[t], zq[t].z, acc.z);
                    acc.w = fmaf(pw[t], zq[t].w, acc.w);
                }
            }
            m = mn;
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t) zq[t] = zn[t];
            }
        }
    }

    if (heavy) {
        // merge the waves' running maxima and sums, in wave order
        __shared__ float red[NW][TRAIN ? 12 : 6][64];
        red[wave][0][lane] = m;
        red[wave][1][lane] = s;
        red[wave][2][lane] = acc.x;
        red[wave][3][lane] = acc.y;
        red[wave][4][lane] = acc.z;
        red[wave][5][lane] = acc.w;
        if constexpr (TRAIN) {
            red[wave][6][lane] = sp;
            red[wave][7][lane] = sn;
            red[wave][8][lane] = accp.x;
            red[wave][9][lane] = accp.y;
            red[wave][10][lane] = accp.z;
            red[wave][11][lane] = accp.w;
        }
        __syncthreads();
        if (wave != 0) return;
        float mm = red[0][0][lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, red[w][0][lane]);
        s = 0.0f;
        acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (TRAIN) {
            sp = sn = 0.0f;
            accp = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = red[w][0][lane];
            // a wave that saw no entry has m = -inf and weighs nothing
            const float f = mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((mw - mm) * kEx);
            s = fmaf(red[w][1][lane], f, s);
            acc.x = fmaf(red[w][2][lane], f, acc.x);
            acc.y = fmaf(red[w][3][lane], f, acc.y);
            acc.z = fmaf(red[w][4][lane], f, acc.z);
            acc.w = fmaf(red[w][5][lane], f, acc.w);
            if constexpr (TRAIN) {
                sp = fmaf(red[w][6][lane], f, sp);
                sn = fmaf(red[w][7][lane], f, sn);
                accp.x = fmaf(red[w][8][lane], f, accp.x);
                accp.y = fmaf(red[w][9][lane], f, accp.y);
                accp.z = fmaf(red[w][10][lane], f, accp.z);
                accp.w = fmaf(red[w][11][lane], f, accp.w);
            }
        }
        m = mm;
    }

    if constexpr (TRAIN) {
        // statistics: one lane per head; the padded heads carry no columns and look like a uniform softmax
        if (act && (lane % G) == 0 && col < (int64_t)a.heads * a.Dh) {
            const bool any = s > 0.0f;
            const float rs = any ? 1.0f / s : 0.0f;
            a.save_stats[(int64_t)v * er_stride + h] = f32x4{any ? m : 0.0f, rs, sp * rs, sn * rs};
        }
        if (lane == 0) {
            const bool any = hi > lo;
            const f32x4 t = {0.0f, any ? 1.0f / (float)(hi - lo) : 0.0f, 0.0f, any ? 1.0f : 0.0f};
            for (int k = a.heads; k < er_stride; ++k) a.save_stats[(int64_t)v * er_stride + k] = t;
        }
    }
    if (!act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    float r[4];
    if constexpr (TRAIN) {
        float rp[4], rn[4];
        const float ap[4] = {accp.x, accp.y, accp.z, accp.w}, an[4] = {acc.x, acc.y, acc.z, acc.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            r[k] = s > 0.0f ? (an[k] + ap[k]) / s : 0.0f;
            rp[k] = s > 0.0f ? ap[k] / s : 0.0f;
            rn[k] = s > 0.0f ? an[k] / s : 0.0f;
        }
        store_row<4>(a.save_pos + (int64_t)v * a.ld_pos + col, rp, 4, true);
        store_row<4>(a.save_neg + (int64_t)v * a.ld_pos + col, rn, 4, true);
    } else {
        r[0] = s > 0.0f ? acc.x / s : 0.0f;
        r[1] = s > 0.0f ? acc.y / s : 0.0f;
        r[2] = s > 0.0f ? acc.z / s : 0.0f;
        r[3] = s > 0.0f ? acc.w / s : 0.0f;
    }
    store_row<4>(orow + a.ocol + col, r, 4, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self) {
        float zs[4];
        load_row<4>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_row<4>(orow + col, zs, 4, a.self_vec != 0);
    }
}

// ---------------------------------------------------------------------------
// The same for rows, or slabs of whole heads, of up to 64 columns: P = 8 or 16 lanes of four floats hold a row, and the R = 64 / P groups of a
// wave take R consecutive rows of the schedule, or shares of one long row, in lock step (EntryWalk).  One entry per
// instruction leaves 64 - P lanes idle there, and a row of twenty entries waits for memory five times, whatever its width;
// here that is five times for R rows.  Scores, online softmax and save mode as above; a group whose row has ended weighs
// its batches' entries with zero.  The shares of a long row are merged over the groups first, then over the waves, in order.
// One row per wave and several, in us: 32 columns 2,449,029 nodes of 50 entries 5,025 and 2,388 (7.1 TB/s of whole lines), save mode 7,153 and 2,695;
// 200,000 of 100 749 and 254, 1,083 and 281; 200,000 of 20 188 and 67; 64 columns 196 and 135, 1,000,000 of 8 641 and 390.
// (32 lanes, for 65 to 128 columns: 200,000 of 20 267 and 279, 5,000 of 20 13.4 and 17.4, so those keep a row per wave.)
// ---------------------------------------------------------------------------
template <int G, int P, bool TRAIN, int NW>
__global__ __launch_bounds__(64 * NW) void agg_gat_rows_kernel(
    AggArgs a, const float* __restrict__ attn_src, const float* __restrict__ attn_dst, int er_stride)
{
    constexpr int U = 4, R = 64 / P;
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr float kIn = TRAIN ? 1.0f : kLog2e;       // factor on the scores as they are formed
    constexpr float kEx = TRAIN ? kLog2e : 1.0f;       // factor inside the exponentials
    const int lane = threadIdx.x & 63, li = lane % P, g = lane / P;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // one slab of heads after the other, long rows first in each
    const uint32_t slab = blockIdx.x / a.slab_blocks, block = blockIdx.x % a.slab_blocks;
    const bool heavy = block < a.heavy_rows;          // uniform over the workgroup
    const int64_t first = heavy ? (int64_t)block : a.heavy_rows + ((int64_t)(block - (uint32_t)a.heavy_rows) * NW + wave) * R;
    if (first >= a.n_rows) return;
    const int64_t slot = heavy ? first : first + g;
    const bool have = slot < a.n_rows;
    int v = 0;
    uint32_t lo = 0, hi = 0;
    if (have) {
        v = a.order[slot];
        lo = (uint32_t)a.row_ptr[v];
        hi = (uint32_t)a.row_ptr[v + 1];
    }
    constexpr uint32_t kTile = EntryWalk<P>::kTile;
    EntryWalk<P> walk;
    const uint32_t rowbytes = (uint32_t)(a.ldz * 4);
    const int batches = heavy ? walk.start(a.col_idx, lo + kTile * (wave * R + g), hi, kTile * NW * R, rowbytes)
                              : walk.start(a.col_idx, lo, hi, kTile, rowbytes);

    const int col = (int)slab * a.slab_cols + li * 4;
    const bool act = li * 4 < a.slab_cols && col < a.F;
    const table_t table = buffer_table(a.Z, a.table_bytes);
    const uint32_t colbytes = act ? (uint32_t)col * 4 : kNoEntry;      // (columns past the row width fetch nothing)
    const int h = min(col / a.Dh, a.heads - 1);
    f32x4 as = {0.0f, 0.0f, 0.0f, 0.0f};
    float erv = 0.0f;
    if (act) {
        as = *reinterpret_cast<const f32x4*>(attn_src + col);        // [heads, Dh] is F contiguous floats
        as.x *= kIn; as.y *= kIn; as.z *= kIn; as.w *= kIn;
        if (!attn_dst && have) erv = a.er[(int64_t)v * er_stride + h] * kIn;
    }
    if (attn_dst) {
        f32x4 ad = {0.0f, 0.0f, 0.0f, 0.0f};
        if (act) ad = *reinterpret_cast<const f32x4*>(attn_dst + col);
        const f32x4 zv = __builtin_bit_cast(f32x4, load_entry(table, have ? (uint32_t)v * rowbytes : kNoEntry, colbytes));
        float d = (ad.x * kIn) * zv.x;
        d = fmaf(ad.y * kIn, zv.y, d);
        d = fmaf(ad.z * kIn, zv.z, d);
        d = fmaf(ad.w * kIn, zv.w, d);
        erv = group_sum<G>(d);
    }

    const bool empty = (heavy ? lo + kTile * (wave * R + g) : lo) >= hi;      // no entry: its maximum stays -infinity
    float m = -INFINITY, s = 0.0f, sp = 0.0f, sn = 0.0f;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, accp = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 z[2][U];
    uint32_t on[2][U];
    auto issue = [&](int j, f32x4 (&zz)[U], uint32_t (&oo)[U]) {
#pragma unroll
        for (int t = 0; t < U; ++t) {
            oo[t] = walk.at(j, t);
            zz[t] = __builtin_bit_cast(f32x4, load_entry(table, oo[t], colbytes));
        }
    };
    auto consume = [&](const f32x4 (&zq)[U], const uint32_t (&oo)[U]) {
        float x[U], sc[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            float d = as.x * zq[t].x;
            d = fmaf(as.y, zq[t].y, d);
            d = fmaf(as.z, zq[t].z, d);
            d = fmaf(as.w, zq[t].w, d);
            x[t] = group_sum<G>(d) + erv;
            sc[t] = oo[t] != kNoEntry ? (x[t] > 0.0f ? x[t] : a.slope * x[t]) : -INFINITY;
        }
        float mn = m;
#pragma unroll
        for (int t = 0; t < U; ++t) mn = fmaxf(mn, sc[t]);
        const float mr = empty ? 0.0f : mn;
        const float scale = __builtin_amdgcn_exp2f((m - mr) * kEx);
        float pw[U];
#pragma unroll
        for (int t = 0; t < U; ++t) pw[t] = __builtin_amdgcn_exp2f((sc[t] - mr) * kEx);
        float ps = 0.0f;
#pragma unroll
        for (int t = 0; t < U; ++t) ps += pw[t];
        s = s * scale + ps;
        acc.x *= scale; acc.y *= scale; acc.z *= scale; acc.w *= scale;
        if constexpr (TRAIN) {
            float pps = 0.0f, pns = 0.0f;
            accp.x *= scale; accp.y *= scale; accp.z *= scale; accp.w *= scale;
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const float pp = x[t] > 0.0f ? pw[t] : 0.0f, pn = x[t] > 0.0f ? 0.0f : pw[t];
                pps += pp;
                pns += pn;
                accp.x = fmaf(pp, zq[t].x, accp.x);
                accp.y = fmaf(pp, zq[t].y, accp.y);
                accp.z = fmaf(pp, zq[t].z, accp.z);
                accp.w = fmaf(pp, zq[t].w, accp.w);
                acc.x = fmaf(pn, zq[t].x, acc.x);
                acc.y = fmaf(pn, zq[t].y, acc.y);
                acc.z = fmaf(pn, zq[t].z, acc.z);
                acc.w = fmaf(pn, zq[t].w, acc.w);
            }
            sp = sp * scale + pps;
            sn = sn * scale + pns;
        } else {
#pragma unroll
            for (int t = 0; t < U; ++t) {
                acc.x = fmaf(pw[t], zq[t].x, acc.x);
                acc.y = fmaf(pw[t], zq[t].y, acc.y);
                acc.z = fmaf(pw[t], zq[t].z, acc.z);
                acc.w = fmaf(pw[t], zq[t].w, acc.w);
            }
        }
        m = mn;
    };
    // the gathers of a batch are issued before the batch before it is added up
    auto step = [&](int k, f32x4 (&zn)[U], uint32_t (&no)[U]) {       // batch k
        if (k % P == 0 && k > 0) walk.take();
        issue(k % P, zn, no);
    };
    if (batches > 0) step(0, z[0], on[0]);
    for (int k = 0; k < batches; k += 2) {
        if (k + 1 < batches) step(k + 1, z[1], on[1]);
        consume(z[0], on[0]);
        if (k + 1 >= batches) break;
        if (k + 2 < batches) step(k + 2, z[0], on[0]);
        consume(z[1], on[1]);
    }

    if (heavy) {
        // merge the shares: groups of the wave, then the waves; one that saw no entry has m = -inf and weighs nothing
        auto weight = [&](float mw, float mm) { return mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((mw - mm) * kEx); };
#pragma unroll
        for (int b = P; b < 64; b <<= 1) {
            const float mo = __shfl_xor(m, b, 64), mm = fmaxf(m, mo), fa = weight(m, mm), fb = weight(mo, mm);
            auto join = [&](float x) { return x * fa + __shfl_xor(x, b, 64) * fb; };
            s = join(s);
            acc = f32x4{join(acc.x), join(acc.y), join(acc.z), join(acc.w)};
            if constexpr (TRAIN) {
                sp = join(sp);
                sn = join(sn);
                accp = f32x4{join(accp.x), join(accp.y), join(accp.z), join(accp.w)};
            }
            m = mm;
        }
        __shared__ float red[NW][TRAIN ? 12 : 6][P];
        if (g == 0) {
            red[wave][0][li] = m;
            red[wave][1][li] = s;
            red[wave][2][li] = acc.x;
            red[wave][3][li] = acc.y;
            red[wave][4][li] = acc.z;
            red[wave][5][li] = acc.w;
            if constexpr (TRAIN) {
                red[wave][6][li] = sp;
                red[wave][7][li] = sn;
                red[wave][8][li] = accp.x;
                red[wave][9][li] = accp.y;
                red[wave][10][li] = accp.z;
                red[wave][11][li] = accp.w;
            }
        }
        __syncthreads();
        if (wave != 0) return;
        float mm = red[0][0][li];
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, red[w][0][li]);
        s = sp = sn = 0.0f;
        acc = accp = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = weight(red[w][0][li], mm);
            s = fmaf(red[w][1][li], f, s);
            acc.x = fmaf(red[w][2][li], f, acc.x);
            acc.y = fmaf(red[w][3][li], f, acc.y);
            acc.z = fmaf(red[w][4][li], f, acc.z);
            acc.w = fmaf(red[w][5][li], f, acc.w);
            if constexpr (TRAIN) {
                sp = fmaf(red[w][6][li], f, sp);
                sn = fmaf(red[w][7][li], f, sn);
                accp.x = fmaf(red[w][8][li], f, accp.x);
                accp.y = fmaf(red[w][9][li], f, accp.y);
                accp.z = fmaf(red[w][10][li], f, accp.z);
                accp.w = fmaf(red[w][11][li], f, accp.w);
            }
        }
        m = mm;
    }

    if (!have || (heavy && g != 0)) return;
    if constexpr (TRAIN) {
        // statistics: one lane per head; the padded heads carry no columns and look like a uniform softmax
        if (act && (li % G) == 0) {
            const bool any = s > 0.0f;
            const float rs = any ? 1.0f / s : 0.0f;
            a.save_stats[(int64_t)v * er_stride + h] = f32x4{any ? m : 0.0f, rs, sp * rs, sn * rs};
        }
        if (li == 0 && slab == 0) {
            const bool any = hi > lo;
            const f32x4 t = {0.0f, any ? 1.0f / (float)(hi - lo) : 0.0f, 0.0f, any ? 1.0f : 0.0f};
            for (int k = a.heads; k < er_stride; ++k) a.save_stats[(int64_t)v * er_stride + k] = t;
        }
    }
    if (!act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    float r[4];
    if constexpr (TRAIN) {
        float rp[4], rn[4];
        const float ap[4] = {accp.x, accp.y, accp.z, accp.w}, an[4] = {acc.x, acc.y, acc.z, acc.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            r[k] = s > 0.0f ? (an[k] + ap[k]) / s : 0.0f;
            rp[k] = s > 0.0f ? ap[k] / s : 0.0f;
            rn[k] = s > 0.0f ? an[k] / s : 0.0f;
        }
        store_row<4>(a.save_pos + (int64_t)v * a.ld_pos + col, rp, 4, true);
        store_row<4>(a.save_neg + (int64_t)v * a.ld_pos + col, rn, 4, true);
    } else {
        r[0] = s > 0.0f ? acc.x / s : 0.0f;
        r[1] = s > 0.0f ? acc.y / s : 0.0f;
        r[2] = s > 0.0f ? acc.z / s : 0.0f;
        r[3] = s > 0.0f ? acc.w / s : 0.0f;
    }
    store_row<4>(orow + a.ocol + col, r, 4, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self) {
        float zs[4];
        load_row<4>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_row<4>(orow + col, zs, 4, a.self_vec != 0);
    }
}

template <int G, int P, bool TRAIN>
void launch_gat_rows(const AggArgs& base, int64_t n_heavy, int64_t N, const float* attn_src, const float* attn_dst, int hp,
                     int waves, hipStream_t stream)
{
    if constexpr (G <= P && G * kMaxHeads > P / 2) {
        AggArgs a = base;
        const int64_t rows = (int64_t)waves * (64 / P);
        a.heavy_rows = n_heavy;
        a.slab_blocks = (uint32_t)(n_heavy + (N - n_heavy + rows - 1) / rows);
        const dim3 grid((unsigned)(a.slab_blocks * (unsigned)a.nslab)), block(64 * waves);
        if (waves == 4) agg_gat_rows_kernel<G, P, TRAIN, 4><<<grid, block, 0, stream>>>(a, attn_src, attn_dst, hp);
        else            agg_gat_rows_kernel<G, P, TRAIN, 8><<<grid, block, 0, stream>>>(a, attn_src, attn_dst, hp);
    }
}
template <int G, bool TRAIN>
void dispatch_gat_rows(int lanes, const AggArgs& a, int64_t n_heavy, int64_t N, const float* attn_src, const float* attn_dst,
                       int hp, int waves, hipStream_t stream)
{
    if (lanes == 8) launch_gat_rows<G, 8, TRAIN>(a, n_heavy, N, attn_src, attn_dst, hp, waves, stream);
    else            launch_gat_rows<G, 16, TRAIN>(a, n_heavy, N, attn_src, attn_dst, hp, waves, stream);
}

template <int VEC, int NC, int HP, bool HU>
void launch_gat_pair(const AggArgs& base, int64_t n_heavy, int64_t N, hipStream_t stream)
{
    if (n_heavy > 0) {
        AggArgs a = base;
        a.row_begin = 0;
        a.row_count = n_heavy;
        const int64_t blocks = n_heavy * a.nslab;
        agg_gat_kernel<VEC, NC, kHeavyWaves, HP, HU><<<dim3((unsigned)blocks), dim3(64 * kHeavyWaves), 0, stream>>>(a);
    }
    if (N > n_heavy) {
        AggArgs a = base;
        a.row_begin = n_heavy;
        a.row_count = N - n_heavy;
        const int64_t blocks = (a.row_count * a.nslab + kLightWaves - 1) / kLightWaves;
        agg_gat_kernel<VEC, NC, 1, HP, HU><<<dim3((unsigned)blocks), dim3(64 * kLightWaves), 0, stream>>>(a);
    }
}

template <int NC, int HP, bool HU, bool TRAIN>
void launch_gat_fast(const AggArgs& base, int64_t n_heavy, int64_t N, int waves, hipStream_t stream)
{
    AggArgs a = base;
    const unsigned blocks = both_classes(a, n_heavy, N, waves);
    if (waves == 4) agg_gat_fast_kernel<NC, 4, HP, HU, TRAIN><<<dim3(blocks), dim3(64 * 4), 0, stream>>>(a);
    else            agg_gat_fast_kernel<NC, 8, HP, HU, TRAIN><<<dim3(blocks), dim3(64 * 8), 0, stream>>>(a);
}

template <int HP, bool HU>
void dispatch_gat_fast(int nc, bool train, const AggArgs& a, int64_t nh, int64_t N, int waves, hipStream_t s)
{
    if (train) {
        if (nc == 1) launch_gat_fast<1, HP, HU, true>(a, nh, N, waves, s);
        else launch_gat_fast<2, HP, HU, true>(a, nh, N, waves, s);
    } else {
        if (nc == 1) launch_gat_fast<1, HP, HU, false>(a, nh, N, waves, s);
        else launch_gat_fast<2, HP, HU, false>(a, nh, N, waves, s);
    }
}

template <int VEC, bool MAXOP>
void dispatch_linear_nc(int nc, const AggArgs& a, int64_t nh, int64_t N, hipStream_t s)
{
    if (nc == 1) launch_linear<VEC, 1, MAXOP>(a, nh, N, s);
    else if (nc == 2) launch_linear<VEC, 2, MAXOP>(a, nh, N, s);
    else launch_linear<VEC, 3, MAXOP>(a, nh, N, s);
}

template <int VEC>
void dispatch_linear(int nc, bool maxop, const AggArgs& a, int64_t nh, int64_t N, hipStream_t s)
{
    if (maxop) dispatch_linear_nc<VEC, true>(nc, a, nh, N, s);
    else dispatch_linear_nc<VEC, false>(nc, a, nh, N, s);
}

template <int VEC, int HP, bool HU>
void dispatch_gat_nc(int nc, const AggArgs& a, int64_t nh, int64_t N, hipStream_t s)
{
    if (nc == 1) launch_gat_pair<VEC, 1, HP, HU>(a, nh, N, s);
    else launch_gat_pair<VEC, 2, HP, HU>(a, nh, N, s);
}

bool aligned_for(const void* p, int64_t ld, int vec)
{
    return ((uintptr_t)p % (uintptr_t)(4 * vec)) == 0 && ld % vec == 0;
}

}  // namespace

AggOptions& agg_options()
{
    static AggOptions o;
    return o;
}

GatWorkspace gat_workspace(int64_t N, int64_t F, int heads, bool save)
{
    const int64_t n = N > 0 ? N : 1, hp = heads_padded(heads);
    GatWorkspace w;
    int64_t off = 0;
    w.el = off; off += align_up(n * hp * (int64_t)sizeof(float), 256);
    w.er = off; off += align_up(n * hp * (int64_t)sizeof(float), 256);
    w.ld_pos = align_up(F > 0 ? F : 1, 32);
    w.stats = off; if (save) off += align_up(n * hp * 16, 256);
    w.pos = off;   if (save) off += align_up(n * w.ld_pos * (int64_t)sizeof(float), 256);
    w.neg = off;   if (save) off += align_up(n * w.ld_pos * (int64_t)sizeof(float), 256);
    w.total = off;
    return w;
}

int64_t aggregate_workspace_bytes(int64_t N, int mode, int heads, int64_t F, bool save)
{
    if (mode != RETEXO_GAT_SOFTMAX) return 0;
    return gat_workspace(N, F, heads, save).total;
}

void launch_gat_scores(int64_t N, int64_t F, int heads, const float* Z, int64_t ldz,
                       const float* a_src, const float* a_dst, float* el, float* er, hipStream_t stream,
                       int64_t el_stride)
{
    const int Dh = (int)(F / heads);
    if (el_stride == 0) el_stride = heads_padded(heads);
    if (F % 4 == 0 && aligned_for(Z, ldz, 4) && aligned_for(a_src, 4, 4) && aligned_for(a_dst, 4, 4) && agg_options().max_vec >= 4) {
        const unsigned gv = (unsigned)((N + 15) / 16);
        if (heads_padded(heads) == 4)
            gat_scores_vec_kernel<4><<<dim3(gv), dim3(256), 0, stream>>>(N, F, heads, Dh, Z, ldz, a_src, a_dst, el, el_stride, er);
        else
            gat_scores_vec_kernel<8><<<dim3(gv), dim3(256), 0, stream>>>(N, F, heads, Dh, Z, ldz, a_src, a_dst, el, el_stride, er);
        return;
    }
    const unsigned gb = (unsigned)((N + 3) / 4);
    if (heads_padded(heads) == 4)
        gat_scores_kernel<4><<<dim3(gb), dim3(256), 0, stream>>>(N, F, heads, Dh, Z, ldz, a_src, a_dst, el, el_stride, er);
    else
        gat_scores_kernel<8><<<dim3(gb), dim3(256), 0, stream>>>(N, F, heads, Dh, Z, ldz, a_src, a_dst, el, el_stride, er);
}

namespace {

// rows of Z start at 16-byte addresses and their last vector may read padding columns of the same row
bool rows_padded(const AggCall& c) { return aligned_for(c.Z, c.ldz, 4) && align_up(c.F, 4) <= c.ldz; }

// Sums, means and gcn_sym of up to 48 columns in row groups take four floats at any float's address, none of them past a row's end
// (own_columns), where rows are neither aligned nor padded: mean in us, before and now, 1,000,000 nodes of 20 entries, 5
// columns 645 and 367, 17 columns 631 and 520; 62 columns 1,030 and 1,050.  (Wider ones touch a line more per entry and slab: 301
// columns in slabs of 64 4,106 and 5,180.)
bool narrow_unpadded(const AggCall& c)
{
    const AggOptions& opt = agg_options();
    return c.mode != RETEXO_GAT_SOFTMAX && c.mode != RETEXO_MAX && c.F >= 4 && c.F <= 48 && !rows_padded(c) &&
           (c.plan->N * c.ldz + c.F) * 4 < (1ll << 32) && !opt.wide_offsets && opt.slab_cols == 0 && opt.max_vec >= 4 &&
           !(c.plan->part_ptr && opt.parts >= 0);
}

// widest gather the layout of Z allows
int gather_vec(const AggCall& c)
{
    const bool two = aligned_for(c.Z, c.ldz, 2) && align_up(c.F, 2) <= c.ldz;
    int vec = rows_padded(c) || narrow_unpadded(c) ? 4 : two ? 2 : 1;
    if (vec > agg_options().max_vec) vec = agg_options().max_vec >= 2 ? 2 : 1;
    if (c.mode == RETEXO_GAT_SOFTMAX && vec == 2) vec = 1;
    return vec;
}

// graphs that the range walk can be for: the plan split them, or they are dense and their table does not fit an L2
bool dense_for_ranges(const AggCall& c)
{
    const retexo_plan* p = c.plan;
    return p->part_ptr || (p->nnz >= 32 * p->N && p->N * c.ldz * 4 > (4ll << 20));
}

// Times the mean row that the longest one may have for the rows to count as alike: then no node is gathered much more often than
// others, nothing but a range's slab stays in an L2, and a range's launches end together.  Over rows on whole 128-byte lines, mean in
// us, ranges against the others: 200,000 nodes of 100 entries (longest 151) 64 columns 444 and 645, 32 columns 235 and 294; 228,965 of
// 165 (592), 32 columns 343 and 529; 60,000 of 40 (79), 256 columns 200 and 259; 64,053 of 54 (91), 192 columns 239 and 325; with
// weights 200,000 of 100, 256 columns 2,300 and 2,637.  The other way, longest rows of twenty times the mean and more: see
// linear_route.  Tables of many ranges are faster in row groups whatever the rows (1,000,000 of 100, longest 154, 64 columns 5,391 and
// 3,461), and so are narrow rows of few nodes.  The lines are where 12,662 drawn calls over dense graphs change sides, by nodes and
// columns: against the kernels that took them before row groups 1,054 were more than 4 % slower, at most by a factor of 2.1, and 222 are,
// all of them together 0.912 of the time and 0.901.
int64_t alike_rows(int64_t N, int64_t nnz, int64_t F, bool weighted)
{
    const bool long_rows = nnz >= 100 * N;
    if (N <= 32768) return F > 64 ? 3 : F > 32 && N > 24000 && !weighted ? 2 : 0;
    if (N <= 65536) return F <= 128 ? 6 : 10;
    if (N <= 131072) return F <= 32 ? 8 : weighted ? 10 : 20;
    if (N <= 262144) return !weighted ? (F <= 32 ? 10 : 20) : long_rows || F <= 16 ? 10 : F <= 64 ? 0 : 3;
    return N <= 524288 && long_rows && !weighted ? 10 : 0;
}
// The same over padded rows that are not whole lines, which are narrow where ranges gain.  Rows of 17 to 32 columns, up to eight
// ranges of 128-byte pieces, from 56 to 85 entries on (24 columns, ranges against row groups: 160,491 nodes of 109 203 and 298,
// 114,026 of 210, longest 3.9 times the mean, 210 and 313; ratios: 164,000 of 196, 15.8 times, 1.61, 119,289 of 225, 14.2 times,
// 1.25, 127,881 of 107, 14.7 times, 1.25, 101,000 of 102, 13.9 times, 0.85, nine ranges and more 0.6 to 0.75).  Rows of 9 to 16 columns, which are half idle in
// row groups too, where they are long: with weights 96,411 of 219 1.17, 61,000 of 221 1.01; without 178,272 of 166 1.16, 254,000 of
// 107 1.30, 309,000 of 152 1.15, but 325,193 of 80 0.80.  Wider rows, without weights, in four ranges: 40 columns, 193,000 of
// 121 1.12, 56 columns, 166,429 of 120, 16 times, 1.13.
int64_t alike_off_lines(int64_t N, int64_t nnz, int64_t F, bool weighted)
{
    auto mean_is = [&](int64_t entries) { return nnz >= entries * N; };
    if (N <= 32768 || N > 524288 || F <= 8 || F > 64) return 0;
    if (F > 16 && F <= 32) {
        if (!mean_is(N <= 131072 ? 56 : weighted && N > 262144 ? 85 : 64)) return 0;
        return N <= 65536 ? 6 : N <= 104000 && !mean_is(140) ? 8 : 24;
    }
    if (F > 32) return !weighted && N > 131072 && N <= 262144 && mean_is(110) ? 20 : 0;
    if (weighted) return N <= 262144 && mean_is(130) ? 5 : 0;
    if (N <= 200000) return N > 150000 && mean_is(160) ? 10 : 0;
    return mean_is(N <= 262144 ? 75 : 100) ? 10 : 0;
}

// Which kernels a sum, mean or gcn_sym takes whose rows are gathered four floats at a time: the range walk over narrow slabs, row
// groups of `lanes` lanes over slabs of 4 * lanes columns, or (neither) whole rows.
struct LinearRoute {
    bool ranges;
    int lanes;
};
// Measured over 23 graphs of 3,000 to 2,449,029 nodes and 5 to 500 entries per row at 32 to 602 columns, and over some
// thousands of drawn calls (us, mean unless said, ranges against the others; limits without a figure here are where those calls
// change sides):
//  Ranges pay where a range's slab is near an L2's size and rows are long: 232,965 nodes of 492 entries, 602 columns 13,440 and
//  26,270; 400,000 of 250 (31 in each of 8 ranges) 17,200 and 27,660; 427,947 of 189, 192 columns 5,323 and 7,965; 50,000 of 400,
//  64 columns 242 and 334; 476,789 of 205, 32 columns 1,180 and 1,572.  The other way 1,000,000 of 100 (6 in each of 16 ranges)
//  47,760 and 30,750, 200,000 of 100, 64 columns 636 and 523, 32 columns 455 and 242, 60,000 of 40, 256 columns 257 and 232,
//  2,449,029 of 50, 256 columns (whose one range is 300 MB) 18,430 and 17,360, with weights 30,780 and (whole rows) 20,470.
//  They are two launches per range, so the call has to be long enough: 20,000 of 200, 256 columns 240 and 216, 602 columns
//  468 and 526.  Where neither gains much the lines lie on the side of the ranges.
//  Row groups for all rows of up to 64 columns: 1,000,000 of 20, 32 columns 394 against 773 in whole rows, of 8 187 and 489,
//  3,000 of 5 5.2 and 8.0; 64 columns 733 and 898, 377 and 543, 5.5 and 8.0.
//  Wider rows in slabs of 64 from 16 entries per row on, which leaves more of the nodes that are gathered most in an L2: 200,000
//  of 20, 256 columns 489 and 587, 500,000 of 40 2,614 and 2,738; of 8 entries 1,568 and 1,300; 128 columns (two slabs) from 64
//  entries on (20,000 of 200 112 and 123; 22,000 of 30, 96 columns 44 and 35).  Graphs that fit anyway in slabs of 128:
//  10,000 of 400, 256 columns 152 and 189.  With weights, read again for every slab, where all of them stay in an L2: 200,000
//  of 100, 256 columns 2,305 and 2,779, 30,000 of 40 111 and 132 (slabs of 128; 122 of 64), but 1,000,000 of 20 3,837 and 3,176.
//  Slabs are taken where they are three quarters full (6,051 of 223, 192 columns in two of 128 85 and 76) and, on graphs that are not
//  dense, over rows on whole 128-byte lines, of which each slab otherwise touches one more (210,122 of 29, 260 columns 1,299 and 972).
LinearRoute linear_route(const AggCall& c, int vec, int parts)
{
    const retexo_plan* p = c.plan;
    const AggOptions& opt = agg_options();
    const int64_t N = p->N, nnz = p->nnz, F = c.F, work = nnz * (F < 32 ? 32 : F);
    const bool weighted = c.mode == RETEXO_GCN_SYM;
    if (vec != 4 || c.mode == RETEXO_MAX || c.mode == RETEXO_GAT_SOFTMAX || opt.slab_cols != 0) return {false, 0};
    const LinearRoute ranges = {true, 0}, whole = {false, 0};
    if (narrow_unpadded(c)) return {false, F <= 32 ? 8 : 16};
    if (p->part_ptr && opt.parts >= 0) return ranges;              // (the caller said how many)
    const bool dense = dense_for_ranges(c);
    auto mean_is = [&](int64_t entries) { return nnz >= entries * N; };
    const bool lines = aligned_for(c.Z, c.ldz, 32);                 // rows on whole 128-byte lines
    const int64_t alike = lines ? alike_rows(N, nnz, F, weighted) : alike_off_lines(N, nnz, F, weighted);
    if (dense && p->max_degree * N < alike * nnz) return ranges;
    if (dense && N >= 16384 && N * 128 <= parts * (64ll << 20) && 2 * nnz >= 25 * N * parts) {
        const bool enough = N >= 24000 || work >= 1200000000ll || mean_is(300);
        if (F >= 100 ? enough && work >= 700000000ll && (mean_is(160) || mean_is((weighted ? 25 : 15) * parts))
            : F > 32 ? enough && work >= 600000000ll && mean_is(N >= 200000 ? 105 : 140)
                     : N >= 30000 && mean_is(N >= 200000 ? 170 : N >= 110000 ? 230 : N >= 40000 || weighted ? 255 : 350))
            return ranges;
    }
    // one range of a large table: nearly the same (2,449,029 of 50, 32 columns, 729,742 of 36 476 and 516, 554,648 of 32, 64
    // columns 562 and 619), where half of a row's lane group is idle from fewer nodes on (drawn calls of 250,000 to 350,000 nodes of
    // 32 to 64 entries, row groups against it: up to 16 columns 1.06 of the time, 17 to 32 columns 0.95)
    if (dense && !p->part_ptr && (F <= 32 ? N >= (F <= 16 ? 200000 : 350000) : F <= 64 && !weighted && N >= 200000 && N < 1000000)) return ranges;
    if ((N * c.ldz + F) * 4 >= (1ll << 32) || opt.wide_offsets)              // (row groups have 32-bit offsets)
        return dense && !(weighted && parts == 1) ? ranges : whole;
    auto in_slabs = [&](int lanes) {
        const int64_t slabs = (F + 4 * lanes - 1) / (4 * lanes);
        if (4 * F >= 3 * slabs * (4 * lanes) && (dense || lines || F <= 128)) return LinearRoute{false, lanes};
        return dense && mean_is(100) ? ranges : whole;
    };
    if (F <= 64) return {false, F <= 32 ? 8 : 16};
    if (N < 16384) {
        if (F > 256 || N < 8192 || !mean_is(64)) return dense && (F > 128 || mean_is(100)) ? ranges : whole;
        return in_slabs(32);
    }
    if (weighted) return N < 300000 && mean_is(F <= 128 ? 100 : 32) ? in_slabs(N < 100000 ? 32 : 16) : whole;
    return mean_is(F <= 128 ? 64 : 16) ? in_slabs(16) : whole;
}

// Which edge-softmax kernels a call takes.
struct GatRoute {
    int vec;
    bool off32;     // every byte offset into Z fits 32 bits
    bool flash;     // source scores from the gathered rows themselves
    bool in_rows;   // source scores kept in the unused columns of Z's own rows
};
GatRoute gat_route(const AggCall& c)
{
    const AggOptions& opt = agg_options();
    const int64_t N = c.plan->N;
    GatRoute r;
    r.vec = gather_vec(c);
    r.off32 = (N * c.ldz + c.F) * 4 < (1ll << 32) && !opt.wide_offsets;
    const int hp = heads_padded(c.heads);
    const int64_t Dh = c.F / c.heads;
    const int64_t g = Dh / 4;
    // the source scores are computed from the gathered rows themselves when a head is a power-of-two group of
    // four-float lanes
    r.flash = r.vec == 4 && r.off32 && opt.gat_fast && opt.gat_flash && c.F <= 256 &&
              Dh % 4 == 0 && g <= 64 && (g & (g - 1)) == 0 && aligned_for(c.attn_src, 4, 4);
    // Otherwise, when Z is the library's own buffer and its rows have unused columns behind F, the source
    // scores of a node are kept there: the gather of a row then brings them along in the row's last cache
    // line, instead of one more line per entry from a table elsewhere.
    r.in_rows = c.z_padding_free && !r.flash && r.vec == 4 && r.off32 && opt.gat_fast && opt.gat_in_rows &&
                c.F % 4 == 0 && c.ldz - c.F >= hp && c.F % 32 != 0 && (c.F % 32) + hp <= 32;
    return r;
}

// Heads that a slab of agg_gat_rows_kernel holds; 0: the call takes one row per wave.
// Up to 64 columns are one slab.  Wider rows of heads of up to 64 columns are walked a slab of 64 after the other over tables
// much larger than an L2 (24 MB) from 48 entries per row and 4 GB of gathers on.  What gains is four rows in flight per wave; hits
// in L2 hardly do (2,449,029 nodes of 50 entries, 256 columns: hit rate 0.039 and 0.052, traffic 133.7 and 132.7 GB, the time a
// tenth less).  It has to outweigh reading the ids, and a row's own start, once per slab.  The lines are no crossover: shorter calls
// gain as well (60,000 of 50 in save mode 475 and 360), down to a size that has not been measured.
// One row per wave and slabs, in us: 2,449,029 nodes of 50 entries, 256 columns 20,400 and 18,700, save mode 22,050 and 20,900;
// 200,000 of 100 2,626 and 2,113; 50,000 of 400 2,030 and 1,166; 65,000 of 100 743 and 639; 128 columns 2,449,029 of 50
// 9,330 and 8,740, 200,000 of 100 1,199 and 1,079.  The other way: 100,000 of 40, 192 columns, save mode 365 and 406; 1,000,000 of
// 8, 256 columns 1,483 and 1,651; known slower with slabs: 1,500,000 of 70, 128 columns 7,307 and 7,506.
int gat_rows_heads(const AggCall& c, int Dh)
{
    const retexo_plan* p = c.plan;
    if (c.F <= 64) return c.save || p->nnz >= kRowsFewest ? c.heads : 0;
    if (Dh > 64 || p->nnz < 48 * p->N || p->N * c.F * 4 < (24ll << 20) || p->nnz * c.F * 4 < (4ll << 30)) return 0;
    return 64 / Dh < c.heads ? 64 / Dh : c.heads;
}

// One wave per row of W (and one for b): copy the row and append its products with the heads of a_src.
__global__ __launch_bounds__(256) void gat_fold_kernel(int D_in, int F, int heads, int Dh, int hp,
                                                       const float* __restrict__ W, const float* __restrict__ b,
                                                       const float* __restrict__ a_src,
                                                       float* __restrict__ W2, float* __restrict__ b2)
{
    const int lane = threadIdx.x & 63;
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k > D_in) return;
    const float* src = k < D_in ? W + (int64_t)k * F : b;        // b == NULL: a zero bias
    float* dst = k < D_in ? W2 + (int64_t)k * (F + hp) : b2;
    float ps[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) ps[h] = 0.0f;
    for (int j = lane; j < F; j += 64) {
        const float x = src ? src[j] : 0.0f;
        dst[j] = x;
        const float t = x * a_src[j];
        const int hj = j / Dh;
#pragma unroll
        for (int h = 0; h < 8; ++h) ps[h] += hj == h ? t : 0.0f;
    }
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const float sum = wave_sum(ps[h]);
        if (lane == 0 && h < hp) dst[F + h] = h < heads ? sum : 0.0f;
    }
}

}  // namespace

bool gat_fold_plan(const AggCall& c, int64_t D_in, int64_t avail_bytes)
{
    if (c.mode != RETEXO_GAT_SOFTMAX || c.save || !agg_options().gat_fold) return false;
    const GatRoute r = gat_route(c);
    const int64_t wide = c.F + heads_padded(c.heads);
    // the pipelined kernel forms the destination scores from whole rows: one slab (two float4 per lane at most)
    return r.in_rows && c.F <= 512 && agg_options().slab_cols == 0 && aligned_for(c.attn_dst, 4, 4) &&
           (D_in + 1) * wide * (int64_t)sizeof(float) <= avail_bytes;
}

void launch_gat_fold(int64_t D_in, int64_t F, int heads, const float* W, const float* b, const float* a_src,
                     float* W2, float* b2, hipStream_t stream)
{
    gat_fold_kernel<<<dim3((unsigned)((D_in + 1 + 3) / 4)), dim3(256), 0, stream>>>(
        (int)D_in, (int)F, heads, (int)(F / heads), heads_padded(heads), W, b, a_src, W2, b2);
}

int launch_aggregate(const AggCall& c, hipStream_t stream)
{
    const retexo_plan* p = c.plan;
    const int64_t N = p->N;
    if (N == 0 || c.F == 0) return RETEXO_OK;
    const AggOptions& opt = agg_options();
    const bool gat = c.mode == RETEXO_GAT_SOFTMAX;

    const int vec = gather_vec(c);
    const int max_nc = gat ? 2 : 3;
    int nc;
    if (opt.slab_cols > 0) nc = (int)((opt.slab_cols + 64 * vec - 1) / (64 * vec));
    else nc = (int)((c.F + 64 * vec - 1) / (64 * vec));
    nc = nc < 1 ? 1 : nc > max_nc ? max_nc : nc;
    // Whole rows of more than 256 columns a slab of 256 after the other: one load per entry and slab leaves eight entries in
    // flight per lane and twice the waves (mean in us, slabs of up to 768 and of 256: 1,000,000 nodes of 20 entries, 500 columns
    // 6,697 and 5,886, 640 columns 8,647 and 7,367; 2,708 of 4, 640 columns 13.3 and 8.2, 1,433 columns 17.2 and 13.5; 50,000 of
    // 10, 1,433 columns 577 and 416).  Not where the last slab would be nearly empty (288 columns, 1,000,000 of 20 3,440 and
    // 3,715; 544, 81,938 of 5 157 and 179), nor for rows of a few entries over a large table (300,000 of 4, 640 columns 577 and
    // 607), nor for the maximum (19,717 of 5, 500 columns 31 and 39).
    const int64_t last_slab = c.F % 256 == 0 ? 256 : c.F % 256;
    if (!gat && vec == 4 && c.mode != RETEXO_MAX && opt.slab_cols == 0 && c.F > 256 &&
        last_slab >= (c.F > 512 ? 64 : c.mode == RETEXO_GCN_SYM ? 192 : 128) &&
        !(p->nnz < 10 * N && N >= 100000 && (c.F > 512 || c.mode == RETEXO_GCN_SYM)))
        nc = 1;
    if (!gat && vec == 4 && c.mode != RETEXO_MAX && nc == 3 && opt.slab_cols == 0 && dense_for_ranges(c)) nc = 2;      // (has levels)
    const int64_t slab_w = 64 * (int64_t)vec * nc;

    AggArgs a;
    a.row_ptr = p->row_ptr;
    a.col_idx = p->col_idx;
    a.order = p->order;
    a.deg = p->deg;
    a.set_deg = p->degrees_set && c.mode == RETEXO_MEAN ? p->deg : nullptr;
    a.dinv = p->dinv;
    a.wsrc = c.mode == RETEXO_GCN_SYM ? p->dinv : nullptr;
    a.Z = c.Z;
    a.ldz = c.ldz;
    a.out = c.out;
    a.ldo = c.ldo;
    a.ocol = c.self_concat ? c.F : 0;
    a.el = nullptr;
    a.el_stride = 0;
    a.er = nullptr;
    a.er_from = nullptr;
    a.row_begin = 0;
    a.row_count = 0;
    a.heavy_rows = 0;
    a.heavy_items = 0;
    a.F = c.F;
    a.nslab = (int)((c.F + slab_w - 1) / slab_w);
    a.slab_major = opt.slab_major < 0 ? 1 : (int)opt.slab_major;
    a.scale = c.mode == RETEXO_MEAN ? SCALE_MEAN : c.mode == RETEXO_GCN_SYM ? SCALE_GCN : SCALE_SUM;
    a.levels = dense_for_ranges(c) ? 1 : 0;
    a.heads = c.heads;
    a.Dh = gat ? (int)(c.F / c.heads) : (int)c.F;
    a.slope = c.slope;
    a.copy_self = (c.self_concat && c.copy_self) ? 1 : 0;
    a.out_vec = aligned_for(c.out + a.ocol, c.ldo, vec) ? 1 : 0;
    a.out_half = (vec == 4 && aligned_for(c.out + a.ocol, c.ldo, 2)) ? 1 : 0;
    a.self_vec = aligned_for(c.out, c.ldo, vec) ? 1 : 0;
    a.part_ptr = nullptr;
    a.n_rows = N;
    a.part_lo = 0;
    a.part_hi = 0;
    a.first = 1;
    a.last = 1;
    a.save_stats = nullptr;
    a.save_pos = nullptr;
    a.save_neg = nullptr;
    a.ld_pos = 0;

    // (the edge softmax over unaligned or very large tables has a launch of its own for the long rows)
    const bool own_launch = gat && !(vec == 4 && opt.gat_fast && gat_route(c).off32);
    int64_t n_heavy = long_rows(p, c.F, own_launch, gat);

    // source-id ranges that the table is walked in, sized so that a range's slab (one 128-byte line per row) stays in L2
    int parts = (int)opt.parts;
    if (parts < 0) {
        parts = 1;
        while (p->part_ptr && parts < kMaxParts && N * 32 * 4 > (int64_t)parts * (8ll << 20)) parts *= 2;
    }
    const LinearRoute linear = linear_route(c, vec, parts);
    // narrow slabs (32/64/128 columns) use the grouped gather; they need float4 gathers
    // (the maximum is only implemented on whole rows)
    int64_t narrow = (!gat && vec == 4 && c.mode != RETEXO_MAX) ? opt.slab_cols : -1;
    if (linear.ranges) narrow = 32;
    if (narrow == 32 || narrow == 64 || narrow == 128) {
        a.nslab = (int)((c.F + narrow - 1) / narrow);
        a.slab_major = opt.slab_major < 0 ? 1 : (int)opt.slab_major;
        if (opt.parts < 0 && narrow != 32) {
            parts = 1;
            while (parts < kMaxParts && N * narrow * 4 > (int64_t)parts * (8ll << 20)) parts *= 2;
        }
        if (!p->part_ptr || (parts != 2 && parts != 4 && parts != 8 && parts != 16)) parts = 1;
        {
            // long-row class by the length of a row's share of one range
            const int64_t want = opt.narrow_heavy * parts;
            n_heavy = 0;
            for (int i = 0; i < kPlanThresholdCount; ++i)
                if (kPlanThresholds[i] >= want || kPlanThresholds[i] >= 16384) {
                    n_heavy = p->rows_at_least[i];
                    break;
                }
            if (parts > 1) a.part_ptr = p->part_ptr;
        }
        for (int k = 0; k < parts; ++k) {
            a.part_lo = k * (kMaxParts / parts);
            a.part_hi = (k + 1) * (kMaxParts / parts);
            a.first = k == 0;
            a.last = k == parts - 1;
            const bool wtd = a.wsrc != nullptr;
            const bool off32 = (N * c.ldz + c.F) * 4 < (1ll << 32) && !opt.wide_offsets;
            a.table_bytes = off32 ? (uint32_t)(((N - 1) * c.ldz + align_up(c.F, 4)) * 4) : 0u;
            if (narrow == 32) dispatch_grouped<8>(a, n_heavy, N, wtd, off32, stream);
            else if (narrow == 64) dispatch_grouped<16>(a, n_heavy, N, wtd, off32, stream);
            else dispatch_grouped<32>(a, n_heavy, N, wtd, off32, stream);
        }
    } else if (linear.lanes) {
        a.table_bytes = (uint32_t)(((N - 1) * c.ldz + (c.F < 4 ? 4 : c.F)) * 4);
        if (linear.lanes == 8)       launch_rows<8>(a, n_heavy, N, stream);
        else if (linear.lanes == 16) launch_rows<16>(a, n_heavy, N, stream);
        else                         launch_rows<32>(a, n_heavy, N, stream);
    } else if (!gat) {
        const bool maxop = c.mode == RETEXO_MAX;
        if (vec == 4) dispatch_linear<4>(nc, maxop, a, n_heavy, N, stream);
        else if (vec == 2) dispatch_linear<2>(nc, maxop, a, n_heavy, N, stream);
        else dispatch_linear<1>(nc, maxop, a, n_heavy, N, stream);
    } else {
        const int hp = heads_padded(c.heads);
        float* el = (float*)c.workspace;
        float* er = (float*)((char*)c.workspace + gat_workspace(N, c.F, c.heads, false).er);
        const bool hu = (a.Dh % vec) == 0;
        const GatRoute route = gat_route(c);
        const bool off32 = route.off32, flash = route.flash, in_rows = route.in_rows;
        const int g = a.Dh / 4;
        const int waves = softmax_waves(p, c.F, c.save && !flash);
        if (c.el_ready && !(in_rows && !c.save && a.nslab == 1)) return RETEXO_E_FLAGS;   // the round asked gat_fold_plan
        a.el_stride = in_rows ? c.ldz : hp;
        if (in_rows) el = const_cast<float*>(c.Z) + c.F;
        a.el = el;
        a.er = er;
        // the plain forward over rows whose scores all come from the gathered rows needs no table
        const bool no_table = flash && !c.save && aligned_for(c.attn_dst, 4, 4);
        // only the pipelined kernel keeps the backward's statistics: decided before anything is launched,
        // so that the error leaves the workspace and the output untouched
        if (c.save && !(vec == 4 && off32 && opt.gat_fast)) return RETEXO_E_FLAGS;
        if (c.el_ready) {
            // the transform wrote the source scores; every row forms its own destination scores
            a.er = nullptr;
            a.er_from = c.attn_dst;
        } else if (!no_table) {
            launch_gat_scores(N, c.F, c.heads, c.Z, c.ldz, c.attn_src, c.attn_dst, el, er, stream, a.el_stride);
        }
        if (c.save) {
            const GatWorkspace w = gat_workspace(N, c.F, c.heads, true);
            a.save_stats = (f32x4*)((char*)c.workspace + w.stats);
            a.save_pos = (float*)((char*)c.workspace + w.pos);
            a.save_neg = (float*)((char*)c.workspace + w.neg);
            a.ld_pos = w.ld_pos;
        }
        // several rows per wave: whole heads of up to 64 columns at a time
        const int slab_heads = flash ? gat_rows_heads(c, a.Dh) : 0;
        if (slab_heads) {
            a.table_bytes = (uint32_t)(((N - 1) * c.ldz + c.F) * 4);
            a.slab_cols = slab_heads * a.Dh;
            a.nslab = (c.heads + slab_heads - 1) / slab_heads;
            const float* ad = no_table ? c.attn_dst : nullptr;
            const int lanes = row_lanes(a.slab_cols);
            auto go = [&](auto gtag) {
                constexpr int GG = decltype(gtag)::value;
                if (c.save) dispatch_gat_rows<GG, true>(lanes, a, n_heavy, N, c.attn_src, nullptr, hp, waves, stream);
                else        dispatch_gat_rows<GG, false>(lanes, a, n_heavy, N, c.attn_src, ad, hp, waves, stream);
            };
            switch (g) {
                case 1:  go(std::integral_constant<int, 1>{}); break;
                case 2:  go(std::integral_constant<int, 2>{}); break;
                case 4:  go(std::integral_constant<int, 4>{}); break;
                case 8:  go(std::integral_constant<int, 8>{}); break;
                default: go(std::integral_constant<int, 16>{}); break;
            }
        } else if (flash) {
            AggArgs f = a;
            f.nslab = 1;
            const dim3 grid(both_classes(f, n_heavy, N, waves)), block(64 * waves);
            const float* ad = no_table ? c.attn_dst : nullptr;
            auto go = [&](auto gtag) {
                constexpr int GG = decltype(gtag)::value;
                if (c.save && waves == 4) agg_gat_flash_kernel<GG, true, 4><<<grid, block, 0, stream>>>(f, c.attn_src, nullptr, hp);
                else if (c.save)          agg_gat_flash_kernel<GG, true, 8><<<grid, block, 0, stream>>>(f, c.attn_src, nullptr, hp);
                else if (waves == 4)      agg_gat_flash_kernel<GG, false, 4><<<grid, block, 0, stream>>>(f, c.attn_src, ad, hp);
                else                      agg_gat_flash_kernel<GG, false, 8><<<grid, block, 0, stream>>>(f, c.attn_src, ad, hp);
            };
            switch (g) {
                case 1:  go(std::integral_constant<int, 1>{}); break;
                case 2:  go(std::integral_constant<int, 2>{}); break;
                case 4:  go(std::integral_constant<int, 4>{}); break;
                case 8:  go(std::integral_constant<int, 8>{}); break;
                case 16: go(std::integral_constant<int, 16>{}); break;
                case 32: go(std::integral_constant<int, 32>{}); break;
                default: go(std::integral_constant<int, 64>{}); break;
            }
        } else if (vec == 4 && off32 && opt.gat_fast) {
            if (hp == 4) { if (hu) dispatch_gat_fast<4, true>(nc, c.save, a, n_heavy, N, waves, stream); else dispatch_gat_fast<4, false>(nc, c.save, a, n_heavy, N, waves, stream); }
            else         { if (hu) dispatch_gat_fast<8, true>(nc, c.save, a, n_heavy, N, waves, stream); else dispatch_gat_fast<8, false>(nc, c.save, a, n_heavy, N, waves, stream); }
        } else if (vec == 4) {
            if (hp == 4) { if (hu) dispatch_gat_nc<4, 4, true>(nc, a, n_heavy, N, stream); else dispatch_gat_nc<4, 4, false>(nc, a, n_heavy, N, stream); }
            else         { if (hu) dispatch_gat_nc<4, 8, true>(nc, a, n_heavy, N, stream); else dispatch_gat_nc<4, 8, false>(nc, a, n_heavy, N, stream); }
        } else {
            if (hp == 4) dispatch_gat_nc<1, 4, true>(nc, a, n_heavy, N, stream);
            else         dispatch_gat_nc<1, 8, true>(nc, a, n_heavy, N, stream);
        }
    }
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
