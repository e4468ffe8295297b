// Device helpers shared by the gather kernels (aggregation forward and backward):
// row loads/stores of VEC floats per lane, wave reductions and lane broadcasts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // at any float's address

constexpr int kLightWaves = 4;   // independent rows per workgroup in the light kernels
constexpr int kHeavyWaves = 8;   // cooperating waves per row in the heavy kernels
constexpr int kUnroll = 4;       // neighbours fetched per unrolled step

template <int VEC>
__device__ __forceinline__ void load_row(const float* p, float (&v)[VEC])
{
    if constexpr (VEC == 4) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else if constexpr (VEC == 2) {
        const f32x2 t = *reinterpret_cast<const f32x2*>(p);
        v[0] = t.x; v[1] = t.y;
    } else {
        v[0] = *p;
    }
}

// vec_ok: p allows one VEC-wide store; half_ok (VEC == 4 only): p is 8-byte aligned, two 8-byte stores — the
// aggregate half of a concatenated row of odd half-width (602 columns) starts 8 bytes into a 16-byte piece,
// and four scalar stores per lane cost six times the L2 write requests of one wide store
template <int VEC>
__device__ __forceinline__ void store_row(float* p, const float (&v)[VEC], int valid, bool vec_ok, bool half_ok = false)
{
    if constexpr (VEC == 4) {
        if (!vec_ok && half_ok && valid >= 4) {
            *reinterpret_cast<f32x2*>(p) = f32x2{v[0], v[1]};
            *reinterpret_cast<f32x2*>(p + 2) = f32x2{v[2], v[3]};
            return;
        }
    }
    if (vec_ok && valid >= VEC) {
        if constexpr (VEC == 4) {
            f32x4 t = {v[0], v[1], v[2], v[3]};
            *reinterpret_cast<f32x4*>(p) = t;
        } else if constexpr (VEC == 2) {
            f32x2 t = {v[0], v[1]};
            *reinterpret_cast<f32x2*>(p) = t;
        } else {
            *p = v[0];
        }
    } else {
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            if (k < valid) p[k] = v[k];
    }
}

// those of four floats that are the lane's own (see own_columns): [skip, valid)
__device__ __forceinline__ void store_own(float* p, const float (&v)[4], int skip, int valid, bool vec_ok, bool half_ok = false)
{
    if (skip == 0 && valid == 4) {
        if (vec_ok || half_ok) store_row<4>(p, v, 4, vec_ok, half_ok);
        else *reinterpret_cast<f32x4u*>(p) = f32x4u{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k >= skip && k < valid) p[k] = v[k];
    }
}

// data that is read once per pass (indices, row bookkeeping, running sums) is fetched with a
// non-temporal hint so that it does not push the reused feature rows out of L2
template <typename T>
__device__ __forceinline__ T ldg_stream(const T* p) { return __builtin_nontemporal_load(p); }

// A table below 4 GiB as a buffer: a 16-byte load at an offset past its end fetches nothing and returns zeros.  So an entry
// that does not exist is an offset (kNoEntry, which stays the largest under the saturating addition of a column offset)
// and costs neither a comparison nor a cleared register in the loops that gather.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kNoEntry = 0xffffffffu;
typedef __amdgpu_buffer_rsrc_t table_t;
__device__ __forceinline__ table_t buffer_table(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 load_entry(table_t t, uint32_t row, uint32_t col)
{
    return __builtin_amdgcn_raw_buffer_load_b128(t, __builtin_elementwise_add_sat(row, col), 0, 0);
}

// Rows, or slabs of rows, that a wave need not hold alone: P lanes (4 to 64) of four floats, or of four or eight 16-bit elements, hold
// one, and the R = 64 / P groups of a wave walk a list of entries each, in lock step: R rows of neighbouring length, or R shares of one long row.  A
// gather instruction so carries R entries, where one entry per instruction leaves 64 - P lanes idle and the kernels wait
// for as many round trips to memory as a row has batches.
// Every lane fetches four consecutive ids at a time (a tile of 4 P entries per group, whole cache lines of col_idx, a tile
// ahead of its use); entry t of the four in lane l of the group is entry 4 l + t of the tile.  A batch is the four entries
// of one lane.  What does not exist is the offset kNoEntry and fetches nothing.
// KEEP_ID: the ids themselves as well (for a second table).
template <int P, bool KEEP_ID = false>
struct EntryWalk {
    static constexpr uint32_t kTile = 4 * P;
    const int32_t* __restrict__ col;
    uint32_t hi, ahead, step;            // end of the list; first entry of the tile in `nxt`; distance of a group's tiles
    uint32_t rowbytes;
    int li, gaddr;
    uint32_t off[4], nxt[4];             // byte offsets of the current tile's entries; ids of the one after it
    uint32_t id[KEEP_ID ? 4 : 1];

    __device__ __forceinline__ void fetch()
    {
        typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));
        const uint32_t at = ahead + 4 * li;          // (entry counts stay below 2^31)
        if (at + 4 <= hi) {
            const i32x4u t = *reinterpret_cast<const i32x4u*>(col + at);
            nxt[0] = (uint32_t)t.x; nxt[1] = (uint32_t)t.y; nxt[2] = (uint32_t)t.z; nxt[3] = (uint32_t)t.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) nxt[k] = at + k < hi ? (uint32_t)col[at + k] : kNoEntry;
        }
    }
    // The group's entries: tiles that start at first, first + step_, ... up to hi_.  Returns the number of batches of the
    // wave's longest list (uniform).
    __device__ __forceinline__ int start(const int32_t* col_idx, uint32_t first, uint32_t hi_, uint32_t step_, uint32_t rowbytes_)
    {
        const int lane = threadIdx.x & 63;
        col = col_idx; hi = hi_; ahead = min(first, hi_); step = step_; rowbytes = rowbytes_;
        li = lane % P; gaddr = (lane - li) * 4;
        fetch();
        int n = 0;
        if (first < hi) {
            const uint32_t tiles = (hi - first - 1) / step, rest = hi - (first + tiles * step);
            n = (int)(tiles * P + (min(rest, kTile) + 3) / 4);
        }
#pragma unroll
        for (int m = P; m < 64; m <<= 1) n = max(n, __shfl_xor(n, m, 64));
        take();
        return __builtin_amdgcn_readfirstlane(n);
    }
    // the tile that was fetched becomes the current one, the next is requested
    __device__ __forceinline__ void take()
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            off[k] = nxt[k] == kNoEntry ? kNoEntry : nxt[k] * rowbytes;
            if constexpr (KEEP_ID) id[k] = nxt[k];
        }
        ahead = hi - ahead > step ? ahead + step : hi;
        fetch();
    }
    // byte offset of entry t of batch j of the current tile
    __device__ __forceinline__ uint32_t at(int j, int t) const
    {
        return (uint32_t)__builtin_amdgcn_ds_bpermute(gaddr + 4 * j, (int)off[t]);
    }
    __device__ __forceinline__ uint32_t id_at(int j, int t) const
    {
        return (uint32_t)__builtin_amdgcn_ds_bpermute(gaddr + 4 * j, (int)id[t]);
    }
};

// The running sum of a list of entries that a lane group walks by itself, from the sums of its batches of eight.  LEVELS: of two
// batches, of eight such pairs (128 entries), then of the 128s.  One sum over the whole list loses more the longer it is: terms of
// one sign, 2-norm of the error, 70, 100 and 300 entries 1.2e-7, 1.5e-7 and 2.4e-7, so 4.9e-8, 5.5e-8 and 4.9e-8, where a walk in
// source ranges that each add to the result, which takes such lists too, gives 5.4e-8 and 6.0e-8 (70 in eight, 100 in four).  A list of a few
// entries pays for it (1,000,000 rows of 8, 64 columns, with weights 459 us and 481), so the calls that could take ranges have it.
template <int K, bool LEVELS>
struct BatchSums {
    float all[K], tile[LEVELS ? K : 1], pair[LEVELS ? K : 1];
    __device__ __forceinline__ BatchSums()
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            all[k] = 0.0f;
            if constexpr (LEVELS) tile[k] = 0.0f;
        }
    }
    // batch i, i even; its sum
    __device__ __forceinline__ void even(const float (&sum)[K])
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (LEVELS) pair[k] = sum[k];
            else all[k] += sum[k];
        }
    }
    // ... and that of batch i + 1
    __device__ __forceinline__ void odd(int i, const float (&sum)[K])
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (LEVELS) tile[k] += pair[k] + sum[k];
            else all[k] += sum[k];
        }
        if constexpr (LEVELS) {
            if ((i & 14) == 14) flush();         // (uniform)
        }
    }
    // an even batch without an odd one after it
    __device__ __forceinline__ void last_even()
    {
        if constexpr (LEVELS) {
#pragma unroll
            for (int k = 0; k < K; ++k) tile[k] += pair[k];
        }
    }
    __device__ __forceinline__ void flush()
    {
        if constexpr (LEVELS) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                all[k] += tile[k];
                tile[k] = 0.0f;
            }
        }
    }
};

// lanes that hold a row of F columns, up to 256, four columns each
inline int row_lanes(int64_t F) { return F <= 32 ? 8 : F <= 64 ? 16 : F <= 128 ? 32 : 64; }

__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
    return x;
}

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// several values at once, step by step: COUNT independent moves are in flight at each of the six steps (one value after the
// other is a chain of 6 * COUNT of them, which the compiler may or may not interleave)
template <int COUNT>
__device__ __forceinline__ void wave_max(float (&x)[COUNT])
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        float t[COUNT];
#pragma unroll
        for (int i = 0; i < COUNT; ++i) t[i] = __shfl_xor(x[i], m, 64);
#pragma unroll
        for (int i = 0; i < COUNT; ++i) x[i] = fmaxf(x[i], t[i]);
    }
}
template <int COUNT>
__device__ __forceinline__ void wave_sum(float (&x)[COUNT])
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        float t[COUNT];
#pragma unroll
        for (int i = 0; i < COUNT; ++i) t[i] = __shfl_xor(x[i], m, 64);
#pragma unroll
        for (int i = 0; i < COUNT; ++i) x[i] += t[i];
    }
}

__device__ __forceinline__ int bcast_i(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
__device__ __forceinline__ float bcast_f(float x, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// sum over aligned groups of G neighbouring lanes (G a power of two): up to 16 lanes with DPP moves inside
// a row of 16, beyond that with cross-row shuffles
template <int G>
__device__ __forceinline__ float group_sum(float x)
{
    // butterfly over the G lanes of a head; every lane ends with the group's sum
    if constexpr (G >= 2) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
    if constexpr (G >= 4) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
    if constexpr (G >= 8) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, true));  // row_half_mirror
    if constexpr (G >= 16) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, true)); // row_mirror
    if constexpr (G >= 32) x += __shfl_xor(x, 16, 64);
    if constexpr (G >= 64) x += __shfl_xor(x, 32, 64);
    return x;
}

// pick s[h] for a per-lane head index from per-head wave-uniform values
template <int HP>
__device__ __forceinline__ float select_head(const float (&s)[HP], int h)
{
    float r = s[0];
#pragma unroll
    for (int i = 1; i < HP; ++i) r = (h == i) ? s[i] : r;
    return r;
}

}  // namespace
