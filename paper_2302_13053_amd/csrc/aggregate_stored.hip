// Aggregation over a feature table kept in 16-bit storage (bfloat16 or IEEE half).
//
// The aggregation is bound by the bytes it gathers (one row of Z per CSR entry),
// so a table stored in 16 bits moves half of them.  This is a variant outside
// the fp32 results: the stored value is the float32 value rounded to nearest
// even in the target format (retexo_store_rows), every sum is still accumulated
// in float32 and the output is float32.  Against the same rounded table the
// result obeys the same 1e-5 bound as the fp32 path; against the unrounded
// table the difference is the rounding of the storage format.
//
// Kernels (each decodes 16-byte loads of eight elements per lane):
//   * whole rows per wave, for sum / mean / gcn_sym / max        (any shape; scalar loads when unaligned)
//   * several rows, or slabs of rows, per wave for sum / mean / gcn_sym (up to 128 columns; any width at 4-byte addresses)
//   * 64-column slabs, one row per 8-lane group, walked source range by source range so that the
//     slab of the current range stays in L2 (dense graphs; same plan split as the fp32 path)
//   * edge softmax, whole rows per wave, software-pipelined with per-edge weights in LDS
//   * edge softmax, several rows per wave, scores from the gathered rows (heads of a power of two of four-element lanes)
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "gather.hpp"

namespace {

enum { FMT_BF16 = RETEXO_STORE_BF16, FMT_FP16 = RETEXO_STORE_FP16 };

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int FMT>
__device__ __forceinline__ float decode1(uint16_t x)
{
    if constexpr (FMT == FMT_BF16) {
        return __uint_as_float((uint32_t)x << 16);
    } else {
        _Float16 h;
        __builtin_memcpy(&h, &x, 2);
        return (float)h;
    }
}

// eight stored elements (16 bytes) -> floats
template <int FMT>
__device__ __forceinline__ void decode8(const u32x4& raw, float (&v)[8])
{
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (FMT == FMT_BF16) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        } else {
            v[2 * i] = decode1<FMT>((uint16_t)(w[i] & 0xffffu));
            v[2 * i + 1] = decode1<FMT>((uint16_t)(w[i] >> 16));
        }
    }
}

// acc += w * the eight stored elements; without weights IEEE half still goes through the multiply-add, which converts on
// the way (v_fma_mix_f32; a conversion and an addition otherwise): `w` is then one, held in a register on purpose
template <int FMT, bool WEIGHTED>
__device__ __forceinline__ void add8(const u32x4& raw, float w, float (&acc)[8])
{
    float z[8];
    decode8<FMT>(raw, z);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = WEIGHTED || FMT == FMT_FP16 ? fmaf(w, z[k], acc[k]) : acc[k] + z[k];
}
// the first term of a sum
template <int FMT, bool WEIGHTED>
__device__ __forceinline__ void first8(const u32x4& raw, float w, float (&acc)[8])
{
    float z[8];
    decode8<FMT>(raw, z);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = WEIGHTED ? w * z[k] : FMT == FMT_FP16 ? fmaf(w, z[k], 0.0f) : z[k];
}
__device__ __forceinline__ float register_one()
{
    float one = 1.0f;
    asm("" : "+v"(one));
    return one;
}

template <int FMT>
__device__ __forceinline__ uint16_t encode1(float x)
{
    if constexpr (FMT == FMT_BF16) {
        const uint32_t b = __float_as_uint(x);
        if (x != x) return (uint16_t)((b >> 16) | 0x0040u);                   // NaN stays NaN (quiet)
        return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);            // nearest, ties to even
    } else {
        const _Float16 h = (_Float16)x;                                       // hardware conversion: nearest even
        uint16_t r;
        __builtin_memcpy(&r, &h, 2);
        return r;
    }
}

// `count` (1 to 4) converted elements to p, which is on 8 bytes
template <int FMT>
__device__ __forceinline__ void store4(uint16_t* p, const f32x4& x, int count)
{
    const u32x2 y = {(uint32_t)encode1<FMT>(x.x) | (uint32_t)encode1<FMT>(x.y) << 16,
                     (uint32_t)encode1<FMT>(x.z) | (uint32_t)encode1<FMT>(x.w) << 16};
    if (count == 4) *reinterpret_cast<u32x2*>(p) = y;
    else {
        if (count >= 2) *reinterpret_cast<uint32_t*>(p) = y.x;
        if (count == 3) p[2] = (uint16_t)y.y;
        if (count == 1) p[0] = (uint16_t)y.x;
    }
}

// 2^lg lanes per row, VEC consecutive columns per lane (16-byte reads and 8-byte writes where rows allow them), U rows in
// flight per lane.  Bound by its bytes: Reddit-shaped table, 232,965 x 602, 143 us = 5.9 TB/s.
// Rows that fewer lanes cover have several of them in a wave: with a wave each most lanes
// are idle (2,400,000 x 8 without padding 236 us, 20 now; x 41 in rows of 64 491 and 176).
// STREAM: past the caches, for a table that they cannot hold anyway (2,400,000 x 8 of rows of 128 bytes 159 -> 78 us;
// 1,000,000 x 8, which the last of them holds, 30 -> 37).
template <int FMT, int VEC, int U, bool STREAM>
__global__ __launch_bounds__(256) void store_rows_kernel(int64_t N, int64_t F, const float* __restrict__ src,
                                                          int64_t lds, uint16_t* __restrict__ dst, int64_t ldd, int lg)
{
    const int64_t apart = 256 >> lg, step = (int64_t)gridDim.x * apart * U;      // rows between a thread's
    const int64_t c0 = (int64_t)(threadIdx.x & ((1u << lg) - 1u)) * VEC, cstep = (int64_t)VEC << lg;
    for (int64_t r0 = (int64_t)blockIdx.x * apart * U + (threadIdx.x >> lg); r0 < N; r0 += step) {
        for (int64_t c = c0; c < F; c += cstep) {
            const float* from = src + r0 * lds + c;
            uint16_t* to = dst + r0 * ldd + c;
            const int count = (int)min((int64_t)VEC, F - c);
            if constexpr (VEC == 4) {
                f32x4 x[U];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    if (r0 + t * apart >= N) break;
                    const float* f = from + t * apart * lds;
                    // (behind the last columns of a row lies its padding; the last row may end with the buffer)
                    if (count == 4 || r0 + t * apart < N - 1) {
                        if constexpr (STREAM) x[t] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(f));
                        else x[t] = *reinterpret_cast<const f32x4*>(f);
                    } else {
                        x[t] = f32x4{f[0], 0.0f, 0.0f, 0.0f};
                        if (count > 1) x[t].y = f[1];
                        if (count > 2) x[t].z = f[2];
                    }
                }
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    if (r0 + t * apart >= N) break;
                    store4<FMT>(to + t * apart * ldd, x[t], count);
                }
            } else {
                float x[U];
#pragma unroll
                for (int t = 0; t < U; ++t) x[t] = r0 + t * apart < N ? from[t * apart * lds] : 0.0f;
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (r0 + t * apart < N) to[t * apart * ldd] = encode1<FMT>(x[t]);
            }
        }
    }
}

// the same for rows without padding, which are one run of n elements
template <int FMT>
__global__ __launch_bounds__(256) void store_run_kernel(int64_t n, const float* __restrict__ src, uint16_t* __restrict__ dst)
{
    constexpr int U = 4;
    const int64_t step = (int64_t)gridDim.x * 256 * 4;
    for (int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i0 < n; i0 += step * U) {
        f32x4 x[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int64_t i = i0 + t * step;
            if (i + 4 <= n) {
                x[t] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + i));
            } else if (i < n) {
                x[t] = f32x4{src[i], 0.0f, 0.0f, 0.0f};
                if (i + 1 < n) x[t].y = src[i + 1];
                if (i + 2 < n) x[t].z = src[i + 2];
            }
        }
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int64_t i = i0 + t * step;
            if (i < n) store4<FMT>(dst + i, x[t], (int)min((int64_t)4, n - i));
        }
    }
}

// row loads of E stored elements per lane (E = 8: one 16-byte load; 4: one 8-byte load; 1: one 2-byte load)
template <int FMT, int E>
__device__ __forceinline__ void load_stored(const uint16_t* p, float (&v)[E])
{
    if constexpr (E == 8) {
        const u32x4 raw = *reinterpret_cast<const u32x4*>(p);
        decode8<FMT>(raw, v);
    } else if constexpr (E == 4) {
        const u32x2 raw = *reinterpret_cast<const u32x2*>(p);
        const uint32_t w[2] = {raw.x, raw.y};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if constexpr (FMT == FMT_BF16) {
                v[2 * i] = __uint_as_float(w[i] << 16);
                v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
            } else {
                v[2 * i] = decode1<FMT>((uint16_t)(w[i] & 0xffffu));
                v[2 * i + 1] = decode1<FMT>((uint16_t)(w[i] >> 16));
            }
        }
    } else {
        v[0] = decode1<FMT>(*p);
    }
}

// vec_ok: 16-byte stores; half_ok: p is at least 8-byte aligned (the aggregate half of a concatenated row of odd
// half-width): 8-byte stores instead of one per element
template <int E>
__device__ __forceinline__ void store_floats(float* p, const float (&v)[E], int valid, bool vec_ok, bool half_ok = false)
{
    if (E % 2 == 0 && !vec_ok && half_ok && valid >= E) {
#pragma unroll
        for (int k = 0; k < E; k += 2) *reinterpret_cast<f32x2*>(p + k) = f32x2{v[k], v[k + 1 < E ? k + 1 : k]};
        return;
    }
    if (E == 8 && vec_ok && valid >= 8) {
        const f32x4 a = {v[0], v[1], v[2], v[3]}, b = {v[E > 4 ? 4 : 0], v[E > 5 ? 5 : 0], v[E > 6 ? 6 : 0], v[E > 7 ? 7 : 0]};
        *reinterpret_cast<f32x4*>(p) = a;
        *reinterpret_cast<f32x4*>(p + 4) = b;
    } else if (E == 4 && vec_ok && valid >= 4) {
        const f32x4 a = {v[0], v[E > 1 ? 1 : 0], v[E > 2 ? 2 : 0], v[E > 3 ? 3 : 0]};
        *reinterpret_cast<f32x4*>(p) = a;
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k)
            if (k < valid) p[k] = v[k];
    }
}

struct StoredArgs {
    const int64_t* row_ptr;
    const int32_t* col_idx;
    const int32_t* order;
    const int32_t* deg;
    const int32_t* set_deg;  // what a mean divides by where it is not the row's length (retexo_plan_set_degrees); else NULL: a load less
    const float* dinv;
    const float* wsrc;       // per-source weights (gcn_sym: dinv) or NULL
    const uint16_t* Z;
    int64_t ldz;             // in elements
    float* out;
    int64_t ldo;
    int64_t ocol;
    const float* el;
    const float* er;
    int64_t row_begin, row_count;
    int64_t F;
    int nslab;
    int scale;               // 0 sum, 1 mean, 2 gcn
    int heads, Dh;
    float slope;
    int copy_self;
    int out_vec;             // aggregate half of out allows 16-byte stores
    int out_half;            // ... or at least 8-byte stores
    int self_vec;
    const int32_t* part_ptr;
    int64_t n_rows;
    int part_lo, part_hi;
    int first, last;
    uint32_t table_bytes;    // up to the end of the last row's last vector (narrow slabs and row groups: below 4 GiB)
    int own_rows;            // rows hold whole vectors of eight elements (see stored_rows_kernel)
    uint32_t slab_blocks;    // workgroups per slab of stored_rows_kernel, heavy_rows of them with one row each
    int64_t heavy_rows;
};

// ---------------------------------------------------------------------------
// sum / mean / gcn_sym / max, whole rows: one wave per (row, slab of 64*E*NC columns)
// ---------------------------------------------------------------------------
template <int FMT, int E, int NC, int NW, bool MAXOP>
__global__ __launch_bounds__(64 * (NW == 1 ? kLightWaves : NW)) void stored_linear_kernel(StoredArgs a)
{
    constexpr int U = E == 8 ? 2 : kUnroll;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t items = a.row_count * a.nslab;
    const int64_t item = (NW == 1) ? (int64_t)blockIdx.x * kLightWaves + wave : (int64_t)blockIdx.x;
    if (item >= items) return;
    const int64_t slot = item / a.nslab;
    const int slab = (int)(item % a.nslab);
    const int v = __builtin_amdgcn_readfirstlane(a.order[a.row_begin + slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);
    const int d = a.set_deg ? a.set_deg[v] : hi - lo;

    const int64_t col0 = (int64_t)slab * (64 * E * NC) + lane * E;
    bool act[NC];
    int64_t colsafe[NC];
    float acc[NC][E];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t col = col0 + c * 64 * E;
        act[c] = col < a.F;
        colsafe[c] = act[c] ? col : 0;        // lanes past the row width gather column 0 (never stored)
#pragma unroll
        for (int k = 0; k < E; ++k) acc[c][k] = MAXOP ? -INFINITY : 0.0f;
    }
    const bool weighted = a.wsrc != nullptr;

    for (int base = lo + 64 * (NW == 1 ? 0 : wave); base < hi; base += 64 * NW) {
        const int e = base + lane;
        const bool valid = e < hi;
        int my_u = valid ? a.col_idx[e] : 0;
        my_u = valid ? my_u : bcast_i(my_u, 0);
        const float my_w = weighted ? (valid ? a.wsrc[my_u] : 0.0f) : (valid ? 1.0f : 0.0f);
        const int cnt = min(64, hi - base);
        for (int j = 0; j < cnt; j += U) {
            float z[U][NC][E], w[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int jj = (j + t) & 63;                        // past the tile: a repeat with weight zero
                const uint16_t* zr = a.Z + (int64_t)bcast_i(my_u, jj) * a.ldz;
                w[t] = j + t < cnt ? bcast_f(my_w, jj) : 0.0f;
#pragma unroll
                for (int c = 0; c < NC; ++c) load_stored<FMT, E>(zr + colsafe[c], z[t][c]);
            }
#pragma unroll
            for (int t = 0; t < U; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int k = 0; k < E; ++k) {
                        if constexpr (MAXOP) acc[c][k] = j + t < cnt ? fmaxf(acc[c][k], z[t][c][k]) : acc[c][k];
                        else acc[c][k] = fmaf(w[t], z[t][c][k], acc[c][k]);
                    }
        }
    }

    if constexpr (NW > 1) {
        __shared__ float red[NW][NC * E][64];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) red[wave][c * E + k][lane] = acc[c][k];
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) {
                float s = red[0][c * E + k][lane];
#pragma unroll
                for (int w = 1; w < NW; ++w) s = MAXOP ? fmaxf(s, red[w][c * E + k][lane]) : s + red[w][c * E + k][lane];
                acc[c][k] = s;
            }
    }

    float* orow = a.out + (int64_t)v * a.ldo;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (!act[c]) continue;
        const int64_t col = col0 + c * 64 * E;
        const int valid = (int)min((int64_t)E, a.F - col);
        float r[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            float x = acc[c][k];
            if (MAXOP) x = d > 0 ? x : 0.0f;
            else if (a.scale == 1) x = d > 0 ? x / (float)d : 0.0f;
            else if (a.scale == 2) x = x * a.dinv[v];
            r[k] = x;
        }
        store_floats<E>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
        if (a.copy_self) {
            float zs[E];
            load_stored<FMT, E>(a.Z + (int64_t)v * a.ldz + col, zs);
            store_floats<E>(orow + col, zs, valid, a.self_vec != 0);
        }
    }
}

// ---------------------------------------------------------------------------
// sum / mean / gcn_sym on 64-column slabs: one row per 8-lane group, eight elements per lane, so a
// gathered row-slab is one 128-byte line.  Launched once per group of source-id ranges: the running
// sum is kept in `out` between launches.
//
// Bound by the address units and, with two instructions per element, nearly as much by the vector units.  So an
// entry that a lane's row does not have is an offset past the table's end (a sixth of a bundle's gathers are such fillers),
// which costs neither a fetch nor an instruction (zero bits decode to +0 in both formats), sums without weights hand round
// no weights, and the next step's gathers are issued before the current ones are added up.
// Reddit-shaped graph, 602 columns, bf16, four ranges: 2.17 -> 1.94 ms per range, long rows 0.335 -> 0.297, the whole mean
// 10.36 -> 9.05 ms with the store; gcn_sym 13.0 -> 11.9.  What is left is the L2 requests and misses of the gathers (18.8 TB/s; the
// float32 kernel 20.1) and the running sums, twice its bytes per slab.
// U entries per step: eight keep twice as many gathers in flight per wave, four more waves (85 registers instead of 117).
// Eight where the slab of the table fits L2 or nearly does, so that latency and not misses bounds the call (bf16 mean, 8,847
// nodes of 328 entries, 256 columns 97 us with eight, 108 with four; 100,000 of 100 438 and 472, gcn_sym 606 and 631), and
// without weights also where it is the only slab and a row of a range is walked longer than all others of the launch take:
// eight walk it in half the steps.  That is a share of 64 entries per range the table is cut into, or more (64 columns, eight and
// four: 600,000 nodes of 120, sixteen ranges, longest row 26,500 2,240 and 2,583, 9,640 2,059 and 1,941, all rows alike 2,163
// and 2,008; 300,000 of 120, eight ranges, longest 31,600 798 and 984, 5,000 535 and 651, 3,100 531 and 494, 1,100 538 and 496).
// Four otherwise (200 columns 8,279 and 8,101, gcn_sym 10,748 and 9,640; the Reddit-shaped mean of 602 columns 9,081 and 9,034).
// ---------------------------------------------------------------------------
template <int FMT, bool WEIGHTED, int U>
__global__ __launch_bounds__(64 * kLightWaves) void stored_rowgroup_kernel(StoredArgs a)
{
    constexpr int LPG = 8, G = 64 / LPG;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t bundles = (a.row_count + G - 1) / G;
    const int64_t item = (int64_t)blockIdx.x * kLightWaves + wave;
    if (item >= bundles * a.nslab) return;
    const int slab = (int)(item / bundles);                 // slab-major: neighbouring waves share a slab
    const int64_t bundle = item % bundles;

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
    int maxlen = len;
#pragma unroll
    for (int m = LPG; m < 64; m <<= 1) maxlen = max(maxlen, __shfl_xor(maxlen, m, 64));
    maxlen = __builtin_amdgcn_readfirstlane(maxlen);

    const int64_t col = (int64_t)slab * 64 + li * 8;
    const bool act = col < a.F;
    const bool writer = act && has_row;
    const int valid = (int)min((int64_t)8, a.F - col);
    const table_t table = buffer_table(a.Z, a.table_bytes);
    const uint32_t colbytes = act ? (uint32_t)(col * 2) : kNoEntry;
    const uint32_t rowbytes = (uint32_t)(a.ldz * 2);
    float* orow = a.out + (int64_t)v * a.ldo;

    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
    if (!a.first && writer) {
        if (a.out_vec && valid >= 8) {
            const f32x4 p0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(orow + a.ocol + col));
            const f32x4 p1 = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(orow + a.ocol + col + 4));
            acc[0] = p0.x; acc[1] = p0.y; acc[2] = p0.z; acc[3] = p0.w;
            acc[4] = p1.x; acc[5] = p1.y; acc[6] = p1.z; acc[7] = p1.w;
        } else if (a.out_half && valid >= 8) {
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
                const f32x2 t = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(orow + a.ocol + col + k));
                acc[k] = t.x;
                acc[k + 1] = t.y;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < valid) acc[k] = orow[a.ocol + col + k];
        }
    }

    const int gaddr = (lane - li) * 4;          // ds_bpermute byte address of this group's lane 0
    // Neighbour ids: every lane of a group fetches eight consecutive ids at a time, so a group reads col_idx in
    // whole cache lines (64 entries) a block ahead of its use; entry e of a block sits in component e % 8 of the
    // group's lane e / 8.  Past the end of a row: id -1, which becomes kNoEntry and fetches zeros, so that nothing of an
    // unrelated row can reach the sum.
    constexpr int IPL = 8, BLOCK = IPL * LPG;
    typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));      // 4-byte aligned 16-byte load
    int nxt_u[IPL];
    float nxt_w[IPL];
    auto fetch_ids = [&](int first) {
        const int nb = first + IPL * li;
        if (nb + IPL <= len) {
#pragma unroll
            for (int k = 0; k < IPL; k += 4) {
                const i32x4u t = *reinterpret_cast<const i32x4u*>(a.col_idx + lo + nb + k);
                nxt_u[k] = t.x; nxt_u[k + 1] = t.y; nxt_u[k + 2] = t.z; nxt_u[k + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < IPL; ++k) nxt_u[k] = nb + k < len ? a.col_idx[lo + nb + k] : -1;
        }
        if constexpr (WEIGHTED) {
#pragma unroll
            for (int k = 0; k < IPL; ++k) nxt_w[k] = nb + k < len ? a.wsrc[nxt_u[k]] : 0.0f;
        }
    };
    const float one = WEIGHTED ? 1.0f : register_one();
    fetch_ids(0);
    for (int s0 = 0; s0 < maxlen; s0 += BLOCK) {
        uint32_t my_off[IPL];
        float my_w[IPL];
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            my_off[k] = nxt_u[k] >= 0 ? (uint32_t)nxt_u[k] * rowbytes : kNoEntry;
            my_w[k] = WEIGHTED ? nxt_w[k] : 0.0f;
        }
        fetch_ids(s0 + BLOCK);
        constexpr int T = BLOCK / U;
        u32x4 raw[2][U];
        float w[2][U];
        // e0: first entry of the step in the block
        auto issue = [&](int e0, u32x4 (&rr)[U], float (&ww)[U]) {
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int e = e0 + t;
                rr[t] = load_entry(table, (uint32_t)__builtin_amdgcn_ds_bpermute(gaddr + 4 * (e / IPL), (int)my_off[e % IPL]), colbytes);
                if constexpr (WEIGHTED)
                    ww[t] = __int_as_float(__builtin_amdgcn_ds_bpermute(gaddr + 4 * (e / IPL), __float_as_int(my_w[e % IPL])));
                else
                    ww[t] = one;
            }
        };
        issue(0, raw[0], w[0]);
#pragma unroll
        for (int st = 0; st < T; ++st) {
            const int c0 = s0 + st * U;
            if (c0 >= maxlen) break;                     // (uniform)
            if (st + 1 < T && c0 + U < maxlen) issue((st + 1) * U, raw[(st + 1) & 1], w[(st + 1) & 1]);
#pragma unroll
            for (int t = 0; t < U; ++t) add8<FMT, WEIGHTED>(raw[st & 1][t], w[st & 1][t], acc);
        }
    }
    if (!writer) return;
    const int d = (a.last && a.scale == 1) ? a.deg[v] : 0;      // only the mean's last range needs it
    float r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        float x = acc[k];
        if (a.last) {
            if (a.scale == 1) x = d > 0 ? x / (float)d : 0.0f;
            else if (a.scale == 2) x = x * a.dinv[v];
        }
        r[k] = x;
    }
    store_floats<8>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self && a.first) {
        float zs[8];
        load_stored<FMT, 8>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_floats<8>(orow + col, zs, valid, a.self_vec != 0);
    }
}

// ---------------------------------------------------------------------------
// sum / mean / gcn_sym of rows, or slabs, of 8 P columns: P lanes of eight elements hold a row, and the R = 64 / P groups of a
// wave walk R rows of the schedule, or shares of one long row, in lock step (EntryWalk).  Long rows first in every slab, one per
// workgroup, their shares added up over the groups and then over the waves in order; one launch for both classes.
// Bound by memory latency on small graphs, where R rows wait together, and by the gathered lines on large ones.
// rows_lanes says where it is taken, and what it measures.
// ---------------------------------------------------------------------------
template <int FMT, int P, bool WEIGHTED>
__global__ __launch_bounds__(64 * kHeavyWaves) void stored_rows_kernel(StoredArgs a)
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
    const uint32_t rowbytes = (uint32_t)(a.ldz * 2);
    int batches = heavy ? walk.start(a.col_idx, lo + Walk::kTile * (wave * R + g), hi, Walk::kTile * NW * R, rowbytes)
                        : walk.start(a.col_idx, lo, hi, Walk::kTile, rowbytes);
    batches = (batches + PER - 1) / PER;
    // the weights of the current tile's entries, requested with its first gathers, and of the one before it
    float w_cur[4] = {0.0f, 0.0f, 0.0f, 0.0f}, w_prev[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto weights = [&]() {
        if constexpr (WEIGHTED) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w_prev[k] = w_cur[k];
                w_cur[k] = walk.id[k] != kNoEntry ? a.wsrc[walk.id[k]] : 0.0f;
            }
        }
    };
    weights();

    // eight columns from `col` on, moved back to end with the row where rows don't hold whole vectors (see own_columns)
    const int col0 = (int)slab * (8 * P) + li * 8, F = (int)a.F;
    const bool act = col0 < F;
    const int col = a.own_rows ? col0 : min(col0, F - 8), skip = col0 - col, valid = min(8, F - col);
    const table_t table = buffer_table(a.Z, a.table_bytes);
    const uint32_t colbytes = act ? (uint32_t)col * 2 : kNoEntry;      // (columns past the row width fetch nothing)
    const float one = WEIGHTED ? 1.0f : register_one();
    // Running sums in levels (see BatchSums): 16 entries, 128 entries, and the 128s, which lie in LDS since most rows have none.
    // With weights, which take registers too, the second level lies there as well (otherwise a compute unit holds one workgroup
    // instead of two: bf16, 1,000,000 nodes of 8 entries, 64 columns 321 us and 261).
    float sum[8], tile[WEIGHTED ? 1 : 8];
    __shared__ float far[WEIGHTED ? 2 : 1][8][64 * NW];
    auto put = [&](int n) {                // the sum of the list's n-th 16 entries, others follow
        if constexpr (WEIGHTED) {
            if (n % 8 != 0) {
#pragma unroll
                for (int c = 0; c < 8; ++c) sum[c] += far[1][c][threadIdx.x];
            }
            if (n % 8 != 7) {
#pragma unroll
                for (int c = 0; c < 8; ++c) far[1][c][threadIdx.x] = sum[c];
                return;
            }
            if (n > 7) {
#pragma unroll
                for (int c = 0; c < 8; ++c) sum[c] += far[0][c][threadIdx.x];
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) far[0][c][threadIdx.x] = sum[c];
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) tile[c] += sum[c];
            if (n % 8 != 7) return;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                far[0][c][threadIdx.x] = n > 7 ? far[0][c][threadIdx.x] + tile[c] : tile[c];
                tile[c] = 0.0f;
            }
        }
    };
    if constexpr (!WEIGHTED) {
#pragma unroll
        for (int c = 0; c < 8; ++c) tile[c] = 0.0f;
    }
    u32x4 z[2][U];
    constexpr int kBatches = P / PER;                                   // of a tile
    // batch k of an even number and the next (which is never a tile's first): its place in the tile
    auto place = [](int k, auto odd) { return (k & ~1) % kBatches + (decltype(odd)::value ? 1 : 0); };
    constexpr std::false_type even;
    constexpr std::true_type odd;
    auto issue = [&](int k, u32x4 (&zz)[U], auto is_odd) {
        const int j = place(k, is_odd);
        if (j == 0 && k > 0) {
            walk.take();
            weights();
        }
#pragma unroll
        for (int t = 0; t < U; ++t) zz[t] = load_entry(table, walk.at(j * PER + t / 4, t % 4), colbytes);
    };
    auto consume = [&](int k, const u32x4 (&zz)[U], auto is_odd) {
        const int j = place(k, is_odd);
        // (the next tile's weights have taken the place of this one's when its last batch is added up)
        const bool old = (j + 1) % kBatches == 0 && k + 1 < batches;
#pragma unroll
        for (int t = 0; t < U; ++t) {
            float w = one;
            if constexpr (WEIGHTED)
                w = __int_as_float(__builtin_amdgcn_ds_bpermute(walk.gaddr + 4 * (j * PER + t / 4),
                                                                __float_as_int(old ? w_prev[t % 4] : w_cur[t % 4])));
            if (t == 0 && !decltype(is_odd)::value) first8<FMT, WEIGHTED>(zz[t], w, sum);
            else add8<FMT, WEIGHTED>(zz[t], w, sum);
        }
    };
    if (batches > 0) issue(0, z[0], even);
    for (int k = 0; k < batches; k += 2) {
        if (k + 1 < batches) issue(k + 1, z[1], odd);
        if (k > 0) put(k / 2 - 1);
        consume(k, z[0], even);
        if (k + 1 >= batches) break;
        if (k + 2 < batches) issue(k + 2, z[0], even);
        consume(k + 1, z[1], odd);
    }
    float acc[8];
    const int before = (batches + 1) / 2 - 1;                           // sums that were put away
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        acc[c] = batches > 0 ? sum[c] : 0.0f;
        if constexpr (!WEIGHTED) acc[c] += tile[c];
    }
    if (WEIGHTED && before > 0 && before % 8 != 0) {
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += far[1][c][threadIdx.x];
    }
    if (before >= 8) {
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += far[0][c][threadIdx.x];
    }

    if (heavy) {
#pragma unroll
        for (int b = P; b < 64; b <<= 1)
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] += __shfl_xor(acc[k], b, 64);
        __shared__ float red[NW][8][P];
        if (g == 0) {
#pragma unroll
            for (int k = 0; k < 8; ++k) red[wave][k][li] = acc[k];
        }
        __syncthreads();
        if (wave != 0 || g != 0) return;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            acc[k] = red[0][k][li];
#pragma unroll
            for (int w = 1; w < NW; ++w) acc[k] += red[w][k][li];
        }
    }
    if (!have || !act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    const float dinv = WEIGHTED ? a.dinv[v] : 1.0f;
    float r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        float x = acc[k];
        if constexpr (WEIGHTED) x = x * dinv;
        else if (a.scale == 1) x = d > 0 ? x / (float)d : 0.0f;
        r[k] = x;
    }
    auto store = [&](float* p, const float (&x)[8], bool vec_ok, bool half_ok) {
        if (skip == 0) {
            store_floats<8>(p, x, valid, vec_ok, half_ok);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k >= skip) p[k] = x[k];
        }
    };
    store(orow + a.ocol + col, r, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self) {
        float zs[8];
        decode8<FMT>(load_entry(table, (uint32_t)v * rowbytes, colbytes), zs);
        store(orow + col, zs, a.self_vec != 0, false);
    }
}

// ---------------------------------------------------------------------------
// The same slabs for long rows: a workgroup of eight waves per (row, slab).  A wave reads 64
// consecutive entries of the row at a time; each of its eight 8-lane groups gathers the eight entries
// its own lanes hold.  Partial sums are combined across the groups of a wave by shuffles and across
// waves through LDS, in a fixed order.
// ---------------------------------------------------------------------------
template <int FMT, bool WEIGHTED>
__global__ __launch_bounds__(64 * kHeavyWaves) void stored_grouped_kernel(StoredArgs a)
{
    constexpr int LPG = 8, U = 8;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t item = blockIdx.x;                        // slab-major
    const int slab = (int)(item / a.row_count);
    const int64_t slot = item % a.row_count;
    const int v = a.order[a.row_begin + slot];
    int lo, hi;
    if (a.part_ptr) {
        lo = a.part_ptr[(int64_t)a.part_lo * a.n_rows + a.row_begin + slot];
        hi = a.part_ptr[(int64_t)a.part_hi * a.n_rows + a.row_begin + slot];
    } else {
        lo = (int)a.row_ptr[v];
        hi = (int)a.row_ptr[v + 1];
    }
    const int li = lane % LPG;
    const int64_t col = (int64_t)slab * 64 + li * 8;
    const bool act = col < a.F;
    const int valid = (int)min((int64_t)8, a.F - col);
    const table_t table = buffer_table(a.Z, a.table_bytes);
    const uint32_t colbytes = act ? (uint32_t)(col * 2) : kNoEntry;
    const uint32_t rowbytes = (uint32_t)(a.ldz * 2);
    const int gaddr = (lane - li) * 4;

    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
    // the ids (and weights) of a wave's next tile are requested before the current tile's rows
    const float one = WEIGHTED ? 1.0f : register_one();
    int nxt_u = 0;
    float nxt_w = 0.0f;
    auto fetch_id = [&](int e) {
        nxt_u = e < hi ? a.col_idx[e] : -1;
        if constexpr (WEIGHTED) nxt_w = e < hi ? a.wsrc[nxt_u] : 0.0f;
    };
    fetch_id(lo + 64 * wave + lane);
    for (int base = lo + 64 * wave; base < hi; base += 64 * kHeavyWaves) {
        const uint32_t my_off = nxt_u >= 0 ? (uint32_t)nxt_u * rowbytes : kNoEntry;
        const float my_w = nxt_w;
        fetch_id(base + 64 * kHeavyWaves + lane);
        u32x4 raw[U];
        float w[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            raw[t] = load_entry(table, (uint32_t)__builtin_amdgcn_ds_bpermute(gaddr + 4 * t, (int)my_off), colbytes);
            if constexpr (WEIGHTED) w[t] = __int_as_float(__builtin_amdgcn_ds_bpermute(gaddr + 4 * t, __float_as_int(my_w)));
            else w[t] = one;
        }
#pragma unroll
        for (int t = 0; t < U; ++t) add8<FMT, WEIGHTED>(raw[t], w[t], acc);
    }
    // the eight groups of a wave, then the eight waves
#pragma unroll
    for (int m = LPG; m < 64; m <<= 1)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += __shfl_xor(acc[k], m, 64);
    __shared__ float red[kHeavyWaves][LPG][8];
    if (lane < LPG) {
#pragma unroll
        for (int k = 0; k < 8; ++k) red[wave][lane][k] = acc[k];
    }
    __syncthreads();
    if (wave != 0 || lane >= LPG || !act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    float r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        float x = red[0][lane][k];
#pragma unroll
        for (int w = 1; w < kHeavyWaves; ++w) x += red[w][lane][k];
        if (!a.first && k < valid) x += orow[a.ocol + col + k];
        if (a.last) {
            const int d = (a.last && a.scale == 1) ? a.deg[v] : 0;      // only the mean's last range needs it
            if (a.scale == 1) x = d > 0 ? x / (float)d : 0.0f;
            else if (a.scale == 2) x = x * a.dinv[v];
        }
        r[k] = x;
    }
    store_floats<8>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self && a.first) {
        float zs[8];
        load_stored<FMT, 8>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_floats<8>(orow + col, zs, valid, a.self_vec != 0);
    }
}

// ---------------------------------------------------------------------------
// attention scores from a stored table (one wave per node)
// ---------------------------------------------------------------------------
template <int FMT, int HP>
__global__ __launch_bounds__(256) void stored_scores_kernel(
    int64_t N, int64_t F, int Dh, const uint16_t* __restrict__ Z, int64_t ldz,
    const float* __restrict__ a_src, const float* __restrict__ a_dst, float* __restrict__ el, float* __restrict__ er)
{
    const int lane = threadIdx.x & 63;
    const int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= N) return;
    float ps[HP], pd[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) { ps[h] = 0.0f; pd[h] = 0.0f; }
    for (int64_t c = lane; c < F; c += 64) {
        const float z = decode1<FMT>(Z[v * ldz + c]);
        const int h = (int)(c / Dh);
        const float s = z * a_src[c], t = z * a_dst[c];
#pragma unroll
        for (int i = 0; i < HP; ++i) {
            ps[i] += (h == i) ? s : 0.0f;
            pd[i] += (h == i) ? t : 0.0f;
        }
    }
#pragma unroll
    for (int h = 0; h < HP; ++h) {
        const float s = wave_sum(ps[h]), t = wave_sum(pd[h]);
        if (lane == 0) { el[v * HP + h] = s; er[v * HP + h] = t; }
    }
}

// The same scores with 8-byte loads: 16 lanes per node (four nodes per wave), each lane walks the row in steps
// of 64 columns, four stored elements at a time, all pieces of a row of up to 256 columns requested before the
// first is used; the per-head partial sums are reduced over the 16 lanes of a node.
// Needs 8-byte aligned rows, 16-byte aligned attention vectors and F % 4 == 0.
template <int FMT, int HP>
__global__ __launch_bounds__(256) void stored_scores_vec_kernel(
    int64_t N, int64_t F, int Dh, const uint16_t* __restrict__ Z, int64_t ldz,
    const float* __restrict__ a_src, const float* __restrict__ a_dst, float* __restrict__ el, float* __restrict__ er)
{
    const int li = threadIdx.x & 15;
    const int64_t v = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const bool have = v < N;
    const int64_t vv = have ? v : N - 1;                 // idle groups repeat the last node (nothing stored)
    const bool whole = Dh % 4 == 0;
    float ps[HP], pd[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) { ps[h] = 0.0f; pd[h] = 0.0f; }
    for (int64_t c0 = li * 4; c0 < F; c0 += 256) {
        float zq[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = c0 + 64 * q;
            if (c < F) load_stored<FMT, 4>(Z + vv * ldz + c, zq[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = c0 + 64 * q;
            if (c >= F) break;
            const f32x4 as = *reinterpret_cast<const f32x4*>(a_src + c);
            const f32x4 ad = *reinterpret_cast<const f32x4*>(a_dst + c);
            const float sa[4] = {as.x, as.y, as.z, as.w}, da[4] = {ad.x, ad.y, ad.z, ad.w};
            if (whole) {
                const int h = (int)c / Dh;
                const float s = ((zq[q][0] * sa[0] + zq[q][1] * sa[1]) + zq[q][2] * sa[2]) + zq[q][3] * sa[3];
                const float t = ((zq[q][0] * da[0] + zq[q][1] * da[1]) + zq[q][2] * da[2]) + zq[q][3] * da[3];
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
                const float s = zq[q][k] * sa[k], t = zq[q][k] * da[k];
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
        for (int h = 0; h < HP; ++h) { el[v * HP + h] = ps[h]; er[v * HP + h] = pd[h]; }
    }
}

// ---------------------------------------------------------------------------
// edge softmax over a stored table: whole rows per wave, online softmax at tile granularity, per-edge
// weights through wave-private LDS, next batch of rows requested before the current one is consumed.
//   HU: every lane's E columns lie inside one head (Dh % E == 0)
// ---------------------------------------------------------------------------
template <int FMT, int E, int NC, int NW, int HP, bool HU>
__global__ __launch_bounds__(64 * (NW == 1 ? kLightWaves : NW)) void stored_gat_kernel(StoredArgs a)
{
    constexpr int WAVES = NW == 1 ? kLightWaves : NW;
    constexpr int U = E * NC >= 16 ? 2 : 4;
    constexpr int Q = HU ? 1 : E;
    __shared__ float wl[WAVES][HP][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t items = a.row_count * a.nslab;
    const int64_t item = (NW == 1) ? (int64_t)blockIdx.x * kLightWaves + wave : (int64_t)blockIdx.x;
    if (item >= items) return;
    const int64_t slot = item / a.nslab;
    const int slab = (int)(item % a.nslab);
    const int v = __builtin_amdgcn_readfirstlane(a.order[a.row_begin + slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);

    const int64_t col0 = (int64_t)slab * (64 * E * NC) + lane * E;
    bool act[NC];
    int64_t colsafe[NC];
    int hc[NC][Q];
    float acc[NC][E];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t col = col0 + c * 64 * E;
        act[c] = col < a.F;
        colsafe[c] = act[c] ? col : 0;
#pragma unroll
        for (int k = 0; k < Q; ++k) hc[c][k] = min((int)((col + k) / a.Dh), a.heads - 1);
#pragma unroll
        for (int k = 0; k < E; ++k) acc[c][k] = 0.0f;
    }
    float* myw = &wl[wave][0][0];

    float m[HP], s[HP], erv[HP];
#pragma unroll
    for (int h = 0; h < HP; ++h) {
        m[h] = -INFINITY;
        s[h] = 0.0f;
        erv[h] = a.er[(int64_t)v * HP + h];
    }

    const int first = lo + 64 * (NW == 1 ? 0 : wave);
    for (int base = first; base < hi; base += 64 * NW) {
        const int e = base + lane;
        const bool valid = e < hi;
        const int cnt = min(64, hi - base);
        int my_u = valid ? a.col_idx[e] : 0;
        my_u = valid ? my_u : bcast_i(my_u, 0);

        float zq[U][NC][E];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const uint16_t* zr = a.Z + (int64_t)bcast_i(my_u, t) * a.ldz;
#pragma unroll
            for (int c = 0; c < NC; ++c) load_stored<FMT, E>(zr + colsafe[c], zq[t][c]);
        }
        float elu[HP], scale[HP];
        if constexpr (HP == 4) {
            const f32x4 t = *reinterpret_cast<const f32x4*>(a.el + (int64_t)my_u * 4);
            elu[0] = t.x; elu[1] = t.y; elu[2] = t.z; elu[3] = t.w;
        } else {
#pragma unroll
            for (int h = 0; h < HP; ++h) elu[h] = a.el[(int64_t)my_u * HP + h];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // earlier reads of wl are done
#pragma unroll
        for (int h = 0; h < HP; ++h) {
            const float x = elu[h] + erv[h];
            const float sc = valid ? (x > 0.0f ? x : a.slope * x) : -INFINITY;
            const float mn = fmaxf(m[h], wave_max(sc));
            scale[h] = expf(m[h] - mn);
            const float pe = valid ? expf(sc - mn) : 0.0f;
            s[h] = s[h] * scale[h] + wave_sum(pe);
            m[h] = mn;
            myw[h * 64 + lane] = pe;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (base != first) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int k = 0; k < E; ++k) acc[c][k] *= select_head<HP>(scale, hc[c][HU ? 0 : k]);
        }

        for (int j = 0; j < cnt; j += U) {
            float zn[U][NC][E];
            const bool more = j + U < cnt;
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint16_t* zr = a.Z + (int64_t)bcast_i(my_u, (j + U + t) & 63) * a.ldz;
#pragma unroll
                    for (int c = 0; c < NC; ++c) load_stored<FMT, E>(zr + colsafe[c], zn[t][c]);
                }
            }
#pragma unroll
            for (int t = 0; t < U; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if constexpr (HU) {
                        const float w = myw[hc[c][0] * 64 + j + t];
#pragma unroll
                        for (int k = 0; k < E; ++k) acc[c][k] = fmaf(w, zq[t][c][k], acc[c][k]);
                    } else {
#pragma unroll
                        for (int k = 0; k < E; ++k) acc[c][k] = fmaf(myw[hc[c][k] * 64 + j + t], zq[t][c][k], acc[c][k]);
                    }
                }
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int k = 0; k < E; ++k) zq[t][c][k] = zn[t][c][k];
            }
        }
    }

    if constexpr (NW > 1) {
        __shared__ float red[NW][NC * E][64];
        __shared__ float mred[NW][HP], sred[NW][HP];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) red[wave][c * E + k][lane] = acc[c][k];
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
                f[w][h] = (mred[w][h] == -INFINITY) ? 0.0f : expf(mred[w][h] - mm);
                ss += sred[w][h] * f[w][h];
            }
            s[h] = ss;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < E; ++k) {
                float t = 0.0f;
#pragma unroll
                for (int w = 0; w < NW; ++w) t += red[w][c * E + k][lane] * select_head<HP>(f[w], hc[c][HU ? 0 : k]);
                acc[c][k] = t;
            }
    }

    float* orow = a.out + (int64_t)v * a.ldo;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (!act[c]) continue;
        const int64_t col = col0 + c * 64 * E;
        const int valid = (int)min((int64_t)E, a.F - col);
        float r[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const float den = select_head<HP>(s, hc[c][HU ? 0 : k]);
            r[k] = den > 0.0f ? acc[c][k] / den : 0.0f;
        }
        store_floats<E>(orow + a.ocol + col, r, valid, a.out_vec != 0, a.out_half != 0);
        if (a.copy_self) {
            float zs[E];
            load_stored<FMT, E>(a.Z + (int64_t)v * a.ldz + col, zs);
            store_floats<E>(orow + col, zs, valid, a.self_vec != 0);
        }
    }
}

// ---------------------------------------------------------------------------
// gat_softmax over a stored table for rows of ordinary length when the row fits one wave at four
// elements per lane (F <= 256) and a head is a power-of-two group of lanes: the source score of an
// entry is computed from the gathered (decoded) row itself instead of being read from the score
// table, which costs a cache line per entry — a fifth of the traffic when a row is only 512 bytes.
// Same scheme as the fp32 kernel of that name: per-lane dot product with a_src, sum over the head's
// lanes, online softmax over batches of four entries, scores in units of log2(e).
// ---------------------------------------------------------------------------
template <int FMT, int G>
__global__ __launch_bounds__(64 * kLightWaves) void stored_gat_flash_kernel(StoredArgs a, const float* __restrict__ attn_src,
                                                                            int er_stride)
{
    constexpr int U = 4, E = 4;
    constexpr float kLog2e = 1.4426950408889634f;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t slot = (int64_t)blockIdx.x * kLightWaves + wave;
    if (slot >= a.row_count) return;
    const int v = __builtin_amdgcn_readfirstlane(a.order[a.row_begin + slot]);
    const int lo = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v]);
    const int hi = __builtin_amdgcn_readfirstlane((int)a.row_ptr[v + 1]);

    const int64_t col = lane * E;
    const bool act = col < a.F;
    const int64_t colsafe = act ? col : 0;            // idle lanes read the row start (weight vector zero, never stored)
    const int h = min((int)(col / a.Dh), a.heads - 1);
    float as[E] = {0.0f, 0.0f, 0.0f, 0.0f};
    float erv = 0.0f;
    if (act) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(attn_src + col);
        as[0] = t.x * kLog2e; as[1] = t.y * kLog2e; as[2] = t.z * kLog2e; as[3] = t.w * kLog2e;
        erv = a.er[(int64_t)v * er_stride + h] * kLog2e;
    }

    float m = -INFINITY, s = 0.0f;
    float acc[E] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int base = lo; base < hi; base += 64) {
        const int e = base + lane;
        const bool valid = e < hi;
        const int cnt = min(64, hi - base);
        int my_u = valid ? a.col_idx[e] : 0;
        my_u = valid ? my_u : bcast_i(my_u, 0);

        float zq[U][E];
#pragma unroll
        for (int t = 0; t < U; ++t) load_stored<FMT, E>(a.Z + (int64_t)bcast_i(my_u, t) * a.ldz + colsafe, zq[t]);

        for (int j = 0; j < cnt; j += U) {
            float zn[U][E];
            const bool more = j + U < cnt;
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t)
                    load_stored<FMT, E>(a.Z + (int64_t)bcast_i(my_u, (j + U + t) & 63) * a.ldz + colsafe, zn[t]);
            }
            float sc[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                float d = as[0] * zq[t][0];
                d = fmaf(as[1], zq[t][1], d);
                d = fmaf(as[2], zq[t][2], d);
                d = fmaf(as[3], zq[t][3], d);
                const float x = group_sum<G>(d) + erv;
                sc[t] = (j + t < cnt) ? (x > 0.0f ? x : a.slope * x) : -INFINITY;
            }
            float mn = m;
#pragma unroll
            for (int t = 0; t < U; ++t) mn = fmaxf(mn, sc[t]);      // finite: entry j of the tile is real
            const float scale = __builtin_amdgcn_exp2f(m - mn);
            float pw[U], ps = 0.0f;
#pragma unroll
            for (int t = 0; t < U; ++t) { pw[t] = __builtin_amdgcn_exp2f(sc[t] - mn); ps += pw[t]; }
            s = s * scale + ps;
#pragma unroll
            for (int k = 0; k < E; ++k) acc[k] *= scale;
#pragma unroll
            for (int t = 0; t < U; ++t)
#pragma unroll
                for (int k = 0; k < E; ++k) acc[k] = fmaf(pw[t], zq[t][k], acc[k]);
            m = mn;
            if (more) {
#pragma unroll
                for (int t = 0; t < U; ++t)
#pragma unroll
                    for (int k = 0; k < E; ++k) zq[t][k] = zn[t][k];
            }
        }
    }

    if (!act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    float r[E];
#pragma unroll
    for (int k = 0; k < E; ++k) r[k] = s > 0.0f ? acc[k] / s : 0.0f;
    store_floats<E>(orow + a.ocol + col, r, E, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self) {
        float zs[E];
        load_stored<FMT, E>(a.Z + (int64_t)v * a.ldz + col, zs);
        store_floats<E>(orow + col, zs, E, a.self_vec != 0);
    }
}

// ---------------------------------------------------------------------------
// The same for several rows per wave: P lanes of four elements hold a row, and the R = 64 / P groups of a wave walk R rows of the
// schedule, or shares of one long row, in lock step (EntryWalk); a group whose row has ended weighs its batches' entries with
// zero.  Destination scores come from a row's own elements, so nothing is launched before it, and long rows, one per workgroup
// with their shares merged over the groups and then over the waves in order, run beside the others.
// bf16 in us, scores, long rows and a wave per row before, and now: 32 columns 2,145,631 nodes of 7 entries 1,946 and 537,
// 15,346 of 12 84 and 15; 64 columns 2,222,171 of 51 7,527 and 2,379 (6.2 TB/s of lines), 164,453 of 436 4,188 and 987; 128
// columns 475,093 of 56 1,894 and 939; 256 columns, where a wave is a row either way, 29,969 of 22, longest 2,604, 186 and 90,
// 1,911,625 of 60 9,910 and 8,877.  1,685 drawn calls: 0.47 of the time.
// ---------------------------------------------------------------------------
template <int FMT, int G, int P>
__global__ __launch_bounds__(64 * kHeavyWaves) void stored_gat_rows_kernel(StoredArgs a, const float* __restrict__ attn_src,
                                                                           const float* __restrict__ attn_dst)
{
    constexpr int U = 4, R = 64 / P, NW = kHeavyWaves;
    constexpr float kLog2e = 1.4426950408889634f;
    const int lane = threadIdx.x & 63, li = lane % P, g = lane / P;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool heavy = blockIdx.x < a.heavy_rows;     // uniform over the workgroup
    const int64_t first = heavy ? (int64_t)blockIdx.x : a.heavy_rows + ((int64_t)(blockIdx.x - (uint32_t)a.heavy_rows) * NW + wave) * R;
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
    const uint32_t rowbytes = (uint32_t)(a.ldz * 2);
    const int batches = heavy ? walk.start(a.col_idx, lo + kTile * (wave * R + g), hi, kTile * NW * R, rowbytes)
                              : walk.start(a.col_idx, lo, hi, kTile, rowbytes);

    const int col = li * 4;
    const bool act = col < a.F;
    const table_t table = buffer_table(a.Z, a.table_bytes);
    const uint32_t colbytes = act ? (uint32_t)col * 2 : kNoEntry;      // (columns past the row width fetch nothing)
    auto load = [&](uint32_t row) {
        return __builtin_amdgcn_raw_buffer_load_b64(table, __builtin_elementwise_add_sat(row, colbytes), 0, 0);
    };
    auto decode = [&](const u32x2& raw, float (&z)[4]) {
        if constexpr (FMT == FMT_BF16) {
            z[0] = __uint_as_float(raw.x << 16); z[1] = __uint_as_float(raw.x & 0xffff0000u);
            z[2] = __uint_as_float(raw.y << 16); z[3] = __uint_as_float(raw.y & 0xffff0000u);
        } else {
            z[0] = decode1<FMT>((uint16_t)raw.x); z[1] = decode1<FMT>((uint16_t)(raw.x >> 16));
            z[2] = decode1<FMT>((uint16_t)raw.y); z[3] = decode1<FMT>((uint16_t)(raw.y >> 16));
        }
    };
    auto dot = [](const f32x4& w, const float (&z)[4]) {
        float d = w.x * z[0];
        d = fmaf(w.y, z[1], d);
        d = fmaf(w.z, z[2], d);
        return fmaf(w.w, z[3], d);
    };
    // exponents are kept in units of log2(e): exp(x) = exp2(x * log2(e)), and the leaky step commutes with the factor
    f32x4 as = {0.0f, 0.0f, 0.0f, 0.0f}, ad = as;
    if (act) {
        as = *reinterpret_cast<const f32x4*>(attn_src + col) * kLog2e;        // [heads, Dh] is F contiguous floats
        ad = *reinterpret_cast<const f32x4*>(attn_dst + col) * kLog2e;
    }
    float own[4];
    const u32x2 own_raw = load(have ? (uint32_t)v * rowbytes : kNoEntry);
    decode(own_raw, own);
    const float erv = group_sum<G>(dot(ad, own));

    const bool empty = (heavy ? lo + kTile * (wave * R + g) : lo) >= hi;      // no entry: its maximum stays -infinity
    float m = -INFINITY, s = 0.0f;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    u32x2 z[2][U];
    uint32_t on[2][U];
    auto consume = [&](const u32x2 (&zz)[U], const uint32_t (&oo)[U]) {
        float zq[U][4], sc[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            decode(zz[t], zq[t]);
            const float x = group_sum<G>(dot(as, zq[t])) + erv;
            sc[t] = oo[t] != kNoEntry ? (x > 0.0f ? x : a.slope * x) : -INFINITY;
        }
        float mn = m;
#pragma unroll
        for (int t = 0; t < U; ++t) mn = fmaxf(mn, sc[t]);
        const float mr = empty ? 0.0f : mn;
        const float scale = __builtin_amdgcn_exp2f(m - mr);
        float pw[U], ps = 0.0f;
#pragma unroll
        for (int t = 0; t < U; ++t) { pw[t] = __builtin_amdgcn_exp2f(sc[t] - mr); ps += pw[t]; }
        s = s * scale + ps;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] *= scale;
#pragma unroll
        for (int t = 0; t < U; ++t)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = fmaf(pw[t], zq[t][k], acc[k]);
        m = mn;
    };
    // the gathers of a batch are issued before the batch before it is added up
    auto step = [&](int k, u32x2 (&zn)[U], uint32_t (&no)[U]) {       // batch k
        if (k % P == 0 && k > 0) walk.take();
#pragma unroll
        for (int t = 0; t < U; ++t) {
            no[t] = walk.at(k % P, t);
            zn[t] = load(no[t]);
        }
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
        auto weight = [](float mw, float mm) { return mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mw - mm); };
#pragma unroll
        for (int b = P; b < 64; b <<= 1) {
            const float mo = __shfl_xor(m, b, 64), mm = fmaxf(m, mo), fa = weight(m, mm), fb = weight(mo, mm);
            auto join = [&](float x) { return x * fa + __shfl_xor(x, b, 64) * fb; };
            s = join(s);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = join(acc[k]);
            m = mm;
        }
        __shared__ float red[NW][6][P];
        if (g == 0) {
            red[wave][0][li] = m;
            red[wave][1][li] = s;
#pragma unroll
            for (int k = 0; k < 4; ++k) red[wave][2 + k][li] = acc[k];
        }
        __syncthreads();
        if (wave != 0 || g != 0) return;
        float mm = red[0][0][li];
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, red[w][0][li]);
        s = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = weight(red[w][0][li], mm);
            s = fmaf(red[w][1][li], f, s);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = fmaf(red[w][2 + k][li], f, acc[k]);
        }
    }
    if (!have || !act) return;
    float* orow = a.out + (int64_t)v * a.ldo;
    float r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = s > 0.0f ? acc[k] / s : 0.0f;
    store_floats<4>(orow + a.ocol + col, r, 4, a.out_vec != 0, a.out_half != 0);
    if (a.copy_self) store_floats<4>(orow + col, own, 4, a.self_vec != 0);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <typename K, typename KH>
void launch_pair(K light, KH heavy, const StoredArgs& base, int64_t n_heavy, int64_t N, hipStream_t stream)
{
    if (n_heavy > 0) {
        StoredArgs a = base;
        a.row_begin = 0;
        a.row_count = n_heavy;
        heavy<<<dim3((unsigned)(n_heavy * a.nslab)), dim3(64 * kHeavyWaves), 0, stream>>>(a);
    }
    if (N > n_heavy) {
        StoredArgs a = base;
        a.row_begin = n_heavy;
        a.row_count = N - n_heavy;
        const int64_t blocks = (a.row_count * a.nslab + kLightWaves - 1) / kLightWaves;
        light<<<dim3((unsigned)blocks), dim3(64 * kLightWaves), 0, stream>>>(a);
    }
}

template <int FMT, int E, bool MAXOP>
void dispatch_linear(int nc, const StoredArgs& a, int64_t nh, int64_t N, hipStream_t s)
{
    if (nc == 1) launch_pair(stored_linear_kernel<FMT, E, 1, 1, MAXOP>, stored_linear_kernel<FMT, E, 1, kHeavyWaves, MAXOP>, a, nh, N, s);
    else launch_pair(stored_linear_kernel<FMT, E, 2, 1, MAXOP>, stored_linear_kernel<FMT, E, 2, kHeavyWaves, MAXOP>, a, nh, N, s);
}

template <int FMT, int P>
void launch_rows(const StoredArgs& base, const retexo_plan* p, hipStream_t stream)
{
    StoredArgs a = base;
    const int64_t rows = kHeavyWaves * (64 / P), N = p->N, n_heavy = long_rows(p, a.F, false);
    a.heavy_rows = n_heavy;
    a.nslab = (int)((a.F + 8 * P - 1) / (8 * P));
    a.slab_blocks = (uint32_t)(n_heavy + (N - n_heavy + rows - 1) / rows);
    const dim3 grid(a.slab_blocks * (unsigned)a.nslab), block(64 * kHeavyWaves);
    if (a.wsrc) stored_rows_kernel<FMT, P, true><<<grid, block, 0, stream>>>(a);
    else        stored_rows_kernel<FMT, P, false><<<grid, block, 0, stream>>>(a);
}

template <int FMT, int G, int P>
void launch_gat_rows(const StoredArgs& base, const retexo_plan* p, const float* attn_src, const float* attn_dst, hipStream_t stream)
{
    if constexpr (G <= P && G * kMaxHeads > P / 2) {
        StoredArgs a = base;
        const int64_t rows = kHeavyWaves * (64 / P), N = p->N, n_heavy = long_rows(p, a.F, false, true);
        a.heavy_rows = n_heavy;
        const unsigned blocks = (unsigned)(n_heavy + (N - n_heavy + rows - 1) / rows);
        stored_gat_rows_kernel<FMT, G, P><<<dim3(blocks), dim3(64 * kHeavyWaves), 0, stream>>>(a, attn_src, attn_dst);
    }
}
template <int FMT, int G>
void dispatch_gat_rows(const StoredArgs& a, const retexo_plan* p, const float* as, const float* ad, hipStream_t stream)
{
    switch (row_lanes(a.F)) {
        case 8:  launch_gat_rows<FMT, G, 8>(a, p, as, ad, stream); break;
        case 16: launch_gat_rows<FMT, G, 16>(a, p, as, ad, stream); break;
        case 32: launch_gat_rows<FMT, G, 32>(a, p, as, ad, stream); break;
        default: launch_gat_rows<FMT, G, 64>(a, p, as, ad, stream); break;
    }
}

template <int FMT, int E, int HP, bool HU>
void dispatch_gat(int nc, const StoredArgs& a, int64_t nh, int64_t N, hipStream_t s)
{
    if (nc == 1) launch_pair(stored_gat_kernel<FMT, E, 1, 1, HP, HU>, stored_gat_kernel<FMT, E, 1, kHeavyWaves, HP, HU>, a, nh, N, s);
    else launch_pair(stored_gat_kernel<FMT, E, 2, 1, HP, HU>, stored_gat_kernel<FMT, E, 2, kHeavyWaves, HP, HU>, a, nh, N, s);
}

bool aligned_rows(const void* p, int64_t ld_elems, int bytes_per_elem)
{
    return ((uintptr_t)p % 16) == 0 && (ld_elems * bytes_per_elem) % 16 == 0;
}

// Lanes of eight elements that hold a row, or a slab, of a sum, mean or gcn_sym in row groups; 0: the range walk (`ranges`, over
// `parts` ranges) or whole rows.  bf16 mean in us, row groups against the others, over 29 graphs of 3,000 to 2,400,000 nodes:
//  Rows that 16-byte loads can't take whole (an element per lane in whole rows): always, 1,000,000 nodes of 20 entries, 30
//  columns 521 and 639, 232,965 of 490 1,075 and 2,430; 60,000 of 250, 130 columns 381 and 767, 250 columns 838 and 1,039.
//  Others of up to 128 columns instead of whole rows: 1,000,000 of 20, 32 columns 395 and 745, 64 columns 432 and 790, 128
//  columns 778 and 960; 100,000 of 8 15 and 48, 22 and 49, 40 and 51; 30,000 of 300, 64 columns 55 and 255.  Wider ones where a few
//  long rows, which are walked here beside the others, outlast the rest (19,677 of 30, longest 1,743, 512 columns 87 and 310;
//  172,021 of 10, 608 columns 492 and 1,166), not where all are alike (1,000,000 of 8, 256 columns 947 and 912; 78,691 of 6, longest
//  18, 288 columns 83 and 57; 66,237 of 7, longest 94, 342 columns with weights 86 and 67): from a longest row of 48 entries and of
//  1/300 of the nodes on, 1/100 where the last slab is less than three quarters of the columns; up to 250,000 nodes.  Of 16,248 drawn calls
//  over 16-bit tables 806 were more than 4 % slower than in whole rows when all of up to 250,000 nodes came here, 83 are.
//  With weights, which wait for ids, from 8,192 nodes on, or a longest row of 48 (of up to 64 columns) or a mean of 100 (above): 2,340
//  of 14, longest 28, 32 columns 5.9 and 4.8; 3,000 of 60, 128 columns 10.4 and 9.9.  Fewer nodes whose rows are alike, on which
//  the chip waits for one row as for another, in whole rows: with weights up to 3,500 and a longest row of three times the mean
//  (430 of 36, longest 52, 2 columns 7.6 and 6.0; 1,986 of 81, longest 115, 32 columns 13.0 and 11.2; the other way 4,308 of 89,
//  longest 121, 14.0 and 16.6; 1,799 of 109, longest 339, 22.2 and 27.7), without up to 4,500 and a longest row of 44 entries
//  (1,299 of 7, 64 columns 4.2 and 3.7; 4,187 of 5 4.4 and 4.0; the other way 5,056 of 8 4.2 and 4.6, 2,261 of 34, longest 54, 6.5 and 7.0).
//  Instead of the range walk where a row's share of a range is short: 600,000 of 120 (7 per range) 1,127 and 1,448, 1,003,546
//  of 80 (5), 64 columns 1,483 and 3,670, 576,484 of 113 (7), 96 columns 2,069 and 3,946; the other way 400,000 of 150 (19) 800
//  and 678, 150,000 of 200 (50), 64 columns 355 and 251, with weights 386,048 of 112 (14) 1,012 and 832.  Not in one range, which
//  takes the longest rows apart: 59,657 of 263, longest 5,419, 265 and 110; but 1,330,759 of 85, 104 columns 5,328 and 5,836.
int rows_lanes(const StoredCall& c, bool wide, bool ranges, int parts)
{
    const retexo_plan* p = c.plan;
    const AggOptions& opt = agg_options();
    const int64_t N = p->N, nnz = p->nnz, F = c.F;
    const bool weighted = c.mode == RETEXO_GCN_SYM;
    if (opt.slab_cols != 0 || opt.max_vec < 4 || (p->part_ptr && opt.parts >= 0)) return 0;      // (the caller said how)
    const int lanes = F <= 32 ? 4 : F <= 64 ? 8 : F <= 128 ? 16 : 32;
    if (weighted && N < 8192 && (F > 64 ? nnz < 100 * N : p->max_degree < 48)) return 0;
    if (!wide) {
        // eight elements at 4-byte addresses, none past a row's end: what lies there may not be the caller's
        return (uintptr_t)c.Z % 4 == 0 && c.ldz % 2 == 0 && F >= 8 && F % 2 == 0 ? lanes : 0;
    }
    if (!ranges && F <= 128 && (weighted ? N < 3500 && F <= 64 && p->max_degree * N < 3 * nnz : N < 4500 && p->max_degree < 44)) return 0;
    if (!ranges) {
        const bool filled = 4 * F >= 3 * align_up(F, 256);
        return F <= 128 || (N < 250000 && p->max_degree >= 48 && (filled ? 300 : 100) * (int64_t)p->max_degree >= N) ? lanes : 0;
    }
    if (F > 128) return 0;
    if (parts > 1) return nnz < N * parts * (weighted ? 12 : F > 32 ? 14 : 10) ? lanes : 0;
    return F > 64 && N >= 600000 ? lanes : 0;
}

template <int FMT>
int launch_stored(const StoredCall& c, hipStream_t stream)
{
    const retexo_plan* p = c.plan;
    const int64_t N = p->N, F = c.F;
    const AggOptions& opt = agg_options();
    const bool gat = c.mode == RETEXO_GAT_SOFTMAX;
    const uint16_t* Z = (const uint16_t*)c.Z;

    // 16-byte loads of eight elements need aligned rows padded to whole vectors; rows of at most 256
    // columns use 8-byte loads of four elements so that all 64 lanes of a wave carry a share of the row
    const bool wide = aligned_rows(Z, c.ldz, 2) && align_up(F, 8) <= c.ldz && opt.max_vec >= 4;
    const int E = wide ? (F <= 256 ? 4 : 8) : 1;

    StoredArgs a;
    a.row_ptr = p->row_ptr;
    a.col_idx = p->col_idx;
    a.order = p->order;
    a.deg = p->deg;
    a.set_deg = p->degrees_set && c.mode == RETEXO_MEAN ? p->deg : nullptr;
    a.dinv = p->dinv;
    a.wsrc = c.mode == RETEXO_GCN_SYM ? p->dinv : nullptr;
    a.Z = Z;
    a.ldz = c.ldz;
    a.out = c.out;
    a.ldo = c.ldo;
    a.ocol = c.self_concat ? F : 0;
    a.el = nullptr;
    a.er = nullptr;
    a.row_begin = 0;
    a.row_count = 0;
    a.F = F;
    a.scale = c.mode == RETEXO_MEAN ? 1 : c.mode == RETEXO_GCN_SYM ? 2 : 0;
    a.heads = c.heads;
    a.Dh = gat ? (int)(F / c.heads) : (int)F;
    a.slope = c.slope;
    a.copy_self = (c.self_concat && c.copy_self) ? 1 : 0;
    a.out_vec = aligned_rows(c.out + a.ocol, c.ldo, 4) ? 1 : 0;
    a.out_half = ((uintptr_t)(c.out + a.ocol) % 8 == 0 && c.ldo % 2 == 0) ? 1 : 0;
    a.self_vec = aligned_rows(c.out, c.ldo, 4) ? 1 : 0;
    a.part_ptr = nullptr;
    a.n_rows = N;
    a.part_lo = 0;
    a.part_hi = 0;
    a.first = 1;
    a.last = 1;
    a.table_bytes = 0;
    a.own_rows = wide;

    const int64_t n_heavy = long_rows(p, F, true);

    const int max_nc = 2;
    int nc = (int)((F + 64 * E - 1) / (64 * E));
    nc = nc < 1 ? 1 : nc > max_nc ? max_nc : nc;
    const int64_t slab_w = 64 * (int64_t)E * nc;
    a.nslab = (int)((F + slab_w - 1) / slab_w);

    // dense graphs whose table exceeds L2 although a 64-column slab of one source range fits: narrow slabs
    const bool off32 = (N * c.ldz + F) * 2 < (1ll << 32) && !opt.wide_offsets;
    const bool linear_sum = c.mode == RETEXO_SUM || c.mode == RETEXO_MEAN || c.mode == RETEXO_GCN_SYM;
    bool narrow = linear_sum && wide && off32 && (p->part_ptr || (p->nnz >= 32 * N && N * c.ldz * 2 > (4ll << 20)));
    if (opt.slab_cols > 64) narrow = false;
    if (opt.slab_cols == 64 && linear_sum && wide && off32) narrow = true;
    // workgroups of the range walk read their share of one source range after the other
    int parts = 1;
    if (narrow && p->part_ptr) {
        parts = (int)opt.parts;
        if (parts < 0) {
            parts = 1;
            while (parts < kMaxParts && N * 128 > (int64_t)parts * (8ll << 20)) parts *= 2;
        }
        if (parts != 2 && parts != 4 && parts != 8 && parts != 16) parts = 1;
    }
    if (const int lanes = linear_sum && off32 ? rows_lanes(c, wide, narrow, parts) : 0) {
        a.table_bytes = (uint32_t)(((N - 1) * c.ldz + (a.own_rows ? align_up(F, 8) : F)) * 2);
        if (lanes == 4)       launch_rows<FMT, 4>(a, p, stream);
        else if (lanes == 8)  launch_rows<FMT, 8>(a, p, stream);
        else if (lanes == 16) launch_rows<FMT, 16>(a, p, stream);
        else                  launch_rows<FMT, 32>(a, p, stream);
    } else if (narrow) {
        a.table_bytes = (uint32_t)(((N - 1) * c.ldz + align_up(F, 8)) * 2);
        a.nslab = (int)((F + 63) / 64);
        if (parts > 1) a.part_ptr = p->part_ptr;
        // rows whose share of one range is long get a workgroup each
        int64_t n_long = 0;
        for (int i = 0; i < kPlanThresholdCount; ++i)
            if (kPlanThresholds[i] >= opt.narrow_heavy * parts || kPlanThresholds[i] >= 16384) {
                n_long = p->rows_at_least[i];
                break;
            }
        const int64_t bundles = (N - n_long + 7) / 8;
        const int64_t blocks = (bundles * a.nslab + kLightWaves - 1) / kLightWaves;
        for (int k = 0; k < parts; ++k) {
            a.part_lo = k * (kMaxParts / parts);
            a.part_hi = (k + 1) * (kMaxParts / parts);
            a.first = k == 0;
            a.last = k == parts - 1;
            if (n_long > 0) {
                a.row_begin = 0;
                a.row_count = n_long;
                const dim3 grid((unsigned)(n_long * a.nslab));
                if (a.wsrc) stored_grouped_kernel<FMT, true><<<grid, dim3(64 * kHeavyWaves), 0, stream>>>(a);
                else stored_grouped_kernel<FMT, false><<<grid, dim3(64 * kHeavyWaves), 0, stream>>>(a);
            }
            if (N > n_long) {
                a.row_begin = n_long;
                a.row_count = N - n_long;
                const dim3 grid((unsigned)blocks), block(64 * kLightWaves);
                const bool eight = parts <= 2 || (!a.wsrc && a.nslab == 1 && p->max_degree >= 64 * parts * parts);   // see the kernel
                if (a.wsrc && eight)  stored_rowgroup_kernel<FMT, true, 8><<<grid, block, 0, stream>>>(a);
                else if (a.wsrc)      stored_rowgroup_kernel<FMT, true, 4><<<grid, block, 0, stream>>>(a);
                else if (eight)       stored_rowgroup_kernel<FMT, false, 8><<<grid, block, 0, stream>>>(a);
                else                  stored_rowgroup_kernel<FMT, false, 4><<<grid, block, 0, stream>>>(a);
            }
        }
    } else if (!gat) {
        const bool maxop = c.mode == RETEXO_MAX;
        if (E == 8)      { if (maxop) dispatch_linear<FMT, 8, true>(nc, a, n_heavy, N, stream); else dispatch_linear<FMT, 8, false>(nc, a, n_heavy, N, stream); }
        else if (E == 4) { if (maxop) dispatch_linear<FMT, 4, true>(nc, a, n_heavy, N, stream); else dispatch_linear<FMT, 4, false>(nc, a, n_heavy, N, stream); }
        else             { if (maxop) dispatch_linear<FMT, 1, true>(nc, a, n_heavy, N, stream); else dispatch_linear<FMT, 1, false>(nc, a, n_heavy, N, stream); }
    } else {
        // rows of ordinary length compute the source scores from the gathered rows (see the kernel)
        const int g = a.Dh / 4;
        const bool flash = E == 4 && opt.gat_flash && a.Dh % 4 == 0 && g <= 64 && (g & (g - 1)) == 0 &&
                           (uintptr_t)c.attn_src % 16 == 0;
        // (not over 4 GiB and more, whose byte offsets take 64 bits)
        const bool rows = flash && off32 && (uintptr_t)c.attn_dst % 16 == 0;
        if (rows) {
            a.table_bytes = (uint32_t)(((N - 1) * c.ldz + align_up(F, 4)) * 2);
            switch (g) {
                case 1:  dispatch_gat_rows<FMT, 1>(a, p, c.attn_src, c.attn_dst, stream); break;
                case 2:  dispatch_gat_rows<FMT, 2>(a, p, c.attn_src, c.attn_dst, stream); break;
                case 4:  dispatch_gat_rows<FMT, 4>(a, p, c.attn_src, c.attn_dst, stream); break;
                case 8:  dispatch_gat_rows<FMT, 8>(a, p, c.attn_src, c.attn_dst, stream); break;
                case 16: dispatch_gat_rows<FMT, 16>(a, p, c.attn_src, c.attn_dst, stream); break;
                case 32: dispatch_gat_rows<FMT, 32>(a, p, c.attn_src, c.attn_dst, stream); break;
                default: dispatch_gat_rows<FMT, 64>(a, p, c.attn_src, c.attn_dst, stream); break;
            }
            if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
            return RETEXO_OK;
        }
        const int hp = heads_padded(c.heads);
        const GatWorkspace w = gat_workspace(N, F, c.heads, false);
        float* el = (float*)((char*)c.workspace + w.el);
        float* er = (float*)((char*)c.workspace + w.er);
        a.el = el;
        a.er = er;
        const bool vec_scores = F % 4 == 0 && c.ldz % 4 == 0 && (uintptr_t)Z % 8 == 0 && F < (1ll << 30) &&
                                (uintptr_t)c.attn_src % 16 == 0 && (uintptr_t)c.attn_dst % 16 == 0 && opt.max_vec >= 4;
        if (vec_scores) {
            const unsigned gv = (unsigned)((N + 15) / 16);
            if (hp == 4) stored_scores_vec_kernel<FMT, 4><<<dim3(gv), dim3(256), 0, stream>>>(N, F, a.Dh, Z, c.ldz, c.attn_src, c.attn_dst, el, er);
            else stored_scores_vec_kernel<FMT, 8><<<dim3(gv), dim3(256), 0, stream>>>(N, F, a.Dh, Z, c.ldz, c.attn_src, c.attn_dst, el, er);
        } else {
            const unsigned gb = (unsigned)((N + 3) / 4);
            if (hp == 4) stored_scores_kernel<FMT, 4><<<dim3(gb), dim3(256), 0, stream>>>(N, F, a.Dh, Z, c.ldz, c.attn_src, c.attn_dst, el, er);
            else stored_scores_kernel<FMT, 8><<<dim3(gb), dim3(256), 0, stream>>>(N, F, a.Dh, Z, c.ldz, c.attn_src, c.attn_dst, el, er);
        }
        const bool hu = (a.Dh % E) == 0;
        int64_t n_table = N;          // rows [0, n_table) of the schedule go through the table kernels
        if (flash && N > n_heavy) {
            StoredArgs f = a;
            f.nslab = 1;
            f.row_begin = n_heavy;
            f.row_count = N - n_heavy;
            const dim3 grid((unsigned)((f.row_count + kLightWaves - 1) / kLightWaves)), block(64 * kLightWaves);
            switch (g) {
                case 1:  stored_gat_flash_kernel<FMT, 1><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
                case 2:  stored_gat_flash_kernel<FMT, 2><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
                case 4:  stored_gat_flash_kernel<FMT, 4><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
                case 8:  stored_gat_flash_kernel<FMT, 8><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
                case 16: stored_gat_flash_kernel<FMT, 16><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
                case 32: stored_gat_flash_kernel<FMT, 32><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
                default: stored_gat_flash_kernel<FMT, 64><<<grid, block, 0, stream>>>(f, c.attn_src, hp); break;
            }
            n_table = n_heavy;
        }
        if (n_table == 0) {
            // nothing left for the table kernels
        } else if (E == 8) {
            if (hp == 4) { if (hu) dispatch_gat<FMT, 8, 4, true>(nc, a, n_heavy, N, stream); else dispatch_gat<FMT, 8, 4, false>(nc, a, n_heavy, N, stream); }
            else         { if (hu) dispatch_gat<FMT, 8, 8, true>(nc, a, n_heavy, N, stream); else dispatch_gat<FMT, 8, 8, false>(nc, a, n_heavy, N, stream); }
        } else if (E == 4) {
            if (hp == 4) { if (hu) dispatch_gat<FMT, 4, 4, true>(nc, a, n_heavy, n_table, stream); else dispatch_gat<FMT, 4, 4, false>(nc, a, n_heavy, n_table, stream); }
            else         { if (hu) dispatch_gat<FMT, 4, 8, true>(nc, a, n_heavy, n_table, stream); else dispatch_gat<FMT, 4, 8, false>(nc, a, n_heavy, n_table, stream); }
        } else {
            if (hp == 4) dispatch_gat<FMT, 1, 4, true>(nc, a, n_heavy, N, stream);
            else dispatch_gat<FMT, 1, 8, true>(nc, a, n_heavy, N, stream);
        }
    }
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}

}  // namespace

template <int FMT>
static void store(int64_t N, int64_t F, const float* src, int64_t lds, uint16_t* dst, int64_t ldd, hipStream_t stream)
{
    const bool bases = (uintptr_t)src % 16 == 0 && (uintptr_t)dst % 8 == 0, wide = bases && lds % 4 == 0 && ldd % 4 == 0;
    auto blocks = [](int64_t items, int64_t per) { return dim3((unsigned)std::min<int64_t>((items + per - 1) / per, 16384)); };
    if (bases && lds == F && ldd == F) {
        store_run_kernel<FMT><<<blocks(N * F, 4096), dim3(256), 0, stream>>>(N * F, src, dst);
        return;
    }
    const int64_t vectors = wide ? (F + 3) / 4 : F;
    int lg = 0;
    while (lg < 6 && (1 << lg) < vectors) ++lg;
    auto go = [&](auto kernel, int rows) {
        kernel<<<blocks(N, (256 >> lg) * rows), dim3(256), 0, stream>>>(N, F, src, lds, dst, ldd, lg);
    };
    const bool stream_past = N * lds * 4 > (256ll << 20);
    // (rows of several column steps have enough in flight by themselves: 232,965 x 602 unaligned 226 us with four rows,
    // 209 with one; x 256 73 and 90)
    if (!wide && F <= 256) go(store_rows_kernel<FMT, 1, 4, false>, 4);
    else if (!wide)        go(store_rows_kernel<FMT, 1, 1, false>, 1);
    else if (vectors > 64) go(store_rows_kernel<FMT, 4, 1, true>, 1);
    else if (stream_past)  go(store_rows_kernel<FMT, 4, 4, true>, 4);
    else                   go(store_rows_kernel<FMT, 4, 4, false>, 4);
}

int launch_store_rows(int storage, int64_t N, int64_t F, const float* src, int64_t lds, void* dst, int64_t ldd,
                      hipStream_t stream)
{
    if (N == 0 || F == 0) return RETEXO_OK;
    if (storage == RETEXO_STORE_BF16) store<FMT_BF16>(N, F, src, lds, (uint16_t*)dst, ldd, stream);
    else store<FMT_FP16>(N, F, src, lds, (uint16_t*)dst, ldd, stream);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}

int launch_aggregate_stored(const StoredCall& c, hipStream_t stream)
{
    if (c.plan->N == 0 || c.F == 0) return RETEXO_OK;
    return c.storage == RETEXO_STORE_BF16 ? launch_stored<FMT_BF16>(c, stream) : launch_stored<FMT_FP16>(c, stream);
}
