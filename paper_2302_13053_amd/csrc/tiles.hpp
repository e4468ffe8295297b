// Pieces shared by the MFMA kernels (dense transform and weight gradient).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTileK = 16;    // K extent of one LDS tile

// f(0), f(1), .. f(N - 1) with the index as a constant: register arrays are only ever indexed by constants
template <int... I, class F>
__device__ __forceinline__ void each_index(std::integer_sequence<int, I...>, F&& f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void each(F&& f) { each_index(std::make_integer_sequence<int, N>{}, f); }

#define RETEXO_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// ---------------------------------------------------------------------------
// float32 products on the bf16 matrix cores.
//
// A float32 is the sum of three bf16 values: hi = round(x), mid = round(x - hi), lo = x - hi - mid.  Both
// differences are exact, and the three 8-bit significands with their signs cover all 24 bits, so nothing of x is
// lost.  Of the nine partial products of a * b the six with at least one hi or two mid are computed, each exact in
// float32 and added up in float32 by the matrix core; the three left out (mid*lo, lo*mid, lo*lo) are below 2^-24 of
// the product.  v_mfma_f32_32x32x16_bf16 does sixteen k in the time in which v_mfma_f32_32x32x2_f32 does one: six
// of them against eight.
//
// The five small products have a running sum of their own, added to that of hi*hi at the end: the matrix core rounds the
// sum after every eight k (and drops what lies 25 bits below the largest term), so with small products on the large sum
// it would be rounded twelve times per sixteen k, where the float32 instruction rounds once per k that is not zero;
// this way it is twice.  (All six onto one sum: 512 rectified columns 3.2e-7 off the same in 64 bits in the 2-norm,
// the float32 instruction 2.8e-7.  Small sums of sixteen k added to the large one each time: as exact, 11 % slower.)
//
// Both operands are multiplied by 2^24 before they are split and the sums by 2^-48 at the end, which changes no bit of
// an ordinary result.  The last bit of the smallest float32 (2^-149) is then 2^-125, a normal bf16 number, so that no
// operand loses its mid and lo parts, however small it is (unscaled, one below 2^-110 did: 32 products of operands of
// about 2^-124 and 2^40 were 5.6e-4 off), and what the matrix core does with sums below its normal range stays below
// 2^-174 of the unscaled ones.  At the other end operands from 2^104 on and sums from 2^80 on overflow.
// Where they do, and for infinities and NaN (their remainders are NaN), the float32 instructions take over, one 32 x 32
// tile at a time (see `redo_tile`).
// ---------------------------------------------------------------------------
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));     // 16 bytes at any float's address

__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_low(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_high(uint32_t p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

constexpr float kSplitScale = 0x1p24f;          // of either operand
constexpr float kSplitUnscale = 0x1p-48f;       // of a sum of products

// Two floats, times `scale` (kSplitScale or its negative) -> pair q of their hi, mid and lo parts.
template <class V>
__device__ __forceinline__ void split_pair(float x0, float x1, float scale, int q, V (&part)[3])
{
    x0 *= scale;
    x1 *= scale;
    const uint32_t hi = bf16_pair(x0, x1);
    const float r0 = x0 - bf16_low(hi), r1 = x1 - bf16_high(hi);
    const uint32_t mid = bf16_pair(r0, r1);
    part[0][q] = hi;
    part[1][q] = mid;
    part[2][q] = bf16_pair(r0 - bf16_low(mid), r1 - bf16_high(mid));
}

// Whether any of a wave's 32 x 32 sums formed from split operands is not finite: then it cannot be trusted.
__device__ __forceinline__ bool redo_tile(const f32x16& acc)
{
    uint32_t top = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float x = acc[r];
        const uint32_t m = __builtin_bit_cast(uint32_t, x) & 0x7fffffffu;
        top = m > top ? m : top;
    }
    return __any(top >= 0x7f800000u);
}

// One 32 x 32 tile by the float32 instruction, operands straight from memory: `a` is this lane's row (lane % 32), element k
// at a[k * a_step], `b` its column.  k in ascending pairs, 2 U of them at a time with the next 2 U in flight (one pair at a
// time, a weight gradient with an infinite input waited for memory a thousand times over: 232,965 x 1204 -> 256 2.8 ms, so
// 2.0, 0.9 without the infinity; 1,000,000 x 2000 -> 32 5.6, 3.5 and 1.8; twice as many at a time is no faster).
template <int U>
__device__ __forceinline__ f32x16 float32_tile(const float* a, int64_t a_step, const float* b, int64_t b_step, int K, int lane)
{
    const int lk = lane >> 5;
    f32x16 x;
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = 0.0f;
    float va[2][U], vb[2][U];
    auto take = [&](int k0, auto slot_tag) {
        constexpr int slot = decltype(slot_tag)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 2 * u + lk;
            const bool in = k < K;
            const float av = a[(in ? k : 0) * a_step], bv = b[(in ? k : 0) * b_step];
            va[slot][u] = in ? av : 0.0f;
            vb[slot][u] = in ? bv : 0.0f;
        }
    };
    auto multiply = [&](int k0, auto slot_tag) {
        constexpr int cur = decltype(slot_tag)::value;
        if (k0 + 2 * U < K) take(k0 + 2 * U, std::integral_constant<int, cur ^ 1>{});
#pragma unroll
        for (int u = 0; u < U; ++u) x = __builtin_amdgcn_mfma_f32_32x32x2f32(va[cur][u], vb[cur][u], x, 0, 0, 0);
    };
    take(0, std::integral_constant<int, 0>{});
    for (int k0 = 0; k0 < K; k0 += 4 * U) {
        multiply(k0, std::integral_constant<int, 0>{});
        if (k0 + 2 * U < K) multiply(k0 + 2 * U, std::integral_constant<int, 1>{});
    }
    return x;
}

// LDS image of one K tile of a workgroup: 16-byte units of eight k of one row (of A) or column (of B),
// [part][k / 8][row], first A's BM rows, then B's BN.  The four units of padding per plane put the two k halves of a row,
// which neighbouring lanes write, into different banks; a matrix instruction's operand (lane l: row l % 32,
// k half l / 32) is 32 consecutive units.
template <int BM, int BN> struct SplitTile {
    static constexpr int LA = BM + 4, LB = BN + 4;
    static constexpr int units = 6 * (LA + LB);
    static __device__ __forceinline__ int a(int part, int half, int row) { return (part * 2 + half) * LA + row; }
    static __device__ __forceinline__ int b(int part, int half, int col) { return 6 * LA + (part * 2 + half) * LB + col; }
};

// Staging of an operand whose rows run along k (element (k, c) at src[k * ld + c]): a wave takes pieces of 64
// columns by KW k (one coalesced load per k), so every lane ends up with KW consecutive k of its column: eight where
// the workgroup's waves share the BW columns x 16 k of a tile evenly that way, else four.  (32 columns are staged
// twice, by two waves each with the same values.)  Columns past the end repeat the last one (their products are never
// stored); rows from k_end on repeat the last row and count as zero, which is seen to when they are split: a load whose
// value is looked at where it is issued waits for itself and for all loads before it.
// SETS: tiles held in registers.  Waits count loads in the order of their issue, so where one operand is fetched two tiles
// ahead, the other is too.
// The work on a piece comes in micro steps for split_k_loop: KW / 2 steps that split a pair, one that writes the
// parts to LDS, one that fetches the piece of a later tile.
template <int BW, int WAVES, int SETS = 1> struct KMajorStage {
    static constexpr int KW = BW >= 64 && BW / 32 % WAVES == 0 ? 8 : 4;
    static constexpr int chunks = BW == 32 ? WAVES : BW / 64 * (kTileK / KW);
    static constexpr int count = (chunks + WAVES - 1) / WAVES;
    static constexpr int steps = KW / 2 + 2;                        // micro steps per piece
    typedef uint32_t part_t __attribute__((ext_vector_type(KW / 2)));
    const float* src;
    int64_t ld, k0, k_end;
    int wave, lane;
    uint32_t col[count];              // byte offset of this lane's (clamped) column, per piece
    uint64_t lane_at;                 // BW == 32: byte offset of this lane's first element from the tile's first row
    float r[SETS][count][KW];
    part_t part[3];

    __device__ __forceinline__ int chunk(int i) const { return wave + WAVES * i; }
    __device__ __forceinline__ bool mine(int i) const { return chunks % WAVES == 0 || chunk(i) < chunks; }
    __device__ __forceinline__ int kk(int i) const             // first k of the piece inside the tile
    {
        return BW == 32 ? ((wave & 1) * 2 + (lane >> 5)) * 4 : chunk(i) / (BW / 64) * KW;
    }
    __device__ __forceinline__ int local(int i) const { return BW == 32 ? lane & 31 : (chunk(i) % (BW / 64)) * 64 + lane; }

    __device__ __forceinline__ void init(const float* s, int64_t ld_, int64_t k_begin, int64_t k_end_, int c0, int c_end, int wave_, int lane_)
    {
        src = s; ld = ld_; k0 = k_begin; k_end = k_end_; wave = wave_; lane = lane_;
#pragma unroll
        for (int i = 0; i < count; ++i) {
            const int c = c0 + local(i);
            col[i] = 4u * (uint32_t)(c < c_end ? c : c_end - 1);
        }
        if constexpr (BW == 32) lane_at = col[0] + 4 * (uint64_t)ld * (uint32_t)kk(0);
    }
    // The row's address is the same for all lanes and is formed in scalar registers (the empty asm keeps the compiler from
    // turning every row into a pointer of its own that each tile has to advance: thirty 64-bit additions per tile, and
    // spilled scalar registers).
    typedef const __attribute__((address_space(1))) char* global_t;
    static __device__ __forceinline__ float at(uint64_t row, uint64_t offset)
    {
        return *reinterpret_cast<const __attribute__((address_space(1))) float*>(reinterpret_cast<global_t>(row) + offset);
    }
    // EDGE: the tile may reach over the end
    template <int i, int set, bool EDGE>
    __device__ __forceinline__ void fetch(int kt)
    {
        if (!mine(i)) return;
        const int64_t k = k0 + (int64_t)kt * kTileK + (BW == 32 ? 0 : kk(i));
        const uint64_t first = reinterpret_cast<uint64_t>(src + k * ld);
        uint32_t low = __builtin_amdgcn_readfirstlane((uint32_t)first), high = __builtin_amdgcn_readfirstlane((uint32_t)(first >> 32));
        asm("" : "+s"(low), "+s"(high));
        const uint64_t row = (uint64_t)high << 32 | low;
        const uint64_t pitch = 4 * (uint64_t)ld;
        if constexpr (!EDGE) {
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                if constexpr (BW == 32) r[set][i][q] = at(row + q * pitch, lane_at);       // (the half-waves stage different k)
                else r[set][i][q] = at(row + q * pitch, col[i]);
            }
        } else {
            const int left = (int)(k_end - 1 - k);             // the last row there is, from k on (may lie before it)
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                if constexpr (BW == 32) r[set][i][q] = at(row, col[0] + (uint64_t)min(kk(i) + q, left) * pitch);
                else r[set][i][q] = at(row + (uint64_t)(int64_t)min(q, left) * pitch, col[i]);
            }
        }
    }
    // plane(part, k half, column) -> 16-byte unit of `base`; scale: kSplitScale, or its negative to stage the operand
    // negated; kt: the staged tile
    template <int M, int set, bool EDGE, class Plane>
    __device__ __forceinline__ void micro(u32x4* base, Plane&& plane, float scale, int kt, int nk)
    {
        constexpr int i = M / steps, st = M % steps;
        if (!mine(i)) return;
        if constexpr (EDGE && st == 0) {
            const int left = (int)(k_end - k0 - (int64_t)kt * kTileK) - kk(i);
#pragma unroll
            for (int q = 0; q < KW; ++q) r[set][i][q] = q < left ? r[set][i][q] : 0.0f;
        }
        if constexpr (st < KW / 2) {
            split_pair(r[set][i][2 * st], r[set][i][2 * st + 1], scale, st, part);
        } else if constexpr (st == KW / 2) {
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                u32x4* unit = base + plane(s, kk(i) >> 3, local(i));
                *reinterpret_cast<part_t*>(reinterpret_cast<char*>(unit) + (KW == 4 ? (kk(i) & 4) * 2 : 0)) = part[s];
            }
        } else {
            if (!EDGE || kt + SETS < nk) fetch<i, set, EDGE>(kt + SETS);
        }
    }
};

// the staging registers that belong to an LDS buffer
template <int SETS, class Buf>
__device__ __forceinline__ constexpr int set_of()
{
    if constexpr (SETS == 2) return Buf::value;
    else return 0;
}

// ---------------------------------------------------------------------------
// Software-pipelined K loop of one workgroup tile (six bf16 products per 32 x 32 x 16 block).
//
// A matrix core is kept busy only if what else a wave does fits between its matrix instructions (32 cycles each,
// two waves per SIMD).  So the staging work of a K tile is cut into `MICROS` steps of about ten instructions, spread
// over the matrix instructions before the tile's barrier; sched_barrier pins the order.  micro(m, buf, kt, edge): step m
// of "split the staged pieces (tile kt) into LDS buffer `buf` = kt % 2, and fetch those of tile kt + SETS in their place",
// whose loads so have at least one K tile of matrix instructions to arrive.  One-column tiles pass `buf` as a constant.
// Only the last tile may be partial: the steady loop ends where that one would be fetched, and holds no branch (which
// would leave the number of loads in flight unknown, so that every use waits for more of them than it needs: 232,965 x
// 1204 -> 256 847 us with the checks in the loop, 805 without).
// Columns of the wave's tile are worked through one after the other with B's operands a column ahead.
// The one barrier of a K tile stands before its last column, whose operands are already in registers: behind that
// barrier the next tile's first operands are read as soon as their registers are free.
// Contract on entry: tile 0 is in LDS buffer 0 and a barrier has passed; the next tiles' pieces (if there are any) are staged.
// a0 / b0: first row / column of this wave's 32 x 32 TN block of accumulators, which leave with kSplitScale^2 in them.
// ---------------------------------------------------------------------------
// nk: tiles; n_whole: those that are whole.
template <int TN, int BM, int BN, int MICROS, int SETS, class Micro>
__device__ __forceinline__ void split_k_loop(f32x16 (&acc)[TN], const u32x4* __restrict__ lds, int nk, int n_whole, int a0,
                                             int b0, int lane, Micro&& micro)
{
    using T = SplitTile<BM, BN>;
    constexpr int SLOTS = TN == 1 ? 1 : TN % 2 ? TN : 2;      // register sets of B operands: a column ahead, also across tiles
    constexpr int HI = 0, MID = 1, LO = 2;
    constexpr int pa[6] = {HI, HI, HI, LO, MID, MID}, pb[6] = {HI, LO, MID, HI, MID, HI};
    constexpr int G = (TN > 1 ? TN - 1 : 1) * 6;              // matrix instructions before the barrier
    const int lrow = lane & 31, lk = lane >> 5;
    bf16x8 af[3], bf[SLOTS][3];
    f32x16 small[TN];                                         // sums of all products but hi*hi
    auto read_a = [&](int buf, int part) {
        af[part] = __builtin_bit_cast(bf16x8, lds[buf * T::units + T::a(part, lk, a0 + lrow)]);
    };
    auto read_b = [&](int buf, int j, int slot) {
#pragma unroll
        for (int part = 0; part < 3; ++part)
            bf[slot][part] = __builtin_bit_cast(bf16x8, lds[buf * T::units + T::b(part, lk, b0 + j * 32 + lrow)]);
    };
    read_b(0, 0, 0);
    read_a(0, HI);
    read_a(0, LO);
    read_a(0, MID);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) small[j][r] = 0.0f;
    constexpr std::true_type go_on{}, edge{};
    constexpr std::false_type finish{}, steady{};
    auto tile = [&](int kt, auto more_tag, auto buf, auto next, auto edge_tag) {
        constexpr bool more = decltype(more_tag)::value;
        each<TN * 6>([&](auto at) {
            constexpr int g = decltype(at)::value, j = g / 6, p = g % 6;
            constexpr bool last = TN > 1 && j == TN - 1;
            if constexpr (last && more && p == 0) {
                // every wave has read its operands of this tile and written its share of the next one
                __syncthreads();
                RETEXO_SCHED_FENCE();
                read_b(next, 0, 0);
            }
            f32x16& sum = p == 0 ? acc[j] : small[j];
            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[pa[p]], bf[j % SLOTS][pb[p]], sum, 0, 0, 0);
            RETEXO_SCHED_FENCE();
            if constexpr (p == 0 && j + 1 < TN) read_b(buf, j + 1, (j + 1) % SLOTS);
            if constexpr (last && more) {
                if constexpr (p == 2) read_a(next, HI);
                if constexpr (p == 3) read_a(next, LO);
                if constexpr (p == 5) read_a(next, MID);
            }
            if constexpr (!last && more) {
                constexpr int m0 = g * MICROS / G, m1 = (g + 1) * MICROS / G;
                each<m1 - m0>([&](auto m) { micro(std::integral_constant<int, m0 + decltype(m)::value>{}, next, kt + 1, edge_tag); });
            }
            RETEXO_SCHED_FENCE();
        });
        if constexpr (TN == 1 && more) {
            __syncthreads();
            RETEXO_SCHED_FENCE();
            read_b(next, 0, 0);
            read_a(next, HI);
            read_a(next, LO);
            read_a(next, MID);
        }
    };
    if constexpr (TN == 1) {
        // (unrolled over both buffers, which the wider tiles have no registers for)
        constexpr std::integral_constant<int, 0> even{};
        constexpr std::integral_constant<int, 1> odd{};
        int kt = 0;
        for (; kt + 2 + SETS < n_whole; kt += 2) {
            tile(kt, go_on, even, odd, steady);
            tile(kt + 1, go_on, odd, even, steady);
        }
        for (; kt + 2 < nk; kt += 2) {
            tile(kt, go_on, even, odd, edge);
            tile(kt + 1, go_on, odd, even, edge);
        }
        if (kt + 1 < nk) {
            tile(kt, go_on, even, odd, edge);
            tile(kt + 1, finish, odd, even, edge);
        } else if (kt < nk) {
            tile(kt, finish, even, odd, edge);
        }
    } else {
        int kt = 0;
        for (; kt + 1 + SETS < n_whole; ++kt) tile(kt, go_on, kt & 1, (kt & 1) ^ 1, steady);
        for (; kt + 1 < nk; ++kt) tile(kt, go_on, kt & 1, (kt & 1) ^ 1, edge);
        if (nk > 0) tile(nk - 1, finish, (nk - 1) & 1, nk & 1, edge);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] += small[j][r];
}
