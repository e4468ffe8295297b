// Dense transform Z = act(H W + b): the fully connected layer (+ ReLU) that is
// the f of Eq. 1, evaluated for every node once a layer has been trained.
//
// This is the one dense contraction on the path, so it runs on the matrix
// cores: every float32 as three bf16 values, six exact products of them per
// product, summed in float32 (tiles.hpp).  What is left out is below the
// rounding of a float32 sum, and the sum itself is rounded less often.  Error
// against 64 bits (2-norm, normal inputs; v_mfma_f32_32x32x2_f32, which carried
// this product before, in brackets): K = 100 0.6e-7 (1.8e-7), K = 256 0.9e-7
// (2.9e-7), K = 1204 2.0e-7 (6.2e-7), K = 2866 3.3e-7 (9.6e-7); 512 rectified
// columns 1.0e-7 (2.8e-7).
//
// Tiling.  A workgroup owns a 128 x BN output tile with BN >= D_out whenever
// D_out <= 256, so H — by far the larger operand — is read from HBM exactly
// once.  The K loop moves 16 columns of H and rows of W per step through LDS, as
// bf16 parts in the layout of the matrix operands.  Tiles wider than 128 run
// eight waves, one workgroup per CU (217 registers, 228 where signs are decided, 75 KB of LDS), narrower ones
// four waves and two to four workgroups.  W is split by every workgroup again: the
// call has no scratch memory to keep its parts in.
//
// What bounds the wide tiles is power, the splitting between the matrix
// instructions and the change between loading and storing: a single launch runs at
// 1.8-1.9 of 2.4 GHz with the matrix cores busy half of its cycles (GRBM_GUI_ACTIVE,
// SQ_VALU_MFMA_BUSY_CYCLES), the same launch on zeros is a quarter faster, and a bf16
// library product of 8192^3 reaches 1210-1280 TFLOP/s where this kernel issues
// 960-1110.  Measured (float32 instructions before): 2,449,029 x 256 -> 256 2.01 ms =
// 160 TFLOP/s (2.62 ms), 232,965 x 1204 -> 256 0.805 ms = 178 (1.20), 2,449,029 x 256
// -> 188 1.69 ms (2.01), 232,965 x 512 -> 41 0.136 ms = 3.8 TB/s (0.182), 100,000 x
// 512 -> 128 93 us (134), 40,000 x 2866 -> 64 157 us (345).
//
// Sources are clamped instead of checked (rows past the end repeat the last
// row, columns past D_out the last column), so the loop carries no selects;
// only the last tiles of K, which may be partial, have a form of their own.
// Loads are four bytes wide (W) or 16 bytes at any float's address (H), so every
// alignment and leading dimension takes this kernel, in one order of arithmetic.
// Short rows into narrow outputs are within a few per cent of what they took on the
// float32 instruction, not below it: 1,000,000 x 64 -> 32 79.5 us (75.7),
// 889,043 x 48 -> 8 51.5 (49.5), 300,000 x 8 -> 128 36.8 (35.3).  Bias and ReLU are
// applied to the accumulators on the way out, through one pointer per 32x32 tile
// that walks down the rows: every store covers two whole cache lines.  (Passed
// through LDS first, to leave 16 bytes per lane: 2,449,029 x 256 -> 256 2.15 ms
// where this was 2.08, x 16 -> 256 547 us and 500.)  Matrices of few rows take
// the few-rows kernel at the end (K split over the waves of a workgroup).
#include "common.hpp"
#include "tiles.hpp"

#include <type_traits>

namespace {

// Bias, ReLU, optional mask and store of the accumulators of one wave.
// Accumulator element r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32 of its tile.
// Only the last row block of the matrix checks rows.
// MASKED: sums[c] gets the sum of the wave's 32 rows of its column c.
template <int TN, bool MASKED>
__device__ __forceinline__ void write_out(const f32x16 (&acc)[TN], const float (&bv)[TN], int64_t N, int D_out,
                                          int64_t row_base, int col_base, int lane, int relu,
                                          float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm,
                                          bool whole_block, float* __restrict__ sums)
{
    const int lrow = lane & 31, lk = lane >> 5;
    auto run = [&](auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = col_base + j * 32 + lrow;
            if (col >= D_out) continue;
            const int64_t row0 = row_base + 4 * lk;
            float* p = Z + row0 * ldz + col;
            float mv[16], sum[4] = {};
            if constexpr (MASKED) {
                // backward of a ReLU layer: the value passes only where the forward activation was positive
                const float* pm = mask + row0 * ldm + col;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int ro = 8 * (r / 4) + (r % 4);
                    mv[r] = (FULL || row0 + ro < N) ? pm[ro * ldm] : 0.0f;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ro = 8 * (r / 4) + (r % 4);
                float x = acc[j][r] + bv[j];
                if (relu) x = fmaxf(x, 0.0f);
                if constexpr (MASKED) {
                    x = mv[r] > 0.0f ? x : 0.0f;         // (rows past the end: 0)
                    sum[r % 4] += x;
                }
                if (FULL || row0 + ro < N) p[ro * ldz] = x;
            }
            if constexpr (MASKED) {
                const float half = (sum[0] + sum[1]) + (sum[2] + sum[3]);
                const float both = half + __shfl_xor(half, 32, 64);      // (both lanes hold the same column)
                if (lk == 0) sums[j * 32 + lrow] = both;
            }
        }
    };
    if (whole_block) run(std::true_type{});
    else run(std::false_type{});
}

// Which side of zero a sum lies on, where the caller goes by that: a sum (plus its bias) within rounding of zero is
// formed again as one chain of float32 multiply-adds, k ascending, which is what v_mfma_f32_32x32x2_f32 makes of it.
// "Within rounding": 2^-25 sqrt(K) of the wave's largest finite sum, six to nine times what the two sums were seen apart
// (2-norm, K = 29 to 2866), about one sum in 200,000; less for a row whose largest input (`row_top`, of the wave's 32
// rows) or a column whose largest weight (`col_top`, of the wave's columns) is below a quarter of the wave's, so that rows
// and units of very different size do not all count as near zero beside the largest.
// A sum of exactly zero stays zero: no product, or products that cancel in pairs once they are split (which a chain of
// float32 multiply-adds may leave a rounding of; the exact sum is zero or below 2^-24 of its terms).  The two cannot be
// told apart here, and forming the first again costs steps over sparse inputs and pruned weights dearly: 232,965 x 1204 ->
// 256 with 2 % of the inputs and 10 % of the weights left 7.1 ms instead of 2.0.
// The wave works on one sum at a time: 256 k of the row and the column at once into LDS, then one multiply-add per k in
// every lane: about 3 us at K = 1120.  A 32 x 32 tile with more than kSingles of them takes the float32 instruction as a
// whole, 35 us at that K (which for every tile was a third of a small training step: 39,895 x 1120 -> 64).
// A step with every second unit's weights at 1e-6 of the others' took 11 ms there without `col_top` and the whole tiles,
// 0.25 ms with them; rows between 1e-6 and 1e6 of the mean 0.36 and 0.25.
constexpr int kChain = 256;
constexpr int kSingles = 10;
template <int TN>
__device__ __forceinline__ void decide_near_zero(f32x16 (&acc)[TN], const float (&bv)[TN], int D_in, int D_out,
                                                 const float* __restrict__ H, int64_t ldh, const float* __restrict__ W,
                                                 int64_t row_base, int64_t N, int col_base, int lane, const float* row_top,
                                                 const float* col_top, f32x4* __restrict__ chain)
{
    // what is not finite says nothing about the size of the others
    auto finite = [](float x) { return __builtin_fabsf(x) < INFINITY ? __builtin_fabsf(x) : 0.0f; };
    auto wave_largest = [](float x) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
        return x;
    };
    float top = 0.0f, weight = 0.0f;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) top = fmaxf(top, finite(acc[j][r]));
        weight = fmaxf(weight, finite(col_top[j * 32 + (lane & 31)]));
    }
    top = wave_largest(top);
    weight = wave_largest(weight);
    const float input = wave_largest(finite(row_top[lane & 31]));
    auto share = [](float x, float largest) { return x > 0.0f ? fminf(1.0f, 4.0f * (x / largest)) : 0.0f; };
    const float coarse = top * (0x1p-25f * sqrtf((float)D_in));
    const int64_t rows_left = N - row_base;
    float line[16];                              // of this lane's sums, by row
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int in_tile = 8 * (r / 4) + 4 * (lane >> 5) + r % 4;
        line[r] = in_tile < rows_left ? coarse * share(row_top[in_tile], input) : 0.0f;
    }
    each<TN>([&](auto at) {
        constexpr int j = decltype(at)::value;
        const int col = col_base + j * 32 + (lane & 31);
        const float unit = col < D_out ? share(col_top[j * 32 + (lane & 31)], weight) : 0.0f;
        auto near = [&](int r) {
            return __ballot(__builtin_fabsf(acc[j][r] + bv[j]) < line[r] * unit && acc[j][r] != 0.0f);
        };
        int count = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) count += __popcll(near(r));
        if (count == 0) return;                  // (uniform, as is the next)
        if (count > kSingles) {
            acc[j] = float32_tile<TN == 1 ? 8 : 16>(H + min(row_base + (lane & 31), N - 1) * ldh, 1, W + min(col, D_out - 1), D_out,
                                                   D_in, lane);
            return;
        }
        each<16>([&](auto element) {
            constexpr int r = decltype(element)::value;
            uint64_t close = near(r);
            while (close) {
                const int src = __ffsll((unsigned long long)close) - 1;
                close &= close - 1;
                const float* hp = H + (row_base + 8 * (r / 4) + 4 * (src >> 5) + r % 4) * ldh;
                const float* wp = W + (col_base + j * 32 + (src & 31));
                float sum = 0.0f;
                for (int k0 = 0; k0 < D_in; k0 += kChain) {
                    float h[kChain / 64], w[kChain / 64];
#pragma unroll
                    for (int i = 0; i < kChain / 64; ++i) {
                        const int k = k0 + i * 64 + lane;
                        h[i] = k < D_in ? hp[k] : 0.0f;
                        w[i] = k < D_in ? wp[(int64_t)k * D_out] : 0.0f;
                    }
                    float* c = reinterpret_cast<float*>(chain);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
                    for (int i = 0; i < kChain / 64; ++i) {
                        c[i * 64 + lane] = h[i];
                        c[kChain + i * 64 + lane] = w[i];
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 8
                    for (int q = 0; q < kChain / 4; ++q) {
                        const f32x4 a = chain[q], b = chain[kChain / 4 + q];
                        sum = fmaf(a.x, b.x, sum);
                        sum = fmaf(a.y, b.y, sum);
                        sum = fmaf(a.z, b.z, sum);
                        sum = fmaf(a.w, b.w, sum);
                    }
                }
                if (lane == src) acc[j][r] = sum;
            }
        });
    });
}

// The block kernel: 128 x BN outputs per workgroup, 32 rows and up to 128 columns per wave (whose two running sums then
// take 128 registers): four waves, or eight for the tiles wider than 128; any alignment and leading dimension.
// MASKED (the backward of a ReLU layer) also leaves the column sums of every 128-row block, which the bias gradient is made
// of, as long as the values are in registers: a pass of its own over them takes 45 us for 232,965 x 256.
// HALVES: the halves of K apart, for one workgroup per compute unit, which has the registers: a layer's input is often [self |
// aggregate], and terms of unlike size round each other (in_halves).
template <int BN> constexpr int transform_waves = BN > 128 ? 8 : 4;
template <int BN, bool MASKED, bool KEEP_SIGN, bool HALVES>
__global__ __launch_bounds__(64 * transform_waves<BN>, HALVES ? 1 : BN <= 64 ? 3 : 2) void transform_kernel(
    int64_t N, int D_in, int D_out, const float* __restrict__ H, int64_t ldh,
    const float* __restrict__ W, const float* __restrict__ bias, int relu,
    float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm, float* __restrict__ colsums)
{
    constexpr int BM = 128, WAVES = transform_waves<BN>, WN = BN / (WAVES / 4), TN = WN / 32;
    using T = SplitTile<BM, BN>;
    constexpr int SETS = BN == 32 ? 2 : 1;               // tiles staged in registers
    using WStage = KMajorStage<BN, WAVES, SETS>;
    constexpr int HP = BM * kTileK / (64 * WAVES) / 4;   // 16-byte pieces of H that a thread stages
    __shared__ u32x4 lds[2 * T::units];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int a0 = wave % 4 * 32, b0 = wave / 4 * WN;    // the wave's rows and columns of the tile
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    const int lrow = lane & 31;

    f32x16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

    // H: a thread stages HP pieces of four consecutive k, of rows 16 WAVES apart: four lanes fetch the 64 bytes of a row
    // that a tile holds (rows past the end repeat the last one, never stored).  The 32-column tile, whose matrix
    // instructions are over long before a row arrives from memory, stages two tiles of both operands ahead (2,449,029 x 256
    // -> 7 536 us, 300,000 x 2000 -> 32 513; two of H behind one of W 578 and 578, all one tile ahead 611 and more).
    const int hr = tid / 4, hk = tid % 4 * 4;
    const float* ph[HP];
#pragma unroll
    for (int v = 0; v < HP; ++v) ph[v] = H + min(m0 + hr + 16 * WAVES * v, N - 1) * ldh + hk;
    f32x4 ra[SETS][HP];
    int k0 = 0, K = HALVES ? D_in / 2 : D_in, nk = (K + kTileK - 1) / kTileK;      // the k of the sums at hand: [k0, k0 + K)
    auto fetch_h = [&](int kt, int v, auto set_tag, auto edge) {
        constexpr int set = decltype(set_tag)::value;
        const float* p = ph[v] + kt * kTileK;
        if (!decltype(edge)::value || (kt + 1) * kTileK <= K) {
            ra[set][v] = *reinterpret_cast<const f32x4_any*>(p);
        } else {
            const int last = K - 1 - kt * kTileK - hk;           // the row's last element, from p on (may lie before it)
#pragma unroll
            for (int q = 0; q < 4; ++q) ra[set][v][q] = p[min(q, last)];
        }
    };
    WStage sw;
    sw.init(W, D_out, 0, K, n0, D_out, wave, lane);

    float bv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + b0 + j * 32 + lrow;
        bv[j] = (bias && col < D_out) ? bias[col] : 0.0f;
    }

    constexpr int A_MICROS = HP * 4, MICROS = A_MICROS + WStage::count * WStage::steps;
    typedef uint32_t part_t __attribute__((ext_vector_type(2)));
    part_t part_h[3];
    float h_top[HP] = {};                                // largest input of this thread's parts of its rows
    float w_top[WStage::count] = {};                     // ... and weight of its columns
    auto micro = [&](auto step, auto buf, int kt, auto edge) {
        constexpr int m = decltype(step)::value;
        constexpr bool EDGE = decltype(edge)::value;
        constexpr int set = set_of<SETS, decltype(buf)>();
        u32x4* base = lds + buf * T::units;
        if constexpr (EDGE && m < A_MICROS && m % 4 == 0) {          // what lies past the row's end counts as zero (see KMajorStage)
#pragma unroll
            for (int q = 0; q < 4; ++q) ra[set][m / 4][q] = kt * kTileK + hk + q < K ? ra[set][m / 4][q] : 0.0f;
        }
        if constexpr (KEEP_SIGN && m < A_MICROS && m % 4 == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) h_top[m / 4] = fmaxf(h_top[m / 4], __builtin_fabsf(ra[set][m / 4][q]));
        }
        if constexpr (KEEP_SIGN && m >= A_MICROS && (m - A_MICROS) % WStage::steps == 0) {
            constexpr int i = (m - A_MICROS) / WStage::steps;
            if (sw.mine(i)) {
#pragma unroll
                for (int q = 0; q < WStage::KW; ++q) w_top[i] = fmaxf(w_top[i], __builtin_fabsf(sw.r[set][i][q]));
            }
        }
        if constexpr (m >= A_MICROS) {
            sw.template micro<m - A_MICROS, set, EDGE>(base, [](int s, int half, int c) { return T::b(s, half, c); }, kSplitScale, kt, nk);
        } else if constexpr (m % 4 < 2) {
            split_pair(ra[set][m / 4][m % 4 * 2], ra[set][m / 4][m % 4 * 2 + 1], kSplitScale, m % 4, part_h);
        } else if constexpr (m % 4 == 2) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
                *reinterpret_cast<part_t*>(reinterpret_cast<char*>(base + T::a(s, hk >> 3, hr + 16 * WAVES * (m / 4))) + (hk & 4) * 2) = part_h[s];
        } else {
            if (!EDGE || kt + SETS < nk) fetch_h(kt + SETS, m / 4, std::integral_constant<int, set>{}, edge);
        }
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::true_type edge{};
    auto fetch_all = [&](int kt, auto set_tag) {
#pragma unroll
        for (int v = 0; v < HP; ++v) fetch_h(kt, v, set_tag, edge);
        each<WStage::count>([&](auto i) { sw.template fetch<decltype(i)::value, decltype(set_tag)::value, true>(kt); });
    };
    f32x16 early[HALVES ? TN : 1];                       // the first half's sums
    for (int half = 0;; ++half) {
        fetch_all(0, first);
        if (SETS == 2 && nk > 1) fetch_all(1, std::integral_constant<int, SETS - 1>{});
        each<MICROS>([&](auto m) { micro(m, first, 0, edge); });
        __syncthreads();
        split_k_loop<TN, BM, BN, MICROS, SETS>(acc, lds, nk, K / kTileK, a0, b0, lane, micro);
        if (!HALVES || half == 1) break;
#pragma unroll
        for (int j = 0; j < (HALVES ? TN : 1); ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                early[j][r] = acc[j][r];
                acc[j][r] = 0.0f;
            }
        k0 = K;
        K = D_in - K;
        nk = (K + kTileK - 1) / kTileK;
#pragma unroll
        for (int v = 0; v < HP; ++v) ph[v] += k0;
        sw.init(W, D_out, k0, D_in, n0, D_out, wave, lane);
        __syncthreads();                                 // every wave is done with the last tile
    }
    if constexpr (HALVES) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] += early[j][r];
    }

    each<TN>([&](auto at) {
        constexpr int j = decltype(at)::value;
        const float* hp = H + min(m0 + a0 + lrow, N - 1) * ldh;
        const float* wp = W + min(n0 + b0 + j * 32 + lrow, D_out - 1);
        if (D_in == 1) {              // the float32 instruction rounds the one product once, the split's two sums twice
            acc[j] = float32_tile<1>(hp, 1, wp, D_out, 1, lane);
        } else if (redo_tile(acc[j])) {
            acc[j] = float32_tile<TN == 1 ? 8 : 16>(hp, 1, wp, D_out, D_in, lane);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] *= kSplitUnscale;
        }
    });

    if constexpr (KEEP_SIGN) {
        // the tiles' memory: largest input of every row, largest weight of every column, operands of the waves' chains
        float* row_top = reinterpret_cast<float*>(lds);
        float* col_top = row_top + BM;
        f32x4* chain = reinterpret_cast<f32x4*>(lds) + (BM + BN) / 4 + wave * (2 * kChain / 4);
        static_assert(2 * T::units >= (BM + BN) / 4 + WAVES * (2 * kChain / 4), "they fit there");
        __syncthreads();                                 // every wave is done with the last tile
#pragma unroll
        for (int v = 0; v < HP; ++v) {
            h_top[v] = fmaxf(h_top[v], __shfl_xor(h_top[v], 1, 64));
            row_top[hr + 16 * WAVES * v] = fmaxf(h_top[v], __shfl_xor(h_top[v], 2, 64));
        }
        if (tid < BN) col_top[tid] = 0.0f;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < WStage::count; ++i)          // (numbers that are not negative order as their bits do)
            if (sw.mine(i)) atomicMax(reinterpret_cast<uint32_t*>(col_top + sw.local(i)), __builtin_bit_cast(uint32_t, w_top[i]));
        __syncthreads();
        decide_near_zero<TN>(acc, bv, D_in, D_out, H, ldh, W, m0 + a0, N, n0 + b0, lane, row_top + a0, col_top + b0, chain);
    }
    float* sums = reinterpret_cast<float*>(lds);         // [4][BN], in the tiles' memory
    if constexpr (MASKED) __syncthreads();               // every wave is done with the last tile
    write_out<TN, MASKED>(acc, bv, N, D_out, m0 + a0, n0 + b0, lane, relu, Z, ldz, mask, ldm, m0 + BM <= N,
                          sums + wave % 4 * BN + b0);
    if constexpr (MASKED) {
        __syncthreads();
        if (tid < BN && n0 + tid < D_out)
            colsums[(int64_t)blockIdx.x * D_out + n0 + tid] = (sums[tid] + sums[BN + tid]) + (sums[2 * BN + tid] + sums[3 * BN + tid]);
    }
}

// Few rows: a matrix with so few 128-row blocks that they would leave most compute units idle (a citation
// graph's 2,708 x 2,866 features give 22) is cut into 32-row blocks, and the K extent of each block is cut
// over the eight waves of its workgroup.  A wave needs no LDS and no barrier in its loop: per group of 8 k it
// fetches its operands straight into the MFMA layout — lane l holds k = 4 (l / 32) .. + 3 of row l % 32, so
// MFMA q of the group pairs k = q (lower half-wave) with k = 4 + q (upper half-wave) — eight groups at a time,
// the next eight in flight behind the MFMAs.  The eight partial tiles are then added in a fixed order (wave w + wave
// w + 4 in registers, then ((0 + 1) + 2) + 3 through LDS), so the result is reproducible.  The float32
// instruction carries these products: the kernel waits for memory, not for the matrix cores.
template <int TN, bool MASKED>
__global__ __launch_bounds__(512) void transform_few_rows_kernel(
    int64_t N, int D_in, int D_out, const float* __restrict__ H, int64_t ldh,
    const float* __restrict__ W, const float* __restrict__ bias, int relu,
    float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm, float* __restrict__ colsums)
{
    constexpr int BN = TN * 32, NW = 8;
    __shared__ float part[NW / 2][32][BN];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lrow = lane & 31, lk = lane >> 5;
    const int64_t m0 = (int64_t)blockIdx.x * 32;
    const int n0 = blockIdx.y * BN;

    const int groups = (D_in + 7) / 8;
    const int per = (groups + NW - 1) / NW;
    const int g0 = wave * per;
    const int g1 = g0 + per < groups ? g0 + per : groups;

    int64_t row = m0 + lrow;
    row = row < N ? row : N - 1;                 // rows past the end repeat the last one; never stored
    const float* hp = H + row * ldh;
    int col[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int c = n0 + j * 32 + lrow;
        col[j] = c < D_out ? c : D_out - 1;
    }

    f32x16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

    // operands of U groups at a time, the next U in flight behind this batch's MFMAs (a wave's loop is a chain
    // of memory latencies; the batch is what keeps enough bytes in flight).  A row's bytes come 16 at a time, at any
    // alignment; only a group that reaches over the end of K checks every element.
    constexpr int U = TN == 1 ? 8 : 4;           // (registers: eight groups of two column tiles spill)
    float a[2][U][4], b[2][U][TN][4];
    auto fetch = [&](int gb, auto slot_tag) {    // slot as a type: register arrays want constant indices
        constexpr int slot = decltype(slot_tag)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = gb + u, k = g * 8 + lk * 4;
            if (g >= g1) break;                  // (uniform, as is the next)
            if (g * 8 + 8 <= D_in) {
                const f32x4 t = *reinterpret_cast<const f32x4_any*>(hp + k);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a[slot][u][q] = t[q];
                    const float* wr = W + (int64_t)(k + q) * D_out;
#pragma unroll
                    for (int j = 0; j < TN; ++j) b[slot][u][j][q] = wr[col[j]];
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool in = k + q < D_in;
                    const float t = hp[in ? k + q : 0];
                    a[slot][u][q] = in ? t : 0.0f;
                    const float* wr = W + (int64_t)(in ? k + q : 0) * D_out;
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const float w = wr[col[j]];
                        b[slot][u][j][q] = in ? w : 0.0f;
                    }
                }
            }
        }
    };

    auto batch = [&](int gb, auto slot_tag) {
        constexpr int cur = decltype(slot_tag)::value;
        if (gb + U < g1) fetch(gb + U, std::integral_constant<int, cur ^ 1>{});
        RETEXO_SCHED_FENCE();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (gb + u >= g1) break;
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][u][q], b[cur][u][j][q], acc[j], 0, 0, 0);
        }
    };
    if (g0 < g1) fetch(g0, std::integral_constant<int, 0>{});
    for (int gb = g0; gb < g1; gb += 2 * U) {
        batch(gb, std::integral_constant<int, 0>{});
        if (gb + U < g1) batch(gb + U, std::integral_constant<int, 1>{});
    }

    // accumulator element r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of its tile
    auto put = [&](int slot) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) part[slot][8 * (r / 4) + 4 * lk + (r % 4)][j * 32 + lrow] = acc[j][r];
    };
    if (wave >= NW / 2) put(wave - NW / 2);
    __syncthreads();
    if (wave < NW / 2) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] += part[wave][8 * (r / 4) + 4 * lk + (r % 4)][j * 32 + lrow];
    }
    __syncthreads();
    if (wave < NW / 2) put(wave);
    __syncthreads();

    float sum = 0.0f;                            // of this thread's outputs, which lie in one column
    for (int e = tid; e < 32 * BN; e += 512) {
        const int r = e / BN, c = e % BN;
        const int64_t orow = m0 + r;
        const int ocol = n0 + c;
        if (orow >= N || ocol >= D_out) continue;
        float x = ((part[0][r][c] + part[1][r][c]) + part[2][r][c]) + part[3][r][c];
        x += bias ? bias[ocol] : 0.0f;
        if (relu) x = fmaxf(x, 0.0f);
        if constexpr (MASKED) x = mask[orow * ldm + ocol] > 0.0f ? x : 0.0f;
        Z[orow * ldz + ocol] = x;
        sum += x;
    }
    if constexpr (MASKED) {                      // column sums of the 32 rows, as in the block kernel
        __syncthreads();
        float* sums = &part[0][0][0];            // [512 / BN][BN]
        sums[tid] = sum;
        __syncthreads();
        if (tid < BN && n0 + tid < D_out) {
            float t[4] = {};
#pragma unroll
            for (int i = 0; i < 512 / BN; ++i) t[i % 4] += sums[i * BN + tid];
            colsums[(int64_t)blockIdx.x * D_out + n0 + tid] = (t[0] + t[1]) + (t[2] + t[3]);
        }
    }
}

// The same for long sums: 32 x 32 tiles, sixteen waves, operands through LDS.  The kernel above asks for sixteen
// bytes of 32 rows at a time and for single floats of W, which keeps the address units busy for as long as the matrix cores (2,708
// x 2,866 -> 64: 28.2 us; without its products, without W or without H 20.6, 20.6, 18.6).  Here chunks of 128 k come in whole
// lines, two ahead, and each wave multiplies eight k of every chunk: 24.3 us there (27.9), 1,433 columns 15.7 ->
// 14.4, 2,866 -> 256 82 -> 71.  Its products are 10 of the 24 us (1,433 float32 instructions of 64 cycles per tile, over four
// SIMDs); the rest is 23 chunks with a barrier and a round trip through LDS each.  Less work stays above: 2,708 x 1,433 -> 7 12.4
// and 14.0, 2,000 x 1,300 -> 64 11.6 and 12.9, 1,400 x 2,500 -> 32 20.1 and 21.2; where compute units have two tiles, 2,708 x 500 ->
// 256 18.2 and 19.5, 8,000 x 600 -> 41 15.5 and 17.1, 2,708 x 1,400 -> 256 42.7 and 40.6, 1,053 x 1,421 -> 765 46.6 and 53.9.
constexpr int64_t kStagedWork = 250000;      // tiles times k from which it is taken, up to 256 tiles
constexpr int kStagedMany = 1200;            // k from which it is taken, up to kStagedMost tiles
constexpr int64_t kStagedMost = 700;
template <bool MASKED, bool HALVES>
__global__ __launch_bounds__(1024, HALVES ? 4 : 8) void transform_few_staged_kernel(
    int64_t N, int D_in, int D_out, const float* __restrict__ H, int64_t ldh,
    const float* __restrict__ W, const float* __restrict__ bias, int relu,
    float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm, float* __restrict__ colsums)
{
    constexpr int NW = 16, KC = 128, SLICE = KC / NW;
    constexpr int PH = KC + 4, PW = 36;          // row pitches in LDS: a wave's reads meet no bank twice
    struct Operands { float h[32 * PH], w[KC * PW]; };
    typedef float parts_t[NW / 2][32][33];       // partial tiles, over the operands of a chunk
    static_assert(sizeof(parts_t) <= sizeof(Operands), "they fit there");
    __shared__ __align__(16) Operands sh[2];
    __shared__ float early[HALVES ? 1 : 1024];   // the first half's sums

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lrow = lane & 31, lk = lane >> 5;
    const int64_t m0 = (int64_t)blockIdx.x * 32;
    const int n0 = blockIdx.y * 32;
    // A thread's piece of a chunk: four k of a row of H, four columns of a row of W.  All are loaded without a branch (the
    // loads of two chunks stay in flight): a piece that reaches over the end of its row is loaded from four floats before
    // that (D_in, D_out >= 4) and moved into place, with zeroes behind it, on its way to LDS.
    const int hr = tid / (KC / 4), hk = tid % (KC / 4) * 4, wk = tid / 8, wc = n0 + tid % 8 * 4;
    const float* hp = H + (m0 + hr < N ? m0 + hr : N - 1) * ldh;           // rows past the end repeat the last one; never stored
    const float* wp = W + min(wc, D_out - 4);
    const int w_over = min(max(wc + 4 - D_out, 0), 4);
    const bool whole_columns = n0 + 32 <= D_out;                           // (uniform)
    auto moved = [](f32x4 t, int over) {         // elements past the row's end: zero
        f32x4 r = t;
        if (over & 1) r = f32x4{r[1], r[2], r[3], 0.0f};
        if (over & 2) r = f32x4{r[2], r[3], 0.0f, 0.0f};
        if (over & 4) r = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        return r;
    };

    // The halves of a sum apart: a layer's input is often [self | aggregate], and terms of unlike size round each other ([self | mean
    // of 12 neighbours], 2 % of self not zero, 2,866 -> 256, error against 64 bits 1.3e-7 in one sum, 7.2e-8 so, the kernel above
    // 8.6e-8).  HALVES: in registers of their own, where those cost nothing (one workgroup per compute unit; otherwise 2,708 x 2,866
    // -> 256 62 -> 69 us); without, one half after the other.
    const int half = D_in / 8 * 4;               // (whole pieces)
    int k_begin = 0, k_end = HALVES ? D_in : half, chunks = (k_end + KC - 1) / KC;
    f32x16 acc, first;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = first[r] = 0.0f;
    parts_t& part = *reinterpret_cast<parts_t*>(&sh[0]);
    auto put = [&](int slot) {
#pragma unroll
        for (int r = 0; r < 16; ++r) part[slot][8 * (r / 4) + 4 * lk + (r % 4)][lrow] = acc[r];
    };
    // the sixteen waves' partial tiles in `acc`, added in pairs (the fewest roundings): this thread's output, row tid / 32, column
    // tid % 32.  Begins where no wave uses the operands, ends with a barrier.
    auto reduce = [&]() {
        if (wave >= NW / 2) put(wave - NW / 2);
        __syncthreads();
        if (wave < NW / 2) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += part[wave][8 * (r / 4) + 4 * lk + (r % 4)][lrow];
        }
        __syncthreads();
        if (wave < NW / 2) put(wave);
        __syncthreads();
        float t[NW / 2];
#pragma unroll
        for (int w = 0; w < NW / 2; ++w) t[w] = part[w][tid / 32][tid % 32];
#pragma unroll
        for (int w = NW / 4; w >= 1; w /= 2)
#pragma unroll
            for (int i = 0; i < w; ++i) t[i] += t[i + w];
        __syncthreads();
        return t[0];
    };
    f32x4 rh[2], rw[2];
    auto load = [&](int ch, int slot) {
        const int k0 = k_begin + min(ch, chunks - 1) * KC;
        rh[slot] = *reinterpret_cast<const f32x4_any*>(hp + min(k0 + hk, D_in - 4));
        rw[slot] = *reinterpret_cast<const f32x4_any*>(wp + (int64_t)min(k0 + wk, D_in - 1) * D_out);
    };
    // one chunk of the k of [k_begin, k_end): the registers of `slot` go to its LDS buffer (last read two chunks ago: the barrier of
    // the chunk between lies behind every wave by then); the chunk two ahead takes the registers
    auto chunk = [&](int ch, int slot) {
        f32x4 h = rh[slot], w = rw[slot];
        if (ch == chunks - 1) {                  // (uniform)
            const int k = k_begin + ch * KC;
            h = moved(h, k + hk >= k_end ? 4 : max(k + hk + 4 - D_in, 0));
            w = k + wk < k_end ? w : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        if (!whole_columns) w = moved(w, w_over);
        *reinterpret_cast<f32x4*>(&sh[slot].h[hr * PH + hk]) = h;
        *reinterpret_cast<f32x4*>(&sh[slot].w[wk * PW + (wc - n0)]) = w;
        load(ch + 2, slot);
        __syncthreads();
        auto multiply = [&](f32x16& to) {
            const int kb = wave * SLICE + 4 * lk;    // lower half-wave: the slice's first four k, upper: the others
            const f32x4 a = *reinterpret_cast<const f32x4*>(&sh[slot].h[lrow * PH + kb]);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                to = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], sh[slot].w[(kb + q) * PW + lrow], to, 0, 0, 0);
        };
        if (HALVES && ch * KC + wave * SLICE < half) multiply(first);      // (uniform over the wave)
        else multiply(acc);
    };
    float x;
    for (;;) {
        load(0, 0);
        load(1, 1);
        int ch = 0;
        for (; ch + 1 < chunks; ch += 2) {
            chunk(ch, 0);
            chunk(ch + 1, 1);
        }
        if (ch < chunks) chunk(ch, 0);
        if constexpr (HALVES) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += first[r];
        }
        __syncthreads();                         // every wave is done with the operands
        x = reduce();
        if (k_end == D_in) break;
        if constexpr (!HALVES) early[tid] = x;
        k_begin = k_end;
        k_end = D_in;
        chunks = (k_end - k_begin + KC - 1) / KC;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    }

    if constexpr (!HALVES) x += early[tid];
    int out = tid;                               // one output per thread (its place is not kept in registers meanwhile)
    asm("" : "+v"(out));
    const int r = out / 32, c = out % 32;
    const int64_t orow = m0 + r;
    const int ocol = n0 + c;
    const bool inside = orow < N && ocol < D_out;
    if (inside) {
        x += bias ? bias[ocol] : 0.0f;
        if (relu) x = fmaxf(x, 0.0f);
        if constexpr (MASKED) x = mask[orow * ldm + ocol] > 0.0f ? x : 0.0f;
        Z[orow * ldz + ocol] = x;
    }
    if constexpr (MASKED) {                      // column sums of the 32 rows, as in the block kernel
        float* sums = &sh[0].h[0];
        sums[tid] = inside ? x : 0.0f;
        __syncthreads();
        if (tid < 32 && n0 + tid < D_out) {
            float t[4] = {};
#pragma unroll
            for (int i = 0; i < 32; ++i) t[i % 4] += sums[i * 32 + tid];
            colsums[(int64_t)blockIdx.x * D_out + n0 + tid] = (t[0] + t[1]) + (t[2] + t[3]);
        }
    }
}

// D_in == 0: the product is empty and every row is act(b); H and W are not touched (they may be NULL)
__global__ void bias_rows_kernel(int64_t N, int D_out, const float* __restrict__ bias, int relu,
                                 float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm)
{
    const int64_t total = N * D_out;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = e / D_out;
        const int col = (int)(e % D_out);
        float x = bias ? bias[col] : 0.0f;
        if (relu) x = fmaxf(x, 0.0f);
        if (mask) x = mask[row * ldm + col] > 0.0f ? x : 0.0f;
        Z[row * ldz + col] = x;
    }
}

// Which kernel a shape takes, by the shape only, never by alignment, so that one shape always takes one order of additions.
//  Few rows: fewer than 128 blocks, and up to 832 tiles of 32 x 32 or 512 workgroups of 64 columns, two for each compute unit.  A
//  compute unit takes some 9 ns per k and tile there, and 29 to 59 ns per k for one block of 128 rows, whose loop waits for memory
//  when it is alone: 8,000 x 600 -> 41 (500 tiles) 15.5 us and 20.9, 15,488 x 212 -> 64 (968 tiles, 484 workgroups) 11.0 and 13.3,
//  14,500 x 32 -> 64 5.7 and 5.3; with a third workgroup 9,070 x 2,219 -> 96 (852, 568) 95.8 and 70, 4,227 x 882 -> 216 (931, 532)
//  44.2 and 31.9, 2,708 x 32 -> 500 (1,360, 680) 8.2 and 6.9.  From 128 blocks the split products stay in one sum, which is a quarter
//  closer on inputs of one size, although few rows are faster (20,000 x 500 -> 20 14.7 and 18.3).  (The "transform_few_blocks"
//  setting, unless it is 128: fewer blocks than it says, however many tiles.)
//  Blocks: as wide as the output up to 256 columns; narrower, so that H is read more than once, where that gives up to 256 blocks
//  instead of fewer (14,000 x 500 -> 256 in 110 blocks 37.3, 220 of 128 columns 30.4; 8,000 x 1,000 -> 256 in 63 65.3, 252 of 64
//  38.9; 19,717 x 500 -> 256 in 155 36.6, 310 of 128 42.6), and half as wide where the widest are a few more than compute units
//  (2,708 x 64 -> 2,866 in 264 19.1, 506 of 128 12.9; 40,000 x 256 -> 256 in 313 44.6, 626 40.3), up to three of the narrower for
//  each (49,542 x 86 -> 256 in 388 26.8, 776 of 128 30.2).
int64_t block_width(int64_t D_out) { return D_out <= 32 ? 32 : D_out <= 64 ? 64 : D_out <= 128 ? 128 : D_out <= 192 ? 192 : 256; }
int64_t blocks_of(int64_t N, int64_t D_out, int64_t bn) { return (N + 127) / 128 * ((D_out + bn - 1) / bn); }
bool takes_few_rows(int64_t N, int64_t D_out)
{
    const int64_t few = agg_options().few_blocks, gx = (N + 31) / 32;
    if (blocks_of(N, D_out, block_width(D_out)) >= few) return false;
    return few != 128 || gx * ((D_out + 31) / 32) <= 832 || gx * ((D_out + 63) / 64) <= 512;
}
// The split products of shapes that few rows took before: the halves of K apart (see transform_kernel).  [self | mean of 12
// neighbours], 2 % of self not zero, 2,866 columns, error against 64 bits: few rows 8.6e-8, one sum 1.9e-7, so 5.4e-8; rectified
// normal columns 2.8e-7, 3.2e-7, 1.7e-7; of 127 columns 5.2e-8, 7.3e-8, 3.5e-8, of 16 2.9e-8, 3.4e-8, 2.7e-8.  5,000 x 500 -> 300
// 20.8 us in one sum, 23.1 so; 8,000 x 1,000 -> 256 38.5 and 42.0; 2,708 x 64 -> 500 6.6 and 8.3 (few rows 9.8).
bool in_halves(int64_t N, int64_t D_in, int64_t D_out) { return D_in >= 2 && blocks_of(N, D_out, block_width(D_out)) < 128; }
int64_t block_width_for(int64_t N, int64_t D_out)
{
    const int64_t widest = block_width(D_out), blocks = blocks_of(N, D_out, widest);
    if (blocks > 256) return widest == 256 && blocks <= 384 ? 128 : widest;
    int64_t bn = widest;
    for (int64_t narrower : {128, 64, 32})
        if (narrower < bn && blocks_of(N, D_out, narrower) <= 256) bn = narrower;
    return bn;
}

template <int BN, bool MASKED>
void launch(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh, const float* W,
            const float* b, bool relu, float* Z, int64_t ldz, const float* mask, int64_t ldm, bool keep_sign,
            float* colsums, hipStream_t stream)
{
    const dim3 grid((unsigned)((N + 127) / 128), (unsigned)((D_out + BN - 1) / BN)), block(64 * transform_waves<BN>);
    const int r = relu ? 1 : 0;
    auto go = [&](auto sign, auto halves) {
        transform_kernel<BN, MASKED, decltype(sign)::value, decltype(halves)::value><<<grid, block, 0, stream>>>(
            N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, colsums);
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if constexpr (BN <= 128) {                   // (wider ones are not for so few blocks)
        if (in_halves(N, D_in, D_out)) {
            if constexpr (!MASKED) {
                if (keep_sign) return go(yes, yes);
            }
            return go(no, yes);
        }
    }
    if constexpr (!MASKED) {
        if (keep_sign) return go(yes, no);
    }
    go(no, no);
}

template <bool MASKED>
void launch_few_rows(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh, const float* W,
                     const float* b, bool relu, float* Z, int64_t ldz, const float* mask, int64_t ldm,
                     float* colsums, hipStream_t stream)
{
    const int r = relu ? 1 : 0;
    const unsigned gx = (unsigned)((N + 31) / 32);
    const int64_t tiles = gx * ((D_out + 31) / 32);
    const bool many = tiles > 256;
    if (D_out >= 4 && (many ? D_in >= kStagedMany && tiles <= kStagedMost : tiles * D_in >= kStagedWork)) {
        const dim3 grid(gx, (unsigned)((D_out + 31) / 32));
        if (many) transform_few_staged_kernel<MASKED, false><<<grid, dim3(1024), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, colsums);
        else      transform_few_staged_kernel<MASKED, true><<<grid, dim3(1024), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, colsums);
        return;
    }
    // 32-column tiles when 64-column ones would not give every compute unit a workgroup
    if (D_out <= 32 || (int64_t)gx * ((D_out + 63) / 64) < 256) {
        dim3 grid(gx, (unsigned)((D_out + 31) / 32));
        transform_few_rows_kernel<1, MASKED><<<grid, dim3(512), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, colsums);
    } else {
        dim3 grid(gx, (unsigned)((D_out + 63) / 64));
        transform_few_rows_kernel<2, MASKED><<<grid, dim3(512), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, colsums);
    }
}

template <bool MASKED>
void launch_by_width(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh, const float* W,
                     const float* b, bool relu, float* Z, int64_t ldz, const float* mask, int64_t ldm, bool keep_sign,
                     float* colsums, hipStream_t stream)
{
    if (takes_few_rows(N, D_out)) {
        launch_few_rows<MASKED>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, colsums, stream);
        return;
    }
    auto go = [&](auto width) {
        launch<decltype(width)::value, MASKED>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, keep_sign, colsums, stream);
    };
    const int64_t bn = block_width_for(N, D_out);
    if (bn == 32)       go(std::integral_constant<int, 32>{});
    else if (bn == 64)  go(std::integral_constant<int, 64>{});
    else if (bn == 128) go(std::integral_constant<int, 128>{});
    else if (bn == 192) go(std::integral_constant<int, 192>{});
    else                go(std::integral_constant<int, 256>{});
}

}  // namespace

int64_t transform_row_blocks(int64_t N, int64_t D_out) { return takes_few_rows(N, D_out) ? (N + 31) / 32 : (N + 127) / 128; }

int launch_transform(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh,
                     const float* W, const float* b, bool relu, float* Z, int64_t ldz,
                     hipStream_t stream, const float* mask, int64_t ldm, bool keep_sign, float* colsums)
{
    if (N == 0 || D_out == 0) return RETEXO_OK;
    if (D_in == 0) {
        const int64_t blocks = (N * D_out + 255) / 256;
        bias_rows_kernel<<<dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, stream>>>(
            N, (int)D_out, b, relu ? 1 : 0, Z, ldz, mask, ldm);
        return hipGetLastError() != hipSuccess ? RETEXO_E_HIP : RETEXO_OK;
    }
    if (mask) launch_by_width<true>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, keep_sign, colsums, stream);
    else      launch_by_width<false>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, keep_sign, colsums, stream);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
