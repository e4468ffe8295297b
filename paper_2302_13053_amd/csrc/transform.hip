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
// eight waves, one workgroup per CU (212 registers, 75 KB of LDS), narrower ones
// four waves and two to four workgroups.  W is split by every workgroup again: the
// call has no scratch memory to keep its parts in.
//
// What bounds the wide tiles is power and the change between loading and storing:
// the matrix instructions run at a clock of about 1.5 GHz (GRBM_GUI_ACTIVE), the
// same launch on zeros is 25 % faster, and a bf16 library product of 8192^3
// reaches 1210-1270 TFLOP/s where this kernel issues 900-1000.  Measured (float32
// instructions before): 2,449,029 x 256 -> 256 2.15 ms = 149 TFLOP/s (2.60 ms),
// 232,965 x 1204 -> 256 0.87 ms = 166 (1.28), 2,449,029 x 256 -> 188 1.74 ms (1.98),
// 232,965 x 512 -> 41 0.137 ms = 3.8 TB/s (0.171), 100,000 x 512 -> 128 94 us (150).
//
// Sources are clamped instead of checked (rows past the end repeat the last
// row, columns past D_out the last column), so the loop carries no selects;
// only a partial last K tile takes a checked form.  Loads are four bytes wide
// (W) or 16 bytes at any float's address (H), so every alignment and leading
// dimension takes this kernel, in one order of arithmetic.  Bias and ReLU are
// applied to the accumulators on the way out: through this wave's piece of the
// dead tiles in LDS and from there as 16-byte pieces of rows where the output
// allows it, otherwise through one pointer per 32x32 tile that walks down the
// rows.  Matrices of few rows take the few-rows kernel at the end (K split over
// the waves of a workgroup).
#include "common.hpp"
#include "tiles.hpp"

#include <type_traits>

namespace {

// Bias, ReLU, optional mask and store of the accumulators of one wave.
// Accumulator element r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32 of its tile.
// Only the last row block of the matrix checks rows.
template <int TN, bool MASKED>
__device__ __forceinline__ void write_out(const f32x16 (&acc)[TN], const float (&bv)[TN], int64_t N, int D_out,
                                          int64_t row_base, int col_base, int lane, int relu,
                                          float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm,
                                          bool whole_block)
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
            float mv[16];
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
                if constexpr (MASKED) x = mv[r] > 0.0f ? x : 0.0f;
                if (FULL || row0 + ro < N) p[ro * ldz] = x;
            }
        }
    };
    if (whole_block) run(std::true_type{});
    else run(std::false_type{});
}

// The same epilogue for outputs whose rows allow 16-byte stores (Z and the mask 16-byte aligned, ldz, ldm and
// D_out multiples of four): each 32 x CW block of results goes through this wave's own piece of LDS (T, 32 rows
// of CW + 4 floats; the K loop's tiles are dead by then) and leaves as whole 16-byte pieces of rows, four times
// fewer store instructions, each covering full cache lines.  Same values as write_out.
template <int TN, int CW, bool MASKED>
__device__ __forceinline__ void write_out_rows(const f32x16 (&acc)[TN], const float (&bv)[TN], int64_t N, int D_out,
                                               int64_t row_base, int col_base, int lane, int relu,
                                               float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm,
                                               float* __restrict__ T)
{
    constexpr int P = CW + 4;            // LDS pitch: rows stay 16-byte aligned, column reads spread over the banks
    constexpr int JT = CW / 32;          // accumulator tiles per pass
    constexpr int LPR = CW / 4;          // lanes that cover one row of the pass
    constexpr int RPI = 64 / LPR;        // rows per store instruction
    static_assert(TN % JT == 0, "passes cover whole tiles");
    const int lrow = lane & 31, lk = lane >> 5;
    const int c4 = (lane % LPR) * 4, rsub = lane / LPR;
#pragma unroll
    for (int j0 = 0; j0 < TN; j0 += JT) {
#pragma unroll
        for (int jj = 0; jj < JT; ++jj)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ro = 8 * (r / 4) + (r % 4) + 4 * lk;
                float x = acc[j0 + jj][r] + bv[j0 + jj];
                if (relu) x = fmaxf(x, 0.0f);
                T[ro * P + jj * 32 + lrow] = x;
            }
        const int col = col_base + j0 * 32 + c4;
#pragma unroll
        for (int s = 0; s < 32 / RPI; ++s) {
            const int rr = s * RPI + rsub;
            f32x4 v = *reinterpret_cast<const f32x4*>(&T[rr * P + c4]);
            const int64_t row = row_base + rr;
            if (row < N && col < D_out) {
                if constexpr (MASKED) {
                    const f32x4 m = *reinterpret_cast<const f32x4*>(mask + row * ldm + col);
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = m[q] > 0.0f ? v[q] : 0.0f;
                }
                *reinterpret_cast<f32x4*>(Z + row * ldz + col) = v;
            }
        }
    }
}

// The block kernel: 128 x BN outputs per workgroup, 32 rows and up to 128 columns per wave (whose two running sums then
// take 128 registers): four waves, or eight for the tiles wider than 128; any alignment and leading dimension.
// ZVEC: the output (and the mask) allow 16-byte stores, see write_out_rows.
template <int BN> constexpr int transform_waves = BN > 128 ? 8 : 4;
template <int BN, bool MASKED, bool ZVEC>
__global__ __launch_bounds__(64 * transform_waves<BN>, BN <= 32 ? 4 : BN <= 64 ? 3 : 2) void transform_kernel(
    int64_t N, int D_in, int D_out, const float* __restrict__ H, int64_t ldh,
    const float* __restrict__ W, const float* __restrict__ bias, int relu,
    float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm, int keep_sign)
{
    constexpr int BM = 128, WAVES = transform_waves<BN>, WN = BN / (WAVES / 4), TN = WN / 32;
    using T = SplitTile<BM, BN>;
    using WStage = KMajorStage<BN, WAVES>;
    constexpr int HW = BM * kTileK / (64 * WAVES);       // floats of H a thread stages
    // row-wise epilogue: 64 columns per pass where the tiles leave room for every wave's 32 x 68 block, else 32
    constexpr int CW = (TN % 2 == 0 && 2 * T::units * 4 >= WAVES * 32 * 68) ? 64 : 32;
    static_assert(2 * T::units * 4 >= WAVES * 32 * (CW + 4), "the epilogue's blocks fit in the tiles' memory");
    __shared__ u32x4 lds[2 * T::units];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int a0 = wave % 4 * 32, b0 = wave / 4 * WN;    // the wave's rows and columns of the tile
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    const int lrow = lane & 31, lk = lane >> 5;

    f32x16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

    // H: a thread stages HW consecutive k of one row (rows past the end repeat the last one, never stored)
    const int hr = tid / (kTileK / HW), hk = tid % (kTileK / HW) * HW;
    const float* ph = H + (m0 + hr < N ? m0 + hr : N - 1) * ldh;
    float ra[HW];
    auto fetch_h = [&](int kt) {
        const int k = kt * kTileK + hk;
        if ((kt + 1) * kTileK <= D_in) {
#pragma unroll
            for (int v = 0; v < HW / 4; ++v) {
                const f32x4 t = *reinterpret_cast<const f32x4_any*>(ph + k + 4 * v);
#pragma unroll
                for (int q = 0; q < 4; ++q) ra[4 * v + q] = t[q];
            }
        } else {
#pragma unroll
            for (int q = 0; q < HW; ++q) ra[q] = k + q < D_in ? ph[k + q] : 0.0f;
        }
    };
    WStage sw;
    sw.init(W, D_out, 0, D_in, n0, D_out, wave, lane);

    float bv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + b0 + j * 32 + lrow;
        bv[j] = (bias && col < D_out) ? bias[col] : 0.0f;
    }

    const int nk = (D_in + kTileK - 1) / kTileK;
    constexpr int A_MICROS = HW / 2 + 2, MICROS = A_MICROS + WStage::count * WStage::steps;
    typedef uint32_t part_t __attribute__((ext_vector_type(HW / 2)));
    part_t part_h[3];
    auto micro = [&](auto step, int buf, int kt) {
        constexpr int m = decltype(step)::value;
        u32x4* base = lds + buf * T::units;
        if constexpr (m >= A_MICROS) {
            sw.template micro<m - A_MICROS>(base, [](int s, int half, int c) { return T::b(s, half, c); }, 0u, kt + 1 < nk, kt + 1);
        } else if constexpr (m < HW / 2) {
            split_pair(ra[2 * m], ra[2 * m + 1], m, part_h);
        } else if constexpr (m == HW / 2) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
                *reinterpret_cast<part_t*>(reinterpret_cast<char*>(base + T::a(s, hk >> 3, hr)) + (hk & 7) * 2) = part_h[s];
        } else {
            if (kt + 1 < nk) fetch_h(kt + 1);
        }
    };
    fetch_h(0);
    each<WStage::count>([&](auto i) { sw.template fetch<decltype(i)::value>(0); });
    each<MICROS>([&](auto m) { micro(m, 0, 0); });
    __syncthreads();
    split_k_loop<TN, BM, BN, MICROS>(acc, lds, nk, a0, b0, lane, micro);

    // how close to zero a sum is decided by the float32 instruction: 2^-18 of the wave's largest one, twenty times what
    // the two were seen apart
    float near = 0.0f;
    if (keep_sign) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) near = fmaxf(near, __builtin_fabsf(acc[j][r]));
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) near = fmaxf(near, __shfl_xor(near, m, 64));
        near *= 0x1p-18f;
    }
    each<TN>([&](auto at) {
        constexpr int j = decltype(at)::value;
        if (!redo_tile(acc[j], bv[j], near)) return;
        // the tile once more with the float32 instruction, operands straight from memory, k in ascending pairs
        const int64_t row = m0 + a0 + lrow;
        const int col = n0 + b0 + j * 32 + lrow;
        const float* hp = H + (row < N ? row : N - 1) * ldh;
        const float* wp = W + (col < D_out ? col : D_out - 1);
        f32x16 x;
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = 0.0f;
        constexpr int U = 8;
        for (int k0 = 0; k0 < D_in; k0 += 2 * U) {
            float a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + 2 * u + lk;
                const bool in = k < D_in;
                const float av = hp[in ? k : 0], bw = wp[(int64_t)(in ? k : 0) * D_out];
                a[u] = in ? av : 0.0f;
                b[u] = in ? bw : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) x = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], b[u], x, 0, 0, 0);
        }
        acc[j] = x;
    });

    if constexpr (ZVEC) {
        __syncthreads();                      // every wave is done with the last tile
        write_out_rows<TN, CW, MASKED>(acc, bv, N, D_out, m0 + a0, n0 + b0, lane, relu, Z, ldz, mask, ldm,
                                       reinterpret_cast<float*>(lds) + wave * 32 * (CW + 4));
    } else {
        write_out<TN, MASKED>(acc, bv, N, D_out, m0 + a0, n0 + b0, lane, relu, Z, ldz, mask, ldm, m0 + BM <= N);
    }
}

// Few rows: a matrix with so few 128-row blocks that they would leave most compute units idle (a citation
// graph's 2,708 x 2,866 features give 22) is cut into 32-row blocks, and the K extent of each block is cut
// over the eight waves of its workgroup.  A wave needs no LDS and no barrier in its loop: per group of 8 k it
// fetches its operands straight into the MFMA layout — lane l holds k = 4 (l / 32) .. + 3 of row l % 32, so
// MFMA q of the group pairs k = q (lower half-wave) with k = 4 + q (upper half-wave) — four groups at a time,
// the next four in flight behind the MFMAs.  The eight partial tiles are then added in a fixed order (wave w + wave w + 4 in registers, then
// ((0 + 1) + 2) + 3 through LDS), so the result is reproducible; it differs from the block kernels' only in
// the order of the fp32 additions.
template <int TN, bool HV, bool MASKED>
__global__ __launch_bounds__(512) void transform_few_rows_kernel(
    int64_t N, int D_in, int D_out, const float* __restrict__ H, int64_t ldh,
    const float* __restrict__ W, const float* __restrict__ bias, int relu,
    float* __restrict__ Z, int64_t ldz, const float* __restrict__ mask, int64_t ldm)
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
    // of memory latencies; the batch is what keeps enough bytes in flight)
    constexpr int U = 4;
    float a[2][U][4], b[2][U][TN][4];
    auto wanted_of = [&](int g) {                // how many of this lane's four k of group g are data
        const int left = g < g1 ? D_in - (g * 8 + lk * 4) : 0;
        return left < 0 ? 0 : (left < 4 ? left : 4);
    };
    auto fetch = [&](int gb, int slot) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (gb + u) * 8 + lk * 4;
            const int wanted = wanted_of(gb + u);
            load4<HV>(hp, k, wanted, a[slot][u]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float* wr = W + (int64_t)(q < wanted ? k + q : 0) * D_out;
#pragma unroll
                for (int j = 0; j < TN; ++j) b[slot][u][j][q] = wr[col[j]];
            }
        }
    };
    auto zero = [&](int gb, int slot) {          // what is not data was fetched from k = 0: replace it
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int wanted = wanted_of(gb + u);
            zero4<HV>(wanted, a[slot][u]);
#pragma unroll
            for (int j = 0; j < TN; ++j) zero4<false>(wanted, b[slot][u][j]);
        }
    };

    auto batch = [&](int gb, auto slot_tag) {    // slot as a type: register arrays want constant indices
        constexpr int cur = decltype(slot_tag)::value;
        if (gb + U < g1) fetch(gb + U, cur ^ 1);
        RETEXO_SCHED_FENCE();
        zero(gb, cur);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][u][q], b[cur][u][j][q], acc[j], 0, 0, 0);
    };
    if (g0 < g1) fetch(g0, 0);
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

template <int BN, bool MASKED>
void launch(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh, const float* W,
            const float* b, bool relu, float* Z, int64_t ldz, const float* mask, int64_t ldm, bool keep_sign,
            hipStream_t stream)
{
    const dim3 grid((unsigned)((N + 127) / 128), (unsigned)((D_out + BN - 1) / BN)), block(64 * transform_waves<BN>);
    const int r = relu ? 1 : 0, ks = keep_sign ? 1 : 0;
    const bool zv = (uintptr_t)Z % 16 == 0 && ldz % 4 == 0 && D_out % 4 == 0 &&
                    (!MASKED || ((uintptr_t)mask % 16 == 0 && ldm % 4 == 0));
    if (zv) transform_kernel<BN, MASKED, true><<<grid, block, 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, ks);
    else    transform_kernel<BN, MASKED, false><<<grid, block, 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm, ks);
}

template <bool MASKED>
void launch_few_rows(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh, const float* W,
                     const float* b, bool relu, float* Z, int64_t ldz, const float* mask, int64_t ldm,
                     hipStream_t stream)
{
    const bool hv = (uintptr_t)H % 16 == 0 && ldh % 4 == 0 && D_in % 4 == 0;
    const int r = relu ? 1 : 0;
    const unsigned gx = (unsigned)((N + 31) / 32);
    // 32-column tiles when 64-column ones would not give every compute unit a workgroup
    if (D_out <= 32 || (int64_t)gx * ((D_out + 63) / 64) < 256) {
        dim3 grid(gx, (unsigned)((D_out + 31) / 32));
        if (hv) transform_few_rows_kernel<1, true, MASKED><<<grid, dim3(512), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm);
        else    transform_few_rows_kernel<1, false, MASKED><<<grid, dim3(512), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm);
    } else {
        dim3 grid(gx, (unsigned)((D_out + 63) / 64));
        if (hv) transform_few_rows_kernel<2, true, MASKED><<<grid, dim3(512), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm);
        else    transform_few_rows_kernel<2, false, MASKED><<<grid, dim3(512), 0, stream>>>(N, (int)D_in, (int)D_out, H, ldh, W, b, r, Z, ldz, mask, ldm);
    }
}

// Fewer 128-row blocks (times the column blocks) than the "transform_few_blocks" setting, 128 unless changed:
// the few-rows kernel.  The choice depends on the shape only, never on alignment, so one shape always takes
// one order of additions.

template <bool MASKED>
void launch_by_width(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh, const float* W,
                     const float* b, bool relu, float* Z, int64_t ldz, const float* mask, int64_t ldm, bool keep_sign,
                     hipStream_t stream)
{
    const int64_t bn = D_out <= 32 ? 32 : D_out <= 64 ? 64 : D_out <= 128 ? 128 : D_out <= 192 ? 192 : 256;
    if ((N + 127) / 128 * ((D_out + bn - 1) / bn) < agg_options().few_blocks) {
        launch_few_rows<MASKED>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, stream);
        return;
    }
    auto go = [&](auto width) {
        launch<decltype(width)::value, MASKED>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, keep_sign, stream);
    };
    if (bn == 32)       go(std::integral_constant<int, 32>{});
    else if (bn == 64)  go(std::integral_constant<int, 64>{});
    else if (bn == 128) go(std::integral_constant<int, 128>{});
    else if (bn == 192) go(std::integral_constant<int, 192>{});
    else                go(std::integral_constant<int, 256>{});
}

}  // namespace

int launch_transform(int64_t N, int64_t D_in, int64_t D_out, const float* H, int64_t ldh,
                     const float* W, const float* b, bool relu, float* Z, int64_t ldz,
                     hipStream_t stream, const float* mask, int64_t ldm, bool keep_sign)
{
    if (N == 0 || D_out == 0) return RETEXO_OK;
    if (D_in == 0) {
        const int64_t blocks = (N * D_out + 255) / 256;
        bias_rows_kernel<<<dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, stream>>>(
            N, (int)D_out, b, relu ? 1 : 0, Z, ldz, mask, ldm);
        return hipGetLastError() != hipSuccess ? RETEXO_E_HIP : RETEXO_OK;
    }
    if (mask) launch_by_width<true>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, keep_sign, stream);
    else      launch_by_width<false>(N, D_in, D_out, H, ldh, W, b, relu, Z, ldz, mask, ldm, keep_sign, stream);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
