// Local training of one layer: the work a worker does between two message
// passing rounds (section "Lazy Message Passing").  A layer f (fully connected
// + ReLU, Eq. 1) is trained by itself on its fixed aggregated inputs X with a
// temporary linear classification layer C on top (the appendix sizes C as
// H_m x H_K) and softmax cross-entropy over the labelled nodes; the last layer
// is the classification function itself (H == 0 here).
//
//      A      = ReLU(X W1 + b1)          transform kernel (float32 in three bf16 parts)
//      logits = A Wc + bc                transform kernel
//      dL     = (softmax(logits) - onehot(label)) / n_labelled, 0 for unlabelled nodes
//      gWc    = A^T dL,  gbc = colsum(dL)
//      dA     = (dL Wc^T) where A > 0    transform kernel with Wc^T and a ReLU mask
//      gW1    = X^T dA,  gb1 = colsum(dA)
//
// Bound by the matrix cores in large steps and by the number of dependent launches in small ones: nine of them, ten with
// the input gradient (2,708 x 2866 -> 64 -> 7 with eighteen of them 114 us, now 94).
//
// The two weight gradients are "TN" products whose contraction runs over the
// nodes (hundreds of thousands), with a small output.  wgrad_kernel splits the
// node range over many workgroups, each producing a partial [M, Nq] tile with
// the same split-bf16 tile loop as the transform, and a second kernel adds the
// partials in a fixed order: deterministic, and more accurate than one long
// fp32 accumulation.
#include "common.hpp"
#include "tiles.hpp"

namespace {

constexpr int kThreads = 256;

// ---------------------------------------------------------------------------
// part[z][m][n] = sum over k in chunk z of P[k][m] * Q[k][n]
// ---------------------------------------------------------------------------

// Both operands run along k, so both are staged by columns (KMajorStage) and multiplied by the split K loop shared
// with the dense transform; 128 x BN outputs per workgroup, 32 rows and up to 128 columns per wave, any alignment and
// leading dimension.
template <int BN> constexpr int wgrad_waves = BN > 128 ? 8 : 4;
template <int BN>
__global__ __launch_bounds__(64 * wgrad_waves<BN>, BN <= 32 ? 4 : BN <= 64 ? 3 : 2) void wgrad_kernel(
    int64_t K, int M, int Nq, const float* __restrict__ P, int64_t ldp,
    const float* __restrict__ Q, int64_t ldq, int64_t k_chunk, float* __restrict__ part)
{
    constexpr int BM = 128, WAVES = wgrad_waves<BN>, WN = BN / (WAVES / 4), TN = WN / 32;
    using T = SplitTile<BM, BN>;
    using PStage = KMajorStage<BM, WAVES>;               // (two tiles ahead: 500,000 x 256 -> 32 140 us instead of 136)
    using QStage = KMajorStage<BN, WAVES>;
    __shared__ u32x4 lds[2 * T::units];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int a0 = wave % 4 * 32, b0 = wave / 4 * WN;    // the wave's rows and columns of the tile
    const int lrow = lane & 31, lk = lane >> 5;
    const int m0 = blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    const int64_t k_begin = (int64_t)blockIdx.z * k_chunk;
    const int64_t k_end = min(K, k_begin + k_chunk);

    f32x16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

    // every other chunk is summed with its sign turned and turned back at the end: the matrix core's bf16 additions lean
    // to one side a little, and over the thousands of chunks of a large graph that would add up
    const bool turned = blockIdx.z & 1;
    const float scale_p = turned ? -kSplitScale : kSplitScale;
    const int nk = k_end > k_begin ? (int)((k_end - k_begin + kTileK - 1) / kTileK) : 0;
    if (nk > 0) {
        PStage sp;
        QStage sq;
        sp.init(P, ldp, k_begin, k_end, m0, M, wave, lane);
        sq.init(Q, ldq, k_begin, k_end, n0, Nq, wave, lane);
        constexpr int A_MICROS = PStage::count * PStage::steps;
        constexpr int MICROS = A_MICROS + QStage::count * QStage::steps;
        auto micro = [&](auto step, auto buf, int kt, auto edge_tag) {
            constexpr int m = decltype(step)::value;
            constexpr bool EDGE = decltype(edge_tag)::value;
            u32x4* base = lds + buf * T::units;
            if constexpr (m < A_MICROS)
                sp.template micro<m, 0, EDGE>(base, [](int s, int half, int c) { return T::a(s, half, c); }, scale_p, kt, nk);
            else
                sq.template micro<m - A_MICROS, 0, EDGE>(base, [](int s, int half, int c) { return T::b(s, half, c); }, kSplitScale, kt, nk);
        };
        each<PStage::count>([&](auto i) { sp.template fetch<decltype(i)::value, 0, true>(0); });
        each<QStage::count>([&](auto i) { sq.template fetch<decltype(i)::value, 0, true>(0); });
        each<MICROS>([&](auto m) { micro(m, std::integral_constant<int, 0>{}, 0, std::true_type{}); });
        __syncthreads();
        split_k_loop<TN, BM, BN, MICROS, 1>(acc, lds, nk, (int)((k_end - k_begin) / kTileK), a0, b0, lane, micro);
    }

    // accumulator element r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32 of its 32 x 32 tile
    float* out = part + (int64_t)blockIdx.z * M * Nq;
    const int row0 = m0 + a0 + 4 * lk;
    each<TN>([&](auto at) {
        constexpr int j = decltype(at)::value;
        const int col = n0 + b0 + j * 32 + lrow;
        float turn = turned ? -kSplitUnscale : kSplitUnscale;
        const float* pp = P + k_begin * ldp + min(m0 + a0 + lrow, M - 1);
        const float* qp = Q + k_begin * ldq + min(col, Nq - 1);
        if (k_end - k_begin == 1) {          // (a single product is rounded once by the float32 instruction)
            acc[j] = float32_tile<1>(pp, ldp, qp, ldq, 1, lane);
            turn = 1.0f;
        } else if (redo_tile(acc[j])) {
            acc[j] = float32_tile<BN <= 64 ? 8 : 16>(pp, ldp, qp, ldq, (int)(k_end - k_begin), lane);
            turn = 1.0f;
        }
        if (col >= Nq) return;
        float* p = out + (int64_t)row0 * Nq + col;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ro = 8 * (r / 4) + (r % 4);
            if (row0 + ro < M) p[(int64_t)ro * Nq] = turn * acc[j][r];
        }
    });
}

// out[i] = sum_z part[z][i], i < total.  A workgroup owns 64 outputs; its four waves each add a quarter of the z
// range with four running sums (z mod 4), and the sixteen sums of an output are combined in a fixed order: the
// result does not depend on the launch, and with few outputs and hundreds of partials (a classifier's gradient) the
// additions do not wait for one load at a time.
__device__ __forceinline__ void reduce_partials(int64_t block, int S, int64_t total, const float* __restrict__ part,
                                                float* __restrict__ out, float* sh)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = block * 64 + lane;
    float s = 0.0f;
    if (i < total) {
        const int per = (S + 3) / 4;
        const int z0 = wave * per, z1 = min(S, z0 + per);
        const float* p = part + i;
        float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        int z = z0;
        for (; z + 4 <= z1; z += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] += p[(int64_t)(z + k) * total];
        }
        for (int k = 0; z < z1; ++z, ++k) q[k] += p[(int64_t)z * total];
        s = (q[0] + q[1]) + (q[2] + q[3]);
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    if (wave == 0 && i < total) out[i] = (sh[lane] + sh[64 + lane]) + (sh[128 + lane] + sh[192 + lane]);
}

constexpr int kCountBlocks = 64;         // workgroups that count labelled nodes; a wave adds their counts up
struct TrainHeader {
    int32_t labelled[kCountBlocks];
};

__device__ __forceinline__ int labelled_nodes(const TrainHeader* hdr)
{
    int n = hdr->labelled[threadIdx.x & 63];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) n += __shfl_xor(n, m, 64);
    return n;
}

// out [Cp, R] = scale * transpose of in [R, Cn], rows Cn..Cp of out zero
struct Transpose {
    int R, Cn, Cp;
    const float* in;
    float* out;
    float scale;
};

// What a step needs before its products, in one launch: the first kCountBlocks workgroups count labelled nodes, the next
// `a_blocks` transpose the classifier's weights for the way back, the others the first layer's for the input gradient.
// (Clearing, counting and transposing were four launches of 2 to 12 us, two of them in front of the first product.)
__global__ __launch_bounds__(kThreads) void prepare_kernel(int64_t N, const int32_t* __restrict__ labels,
                                                           TrainHeader* hdr, unsigned a_blocks, Transpose a, Transpose b)
{
    __shared__ int sh[kThreads / 64];
    if (blockIdx.x < kCountBlocks) {
        int cnt = 0;
        constexpr int64_t step = (int64_t)kCountBlocks * kThreads;
        int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x;
        for (; v + 7 * step < N; v += 8 * step) {
            int y[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) y[k] = labels[v + k * step];
#pragma unroll
            for (int k = 0; k < 8; ++k) cnt += y[k] >= 0;
        }
        for (; v < N; v += step) cnt += labels[v] >= 0;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) cnt += __shfl_xor(cnt, m, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) hdr->labelled[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
        return;
    }
    const unsigned block = blockIdx.x - kCountBlocks;
    const bool first = block < a_blocks;
    const Transpose t = first ? a : b;
    const int64_t i = (int64_t)(first ? block : block - a_blocks) * kThreads + threadIdx.x;
    if (i >= (int64_t)t.R * t.Cp) return;
    const int c = (int)(i / t.R), r = (int)(i % t.R);
    t.out[i] = c < t.Cn ? t.scale * t.in[(int64_t)r * t.Cn + c] : 0.0f;
}

__device__ __forceinline__ float wmax(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
    return x;
}
__device__ __forceinline__ float wsum(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// f over the values of sixteen lanes, the same in each of them
template <class F>
__device__ __forceinline__ float fold16(float x, F&& f)
{
    auto with = [&](auto ctrl) {
        x = f(x, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true)));
    };
    with(std::integral_constant<int, 0xb1>{});           // lane ^ 1
    with(std::integral_constant<int, 0x4e>{});           // lane ^ 2
    with(std::integral_constant<int, 0x141>{});          // the other four of eight (mirrored)
    with(std::integral_constant<int, 0x140>{});          // the other eight of sixteen
    return x;
}

// Nodes per workgroup of the loss kernel: sixteen at a time (4 per wave), up to eight times where that leaves 2,048
// workgroups, which is what the chip holds: there are as many partial sums of the loss and the columns to add up.
constexpr int kXentRows = 16;
int xent_turns(int64_t N, bool narrow)
{
    const int64_t t = N / (kXentRows * 2048);
    return !narrow || t < 1 ? 1 : t > 8 ? 8 : (int)t;
}
bool xent_narrow(int64_t ldc) { return ldc <= 64; }
int64_t xent_blocks(int64_t N, int64_t ldc)
{
    const int64_t rows = kXentRows * xent_turns(N, xent_narrow(ldc));
    return (N + rows - 1) / rows;
}

// L[v, 0:C] holds the logits on entry and d loss / d logits on exit (zero for unlabelled nodes and in the padding
// columns C..ld).  Per-workgroup loss sums go to loss_part[blockIdx.x] (unscaled).
// A wave takes four nodes.  Where a row fits sixteen lanes of four columns (NARROW: ld <= 64) all four at once: bound by the
// instructions of a row, of which the reductions are one set for four rows then, and so are the logarithms.  (One row over
// the wave's lanes, 190 instructions each: 232,965 x 41 62 us, 35 now, 58 with the logarithms alone in common; the streaming
// of L takes 25.  2,708 x 7: 5 us, 4 now.)  These rows' column sums, which the bias gradient is made of, go to
// col_part[blockIdx.x][0:C] on the way: in a pass of their own 10 us.
template <bool NARROW>
__global__ __launch_bounds__(kThreads) void softmax_xent_kernel(
    int64_t N, int C, float* __restrict__ L, int64_t ld, const int32_t* __restrict__ labels,
    const TrainHeader* hdr, float* __restrict__ loss_part, int turns, float* __restrict__ col_part)
{
    __shared__ float wl[4];
    __shared__ __attribute__((aligned(16))) float wc[16][64];
    constexpr int R = kXentRows / 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nl = labelled_nodes(hdr);
    const float inv = nl > 0 ? 1.0f / (float)nl : 0.0f;
    const int64_t first = (int64_t)blockIdx.x * kXentRows * turns + wave * R;
    float loss = 0.0f;
    // s: the softmax denominator; so: its part from the classes other than the label.  The label's
    // gradient p_y - 1 is formed as -so / s: for a confidently classified node p_y is close to one and
    // the subtraction would leave only a few correct digits of what is then the whole gradient.
    if constexpr (NARROW) {
        // sixteen lanes per row, four columns per lane (rows of the workspace start on 128-byte lines)
        const int c0 = lane % 16 * 4;
        float column[4] = {};
        f32x4 next = {};
        int next_y = -1;
        auto fetch = [&](int64_t v) {
            v = v < N ? v : N - 1;
            next_y = labels[v];
            if (c0 < ld) next = *reinterpret_cast<const f32x4*>(L + v * ld + c0);
        };
        auto larger = [](float a, float b) { return fmaxf(a, b); };
        auto plus = [](float a, float b) { return a + b; };
        const int64_t mine = first + lane / 16;
        fetch(mine);
        for (int t = 0; t < turns; ++t) {
            const int64_t v = mine + (int64_t)t * kXentRows;
            const int y = next_y;
            float x[4], e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = c0 + k < C ? next[k] : -INFINITY;
            if (t + 1 < turns) fetch(v + kXentRows);
            const float m = fold16(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), larger);
            float at = 0.0f, ey = 0.0f, rest[4];         // logit and exponential of the label, the others' exponentials
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                e[k] = c0 + k < C ? expf(x[k] - m) : 0.0f;
                const bool label = c0 + k == y && c0 + k < C;
                at = label ? x[k] : at;
                ey = label ? e[k] : ey;
                rest[k] = label ? 0.0f : e[k];
            }
            at = fold16(at, plus);                       // (one term that is not zero)
            ey = fold16(ey, plus);
            const float so = fold16((rest[0] + rest[1]) + (rest[2] + rest[3]), plus);
            const float s = so + ey;
            const float off = so / s;                    // 1 - p_y
            const float scale = y >= 0 ? inv : 0.0f;
            f32x4 g;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                g[k] = c0 + k < C ? (c0 + k == y ? -off : e[k] / s) * scale : 0.0f;
                column[k] += v < N ? g[k] : 0.0f;
            }
            if (v < N && c0 < ld) *reinterpret_cast<f32x4*>(L + v * ld + c0) = g;
            if (v < N && y >= 0 && y < C) loss += off <= 0.5f ? -log1pf(-off) : -(at - m - logf(s));
        }
        *reinterpret_cast<f32x4*>(&wc[wave * 4 + lane / 16][c0]) = f32x4{column[0], column[1], column[2], column[3]};
        loss = (__shfl(loss, 0, 64) + __shfl(loss, 16, 64)) + (__shfl(loss, 32, 64) + __shfl(loss, 48, 64));
    } else {
        for (int r = 0; r < R; ++r) {
            const int64_t v = first + r;
            if (v >= N) break;
            float* row = L + v * ld;
            const int y = labels[v];
            const float scale = y >= 0 ? inv : 0.0f;
            float m = -INFINITY;
            for (int j = lane; j < C; j += 64) m = fmaxf(m, row[j]);
            m = wmax(m);
            float s = 0.0f, so = 0.0f;
            for (int j = lane; j < C; j += 64) {
                const float e = expf(row[j] - m);
                s += e;
                so += j == y ? 0.0f : e;
            }
            s = wsum(s);
            so = wsum(so);
            const float rest = so / s;                 // 1 - p_y
            if (y >= 0 && y < C) loss += rest <= 0.5f ? -log1pf(-rest) : -(row[y] - m - logf(s));
            for (int j = lane; j < ld; j += 64) {
                float g = 0.0f;
                if (j < C) g = (j == y ? -rest : expf(row[j] - m) / s) * scale;
                row[j] = g;
            }
        }
    }
    if (lane == 0) wl[wave] = loss;
    __syncthreads();
    if (threadIdx.x == 0) loss_part[blockIdx.x] = (wl[0] + wl[1]) + (wl[2] + wl[3]);
    if (NARROW && wave == 0 && lane < C) {
        float t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = (wc[4 * k][lane] + wc[4 * k + 1][lane]) + (wc[4 * k + 2][lane] + wc[4 * k + 3][lane]);
        col_part[(int64_t)blockIdx.x * C + lane] = (t[0] + t[1]) + (t[2] + t[3]);
    }
}

// The sum of part[0], part[stride], ..: eight loads at a time, then the threads pairwise in a fixed order.  In 64 bits: the
// last additions, between sums that have grown large, are the ones whose rounding shows (232,965 x 7 bias gradient 4.8e-8
// off the same in 64 bits with 1,820 partial sums of 128 rows, 6.0e-8 with 2,081 of 112 in float32).
__device__ __forceinline__ double block_sum(int64_t n, const float* __restrict__ part, int64_t stride, double* sh)
{
    double s = 0.0;
    int64_t i = threadIdx.x;
    for (; i + 7 * kThreads < n; i += 8 * kThreads) {
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = part[(i + k * kThreads) * stride];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += x[k];
    }
    for (; i < n; i += kThreads) s += part[i * stride];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    return sh[0];
}

// The last additions of a layer's gradients, in one launch: workgroup 0 the loss (if there is one to form), then one per
// column of the bias gradient, then the weight gradient's (see reduce_partials).  Launches of a few microseconds of work
// each, they took a third of a small step one after the other.
struct Finish {
    int S;                        // weight gradient: partial products, their size, and where they are
    int64_t total;
    const float* part;
    float* gW;
    int64_t B;                    // bias gradient: partial sums per column, columns (0: none)
    int C;
    const float* colpart;
    float* gb;
    int64_t n_loss;               // loss: partial sums
    const float* losspart;
    const TrainHeader* hdr;
    float* loss;                  // or NULL
};
__global__ __launch_bounds__(kThreads) void finish_kernel(Finish f)
{
    __shared__ double sh[kThreads];
    int64_t block = blockIdx.x;
    if (f.loss) {
        if (block == 0) {
            const int nl = labelled_nodes(f.hdr);
            const double s = block_sum(f.n_loss, f.losspart, 1, sh);
            if (threadIdx.x == 0) *f.loss = nl > 0 ? (float)(s / nl) : 0.0f;
            return;
        }
        --block;
    }
    if (block < f.C) {
        const double s = block_sum(f.B, f.colpart + block, f.C, sh);
        if (threadIdx.x == 0) f.gb[block] = (float)s;
        return;
    }
    reduce_partials(block - f.C, f.S, f.total, f.part, f.gW, reinterpret_cast<float*>(sh));
}

// Column sums of what no kernel here has just written.  A workgroup takes kColRows rows; its four
// waves stride the rows, lanes stride the columns, every wave keeps four running sums (four loads in
// flight) that are combined in a fixed order, and the waves are added in order through LDS.
// finish_kernel adds the workgroups' results.
constexpr int kColRows = 128;

__global__ __launch_bounds__(kThreads) void colsum_kernel(int64_t N, int C, const float* __restrict__ D, int64_t ld,
                                                          float* __restrict__ part)
{
    __shared__ float sh[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * kColRows, r1 = min(N, r0 + kColRows);
    for (int c0 = 0; c0 < C; c0 += 64) {
        const int c = c0 + lane;
        float s = 0.0f;
        if (c < C) {
            float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            int64_t r = r0 + wave;
            for (; r + 12 < r1; r += 16) {
#pragma unroll
                for (int k = 0; k < 4; ++k) q[k] += D[(r + 4 * k) * ld + c];
            }
            for (int k = 0; r < r1; r += 4, ++k) q[k] += D[r * ld + c];
            s = (q[0] + q[1]) + (q[2] + q[3]);
        }
        sh[wave][lane] = s;
        __syncthreads();
        if (wave == 0 && c < C)
            part[(int64_t)blockIdx.x * C + c] = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Dropout on the hidden units (the appendix on hyper-parameters trains with dropout; it is taken on the
// layer's output, in front of the temporary classifier).  The mask is not stored: unit j of node v is
// dropped in draw number `draw` of stream `seed` when word j % 4 of the Philox-4x32-10 block
//      counter = (v, j / 4, draw low, draw high),  key = (seed low, seed high)
// (Salmon, Moraes, Dror, Shaw, SC 2011) is below floor(p * 2^32), so any caller can re-draw it.
// Kept units are scaled by 1 / (1 - p).  The backward pass needs no second draw: a unit of the stored
// activations is positive exactly when it was active and kept.
// ---------------------------------------------------------------------------
struct PhiloxWords { uint32_t w0, w1, w2, w3; };

__device__ __forceinline__ PhiloxWords philox_4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                      uint32_t k0, uint32_t k1)
{
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;      // multipliers of words 0 and 2
    constexpr uint32_t kKeyA = 0x9E3779B9u, kKeyB = 0xBB67AE85u;      // key increments per round
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hiA = __umulhi(kMulA, c0), loA = kMulA * c0;
        const uint32_t hiB = __umulhi(kMulB, c2), loB = kMulB * c2;
        c0 = hiB ^ c1 ^ k0;
        c2 = hiA ^ c3 ^ k1;
        c1 = loB;
        c3 = loA;
        k0 += kKeyA;
        k1 += kKeyB;
    }
    return {c0, c1, c2, c3};
}

__global__ __launch_bounds__(kThreads) void dropout_kernel(int64_t N, int H, float* __restrict__ A, int64_t ld,
                                                           uint32_t threshold, float scale, uint32_t seed_lo,
                                                           uint32_t seed_hi, uint32_t draw_lo, uint32_t draw_hi)
{
    const int Q = (H + 3) / 4;
    const int64_t total = N * Q;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total; i += (int64_t)gridDim.x * kThreads) {
        const int64_t v = i / Q;
        const int q = (int)(i % Q);
        const PhiloxWords w = philox_4x32_10((uint32_t)v, (uint32_t)q, draw_lo, draw_hi, seed_lo, seed_hi);
        float* p = A + v * ld + 4 * q;
        if (4 * q + 3 < H) {
            // rows of the workspace start on 128-byte lines
            f32x4 x = *reinterpret_cast<const f32x4*>(p);
            x.x = w.w0 >= threshold ? x.x * scale : 0.0f;
            x.y = w.w1 >= threshold ? x.y * scale : 0.0f;
            x.z = w.w2 >= threshold ? x.z * scale : 0.0f;
            x.w = w.w3 >= threshold ? x.w * scale : 0.0f;
            *reinterpret_cast<f32x4*>(p) = x;
        } else {
            const uint32_t ws[4] = {w.w0, w.w1, w.w2, w.w3};
            for (int k = 0; k < 4 && 4 * q + k < H; ++k) p[k] = ws[k] >= threshold ? p[k] * scale : 0.0f;
        }
    }
}

__global__ __launch_bounds__(kThreads) void sgd_kernel(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                                                       float lr)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) p[i] = p[i] - lr * g[i];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct Split { int S; int64_t k_chunk; };

Split choose_split(int64_t K, int64_t M, int64_t Nq, int bn)
{
    const int64_t tiles = ((M + 127) / 128) * ((Nq + bn - 1) / bn);
    // at most 1024 workgroups: four rounds of the 256 that the widest tile (eight waves) has room for, two of the 128-column
    // tile's 512 (one more workgroup would add a round for it alone)
    int64_t S = 1024 / tiles;
    const int64_t max_s = (K + 255) / 256;                  // at least 256 nodes per chunk
    if (S > max_s) S = max_s;
    if (S < 1) S = 1;
    int64_t chunk = (K + S - 1) / S;
    chunk = (chunk + kTileK - 1) / kTileK * kTileK;
    S = (K + chunk - 1) / chunk;
    if (S < 1) S = 1;
    return {(int)S, chunk};
}

int bn_for(int64_t Nq) { return Nq <= 32 ? 32 : Nq <= 64 ? 64 : Nq <= 128 ? 128 : 256; }

// f.gW[M][Nq] = P^T Q, and what else f asks for
void wgrad(int64_t K, int64_t M, int64_t Nq, const float* P, int64_t ldp, const float* Q, int64_t ldq, float* part,
           Finish f, hipStream_t stream)
{
    const int bn = bn_for(Nq);
    const Split sp = choose_split(K, M, Nq, bn);
    dim3 grid((unsigned)((M + 127) / 128), (unsigned)((Nq + bn - 1) / bn), (unsigned)sp.S);
    auto go = [&](auto width) {
        constexpr int BN = decltype(width)::value;
        wgrad_kernel<BN><<<grid, dim3(64 * wgrad_waves<BN>), 0, stream>>>(K, (int)M, (int)Nq, P, ldp, Q, ldq, sp.k_chunk, part);
    };
    if (bn == 32)       go(std::integral_constant<int, 32>{});
    else if (bn == 64)  go(std::integral_constant<int, 64>{});
    else if (bn == 128) go(std::integral_constant<int, 128>{});
    else                go(std::integral_constant<int, 256>{});
    f.S = sp.S;
    f.total = M * Nq;
    f.part = part;
    finish_kernel<<<dim3((unsigned)((f.loss ? 1 : 0) + f.C + (f.total + 63) / 64)), dim3(kThreads), 0, stream>>>(f);
}

int64_t colsum(int64_t N, int64_t C, const float* D, int64_t ld, float* part, hipStream_t stream)
{
    const int64_t B = (N + kColRows - 1) / kColRows;
    colsum_kernel<<<dim3((unsigned)B), dim3(kThreads), 0, stream>>>(N, (int)C, D, ld, part);
    return B;
}

struct TrainLayout {
    int64_t ldh, ldc;
    int64_t hdr, A, L, dA, WcT, W1T, part, colpart, losspart, total;
};

int64_t partial_floats(int64_t K, int64_t M, int64_t Nq)
{
    const Split sp = choose_split(K, M, Nq, bn_for(Nq));
    return (int64_t)sp.S * M * Nq;
}

TrainLayout make_layout(int64_t N, int64_t D_in, int64_t H, int64_t C)
{
    TrainLayout t;
    const int64_t n1 = N > 0 ? N : 1;
    t.ldh = align_up(H > 0 ? H : 1, 32);
    t.ldc = align_up(C > 0 ? C : 1, 32);
    int64_t off = 0;
    auto take = [&](int64_t floats) { const int64_t at = off; off += align_up(floats * 4, 256); return at; };
    static_assert(sizeof(TrainHeader) <= 256, "its place");
    t.hdr = off; off += 256;
    t.A = take(H > 0 ? n1 * t.ldh : 0);
    t.L = take(n1 * t.ldc);
    t.dA = take(H > 0 ? n1 * t.ldh : 0);
    t.WcT = take(H > 0 ? t.ldc * H : 0);
    t.W1T = take((H > 0 ? H : t.ldc) * D_in);            // transposed first-layer weights (input gradient)
    int64_t pf = 0;
    if (H > 0) {
        pf = partial_floats(N, D_in, t.ldh);
        const int64_t p2 = partial_floats(N, H, t.ldc);
        if (p2 > pf) pf = p2;
    } else {
        pf = partial_floats(N, D_in, t.ldc);
    }
    t.part = take(pf);
    // (of blocks of 32 rows or more behind a product, of the loss kernel's rows, or of kColRows rows)
    const int64_t cols = (n1 + 31) / 32 * t.ldh;
    const int64_t top = xent_narrow(t.ldc) ? xent_blocks(n1, t.ldc) * C : (n1 + kColRows - 1) / kColRows * t.ldc;
    t.colpart = take(cols > top ? cols : top);
    t.losspart = take(xent_blocks(n1, t.ldc));
    t.total = off;
    return t;
}

int check_sizes(int64_t N, int64_t D_in, int64_t H, int64_t C)
{
    if (N < 0 || D_in < 1 || H < 0 || C < 1) return RETEXO_E_SIZE;
    if (N >= (1ll << 31) || D_in >= (1 << 20) || H >= (1 << 20) || C >= (1 << 20)) return RETEXO_E_SIZE;
    return RETEXO_OK;
}

}  // namespace

extern "C" int64_t retexo_train_workspace_bytes(int64_t N, int64_t D_in, int64_t H, int64_t C)
{
    if (int s = check_sizes(N, D_in, H, C)) return s;
    return make_layout(N, D_in, H, C).total;
}

namespace {
int layer_grad_impl(int64_t N, int64_t D_in, int64_t H, int64_t C,
                    const float* d_X, int64_t ldx, const int32_t* d_labels,
                    const float* d_W1, const float* d_b1, const float* d_Wc, const float* d_bc,
                    float* d_gW1, float* d_gb1, float* d_gWc, float* d_gbc, float* d_loss,
                    float* d_gX, int64_t ldgx, float p_drop, uint64_t seed, uint64_t draw,
                    void* d_workspace, int64_t workspace_bytes, void* stream_)
{
    if (int s = check_sizes(N, D_in, H, C)) return s;
    if (!(p_drop >= 0.0f && p_drop < 1.0f)) return RETEXO_E_SIZE;
    if (p_drop > 0.0f && H == 0) return RETEXO_E_SIZE;        // there is no hidden unit to drop
    const float keep_scale = p_drop > 0.0f ? 1.0f / (1.0f - p_drop) : 1.0f;
    if (ldx < D_in) return RETEXO_E_LD;
    if (d_gX && ldgx < D_in) return RETEXO_E_LD;
    if (d_gX && N > 0 && d_X &&
        !((const char*)d_gX + (size_t)((N - 1) * ldgx + D_in) * 4 <= (const char*)d_X ||
          (const char*)d_X + (size_t)((N - 1) * ldx + D_in) * 4 <= (const char*)d_gX))
        return RETEXO_E_ALIAS;
    if (!d_W1 || !d_b1 || !d_gW1 || !d_gb1 || !d_loss) return RETEXO_E_NULL;
    if (N > 0 && (!d_X || !d_labels)) return RETEXO_E_NULL;
    if (H > 0 && (!d_Wc || !d_bc || !d_gWc || !d_gbc)) return RETEXO_E_NULL;
    const TrainLayout t = make_layout(N, D_in, H, C);
    if (!d_workspace || workspace_bytes < t.total || ((uintptr_t)d_workspace & 255)) return RETEXO_E_WORKSPACE;

    hipStream_t stream = (hipStream_t)stream_;
    char* ws = (char*)d_workspace;
    TrainHeader* hdr = (TrainHeader*)(ws + t.hdr);
    float* A = (float*)(ws + t.A);
    float* L = (float*)(ws + t.L);
    float* dA = (float*)(ws + t.dA);
    float* WcT = (float*)(ws + t.WcT);
    float* W1T = (float*)(ws + t.W1T);
    float* part = (float*)(ws + t.part);
    float* colpart = (float*)(ws + t.colpart);
    float* losspart = (float*)(ws + t.losspart);
    const int64_t W1cols = H > 0 ? H : C;

    if (N == 0) {
        // nothing to learn from: zero loss and gradients
        if (launch_zero(d_gW1, (size_t)(D_in * W1cols) * 4, stream)) return RETEXO_E_HIP;
        if (launch_zero(d_gb1, (size_t)W1cols * 4, stream)) return RETEXO_E_HIP;
        if (H > 0) {
            if (launch_zero(d_gWc, (size_t)(H * C) * 4, stream)) return RETEXO_E_HIP;
            if (launch_zero(d_gbc, (size_t)C * 4, stream)) return RETEXO_E_HIP;
        }
        if (launch_zero(d_loss, 4, stream)) return RETEXO_E_HIP;
        return RETEXO_OK;
    }

    // (the dropout's scale rides on the transposed classifier; the contractions over its and dL's padded width meet zeros)
    const Transpose top = {(int)H, (int)C, H > 0 ? (int)t.ldc : 0, d_Wc, WcT, keep_scale};
    const Transpose low = {(int)D_in, (int)W1cols, !d_gX ? 0 : H > 0 ? (int)H : (int)t.ldc, d_W1, W1T, 1.0f};
    auto blocks_of = [](const Transpose& x) { return ((int64_t)x.R * x.Cp + kThreads - 1) / kThreads; };
    prepare_kernel<<<dim3((unsigned)(kCountBlocks + blocks_of(top) + blocks_of(low))), dim3(kThreads), 0, stream>>>(
        N, d_labels, hdr, (unsigned)blocks_of(top), top, low);

    // forward
    const float* feat = d_X;        // input of the classifier product
    int64_t ldfeat = ldx, dfeat = D_in;
    if (H > 0) {
        // Which units are on goes into every gradient behind them; units whose sum is within rounding of zero are
        // decided by the float32 sums, so that a model trains the same however the products are formed.
        if (int e = launch_transform(N, D_in, H, d_X, ldx, d_W1, d_b1, true, A, t.ldh, stream, nullptr, 0, true)) return e;
        if (p_drop > 0.0f) {
            const uint32_t threshold = (uint32_t)((double)p_drop * 4294967296.0);
            const int64_t quads = N * ((H + 3) / 4);
            const int64_t blocks = (quads + kThreads - 1) / kThreads;
            dropout_kernel<<<dim3((unsigned)(blocks < (1 << 20) ? blocks : (1 << 20))), dim3(kThreads), 0, stream>>>(
                N, (int)H, A, t.ldh, threshold, keep_scale, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)draw,
                (uint32_t)(draw >> 32));
        }
        feat = A; ldfeat = t.ldh; dfeat = H;
    }
    if (int e = launch_transform(N, dfeat, C, feat, ldfeat, H > 0 ? d_Wc : d_W1, H > 0 ? d_bc : d_b1, false,
                                 L, t.ldc, stream))
        return e;

    // loss and d loss / d logits (in place, padding columns zeroed)
    const bool narrow = xent_narrow(t.ldc);
    const int64_t nb = xent_blocks(N, t.ldc);
    auto xent = narrow ? softmax_xent_kernel<true> : softmax_xent_kernel<false>;
    xent<<<dim3((unsigned)nb), dim3(kThreads), 0, stream>>>(N, (int)C, L, t.ldc, d_labels, hdr, losspart, xent_turns(N, narrow), colpart);

    // classifier (or only) layer: weight and bias gradients
    Finish f = {};
    f.n_loss = nb; f.losspart = losspart; f.hdr = hdr; f.loss = d_loss;
    f.C = (int)C; f.colpart = colpart;
    f.B = narrow ? nb : colsum(N, C, L, t.ldc, colpart, stream);
    f.gW = H > 0 ? d_gWc : d_gW1;
    f.gb = H > 0 ? d_gbc : d_gb1;
    wgrad(N, dfeat, C, feat, ldfeat, L, t.ldc, part, f, stream);

    if (H > 0) {
        // back through the classifier, the dropout (its mask is part of "A > 0") and the ReLU, then the layer's own gradients
        if (int e = launch_transform(N, t.ldc, H, L, t.ldc, WcT, nullptr, false, dA, t.ldh, stream, A, t.ldh, false, colpart)) return e;
        Finish g = {};
        g.B = transform_row_blocks(N, H); g.C = (int)H; g.colpart = colpart;
        g.gW = d_gW1;
        g.gb = d_gb1;
        wgrad(N, D_in, H, d_X, ldx, dA, t.ldh, part, g, stream);
        // dL/dX = dA W1^T, contracted over exactly H columns (dA's padding columns are not written)
        if (d_gX)
            if (int e = launch_transform(N, H, D_in, dA, t.ldh, W1T, nullptr, false, d_gX, ldgx, stream)) return e;
    } else if (d_gX) {
        // dL/dX = dL W1^T over the padded width of dL (its padding columns and the padding rows of W1^T are zero)
        if (int e = launch_transform(N, t.ldc, D_in, L, t.ldc, W1T, nullptr, false, d_gX, ldgx, stream)) return e;
    }
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
}  // namespace

extern "C" int retexo_layer_grad_x(int64_t N, int64_t D_in, int64_t H, int64_t C,
                                   const float* d_X, int64_t ldx, const int32_t* d_labels,
                                   const float* d_W1, const float* d_b1, const float* d_Wc, const float* d_bc,
                                   float* d_gW1, float* d_gb1, float* d_gWc, float* d_gbc, float* d_loss,
                                   float* d_gX, int64_t ldgx,
                                   void* d_workspace, int64_t workspace_bytes, void* stream)
{
    return layer_grad_impl(N, D_in, H, C, d_X, ldx, d_labels, d_W1, d_b1, d_Wc, d_bc, d_gW1, d_gb1, d_gWc, d_gbc,
                           d_loss, d_gX, ldgx, 0.0f, 0, 0, d_workspace, workspace_bytes, stream);
}

extern "C" int retexo_layer_grad_dropout(int64_t N, int64_t D_in, int64_t H, int64_t C,
                                         const float* d_X, int64_t ldx, const int32_t* d_labels,
                                         const float* d_W1, const float* d_b1, const float* d_Wc, const float* d_bc,
                                         float* d_gW1, float* d_gb1, float* d_gWc, float* d_gbc, float* d_loss,
                                         float* d_gX, int64_t ldgx, float p_drop, uint64_t seed, uint64_t draw,
                                         void* d_workspace, int64_t workspace_bytes, void* stream)
{
    return layer_grad_impl(N, D_in, H, C, d_X, ldx, d_labels, d_W1, d_b1, d_Wc, d_bc, d_gW1, d_gb1, d_gWc, d_gbc,
                           d_loss, d_gX, ldgx, p_drop, seed, draw, d_workspace, workspace_bytes, stream);
}

extern "C" int retexo_layer_grad(int64_t N, int64_t D_in, int64_t H, int64_t C,
                                 const float* d_X, int64_t ldx, const int32_t* d_labels,
                                 const float* d_W1, const float* d_b1, const float* d_Wc, const float* d_bc,
                                 float* d_gW1, float* d_gb1, float* d_gWc, float* d_gbc, float* d_loss,
                                 void* d_workspace, int64_t workspace_bytes, void* stream)
{
    return retexo_layer_grad_x(N, D_in, H, C, d_X, ldx, d_labels, d_W1, d_b1, d_Wc, d_bc, d_gW1, d_gb1, d_gWc,
                               d_gbc, d_loss, nullptr, 0, d_workspace, workspace_bytes, stream);
}

namespace {
struct TbLayout { int64_t part, colpart, total; };
TbLayout tb_layout(int64_t N, int64_t D_in, int64_t D_out)
{
    TbLayout t;
    const int64_t n1 = N > 0 ? N : 1;
    int64_t off = 0;
    auto take = [&](int64_t floats) { const int64_t at = off; off += align_up(floats * 4, 256); return at; };
    t.part = take(partial_floats(n1, D_in, D_out));
    t.colpart = take(((n1 + kColRows - 1) / kColRows) * D_out);
    t.total = off;
    return t;
}
}  // namespace

extern "C" int64_t retexo_transform_backward_workspace_bytes(int64_t N, int64_t D_in, int64_t D_out)
{
    if (int s = check_sizes(N, D_in, 0, D_out)) return s;
    return tb_layout(N, D_in, D_out).total;
}

extern "C" int retexo_transform_backward(int64_t N, int64_t D_in, int64_t D_out,
                                         const float* d_H, int64_t ldh, const float* d_dZ, int64_t lddz,
                                         float* d_gW, float* d_gb,
                                         void* d_workspace, int64_t workspace_bytes, void* stream_)
{
    if (int s = check_sizes(N, D_in, 0, D_out)) return s;
    if (ldh < D_in || lddz < D_out) return RETEXO_E_LD;
    if (!d_gW) return RETEXO_E_NULL;
    if (N > 0 && (!d_H || !d_dZ)) return RETEXO_E_NULL;
    const TbLayout t = tb_layout(N, D_in, D_out);
    if (!d_workspace || workspace_bytes < t.total || ((uintptr_t)d_workspace & 255)) return RETEXO_E_WORKSPACE;
    hipStream_t stream = (hipStream_t)stream_;
    if (N == 0) {
        if (launch_zero(d_gW, (size_t)(D_in * D_out) * 4, stream)) return RETEXO_E_HIP;
        if (d_gb) if (launch_zero(d_gb, (size_t)D_out * 4, stream)) return RETEXO_E_HIP;
        return RETEXO_OK;
    }
    char* ws = (char*)d_workspace;
    Finish f = {};
    f.gW = d_gW;
    if (d_gb) {
        f.C = (int)D_out; f.gb = d_gb; f.colpart = (float*)(ws + t.colpart);
        f.B = colsum(N, D_out, d_dZ, lddz, (float*)(ws + t.colpart), stream);
    }
    wgrad(N, D_in, D_out, d_H, ldh, d_dZ, lddz, (float*)(ws + t.part), f, stream);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}

extern "C" int retexo_sgd_update(int64_t n, float* d_param, const float* d_grad, float lr, void* stream)
{
    if (n < 0) return RETEXO_E_SIZE;
    if (n == 0) return RETEXO_OK;
    if (!d_param || !d_grad) return RETEXO_E_NULL;
    sgd_kernel<<<dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, (hipStream_t)stream>>>(
        n, d_param, d_grad, lr);
    if (hipGetLastError() != hipSuccess) return RETEXO_E_HIP;
    return RETEXO_OK;
}
