// A whole layer in one kernel -- input transform, channel sums, output transform (Sec. 2.1 steps 1, 3, 4) -- for
// layers with so little work that the launches and the latency of three kernels are what takes the time.
//
// A workgroup takes TB consecutive tiles of the batch (whatever tile rows and images they belong to) and KB output
// channels.  Per block of input channels (32 in binary16, 16 in binary32) it stages the tiles' windows in LDS as
// the input transform does, transforms them -- V of the block stays in LDS -- and adds the block's products
// to M[xi] = sum V[xi] U[xi], which stays in registers: wave w holds the positions xi = w, w + waves, ...,
// all TB tiles and KB channels of each, as 16 x 16 results of the matrix unit.  U comes from L2 straight into
// registers (a fragment of 16 channels x 64 bytes is one contiguous KiB, no two waves want the same one);
// x of the next block and U of this one are under way while a block is transformed.  At the end M goes through
// LDS to the threads that transform it, one (tile, channel) pair each, and their m x m results leave as rows of m
// elements, neighbouring tiles in neighbouring lanes.
// Every value is formed by the same operations in the same order as by the kernels for larger layers, so the
// results are the same bits (the sign of a pooled zero among them, larger_of): V by the contract of the input transform; M in ascending channels (the matrix
// unit's sums do not depend on the shape of the instruction; binary32: two chains, in the order contract.hip gives);
// the output transform columns first, or, for the layers that
// otherwise run contraction and output transform as one kernel (64 input channels, ROWS_FIRST), in its order.
// The windows are transformed again for every KB output channels, which is why large layers do not come here.
#include <algorithm>

#include "input_common.hpp"
#include "output_common.hpp"

namespace nova {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

template <int N, int R>
struct LayerCoef {
    InCoef<N> in;
    OutCoef<N, R> out;
};

// Operand fragments of the 16 x 16 matrix instructions: lane l supplies row l % 16 and the channels of piece l / 16.
//   binary16: 8 channels of the 32, one instruction (16x16x32).
//   binary32: channels 4 p .. 4 p + 3 of the 16 for piece p; four instructions (16x16x4) take one each, the first two
//   for one chain of sums, the others for a second one.
template <typename T> struct Products;
template <> struct Products<f16> {
    static constexpr int CHAINS = 1;
    typedef half8 frag;
    static __device__ __forceinline__ frag load_filter(const f16 *row0, unsigned lane)         // 32 channels of 16 rows of U
    {
        const unsigned off = ((lane & 15u) * kChanBlock + (lane >> 4) * 8u) * (unsigned)sizeof(f16);
        return *reinterpret_cast<const NOVA_GLOBAL frag *>(plane_element(row0, off));
    }
    static __device__ __forceinline__ void add(float4v (&acc)[CHAINS], const frag &u, const half8 &v)
    {
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(u, v, acc[0], 0, 0, 0);
    }
};
template <> struct Products<float> {
    static constexpr int CHAINS = 2;
    typedef float4v frag;
    static __device__ __forceinline__ frag load_filter(const float *row0, unsigned lane)       // 16 channels of 16 rows of U
    {
        const unsigned off = ((lane & 15u) * kChanBlock + (lane >> 4) * 4u) * (unsigned)sizeof(float);
        return *reinterpret_cast<const NOVA_GLOBAL frag *>(plane_element(row0, off));
    }
    static __device__ __forceinline__ void add(float4v (&acc)[CHAINS], const frag &u, const float4v &v)
    {
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int ch = 0; ch < CHAINS; ++ch) acc[ch] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[2 * ch + e], v[2 * ch + e], acc[ch], 0, 0, 0);
    }
};

// Rows [P0, P0 + ROWS) of the m x m outputs of one pair from its n x n products m_at(i, j), rounded to T.  Columns first,
// as output_transform_kernel (without ReLU a binary16 result is rounded together with its last multiply-add there).
template <int N, int R, typename T, bool RELU, int P0, int ROWS, typename F>
__device__ __forceinline__ void outputs_columns_first(F &&m_at, T (&out)[ROWS][N - R + 1], const OutCoef<N, R> &coef)
{
    constexpr int M = N - R + 1, H = (N - 2) / 2;
    float z[ROWS][N], s[H], d[H];
#pragma unroll
    for (int b = 0; b < N; ++b) {
        float v[N];
#pragma unroll
        for (int a = 0; a < N; ++a) v[a] = m_at(a, b);
        output_transform_1d_pairs<N, R>(v, s, d);
#pragma unroll
        for (int p = 0; p < ROWS; ++p) z[p][b] = output_transform_1d_out<N, R>(P0 + p, v[0], v[N - 1], s, d, coef);
    }
#pragma unroll
    for (int p = 0; p < ROWS; ++p) {
        output_transform_1d_pairs<N, R>(z[p], s, d);
        if constexpr (sizeof(T) == 2 && !RELU) {
#pragma unroll
            for (int q = 0; q < M; q += 2) {
                const unsigned word = output_transform_1d_f16_pair<N, R>(q, z[p][0], z[p][N - 1], s, d, coef);
                __builtin_memcpy(&out[p][q], &word, 4);
            }
        } else {
#pragma unroll
            for (int q = 0; q < M; ++q) {
                const float v = output_transform_1d_out<N, R>(q, z[p][0], z[p][N - 1], s, d, coef);
                out[p][q] = (T)(RELU && v < 0.0f ? 0.0f : v);                     // NaN stays NaN
            }
        }
    }
}
// All of them, rows first, folded pair by pair, as fused_contract_output_kernel (rounding is a step of its own there).
template <int N, int R, typename T, bool RELU, typename F>
__device__ __forceinline__ void outputs_rows_first(F &&m_at, T (&out)[N - R + 1][N - R + 1], const OutCoef<N, R> &coef)
{
    constexpr int M = N - R + 1;
    float Y[M][M];
    auto row = [&](int i, float (&o)[M]) __attribute__((always_inline)) {
        float v[N];
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = m_at(i, j);
        output_transform_1d<N, R, true>(v, o, coef);
    };
    float carried[M], w[M];
    row(0, w);
#pragma unroll
    for (int p = 0; p < M; ++p)
#pragma unroll
        for (int q = 0; q < M; ++q) Y[p][q] = fma32(p == 0 ? coef.zero : 0.0f, (p & 1) ? 0.0f - w[q] : 0.0f + w[q], 0.0f);
#pragma unroll
    for (int d = 1; d < N / 2; ++d) {
        row(2 * d - 1, carried);
        row(2 * d, w);
#pragma unroll
        for (int p = 0; p < M; ++p)
#pragma unroll
            for (int q = 0; q < M; ++q)
                Y[p][q] = fma32(coef.pw[(d - 1) * M + p], (p & 1) ? carried[q] - w[q] : carried[q] + w[q], Y[p][q]);
    }
    row(N - 1, w);
#pragma unroll
    for (int q = 0; q < M; ++q) Y[M - 1][q] = fma32(coef.inf, w[q], Y[M - 1][q]);
#pragma unroll
    for (int p = 0; p < M; ++p)
#pragma unroll
        for (int q = 0; q < M; ++q) out[p][q] = round_twice(RELU && Y[p][q] < 0.0f ? 0.0f : Y[p][q], (T *)nullptr);
}

// The outputs of part `part` (wave-uniform) of the SPLIT that share a pair: whole pairs of rows, so that pooling
// stays within a part.
template <int N, int R, typename T, int SPLIT, bool RELU, bool ROWS_FIRST, int I, typename F>
__device__ __forceinline__ void output_part(int part, F &&m_at, const OutCoef<N, R> &coef, T *plane, int tr, int tc, int H, int W, bool pool,
                                            bool zeros)
{
    constexpr int M = N - R + 1;
    if constexpr (I + 1 < SPLIT) {
        if (part != I) return output_part<N, R, T, SPLIT, RELU, ROWS_FIRST, I + 1>(part, m_at, coef, plane, tr, tc, H, W, pool, zeros);
    }
    constexpr int P0 = 2 * ((M / 2 * I + SPLIT - 1) / SPLIT), ROWS = 2 * ((M / 2 * (I + 1) + SPLIT - 1) / SPLIT) - P0;
    static_assert(ROWS >= 2 && (!ROWS_FIRST || SPLIT == 1), "parts");
    T out[ROWS][M];
    if constexpr (ROWS_FIRST) outputs_rows_first<N, R, T, RELU>(m_at, out, coef);
    else outputs_columns_first<N, R, T, RELU, P0, ROWS>(m_at, out, coef);
    store_tile_rows<T, M, P0, ROWS>(out, plane, tr, tc, H, W, pool, zeros);
}

// Where the transform's values go: the thread's word in the row of its tile, position by position.
template <int N, typename T, int V_POS>
struct VToLds {
    unsigned char *to;
    __device__ __forceinline__ void start(int) {}
    template <int CPT>
    __device__ __forceinline__ void value(int i, int j, const float (&o)[CPT][N])
    {
        *reinterpret_cast<unsigned *>(to + (i * N + j) * V_POS) = rounded_word<N>(o, j, (T *)nullptr);
    }
};

template <int N, int R, typename T, int TB, int KB, int RS, bool RELU, bool ROWS_FIRST>
__global__ void __launch_bounds__(TB * 16 * RS)
layer_kernel(const T *__restrict__ x, const T *__restrict__ U, T *__restrict__ y, int C, int H, int W, int K, int Kp,
             int tiles_h, int tiles_w, int c_blocks, int k_groups, int Ttot, long long x_elems, int flags, LayerCoef<N, R> coef)
{
    constexpr int CH = sizeof(T) == 2 ? 32 : 16;            // input channels per turn
    using B = TileWindows<N, T, CH, TB, RS>;
    using P = Products<T>;
    constexpr int M = N - R + 1, THREADS = B::THREADS, WAVES = THREADS / 64;
    constexpr int KF = KB / 16, OWN = N * N / WAVES;         // 16-channel blocks; positions of a wave
    // threads that share a pair's output rows: as many as there are, at most one per two rows
    constexpr int SPLIT = ROWS_FIRST || THREADS < 2 * KB * TB ? 1 : THREADS / (KB * TB) < M / 2 ? THREADS / (KB * TB) : M / 2;
    constexpr int V_POS = TB * 64;                          // bytes of V of one position
    // filters are asked for before the transform where the registers hold both.  Scratch per lane: 44 bytes (10 registers) for n = 8 with
    // 16 tiles in binary16, whose 1024 threads have 128 registers each; n = 10, 168 registers: 20 bytes (4) in binary16, 108 (30, r = 3)
    // and 72 (17, r = 5) in binary32; none elsewhere
    // (with 64 output channels they come after it: 80 bytes of scratch otherwise, 64 -> 64 @224x224 F(4,3) 16.1 us instead of 14.4)
    constexpr bool EARLY = KB < 64 && (N < 8 || (N == 8 && (TB == 8 || sizeof(T) == 4)));
    static_assert(B::GP == 16 && N * N % WAVES == 0 && KB % 16 == 0 && (TB == 8 || TB == 16), "workgroup shape");
    extern __shared__ __align__(16) unsigned char lds_raw[];
    unsigned *windows = reinterpret_cast<unsigned *>(lds_raw);
    unsigned char *v_lds = lds_raw + B::LDS_BYTES;
    float *m_lds = reinterpret_cast<float *>(lds_raw);      // at the end

    const unsigned bid = xcd_local_block_id(blockIdx.x, gridDim.x);
    const int kg = (int)(bid % (unsigned)k_groups), t0 = (int)(bid / (unsigned)k_groups) * TB;
    const int count = Ttot - t0 < TB ? Ttot - t0 : TB;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool pool = (flags & NOVA_FLAG_POOL2) != 0;

    WindowRows<N, R, T, B, true> rows;
    rows.place_tile(t0, count, tiles_h, tiles_w);
    rows.keep_addresses(H, W);
    const T *planes = x + (long long)rows.img * C * H * W;
    const long long block_elems = (long long)CH * H * W;
    long long remaining = x_elems - (planes - x);
    rows.template load<false>(planes, C, remaining, H, W);

    // transform: lanes run over the words of a tile's channel block, a wave over four tiles
    const int g = tid % 16, j = tid / 16 % TB;
    const int part = __builtin_amdgcn_readfirstlane(tid / (16 * TB));
    const unsigned *win = windows + j * B::TILE + g * B::WIN;
    // V in LDS: [position][tile] rows of 64 bytes, 16-byte pieces in the places piece ^ (tile / 2) % 4 (fragment
    // reads of 16 rows are then free of bank conflicts)
    unsigned char *v_to = v_lds + j * 64 + (((g >> 2) ^ ((j >> 1) & 3)) * 16) + (g & 3) * 4;
    const int f_tile = (lane & 15) % TB;
    const unsigned char *v_from = v_lds + f_tile * 64 + (((lane >> 4) ^ ((f_tile >> 1) & 3)) * 16);

    float4v acc[OWN][KF][P::CHAINS];
#pragma unroll
    for (int i = 0; i < OWN; ++i)
#pragma unroll
        for (int f = 0; f < KF; ++f)
#pragma unroll
            for (int c = 0; c < P::CHAINS; ++c) acc[i][f][c] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

    const int turns = (C + CH - 1) / CH;
    for (int turn = 0; turn < turns; ++turn) {
        const int c_lim = C - turn * CH;
        rows.place(windows, c_lim, remaining, H, W);
        __syncthreads();
        if (turn + 1 < turns) {
            planes += block_elems;
            remaining -= block_elems;
            rows.template load<false>(planes, c_lim - CH, remaining, H, W);
        }
        // the wave's filters of this block
        typename P::frag uf[OWN][KF];
        const T *u_at = U + ((size_t)wave * c_blocks + (size_t)(turn * CH / kChanBlock)) * Kp * kChanBlock + (size_t)kg * KB * kChanBlock +
                        (turn * CH) % kChanBlock;
        auto load_filters = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const T *at = uniform_pointer(u_at + (size_t)(i * WAVES) * c_blocks * Kp * kChanBlock);
#pragma unroll
                for (int f = 0; f < KF; ++f) {
                    // (U has whole blocks of 32 output channels: of the last 64 there may be only the first, which is read again then)
                    const int rows = KB <= 32 || kg * KB + f * 16 < Kp ? f * 16 : 0;
                    uf[i][f] = P::load_filter(at + rows * kChanBlock, (unsigned)lane);
                }
            }
        };
        if constexpr (EARLY) load_filters();
        transform_part<N, T, true, B>(part, win, coef.in, VToLds<N, T, V_POS>{v_to});
        if constexpr (!EARLY) load_filters();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            typedef typename std::conditional<sizeof(T) == 2, half8, float4v>::type vfrag;
            const vfrag vf = *reinterpret_cast<const vfrag *>(v_from + (wave + i * WAVES) * V_POS);
#pragma unroll
            for (int f = 0; f < KF; ++f) P::add(acc[i][f], uf[i][f], vf);
        }
    }
    __syncthreads();

    // ---- M to LDS: [position][KB channels][TB tiles], the channels of a block in the order e * 4 + piece in which
    // the lanes hold them (channel 4 * piece + e)
    const bool round_m = sizeof(T) == 2 && (flags & NOVA_FLAG_M_F16);
    const bool zeros = !RELU || round_m;                    // (a sum of products that were rounded to -0 passes the ReLU as -0)
    if (TB == 16 || (lane & 15) < TB) {
#pragma unroll
        for (int i = 0; i < OWN; ++i)
#pragma unroll
            for (int f = 0; f < KF; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float sum = acc[i][f][0][e];
                    if constexpr (P::CHAINS == 2) sum += acc[i][f][P::CHAINS - 1][e];
                    if (round_m) sum = (float)round_twice(sum, (f16 *)nullptr);
                    m_lds[(wave + i * WAVES) * (KB * TB) + (f * 16 + e * 4 + (lane >> 4)) * TB + (lane & 15)] = sum;
                }
    }
    __syncthreads();

    // ---- SPLIT threads per (tile, channel) pair, each with some rows of its outputs; neighbouring tiles in
    // neighbouring lanes
    for (int item = tid; item < KB * TB * SPLIT; item += THREADS) {
        const int pair = item % (KB * TB), q = pair / TB, tile = pair % TB;
        const int k = kg * KB + (q & ~15) + 4 * (q & 3) + ((q >> 2) & 3);
        if (tile >= count || k >= K) continue;
        const int t = t0 + tile, trow = t / tiles_w, tc = t - trow * tiles_w, img = trow / tiles_h, tr = trow - img * tiles_h;
        const float *m_pair = m_lds + pair;
        auto m_at = [&](int a, int b) __attribute__((always_inline)) { return m_pair[(a * N + b) * (KB * TB)]; };
        output_part<N, R, T, SPLIT, RELU, ROWS_FIRST, 0>(SPLIT > 1 ? __builtin_amdgcn_readfirstlane(item / (KB * TB)) : 0, m_at, coef.out,
                                                        y + ((long long)img * K + k) * (pool ? (long long)(H / 2) * (W / 2) : (long long)H * W), tr, tc, H, W, pool,
                                                        zeros);
    }
}

template <int N, int R, typename T, int TB, int KB, int RS, bool ROWS_FIRST>
static int launch_layer_shape(const nova_transforms *t, const void *x, const void *U, void *y, const Geometry &g, int flags, hipStream_t stream)
{
    using B = TileWindows<N, T, sizeof(T) == 2 ? 32 : 16, TB, RS>;
    constexpr int LOOP = B::LDS_BYTES + N * N * TB * 64, END = N * N * TB * KB * 4, LDS = LOOP > END ? LOOP : END;
    static_assert(LDS <= 160 * 1024, "LDS of a workgroup");
    LayerCoef<N, R> coef;
    fill_in_coef<N>(t, coef.in);
    fill_out_coef<N, R>(t, coef.out);
    const int k_groups = ceil_div(g.K, KB);
    const long long blocks = (g.T + TB - 1) / TB * k_groups;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    auto kern = (flags & NOVA_FLAG_RELU) ? layer_kernel<N, R, T, TB, KB, RS, true, ROWS_FIRST> : layer_kernel<N, R, T, TB, KB, RS, false, ROWS_FIRST>;
    if (LDS > 64 * 1024)
        NOVA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS));
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(B::THREADS), LDS, stream, (const T *)x, (const T *)U, (T *)y, g.C, g.H, g.W, g.K,
                       g.Kp, g.tiles_h, g.tiles_w, g.c_blocks, k_groups, (int)g.T, (long long)g.N * g.C * g.H * g.W, flags, coef);
    return (int)hipGetLastError();
}

// Output channels per workgroup.  16 tiles of n = 4 and 6 also take twice as many: the windows are transformed half as often and few
// layers need a second round of workgroups (64 -> 64 @224x224 F(4,3) 18.4 -> 14.4 us, 48 -> 64 5x5 @25x25 batch 22 F(2,5) 21.5
// -> 12.7, binary32 96 -> 64 @16x16 batch 78 F(4,3) 29.9 -> 23.4), but a workgroup by itself takes longer.  (Larger n: the products do not fit
// the LDS or the registers; 8 tiles of n = 8 in binary32 with 32 channels 1.5 to 2 times as long.)
template <int N, typename T> constexpr int kLayerChannels = sizeof(T) == 2 && N < 10 ? 32 : 16;

template <int N, int R, typename T, bool ROWS_FIRST>
static int launch_layer_n(const nova_transforms *t, const void *x, const void *U, void *y, const Geometry &g, int flags, LayerShape shape, hipStream_t s)
{
    if constexpr (N < 8) {
        constexpr int WIDE = 2 * kLayerChannels<N, T>;
        if (shape.channels == WIDE) return launch_layer_shape<N, R, T, 16, WIDE, N / 2, ROWS_FIRST>(t, x, U, y, g, flags, s);
    }
    // (16 windows of 10 x 10 and their V do not fit the LDS)
    if constexpr (N < 10) {
        if (shape.tiles == 16) return launch_layer_shape<N, R, T, 16, kLayerChannels<N, T>, N / 2, ROWS_FIRST>(t, x, U, y, g, flags, s);
    }
    return launch_layer_shape<N, R, T, 8, kLayerChannels<N, T>, N / 2, ROWS_FIRST>(t, x, U, y, g, flags, s);
}

// Which layers run as one kernel, and with how many tiles per workgroup: the shape with the lowest estimate, if
// that is below 0.94 of the estimate for the separate kernels (0.85 from 30 us on, where the estimates are widest).  Estimates (us):
//   one kernel        2 + rounds * (turns * kTurn + kOnce), rounds = workgroups per compute unit, turns = blocks of input channels
//                     (n = 4, where several workgroups share a compute unit: at least 3 + turns * 1.3, binary32 1.0, the serial chain; 16 tiles in
//                     binary32 3 + turns / 2 + workgroups per compute unit, not rounded, * (0.7 turns + 0.55))
//                     + 3 per million results beyond the first two million that lie in tiles cut off at the right edge, whose rows left
//                     element by element when this was fitted and leave in pieces of 4, 2 and 1 now (6 -> 166 @128x5 batch 159 F(6,3), 17 million: 121 in one kernel, 70 apart)
//   separate kernels  kStages + kPerMB for each MB of V and M (or what is left of M) + 11 per GFLOP in binary32
//   twice the         the same with their own times (n = 4: at least 6 + turns * 1.9, binary32 3.9 + turns * 1.35; binary16 up to four turns, with more
//   channels          0.88 times as fast), taken below 0.94 of the estimate without.  600 layers of 200 to 16000 tiles in binary16: 80 run otherwise
//                     than before, 1.2 times as fast in the geometric mean, the slowest 0.92
// Fitted to 2600 layers of 1 to 12000 tiles, 5 to 520 -> 1 to 520 channels, timed both ways on one MI355X (sd 6-13 %, one kernel n = 4
// 20-30 %): 1295 are taken, geometric mean 1.54 times as fast as the separate kernels; nine are slower by more than 2 %, two of
// them by more than 10 % (18 -> 128 5x5 @38x4 batch 7 F(6,5) binary32 20.5 / 16.9 us, 300 -> 33 @7x109 batch 32 F(6,3) binary32 78.7 / 70.9).
// us, separate / one kernel: 16 -> 16 @32x32 F(4,3) binary32 12.3 / 6.7; 40 -> 70 @45x61 batch 8 F(6,3) binary32 29.5 / 16.7; 48
// -> 96 5x5 @35x35 batch 16 27.6 / 16.7; 64 -> 64 @56x56 batch 8 F(6,3) 17.4 / 14.0; 64 -> 128 @112x112 F(4,3) 18.7 / 10.4; not
// taken: 256 -> 256 @56x56 F(4,3) 18.2 / 22, 512 -> 512 @28x28 17 / 38.
struct LayerTimes { double turn[2], once[2], stages, per_mb; };          // [8 tiles, 16 tiles]
static const LayerTimes &layer_times(int n, bool half)
{
    static const LayerTimes kHalf[] = {{{0.78, 0.94}, {1.45, 2.2}, 12.4, 0.40}, {{1.85, 2.15}, {3.6, 3.75}, 13.6, 0.40},
                                       {{3.3, 4.95}, {4.9, 5.4}, 15.6, 0.43}, {{4.55, 0}, {5.9, 0}, 20.3, 0.38}};
    static const LayerTimes kFull[] = {{{0.74, 0.86}, {1.06, 1.6}, 12.5, 0.37}, {{1.7, 1.8}, {2.6, 2.9}, 14.2, 0.35},
                                       {{3.3, 3.6}, {3.2, 3.5}, 15.9, 0.33}, {{6.1, 0}, {5.1, 0}, 19.4, 0.35}};
    return (half ? kHalf : kFull)[n / 2 - 2];
}

LayerShape layer_shape(const nova_transforms *t, const Geometry &g, int dtype, size_t domain_bytes, bool contract_output)
{
    // points in the paired order, whole window rows in x, planes within 32-bit offsets
    const long long x_elems = (long long)g.N * g.C * g.H * g.W;
    if (!t->symmetric || g.C <= few_channels_limit() || g.T > 0x7fffffffLL || x_elems < g.m || (long long)kChanBlock * g.H * g.W >= (1LL << 30))
        return {0, 0};
    const bool half = dtype == NOVA_F16;
    const LayerTimes &lt = layer_times(g.n, half);
    const int turns = ceil_div(g.C, half ? 32 : 16), k_groups = ceil_div(g.K, half && g.n < 10 ? 32 : 16);
    double best = lt.stages + lt.per_mb * 1e-6 * (double)domain_bytes;
    if (!half) best += 11e-9 * 2.0 * g.n * g.n * (double)g.T * g.C * g.Kp;
    best *= best < 30.0 ? 0.94 : 0.85;
    // Where contraction and output transform would run as one kernel (contract_output.hip) domain_bytes is V alone; n = 6 and 4 were timed
    // against it.  n = 6: what its stages, 64 input channels each, add.  (96 -> 128 @39x39 batch 16 F(4,3) 22.9 / 18.3 us, 48 -> 64 5x5 @25x25
    // batch 22 21.5 / 12.7.)  n = 4: 7.6 + 0.3 per 1000 tiles and block of input channels + 1.5 + 2.75 per block for 1000 of its workgroups + 1.5
    // per million tiles x output channels (sd 10 %, 207 layers); one kernel below 0.87 of that (of 500 layers 43 that would run there run as one
    // kernel, 1.19 times as fast, the slowest 0.93: 64 -> 64 @23x24 batch 71 21.4 / 15.9, 48 -> 33 @2x6 batch 2309 17.0 / 10.3).
    if (contract_output) {
        if (!half || g.n > 6) return {0, 0};
        const double groups = 1e-3 * (double)((g.T + 31) / 32 * g.k_blocks);
        best = g.n == 6 ? 0.85 * (lt.stages + lt.per_mb * 1e-6 * (double)domain_bytes + 1.5 * ((g.c_blocks + 1) / 2))
                        : 0.87 * (7.6 + 0.3e-3 * (double)g.T * g.c_blocks + groups * (1.5 + 2.75 * g.c_blocks) + 1.5e-6 * (double)g.T * g.K);
    }
    const double cut = std::max(0.0, (double)g.N * g.K * g.H * (g.W % g.m) - 2e6);
    const int channels = half && g.n < 10 ? 32 : 16;
    const auto rounds_of = [&](int tiles, int groups) {
        return (double)(((g.T + tiles - 1) / tiles * groups + device_cu_count() - 1) / device_cu_count());
    };
    LayerShape shape = {0, 0};
    for (int i = 0; i < (g.n < 10 ? 2 : 1); ++i) {
        double time = 2.0 + rounds_of(8 * (i + 1), k_groups) * (turns * lt.turn[i] + lt.once[i]);
        if (g.n == 4 && !half && i == 1) time = 3.0 + 0.5 * turns + (double)((g.T + 15) / 16 * k_groups) / device_cu_count() * (0.7 * turns + 0.55);
        if (g.n == 4) time = std::max(time, 3.0 + turns * (half ? 1.3 : 1.0));
        time += 3e-6 * cut;
        if (time < best) { best = time; shape = {8 * (i + 1), channels}; }
    }
    if (g.n < 8 && g.K > channels && (!half || g.n == 6 || turns <= 4)) {
        static const LayerTimes kWideHalf[] = {{{0, 1.15}, {0, 1.9}, 0, 0}, {{0, 3.5}, {0, 5.3}, 0, 0}}, kWideFull[] = {{{0, 1.3}, {0, 0.9}, 0, 0}, {{0, 3.15}, {0, 3.6}, 0, 0}};
        const LayerTimes &wide = (half ? kWideHalf : kWideFull)[g.n / 2 - 2];
        double time = 2.0 + rounds_of(16, ceil_div(g.K, 2 * channels)) * (turns * wide.turn[1] + wide.once[1]);
        if (g.n == 4) time = std::max(time, half ? 6.0 + turns * 1.9 : 3.9 + turns * 1.35);
        time += 3e-6 * cut;
        if (time < best * (shape.tiles ? 0.94 : 1.0)) shape = {16, 2 * channels};
    }
    return shape;
}

int launch_layer(const nova_transforms *t, const void *x, const void *U, void *y, const Geometry &g, int dtype, int flags, LayerShape shape,
                 void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    const bool h = dtype == NOVA_F16;
    const bool rows_first = fused_contract_output_preferred(t, g, dtype, flags);
#define NOVA_LAYER(N, R) (h ? launch_layer_n<N, R, f16, false>(t, x, U, y, g, flags, shape, s) \
                            : launch_layer_n<N, R, float, false>(t, x, U, y, g, flags, shape, s))
    if (t->r == 3) {
        switch (t->n) {
        case 4: return NOVA_LAYER(4, 3);
        case 6: return NOVA_LAYER(6, 3);
        case 8: return rows_first ? launch_layer_n<8, 3, f16, true>(t, x, U, y, g, flags, shape, s) : NOVA_LAYER(8, 3);
        case 10: return rows_first ? launch_layer_n<10, 3, f16, true>(t, x, U, y, g, flags, shape, s) : NOVA_LAYER(10, 3);
        }
    } else if (t->r == 5) {
        switch (t->n) {
        case 6: return NOVA_LAYER(6, 5);
        case 8: return NOVA_LAYER(8, 5);
        case 10: return NOVA_LAYER(10, 5);
        }
    }
#undef NOVA_LAYER
    return (int)hipErrorInvalidValue;
}

}  // namespace nova
