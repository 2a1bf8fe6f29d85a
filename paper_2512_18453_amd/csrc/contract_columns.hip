// Contraction over input channels and the first half of the output transform in one kernel (Sec. 2.1 steps 3 and 4):
//     Z[j][p][t][k] = sum_i A[i][p] M[i*n + j][t][k],   M[xi][t][k] = sum_c V[xi][t][c] U[xi][k][c]
// for the calls that run the whole layer.  A wave keeps the products of the n positions of a column j for its tiles and
// output channels in registers (the matrix unit leaves the same (tile, channel) in the same place for each of them),
// transforms them along the column and stores m values instead of n: of what the separate kernels write and
// read again, 20 % (n = 10), 25 % (8), 33 % (6) or half (4) never exists.  What is left for the output transform is
// one 1D transform per row.  Products and sums are those of the separate kernels in the same order, so the results
// are the same bits.
//
// The channel loop (contract_loop.hpp) runs without a break over the n positions.  A lane holds one
// channel of a block and 16 tiles, so a store covers two whole 128-byte rows of Z.
#include "contract_loop.hpp"
#include "output_common.hpp"

namespace nova {

template <int N, int R, int BM, int BN, int WM, int WN, int S, int OCC>
__global__ void __launch_bounds__(64 * WM * WN, (OCC * WM * WN + 3) / 4)
contract_columns_kernel(const f16 *__restrict__ U, const f16 *__restrict__ V, float *__restrict__ Z, int T, int Tp, int Kp,
                        int c_blocks, int k_blocks, int row_blocks, int col_blocks, OutCoef<N, R> coef)
{
    constexpr int M = N - R + 1;
    using Loop = ChannelLoop<BM, BN, WM, WN, S>;
    constexpr int MB = Loop::MB, NB = Loop::NB;
    extern __shared__ __align__(1024) unsigned char ring[];

    unsigned bid = xcd_local_block_id(blockIdx.x, gridDim.x);
    const int cbk = bid % col_blocks; bid /= col_blocks;
    const int rbk = bid % row_blocks; bid /= row_blocks;
    const int column = bid;
    const int t0 = rbk * BM, k0 = cbk * BN;
    const int lane = (int)(threadIdx.x & 63), frag_row = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave / WN, wn = wave % WN;

    Loop loop;
    loop.start(ring, V + ((size_t)column * c_blocks * T + t0) * kChanBlock, U + ((size_t)column * c_blocks * Kp + k0) * kChanBlock, T, Kp,
               T - 1 - t0, Kp - 1 - k0, c_blocks, N, (long long)N * c_blocks);
    float16v acc[N][NB][MB];
    int slot = 0;
    loop.fill();
#pragma unroll
    for (int a = 0; a < N; ++a) loop.position(ring, slot, acc[a]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the surplus loads must land before the LDS is released

    // D[row = t][col = k]: lane holds channel lane % 32 of a block and tiles 8 (e / 4) + 4 (lane / 32) + e % 4.  Rows up to Tp
    // exist, so no store asks for its row.
    const size_t plane = (size_t)k_blocks * Tp * kChanBlock;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int kb = (k0 >> 5) + wn * NB + j;
        if (kb >= k_blocks) continue;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            float *base = uniform_pointer(Z + (size_t)column * M * plane + (size_t)kb * Tp * kChanBlock);
            const unsigned row0 = (unsigned)(t0 + (wm * MB + i) * 32 + (lane >> 5) * 4);
            if (t0 + (wm * MB + i) * 32 >= T) continue;
            const unsigned at = (row0 * kChanBlock + (unsigned)frag_row) * 4u;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float v[N], o[M];
#pragma unroll
                for (int a = 0; a < N; ++a) v[a] = acc[a][j][i][e];
                output_transform_1d<N, R, true>(v, o, coef);
#pragma unroll
                for (int p = 0; p < M; ++p)
                    *plane_element(base + (size_t)p * plane + ((e >> 2) * 8 + (e & 3)) * kChanBlock, at) = o[p];
            }
        }
    }
}

template <int N, int R, int BM, int BN, int WM, int WN, int S, int OCC>
static int launch_columns(const nova_transforms *t, const void *U, const void *V, void *Z, const Geometry &g, hipStream_t stream)
{
    const int row_blocks = ceil_div((int)g.T, BM), col_blocks = ceil_div(g.Kp, BN);
    const long long blocks = (long long)N * row_blocks * col_blocks;
    constexpr int LDS = ChannelLoop<BM, BN, WM, WN, S>::LDS_BYTES;
    static_assert(LDS * OCC <= 160 * 1024, "ring");
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    OutCoef<N, R> coef;
    fill_out_coef<N, R>(t, coef);
    auto kern = contract_columns_kernel<N, R, BM, BN, WM, WN, S, OCC>;
    if (LDS > 64 * 1024)
        NOVA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS));
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * WM * WN), LDS, stream, (const f16 *)U, (const f16 *)V, (float *)Z, (int)g.T,
                       (int)g.Tp, g.Kp, g.c_blocks, g.k_blocks, row_blocks, col_blocks, coef);
    return (int)hipGetLastError();
}

template <int N, int R>
static int launch_columns_n(const nova_transforms *t, const void *U, const void *V, void *Z, const Geometry &g, hipStream_t s)
{
    // 64 x 64 by 4 waves, a ring of 4: us for the whole call, ring of 3 / 4 / 5 and 128 x 64 by 8 waves, 128 -> 128 @112x112 batch 32
    // F(6,3): 233.7 / 232.3 / 231.6 / 238.8, 256 -> 256 @56x56 batch 32 F(8,3): 133 / 128 / 126 / 145.  (Rings of
    // 4 and 5 differ by less than the runs do; with 5, 40 KB, n = 4 would lose the fifth workgroup per compute unit that its 89
    // registers allow.  Two channel blocks per stage with the next fragments read ahead, 64 KB of LDS: 241 and 130 -- two workgroups
    // per compute unit instead of three or four.)
    // One block of output channels: 128 x 32, none of it padding.
    if (g.Kp == 32) return launch_columns<N, R, 128, 32, 4, 1, 4, 2>(t, U, V, Z, g, s);
    return launch_columns<N, R, 64, 64, 2, 2, 4, 2>(t, U, V, Z, g, s);
}

// Where the whole call runs this way (g: a slab), once contract_output.hip has not taken the layer: F(8,3); F(6,3) and F(4,5) from 129, F(4,3) and F(6,5) from
// 193 input channels on, F(2,5) from 129; fewer where the workgroups are too few for it (F(6,5) mostly); one block of output channels.  The rest of the
// layers below -- all of F(2,3) -- come here only with a y that lies over x or U, which a kernel that writes y while others read U cannot serve:
// there these figures are against the separate kernels.  A wave goes through n positions in turn where the separate contraction has
// a wave for each, so there have to be tiles and output channels enough to fill the chip without them, and the fewer input
// channels there are, the more of the time is M's.  Whole calls, separate kernels / this way, geometric means over 286
// layers by n * n * T * K (1.5-6 / 6-15 / 15-30 / 30-60 / more millions) and blocks of 32 input channels:
//   up to 2    n = 4: 1.01 / - / 1.25 / 1.20 / 1.48   6: 0.98 / 1.08 / 1.20 / - / 1.25   8: 0.93 / 1.05 / 1.10 / 1.22 / 1.44   10: 0.93 / 1.02 / 1.10 / 1.13 / 1.23
//   3, 4       n = 4: 0.99 / 1.12 / 1.22 / 1.19 / -   6: 0.91 / 1.04 / 1.14 / 1.20 / 1.18   8: 0.88 / 1.06 / 1.13 / 1.15 / 1.30   10: 0.85 / 0.99 / 1.07 / 1.14 / 1.22
//   5 to 8     n = 4: 0.87 / 1.11 / - / 0.97 / 1.06   6: 0.93 / 1.05 / 1.05 / 1.08 / 1.12   8: 0.78 / 1.04 / 1.05 / 1.01 / -   10: 0.73 / 1.02 / 0.96 / 0.95 / -
//   more       0.67-0.83 / 0.95-1.04 / 0.89-1.01
bool contract_columns_preferred(const nova_transforms *t, const Geometry &g, int dtype, int flags)
{
    if (dtype != NOVA_F16 || (flags & NOVA_FLAG_M_F16) || !t->symmetric || g.C <= few_channels_limit() || g.T > 0x7fffffffLL) return false;
    if ((size_t)g.k_blocks * g.Tp * kChanBlock * sizeof(float) >= ((size_t)1 << 32)) return false;             // (32-bit offsets inside a plane)
    const double products = (double)g.n * g.n * (double)g.T * g.Kp;
    // (n = 10 beside the streaming contraction with its U in registers, which starts at 24 M products: 128 -> 128 @28x28 batch 256 in
    // two slabs of 26 M, 141.9 us with it, 144.3 this way; 34 to 60 M products 1.00 to 1.15 times faster this way)
    if (g.n == 10) return g.c_blocks <= 4 && products >= (g.c_blocks == 4 && g.Kp % 128 == 0 ? 30e6 : 15e6);
    // F(6,3) from later on where there are many output channels, or few tiles for the same products: up to 14 M (a workgroup or two per
    // compute unit) these are 0.93 to 1.0 times as fast this way, with 5 blocks and more up to 20 M 0.97 to 1.1; 8 blocks and K a
    // multiple of 256 (the streaming contraction of 8 waves) 0.89 to 1.05 up to 45 M, 0.98 to 1.32 from there.  Of 1800 layers of
    // all n 1020 are taken, geometric mean 1.18; 21 are 0.93 to 0.98 times as fast, most of them F(6,3) with 192 to 224 channels.
    if (g.n == 8 && g.r == 3) {
        if (g.c_blocks == 8 && g.Kp % 256 == 0) return products >= 45e6;
        return g.c_blocks <= 8 && products >= (g.Kp > 256 ? (g.c_blocks < 5 ? 14e6 : 20e6) : g.c_blocks == 8 ? 13e6 : 10.5e6);
    }
    return g.c_blocks <= 8 && products >= 9e6;
}

int launch_contract_columns(const nova_transforms *t, const void *U, const void *V, void *Z, const Geometry &g, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (t->r == 3) {
        switch (t->n) {
        case 4: return launch_columns_n<4, 3>(t, U, V, Z, g, s);
        case 6: return launch_columns_n<6, 3>(t, U, V, Z, g, s);
        case 8: return launch_columns_n<8, 3>(t, U, V, Z, g, s);
        case 10: return launch_columns_n<10, 3>(t, U, V, Z, g, s);
        }
    } else if (t->r == 5) {
        switch (t->n) {
        case 6: return launch_columns_n<6, 5>(t, U, V, Z, g, s);
        case 8: return launch_columns_n<8, 5>(t, U, V, Z, g, s);
        case 10: return launch_columns_n<10, 5>(t, U, V, Z, g, s);
        }
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace nova
