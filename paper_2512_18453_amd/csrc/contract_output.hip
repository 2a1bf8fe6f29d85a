// Contraction over input channels and output transform in one kernel (Sec. 2.1 steps 3 and 4), for layers of up to 256
// input channels with tiles and output channels enough to fill the chip: neither the products M nor half of their transform
// exists in memory (up to now contract_columns.hip and the row half of output_transform.hip, which write and read m of every n
// planes of M).  binary16, points in the paired order.  Products and sums are those of the separate kernels in the same order:
// the same bits.
//
// A workgroup of 4 waves takes 32 consecutive tiles of the batch (whatever tile rows and images they belong to) and 32 output
// channels, a wave 16 x 16 of them: the 16 x 16 matrix instruction leaves a lane 4 channels of one tile, whose 4 m^2 outputs it
// keeps in registers (n = 8: 144 of 256, two workgroups per compute unit).  The positions are visited column by column, n - 1
// and 0 first, then the pairs of columns of the points +a and -a; in a column the rows 0 and n - 1, then the pairs of rows: a
// stage is two positions x 64 input channels.  A pair's products enter the column's transform z through their sum and
// difference, a pair of columns' z the outputs in the same way (as in few_channels.hip).
// Stages arrive in a ring of S in LDS, S - 1 ahead, by direct global->LDS loads (a wave loads one of the stage's positions and
// blocks of 32 channels; rows of 64 bytes, XOR-swizzled by 16-byte piece, piece ^ (row / 2) % 4, for reads of 16 rows), one
// barrier per stage.  The stages of a column are unrolled; a stage's addresses are those of its column and an offset.
// Scratch per lane: 28 to 48 bytes (7 to 12 registers) with m = 6, none elsewhere; outside the stages, but for 5 x 5 with more than 64 input channels,
// which store and read back 6 or 7 registers for each pair of columns (and wait for all of the ring then).
// What bounds it: the units' time beside the waits.  64 stages, two workgroups per compute unit, 128 -> 128 @112x112 F(6,3), by counters: a
// wave takes 908 clocks per stage, 258 of them at barriers and for loads, 296 until a unit takes its next instruction; the two waves of a SIMD
// keep it busy with vector instructions for 287 clocks, scalar 232, matrix 128, and the loads of both workgroups take 512 at the 64 bytes per
// clock of L2 (0.84 of them hit).  HBM: 136 MB read, 15 written in 48.5 us, 3.1 TB/s; no bank conflicts.  That layer, batch 32, pooled: 97 us for 189 MB
// of V where contraction with columns and row transform took 152, whole call 231 -> 173.
// Tried: all n^2 products in registers (each operand then read by one wave only, no barriers), transformed at the end through
// LDS: 167 us, the transform's 70 of them beside nothing else; 8 waves with 32 x 64 per workgroup and compute unit, a quarter fewer
// loads: 112, 156 against 139 for the whole call 128 -> 256 batch 16; rings of 3 and 5: 110, 108; n = 10 (M = 8) with the 256 outputs of a
// lane in accumulation registers, added to by the matrix unit, one wave per SIMD: 64 -> 64 @224x224 196 us against 134 for fused_output.hip.
#include <algorithm>

#include "output_common.hpp"

namespace nova {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

// Four loads of 16 rows of 64 bytes, two from v and two from u, to four consecutive KiB of LDS
__device__ __forceinline__ void co_loads(const void *v, const unsigned (&v_off)[2], const void *u, const unsigned (&u_off)[2], unsigned lds)
{
    unsigned saved_m0;
#define NOVA_CO_NEXT(OFF, BASE) "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 " OFF ", " BASE "\n\t"
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %2\n\t"
                 NOVA_CO_NEXT("%5", "%2") NOVA_CO_NEXT("%6", "%3") NOVA_CO_NEXT("%7", "%3") "s_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "s"(lds), "s"(v), "s"(u), "v"(v_off[0]), "v"(v_off[1]), "v"(u_off[0]), "v"(u_off[1]) : "memory", "scc");
#undef NOVA_CO_NEXT
}

static size_t co_v_bytes(const Geometry &g) { return (size_t)g.n * g.n * g.c_blocks * (size_t)g.T * kChanBlock * sizeof(f16); }

// CHUNKS: stages of a pair of positions, 64 input channels each (an odd number of blocks of 32:
// half of the last one is not used); OCC: workgroups per compute unit; HINT: streaming hint for the rows of y that leave from registers
constexpr int WT = 2, WK = 2;      // waves of a workgroup: WT x WK of 16 tiles x 16 channels each; a wave loads one (position, channel block) of a stage's four

template <int N, int R, int CHUNKS, int S, int OCC, bool HINT>
__global__ void __launch_bounds__(64 * WT * WK, OCC)
contract_output_kernel(const f16 *__restrict__ U, const f16 *__restrict__ V, f16 *__restrict__ y, int K, int H, int W, int tiles_h,
                       int tiles_w, int Kp, int Ttot, int c_blocks, int k_groups, int flags, int narrow, OutCoef<N, R> coef)
{
    constexpr int M = N - R + 1, HP = (N - 2) / 2, STEPS = N / 2, TILES = 16 * WT, CHANNELS = 16 * WK;
    constexpr int PLANE = (TILES + CHANNELS) * 64, STAGE = 4 * PLANE;
    extern __shared__ __align__(1024) unsigned char ring[];
    const unsigned lds_base = (unsigned)(size_t)((__attribute__((address_space(3))) void *)ring);
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wt = wave / WK, wk = wave % WK;

    const unsigned bid = xcd_local_block_id(blockIdx.x, gridDim.x);
    const int kg = (int)(bid % (unsigned)k_groups), t0 = (int)(bid / (unsigned)k_groups) * TILES, k0 = kg * CHANNELS;

    // ---- loads: the wave's position (of the two) and channel block (of the two) of every stage
    const int my_pos = wave >> 1, my_cb = wave & 1;
    // a load is 16 rows: lane l -> row l / 4, place l % 4 (rows past the last tile: that again, its results are not stored)
    unsigned v_off[WT], u_off[WK];
    {
        const int row = lane >> 2;
        const unsigned piece = (unsigned)((lane & 3) ^ ((row >> 1) & 3)) * 16u;
#pragma unroll
        for (int i = 0; i < WT; ++i) v_off[i] = (unsigned)(t0 + i * 16 + row < Ttot ? i * 16 + row : Ttot - 1 - t0) * 64u + piece;
#pragma unroll
        for (int i = 0; i < WK; ++i) u_off[i] = (unsigned)(i * 16 + row) * 64u + piece;                      // (Kp is a multiple of 32)
    }
    // The stages of a column of positions, (step q, chunk c): step 0 takes the rows 0 and N - 1, step q the rows 2q - 1 and 2q.  Byte offsets
    // of the wave's operands from those of row 0 and channel block 0 of the column (32 bits: the launcher checks)
    constexpr int PER_COLUMN = STEPS * CHUNKS;
    const unsigned v_plane = (unsigned)Ttot * 64u, u_plane = (unsigned)Kp * 64u;
    const unsigned v_row = v_plane * (unsigned)(N * c_blocks), u_row = u_plane * (unsigned)(N * c_blocks);
    const unsigned last_block = (unsigned)(2 * (CHUNKS - 1) + my_cb < c_blocks ? 2 * (CHUNKS - 1) + my_cb : c_blocks - 1);   // (an odd number of blocks: the last again)
    auto offset_of = [&](int stage, unsigned row, unsigned plane) __attribute__((always_inline)) {
        const int q = stage / CHUNKS, c = stage % CHUNKS;
        return (unsigned)(q == 0 ? my_pos * (N - 1) : 2 * q - 1 + my_pos) * row + (c == CHUNKS - 1 ? last_block : (unsigned)(2 * c + my_cb)) * plane;
    };
    // Kept in a table; for m = 6 with more than 64 input channels, 16 to 30 scalars too many beside the others (47 to 127 scalar spills), each is worked
    // out when its loads are issued: F(6,3) 1.01 to 1.03 times as fast, 0.99 to 1.0 with pooling; F(6,5) 1.0 to 1.05; elsewhere 0.98 to 1.0.
    constexpr bool TABLE = M < 6 || CHUNKS == 1;
    unsigned v_stage[TABLE ? PER_COLUMN : 1], u_stage[TABLE ? PER_COLUMN : 1];
    if constexpr (TABLE) {
#pragma unroll
        for (int s = 0; s < PER_COLUMN; ++s) {
            v_stage[s] = (unsigned)__builtin_amdgcn_readfirstlane((int)offset_of(s, v_row, v_plane));
            u_stage[s] = (unsigned)__builtin_amdgcn_readfirstlane((int)offset_of(s, u_row, u_plane));
        }
    }
    auto stage_offset = [&](const unsigned *table, int s, unsigned row, unsigned plane) __attribute__((always_inline)) {
        if constexpr (TABLE) return table[s];
        asm volatile("" : "+s"(row), "+s"(plane));             // (not moved out of the loop over columns: the table again)
        return offset_of(s, row, plane);
    };
    const char *v_first = uniform_pointer(reinterpret_cast<const char *>(V) + (size_t)t0 * 64u), *u_first = uniform_pointer(reinterpret_cast<const char *>(U) + (size_t)k0 * 64u);
    const unsigned v_column = v_plane * (unsigned)c_blocks, u_column = u_plane * (unsigned)c_blocks;      // from one column to the next
    const char *v_col = v_first + (size_t)(N - 1) * v_column, *u_col = u_first + (size_t)(N - 1) * u_column;        // of the column loaded now
    int columns_left = N;
    const unsigned my_lds = (unsigned)__builtin_amdgcn_readfirstlane((int)(lds_base + (unsigned)(wave * PLANE)));
    // stage `s` of its column to place `slot`; past the last column its stages again, so that the wait counts are constants
    auto issue = [&](int s, int slot) __attribute__((always_inline)) {
        co_loads(v_col + stage_offset(v_stage, s, v_row, v_plane), v_off, u_col + stage_offset(u_stage, s, u_row, u_plane), u_off, my_lds + (unsigned)(slot * STAGE));
        if (s == PER_COLUMN - 1) {
            --columns_left;
            const bool first = columns_left == N - 1, more = columns_left > 0;
            v_col = first ? v_first : more ? v_col + v_column : v_col;
            u_col = first ? u_first : more ? u_col + u_column : u_col;
        }
    };

    const int f_row = lane & 15;
    const unsigned char *f_at = ring + f_row * 64 + (((lane >> 4) ^ ((f_row >> 1) & 3)) * 16);
    const unsigned char *vf_at = f_at + wt * 1024, *uf_at = f_at + TILES * 64 + wk * 1024;

    int slot = 0;
    const bool odd = (c_blocks & 1) != 0;
    // the products of the two positions of step q; `work`: between the reads of its first fragments and their use
    auto step = [&](auto q_tag, float4v (&m)[2], auto &&work) __attribute__((always_inline)) {
        constexpr int q = decltype(q_tag)::value;
        float4v acc[2];
        acc[0] = acc[1] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"((S - 2) * (WT + WK)) : "memory");
            __syncthreads();
            half8 vf[2][2], uf[2][2];
            const unsigned char *va = vf_at + slot * STAGE, *ua = uf_at + slot * STAGE;
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    vf[p][cb] = *reinterpret_cast<const half8 *>(va + (p * 2 + cb) * PLANE);
                    uf[p][cb] = *reinterpret_cast<const half8 *>(ua + (p * 2 + cb) * PLANE);
                }
            __builtin_amdgcn_sched_barrier(0);
            issue((q * CHUNKS + c + S - 1) % PER_COLUMN, slot == 0 ? S - 1 : slot - 1);
            if (c == 0) work();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(uf[p][0], vf[p][0], acc[p], 0, 0, 0);
            if (c < CHUNKS - 1 || !odd) {
#pragma unroll
                for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(uf[p][1], vf[p][1], acc[p], 0, 0, 0);
            }
            slot = slot == S - 1 ? 0 : slot + 1;
        }
        m[0] = acc[0];
        m[1] = acc[1];
    };
    // One column of positions: `first` with the products of step 0 (positions 0 and N - 1), then `pair` with the sums' operands of each pair
    auto column = [&](auto &&first, auto &&pair) __attribute__((always_inline)) {
        float4v m[2];
        static_for<STEPS>([&](auto q_tag) __attribute__((always_inline)) {
            constexpr int q = decltype(q_tag)::value;
            float4v next[2];
            step(q_tag, next, [&]() __attribute__((always_inline)) {
                if constexpr (q == 1) first(m);
                if constexpr (q > 1) pair(std::integral_constant<int, q - 2>{}, m);
            });
            m[0] = next[0];
            m[1] = next[1];
        });
        pair(std::integral_constant<int, STEPS - 2>{}, m);
    };

#pragma unroll
    for (int j = 0; j < S - 1; ++j) issue(j % PER_COLUMN, j);
    float Y[4][M][M], z0[4][M], z1[4][M];
    auto column1 = [&](float (&z)[4][M]) __attribute__((always_inline)) {
        column([&](const float4v (&m)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int p = 0; p < M; ++p) z[e][p] = p == 0 ? coef.zero * m[0][e] : p == M - 1 ? coef.inf * m[1][e] : 0.0f;
        }, [&](auto j_tag, const float4v (&m)[2]) __attribute__((always_inline)) {
            constexpr int j = decltype(j_tag)::value;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float s = m[0][e] + m[1][e], d = m[0][e] - m[1][e];
#pragma unroll
                for (int p = 0; p < M; ++p) z[e][p] = fma32(coef.pw[j * M + p], (p & 1) ? d : s, z[e][p]);
            }
        });
    };
    column1(z0);
    column1(z1);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int p = 0; p < M; ++p)
#pragma unroll
            for (int q = 0; q < M; ++q) Y[e][p][q] = q == 0 ? coef.zero * z1[e][p] : q == M - 1 ? coef.inf * z0[e][p] : 0.0f;
#pragma unroll 1
    for (int d = 0; d < HP - 1; ++d) {
        column1(z0);
        column1(z1);
        const float *c = coef.pw + d * M;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int p = 0; p < M; ++p) {
                const float s = z0[e][p] + z1[e][p], t = z0[e][p] - z1[e][p];
#pragma unroll
                for (int q = 0; q < M; ++q) Y[e][p][q] = fma32(c[q], (q & 1) ? t : s, Y[e][p][q]);
            }
    }
    column1(z0);
    column1(z1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    const bool relu = (flags & NOVA_FLAG_RELU) != 0, pool = (flags & NOVA_FLAG_POOL2) != 0;
    // the last pair of columns, rounded as the separate output transform does (without ReLU together with the last multiply-add)
    auto outputs = [&](int e, f16 (&out)[M][M]) __attribute__((always_inline)) {
        const float *c = coef.pw + (HP - 1) * M;
#pragma unroll
        for (int p = 0; p < M; ++p) {
            // (not moved in front of the branches that it is called in: sums and differences beside the columns would not fit the registers)
            asm volatile("" : "+v"(z0[e][p]));
            const float s = z0[e][p] + z1[e][p], d = z0[e][p] - z1[e][p];
#pragma unroll
            for (int q = 0; q < M; q += 2) {
                unsigned word;
                if (relu) {
                    float v0 = fma32(c[q], s, Y[e][p][q]), v1 = fma32(c[q + 1], d, Y[e][p][q + 1]);
                    asm volatile("" : "+v"(v0), "+v"(v1));
                    half2v pair = {(f16)v0, (f16)v1};
                    pair = __builtin_elementwise_maximum(pair, half2v{(f16)0.0f, (f16)0.0f});          // NaN stays NaN
                    word = __builtin_bit_cast(unsigned, pair);
                } else {
                    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[0,0,0]" : "=v"(word) : "s"(c[q]), "v"(s), "v"(Y[e][p][q]));
                    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel_hi:[0,0,0]" : "+v"(word) : "s"(c[q + 1]), "v"(d), "v"(Y[e][p][q + 1]));
                }
                __builtin_memcpy(&out[p][q], &word, 4);
            }
        }
    };
    const int channel = wk * 16 + 4 * (lane >> 4);             // the lane's first, of the workgroup's
    if (narrow) {                                              // the results leave through LDS, 16 tiles at a time
        static_assert(CHANNELS == TileRowsInLds<M>::CHANNELS && 64 * WT * WK == 256 && TileRowsInLds<M>::BYTES <= S * STAGE, "block");
        f16 *block = reinterpret_cast<f16 *>(ring);
#pragma unroll 1
        for (int part = 0; part < WT; ++part) {
            __syncthreads();                                   // the operands, or the part before, have been read
            if (wt == part) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    f16 out[M][M];
                    outputs(e, out);
#pragma unroll
                    for (int p = 0; p < M; ++p) TileRowsInLds<M>::put(block, channel + e, lane & 15, p, out[p]);
                }
            }
            __syncthreads();
            TileRowsInLds<M>::store(block, y, k0, K, t0 + part * 16, Ttot, tiles_h, tiles_w, H, W);
        }
        return;
    }
    // rows of m elements straight from registers, neighbouring tiles in neighbouring lanes
    const int t = t0 + wt * 16 + (lane & 15);
    if (t >= Ttot) return;
    const int trow = t / tiles_w, tc = t - trow * tiles_w, img = trow / tiles_h, tr = trow - img * tiles_h;
    const long long plane = pool ? (long long)(H / 2) * (W / 2) : (long long)H * W;
    f16 *at = y + ((long long)img * K + k0 + channel) * plane;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f16 out[M][M];
        outputs(e, out);
        if (k0 + channel + e < K) store_tile_rows<f16, M, 0, M, HINT>(out, at + e * plane, tr, tc, H, W, pool, !relu);
    }
}

template <int N, int R, int CHUNKS, int S, int OCC>
static int launch_co_chunks(const nova_transforms *t, const void *U, const void *V, void *y, const Geometry &g, int flags, hipStream_t stream)
{
    constexpr int M = N - R + 1;
    OutCoef<N, R> coef;
    fill_out_coef<N, R>(t, coef);
    const int k_groups = g.Kp / (16 * WK);
    const long long blocks = (g.T + 16 * WT - 1) / (16 * WT) * k_groups;
    if (blocks <= 0 || blocks > 0x7fffffffLL || g.c_blocks > 2 * CHUNKS) return (int)hipErrorInvalidValue;
    // Results through LDS only where rows from registers take two pieces each for the last tile (3 or 5 columns), in images of one or two tiles' width
    // of whose tile rows more than half exist.  Time of the call with it / from registers, 700 layers: there 0.71 to 1.08 (m = 6, geometric
    // mean 0.93), 0.75 to 1.03 (m = 4, 0.91); with half of the rows or fewer 1.0 to 1.45 (most of a tile's lanes have no row: 24 -> 60 @2x2
    // batch 3205 F(6,3) 28.0 us / 21.2); other numbers of columns 1.0 to 1.3; wider images 1.0 to 1.3; m = 2 1.0 to 1.1.
    const int last_columns = g.W - M * (g.tiles_w - 1);
    const bool narrow = M > 2 && !(flags & NOVA_FLAG_POOL2) && g.tiles_w <= 2 && last_columns % 2 == 1 && last_columns >= 3 && 2 * g.H > M * g.tiles_h;
    // Streaming hint for rows of 12 bytes as in fused_output.hip, in images of three tiles or more (80 -> 128 5x5 @13x19 batch 1852, V and y 259 MB,
    // 366 us with it, 389 without; 72 -> 161 @4x6 batch 14517, 277 MB, 457 / 218).  Shorter rows never: 128 -> 256 @3x4 batch 7006 F(4,3)
    // 210 us with it, 87 without.  (Pooled rows of m = 6 leave value by value, without it.)
    auto kern = contract_output_kernel<N, R, CHUNKS, S, OCC, false>;
    if constexpr (M == 6) {
        constexpr size_t kCacheBytes = (size_t)256 << 20;
        if (g.W > 2 * M && co_v_bytes(g) + (size_t)g.N * g.K * g.H * g.W * sizeof(f16) > kCacheBytes) kern = contract_output_kernel<N, R, CHUNKS, S, OCC, true>;
    }
    constexpr int LDS = S * 4 * (WT + WK) * 1024;
    static_assert(LDS * OCC <= 160 * 1024, "LDS of the workgroups of a compute unit");
    if (LDS >= 64 * 1024) NOVA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS));
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * WT * WK), LDS, stream, (const f16 *)U, (const f16 *)V, (f16 *)y, g.K, g.H, g.W, g.tiles_h,
                       g.tiles_w, g.Kp, (int)g.T, g.c_blocks, k_groups, flags, narrow ? 1 : 0, coef);
    return (int)hipGetLastError();
}

// Input channels from which on the separate kernels are as fast again (in blocks of 32), and workgroups it takes to be faster than
// all else.  789 layers (33 to 256 -> 16 to 512 channels, 0.8 to 100 M products, all n but F(8,3)), time of the other paths -- one
// kernel, columns, separate -- against this one by workgroups:
//   n = 4          up to 350 0.7-1.0, from 400 on 1.1-2.0 (up to 128 channels), 1.0-1.4 (up to 256)
//   n = 6, r = 3   up to 140 0.6-1.0, from 144 on 1.0-1.65 (up to 128 channels; up to 64 from 256 on: 64 -> 64 @224x224, 196, 0.85), 1.0-1.2 (up to 192, from 200 on), 0.9-1.1 (up to 256)
//   n = 8, r = 3   up to 150 0.5-0.95, from 160 on 1.0-1.7 (up to 128 channels; 64 the same as fused_output.hip, which has them), 0.9-1.2 above
//   n = 6, r = 5   up to 130 0.55-0.9, from 136 on 1.0-1.4 (up to 128), 0.8-1.1 above
//   n = 8, r = 5   up to 130 0.5-1.0, from 144 on 1.0-1.6 (up to 128), 0.8-1.1 above
//   n = 10, r = 5  from 236 on 1.25-1.7 (up to 64), from 368 on 1.0-1.3 (up to 128), from 500 on 1.1-1.5 (up to 192), less below
// One block of output channels 0.45-1.06: not taken.  (Workgroups on the whole chip, 256 compute units; partitions of it
// were not timed.)
struct CoRange { int max_blocks, workgroups[3]; };     // (up to 2 blocks of input channels, 4, more)
static CoRange co_range(int n, int r)
{
    if (r == 3) return n == 4 ? CoRange{8, {400, 400, 400}} : n == 6 ? CoRange{6, {256, 144, 200}} : n == 8 ? CoRange{4, {180, 172, 0}} : CoRange{};
    if (r == 5) return n == 6 ? CoRange{4, {140, 140, 0}} : n == 8 ? CoRange{4, {144, 144, 0}} : n == 10 ? CoRange{6, {236, 368, 500}} : CoRange{};
    return CoRange{};
}

static bool co_applies(const nova_transforms *t, const Geometry &g, int dtype, int flags)
{
    const CoRange range = co_range(t->n, t->r);
    return dtype == NOVA_F16 && !(flags & NOVA_FLAG_M_F16) && t->symmetric && g.C > few_channels_limit() && g.c_blocks <= range.max_blocks &&
           g.T <= 0x7fffffffLL && co_v_bytes(g) < ((size_t)1 << 32) && (size_t)g.n * g.n * g.c_blocks * g.Kp * 64 < ((size_t)1 << 32);
}

bool contract_output_preferred(const nova_transforms *t, const Geometry &g, int dtype, int flags)
{
    if (!co_applies(t, g, dtype, flags) || g.Kp == 32) return false;
    const CoRange range = co_range(t->n, t->r);
    return (g.T + 31) / 32 * g.k_blocks >= range.workgroups[g.c_blocks <= 2 ? 0 : g.c_blocks <= 4 ? 1 : 2];
}

int launch_contract_output(const nova_transforms *t, const void *U, const void *V, void *y, const Geometry &g, int flags, void *stream)
{
    if (!co_applies(t, g, NOVA_F16, flags)) return (int)hipErrorInvalidValue;
    hipStream_t s = (hipStream_t)stream;
    const int chunks = (g.c_blocks + 1) / 2;
#define NOVA_CO(N, R, CHUNKS, S, OCC) launch_co_chunks<N, R, CHUNKS, S, OCC>(t, U, V, y, g, flags, s)
    if (t->r == 3) {
        switch (t->n) {
        case 4: return chunks == 1 ? NOVA_CO(4, 3, 1, 3, 3) : chunks == 2 ? NOVA_CO(4, 3, 2, 3, 3) : chunks == 3 ? NOVA_CO(4, 3, 3, 3, 3) : NOVA_CO(4, 3, 4, 3, 3);
        case 6: return chunks == 1 ? NOVA_CO(6, 3, 1, 4, 2) : chunks == 2 ? NOVA_CO(6, 3, 2, 4, 2) : NOVA_CO(6, 3, 3, 4, 2);
        case 8: return chunks == 1 ? NOVA_CO(8, 3, 1, 4, 2) : NOVA_CO(8, 3, 2, 4, 2);
        }
    } else if (t->r == 5) {
        switch (t->n) {
        case 6: return chunks == 1 ? NOVA_CO(6, 5, 1, 3, 3) : NOVA_CO(6, 5, 2, 3, 3);
        case 8: return chunks == 1 ? NOVA_CO(8, 5, 1, 4, 2) : NOVA_CO(8, 5, 2, 4, 2);
        case 10: return chunks == 1 ? NOVA_CO(10, 5, 1, 4, 2) : chunks == 2 ? NOVA_CO(10, 5, 2, 4, 2) : NOVA_CO(10, 5, 3, 4, 2);
        }
    }
#undef NOVA_CO
    return (int)hipErrorInvalidValue;
}

}  // namespace nova
