// Products and output transform for layers of at most 4 input channels (the first layer of an image network) in
// binary16, points in the paired order (Sec. 2.1 steps 3 and 4).  V comes in the compact layout Vc [n*n][T][4] and the filters'
// first channels packed, Uc [n*n][Kp][4]; M is never formed in memory.
//
// A workgroup of 4 waves takes 16 consecutive tiles (whatever tile rows and images they belong to) and 32 output
// channels, whose operands it stages in LDS.  The products of a position -- 4 channels long -- are one v_mfma_f32_4x4x4_16b_f16:
// of its sixteen 4 x 4 blocks, block b covers channels 4 (b / 4) .. + 3 and tiles 4 (b % 4) .. + 3, so a lane is left with 4
// channels of tile lane % 16 and every product it makes is used.
// Four pairs' outputs would not fit a lane's registers; but in a column's transform the even outputs take only the
// sums of the (+a, -a) rows and the odd ones only their differences, so two waves share the pairs, one with the even output
// rows, one with the odd ones, and no addition or multiplication is done twice (the products are; the matrix unit has
// the time).  Column by column: transformed to the wave's m / 2 rows, columns of +a and -a folded into the outputs together.  The order
// of every sum is the separate output transform's.  Rows of m elements leave straight from registers, neighbouring tiles
// in neighbouring lanes.
// What bounds it: vector instructions, 1900 per lane and wave at n = 10 (4 pairs, half of their rows), about 40 us on 3 -> 64 @224x224
// batch 32 F(8,3), beside the 42 us that its 205 MB of y take; 61 us in all.  Products as multiply-add chains on the vector
// unit, one pair per thread and the output block through LDS (the kernel for other points and binary32 still,
// output_transform.hip) took 110.  On the way: as below but operands read column by column when needed 67, cropping and
// comparisons per store and a select for the ReLU 72.
// The matrix unit's sum of 4 products is nearer to 64 bits than the chain's (relative error 2.3e-8 against 2.7e-8).
#include <algorithm>

#include "output_common.hpp"

namespace nova {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kFewTiles = 16, kFewGroup = 32;      // tiles and output channels of a workgroup

// The wave's M / 2 output rows (p = HALF, HALF + 2, ..) of its lane's 4 pairs.  u, v: the lane's operands of position 0 in LDS.
template <int N, int R, int HALF, bool ROUND_M>
__device__ __forceinline__ void few_outputs(const half4 *u, const half4 *v, float (&Y)[4][(N - R + 1) / 2][N - R + 1], const OutCoef<N, R> &k)
{
    constexpr int M = N - R + 1, H = (N - 2) / 2, MH = M / 2;
    half4 uf[N], vf[N];                       // operands of the column taken next: read while this one is transformed
    auto read = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uf[i] = u[(i * N + j) * kFewGroup];
            vf[i] = v[(i * N + j) * kFewTiles];
        }
    };
    auto column = [&](int next, float (&z)[4][MH]) __attribute__((always_inline)) {
        float4v m[N];
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = __builtin_amdgcn_mfma_f32_4x4x4f16(uf[i], vf[i], float4v{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
        if (next >= 0) read(next);
        // (what is further ahead would take the registers that the outputs need)
        if constexpr (N >= 8) __builtin_amdgcn_sched_barrier(0);
        auto product = [&](int i, int e) __attribute__((always_inline)) { return ROUND_M ? (float)round_twice(m[i][e], (f16 *)nullptr) : m[i][e]; };
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float sd[H];
#pragma unroll
            for (int q = 0; q < H; ++q) sd[q] = HALF ? product(2 * q + 1, e) - product(2 * q + 2, e) : product(2 * q + 1, e) + product(2 * q + 2, e);
#pragma unroll
            for (int pi = 0; pi < MH; ++pi) {
                const int p = 2 * pi + HALF;
                float acc = p == 0 ? k.zero * product(0, e) : p == M - 1 ? k.inf * product(N - 1, e) : 0.0f;
#pragma unroll
                for (int q = 0; q < H; ++q) acc = fma32(k.pw[q * M + p], sd[q], acc);
                z[e][pi] = acc;
            }
        }
        if constexpr (N >= 8) __builtin_amdgcn_sched_barrier(0);
    };
    float z0[4][MH], z1[4][MH];
    read(N - 1);
    column(0, z0);
    column(1, z1);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int pi = 0; pi < MH; ++pi)
#pragma unroll
            for (int q = 0; q < M; ++q) Y[e][pi][q] = q == 0 ? k.zero * z1[e][pi] : q == M - 1 ? k.inf * z0[e][pi] : 0.0f;
#pragma unroll
    for (int d = 0; d < H; ++d) {
        column(2 * d + 2, z0);
        column(d + 1 < H ? 2 * d + 3 : -1, z1);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int pi = 0; pi < MH; ++pi) {
                const float s = z0[e][pi] + z1[e][pi], t = z0[e][pi] - z1[e][pi];
#pragma unroll
                for (int q = 0; q < M; ++q) Y[e][pi][q] = fma32(k.pw[d * M + q], (q & 1) ? t : s, Y[e][pi][q]);
            }
    }
}

template <int N, int R, bool ROUND_M, bool POOL>
__global__ void __launch_bounds__(256, 2)
few_channels_kernel(const f16 *__restrict__ Vc, const f16 *__restrict__ Uc, f16 *__restrict__ y, int K, int H, int W, int tiles_h, int tiles_w,
                    int Kp, int Ttot, int k_groups, int relu, int narrow, OutCoef<N, R> coef)
{
    constexpr int M = N - R + 1, MH = M / 2, N2 = N * N, THREADS = 256;
    // Streaming hint for the rows, but not for those of 12 bytes: 3 -> 64 @224x224 batch 32 F(6,3) 66 us without, 72 as 8 + 4 bytes
    // with it, 128 with it on 12 (the fused 64-channel kernel decides by the size of V and y)
    constexpr bool kHint = M != 6;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    half4 *Vs = reinterpret_cast<half4 *>(lds_raw), *Us = Vs + N2 * kFewTiles;        // [position][16 tiles], [position][32 channels]

    const unsigned bid = xcd_local_block_id(blockIdx.x, gridDim.x);
    const int kg = (int)(bid % (unsigned)k_groups), t0 = (int)(bid / (unsigned)k_groups) * kFewTiles;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // all loads of the operands in flight together
    const half4 *Vg = reinterpret_cast<const half4 *>(Vc), *Ug = reinterpret_cast<const half4 *>(Uc);
    constexpr int NV = (N2 * kFewTiles + THREADS - 1) / THREADS, NU = (N2 * kFewGroup + THREADS - 1) / THREADS;
    {
        half4 v[NV], u[NU];
        const int t = t0 + (tid & 15) < Ttot ? t0 + (tid & 15) : Ttot - 1;        // (slots past the last tile: the last one again)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int xi = (tid >> 4) + i * (THREADS / kFewTiles);
            v[i] = Vg[(size_t)(xi < N2 ? xi : N2 - 1) * Ttot + t];
        }
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int xi = (tid >> 5) + i * (THREADS / kFewGroup);
            u[i] = Ug[(size_t)(xi < N2 ? xi : N2 - 1) * Kp + kg * kFewGroup + (tid & 31)];
        }
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (tid + i * THREADS < N2 * kFewTiles) Vs[tid + i * THREADS] = v[i];
#pragma unroll
        for (int i = 0; i < NU; ++i)
            if (tid + i * THREADS < N2 * kFewGroup) Us[tid + i * THREADS] = u[i];
    }
    __syncthreads();

    const half4 *v_at = Vs + (lane & 15), *u_at = Us + (wave >> 1) * 16 + 4 * (lane >> 4) + (lane & 3);
    const int half = wave & 1;
    float Y[4][MH][M];
    if (half == 0) few_outputs<N, R, 0, ROUND_M>(u_at, v_at, Y, coef);
    else few_outputs<N, R, 1, ROUND_M>(u_at, v_at, Y, coef);

    const int t = t0 + (lane & 15), trow = t / tiles_w, tc = t - trow * tiles_w, img = trow / tiles_h, tr = trow - img * tiles_h;
    const int k0 = kg * kFewGroup + (wave >> 1) * 16 + 4 * (lane >> 4);               // the lane's first channel
    const bool active = t < Ttot;
    f16 out[4][MH][M];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int pi = 0; pi < MH; ++pi)
#pragma unroll
            for (int q = 0; q < M; q += 2) {
                // (rounded in a step of its own, as round_twice does, so that pooled and plain calls agree bit for bit)
                asm volatile("" : "+v"(Y[e][pi][q]), "+v"(Y[e][pi][q + 1]));
                half2v pair = {(f16)Y[e][pi][q], (f16)Y[e][pi][q + 1]};
                if (relu) pair = __builtin_elementwise_maximum(pair, half2v{(f16)0.0f, (f16)0.0f});         // NaN stays NaN
                out[e][pi][q] = pair[0];
                out[e][pi][q + 1] = pair[1];
            }
    if constexpr (!POOL) {
        if (narrow) {                             // the results leave through LDS
            f16 *block = reinterpret_cast<f16 *>(lds_raw);
            __syncthreads();                      // the operands have been read
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int pi = 0; pi < MH; ++pi)
                    TileRowsInLds<M>::put(block, (wave >> 1) * 16 + 4 * (lane >> 4) + e, lane & 15, 2 * pi + half, out[e][pi]);
            __syncthreads();
            TileRowsInLds<M>::store(block, y, kg * kFewGroup, K, t0, Ttot, tiles_h, tiles_w, H, W);
            return;
        }
        const int w0 = tc * M, h0 = tr * M;
        f16 *plane = y + (((long long)img * K + k0) * H + h0) * W + w0;
        if (__all(active && k0 + 4 <= K && h0 + M <= H && w0 + M <= W)) {             // nothing to crop in the whole wave
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int pi = 0; pi < MH; ++pi) store_row<f16, M, kHint>(plane + ((long long)e * H + 2 * pi + half) * W, out[e][pi]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int pi = 0; pi < MH; ++pi) {
                    const int p = 2 * pi + half;
                    if (!active || k0 + e >= K || h0 + p >= H) continue;
                    f16 *row = plane + ((long long)e * H + p) * W;
                    if (w0 + M <= W) {
                        store_row<f16, M, kHint>(row, out[e][pi]);
                    } else {
#pragma unroll
                        for (int q = 0; q < M; ++q)
                            if (w0 + q < W) row[q] = out[e][pi][q];
                    }
                }
        }
    } else {
        // 2 x 2 max-pool (H, W, m even): the wave with the odd rows hands their pairwise maxima over
        auto pooled = [&](auto zeros) __attribute__((always_inline)) {
            auto larger = [](f16 a, f16 b) __attribute__((always_inline)) { return larger_of<decltype(zeros)::value>(a, b); };
            f16 row_max[4][MH][MH];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int pi = 0; pi < MH; ++pi)
#pragma unroll
                    for (int q = 0; q < MH; ++q) row_max[e][pi][q] = larger(out[e][pi][2 * q], out[e][pi][2 * q + 1]);
            f16 *handed = reinterpret_cast<f16 *>(lds_raw) + (wave >> 1) * (4 * MH * MH * 64) + lane;
            static_assert(2 * 4 * MH * MH * 64 * 2 <= N2 * (kFewTiles + kFewGroup) * 8, "what is handed over takes the operands' place");
            __syncthreads();                      // the operands have been read
            if (half == 1) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int pi = 0; pi < MH; ++pi)
#pragma unroll
                        for (int q = 0; q < MH; ++q) handed[((e * MH + pi) * MH + q) * 64] = row_max[e][pi][q];
            }
            __syncthreads();
            if (half == 0 && active) {
                const int Hp = H / 2, Wp = W / 2, w0 = tc * MH;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    f16 *plane = y + (((long long)img * K + k0 + e) * Hp + tr * MH) * Wp + w0;
#pragma unroll
                    for (int pi = 0; pi < MH; ++pi) {
                        if (k0 + e >= K || tr * MH + pi >= Hp) continue;
                        f16 best[MH];
#pragma unroll
                        for (int q = 0; q < MH; ++q) best[q] = larger(row_max[e][pi][q], handed[((e * MH + pi) * MH + q) * 64]);
                        if (w0 + MH <= Wp) {
                            store_row<f16, MH, true>(plane + (long long)pi * Wp, best);
                        } else {
#pragma unroll
                            for (int q = 0; q < MH; ++q)
                                if (w0 + q < Wp) plane[(long long)pi * Wp + q] = best[q];
                        }
                    }
                }
            }
        };
        if (relu) pooled(std::false_type{});                // (no -0 is left)
        else pooled(std::true_type{});
    }
}

template <int N, int R>
static int launch_few(const nova_transforms *t, const void *Vc, const void *Uc, void *y, const Geometry &g, int flags, hipStream_t stream)
{
    if (g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    OutCoef<N, R> coef;
    fill_out_coef<N, R>(t, coef);
    const int k_groups = g.Kp / kFewGroup;
    const long long blocks = (g.T + kFewTiles - 1) / kFewTiles * k_groups;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    const bool round_m = (flags & NOVA_FLAG_M_F16) != 0, pool = (flags & NOVA_FLAG_POOL2) != 0;
    auto kern = round_m ? (pool ? few_channels_kernel<N, R, true, true> : few_channels_kernel<N, R, true, false>)
                        : (pool ? few_channels_kernel<N, R, false, true> : few_channels_kernel<N, R, false, false>);
    // Results through LDS (TileRowsInLds): time of the call with it against rows straight from registers, 280 layers of 2 to
    // 224 columns: where tiles overhang the right edge 1.05 to 3.2 times as fast in up to 30 columns, up to 40 still 1.0 to 1.65 but
    // for F(6,3), whose 12-byte rows store as fast then (0.93 to 1.01); up to two whole tiles 0.97 to 2.6 (F(2,3) 0.92); 0.7 to
    // 1.2 in more.  (Pooled as well it gained 0.98 to 1.07.)
    const bool narrow = !pool && g.W <= (g.m == 6 ? 30 : 40) && (g.W % g.m != 0 || (g.m > 2 && g.tiles_w <= 2));
    constexpr int M = N - R + 1, OPERANDS = N * N * (kFewTiles + kFewGroup) * 8;
    const int lds_bytes = narrow ? std::max(OPERANDS, TileRowsInLds<M>::BYTES) : OPERANDS;
    if (lds_bytes > 64 * 1024)
        NOVA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), (size_t)lds_bytes, stream, (const f16 *)Vc, (const f16 *)Uc,
                       (f16 *)y, g.K, g.H, g.W, g.tiles_h, g.tiles_w, g.Kp, (int)g.T, k_groups, (flags & NOVA_FLAG_RELU) ? 1 : 0, narrow ? 1 : 0, coef);
    return (int)hipGetLastError();
}

int launch_few_channels_f16(const nova_transforms *t, const void *Vc, const void *Uc, void *y, const Geometry &g, int flags, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (t->r == 3) {
        switch (t->n) {
        case 4: return launch_few<4, 3>(t, Vc, Uc, y, g, flags, s);
        case 6: return launch_few<6, 3>(t, Vc, Uc, y, g, flags, s);
        case 8: return launch_few<8, 3>(t, Vc, Uc, y, g, flags, s);
        case 10: return launch_few<10, 3>(t, Vc, Uc, y, g, flags, s);
        }
    } else if (t->r == 5) {
        switch (t->n) {
        case 6: return launch_few<6, 5>(t, Vc, Uc, y, g, flags, s);
        case 8: return launch_few<8, 5>(t, Vc, Uc, y, g, flags, s);
        case 10: return launch_few<10, 5>(t, Vc, Uc, y, g, flags, s);
        }
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace nova
