// INT8 operands in the Winograd domain (Sec. 4.1 "INT8 Setup"; "CNN Quantization Setup"): the
// transformed weights U and the transformed input tiles V are quantised symmetrically -- scale
// s = max|.| / 127 per tensor, per output channel for U, or per Winograd-domain position; code = value / s rounded to nearest even,
// saturated to [-128, 127] -- and the channel contraction runs on the integer codes,
//     Mi[xi][t][k] = sum_c Vq[xi][t][c] * Uq[xi][k][c]        (exact, 32-bit accumulators),
// on the matrix cores (v_mfma_i32_32x32x32_i8).  The transforms themselves stay in floating point.
//
// Layouts as in the floating-point path, one byte per element: Uq [n*n][C/32][Kp][32],
// Vq [n*n][C/32][T][32]; Mi [n*n][K/32][Tp][32] of int32, or M of the same shape in binary32 with
// M = fl(fl(Mi) * fl(s_U[k] * s_V)).
// Every floating-point step that decides a code is binary32 and correctly rounded: s = max / 127,
// code = rint(value / s); a tensor or channel that is all zero has s = 1.
#include "device_common.hpp"

namespace nova {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int16v __attribute__((ext_vector_type(16)));

__global__ void __launch_bounds__(256)
fill_u32_kernel(unsigned *dst, unsigned value, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = value;
}

// which scale an 8-element piece p belongs to.  kind 0: the only one; 1: its row index inside a
// (position, channel block) plane; 2: its position xi (plane_pieces = pieces per position)
__device__ __forceinline__ int scale_index(long long p, int kind, int rows, long long plane_pieces)
{
    return kind == 0 ? 0 : kind == 1 ? (int)((p >> 2) % rows) : (int)(p / plane_pieces);
}

__device__ __forceinline__ float scale_of(unsigned top_bits)
{
    const float top = __uint_as_float(top_bits);
    return top > 0.0f ? __fdiv_rn(top, 127.0f) : 1.0f;
}

__device__ __forceinline__ float block_max(float m)
{
    __shared__ float per_wave[16];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) per_wave[threadIdx.x >> 6] = m;
    __syncthreads();
    float all = 0.0f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) all = fmaxf(all, per_wave[w]);
    return all;
}

template <typename T>
__device__ __forceinline__ float piece_max(const T *at, float m)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(load_f32(at + e)));
    return m;
}

// Largest magnitude per row index k over all planes [positions * channel blocks][rows][32]: one workgroup per
// row, result stored as it is (one atomic per piece, as before, took 144 us for 128 -> 128 channels at n = 6;
// this form 5 us).
template <typename T>
__global__ void __launch_bounds__(256)
absmax_rows_kernel(const T *__restrict__ src, unsigned *__restrict__ top, long long planes, int rows)
{
    const int row = (int)blockIdx.x;
    float m = 0.0f;
    for (long long q = threadIdx.x; q < planes * 4; q += 256) m = piece_max(src + (((q >> 2) * rows + row) * 4 + (q & 3)) * 8, m);
    m = block_max(m);
    if (threadIdx.x == 0) top[row] = __float_as_uint(m);
}

// Largest magnitudes of `segments` equal runs of seg_pieces pieces: a run is shared by blocks_per_seg workgroups
// with one atomic each on the run's result (for non-negative binary32 numbers the order of the values is the
// order of their bit patterns).  An atomic per wave of 8-element pieces on one address took 11 ns apiece,
// 162 us for the V of 128 ch @28x28 batch 32.
template <typename T>
__global__ void __launch_bounds__(512)
absmax_runs_kernel(const T *__restrict__ src, unsigned *__restrict__ top, long long seg_pieces, int blocks_per_seg)
{
    const int seg = (int)blockIdx.x / blocks_per_seg, part = (int)blockIdx.x - seg * blocks_per_seg;
    const T *run = src + (size_t)seg * seg_pieces * 8;
    float m = 0.0f;
    for (long long p = (long long)part * 512 + threadIdx.x; p < seg_pieces; p += (long long)blocks_per_seg * 512) m = piece_max(run + p * 8, m);
    m = block_max(m);
    if (threadIdx.x == 0 && m > 0.0f) atomicMax(top + seg, __float_as_uint(m));
}

__device__ __forceinline__ unsigned code_of(float value, float s)
{
    float q = __builtin_rintf(__fdiv_rn(value, s));         // ties to even
    q = q < -128.0f ? -128.0f : (q > 127.0f ? 127.0f : q);
    return (unsigned)((int)q & 0xff);
}

template <typename T>
__global__ void __launch_bounds__(256)
quantize_kernel(const T *__restrict__ src, signed char *__restrict__ dst, const unsigned *__restrict__ top,
                long long pieces, int rows, int valid, int kind, long long plane_pieces)
{
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < pieces; p += (long long)gridDim.x * blockDim.x) {
        // (rows beyond `valid` are padding: all zero, and without a scale of their own)
        const int idx = scale_index(p, kind, rows, plane_pieces);
        const float s = scale_of(idx < valid ? top[idx] : 0u);
        const T *at = src + p * 8;
        unsigned lo = 0, hi = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned byte = code_of(load_f32(at + e), s);
            if (e < 4) lo |= byte << (8 * e); else hi |= byte << (8 * (e - 4));
        }
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u32x2 *>(dst + p * 8) = u32x2{lo, hi};
    }
}

// top (bit patterns of the largest magnitudes) -> scales, in place
__global__ void __launch_bounds__(256)
finish_scales_kernel(unsigned *top_then_scale, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) top_then_scale[i] = __float_as_uint(scale_of(top_then_scale[i]));
}

// src: [positions][channel blocks][rows][32]; kind 0: one scale; 1: one per row index below n_scales (the
// other rows are zero padding); 2: one per position (n_scales = positions)
template <typename T>
static int quantize_rows(const void *src, void *dst, void *scales, long long elements, int rows, int n_scales,
                         int kind, long long plane_pieces, hipStream_t stream)
{
    const long long pieces = elements / 8;                  // rows are 32 elements: always whole pieces
    long long want = (pieces + 255) / 256;
    const unsigned blocks = (unsigned)(want < 1 ? 1 : want > 4096 ? 4096 : want);
    hipLaunchKernelGGL(fill_u32_kernel, dim3((n_scales + 255) / 256), dim3(256), 0, stream, (unsigned *)scales, 0u, n_scales);
    if (kind == 1) {
        hipLaunchKernelGGL(absmax_rows_kernel<T>, dim3(n_scales), dim3(256), 0, stream, (const T *)src, (unsigned *)scales,
                           pieces / 4 / rows, rows);
    } else {
        // (about two workgroups per compute unit over all runs)
        const long long seg_pieces = kind == 2 ? plane_pieces : pieces;
        int per_seg = ceil_div(512, n_scales);
        if (per_seg > (seg_pieces + 511) / 512) per_seg = (int)((seg_pieces + 511) / 512);
        hipLaunchKernelGGL(absmax_runs_kernel<T>, dim3((unsigned)n_scales * per_seg), dim3(512), 0, stream, (const T *)src,
                           (unsigned *)scales, seg_pieces, per_seg);
    }
    hipLaunchKernelGGL(quantize_kernel<T>, dim3(blocks), dim3(256), 0, stream, (const T *)src, (signed char *)dst,
                       (const unsigned *)scales, pieces, rows, n_scales, kind, plane_pieces);
    hipLaunchKernelGGL(finish_scales_kernel, dim3((n_scales + 255) / 256), dim3(256), 0, stream, (unsigned *)scales, n_scales);
    return (int)hipGetLastError();
}

int launch_quantize_int8(const void *src, void *dst, void *scales, long long elements, int positions, int rows,
                         int n_scales, int kind, int dtype, void *stream)
{
    if (positions < 1 || rows < 1 || elements % ((long long)positions * rows * kChanBlock) != 0) return (int)hipErrorInvalidValue;
    if ((kind == 0 && n_scales != 1) || (kind == 1 && (n_scales < 1 || n_scales > rows)) || (kind == 2 && n_scales != positions) ||
        kind < 0 || kind > 2)
        return (int)hipErrorInvalidValue;
    const long long plane_pieces = elements / positions / 8;
    return dtype == NOVA_F16 ? quantize_rows<f16>(src, dst, scales, elements, rows, n_scales, kind, plane_pieces, (hipStream_t)stream)
                             : quantize_rows<float>(src, dst, scales, elements, rows, n_scales, kind, plane_pieces, (hipStream_t)stream);
}

// ---- contraction.  A workgroup of 4 waves owns a BM x BN tile of one Mi[xi]; a step moves 32 channels
// (one 32x32x32 matrix instruction per pair of 32-row blocks) through double-buffered LDS, rows padded
// from 32 to 48 bytes so that the 16 lanes of a 128-bit read phase fall into different bank groups.
// The two halves of a wave supply the two 16-channel halves of a row; the sum over the 32 channels of
// a step does not depend on how the instruction orders them, as long as both operands use the same
// order -- they do: both are read with the same row and half-row indexing.
//   VT = signed char: Vq holds codes.  VT = the storage type: V itself, quantised on the way into LDS with
//   the scale of the tensor (or position), which every workgroup forms from the `partials` the input
//   transform left: partial maxima (per position with scale_kind 2).
//   Saves a pass that reads V, one that reads V and writes the codes, and the atomics: 128 ch @28x28
//   batch 32 n = 6, whole call: 208 us with an atomic per wave in the maximum, about 50 with the separate
//   passes as they are now, 33 this way.  Per position 7600 -> 40.
// U supplies the rows of the instruction and V the columns: a lane then holds four neighbouring output
// channels per store.
constexpr int kRowBytes8 = 48;

// partial maxima of one run: count of them, `step` apart; runs (one per position with scale_kind 2) `pitch` apart
struct MaximaRuns { int count, step, pitch; };

template <typename VT> struct Codes16 {               // 16 values of V on their way to 16 codes
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    static constexpr int PIECES = (int)sizeof(VT);
    u32x4 raw[PIECES];
    __device__ __forceinline__ void load(const VT *src)
    {
#pragma unroll
        for (int q = 0; q < PIECES; ++q) raw[q] = reinterpret_cast<const u32x4 *>(src)[q];
    }
    // The codes for scale s, inv = fl(1 / s).  value * inv is within 2^-23 of the quotient, so it rounds to the same
    // integer unless it lies within 127 * 2^-23 = 1.6e-5 of a tie; a lane that has such a value (or one that is
    // not finite) divides.  Adding 1.5 * 2^23 rounds to an integer, ties to even, and leaves its code in
    // the low byte: 5 instructions per value instead of 20.
    __device__ __forceinline__ u32x4 codes(float s, float inv) const
    {
        if constexpr (sizeof(VT) == 1) {
            return raw[0];
        } else {
            VT val[16];
            __builtin_memcpy(val, raw, sizeof(val));
            constexpr float kRound = 12582912.0f;
            u32x4 out;
            bool sure = true;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned bits[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = load_f32(&val[4 * q + e]) * inv, r = p + kRound;
                    sure = sure && fabsf(p - (r - kRound)) < 0.5f - 2.0e-5f;
                    bits[e] = __float_as_uint(r);
                }
                out[q] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(bits[3], bits[2], 0x0c0c0400u),
                                               __builtin_amdgcn_perm(bits[1], bits[0], 0x0c0c0400u), 0x05040100u);
            }
            if (!sure) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    out[q] = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[q] |= code_of(load_f32(&val[4 * q + e]), s) << (8 * e);
                }
            }
            return out;
        }
    }
};

template <int BM, int BN, int WM, int WN, bool DEQUANT, typename VT>
__global__ void __launch_bounds__(256)
contract_i8_kernel(const signed char *__restrict__ Uq, const VT *__restrict__ Vq, void *__restrict__ Mo,
                   const float *__restrict__ u_scales, const float *__restrict__ v_scale, MaximaRuns runs, int scale_kind,
                   int T, int Tp, int Kp, int K, int c_blocks, int k_blocks, int row_blocks, int col_blocks)
{
    constexpr int MB = BM / WM / 32, NB = BN / WN / 32;
    static_assert(WM * WN == 4 && BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "tile shape");
    static_assert(BM * 2 <= 256 && BN * 2 <= 256, "one 16-code segment per thread and operand");
    __shared__ __align__(16) signed char lds_a[2][BM * kRowBytes8];
    __shared__ __align__(16) signed char lds_b[2][BN * kRowBytes8];

    unsigned bid = xcd_local_block_id(blockIdx.x, gridDim.x);
    const int cbk = bid % col_blocks; bid /= col_blocks;
    const int rbk = bid % row_blocks; bid /= row_blocks;
    const int xi = bid;
    const int t0 = rbk * BM, k0 = cbk * BN;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WN, wn = wave % WN;

    // segment s of an operand tile: row s/2, 16-channel half s%2; rows beyond the tensor are clamped to the
    // last valid row (their products are never stored)
    const int row = tid >> 1, halfrow = tid & 1;
    const bool has_a = tid < BM * 2, has_b = tid < BN * 2;
    int ta = t0 + row; if (ta > T - 1) ta = T - 1;
    int kb_row = k0 + row; if (kb_row > Kp - 1) kb_row = Kp - 1;
    const VT *a_src = Vq + ((size_t)xi * c_blocks * T + ta) * kChanBlock + halfrow * 16;
    const signed char *b_src = Uq + ((size_t)xi * c_blocks * Kp + kb_row) * kChanBlock + halfrow * 16;
    const size_t a_step = (size_t)T * kChanBlock, b_step = (size_t)Kp * kChanBlock;
    const int dst_off = row * kRowBytes8 + halfrow * 16;

    int16v acc[NB][MB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][i][e] = 0;

    Codes16<VT> a_reg;
    Codes16<signed char> b_reg;
    auto load_global = [&](int cb) {
        if (has_a) a_reg.load(a_src + cb * a_step);
        if (has_b) b_reg.load(b_src + cb * b_step);
    };
    load_global(0);
    // scale_kind 0: one scale each; 1: U per output channel; 2: both per position
    float sv = 0.0f, inv = 0.0f;
    if constexpr (sizeof(VT) > 1) {
        float m = 0.0f;
        const float *parts = v_scale + (scale_kind == 2 ? (size_t)xi * runs.pitch : 0);
        for (int p = tid; p < runs.count; p += 256) m = fmaxf(m, parts[(size_t)p * runs.step]);
        sv = scale_of(__float_as_uint(block_max(m)));
        inv = __fdiv_rn(1.0f, sv);
    } else if constexpr (DEQUANT) {
        sv = v_scale[scale_kind == 2 ? xi : 0];
    }
    auto store_lds = [&](int buf) {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        if (has_a) *reinterpret_cast<u32x4 *>(&lds_a[buf][dst_off]) = a_reg.codes(sv, inv);
        if (has_b) *reinterpret_cast<u32x4 *>(&lds_b[buf][dst_off]) = b_reg.codes(0.0f, 0.0f);
    };
    store_lds(0);
    __syncthreads();

    const int frag_row = lane & 31, frag_half = (lane >> 5) * 16;
    for (int cb = 0; cb < c_blocks; ++cb) {
        const int buf = cb & 1;
        if (cb + 1 < c_blocks) load_global(cb + 1);
        int4v af[MB], bf[NB];
#pragma unroll
        for (int i = 0; i < MB; ++i)
            af[i] = *reinterpret_cast<const int4v *>(&lds_a[buf][((wm * MB + i) * 32 + frag_row) * kRowBytes8 + frag_half]);
#pragma unroll
        for (int j = 0; j < NB; ++j)
            bf[j] = *reinterpret_cast<const int4v *>(&lds_b[buf][((wn * NB + j) * 32 + frag_row) * kRowBytes8 + frag_half]);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < MB; ++i)
                acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[i], bf[j], acc[j][i], 0, 0, 0);
        if (cb + 1 < c_blocks) store_lds(buf ^ 1);
        __syncthreads();
    }

    // D[row = t][col = k]: lane holds channel lane % 32 of a block and tiles 8 (e / 4) + 4 (lane / 32) + e % 4; a store covers two
    // whole 128-byte rows of M
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int kb = (k0 >> 5) + wn * NB + j;
        if (kb >= k_blocks) continue;
        float both = 0.0f;
        if constexpr (DEQUANT) {
            const int k = kb * kChanBlock + frag_row;
            both = u_scales[scale_kind == 1 ? (k < K ? k : K - 1) : scale_kind == 2 ? xi : 0] * sv;
        }
        int *plane = reinterpret_cast<int *>(Mo) + ((size_t)xi * k_blocks + kb) * (size_t)Tp * kChanBlock + frag_row;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int t = t0 + (wm * MB + i) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                if (t < T) plane[(size_t)t * kChanBlock] = DEQUANT ? __float_as_int((float)acc[j][i][e] * both) : acc[j][i][e];
            }
    }
}

template <bool DEQUANT, typename VT>
static int launch_ci8(const void *Uq, const void *Vq, void *Mo, const float *u_scales, const float *v_scale, MaximaRuns runs,
                      int scale_kind, const Geometry &g, hipStream_t stream)
{
    constexpr int BM = 64, BN = 128;         // (128 rows: 1-4 % slower on every shape timed)
    const int row_blocks = ceil_div((int)g.T, BM), col_blocks = ceil_div(g.Kp, BN);
    const long long blocks = (long long)g.n * g.n * row_blocks * col_blocks;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL((contract_i8_kernel<BM, BN, 2, 2, DEQUANT, VT>), dim3((unsigned)blocks), dim3(256), 0, stream,
                       (const signed char *)Uq, (const VT *)Vq, Mo, u_scales, v_scale, runs, scale_kind,
                       (int)g.T, (int)g.Tp, g.Kp, g.K, g.c_blocks, g.k_blocks, row_blocks, col_blocks);
    return (int)hipGetLastError();
}

int launch_contract_int8(const void *Uq, const void *Vq, void *Mo, const void *u_scales, const void *v_scale,
                         int scale_kind, int dequantise, const Geometry &g, void *stream)
{
    if (g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    const float *us = (const float *)u_scales, *vs = (const float *)v_scale;
    return dequantise ? launch_ci8<true, signed char>(Uq, Vq, Mo, us, vs, MaximaRuns{}, scale_kind, g, (hipStream_t)stream)
                      : launch_ci8<false, signed char>(Uq, Vq, Mo, us, vs, MaximaRuns{}, scale_kind, g, (hipStream_t)stream);
}

// Slices of kSlice partial maxima of each of gridDim.y runs folded in place into the slice's first entry.
constexpr int kSlice = 2048;
__global__ void __launch_bounds__(256)
fold_maxima_kernel(float *maxima, int n_part)
{
    float *run = maxima + (size_t)blockIdx.y * n_part;
    const int first = (int)blockIdx.x * kSlice, last = n_part - first < kSlice ? n_part : first + kSlice;
    float m = 0.0f;
    for (int p = first + (int)threadIdx.x; p < last; p += 256) m = fmaxf(m, run[p]);
    m = block_max(m);
    if (threadIdx.x == 0) run[first] = m;
}

// Contraction of V itself (de-quantised products), its scale formed from the partial maxima of the input transform.
// A workgroup reads up to 2 * kSlice of them by itself (16 per thread, from L2); beyond that they are folded
// first: a launch, on a layer of more than 60 us.
int launch_contract_int8_of_v(const void *Uq, const void *V, void *Mo, const void *u_scales, float *partials, int n_part,
                              int scale_kind, const Geometry &g, int dtype, void *stream)
{
    if (g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipStream_t s = (hipStream_t)stream;
    MaximaRuns runs = {n_part, 1, n_part};
    if (n_part > 2 * kSlice) {
        runs.count = ceil_div(n_part, kSlice);
        runs.step = kSlice;
        hipLaunchKernelGGL(fold_maxima_kernel, dim3((unsigned)runs.count, scale_kind == 2 ? g.n * g.n : 1), dim3(256), 0, s,
                           partials, n_part);
    }
    const float *us = (const float *)u_scales;
    return dtype == NOVA_F16 ? launch_ci8<true, f16>(Uq, V, Mo, us, partials, runs, scale_kind, g, s)
                             : launch_ci8<true, float>(Uq, V, Mo, us, partials, runs, scale_kind, g, s);
}

}  // namespace nova
