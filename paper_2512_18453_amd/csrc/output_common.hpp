// What the output-transform kernels share: the 1D transform with A, the geometry of a tile group's
// output block in LDS, and the code that moves such a block to y.
#pragma once
#include <type_traits>

#include "device_common.hpp"

namespace nova {

// The 1D transform with A for points in the paired order (0, +a1, -a1, ..., infinity), in two steps that
// can be issued apart: sums and differences of the pairs, then one output at a time.
template <int N, int R>
__device__ __forceinline__ void output_transform_1d_pairs(const float (&v)[N], float (&s)[(N - 2) / 2 > 0 ? (N - 2) / 2 : 1],
                                                          float (&d)[(N - 2) / 2 > 0 ? (N - 2) / 2 : 1])
{
    constexpr int H = (N - 2) / 2;
#pragma unroll
    for (int j = 0; j < H; ++j) {
        s[j] = v[2 * j + 1] + v[2 * j + 2];
        d[j] = v[2 * j + 1] - v[2 * j + 2];
    }
}

// output i from the values at 0 and at infinity and the pairs' sums and differences
// (with unscaled rows zero = inf = pw[j][0] = 1 and these are plain sums)
template <int N, int R>
__device__ __forceinline__ float output_transform_1d_out(int i, float v_zero, float v_inf,
                                                         const float (&s)[(N - 2) / 2 > 0 ? (N - 2) / 2 : 1],
                                                         const float (&d)[(N - 2) / 2 > 0 ? (N - 2) / 2 : 1], const OutCoef<N, R> &k)
{
    constexpr int M = N - R + 1;
    constexpr int H = (N - 2) / 2;
    float acc = i == 0 ? k.zero * v_zero : (i == M - 1) ? k.inf * v_inf : 0.0f;
#pragma unroll
    for (int j = 0; j < H; ++j) acc = fma32(k.pw[j * M + i], (i & 1) ? d[j] : s[j], acc);
    if (M == 1) acc = fma32(k.inf, v_inf, acc);
    return acc;
}

// Outputs i and i + 1 as two binary16 values in a word, each rounded together with its last multiply-add: what the
// compiler makes of `(f16)output_transform_1d_out(...)` where nothing stands between the two (v_fma_mixlo_f16), spelled
// out where results have to be the same bits from several kernels.
template <int N, int R>
__device__ __forceinline__ unsigned output_transform_1d_f16_pair(int i, float v_zero, float v_inf,
                                                                 const float (&s)[(N - 2) / 2 > 0 ? (N - 2) / 2 : 1],
                                                                 const float (&d)[(N - 2) / 2 > 0 ? (N - 2) / 2 : 1], const OutCoef<N, R> &k)
{
    constexpr int M = N - R + 1, H = (N - 2) / 2;
    static_assert(M % 2 == 0 && H >= 1, "pairs of outputs");
    float acc[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        acc[e] = i + e == 0 ? k.zero * v_zero : (i + e == M - 1) ? k.inf * v_inf : 0.0f;
#pragma unroll
        for (int j = 0; j < H - 1; ++j) acc[e] = fma32(k.pw[j * M + i + e], e ? d[j] : s[j], acc[e]);      // (i is even)
    }
    unsigned word;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[0,0,0]" : "=v"(word) : "s"(k.pw[(H - 1) * M + i]), "v"(s[H - 1]), "v"(acc[0]));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel_hi:[0,0,0]" : "+v"(word) : "s"(k.pw[(H - 1) * M + i + 1]), "v"(d[H - 1]), "v"(acc[1]));
    return word;
}

template <int N, int R, bool SYM>
__device__ __forceinline__ void output_transform_1d(const float (&v)[N], float (&out)[N - R + 1], const OutCoef<N, R> &k)
{
    constexpr int M = N - R + 1;
    constexpr int H = (N - 2) / 2;
    if constexpr (SYM) {
        float s[H > 0 ? H : 1], d[H > 0 ? H : 1];
        output_transform_1d_pairs<N, R>(v, s, d);
#pragma unroll
        for (int i = 0; i < M; ++i) out[i] = output_transform_1d_out<N, R>(i, v[0], v[N - 1], s, d, k);
    } else {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            float acc = 0.0f;
#pragma unroll
            for (int p = 0; p < N; ++p) acc = fma32(k.a[p * M + i], v[p], acc);
            out[i] = acc;
        }
    }
}

// A row of M results to its place in the LDS block, in the widest pieces its alignment allows (M elements are a
// whole number of them; block pitches are multiples of 4 elements, tile columns multiples of M): a quarter to a
// half of the LDS instructions of element stores, and conversions two at a time.
template <int M>
__device__ __forceinline__ void store_block_row(f16 *dst, const float (&o)[M])
{
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    static_assert(M % 2 == 0, "whole pieces");
    if constexpr (M % 4 == 0) {
#pragma unroll
        for (int q = 0; q < M; q += 4)
            *reinterpret_cast<half4 *>(__builtin_assume_aligned(dst + q, 8)) = half4{(f16)o[q], (f16)o[q + 1], (f16)o[q + 2], (f16)o[q + 3]};
    } else {
#pragma unroll
        for (int q = 0; q < M; q += 2) *reinterpret_cast<half2v *>(__builtin_assume_aligned(dst + q, 4)) = half2v{(f16)o[q], (f16)o[q + 1]};
    }
}
template <int M>
__device__ __forceinline__ void store_block_row(float *dst, const float (&o)[M])
{
    typedef float float4v __attribute__((ext_vector_type(4)));
    typedef float float2v __attribute__((ext_vector_type(2)));
    if constexpr (M % 4 == 0) {
#pragma unroll
        for (int q = 0; q < M; q += 4)
            *reinterpret_cast<float4v *>(__builtin_assume_aligned(dst + q, 16)) = float4v{o[q], o[q + 1], o[q + 2], o[q + 3]};
    } else {
#pragma unroll
        for (int q = 0; q < M; q += 2) *reinterpret_cast<float2v *>(__builtin_assume_aligned(dst + q, 8)) = float2v{o[q], o[q + 1]};
    }
}

// The same for values already rounded, two to a word
template <int M>
__device__ __forceinline__ void store_block_words(f16 *dst, const unsigned (&w)[M / 2])
{
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    unsigned *at = reinterpret_cast<unsigned *>(__builtin_assume_aligned(dst, 4));
    if constexpr (M % 4 == 0) {
#pragma unroll
        for (int q = 0; q < M / 2; q += 2) *reinterpret_cast<u32x2 *>(__builtin_assume_aligned(at + q, 8)) = u32x2{w[q], w[q + 1]};
    } else {
#pragma unroll
        for (int q = 0; q < M / 2; ++q) at[q] = w[q];
    }
}

struct OutShape {
    int twb;          // tiles per group (all tile rows of the group together)
    int twc;          // tile columns per group
    int trb;          // tile rows per group
    int rows;         // output rows per group = trb * m
    int groups;       // tile groups per tile row
    int cols_pitch;   // LDS elements per output row of the group
    int k_pitch;      // LDS elements per channel
    int images;       // images per group (of which it takes all tiles then), in LDS one behind the other like further channels
    int batch;        // images of the call
    int pieces;       // kStoreFlat: 16-byte pieces that can touch one channel's run of rows * W elements
    unsigned piece_magic, w_magic;                 // ceil(2^32 / d) for d = pieces, W
    unsigned rows_magic, line_magic;               // ceil(2^32 / d) for d = rows, pieces of a row (0 for 1)
    int pool;         // 1: 2 x 2 max-pool while storing (H, W even)
    unsigned half_rows_magic;                      // ceil(2^32 / (rows / 2)), rows / 2 >= 2
};

// COUNT elements to an element-aligned address; NT: with the streaming cache hint
#define NOVA_STORE(type, at, value)                                                              \
    do {                                                                                         \
        type *nova_at_ = reinterpret_cast<type *>(at);                                           \
        if constexpr (NT) __builtin_nontemporal_store(value, nova_at_); else *nova_at_ = value;  \
    } while (0)
template <typename T, int COUNT, bool NT = false>
__device__ __forceinline__ void store_row(T *dst, const T (&v)[COUNT])
{
    constexpr int WORDS = COUNT * (int)sizeof(T) / 4;
    typedef unsigned int piece4 __attribute__((ext_vector_type(4), aligned(2)));
    typedef unsigned int piece3 __attribute__((ext_vector_type(3), aligned(2)));
    typedef unsigned int piece2 __attribute__((ext_vector_type(2), aligned(2)));
    typedef unsigned int piece1 __attribute__((aligned(2)));
    if constexpr (COUNT * (int)sizeof(T) % 4 != 0) {
#pragma unroll
        for (int e = 0; e < COUNT; ++e) dst[e] = v[e];
    } else {
        unsigned w[WORDS];
        __builtin_memcpy(w, v, WORDS * 4);
        unsigned char *at = reinterpret_cast<unsigned char *>(dst);
        constexpr int FOURS = WORDS / 4 * 4;
#pragma unroll
        for (int e = 0; e < FOURS; e += 4) NOVA_STORE(piece4, at + 4 * e, (piece4{w[e], w[e + 1], w[e + 2], w[e + 3]}));
        if constexpr (WORDS - FOURS == 3) NOVA_STORE(piece3, at + 4 * FOURS, (piece3{w[FOURS], w[FOURS + 1], w[FOURS + 2]}));
        if constexpr (WORDS - FOURS == 2) NOVA_STORE(piece2, at + 4 * FOURS, (piece2{w[FOURS], w[FOURS + 1]}));
        if constexpr (WORDS - FOURS == 1) NOVA_STORE(piece1, at + 4 * (WORDS - 1), w[WORDS - 1]);
    }
}
#undef NOVA_STORE

// The first `left` of COUNT elements (COUNT <= 8).  Rows cut off at the right edge leave this way from every kernel: element by element, four or five
// of six columns took up to half of a call (5 -> 350 @6x4 batch 1004 F(6,3) 61 us through contract_output.hip, 33 through LDS)
template <typename T, int COUNT>
__device__ __forceinline__ void store_row_part(T *dst, const T (&v)[COUNT], int left)
{
    if (left >= COUNT) {
        store_row<T, COUNT>(dst, v);
        return;
    }
    // pieces of 4, 2 and 1 elements; the values move up behind each
    T rest[COUNT];
#pragma unroll
    for (int e = 0; e < COUNT; ++e) rest[e] = v[e];
    if constexpr (COUNT > 4) {
        if (left & 4) {
            const T four[4] = {rest[0], rest[1], rest[2], rest[3]};
            store_row<T, 4>(dst, four);
            dst += 4;
#pragma unroll
            for (int e = 0; e + 4 < COUNT; ++e) rest[e] = rest[e + 4];
        }
    }
    if constexpr (COUNT > 2) {
        if (left & 2) {
            const T two[2] = {rest[0], rest[1]};
            store_row<T, 2>(dst, two);
            dst += 2;
            rest[0] = rest[2];
        }
    }
    if (left & 1) dst[0] = rest[0];
}
// How the block leaves LDS.
//   kStoreRows    a piece of an image row per thread (kRowPiece elements), neighbouring pieces in neighbouring lanes: any W, any group, any alignment
//   kStoreVec     W (and the group width) a multiple of a 16-byte piece, y 16-byte aligned: whole aligned pieces
//   kStoreFlat    the group spans the image width and y is 16-byte aligned: the rows of one channel are one contiguous run of y, written in
//                 aligned 16-byte pieces, gathered element by element, whatever W is (element stores at its two ends)
enum { kStoreRows = 0, kStoreVec = 1, kStoreFlat = 2 };
// Elements of a piece, a whole number of which the row pitch of the LDS block is: a tile's row, but four of m = 6 in binary32 (12-byte pieces 0.95 times
// as fast, 400 widths) and of m = 2 in binary16 (a tile's row there, 4 bytes, 0.97 with M in binary32, 0.95 in binary16).
template <typename T, int M> constexpr int kRowPiece = (sizeof(T) == 4 && M == 6) || (sizeof(T) == 2 && M == 2) ? 4 : M;

// Rows against the ways before them (kStoreFlat where a group spans the width, else element by element), the output transform alone, their time against
// rows: binary16 1.0 to 1.45 (spanning) and 1.0 to 1.9, products in binary16 0.95 to 1.8; binary32 0.8 to 1.4 and 1.0 to 1.6.  Flat stays for binary32
// where it is the faster one:
//   M and y of 192 MB or more, most of the last-level cache, past which its stores go.  Whole calls, 470 layers of 40 to 500 MB of M, flat over rows: up to
//   128 MB 1.01, 192 1.0, 256 0.88 to 1.05 (0.97), more 0.80 to 1.0 (0.90).  8 -> 350 @14x11 batch 350 F(4,3) 122 us in rows, 105 flat.
//   64 MB or more and a last tile of two or three columns (F(4,3)), any number (m = 6) or six and seven (m = 8, two tiles or more), where the transform
//   alone takes 0.77 to 1.06 (other numbers 0.97 to 1.2) and the whole call 1.0 to 1.02: 64 ch @50x50 batch 48 F(6,3) 23.4 and 19.9.
//   Images of one tile with at most half of its rows (m = 6 and 8: 0.79 to 1.0, with more 0.9 to 1.2).
//   Not F(8,3) of at most four input channels (1.0 to 1.3).

// The [32 channels][rows][columns] block of a group, staged in LDS (channel pitch sh.k_pitch, row pitch
// sh.cols_pitch), to y [N][K][H][W] (or its 2 x 2 max-pooled form): lanes along W.  Called by all
// threads of the workgroup after a barrier; img, kb (block of 32 channels), tr (first tile row of the
// group), tc0 (first tile column) say where the block sits.
template <typename T, int M, int STG>
__device__ __forceinline__ void store_output_block(const T *lds, T *__restrict__ y, int img, int kb, int tr, int tc0,
                                                   int K, int H, int W, int tiles_w, const OutShape &sh)
{
    constexpr int PE = 16 / (int)sizeof(T);
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const int w0 = tc0 * M;
    int cols = sh.twc * M;
    if (w0 + cols > W) cols = W - w0;
    if (sh.pool) {
        // 2 x 2 max-pool on the way out: rows, columns, H, W, tr*M and w0 are all even, so no window
        // straddles two groups.  One output element per thread and round, lanes along the pooled row.
        const int Hp = H / 2, Wp = W / 2, pcols = cols / 2, prows = sh.rows / 2;
        if constexpr (STG == kStoreVec && sizeof(T) == 2) {
            // W, w0 and cols are multiples of a 16-byte piece of y and y is 16-byte aligned.  If they are multiples
            // of two pieces, the pooled rows leave in 16-byte pieces too: a thread takes 2 rows x 16 columns.
            if (W % (2 * PE) == 0 && w0 % (2 * PE) == 0 && cols % (2 * PE) == 0) {
                const int pieces = pcols / PE;
                const unsigned magic = (unsigned)((((unsigned long long)1 << 32) + pieces - 1) / pieces);
                const int slots = kChanBlock * prows * pieces;
                for (int s = threadIdx.x; s < slots; s += (int)blockDim.x) {
                    const int line = pieces > 1 ? (int)__umulhi((unsigned)s, magic) : s;
                    const int q = s - line * pieces;
                    const int kk = prows > 1 ? (int)__umulhi((unsigned)line, sh.half_rows_magic) : line;
                    const int pp = line - kk * prows;
                    const int k = kb * kChanBlock + kk, hp = (tr * M) / 2 + pp;
                    if (k >= K || hp >= Hp) continue;
                    const T *top = lds + kk * sh.k_pitch + 2 * pp * sh.cols_pitch + 2 * q * PE;     // 8-byte aligned
                    const T *bottom = top + sh.cols_pitch;
                    T a[2 * PE], b[2 * PE], out[PE];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        reinterpret_cast<u32x2 *>(a)[e] = reinterpret_cast<const u32x2 *>(top)[e];
                        reinterpret_cast<u32x2 *>(b)[e] = reinterpret_cast<const u32x2 *>(bottom)[e];
                    }
#pragma unroll
                    for (int e = 0; e < PE; ++e) {
                        const float v0 = (float)a[2 * e], v1 = (float)a[2 * e + 1], v2 = (float)b[2 * e], v3 = (float)b[2 * e + 1];
                        float best = v0;                                  // a NaN in the window wins
                        best = (v1 > best || v1 != v1) ? v1 : best;
                        best = (v2 > best || v2 != v2) ? v2 : best;
                        best = (v3 > best || v3 != v3) ? v3 : best;
                        out[e] = (T)best;                                 // one of the four values: exact
                    }
                    u32x4 piece;
                    __builtin_memcpy(&piece, out, 16);
                    __builtin_nontemporal_store(piece, reinterpret_cast<u32x4 *>(y + (((size_t)img * K + k) * Hp + hp) * Wp + w0 / 2 + q * PE));
                }
                return;
            }
        }
        const unsigned pc_magic = (unsigned)((((unsigned long long)1 << 32) + pcols - 1) / pcols);
        const int slots = kChanBlock * prows * pcols;
        for (int s = threadIdx.x; s < slots; s += (int)blockDim.x) {
            const int line = pcols > 1 ? (int)__umulhi((unsigned)s, pc_magic) : s;
            const int qq = s - line * pcols;
            const int kk = prows > 1 ? (int)__umulhi((unsigned)line, sh.half_rows_magic) : line;
            const int pp = line - kk * prows;
            const int k = kb * kChanBlock + kk, hp = (tr * M) / 2 + pp;
            if (k >= K || hp >= Hp) continue;
            const T *win = lds + kk * sh.k_pitch + 2 * pp * sh.cols_pitch + 2 * qq;
            const float a = load_f32(win), b = load_f32(win + 1);
            const float c = load_f32(win + sh.cols_pitch), d = load_f32(win + sh.cols_pitch + 1);
            float best = a;                                   // a NaN in the window wins
            best = (b > best || b != b) ? b : best;
            best = (c > best || c != c) ? c : best;
            best = (d > best || d != d) ? d : best;
            store_from_f32(y + (((size_t)img * K + k) * Hp + hp) * Wp + w0 / 2 + qq, best);
        }
        return;
    }
    if constexpr (STG == kStoreVec) {
        // W, w0 and cols are multiples of PE and y is 16-byte aligned
        const int pieces = cols / PE;
        const unsigned magic = (unsigned)((((unsigned long long)1 << 32) + pieces - 1) / pieces);
        const int slots = kChanBlock * sh.rows * pieces;
        for (int s = threadIdx.x; s < slots; s += (int)blockDim.x) {
            const int line = pieces > 1 ? (int)__umulhi((unsigned)s, magic) : s;
            const int q = s - line * pieces;
            const int kk = (int)__umulhi((unsigned)line, sh.rows_magic), p = line - kk * sh.rows;
            const int k = kb * kChanBlock + kk, h = tr * M + p;
            if (k >= K || h >= H) continue;
            const u32x2 *in = reinterpret_cast<const u32x2 *>(lds + kk * sh.k_pitch + p * sh.cols_pitch + q * PE);
            const u32x2 lo = in[0], hi = in[1];
            u32x4 *dst = reinterpret_cast<u32x4 *>(y + (((size_t)img * K + k) * H + h) * W + w0 + q * PE);
            __builtin_nontemporal_store(u32x4{lo.x, lo.y, hi.x, hi.y}, dst);    // y is not read again by this call
        }
    } else if constexpr (STG == kStoreFlat) {
        // the group spans the width: rows h0 .. h1-1 of one channel are one run of y
        const int h0 = tr * M;
        int h1 = h0 + sh.rows; if (h1 > H) h1 = H;
        const int run = (h1 - h0) * W;
        const int slots = kChanBlock * sh.pieces;
        for (int s = threadIdx.x; s < slots; s += (int)blockDim.x) {
            const int kk = (int)__umulhi((unsigned)s, sh.piece_magic);
            const int kq = s - kk * sh.pieces;
            const int k = kb * kChanBlock + kk;
            if (k >= K) continue;
            const long long e0 = (((long long)img * K + k) * H + h0) * W;         // first element of the run
            const long long p0 = (e0 & ~(long long)(PE - 1)) + (long long)kq * PE;   // piece, aligned in y
            const int rel = (int)(p0 - e0);                                        // -(PE-1) .. run-1 if needed
            if (rel >= run) continue;
            // (row, column) of the piece's first element inside the run, then step along it
            const int q = rel < 0 ? 0 : rel;
            int hr = (int)__umulhi((unsigned)q, sh.w_magic);
            int w = q - hr * W;
            const T *src = lds + kk * sh.k_pitch;
            T val[PE];
#pragma unroll
            for (int e = 0; e < PE; ++e) {
                const int pos = rel + e;
                val[e] = (T)0.0f;
                if (pos >= 0 && pos < run) {
                    val[e] = src[hr * sh.cols_pitch + w];
                    if (++w == W) { w = 0; ++hr; }
                }
            }
            if (rel >= 0 && rel + PE <= run) {
                u32x4 piece;
                __builtin_memcpy(&piece, val, 16);
                __builtin_nontemporal_store(piece, reinterpret_cast<u32x4 *>(y + p0));
            } else {
#pragma unroll
                for (int e = 0; e < PE; ++e)
                    if (rel + e >= 0 && rel + e < run) y[p0 + e] = val[e];
            }
        }
    } else {
        constexpr int P = kRowPiece<T, M>;
        const int per_line = (sh.twc * M + P - 1) / P;
        const int slots = sh.images * kChanBlock * sh.rows * per_line;
        for (int s = threadIdx.x; s < slots; s += (int)blockDim.x) {
            const int line = per_line > 1 ? (int)__umulhi((unsigned)s, sh.line_magic) : s;
            const int w = (s - line * per_line) * P;
            const int plane = (int)__umulhi((unsigned)line, sh.rows_magic), p = line - plane * sh.rows;
            const int k = kb * kChanBlock + plane % kChanBlock, h = tr * M + p, image = img + plane / kChanBlock;
            if (k >= K || h >= H || w >= cols || image >= sh.batch) continue;
            T v[P];
            __builtin_memcpy(v, __builtin_assume_aligned(lds + plane * sh.k_pitch + p * sh.cols_pitch + w, P * sizeof(T) % 8 == 0 ? 8 : 4), P * sizeof(T));
            T *to = y + (((size_t)image * K + k) * H + h) * W + w0 + w;
            store_row_part<T, P>(to, v, cols - w);
        }
    }
}

// The larger of two values, of which a is the earlier one of its window: a NaN wins, and of a zero of either sign the
// earlier stays, as in the separate output transform's comparisons one after the other (elementwise maximum alone makes
// +0 of the two).  ZEROS: whether zeros of both signs can meet; where a ReLU leaves +0 only, the maximum alone will do.
template <bool ZEROS, typename T>
__device__ __forceinline__ T larger_of(T a, T b)
{
    const T top = __builtin_elementwise_maximum(a, b);
    if constexpr (ZEROS) return top == a ? a : top;
    return top;
}

// Rows [P0, P0 + ROWS) of a tile's outputs, rounded, 2 x 2 max-pooled to the image plane at `plane` (H, W, m even, so no
// window straddles two tiles).
template <typename T, int M, int P0, int ROWS, bool NT, bool ZEROS>
__device__ __forceinline__ void store_pooled_rows(const T (&out)[ROWS][M], T *plane, int tr, int tc, int H, int W)
{
    const int Hp = H / 2, Wp = W / 2, h0 = (tr * M + P0) / 2, w0 = tc * (M / 2);
    T *at = plane + (long long)h0 * Wp + w0;
#pragma unroll
    for (int p = 0; p < ROWS / 2; ++p) {
        if (h0 + p >= Hp) continue;
        T best[M / 2];
#pragma unroll
        for (int s = 0; s < M / 2; ++s)
            best[s] = larger_of<ZEROS>(larger_of<ZEROS>(out[2 * p][2 * s], out[2 * p][2 * s + 1]),
                                       larger_of<ZEROS>(out[2 * p + 1][2 * s], out[2 * p + 1][2 * s + 1]));
        if (w0 + M / 2 <= Wp) {
            store_row<T, M / 2, NT>(at + (long long)p * Wp, best);
        } else {
#pragma unroll
            for (int s = 0; s < M / 2; ++s)
                if (w0 + s < Wp) at[(long long)p * Wp + s] = best[s];
        }
    }
}

// Rows [P0, P0 + ROWS) of a tile's outputs, rounded, to the image plane at `plane`, or pooled; zeros: as ZEROS above.
template <typename T, int M, int P0, int ROWS, bool NT = false>
__device__ __forceinline__ void store_tile_rows(const T (&out)[ROWS][M], T *plane, int tr, int tc, int H, int W, bool pool, bool zeros)
{
    if (pool) {
        if (zeros) store_pooled_rows<T, M, P0, ROWS, NT, true>(out, plane, tr, tc, H, W);
        else store_pooled_rows<T, M, P0, ROWS, NT, false>(out, plane, tr, tc, H, W);
    } else {
        const int h0 = tr * M + P0, w0 = tc * M;
        T *at = plane + (long long)h0 * W + w0;
#pragma unroll
        for (int p = 0; p < ROWS; ++p) {
            if (h0 + p >= H) continue;
            if (w0 + M <= W) {
                store_row<T, M, NT>(at + (long long)p * W, out[p]);
            } else {
                store_row_part<T, M>(at + (long long)p * W, out[p], W - w0);
            }
        }
    }
}

// Results of 16 consecutive tiles and 32 channels (M x M binary16 values of each) that leave through LDS,
// [channel][tile][row][column], for narrow images: there neighbouring tiles are neighbours in few rows of y, so a store of one
// row per lane, the tiles in neighbouring lanes, touches a memory line of its own with almost every lane.  Here the
// rows of a tile go to neighbouring lanes, and rows of narrow images lie one behind the other.
template <int M>
struct TileRowsInLds {
    static constexpr int TILES = 16, CHANNELS = 32;
    static constexpr int PITCH = M * M + (M == 8 ? 8 : M == 4 ? 4 : 0);           // values of a tile: 16 tiles' rows in different banks
    static constexpr int BYTES = CHANNELS * TILES * PITCH * 2;
    static constexpr int ALIGN = M == 8 ? 16 : M == 4 ? 8 : 4;                    // bytes, of a row
    static constexpr int SLOTS = M > 4 ? 8 : M;                                   // lanes per tile
    static_assert(M == 2 || M == 4 || M == 6 || M == 8, "tile size");

    __device__ __forceinline__ static void put(f16 *block, int channel, int tile, int row, const f16 (&v)[M])
    {
        f16 *to = block + (channel * TILES + tile) * PITCH + row * M;
        __builtin_memcpy(__builtin_assume_aligned(to, ALIGN), v, M * 2);
    }

    // By 256 threads, after a barrier
    __device__ __forceinline__ static void store(const f16 *block, f16 *y, int k0, int K, int t0, int Ttot, int tiles_h, int tiles_w, int H, int W)
    {
        const int tid = (int)threadIdx.x, row = tid % SLOTS, tile = tid / SLOTS % TILES;
        const int t = t0 + tile, trow = t / tiles_w, tc = t - trow * tiles_w, img = trow / tiles_h, tr = trow - img * tiles_h;
        const int h = tr * M + row, w0 = tc * M, left = W - w0;
        if (t >= Ttot || row >= M || h >= H) return;
        constexpr int STEP = 256 / (SLOTS * TILES);                               // channels at a time
#pragma unroll 4
        for (int c = tid / (SLOTS * TILES); c < CHANNELS; c += STEP) {
            if (k0 + c >= K) break;
            f16 v[M];
            __builtin_memcpy(v, __builtin_assume_aligned(block + (c * TILES + tile) * PITCH + row * M, ALIGN), M * 2);
            f16 *to = y + (((long long)img * K + k0 + c) * H + h) * W + w0;
            store_row_part<f16, M>(to, v, left);
        }
    }
};

template <int N, int R>
static void fill_out_coef(const nova_transforms *t, OutCoef<N, R> &k)
{
    constexpr int M = N - R + 1, H = OutCoef<N, R>::H;
    for (int i = 0; i < N * M; ++i) k.a[i] = t->A32[i];
    for (int j = 0; j < H; ++j)
        for (int i = 0; i < M; ++i) k.pw[j * M + i] = t->A32[(2 * j + 1) * M + i];
    k.zero = t->A32[0];
    k.inf = t->A32[(N - 1) * M + (M - 1)];
}

template <int N, int R, typename T>
static size_t out_shape(int twb, int trb, OutShape &sh)
{
    constexpr int M = N - R + 1;
    sh.twb = twb * trb;
    sh.twc = twb;
    sh.trb = trb;
    sh.rows = trb * M;
    sh.rows_magic = (unsigned)((((unsigned long long)1 << 32) + sh.rows - 1) / sh.rows);
    sh.cols_pitch = (twb * M + 3) / 4 * 4;              // rows stay 8-byte aligned
    int kp = sh.rows * sh.cols_pitch;                   // multiple of 4
    // channel pitch 4 * odd elements: 8-byte aligned rows, and the 32 channels of a half-wave
    // writing one (row, column) fall into different banks
    if ((kp / 4) % 2 == 0) kp += 4;
    sh.k_pitch = kp;
    const int per_line = (twb * M + kRowPiece<T, M> - 1) / kRowPiece<T, M>;
    sh.pieces = 1; sh.piece_magic = 0; sh.w_magic = 0;
    sh.line_magic = per_line > 1 ? (unsigned)((((unsigned long long)1 << 32) + per_line - 1) / per_line) : 0;
    sh.images = 1;
    sh.pool = 0;
    sh.half_rows_magic = sh.rows / 2 > 1 ? (unsigned)((((unsigned long long)1 << 32) + sh.rows / 2 - 1) / (sh.rows / 2)) : 0;
    return (size_t)kChanBlock * kp * sizeof(T);
}


}  // namespace nova
