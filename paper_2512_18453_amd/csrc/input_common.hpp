// What the kernels that transform input tiles share: the 1D transform with B^T in the contracted order, the
// windows of a group of tiles in LDS, and the code that brings them there from x [N][C][H][W].
#pragma once
#include "device_common.hpp"

namespace nova {

// Rows [LO, HI) of one 1D transform: out[p - LO] = sum_a B^T[p][a] v[a] in the contracted order.
// With SYM the range must not cut a (+a, -a) pair of rows (rows 2q+1, 2q+2).
template <int N, bool SYM, int LO, int HI>
__device__ __forceinline__ void input_transform_rows(const float (&v)[N], float (&out)[HI - LO], const InCoef<N> &k)
{
    constexpr int H = (N - 2) / 2;
    if constexpr (SYM) {
        if constexpr (LO == 0) {
            float e0 = 0.0f;
#pragma unroll
            for (int q = 0; q <= H; ++q) e0 = fma32(k.zero[q], v[2 * q], e0);
            out[0] = e0;
        }
#pragma unroll
        for (int j = 0; j < H; ++j) {
            if (2 * j + 1 >= LO && 2 * j + 2 < HI) {
                float E = 0.0f, O = 0.0f;
#pragma unroll
                for (int q = 0; q < H; ++q) E = fma32(k.ev[j * H + q], v[2 * q + 2], E);
#pragma unroll
                for (int q = 0; q < H; ++q) O = fma32(k.od[j * H + q], v[2 * q + 1], O);
                out[2 * j + 1 - LO] = E + O;
                out[2 * j + 2 - LO] = E - O;
            }
        }
        if constexpr (HI == N) {
            float oi = 0.0f;
#pragma unroll
            for (int q = 0; q <= H; ++q) oi = fma32(k.inf[q], v[2 * q + 1], oi);
            out[N - 1 - LO] = oi;
        }
    } else {
#pragma unroll
        for (int p = LO; p < HI; ++p) {
            float E = 0.0f, O = 0.0f;
#pragma unroll
            for (int a = 0; a < N; a += 2) E = fma32(k.bt[p * N + a], v[a], E);
#pragma unroll
            for (int a = 1; a < N; a += 2) O = fma32(k.bt[p * N + a], v[a], O);
            out[p - LO] = E + O;
        }
    }
}

// Where the rows are split between two threads (or waves) that share a tile: half 0 takes rows
// [0, SP), half 1 rows [SP, N); SP is odd so that no (+a, -a) pair of rows is cut.
template <int N> struct RowSplit { static constexpr int value = ((N / 2) % 2 == 1) ? N / 2 : N / 2 + 1; };

// The windows of TB tiles that are neighbours in t (whatever tile rows and images they belong to) and of one block
// of CH channels, for TB * (words per pixel) * RS threads.  A word of LDS holds one pixel of CPT channels: two
// neighbouring channels in binary16, one in binary32.  RS threads share the transform rows of one tile and word.
template <int N, typename T, int CH, int TB_, int RS_>
struct TileWindows {
    static constexpr int CPT = 4 / (int)sizeof(T);              // channels per word
    static constexpr int GP = CH / CPT;                         // words per pixel of a channel block
    static constexpr int TB = TB_, RS = RS_;
    // rows [bound(i), bound(i + 1)) are thread i's; no (+a, -a) pair (2q + 1, 2q + 2) is cut
    static constexpr int bound(int i) { return i == 0 ? 0 : i == RS ? N : RS == N / 2 ? 2 * i + 1 : RowSplit<N>::value; }
    static constexpr int RUN = TB < 16 ? TB : 16;               // neighbouring tiles whose lanes exchange columns (16: a DPP row)
    static constexpr int THREADS = TB * GP * RS;
    static constexpr int TILE_PAD = 2;
    // Pitches in words.  The window reads take two pixels (8 bytes) per lane, 32 lanes (two tiles' 16 windows, or
    // one tile's 32) per phase: with a window pitch of 2 * odd 8-byte units (binary32: odd) and a tile pitch of
    // an odd number of them, the lanes fall into different banks.
    static constexpr int WIN = CPT == 2 ? ((N * N / 4) % 2 == 1 ? N * N : N * N + 4) : N * N + 2;
    static constexpr int TILE = GP * WIN + TILE_PAD;
    static constexpr int LDS_BYTES = TB * TILE * 4;
    static_assert(WIN % 2 == 0 && N % RS == 0 && (RS <= 2 || RS == N / 2) && (TB * GP) % 64 == 0, "block shape");
};

// COUNT words of x from any (element-aligned) address; STREAM: with the streaming cache hint.
// (The hint is an argument of the builtin, not of a type: the element-aligned vector types below would lose
// their alignment as template arguments.)
#define NOVA_LOAD_X(at) (STREAM ? __builtin_nontemporal_load(at) : *(at))
template <bool STREAM, int COUNT>
__device__ __forceinline__ void load_words(const void *src, unsigned (&w)[COUNT])
{
    typedef unsigned int piece4 __attribute__((ext_vector_type(4), aligned(2)));
    typedef unsigned int piece3 __attribute__((ext_vector_type(3), aligned(2)));
    typedef unsigned int piece2 __attribute__((ext_vector_type(2), aligned(2)));
    typedef unsigned int piece1 __attribute__((aligned(2)));
    const char *at = reinterpret_cast<const char *>(src);
    constexpr int FOURS = COUNT / 4 * 4;
#pragma unroll
    for (int e = 0; e < FOURS; e += 4) {
        const piece4 *p = reinterpret_cast<const piece4 *>(at + 4 * e);
        const piece4 v = NOVA_LOAD_X(p);
#pragma unroll
        for (int q = 0; q < 4; ++q) w[e + q] = v[q];
    }
    if constexpr (COUNT - FOURS == 3) {
        const piece3 *p = reinterpret_cast<const piece3 *>(at + 4 * FOURS);
        const piece3 v = NOVA_LOAD_X(p);
        w[FOURS] = v[0]; w[FOURS + 1] = v[1]; w[FOURS + 2] = v[2];
    } else if constexpr (COUNT - FOURS == 2) {
        const piece2 *p = reinterpret_cast<const piece2 *>(at + 4 * FOURS);
        const piece2 v = NOVA_LOAD_X(p);
        w[FOURS] = v[0]; w[FOURS + 1] = v[1];
    } else if constexpr (COUNT - FOURS == 1) {
        const piece1 *p = reinterpret_cast<const piece1 *>(at + 4 * FOURS);
        w[FOURS] = NOVA_LOAD_X(p);
    }
}
template <bool STREAM> __device__ __forceinline__ unsigned element_bits(const float *p) { return __float_as_uint(NOVA_LOAD_X(p)); }
template <bool STREAM> __device__ __forceinline__ unsigned element_bits(const f16 *p)
{
    const unsigned short *bits = reinterpret_cast<const unsigned short *>(p);
    return (unsigned)NOVA_LOAD_X(bits);
}
#undef NOVA_LOAD_X

// A thread's part of staging the windows of B: window rows (channel word g, row a) of one tile, with the tiles of
// the group in neighbouring lanes, so that a load runs along image rows and the columns a window shares with its
// neighbours come from the lanes beside it.  The M elements loaded are aligned to an element only.
// load() brings a channel block's rows into registers, place() puts them into LDS; the two may be far apart.
// KEEP: the items' addresses are worked out once (keep_addresses()) and kept in registers, for kernels that load several
// channel blocks.
template <int N, int R, typename T, typename B, bool KEEP>
struct WindowRows {
    static constexpr int M = N - R + 1;                          // outputs per tile side = tile stride
    static constexpr int PAD = (R - 1) / 2;                      // zero border of the convolution
    static constexpr int CPT = B::CPT, CH = B::GP * B::CPT;
    static constexpr int ITEMS = N / B::RS;                      // window rows a thread stages
    static constexpr int WORDS = M * (int)sizeof(T) / 4;         // words of a tile's own columns in one row

    int j, tc, h_lo, w0, img;                                    // the thread's tile: slot, tile column, first row and column, image
    bool first_lane, last_lane, right_edge;
    bool loaded_tail;                                            // what near_end() said of the block loaded last
    struct Item { int off, chan, dst; };                         // its row in x (elements) and in LDS (words), first channel
    Item kept[KEEP ? ITEMS : 1];
    unsigned raw[ITEMS][CPT][WORDS], halo[ITEMS][CPT][PAD];

    // the slots from `count` on are given the last tile again; their windows are never used
    __device__ __forceinline__ void place_tile(int t0, int count, int tiles_h, int tiles_w)
    {
        j = (int)threadIdx.x % B::TB;
        const int t = t0 + (j < count ? j : count - 1);
        const int trow = t / tiles_w;
        tc = t - trow * tiles_w;
        img = trow / tiles_h;
        h_lo = (trow - img * tiles_h) * M - PAD;
        w0 = tc * M;
        // the first tile of a run of lanes loads its left halo, the last one the right one (never the same tile: a run
        // has several; lanes past the group's last tile load it again)
        first_lane = j % B::RUN == 0;
        last_lane = j % B::RUN == B::RUN - 1 || j == count - 1;
        right_edge = tc == tiles_w - 1;
    }

    // (planes within 32-bit offsets)
    __device__ __forceinline__ static int word(int k) { return ((int)threadIdx.x + k * B::THREADS) / B::TB / N; }
    __device__ __forceinline__ static int row(int k) { return ((int)threadIdx.x + k * B::THREADS) / B::TB - word(k) * N; }
    __device__ __forceinline__ void keep_addresses(int H, int W)
    {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            kept[KEEP ? k : 0] = {word(k) * CPT * (H * W) + (h_lo + row(k)) * W + w0,
                                  (unsigned)(h_lo + row(k)) < (unsigned)H ? word(k) * CPT : 1 << 30,       // (outside the image: no channel)
                                  j * B::TILE + word(k) * B::WIN + row(k) * N};
    }

    // x may end before the M elements of a row do; then they are taken from the end of x and moved
    __device__ __forceinline__ static bool near_end(long long remaining, int c_lim, int HW)
    {
        return __any(remaining < (long long)(c_lim < CH ? c_lim : CH) * HW + M);
    }

    // planes: first channel plane of the block in the tile's image; c_lim: channels of x from there on;
    // remaining: elements of x from there on
    template <bool STREAM>
    __device__ __forceinline__ void load(const T *planes, int c_lim, long long remaining, int H, int W)
    {
        const int HW = H * W, first = h_lo * W + w0;
        const bool tail = loaded_tail = near_end(remaining, c_lim, HW);
        const int room = remaining < 0x7fffffffLL ? (int)remaining : 0x7fffffff;
        const bool lead = first_lane && tc > 0, trail = last_lane && !right_edge;
        const int halo_w = lead ? w0 - PAD : w0 + M;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
#pragma unroll
                for (int e = 0; e < WORDS; ++e) raw[k][c][e] = 0u;
#pragma unroll
                for (int q = 0; q < PAD; ++q) halo[k][c][q] = 0u;
            }
            const int g = word(k), a = row(k);
            if (KEEP ? kept[KEEP ? k : 0].chan < c_lim : (unsigned)(h_lo + a) < (unsigned)H && g * CPT < c_lim) {
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const int ch = c == 0 || g * CPT + c < c_lim ? g * CPT + c : g * CPT;       // (no such channel: zeroed in place())
                    const int at = KEEP ? kept[KEEP ? k : 0].off + (ch - g * CPT) * HW : ch * HW + first + a * W;
                    load_words<STREAM>(planes + (tail && at > room - M ? room - M : at), raw[k][c]);
                    if (lead || trail) {
#pragma unroll
                        for (int q = 0; q < PAD; ++q)
                            if (halo_w + q < W) halo[k][c][q] = element_bits<STREAM>(planes + (at - w0 + halo_w + q));
                    }
                }
            }
        }
    }

    __device__ __forceinline__ void place(unsigned *lds, int c_lim, long long remaining, int H, int W)
    {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const int HW = H * W, first = h_lo * W + w0, valid = W - w0;     // columns of the tile at or beyond `valid` lie outside
        // (kernels of several blocks work it out again: kept, it costs the one-kernel layers spills)
        const bool tail = KEEP ? near_end(remaining, c_lim, HW) : loaded_tail;
        const int room = remaining < 0x7fffffffLL ? (int)remaining : 0x7fffffff;
        const bool any_right = __any(valid < M), odd_channel = CPT == 2 && c_lim < CH && (c_lim & 1);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int g = word(k), a = row(k);
            if (tail) {
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    int shift = (g * CPT + c) * HW + first + a * W - (room - M);
                    if (shift > M) shift = M;
                    while (__any(shift > 0)) {                   // one element further per turn
                        if (shift > 0) {
#pragma unroll
                            for (int e = 0; e < WORDS; ++e) {
                                const unsigned next = e + 1 < WORDS ? raw[k][c][e + 1 < WORDS ? e + 1 : e] : 0u;
                                raw[k][c][e] = sizeof(T) == 2 ? (raw[k][c][e] >> 16) | (next << 16) : next;
                            }
                        }
                        --shift;
                    }
                }
            }
            unsigned px[N], edge[PAD];                           // the window row; a word per pixel
            if constexpr (CPT == 2) {
                if (odd_channel && g * CPT + 1 >= c_lim) {
#pragma unroll
                    for (int e = 0; e < WORDS; ++e) raw[k][1][e] = 0u;
#pragma unroll
                    for (int q = 0; q < PAD; ++q) halo[k][1][q] = 0u;
                }
#pragma unroll
                for (int e = 0; e < M; ++e)
                    px[PAD + e] = __builtin_amdgcn_perm(raw[k][1][e / 2], raw[k][0][e / 2], (e & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
                for (int q = 0; q < PAD; ++q) edge[q] = halo[k][0][q] | (halo[k][1][q] << 16);
            } else {
#pragma unroll
                for (int e = 0; e < M; ++e) px[PAD + e] = raw[k][0][e];
#pragma unroll
                for (int q = 0; q < PAD; ++q) edge[q] = halo[k][0][q];
            }
            if (any_right) {
#pragma unroll
                for (int e = 0; e < M; ++e) px[PAD + e] = e < valid ? px[PAD + e] : 0u;
            }
            // the columns beside the tile belong to the neighbouring lanes' tiles (row_shr:1, row_shl:1)
#pragma unroll
            for (int q = 0; q < PAD; ++q) {
                const unsigned before = (unsigned)__builtin_amdgcn_update_dpp(0, (int)px[M + q], 0x111, 0xf, 0xf, true);
                const unsigned after = (unsigned)__builtin_amdgcn_update_dpp(0, (int)px[PAD + q], 0x101, 0xf, 0xf, true);
                px[q] = tc == 0 ? 0u : first_lane ? edge[q] : before;
                px[PAD + M + q] = right_edge ? 0u : last_lane ? edge[q] : after;
            }
            unsigned *dst = lds + (KEEP ? kept[KEEP ? k : 0].dst : j * B::TILE + g * B::WIN + a * N);
#pragma unroll
            for (int e = 0; e < N; e += 2)
                *reinterpret_cast<u32x2 *>(__builtin_assume_aligned(dst + e, 8)) = u32x2{px[e], px[e + 1]};
        }
    }
};

// Rows [LO, HI) of the transform of the CPT windows in `win` (pitch between pixels: a word; N words per row):
// emit.start(LO), then emit.value(i, j, o) is handed V[i][j] of each of them, o[c][j], unrounded, for i, j ascending.
template <int N, typename T, bool SYM, int LO, int HI, typename F>
__device__ __forceinline__ void transform_window(const unsigned *win, const InCoef<N> &coef, F &&emit)
{
    constexpr int CPT = 4 / (int)sizeof(T);
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    // columns of the tile first, two at a time: tmp[c][i - LO][b] = sum_a B^T[i][a] d[a][b]
    float tmp[CPT][HI - LO][N];
#pragma unroll
    for (int bp = 0; bp < N; bp += 2) {
        u32x2 px[N];
#pragma unroll
        for (int a = 0; a < N; ++a) px[a] = *reinterpret_cast<const u32x2 *>(__builtin_assume_aligned(win + a * N + bp, 8));
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                float d[N], o[HI - LO];
#pragma unroll
                for (int a = 0; a < N; ++a) {
                    if constexpr (CPT == 2) {
                        const unsigned short bits = (unsigned short)(px[a][bb] >> (16 * c));
                        f16 h;
                        __builtin_memcpy(&h, &bits, 2);
                        d[a] = (float)h;
                    } else {
                        d[a] = __uint_as_float(px[a][bb]);
                    }
                }
                input_transform_rows<N, SYM, LO, HI>(d, o, coef);
#pragma unroll
                for (int i = 0; i < HI - LO; ++i) tmp[c][i][bp + bb] = o[i];
            }
    }
    // then along each of those rows: V[i][j] = sum_b tmp[i][b] B^T[j][b]
    emit.start(LO);
#pragma unroll
    for (int i = LO; i < HI; ++i) {
        float o[CPT][N];
#pragma unroll
        for (int c = 0; c < CPT; ++c) input_transform_rows<N, SYM, 0, N>(tmp[c][i - LO], o[c], coef);
#pragma unroll
        for (int j = 0; j < N; ++j) emit.value(i, j, o);
    }
}

// The row range of thread `part` (wave-uniform) of the B::RS that share a tile and word.
template <int N, typename T, bool SYM, typename B, int I = 0, typename F>
__device__ __forceinline__ void transform_part(int part, const unsigned *win, const InCoef<N> &coef, F &&emit)
{
    if constexpr (I + 1 < B::RS) {
        if (part != I) return transform_part<N, T, SYM, B, I + 1>(part, win, coef, emit);
    }
    // Keeps the parts' common beginning, the first window reads and their conversions to binary32, from being moved in
    // front of the branch: converted there, those values no longer enter the first multiply-adds as binary16 operands
    // (n = 10: 50 of 3836 instructions and 14 of 133 registers more; 256 ch @56x56 batch 33 F(8,3) 34.4 -> 33.6 us)
    asm volatile("; part %0" : : "n"(I) : "memory");
    transform_window<N, T, SYM, B::bound(I), B::bound(I + 1)>(win, coef, emit);
}

// One word of V: CPT rounded values of position j of a row
template <int N>
__device__ __forceinline__ unsigned rounded_word(const float (&o)[2][N], int j, f16 *)
{
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    float a = o[0][j], b = o[1][j];
    asm volatile("" : "+v"(a), "+v"(b));                         // (as round_twice; both in one conversion)
    return __builtin_bit_cast(unsigned, half2v{(f16)a, (f16)b});
}
template <int N>
__device__ __forceinline__ unsigned rounded_word(const float (&o)[1][N], int j, float *) { return __float_as_uint(o[0][j]); }

template <int N>
static void fill_in_coef(const nova_transforms *t, InCoef<N> &k)
{
    constexpr int H = InCoef<N>::H;
    for (int i = 0; i < N * N; ++i) k.bt[i] = t->BT32[i];
    for (int q = 0; q <= H; ++q) {
        k.zero[q] = t->BT32[0 * N + 2 * q];
        k.inf[q] = t->BT32[(N - 1) * N + 2 * q + 1];
    }
    for (int j = 0; j < H; ++j)
        for (int q = 0; q < H; ++q) {
            k.ev[j * H + q] = t->BT32[(2 * j + 1) * N + 2 * q + 2];
            k.od[j * H + q] = t->BT32[(2 * j + 1) * N + 2 * q + 1];
        }
}

}  // namespace nova
