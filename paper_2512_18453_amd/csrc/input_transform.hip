// Input transform V = B^T d B (Sec. 2.1 step 1, nested in 2D) for every n x n tile of the
// zero-padded image, x [N][C][H][W] -> V [n*n][C/32][T][32].
//
// A workgroup takes TB consecutive tiles of the batch (4, 8 or 16; whatever tile rows and images they belong
// to) and one block of 32 channels.  Every tile's own n x n window is staged in LDS, two neighbouring
// channels of a pixel in one word (binary16), so that a thread transforms one tile of two channels and its
// results leave as whole words straight from registers: 16 lanes = 32 channels of a tile = 64 bytes of V,
// a wave = 4 neighbouring tiles = 256 contiguous bytes per position.  Two threads share the rows of a
// tile from n = 8 on.  A window's row is loaded as the tile's own m columns; the columns it shares with the
// tiles beside it come from the neighbouring lanes.
// What bounds it: the vector instructions (about 1450 per tile and channel pair and half at n = 10, 14 us of
// issue slots on the 256 x 56 x 56 x batch 32 layer) beside the bytes of x and V.  Earlier form (a strip of
// one tile row staged once, thread = one tile of one channel, results back through LDS for 16-byte stores)
// against this one, us per launch, MI355X: 256 ch @56x56 batch 32 F(8,3) 35.4 -> 29.1; F(4,3) 70 -> 29;
// 64 ch @224x224 batch 8 F(8,3) 40.5 -> 29.3; 128 ch @112x112 batch 32 F(6,3) 94.5 -> 74; 512 ch @7x7 batch
// 256 F(8,3) 32.2 -> 13.4 (the strip form left half of the lanes without a tile); binary32 40 ch @45x61
// batch 8 F(6,3) 14.0 -> 7.5.
//
// Arithmetic contract (binary32): a 1D transform row is E + O, with E / O fused multiply-add
// chains over the even / odd input indices in ascending order, columns of the tile first, then
// rows.  For points given as 0, +a, -a, ... the rows of +a and -a share E and O (the even
// coefficients agree, the odd ones are negated), which gives bit-identical results at half the
// multiplications.  The result is rounded once to the storage format.
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

// A workgroup takes TB tiles that are neighbours in t (whatever tile rows and images they belong to) and one
// block of CH channels: 32, or 4 for the compact layout of the first layer.  A word of LDS holds one pixel of CPT
// channels: two neighbouring channels in binary16, one in binary32.
template <int N, typename T, int CH, bool WIDE>
struct TileBlock {
    static constexpr int CPT = 4 / (int)sizeof(T);              // channels per word
    static constexpr int GP = CH / CPT;                         // words per pixel of a channel block
    // threads that share the transform rows of one tile and word; WIDE: one per pair of rows (+a, -a), for launches
    // that leave the chip half empty, where a thread's chain of instructions is what takes the time
    static constexpr int RS = WIDE ? N / 2 : N >= 8 ? 2 : 1;
    // rows [bound(i), bound(i + 1)) are thread i's; no (+a, -a) pair (2q + 1, 2q + 2) is cut
    static constexpr int bound(int i) { return i == 0 ? 0 : i == RS ? N : WIDE ? 2 * i + 1 : RowSplit<N>::value; }
    static constexpr int TB = CH == 4 ? 64 / GP : sizeof(T) == 2 ? (N >= 8 ? 8 : 16) : (N >= 8 ? 4 : 8);
    static constexpr int RUN = TB < 16 ? TB : 16;               // neighbouring tiles whose lanes exchange columns (16: a DPP row)
    static constexpr int THREADS = TB * GP * RS;
    static constexpr int WAVES_PER_XI = TB * GP / 64;
    static constexpr int TILE_PAD = 2;
    // Pitches in words.  The window reads take two pixels (8 bytes) per lane, 32 lanes (two tiles' 16 windows, or
    // one tile's 32) per phase: with a window pitch of 2 * odd 8-byte units (binary32: odd) and a tile pitch of
    // an odd number of them, the lanes fall into different banks.
    static constexpr int WIN = CPT == 2 ? ((N * N / 4) % 2 == 1 ? N * N : N * N + 4) : N * N + 2;
    static constexpr int TILE = GP * WIN + TILE_PAD;
    static constexpr int LDS_BYTES = TB * TILE * 4;
    static_assert(WIN % 2 == 0 && N % RS == 0 && (TB * GP) % 64 == 0, "block shape");
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

// What the transform leaves about the largest magnitude of V, for a later quantisation (partial maxima, in the
// storage format's rounding -- rounding is monotonic, so the largest rounded value is the rounded largest):
//   kMaxTensor     one per wave
//   kMaxPosition   four per wave and position (16 lanes each)
enum { kMaxNone = 0, kMaxTensor = 1, kMaxPosition = 2 };

// Rows [LO, HI) of the transform of the CPT windows in `win`, stored to V as they are finished.
// top (kMaxTensor): running maximum; partials, n_part (kMaxPosition): where this wave's go, entries per position.
template <int N, typename T, bool SYM, int MAXIMA, int LO, int HI>
__device__ __forceinline__ void transform_window(const unsigned *win, T *v_block, size_t xi_stride, unsigned lane_off, bool active,
                                                 const InCoef<N> &coef, float &top, float *partials, int n_part)
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
    // then along each of those rows: V[i][j] = sum_b tmp[i][b] B^T[j][b], rounded to storage
    T *plane = uniform_pointer(v_block + (size_t)(LO * N) * xi_stride);
#pragma unroll
    for (int i = LO; i < HI; ++i) {
        float o[CPT][N];
#pragma unroll
        for (int c = 0; c < CPT; ++c) input_transform_rows<N, SYM, 0, N>(tmp[c][i - LO], o[c], coef);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            unsigned word;
            if constexpr (CPT == 2) {
                const f16 pair[2] = {round_twice(o[0][j], (f16 *)nullptr), round_twice(o[1][j], (f16 *)nullptr)};
                __builtin_memcpy(&word, pair, 4);
            } else {
                word = __float_as_uint(o[0][j]);
            }
            if (MAXIMA == kMaxNone || active) *reinterpret_cast<NOVA_GLOBAL unsigned *>(plane_element(plane, lane_off)) = word;
            plane = uniform_pointer(plane + xi_stride);
            if constexpr (MAXIMA == kMaxTensor) {
#pragma unroll
                for (int c = 0; c < CPT; ++c) top = fmaxf(top, fabsf(o[c][j]));
            }
            if constexpr (MAXIMA == kMaxPosition) {
                float m = fabsf(o[0][j]);
                if constexpr (CPT == 2) m = fmaxf(m, fabsf(o[CPT - 1][j]));
                // maximum over 16 lanes (row_ror 8, 4, 2, 1); fmaxf drops a NaN
                m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x128, 0xf, 0xf, true)));
                m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x124, 0xf, 0xf, true)));
                m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x122, 0xf, 0xf, true)));
                m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x121, 0xf, 0xf, true)));
                if ((threadIdx.x & 15) == 0)
                    partials[(size_t)(i * N + j) * n_part + (threadIdx.x >> 4 & 3)] = fmaxf(0.0f, (float)round_twice(m, (T *)nullptr));
            }
        }
    }
}

// The row range of thread `part` (wave-uniform) of the B::RS that share a tile and word.
template <int N, typename T, bool SYM, int MAXIMA, typename B, int I>
__device__ __forceinline__ void transform_part(int part, const unsigned *win, T *v_block, size_t xi_stride, unsigned lane_off, bool active,
                                               const InCoef<N> &coef, float &top, float *partials, int n_part)
{
    if constexpr (I + 1 < B::RS) {
        if (part != I) return transform_part<N, T, SYM, MAXIMA, B, I + 1>(part, win, v_block, xi_stride, lane_off, active, coef, top, partials, n_part);
    }
    transform_window<N, T, SYM, MAXIMA, B::bound(I), B::bound(I + 1)>(win, v_block, xi_stride, lane_off, active, coef, top, partials, n_part);
}

// Filters to pack beside the transform (blocks of 4 channels only): to[row][c] = from[row][0][c] for c < 4, a row
// being (xi, k) of U [n*n][1][Kp][32].  Done by workgroups of the same launch: a launch of its own cost 3.5 us of
// host time and 3-5 us on the device (3 -> 64 @224x224 batch 32 F(8,3), whole call 125 -> 121 us).
template <typename T>
struct PackFilters { const T *from; T *to; long long rows; };

// Groups of tiles: a row of row_tiles consecutive t (the whole batch, or one tile row of an image) is cut into
// groups_per_row groups of `per` tiles.
template <int N, int R, typename T, bool SYM, int CH, bool WIDE, bool STREAM, int MAXIMA>
__global__ void __launch_bounds__((TileBlock<N, T, CH, WIDE>::THREADS), 3)     // (three waves per SIMD: as many as the windows in LDS allow)
input_transform_kernel(const T *__restrict__ x, T *__restrict__ V, int C, int H, int W, int tiles_h, int tiles_w,
                       int c_blocks, unsigned t_groups, int row_tiles, int groups_per_row, int per, int Ttot, long long x_elems,
                       int by_element, float *partials, int n_part, PackFilters<T> pack, InCoef<N> coef)
{
    using B = TileBlock<N, T, CH, WIDE>;
    constexpr int M = N - R + 1;                 // outputs per tile side = tile stride
    constexpr int PAD = (R - 1) / 2;             // zero border of the convolution
    constexpr int CPT = B::CPT;
    constexpr int ITEMS = N / B::RS;             // window rows a thread stages
    constexpr int WORDS = M * (int)sizeof(T) / 4;                  // words of a tile's own columns in one row
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) unsigned lds[];

    const unsigned tile_blocks = t_groups * (unsigned)c_blocks;
    if constexpr (CH == 4) {
        if (blockIdx.x >= tile_blocks) {                         // the workgroups after the tiles' pack filters
            const long long row = (long long)(blockIdx.x - tile_blocks) * B::THREADS + threadIdx.x;
            if (row < pack.rows) {
#pragma unroll
                for (int c = 0; c < CH; ++c) pack.to[row * CH + c] = pack.from[row * kChanBlock + c];
            }
            return;
        }
    }
    const unsigned bid = xcd_local_block_id(blockIdx.x, tile_blocks);
    const int cb = (int)(bid / t_groups);
    const int group = (int)(bid - (unsigned)cb * t_groups), group_row = group / groups_per_row;
    const int in_row = (group - group_row * groups_per_row) * per;                  // the group's first tile within its row
    const int t0 = group_row * row_tiles + in_row;
    const int count = row_tiles - in_row < per ? row_tiles - in_row : per;
    const int tid = (int)threadIdx.x;

    // ---- stage the windows.  A thread's items are window rows of one tile: (channel word g, row a), with
    // the tiles of the group in neighbouring lanes, so that a load runs along image rows and the columns a
    // window shares with its neighbours come from the lanes beside it.  The M elements loaded are aligned to
    // an element only.
    {
        const int j = tid % B::TB;
        const int t = t0 + (j < count ? j : count - 1);
        const int trow = t / tiles_w, tc = t - trow * tiles_w, img = trow / tiles_h, tr = trow - img * tiles_h;
        const int h_lo = tr * M - PAD, w_lo = tc * M - PAD;
        const int c_lim = C - cb * CH;
        const T *planes = x + ((long long)img * C + (long long)cb * CH) * H * W;     // this block's first channel plane
        unsigned *tile_lds = lds + j * B::TILE;
        if (by_element) {
            // planes too large for 32-bit offsets, or x shorter than a window row
#pragma unroll 1
            for (int k = 0; k < ITEMS; ++k) {
                const int rest = (tid + k * B::THREADS) / B::TB, g = rest / N, a = rest - g * N;
                const int h = h_lo + a;
                T *dst = reinterpret_cast<T *>(tile_lds + g * B::WIN + a * N);
#pragma unroll 1
                for (int e = 0; e < N * CPT; ++e) {
                    const int c = g * CPT + e % CPT, w = w_lo + e / CPT;
                    T val = (T)0.0f;
                    if (c < c_lim && h >= 0 && h < H && w >= 0 && w < W) val = planes[((long long)c * H + h) * W + w];
                    dst[e] = val;
                }
            }
        } else {
            const int w0 = tc * M, valid = W - w0;               // columns of the tile at or beyond `valid` lie outside
            const int HW = H * W, first = h_lo * W + w0;
            // x may end before the M elements of a row do; then they are taken from the end of x and moved
            const long long remaining = x_elems - (planes - x);
            const bool tail = __any(remaining < (long long)(c_lim < CH ? c_lim : CH) * HW + M);
            const int room = remaining < 0x7fffffffLL ? (int)remaining : 0x7fffffff;
            // the first tile of a run of lanes loads its left halo, the last one the right one (never the same tile: a run
            // has several; lanes past the group's last tile load it again and stage a window that is never read)
            const bool first_lane = j % B::RUN == 0, last_lane = j % B::RUN == B::RUN - 1 || j == count - 1;
            const bool lead = first_lane && tc > 0, trail = last_lane && tc < tiles_w - 1;
            const int halo_w = lead ? w0 - PAD : w0 + M;
            unsigned raw[ITEMS][CPT][WORDS], halo[ITEMS][CPT][PAD];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int rest = (tid + k * B::THREADS) / B::TB, g = rest / N, a = rest - g * N;
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
#pragma unroll
                    for (int e = 0; e < WORDS; ++e) raw[k][c][e] = 0u;
#pragma unroll
                    for (int q = 0; q < PAD; ++q) halo[k][c][q] = 0u;
                }
                if ((unsigned)(h_lo + a) < (unsigned)H && g * CPT < c_lim) {
#pragma unroll
                    for (int c = 0; c < CPT; ++c) {
                        const int ch = c == 0 || g * CPT + c < c_lim ? g * CPT + c : g * CPT;   // (no such channel: zeroed below)
                        const int off = ch * HW + first + a * W;
                        load_words<STREAM>(planes + (tail && off > room - M ? room - M : off), raw[k][c]);
                        if (lead || trail) {
#pragma unroll
                            for (int q = 0; q < PAD; ++q)
                                if (halo_w + q < W) halo[k][c][q] = element_bits<STREAM>(planes + (off - w0 + halo_w + q));
                        }
                    }
                }
            }
            const bool any_right = __any(valid < M), odd_channel = CPT == 2 && c_lim < CH && (c_lim & 1);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int rest = (tid + k * B::THREADS) / B::TB, g = rest / N, a = rest - g * N;
                if (tail) {
#pragma unroll
                    for (int c = 0; c < CPT; ++c) {
                        int shift = (g * CPT + c) * HW + first + a * W - (room - M);
                        if (shift > M) shift = M;
                        while (__any(shift > 0)) {               // one element further per turn
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
                unsigned px[N], edge[PAD];                       // the window row; a word per pixel
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
                    px[PAD + M + q] = tc == tiles_w - 1 ? 0u : last_lane ? edge[q] : after;
                }
                unsigned *dst = tile_lds + g * B::WIN + a * N;
#pragma unroll
                for (int e = 0; e < N; e += 2)
                    *reinterpret_cast<u32x2 *>(__builtin_assume_aligned(dst + e, 8)) = u32x2{px[e], px[e + 1]};
            }
        }
    }
    __syncthreads();

    // ---- transform: lanes run over the words of a tile's channel block, a wave over 64 / GP tiles
    const int g = tid % B::GP, j = tid / B::GP % B::TB;
    const int part = __builtin_amdgcn_readfirstlane(tid / (B::GP * B::TB));          // which of the RS row ranges
    // (for the maxima every lane stays, and one without a tile reads the group's last one; the place of its own holds
    // a window that no tile has: the last tile's columns between halos taken from the same tile)
    const unsigned *win = lds + (MAXIMA == kMaxNone || j < count ? j : count - 1) * B::TILE + g * B::WIN;
    T *v_block = V + ((size_t)cb * Ttot + t0) * CH;
    const size_t xi_stride = (size_t)c_blocks * Ttot * CH;
    const unsigned lane_off = (unsigned)(j * CH + g * CPT) * (unsigned)sizeof(T);
    const bool active = j < count;
    if constexpr (MAXIMA == kMaxNone)
        if (!active) return;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float top = 0.0f;
    float *mine = partials;
    if constexpr (MAXIMA == kMaxPosition) mine += ((size_t)blockIdx.x * B::WAVES_PER_XI + wave % B::WAVES_PER_XI) * 4;
    transform_part<N, T, SYM, MAXIMA, B, 0>(part, win, v_block, xi_stride, lane_off, active, coef, top, mine, n_part);
    if constexpr (MAXIMA == kMaxTensor) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
        if ((tid & 63) == 0) mine[(size_t)blockIdx.x * (B::THREADS / 64) + wave] = (float)round_twice(top, (T *)nullptr);
    }
}

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

// partial maxima (per position with kMaxPosition) of a launch over all of g; -1: more than an int holds
template <int N, typename T>
static int maxima_count(const Geometry &g, int maxima)
{
    using B = TileBlock<N, T, kChanBlock, false>;
    const long long blocks = (g.T + B::TB - 1) / B::TB * g.c_blocks;
    const long long count = maxima == kMaxTensor ? blocks * (B::THREADS / 64) : maxima == kMaxPosition ? blocks * B::WAVES_PER_XI * 4 : 0;
    return count > 0x7fffffffLL ? -1 : (int)count;
}

template <int N, int R, typename T>
static int launch_it(const nova_transforms *t, const void *x, void *V, const Geometry &g, bool stream_x, int maxima, float *partials,
                     hipStream_t stream)
{
    using B = TileBlock<N, T, kChanBlock, false>;
    InCoef<N> coef;
    fill_in_coef<N>(t, coef);
    if (g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    // Groups of TB consecutive tiles, whatever rows and images they belong to: every lane has a tile.  With the
    // streaming hint on x a group keeps to one tile row instead: what it shares with a neighbour is not
    // found in the cache again (56 x 56 x 256 channels, batch 32, F(8,3), whole call: 110 us with rows and the
    // hint, 114 with the hint alone, 116 with neither; the transform alone, repeated on the same buffers, 34 / 39 / 29,
    // with x and V from memory 34.7 with both against 36.9 with neither).  Taken where a row is one nearly full
    // group.  Whole calls, time without / with both, layers whose x, V and M are 300 MB, n = 8 and 10, five pairs of
    // channel counts, by tiles per row: 4 and 5 0.94-0.99, 6 0.98-1.06, 7 0.98-1.08, 8 0.98-1.11, 9 and 10 (two groups)
    // 0.90-0.96, 12 0.93-0.99, 14 0.96-0.99, 15 and 16 0.96-1.03, 21 and 28 0.91-1.00.
    auto kern = t->symmetric ? input_transform_kernel<N, R, T, true, kChanBlock, false, false, kMaxNone>
                             : input_transform_kernel<N, R, T, false, kChanBlock, false, false, kMaxNone>;
    if (maxima != kMaxNone && !t->symmetric) return (int)hipErrorInvalidValue;
    if (maxima == kMaxTensor) kern = input_transform_kernel<N, R, T, true, kChanBlock, false, false, kMaxTensor>;
    if (maxima == kMaxPosition) kern = input_transform_kernel<N, R, T, true, kChanBlock, false, false, kMaxPosition>;
    bool rows = false;
    if constexpr (N >= 8 && sizeof(T) == 2)
        if (stream_x && maxima == kMaxNone && t->symmetric && g.tiles_w > B::TB * 3 / 4 && g.tiles_w <= B::TB) {
            kern = input_transform_kernel<N, R, T, true, kChanBlock, false, true, kMaxNone>;
            rows = true;
        }
    int threads = B::THREADS;
    // no more workgroups than compute units: one thread per pair of transform rows.  us per launch, without / with:
    // 512 ch @14x14 F(4,3) 6.2 / 5.2, 33 ch @30x41 batch 3 F(4,3) 7.5 / 5.4, binary32 16 ch @32x32 F(4,3) 5.7 / 4.6,
    // 256 ch @28x28 batch 16 F(8,3) (256 workgroups) 9.4 / 9.0, batch 32 (512) 13.3 / 15.0
    if (!rows && maxima == kMaxNone && t->symmetric && (g.T + B::TB - 1) / B::TB * g.c_blocks <= device_cu_count()) {
        kern = input_transform_kernel<N, R, T, true, kChanBlock, true, false, kMaxNone>;
        threads = TileBlock<N, T, kChanBlock, true>::THREADS;
    }
    const int row_tiles = rows ? g.tiles_w : (int)g.T;
    const int groups_per_row = ceil_div(row_tiles, B::TB);
    const int per = rows ? row_tiles : B::TB;               // (a row is one group)
    const long long t_groups = g.T / row_tiles * groups_per_row;
    const long long blocks = t_groups * g.c_blocks;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    const long long x_elems = (long long)g.N * g.C * g.H * g.W;
    const int by_element = x_elems < N - R + 1 || (long long)kChanBlock * g.H * g.W >= (1LL << 30) ? 1 : 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), B::LDS_BYTES, stream, (const T *)x, (T *)V, g.C, g.H, g.W,
                       g.tiles_h, g.tiles_w, g.c_blocks, (unsigned)t_groups, row_tiles, groups_per_row, per, (int)g.T, x_elems,
                       by_element, partials, maxima_count<N, T>(g, maxima), PackFilters<T>{nullptr, nullptr, 0}, coef);
    return (int)hipGetLastError();
}

static int launch_it_any(const nova_transforms *t, const void *x, void *V, const Geometry &g, int dtype, bool stream_x, int maxima,
                         float *partials, hipStream_t s)
{
    const bool h = dtype == NOVA_F16;
#define NOVA_IT(N, R) (h ? launch_it<N, R, f16>(t, x, V, g, stream_x, maxima, partials, s) \
                         : launch_it<N, R, float>(t, x, V, g, stream_x, maxima, partials, s))
    if (t->r == 3) {
        switch (t->n) {
        case 4: return NOVA_IT(4, 3);
        case 6: return NOVA_IT(6, 3);
        case 8: return NOVA_IT(8, 3);
        case 10: return NOVA_IT(10, 3);
        }
    } else if (t->r == 5) {
        switch (t->n) {
        case 6: return NOVA_IT(6, 5);
        case 8: return NOVA_IT(8, 5);
        case 10: return NOVA_IT(10, 5);
        }
    }
#undef NOVA_IT
    return (int)hipErrorInvalidValue;
}

int launch_input_transform(const nova_transforms *t, const void *x, void *V, const Geometry &g,
                           int dtype, void *stream, bool stream_x)
{
    return launch_it_any(t, x, V, g, dtype, stream_x, kMaxNone, nullptr, (hipStream_t)stream);
}

int input_maxima_count(const Geometry &g, int dtype, bool per_position)
{
    const int maxima = per_position ? kMaxPosition : kMaxTensor;
    const bool h = dtype == NOVA_F16;
    switch (g.n) {
    case 4: return h ? maxima_count<4, f16>(g, maxima) : maxima_count<4, float>(g, maxima);
    case 6: return h ? maxima_count<6, f16>(g, maxima) : maxima_count<6, float>(g, maxima);
    case 8: return h ? maxima_count<8, f16>(g, maxima) : maxima_count<8, float>(g, maxima);
    case 10: return h ? maxima_count<10, f16>(g, maxima) : maxima_count<10, float>(g, maxima);
    }
    return -1;
}

int launch_input_transform_maxima(const nova_transforms *t, const void *x, void *V, float *partials, bool per_position,
                                  const Geometry &g, int dtype, void *stream)
{
    return launch_it_any(t, x, V, g, dtype, false, per_position ? kMaxPosition : kMaxTensor, partials, (hipStream_t)stream);
}

// ---- Few input channels (C <= 4): V in the compact layout Vc [n*n][T][4] that the few-channel output transform
// reads (no 32-channel blocks: 3 of 32 channels would carry data).  The same kernel with blocks of 4
// channels: a wave takes 32 tiles (binary16) or 16 (binary32) and stores 256 contiguous bytes per position.
// (A kernel of its own, strip staged element by element, one channel per lane, 2-byte stores: 24.7 us on
// 3 x 224 x 224, batch 32, F(8,3); this one 12.0.)
constexpr int kFewIn = 4;                  // channels

template <int N, int R, typename T>
static int launch_it_few(const nova_transforms *t, const void *x, void *Vc, const Geometry &g, const void *U, void *Uc,
                         hipStream_t stream)
{
    using B = TileBlock<N, T, kFewIn, false>;
    if (g.C > kFewIn || g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    InCoef<N> coef;
    fill_in_coef<N>(t, coef);
    const long long blocks = (g.T + B::TB - 1) / B::TB;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    const long long x_elems = (long long)g.N * g.C * g.H * g.W;
    const int by_element = x_elems < N - R + 1 || (long long)kFewIn * g.H * g.W >= (1LL << 30) ? 1 : 0;
    auto kern = t->symmetric ? input_transform_kernel<N, R, T, true, kFewIn, false, false, kMaxNone>
                             : input_transform_kernel<N, R, T, false, kFewIn, false, false, kMaxNone>;
    const PackFilters<T> pack = {(const T *)U, (T *)Uc, U ? (long long)g.n * g.n * g.Kp : 0};
    const long long pack_blocks = (pack.rows + B::THREADS - 1) / B::THREADS;
    if (blocks + pack_blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks + pack_blocks)), dim3(B::THREADS), B::LDS_BYTES, stream, (const T *)x, (T *)Vc, g.C, g.H, g.W,
                       g.tiles_h, g.tiles_w, 1, (unsigned)blocks, (int)g.T, (int)blocks, B::TB, (int)g.T, x_elems, by_element,
                       (float *)nullptr, 0, pack, coef);
    return (int)hipGetLastError();
}

size_t few_channels_input_bytes(const Geometry &g, int dtype)
{
    return (size_t)g.n * g.n * (size_t)g.T * kFewIn * dtype_size(dtype);
}

int launch_input_transform_few(const nova_transforms *t, const void *x, void *Vc, const Geometry &g,
                               const void *U, void *Uc, int dtype, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    const bool h = dtype == NOVA_F16;
    if (t->r == 3) {
        switch (t->n) {
        case 4: return h ? launch_it_few<4, 3, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<4, 3, float>(t, x, Vc, g, U, Uc, s);
        case 6: return h ? launch_it_few<6, 3, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<6, 3, float>(t, x, Vc, g, U, Uc, s);
        case 8: return h ? launch_it_few<8, 3, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<8, 3, float>(t, x, Vc, g, U, Uc, s);
        case 10: return h ? launch_it_few<10, 3, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<10, 3, float>(t, x, Vc, g, U, Uc, s);
        }
    } else if (t->r == 5) {
        switch (t->n) {
        case 6: return h ? launch_it_few<6, 5, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<6, 5, float>(t, x, Vc, g, U, Uc, s);
        case 8: return h ? launch_it_few<8, 5, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<8, 5, float>(t, x, Vc, g, U, Uc, s);
        case 10: return h ? launch_it_few<10, 5, f16>(t, x, Vc, g, U, Uc, s) : launch_it_few<10, 5, float>(t, x, Vc, g, U, Uc, s);
        }
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace nova
