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
#include "input_common.hpp"

namespace nova {

// A workgroup's windows: 32 channels, or 4 for the compact layout of the first layer.  Threads per tile and word --
// WIDE: one per pair of transform rows (+a, -a), for launches that leave the chip half empty, where a thread's chain
// of instructions is what takes the time; 2: also only 4 tiles, so that they are spread over more compute units.
template <typename T, int CH> constexpr int kWords = CH * (int)sizeof(T) / 4;
template <int N, typename T, int CH, int WIDE>
constexpr int kTilesOf = CH == 4 ? 64 / kWords<T, CH> : WIDE == 2 ? 4 : sizeof(T) == 2 ? (N >= 8 ? 8 : 16) : (N >= 8 ? 4 : 8);
template <int N, typename T, int CH, int WIDE>
struct TileBlock : TileWindows<N, T, CH, kTilesOf<N, T, CH, WIDE>, WIDE ? N / 2 : N >= 8 ? 2 : 1> {
    using W = TileWindows<N, T, CH, kTilesOf<N, T, CH, WIDE>, WIDE ? N / 2 : N >= 8 ? 2 : 1>;
    static constexpr int WAVES_PER_XI = W::TB * W::GP / 64;
};

// What the transform leaves about the largest magnitude of V, for a later quantisation (partial maxima, in the
// storage format's rounding -- rounding is monotonic, so the largest rounded value is the rounded largest):
//   kMaxTensor     one per wave
//   kMaxPosition   four per wave and position (16 lanes each)
enum { kMaxNone = 0, kMaxTensor = 1, kMaxPosition = 2 };

// Where the transform's values go: the planes of V, one after the other.
// top (kMaxTensor): running maximum; partials, n_part (kMaxPosition): where this wave's go, entries per position.
template <int N, typename T, int MAXIMA>
struct VToPlanes {
    T *v_block;
    size_t xi_stride;
    unsigned lane_off;
    bool active;
    T *plane;
    float top;
    float *partials;
    int n_part;
    __device__ __forceinline__ void start(int first_row) { plane = uniform_pointer(v_block + (size_t)(first_row * N) * xi_stride); }
    template <int CPT>
    __device__ __forceinline__ void value(int i, int j, const float (&o)[CPT][N])
    {
        const unsigned word = rounded_word<N>(o, j, (T *)nullptr);
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
};

// Filters to pack beside the transform (blocks of 4 channels only): to[row][c] = from[row][0][c] for c < 4, a row
// being (xi, k) of U [n*n][1][Kp][32].  Done by workgroups of the same launch: a launch of its own cost 3.5 us of
// host time and 3-5 us on the device (3 -> 64 @224x224 batch 32 F(8,3), whole call 125 -> 121 us).
template <typename T>
struct PackFilters { const T *from; T *to; long long rows; };

// Groups of tiles: a row of row_tiles consecutive t (the whole batch, or one tile row of an image) is cut into
// groups_per_row groups of `per` tiles.
template <int N, int R, typename T, bool SYM, int CH, int WIDE, bool STREAM, int MAXIMA>
__global__ void __launch_bounds__((TileBlock<N, T, CH, WIDE>::THREADS), 3)     // (three waves per SIMD: as many as the windows in LDS allow)
input_transform_kernel(const T *__restrict__ x, T *__restrict__ V, int C, int H, int W, int tiles_h, int tiles_w,
                       int c_blocks, unsigned t_groups, int row_tiles, int groups_per_row, int per, int Ttot, long long x_elems,
                       int by_element, float *partials, int n_part, PackFilters<T> pack, InCoef<N> coef)
{
    using B = TileBlock<N, T, CH, WIDE>;
    constexpr int CPT = B::CPT;
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

    // ---- stage the windows
    {
        const int c_lim = C - cb * CH;
        WindowRows<N, R, T, B, false> rows;
        rows.place_tile(t0, count, tiles_h, tiles_w);
        const T *planes = x + ((long long)rows.img * C + (long long)cb * CH) * H * W;     // this block's first channel plane
        if (by_element) {
            // planes too large for 32-bit offsets, or x shorter than a window row
            constexpr int PAD = (R - 1) / 2;
#pragma unroll 1
            for (int k = 0; k < N / B::RS; ++k) {
                const int rest = (tid + k * B::THREADS) / B::TB, g = rest / N, a = rest - g * N;
                const int h = rows.h_lo + a;
                T *dst = reinterpret_cast<T *>(lds + rows.j * B::TILE + g * B::WIN + a * N);
#pragma unroll 1
                for (int e = 0; e < N * CPT; ++e) {
                    const int c = g * CPT + e % CPT, w = rows.w0 - PAD + e / CPT;
                    T val = (T)0.0f;
                    if (c < c_lim && h >= 0 && h < H && w >= 0 && w < W) val = planes[((long long)c * H + h) * W + w];
                    dst[e] = val;
                }
            }
        } else {
            const long long remaining = x_elems - (planes - x);
            rows.template load<STREAM>(planes, c_lim, remaining, H, W);
            rows.place(lds, c_lim, remaining, H, W);
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
    VToPlanes<N, T, MAXIMA> sink{v_block, xi_stride, lane_off, active, nullptr, 0.0f, mine, n_part};
    transform_part<N, T, SYM, B>(part, win, coef, sink);
    top = sink.top;
    if constexpr (MAXIMA == kMaxTensor) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
        if ((tid & 63) == 0) mine[(size_t)blockIdx.x * (B::THREADS / 64) + wave] = (float)round_twice(top, (T *)nullptr);
    }
}

// partial maxima (per position with kMaxPosition) of a launch over all of g; -1: more than an int holds
template <int N, typename T>
static int maxima_count(const Geometry &g, int maxima)
{
    using B = TileBlock<N, T, kChanBlock, 0>;
    const long long blocks = (g.T + B::TB - 1) / B::TB * g.c_blocks;
    const long long count = maxima == kMaxTensor ? blocks * (B::THREADS / 64) : maxima == kMaxPosition ? blocks * B::WAVES_PER_XI * 4 : 0;
    return count > 0x7fffffffLL ? -1 : (int)count;
}

template <int N, int R, typename T>
static int launch_it(const nova_transforms *t, const void *x, void *V, const Geometry &g, bool stream_x, int maxima, float *partials,
                     hipStream_t stream)
{
    using B = TileBlock<N, T, kChanBlock, 0>;
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
    auto kern = t->symmetric ? input_transform_kernel<N, R, T, true, kChanBlock, 0, false, kMaxNone>
                             : input_transform_kernel<N, R, T, false, kChanBlock, 0, false, kMaxNone>;
    if (maxima != kMaxNone && !t->symmetric) return (int)hipErrorInvalidValue;
    if (maxima == kMaxTensor) kern = input_transform_kernel<N, R, T, true, kChanBlock, 0, false, kMaxTensor>;
    if (maxima == kMaxPosition) kern = input_transform_kernel<N, R, T, true, kChanBlock, 0, false, kMaxPosition>;
    bool rows = false;
    if constexpr (N >= 8 && sizeof(T) == 2)
        if (stream_x && maxima == kMaxNone && t->symmetric && g.tiles_w > B::TB * 3 / 4 && g.tiles_w <= B::TB) {
            kern = input_transform_kernel<N, R, T, true, kChanBlock, 0, true, kMaxNone>;
            rows = true;
        }
    int threads = B::THREADS, tiles = B::TB, lds_bytes = B::LDS_BYTES;
    // no more workgroups than compute units: one thread per pair of transform rows.  us per launch, without / with:
    // 512 ch @14x14 F(4,3) 6.2 / 5.2, 33 ch @30x41 batch 3 F(4,3) 7.5 / 5.4, binary32 16 ch @32x32 F(4,3) 5.7 / 4.6,
    // 256 ch @28x28 batch 16 F(8,3) (256 workgroups) 9.4 / 9.0, batch 32 (512) 13.3 / 15.0
    if (!rows && maxima == kMaxNone && t->symmetric && (g.T + B::TB - 1) / B::TB * g.c_blocks <= device_cu_count()) {
        kern = input_transform_kernel<N, R, T, true, kChanBlock, 1, false, kMaxNone>;
        threads = TileBlock<N, T, kChanBlock, 1>::THREADS;
        // Four tiles per workgroup while those are no more than compute units either (binary16 n = 6: twice as many).  The transform alone, time
        // with more over time with four, 280 launches: n = 10 1.11-1.52 (up to twice the units 0.97-1.03), n = 8 1.08-1.33 (1.01-1.02), n = 6
        // 0.99-1.22 (1.05-1.09; more 0.95-1.02), binary32 n = 6 0.93-1.10 (0.95-1.00); n = 4 0.84-1.08, not taken.  512 ch @14x14 F(4,3) 5.2 / 4.3 us.
        if constexpr (B::TB > 4 && N > 4) {
            if ((g.T + 3) / 4 * g.c_blocks <= device_cu_count() * (N == 6 && sizeof(T) == 2 ? 2 : 1)) {
                using S = TileBlock<N, T, kChanBlock, 2>;
                kern = input_transform_kernel<N, R, T, true, kChanBlock, 2, false, kMaxNone>;
                threads = S::THREADS;
                tiles = S::TB;
                lds_bytes = S::LDS_BYTES;
            }
        }
    }
    const int row_tiles = rows ? g.tiles_w : (int)g.T;
    const int groups_per_row = ceil_div(row_tiles, tiles);
    const int per = rows ? row_tiles : tiles;               // (a row is one group)
    const long long t_groups = g.T / row_tiles * groups_per_row;
    const long long blocks = t_groups * g.c_blocks;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    const long long x_elems = (long long)g.N * g.C * g.H * g.W;
    const int by_element = x_elems < N - R + 1 || (long long)kChanBlock * g.H * g.W >= (1LL << 30) ? 1 : 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), lds_bytes, stream, (const T *)x, (T *)V, g.C, g.H, g.W,
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
    using B = TileBlock<N, T, kFewIn, 0>;
    if (g.C > kFewIn || g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    InCoef<N> coef;
    fill_in_coef<N>(t, coef);
    const long long blocks = (g.T + B::TB - 1) / B::TB;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    const long long x_elems = (long long)g.N * g.C * g.H * g.W;
    const int by_element = x_elems < N - R + 1 || (long long)kFewIn * g.H * g.W >= (1LL << 30) ? 1 : 0;
    auto kern = t->symmetric ? input_transform_kernel<N, R, T, true, kFewIn, 0, false, kMaxNone>
                             : input_transform_kernel<N, R, T, false, kFewIn, 0, false, kMaxNone>;
    int threads = B::THREADS;
    // (as in launch_it; us for the whole call without / with: 3 -> 64 @48x18 batch 12 F(8,3) 21.0 / 18.4, 4 -> 41 @44x14 batch 32
    // F(6,3) 13.8 / 12.3, but 3 -> 10 @24x57 batch 12 F(2,3) 8.5 / 9.0)
    if (N > 4 && t->symmetric && blocks <= device_cu_count()) {
        kern = input_transform_kernel<N, R, T, true, kFewIn, 1, false, kMaxNone>;
        threads = TileBlock<N, T, kFewIn, 1>::THREADS;
    }
    const PackFilters<T> pack = {(const T *)U, (T *)Uc, U ? (long long)g.n * g.n * g.Kp : 0};
    const long long pack_blocks = (pack.rows + threads - 1) / threads;
    if (blocks + pack_blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks + pack_blocks)), dim3(threads), B::LDS_BYTES, stream, (const T *)x, (T *)Vc, g.C, g.H, g.W,
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
