// Winograd-domain contraction over input channels (Sec. 2.1 step 3, summed over channels):
//     M[xi][t][k] = sum_c V[xi][t][c] * U[xi][k][c]      for each of the n*n positions xi,
// i.e. n*n independent (T x C) . (C x K) matrix products.  Both operands are stored with the
// contraction index blocked by 32 and fastest (V [xi][C/32][T][32], U [xi][C/32][Kp][32]), so a
// (rows x 32-channel) operand tile is one contiguous piece of memory and every lane's MFMA
// fragment is a 16-byte read.
//
// binary16 path: v_mfma_f32_32x32x16_f16, binary32 accumulation, two kernels with the same order of summation
// (ascending channels, 16 per instruction), so that which of them runs does not show in M:
//   streaming kernel (large layers with C = 64, 128 or 256; further down): U stays in registers, V streams once
//     through an LDS ring filled by direct global->LDS loads;
//   tiled kernel (everything else): a ring of LDS stages of 32 channels, filled the same way.
// Both store M a whole 128-byte row of 32 output channels per half-wave: 16-byte stores of four neighbouring
// channels per lane, 32 bytes of each row at a time, moved the same bytes in 5-30 % more time (streaming kernel,
// us: 256 -> 256 @14x14 batch 256 binary16 M 28.5 -> 22.8, binary32 30.0 -> 26.4; 128 -> 128 @28x28 batch 128
// 28.0 -> 24.8; 256 -> 256 @56x56 batch 32 40.7 -> 39.3).
// binary32 path: the tiled kernel on v_mfma_f32_32x32x2_f32.
#include <type_traits>

#include "device_common.hpp"

namespace nova {

int device_cu_count()
{
    static int cached[64] = {};
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4f __attribute__((ext_vector_type(4)));

// s_waitcnt vmcnt(X): at most X of the wave's vector-memory operations are outstanding afterwards (they retire
// in the order issued)
template <int X>
__device__ __forceinline__ void stream_wait()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(X < 63 ? X : 63) : "memory");
}

// Tiled variant.  WM x WN waves own BM tiles x BN output channels of one M[xi].  The channel loop takes 32
// channels per stage from a ring of S stages in LDS, filled by direct global->LDS loads S - 1 stages ahead: a
// stage costs one round trip to memory only where the loop begins (with one stage in flight, as before,
// every 32 channels cost one: 16 us for 512 channels on a 14 x 14 image however few tiles).  A stage is BM rows
// of V and BN rows of U, 64 bytes each, XOR-swizzled by 16-byte slot like the streaming kernel's; a wave-wide
// load moves 16 rows.  Rows beyond the tensors are clamped to the last valid row (their products are
// never stored); past the last channel block loads are still issued, so that the wait counts are constants, but
// every lane rereads the same 16 bytes: one cached request.  Summation order per product: ascending channels in steps of 16, as in the
// streaming kernel -- M does not depend on which kernel or tile shape formed it.
// binary32 storage: v_mfma_f32_32x32x2_f32.  A row is 128 bytes (slots XOR-swizzled with (row / 2) % 8, a wave-wide
// load moves 8 rows); a 128-bit read gives a lane four channels, which four instructions take in turn, two reads
// for every 16 channels, which enter in the order 0, 4, 8, 12, 1, 5, 9, 13 (one chain of sums) and 2, 6, 10, 14, 3, 7, 11,
// 15 (a second one): the order in which a 16 x 16 x 4 instruction meets them in 64-byte rows (layer.hip) (rounding error of M against 64 bits, geometric mean over 40 drawn layers: 0.83 times that of one
// multiply-add chain over the channels).  With plain multiply-add tiles (one
// 4-byte LDS read per 2 products, one step in flight) 40 -> 70 @45x61 batch 8 F(6,3) took 23.9 us, this way 13.5.
template <int BM, int BN, int WM, int WN, int S, typename ST, typename MT>
__global__ void __launch_bounds__(64 * WM * WN)
contract_tile_kernel(const ST *__restrict__ U, const ST *__restrict__ V, MT *__restrict__ Mo, int C,
                     int T, int Tp, int Kp, int c_blocks, int k_blocks, int row_blocks, int col_blocks)
{
    constexpr int ROW = kChanBlock * (int)sizeof(ST);       // bytes of 32 channels
    constexpr int SLOTS = ROW / 16, LOAD_ROWS = 1024 / ROW; // 16-byte slots per row, rows per wave-wide load
    constexpr int SWZ = sizeof(ST) == 2 ? 2 : 1;            // slot ^ (row >> SWZ) % SLOTS
    constexpr int WAVES = WM * WN;
    constexpr int MB = BM / WM / 32, NB = BN / WN / 32;     // 32 x 32 blocks per wave
    constexpr int GROUPS = (BM + BN) / LOAD_ROWS;           // wave-wide loads per stage
    constexpr int NP = (GROUPS + WAVES - 1) / WAVES;        // ... per wave (a surplus one repeats the wave's first)
    constexpr int STAGE = (BM + BN) * ROW;
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0 && S >= 3 && S * STAGE <= 64 * 1024, "tile shape");
    __shared__ __align__(1024) unsigned char ring[S * STAGE];
    const unsigned ring_base = (unsigned)(size_t)((__attribute__((address_space(3))) void *)ring);

    unsigned bid = xcd_local_block_id(blockIdx.x, gridDim.x);
    const int cbk = bid % col_blocks; bid /= col_blocks;
    const int rbk = bid % row_blocks; bid /= row_blocks;
    const int xi = bid;
    const int t0 = rbk * BM, k0 = cbk * BN;
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave / WN, wn = wave % WN;

    // lane l of a load: row l / SLOTS of the LOAD_ROWS, physical slot l % SLOTS
    const ST *src[NP];
    unsigned off[NP], dst[NP];
    size_t step[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        int grp = wave + i * WAVES;
        if (grp >= GROUPS) grp = wave;
        const bool of_v = grp * LOAD_ROWS < BM;
        int row = grp * LOAD_ROWS - (of_v ? 0 : BM) + lane / SLOTS;
        const unsigned slot = (unsigned)((lane % SLOTS) ^ ((row >> SWZ) % SLOTS));
        const int last = of_v ? T - 1 - t0 : Kp - 1 - k0;
        if (row > last) row = last;
        off[i] = (unsigned)row * (unsigned)ROW + slot * 16u;
        src[i] = uniform_pointer(of_v ? V + ((size_t)xi * c_blocks * T + t0) * kChanBlock : U + ((size_t)xi * c_blocks * Kp + k0) * kChanBlock);
        step[i] = (size_t)(of_v ? T : Kp) * kChanBlock;
        dst[i] = ring_base + (unsigned)grp * 1024u;
    }
    int issued = 0;
    auto issue_stage = [&](int slot) __attribute__((always_inline)) {
        const bool surplus = issued >= c_blocks;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            global_to_lds16<false>(src[i], surplus ? 0u : off[i], (unsigned)__builtin_amdgcn_readfirstlane((int)(dst[i] + (unsigned)(slot * STAGE))));
            if (issued + 1 < c_blocks) src[i] = uniform_pointer(src[i] + step[i]);
        }
        ++issued;
    };

    constexpr int CHAINS = sizeof(ST) == 4 ? 2 : 1;
    float16v acc[CHAINS][NB][MB];
#pragma unroll
    for (int ch = 0; ch < CHAINS; ++ch)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[ch][j][i][e] = 0.0f;

    for (int j = 0; j < S - 1; ++j) issue_stage(j);
    const int frag_row = lane & 31, swz = (frag_row >> SWZ) % SLOTS;
    int frag_off[SLOTS / 2];
#pragma unroll
    for (int kk = 0; kk < SLOTS / 2; ++kk) frag_off[kk] = frag_row * ROW + (((kk * 2 + (lane >> 5)) ^ swz) * 16);
    int slot = 0;
    for (int cb = 0; cb < c_blocks; ++cb) {
        stream_wait<(S - 2) * NP>();                       // this wave's pieces of the stage have landed
        __syncthreads();                                   // everyone's have; the slot before is free again
        issue_stage(slot == 0 ? S - 1 : slot - 1);
        const unsigned char *stage = ring + slot * STAGE;
        // fragments of 16 channels: one read in binary16, two (channels 0..7 and 8..15) in binary32
        typedef typename std::conditional<sizeof(ST) == 2, half8, float4f>::type frag_t;
        constexpr int READS = sizeof(ST) == 2 ? 1 : 2;
#pragma unroll
        for (int kk = 0; kk < SLOTS / 2; kk += READS) {
            // (binary32: channels past C are zero on both sides and need not be multiplied)
            const int left = C - cb * kChanBlock - kk * 8;
            if (sizeof(ST) == 4 && left <= 0) break;
            frag_t vf[READS][MB], uf[READS][NB];
#pragma unroll
            for (int q = 0; q < READS; ++q) {
#pragma unroll
                for (int i = 0; i < MB; ++i) vf[q][i] = *reinterpret_cast<const frag_t *>(stage + (wm * MB + i) * 32 * ROW + frag_off[kk + q]);
#pragma unroll
                for (int j = 0; j < NB; ++j) uf[q][j] = *reinterpret_cast<const frag_t *>(stage + BM * ROW + (wn * NB + j) * 32 * ROW + frag_off[kk + q]);
            }
            if constexpr (sizeof(ST) == 2) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int i = 0; i < MB; ++i) acc[0][j][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[0][i], uf[0][j], acc[0][j][i], 0, 0, 0);
            } else {
                // (the two chains in turn, so that one's instruction does not wait for the one before)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int q = 0; q < READS; ++q) {
                        if (q == 1 && left <= 8) continue;
#pragma unroll
                        for (int ch = 0; ch < 2; ++ch)
#pragma unroll
                            for (int j = 0; j < NB; ++j)
#pragma unroll
                                for (int i = 0; i < MB; ++i) {
                                    float16v &sum = acc[ch % CHAINS][j][i];
                                    sum = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[q][i][2 * ch + e], uf[q][j][2 * ch + e], sum, 0, 0, 0);
                                }
                    }
            }
        }
        slot = slot == S - 1 ? 0 : slot + 1;
    }
    // the surplus loads must land before the LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // D[row = t][col = k]: lane holds channel lane%32 of a block and tiles 8*(e/4) + 4*(lane/32) + e%4, so that a
    // store covers two whole 128-byte rows of M (with U as the row operand a lane has four neighbouring channels,
    // and a store 32 pieces of 32 bytes: a quarter as many stores, 5-30 % slower)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int kb = (k0 >> 5) + wn * NB + j;
        if (kb >= k_blocks) continue;
        MT *plane = Mo + ((size_t)xi * k_blocks + kb) * (size_t)Tp * kChanBlock + frag_row;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int t = t0 + (wm * MB + i) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                float sum = acc[0][j][i][e];
                if constexpr (CHAINS == 2) sum += acc[CHAINS - 1][j][i][e];
                if (t < T) store_from_f32(plane + (size_t)t * kChanBlock, sum);
            }
    }
}

// ---------------------------------------------------------------------------------------------
// Weight-stationary streaming variant.
//
// The contraction is bound by HBM traffic (V in, M out), not by the matrix cores, and a tiled
// GEMM that reloads U and V per output tile is held back by load latency: it never has enough
// bytes in flight.  Here a workgroup keeps its slice of U[xi] -- NB*32 output channels x all C
// input channels per wave -- in VGPRs as ready-made MFMA fragments, and streams its share of
// V[xi] exactly once through a ring of S stages in LDS, filled by direct global->LDS loads (no
// destination registers), S-1 stages in flight.  A stage is SR = 32*WM consecutive tiles t with
// all C channels, so each stage yields finished outputs (no accumulation across stages) which go
// straight from the accumulators to M.  A segment = all stages of one (k-group, xi): the unit
// that shares one set of U fragments.  The grid is sized to what is resident at once (OCC
// workgroups per CU); if that is at least the number of segments, each segment is split among
// several workgroups and nobody reloads U, otherwise each workgroup takes a contiguous, equal
// share of all stages and walks through it segment by segment.
//   WN x WM waves; WN split the output channels, WM the rows of a stage.
//   CB = C/32 (fixes the registers for the U fragments).
// Two workgroups per CU where registers and LDS allow: the stores throttle the wave that issues
// them when HBM writes back up, and a second workgroup's MFMAs and loads fill those gaps.
//
// Waiting.  The hardware retires the vector-memory operations of a wave in issue order, and
// `s_waitcnt vmcnt(X)` waits until at most X are outstanding; so an operation with at least X
// younger ones is complete after the wait.  The compiler's own bookkeeping cannot express "all
// but the newest S-2 stages" across the loop, so the streaming loads and the stores are issued
// through inline assembly (which it does not count) and waited for with explicit counts.  Every
// stage issues exactly NP loads and NS stores per thread, nothing conditional; the compiler's own
// loads of U are complete before the loop over stages starts.
// The direct loads write LDS, not registers, so nothing the compiler allocates is written behind
// its back; their "memory" clobber keeps LDS reads from moving across them.
// Addresses are `uniform 64-bit base (scalar registers) + 32-bit per-lane byte offset`: one VGPR
// per access instead of two, which this kernel's register budget needs.
__device__ __forceinline__ void stream_to_lds16(const void *uniform_base, unsigned byte_offset, unsigned lds_wave_base)
{
    global_to_lds16<false>(uniform_base, byte_offset, lds_wave_base);
}
template <int IMM>
__device__ __forceinline__ void stream_store(float *uniform_base, unsigned byte_offset, float a)
{
    asm volatile("global_store_dword %0, %1, %2 offset:%3" : : "v"(byte_offset), "v"(a), "s"(uniform_base), "n"(IMM) : "memory");
}
template <int IMM>
__device__ __forceinline__ void stream_store(f16 *uniform_base, unsigned byte_offset, float a)
{
    const f16 v = (f16)a;
    asm volatile("global_store_short %0, %1, %2 offset:%3" : : "v"(byte_offset), "v"(v), "s"(uniform_base), "n"(IMM) : "memory");
}
template <typename MT, int E = 0>
__device__ __forceinline__ void stream_store_block(MT *plane, unsigned m_off, const float16v &acc)
{
    if constexpr (E < 16) {
        stream_store<((E >> 2) * 8 + (E & 3)) * kChanBlock * (int)sizeof(MT)>(plane, m_off, acc[E]);
        stream_store_block<MT, E + 1>(plane, m_off, acc);
    }
}
// wait for the loads of the i-th stage of this workgroup (i counted from its first stage):
// younger operations = (S-2) stages of loads plus the stores of the min(i, S-1) stages completed
// since that stage was issued
template <int I, int S, int NP, int NS>
__device__ __forceinline__ void stream_wait_stage(int i)
{
    if constexpr (I == S - 1) {
        stream_wait<(S - 2) * NP + NS * (S - 1)>();
    } else {
        if (i == I) stream_wait<(S - 2) * NP + NS * I>();
        else stream_wait_stage<I + 1, S, NP, NS>(i);
    }
}

// WN x WM waves: WN split the output channels (NB blocks of 32 each, so WN*NB*32 per workgroup),
// WM split the rows of a stage (SR = 32*WM tiles).  OCC = workgroups per CU the registers and the
// LDS ring are budgeted for: with two, one workgroup's MFMAs overlap the other's stores, which
// throttle the issuing wave when HBM writes back up.
template <int WN, int WM, int NB, int CB, int S, int OCC, typename MT>
// (the second launch bound is waves per SIMD: a workgroup puts WN*WM/4 on each)
__global__ void __launch_bounds__(64 * WN * WM, (OCC * WN * WM + 3) / 4)
contract_stream_kernel(const f16 *__restrict__ U, const f16 *__restrict__ V, MT *__restrict__ Mo,
                       int T, int Tp, int Kp, int k_blocks, int stages_per_xi, int xi_count, int items_total, int wgs_per_seg)
{
    constexpr int THREADS = 64 * WN * WM;
    constexpr int SR = 32 * WM;                      // rows (tiles t) per stage
    constexpr int NP = CB * SR * 4 / THREADS;        // 16-byte loads per thread and stage
    constexpr int NS = 16 * NB;                      // stores per thread and stage
    constexpr int STAGE_BYTES = CB * SR * 64;        // [CB][SR] rows of 32 binary16 channels
    static_assert(NP >= 1 && NP * THREADS == CB * SR * 4 && S >= 3 && S * STAGE_BYTES * OCC <= 144 * 1024,
                  "pipeline shape");
    static_assert(THREADS / 4 % 16 == 0, "the swizzle term (r/4)%4 must not depend on the piece index i");

    __shared__ __align__(1024) unsigned char ring[S * STAGE_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int frag_row = lane & 31;
    const unsigned ring_base = (unsigned)(size_t)((__attribute__((address_space(3))) void *)ring);

    // Work items: item = ((kg * xi_count) + xi) * stages_per_xi + tb; a run of stages_per_xi items
    // with the same (kg, xi) is a segment and needs one load of U fragments.  If there are at least
    // as many workgroups as segments, wgs_per_seg of them share each segment and nobody reloads U in
    // mid-stream; otherwise every workgroup takes a contiguous, equal share of all items.
    // (Workgroups that are neighbours in this order run on the same XCD, so a U[xi] slice shared by
    // several of them is fetched into one L2 only.)
    const unsigned wg = xcd_local_block_id(blockIdx.x, gridDim.x);
    int g0, g1;
    if (wgs_per_seg > 0) {
        const int seg0 = wg / wgs_per_seg, part = wg - seg0 * wgs_per_seg;
        g0 = seg0 * stages_per_xi + (int)((long long)stages_per_xi * part / wgs_per_seg);
        g1 = seg0 * stages_per_xi + (int)((long long)stages_per_xi * (part + 1) / wgs_per_seg);
    } else {
        g0 = (int)((long long)items_total * wg / gridDim.x);
        g1 = (int)((long long)items_total * (wg + 1) / gridDim.x);
    }
    if (g0 >= g1) return;

    // Piece p = tid + THREADS*i of a stage sits at LDS offset 16*p: row r = p/4 of the stage
    // ([channel block][tile] order), physical 16-byte slot p%4.  The logical slot (which 8 channels
    // of the row) is XOR-ed with (r/4)%4, so that the 16 rows a 128-bit fragment read touches in one
    // phase fall into 16 different bank groups.  Each lane picks the global address that belongs in
    // its fixed LDS slot.
    const int p_q = (tid & 3) ^ ((tid >> 4) & 3);        // (r/4)%4 with r = tid/4 + (THREADS/4)*i
    // fragment reads: row cb*SR + wm*32 + frag_row, logical slot 2*kk + lane/32
    const int swz = (frag_row >> 2) & 3;                 // (r/4)%4 of those rows (SR is a multiple of 32)
    int frag_off[2];
    for (int kk = 0; kk < 2; ++kk) frag_off[kk] = (wm * 32 + frag_row) * 64 + (((kk * 2 + (lane >> 5)) ^ swz) * 16);
    const unsigned u_lane_off = (unsigned)((frag_row * kChanBlock + (lane >> 5) * 8) * (int)sizeof(f16));

    // One pass of the outer loop = the part of this workgroup's range that lies in one segment.
    for (int g = g0; g < g1;) {
        const int seg = g / stages_per_xi;                 // = kg * xi_count + xi
        const int kg = seg / xi_count, xi = seg - kg * xi_count;
        const int tb0 = g - seg * stages_per_xi;
        int count = stages_per_xi - tb0;                   // stages of this pass
        if (count > g1 - g) count = g1 - g;
        g += count;
        const f16 *v_plane = uniform_pointer(V + (size_t)xi * CB * T * kChanBlock);

        // stage j of the pass -> ring slot; past the end of the pass the loads are still issued
        // (the wait counts assume a fixed number per stage) but every lane rereads the first 16
        // bytes of the plane: one cached request
        auto issue_stage = [&](int j, int slot) __attribute__((always_inline)) {
            const bool surplus = j > count - 1;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int r = (tid >> 2) + i * (THREADS / 4);    // row of the stage: [channel block][tile]
                const int cb = r / SR, row = r % SR;             // SR is a power of two
                int t = (tb0 + j) * SR + row; if (t > T - 1) t = T - 1;      // rows past the end: reread the last
                const unsigned off = surplus ? 0u : ((unsigned)(cb * T + t) * kChanBlock + (unsigned)p_q * 8u) * (unsigned)sizeof(f16);
                stream_to_lds16(v_plane, off, ring_base + slot * STAGE_BYTES + (i * THREADS + wave * 64) * 16);
            }
        };
        for (int j = 0; j < S - 1; ++j) issue_stage(j, j);       // S-1 stages in flight

        // this wave's NB*32 output channels x all C channels of U[xi], as ready-made MFMA fragments:
        // uniform base per (block of 32 channels out, block of 32 channels in) + one per-lane offset
        half8 ufrag[NB][CB][2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int k0 = ((kg * WN + wn) * NB + nb) * 32;               // k0 + 31 < Kp: Kp is a multiple of WN*NB*32
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const f16 *blk = U + (((size_t)xi * CB + cb) * Kp + k0) * kChanBlock;
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
                    ufrag[nb][cb][kk] = *reinterpret_cast<const NOVA_GLOBAL half8 *>(plane_element(blk + kk * 16, u_lane_off));
            }
        }
        // Pin the fragments here: each empty statement below consumes and redefines one of them, so
        // the compiler must have the load issued and waited for at this point and cannot sink either
        // into the loop.  Its wait for the youngest of them is vmcnt(0), which also covers the S-1
        // stages above (they are older); from here on only operations issued through inline
        // assembly are outstanding, as the counts in the loop assume.
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) asm volatile("" : "+v"(ufrag[nb][cb][kk]));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

        MT *m_plane = uniform_pointer(Mo + ((size_t)xi * k_blocks + (size_t)(kg * WN + wn) * NB) * Tp * kChanBlock);
        // lane holds output channel lane%32 of each block and t = 8*(e/4) + 4*(lane/32) + e%4: a store covers two
        // whole 128-byte rows of M; rows up to Tp exist, so no store is conditional
        unsigned m_off = ((unsigned)(tb0 * SR + wm * 32 + (lane >> 5) * 4) * kChanBlock + (unsigned)frag_row) * (unsigned)sizeof(MT);
        int slot = 0;
        for (int j = 0; j < count; ++j) {
            stream_wait_stage<0, S, NP, NS>(j);                // this wave's pieces of stage j have landed
            __syncthreads();                                   // everyone's have; slot-1 is free again
            issue_stage(j + S - 1, slot == 0 ? S - 1 : slot - 1);

            // acc[nb] = V-stage rows (32 tiles) x U-block (32 output channels): D[row = t][col = k]
            float16v acc[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[nb][e] = 0.0f;
            const unsigned char *stage = ring + slot * STAGE_BYTES;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const half8 vf = *reinterpret_cast<const half8 *>(stage + cb * SR * 64 + frag_off[kk]);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, ufrag[nb][cb][kk], acc[nb], 0, 0, 0);
                    // keep the fragment reads of later channel blocks from being hoisted all the way
                    // up: sixteen 128-bit fragments in flight at once do not fit the register budget
                    if (kk == 1) __builtin_amdgcn_sched_barrier(0);
                }

            // The stores are inline assembly and read the accumulators directly; the compiler inserts
            // the wait states an MFMA result needs before a vector-memory instruction may read it
            // only for instructions it schedules itself, so they are spelled out here (the longest
            // requirement, for a 16-pass MFMA, is 18).
            asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                MT *plane = m_plane + (size_t)nb * Tp * kChanBlock;
                stream_store_block<MT>(plane, m_off, acc[nb]);
            }
            m_off += (unsigned)(SR * kChanBlock) * (unsigned)sizeof(MT);
            slot = slot == S - 1 ? 0 : slot + 1;
        }
        // the surplus prefetches of the tail must land before the ring is refilled or released,
        // and every wave must be done reading before the next pass overwrites it
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
}

template <int BM, int BN, int WM, int WN, int S, typename ST, typename MT>
static int launch_tile(const void *U, const void *V, void *Mo, const Geometry &g, hipStream_t stream)
{
    const int row_blocks = ceil_div((int)g.T, BM), col_blocks = ceil_div(g.Kp, BN);
    const long long blocks = (long long)g.n * g.n * row_blocks * col_blocks;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL((contract_tile_kernel<BM, BN, WM, WN, S, ST, MT>), dim3((unsigned)blocks), dim3(64 * WM * WN), 0, stream,
                       (const ST *)U, (const ST *)V, (MT *)Mo, g.C, (int)g.T, (int)g.Tp, g.Kp, g.c_blocks, g.k_blocks,
                       row_blocks, col_blocks);
    return (int)hipGetLastError();
}

template <int WN, int WM, int NB, int CB, int S, int OCC, typename MT>
static int launch_stream(const void *U, const void *V, void *Mo, const Geometry &g, hipStream_t stream)
{
    constexpr int SR = 32 * WM;
    const int slots = device_cu_count() * OCC;           // workgroups resident at once
    const int stages_per_xi = ceil_div((int)g.T, SR);
    const int kgroups = g.Kp / (WN * NB * 32);
    const long long segs = (long long)kgroups * g.n * g.n;
    const long long items = segs * stages_per_xi;
    if (items <= 0 || items > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    // 32-bit byte offsets inside one xi plane of V and one (xi, channel block) plane of M
    if ((size_t)g.c_blocks * g.T * kChanBlock * sizeof(f16) >= ((size_t)1 << 32) ||
        (size_t)g.Tp * kChanBlock * sizeof(MT) >= ((size_t)1 << 32)) return (int)hipErrorInvalidValue;
    int wgs_per_seg = (int)(slots / segs);
    if (wgs_per_seg > stages_per_xi) wgs_per_seg = stages_per_xi;
    const int blocks = wgs_per_seg > 0 ? (int)(segs * wgs_per_seg) : (int)(items < slots ? items : slots);
    hipLaunchKernelGGL((contract_stream_kernel<WN, WM, NB, CB, S, OCC, MT>), dim3(blocks), dim3(64 * WN * WM), 0, stream,
                       (const f16 *)U, (const f16 *)V, (MT *)Mo, (int)g.T, (int)g.Tp, g.Kp, g.k_blocks,
                       stages_per_xi, g.n * g.n, (int)items, wgs_per_seg);
    return (int)hipGetLastError();
}

// Tile shape (us per launch, buffers alternating so that nothing is found in the cache).  64 x 64 fills the chip
// soonest and is the fastest one on small layers: 48 -> 96 5x5 @35x35 batch 16 12.0 (128 x 64: 15.2), 512 -> 512
// @14x14 batch 1 F(4,3) 6.6 (8.2), 128 -> 128 @112x112 batch 5 F(6,3), 15 M products, 15.6 (16.6).  Larger tiles read
// U and V less often: 128 x 128 by 8 waves in long channel loops once it fills the chip as well (512 -> 512 @7x7
// F(8,3) batch 256 30.7 against 36.0 and 41.8 for 128 x 64 and 64 x 64, batch 128 15.8 against 20.3 and 17.4), but not
// for 64 output channels or fewer, where half of them would be padding (whole calls, 128 x 128 / the tile taken instead:
// 256 -> 64 @56x56 F(6,3) batch 16 42.7 / 41.0, 512 -> 64 @60x60 F(8,3) batch 7 44.7 / 43.3; the contraction alone there
// 12.9 / 11.5), nor for 64 tiles or fewer, where half of the rows would be (512 -> 512 @7x7 F(8,3), 9 images 11.9 / 10.7, 40 13.2 / 12.8;
// 241 -> 512 with 9 tiles 7.9 / 7.2); 128 x 64 in other large layers (164 -> 33 @98x29 batch 43 F(4,3), 20 M, 38.4 against 41.4; 64 -> 64
// @112x112 batch 32 F(4,3), 58 M, 56.0 against 59.7).  One block of output channels: 128 x 32, none of it padding.
template <typename MT>
static int launch_c16_tiled(const void *U, const void *V, void *Mo, const Geometry &g, hipStream_t s)
{
    if (g.Kp == 32) return launch_tile<128, 32, 4, 1, 3, f16, MT>(U, V, Mo, g, s);
    const double positions = (double)g.n * g.n;
    if (g.c_blocks >= 8 && g.Kp > 64 && g.T > 64 && positions * ceil_div((int)g.T, 128) * ceil_div(g.Kp, 128) >= 400)
        return launch_tile<128, 128, 2, 4, 3, f16, MT>(U, V, Mo, g, s);
    if (positions * (double)g.T * g.Kp >= 16e6) return launch_tile<128, 64, 2, 2, 3, f16, MT>(U, V, Mo, g, s);
    // Long channel loops on a chip that few workgroups leave half empty: a ring of 5, more in flight per workgroup.  With U from
    // memory (the 13-layer stack on one image, 118 MB of U, eight layers of 512 channels or to them) 209.7 us with 3, 203.5 with 4, 203.2 with 5; with U in
    // the last-level cache the same (0.99 to 1.0 up to 384 workgroups, 0.96 from there on, 0.92 from 1000 on).
    if (g.c_blocks >= 8 && positions * ceil_div((int)g.T, 64) * ceil_div(g.Kp, 64) <= 384) return launch_tile<64, 64, 2, 2, 5, f16, MT>(U, V, Mo, g, s);
    return launch_tile<64, 64, 2, 2, 3, f16, MT>(U, V, Mo, g, s);
}

// The streaming kernel takes C in {64, 128, 256} and K a multiple of 128 where there are enough stages per
// workgroup to pay for its start (the U fragments): by the number of products, streaming / best tile in us:
//   C = 256, M binary32: from 12 M  (256 -> 256 @56x56 F(8,3) batch 12, 15 M: 19.3 / 20.1, batch 32, 40 M: 44 / 64;
//                                    F(6,3) @28x28 batch 24, 10 M: 15.6 / 14.6)
//   C = 128: from 24 M              (128 -> 128 @112x112 F(6,3) batch 11, 33 M: 32.5 / 35.8, batch 5, 15 M: 16.5 / 15.6)
//   C = 64: from 40 M               (64 -> 128 @224x224 F(4,3) batch 8, 116 M: 99 / 107; 64 -> 256 @56x56, 36 M: 26 / 26)
//   M binary16: from 16 M           (256 -> 256 @14x14 F(8,3) batch 256, 26 M: 22.9 / 31.8; 64 -> 256 @56x56, 60 M: 27 / 45)
// (C = 512 variants, 16 channel blocks in 128 fragment registers at one workgroup per CU, measured no faster than
// tiles at T = 512 and slower at T = 128.)  Ring depth S: as many stages as fit about 128 KiB of LDS, at most 8.
template <typename MT>
static int launch_c16_shape(const void *U, const void *V, void *Mo, const Geometry &g, hipStream_t s)
{
    const int cb = g.c_blocks;
    const double products = (double)g.n * g.n * (double)g.T * g.Kp;
    const double from = sizeof(MT) == 2 ? 16e6 : cb == 8 ? 12e6 : cb == 4 ? 24e6 : 40e6;
    if ((cb == 2 || cb == 4 || cb == 8) && g.Kp % 128 == 0 && products >= from) {
        const bool wide = g.Kp % 256 == 0;
        //                                              WN WM NB CB  S OCC
        if (wide && cb == 8) return launch_stream<8, 1, 1, 8, 4, 2, MT>(U, V, Mo, g, s);   // 8 waves x 32 channels
        if (wide && cb == 4) return launch_stream<4, 1, 2, 4, 8, 2, MT>(U, V, Mo, g, s);
        if (wide) return launch_stream<4, 1, 2, 2, 8, 2, MT>(U, V, Mo, g, s);
        if (cb == 8) return launch_stream<2, 2, 2, 8, 4, 1, MT>(U, V, Mo, g, s);
        if (cb == 4) return launch_stream<2, 2, 2, 4, 4, 2, MT>(U, V, Mo, g, s);
        return launch_stream<2, 2, 2, 2, 8, 2, MT>(U, V, Mo, g, s);
    }
    return launch_c16_tiled<MT>(U, V, Mo, g, s);
}

int launch_contract(const nova_transforms *, const void *U, const void *V, void *Mo, const Geometry &g,
                    int dtype, int flags, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (g.T > 0x7fffffffLL) return (int)hipErrorInvalidValue;
    if (dtype == NOVA_F16)
        return (flags & NOVA_FLAG_M_F16) ? launch_c16_shape<f16>(U, V, Mo, g, s)
                                         : launch_c16_shape<float>(U, V, Mo, g, s);
    if (g.Kp == 32) return launch_tile<64, 32, 2, 1, 3, float, float>(U, V, Mo, g, s);
    return launch_tile<64, 64, 2, 2, 3, float, float>(U, V, Mo, g, s);
}

}  // namespace nova
