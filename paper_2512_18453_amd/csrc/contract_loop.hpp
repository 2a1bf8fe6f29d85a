// The channel loop of contract_columns.hip: tiles of BM rows of V (winograd tiles) by BN rows of U (output channels), binary16, on
// v_mfma_f32_32x32x16_f16 with WM x WN waves.  (The tiled contraction of contract.hip has a ring of its own; with this loop in its
// place it was 0.8 to 1.0 times as fast: there workgroups per compute unit count for more than instructions per stage.)
//
// A stage is one block of 32 channels: (BM + BN) rows of 64 bytes each, XOR-swizzled by 16-byte slot (slot ^ (row / 4) % 4: the 16
// rows that a 128-bit fragment read touches in one phase fall into different bank groups).  Stages arrive in a
// ring of S in LDS by direct global->LDS loads, S - 1 ahead.
// With few waves per SIMD the number of instructions counts: a wave alone issues one about every four clocks.  A 64-bit
// pointer per load and M0 handed back after each made 150 scalar instructions per stage, 0.2 us with nothing to wait
// for; hence one pointer per operand, a 32-bit offset per load that never changes, and the loads of an operand in one
// statement (45 scalar instructions; 256 -> 256 @56x56 F(8,3) batch 32, contraction with columns, 53 -> 46 us).
#pragma once
#include "device_common.hpp"

namespace nova {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

// COUNT direct loads of 64 16-byte pieces each, uniform_base + off[k] -> LDS at lds_base + AT(k)
template <int A1, int A2, int A3, int COUNT>
__device__ __forceinline__ void loads_to_lds(const void *uniform_base, const unsigned (&off)[COUNT], unsigned lds_base)
{
    unsigned saved_m0;
#define NOVA_FIRST "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %2\n\t"
#define NOVA_NEXT(AT, OFF) "s_add_u32 m0, %1, " AT "\n\ts_nop 0\n\tglobal_load_lds_dwordx4 " OFF ", %2\n\t"
    if constexpr (COUNT == 1)
        asm volatile(NOVA_FIRST "s_mov_b32 m0, %0" : "=&s"(saved_m0) : "s"(lds_base), "s"(uniform_base), "v"(off[0]) : "memory");
    else if constexpr (COUNT == 2)
        asm volatile(NOVA_FIRST NOVA_NEXT("%5", "%4") "s_mov_b32 m0, %0"
                     : "=&s"(saved_m0) : "s"(lds_base), "s"(uniform_base), "v"(off[0]), "v"(off[1]), "n"(A1) : "memory", "scc");
    else {
        static_assert(COUNT == 4, "loads per statement");
        asm volatile(NOVA_FIRST NOVA_NEXT("%7", "%4") NOVA_NEXT("%8", "%5") NOVA_NEXT("%9", "%6") "s_mov_b32 m0, %0"
                     : "=&s"(saved_m0)
                     : "s"(lds_base), "s"(uniform_base), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "n"(A1), "n"(A2), "n"(A3)
                     : "memory", "scc");
    }
#undef NOVA_FIRST
#undef NOVA_NEXT
}

template <int BM, int BN, int WM, int WN, int S>
struct ChannelLoop {
    static constexpr int ROW = 64, STAGE = (BM + BN) * ROW, WAVES = WM * WN;
    static constexpr int LDS_BYTES = S * STAGE;
    static constexpr int MB = BM / WM / 32, NB = BN / WN / 32;              // 32 x 32 blocks per wave
    static constexpr int VG = BM / 16, UG = BN / 16;                        // wave-wide loads (16 rows) of a channel block
    static constexpr int NV = (VG + WAVES - 1) / WAVES, NU = (UG + WAVES - 1) / WAVES;      // ... per wave (a surplus one repeats another's)
    static_assert((VG % WAVES == 0 || WAVES % VG == 0) && (UG % WAVES == 0 || WAVES % UG == 0) && MB >= 1 && NB >= 1 && S >= 3, "tile shape");

    const f16 *v_at, *u_at;                       // first row of the stage issued next
    unsigned v_off[NV], u_off[NU];                // bytes from there, of the lane's piece of each load
    long long v_step, u_step, v_turn, u_turn;     // elements to the next stage, and from a position's last stage to the next position
    int c_blocks, to_issue, in_turn;              // stages per position; not yet issued: in all, of the position
    unsigned v_lds, u_lds;
    int v_frag[2], u_frag[2];

    // v0, u0: the first position's first channel block at the tile's first rows; v_rows, u_rows: rows of a channel block;
    // v_last, u_last: last row, from the tile's first, that exists (rows beyond it reread it; their products are not
    // stored); positions visited, position_step channel blocks from one to the next
    __device__ __forceinline__ void start(const unsigned char *ring, const f16 *v0, const f16 *u0, int v_rows, int u_rows, int v_last, int u_last,
                                          int blocks, int positions, long long position_step)
    {
        const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int wm = wave / WN, wn = wave % WN;
        v_at = uniform_pointer(v0);
        u_at = uniform_pointer(u0);
        auto offset = [&](int g, int last) __attribute__((always_inline)) {
            int row = g * 16 + lane / 4;
            const unsigned slot = (unsigned)((lane % 4) ^ ((row >> 2) % 4));
            if (row > last) row = last;
            return (unsigned)row * (unsigned)ROW + slot * 16u;
        };
        const int vw = wave % VG, uw = wave % UG;
#pragma unroll
        for (int i = 0; i < NV; ++i) v_off[i] = offset(vw + i * WAVES, v_last);
#pragma unroll
        for (int i = 0; i < NU; ++i) u_off[i] = offset(uw + i * WAVES, u_last);
        c_blocks = blocks;
        to_issue = blocks * positions;
        in_turn = blocks;
        v_step = (long long)v_rows * kChanBlock;
        u_step = (long long)u_rows * kChanBlock;
        v_turn = (position_step - (blocks - 1)) * v_rows * kChanBlock;
        u_turn = (position_step - (blocks - 1)) * u_rows * kChanBlock;
        const unsigned ring_at = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(size_t)((__attribute__((address_space(3))) const void *)ring));
        v_lds = ring_at + (unsigned)(vw * 1024);
        u_lds = ring_at + (unsigned)(BM * ROW + uw * 1024);
        const int frag_row = lane & 31, swz = (frag_row >> 2) % 4;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int in_row = ((kk * 2 + (lane >> 5)) ^ swz) * 16;
            v_frag[kk] = (wm * MB * 32 + frag_row) * ROW + in_row;
            u_frag[kk] = (BM + wn * NB * 32 + frag_row) * ROW + in_row;
        }
    }

    // The next stage's loads, to place `slot` of the ring.  Past the last stage every lane rereads the same 16 bytes, so that
    // the wait counts are constants.
    __device__ __forceinline__ void issue(int slot)
    {
        const unsigned mask = to_issue > 0 ? ~0u : 0u;
        unsigned off[NV], offu[NU];
#pragma unroll
        for (int i = 0; i < NV; ++i) off[i] = v_off[i] & mask;
#pragma unroll
        for (int i = 0; i < NU; ++i) offu[i] = u_off[i] & mask;
        loads_to_lds<WAVES * 1024, 2 * WAVES * 1024, 3 * WAVES * 1024>(v_at, off, v_lds + (unsigned)(slot * STAGE));
        loads_to_lds<WAVES * 1024, 2 * WAVES * 1024, 3 * WAVES * 1024>(u_at, offu, u_lds + (unsigned)(slot * STAGE));
        const bool more = to_issue > 1, turn = in_turn == 1;
        v_at += more ? (turn ? v_turn : v_step) : 0;
        u_at += more ? (turn ? u_turn : u_step) : 0;
        --to_issue;
        in_turn = turn ? c_blocks : in_turn - 1;
    }

    __device__ __forceinline__ void fill()
    {
        for (int j = 0; j < S - 1; ++j) issue(j);
    }
    // The products of one position; slot: of its first stage, moved on to that of the next position's.
    // D[row = t][col = k]: lane holds channel lane % 32 of a block and tiles 8 (e / 4) + 4 (lane / 32) + e % 4
    __device__ __forceinline__ void position(const unsigned char *ring, int &slot, float16v (&sum)[NB][MB])
    {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[j][i][e] = 0.0f;
#pragma unroll 1
        for (int st = 0; st < c_blocks; ++st) {
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"((S - 2) * (NV + NU)) : "memory");      // this wave's pieces of the stage have landed
            __syncthreads();                                                                 // everyone's have; the slot before is free again
            const unsigned char *stage = ring + slot * STAGE;
            half8 vf[2][MB], uf[2][NB];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int i = 0; i < MB; ++i) vf[kk][i] = *reinterpret_cast<const half8 *>(stage + v_frag[kk] + i * 32 * ROW);
#pragma unroll
                for (int j = 0; j < NB; ++j) uf[kk][j] = *reinterpret_cast<const half8 *>(stage + u_frag[kk] + j * 32 * ROW);
            }
            issue(slot == 0 ? S - 1 : slot - 1);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int i = 0; i < MB; ++i) sum[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[kk][i], uf[kk][j], sum[j][i], 0, 0, 0);
            slot = slot == S - 1 ? 0 : slot + 1;
        }
    }
};

}  // namespace nova
