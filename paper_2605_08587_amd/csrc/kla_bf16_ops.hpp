// Device helpers shared by the bf16 chunk kernels (gfx950 only): native 128-bit register values,
// direct global->LDS copies, the transposing LDS read, the swizzle of token-major LDS tiles, the bf16
// MFMA with the slot order of kla_mma.hpp, and a wait on the vector-memory counter alone.
#pragma once
#include "kla_common.hpp"
#include "kla_mma.hpp"

namespace kla {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native 128-bit register value (never a stack object)
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void st16(void* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

// Swizzle of a token-major [64 x DK] bf16 tile in LDS: the index of a row's 16-byte piece is XORed with this function
// of the row (period 8 rows).  It is built for the way gfx950 serves a wave's LDS accesses, found with two-lane probes
// under the bank-conflict counter:
//   * a 128-bit read goes 16 lanes per cycle (256 bytes), in the lane sets {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31}
//     and the same + 32: the row-slot read of an A operand (lane (r, g): row r, piece 4 kp + g) puts, in one cycle,
//     eight rows at piece p and the other eight rows of the block at piece p ^ 1;
//   * a 64-bit read, the transposing one included, goes 32 lanes per cycle (0-31, 32-63): the K^T read puts rows
//     8 m .. 8 m + 7 at four consecutive pieces in one cycle, each lane taking one half of its piece, so two lanes per
//     piece position is the best possible (4 cycles per read);
//   * a 128-bit write goes 8 consecutive lanes per cycle (128 bytes), and positions 128 bytes apart collide: a wave that
//     stores row slots puts rows 8 m .. 8 m + 7 at one piece.
// With the masks below all three run without avoidable conflicts: 4, 4 and 8 cycles (a plain XOR with the low row
// bits costs 8, 8 and 8).  A row of DK = 64 covers half of the banks, so the row parity is part of the position.
template <int DK> __device__ __forceinline__ int swz_piece(int row)
{
    static_assert(DK == 64 || DK == 128, "tile widths of the chunk kernels");
    const int b0 = row & 1, b1 = (row >> 1) & 1, b2 = (row >> 2) & 1;
    return DK == 128 ? (b2 * 9) | (b0 << 2) | (b1 << 1) : (b1 << 2) | ((b0 ^ b2) << 1) | b2;
}

__device__ __forceinline__ u32x2 lds_read_tr(const char* p)
{
    const short4v v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(p));
    return __builtin_bit_cast(u32x2, v);
}

// 16 bytes per lane, global -> LDS without passing through registers: lane l's bytes land at
// lds_wave_base + 16 l.  `lds_wave_base` must be wave-uniform (it goes to M0).  Written as inline
// assembly on purpose: the compiler then keeps no book of these copies, so it puts no wait for them in
// front of LDS reads of OTHER ring stages; completion is awaited explicitly (wait_vmcnt + barrier).
// The global address is a wave-uniform base plus a 32-bit per-lane byte offset.
__device__ __forceinline__ void dma16(const char* gbase_uniform, int lane_off, char* lds_wave_base)
{
    const uint32_t m = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)lds_wave_base);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(gbase_uniform), "s"(m)
                 : "memory");
}

// One dword of one 128-byte line that all slices of a head will copy: the lines of two [64 x d_k] tiles (rows of RB bytes, `stride` apart,
// from row `row0` of `rows` on) and the first `n_rec` lines at `rec`, counted through in this order; i: which.  A wave that has nothing
// else to wait for asks for 128 of them, slice s for 128 s .. 128 s + 127, some chunks ahead of the copies, which then find their lines in
// L2: a CU's copies are in flight by the 64 KB, so what they take in per cycle falls with their latency.  (Where there are fewer slices
// than lines by the 128, the last lines are nobody's.)  The value is of no interest, but has to be
// waited for (by the next call's caller) before its register is free.
template <int RB> __device__ __forceinline__ uint32_t touch_line(const char* tile0, const char* tile1, size_t stride, int row0, int rows,
                                                                 const char* rec, int n_rec, int i)
{
    constexpr int LPR = RB / 128, NL = 64 * LPR;
    if (i >= 2 * NL + n_rec) return 0u;
    const int l = i % NL;
    const char* p = i < 2 * NL ? (i < NL ? tile0 : tile1) + (size_t)min(row0 + l / LPR, rows - 1) * stride + (l % LPR) * 128 : rec + (size_t)(i - 2 * NL) * 128;
    return *reinterpret_cast<const uint32_t*>(p);
}

// s_waitcnt on the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ void mma_bf16(floatx4& acc, u32x4 a, u32x2 b0, u32x2 b1)
{
    const u32x4 b = {b0.x, b0.y, b1.x, b1.y};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                  acc, 0, 0, 0);
}
__device__ __forceinline__ void mma_bf16(floatx4& acc, u32x2 a0, u32x2 a1, u32x2 b0, u32x2 b1)
{
    const u32x4 a = {a0.x, a0.y, a1.x, a1.y};
    mma_bf16(acc, a, b0, b1);
}
__device__ __forceinline__ u32x2 to_quad(floatx4 x)
{
    const u32x2 q = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])};
    return q;
}
__device__ __forceinline__ floatx4 quad_to_f(u32x2 q)
{
    floatx4 r;
    r[0] = __uint_as_float(q.x << 16); r[1] = __uint_as_float(q.x & 0xffff0000u);
    r[2] = __uint_as_float(q.y << 16); r[3] = __uint_as_float(q.y & 0xffff0000u);
    return r;
}
// A quad of lanes (r = 4 q .. 4 q + 3) holds a 4x4 block of bf16 of an accumulator tile: lane j rows 4 g + e (e = 0..3,
// packed in two dwords) of column 4 q + j.  Transposed inside the quad by two exchange steps (dwords with lane j ^ 2,
// halves with lane j ^ 1) each lane then owns 4 consecutive columns of row 4 g + (r & 3): one 64-bit LDS write per tile
// instead of four 16-bit ones.  q_lo = (r & 3) < 2; psel = (r & 1) ? 0x03020706 : 0x05040100.
__device__ __forceinline__ u32x2 quad_transpose4x4(u32x2 ob, bool q_lo, uint32_t psel)
{
    const uint32_t snd = q_lo ? ob.y : ob.x;
    const uint32_t rcv = (uint32_t)__builtin_amdgcn_mov_dpp((int)snd, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
    if (q_lo) ob.y = rcv; else ob.x = rcv;
    const uint32_t px = (uint32_t)__builtin_amdgcn_mov_dpp((int)ob.x, 0xB1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
    const uint32_t py = (uint32_t)__builtin_amdgcn_mov_dpp((int)ob.y, 0xB1, 0xf, 0xf, true);
    ob.x = __builtin_amdgcn_perm(px, ob.x, psel);
    ob.y = __builtin_amdgcn_perm(py, ob.y, psel);
    return ob;
}

// ---- what the sweeps leave in memory for the backward's assembly, written by the wave that holds it in registers ----
// Both in the order in which the registers are: every store instruction fills whole 1 KiB blocks, and no wave transposes or
// stages anything for them.  8 x 4096 tokens, 8 heads, d = 128, the whole backward: 476 us with rows transposed and staged in
// LDS and checkpoints in rows of d_k (64 bytes per row and store instruction), 468 with X and Y in operand order, 457 with
// the checkpoints too (the reverse sweep alone 157 -> 144 us).
//
// A state checkpoint (bf16, fragments q of the permuted feature index above), per chunk-head and 16 columns: 1 KiB per 32
// features, in it column r's 64 bytes = features 32 kp + 8 g .. + 7 for g = 0 .. 3.  chk: the chunk-head's first byte.
template <int DK> __device__ __forceinline__ void put_checkpoint(char* chk, int col_tile, const u32x2 (&q)[DK / 16], int r, int g)
{
    char* p = chk + col_tile * (16 * DK * 2) + r * 64 + g * 16;
#pragma unroll
    for (int kp = 0; kp < DK / 32; ++kp) {
        const u32x4 w = {q[2 * kp].x, q[2 * kp].y, q[2 * kp + 1].x, q[2 * kp + 1].y};
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p + kp * 1024));
    }
}
// The 64 rows of X or Y (quads q[it]: tokens 16 it + 4 g .. + 3 of column r), 16 columns at a time.  A whole chunk takes the
// bytes of its 64 rows of a [tokens][H][d_v] tensor and keeps them head after head, per head and 16 columns as the two 1 KiB
// tile-pairs of B-operand slots (kla_mma.hpp).  A short one has no room for its 64 rows: it is stored as rows.
// chunk: the first byte of the chunk's rows; v_row: bytes between tokens; hd: head.
__device__ __forceinline__ void put_rows(char* chunk, size_t v_row, int dv, int hd, int col_tile, const u32x2 (&q)[4], int clen, int r, int g)
{
    if (clen == 64) {
        char* p = chunk + (size_t)hd * dv * 128 + col_tile * 2048 + (16 * g + r) * 16;
#pragma unroll
        for (int jp = 0; jp < 2; ++jp) {
            const u32x4 w = {q[2 * jp].x, q[2 * jp].y, q[2 * jp + 1].x, q[2 * jp + 1].y};
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p + jp * 1024));
        }
    } else {
        // (once per sequence: the lane goes through an empty asm so that none of these addresses is kept in registers)
        asm volatile("" : "+v"(r), "+v"(g));
        char* p = chunk + (size_t)hd * dv * 2 + (16 * col_tile + r) * 2;
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * it + 4 * g + e;
                const uint32_t w = e < 2 ? q[it].x : q[it].y;
                if (row < clen) *reinterpret_cast<uint16_t*>(p + (size_t)row * v_row) = (uint16_t)((e & 1) ? w >> 16 : w & 0xffffu);
            }
    }
}
__device__ __forceinline__ floatx4 ld_f4(const char* p) { return *reinterpret_cast<const floatx4*>(p); }

}  // namespace kla
