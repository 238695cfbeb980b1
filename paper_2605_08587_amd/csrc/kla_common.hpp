// Shared device helpers for the gfx950 KLA kernels: element types, bf16 conversion,
// wave-level reductions.  gfx950 only (64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kla {

constexpr int kWave = 64;
constexpr int kChunk = 64;   // tokens per chunk (C in Algorithm 1, right panel)

// Storage type of a bf16 element: raw bits.  Arithmetic is never done in bf16; values are
// widened to fp32 exactly and rounded back with round-to-nearest-even.
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float to_float(float x) { return x; }
__device__ __forceinline__ float to_float(bf16_t x) { return __uint_as_float(((uint32_t)x.bits) << 16); }
__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ uint32_t float_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);                                    // round to nearest even
    return u >> 16;
}
// two fp32 -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float floatx2_t __attribute__((ext_vector_type(2)));
    const floatx2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

template <typename T> __device__ __forceinline__ T from_float(float f);
template <> __device__ __forceinline__ float from_float<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16_t from_float<bf16_t>(float f)
{
    bf16_t r; r.bits = (uint16_t)float_to_bf16_bits(f); return r;
}

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>).  Used where a
// register array must be indexed by constants from the start (so that it never becomes a stack object).
template <int I> struct IntC { static constexpr int value = I; constexpr operator int() const { return I; } };
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) { f(IntC<I>()); static_for<N, I + 1>(f); }
}

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, kWave);
    return x;
}

// Sums by DPP moves, which stay on the vector ALU (a shuffle goes through LDS): over the 16 lanes of a row, in every lane; over
// the wave, in every lane; and the inclusive prefix sum over the 64 lanes (shifts within rows, the rows joined through the scalar unit).
template <int CTRL> __device__ __forceinline__ float dpp_mov(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)); }
__device__ __forceinline__ float row_sum16(float x)
{
    x += dpp_mov<0xB1>(x);       // quad_perm [1,0,3,2]
    x += dpp_mov<0x4E>(x);       // quad_perm [2,3,0,1]
    x += dpp_mov<0x141>(x);      // row_half_mirror
    x += dpp_mov<0x140>(x);      // row_mirror
    return x;
}
__device__ __forceinline__ float lane_value(float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); }
__device__ __forceinline__ float wave_sum_rows(float x)
{
    x = row_sum16(x);
    return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}
__device__ __forceinline__ float prefix_sum64(float x, int lane)
{
    x += dpp_mov<0x111>(x);      // row_shr:1, 2, 4, 8
    x += dpp_mov<0x112>(x);
    x += dpp_mov<0x114>(x);
    x += dpp_mov<0x118>(x);
    const float r0 = lane_value(x, 15), r1 = lane_value(x, 31), r2 = lane_value(x, 47);
    return x + (lane < 16 ? 0.f : (lane < 32 ? r0 : (lane < 48 ? r0 + r1 : (r0 + r1) + r2)));
}

// Where a per-chunk workgroup works: global chunk index cg (sequences in order, chunks of 64 tokens counted from each
// sequence's own first token) -> first token of the chunk and its length (64, or less for a ragged last chunk).
// cu_seqlens / chunk_off (chunk_off[s] = number of chunks before sequence s) describe a packed batch; both NULL for a
// fixed-length batch of sequences of T tokens (NT chunks each).
struct ChunkPos { long tok0; int clen; };
__device__ __forceinline__ ChunkPos chunk_pos(const int* cu_seqlens, const int* chunk_off, int n_seq, int T, int NT, int cg)
{
    ChunkPos p;
    if (cu_seqlens) {
        int lo = 0, hi = n_seq - 1;                  // last s with chunk_off[s] <= cg
        while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (chunk_off[mid] <= cg) lo = mid; else hi = mid - 1; }
        const int c = cg - chunk_off[lo];
        const int s0 = cu_seqlens[lo], s1 = cu_seqlens[lo + 1];
        p.tok0 = (long)s0 + 64L * c;
        p.clen = min(64, s1 - (int)p.tok0);
    } else {
        const int n = cg / NT, c = cg % NT;
        p.tok0 = (long)n * T + 64L * c;
        p.clen = min(64, T - 64 * c);
    }
    return p;
}

// The same for a packed batch of at most 64 sequences straight from cu_seqlens, lane = sequence: one trip to memory instead
// of a kernel before this one and a binary search (16 sequences: 5 us per call).  Every lane of the wave takes part.
// out, if not NULL, receives what chunk_offsets_kernel leaves for the kernels behind: n_seq + 1 chunk offsets, then the
// sequences, most chunks first.
constexpr int kPosScanMax = 64;
__device__ __forceinline__ ChunkPos chunk_pos_scan(const int* cu_seqlens, int n_seq, int cg, int lane, int* out)
{
    const int s = min(lane, n_seq - 1);
    const int c0 = cu_seqlens[s], c1 = cu_seqlens[s + 1];
    const int nc = lane < n_seq ? (c1 - c0 + 63) / 64 : 0;
    int x = nc;                                          // inclusive prefix sum: DPP shifts within rows of 16 lanes, then the rows
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    const int r0 = __builtin_amdgcn_readlane(x, 15), r1 = __builtin_amdgcn_readlane(x, 31), r2 = __builtin_amdgcn_readlane(x, 47);
    x += lane < 16 ? 0 : (lane < 32 ? r0 : (lane < 48 ? r0 + r1 : r0 + r1 + r2));
    const int excl = x - nc;
    const int sel = 63 - __builtin_clzll(__ballot(lane < n_seq && excl <= cg));     // the last sequence that starts at or before cg
    ChunkPos p;
    p.tok0 = (long)__builtin_amdgcn_readlane(c0, sel) + 64L * (cg - __builtin_amdgcn_readlane(excl, sel));
    p.clen = min(64, __builtin_amdgcn_readlane(c1, sel) - (int)p.tok0);
    if (out) {
        int rank = 0;
        for (int j = 0; j < n_seq; ++j) {
            const int o = __builtin_amdgcn_readlane(nc, j);
            rank += (o > nc || (o == nc && j < lane)) ? 1 : 0;
        }
        if (lane < n_seq) { out[lane] = excl; out[n_seq + 1 + rank] = lane; }
        if (lane == 63) out[n_seq] = x;
    }
    return p;
}

// Kaczmarz coefficient of eq. (3); a zero denominator (zero key, eps = 0) gives beta = 0
// because the write beta k e^T is then zero for every finite beta.
__device__ __forceinline__ float kaczmarz_beta(float eta, float knorm2, float eps)
{
    const float den = knorm2 + eps;
    return den == 0.0f ? 0.0f : eta / den;
}

// The same with the hardware reciprocal (1 ulp) instead of an IEEE division: for results that are rounded to
// bf16 right afterwards.
__device__ __forceinline__ float kaczmarz_beta_fast(float eta, float knorm2, float eps)
{
    const float den = knorm2 + eps;
    return den == 0.0f ? 0.0f : eta * __builtin_amdgcn_rcpf(den);
}

}  // namespace kla
