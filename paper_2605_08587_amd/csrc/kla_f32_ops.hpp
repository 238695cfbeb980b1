// Device helpers shared by the fp32 chunk kernels: a [64, d_k] tile in LDS that is read row- and column-wise without bank
// conflicts, its way there from global memory, and the record's operand order.
#pragma once
#include "kla_common.hpp"
#include "kla_mma.hpp"

namespace kla {

__device__ __forceinline__ float4 ldf4(const void* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ floatx4 lda4(const void* p) { return *reinterpret_cast<const floatx4*>(p); }
__device__ __forceinline__ float4 quad(floatx4 x) { return make_float4(x[0], x[1], x[2], x[3]); }

template <int DK> struct F32 {
    static constexpr int KB = DK / 16;               // feature tiles
    static constexpr int TS = KB / 4;                // of them per wave
    static constexpr int RB = DK * 4, PPR = DK / 4;  // bytes and 16-byte pieces of a row
    static constexpr int NLD = 64 * PPR / 256;       // pieces of a [64, d_k] tile per thread
    static constexpr int TILE = 64 * RB;
    static constexpr int SXB = KB * 1024, RXB = 4 * 1024;   // exchanged state / token-shaped result of one column tile
};

// A [64, d_k] tile on its way from global memory to LDS.
template <int DK> struct TileRegs {
    typedef F32<DK> C;
    float4 d[C::NLD];
    __device__ __forceinline__ void load(const float* base, size_t stride, int clen, int tid)
    {
#pragma unroll
        for (int i = 0; i < C::NLD; ++i) {
            const int idx = tid + 256 * i, row = idx / C::PPR, p = idx % C::PPR;
            d[i] = ldf4(base + (size_t)min(row, clen - 1) * stride + 4 * p);
        }
    }
    // ZERO: rows beyond clen are stored as zeros (else as the copies of the last row that load() brought)
    template <bool ZERO = false> __device__ __forceinline__ void stash(char* tile, int tid, int clen = 64) const
    {
#pragma unroll
        for (int i = 0; i < C::NLD; ++i) {
            const int idx = tid + 256 * i, row = idx / C::PPR, p = idx % C::PPR;
            *reinterpret_cast<float4*>(tile + row * C::RB + ((p ^ (row & 15)) * 16)) =
                (!ZERO || row < clen) ? d[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
};

// Lane offsets into such a tile.  Row operand (contraction along the row): row 16 w + r, piece 4 kb + g.  Column operand
// (contraction over the tokens, tile kt = w TS + t of the features): rows 16 jb + 4 g + e, feature 16 kt + r, i.e.
// piece 4 kt + r / 4, whose position is its XOR with 4 g + e.
template <int DK> struct TileOps {
    typedef F32<DK> C;
    int row_off[4], col_off[4], t_off[C::TS];
    __device__ __forceinline__ void init(int wave, int r, int g)
    {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            row_off[x] = (16 * wave + r) * C::RB + 16 * ((g ^ r) & 3) + 64 * (x ^ (r >> 2));
            col_off[x] = (4 * g + x) * C::RB + 16 * ((r >> 2) ^ x) + 4 * (r & 3);
        }
#pragma unroll
        for (int t = 0; t < C::TS; ++t) {
            const int kt = wave * C::TS + t;
            t_off[t] = 64 * ((kt & 3) ^ g) + 256 * (kt >> 2);
        }
    }
    __device__ __forceinline__ float4 row_quad(const char* tile, int kb) const { return ldf4(tile + row_off[kb & 3] + 256 * (kb >> 2)); }
    __device__ __forceinline__ float4 col_quad(const char* tile, int t, int jb) const
    {
        const char* p = tile + t_off[t] + 16 * jb * C::RB;
        return make_float4(*reinterpret_cast<const float*>(p + col_off[0]), *reinterpret_cast<const float*>(p + col_off[1]),
                           *reinterpret_cast<const float*>(p + col_off[2]), *reinterpret_cast<const float*>(p + col_off[3]));
    }
};

// A triangular 64x64 fp32 matrix m (row stride 68) -> 6 stored tile-pairs of operand slots at `out` (see write_tri in
// kla_chunk_intra.hip): the matrix itself, column j scaled by colscale[j] if SCALE, or its transpose.  All 256 threads.
template <bool TRANSPOSE, bool SCALE>
__device__ __forceinline__ void write_tri_f32(char* out, const float* m, const float* colscale, int tid)
{
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int sl = tid + 256 * it;
        if (sl >= kTriPairs * 64) break;
        const int ctp = sl >> 6, ln = sl & 63;
        int ti, jp;
        if constexpr (TRANSPOSE) { ti = ctp < 4 ? (ctp >> 1) : ctp - 2; jp = ctp < 4 ? (ctp & 1) : 1; }
        else                     { ti = ctp < 2 ? ctp : 2 + ((ctp - 2) >> 1); jp = ctp < 2 ? 0 : ((ctp - 2) & 1); }
        const int row = 16 * ti + (ln & 15), col = 32 * jp + 4 * (ln >> 4);
        floatx4 v0, v1;
        if constexpr (TRANSPOSE) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { v0[e] = m[(col + e) * 68 + row]; v1[e] = m[(col + 16 + e) * 68 + row]; }
        } else {
            v0 = lda4(m + row * 68 + col); v1 = lda4(m + row * 68 + col + 16);
            if constexpr (SCALE) { v0 = v0 * lda4(colscale + col); v1 = v1 * lda4(colscale + col + 16); }
        }
        *reinterpret_cast<float4*>(out + (size_t)sl * 32) = quad(v0);
        *reinterpret_cast<float4*>(out + (size_t)sl * 32 + 16) = quad(v1);
    }
}

}  // namespace kla
