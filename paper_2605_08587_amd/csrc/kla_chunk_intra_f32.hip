// Intra-chunk stage for single-precision inputs (eqs. (3), (6), (7) per chunk and head; the algebra and the record are
// those of kla_chunk_intra.hip), all products on v_mfma_f32_16x16x4_f32, one workgroup of four waves per chunk-head.
//
// What bounds it: latency.  A chunk-head is 20 Gram tiles - 2.1 us of one CU's matrix cores at d_k = 128 - behind a trip to
// memory and in front of the serial 16-row substitutions and block products of (I + L)^{-1}, so the only way to a busy
// chip is several chunk-heads per CU.  The footprint is therefore one K tile (32 KB at d_k = 128; the matrices of the
// inverse overlay it): four workgroups per CU.
//   * Wave w forms the Q K^T tiles of row tile w and the K K^T tiles of row tile 3 - w: five tiles for every wave, and a
//     wave needs the Q rows of one row tile only, which go from memory straight into its registers.
//   * The Gram tiles of P come out of the product in the orientation in which an accumulator tile is the operand quad
//     that the record stores (K Q^T for P, Q K^T for the backward's P^T), so P never passes through LDS.
//   * ||k_i||^2 and ||q_i||^2 are sums over the operand registers of the lanes that hold row i, as a tree (the diagonal of
//     K K^T is the same sum, but one chain of d_k roundings: beta 1.7e-7 off instead of 0.5e-7, d_k = 128).
// Measured, K and Q staged as operand slots (101 KB, one workgroup per CU) -> this kernel: 1024 chunk-heads of d_k = 128
// 79 -> 34 us, 64 chunk-heads of d_k = 64 13.3 -> 9.7 us; with the rows of the substitutions read two ahead instead of all
// at once (no spilled register) 31.9 -> 29.4 us.
#include "kla_common.hpp"
#include "kla_kernels.hpp"
#include "kla_f32_ops.hpp"

namespace kla {

namespace {

constexpr int kLdm = 68;   // row stride (floats) of the fp32 64x64 matrices in LDS: 16-byte aligned rows

__device__ __forceinline__ float4 bquad(const float* m, int row0, int col0, int r, int g)   // rows 4g..4g+3 of column r
{
    const float* p = m + (row0 + 4 * g) * kLdm + col0 + r;
    return make_float4(p[0], p[kLdm], p[2 * kLdm], p[3 * kLdm]);
}
__device__ __forceinline__ float4 aquad(const float* m, int row0, int col0, int r, int g)   // columns 4g..4g+3 of row r
{
    return ldf4(m + (row0 + r) * kLdm + col0 + 4 * g);
}
// the squares of a row's values, summed as a tree over its quads (N: a power of two)
__device__ __forceinline__ float sum_squares(float4 v) { return v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w; }
template <int N> __device__ __forceinline__ float tree_sum(float (&x)[N])
{
#pragma unroll
    for (int w = N / 2; w > 0; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) x[i] += x[i + w];
    return x[0];
}

}  // namespace

// MODE (IntraMode): the forward's records [T' | P | three vectors], those of the backward pass, [T' | M^T | P^T | five vectors]
// (see bwd_record_bytes in kla_mma.hpp), or the backward's and [P | three vectors].
template <int DK, int MODE>
__global__ __launch_bounds__(256, 4) void intra_f32_kernel(IntraArgs<float> a)
{
    typedef F32<DK> C;
    constexpr bool FWD = MODE != kIntraBwd, BWD = MODE != kIntraFwd;
    constexpr int KB = C::KB, REC = BWD ? bwd_record_bytes<float>() : ws_record_bytes<float>(), HALF = ws_half_bytes<float>();
    constexpr int MB = 64 * kLdm * 4;
    __shared__ __attribute__((aligned(1024))) char area[C::TILE > 2 * MB ? C::TILE : 2 * MB];
    __shared__ __attribute__((aligned(16))) float g_s[4][64];        // running sums of log alpha, one copy per wave
    __shared__ __attribute__((aligned(16))) float beta_s[64];
    float* Lm = reinterpret_cast<float*>(area);                      // these two overlay the K tile once the Gram products are done
    float* Tm = reinterpret_cast<float*>(area + MB);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int h = blockIdx.x % a.H;
    const ChunkPos cp = a.pos_out ? chunk_pos_scan(a.cu_seqlens, a.n_seq, blockIdx.x / a.H, lane, tid < 64 && blockIdx.x == 0 ? a.pos_out : nullptr)
                                  : chunk_pos(a.cu_seqlens, a.chunk_off, a.n_seq, a.T, a.NT, blockIdx.x / a.H);
    const int clen = cp.clen;
    const size_t ks = (size_t)a.H * DK;
    char* rec = reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC;
    char* recp = MODE == kIntraPair ? reinterpret_cast<char*>(a.wsP) + (size_t)blockIdx.x * pair_record_bytes<float>() : rec + HALF;
    float* vec = reinterpret_cast<float*>(rec + 3 * HALF);   // the backward's five vectors
    float* vecf = reinterpret_cast<float*>(recp + HALF);     // the forward's three
    const bool gdn = (a.opts & kOptGdnBeta) != 0;

    // ---- everything the workgroup reads, requested at once (rows beyond a short chunk: its last row, zeroed below)
    TileRegs<DK> kr;
    kr.load(a.k + (size_t)cp.tok0 * ks + (size_t)h * DK, ks, clen, tid);
    float4 qf[KB];
    {
        const float* q = a.q + (size_t)(cp.tok0 + min(16 * wave + r, clen - 1)) * ks + (size_t)h * DK + 4 * g;
#pragma unroll
        for (int b = 0; b < KB; ++b) qf[b] = ldf4(q + 16 * b);
    }
    const size_t gate = (size_t)(cp.tok0 + min(lane, clen - 1)) * a.H + h;
    float x = a.log_alpha[gate];
    float et = a.eta[gate];
    x = lane < clen ? x : 0.f;
    et = lane < clen ? et : 0.f;

    // ---- g_i = log gamma_i; the decay vectors of the record
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { const float y = __shfl_up(x, off, kWave); if (lane >= off) x += y; }
    g_s[wave][lane] = x;
    if (wave == 0) {
        const float gam = expf(x), dec = expf(__shfl(x, 63, kWave) - x);
        if constexpr (BWD) { vec[lane] = gam; vec[64 + lane] = dec; }
        if constexpr (FWD) { vecf[lane] = gam; vecf[64 + lane] = dec; }
        if constexpr (!BWD) a.wsG[(size_t)blockIdx.x * 128 + lane] = x;
    }
    kr.template stash<true>(area, tid, clen);
    // ---- 1/||q_i|| of row 16 w + r (1 when the read-out is not normalised; 0 for a zero query)
    float rq = 1.f;
    {
        const bool live = 16 * wave + r < clen;
        float sq[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            if (!live) qf[b] = make_float4(0.f, 0.f, 0.f, 0.f);
            sq[b] = sum_squares(qf[b]);
        }
        float ss = tree_sum(sq);
        ss += __shfl_xor(ss, 16, kWave);
        ss += __shfl_xor(ss, 32, kWave);
        if (a.opts & kOptNormalizeQ) rq = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
        if (g == 0) {
            if constexpr (BWD) vec[256 + 16 * wave + r] = rq;
            if constexpr (FWD) vecf[128 + 16 * wave + r] = expf(g_s[wave][16 * wave + r]) * rq;
            if constexpr (!BWD) a.wsG[(size_t)blockIdx.x * 128 + 64 + 16 * wave + r] = rq;
        }
    }
    __syncthreads();

    // ---- Gram tiles, P to the record, L and beta to LDS.  One instance per wave: every tile index is a constant.
    auto gram = [&](auto wc) {
        constexpr int W = wc, A = 3 - W, NT = (A > W ? A : W) + 1;
        TileOps<DK> ops;
        ops.init(A, r, g);
        int boff[4];                                     // row operand of any tile: that of tile 0 + 16 rows per tile
#pragma unroll
        for (int y = 0; y < 4; ++y) boff[y] = ops.row_off[y] - 16 * A * C::RB;
        floatx4 kk[A + 1], qk[W + 1];
#pragma unroll
        for (int t = 0; t <= A; ++t) kk[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        float sq[KB];
        // KK: the tiles of K K^T and the key norms too.  TR = false: tiles of P, TR = true: of P^T
        auto products = [&](auto kkc, auto trc) {
            constexpr bool KK = decltype(kkc)::value != 0, TR = decltype(trc)::value != 0;
            constexpr int N = KK ? NT : W + 1;
#pragma unroll
            for (int t = 0; t <= W; ++t) qk[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                float4 ka;
                if constexpr (KK) { ka = ops.row_quad(area, b); sq[b] = sum_squares(ka); }
                static_for<N>([&](auto tc) {
                    constexpr int t = tc;
                    const float4 kb = KK && t == A ? ka : ldf4(area + boff[b & 3] + 16 * t * C::RB + 256 * (b >> 2));
                    if constexpr (KK && t <= A) mma16(kk[t], ka, kb);        // rows: token of tile A, column: token of tile t
                    if constexpr (t <= W) {
                        if constexpr (TR) mma16(qk[t], qf[b], kb);           // rows: query of tile W, column: key of tile t
                        else              mma16(qk[t], kb, qf[b]);           // rows: key of tile t, column: query of tile W
                    }
                });
            }
        };
        products(IntC<1>(), IntC<FWD ? 0 : 1>());
        const float* gw = g_s[W];
        // ---- P (or P^T): decay, mask, 1/||q||; straight into the record
        const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
        auto put = [&](char* half, int pair, int blk, floatx4 v) {
            *reinterpret_cast<float4*>(half + ((size_t)pair * 64 + lane) * 32 + 16 * blk) = quad(v);
        };
        // (and, zero, the tile of a stored pair that lies on the other side of the diagonal)
        if constexpr (FWD) {
            static_for<W + 1>([&](auto tc) {             // lane: P[16 W + r][16 t + 4 g + e]
                constexpr int t = tc;
                floatx4 v;
                const float gi = gw[16 * W + r];
                const floatx4 gj = lda4(gw + 16 * t + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (t < W || 4 * g + e <= r) ? expf(gi - gj[e]) * qk[t][e] * rq : 0.f;
                put(recp, tri_pair(W, t >> 1), t & 1, v);
            });
            if constexpr ((W & 1) == 0) put(recp, tri_pair(W, W >> 1), 1, z4);
        }
        if constexpr (BWD) {
            if constexpr (FWD) {
                asm volatile("" ::: "memory");           // K is read again: kept from the first time, it would spill
                products(IntC<0>(), IntC<1>());
            }
            static_for<W + 1>([&](auto tc) {             // lane: P[16 W + 4 g + e][16 t + r], the quad of row 16 t + r of P^T
                constexpr int t = tc;
                floatx4 v;
                const float gj = gw[16 * t + r];
                const floatx4 gi = lda4(gw + 16 * W + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float rqi = __shfl(rq, 4 * g + e, kWave);
                    v[e] = (t < W || r <= 4 * g + e) ? expf(gi[e] - gj) * qk[t][e] * rqi : 0.f;
                }
                put(rec + 2 * HALF, triu_pair(t, W >> 1), W & 1, v);
            });
            if constexpr ((W & 1) == 1) put(rec + 2 * HALF, triu_pair(W, W >> 1), 0, z4);
        }
        // ---- beta of the rows of tile A (||k_i||^2 of row 16 A + r in the lanes of r)
        float kn = tree_sum(sq);
        kn += __shfl_xor(kn, 16, kWave);
        kn += __shfl_xor(kn, 32, kWave);
        floatx4 be;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ss = __shfl(kn, 4 * g + e, kWave), eta = __shfl(et, 16 * A + 4 * g + e, kWave);
            be[e] = gdn ? eta : kaczmarz_beta(eta, ss, a.eps);
            if (r == 4 * g + e) {
                beta_s[16 * A + r] = be[e];
                if constexpr (BWD) {
                    vec[128 + 16 * A + r] = be[e];
                    vec[192 + 16 * A + r] = gdn ? 1.f : ((ss + a.eps == 0.f) ? 0.f : 1.0f / (ss + a.eps));
                }
            }
        }
        __syncthreads();                                 // the K tile is dead from here on
        static_for<A + 1>([&](auto tc) {
            constexpr int t = tc;
            const float gj = gw[16 * t + r];
            const floatx4 gi = lda4(gw + 16 * A + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                Lm[(16 * A + 4 * g + e) * kLdm + 16 * t + r] = (t < A || r < 4 * g + e) ? be[e] * expf(gi[e] - gj) * kk[t][e] : 0.f;
        });
        if constexpr ((W & 1) == 0) {                    // tiles (0, 1) and (2, 3) of (I + L)^{-1}: stored, and zero
#pragma unroll
            for (int e = 0; e < 4; ++e) Tm[(16 * W + 4 * g + e) * kLdm + 16 * (W + 1) + r] = 0.f;
        }
    };
    if (wave == 0) gram(IntC<0>()); else if (wave == 1) gram(IntC<1>()); else if (wave == 2) gram(IntC<2>()); else gram(IntC<3>());
    __syncthreads();

    // ---- (I + L)^{-1}: the diagonal 16x16 blocks by forward substitution (wave w: block w, lane r: column r; the rows
    //      of L are read ahead, they do not depend on the result)
    {
        constexpr int AHEAD = 2;
        const float* Lb = Lm + 16 * wave * kLdm + 16 * wave;
        float xs[16];
        floatx4 rows[AHEAD + 1][4];
        auto read_row = [&](auto ic) {
            constexpr int i = ic;
            if constexpr (i < 16) {
#pragma unroll
                for (int c4 = 0; c4 < (i + 3) / 4; ++c4) rows[i % (AHEAD + 1)][c4] = lda4(Lb + i * kLdm + 4 * c4);
            }
        };
        static_for<AHEAD>([&](auto ic) { read_row(IntC<ic + 1>()); });
        xs[0] = (r == 0) ? 1.f : 0.f;
        static_for<15>([&](auto ic) {
            constexpr int i = ic + 1;
            read_row(IntC<i + AHEAD>());
            float s0 = (i == r) ? 1.f : 0.f, s1 = 0.f;
            static_for<i>([&](auto rc) {
                constexpr int rr = rc;
                if constexpr (rr & 1) s1 -= rows[i % (AHEAD + 1)][rr >> 2][rr & 3] * xs[rr];
                else                  s0 -= rows[i % (AHEAD + 1)][rr >> 2][rr & 3] * xs[rr];
            });
            xs[i] = s0 + s1;
            asm volatile("" : "+v"(xs[i]) : : "memory");     // no row is read earlier than said: 15 rows at once spill
        });
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((i >> 2) == g) Tm[(16 * wave + i) * kLdm + 16 * wave + r] = xs[i];
    }
    __syncthreads();
    // ---- 32x32 level, waves 0 and 1: T_ba = -D_b (L_ba D_a)
    if (wave < 2) {
        const int ra = 32 * wave, rb = ra + 16;
        floatx4 y = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
        mma16(y, aquad(Lm, rb, ra, r, g), bquad(Tm, ra, ra, r, g));
        mma16(z, aquad(Tm, rb, rb, r, g), quad(y));
#pragma unroll
        for (int e = 0; e < 4; ++e) Tm[(rb + 4 * g + e) * kLdm + ra + r] = -z[e];
    }
    __syncthreads();
    // ---- 64x64 level: T[32:64, 0:32] = -T22 (L21 T11); wave = (row tile ti, column tile tj)
    {
        const int ti = wave >> 1, tj = wave & 1;
        floatx4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const float4 b = bquad(Tm, 16 * tm, 16 * tj, r, g);
            mma16(y0, aquad(Lm, 32, 16 * tm, r, g), b);
            mma16(y1, aquad(Lm, 48, 16 * tm, r, g), b);
        }
        mma16(z, aquad(Tm, 32 + 16 * ti, 32, r, g), quad(y0));
        mma16(z, aquad(Tm, 32 + 16 * ti, 48, r, g), quad(y1));
        // the block written below is read by no wave in this phase, so no barrier is needed here
#pragma unroll
        for (int e = 0; e < 4; ++e) Tm[(32 + 16 * ti + 4 * g + e) * kLdm + 16 * tj + r] = -z[e];
    }
    __syncthreads();
    // ---- T' = (I + L)^{-1} diag(beta) (and, for the backward, M^T) -> record, in operand order
    write_tri_f32<false, true>(rec, Tm, beta_s, tid);
    if constexpr (BWD) write_tri_f32<true, false>(rec + HALF, Tm, nullptr, tid);
}

template <int DK>
static hipError_t launch_dk(const IntraArgs<float>& a, IntraMode mode, int n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const dim3 grid((unsigned)n_chunks * a.H), block(256);
    if (mode == kIntraFwd)      hipLaunchKernelGGL((intra_f32_kernel<DK, kIntraFwd>), grid, block, 0, st, a);
    else if (mode == kIntraBwd) hipLaunchKernelGGL((intra_f32_kernel<DK, kIntraBwd>), grid, block, 0, st, a);
    else                        hipLaunchKernelGGL((intra_f32_kernel<DK, kIntraPair>), grid, block, 0, st, a);
    return hipGetLastError();
}
hipError_t launch_intra_f32(const IntraArgs<float>& a, int dk, IntraMode mode, int n_chunks, hipStream_t st)
{
    return dk == 64 ? launch_dk<64>(a, mode, n_chunks, st) : launch_dk<128>(a, mode, n_chunks, st);
}

}  // namespace kla
