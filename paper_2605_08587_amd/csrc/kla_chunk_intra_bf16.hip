// bf16 intra-chunk stage: same objects as kla_chunk_intra.hip (beta of eq. (3), g = log gamma,
// T' = (I + B(A^- o KK^T))^{-1} B of eq. (6), P = A o QK^T of eq. (7), and the decay factors the scan
// stage multiplies with), laid out for gfx950.  One workgroup of four waves per chunk-head.
//
// What bounds it: the latency of one chunk-head (a trip to memory, then the serial 16-row substitutions and the block
// products of the inverse between barriers), so the layout is chosen for the number of chunk-heads a CU holds:
//   * K goes global -> LDS directly (global_load_lds_dwordx4) as token-major rows with the 16-byte columns
//     XOR-swizzled by the row; every MFMA operand slot is then one conflict-free 128-bit LDS read of 8
//     consecutive features.  Wave w forms the Q K^T tiles of row tile w and the K K^T tiles of row tile 3 - w: five
//     tiles each, and it needs the Q rows of one row tile only, which go from memory straight into its registers.
//   * The tiles of P come out of the product in the orientation in which an accumulator tile is the operand quad that
//     the record stores (K Q^T for P, Q K^T for the backward's P^T): P never passes through LDS.
//   * (I+L)^{-1} is built in one fp32 64x64 LDS matrix that overlays the K tile (diagonal 16x16 blocks by forward
//     substitution, by the wave that formed them; off-diagonal blocks by two levels of fp32 MFMA block products, the
//     last of which lands in the unused upper right corner, so that no wave has to wait for its operands' readers).
//   * Rows beyond a short last chunk re-read its last row; beta = 0 there zeroes their rows and columns
//     of T', and their rows of P are masked.
// 18 KB of LDS and at most 80 VGPRs: six workgroups per CU.  Measured, K, Q and P all staged in LDS (50 KB, three
// workgroups per CU) -> this kernel: 7824 chunk-heads of d_k = 128 109 -> 76 us, 4096 with the backward's records 58 -> 43 us;
// with the clocks up 69 and 40 us for 0.39 and 0.23 GB (5.7 TB/s by the counters, part of it out of the memory-side cache).
#include "kla_bf16_ops.hpp"
#include "kla_common.hpp"
#include "kla_kernels.hpp"
#include "kla_mma.hpp"

namespace kla {

namespace {

constexpr int kLd = 68;   // row stride (floats) of the fp32 64x64 matrices in LDS

__device__ __forceinline__ floatx4 ldf4(const float* p) { return *reinterpret_cast<const floatx4*>(p); }
// fp32 MFMA 16x16x16 = four 16x16x4 steps; quads hold contraction indices 4g..4g+3
__device__ __forceinline__ void mma16f(floatx4& acc, floatx4 a, floatx4 b)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], acc, 0, 0, 0);
}
// A-operand quad of a row-major fp32 matrix: columns 4g..4g+3 of row r
__device__ __forceinline__ floatx4 aq(const float* m, int row0, int col0, int r, int g)
{
    return ldf4(m + (row0 + r) * kLd + col0 + 4 * g);
}
// B-operand quad: rows 4g..4g+3 of column r
__device__ __forceinline__ floatx4 bq(const float* m, int row0, int col0, int r, int g)
{
    const float* p = m + (row0 + 4 * g) * kLd + col0 + r;
    floatx4 x; x[0] = p[0]; x[1] = p[kLd]; x[2] = p[2 * kLd]; x[3] = p[3 * kLd]; return x;
}

// The transpose of a lower-triangular fp32 64x64 matrix (row stride kLd; its block [32:64, 0:32] is kept in place of the
// block [0:32, 32:64], the other strictly-upper tiles hold garbage) as
// the 6 upper-triangular tile-pairs of bf16 operand slots: pair ctp = wave (+ 4) is row tile jt, column pair ip with
// (jt, ip) = (0,0) (0,1) (1,0) (1,1) (2,1) (3,1); slot entry (row j, column i) is m[i][j].
__device__ __forceinline__ void write_transposed(char* out, const float* m, int wave, int lane)
{
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int ctp = wave + 4 * it;
        if (ctp < kTriPairs) {
            const int jt = ctp < 4 ? (ctp >> 1) : ctp - 2, ip = ctp < 4 ? (ctp & 1) : 1;
            const float* src = m + (ip == 1 && jt < 2 ? 4 * g * kLd + 32 + 16 * jt : (32 * ip + 4 * g) * kLd + 16 * jt) + r;
            const bool low = ctp == 2 || ctp == 5;        // first block of the pair lies below the diagonal of m^T: zero
            floatx4 x0, x1;
#pragma unroll
            for (int e = 0; e < 4; ++e) { x0[e] = src[e * kLd]; x1[e] = src[(16 + e) * kLd]; }
            const u32x2 q0 = low ? u32x2{0u, 0u} : to_quad(x0);
            const u32x2 q1 = to_quad(x1);
            const u32x4 v = {q0.x, q0.y, q1.x, q1.y};
            st16(out + (size_t)(ctp * 64 + lane) * 16, v);
        }
    }
}

}  // namespace

// BWD = true: the record of the backward pass,
// [T' | M^T | P^T | gamma_i | gamma_C/gamma_i | beta_i | 1/(||k_i||^2+eps) | 1/||q_i||]
// (M = (I + L)^{-1}; the transposes as the 6 upper-triangular tile-pairs, see kla_mma.hpp).  kOptGdnBeta: beta = eta
// and the fourth vector, d beta / d eta, is 1; kOptNormalizeQ: P^T carries 1/||q_i|| and the fifth vector holds it
// (1 otherwise).
// MODE (IntraMode): the forward's record, the backward's, or both but for the forward's copy of T'.  For both, Q K^T is formed twice, in
// the orientation of P and in that of P^T: 48 us for 4096 chunk-heads of d_k = 128 where the two separate launches take 35 + 40.
template <int DK, int MODE>
__global__ __launch_bounds__(256, MODE == kIntraPair ? 5 : 6) void intra_bf16_kernel(IntraArgs<bf16_t> a)
{
    constexpr int RB = DK * 2, PPR = DK / 8, KP = DK / 32;
    constexpr int RPB = 1024 / RB, NKB = 64 / RPB;           // rows per 1 KiB copy block, blocks per tile
    constexpr int TILE = 64 * RB, MB = 64 * kLd * 4;
    constexpr bool FWD = MODE != kIntraBwd, BWD = MODE != kIntraFwd;
    constexpr int REC = BWD ? bwd_record_bytes<bf16_t>() : ws_record_bytes<bf16_t>(), HALF = ws_half_bytes<bf16_t>();
    constexpr int PREC = pair_record_bytes<bf16_t>();

    __shared__ __attribute__((aligned(1024))) char area[TILE > MB ? TILE : MB];   // the K tile, then M
    __shared__ __attribute__((aligned(16))) float beta_s[64];
    __shared__ __attribute__((aligned(16))) float g_s[64];
    __shared__ __attribute__((aligned(16))) float eta_s[64];
    float* M = reinterpret_cast<float*>(area);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const bool norm_q = (a.opts & kOptNormalizeQ) != 0, gdn = (a.opts & kOptGdnBeta) != 0;

    // ---- which chunk of which sequence -------------------------------------------------------
    const int h = blockIdx.x % a.H;
    const int cg = blockIdx.x / a.H;
    const ChunkPos cp = a.pos_out ? chunk_pos_scan(a.cu_seqlens, a.n_seq, cg, lane, tid < 64 && blockIdx.x == 0 ? a.pos_out : nullptr)
                                  : chunk_pos(a.cu_seqlens, a.chunk_off, a.n_seq, a.T, a.NT, cg);
    const long tok0 = cp.tok0;
    const int clen = cp.clen;
    char* rec = reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC;
    // P and the forward's vectors: behind T', or records of their own
    char* recp = MODE == kIntraPair ? reinterpret_cast<char*>(a.wsP) + (size_t)blockIdx.x * PREC : rec + HALF;
    float* vec = reinterpret_cast<float*>(rec + 3 * HALF);   // the backward's five
    float* vecf = reinterpret_cast<float*>(recp + HALF);     // the forward's three

    // ---- everything the workgroup reads, requested at once: K -> LDS by the copy engine, this wave's Q rows -> registers
    //      (lane (r, g): features 32 kp + 8 g .. + 7 of row 16 w + r), the gates (wave 0) ---------------------------
    const size_t kq_row = (size_t)a.H * DK * 2;
    const char* kb = reinterpret_cast<const char*>(a.k) + (size_t)tok0 * kq_row + (size_t)h * DK * 2;
    const char* qb = reinterpret_cast<const char*>(a.q) + (size_t)tok0 * kq_row + (size_t)h * DK * 2;
    {
        const int lrow = lane / PPR, pcol = lane % PPR;
#pragma unroll
        for (int i = 0; i < NKB / 4; ++i) {
            const int b = wave + 4 * i;
            const int row = b * RPB + lrow;
            dma16(kb, min(row, clen - 1) * (int)kq_row + ((pcol ^ swz_piece<DK>(row)) * 16), area + b * 1024);
        }
    }
    float x = 0.f, et = 0.f;
    if (wave == 0 && lane < clen) {
        x = a.log_alpha[(size_t)(tok0 + lane) * a.H + h];
        et = a.eta[(size_t)(tok0 + lane) * a.H + h];
    }
    u32x4 qf[KP];
    {
        const char* q = qb + (size_t)min(16 * wave + r, clen - 1) * kq_row + 16 * g;
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) qf[kp] = ld16(q + 64 * kp);
    }
    if (wave == 0) {
        // inclusive prefix sum: within rows of 16 lanes by DPP shifts, the rows joined through the scalar unit
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf, true));   // row_shr:1
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xf, 0xf, true));   // row_shr:2
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xf, 0xf, true));   // row_shr:4
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xf, 0xf, true));   // row_shr:8
        const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 15));
        const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 31));
        const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 47));
        x += g == 0 ? 0.f : (g == 1 ? r0 : (g == 2 ? r0 + r1 : (r0 + r1) + r2));
        const float x2 = x * 1.44269504088896341f;       // in units of log 2: every decay ratio is one v_exp_f32
        g_s[lane] = x2;
        eta_s[lane] = et;
        if constexpr (!BWD) a.wsG[(size_t)blockIdx.x * 128 + lane] = x;
        const float gl2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x2), 63));
        const float gam = __builtin_amdgcn_exp2f(x2), dec = __builtin_amdgcn_exp2f(gl2 - x2);   // gamma_i, gamma_C / gamma_i
        if constexpr (BWD) { vec[lane] = gam; vec[64 + lane] = dec; }
        if constexpr (FWD) { vecf[lane] = gam; vecf[64 + lane] = dec; }
    }
    wait_vmcnt<0>();
    __syncthreads();

    // ---- 1/||q_i|| of row 16 w + r for the normalised read-out o_t = S_t^T q_t / ||q_t|| (Sec. 3.3); 1 otherwise
    float rq = 1.f;
    if (norm_q) {
        float ss = 0.f;
#pragma unroll
        for (int kp = 0; kp < KP; ++kp)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const float x0 = __uint_as_float(qf[kp][m] << 16), x1 = __uint_as_float(qf[kp][m] & 0xffff0000u);
                ss += x0 * x0; ss += x1 * x1;
            }
        ss += __shfl_xor(ss, 16, kWave);
        ss += __shfl_xor(ss, 32, kWave);
        rq = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
    }
    if (g == 0) {
        if constexpr (BWD) vec[256 + 16 * wave + r] = rq;
        if constexpr (FWD) vecf[128 + 16 * wave + r] = __builtin_amdgcn_exp2f(g_s[16 * wave + r]) * rq;
        if constexpr (!BWD) a.wsG[(size_t)blockIdx.x * 128 + 64 + 16 * wave + r] = rq;
    }

    // ---- Gram tiles, P to the record, L to LDS, the diagonal block of the inverse.  One instance per wave: every tile
    //      index is a constant, and only the diagonal tiles pay for the triangular mask
    auto gram = [&](auto wc) {
        constexpr int W = wc, A = 3 - W, NT = (A > W ? A : W) + 1;
        const int sw = swz_piece<DK>(r);                 // the swizzle has period 8 rows
        const char* rowp = area + r * RB;
        floatx4 kk[A + 1], qk[W + 1];
#pragma unroll
        for (int t = 0; t <= A; ++t) kk[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        u32x4 sl[2][NT];
        auto load = [&](int kp, u32x4 (&dst)[NT]) {
            const int c16 = ((4 * kp + g) ^ sw) * 16;
#pragma unroll
            for (int t = 0; t < NT; ++t) dst[t] = ld16(rowp + t * 16 * RB + c16);
        };
        // KK: the tiles of K K^T too.  TR = false: tiles of P, TR = true: of P^T
        auto products = [&](auto kkc, auto trc) {
            constexpr bool KK = decltype(kkc)::value != 0, TR = decltype(trc)::value != 0;
            constexpr int N = KK ? NT : W + 1;
#pragma unroll
            for (int t = 0; t <= W; ++t) qk[t] = floatx4{0.f, 0.f, 0.f, 0.f};
            load(0, sl[0]);
            static_for<KP>([&](auto kc) {
                constexpr int kp = kc;
                if constexpr (kp + 1 < KP) load(kp + 1, sl[(kp + 1) & 1]);
                static_for<N>([&](auto tc) {
                    constexpr int t = tc;
                    const u32x4 b = sl[kp & 1][t];
                    const u32x2 b0 = {b[0], b[1]}, b1 = {b[2], b[3]};
                    if constexpr (KK && t <= A) mma_bf16(kk[t], sl[kp & 1][A], b0, b1);   // rows: token of tile A, column: token of tile t
                    if constexpr (t <= W) {
                        const u32x2 q0 = {qf[kp][0], qf[kp][1]}, q1 = {qf[kp][2], qf[kp][3]};
                        if constexpr (TR) mma_bf16(qk[t], qf[kp], b0, b1);               // rows: query of tile W, column: key of tile t
                        else              mma_bf16(qk[t], b, q0, q1);                    // rows: key of tile t, column: query of tile W
                    }
                });
            });
        };
        products(IntC<1>(), IntC<FWD ? 0 : 1>());
        // ||k_i||^2 is the diagonal of K K^T (exact bf16 products, fp32 sums): beta of eq. (3) by the lane that holds
        // element (i, i)
        if ((r >> 2) == g) {
            const float ss = (r & 2) ? ((r & 1) ? kk[A][3] : kk[A][2]) : ((r & 1) ? kk[A][1] : kk[A][0]);
            const float eta = eta_s[16 * A + r];
            const float be = gdn ? eta : kaczmarz_beta_fast(eta, ss, a.eps);
            beta_s[16 * A + r] = be;
            if constexpr (BWD) {
                vec[128 + 16 * A + r] = be;
                vec[192 + 16 * A + r] = gdn ? 1.f : kaczmarz_beta_fast(1.f, ss, a.eps);
            }
        }
        // ---- P (or P^T): decay, mask, 1/||q||; straight into the record
        const u32x2 zq = {0u, 0u};
        u32x2 pt[W + 1];
        if constexpr (FWD) {
            static_for<W + 1>([&](auto tc) {             // lane: P[16 W + r][16 t + 4 g + e]
                constexpr int t = tc;
                floatx4 v;
                const float gi = g_s[16 * W + r];
                const floatx4 gj = ldf4(g_s + 16 * t + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float y = __builtin_amdgcn_exp2f(t == W ? fminf(gi - gj[e], 0.f) : gi - gj[e]) * qk[t][e] * rq;
                    if (t == W) y = (4 * g + e <= r) ? y : 0.f;
                    if (clen < 64) y = (16 * W + r < clen) ? y : 0.f;                  // rows beyond a short chunk
                    v[e] = y;
                }
                pt[t] = to_quad(v);
            });
            char* out = recp + lane * 16;
            static_for<W / 2 + 1>([&](auto pc) {
                constexpr int jp = pc;
                const u32x2 q0 = pt[2 * jp], q1 = 2 * jp + 1 <= W ? pt[2 * jp + 1 <= W ? 2 * jp + 1 : 0] : zq;
                const u32x4 v = {q0.x, q0.y, q1.x, q1.y};
                st16(out + tri_pair(W, jp) * 1024, v);
            });
        }
        if constexpr (BWD) {
            if constexpr (FWD) {
                asm volatile("" ::: "memory");           // K is read again: kept from the first time, it would spill
                products(IntC<0>(), IntC<1>());
            }
            static_for<W + 1>([&](auto tc) {             // lane: P[16 W + 4 g + e][16 t + r], the quad of row 16 t + r of P^T
                constexpr int t = tc;
                floatx4 v;
                const float gj = g_s[16 * t + r];
                const floatx4 gi = ldf4(g_s + 16 * W + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float y = __builtin_amdgcn_exp2f(t == W ? fminf(gi[e] - gj, 0.f) : gi[e] - gj) * qk[t][e];
                    if (norm_q) y *= __shfl(rq, 4 * g + e, kWave);
                    if (t == W) y = (r <= 4 * g + e) ? y : 0.f;
                    if (clen < 64) y = (16 * W + 4 * g + e < clen) ? y : 0.f;
                    v[e] = y;
                }
                pt[t] = to_quad(v);
            });
            // pair (t, W / 2) of P^T holds the quads of waves W & ~1 and W | 1 side by side; below the diagonal it is zero
            char* out = rec + 2 * HALF + lane * 16;
            static_for<W + 1>([&](auto tc) {
                constexpr int t = tc;
                char* p = out + triu_pair(t, W >> 1) * 1024;
                if constexpr (t == W && (W & 1)) { const u32x4 v = {0u, 0u, pt[t].x, pt[t].y}; st16(p, v); }
                else *reinterpret_cast<u32x2*>(p + 8 * (W & 1)) = pt[t];
            });
        }
        __syncthreads();                                 // the K tile is dead from here on: M overlays it
        // ---- L: decay, mask, beta.  The six strictly-upper tiles are never written: every reader knows they are zero
        const floatx4 bi = ldf4(beta_s + 16 * A + 4 * g);
        const floatx4 gi = ldf4(g_s + 16 * A + 4 * g);
        static_for<A + 1>([&](auto tc) {
            constexpr int t = A - tc;                    // the diagonal tile first: it is what this wave goes on with
            const float gj = g_s[16 * t + r];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float y = bi[e] * __builtin_amdgcn_exp2f(t == A ? fminf(gi[e] - gj, 0.f) : gi[e] - gj) * kk[t][e];
                if (t == A) y = (r < 4 * g + e) ? y : 0.f;                             // strictly lower
                M[(16 * A + 4 * g + e) * kLd + 16 * t + r] = y;
            }
        });
    };
    if (wave == 0) gram(IntC<0>()); else if (wave == 1) gram(IntC<1>()); else if (wave == 2) gram(IntC<2>()); else gram(IntC<3>());

    // ---- diagonal 16x16 block D = (I + L_bb)^{-1} by forward substitution, in place, by the wave that wrote L_bb (lane
    //      column r, the four 16-lane groups redundantly), rows read ahead
    {
        constexpr int AHEAD = 2;
        const int blk = 3 - wave;
        const float* Lb = M + (16 * blk) * kLd + 16 * blk;
        float xs[16];
        floatx4 rows[AHEAD + 1][4];
        auto read_row = [&](auto ic) {
            constexpr int i = ic;
            if constexpr (i < 16) {
#pragma unroll
                for (int c4 = 0; c4 < (i + 3) / 4; ++c4) rows[i % (AHEAD + 1)][c4] = ldf4(Lb + i * kLd + 4 * c4);
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
        // only this wave touches block (blk, blk), and its reads above precede these writes in program order
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((i >> 2) == g) M[(16 * blk + i) * kLd + 16 * blk + r] = xs[i];
    }
    __syncthreads();

    // ---- 32x32 level, in place.  Waves 0,1: block pair (a, b) = (2m, 2m+1): T_ba = -D_b (L_ba D_a)
    if (wave < 2) {
        const int ra = 32 * wave, rb = ra + 16;
        floatx4 y = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
        mma16f(y, aq(M, rb, ra, r, g), bq(M, ra, ra, r, g));
        mma16f(z, aq(M, rb, rb, r, g), y);           // an accumulator tile is the next product's B quad
#pragma unroll
        for (int e = 0; e < 4; ++e) M[(rb + 4 * g + e) * kLd + ra + r] = -z[e];    // only this wave read L_ba
    }
    __syncthreads();

    // ---- 64x64 level.  T[32:64, 0:32] = -T22 (L21 T11); wave = (row tile ti, col tile tj); kept at [0:32, 32:64], where
    //      nobody reads in this phase
    {
        const int ti = wave >> 1, tj = wave & 1;
        floatx4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            if (tm == 0 && tj == 1) continue;        // T11 tile (0, 1) is zero
            const floatx4 b = bq(M, 16 * tm, 16 * tj, r, g);
            mma16f(y0, aq(M, 32, 16 * tm, r, g), b);
            if (ti == 1) mma16f(y1, aq(M, 48, 16 * tm, r, g), b);
        }
        mma16f(z, aq(M, 32 + 16 * ti, 32, r, g), y0);
        if (ti == 1) mma16f(z, aq(M, 32 + 16 * ti, 48, r, g), y1);   // T22 tile (0, 1) is zero
#pragma unroll
        for (int e = 0; e < 4; ++e) M[(16 * ti + 4 * g + e) * kLd + 32 + 16 * tj + r] = -z[e];
    }
    __syncthreads();

    // ---- T' = T diag(beta) -> workspace in operand order (stored tile-pair ctp = wave (+ 4): wave-uniform, so its tile
    //      coordinates are scalars; slot = ctp * 64 + lane) ------------------------------
    {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int ctp = wave + 4 * it;
            if (ctp < kTriPairs) {
                const int ti = ctp < 2 ? ctp : 2 + ((ctp - 2) >> 1), jp = ctp < 2 ? 0 : ((ctp - 2) & 1);
                const int cl = 32 * jp + 4 * g;
                const float* src = M + (ti >= 2 && jp == 0 ? (16 * (ti - 2) + r) * kLd + 32 : (16 * ti + r) * kLd) + cl;
                const bool up = ctp == 0 || ctp == 3;         // second block of the pair is an upper tile: zero
                const u32x2 q0 = to_quad(ldf4(src) * ldf4(beta_s + cl));
                const u32x2 q1 = up ? u32x2{0u, 0u} : to_quad(ldf4(src + 16) * ldf4(beta_s + cl + 16));
                const u32x4 v = {q0.x, q0.y, q1.x, q1.y};
                st16(rec + (size_t)(ctp * 64 + lane) * 16, v);
            }
        }
        if constexpr (BWD) write_transposed(rec + HALF, M, wave, lane);      // M^T
    }
}

template <int DK>
static hipError_t launch_dk(const IntraArgs<bf16_t>& a, IntraMode mode, int n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const dim3 grid((unsigned)n_chunks * a.H), block(256);
    if (mode == kIntraFwd)      hipLaunchKernelGGL((intra_bf16_kernel<DK, kIntraFwd>), grid, block, 0, st, a);
    else if (mode == kIntraBwd) hipLaunchKernelGGL((intra_bf16_kernel<DK, kIntraBwd>), grid, block, 0, st, a);
    else                        hipLaunchKernelGGL((intra_bf16_kernel<DK, kIntraPair>), grid, block, 0, st, a);
    return hipGetLastError();
}
hipError_t launch_intra_bf16(const IntraArgs<bf16_t>& a, int dk, IntraMode mode, int n_chunks, hipStream_t st)
{
    return dk == 64 ? launch_dk<64>(a, mode, n_chunks, st) : launch_dk<128>(a, mode, n_chunks, st);
}

}  // namespace kla
