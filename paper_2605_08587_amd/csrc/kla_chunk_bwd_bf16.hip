// bf16 state sweeps of the backward pass (see kla_chunk_bwd.hip for the algebra and for what each sweep leaves
// behind), built like the forward's bf16 scan kernel (kla_chunk_scan_bf16.hip): operands travel global -> LDS
// directly through a ring of stages filled by a copy wave, K and Q sit as swizzled token-major rows, the
// contraction-along-a-column operands (K^T, Q^T, the V / dO tile) come from the transposing LDS read, and the
// fp32 state (or state gradient) of 16 columns per wave stays in MFMA accumulators with the permuted feature
// index of that kernel: element e of lane (r, g) of tile kt = 2 kp + b is feature 32 kp + 8 g + 4 b + e.
//
//   REV = false   forward sweep:  X = V - D_gamma K S,  U = T' X,  S <- gamma_C S + K^T diag(gamma_C/gamma_i) U;
//                 leaves S_c (before the chunk) and X.
//   REV = true    backward sweep: dU = P^T dO + diag(gamma_C/gamma_i) K dS',  Y = M^T dU,  dV = B Y,
//                 dS <- gamma_C dS' + Q^T D_gamma dO - K^T D_gamma dV;  leaves dS'_c, Y, dV and finally dh0.
//
// X, Y and the checkpoints go to memory as the registers hold them (put_rows, put_checkpoint in kla_bf16_ops.hpp).
//
// A short last chunk re-reads its last valid row for the rows beyond it (as in the forward).  Those rows have
// beta = 0, zero rows and columns in T' and P^T and unit rows in M, so they reach neither U, Y (valid rows), dV nor
// the state; the one place where they would, Q^T D_gamma dO, has their gamma masked to zero.
#include "kla_bf16_ops.hpp"
#include "kla_common.hpp"
#include "kla_kernels.hpp"
#include "kla_mma.hpp"

namespace kla {

namespace {

template <int DK, int NW, bool REV>
struct SweepCfg16 {
    static constexpr int NTH = 64 * NW;                  // compute threads (the workgroup has one more wave)
    static constexpr int KB = DK / 16, KP = DK / 32;
    static constexpr int SLW = 16 * NW;                  // state columns per workgroup
    static constexpr int RB = DK * 2;                    // bytes per K/Q row
    static constexpr int PPR = DK / 8;                   // 16-byte pieces per K/Q row
    static constexpr int RPB = 1024 / RB;                // K/Q rows per 1 KiB copy block
    static constexpr int NKB = 64 / RPB;                 // copy blocks of a K (or Q) tile
    static constexpr int VRW = SLW * 2;                  // bytes per row of the V / dO slice
    static constexpr int VPP = VRW / 16;
    static constexpr int RPV = 64 / VPP;
    static constexpr int NVB = 64 / RPV;
    static constexpr int TPB = kTriPairs * 64 * 16;      // bytes of one triangular operand area
    static constexpr int NTB = (REV ? 2 : 1) * TPB / 1024;   // forward: T'; backward: M^T | P^T
    // TWO (reverse, four compute waves at d_k = 128): two rings, as in the forward kernel (both sweeps of 8 x 4096 tokens, 8 heads,
    // d_v = 256, and the assembly: 632 -> 594 us).  Q and P^T have one of two stages, from which OFF_Q and OFF_P count.
    static constexpr bool TWO = REV && NW == 4 && DK == 128;
    // stage: K rows | (Q rows) | T'  or  M^T | P^T | V or dO slice | gamma_i | gamma_C/gamma_i | beta_i | (1/||q_i||)
    static constexpr int OFF_Q = TWO ? 0 : 64 * RB;
    static constexpr int OFF_T = (REV && !TWO ? 2 : 1) * 64 * RB, OFF_P = TWO ? 64 * RB : OFF_T + TPB, OFF_V = OFF_T + (REV && !TWO ? 2 : 1) * TPB,
                         OFF_EG = OFF_V + 64 * VRW, STAGE = OFF_EG + (REV ? 1024 : 768);
    static constexpr int ORB = NW <= 2 ? 96 : 160;       // row stride of a staging tile (see the forward kernel)
    static constexpr int OSB = 64 * ORB;
    // Reverse sweep: the rows of dV are staged, in two parities, for the store wave.
    static constexpr int QST = TWO ? 64 * RB + TPB : 0;  // a stage of the second ring
    static constexpr int NST = (3 * STAGE + 2 * QST + (REV ? 2 * OSB : 0) <= 160 * 1024) ? 3 : 2;   // LDS ring depth
    static constexpr int OFF_OST = NST * STAGE + 2 * QST;
    static constexpr int N_FIRST = NKB + TPB / 1024 + NVB + 1;   // TWO: copies of the first part
    static_assert(!TWO || (NST == 3 && N_FIRST < 64), "two rings; 6-bit vmcnt");
    // swizzle of the V / dO slice, as in the forward kernel (period 8 rows: the same for every copy block)
    __host__ __device__ static constexpr int vswz(int row) { return NW == 4 ? 2 * ((row >> 1) & 3) : 0; }
    static constexpr int LDS = OFF_OST + (REV ? 2 * OSB : 0);
    static constexpr int NDMA = (REV ? 2 : 1) * NKB + NTB + NVB + 1;
    static_assert(LDS <= 160 * 1024 && NDMA < 64, "LDS budget of a gfx950 CU; 6-bit vmcnt");
};

}  // namespace

template <int DK, int NW, bool REV>
__global__ __launch_bounds__(64 * NW + (REV ? 128 : 64)) void bwd_sweep_bf16_kernel(BwdArgs<bf16_t> a)
{
    typedef SweepCfg16<DK, NW, REV> C;
    constexpr int NTH = C::NTH, KB = C::KB, KP = C::KP, SLW = C::SLW, RB = C::RB, PPR = C::PPR, RPB = C::RPB,
                  VRW = C::VRW, VPP = C::VPP, RPV = C::RPV, ORB = C::ORB, NST = C::NST;

    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    const int nsl = a.dv_dim / SLW;
    const int n_states = a.n_seq > 0 ? a.n_seq : (a.seg_G > 0 ? a.N * a.seg_G : a.N);
    const int xcd = blockIdx.x & 7, pidx = blockIdx.x >> 3;
    const int rank = (pidx / nsl) * 8 + xcd, slice = pidx % nsl;
    if (rank >= n_states * a.H) return;
    const int h = rank % a.H;
    const int s = a.seq_order ? a.seq_order[rank / a.H] : rank / a.H;
    const int chain = s * a.H + h;
    long t0; int len, ch0;
    if (a.cu_seqlens) { t0 = a.cu_seqlens[s]; len = a.cu_seqlens[s + 1] - (int)t0; ch0 = a.chunk_off[s]; }
    else if (a.seg_G > 0) {                              // segment sg of sequence n: chunks [sg Lc, (sg + 1) Lc)
        const int n = s / a.seg_G, sg = s % a.seg_G;
        const int tok = min(sg * a.seg_Lc * 64, a.T);
        t0 = (long)n * a.T + tok;
        len = min(a.seg_Lc * 64, a.T - tok);
        ch0 = n * a.NT + sg * a.seg_Lc;
    }
    else              { t0 = (long)s * a.T;   len = a.T;                           ch0 = s * a.NT; }
    const bool store = (a.opts & kOptNoStore) == 0;      // off: only the state is carried (segment pre-pass)
    const int nch = (len + 63) / 64;
    const int col = slice * SLW + 16 * wave + r;

    // forward: the state; backward: its gradient
    const float* init = REV ? a.d_hT : a.h0;
    floatx4 S[KB];
#pragma unroll
    for (int kt = 0; kt < KB; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int f = 32 * (kt >> 1) + 8 * g + 4 * (kt & 1) + e;
            S[kt][e] = (init && wave < NW) ? init[((size_t)chain * DK + f) * a.dv_dim + col] : 0.f;   // not the copy wave
        }

    const size_t kq_row = (size_t)a.H * DK * 2, v_row = (size_t)a.H * a.dv_dim * 2;     // bytes between tokens
    const char* kbase = reinterpret_cast<const char*>(a.k) + (size_t)t0 * kq_row + (size_t)h * DK * 2;
    const char* qbase = reinterpret_cast<const char*>(a.q) + (size_t)t0 * kq_row + (size_t)h * DK * 2;
    const char* vbase = reinterpret_cast<const char*>(REV ? a.d_o : a.v) + (size_t)t0 * v_row + ((size_t)h * a.dv_dim + slice * SLW) * 2;
    constexpr int REC = bwd_record_bytes<bf16_t>();
    const char* tpbase = a.rec + ((size_t)ch0 * a.H + h) * REC;

    // ---- loop-invariant per-lane offsets (as in the forward kernel) -----------------------------------
    const int lrow = lane / PPR, pcol = lane % PPR;
    constexpr int NGK = 8 / RPB;                        // the swizzle has period 8 rows
    int gk[NGK];
#pragma unroll
    for (int j = 0; j < NGK; ++j)
        gk[j] = lrow * (int)kq_row + ((pcol ^ swz_piece<DK>(RPB * j + lrow)) * 16);
    const int gv = (lane / VPP) * (int)v_row + (((lane % VPP) ^ C::vswz(lane / VPP)) * 16);
    int oK[KP];
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) oK[kp] = r * RB + (((4 * kp + g) ^ swz_piece<DK>(r)) * 16);
    const int a4 = r >> 2, c4 = r & 3;
    int oKT[KP];
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) oKT[kp] = (4 * g + a4) * RB + (((4 * kp + c4) ^ swz_piece<DK>(4 * g + a4)) * 16);
    const int oV = (4 * g + a4) * VRW + (((2 * wave + (c4 >> 1)) ^ C::vswz(4 * g + a4)) * 16) + (c4 & 1) * 8;
    const int oO = (4 * g + (r & 3)) * ORB + (16 * wave + 4 * (r >> 2)) * 2;
    const bool q_lo = (r & 3) < 2;
    const uint32_t psel = (r & 1) ? 0x03020706u : 0x05040100u;

    // ---- global -> LDS copy of everything chunk c needs ---------------------------------------------------
    // part 0: all of it; TWO: part 1 = K, M^T, the dO slice, the vectors, part 2 = Q and P^T (at sq)
    auto issue = [&](int c, char* st, char* sq, auto part_c) {
        constexpr int part = decltype(part_c)::value;
        constexpr bool first = part != 2, rest = REV && part != 1;
        const int clen = min(64, len - 64 * c);
        const char* kc = kbase + (size_t)(64 * c) * kq_row;
        const char* qc = qbase + (size_t)(64 * c) * kq_row;
        const char* vc = vbase + (size_t)(64 * c) * v_row;
        const char* tc = tpbase + (size_t)c * a.H * REC;
        if (clen == 64) {
            static_for<C::NKB>([&](auto i) {
                const int b = i;
                const size_t o = (size_t)(b * RPB) * kq_row;
                const int lo = gk[b % NGK];
                if constexpr (first) dma16(kc + o, lo, st + b * 1024);
                if constexpr (rest) dma16(qc + o, lo, sq + C::OFF_Q + b * 1024);
            });
            if constexpr (first)
                static_for<C::NVB>([&](auto i) {
                    const int b = i;
                    dma16(vc + (size_t)(b * RPV) * v_row, gv, st + C::OFF_V + b * 1024);
                });
        } else {                                         // ragged last chunk: clamp the row
            static_for<C::NKB>([&](auto i) {
                const int b = i;
                const int row = b * RPB + lrow;
                const int lo = min(row, clen - 1) * (int)kq_row + ((pcol ^ swz_piece<DK>(row)) * 16);
                if constexpr (first) dma16(kc, lo, st + b * 1024);
                if constexpr (rest) dma16(qc, lo, sq + C::OFF_Q + b * 1024);
            });
            if constexpr (first)
                static_for<C::NVB>([&](auto i) {
                    const int b = i;
                    const int row = b * RPV + lane / VPP;
                    dma16(vc, min(row, clen - 1) * (int)v_row + (((lane % VPP) ^ C::vswz(row)) * 16), st + C::OFF_V + b * 1024);
                });
        }
        // forward: T' (first part of the record); backward: M^T, P^T (second and third)
        static_for<C::TPB / 1024>([&](auto i) {
            const int b = i;
            if constexpr (first) dma16(tc + (REV ? C::TPB : 0) + b * 1024, lane * 16, st + C::OFF_T + b * 1024);
            if constexpr (rest) dma16(tc + 2 * C::TPB + b * 1024, lane * 16, sq + C::OFF_P + b * 1024);
        });
        // gamma_i | gamma_C/gamma_i | beta_i, and for the reverse sweep 1/||q_i|| (the fifth vector of the record)
        if constexpr (first) {
            if constexpr (REV) dma16(tc + 3 * C::TPB, lane < 48 ? lane * 16 : 1024 + (lane - 48) * 16, st + C::OFF_EG);
            else if (lane < 48) dma16(tc + 3 * C::TPB, lane * 16, st + C::OFF_EG);
        }
    };

    // 4x4 transposition inside each quad of lanes, then one 64-bit write: lane (r, g) ends up with row 4 g + (r & 3),
    // columns 4 (r >> 2) .. + 3 of the wave's 16
    auto stage_quad = [&](u32x2 ob, char* dst) { *reinterpret_cast<u32x2*>(dst) = quad_transpose4x4(ob, q_lo, psel); };

    // ---- one chunk for this wave's 16 columns -----------------------------------------------------------
    // sq: where Q and P^T are (TWO: a stage of the second ring; else st)
    auto compute = [&](const char* st, [[maybe_unused]] const char* sq, char* ost, int c) {
        const int clen = min(64, len - 64 * c);
        const char* pS = st + lane * 16;
        const char* pV = st + C::OFF_V + oV;
        const char* pG = st + C::OFF_EG + 16 * g;
        auto kslot = [&](int it, int kp) {
            return ld16(st + oK[kp] + 16 * it * RB);
        };
        auto ktslot = [&](int kt, int jp, const char* tile, u32x2& q0, u32x2& q1) {      // tile: K or Q
            const int kp = kt >> 1, b = kt & 1;
            const char* p = tile + oKT[kp] + 32 * jp * RB + 8 * b;
            q0 = lds_read_tr(p);
            q1 = lds_read_tr(p + 16 * RB);
        };

        const float gC = *reinterpret_cast<const float*>(st + C::OFF_EG + 63 * 4);
        u32x2 Sq[KB];
#pragma unroll
        for (int kt = 0; kt < KB; ++kt) { Sq[kt] = to_quad(S[kt]); if constexpr (!REV) S[kt] = S[kt] * gC; }
        if (store) put_checkpoint<DK>(reinterpret_cast<char*>(REV ? a.ds_chk : a.s_chk) + ((size_t)(ch0 + c) * a.H + h) * a.dv_dim * RB,
                                      slice * NW + wave, Sq, r, g);

        // ---- K S or K dS'
        floatx4 ks[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) ks[it] = floatx4{0.f, 0.f, 0.f, 0.f};
        u32x4 ka[2][4];
#pragma unroll
        for (int it = 0; it < 4; ++it) ka[0][it] = kslot(it, 0);
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) {
            if (kp + 1 < KP) {
#pragma unroll
                for (int it = 0; it < 4; ++it) ka[(kp + 1) & 1][it] = kslot(it, kp + 1);
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) mma_bf16(ks[it], ka[kp & 1][it], Sq[2 * kp], Sq[2 * kp + 1]);
        }
        u32x2 vq[4];
        floatx4 egv[4], edv[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            vq[it] = lds_read_tr(pV + 16 * it * VRW);
            egv[it] = ld_f4(pG + 64 * it);
            edv[it] = ld_f4(pG + 256 + 64 * it);
        }
        u32x4 tsl[kTriPairs];
#pragma unroll
        for (int i = 0; i < kTriPairs; ++i) tsl[i] = ld16(pS + C::OFF_T + i * 1024);
        u32x2 kt[2][KB][2];                              // [token pair jp][state tile][token block]

        if constexpr (!REV) {
            u32x2 Xq[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                Xq[it] = to_quad(quad_to_f(vq[it]) - egv[it] * ks[it]);       // eq. (6), right-hand side without B
            }
            put_rows(reinterpret_cast<char*>(a.X) + (size_t)(t0 + 64L * c) * v_row, v_row, a.dv_dim, h, slice * NW + wave, Xq, clen, r, g);
#pragma unroll
            for (int t = 0; t < KB; ++t) ktslot(t, 0, st, kt[0][t][0], kt[0][t][1]);
            floatx4 U[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                U[it] = floatx4{0.f, 0.f, 0.f, 0.f};
                mma_bf16(U[it], tsl[tri_pair(it, 0)], Xq[0], Xq[1]);
            }
            mma_bf16(U[2], tsl[tri_pair(2, 1)], Xq[2], Xq[3]);
            mma_bf16(U[3], tsl[tri_pair(3, 1)], Xq[2], Xq[3]);
#pragma unroll
            for (int t = 0; t < KB; ++t) ktslot(t, 1, st, kt[1][t][0], kt[1][t][1]);
            u32x2 Udq[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) Udq[it] = to_quad(U[it] * edv[it]);   // U itself is not kept: the assembly forms it again from T' and X
#pragma unroll
            for (int t = 0; t < KB; ++t) mma_bf16(S[t], kt[0][t][0], kt[0][t][1], Udq[0], Udq[1]);
#pragma unroll
            for (int t = 0; t < KB; ++t) mma_bf16(S[t], kt[1][t][0], kt[1][t][1], Udq[2], Udq[3]);
        } else {
            u32x4 psl[kTriPairs];
#pragma unroll
            for (int i = 0; i < kTriPairs; ++i) psl[i] = ld16(sq + lane * 16 + C::OFF_P + i * 1024);
            // ---- dU = diag(gamma_C/gamma_i) K dS' + P^T dO   (P^T upper triangular; the order of the sums here and in the state
            //      update is that of kla_chunk_rev_bf16.hip, to the last bit)
            floatx4 dU[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) dU[it] = floatx4{0.f, 0.f, 0.f, 0.f};
            mma_bf16(dU[0], psl[triu_pair(0, 0)], vq[0], vq[1]);
            mma_bf16(dU[1], psl[triu_pair(1, 0)], vq[0], vq[1]);
#pragma unroll
            for (int it = 0; it < 4; ++it) mma_bf16(dU[it], psl[triu_pair(it, 1)], vq[2], vq[3]);
            u32x2 dUq[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) dUq[it] = to_quad(edv[it] * ks[it] + dU[it]);
#pragma unroll
            for (int t = 0; t < KB; ++t) ktslot(t, 0, sq + C::OFF_Q, kt[0][t][0], kt[0][t][1]);
            // ---- Y = M^T dU
            floatx4 Y[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) Y[it] = floatx4{0.f, 0.f, 0.f, 0.f};
            mma_bf16(Y[0], tsl[triu_pair(0, 0)], dUq[0], dUq[1]);
            mma_bf16(Y[1], tsl[triu_pair(1, 0)], dUq[0], dUq[1]);
#pragma unroll
            for (int it = 0; it < 4; ++it) mma_bf16(Y[it], tsl[triu_pair(it, 1)], dUq[2], dUq[3]);
#pragma unroll
            for (int t = 0; t < KB; ++t) ktslot(t, 1, sq + C::OFF_Q, kt[1][t][0], kt[1][t][1]);
            u32x2 gdOq[4], gdXq[4];
            u32x2 Yq[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const floatx4 dx = Y[it] * ld_f4(pG + 512 + 64 * it);           // dV = B Y
                Yq[it] = to_quad(Y[it]);
                stage_quad(to_quad(dx), ost + oO + 16 * it * ORB);
                floatx4 eg = egv[it];
#pragma unroll
                for (int e = 0; e < 4; ++e) eg[e] = (16 * it + 4 * g + e < clen) ? eg[e] : 0.f;   // rows past a ragged end
                gdOq[it] = to_quad(eg * ld_f4(pG + 768 + 64 * it) * quad_to_f(vq[it]));   // D_gamma dO / ||q||
                gdXq[it] = to_quad(-(eg * dx));
            }
            if (store) put_rows(reinterpret_cast<char*>(a.Y) + (size_t)(t0 + 64L * c) * v_row, v_row, a.dv_dim, h, slice * NW + wave, Yq, clen, r, g);
            // ---- dS = gamma_C dS' + Q^T D_gamma dO - K^T D_gamma dV
            floatx4 inc[KB];
#pragma unroll
            for (int t = 0; t < KB; ++t) { inc[t] = floatx4{0.f, 0.f, 0.f, 0.f}; mma_bf16(inc[t], kt[0][t][0], kt[0][t][1], gdOq[0], gdOq[1]); }
#pragma unroll
            for (int t = 0; t < KB; ++t) mma_bf16(inc[t], kt[1][t][0], kt[1][t][1], gdOq[2], gdOq[3]);
#pragma unroll
            for (int t = 0; t < KB; ++t) S[t] = S[t] * gC + inc[t];
#pragma unroll
            for (int t = 0; t < KB; ++t) ktslot(t, 0, st, kt[0][t][0], kt[0][t][1]);
#pragma unroll
            for (int t = 0; t < KB; ++t) ktslot(t, 1, st, kt[1][t][0], kt[1][t][1]);
#pragma unroll
            for (int t = 0; t < KB; ++t) mma_bf16(S[t], kt[0][t][0], kt[0][t][1], gdXq[0], gdXq[1]);
#pragma unroll
            for (int t = 0; t < KB; ++t) mma_bf16(S[t], kt[1][t][0], kt[1][t][1], gdXq[2], gdXq[3]);
        }
    };

    // Reverse sweep: the staged rows of dV go out through a wave that does nothing else, 16 bytes per lane
    auto write_out = [&](int c, const char* ost) {
        const int clen = min(64, len - 64 * c);
        char* o1 = reinterpret_cast<char*>(a.dv) + (size_t)(t0 + 64L * c) * v_row + ((size_t)h * a.dv_dim + slice * SLW) * 2;
#pragma unroll
        for (int it = 0; it < VPP; ++it) {
            const int i = lane + 64 * it;
            const int row = i / VPP, pv = i % VPP;
            if (row < clen) __builtin_nontemporal_store(ld16(ost + row * ORB + pv * 16), reinterpret_cast<u32x4*>(o1 + (size_t)row * v_row + pv * 16));
        }
    };

    char* ost0 = lds + C::OFF_OST;                       // reverse sweep only
    char* ost1 = ost0 + C::OSB;
    // chunks are visited in the order i = 0 .. nch-1; the backward sweep starts at the last chunk
    auto chunk_of = [&](int i) { return REV ? nch - 1 - i : i; };

    if constexpr (REV) {
        if (wave == NW + 1) {
            // ---- the store wave: after the barrier that ends visit i, chunk_of(i) is complete in the staging area of
            //      parity i & 1, which the compute waves write again only in visit i + 2, behind the barrier this wave
            //      reaches next
            //      Two chains: it also touches lines of K, Q, M^T and P^T of the visit AHEAD later (a.touch: where these are more
            //      than the memory-side cache holds on to). At d_k = 128 the 352 lines are those of three slices; the two slices of
            //      d_v = 64 ask for K and Q alone.  At d_k = 64 two slices ask for all 224.
            constexpr int AHEAD = 4;
            uint32_t seen[2] = {0u, 0u};
            __syncthreads();
            for (int i = 0; i < nch; ++i) {
                if constexpr (NW == 2) {
                    asm volatile("" ::"v"(seen[0]), "v"(seen[1]));
                    if (a.touch && i + AHEAD < nch) {
                        const int c = chunk_of(i + AHEAD);
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            seen[j] = touch_line<RB>(kbase, qbase, kq_row, 64 * c, len, tpbase + (size_t)c * a.H * REC + C::TPB, 2 * C::TPB / 128, (2 * slice + j) * 64 + lane);
                    }
                }
                __syncthreads();
                if (store) write_out(chunk_of(i), (i & 1) ? ost1 : ost0);
            }
            return;
        }
    }

    if constexpr (C::TWO) {
        if (wave == NW) {
            // ---- the copy wave of two rings, as in the forward kernel (i: visits)
            auto first = [&](int i) { issue(chunk_of(i), lds + (i % 3) * C::STAGE, nullptr, IntC<1>()); };
            auto rest = [&](int i) { issue(chunk_of(i), nullptr, lds + 3 * C::STAGE + (i & 1) * C::QST, IntC<2>()); };
            if (nch > 0) { first(0); rest(0); }
            if (nch > 1) { first(1); wait_vmcnt<C::N_FIRST>(); } else wait_vmcnt<0>();
            __syncthreads();
            for (int i = 0; i < nch; ++i) {
                if (i + 1 < nch) rest(i + 1);
                if (i + 2 < nch) { first(i + 2); wait_vmcnt<C::N_FIRST>(); } else wait_vmcnt<0>();
                __syncthreads();
            }
            return;
        }
    }
    if (wave == NW) {
        // ---- the copy wave: keeps the next NST-1 chunks on their way while one is computed -----------------
#pragma unroll
        for (int p = 0; p < NST - 1; ++p)
            if (p < nch) issue(chunk_of(p), lds + p * C::STAGE, lds + p * C::STAGE, IntC<0>());
        if (NST == 3 && nch > 1) wait_vmcnt<C::NDMA>(); else wait_vmcnt<0>();
        __syncthreads();
        int spre = NST - 1;
        for (int i = 0; i < nch; ++i) {
            const bool ahead = i + NST - 1 < nch;
            if (ahead) issue(chunk_of(i + NST - 1), lds + spre * C::STAGE, lds + spre * C::STAGE, IntC<0>());
            if (NST == 3 && ahead) wait_vmcnt<C::NDMA>(); else wait_vmcnt<0>();
            __syncthreads();
            spre = (spre + 1 == NST) ? 0 : spre + 1;
        }
        return;
    }

    // ---- compute waves (same barrier discipline as the forward kernel) --------------------------------------
    __syncthreads();
    int scur = 0;
    for (int i = 0; i < nch; ++i) {
        const int c = chunk_of(i);
        char* st = lds + scur * C::STAGE;
        compute(st, C::TWO ? lds + 3 * C::STAGE + (i & 1) * C::QST : st, (i & 1) ? ost1 : ost0, c);
        __syncthreads();
        scur = (scur + 1 == NST) ? 0 : scur + 1;
    }

    if (REV && a.dh0) {
#pragma unroll
        for (int kt = 0; kt < KB; ++kt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int f = 32 * (kt >> 1) + 8 * g + 4 * (kt & 1) + e;
                a.dh0[((size_t)chain * DK + f) * a.dv_dim + col] = S[kt][e];
            }
    }
}

// =================================================================================================
// per chunk-head contractions (bf16): the algebra of bwd_assemble_kernel in kla_chunk_bwd.hip on direct
// global -> LDS copies.  Every operand sits in LDS as plain swizzled rows: the slab of S^T and dS'^T (64 rows of
// d_k) and the K, Q tiles exactly like a K tile of the sweeps, the [64 tokens x 32 columns] slabs of dO
// in rows of 64 bytes.  Operands contracted along a row are two 64-bit reads, operands contracted down a
// column (S^T, dS'^T, K, Q) come from the transposing read, which makes lane r of an output tile the feature
// 32 kp + 8 (r / 4) + 4 b + r % 4 of tile 2 kp + b; the K and Q values that meet those outputs are read the same
// way, and the 4x4 transposition before the staged write-out puts the features back in order.  X, Y and U are in the
// operand order the sweeps leave them in: X is the B operand of T' X as it lies, and token rows of Y, U (and X) are the
// columns of such a slot area, read with the transposing read.  (X and Y of a short chunk are rows in memory, and here.)
// A short last chunk re-reads its last valid row for the rows beyond it; the rows of A o dP and D', of the
// <.,k> sums and of dg that belong to those rows are masked to zero.
// =================================================================================================
namespace {
// acc + x.lo * y.lo + x.hi * y.hi for two packed bf16 pairs (v_dot2c_f32_bf16)
__device__ __forceinline__ float dot2_bf16(uint32_t x, uint32_t y, float acc)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, x), __builtin_bit_cast(bf16x2_t, y), acc, false);
}
}  // namespace

template <int DK>
__global__ __launch_bounds__(256, 2) void bwd_assemble_bf16_kernel(BwdArgs<bf16_t> a)
{
    constexpr int KB = DK / 16, KP = DK / 32;
    constexpr int RB = DK * 2, PPR = DK / 8, RPB = 1024 / RB, NKB = 64 / RPB;      // [64 x d_k] tiles
    constexpr int RBA = 64, NAB = 4;                 // [64 tokens x 32 columns] slabs: 4 blocks of 16 rows of 64 bytes
    constexpr int TK = 64 * RB, TS = 32 * RB, NSB = TS / 1024, TA = 64 * RBA;
    constexpr int ORQ = RB + 16, MB = 64 * ORQ > 16384 ? 64 * ORQ : 16384;       // row stride and room of the dq / dk staging tiles
    // first phase, two buffers of one 32-column slab each: S^T | dS'^T | dO | U | Y | X (U is formed here, from T' and X)
    constexpr int OFF_S = 0, OFF_DS = TS, OFF_DO = 2 * TS, OFF_U = OFF_DO + TA, OFF_Y = OFF_U + TA, OFF_X = OFF_Y + TA;
    constexpr int SLAB = 2 * TS + 4 * TA;
    constexpr int PH1 = 2 * SLAB;
    // second phase: K | Q | A o dP, D' | B D', the latter two areas also the staging tiles of dq and dk.  K and Q are fetched into the
    // first buffer while the last slab (always in the second one: d_v / 32 is even) is being used.
    constexpr int OFF_K = 0, OFF_Q = TK, OFF_E1 = 2 * TK, OFF_DP = 2 * TK + MB;
    constexpr int PH2 = 2 * TK + 2 * MB;
    constexpr int BIG = PH1 > PH2 ? PH1 : PH2;
    static_assert(2 * TK <= SLAB, "the K and Q tiles fit one slab buffer");
    __shared__ __attribute__((aligned(1024))) char lds[BIG];
    __shared__ __attribute__((aligned(1024))) char tp_s[kTriPairs * 1024];       // T' of the chunk, as the record holds it
    __shared__ __attribute__((aligned(16))) float eg_s[64], ed_s[64], beta_s[64], invden_s[64], rq_s[64], g_s[64], yx_s[64],
        dg_s[64], dbeta_s[64];
    __shared__ float red_s[8];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    const int h = blockIdx.x % a.H;
    const int cg = blockIdx.x / a.H;
    const ChunkPos cp = chunk_pos(a.cu_seqlens, a.chunk_off, a.n_seq, a.T, a.NT, cg);
    const long tok0 = cp.tok0;
    const int clen = cp.clen;
    const size_t kq_row = (size_t)a.H * DK * 2, v_row = (size_t)a.H * a.dv_dim * 2;
    const char* rec = a.rec + (size_t)blockIdx.x * bwd_record_bytes<bf16_t>();
    // With the normalised read-out (Sec. 3.3) the query that meets the state is q^ = q / ||q||.  Scaling the rows of dO
    // by 1/||q_i|| wherever they meet U or S gives dQ' = diag(1/||q||) dL/dq^ directly, (A o dP')^T Q is what dK
    // needs, q_i . dQ'_i is what dg needs, and dq_i = dQ'_i - (q_i . dQ'_i) q_i / ||q_i||^2 at the end.
    const bool norm_q = (a.opts & kOptNormalizeQ) != 0;
    {
        const float* vec = reinterpret_cast<const float*>(rec + 3 * ws_half_bytes<bf16_t>());
        float* dst = wave == 0 ? eg_s : (wave == 1 ? ed_s : (wave == 2 ? beta_s : invden_s));
        dst[lane] = vec[tid];
        if (wave == 1) rq_s[lane] = vec[256 + lane];
        if (wave == 0) {                                 // g_i = log gamma_i, in units of log 2: the decay ratios below are exp2 of differences
            const float la = lane < clen ? a.log_alpha[(size_t)(tok0 + lane) * a.H + h] : 0.f;
            g_s[lane] = prefix_sum64(la, lane) * 1.44269504088896341f;
        }
    }

    // ---- per-lane offsets ---------------------------------------------------------------------------
    // copies of [rows x d_k] tiles and of [64 x 32] slabs, swizzled on the global side (the 16-byte column index is
    // XORed with swz_piece(row) resp. (row / 2) % 4)
    const int lrow = lane / PPR, pcol = lane % PPR;
    const int lrowA = lane >> 2, pcolA = lane & 3;
    // The per-lane part of a checkpoint copy's address depends on the block only through b % NGK (the swizzle has
    // period 8 rows).  Rows past the end of a ragged chunk re-read its last one.
    const bool full = clen == 64;
    constexpr int NGK = 8 / RPB;
    int gst[NGK];                                    // piece 4 kp + g of column lrow (see put_checkpoint)
#pragma unroll
    for (int j = 0; j < NGK; ++j) { const int pc = pcol ^ swz_piece<DK>(RPB * j + lrow); gst[j] = lrow * 64 + (pc >> 2) * 1024 + (pc & 3) * 16; }
    const int gsl = lrowA * (int)v_row + ((pcolA ^ ((lrowA >> 1) & 3)) * 16);
    auto copy_tile = [&](const char* src, size_t stride, char* dst, int b0, int b1) {       // blocks [b0, b1) of a [64 x d_k] tile
        for (int b = b0; b < b1; ++b) {
            const int row = b * RPB + lrow;
            dma16(src, min(row, clen - 1) * (int)stride + ((pcol ^ swz_piece<DK>(row)) * 16), dst + b * 1024);
        }
    };
    auto copy_state = [&](const char* src, char* dst) {                                      // 32 columns of a checkpoint: never ragged
        static_for<NSB>([&](auto bb) {
            const int b = bb;
            dma16(src + (b * RPB / 16) * (16 * RB) + (b * RPB % 16) * 64, gst[b % NGK], dst + b * 1024);
        });
    };
    auto copy_slab = [&](const char* src, char* dst) {                                       // 4 blocks of 16 token rows x 64 bytes
        static_for<NAB>([&](auto bb) {
            const int b = bb;
            if (full) dma16(src + (size_t)(b * 16) * v_row, gsl, dst + b * 1024);
            else      dma16(src, min(b * 16 + lrowA, clen - 1) * (int)v_row + ((pcolA ^ ((lrowA >> 1) & 3)) * 16), dst + b * 1024);
        });
    };
    // row-contracted operand of a slab: token row 16 t + r, contraction indices {4 g .. +3 | 16 + 4 g .. +3}
    const int arow = r * RBA + (g & 1) * 8, asw = (r >> 1) & 3;
    const int acol0 = ((g >> 1) ^ asw) * 16, acol1 = ((2 + (g >> 1)) ^ asw) * 16;
    auto aslot = [&](const char* tile, int t, u32x2& q0, u32x2& q1) {
        const char* p = tile + 16 * t * RBA + arow;
        q0 = *reinterpret_cast<const u32x2*>(p + acol0);
        q1 = *reinterpret_cast<const u32x2*>(p + acol1);
    };
    // column-contracted operand of a [64 x d_k] tile through the transposing read (as K^T in the sweeps)
    const int a4 = r >> 2, c4 = r & 3;
    int oKT[KP];
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) oKT[kp] = (4 * g + a4) * RB + (((4 * kp + c4) ^ swz_piece<DK>(4 * g + a4)) * 16);
    auto tslot = [&](const char* tile, int kt, int jp, u32x2& q0, u32x2& q1) {
        const int kp = kt >> 1, b = kt & 1;
        const char* p = tile + oKT[kp] + 32 * jp * RB + 8 * b;
        q0 = lds_read_tr(p);
        q1 = lds_read_tr(p + 16 * RB);
    };

    // Slot areas of a slab: [column tile ct][token pair jp][64 slots], 4 KiB.  Token row 16 t + r of one, contraction indices =
    // columns {4 g .. +3 | 16 + 4 g .. +3}: source lane (a4, c4) of the transposing read points at the four tokens
    // 16 t + 4 c4 .. of column 4 g + a4, i.e. at slot (r' = 4 g + a4, g' = c4).  In the areas of Y and U the slots of odd g'
    // are exchanged by halves (slot index XOR 8), so that the 32 lanes served at once meet in pairs and not in fours.
    const int oT = ((16 * c4 + 4 * g + a4) ^ (8 * (c4 & 1))) * 16, oTx = (16 * c4 + 4 * g + a4) * 16;
    auto rowslot = [&](const char* tile, int t, int off, u32x2& q0, u32x2& q1) {
        const char* p = tile + (t >> 1) * 1024 + 8 * (t & 1) + off;
        q0 = lds_read_tr(p);
        q1 = lds_read_tr(p + 2048);
    };
    const int swl = (lane ^ (8 * (g & 1))) * 16;         // this lane's slot of such an area
    // rows of X (a short chunk), column-contracted: where this lane's 8 bytes sit (column tile 0; tile 1: bit 5 flipped)
    const int xo = (4 * g + a4) * RBA + ((((c4 >> 1)) ^ ((2 * g + (a4 >> 1)) & 3)) * 16) + (c4 & 1) * 8;
    // U = T' X is not read back from the forward sweep but formed again, slab by slab: the T' tile pairs of this wave's 16
    // rows (A operands, copied from the record into LDS once) times the X slots, the result put into the slab's U area.
    for (int i = wave; i < kTriPairs; i += 4) dma16(rec + i * 1024, lane * 16, tp_s + i * 1024);   // lands with the first slab
    floatx4 dQ[KB], dKr[KB], dKw[KB], dP[4], N1[4];
#pragma unroll
    for (int ct = 0; ct < KB; ++ct) { dQ[ct] = floatx4{0.f, 0.f, 0.f, 0.f}; dKr[ct] = dQ[ct]; dKw[ct] = dQ[ct]; }
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) { dP[jt] = floatx4{0.f, 0.f, 0.f, 0.f}; N1[jt] = dP[jt]; }
    floatx4 YX = floatx4{0.f, 0.f, 0.f, 0.f};        // tile (wave, wave) of Y X^T: its diagonal is wanted
    float sdot = 0.f;

    // ---- first phase: everything that contracts over d_v, 32 columns at a time.  The products of a slab take a quarter of a
    //      trip to memory, so a buffer is refilled as soon as every wave is done with it (one more barrier per slab), while
    //      the slab in the other one is still on its way; K and Q come behind the last slab.  12 sequences of 100 .. 2100 tokens,
    //      8 heads, d_v = 256: assembly 151 -> 144 us; 8 x 4096 tokens, d_v = 128: 164 -> 156. (With row sums by DPP and the
    //      bf16 tiles of the second phase 133 and 150 us, 5.3 TB/s of its bytes.) -----------------
    const char* Sg = reinterpret_cast<const char*>(a.s_chk) + (size_t)blockIdx.x * DK * a.dv_dim * 2;
    const char* dSg = reinterpret_cast<const char*>(a.ds_chk) + (size_t)blockIdx.x * DK * a.dv_dim * 2;
    // X and Y of a whole chunk: slots, 4 KiB per slab; of a short one: rows (put_rows)
    const size_t xy0 = (size_t)tok0 * v_row + (size_t)h * a.dv_dim * (full ? 128 : 2);
    const char* Xg = reinterpret_cast<const char*>(a.X) + xy0;
    const char* Yg = reinterpret_cast<const char*>(a.Y) + xy0;
    const size_t vrow0 = (size_t)tok0 * v_row + (size_t)h * a.dv_dim * 2;
    auto issue_slab = [&](int sl, char* buf) {
        if (wave == 0)      copy_state(Sg + (size_t)(32 * sl) * RB, buf + OFF_S);
        else if (wave == 1) copy_state(dSg + (size_t)(32 * sl) * RB, buf + OFF_DS);
        else if (wave == 2) copy_slab(reinterpret_cast<const char*>(a.d_o) + vrow0 + 64 * sl, buf + OFF_DO);
        else {
            if (full) {
                static_for<4>([&](auto bb) {
                    const int b = bb;
                    dma16(Yg + (size_t)sl * 4096 + b * 1024, swl, buf + OFF_Y + b * 1024);
                    dma16(Xg + (size_t)sl * 4096 + b * 1024, lane * 16, buf + OFF_X + b * 1024);
                });
            } else {
                copy_slab(Yg + 64 * sl, buf + OFF_Y);
                copy_slab(Xg + 64 * sl, buf + OFF_X);
            }
        }
    };
    const int ns = a.dv_dim / 32;
    issue_slab(0, lds);
    issue_slab(1, lds + SLAB);
    for (int sl = 0; sl < ns; ++sl) {
        const char* buf = lds + (sl & 1) * SLAB;
        // all but the copies issued last, which are the next slab's or (NKB / 2 of each wave) K's and Q's
        if (sl + 1 == ns)   wait_vmcnt<NKB / 2>();
        else if (wave < 2)  wait_vmcnt<NSB>();
        else if (wave == 2) wait_vmcnt<NAB>();
        else                wait_vmcnt<2 * NAB>();
        __syncthreads();                             // slab sl has landed
        // U = T' X: this wave's 16 rows of the slab
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
            floatx4 u = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int jp = 0; jp < 2; ++jp) {
                if (2 * jp <= wave) {                      // T' is lower triangular (wave-uniform)
                    u32x2 x0, x1;
                    if (full) {
                        const u32x4 xs = ld16(buf + OFF_X + (2 * ct + jp) * 1024 + lane * 16);
                        x0 = u32x2{xs[0], xs[1]}; x1 = u32x2{xs[2], xs[3]};
                    } else {
                        const char* xp = buf + OFF_X + 32 * jp * RBA + (xo ^ (32 * ct));
                        x0 = lds_read_tr(xp); x1 = lds_read_tr(xp + 16 * RBA);
                    }
                    mma_bf16(u, ld16(tp_s + tri_pair(wave, jp) * 1024 + lane * 16), x0, x1);
                }
            }
            *reinterpret_cast<u32x2*>(lds + (sl & 1) * SLAB + OFF_U + ct * 2048 + (wave >> 1) * 1024 + 8 * (wave & 1) + swl) = to_quad(u);
        }
        u32x2 y0, y1;
        {   // Y_i . X_i
            u32x2 x0, x1;
            if (full) { rowslot(buf + OFF_Y, wave, oT, y0, y1); rowslot(buf + OFF_X, wave, oTx, x0, x1); }
            else      { aslot(buf + OFF_Y, wave, y0, y1); aslot(buf + OFF_X, wave, x0, x1); }
            mma_bf16(YX, y0, y1, x0, x1);
        }
        {   // <dS', S>: plain 16-byte pieces, the swizzle is the same for both tiles
#pragma unroll
            for (int pc = 0; pc < TS / 16 / 256; ++pc) {
                const int o = (tid + 256 * pc) * 16;
                const u32x4 sv = ld16(buf + OFF_S + o), dv = ld16(buf + OFF_DS + o);
#pragma unroll
                for (int m = 0; m < 4; ++m) sdot = dot2_bf16(sv[m], dv[m], sdot);
            }
        }
        __syncthreads();                             // every wave's rows of U are in the slab
        u32x2 do0, do1, u0, u1;
        aslot(buf + OFF_DO, wave, do0, do1);
        rowslot(buf + OFF_U, wave, oT, u0, u1);
#pragma unroll
        for (int ct = 0; ct < KB; ++ct) {
            u32x2 s0, s1, d0, d1;
            tslot(buf + OFF_S, ct, 0, s0, s1);
            tslot(buf + OFF_DS, ct, 0, d0, d1);
            mma_bf16(dQ[ct], do0, do1, s0, s1);            // dO S^T
            mma_bf16(dKr[ct], y0, y1, s0, s1);             // Y S^T
            mma_bf16(dKw[ct], u0, u1, d0, d1);             // U dS'^T
        }
        static_for<4>([&](auto jt) {
            if (jt <= wave) {                              // lower-triangular tiles only
                u32x2 b0, b1;
                rowslot(buf + OFF_U, jt, oT, b0, b1);
                mma_bf16(dP[jt], do0, do1, b0, b1);        // dO U^T
                mma_bf16(N1[jt], y0, y1, b0, b1);          // Y U^T
            }
        });
        if (sl + 1 < ns) {
            __syncthreads();                         // slab sl is no longer read
            if (sl + 2 < ns) issue_slab(sl + 2, lds + (sl & 1) * SLAB);
            else {
                const char* kb = reinterpret_cast<const char*>(a.k) + (size_t)tok0 * kq_row + (size_t)h * DK * 2;
                const char* qb = reinterpret_cast<const char*>(a.q) + (size_t)tok0 * kq_row + (size_t)h * DK * 2;
                if (wave < 2) copy_tile(kb, kq_row, lds + OFF_K, wave * (NKB / 2), (wave + 1) * (NKB / 2));
                else          copy_tile(qb, kq_row, lds + OFF_Q, (wave - 2) * (NKB / 2), (wave - 1) * (NKB / 2));
            }
        }
    }
    {   // D_gamma dO S^T,  -D_gamma dX S^T (dX = B Y),  diag(gamma_C/gamma_i) U dS'^T
        const floatx4 egv = ld_f4(reinterpret_cast<const char*>(eg_s + 16 * wave + 4 * g));
        const floatx4 edv = ld_f4(reinterpret_cast<const char*>(ed_s + 16 * wave + 4 * g));
        const floatx4 ngb = -(egv * ld_f4(reinterpret_cast<const char*>(beta_s + 16 * wave + 4 * g)));
        const floatx4 egq = egv * ld_f4(reinterpret_cast<const char*>(rq_s + 16 * wave + 4 * g));
#pragma unroll
        for (int ct = 0; ct < KB; ++ct) { dQ[ct] = dQ[ct] * egq; dKr[ct] = dKr[ct] * ngb; dKw[ct] = dKw[ct] * edv; }
    }
    if ((r >> 2) == g) yx_s[16 * wave + r] = (r & 2) ? ((r & 1) ? YX[3] : YX[2]) : ((r & 1) ? YX[1] : YX[0]);
    sdot = wave_sum_rows(sdot);
    if (lane == 0) red_s[wave] = sdot;
    wait_vmcnt<0>();                                 // this wave's part of K and Q
    __syncthreads();                                 // the slab areas are dead from here on

    // ---- second phase: A o dP, D' = -A^- o (Y U^T) and B D' as bf16 tiles of 512 bytes, tile (ti, tj) at 4 ti + tj, each as the
    //      accumulators hold it: lane (r, g)'s quad is rows 4 g .. + 3 of column r, which is the A operand of the transposed
    //      products as it lies and of the others through the transposing read. (As fp32 matrices they took 32 writes of one float, 24 to 48 reads
    //      and the conversions per wave: 152.6 -> 150 us, 136.5 -> 133, one round of chunk-heads 15.6 -> 13.9.) Tiles right of the diagonal that a pair of tiles drags in are zero.
    char* Et = lds + OFF_E1;
    char* Dt = Et + 8192;
    char* Bt = lds + OFF_DP;
    static_assert(2 * 8192 <= MB, "the tiles fit where the staging tiles of dq and dk go");
    {
        const floatx4 gi = ld_f4(reinterpret_cast<const char*>(g_s + 16 * wave + 4 * g)), rqi = ld_f4(reinterpret_cast<const char*>(rq_s + 16 * wave + 4 * g)),
                      bi = ld_f4(reinterpret_cast<const char*>(beta_s + 16 * wave + 4 * g));
        static_for<4>([&](auto jt) {
            if (jt <= (wave | 1)) {
                const int j = 16 * jt + r;
                const float gj = g_s[j];
                floatx4 ev, dv;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 16 * wave + 4 * g + e;
                    const float dec = (jt <= wave && j <= i && i < clen) ? __builtin_amdgcn_exp2f(gi[e] - gj) : 0.f;
                    ev[e] = dec * rqi[e] * dP[jt][e];
                    dv[e] = (j < i) ? -dec * N1[jt][e] : 0.f;
                }
                const int at = (4 * wave + jt) * 512 + lane * 8;
                *reinterpret_cast<u32x2*>(Et + at) = to_quad(ev);
                *reinterpret_cast<u32x2*>(Dt + at) = to_quad(dv);
                *reinterpret_cast<u32x2*>(Bt + at) = to_quad(dv * bi);
            }
        });
    }
    __syncthreads();

    // K and Q of this wave's rows as accumulator tiles: token 16 wave + 4 g + e, feature of (tile ct, lane r)
    auto kacc = [&](int off, int ct) {
        u32x2 q0, q1;
        tslot(lds + off, ct, wave >> 1, q0, q1);
        return quad_to_f((wave & 1) ? q1 : q0);
    };
    floatx4 rowmask;                                 // 1 for the rows of the chunk, 0 past a ragged end
#pragma unroll
    for (int e = 0; e < 4; ++e) rowmask[e] = (16 * wave + 4 * g + e < clen) ? 1.f : 0.f;
    float zsum = 0.f;                                // sum_i (gamma_C/gamma_i) k_i . (dS' U_i)
#pragma unroll
    for (int ct = 0; ct < KB; ++ct) {
        const floatx4 kk = kacc(OFF_K, ct);
#pragma unroll
        for (int e = 0; e < 4; ++e) zsum += rowmask[e] * dKw[ct][e] * kk[e];
    }
    zsum = wave_sum_rows(zsum);
    if (lane == 0) red_s[4 + wave] = zsum;

    floatx4 E2[KB];
#pragma unroll
    for (int ct = 0; ct < KB; ++ct) E2[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int otr = (16 * c4 + 4 * g + a4) * 8;          // source of the transposing read: rows 4 c4 .. + 3 of column 4 g + a4
    auto rows_slot = [&](const char* m, int jp, u32x2& q0, u32x2& q1) {      // rows 16 wave + r, columns 32 jp + (16 +) 4 g ..
        const char* p = m + (4 * wave + 2 * jp) * 512 + otr;
        q0 = lds_read_tr(p);
        q1 = lds_read_tr(p + 512);
    };
    auto cols_slot = [&](const char* m, int jp, u32x2& q0, u32x2& q1) {      // column 16 wave + r, rows 32 jp + (16 +) 4 g ..
        const char* p = m + (8 * jp + wave) * 512 + lane * 8;
        q0 = *reinterpret_cast<const u32x2*>(p);
        q1 = *reinterpret_cast<const u32x2*>(p + 4 * 512);
    };
    static_for<2>([&](auto jp) {
        if (jp <= (wave >> 1)) {
            u32x2 e0, e1, d0, d1;
            rows_slot(Et, jp, e0, e1);
            rows_slot(Dt, jp, d0, d1);
#pragma unroll
            for (int ct = 0; ct < KB; ++ct) {
                u32x2 k0, k1;
                tslot(lds + OFF_K, ct, jp, k0, k1);
                mma_bf16(dQ[ct], e0, e1, k0, k1);          // (A o dP) K
                mma_bf16(E2[ct], d0, d1, k0, k1);          // D' K
            }
        }
        if (jp >= (wave >> 1)) {
            u32x2 e0, e1, d0, d1;
            cols_slot(Et, jp, e0, e1);
            cols_slot(Bt, jp, d0, d1);
#pragma unroll
            for (int ct = 0; ct < KB; ++ct) {
                u32x2 k0, k1, q0, q1;
                tslot(lds + OFF_Q, ct, jp, q0, q1);
                tslot(lds + OFF_K, ct, jp, k0, k1);
                mma_bf16(dKw[ct], e0, e1, q0, q1);         // (A o dP)^T Q
                mma_bf16(dKw[ct], d0, d1, k0, k1);         // (B D')^T K
            }
        }
    });

    // ---- rows: dbeta, dg, the beta term of dK -----------------------------------------------------------
    float dbr[4] = {0.f, 0.f, 0.f, 0.f}, dgr[4] = {0.f, 0.f, 0.f, 0.f}, dqr[4] = {0.f, 0.f, 0.f, 0.f};
    floatx4 kk[KB];
    const floatx4 bev = ld_f4(reinterpret_cast<const char*>(beta_s + 16 * wave + 4 * g));
#pragma unroll
    for (int ct = 0; ct < KB; ++ct) {
        kk[ct] = kacc(OFF_K, ct);
        const floatx4 qq = kacc(OFF_Q, ct);
        dKr[ct] = dKr[ct] + bev * E2[ct];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dbr[e] += E2[ct][e] * kk[ct][e];
            dqr[e] += dQ[ct][e] * qq[e];
            dgr[e] += (dKr[ct][e] - dKw[ct][e]) * kk[ct][e];
        }
    }
    floatx4 c5, cq;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 16 * wave + 4 * g + e;
        float db = row_sum16(dbr[e]);
        const float dgv = row_sum16(dgr[e]), dqv = row_sum16(dqr[e]);
        db += yx_s[i];
        if (r == 0) { dbeta_s[i] = db; dg_s[i] = rowmask[e] * (dgv + dqv); }
        cq[e] = -dqv * rq_s[i] * rq_s[i];
        c5[e] = (a.opts & kOptGdnBeta) ? 0.f : -2.f * beta_s[i] * db * invden_s[i];   // beta = eta does not depend on k
    }
    __syncthreads();                                 // every wave is done with A o dP and D': they become staging tiles

    // ---- dq, dk: 4x4 transposition inside each quad of lanes, staged rows, 16-byte stores ----------------
    {
        char* sq = lds + OFF_E1;
        char* sk = lds + OFF_DP;
        const bool q_lo = (r & 3) < 2;
        const uint32_t psel = (r & 1) ? 0x03020706u : 0x05040100u;
        auto stage_quad = [&](u32x2 ob, char* dst) { *reinterpret_cast<u32x2*>(dst) = quad_transpose4x4(ob, q_lo, psel); };
        // after the transposition lane (r, g) holds token row 16 wave + 4 g + r % 4, features 32 kp + 8 (r / 4) + 4 b .. + 3
        const int orow = (16 * wave + 4 * g + (r & 3)) * ORQ + 16 * (r >> 2);
#pragma unroll
        for (int ct = 0; ct < KB; ++ct) {
            const int fo = orow + 64 * (ct >> 1) + 8 * (ct & 1);
            if (norm_q) dQ[ct] = dQ[ct] + cq * kacc(OFF_Q, ct);
            stage_quad(to_quad(dQ[ct]), sq + fo);
            stage_quad(to_quad(dKr[ct] + dKw[ct] + c5 * kk[ct]), sk + fo);
        }
        __syncthreads();
        char* qo = reinterpret_cast<char*>(a.dq) + (size_t)tok0 * kq_row + (size_t)h * DK * 2;
        char* ko = reinterpret_cast<char*>(a.dk) + (size_t)tok0 * kq_row + (size_t)h * DK * 2;
#pragma unroll
        for (int it = 0; it < 64 * PPR / 256; ++it) {
            const int i = tid + 256 * it, row = i / PPR, pc = i % PPR;
            if (row < clen) {
                __builtin_nontemporal_store(ld16(sq + row * ORQ + pc * 16), reinterpret_cast<u32x4*>(qo + (size_t)row * kq_row + pc * 16));
                __builtin_nontemporal_store(ld16(sk + row * ORQ + pc * 16), reinterpret_cast<u32x4*>(ko + (size_t)row * kq_row + pc * 16));
            }
        }
    }
    if (wave == 0) {
        const int i = 63 - lane;                         // suffix sums: prefix sums from the last token on
        float x = dg_s[i];
        if (lane == 0) x += eg_s[63] * (red_s[0] + red_s[1] + red_s[2] + red_s[3]) + (red_s[4] + red_s[5] + red_s[6] + red_s[7]);
        x = prefix_sum64(x, lane);
        if (i < clen) {
            a.dlog_alpha[(size_t)(tok0 + i) * a.H + h] = x;
            a.deta[(size_t)(tok0 + i) * a.H + h] = dbeta_s[i] * invden_s[i];
        }
    }
}

hipError_t launch_bwd_assemble_bf16(const BwdArgs<bf16_t>& a, int dk, long n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const dim3 grid((unsigned)(n_chunks * a.H)), block(256);
    if (dk == 64) hipLaunchKernelGGL((bwd_assemble_bf16_kernel<64>), grid, block, 0, st, a);
    else          hipLaunchKernelGGL((bwd_assemble_bf16_kernel<128>), grid, block, 0, st, a);
    return hipGetLastError();
}

template <int DK, int NW, bool REV>
static hipError_t launch_sweep(const BwdArgs<bf16_t>& a, hipStream_t st)
{
    const int n_chains = (a.n_seq > 0 ? a.n_seq : (a.seg_G > 0 ? a.N * a.seg_G : a.N)) * a.H;
    if (n_chains == 0) return hipSuccess;
    const dim3 grid((unsigned)(((n_chains + 7) / 8) * 8 * (a.dv_dim / (16 * NW))));
    hipLaunchKernelGGL((bwd_sweep_bf16_kernel<DK, NW, REV>), grid, dim3(64 * NW + (REV ? 128 : 64)), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_bwd_states_bf16(const BwdArgs<bf16_t>& a, int dk, int waves, hipStream_t st)
{
    switch (waves) {
        case 1: return dk == 64 ? launch_sweep<64, 1, false>(a, st) : launch_sweep<128, 1, false>(a, st);
        case 2: return dk == 64 ? launch_sweep<64, 2, false>(a, st) : launch_sweep<128, 2, false>(a, st);
        case 4: return dk == 64 ? launch_sweep<64, 4, false>(a, st) : launch_sweep<128, 4, false>(a, st);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_bwd_scan_bf16(const BwdArgs<bf16_t>& a, int dk, int waves, hipStream_t st)
{
    switch (waves) {
        case 1: return launch_bwd_rev_bf16(a, dk, st);
        case 2: return dk == 64 ? launch_sweep<64, 2, true>(a, st) : launch_sweep<128, 2, true>(a, st);
        case 4: return dk == 64 ? launch_sweep<64, 4, true>(a, st) : launch_sweep<128, 4, true>(a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kla
