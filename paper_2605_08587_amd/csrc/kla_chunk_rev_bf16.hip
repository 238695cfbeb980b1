// bf16 reverse state sweep of the backward pass for batches of at most 256 chains of sixteen state columns, a CU for each, and packed ones
// whose further chains are so short that they fit behind the others (kla_widths.hpp; kla_chunk_bwd.hip has the algebra,
// kla_chunk_bwd_bf16.hip the reverse sweep of two and four chains per workgroup):
//
//     dU = P^T dO + diag(gamma_C/gamma_i) K dS',   Y = M^T dU,   dV = B Y,
//     dS <- gamma_C dS' + Q^T D_gamma dO - K^T D_gamma dV;      leaves dS'_c, Y, dV and finally dh0.
//
// What bounds it: the instructions of the wave that carries dS', one visit of a chunk after the other, with three SIMDs idle. Two of
// a visit's five products, P^T dO and Q^T D_gamma dO, do not depend on dS', so a second wave, on a SIMD of its own, forms them one
// visit ahead (fp32, handed over through LDS in accumulator order: they enter the chain as the addends of multiply-adds it
// has anyway), and the wave that stores rows takes Y in fp32 and the checkpoint from the chain and does the scaling by beta, the
// roundings and the transposition. The chain keeps K dS', Y and K^T D_gamma dV: a visit is 1.2 us instead of 1.5.
// LDS: ring A, three stages (K, M^T, the vectors), feeds the chain; ring B, two stages (Q, P^T, the dO slice, the vectors), its helper.
// The order of the sums is that of the wider sweeps, so the bits do not depend on the batch that a sequence comes in.
// A second barrier in the visit, passed as soon as the chain and the store wave have read what they were handed, lets each of the
// hand-over areas exist once.
// Measured, one wave per chain -> this, 8 heads, d = 128: 3000 tokens 70 -> 57 us; 2 x 700 22.8 -> 18.6; 3 x 2000 (192 chains)
// 50 -> 44; 4 x 2000 (256) 51 -> 50, where the 56 KB that a CU takes and gives per visit are what is left. With two chains per workgroup
// it gains nothing for the same reason: 5, 6, 7, 8 x 2000 tokens 55, 58, 63, 66 us against 55, 58, 62, 63.
#include "kla_bf16_ops.hpp"
#include "kla_common.hpp"
#include "kla_kernels.hpp"
#include "kla_mma.hpp"

namespace kla {

namespace {

template <int DK>
struct RevCfg {
    static constexpr int KB = DK / 16, KP = DK / 32;
    static constexpr int RB = DK * 2, PPR = DK / 8, RPB = 1024 / RB, NKB = 64 / RPB;         // K / Q rows, 16-byte pieces, copy blocks
    static constexpr int VRW = 32, VPP = VRW / 16, RPV = 64 / VPP, NVB = 64 / RPV;      // the same of the dO slice
    static constexpr int TPB = kTriPairs * 64 * 16;
    // ring A: K | M^T | gamma_i | gamma_C/gamma_i | beta_i | 1/||q_i||; ring B: Q | P^T | dO slice | the same vectors
    static constexpr int OFF_M = 64 * RB, A_VEC = OFF_M + TPB, STA = A_VEC + 1024, NSA = 3;
    static constexpr int OFF_P = 64 * RB, OFF_V = OFF_P + TPB, B_VEC = OFF_V + 64 * VRW, STB = B_VEC + 1024, NSB = 2;
    static constexpr int N_A = NKB + TPB / 1024 + 1, N_B = NKB + TPB / 1024 + NVB + 1;        // copies of a chunk
    // hand-over areas: P^T dO (4 tiles of 1 KiB), Q^T D_gamma dO (KB); Y (4), the checkpoint (KP)
    static constexpr int HB = (4 + KB) * 1024, YB = (4 + KP) * 1024;
    static constexpr int OFF_B = NSA * STA, OFF_H = OFF_B + NSB * STB, OFF_Y = OFF_H + HB, LDS = OFF_Y + YB;
    static constexpr int W_HELP = 1, W_COPY = 2, W_STORE = 3, NWAVES = 4;
    static_assert(LDS <= 160 * 1024 && N_A + N_B < 64, "LDS budget of a gfx950 CU; 6-bit vmcnt");
};

}  // namespace

template <int DK>
__global__ __launch_bounds__((64 * RevCfg<DK>::NWAVES)) void bwd_rev_bf16_kernel(BwdArgs<bf16_t> a)
{
    typedef RevCfg<DK> C;
    constexpr int KB = C::KB, KP = C::KP, RB = C::RB, PPR = C::PPR, RPB = C::RPB, VRW = C::VRW, VPP = C::VPP, RPV = C::RPV;
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    // ---- workgroup -> (sequence, head, column slice), as in the forward sweep
    const int nsl = a.dv_dim / 16;
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
    const bool store = (a.opts & kOptNoStore) == 0;      // off: only the state gradient is carried (segment pre-pass)
    const int nch = (len + 63) / 64;

    const size_t kq_row = (size_t)a.H * DK * 2, v_row = (size_t)a.H * a.dv_dim * 2;     // bytes between tokens
    auto chunk_of = [&](int i) { return nch - 1 - i; };  // visit i
    const int a4 = r >> 2, c4 = r & 3;
    // K^T / Q^T slots through the transposing read (see kla_chunk_scan_bf16.hip)
    int oKT[KP];
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) oKT[kp] = (4 * g + a4) * RB + (((4 * kp + c4) ^ swz_piece<DK>(4 * g + a4)) * 16);
    auto ktslot = [&](int kt, int jp, const char* tile, u32x2& q0, u32x2& q1) {
        const int kp = kt >> 1, b = kt & 1;
        const char* p = tile + oKT[kp] + 32 * jp * RB + 8 * b;
        q0 = lds_read_tr(p);
        q1 = lds_read_tr(p + 16 * RB);
    };

    // Every wave passes two barriers before the first visit and two in each: "mid" (what the visit before handed over has been
    // read) and the one that ends the visit.
    if (wave == C::W_COPY) {
        // ---- the copy wave.  Visit i brings ring B of visit i + 2 into the stage that the helpers left at the end of visit
        // i - 1, and ring A of visit i + 2 into the one that the chains left then.
        const char* kbase = reinterpret_cast<const char*>(a.k) + (size_t)t0 * kq_row + (size_t)h * DK * 2;
        const char* qbase = reinterpret_cast<const char*>(a.q) + (size_t)t0 * kq_row + (size_t)h * DK * 2;
        const char* vbase = reinterpret_cast<const char*>(a.d_o) + (size_t)t0 * v_row + ((size_t)h * a.dv_dim + slice * 16) * 2;
        constexpr int REC = bwd_record_bytes<bf16_t>();
        const char* rbase = a.rec + ((size_t)ch0 * a.H + h) * REC;
        const int lrow = lane / PPR, pcol = lane % PPR;
        constexpr int NGK = 8 / RPB;                     // the swizzle has period 8 rows
        int gk[NGK];
#pragma unroll
        for (int j = 0; j < NGK; ++j) gk[j] = lrow * (int)kq_row + ((pcol ^ swz_piece<DK>(RPB * j + lrow)) * 16);
        const int gv = (lane / VPP) * (int)v_row + (lane % VPP) * 16;
        auto tile = [&](const char* src, int clen, char* dst) {         // a [64 x d_k] tile; rows past a ragged end re-read the last one
            if (clen == 64)
                static_for<C::NKB>([&](auto i) { const int b = i; dma16(src + (size_t)(b * RPB) * kq_row, gk[b % NGK], dst + b * 1024); });
            else
                static_for<C::NKB>([&](auto i) {
                    const int b = i, row = b * RPB + lrow;
                    dma16(src, min(row, clen - 1) * (int)kq_row + ((pcol ^ swz_piece<DK>(row)) * 16), dst + b * 1024);
                });
        };
        auto vectors = [&](const char* rec, char* dst) { dma16(rec + 3 * C::TPB, lane < 48 ? lane * 16 : 1024 + (lane - 48) * 16, dst); };
        auto issue_a = [&](int i) {
            const int c = chunk_of(i);
            char* st = lds + (i % C::NSA) * C::STA;
            const char* rec = rbase + (size_t)c * a.H * REC;
            tile(kbase + (size_t)(64 * c) * kq_row, min(64, len - 64 * c), st);
            static_for<C::TPB / 1024>([&](auto j) { const int b = j; dma16(rec + C::TPB + b * 1024, lane * 16, st + C::OFF_M + b * 1024); });
            vectors(rec, st + C::A_VEC);
        };
        auto issue_b = [&](int i) {
            const int c = chunk_of(i), clen = min(64, len - 64 * c);
            char* st = lds + C::OFF_B + (i % C::NSB) * C::STB;
            const char* rec = rbase + (size_t)c * a.H * REC;
            tile(qbase + (size_t)(64 * c) * kq_row, clen, st);
            static_for<C::TPB / 1024>([&](auto j) { const int b = j; dma16(rec + 2 * C::TPB + b * 1024, lane * 16, st + C::OFF_P + b * 1024); });
            const char* vc = vbase + (size_t)(64 * c) * v_row;
            if (clen == 64)
                static_for<C::NVB>([&](auto j) { const int b = j; dma16(vc + (size_t)(b * RPV) * v_row, gv, st + C::OFF_V + b * 1024); });
            else
                static_for<C::NVB>([&](auto j) {
                    const int b = j;
                    dma16(vc, min(b * RPV + lane / VPP, clen - 1) * (int)v_row + (lane % VPP) * 16, st + C::OFF_V + b * 1024);
                });
            vectors(rec, st + C::B_VEC);
        };
        // Copies retire in order: a wait for all but the last n
        if (nch > 0) { issue_b(0); issue_a(0); }
        if (nch > 1) { issue_b(1); wait_vmcnt<C::N_A + C::N_B>(); } else if (nch > 0) wait_vmcnt<C::N_A>();
        __syncthreads();                                 // ring B of visit 0 is there
        if (nch > 1) { issue_a(1); wait_vmcnt<C::N_A>(); } else wait_vmcnt<0>();
        __syncthreads();                                 // ring A of visit 0, ring B of visit 1
        for (int i = 0; i < nch; ++i) {
            __syncthreads();                             // mid
            if (i + 2 < nch) { issue_b(i + 2); issue_a(i + 2); wait_vmcnt<C::N_A>(); } else wait_vmcnt<0>();
            __syncthreads();
        }
        return;
    }

    if (wave == C::W_STORE) {
        // ---- the store wave: in visit i the checkpoint, Y and dV of visit i - 1
        const bool q_lo = (r & 3) < 2;
        const uint32_t psel = (r & 1) ? 0x03020706u : 0x05040100u;
        floatx4 y[4], be[4];
        u32x4 chk[KP];
        auto take = [&](int i) {                         // of visit i: before the stage of ring A and the areas are written again
            const char* st = lds + (i % C::NSA) * C::STA;
#pragma unroll
            for (int it = 0; it < 4; ++it) be[it] = ld_f4(st + C::A_VEC + 512 + 64 * it + 16 * g);
            const char* p = lds + C::OFF_Y + lane * 16;
#pragma unroll
            for (int it = 0; it < 4; ++it) y[it] = ld_f4(p + it * 1024);
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) chk[kp] = ld16(p + (4 + kp) * 1024);
        };
        auto put = [&](int i) {
            const int c = chunk_of(i), clen = min(64, len - 64 * c);
            char* cp = reinterpret_cast<char*>(a.ds_chk) + ((size_t)(ch0 + c) * a.H + h) * a.dv_dim * RB + slice * (16 * RB);
#pragma unroll
            for (int kp = 0; kp < KP; ++kp)              // put_checkpoint's order
                __builtin_nontemporal_store(chk[kp], reinterpret_cast<u32x4*>(cp + kp * 1024 + r * 64 + g * 16));
            u32x2 yq[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) yq[it] = to_quad(y[it]);
            put_rows(reinterpret_cast<char*>(a.Y) + (size_t)(t0 + 64L * c) * v_row, v_row, a.dv_dim, h, slice, yq, clen, r, g);
            // dV = B Y.  After the transposition lane (r, g) has row 4 g + r % 4 (+ 16 it), columns 4 (r / 4) .. + 3
            char* o = reinterpret_cast<char*>(a.dv) + (size_t)(t0 + 64L * c) * v_row + ((size_t)h * a.dv_dim + slice * 16) * 2;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int row = 16 * it + 4 * g + (r & 3);
                const u32x2 d = quad_transpose4x4(to_quad(y[it] * be[it]), q_lo, psel);
                if (row < clen) __builtin_nontemporal_store(d, reinterpret_cast<u32x2*>(o + (size_t)row * v_row + 8 * (r >> 2)));
            }
        };
        __syncthreads();
        __syncthreads();
        for (int i = 0; i < nch; ++i) {
            if (i > 0) take(i - 1);
            __syncthreads();                             // mid
            if (i > 0 && store) put(i - 1);
            __syncthreads();
        }
        if (nch > 0 && store) { take(nch - 1); put(nch - 1); }
        return;
    }

    if (wave == C::W_HELP) {
        // ---- the helper: P^T dO and Q^T D_gamma dO of the visit ahead
        const int oV = C::OFF_V + (4 * g + a4) * VRW + (c4 >> 1) * 16 + (c4 & 1) * 8;
        char* hand = lds + C::OFF_H + lane * 16;
        auto step = [&](int i) {
            const int clen = min(64, len - 64 * chunk_of(i));
            const char* st = lds + C::OFF_B + (i % C::NSB) * C::STB;
            floatx4 hu[4], hs[KB];
            u32x2 vq[4], gd[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                vq[it] = lds_read_tr(st + oV + 16 * it * VRW);
                hu[it] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            u32x4 psl[kTriPairs];
#pragma unroll
            for (int j = 0; j < kTriPairs; ++j) psl[j] = ld16(st + C::OFF_P + j * 1024 + lane * 16);
            u32x2 kt[2][KB][2];
#pragma unroll
            for (int jp = 0; jp < 2; ++jp)
#pragma unroll
                for (int t = 0; t < KB; ++t) ktslot(t, jp, st, kt[jp][t][0], kt[jp][t][1]);
#pragma unroll
            for (int it = 0; it < 4; ++it) {             // D_gamma dO / ||q||; rows past a ragged end have no part in Q^T D_gamma dO
                floatx4 eg = ld_f4(st + C::B_VEC + 64 * it + 16 * g) * ld_f4(st + C::B_VEC + 768 + 64 * it + 16 * g);
                if (clen < 64) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) eg[e] = (16 * it + 4 * g + e < clen) ? eg[e] : 0.f;
                }
                gd[it] = to_quad(eg * quad_to_f(vq[it]));
            }
            mma_bf16(hu[0], psl[triu_pair(0, 0)], vq[0], vq[1]);      // P^T is upper triangular
            mma_bf16(hu[1], psl[triu_pair(1, 0)], vq[0], vq[1]);
#pragma unroll
            for (int t = 0; t < KB; ++t) { hs[t] = floatx4{0.f, 0.f, 0.f, 0.f}; mma_bf16(hs[t], kt[0][t][0], kt[0][t][1], gd[0], gd[1]); }
#pragma unroll
            for (int it = 0; it < 4; ++it) mma_bf16(hu[it], psl[triu_pair(it, 1)], vq[2], vq[3]);
#pragma unroll
            for (int t = 0; t < KB; ++t) mma_bf16(hs[t], kt[1][t][0], kt[1][t][1], gd[2], gd[3]);
#pragma unroll
            for (int it = 0; it < 4; ++it) *reinterpret_cast<floatx4*>(hand + it * 1024) = hu[it];
#pragma unroll
            for (int t = 0; t < KB; ++t) *reinterpret_cast<floatx4*>(hand + (4 + t) * 1024) = hs[t];
        };
        __syncthreads();
        if (nch > 0) step(0);
        __syncthreads();
        for (int i = 0; i < nch; ++i) {
            __syncthreads();                             // mid: the chain has read what it was handed
            if (i + 1 < nch) step(i + 1);
            __syncthreads();
        }
        return;
    }

    // ---- the chain: dS' of sixteen columns; element e of lane (r, g) of tile kt = 2 kp + b is feature 32 kp + 8 g + 4 b + e
    const int col = slice * 16 + r;
    floatx4 S[KB];
#pragma unroll
    for (int kt = 0; kt < KB; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int f = 32 * (kt >> 1) + 8 * g + 4 * (kt & 1) + e;
            S[kt][e] = a.d_hT ? a.d_hT[((size_t)chain * DK + f) * a.dv_dim + col] : 0.f;
        }
    int oK[KP];
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) oK[kp] = r * RB + (((4 * kp + g) ^ swz_piece<DK>(r)) * 16);
    const char* hand = lds + C::OFF_H + lane * 16;
    char* yarea = lds + C::OFF_Y + lane * 16;
    __syncthreads();
    __syncthreads();
    int stage = 0;
    for (int i = 0; i < nch; ++i) {
        const int clen = min(64, len - 64 * chunk_of(i));
        const char* st = lds + stage * C::STA;
        stage = stage + 1 == C::NSA ? 0 : stage + 1;
        const char* pG = st + C::A_VEC + 16 * g;
        floatx4 hu[4], hs[KB];
#pragma unroll
        for (int t = 0; t < KB; ++t) hs[t] = ld_f4(hand + (4 + t) * 1024);
#pragma unroll
        for (int it = 0; it < 4; ++it) hu[it] = ld_f4(hand + it * 1024);
        const float gC = *reinterpret_cast<const float*>(st + C::A_VEC + 63 * 4);
        u32x2 Sq[KB];
#pragma unroll
        for (int kt = 0; kt < KB; ++kt) Sq[kt] = to_quad(S[kt]);
        // ---- K dS'
        floatx4 ks[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) ks[it] = floatx4{0.f, 0.f, 0.f, 0.f};
        u32x4 ka[2][4];
#pragma unroll
        for (int it = 0; it < 4; ++it) ka[0][it] = ld16(st + oK[0] + 16 * it * RB);
#pragma unroll
        for (int kt = 0; kt < KB; ++kt) S[kt] = S[kt] * gC + hs[kt];
        __syncthreads();                                 // mid
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) {
            if (kp + 1 < KP) {
#pragma unroll
                for (int it = 0; it < 4; ++it) ka[(kp + 1) & 1][it] = ld16(st + oK[kp + 1] + 16 * it * RB);
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) mma_bf16(ks[it], ka[kp & 1][it], Sq[2 * kp], Sq[2 * kp + 1]);
        }
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) st16(yarea + (4 + kp) * 1024, u32x4{Sq[2 * kp].x, Sq[2 * kp].y, Sq[2 * kp + 1].x, Sq[2 * kp + 1].y});
        u32x4 tsl[kTriPairs];
#pragma unroll
        for (int j = 0; j < kTriPairs; ++j) tsl[j] = ld16(st + C::OFF_M + j * 1024 + lane * 16);
        floatx4 edv[4], egv[4], bev[4];                  // gamma_C/gamma_i; gamma_i, zero past a ragged end; beta_i
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            edv[it] = ld_f4(pG + 256 + 64 * it);
            egv[it] = ld_f4(pG + 64 * it);
            bev[it] = ld_f4(pG + 512 + 64 * it);
            if (clen < 64) {
#pragma unroll
                for (int e = 0; e < 4; ++e) egv[it][e] = (16 * it + 4 * g + e < clen) ? egv[it][e] : 0.f;
            }
        }
        // ---- dU = diag(gamma_C/gamma_i) K dS' + P^T dO
        u32x2 dUq[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) dUq[it] = to_quad(edv[it] * ks[it] + hu[it]);
        u32x2 kt[2][KB][2];                              // K^T slots [token pair jp][state tile][token block]
#pragma unroll
        for (int t = 0; t < KB; ++t) ktslot(t, 0, st, kt[0][t][0], kt[0][t][1]);
        // ---- Y = M^T dU (upper triangular)
        floatx4 Y[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) Y[it] = floatx4{0.f, 0.f, 0.f, 0.f};
        mma_bf16(Y[0], tsl[triu_pair(0, 0)], dUq[0], dUq[1]);
        mma_bf16(Y[1], tsl[triu_pair(1, 0)], dUq[0], dUq[1]);
#pragma unroll
        for (int it = 0; it < 4; ++it) mma_bf16(Y[it], tsl[triu_pair(it, 1)], dUq[2], dUq[3]);
#pragma unroll
        for (int t = 0; t < KB; ++t) ktslot(t, 1, st, kt[1][t][0], kt[1][t][1]);
        // ---- dS = gamma_C dS' + Q^T D_gamma dO - K^T D_gamma dV
        u32x2 gdXq[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) gdXq[it] = to_quad(-(egv[it] * (Y[it] * bev[it])));
#pragma unroll
        for (int t = 0; t < KB; ++t) mma_bf16(S[t], kt[0][t][0], kt[0][t][1], gdXq[0], gdXq[1]);
#pragma unroll
        for (int it = 0; it < 4; ++it) *reinterpret_cast<floatx4*>(yarea + it * 1024) = Y[it];
#pragma unroll
        for (int t = 0; t < KB; ++t) mma_bf16(S[t], kt[1][t][0], kt[1][t][1], gdXq[2], gdXq[3]);
        __syncthreads();
    }
    if (a.dh0) {
#pragma unroll
        for (int kt = 0; kt < KB; ++kt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int f = 32 * (kt >> 1) + 8 * g + 4 * (kt & 1) + e;
                a.dh0[((size_t)chain * DK + f) * a.dv_dim + col] = S[kt][e];
            }
    }
}

template <int DK>
static hipError_t launch_dk(const BwdArgs<bf16_t>& a, hipStream_t st)
{
    const int n_chains = (a.n_seq > 0 ? a.n_seq : (a.seg_G > 0 ? a.N * a.seg_G : a.N)) * a.H;
    if (n_chains == 0) return hipSuccess;
    const dim3 grid((unsigned)(((n_chains + 7) / 8) * 8 * (a.dv_dim / 16)));
    hipLaunchKernelGGL((bwd_rev_bf16_kernel<DK>), grid, dim3(64 * RevCfg<DK>::NWAVES), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_bwd_rev_bf16(const BwdArgs<bf16_t>& a, int dk, hipStream_t st) { return dk == 64 ? launch_dk<64>(a, st) : launch_dk<128>(a, st); }

}  // namespace kla
