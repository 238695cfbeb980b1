// bf16 inter-chunk stage for batches of at most 256 chains of sixteen state columns, a CU for each: the recurrence of
// kla_chunk_scan_bf16.hip, the same arithmetic in the same order (same bits), with the work of a chunk split by rows.
//
// What bounds it: the latency of a chunk step. With one wave per chain a step is that wave's 480 instructions one after the
// other, and three of four SIMDs have none of them. Here, as in the fp32 scans, four waves ("the chain") share the sixteen columns, one
// per SIMD: wave w owns rows 16 w .. of what is indexed by tokens (K S, X, U) and d_k / 64 feature tiles of the state, and what the
// next product contracts over is exchanged through LDS as operand quads, behind three barriers per step. Four more waves take Q S,
// P U, the outputs and what the backward wants off the chain, a ninth brings K, V and the decay vectors through a ring of five stages,
// a third of a chunk between two barriers (in one piece it kept the others waiting at the first). T', P and Q rows go
// from memory into the registers of the one wave that uses them, three chunks ahead. What is left is the rate at which a CU takes
// its 47 KB per step, 1 KB every 35 .. 40 cycles: steps of 0.8 us. (A form with 32 columns per workgroup, for up to 512 chains, was no
// faster than the column split: 25.1 against 24.8 us for 4 x 700 tokens, 8 heads, d_v = 256.)
// Measured, column split -> this, call with stage 1: 8 heads, d = 128: 200 tokens 13.4 -> 12.3 us, 700 20.3 -> 17.7, 4000 72.8 -> 64.4;
// 4 x 1000 tokens (256 chains) 28.8 -> 26.6; leaving intermediates, 4000 tokens 80.9 -> 73.1.
#include "kla_bf16_ops.hpp"
#include "kla_common.hpp"
#include "kla_kernels.hpp"
#include "kla_mma.hpp"

namespace kla {

namespace {

template <int DK>
struct RowsCfg {
    static constexpr int KP = DK / 32, TW = DK / 64;     // pairs of feature tiles; feature tiles per chain wave
    static constexpr int RB = DK * 2, PPR = DK / 8, RPB = 1024 / RB, NKB = 64 / RPB;         // K rows, copy blocks of a K tile
    static constexpr int VRW = 32, VPP = VRW / 16, RPV = 64 / VPP, NVB = 64 / RPV;           // the same of the V slice
    static constexpr int TPB = kTriPairs * 64 * 16;
    static constexpr int OFF_V = 64 * RB, OFF_VEC = OFF_V + 64 * VRW, STAGE = OFF_VEC + 1024;   // K | V slice | the record's vectors
    static constexpr int NST = 5, NDMA = NKB + NVB + 1;
    // exchange areas: the state in bf16 (two images), X, U, diag(gamma_C/gamma_i) U
    static constexpr int SIMG = KP * 1024, XB = 2048;
    static constexpr int OFF_S = NST * STAGE, OFF_X = OFF_S + 2 * SIMG, OFF_U = OFF_X + XB, OFF_UD = OFF_U + XB, LDS = OFF_UD + XB;
    static_assert(LDS <= 160 * 1024 && (NST - 2) * NDMA < 64, "LDS budget of a gfx950 CU; 6-bit vmcnt");
};

// an address that is the same in every lane, said so to the compiler
__device__ __forceinline__ const char* uniform(const char* p)
{
    const uint64_t x = reinterpret_cast<uintptr_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x), hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return reinterpret_cast<const char*>((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ void mma_slots(floatx4& acc, u32x4 a, u32x4 b) { mma_bf16(acc, a, u32x2{b[0], b[1]}, u32x2{b[2], b[3]}); }

}  // namespace

// SV: the incoming state of every chunk and X stay behind for the backward pass (see ScanArgs)
template <int DK, bool SV>
__global__ __launch_bounds__(576) void scan_rows_bf16_kernel(ScanArgs<bf16_t> a)
{
    typedef RowsCfg<DK> C;
    constexpr int KP = C::KP, TW = C::TW, RB = C::RB, PPR = C::PPR, RPB = C::RPB, VRW = C::VRW, VPP = C::VPP, RPV = C::RPV, NST = C::NST;
    constexpr int PF = 3;                                // chunks a wave's register operands are requested ahead
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), w = wid & 3;
    const int r = lane & 15, g = lane >> 4;

    // ---- workgroup -> (sequence, head, column slice); slices of one head share an XCD (ids congruent mod 8)
    const int nsl = a.dv / 16;
    const int xcd = blockIdx.x & 7, pidx = blockIdx.x >> 3;
    const int rank = (pidx / nsl) * 8 + xcd, slice = pidx % nsl;
    if (rank >= (a.n_seq > 0 ? a.n_seq : a.N) * a.H) return;
    const int h = rank % a.H;
    const int s = a.seq_order ? a.seq_order[rank / a.H] : rank / a.H;
    const int chain = s * a.H + h;
    long t0; int len, ch0;
    if (a.cu_seqlens) { t0 = a.cu_seqlens[s]; len = a.cu_seqlens[s + 1] - (int)t0; ch0 = a.chunk_off[s]; }
    else              { t0 = (long)s * a.T;   len = a.T;                           ch0 = s * a.NT; }
    const int nch = (len + 63) / 64;
    const int col = slice * 16 + r;

    const size_t kq_row = (size_t)a.H * DK * 2, v_row = (size_t)a.H * a.dv * 2;
    // records: T', and P with the vectors behind it
    constexpr int REC = SV ? bwd_record_bytes<bf16_t>() : ws_record_bytes<bf16_t>(), RECP = SV ? pair_record_bytes<bf16_t>() : REC;
    const char* tpbase = reinterpret_cast<const char*>(a.wsT) + ((size_t)ch0 * a.H + h) * REC;
    const char* ppbase = SV ? reinterpret_cast<const char*>(a.wsP) + ((size_t)ch0 * a.H + h) * RECP : tpbase + C::TPB;
    // the slot areas of X, U, Ud: row tile w is half (w & 1) of pair w / 2
    const int own = (w >> 1) * 1024 + lane * 16 + 8 * (w & 1);

    if (wid == 8) {
        // ---- the copy wave: K, the V slice and the decay vectors of the next NST - 1 chunks
        const char* kbase = reinterpret_cast<const char*>(a.k) + (size_t)t0 * kq_row + (size_t)h * DK * 2;
        const char* vbase = reinterpret_cast<const char*>(a.v) + (size_t)t0 * v_row + ((size_t)h * a.dv + slice * 16) * 2;
        const int lrow = lane / PPR, pcol = lane % PPR;
        constexpr int NGK = 8 / RPB;                     // the swizzle of K has period 8 rows
        int gk[NGK];
#pragma unroll
        for (int j = 0; j < NGK; ++j) gk[j] = lrow * (int)kq_row + ((pcol ^ swz_piece<DK>(RPB * j + lrow)) * 16);
        const int gv = (lane / VPP) * (int)v_row + (lane % VPP) * 16;
        // a third of a chunk's copies; rows beyond a short chunk re-read its last one (T' has zeros there)
        auto issue = [&](int c, auto part_c) {
            constexpr int part = decltype(part_c)::value, i0 = part * C::NDMA / 3, i1 = (part + 1) * C::NDMA / 3;
            const int clen = min(64, len - 64 * c);
            char* st = lds + (c % NST) * C::STAGE;
            const char* kc = uniform(kbase + (size_t)(64 * c) * kq_row);
            const char* vc = uniform(vbase + (size_t)(64 * c) * v_row);
            auto blocks = [&](auto whole_c) {
                constexpr bool whole = decltype(whole_c)::value != 0;
                static_for<C::NDMA>([&](auto i) {
                    if constexpr (i >= i0 && i < i1) {
                        if constexpr (i < C::NKB) {
                            const int row = i * RPB + lrow;
                            if constexpr (whole) dma16(kc + (size_t)(i * RPB) * kq_row, gk[i % NGK], st + i * 1024);
                            else                 dma16(kc, min(row, clen - 1) * (int)kq_row + ((pcol ^ swz_piece<DK>(row)) * 16), st + i * 1024);
                        } else if constexpr (i < C::NKB + C::NVB) {
                            constexpr int b = i - C::NKB;
                            if constexpr (whole) dma16(vc + (size_t)(b * RPV) * v_row, gv, st + C::OFF_V + b * 1024);
                            else                 dma16(vc, min(b * RPV + lane / VPP, clen - 1) * (int)v_row + (lane % VPP) * 16, st + C::OFF_V + b * 1024);
                        } else if (lane < 48) dma16(uniform(ppbase + (size_t)c * a.H * RECP + C::TPB), lane * 16, st + C::OFF_VEC);
                    }
                });
            };
            if (clen == 64) blocks(IntC<1>()); else blocks(IntC<0>());
        };
        // all copies but those of the last n chunks issued have landed
        auto landed = [&](int n) { static_for<NST - 1>([&](auto k) { if (n == k) wait_vmcnt<k * C::NDMA>(); }); };
        for (int c = 0; c < min(NST - 1, nch); ++c) static_for<3>([&](auto i) { issue(c, i); });
        landed(max(min(NST - 1, nch) - 2, 0));           // chunks 0 and 1
        __syncthreads();
        for (int c = 0; c < nch; ++c) {
            const bool ahead = c + NST - 1 < nch;        // into the stage that chunk c - 1 left
            if (ahead) issue(c + NST - 1, IntC<0>());
            __syncthreads();
            if (ahead) issue(c + NST - 1, IntC<1>());
            __syncthreads();
            if (ahead) issue(c + NST - 1, IntC<2>());
            landed(max(min(NST - 3, nch - 3 - c), 0));   // chunk c + 2: the chain reads a chunk's K one step early
            __syncthreads();
        }
        return;
    }

    if (wid < 4) {
        // ---- the chain
        const int a4 = r >> 2, c4 = r & 3;
        int oK[KP];
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) oK[kp] = (16 * w + r) * RB + (((4 * kp + g) ^ swz_piece<DK>(r)) * 16);
        const int kpw = DK == 128 ? w : w >> 1;          // this wave's feature tiles are (half of) pair kpw
        const int oKT = (4 * g + a4) * RB + (((4 * kpw + c4) ^ swz_piece<DK>(4 * g + a4)) * 16) + (DK == 128 ? 0 : 8 * (w & 1));
        const int oV = C::OFF_V + (16 * w + 4 * g + a4) * VRW + (c4 >> 1) * 16 + (c4 & 1) * 8;
        const int oG = C::OFF_VEC + 16 * (4 * w + g);
        auto feature = [&](int t, int e) { return 32 * kpw + 8 * g + 4 * (DK == 128 ? t : w & 1) + e; };

        floatx4 S[TW];
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) S[t][e] = a.h0 ? a.h0[((size_t)chain * DK + feature(t, e)) * a.dv + col] : 0.f;
        auto put_state = [&](char* img) {
            char* p = img + kpw * 1024 + lane * 16;
            if constexpr (DK == 128) {
                const u32x2 q0 = to_quad(S[0]), q1 = to_quad(S[TW - 1]);
                st16(p, u32x4{q0.x, q0.y, q1.x, q1.y});
            } else *reinterpret_cast<u32x2*>(p + 8 * (w & 1)) = to_quad(S[0]);
        };
        u32x4 ka[KP];                                    // of the next chunk: K rows 16 w + r, V, gamma
        u32x2 vq;
        floatx4 eg;
        auto fetch = [&](const char* st) {
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) ka[kp] = ld16(st + oK[kp]);
            vq = lds_read_tr(st + oV);
            eg = ld_f4(st + oG);
        };
        // TWO: T' has two tile-pairs in this wave's rows.  (A load behind a condition inside the loop would leave the compiler no
        // choice but to wait for more than it needs; so would a step behind one.)
        auto run = [&](auto two_c) {
            constexpr bool TWO = decltype(two_c)::value != 0;
            struct Regs { u32x4 t[TWO ? 2 : 1]; } R[PF];
            const char* pt = tpbase + tri_pair(w, 0) * 1024 + lane * 16;   // T' of the chunk that is requested next
            int asked = 0;                               // chunks requested (behind the last one, that one again)
            auto load = [&](Regs& x) {
                x.t[0] = ld16(pt);
                if constexpr (TWO) x.t[1] = ld16(pt + 1024);
                pt += ++asked < nch ? (size_t)a.H * REC : 0;
            };
            if (nch > 0) {
                static_for<PF>([&](auto i) { load(R[i]); });
                put_state(lds + C::OFF_S);
            }
            __syncthreads();
            if (nch > 0) fetch(lds);
            int stage = 0;
            auto step = [&](int c, Regs& x, auto more) {
                const char* st = lds + stage * C::STAGE;
                stage = stage + 1 == NST ? 0 : stage + 1;
                const char* img = lds + C::OFF_S + (c & 1) * C::SIMG;
                // ---- X = V - D_gamma K S
                u32x4 sq[KP];
#pragma unroll
                for (int kp = 0; kp < KP; ++kp) sq[kp] = ld16(img + kp * 1024 + lane * 16);
                floatx4 ks = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kp = 0; kp < KP; ++kp) mma_slots(ks, ka[kp], sq[kp]);
                *reinterpret_cast<u32x2*>(lds + C::OFF_X + own) = to_quad(quad_to_f(vq) - eg * ks);
                __syncthreads();
                // ---- U = T' X; K^T of this wave's feature tiles on its way to the state update
                u32x4 xs[2];
                xs[0] = ld16(lds + C::OFF_X + lane * 16);
                if constexpr (TWO) xs[1] = ld16(lds + C::OFF_X + 1024 + lane * 16);
                const floatx4 ed = ld_f4(st + oG + 256);
                const float gC = *reinterpret_cast<const float*>(st + C::OFF_VEC + 252);
                u32x2 kt[TW][2][2];
#pragma unroll
                for (int t = 0; t < TW; ++t)
#pragma unroll
                    for (int jp = 0; jp < 2; ++jp) {
                        const char* p = st + oKT + 32 * jp * RB + 8 * t;
                        kt[t][jp][0] = lds_read_tr(p);
                        kt[t][jp][1] = lds_read_tr(p + 16 * RB);
                    }
                floatx4 u = {0.f, 0.f, 0.f, 0.f};
                mma_slots(u, x.t[0], xs[0]);
                if constexpr (TWO) mma_slots(u, x.t[1], xs[1]);
                *reinterpret_cast<u32x2*>(lds + C::OFF_UD + own) = to_quad(u * ed);
                *reinterpret_cast<u32x2*>(lds + C::OFF_U + own) = to_quad(u);
#pragma unroll
                for (int t = 0; t < TW; ++t) S[t] = S[t] * gC;
                __syncthreads();
                // ---- S = gamma_C S + K^T (diag(gamma_C/gamma_i) U)
                u32x4 ud[2];
#pragma unroll
                for (int jp = 0; jp < 2; ++jp) ud[jp] = ld16(lds + C::OFF_UD + jp * 1024 + lane * 16);
                fetch(lds + stage * C::STAGE);           // (behind the last chunk: what the ring happens to hold, not used)
#pragma unroll
                for (int jp = 0; jp < 2; ++jp)
#pragma unroll
                    for (int t = 0; t < TW; ++t) mma_bf16(S[t], kt[t][jp][0], kt[t][jp][1], u32x2{ud[jp][0], ud[jp][1]}, u32x2{ud[jp][2], ud[jp][3]});
                if constexpr (decltype(more)::value) load(x);
                put_state(lds + C::OFF_S + ((c + 1) & 1) * C::SIMG);
                __syncthreads();
            };
            int c = 0;
            for (; c + PF <= nch; c += PF) static_for<PF>([&](auto i) { step(c + i, R[i], IntC<1>()); });
            static_for<PF - 1>([&](auto i) { if (c + i < nch) step(c + i, R[i], IntC<0>()); });
        };
        if (w >= 2) run(IntC<1>()); else run(IntC<0>());

        if (a.hT) {
#pragma unroll
            for (int t = 0; t < TW; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) a.hT[((size_t)chain * DK + feature(t, e)) * a.dv + col] = S[t][e];
        }
        return;
    }

    // ---- off the chain: O = D_gamma Q S + P U, rows 16 w ..; SV: what the backward needs
    const char* qbase = reinterpret_cast<const char*>(a.q) + (size_t)t0 * kq_row + (size_t)h * DK * 2 + 16 * g;
    char* obase = reinterpret_cast<char*>(a.o) + (size_t)t0 * v_row + ((size_t)h * a.dv + slice * 16) * 2 + 8 * (r >> 2);
    const bool q_lo = (r & 3) < 2;
    const uint32_t psel = (r & 1) ? 0x03020706u : 0x05040100u;
    auto run = [&](auto two_c) {
        constexpr bool TWO = decltype(two_c)::value != 0;
        struct Regs { u32x4 q[KP], p[TWO ? 2 : 1]; } R[PF];
        const char* pp = ppbase + tri_pair(w, 0) * 1024 + lane * 16;      // P of the chunk that is requested next
        int asked = 0, stage = 0;
        auto load_q = [&](Regs& x, int c) {
            const char* q = qbase + (size_t)min(64 * c + 16 * w + r, len - 1) * kq_row;
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) x.q[kp] = ld16(q + 64 * kp);
        };
        auto load_p = [&](Regs& x) {
            x.p[0] = ld16(pp);
            if constexpr (TWO) x.p[1] = ld16(pp + 1024);
            pp += ++asked < nch ? (size_t)a.H * RECP : 0;
        };
        floatx4 o;
        auto put_out = [&](int c) {
            const int row = 64 * c + 16 * w + 4 * g + (r & 3);
            const u32x2 y = quad_transpose4x4(to_quad(o), q_lo, psel);
            if (row < len) *reinterpret_cast<u32x2*>(obase + (size_t)row * v_row) = y;
        };
        if (nch > 0) static_for<PF>([&](auto i) { load_q(R[i], i); load_p(R[i]); });
        __syncthreads();
        auto step = [&](int c, Regs& x, auto more) {
            const char* img = lds + C::OFF_S + (c & 1) * C::SIMG;
            // ---- before the chain's first barrier: the outputs of the chunk before, Q S of this one
            u32x4 sq[KP];
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) sq[kp] = ld16(img + kp * 1024 + lane * 16);
            const floatx4 eq = ld_f4(lds + stage * C::STAGE + C::OFF_VEC + 512 + 16 * (4 * w + g));   // gamma_i / ||q_i||, or gamma_i
            stage = stage + 1 == NST ? 0 : stage + 1;
            if (c > 0) put_out(c - 1);
            o = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) mma_slots(o, x.q[kp], sq[kp]);
            __syncthreads();
            if constexpr (SV) {
                const int clen = min(64, len - 64 * c);
                char* xc = reinterpret_cast<char*>(a.X) + (size_t)(t0 + 64L * c) * v_row;
                if (w < KP)                              // put_checkpoint, a wave per 1 KiB block
                    __builtin_nontemporal_store(ld16(img + w * 1024 + lane * 16),
                                                reinterpret_cast<u32x4*>(reinterpret_cast<char*>(a.s_chk) + (((size_t)(ch0 + c) * a.H + h) * a.dv + slice * 16) * RB + w * 1024 + r * 64 + g * 16));
                if (clen == 64) {                        // put_rows, a wave per 1 KiB block
                    if (w < 2)
                        __builtin_nontemporal_store(ld16(lds + C::OFF_X + w * 1024 + lane * 16),
                                                    reinterpret_cast<u32x4*>(xc + (size_t)h * a.dv * 128 + slice * 2048 + w * 1024 + lane * 16));
                } else {
                    int r1 = r, g1 = g;
                    asm volatile("" : "+v"(r1), "+v"(g1));   // nothing of this path is kept in registers
                    const u32x2 xq = *reinterpret_cast<const u32x2*>(lds + C::OFF_X + own);
                    char* p = xc + ((size_t)h * a.dv + slice * 16 + r1) * 2;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int row = 16 * w + 4 * g1 + e;
                        const uint32_t v = e < 2 ? xq.x : xq.y;
                        if (row < clen) *reinterpret_cast<uint16_t*>(p + (size_t)row * v_row) = (uint16_t)((e & 1) ? v >> 16 : v & 0xffffu);
                    }
                }
            }
            o = eq * o;
            if constexpr (decltype(more)::value) load_q(x, min(c + PF, nch - 1));
            __syncthreads();
            // ---- + P U
            u32x4 us[2];
            us[0] = ld16(lds + C::OFF_U + lane * 16);
            if constexpr (TWO) us[1] = ld16(lds + C::OFF_U + 1024 + lane * 16);
            mma_slots(o, x.p[0], us[0]);
            if constexpr (TWO) mma_slots(o, x.p[1], us[1]);
            if constexpr (decltype(more)::value) load_p(x);
            __syncthreads();
        };
        int c = 0;
        for (; c + PF <= nch; c += PF) static_for<PF>([&](auto i) { step(c + i, R[i], IntC<1>()); });
        static_for<PF - 1>([&](auto i) { if (c + i < nch) step(c + i, R[i], IntC<0>()); });
        if (nch > 0) put_out(nch - 1);
    };
    if (w >= 2) run(IntC<1>()); else run(IntC<0>());
}

template <int DK>
static hipError_t launch_dk(const ScanArgs<bf16_t>& a, hipStream_t st)
{
    const int n_chains = (a.n_seq > 0 ? a.n_seq : a.N) * a.H;
    if (n_chains == 0) return hipSuccess;
    const dim3 grid((unsigned)(((n_chains + 7) / 8) * 8 * (a.dv / 16))), block(576);
    if (a.s_chk) hipLaunchKernelGGL((scan_rows_bf16_kernel<DK, true>), grid, block, 0, st, a);
    else         hipLaunchKernelGGL((scan_rows_bf16_kernel<DK, false>), grid, block, 0, st, a);
    return hipGetLastError();
}
hipError_t launch_scan_rows_bf16(const ScanArgs<bf16_t>& a, int dk, hipStream_t st)
{
    if (a.seg_G > 0 || a.kt_src) return hipErrorInvalidValue;
    return dk == 64 ? launch_dk<64>(a, st) : launch_dk<128>(a, st);
}

}  // namespace kla
