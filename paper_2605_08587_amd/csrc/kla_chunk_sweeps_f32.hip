// fp32 chunk sweeps: the forward recurrence (outputs and final state) and the two sweeps of the backward pass for
// single-precision inputs, all products on v_mfma_f32_16x16x4_f32.  The algebra is that of kla_chunk_scan.hip and
// kla_chunk_bwd.hip; what differs is the split of the work.
//
// What bounds them: the matrix pipe.  A chunk of 64 tokens and 16 state columns takes 480 fp32 MFMAs at d_k = 128, each
// 32 cycles of one SIMD: 6.4 us if one wave does them all, and there are few such chains (256 for 4 sequences of 8
// heads of 128 columns), so a wave per chain leaves three of four SIMDs without work for the whole call.  Here FOUR
// waves share a chain, one per SIMD, and split every product of a chunk by its output rows:
//     token-shaped results (K S, X, U, Q S, P U; K dS', dU, Y): wave w owns the rows 16 w .. 16 w + 15
//     state-shaped results (S, dS)                            : wave w owns d_k / 64 of the 16-row feature tiles
// so each accumulator exists once, and what the next product contracts over (S, X, U; dS, dU, dX) is exchanged through
// LDS as operand quads (kla_mma.hpp): one conflict-free 16-byte write and read per lane and tile.  A workgroup takes
// NC = 1 or 2 column tiles; two halve the LDS reads per product and are used once there are more tiles than CUs.  The
// forward has a form with four more waves (scan_f32_split_kernel) for batches that leave a workgroup a CU of its own.
//
// Operands.  K (and Q where it is contracted over the tokens) is needed row- and column-wise: it sits in LDS as plain
// token rows whose 16-byte pieces are XORed with the row index mod 16, which makes the 128-bit row reads and the 32-bit
// column reads free of bank conflicts, so no transposed copy exists.  Everything that only one wave needs - its rows of
// Q, its tile-pairs of T', P, M^T, P^T, its rows of V - goes from global memory straight into the registers of the
// product that uses it, and is requested again for the next chunk as soon as that product has been issued.
//
// No load is conditional.  The vector-memory counter retires in order, and behind a branch that may or may not have
// issued a load the compiler can only wait for everything; with conditional loads a step waited for its own prefetches.
// So rows beyond a short last chunk repeat its last row - their rows and columns of T' and P are zero (beta = 0 there),
// so they reach no result; in the reverse sweep dO is zeroed there - and behind the last chunk that chunk is read again.
//
// Measured, one wave per chain -> this file: forward of 4 sequences of 2000 tokens, 8 heads, d = 128 (256 column tiles):
// 590 -> 118 us, 3.7 us per chunk against 1.7 us of MFMA per wave (143 us with conditional loads; 100 us with eight waves); 2 sequences of 500
// tokens, 4 heads, d = 64 (32 tiles): forward 71 -> 20 us, forward sweep 53 -> 17 us, reverse sweep 124 -> 28 us.
#include "kla_common.hpp"
#include "kla_f32_ops.hpp"
#include "kla_kernels.hpp"

namespace kla {

namespace {

// The (at most two) tile-pairs of one row tile of a triangular operand, in registers.
struct TriRegs { float4 q[2][2]; };
__device__ __forceinline__ void load_tri(TriRegs& t, const char* area, int wave, int lane)       // lower triangular: pairs 0 .. wave / 2
{
    const char* p = area + ((size_t)tri_pair(wave, 0) * 64 + lane) * 32;
    const char* p1 = p + (wave >= 2 ? 2048 : 0);         // one pair only: loaded twice, the second copy is not used
    t.q[0][0] = ldf4(p); t.q[0][1] = ldf4(p + 16);
    t.q[1][0] = ldf4(p1); t.q[1][1] = ldf4(p1 + 16);
}
__device__ __forceinline__ void load_triu(TriRegs& t, const char* area, int wave, int lane)      // upper triangular: pairs wave / 2 .. 1
{
    const char* p = area + ((size_t)triu_pair(wave, 1) * 64 + lane) * 32;
    const char* p0 = p - (wave < 2 ? 2048 : 0);
    t.q[1][0] = ldf4(p); t.q[1][1] = ldf4(p + 16);
    t.q[0][0] = ldf4(p0); t.q[0][1] = ldf4(p0 + 16);
}
// acc += (row tile of the operand) x (token-shaped matrix exchanged at x: tile jt of this lane at x + 1024 jt + 16 lane)
__device__ __forceinline__ void mma_tri(floatx4& acc, const TriRegs& t, const char* x, int wave, int lane)
{
    const char* p = x + 16 * lane;
    mma32(acc, t.q[0][0], t.q[0][1], ldf4(p), ldf4(p + 1024));
    if (wave >= 2) mma32(acc, t.q[1][0], t.q[1][1], ldf4(p + 2048), ldf4(p + 3072));
}
__device__ __forceinline__ void mma_triu(floatx4& acc, const TriRegs& t, const char* x, int wave, int lane)
{
    const char* p = x + 16 * lane;
    if (wave < 2) mma32(acc, t.q[0][0], t.q[0][1], ldf4(p), ldf4(p + 1024));
    mma32(acc, t.q[1][0], t.q[1][1], ldf4(p + 2048), ldf4(p + 3072));
}

// rows 16 wave + 4 g + e, one column, of a [tokens, H, d_v] tensor (p: chunk's first row at that column) <-> registers
__device__ __forceinline__ floatx4 load_col(const float* p, size_t stride, int row0, int clen)
{
    floatx4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = p[(size_t)min(row0 + e, clen - 1) * stride];
    return x;
}
__device__ __forceinline__ void store_col(float* p, size_t stride, int row0, int clen, floatx4 x)
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (row0 + e < clen) p[(size_t)(row0 + e) * stride] = x[e];
}

// workgroup -> (sequence, head, column slice): slices of one (sequence, head) get ids congruent mod 8 and share an XCD's L2
struct Pos { int chain, h, slice, nch, ch0, len; long t0; bool valid; };
template <typename A> __device__ __forceinline__ Pos sweep_pos(const A& a, int dv, int slw)
{
    Pos p;
    const int nsl = dv / slw, xcd = blockIdx.x & 7, pidx = blockIdx.x >> 3;
    const int rank = (pidx / nsl) * 8 + xcd;
    p.slice = pidx % nsl;
    p.valid = rank < (a.n_seq > 0 ? a.n_seq : a.N) * a.H;
    const int s = !p.valid ? 0 : (a.seq_order ? a.seq_order[rank / a.H] : rank / a.H);
    p.h = rank % a.H;
    p.chain = s * a.H + p.h;
    if (a.cu_seqlens) { p.t0 = a.cu_seqlens[s]; p.len = a.cu_seqlens[s + 1] - (int)p.t0; p.ch0 = a.chunk_off[s]; }
    else              { p.t0 = (long)s * a.T;   p.len = a.T;                             p.ch0 = s * a.NT; }
    p.nch = (p.len + 63) / 64;
    return p;
}

// this wave's tiles of a [.., d_k, d_v] fp32 state <-> accumulators (base: first row, this lane's column)
template <int DK> __device__ __forceinline__ void load_state(floatx4 (&S)[DK / 64], const float* base, int dv, int wave, int g)
{
#pragma unroll
    for (int t = 0; t < DK / 64; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) S[t][e] = base[(size_t)(16 * (wave * (DK / 64) + t) + 4 * g + e) * dv];
}
template <int DK> __device__ __forceinline__ void store_state(const floatx4 (&S)[DK / 64], float* base, int dv, int wave, int g)
{
#pragma unroll
    for (int t = 0; t < DK / 64; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) base[(size_t)(16 * (wave * (DK / 64) + t) + 4 * g + e) * dv] = S[t][e];
}

}  // namespace

// =================================================================================================
// forward: o and the final state.  Per chunk (eqs. (6)-(8)):
//     X = V - D_gamma (K S)    U = T' X    O = D_gamma (Q S) + P U    S = gamma_C S + K^T diag(gamma_C/gamma_i) U
// DIAG: diagonal gating (App. B): a.k = K o Gamma, a.q = Q o Gamma, a.kt_src = K o (gamma_C/Gamma), unit decay vectors in
// the records, and the state decays per row by a.gc_vec.
// SV: S of every chunk, X and U stay behind for the backward pass (see ScanArgs), as bwd_states_f32_kernel leaves them.
// =================================================================================================
template <int DK, int NC, bool DIAG, bool SV>
__global__ __launch_bounds__(256, 2) void scan_f32_kernel(ScanArgs<float> a)
{
    typedef F32<DK> C;
    constexpr int KB = C::KB, TS = C::TS;
    constexpr int OFF_K2 = C::TILE, OFF_S = (DIAG ? 2 : 1) * C::TILE, OFF_X = OFF_S + NC * C::SXB, OFF_U = OFF_X + NC * C::RXB,
                  OFF_UD = OFF_U + NC * C::RXB, LDS = OFF_UD + NC * C::RXB;
    static_assert(LDS <= 160 * 1024, "LDS budget of a gfx950 CU");
    __shared__ __attribute__((aligned(1024))) char lds[LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const Pos p = sweep_pos(a, a.dv, 16 * NC);
    if (!p.valid) return;
    const int col0 = p.slice * 16 * NC + r;
    const size_t ks = (size_t)a.H * DK, vs = (size_t)a.H * a.dv;
    const float* kb = a.k + (size_t)p.t0 * ks + (size_t)p.h * DK;
    const float* qb = a.q + (size_t)p.t0 * ks + (size_t)p.h * DK;
    const float* k2b = DIAG ? a.kt_src + (size_t)p.t0 * ks + (size_t)p.h * DK : nullptr;
    const float* vb = a.v + (size_t)p.t0 * vs + (size_t)p.h * a.dv + col0;
    float* ob = a.o + (size_t)p.t0 * vs + (size_t)p.h * a.dv + col0;
    // records: T', and P with the vectors behind it
    constexpr int HALF = ws_half_bytes<float>(), REC = SV ? bwd_record_bytes<float>() : ws_record_bytes<float>(),
                  RECP = SV ? pair_record_bytes<float>() : REC;
    const char* rec0 = reinterpret_cast<const char*>(a.wsT) + ((size_t)p.ch0 * a.H + p.h) * REC;
    const char* recp0 = SV ? reinterpret_cast<const char*>(a.wsP) + ((size_t)p.ch0 * a.H + p.h) * RECP : rec0 + HALF;
    const size_t rec_step = (size_t)a.H * REC, recp_step = (size_t)a.H * RECP;
    const int row0 = 16 * wave + 4 * g;

    TileOps<DK> ops;
    ops.init(wave, r, g);

    floatx4 S[NC][TS];
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        if (a.h0) load_state<DK>(S[n], a.h0 + (size_t)p.chain * DK * a.dv + col0 + 16 * n, a.dv, wave, g);
        else
#pragma unroll
            for (int t = 0; t < TS; ++t) S[n][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // to the exchange area (and to the checkpoint of chunk c)
    auto put_state = [&]([[maybe_unused]] int c) {
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                *reinterpret_cast<float4*>(lds + OFF_S + n * C::SXB + ((wave * TS + t) * 64 + lane) * 16) = quad(S[n][t]);
                if constexpr (SV) {
                    if (c < p.nch) *reinterpret_cast<float4*>(a.s_chk + (((size_t)(p.ch0 + c) * a.H + p.h) * a.dv + col0 + 16 * n) * DK + 16 * (wave * TS + t) + 4 * g) = quad(S[n][t]);
                }
            }
    };

    // operands of one wave alone, each requested as soon as its previous value has been used
    float4 qf[KB];
    TriRegs tf, pf;
    floatx4 vf[NC], eg, ed, eq, gcv[TS];
    float gC = 1.f;
    auto get_q = [&](int c) {
        const float* q = qb + (size_t)min(64 * c + 16 * wave + r, p.len - 1) * ks + 4 * g;
#pragma unroll
        for (int b = 0; b < KB; ++b) qf[b] = ldf4(q + 16 * b);
    };
    auto get_v = [&](int c) {
        const int clen = min(64, p.len - 64 * c);
#pragma unroll
        for (int n = 0; n < NC; ++n) vf[n] = load_col(vb + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen);
        const char* rec = recp0 + (size_t)c * recp_step + HALF;
        eg = lda4(rec + 4 * row0);
        ed = lda4(rec + 256 + 4 * row0);
        eq = lda4(rec + 512 + 4 * row0);
        gC = *reinterpret_cast<const float*>(rec + 252);
        if constexpr (DIAG) {
            const float* gc = a.gc_vec + ((size_t)(p.ch0 + c) * a.H + p.h) * DK + 4 * g;
#pragma unroll
            for (int t = 0; t < TS; ++t) gcv[t] = lda4(gc + 16 * (wave * TS + t));
        }
    };

    TileRegs<DK> kr, k2r;
    auto fetch_k = [&](int c) {
        const int clen = min(64, p.len - 64 * c);
        kr.load(kb + (size_t)(64 * c) * ks, ks, clen, tid);
        if constexpr (DIAG) k2r.load(k2b + (size_t)(64 * c) * ks, ks, clen, tid);
    };
    auto stash_k = [&]() {
        kr.stash(lds, tid);
        if constexpr (DIAG) k2r.stash(lds + OFF_K2, tid);
    };

    if (p.nch > 0) {
        fetch_k(0);
        get_v(0);
        load_tri(tf, rec0, wave, lane);
        get_q(0);
        load_tri(pf, recp0, wave, lane);
        stash_k();
        put_state(0);
    }
    __syncthreads();
    for (int c = 0; c < p.nch; ++c) {
        const int cn = min(c + 1, p.nch - 1);
        const char* rec_n = rec0 + (size_t)cn * rec_step;
        fetch_k(cn);                                     // lands during this chunk's products
        // ---- X = V - D_gamma K S (on the serial chain), then Q S, which fills the wait for the other rows of X
        floatx4 x[NC], o[NC];
#pragma unroll
        for (int n = 0; n < NC; ++n) { x[n] = floatx4{0.f, 0.f, 0.f, 0.f}; o[n] = x[n]; }
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            const float4 ka = ops.row_quad(lds, b);
#pragma unroll
            for (int n = 0; n < NC; ++n) mma16(x[n], ka, ldf4(lds + OFF_S + n * C::SXB + (b * 64 + lane) * 16));
        }
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            x[n] = vf[n] - eg * x[n];
            *reinterpret_cast<float4*>(lds + OFF_X + n * C::RXB + (wave * 64 + lane) * 16) = quad(x[n]);
        }
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int n = 0; n < NC; ++n) mma16(o[n], qf[b], ldf4(lds + OFF_S + n * C::SXB + (b * 64 + lane) * 16));
        __syncthreads();
        get_q(cn);
        // ---- U = T' X
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            floatx4 u = {0.f, 0.f, 0.f, 0.f};
            mma_tri(u, tf, lds + OFF_X + n * C::RXB, wave, lane);
            *reinterpret_cast<float4*>(lds + OFF_UD + n * C::RXB + (wave * 64 + lane) * 16) = quad(u * ed);
            *reinterpret_cast<float4*>(lds + OFF_U + n * C::RXB + (wave * 64 + lane) * 16) = quad(u);
            o[n] = o[n] * eq;
            if constexpr (SV) {
                const size_t at = (size_t)(p.t0 + 64L * c) * vs + (size_t)p.h * a.dv + col0 + 16 * n;
                store_col(a.X + at, vs, row0, min(64, p.len - 64 * c), x[n]);
                store_col(a.U + at, vs, row0, min(64, p.len - 64 * c), u);
            }
        }
        __syncthreads();
        load_tri(tf, rec_n, wave, lane);
        // ---- S = gamma_C S + K^T (diag(gamma_C/gamma_i) U)
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) { if constexpr (DIAG) S[n][t] = S[n][t] * gcv[t]; else S[n][t] = S[n][t] * gC; }
        get_v(cn);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            float4 ud[NC];
#pragma unroll
            for (int n = 0; n < NC; ++n) ud[n] = ldf4(lds + OFF_UD + n * C::RXB + (jb * 64 + lane) * 16);
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const float4 kt = ops.col_quad(lds + (DIAG ? OFF_K2 : 0), t, jb);
#pragma unroll
                for (int n = 0; n < NC; ++n) mma16(S[n][t], kt, ud[n]);
            }
        }
        __syncthreads();                                 // K and the exchanged state are no longer read
        stash_k();
        put_state(c + 1);
        // ---- O = D_gamma (Q S) + P U, off the chain
        const int clen = min(64, p.len - 64 * c);
#pragma unroll
        for (int n = 0; n < NC; ++n) mma_tri(o[n], pf, lds + OFF_U + n * C::RXB, wave, lane);
        load_tri(pf, recp0 + (size_t)cn * recp_step, wave, lane);
#pragma unroll
        for (int n = 0; n < NC; ++n) store_col(ob + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen, o[n]);
        __syncthreads();
    }
    if (a.hT) {
#pragma unroll
        for (int n = 0; n < NC; ++n) store_state<DK>(S[n], a.hT + (size_t)p.chain * DK * a.dv + col0 + 16 * n, a.dv, wave, g);
    }
}

// The same with eight waves, two per SIMD: waves 0 .. 3 carry the chain (K S, X, U, the state update), waves 4 .. 7, which
// share their SIMDs, do everything off it (Q S, P U, the outputs, the copies of K).  With four waves a SIMD stands idle
// whenever its only wave waits for LDS or a barrier: 3.7 us per chunk for 1.7 us of MFMA, here 3.1 us.  K and the exchanged
// state have two images each, so a step needs three barriers instead of four.  (Loads requested two chunks ahead, two
// accumulators per product and a raised priority of the chain change nothing: 123 us either way.)
// SV: the waves off the chain store what the backward needs, which they find in the exchange areas.
template <int DK, int NC, bool DIAG, bool SV>
__global__ __launch_bounds__(512, 2) void scan_f32_split_kernel(ScanArgs<float> a)
{
    typedef F32<DK> C;
    constexpr int KB = C::KB, TS = C::TS;
    constexpr int KIMG = (DIAG ? 2 : 1) * C::TILE, SIMG = NC * C::SXB;
    constexpr int OFF_K2 = C::TILE, OFF_S = 2 * KIMG, OFF_X = OFF_S + 2 * SIMG, OFF_U = OFF_X + NC * C::RXB,
                  OFF_UD = OFF_U + NC * C::RXB, LDS = OFF_UD + NC * C::RXB;
    static_assert(LDS <= 160 * 1024, "LDS budget of a gfx950 CU");
    __shared__ __attribute__((aligned(1024))) char lds[LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;       // row tile, in either role
    const bool chain = __builtin_amdgcn_readfirstlane(tid >> 8) == 0;
    const int r = lane & 15, g = lane >> 4;
    const Pos p = sweep_pos(a, a.dv, 16 * NC);
    if (!p.valid) return;
    const int col0 = p.slice * 16 * NC + r;
    const size_t ks = (size_t)a.H * DK, vs = (size_t)a.H * a.dv;
    // records: T', and P with the vectors behind it
    constexpr int HALF = ws_half_bytes<float>(), REC = SV ? bwd_record_bytes<float>() : ws_record_bytes<float>(),
                  RECP = SV ? pair_record_bytes<float>() : REC;
    const char* rec0 = reinterpret_cast<const char*>(a.wsT) + ((size_t)p.ch0 * a.H + p.h) * REC;
    const char* recp0 = SV ? reinterpret_cast<const char*>(a.wsP) + ((size_t)p.ch0 * a.H + p.h) * RECP : rec0 + HALF;
    const size_t rec_step = (size_t)a.H * REC, recp_step = (size_t)a.H * RECP;
    const int row0 = 16 * wave + 4 * g;

    if (chain) {
        const float* vb = a.v + (size_t)p.t0 * vs + (size_t)p.h * a.dv + col0;
        TileOps<DK> ops;
        ops.init(wave, r, g);
        floatx4 S[NC][TS];
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            if (a.h0) load_state<DK>(S[n], a.h0 + (size_t)p.chain * DK * a.dv + col0 + 16 * n, a.dv, wave, g);
            else
#pragma unroll
                for (int t = 0; t < TS; ++t) S[n][t] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        auto put_state = [&](char* img) {
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int t = 0; t < TS; ++t)
                    *reinterpret_cast<float4*>(img + n * C::SXB + ((wave * TS + t) * 64 + lane) * 16) = quad(S[n][t]);
        };
        TriRegs tf;
        floatx4 vf[NC], eg, ed, gcv[TS];
        float gC = 1.f;
        auto get_v = [&](int c) {
            const int clen = min(64, p.len - 64 * c);
#pragma unroll
            for (int n = 0; n < NC; ++n) vf[n] = load_col(vb + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen);
            const char* rec = recp0 + (size_t)c * recp_step + HALF;
            eg = lda4(rec + 4 * row0);
            ed = lda4(rec + 256 + 4 * row0);
            gC = *reinterpret_cast<const float*>(rec + 252);
            if constexpr (DIAG) {
                const float* gc = a.gc_vec + ((size_t)(p.ch0 + c) * a.H + p.h) * DK + 4 * g;
#pragma unroll
                for (int t = 0; t < TS; ++t) gcv[t] = lda4(gc + 16 * (wave * TS + t));
            }
        };
        if (p.nch > 0) {
            get_v(0);
            load_tri(tf, rec0, wave, lane);
            put_state(lds + OFF_S);
        }
        __syncthreads();
        for (int c = 0; c < p.nch; ++c) {
            const int cn = min(c + 1, p.nch - 1);
            const char* kt_img = lds + (c & 1) * KIMG;
            const char* s_img = lds + OFF_S + (c & 1) * SIMG;
            // ---- X = V - D_gamma K S
            floatx4 x[NC];
#pragma unroll
            for (int n = 0; n < NC; ++n) x[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const float4 ka = ops.row_quad(kt_img, b);
#pragma unroll
                for (int n = 0; n < NC; ++n) mma16(x[n], ka, ldf4(s_img + n * C::SXB + (b * 64 + lane) * 16));
            }
#pragma unroll
            for (int n = 0; n < NC; ++n)
                *reinterpret_cast<float4*>(lds + OFF_X + n * C::RXB + (wave * 64 + lane) * 16) = quad(vf[n] - eg * x[n]);
            __syncthreads();
            // ---- U = T' X
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                floatx4 u = {0.f, 0.f, 0.f, 0.f};
                mma_tri(u, tf, lds + OFF_X + n * C::RXB, wave, lane);
                *reinterpret_cast<float4*>(lds + OFF_UD + n * C::RXB + (wave * 64 + lane) * 16) = quad(u * ed);
                *reinterpret_cast<float4*>(lds + OFF_U + n * C::RXB + (wave * 64 + lane) * 16) = quad(u);
            }
            __syncthreads();
            load_tri(tf, rec0 + (size_t)cn * rec_step, wave, lane);
            // ---- S = gamma_C S + K^T (diag(gamma_C/gamma_i) U)
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int t = 0; t < TS; ++t) { if constexpr (DIAG) S[n][t] = S[n][t] * gcv[t]; else S[n][t] = S[n][t] * gC; }
            get_v(cn);
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                float4 ud[NC];
#pragma unroll
                for (int n = 0; n < NC; ++n) ud[n] = ldf4(lds + OFF_UD + n * C::RXB + (jb * 64 + lane) * 16);
#pragma unroll
                for (int t = 0; t < TS; ++t) {
                    const float4 kt = ops.col_quad(kt_img + (DIAG ? OFF_K2 : 0), t, jb);
#pragma unroll
                    for (int n = 0; n < NC; ++n) mma16(S[n][t], kt, ud[n]);
                }
            }
            put_state(lds + OFF_S + ((c + 1) & 1) * SIMG);       // the image chunk c - 1 was read from
            __syncthreads();
        }
        if (a.hT) {
#pragma unroll
            for (int n = 0; n < NC; ++n) store_state<DK>(S[n], a.hT + (size_t)p.chain * DK * a.dv + col0 + 16 * n, a.dv, wave, g);
        }
    } else {
        const int t2 = tid - 256;
        const float* kb = a.k + (size_t)p.t0 * ks + (size_t)p.h * DK;
        const float* qb = a.q + (size_t)p.t0 * ks + (size_t)p.h * DK;
        const float* k2b = DIAG ? a.kt_src + (size_t)p.t0 * ks + (size_t)p.h * DK : nullptr;
        float* ob = a.o + (size_t)p.t0 * vs + (size_t)p.h * a.dv + col0;
        float4 qf[KB];
        TriRegs pf;
        floatx4 eq;
        auto get_q = [&](int c) {
            const float* q = qb + (size_t)min(64 * c + 16 * wave + r, p.len - 1) * ks + 4 * g;
#pragma unroll
            for (int b = 0; b < KB; ++b) qf[b] = ldf4(q + 16 * b);
            eq = lda4(recp0 + (size_t)c * recp_step + HALF + 512 + 4 * row0);
        };
        TileRegs<DK> kr, k2r;
        auto fetch_k = [&](int c) {
            const int clen = min(64, p.len - 64 * c);
            kr.load(kb + (size_t)(64 * c) * ks, ks, clen, t2);
            if constexpr (DIAG) k2r.load(k2b + (size_t)(64 * c) * ks, ks, clen, t2);
        };
        auto stash_k = [&](char* img) {
            kr.stash(img, t2);
            if constexpr (DIAG) k2r.stash(img + OFF_K2, t2);
        };
        if (p.nch > 0) {
            fetch_k(0);
            get_q(0);
            load_tri(pf, recp0, wave, lane);
            stash_k(lds);
        }
        __syncthreads();
        for (int c = 0; c < p.nch; ++c) {
            const int cn = min(c + 1, p.nch - 1);
            const char* s_img = lds + OFF_S + (c & 1) * SIMG;
            fetch_k(cn);                                 // lands during this chunk's products
            // ---- Q S, half of it on either side of the chain's first barrier
            floatx4 o[NC];
#pragma unroll
            for (int n = 0; n < NC; ++n) o[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                if (b == KB / 2) __syncthreads();
#pragma unroll
                for (int n = 0; n < NC; ++n) mma16(o[n], qf[b], ldf4(s_img + n * C::SXB + (b * 64 + lane) * 16));
            }
            const int clen = min(64, p.len - 64 * c);
            if constexpr (SV) {
                float* chk = a.s_chk + (((size_t)(p.ch0 + c) * a.H + p.h) * a.dv + col0) * DK + 4 * g;
#pragma unroll
                for (int n = 0; n < NC; ++n) {
#pragma unroll
                    for (int t = 0; t < TS; ++t)
                        *reinterpret_cast<float4*>(chk + (size_t)(16 * n) * DK + 16 * (wave * TS + t)) =
                            ldf4(s_img + n * C::SXB + ((wave * TS + t) * 64 + lane) * 16);
                    store_col(a.X + (size_t)(p.t0 + 64L * c) * vs + (size_t)p.h * a.dv + col0 + 16 * n, vs, row0, clen,
                              lda4(lds + OFF_X + n * C::RXB + (wave * 64 + lane) * 16));
                }
            }
#pragma unroll
            for (int n = 0; n < NC; ++n) o[n] = o[n] * eq;
            get_q(cn);
            __syncthreads();
            // ---- O = D_gamma (Q S) + P U
#pragma unroll
            for (int n = 0; n < NC; ++n) mma_tri(o[n], pf, lds + OFF_U + n * C::RXB, wave, lane);
            load_tri(pf, recp0 + (size_t)cn * recp_step, wave, lane);
            stash_k(lds + ((c + 1) & 1) * KIMG);         // the image chunk c - 1 was read from
#pragma unroll
            for (int n = 0; n < NC; ++n) store_col(ob + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen, o[n]);
            if constexpr (SV)
#pragma unroll
                for (int n = 0; n < NC; ++n)
                    store_col(a.U + (size_t)(p.t0 + 64L * c) * vs + (size_t)p.h * a.dv + col0 + 16 * n, vs, row0, clen,
                              lda4(lds + OFF_U + n * C::RXB + (wave * 64 + lane) * 16));
            __syncthreads();
        }
    }
}

// =================================================================================================
// backward, forward sweep: incoming state of every chunk (transposed, [d_v][d_k]), X and U
// =================================================================================================
template <int DK, int NC>
__global__ __launch_bounds__(256, 2) void bwd_states_f32_kernel(BwdArgs<float> a)
{
    typedef F32<DK> C;
    constexpr int KB = C::KB, TS = C::TS;
    constexpr int OFF_S = C::TILE, OFF_X = OFF_S + NC * C::SXB, OFF_UD = OFF_X + NC * C::RXB, LDS = OFF_UD + NC * C::RXB;
    __shared__ __attribute__((aligned(1024))) char lds[LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const Pos p = sweep_pos(a, a.dv_dim, 16 * NC);
    if (!p.valid) return;
    const int col0 = p.slice * 16 * NC + r, row0 = 16 * wave + 4 * g;
    const size_t ks = (size_t)a.H * DK, vs = (size_t)a.H * a.dv_dim;
    const float* kb = a.k + (size_t)p.t0 * ks + (size_t)p.h * DK;
    const size_t vo = (size_t)p.t0 * vs + (size_t)p.h * a.dv_dim + col0;
    constexpr int HALF = ws_half_bytes<float>(), REC = bwd_record_bytes<float>();
    const char* rec0 = a.rec + ((size_t)p.ch0 * a.H + p.h) * REC;
    const size_t rec_step = (size_t)a.H * REC;

    TileOps<DK> ops;
    ops.init(wave, r, g);
    floatx4 S[NC][TS];
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        if (a.h0) load_state<DK>(S[n], a.h0 + (size_t)p.chain * DK * a.dv_dim + col0 + 16 * n, a.dv_dim, wave, g);
        else
#pragma unroll
            for (int t = 0; t < TS; ++t) S[n][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // to the exchange area, and to the checkpoint of chunk c
    auto put_state = [&](int c) {
        float* chk = a.s_chk + (((size_t)(p.ch0 + c) * a.H + p.h) * a.dv_dim + col0) * DK + 4 * g;
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                *reinterpret_cast<float4*>(lds + OFF_S + n * C::SXB + ((wave * TS + t) * 64 + lane) * 16) = quad(S[n][t]);
                *reinterpret_cast<float4*>(chk + (size_t)(16 * n) * DK + 16 * (wave * TS + t)) = quad(S[n][t]);
            }
    };
    TriRegs tf;
    floatx4 vf[NC], eg, ed;
    float gC = 1.f;
    auto get_v = [&](int c) {
        const int clen = min(64, p.len - 64 * c);
#pragma unroll
        for (int n = 0; n < NC; ++n) vf[n] = load_col(a.v + vo + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen);
        const char* rec = rec0 + (size_t)c * rec_step + 3 * HALF;
        eg = lda4(rec + 4 * row0);
        ed = lda4(rec + 256 + 4 * row0);
        gC = *reinterpret_cast<const float*>(rec + 252);
    };
    TileRegs<DK> kr;
    if (p.nch > 0) {
        kr.load(kb, ks, min(64, p.len), tid);
        get_v(0);
        load_tri(tf, rec0, wave, lane);
        kr.stash(lds, tid);
        put_state(0);
    }
    __syncthreads();
    for (int c = 0; c < p.nch; ++c) {
        const int cn = min(c + 1, p.nch - 1);
        const int clen = min(64, p.len - 64 * c);
        kr.load(kb + (size_t)(64 * cn) * ks, ks, min(64, p.len - 64 * cn), tid);
        floatx4 x[NC];
#pragma unroll
        for (int n = 0; n < NC; ++n) x[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            const float4 ka = ops.row_quad(lds, b);
#pragma unroll
            for (int n = 0; n < NC; ++n) mma16(x[n], ka, ldf4(lds + OFF_S + n * C::SXB + (b * 64 + lane) * 16));
        }
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            x[n] = vf[n] - eg * x[n];
            *reinterpret_cast<float4*>(lds + OFF_X + n * C::RXB + (wave * 64 + lane) * 16) = quad(x[n]);
        }
        __syncthreads();
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            floatx4 u = {0.f, 0.f, 0.f, 0.f};
            mma_tri(u, tf, lds + OFF_X + n * C::RXB, wave, lane);
            *reinterpret_cast<float4*>(lds + OFF_UD + n * C::RXB + (wave * 64 + lane) * 16) = quad(u * ed);
            store_col(a.X + vo + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen, x[n]);
            store_col(a.U + vo + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen, u);
        }
        __syncthreads();
        load_tri(tf, rec0 + (size_t)cn * rec_step, wave, lane);
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) S[n][t] = S[n][t] * gC;
        get_v(cn);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            float4 ud[NC];
#pragma unroll
            for (int n = 0; n < NC; ++n) ud[n] = ldf4(lds + OFF_UD + n * C::RXB + (jb * 64 + lane) * 16);
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const float4 kt = ops.col_quad(lds, t, jb);
#pragma unroll
                for (int n = 0; n < NC; ++n) mma16(S[n][t], kt, ud[n]);
            }
        }
        __syncthreads();                                 // K and the exchanged state are no longer read
        kr.stash(lds, tid);
        if (c + 1 < p.nch) put_state(c + 1);
        __syncthreads();
    }
}

// =================================================================================================
// backward, reverse sweep: gradient dS' of the state every chunk hands on (transposed), Y, dv, dh0
//     dU = P^T dO + diag(gamma_C/gamma_i) K dS'    Y = M^T dU    dX = B Y = dv
//     dS = gamma_C dS' + Q^T D_gamma diag(1/||q||) dO - K^T D_gamma dX
// =================================================================================================
template <int DK, int NC>
__global__ __launch_bounds__(256, DK == 128 ? 1 : 2) void bwd_scan_f32_kernel(BwdArgs<float> a)
{
    typedef F32<DK> C;
    constexpr int KB = C::KB, TS = C::TS;
    constexpr int OFF_Q = C::TILE, OFF_S = 2 * C::TILE, OFF_U = OFF_S + NC * C::SXB, OFF_G = OFF_U + NC * C::RXB,
                  LDS = OFF_G + NC * C::RXB;
    static_assert(LDS <= 160 * 1024, "LDS budget of a gfx950 CU");
    __shared__ __attribute__((aligned(1024))) char lds[LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const Pos p = sweep_pos(a, a.dv_dim, 16 * NC);
    if (!p.valid) return;
    const int col0 = p.slice * 16 * NC + r, row0 = 16 * wave + 4 * g;
    const size_t ks = (size_t)a.H * DK, vs = (size_t)a.H * a.dv_dim;
    const float* kb = a.k + (size_t)p.t0 * ks + (size_t)p.h * DK;
    const float* qb = a.q + (size_t)p.t0 * ks + (size_t)p.h * DK;
    const size_t vo = (size_t)p.t0 * vs + (size_t)p.h * a.dv_dim + col0;
    constexpr int HALF = ws_half_bytes<float>(), REC = bwd_record_bytes<float>();
    const char* rec0 = a.rec + ((size_t)p.ch0 * a.H + p.h) * REC;
    const size_t rec_step = (size_t)a.H * REC;

    TileOps<DK> ops;
    ops.init(wave, r, g);
    floatx4 dS[NC][TS];
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        if (a.d_hT) load_state<DK>(dS[n], a.d_hT + (size_t)p.chain * DK * a.dv_dim + col0 + 16 * n, a.dv_dim, wave, g);
        else
#pragma unroll
            for (int t = 0; t < TS; ++t) dS[n][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    auto put_state = [&](int c) {
        float* chk = a.ds_chk + (((size_t)(p.ch0 + c) * a.H + p.h) * a.dv_dim + col0) * DK + 4 * g;
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                *reinterpret_cast<float4*>(lds + OFF_S + n * C::SXB + ((wave * TS + t) * 64 + lane) * 16) = quad(dS[n][t]);
                *reinterpret_cast<float4*>(chk + (size_t)(16 * n) * DK + 16 * (wave * TS + t)) = quad(dS[n][t]);
            }
    };
    TriRegs mf, pf;                                      // this wave's rows of M^T and P^T
    floatx4 df[NC][4];                                   // dO, all 64 rows of this lane's columns
    floatx4 eg, ed, be, sc[4];                           // sc: gamma_i / ||q_i|| of all rows 16 jt + 4 g + e
    float gC = 1.f;
    auto get_do = [&](int c) {
        const int clen = min(64, p.len - 64 * c);
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int jt = 0; jt < 4; ++jt) df[n][jt] = load_col(a.d_o + vo + (size_t)(64 * c) * vs + 16 * n, vs, 16 * jt + 4 * g, clen);
    };
    auto get_vec = [&](int c) {
        const char* rec = rec0 + (size_t)c * rec_step + 3 * HALF;
        eg = lda4(rec + 4 * row0);
        ed = lda4(rec + 256 + 4 * row0);
        be = lda4(rec + 512 + 4 * row0);
        gC = *reinterpret_cast<const float*>(rec + 252);
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) sc[jt] = lda4(rec + 64 * jt + 16 * g) * lda4(rec + 1024 + 64 * jt + 16 * g);
    };
    TileRegs<DK> kr, qr;
    auto fetch = [&](int c) {
        const int clen = min(64, p.len - 64 * c);
        kr.load(kb + (size_t)(64 * c) * ks, ks, clen, tid);
        qr.load(qb + (size_t)(64 * c) * ks, ks, clen, tid);
    };
    if (p.nch > 0) {
        const int c = p.nch - 1;
        fetch(c);
        get_do(c);
        get_vec(c);
        load_triu(pf, rec0 + (size_t)c * rec_step + 2 * HALF, wave, lane);
        load_triu(mf, rec0 + (size_t)c * rec_step + HALF, wave, lane);
        kr.stash(lds, tid); qr.stash(lds + OFF_Q, tid);
        put_state(c);
    }
    __syncthreads();
    for (int c = p.nch - 1; c >= 0; --c) {
        const int cn = max(c - 1, 0);
        const int clen = min(64, p.len - 64 * c);
        const char* rec_n = rec0 + (size_t)cn * rec_step;
        fetch(cn);
        if (clen < 64)                                   // dO of the rows that are not there
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int jt = 0; jt < 4; ++jt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) df[n][jt][e] = 16 * jt + 4 * g + e < clen ? df[n][jt][e] : 0.f;
        // ---- dU = P^T dO + diag(gamma_C/gamma_i) K dS'
        floatx4 kd[NC];
#pragma unroll
        for (int n = 0; n < NC; ++n) kd[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            const float4 ka = ops.row_quad(lds, b);
#pragma unroll
            for (int n = 0; n < NC; ++n) mma16(kd[n], ka, ldf4(lds + OFF_S + n * C::SXB + (b * 64 + lane) * 16));
        }
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            floatx4 du = kd[n] * ed;
            if (wave < 2) mma32(du, pf.q[0][0], pf.q[0][1], quad(df[n][0]), quad(df[n][1]));
            mma32(du, pf.q[1][0], pf.q[1][1], quad(df[n][2]), quad(df[n][3]));
            *reinterpret_cast<float4*>(lds + OFF_U + n * C::RXB + (wave * 64 + lane) * 16) = quad(du);
        }
        load_triu(pf, rec_n + 2 * HALF, wave, lane);
        // The half of the state update that waits for nothing fills the wait for the other rows of dU.  Its terms and those of
        // the other half largely cancel where keys are correlated, so they meet in sums of their own and dS takes one
        // rounding per chunk: added to dS one by one, all of Q^T before all of K^T, d_h0 was 3.4e-7 off 64 bits, so 2.7e-7
        // (4 x 300 tokens, 8 heads; the sweep of 2 x 500 tokens, 4 heads, d = 64: 28.1 -> 28.7 us).
        floatx4 inc[NC][TS];
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) inc[n][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const float4 qt = ops.col_quad(lds + OFF_Q, t, jb);
#pragma unroll
                for (int n = 0; n < NC; ++n) mma16(inc[n][t], qt, quad(df[n][jb] * sc[jb]));
            }
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) dS[n][t] = dS[n][t] * gC;
        __syncthreads();
        get_do(cn);
        // ---- Y = M^T dU, dX = B Y
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            floatx4 y = {0.f, 0.f, 0.f, 0.f};
            mma_triu(y, mf, lds + OFF_U + n * C::RXB, wave, lane);
            const floatx4 dx = y * be;
            *reinterpret_cast<float4*>(lds + OFF_G + n * C::RXB + (wave * 64 + lane) * 16) = quad(-(eg * dx));
            store_col(a.Y + vo + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen, y);
            store_col(a.dv + vo + (size_t)(64 * c) * vs + 16 * n, vs, row0, clen, dx);
        }
        __syncthreads();
        load_triu(mf, rec_n + HALF, wave, lane);
        get_vec(cn);
        // ---- dS += K^T (-D_gamma dX)
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            float4 gd[NC];
#pragma unroll
            for (int n = 0; n < NC; ++n) gd[n] = ldf4(lds + OFF_G + n * C::RXB + (jb * 64 + lane) * 16);
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const float4 kt = ops.col_quad(lds, t, jb);
#pragma unroll
                for (int n = 0; n < NC; ++n) mma16(inc[n][t], kt, gd[n]);
            }
        }
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < TS; ++t) dS[n][t] = dS[n][t] + inc[n][t];
        __syncthreads();                                 // K, Q and the exchanged gradient are no longer read
        kr.stash(lds, tid); qr.stash(lds + OFF_Q, tid);
        if (c > 0) put_state(c - 1);
        __syncthreads();
    }
    if (a.dh0) {
#pragma unroll
        for (int n = 0; n < NC; ++n) store_state<DK>(dS[n], a.dh0 + (size_t)p.chain * DK * a.dv_dim + col0 + 16 * n, a.dv_dim, wave, g);
    }
}

// =================================================================================================
// launchers: tiles = 1 or 2 column tiles (16 state columns each) per workgroup
// =================================================================================================
static dim3 sweep_grid(int n_chains, int dv, int tiles) { return dim3((unsigned)(((n_chains + 7) / 8) * 8 * (dv / (16 * tiles)))); }

template <int DK, bool DIAG, bool SV>
static hipError_t launch_scan_dk(const ScanArgs<float>& a, int tiles, hipStream_t st)
{
    const int n_chains = (a.n_seq > 0 ? a.n_seq : a.N) * a.H;
    if (n_chains == 0) return hipSuccess;
    const dim3 grid = sweep_grid(n_chains, a.dv, tiles);
    // Eight waves per workgroup while every workgroup has a CU to itself: 256 tiles 139 -> 123 us per call (4 x 2000 tokens, 8
    // heads, d = 128), 512 tiles, two per workgroup, 126 -> 111 us, 256 tiles with per-channel decay 97 -> 81 us.  With more
    // tiles two workgroups of four waves share a CU and cover each other (1024 tiles 209 us against 217 us with eight
    // waves); per-channel decay with two tiles per workgroup would not fit the second image of its two K tiles.
    const long wgs = ((long)n_chains + 7) / 8 * 8 * (a.dv / (16 * tiles));
    if (tiles == 1) hipLaunchKernelGGL((scan_f32_split_kernel<DK, 1, DIAG, SV>), grid, dim3(512), 0, st, a);
    else {
        if constexpr (!DIAG) {
            if (wgs <= 256) {
                hipLaunchKernelGGL((scan_f32_split_kernel<DK, 2, DIAG, SV>), grid, dim3(512), 0, st, a);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((scan_f32_kernel<DK, 2, DIAG, SV>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}
hipError_t launch_scan_f32(const ScanArgs<float>& a, int dk, int tiles, hipStream_t st)
{
    if (tiles != 1 && tiles != 2) return hipErrorInvalidValue;
    if (a.kt_src) return dk == 64 ? launch_scan_dk<64, true, false>(a, tiles, st) : launch_scan_dk<128, true, false>(a, tiles, st);
    if (a.s_chk) return dk == 64 ? launch_scan_dk<64, false, true>(a, tiles, st) : launch_scan_dk<128, false, true>(a, tiles, st);
    return dk == 64 ? launch_scan_dk<64, false, false>(a, tiles, st) : launch_scan_dk<128, false, false>(a, tiles, st);
}

template <int DK>
static hipError_t launch_bwd_dk(const BwdArgs<float>& a, int tiles, bool reverse, hipStream_t st)
{
    const int n_chains = (a.n_seq > 0 ? a.n_seq : a.N) * a.H;
    if (n_chains == 0) return hipSuccess;
    const dim3 grid = sweep_grid(n_chains, a.dv_dim, tiles);
    if (reverse) {
        if (tiles == 1) hipLaunchKernelGGL((bwd_scan_f32_kernel<DK, 1>), grid, dim3(256), 0, st, a);
        else            hipLaunchKernelGGL((bwd_scan_f32_kernel<DK, 2>), grid, dim3(256), 0, st, a);
    } else {
        if (tiles == 1) hipLaunchKernelGGL((bwd_states_f32_kernel<DK, 1>), grid, dim3(256), 0, st, a);
        else            hipLaunchKernelGGL((bwd_states_f32_kernel<DK, 2>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}
hipError_t launch_bwd_states_f32(const BwdArgs<float>& a, int dk, int tiles, hipStream_t st)
{
    if (tiles != 1 && tiles != 2) return hipErrorInvalidValue;
    return dk == 64 ? launch_bwd_dk<64>(a, tiles, false, st) : launch_bwd_dk<128>(a, tiles, false, st);
}
hipError_t launch_bwd_scan_f32(const BwdArgs<float>& a, int dk, int tiles, hipStream_t st)
{
    if (tiles != 1 && tiles != 2) return hipErrorInvalidValue;
    return dk == 64 ? launch_bwd_dk<64>(a, tiles, true, st) : launch_bwd_dk<128>(a, tiles, true, st);
}

}  // namespace kla
