// Intra-chunk stage of the chunkwise forward (Algorithm 1 right panel, lines 1-4 and the
// matrix of eq. (6)); fully parallel over (chunk, head).
//
// Per chunk of C = 64 tokens of one head it computes
//   beta_i = eta_i / (||k_i||^2 + eps)                                   eq. (3)
//   g_i    = sum_{r<=i} log alpha_r   (log gamma_i, restarting at the chunk)
//   L      = B (A^- o K K^T),  L_ij = beta_i exp(g_i - g_j) k_i.k_j  (j < i)
//   T'     = (I + L)^{-1} B          so that eq. (6) reads  U = T' (V - D_gamma K S_0)
//   P      = A o Q K^T,  P_ij = exp(g_i - g_j) q_i.k_j  (j <= i)         eq. (7)
// and leaves T', P (in the element type, in MFMA operand order) and g in the workspace for the
// scan stage.  Every decay ratio is formed as exp of a difference of g, masked before the exp,
// because gamma itself underflows fp32 inside a chunk for fast decays.
//
// (I + L)^{-1} is built in fp32: the four 16x16 diagonal blocks by forward substitution in LDS,
// then the off-diagonal blocks by two levels of block products on fp32 MFMA,
//   [T11 0; T21 T22] with T21 = -T22 (L21 T11).
//
// intra_kernel is the plain form, kept for bf16 as the A/B reference (KLA_TUNE_GENERIC_INTRA) of kla_chunk_intra_bf16.hip;
// fp32 inputs run kla_chunk_intra_f32.hip.  The diagonal-gating stage below serves both element types.
#include "kla_common.hpp"
#include "kla_kernels.hpp"
#include "kla_mma.hpp"

namespace kla {

namespace {

constexpr int kLdm = 68;   // row stride (floats) of the fp32 64x64 matrices in LDS: 16-byte aligned rows

// lower-triangular 16x16 tile enumeration of a 64x64 matrix: 10 tiles
__device__ __constant__ const int8_t kTileI[10] = {0, 1, 1, 2, 2, 2, 3, 3, 3, 3};
__device__ __constant__ const int8_t kTileJ[10] = {0, 0, 1, 0, 1, 2, 0, 1, 2, 3};

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// B-operand quad of a row-major fp32 matrix: rows 4g..4g+3 of column r
__device__ __forceinline__ float4 bquad(const float* m, int row0, int col0, int r, int g)
{
    const float* p = m + (row0 + 4 * g) * kLdm + col0 + r;
    return make_float4(p[0], p[kLdm], p[2 * kLdm], p[3 * kLdm]);
}
// A-operand quad: columns 4g..4g+3 of row r
__device__ __forceinline__ float4 aquad(const float* m, int row0, int col0, int r, int g)
{
    return ld4(m + (row0 + r) * kLdm + col0 + 4 * g);
}
__device__ __forceinline__ float4 acc_as_quad(floatx4 x) { return make_float4(x[0], x[1], x[2], x[3]); }

// A triangular 64x64 fp32 matrix m (row stride kLdm) -> 6 stored tile-pairs of operand slots at `out`.
// TRANSPOSE = false: the lower-triangular matrix itself (pairs tri_pair(it, jp), jp <= it/2), optionally with
// column j scaled by colscale[j].  TRANSPOSE = true: its transpose, which is upper triangular (pairs
// triu_pair(it, jp), jp >= it/2).  Called by all 256 threads.
template <typename E, bool TRANSPOSE, bool SCALE>
__device__ __forceinline__ void write_tri(char* out, const float* m, const float* colscale, int tid)
{
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int sl = tid + 256 * it;           // slot index: stored tile-pair * 64 + lane
        if (sl >= kTriPairs * 64) break;
        const int ctp = sl >> 6, ln = sl & 63;
        int ti, jp;
        if constexpr (TRANSPOSE) { ti = ctp < 4 ? (ctp >> 1) : ctp - 2; jp = ctp < 4 ? (ctp & 1) : 1; }
        else                     { ti = ctp < 2 ? ctp : 2 + ((ctp - 2) >> 1); jp = ctp < 2 ? 0 : ((ctp - 2) & 1); }
        const int row = 16 * ti + (ln & 15), col = 32 * jp + 4 * (ln >> 4);
        floatx4 v0, v1;
        if constexpr (TRANSPOSE) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { v0[e] = m[(col + e) * kLdm + row]; v1[e] = m[(col + 16 + e) * kLdm + row]; }
        } else {
            const float4 f0 = ld4(m + row * kLdm + col), f1 = ld4(m + row * kLdm + col + 16);
            v0[0] = f0.x; v0[1] = f0.y; v0[2] = f0.z; v0[3] = f0.w;
            v1[0] = f1.x; v1[1] = f1.y; v1[2] = f1.z; v1[3] = f1.w;
            if constexpr (SCALE) {
                const float4 b0 = ld4(colscale + col), b1 = ld4(colscale + col + 16);
                v0[0] *= b0.x; v0[1] *= b0.y; v0[2] *= b0.z; v0[3] *= b0.w;
                v1[0] *= b1.x; v1[1] *= b1.y; v1[2] *= b1.z; v1[3] *= b1.w;
            }
        }
        Slot<E> s; s.q0 = acc_to_quad<E>(v0); s.q1 = acc_to_quad<E>(v1);
        *reinterpret_cast<Slot<E>*>(out + (size_t)sl * slot_bytes<E>()) = s;
    }
}


// Phases 3-6 of the intra-chunk stage, shared by its variants: from L (strictly lower triangular, fp32, in Lm) and
// the fp32 image of P (in Pm) to the record at `rec`: T' = (I + L)^{-1} B and P (forward), or T', M^T and P^T
// (backward).  Tm receives (I + L)^{-1}.  What must be zero on entry: the 16x16 tiles (0,1) and (2,3) of Pm and of Tm, and Pm above
// the diagonal inside its diagonal tiles - the stored tile-pairs, of the matrix or of its transpose, take these in, and phase 5 those
// two tiles of Tm.  The other upper tiles of both, and Lm on and above its diagonal, are not read and may hold anything.  Called by
// all 256 threads after a barrier; contains barriers.
template <typename E, bool BWD>
__device__ __forceinline__ void invert_and_store(const float* Lm, float* Tm, const float* Pm, const float* beta_s, char* rec,
                                                 int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, g = lane >> 4;
    // ---- phase 3: diagonal 16x16 blocks of (I+L)^{-1} by forward substitution (wave w: block w);
    //      meanwhile P goes out to the workspace in operand order ------------------------------
    {
        const int b0 = 16 * wave;
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float s = (i == r) ? 1.f : 0.f;
#pragma unroll
            for (int rr = 0; rr < i; ++rr) s -= Lm[(b0 + i) * kLdm + b0 + rr] * x[rr];
            x[i] = s;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((i >> 2) == g) Tm[(b0 + i) * kLdm + b0 + r] = x[i];
    }
    if constexpr (BWD) write_tri<E, true, false>(rec + 2 * ws_half_bytes<E>(), Pm, nullptr, tid);      // P^T
    else               write_tri<E, false, false>(rec + ws_half_bytes<E>(), Pm, nullptr, tid);
    __syncthreads();

    // ---- phase 4: 32x32 level.  Waves 0,1: block pair (a, b) = (2m, 2m+1): T_ba = -D_b (L_ba D_a)
    if (wave < 2) {
        const int ra = 32 * wave, rb = ra + 16;
        floatx4 y = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
        mma16(y, aquad(Lm, rb, ra, r, g), bquad(Tm, ra, ra, r, g));
        mma16(z, aquad(Tm, rb, rb, r, g), acc_as_quad(y));
#pragma unroll
        for (int e = 0; e < 4; ++e) Tm[(rb + 4 * g + e) * kLdm + ra + r] = -z[e];
    }
    __syncthreads();

    // ---- phase 5: 64x64 level.  T[32:64, 0:32] = -T22 (L21 T11); wave = (row tile ti, col tile tj)
    {
        const int ti = wave >> 1, tj = wave & 1;
        floatx4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const float4 b = bquad(Tm, 16 * tm, 16 * tj, r, g);
            mma16(y0, aquad(Lm, 32, 16 * tm, r, g), b);
            mma16(y1, aquad(Lm, 48, 16 * tm, r, g), b);
        }
        mma16(z, aquad(Tm, 32 + 16 * ti, 32, r, g), acc_as_quad(y0));
        mma16(z, aquad(Tm, 32 + 16 * ti, 48, r, g), acc_as_quad(y1));
        // the block written below is read by no wave in this phase, so no barrier is needed here
#pragma unroll
        for (int e = 0; e < 4; ++e) Tm[(32 + 16 * ti + 4 * g + e) * kLdm + 16 * tj + r] = -z[e];
    }
    __syncthreads();

    // ---- phase 6: T' = T diag(beta) (and T^T for the backward) -> workspace in operand order ------------------
    {
        char* out = rec;
        if constexpr (BWD) {
            write_tri<E, false, true>(out, Tm, beta_s, tid);
            write_tri<E, true, false>(out + ws_half_bytes<E>(), Tm, nullptr, tid);
        } else {
            write_tri<E, false, true>(out, Tm, beta_s, tid);
        }
    }
}

}  // namespace

// BWD = false: the forward's records [T' | P | three vectors].  BWD = true: the records of the backward pass,
// [T' | M^T | P^T | gamma_i | gamma_C/gamma_i | beta_i | 1/(||k_i||^2+eps)] with M = (I + L)^{-1}, T' = M B; the transposes are stored as the
// 6 upper-triangular tile-pairs (see bwd_record_bytes in kla_mma.hpp).
template <int DK, bool BWD>
__global__ __launch_bounds__(256) void intra_kernel(IntraArgs<bf16_t> a)
{
    typedef bf16_t E;
    constexpr int REC = BWD ? bwd_record_bytes<E>() : ws_record_bytes<E>();
    constexpr int PPR = DK * (int)sizeof(E) / 16;    // 16-byte pieces per row
    constexpr int EPP = 16 / (int)sizeof(E);         // elements per piece
    constexpr int KP = DK / 32;                      // contraction pairs per row
    constexpr int OPB = 64 * DK * (int)sizeof(E);    // bytes of one operand area

    __shared__ __attribute__((aligned(16))) char op_area[2 * OPB > 64 * kLdm * 4 ? 2 * OPB : 64 * kLdm * 4];
    __shared__ __attribute__((aligned(16))) float Lm[64 * kLdm];
    __shared__ __attribute__((aligned(16))) float Tm[64 * kLdm];
    __shared__ __attribute__((aligned(16))) float beta_s[64];
    __shared__ __attribute__((aligned(16))) float rq_s[64];      // 1/||q_i|| when the read-out is normalised, else 1
    __shared__ __attribute__((aligned(16))) float g_s[64];
    __shared__ __attribute__((aligned(16))) float invden_s[BWD ? 64 : 4];   // 1/(||k_i||^2 + eps), for the backward pass
    E* Krq = reinterpret_cast<E*>(op_area);
    E* Qrq = reinterpret_cast<E*>(op_area + OPB);
    float* Pm = reinterpret_cast<float*>(op_area);   // reused after the Gram products are in registers

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, g = lane >> 4;

    // ---- which chunk of which sequence -------------------------------------------------------
    const int h = blockIdx.x % a.H;
    const int cg = blockIdx.x / a.H;                 // global chunk index
    const ChunkPos cp = chunk_pos(a.cu_seqlens, a.chunk_off, a.n_seq, a.T, a.NT, cg);
    const long tok0 = cp.tok0;
    const int clen = cp.clen;

    // ---- phase 1: K, Q -> LDS (operand order), key norms -> beta, log-decay prefix sum -> g ---
    {
        const size_t row_stride = (size_t)a.H * DK;
        const E* kb = a.k + (size_t)tok0 * row_stride + (size_t)h * DK;
        const E* qb = a.q + (size_t)tok0 * row_stride + (size_t)h * DK;
#pragma unroll
        for (int it = 0; it < 64 * PPR / 256; ++it) {
            const int pi = tid + 256 * it;
            const int row = pi / PPR, piece = pi % PPR;
            uint4 kd = make_uint4(0, 0, 0, 0), qd = make_uint4(0, 0, 0, 0);
            if (row < clen) {
                kd = *reinterpret_cast<const uint4*>(kb + (size_t)row * row_stride + piece * EPP);
                qd = *reinterpret_cast<const uint4*>(qb + (size_t)row * row_stride + piece * EPP);
            }
            store_rq_piece(Krq, KP, row, piece, kd);
            store_rq_piece(Qrq, KP, row, piece, qd);
            auto sum_squares = [](uint4 d) {
                float ss = 0.f;
                const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const float x0 = bf16_bits_to_float(w[m] & 0xffffu), x1 = bf16_bits_to_float(w[m] >> 16);
                    ss += x0 * x0; ss += x1 * x1;
                }
                return ss;
            };
            float ss = sum_squares(kd), sq = sum_squares(qd);
#pragma unroll
            for (int off = 1; off < PPR; off <<= 1) { ss += __shfl_xor(ss, off, kWave); sq += __shfl_xor(sq, off, kWave); }
            if (piece == 0) {
                const float et = row < clen ? a.eta[(size_t)(tok0 + row) * a.H + h] : 0.f;
                beta_s[row] = (a.opts & kOptGdnBeta) ? et : kaczmarz_beta(et, ss, a.eps);
                // scale of the normalised read-out o_t = S_t^T q_t / ||q_t|| (Sec. 3.3); a zero query gives 0
                rq_s[row] = (a.opts & kOptNormalizeQ) ? (sq > 0.f ? 1.0f / sqrtf(sq) : 0.f) : 1.f;
                if constexpr (BWD) invden_s[row] = (a.opts & kOptGdnBeta) ? 1.f : ((ss + a.eps == 0.f) ? 0.f : 1.0f / (ss + a.eps));
            }
        }
        if (wave == 0) {
            float x = lane < clen ? a.log_alpha[(size_t)(tok0 + lane) * a.H + h] : 0.f;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const float y = __shfl_up(x, off, kWave);
                if (lane >= off) x += y;
            }
            g_s[lane] = x;
            if constexpr (!BWD) a.wsG[(size_t)blockIdx.x * 128 + lane] = x;
            // decay factors the scan stage multiplies with: gamma_i and gamma_C / gamma_i
            const float gl = __shfl(x, 63, kWave);
            float* dec = reinterpret_cast<float*>(reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC
                                                  + (BWD ? 3 : 2) * ws_half_bytes<E>());
            dec[lane] = expf(x);
            dec[64 + lane] = expf(gl - x);
        }
    }
    __syncthreads();
    if (wave == 0) {                                     // third vector of the record (and the scale itself)
        float* dec = reinterpret_cast<float*>(reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC
                                              + (BWD ? 3 : 2) * ws_half_bytes<E>());
        if constexpr (BWD) { dec[128 + lane] = beta_s[lane]; dec[192 + lane] = invden_s[lane]; dec[256 + lane] = rq_s[lane]; }
        else {
            dec[128 + lane] = expf(g_s[lane]) * rq_s[lane];
            a.wsG[(size_t)blockIdx.x * 128 + 64 + lane] = rq_s[lane];
        }
    }

    // ---- phase 2a: Gram products K K^T and Q K^T on the lower-triangular tiles ---------------
    floatx4 acc[5];
#pragma unroll
    for (int jb = 0; jb < 5; ++jb) {
        const int job = wave + 4 * jb;               // 0..9: K K^T tiles, 10..19: Q K^T tiles
        const int lt = job % 10;
        const int ti = kTileI[lt], tj = kTileJ[lt];
        const E* A = job < 10 ? Krq : Qrq;
        floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) {
            const Slot<E> sa = load_slot(A, ti * KP + kp, lane);
            const Slot<E> sb = load_slot(Krq, tj * KP + kp, lane);
            mma32<E>(c, sa, sb.q0, sb.q1);
        }
        acc[jb] = c;
    }
    __syncthreads();   // operand areas are dead from here on; Pm overlays them

    // ---- phase 2b: decay, mask, beta -> L and P as fp32 matrices; zero the upper tiles --------
#pragma unroll
    for (int jb = 0; jb < 5; ++jb) {
        const int job = wave + 4 * jb;
        const int lt = job % 10;
        const int ti = kTileI[lt], tj = kTileJ[lt];
        const int j = 16 * tj + r;
        const float gj = g_s[j];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * ti + 4 * g + e;
            const float gi = g_s[i];
            if (job < 10) {
                const float val = (j < i) ? beta_s[i] * expf(gi - gj) * acc[jb][e] : 0.f;
                Lm[i * kLdm + j] = val;
            } else {
                const float val = (j <= i) ? expf(gi - gj) * acc[jb][e] * rq_s[i] : 0.f;
                Pm[i * kLdm + j] = val;
            }
        }
    }
    for (int x = tid; x < 6 * 256; x += 256) {       // the six strictly-upper tiles
        const int t = x >> 8, e = x & 255;
        const int ti = t < 3 ? 0 : (t < 5 ? 1 : 2);
        const int tj = t < 3 ? t + 1 : (t < 5 ? t - 1 : 3);
        const int idx = (16 * ti + (e >> 4)) * kLdm + 16 * tj + (e & 15);
        Lm[idx] = 0.f; Pm[idx] = 0.f; Tm[idx] = 0.f;
    }
    __syncthreads();

    invert_and_store<E, BWD>(Lm, Tm, Pm, beta_s, reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC, tid);
}

hipError_t launch_intra(const IntraArgs<bf16_t>& a, int dk, int n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const dim3 grid((unsigned)n_chunks * a.H), block(256);
    if (dk == 64) hipLaunchKernelGGL((intra_kernel<64, false>), grid, block, 0, st, a);
    else          hipLaunchKernelGGL((intra_kernel<128, false>), grid, block, 0, st, a);
    return hipGetLastError();
}

// The records of the backward pass: a.wsT points at them, a.wsP and a.wsG are not used.  kOptGdnBeta: beta = eta, and
// the record's fourth vector, d beta / d eta, is 1; kOptNormalizeQ: P^T carries 1/||q_i||, which is also the fifth vector.
hipError_t launch_intra_bwd(const IntraArgs<bf16_t>& a, int dk, int n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const dim3 grid((unsigned)n_chunks * a.H), block(256);
    if (dk == 64) hipLaunchKernelGGL((intra_kernel<64, true>), grid, block, 0, st, a);
    else          hipLaunchKernelGGL((intra_kernel<128, true>), grid, block, 0, st, a);
    return hipGetLastError();
}

// ---- diagonal gating (App. B, "Extension to diagonal gating") -----------------------------------------------
// log_alpha holds d_k values per token and head; gamma_i is a vector and every decay ratio acts inside the inner
// products:  L_ij = beta_i sum_c k_ic k_jc gamma_ic/gamma_jc (j < i),  P_ij = sum_c q_ic k_jc gamma_ic/gamma_jc (j <= i).
// Every ratio is split at a reference row e with j <= e < i, gamma_i/gamma_j = [gamma_i/gamma_e][gamma_e/gamma_j], so
// that both factors are <= 1 (gamma itself may underflow inside a chunk; nothing can overflow): the off-diagonal
// 16x16 tiles and the lower-left 8x8 block of each diagonal tile become ordinary MFMA products of rescaled rows,
// formed in registers from fp32 tables of K, Q and the running log sums; only the 8x8 blocks on the diagonal are
// summed pair by pair on the vector ALUs (there gamma_i/gamma_j <= 1 directly).  The triangular inverse and the records are those of
// the scalar kernel, with unit decay vectors: the decay travels in the operands the scan is given instead,
//     K+ = K o Gamma,  Q+ = Q o Gamma,  K~ = K o (gamma_C / Gamma)   (all factors <= 1)  and gamma_C per channel,
// which this kernel writes next to the records.  Options: kOptGdnBeta (beta = eta); kOptNormalizeQ, for which the
// rows of Q+ and of P are divided by ||q_i|| here, so that the scan needs no variant of its own.
template <typename E, int DK>
__global__ __launch_bounds__(256, 3) void intra_diag_kernel(IntraDiagArgs<E> a)
{
    // The tables hold CH = 64 channels at a time: d_k = 128 takes two passes, whose partial sums meet in the registers
    // that hold the products.  That keeps the kernel at the LDS footprint of the 64x64 fp32 matrices of the later
    // phases (52.5 KB), i.e. three workgroups per CU instead of two.
    constexpr int CH = 64, NPASS = DK / CH;
    constexpr int EPP = 16 / (int)sizeof(E), PPR = DK / EPP, PPH = CH / EPP;
    constexpr int LE = CH + EPP;                     // row stride of the K, Q tables (elements): one 16-byte piece of padding
    constexpr int LD = CH + 4;                       // row stride of the log-sum table (floats)
    constexpr int TE = 64 * LE * (int)sizeof(E), TG = 64 * LD * 4;
    constexpr int NSEG = 256 / CH, SROWS = 64 / NSEG;   // the running sums: 256 threads = CH channels x NSEG row segments
    constexpr int REC = ws_record_bytes<E>();
    // bf16: alpha itself too, for the pair sums (with fp32 rows a fourth table would leave room for two workgroups per CU; there it is
    // formed from the running sums again)
    constexpr bool AT = sizeof(E) == 2;
    constexpr int TABLES = 2 * TE + TG + (AT ? 64 * CH * 4 : 0);
    __shared__ __attribute__((aligned(16))) char area[TABLES > 3 * 64 * kLdm * 4 ? TABLES : 3 * 64 * kLdm * 4];
    __shared__ __attribute__((aligned(16))) float beta_s[64];
    __shared__ __attribute__((aligned(16))) float rq_s[64];      // 1/||q_i|| for the normalised read-out (Sec. 3.3), else 1
    __shared__ float segsum[NSEG][CH];
    const E* Kp = reinterpret_cast<const E*>(area);           // K rows (element type), later overlaid by Lm, Pm, Tm
    const E* Qp = reinterpret_cast<const E*>(area + TE);      // Q rows
    float* Gs = reinterpret_cast<float*>(area + 2 * TE);      // running sums of log2 alpha per channel
    float* As = reinterpret_cast<float*>(area + 2 * TE + TG);
    float* Lm = reinterpret_cast<float*>(area);
    float* Pm = reinterpret_cast<float*>(area + 64 * kLdm * 4);
    float* Tm = reinterpret_cast<float*>(area + 2 * 64 * kLdm * 4);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = blockIdx.x % a.H;
    const int cg = blockIdx.x / a.H;
    const ChunkPos cp = a.pos_out ? chunk_pos_scan(a.cu_seqlens, a.n_seq, cg, lane, tid < 64 && blockIdx.x == 0 ? a.pos_out : nullptr)
                                  : chunk_pos(a.cu_seqlens, a.chunk_off, a.n_seq, a.T, a.NT, cg);
    const long tok0 = cp.tok0;
    const int clen = cp.clen;
    const size_t row_stride = (size_t)a.H * DK;
    auto unpack = [](uint4 d, float (&f)[EPP]) {
        if constexpr (sizeof(E) == 2) {
            const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int m = 0; m < 4; ++m) { f[2 * m] = bf16_bits_to_float(w[m] & 0xffffu); f[2 * m + 1] = bf16_bits_to_float(w[m] >> 16); }
        } else {
            f[0] = __uint_as_float(d.x); f[1] = __uint_as_float(d.y); f[2] = __uint_as_float(d.z); f[3] = __uint_as_float(d.w);
        }
    };
    auto pack = [](const float (&f)[EPP]) {
        if constexpr (sizeof(E) == 2)
            return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
        else
            return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    };

    auto ld4e = [](const E* p) {                     // 4 consecutive elements (8- resp. 16-byte aligned) as floats
        floatx4 f;
        if constexpr (sizeof(E) == 2) {
            const uint2 w = *reinterpret_cast<const uint2*>(p);
            f[0] = bf16_bits_to_float(w.x & 0xffffu); f[1] = bf16_bits_to_float(w.x >> 16);
            f[2] = bf16_bits_to_float(w.y & 0xffffu); f[3] = bf16_bits_to_float(w.y >> 16);
        } else {
            const float4 w = *reinterpret_cast<const float4*>(p);
            f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w;
        }
        return f;
    };
    auto ld4f = [](const float* p) { const float4 w = *reinterpret_cast<const float4*>(p); floatx4 f; f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w; return f; };

    const E* kb = a.k + (size_t)tok0 * row_stride + (size_t)h * DK;
    const E* qb = a.q + (size_t)tok0 * row_stride + (size_t)h * DK;
    const float* lb = a.log_alpha + (size_t)tok0 * row_stride + (size_t)h * DK;

    // ---- phase 0: the normalised read-out (Sec. 3.3) needs 1/||q_i|| over all channels before the first pass scales
    //      Q; otherwise nothing is read ahead of the passes (the key norms are summed up pass by pass)
    if (a.opts & kOptNormalizeQ) {
#pragma unroll
        for (int it = 0; it < 64 * PPR / 256; ++it) {
            const int pi = tid + 256 * it;
            const int row = pi / PPR, piece = pi % PPR;
            uint4 qd = make_uint4(0, 0, 0, 0);
            if (row < clen) qd = *reinterpret_cast<const uint4*>(qb + (size_t)row * row_stride + piece * EPP);
            float qf0[EPP];
            unpack(qd, qf0);
            float sq = 0.f;
#pragma unroll
            for (int i = 0; i < EPP; ++i) sq += qf0[i] * qf0[i];
#pragma unroll
            for (int off = 1; off < PPR; off <<= 1) sq += __shfl_xor(sq, off, kWave);
            if (piece == 0) rq_s[row] = sq > 0.f ? 1.0f / sqrtf(sq) : 0.f;
        }
    } else if (tid < 64) rq_s[tid] = 1.f;
    if (tid < 128) {                                 // unit decay vectors for the scan: g = 0, 1/||q|| = 1
        a.wsG[(size_t)blockIdx.x * 128 + tid] = tid < 64 ? 0.f : 1.f;
        float* dec = reinterpret_cast<float*>(reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC + 2 * ws_half_bytes<E>());
        dec[tid] = 1.f;
        if (tid < 64) dec[128 + tid] = 1.f;
    }

    // accumulators of phase 2a, over all passes
    const int r = lane & 15, g = lane >> 4;
    floatx4 tkk[2], tqk[2];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) { tkk[jb] = floatx4{0.f, 0.f, 0.f, 0.f}; tqk[jb] = tkk[jb]; }
    // The MFMA jobs of phase 2a, two per wave: the six off-diagonal tiles (ti, tj), split at e = the last row before tile ti, so
    // that the A operands do not depend on tj: waves 0 and 1 take two tiles of a row each and form them once; and two
    // jobs of which each takes the lower-left 8x8 blocks of TWO diagonal tiles (2 d and the next) in one 16x16 product - operand rows
    // 0..7 belong to the first tile, rows 8..15 to the second, and the two off-diagonal 8x8 blocks of the result are not used.
    //     wave 0: (3,0) (3,1)    wave 1: (2,0) (2,1)    wave 2: (3,2), d = 0    wave 3: (1,0), d = 1
    const bool same_a = wave < 2;
    auto job_tile = [&](int jb, int& ti, int& tj) {          // (not of the two jobs on the diagonal: wave >= 2, jb = 1)
        ti = wave == 1 ? 2 : (wave == 3 ? 1 : 3);
        tj = wave == 2 ? 2 : (wave == 3 ? 0 : jb);
    };
    // Per lane: the table row of its A operand row (ja), of its B operand row (jbr) and of the reference row.
    auto job_rows = [&](int jb, int r, int& ja, int& jbr, int& e) {
        if (wave < 2 || jb == 0) {
            int ti, tj;
            job_tile(jb, ti, tj);
            ja = 16 * ti + r; jbr = 16 * tj + r; e = 16 * ti - 1;
        } else {
            const int t = 2 * (wave - 2) + (r >> 3);         // the diagonal tile this lane's operand rows belong to
            ja = 16 * t + 8 + (r & 7); jbr = 16 * t + (r & 7); e = 16 * t + 7;
        }
    };
    // The 8x8 blocks on the diagonal: a thread takes eight channels of a pass and, of one block, the pairs of two columns, j = m with
    // the 7 - m rows below it and j = 7 - m with the m below that one: seven steps down the rows, k_j multiplied by alpha on
    // the way, so a pair costs three operations per channel. (One pair per thread over all channels, gamma_i/gamma_j an exponential
    // each, was a third of the kernel's instructions: with the running sums in registers,
    // two shared A operands and the zeros of phase 2b only where they are read 137 -> 120 us for 4096 chunk-heads of d_k = 128, 4.5 TB/s.)
    struct Pairs {
        int cg8, m, b;                                       // channel group, column pair, first row of the block
        __device__ __forceinline__ Pairs(int lane, int wave) : cg8(lane & 7), m((lane >> 3) & 3), b(8 * (2 * wave + (lane >> 5))) {}
        __device__ __forceinline__ int row(int x) const { return b + x + 1 + (x < 7 - m ? m : 0); }      // i of step x
        __device__ __forceinline__ int col(int x) const { return b + (x < 7 - m ? m : 7 - m); }          // j
    };
    float skk[7], sqk[7], sdg[2] = {0.f, 0.f};               // sdg: q_i . k_i of rows m and 7 - m
#pragma unroll
    for (int x = 0; x < 7; ++x) { skk[x] = 0.f; sqk[x] = 0.f; }

    float ksq[64 * PPH / 256];                       // this thread's share of ||k_row||^2, rows (tid + 256 it) / PPH
#pragma unroll
    for (int it = 0; it < 64 * PPH / 256; ++it) ksq[it] = 0.f;
    // A pass's rows of K, Q and log alpha come from memory into registers (fetch) and go on into the tables once the
    // pass before has read them; the fetch of the next pass is issued ahead of the last, long, lightly loaded phase of
    // a pass, so that a workgroup waits for memory once, not once per pass.
    constexpr int NKQ = 64 * PPH / 256, NLA = 64 * CH / 4 / 256;
    uint4 kd[NKQ], qd[NKQ];
    float4 lad[NLA];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int it = 0; it < NKQ; ++it) {
            const int x = tid + 256 * it;
            const int row = x / PPH, piece = x % PPH;
            kd[it] = make_uint4(0, 0, 0, 0); qd[it] = make_uint4(0, 0, 0, 0);
            if (row < clen) {
                kd[it] = *reinterpret_cast<const uint4*>(kb + (size_t)row * row_stride + c0 + piece * EPP);
                qd[it] = *reinterpret_cast<const uint4*>(qb + (size_t)row * row_stride + c0 + piece * EPP);
            }
        }
#pragma unroll
        for (int it = 0; it < NLA; ++it) {
            const int x = tid + 256 * it, row = x / (CH / 4), c4 = x % (CH / 4);
            lad[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < clen) lad[it] = *reinterpret_cast<const float4*>(lb + (size_t)row * row_stride + c0 + 4 * c4);
        }
    };
    constexpr bool AHEAD = sizeof(E) == 2;           // fp32 rows are twice the registers: fetched pass by pass
    if constexpr (AHEAD) fetch(0);
    float et[NKQ];                                   // of the rows whose norms this thread ends up with
#pragma unroll
    for (int it = 0; it < NKQ; ++it) {
        const int x = tid + 256 * it, row = x / PPH;
        et[it] = x % PPH == 0 && row < clen ? a.eta[(size_t)(tok0 + row) * a.H + h] : 0.f;
    }
    for (int pass = 0; pass < NPASS; ++pass) {
        const int c0 = pass * CH;                    // first channel of this pass
        // a lane index that the compiler cannot see through: the addresses of a pass are formed in it, not kept over all of them
        int tv = threadIdx.x;
        asm volatile("" : "+v"(tv));
        const int tid = tv, lane = tid & 63, r = lane & 15, g = lane >> 4;
        const Pairs pr(lane, wave);
        if (pass > 0) __syncthreads();               // the previous pass has read its tables
        if constexpr (!AHEAD) fetch(c0);
        // ---- phase 1: K, Q rows and log2 alpha of CH channels -> LDS (the squares of K summed for the key norms on the way)
#pragma unroll
        for (int it = 0; it < NKQ; ++it) {
            const int x = tid + 256 * it;
            const int row = x / PPH, piece = x % PPH;
            *reinterpret_cast<uint4*>(area + (size_t)(row * LE + piece * EPP) * sizeof(E)) = kd[it];
            *reinterpret_cast<uint4*>(area + TE + (size_t)(row * LE + piece * EPP) * sizeof(E)) = qd[it];
            float kf[EPP];
            unpack(kd[it], kf);
#pragma unroll
            for (int i = 0; i < EPP; ++i) ksq[it] += kf[i] * kf[i];
        }
#pragma unroll
        for (int it = 0; it < NLA; ++it) {
            const int x = tid + 256 * it, row = x / (CH / 4), c4 = x % (CH / 4);
            const float4 v = lad[it];
            const float s2 = 1.44269504088896341f;
            const float4 l2 = make_float4(v.x * s2, v.y * s2, v.z * s2, v.w * s2);
            *reinterpret_cast<float4*>(Gs + row * LD + 4 * c4) = l2;
            if constexpr (AT)
                *reinterpret_cast<float4*>(As + row * CH + 4 * (c4 ^ (row & 15))) =
                    make_float4(__builtin_amdgcn_exp2f(l2.x), __builtin_amdgcn_exp2f(l2.y), __builtin_amdgcn_exp2f(l2.z), __builtin_amdgcn_exp2f(l2.w));
        }
        __syncthreads();
        {   // per channel: running sum over the tokens of the chunk, NSEG row segments side by side, then their offsets
            const int c = tid % CH, sg = tid / CH;
            float* col = Gs + sg * SROWS * LD + c;
            float acc[SROWS];
#pragma unroll
            for (int i = 0; i < SROWS; ++i) acc[i] = col[i * LD];
#pragma unroll
            for (int i = 1; i < SROWS; ++i) acc[i] += acc[i - 1];
            segsum[sg][c] = acc[SROWS - 1];
            __syncthreads();
            float base = 0.f;
            for (int s2 = 0; s2 < sg; ++s2) base += segsum[s2][c];
#pragma unroll
            for (int i = 0; i < SROWS; ++i) col[i * LD] = acc[i] + base;
            if (sg == NSEG - 1) a.gc[(size_t)blockIdx.x * DK + c0 + c] = __builtin_amdgcn_exp2f(base + acc[SROWS - 1]);      // gamma_C
        }
        __syncthreads();

        // ---- phase 1b: the scan's operands K+, Q+, K~ in the element type -------------------------------------
        {
            E* kpo = a.kplus + (size_t)tok0 * row_stride + (size_t)h * DK + c0;
            E* qpo = a.qplus + (size_t)tok0 * row_stride + (size_t)h * DK + c0;
            E* kto = a.ktilde + (size_t)tok0 * row_stride + (size_t)h * DK + c0;
#pragma unroll
            for (int it = 0; it < 64 * PPH / 256; ++it) {
                const int x = tid + 256 * it;
                const int row = x / PPH, piece = x % PPH;
                if (row < clen) {
                    float kf[EPP], qf[EPP], kp[EPP], qp[EPP], kt[EPP];
                    unpack(*reinterpret_cast<const uint4*>(area + (size_t)(row * LE + piece * EPP) * sizeof(E)), kf);
                    unpack(*reinterpret_cast<const uint4*>(area + TE + (size_t)(row * LE + piece * EPP) * sizeof(E)), qf);
#pragma unroll
                    for (int i = 0; i < EPP; ++i) {
                        const float gi = Gs[row * LD + piece * EPP + i], gl = Gs[63 * LD + piece * EPP + i];
                        const float up = __builtin_amdgcn_exp2f(gi);
                        kp[i] = kf[i] * up; qp[i] = qf[i] * (up * rq_s[row]); kt[i] = kf[i] * __builtin_amdgcn_exp2f(gl - gi);
                    }
                    const size_t off = (size_t)row * row_stride + piece * EPP;
                    typedef uint32_t u32x4n __attribute__((ext_vector_type(4)));
                    auto nts = [](E* p, uint4 v) { const u32x4n w = {v.x, v.y, v.z, v.w}; __builtin_nontemporal_store(w, reinterpret_cast<u32x4n*>(p)); };
                    nts(kpo + off, pack(kp));
                    nts(qpo + off, pack(qp));
                    nts(kto + off, pack(kt));
                }
            }
        }
        // (no barrier: phase 2a only reads the tables, like phase 1b)

        // ---- phase 2a: K K^T and Q K^T with the decay ratios inside the sums, the channels of this pass ---------
        // (1) MFMA jobs, operands formed in registers from the tables: A row i = k_i (or q_i) o gamma_i/gamma_e, B row
        //     j = k_j o gamma_e/gamma_j, every factor <= 1.
        // (2) the 8x8 blocks on the diagonal, pair by pair on the vector ALUs.
#pragma unroll 1
        for (int kp = 0; kp < CH / 32; ++kp) {
            Slot<E> sk, sq;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
                int ja, jbr, e;
                job_rows(jb, r, ja, jbr, e);
                const float* ge = Gs + e * LD;
                if (jb == 0 || !same_a) {
                    const float* gi = Gs + ja * LD;
                    const E* ki = Kp + ja * LE;
                    const E* qi = Qp + ja * LE;
                    floatx4 ka[2], qa[2];
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk) {
                        const int c = 32 * kp + 16 * blk + 4 * g;
                        const floatx4 gev = ld4f(ge + c), giv = ld4f(gi + c), kiv = ld4e(ki + c), qiv = ld4e(qi + c);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            const float up = __builtin_amdgcn_exp2f(giv[x] - gev[x]);      // gamma_i / gamma_e <= 1
                            ka[blk][x] = kiv[x] * up; qa[blk][x] = qiv[x] * up;
                        }
                    }
                    sk.q0 = acc_to_quad<E>(ka[0]); sk.q1 = acc_to_quad<E>(ka[1]);
                    sq.q0 = acc_to_quad<E>(qa[0]); sq.q1 = acc_to_quad<E>(qa[1]);
                }
                const float* gj = Gs + jbr * LD;
                const E* kj = Kp + jbr * LE;
                floatx4 kbv[2];
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    const int c = 32 * kp + 16 * blk + 4 * g;
                    const floatx4 gev = ld4f(ge + c), gjv = ld4f(gj + c), kjv = ld4e(kj + c);
#pragma unroll
                    for (int x = 0; x < 4; ++x) kbv[blk][x] = kjv[x] * __builtin_amdgcn_exp2f(gev[x] - gjv[x]);      // gamma_e / gamma_j <= 1
                }
                const typename QuadT<E>::type b0 = acc_to_quad<E>(kbv[0]), b1 = acc_to_quad<E>(kbv[1]);
                mma32<E>(tkk[jb], sk, b0, b1);
                mma32<E>(tqk[jb], sq, b0, b1);
            }
        }
        if constexpr (AHEAD) { if (pass + 1 < NPASS) fetch(c0 + CH); }   // on their way during the pair sums
#pragma unroll 1
        for (int c4 = 0; c4 < 2; ++c4) {                 // this thread's channels: 4 cg8 .. + 3 and 32 more
            const int c = 32 * c4 + 4 * pr.cg8;
            floatx4 w = ld4e(Kp + (pr.b + pr.m) * LE + c);
            const floatx4 k2 = ld4e(Kp + (pr.b + 7 - pr.m) * LE + c);
            const floatx4 q1 = ld4e(Qp + (pr.b + pr.m) * LE + c), q2 = ld4e(Qp + (pr.b + 7 - pr.m) * LE + c);
#pragma unroll
            for (int x = 0; x < 4; ++x) { sdg[0] += q1[x] * w[x]; sdg[1] += q2[x] * k2[x]; }
            static_for<7>([&](auto sc) {
                constexpr int st = sc;
                const int i = pr.row(st);
                if constexpr (st >= 4) { if (st == 7 - pr.m) w = k2; }
                floatx4 al;
                if constexpr (AT) al = ld4f(As + i * CH + 4 * ((8 * c4 + pr.cg8) ^ (i & 15)));
                else {
                    const floatx4 g1 = ld4f(Gs + i * LD + c), g0 = ld4f(Gs + (i - 1) * LD + c);
#pragma unroll
                    for (int x = 0; x < 4; ++x) al[x] = __builtin_amdgcn_exp2f(g1[x] - g0[x]);
                }
                const floatx4 kv = ld4e(Kp + i * LE + c), qv = ld4e(Qp + i * LE + c);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    w[x] *= al[x];
                    skk[st] += kv[x] * w[x]; sqk[st] += qv[x] * w[x];
                }
            });
        }
    }
    // over the eight threads of a block's column pair (exchange with lane ^ 1, ^ 2, then the mirror of eight lanes)
    auto sum8 = [](float v) {
        v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));     // quad_perm [1,0,3,2]
        v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true));     // quad_perm [2,3,0,1]
        v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, true));    // row_half_mirror
        return v;
    };
#pragma unroll
    for (int x = 0; x < 7; ++x) { skk[x] = sum8(skk[x]); sqk[x] = sum8(sqk[x]); }
    sdg[0] = sum8(sdg[0]); sdg[1] = sum8(sdg[1]);
    // ---- beta of eq. (3) from the key norms (the PPH threads of a row sit in consecutive lanes)
#pragma unroll
    for (int it = 0; it < 64 * PPH / 256; ++it) {
        const int x = tid + 256 * it;
        const int row = x / PPH;
        float ss = ksq[it];
#pragma unroll
        for (int off = 1; off < PPH; off <<= 1) ss += __shfl_xor(ss, off, kWave);
        if (x % PPH == 0) {
            beta_s[row] = (a.opts & kOptGdnBeta) ? et[it] : kaczmarz_beta(et[it], ss, a.eps);
        }
    }
    __syncthreads();   // the tables are dead from here on; Lm, Pm, Tm overlay them

    // ---- phase 2b: beta -> L and P.  What is read besides the products must be zero: of P the diagonal tiles and the tiles (0,1) and
    //      (2,3) to their right (tile-pairs are stored whole), of T' these two; of L only the strict lower triangle is read.
    for (int x = tid; x < 512; x += 256) {
        const int t = x >> 6, row = (x >> 2) & 15, c4 = x & 3;                                  // eight 16x16 tiles
        const int ti = t < 4 ? t : (t & 1) * 2, tj = t < 4 ? t : ti + 1;
        *reinterpret_cast<float4*>((t < 6 ? Pm : Tm) + (16 * ti + row) * kLdm + 16 * tj + 4 * c4) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int il = 4 * g + e;                // row inside the product tile; its column is r
            int i, j; bool ok;
            if (wave < 2 || jb == 0) {
                int ti, tj;
                job_tile(jb, ti, tj);
                i = 16 * ti + il; j = 16 * tj + r; ok = true;
            } else {                                 // the two diagonal 8x8 blocks of the product
                const int t = 2 * (wave - 2) + (il >> 3);
                i = 16 * t + 8 + (il & 7); j = 16 * t + (r & 7); ok = (il >> 3) == (r >> 3);
            }
            if (ok) {
                Lm[i * kLdm + j] = beta_s[i] * tkk[jb][e];
                Pm[i * kLdm + j] = tqk[jb][e] * rq_s[i];
            }
        }
    }
    const Pairs pr(lane, wave);
    if (pr.cg8 == 0) {
#pragma unroll
        for (int x = 0; x < 7; ++x) {
            const int i = pr.row(x), j = pr.col(x);
            Lm[i * kLdm + j] = beta_s[i] * skk[x]; Pm[i * kLdm + j] = sqk[x] * rq_s[i];
        }
        Pm[(pr.b + pr.m) * (kLdm + 1)] = sdg[0] * rq_s[pr.b + pr.m];
        Pm[(pr.b + 7 - pr.m) * (kLdm + 1)] = sdg[1] * rq_s[pr.b + 7 - pr.m];
    }
    __syncthreads();
    invert_and_store<E, false>(Lm, Tm, Pm, beta_s, reinterpret_cast<char*>(a.wsT) + (size_t)blockIdx.x * REC, tid);
}

template <typename E>
hipError_t launch_intra_diag(const IntraDiagArgs<E>& a, int dk, int n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const dim3 grid((unsigned)n_chunks * a.H), block(256);
    if (dk == 64) hipLaunchKernelGGL((intra_diag_kernel<E, 64>), grid, block, 0, st, a);
    else          hipLaunchKernelGGL((intra_diag_kernel<E, 128>), grid, block, 0, st, a);
    return hipGetLastError();
}
template hipError_t launch_intra_diag<float>(const IntraDiagArgs<float>&, int, int, hipStream_t);
template hipError_t launch_intra_diag<bf16_t>(const IntraDiagArgs<bf16_t>&, int, int, hipStream_t);

// ---- chunk offsets of a packed batch: chunk_off[s] = sum_{s'<s} ceil(len_s'/64), and the order in which the sweeps take
//      the sequences: most chunks first, so that the workgroups that run longest start first and the short ones fill
//      the CUs that become free (up to kOrderMax sequences; more of them balance by number, keep their order, and `order` is NULL).
__global__ __launch_bounds__(256) void chunk_offsets_kernel(const int* __restrict__ cu_seqlens, int n_seq, int* __restrict__ chunk_off,
                                                            int* __restrict__ order)
{
    static_assert(kOrderMax <= 256, "a thread per sequence");
    __shared__ int nc_s[256];
    __shared__ int wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int carry = 0;
    for (int s0 = 0; s0 < n_seq; s0 += 256) {            // 256 sequences at a time: prefix sum in each wave, then over the waves
        const int s = s0 + tid;
        const int nc = s < n_seq ? (cu_seqlens[s + 1] - cu_seqlens[s] + 63) / 64 : 0;
        int x = nc;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) { const int y = __shfl_up(x, off, kWave); if (lane >= off) x += y; }
        if (lane == 63) wsum[wave] = x;
        nc_s[tid] = nc;
        __syncthreads();
        int base = carry;
        for (int w = 0; w < wave; ++w) base += wsum[w];
        if (s < n_seq) chunk_off[s] = base + x - nc;
        carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
        if (order && s < n_seq) {                        // one pass: n_seq <= 256
            int rank = 0;
            for (int j = 0; j < n_seq; ++j) rank += (nc_s[j] > nc || (nc_s[j] == nc && j < s)) ? 1 : 0;
            order[rank] = s;
        }
        __syncthreads();
    }
    if (tid == 0) chunk_off[n_seq] = carry;
}
hipError_t launch_chunk_offsets(const int* cu_seqlens, int n_seq, int* chunk_off, int* order, hipStream_t st)
{
    hipLaunchKernelGGL(chunk_offsets_kernel, dim3(1), dim3(256), 0, st, cu_seqlens, n_seq, chunk_off, order);
    return hipGetLastError();
}

// ---- test hook: unpack operand-order T', P to plain row-major fp32 ---------------------------
template <typename E>
__global__ void unpack_kernel(const E* __restrict__ wsT, const E* __restrict__ wsP, const float* __restrict__ wsG,
                              float* __restrict__ Tb, float* __restrict__ P, float* __restrict__ gout, long n_ch)
{
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n_ch * 4096) return;
    const long ch = idx >> 12;
    const int i = (int)((idx >> 6) & 63), j = (int)(idx & 63);
    const int ti = i >> 4, jp = j >> 5, ln = (i & 15) + 16 * ((j & 15) >> 2);
    const bool stored = jp <= (ti >> 1);             // only the lower-triangular tile-pairs exist
    const size_t e = (size_t)ch * (ws_record_bytes<E>() / sizeof(E)) + ((size_t)tri_pair(ti, jp) * 64 + ln) * 8 + ((j >> 4) & 1) * 4 + (j & 3);
    Tb[idx] = stored ? to_float(wsT[e]) : 0.f;
    P[idx] = stored ? to_float(wsP[e]) : 0.f;
    if (j == 0) gout[ch * 64 + i] = wsG[ch * 128 + i];
}
template <typename E>
hipError_t launch_unpack(const E* wsT, const E* wsP, const float* wsG, float* Tb, float* P, float* gout, long n_ch,
                         hipStream_t st)
{
    if (n_ch == 0) return hipSuccess;
    const long n = n_ch * 4096;
    hipLaunchKernelGGL((unpack_kernel<E>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, wsT, wsP, wsG, Tb, P,
                       gout, n_ch);
    return hipGetLastError();
}
template hipError_t launch_unpack<float>(const float*, const float*, const float*, float*, float*, float*, long, hipStream_t);
template hipError_t launch_unpack<bf16_t>(const bf16_t*, const bf16_t*, const float*, float*, float*, float*, long, hipStream_t);

}  // namespace kla
