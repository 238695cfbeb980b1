// C ABI of the library (declared in include/kla.h): argument validation, workspace carving and
// launch sequencing.  No allocation, no state but the per-device address of the static scratch array, nothing read
// from the environment; everything is enqueued on the caller's stream.
#include <math.h>

#include <mutex>

#include "../../include/kla.h"
#include "kla_kernels.hpp"
#include "kla_widths.hpp"

namespace {

using kla::bf16_t;
using kla::busiest_cu;
using kla::Lengths;

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }
inline bool dk_ok(int dk) { return dk == 64 || dk == 128; }
inline bool dv_ok(int dv) { return dv == 64 || dv == 128 || dv == 256; }
inline bool dt_ok(int dt) { return dt == KLA_F32 || dt == KLA_BF16; }
inline size_t elem_bytes(int dt) { return dt == KLA_BF16 ? 2 : 4; }

static_assert(KLA_OPT_NORMALIZE_Q == (int)kla::kOptNormalizeQ && KLA_OPT_GDN_BETA == (int)kla::kOptGdnBeta, "option bits");

// The tuning fields of the `opts` argument (KLA_TUNE_* in include/kla.h), decoded.  Zero everywhere = the library's choice.
struct Tune {
    int scan_waves = 0;      // 1, 2, 4 compute waves per scan workgroup
    int segments = 0;        // 1 = never cut sequences into segments, n = cut into n
    bool generic_scan = false, generic_intra = false, generic_bwd = false, unfused = false, fused = false;
    int decode_slice = 0;    // 32, 64, 128, 256 state columns per decode workgroup
    int decode_nt = -1;      // bit 0: non-temporal state loads, bit 1: non-temporal state stores
};
constexpr unsigned kOptMask = KLA_OPT_NORMALIZE_Q | KLA_OPT_GDN_BETA;
constexpr unsigned kTuneMask = 0x03ffff00u;

bool parse_tune(unsigned opts, Tune* t)
{
    if (opts & ~(kOptMask | kTuneMask)) return false;
    const unsigned w = (opts >> 8) & 3u, sg = (opts >> 10) & 31u, ds = (opts >> 18) & 7u, nt = (opts >> 21) & 7u;
    if (sg > 16 || ds > 4 || nt > 4) return false;
    t->scan_waves = w == 0 ? 0 : (w == 3 ? 4 : (int)w);
    t->segments = (int)sg;
    t->generic_scan = (opts & KLA_TUNE_GENERIC_SCAN) != 0;
    t->generic_intra = (opts & KLA_TUNE_GENERIC_INTRA) != 0;
    t->generic_bwd = (opts & KLA_TUNE_GENERIC_BWD) != 0;
    t->unfused = (opts & KLA_TUNE_UNFUSED) != 0;
    t->fused = (opts & KLA_TUNE_FUSED) != 0;
    if (t->fused && t->unfused) return false;
    t->decode_slice = ds == 0 ? 0 : 16 << ds;
    t->decode_nt = nt == 0 ? -1 : (int)nt - 1;
    return true;
}

struct Plan {
    long n_chunks;       // over all sequences
    int n_states;        // sequences
    size_t off_T, off_P, off_G, off_C, off_M, off_S, total;
    size_t order_bytes;  // of these, what the scan order of a packed batch adds
    int seg_G, seg_Lc;   // segment-parallel scan: segments per sequence (1 = off) and chunks per segment
    Lengths seqs;        // (cu: the caller's, for the length of the call)
    bool rows;           // bf16 only: the scan that splits a chunk by rows
    bool fused;          // bf16 only: one kernel, no intra-chunk stage, nothing in the workspace
    int fwd_seg_G;       // make_bwd_plan only: the forward's segments (seg_G are the backward's there)
    Tune tune;
};

// Segments per sequence for the scan stage.  A small fixed-length bf16 batch of long sequences (at most 128
// sixteen-column chains, at least 64 chunks) is cut until max_chains sixteen-column chains run, into segments of at least
// 16 chunks.  Forward: 1024 of them, 256 workgroups of four compute waves; 512, workgroups of two, where the value head
// is narrow and the maps' d_k more columns weigh most (one 65K sequence of 8 heads 345 against 414 us, 8192 tokens of
// d_v = 256 84 against 98 us; 2 x 16K tokens of d_v = 64 154 against 137 us).  Backward: 512, its segmented sweeps
// have two compute waves at most.  Beyond 16 segments their serial composition outweighs the shorter scans (32K tokens of 4 heads: 139 us
// with 32, 128 us with 16).  The tuning field KLA_TUNE_SCAN_SEGMENTS(n) forces n (1 = never).  Returns the number of
// non-empty segments and sets the chunks per segment.
int plan_segments(int N, int NT, int H, int dv, int dt, int n_seq, const Tune& tune, int max_chains, int* Lc)
{
    *Lc = NT;
    if (dt != KLA_BF16 || n_seq > 0 || N <= 0 || NT < 2) return 1;
    if (tune.generic_scan) return 1;                 // generic kernels: never
    const long groups = (long)N * H * (dv / 16);
    int want = 1;
    if (tune.segments >= 1) want = tune.segments;
    else if (groups <= 128 && NT >= 64) {
        while (want < 16 && (long)want * 2 * groups <= max_chains && NT / (want * 2) >= 16) want *= 2;
    }
    if (want > NT) want = NT;
    if (want <= 1) return 1;
    const int lc = (NT + want - 1) / want;
    const int G = (NT + lc - 1) / lc;
    if (G <= 1) return 1;
    *Lc = lc;
    return G;
}

int scan_waves(const Lengths& seqs, int H, int dv, int dt, bool saves, const Tune& tune);

// Packed batches: the order in which the scans take the sequences, behind the n_seq + 1 chunk offsets.  More than
// kla::kOrderMax sequences have none: they are taken as they come.
inline int order_ints(int n_seq) { return n_seq <= kla::kOrderMax ? n_seq : 0; }
inline int* order_at(int* chunk_off, int n_seq) { return order_ints(n_seq) > 0 ? chunk_off + n_seq + 1 : nullptr; }

// fp32 sweeps (kla_chunk_sweeps_f32.hip): column tiles per workgroup.  Four waves share a tile whatever the number; with
// more tiles than CUs two per workgroup halve the LDS reads of every product, with fewer they would leave CUs idle.
inline int f32_tiles(long n_tiles) { return n_tiles > 256 ? 2 : 1; }

// Validates the size arguments shared by the chunk entry points and lays out the workspace.
int make_plan(int N, int T, int H, int dk, int dv, int chunk, int dt, const int32_t* cu_host, int n_seq, unsigned opts, Plan* p)
{
    if (!parse_tune(opts, &p->tune)) return KLA_ERR_SHAPE;
    if (!dt_ok(dt)) return KLA_ERR_DTYPE;
    if (N < 0 || T < 0 || H <= 0 || n_seq < 0 || !dk_ok(dk) || !dv_ok(dv) || chunk != 64) return KLA_ERR_SHAPE;
    long n_chunks = 0;
    if (n_seq > 0) {
        if (N != 1) return KLA_ERR_SHAPE;
        if (!cu_host) return KLA_ERR_NULL;
        if (cu_host[0] != 0) return KLA_ERR_SEQLENS;
        for (int s = 0; s < n_seq; ++s) {
            if (cu_host[s + 1] < cu_host[s]) return KLA_ERR_SEQLENS;
            n_chunks += (cu_host[s + 1] - cu_host[s] + 63) / 64;
        }
        if (cu_host[n_seq] != T) return KLA_ERR_SEQLENS;
        p->n_states = n_seq;
    } else {
        if (cu_host) return KLA_ERR_SHAPE;
        n_chunks = (long)N * ((T + 63) / 64);
        p->n_states = N;
    }
    if (n_chunks * H > 0x7fffffffL || (long)p->n_states * H * (dv / 16) > 0x7fffffffL) return KLA_ERR_SHAPE;
    p->n_chunks = n_chunks;
    // per chunk-head one record [T' | P], each 6 tile-pairs x 64 slots of 8 elements
    const size_t half = (size_t)384 * 8 * elem_bytes(dt);
    p->off_T = 0;
    p->off_P = half;
    p->off_G = round256((size_t)n_chunks * H * (2 * half + 768));   // + three vectors of 64 fp32 (see kla_mma.hpp)
    p->off_C = round256(p->off_G + (size_t)n_chunks * H * 128 * sizeof(float));      // g and 1/||q||
    p->off_M = round256(p->off_C + (size_t)(n_seq + 1 + order_ints(n_seq)) * sizeof(int32_t));   // chunk offsets, scan order of the sequences
    p->order_bytes = p->off_M - round256(p->off_C + (size_t)(n_seq + 1) * sizeof(int32_t));
    auto segments = [&](int max_chains) {
        p->seg_G = plan_segments(N, (T + 63) / 64, H, dv, dt, n_seq, p->tune, max_chains, &p->seg_Lc);
        // per (sequence, head): G - 1 maps [N | M] and G incoming states, fp32
        const size_t maps = p->seg_G > 1 ? (size_t)N * (p->seg_G - 1) * H * dk * (dv + dk) * sizeof(float) : 0;
        const size_t states = p->seg_G > 1 ? (size_t)N * p->seg_G * H * dk * dv * sizeof(float) : 0;
        p->off_S = round256(p->off_M + maps);
        p->total = round256(p->off_S + states);
    };
    segments(dv >= 128 ? 1024 : 512);
    if (p->total > (size_t)KLA_STATIC_SCRATCH_BYTES && p->seg_G > 1) {
        // the larger number of segments is not to put a batch out of reach of the entry point with the fixed scratch, nor
        // to make that entry point's results differ from this one's
        const size_t all = p->total;
        segments(512);
        if (p->total > (size_t)KLA_STATIC_SCRATCH_BYTES && p->total != all) segments(dv >= 128 ? 1024 : 512);
    }
    p->seqs = {p->n_states, (T + 63) / 64, cu_host};
    // Up to 256 chains of sixteen columns each have a CU to themselves: the scan that shares a chain among the waves of one (8
    // heads of 128 columns, 700 tokens: 17.7 against 20.3 us; 256 chains, 4 x 1000 tokens of 8 heads: 26.6 against 28.8; 384: 35.7
    // against 26.0).  Same bits.
    p->rows = dt == KLA_BF16 && !p->tune.scan_waves && !p->tune.generic_scan && ((long)p->n_states * H + 7) / 8 * 8 * (dv / 16) <= 256;
    // The fused kernel (two compute waves per workgroup) keeps the per-chunk objects on chip and needs nothing of the
    // workspace (a token size is still reported and asked for).  It runs batches of 384 to 2047 chains of sixteen state
    // columns with d_v <= 128 (8 x 8 heads x 4096 tokens: 116 against 124 us); below that its helper waves redo the
    // per-chunk work too often (one 65K sequence, unsegmented: 1.83 against 1.38 ms).  The line is part of what a call
    // returns and does not follow speed alone: the two forms round different things to 16 bits - here the off-diagonal
    // blocks of L, which the intra-chunk stage inverts in fp32, there X = V - D_gamma K S - and neither is the closer one
    // everywhere.  Measured against 64 bits, final state, fused / two kernels: 200 tokens of 8 heads, correlated keys and
    // slow decay 5.1e-3 / 3.8e-3; 9 x 300 tokens of 8 heads, independent keys 2.5e-3 / 3.0e-3 (o: within 8 % of each other).
    // A batch without a token (whose inputs may be NULL) only hands its states on: the plain scan does that.
    // KLA_TUNE_FUSED forces the fused kernel wherever it can run (one or two compute waves, no segments).
    const long tiles = ((long)p->n_states * H + 7) / 8 * 8 * (dv / 16);
    const int forced = p->tune.scan_waves ? scan_waves(p->seqs, H, dv, dt, false, p->tune) : 0;
    const bool pair = forced ? forced == 2 : tiles >= 384 && tiles < 2048;
    p->fused = dt == KLA_BF16 && n_chunks > 0 && p->seg_G <= 1 && !p->tune.unfused && !p->tune.generic_scan && !p->tune.generic_intra &&
               (p->tune.fused ? forced <= 2 : pair && dv <= 128);
    if (p->fused) { p->total = 256; p->order_bytes = 0; }
    return KLA_OK;
}

int scan_waves(const Lengths& seqs, int H, int dv, int dt, bool saves, const Tune& tune)
{
    int w;
    if (tune.scan_waves) w = tune.scan_waves;        // tuning field: 1, 2 or 4 waves (16 state columns each) per workgroup
    else if (dt == KLA_F32) w = f32_tiles((long)seqs.n * H * (dv / 16));
    else {
        // bf16: relative lengths of a chunk step with 1, 2, 4 and 8 waves, times the steps of the busiest CU; the cheapest wins,
        // between equals the narrower, which uses more CUs.  Steps measured with the chip full (8 x 2048 tokens, 8 heads, d_v = 256:
        // 174, 107, 85 us per call for 4, 2, 1 rounds of 1, 2, 4 waves; 16 x 2048, 16 heads, d_v = 256: 361 us for 4 rounds of 4
        // waves, 305 us for 2 of 8; 20 x 1024, 8 heads, d_v = 256: 117 us for 3 of 4, 125 us for 2 of 8; with the two rings of the four
        // waves 300, 299, 101 us and, 40 x 1024, 16 heads, d_v = 128, 265 us for 5 of 4, 282 us for 3 of 8).  A forward that
        // leaves its intermediates also stores 512 bytes per token, head and 16 columns, which more waves share a CU for: 8 x 700
        // tokens, 8 heads, d_v = 256 48 us for 2 rounds of 2 waves, 40 for one of 4; 16 x 700 88 us for 2 of 4, 81 for one of 8.
        // Packed, 12 sequences of 653 .. 2056 tokens, 8 heads, d_v = 256: 113 us with 8 waves, 93 with 4, whose second round is of
        // short sequences (leaving intermediates: 174 and 143); 5 of 422 .. 1597, 16 heads, d_v = 128: 51 with 4, 45 with 2.
        const int plain[4] = {100, 100, 128, 215}, saving[4] = {100, 100, 150, 290};
        const int* step = saves ? saving : plain;
        long best = 0;
        w = 1;
        for (int i = 0; i < 4 && 16 << i <= dv; ++i) {
            const long cost = busiest_cu(seqs, H, dv / (16 << i)) * step[i];
            if (i == 0 || cost < best) { best = cost; w = 1 << i; }
        }
    }
    if (dt == KLA_F32 && w > 2) w = 2;            // fp32: column tiles per workgroup, 1 or 2
    while (16 * w > dv) w >>= 1;
    return w;
}

// Compute waves per workgroup of the forward's scan.  The widths of a packed batch cost the host some microseconds (busiest_cu), so
// they are chosen where a kernel is launched and not with the plan, which is made several times per call, also for its sizes alone
// (kla_chunk_saved_bytes through ctypes, 64 sequences: 1.3 us; with the widths in the plan 7.1).
int fwd_waves(const Plan& p, int H, int dv, int dt)
{
    if (p.fused && !p.tune.scan_waves && !p.tune.fused) return 2;
    const int w = scan_waves(p.seqs, H, dv, dt, false, p.tune);
    return p.fused && !p.tune.scan_waves && w > 2 ? 2 : w;
}

// Whether the intra-chunk stage finds its chunks by itself and leaves the offsets and the scan order of a packed batch to the
// kernels behind it; a batch without a single chunk has no such stage.
bool intra_places(int n_seq, long n_chunks, bool generic)
{
    return n_seq > 0 && n_seq <= kla::kPosScanMax && n_chunks > 0 && !generic;
}

template <typename E>
int chunk_fwd_impl(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                   const float* h0, void* o, float* hT, const int32_t* cu_dev, int n_seq, int N, int T, int H, int dk,
                   int dv, const Plan& pl, char* ws, int stages, float* Tb_out, float* P_out, float* g_out,
                   hipStream_t st, unsigned opts)
{
    E* wsT = reinterpret_cast<E*>(ws + pl.off_T);
    E* wsP = reinterpret_cast<E*>(ws + pl.off_P);
    float* wsG = reinterpret_cast<float*>(ws + pl.off_G);
    int* chunk_off = reinterpret_cast<int*>(ws + pl.off_C);
    const int NT = (T + 63) / 64;
    const bool intra = (stages & 1) != 0, scan = (stages & 2) != 0, unpack = (stages & 4) != 0;

    kla::IntraArgs<E> ia;
    ia.q = static_cast<const E*>(q); ia.k = static_cast<const E*>(k);
    ia.log_alpha = log_alpha; ia.eta = eta; ia.eps = eps;
    ia.cu_seqlens = n_seq > 0 ? cu_dev : nullptr; ia.chunk_off = chunk_off; ia.n_seq = n_seq;
    ia.T = T; ia.NT = NT; ia.H = H;
    ia.wsT = wsT; ia.wsP = wsP; ia.wsG = wsG; ia.opts = opts;   // option bits only (the callers strip the tuning fields)
    if constexpr (sizeof(E) == 2) {
        if (stages == 3 && pl.fused) {
            kla::ScanArgs<E> fa;
            fa.q = static_cast<const E*>(q); fa.k = static_cast<const E*>(k); fa.v = static_cast<const E*>(v);
            fa.h0 = h0; fa.o = static_cast<E*>(o); fa.hT = hT;
            fa.cu_seqlens = n_seq > 0 ? cu_dev : nullptr; fa.chunk_off = nullptr; fa.n_seq = n_seq;
            fa.N = N; fa.T = T; fa.NT = NT; fa.H = H; fa.dv = dv;
            fa.wsT = nullptr; fa.wsP = nullptr; fa.wsG = nullptr; fa.opts = opts;
            fa.seg_G = 0; fa.seg_Lc = 0; fa.kt_src = nullptr; fa.gc_vec = nullptr;
            fa.log_alpha = log_alpha; fa.eta = eta; fa.eps = eps;
            return kla::launch_scan_fused_bf16(fa, dk, fwd_waves(pl, H, dv, KLA_BF16), st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
        }
    }
    const bool generic_intra = sizeof(E) == 2 && pl.tune.generic_intra;
    if (intra && !intra_places(n_seq, pl.n_chunks, generic_intra)) {
        if (n_seq > 0 && kla::launch_chunk_offsets(cu_dev, n_seq, chunk_off, order_at(chunk_off, n_seq), st) != hipSuccess) return KLA_ERR_HIP;
    } else if (intra) ia.pos_out = chunk_off;
    if (intra) {
        [[maybe_unused]] bool done = false;
        if constexpr (sizeof(E) == 2) {
            if (!pl.tune.generic_intra) {                // else the plain kernel (A/B testing)
                if (kla::launch_intra_bf16(ia, dk, kla::kIntraFwd, (int)pl.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
                done = true;
            }
        }
        if constexpr (sizeof(E) == 4) {
            if (kla::launch_intra_f32(ia, dk, kla::kIntraFwd, (int)pl.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
        } else {
            if (!done && kla::launch_intra(ia, dk, (int)pl.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
        }
    }
    if (unpack && kla::launch_unpack<E>(wsT, wsP, wsG, Tb_out, P_out, g_out, pl.n_chunks * H, st) != hipSuccess)
        return KLA_ERR_HIP;
    if (!scan) return KLA_OK;
    kla::ScanArgs<E> sa;
    sa.q = static_cast<const E*>(q); sa.k = static_cast<const E*>(k); sa.v = static_cast<const E*>(v);
    sa.h0 = h0; sa.o = static_cast<E*>(o); sa.hT = hT;
    sa.cu_seqlens = ia.cu_seqlens; sa.chunk_off = chunk_off; sa.n_seq = n_seq;
    sa.seq_order = order_at(chunk_off, n_seq);
    sa.N = N; sa.T = T; sa.NT = NT; sa.H = H; sa.dv = dv;
    sa.wsT = wsT; sa.wsP = wsP; sa.wsG = wsG; sa.opts = opts;
    sa.seg_G = 0; sa.seg_Lc = 0; sa.kt_src = nullptr; sa.gc_vec = nullptr;
    sa.log_alpha = log_alpha; sa.eta = eta; sa.eps = eps;
    if constexpr (sizeof(E) == 2) {
        if (pl.seg_G > 1) {
            // segment-parallel scan: maps of all segments but the last, their prefix composition, then every
            // segment at once from its incoming state (see kla_chunk_segments.hip)
            float* maps = reinterpret_cast<float*>(ws + pl.off_M);
            float* seg_state = reinterpret_cast<float*>(ws + pl.off_S);
            sa.seg_G = pl.seg_G; sa.seg_Lc = pl.seg_Lc;
            if (kla::launch_segment_maps_bf16(sa, dk, maps, st) != hipSuccess) return KLA_ERR_HIP;
            if (kla::launch_segment_combine(h0, maps, seg_state, N, H, dk, dv, pl.seg_G, st) != hipSuccess) return KLA_ERR_HIP;
            sa.h0 = seg_state;
            const int wseg = scan_waves({pl.n_states * pl.seg_G, pl.seg_Lc, nullptr}, H, dv, KLA_BF16, false, pl.tune);
            return kla::launch_scan_bf16(sa, dk, wseg, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
        }
    }
    if constexpr (sizeof(E) == 2) {
        if (pl.rows) return kla::launch_scan_rows_bf16(sa, dk, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
    }
    const int waves = fwd_waves(pl, H, dv, sizeof(E) == 2 ? KLA_BF16 : KLA_F32);
    if constexpr (sizeof(E) == 2) {
        if (!pl.tune.generic_scan)                       // else the plain kernel (A/B testing)
            return kla::launch_scan_bf16(sa, dk, waves, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
    }
    if constexpr (sizeof(E) == 4) return kla::launch_scan_f32(sa, dk, waves, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
    else                          return kla::launch_scan(sa, dk, waves > 4 ? 4 : waves, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

// ---- backward pass ---------------------------------------------------------------------------------
struct BwdPlan {
    Plan base;
    // The first `saved` bytes of the workspace hold what follows from the inputs of the forward alone; a forward that leaves
    // them behind (kla_chunk_fwd_save) spares the backward its first two kernels.  Offsets from off_dS on count from there.
    size_t off_rec, off_C, off_S, off_X, off_U, saved;
    size_t off_dS, off_Y, total;             // total: of both parts
    bool can_save;
    // segment-parallel sweeps (base.seg_G > 1): maps of the segments, states entering them, and for the reverse
    // direction the state gradients leaving them and what each segment's pre-pass returns; all fp32
    size_t off_maps, off_segS, off_segG, off_segB;
};

int make_bwd_plan(int N, int T, int H, int dk, int dv, int chunk, int dt, const int32_t* cu_host, int n_seq, unsigned opts,
                  BwdPlan* p)
{
    const int rc = make_plan(N, T, H, dk, dv, chunk, dt, cu_host, n_seq, opts, &p->base);
    if (rc != KLA_OK) return rc;
    p->base.fwd_seg_G = p->base.seg_G;
    p->base.seg_G = plan_segments(N, (T + 63) / 64, H, dv, dt, n_seq, p->base.tune, 512, &p->base.seg_Lc);
    const size_t half = (size_t)384 * 8 * elem_bytes(dt);
    const size_t ch = (size_t)p->base.n_chunks * H;
    const size_t states = ch * dk * dv * elem_bytes(dt);          // checkpoints are kept in the element type
    const size_t rows = (size_t)N * T * H * dv * elem_bytes(dt);
    p->off_rec = 0;                                              // [T' | M^T | P^T | five vectors] per chunk-head
    p->off_C = round256(ch * (3 * half + 1280));
    p->off_S = round256(p->off_C + (size_t)(n_seq + 1 + order_ints(n_seq)) * sizeof(int32_t));
    p->off_X = round256(p->off_S + states);
    // the bf16 kernels do not keep U (their assembly forms it again from T' and X); the generic ones do
    const size_t rows_u = (dt == KLA_BF16 && !p->base.tune.generic_bwd) ? 0 : rows;
    p->off_U = round256(p->off_X + rows);
    p->saved = round256(p->off_U + rows_u);
    p->off_dS = 0;
    p->off_Y = round256(p->off_dS + states);
    const int G = p->base.seg_G;
    const size_t maps = G > 1 ? (size_t)N * (G - 1) * H * dk * (dv + dk) * sizeof(float) : 0;
    const size_t segst = G > 1 ? (size_t)N * G * H * dk * dv * sizeof(float) : 0;
    p->off_maps = round256(p->off_Y + rows);
    p->off_segS = round256(p->off_maps + maps);
    p->off_segG = round256(p->off_segS + segst);
    p->off_segB = round256(p->off_segG + segst);
    p->total = p->saved + round256(p->off_segB + segst);
    // A forward leaves its intermediates where it forms the very ones the backward would: not in one kernel (which rounds other
    // things), not in segments (whose number differs), not through the plain kernels.  And within a bound: what is kept lives
    // until the backward, in every layer of a model.
    const Tune& t = p->base.tune;
    p->can_save = p->base.n_chunks > 0 && !p->base.fused && p->base.fwd_seg_G <= 1 && G <= 1 && !t.generic_scan && !t.generic_intra &&
                  !t.generic_bwd && p->saved <= (size_t)KLA_SAVED_MAX_BYTES;
    return KLA_OK;
}

template <typename E>
int chunk_bwd_impl(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                   const float* h0, const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_,
                   float* dlog_alpha, float* deta, float* dh0, const int32_t* cu_dev, int n_seq, int N, int T, int H,
                   int dk, int dv, const BwdPlan& pl, char* sv, char* ws, bool have, hipStream_t st, unsigned opts)
{
    // sv: what the forward leaves behind (have: it has; else it is made here); ws: the rest of the workspace
    int* chunk_off = reinterpret_cast<int*>(sv + pl.off_C);
    const int NT = (T + 63) / 64;
    const bool placed = intra_places(n_seq, pl.base.n_chunks, sizeof(E) == 2 && pl.base.tune.generic_bwd);
    if (n_seq > 0 && !placed && !have && kla::launch_chunk_offsets(cu_dev, n_seq, chunk_off, order_at(chunk_off, n_seq), st) != hipSuccess) return KLA_ERR_HIP;

    kla::IntraArgs<E> ia;
    if (placed) ia.pos_out = chunk_off;
    ia.q = static_cast<const E*>(q); ia.k = static_cast<const E*>(k);
    ia.log_alpha = log_alpha; ia.eta = eta; ia.eps = eps;
    ia.cu_seqlens = n_seq > 0 ? cu_dev : nullptr; ia.chunk_off = chunk_off; ia.n_seq = n_seq;
    ia.T = T; ia.NT = NT; ia.H = H;
    ia.wsT = reinterpret_cast<E*>(sv + pl.off_rec); ia.wsP = nullptr; ia.wsG = nullptr; ia.opts = opts;
    bool fast = false;                                // bf16: the specialised kernels, unless the generic ones are asked for (A/B testing)
    if constexpr (sizeof(E) == 2) fast = !pl.base.tune.generic_bwd;
    if constexpr (sizeof(E) == 2) {
        if (fast && !have && kla::launch_intra_bf16(ia, dk, kla::kIntraBwd, (int)pl.base.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
    }
    if constexpr (sizeof(E) == 4) {
        if (!have && kla::launch_intra_f32(ia, dk, kla::kIntraBwd, (int)pl.base.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
    } else {
        if (!fast && kla::launch_intra_bwd(ia, dk, (int)pl.base.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
    }

    kla::BwdArgs<E> ba;
    ba.q = ia.q; ba.k = ia.k; ba.v = static_cast<const E*>(v);
    ba.log_alpha = log_alpha; ba.eta = eta; ba.eps = eps;
    ba.h0 = h0; ba.d_o = static_cast<const E*>(d_o); ba.d_hT = d_hT;
    ba.dq = static_cast<E*>(dq); ba.dk = static_cast<E*>(dk_); ba.dv = static_cast<E*>(dv_);
    ba.dlog_alpha = dlog_alpha; ba.deta = deta; ba.dh0 = dh0;
    ba.cu_seqlens = ia.cu_seqlens; ba.chunk_off = chunk_off; ba.n_seq = n_seq;
    ba.seq_order = order_at(chunk_off, n_seq);
    ba.N = N; ba.T = T; ba.NT = NT; ba.H = H; ba.dv_dim = dv;
    ba.rec = sv + pl.off_rec;
    ba.s_chk = reinterpret_cast<E*>(sv + pl.off_S); ba.ds_chk = reinterpret_cast<E*>(ws + pl.off_dS);
    ba.X = reinterpret_cast<E*>(sv + pl.off_X); ba.U = reinterpret_cast<E*>(sv + pl.off_U);
    ba.Y = reinterpret_cast<E*>(ws + pl.off_Y);
    ba.opts = opts;
    ba.seg_G = 0; ba.seg_Lc = 0;
    // What the slices of a head all copy in the reverse sweep, K, Q, M^T and P^T: beyond some 144 MB (of a memory-side cache of 256, which
    // the checkpoints, Y and dO go through too) it comes from HBM, and asking ahead shortens the copies' way (8 x 4096 tokens, 8
    // heads: 143 -> 122 us; 7 x 4096, 161 MB: 130 -> 119); below, it is there already (8 x 3000, 135 MB: 90.3, 90.5; 8 x 2048: 63.7, 65.7).
    // Whole backward, not asked and asked, 8 heads: 4 x 8192, d_v = 256 729 and 678 us; 16 x 2048, d_v = 64 (two slices, which ask for K and
    // Q alone) 271 and 267; one sequence of 65536 in segments 1244 and 1224; d_k = 64: 16 x 4096, d_v = 64 408 and 402, 8 x 8192, d_v = 128
    // 609 and 605.
    ba.touch = (size_t)pl.base.n_chunks * H * (2 * 64 * dk * sizeof(E) + (size_t)2 * 384 * 8 * sizeof(E)) > ((size_t)144 << 20);
    if constexpr (sizeof(E) == 2) {
        if (fast && pl.base.seg_G > 1) {
            // Segment-parallel sweeps for a few long sequences (see kla_chunk_segments.hip).  Forward: maps of all
            // segments but the last, their composition, then every segment at once from its incoming state.  Reverse:
            // the recursion dS = A dS' + b of a segment is affine with A the transpose of the forward map, so a
            // pre-pass that stores nothing gives every b (the last segment runs with its true d_hT), the composition
            // runs down the segments, and the real sweep starts every segment from its incoming gradient.
            const int G = pl.base.seg_G;
            float* maps = reinterpret_cast<float*>(ws + pl.off_maps);
            float* segS = reinterpret_cast<float*>(ws + pl.off_segS);
            float* segG = reinterpret_cast<float*>(ws + pl.off_segG);
            float* segB = reinterpret_cast<float*>(ws + pl.off_segB);
            kla::ScanArgs<E> sa;
            sa.q = ba.q; sa.k = ba.k; sa.v = ba.v; sa.h0 = nullptr; sa.o = nullptr; sa.hT = nullptr;
            sa.cu_seqlens = nullptr; sa.chunk_off = chunk_off; sa.n_seq = 0;
            sa.N = N; sa.T = T; sa.NT = NT; sa.H = H; sa.dv = dv;
            sa.wsT = reinterpret_cast<const E*>(sv + pl.off_rec); sa.wsP = nullptr; sa.wsG = nullptr; sa.opts = 0u;
            sa.seg_G = G; sa.seg_Lc = pl.base.seg_Lc; sa.kt_src = nullptr; sa.gc_vec = nullptr;
            if (kla::launch_segment_maps_bwdrec_bf16(sa, dk, maps, st) != hipSuccess) return KLA_ERR_HIP;
            if (kla::launch_segment_combine(h0, maps, segS, N, H, dk, dv, G, st) != hipSuccess) return KLA_ERR_HIP;
            if (kla::launch_segment_scatter(d_hT, segG, N, H, dk, dv, G, st) != hipSuccess) return KLA_ERR_HIP;
            ba.seg_G = G; ba.seg_Lc = pl.base.seg_Lc;
            const long sc8 = ((long)N * G * H + 7) / 8 * 8;
            const int wseg = sc8 * (dv / 16) > 256 ? 2 : 1;
            ba.h0 = segS;
            if (kla::launch_bwd_states_bf16(ba, dk, wseg, st) != hipSuccess) return KLA_ERR_HIP;
            ba.d_hT = segG; ba.dh0 = segB; ba.opts = opts | kla::kOptNoStore;
            if (kla::launch_bwd_scan_bf16(ba, dk, wseg, st) != hipSuccess) return KLA_ERR_HIP;          // pre-pass: b per segment
            if (kla::launch_segment_combine_rev(maps, segB, segG, N, H, dk, dv, G, st) != hipSuccess) return KLA_ERR_HIP;
            ba.opts = opts;
            if (kla::launch_bwd_scan_bf16(ba, dk, wseg, st) != hipSuccess) return KLA_ERR_HIP;          // the real sweep
            if (dh0 && kla::launch_segment_gather(segB, dh0, N, H, dk, dv, G, st) != hipSuccess) return KLA_ERR_HIP;
            ba.seg_G = 0; ba.seg_Lc = 0; ba.h0 = h0; ba.d_hT = d_hT; ba.dh0 = dh0;
            return kla::launch_bwd_assemble_bf16(ba, dk, pl.base.n_chunks, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
        }
    }
    [[maybe_unused]] const int waves = sizeof(E) == 2 ? kla::sweep_waves(pl.base.seqs, H, dv, !pl.base.tune.generic_bwd) : 0;
    if constexpr (sizeof(E) == 2) {
        if (fast) {
            if (!have && kla::launch_bwd_states_bf16(ba, dk, waves, st) != hipSuccess) return KLA_ERR_HIP;
            if (kla::launch_bwd_scan_bf16(ba, dk, waves, st) != hipSuccess) return KLA_ERR_HIP;
            return kla::launch_bwd_assemble_bf16(ba, dk, pl.base.n_chunks, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
        }
    }
    if constexpr (sizeof(E) == 4) {
        const int tiles = f32_tiles((long)pl.base.n_states * H * (dv / 16));
        if (!have && kla::launch_bwd_states_f32(ba, dk, tiles, st) != hipSuccess) return KLA_ERR_HIP;
        if (kla::launch_bwd_scan_f32(ba, dk, tiles, st) != hipSuccess) return KLA_ERR_HIP;
    } else {
        if (kla::launch_bwd_states(ba, dk, waves, st) != hipSuccess) return KLA_ERR_HIP;
        if (kla::launch_bwd_scan(ba, dk, waves, st) != hipSuccess) return KLA_ERR_HIP;
    }
    if (kla::launch_bwd_assemble<E>(ba, dk, pl.base.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;
    return KLA_OK;
}

// The forward that leaves its intermediates (pl: its own plan, bp: the backward's, bp.can_save): stage 1 writes both kinds of
// record at once, the scan stores every chunk's incoming state and X (and, fp32, U) on its way.
template <typename E>
int chunk_fwd_save_impl(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                        const float* h0, void* o, float* hT, const int32_t* cu_dev, int n_seq, int N, int T, int H, int dk, int dv,
                        const Plan& pl, const BwdPlan& bp, char* ws, char* sv, hipStream_t st, unsigned opts)
{
    // (the records of P take half of the room the plain forward's records have in the workspace)
    int* chunk_off = reinterpret_cast<int*>(sv + bp.off_C);
    kla::IntraArgs<E> ia;
    ia.q = static_cast<const E*>(q); ia.k = static_cast<const E*>(k);
    ia.log_alpha = log_alpha; ia.eta = eta; ia.eps = eps;
    ia.cu_seqlens = n_seq > 0 ? cu_dev : nullptr; ia.chunk_off = chunk_off; ia.n_seq = n_seq;
    ia.T = T; ia.NT = (T + 63) / 64; ia.H = H;
    ia.wsT = reinterpret_cast<E*>(sv + bp.off_rec); ia.wsP = reinterpret_cast<E*>(ws + pl.off_T); ia.wsG = nullptr; ia.opts = opts;
    if (intra_places(n_seq, pl.n_chunks, false)) ia.pos_out = chunk_off;
    else if (n_seq > 0 && kla::launch_chunk_offsets(cu_dev, n_seq, chunk_off, order_at(chunk_off, n_seq), st) != hipSuccess) return KLA_ERR_HIP;

    kla::ScanArgs<E> sa;
    sa.q = ia.q; sa.k = ia.k; sa.v = static_cast<const E*>(v);
    sa.h0 = h0; sa.o = static_cast<E*>(o); sa.hT = hT;
    sa.cu_seqlens = ia.cu_seqlens; sa.chunk_off = chunk_off; sa.n_seq = n_seq;
    sa.seq_order = order_at(chunk_off, n_seq);
    sa.N = N; sa.T = T; sa.NT = ia.NT; sa.H = H; sa.dv = dv;
    sa.wsT = ia.wsT; sa.wsP = ia.wsP; sa.wsG = nullptr; sa.opts = opts;
    sa.seg_G = 0; sa.seg_Lc = 0; sa.kt_src = nullptr; sa.gc_vec = nullptr;
    sa.s_chk = reinterpret_cast<E*>(sv + bp.off_S); sa.X = reinterpret_cast<E*>(sv + bp.off_X); sa.U = reinterpret_cast<E*>(sv + bp.off_U);
    hipError_t e;
    if constexpr (sizeof(E) == 2) {
        e = kla::launch_intra_bf16(ia, dk, kla::kIntraPair, (int)pl.n_chunks, st);
        if (e == hipSuccess) e = pl.rows ? kla::launch_scan_rows_bf16(sa, dk, st) : kla::launch_scan_bf16(sa, dk, scan_waves(pl.seqs, H, dv, KLA_BF16, true, pl.tune), st);
    } else {
        e = kla::launch_intra_f32(ia, dk, kla::kIntraPair, (int)pl.n_chunks, st);
        if (e == hipSuccess) e = kla::launch_scan_f32(sa, dk, fwd_waves(pl, H, dv, KLA_F32), st);
    }
    return e == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

// ---- diagonal gating ----------------------------------------------------------------------------------
struct DiagPlan {
    Plan base;
    size_t off_kp, off_qp, off_kt, off_gc, total;
};

int make_diag_plan(int N, int T, int H, int dk, int dv, int chunk, int dt, const int32_t* cu_host, int n_seq, unsigned opts,
                   DiagPlan* p)
{
    // the layout of the two-kernel forward (the fused kernel has no diagonal-gating variant), no segments
    const int rc = make_plan(N, T, H, dk, dv, chunk, dt, cu_host, n_seq, (opts & ~(31u << 10) & ~KLA_TUNE_FUSED) | KLA_TUNE_UNFUSED | KLA_TUNE_SCAN_SEGMENTS(1), &p->base);
    if (rc != KLA_OK) return rc;
    const size_t rows = (size_t)N * T * H * dk * elem_bytes(dt);
    // The three operand arrays are read row by row at the same time.  Their sizes are large powers of two for the usual
    // shapes, so without the 256-byte steps below the rows of one token would sit in the same memory channel in all
    // three (measured: the scan of the config-2 shape takes 13 us longer).
    p->off_kp = round256(p->base.off_M);             // the forward plan up to its chunk offsets; no segment maps here
    p->off_qp = round256(p->off_kp + rows) + 256;
    p->off_kt = round256(p->off_qp + rows) + 256;
    p->off_gc = round256(p->off_kt + rows) + 256;
    p->total = round256(p->off_gc + (size_t)p->base.n_chunks * H * dk * sizeof(float));
    return KLA_OK;
}

template <typename E>
int chunk_fwd_diag_impl(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                        const float* h0, void* o, float* hT, const int32_t* cu_dev, int n_seq, int N, int T, int H,
                        int dk, int dv, const DiagPlan& pl, char* ws, hipStream_t st, unsigned opts)
{
    int* chunk_off = reinterpret_cast<int*>(ws + pl.base.off_C);
    const int NT = (T + 63) / 64;
    const bool placed = intra_places(n_seq, pl.base.n_chunks, false);
    if (n_seq > 0 && !placed && kla::launch_chunk_offsets(cu_dev, n_seq, chunk_off, order_at(chunk_off, n_seq), st) != hipSuccess) return KLA_ERR_HIP;
    kla::IntraDiagArgs<E> ia;
    if (placed) ia.pos_out = chunk_off;
    ia.q = static_cast<const E*>(q); ia.k = static_cast<const E*>(k);
    ia.log_alpha = log_alpha; ia.eta = eta; ia.eps = eps;
    ia.cu_seqlens = n_seq > 0 ? cu_dev : nullptr; ia.chunk_off = chunk_off; ia.n_seq = n_seq;
    ia.T = T; ia.NT = NT; ia.H = H;
    ia.wsT = reinterpret_cast<E*>(ws + pl.base.off_T); ia.wsG = reinterpret_cast<float*>(ws + pl.base.off_G);
    ia.kplus = reinterpret_cast<E*>(ws + pl.off_kp); ia.qplus = reinterpret_cast<E*>(ws + pl.off_qp);
    ia.ktilde = reinterpret_cast<E*>(ws + pl.off_kt); ia.gc = reinterpret_cast<float*>(ws + pl.off_gc);
    ia.opts = opts;
    if (kla::launch_intra_diag<E>(ia, dk, (int)pl.base.n_chunks, st) != hipSuccess) return KLA_ERR_HIP;

    kla::ScanArgs<E> sa;
    sa.q = ia.qplus; sa.k = ia.kplus; sa.v = static_cast<const E*>(v);
    sa.h0 = h0; sa.o = static_cast<E*>(o); sa.hT = hT;
    sa.cu_seqlens = ia.cu_seqlens; sa.chunk_off = chunk_off; sa.n_seq = n_seq;
    sa.seq_order = order_at(chunk_off, n_seq);
    sa.N = N; sa.T = T; sa.NT = NT; sa.H = H; sa.dv = dv;
    sa.wsT = ia.wsT; sa.wsP = reinterpret_cast<E*>(ws + pl.base.off_P); sa.wsG = ia.wsG; sa.opts = 0u;
    sa.seg_G = 0; sa.seg_Lc = 0; sa.kt_src = ia.ktilde; sa.gc_vec = ia.gc;
    const int waves = kla::diag_scan_waves(pl.base.seqs, H, dk, dv);
    if constexpr (sizeof(E) == 2) {
        if (!pl.base.tune.generic_scan)                  // else the plain kernel (A/B testing)
            return kla::launch_scan_bf16_diag(sa, dk, waves, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
    }
    if constexpr (sizeof(E) == 4)
        return kla::launch_scan_f32(sa, dk, f32_tiles((long)pl.base.n_states * H * (dv / 16)), st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
    else
        return kla::launch_scan_diag(sa, dk, waves, st) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

// ---- scratch of the entry point that allocates nothing (kla_chunk_fwd_static) --------------------------
// A file-scope device array: every GPU the library runs on holds its own copy at its own address until the
// process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the address that
// kernels receive is looked up once per device, with that device current, and kept.
// The bound that callers know, KLA_STATIC_SCRATCH_BYTES, does not count the scan order of a packed batch: it has room of
// its own behind (kOrderMax numbers, rounded up to 256 bytes).
constexpr size_t kStaticScratchBytes = (size_t)KLA_STATIC_SCRATCH_BYTES + 4 * (size_t)kla::kOrderMax + 256;
constexpr int kMaxDevices = 64;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
std::mutex scratch_mutex;
void* scratch_ptr[kMaxDevices];        // device address of `scratch` per device ordinal, NULL until looked up

// Device address of this device's copy of `scratch` (first call on a device: one symbol lookup), or NULL.
void* static_scratch()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        scratch_ptr[dev] = p;
    }
    return scratch_ptr[dev];
}

}  // namespace

extern "C" {

const char* kla_status_string(int code)
{
    switch (code) {
        case KLA_OK: return "KLA_OK";
        case KLA_ERR_NULL: return "KLA_ERR_NULL: a required pointer is NULL";
        case KLA_ERR_SHAPE: return "KLA_ERR_SHAPE: unsupported or inconsistent sizes";
        case KLA_ERR_DTYPE: return "KLA_ERR_DTYPE: unknown element type";
        case KLA_ERR_ALIGN: return "KLA_ERR_ALIGN: pointer not 16-byte aligned";
        case KLA_ERR_WORKSPACE: return "KLA_ERR_WORKSPACE: workspace missing, misaligned or too small";
        case KLA_ERR_SEQLENS: return "KLA_ERR_SEQLENS: bad cu_seqlens";
        case KLA_ERR_HIP: return "KLA_ERR_HIP: kernel launch failed";
        default: return "unknown kla status";
    }
}

size_t kla_chunk_fwd_workspace_bytes(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt,
                                     const int32_t* cu_seqlens_host, int n_seq)
{
    return kla_chunk_fwd_workspace_bytes_opts(N, T, H, dk, dv, chunk, dt, cu_seqlens_host, n_seq, 0u);
}

size_t kla_chunk_fwd_workspace_bytes_opts(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt,
                                          const int32_t* cu_seqlens_host, int n_seq, unsigned opts)
{
    Plan pl;
    if (make_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, &pl) != KLA_OK) return 0;
    return pl.total;
}

// Everything kla_chunk_fwd checks except its workspace; fills the plan.
static int chunk_fwd_validate(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                              float eps, const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                              const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                              kla_dtype dt, unsigned opts, Plan* pl)
{
    const int rc = make_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, pl);
    if (rc != KLA_OK) return rc;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (n_seq > 0 && !cu_seqlens_dev) return KLA_ERR_NULL;
    if (n_seq == 0 && cu_seqlens_dev) return KLA_ERR_SHAPE;
    const bool any_tokens = (long)N * T > 0;
    if (any_tokens && (!q || !k || !v || !log_alpha || !eta || !o)) return KLA_ERR_NULL;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(h0) || !aligned16(hT) ||
        (reinterpret_cast<uintptr_t>(log_alpha) & 3u) || (reinterpret_cast<uintptr_t>(eta) & 3u))
        return KLA_ERR_ALIGN;
    return KLA_OK;
}

static int chunk_fwd_launch(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                            float eps, const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev, int n_seq,
                            int N, int T, int H, int dk, int dv, kla_dtype dt, const Plan& pl, void* workspace,
                            void* hip_stream, int stages, unsigned opts)
{
    if (pl.n_states == 0) return KLA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char* ws = static_cast<char*>(workspace);
    opts &= kOptMask;                                    // the tuning fields live on in pl.tune
    if (dt == KLA_BF16)
        return chunk_fwd_impl<bf16_t>(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv,
                                      pl, ws, stages, nullptr, nullptr, nullptr, st, opts);
    return chunk_fwd_impl<float>(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv, pl, ws,
                                 stages, nullptr, nullptr, nullptr, st, opts);
}

static int chunk_fwd_checked(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                             float eps, const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                             const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                             kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream, int stages,
                             unsigned opts)
{
    Plan pl;
    const int rc = chunk_fwd_validate(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N,
                                      T, H, dk, dv, chunk, dt, opts, &pl);
    if (rc != KLA_OK) return rc;
    if (!workspace) return KLA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < pl.total) return KLA_ERR_WORKSPACE;
    return chunk_fwd_launch(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv, dt, pl,
                            workspace, hip_stream, stages, opts);
}

int kla_chunk_fwd(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                  const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev, const int32_t* cu_seqlens_host,
                  int n_seq, int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt, void* workspace,
                  size_t workspace_bytes, void* hip_stream)
{
    return chunk_fwd_checked(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N, T, H,
                             dk, dv, chunk, dt, workspace, workspace_bytes, hip_stream, 3, 0u);
}

int kla_chunk_fwd_opts(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                       const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                       const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                       kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream, unsigned opts)
{
    return chunk_fwd_checked(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N, T, H,
                             dk, dv, chunk, dt, workspace, workspace_bytes, hip_stream, 3, opts);
}

int kla_chunk_fwd_static(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                         float eps, const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                         const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                         kla_dtype dt, void* hip_stream)
{
    Plan pl;
    const int rc = chunk_fwd_validate(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N,
                                      T, H, dk, dv, chunk, dt, 0u, &pl);
    if (rc != KLA_OK) return rc;
    if (pl.total - pl.order_bytes > (size_t)KLA_STATIC_SCRATCH_BYTES) return KLA_ERR_WORKSPACE;   // refused before any HIP call
    if (pl.n_states == 0) return KLA_OK;
    void* ws = static_scratch();
    if (!ws) return KLA_ERR_HIP;
    return chunk_fwd_launch(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv, dt, pl, ws,
                            hip_stream, 3, 0u);
}

size_t kla_chunk_bwd_workspace_bytes(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt,
                                     const int32_t* cu_seqlens_host, int n_seq)
{
    return kla_chunk_bwd_workspace_bytes_opts(N, T, H, dk, dv, chunk, dt, cu_seqlens_host, n_seq, 0u);
}

size_t kla_chunk_bwd_workspace_bytes_opts(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt,
                                          const int32_t* cu_seqlens_host, int n_seq, unsigned opts)
{
    BwdPlan pl;
    if (make_bwd_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, &pl) != KLA_OK) return 0;
    return pl.total;
}

int kla_chunk_bwd(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                  const float* h0, const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_,
                  float* dlog_alpha, float* deta, float* dh0, const int32_t* cu_seqlens_dev,
                  const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                  kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    return kla_chunk_bwd_opts(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0,
                              cu_seqlens_dev, cu_seqlens_host, n_seq, N, T, H, dk, dv, chunk, dt, workspace,
                              workspace_bytes, hip_stream, 0u);
}

// Everything kla_chunk_bwd checks except its workspace; fills the plan.
static int chunk_bwd_validate(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                              const float* h0, const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_,
                              float* dlog_alpha, float* deta, float* dh0, const int32_t* cu_seqlens_dev,
                              const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                              kla_dtype dt, unsigned opts, BwdPlan* pl)
{
    const int rc = make_bwd_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, pl);
    if (rc != KLA_OK) return rc;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (n_seq > 0 && !cu_seqlens_dev) return KLA_ERR_NULL;
    if (n_seq == 0 && cu_seqlens_dev) return KLA_ERR_SHAPE;
    const bool any_tokens = (long)N * T > 0;
    if (any_tokens && (!q || !k || !v || !log_alpha || !eta || !d_o || !dq || !dk_ || !dv_ || !dlog_alpha || !deta))
        return KLA_ERR_NULL;
    return KLA_OK;
}
static int chunk_bwd_align(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, const float* h0,
                           const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_, float* dlog_alpha, float* deta, float* dh0)
{
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o) || !aligned16(dq) || !aligned16(dk_) ||
        !aligned16(dv_) || !aligned16(h0) || !aligned16(d_hT) || !aligned16(dh0) ||
        (reinterpret_cast<uintptr_t>(log_alpha) & 3u) || (reinterpret_cast<uintptr_t>(eta) & 3u) ||
        (reinterpret_cast<uintptr_t>(dlog_alpha) & 3u) || (reinterpret_cast<uintptr_t>(deta) & 3u))
        return KLA_ERR_ALIGN;
    return KLA_OK;
}
// a buffer of the caller's: present, 256-byte aligned, large enough
static bool buffer_ok(const void* p, size_t bytes, size_t need) { return p && (reinterpret_cast<uintptr_t>(p) & 255u) == 0 && bytes >= need; }

static int chunk_bwd_launch(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                            const float* h0, const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_,
                            float* dlog_alpha, float* deta, float* dh0, const int32_t* cu_seqlens_dev, int n_seq, int N, int T,
                            int H, int dk, int dv, kla_dtype dt, const BwdPlan& pl, char* sv, char* ws, bool have, void* hip_stream,
                            unsigned opts)
{
    if (pl.base.n_states == 0) return KLA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    opts &= kOptMask;
    if (dt == KLA_BF16)
        return chunk_bwd_impl<bf16_t>(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0,
                                      cu_seqlens_dev, n_seq, N, T, H, dk, dv, pl, sv, ws, have, st, opts);
    return chunk_bwd_impl<float>(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0,
                                 cu_seqlens_dev, n_seq, N, T, H, dk, dv, pl, sv, ws, have, st, opts);
}

int kla_chunk_bwd_opts(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                       const float* h0, const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_,
                       float* dlog_alpha, float* deta, float* dh0, const int32_t* cu_seqlens_dev,
                       const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                       kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream, unsigned opts)
{
    BwdPlan pl;
    int rc = chunk_bwd_validate(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0, cu_seqlens_dev,
                                cu_seqlens_host, n_seq, N, T, H, dk, dv, chunk, dt, opts, &pl);
    if (rc != KLA_OK) return rc;
    if (!buffer_ok(workspace, workspace_bytes, pl.total)) return KLA_ERR_WORKSPACE;
    rc = chunk_bwd_align(q, k, v, log_alpha, eta, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0);
    if (rc != KLA_OK) return rc;
    char* ws = static_cast<char*>(workspace);
    return chunk_bwd_launch(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0, cu_seqlens_dev, n_seq, N,
                            T, H, dk, dv, dt, pl, ws, ws + pl.saved, false, hip_stream, opts);
}

// ---- a forward that leaves its intermediates, and the backward that takes them ---------------------------------------
size_t kla_chunk_saved_bytes(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt, const int32_t* cu_seqlens_host, int n_seq,
                             unsigned opts)
{
    BwdPlan pl;
    if (make_bwd_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, &pl) != KLA_OK) return 0;
    return pl.can_save ? pl.saved : 0;
}

size_t kla_chunk_bwd_saved_workspace_bytes(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt, const int32_t* cu_seqlens_host,
                                           int n_seq, unsigned opts)
{
    BwdPlan pl;
    if (make_bwd_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, &pl) != KLA_OK) return 0;
    return pl.can_save ? pl.total - pl.saved : 0;
}

int kla_chunk_fwd_save(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                       const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev, const int32_t* cu_seqlens_host,
                       int n_seq, int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt, void* workspace,
                       size_t workspace_bytes, void* saved, size_t saved_bytes, void* hip_stream, unsigned opts)
{
    Plan pl;
    int rc = chunk_fwd_validate(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N, T, H, dk, dv, chunk,
                                dt, opts, &pl);
    if (rc != KLA_OK) return rc;
    BwdPlan bp;
    rc = make_bwd_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, &bp);
    if (rc != KLA_OK) return rc;
    if (!bp.can_save) return KLA_ERR_SHAPE;
    if (!buffer_ok(workspace, workspace_bytes, pl.total) || !buffer_ok(saved, saved_bytes, bp.saved)) return KLA_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char*>(workspace), *sv = static_cast<char*>(saved);
    opts &= kOptMask;
    if (dt == KLA_BF16)
        return chunk_fwd_save_impl<bf16_t>(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv, pl, bp, ws, sv, st, opts);
    return chunk_fwd_save_impl<float>(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv, pl, bp, ws, sv, st, opts);
}

int kla_chunk_bwd_saved(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                        const float* h0, const void* d_o, const float* d_hT, void* dq, void* dk_, void* dv_,
                        float* dlog_alpha, float* deta, float* dh0, const int32_t* cu_seqlens_dev,
                        const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                        kla_dtype dt, void* workspace, size_t workspace_bytes, const void* saved, size_t saved_bytes,
                        void* hip_stream, unsigned opts)
{
    BwdPlan pl;
    int rc = chunk_bwd_validate(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0, cu_seqlens_dev,
                                cu_seqlens_host, n_seq, N, T, H, dk, dv, chunk, dt, opts, &pl);
    if (rc != KLA_OK) return rc;
    if (!pl.can_save) return KLA_ERR_SHAPE;
    if (!buffer_ok(workspace, workspace_bytes, pl.total - pl.saved) || !buffer_ok(saved, saved_bytes, pl.saved)) return KLA_ERR_WORKSPACE;
    rc = chunk_bwd_align(q, k, v, log_alpha, eta, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0);
    if (rc != KLA_OK) return rc;
    return chunk_bwd_launch(q, k, v, log_alpha, eta, eps, h0, d_o, d_hT, dq, dk_, dv_, dlog_alpha, deta, dh0, cu_seqlens_dev, n_seq, N,
                            T, H, dk, dv, dt, pl, const_cast<char*>(static_cast<const char*>(saved)), static_cast<char*>(workspace), true,
                            hip_stream, opts);
}

size_t kla_chunk_fwd_diag_workspace_bytes(int N, int T, int H, int dk, int dv, int chunk, kla_dtype dt,
                                          const int32_t* cu_seqlens_host, int n_seq)
{
    DiagPlan pl;
    if (make_diag_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, 0u, &pl) != KLA_OK) return 0;
    return pl.total;
}

int kla_chunk_fwd_diag(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                       const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                       const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                       kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    return kla_chunk_fwd_diag_opts(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N, T, H,
                                   dk, dv, chunk, dt, workspace, workspace_bytes, hip_stream, 0u);
}

int kla_chunk_fwd_diag_opts(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                            const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                            const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                            kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream, unsigned opts)
{
    DiagPlan pl;
    const int rc = make_diag_plan(N, T, H, dk, dv, chunk, (int)dt, cu_seqlens_host, n_seq, opts, &pl);
    if (rc != KLA_OK) return rc;
    opts &= kOptMask;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (n_seq > 0 && !cu_seqlens_dev) return KLA_ERR_NULL;
    if (n_seq == 0 && cu_seqlens_dev) return KLA_ERR_SHAPE;
    const bool any_tokens = (long)N * T > 0;
    if (any_tokens && (!q || !k || !v || !log_alpha || !eta || !o)) return KLA_ERR_NULL;
    if (!workspace) return KLA_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < pl.total) return KLA_ERR_WORKSPACE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(h0) || !aligned16(hT) ||
        (reinterpret_cast<uintptr_t>(log_alpha) & 3u) || (reinterpret_cast<uintptr_t>(eta) & 3u))
        return KLA_ERR_ALIGN;
    if (pl.base.n_states == 0) return KLA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char* ws = static_cast<char*>(workspace);
    if (dt == KLA_BF16)
        return chunk_fwd_diag_impl<bf16_t>(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv,
                                           pl, ws, st, opts);
    return chunk_fwd_diag_impl<float>(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, n_seq, N, T, H, dk, dv, pl,
                                      ws, st, opts);
}

int kla_decode_step_diag(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                         float eps, float* S, void* o, int B, int H, int dk, int dv, kla_dtype dt, void* hip_stream)
{
    return kla_decode_step_diag_opts(q, k, v, log_alpha, eta, eps, S, o, B, H, dk, dv, dt, hip_stream, 0u);
}

int kla_decode_step_diag_opts(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                              float eps, float* S, void* o, int B, int H, int dk, int dv, kla_dtype dt, void* hip_stream,
                              unsigned opts)
{
    if (!dt_ok((int)dt)) return KLA_ERR_DTYPE;
    Tune tune;
    if (!parse_tune(opts, &tune)) return KLA_ERR_SHAPE;
    opts &= kOptMask;
    if (B < 0 || H <= 0 || !dk_ok(dk) || !dv_ok(dv) || (long)B * H > 0x7fffffffL) return KLA_ERR_SHAPE;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (B == 0) return KLA_OK;
    if (!q || !k || !v || !log_alpha || !eta || !S || !o) return KLA_ERR_NULL;
    if (!aligned16(S) || (reinterpret_cast<uintptr_t>(q) & 3u) || (reinterpret_cast<uintptr_t>(k) & 3u) ||
        (reinterpret_cast<uintptr_t>(v) & 3u) || (reinterpret_cast<uintptr_t>(o) & 3u) ||
        (reinterpret_cast<uintptr_t>(log_alpha) & 3u) || (reinterpret_cast<uintptr_t>(eta) & 3u))
        return KLA_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e;
    if (dt == KLA_BF16)
        e = kla::launch_decode<bf16_t>(static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k),
                                       static_cast<const bf16_t*>(v), log_alpha, eta, eps, S, static_cast<bf16_t*>(o),
                                       B * H, dk, dv, 64, tune.decode_nt, kla::kOptDiagDecay | opts, st);
    else
        e = kla::launch_decode<float>(static_cast<const float*>(q), static_cast<const float*>(k),
                                      static_cast<const float*>(v), log_alpha, eta, eps, S, static_cast<float*>(o),
                                      B * H, dk, dv, 64, tune.decode_nt, kla::kOptDiagDecay | opts, st);
    return e == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

int kla_debug_chunk_stage(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                          float eps, const float* h0, void* o, float* hT, const int32_t* cu_seqlens_dev,
                          const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int dv, int chunk,
                          kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream, int stage)
{
    if (stage != 1 && stage != 2) return KLA_ERR_SHAPE;
    return chunk_fwd_checked(q, k, v, log_alpha, eta, eps, h0, o, hT, cu_seqlens_dev, cu_seqlens_host, n_seq, N, T, H,
                             dk, dv, chunk, dt, workspace, workspace_bytes, hip_stream, stage, KLA_TUNE_UNFUSED);
}

int kla_debug_intra_chunk(const void* q, const void* k, const float* log_alpha, const float* eta, float eps,
                          float* Tb_out, float* P_out, float* g_out, const int32_t* cu_seqlens_dev,
                          const int32_t* cu_seqlens_host, int n_seq, int N, int T, int H, int dk, int chunk,
                          kla_dtype dt, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    Plan pl;
    const int rc = make_plan(N, T, H, dk, 64, chunk, (int)dt, cu_seqlens_host, n_seq, KLA_TUNE_UNFUSED, &pl);
    if (rc != KLA_OK) return rc;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (n_seq > 0 && !cu_seqlens_dev) return KLA_ERR_NULL;
    if (n_seq == 0 && cu_seqlens_dev) return KLA_ERR_SHAPE;
    if (!q || !k || !log_alpha || !eta || !Tb_out || !P_out || !g_out) return KLA_ERR_NULL;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < pl.total)
        return KLA_ERR_WORKSPACE;
    if (!aligned16(q) || !aligned16(k)) return KLA_ERR_ALIGN;
    if (pl.n_chunks == 0) return KLA_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char* ws = static_cast<char*>(workspace);
    if (dt == KLA_BF16)
        return chunk_fwd_impl<bf16_t>(q, k, nullptr, log_alpha, eta, eps, nullptr, nullptr, nullptr, cu_seqlens_dev,
                                      n_seq, N, T, H, dk, 64, pl, ws, 5, Tb_out, P_out, g_out, st, 0u);
    return chunk_fwd_impl<float>(q, k, nullptr, log_alpha, eta, eps, nullptr, nullptr, nullptr, cu_seqlens_dev, n_seq, N,
                                 T, H, dk, 64, pl, ws, 5, Tb_out, P_out, g_out, st, 0u);
}

int kla_debug_peak_probe(int kind, void* buf, void* aux, size_t bytes, int iters, void* hip_stream)
{
    if (kind < 0 || kind > 3 || iters < 0) return KLA_ERR_SHAPE;
    if (kind == 3) {
        const int ni = iters & 255, depth = 1 + (iters >> 8);
        if ((ni != 16 && ni != 32 && ni != 48 && ni != 60) || depth > 2) return KLA_ERR_SHAPE;
        if (!buf) return KLA_ERR_NULL;
        if (!aligned16(buf)) return KLA_ERR_ALIGN;
        if (bytes < (size_t)8 * 64 * ni * 4 * 2048) return KLA_ERR_WORKSPACE;
    } else if (kind == 2) {
        if (bytes == 0 || bytes > 0x7fffffffu || iters == 0) return KLA_ERR_SHAPE;
        if (!aux) return KLA_ERR_NULL;
    } else {
        if (bytes == 0 || bytes % 65536 != 0 || bytes / 65536 > 0x7fffffffu) return KLA_ERR_SHAPE;
        if (!buf || (kind == 1 && !aux)) return KLA_ERR_NULL;
        if (!aligned16(buf)) return KLA_ERR_ALIGN;
    }
    return kla::launch_probe(kind, buf, aux, bytes, iters, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

int kla_decode_step(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta, float eps,
                    float* S, void* o, int B, int H, int dk, int dv, kla_dtype dt, void* hip_stream)
{
    return kla_decode_step_opts(q, k, v, log_alpha, eta, eps, S, o, B, H, dk, dv, dt, hip_stream, 0u);
}

int kla_decode_step_opts(const void* q, const void* k, const void* v, const float* log_alpha, const float* eta,
                         float eps, float* S, void* o, int B, int H, int dk, int dv, kla_dtype dt, void* hip_stream,
                         unsigned opts)
{
    if (!dt_ok((int)dt)) return KLA_ERR_DTYPE;
    Tune tune;
    if (!parse_tune(opts, &tune)) return KLA_ERR_SHAPE;
    opts &= kOptMask;
    if (B < 0 || H <= 0 || !dk_ok(dk) || !dv_ok(dv) || (long)B * H > 0x7fffffffL) return KLA_ERR_SHAPE;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (B == 0) return KLA_OK;
    if (!q || !k || !v || !log_alpha || !eta || !S || !o) return KLA_ERR_NULL;
    if (!aligned16(S) || (reinterpret_cast<uintptr_t>(q) & 3u) || (reinterpret_cast<uintptr_t>(k) & 3u) ||
        (reinterpret_cast<uintptr_t>(v) & 3u) || (reinterpret_cast<uintptr_t>(o) & 3u) ||
        (reinterpret_cast<uintptr_t>(log_alpha) & 3u) || (reinterpret_cast<uintptr_t>(eta) & 3u))
        return KLA_ERR_ALIGN;
    // State columns per workgroup: 128 (measured best at 512 workgroups, e.g. 64 x 8 states of 128 columns), narrower for
    // small batches so that about 512 workgroups still share the chip (B = 1, H = 8: 3.2 us per step with 32 columns,
    // 4.2 us with 128).  The tuning field KLA_TUNE_DECODE_SLICE(32 | 64 | 128 | 256) overrides.
    int slice = dv < 128 ? dv : 128;
    while (slice > 32 && (long)B * H * (dv / slice) < 512) slice >>= 1;
    if (tune.decode_slice) slice = tune.decode_slice;
    if (slice > dv) slice = dv;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e;
    if (dt == KLA_BF16)
        e = kla::launch_decode<bf16_t>(static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k),
                                       static_cast<const bf16_t*>(v), log_alpha, eta, eps, S, static_cast<bf16_t*>(o),
                                       B * H, dk, dv, slice, tune.decode_nt, opts, st);
    else
        e = kla::launch_decode<float>(static_cast<const float*>(q), static_cast<const float*>(k),
                                      static_cast<const float*>(v), log_alpha, eta, eps, S, static_cast<float*>(o),
                                      B * H, dk, dv, slice, tune.decode_nt, opts, st);
    return e == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

int kla_beta(const void* k, const float* eta, float eps, float* beta, long n_token_heads, int dk, kla_dtype dt,
             void* hip_stream)
{
    if (!dt_ok((int)dt)) return KLA_ERR_DTYPE;
    if (n_token_heads < 0 || !dk_ok(dk) || (n_token_heads * (dk / 8) + 255) / 256 > 0x7fffffffL) return KLA_ERR_SHAPE;
    if (!(eps >= 0.0f) || isinf(eps)) return KLA_ERR_SHAPE;
    if (n_token_heads == 0) return KLA_OK;
    if (!k || !eta || !beta) return KLA_ERR_NULL;
    if (!aligned16(k)) return KLA_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const hipError_t e = dt == KLA_BF16
        ? kla::launch_beta<bf16_t>(static_cast<const bf16_t*>(k), eta, eps, beta, n_token_heads, dk, st)
        : kla::launch_beta<float>(static_cast<const float*>(k), eta, eps, beta, n_token_heads, dk, st);
    return e == hipSuccess ? KLA_OK : KLA_ERR_HIP;
}

}  // extern "C"
