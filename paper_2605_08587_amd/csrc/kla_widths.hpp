// Compute waves per workgroup (16 state columns each) of the sweeps whose width follows from the lengths of the sequences. Host
// code without GPU calls.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <functional>

namespace kla {

// The sequences of a call, as far as the lengths of its sweeps go: n of them of NT chunks each, or (cu != NULL) packed.
struct Lengths { int n, NT; const int32_t* cu; };

// Chunk steps the busiest CU takes in a sweep of `slices` workgroups per (sequence, head), one at a time on a CU (a bf16
// workgroup fills one with its LDS).  Equal lengths: rounds of workgroups times chunks.  A packed batch starts its workgroups
// longest sequence first, each on the first CU to become free, so a second round of shorter ones costs less than a
// round: that schedule is played through, for batches small enough that it matters. `start`: what a workgroup takes besides its
// chunks, in steps.
inline long busiest_cu(const Lengths& s, int H, int slices, int start = 0)
{
    constexpr int kCUs = 256;
    if (!s.cu) return (((long)s.n * H + 7) / 8 * 8 * slices + kCUs - 1) / kCUs * ((s.NT > 1 ? s.NT : 1) + start);
    const long per_seq = (long)H * slices;
    auto steps = [&](int i) { const int c = (s.cu[i + 1] - s.cu[i] + 63) / 64; return c > 0 ? c + start : 0; };
    long longest = 0, total = 0;
    for (int i = 0; i < s.n; ++i) {
        const long c = steps(i);
        longest = std::max(longest, c);
        total += c;
    }
    if (s.n > 64 || s.n * per_seq > 4096) return std::max(longest, (total * per_seq + kCUs - 1) / kCUs);
    int len[64];
    for (int i = 0; i < s.n; ++i) len[i] = steps(i);
    std::sort(len, len + s.n, std::greater<int>());
    struct { long load; int n; } level[kCUs + 1] = {{0, kCUs}};   // CUs by load, least first
    int k = 1;
    for (int i = 0; i < s.n && len[i] > 0; ++i) {
        for (long left = per_seq; left > 0;) {
            const int m = (int)std::min<long>(left, level[0].n);
            const long to = level[0].load + len[i];
            left -= m;
            if ((level[0].n -= m) == 0) std::copy(level + 1, level + k--, level);
            int at = 0;
            while (at < k && level[at].load < to) ++at;
            if (at < k && level[at].load == to) level[at].n += m;
            else { std::copy_backward(level + at, level + k, level + k + 1); ++k; level[at] = {to, m}; }
        }
    }
    return level[k - 1].load;
}

// Whether a sweep with one wave per workgroup ends before one with two (32 columns), whose step is `step2` percent as long: while every
// chain has a CU to itself, and for a packed batch so unequal that the second round fits behind the longest sequence. A
// workgroup's start is taken as three steps, which decides for short sequences (backward of {211, 186, 148, 128, 329, 346, 265, 82, 254}
// tokens, d_k = d_v = 64, 8 heads, training step 52 us with two waves and 53 with one: 9 steps against 10, by two steps a tie).
inline bool one_wave(const Lengths& s, int H, int dv, int step2)
{
    const long chains8 = ((long)s.n * H + 7) / 8 * 8;
    return chains8 * (dv / 16) <= 256 || busiest_cu(s, H, dv / 16, 3) * 100 <= busiest_cu(s, H, dv / 32, 3) * step2;
}

// Compute waves of the backward's bf16 sweeps: one, two or (where the kernel has them) four. Two against one: a step of the reverse
// sweep is 1.1 (every CU busy) to 1.4 times as long, of the forward sweep 1.0 to 1.1. Whole backward, d_k = d_v = 128, 8 heads, with one and
// with two: 4 x 2000 tokens (256 chains) 139 and 143 us; 5 x 2000 (two rounds against one) 201 and 159; packed {4000, 300, 300, 300,
// 200} 168 and 203, {2500, 1200, 1000, 800, 600} 134 and 155, {2000, 1900, 1900, 1800, 300} (40 steps against 35) 145.5 and 145.1 (d_k =
// d_v = 64, 16 heads: 138 and 136), {3000, 100} of 16 heads, d_v = 256 (55 against 50) 190 and 193; 4000 and 40 x 200 (87 against 66) 260
// and 256; 8000 and 70 x 100 392 and 420. (The forward sweep by itself, whose workgroups of one wave fit twice on a CU, goes the same
// way: 5 x 2000 8 us longer with one, {4000, ..} 2 shorter.)
// Four (64 columns) where that shortens the work of the busiest CU: their visits are about 1.15 times as long as with two (8 x 4096
// tokens, 8 heads, one round either way: 469 us with two, 511 us with four; 9 x 2000, two rounds against one: 305, 251; 8 x 2048, d_v =
// 256: 392, 347; 40 x 1000, five rounds against three: 584, 520).
inline int sweep_waves(const Lengths& s, int H, int dv, bool four)
{
    if (one_wave(s, H, dv, 110)) return 1;
    return four && dv >= 64 && busiest_cu(s, H, dv / 64) * 115 < busiest_cu(s, H, dv / 32) * 100 ? 4 : 2;
}

// Compute waves of the per-channel scan (bf16). Whole call, d_k = 128, 8 heads, d_v = 128, with one and two: 5 x 2000 tokens 132 and 94 us,
// packed {4000, 300, 300, 300, 200} 109 and 114, {2500, 1200, 1000, 800, 600} 90 and 93, {2000, 1800, 1700, 1600, 300} (36 steps
// against 35) 83 and 84, {2000, 1900, 1900, 1800, 300} (40 against 35) 87 and 84, {130, 70, 60, 30, 20} (8 against 6) 25.5 and 23.8.
// At d_k = 64 two are as fast at equal steps ({4000, 300, 300, 300, 200}, 16 heads, d_v = 64: 103 and 100; 8 heads, d_v = 128: 79 and 79).
inline int diag_scan_waves(const Lengths& s, int H, int dk, int dv) { return one_wave(s, H, dv, dk == 128 ? 100 : 0) ? 1 : 2; }

}  // namespace kla
