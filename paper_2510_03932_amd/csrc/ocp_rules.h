// Which kernel variant or tile shape a call takes, as plain functions of its
// sizes, so that they can be looked over and tested without a GPU.  Each
// comment says what was measured on both sides of the line (MI355X, 256 CUs).
#pragma once

#include <algorithm>
#include <cstdint>

namespace ocp {
namespace rules {

constexpr int64_t kMiB = 1 << 20;
constexpr int kLineDoubles = 16;     // doubles per 128-byte line
constexpr int kJacLinesSpan = 496;   // intervals a workgroup of 256 lanes stores in whole lines (2 * 256 - 16)

enum JacPath { kJacSingle = 0, kJacPair, kJacLines };

// Single-instance Jacobian values: `slots` slot rows of N values for each of n
// components, from address `addr`; one interval per lane, two (16-byte stores),
// or whole lines from LDS.
//
// Rows in whole lines need enough workgroups to hide the LDS pass: 560 of them
// (700 under forward Euler, which stores one row per column, not two) gain at
// odd N (n = 4: 6.4 -> 5.7 us at N = 52,081; n = 32: 43.5 -> 30.5 at N = 5457),
// fewer lose (n = 8: 6.3 -> 8.6 at N = 13,009; n = 32: 15.3 -> 22.4 at
// N = 2049).  Rows that can take pairs (an even N) gain only beyond the size of
// the L2s, which merge the partial lines (n = 8, lines against pairs: 28 MB 9.0
// and 7.6, 90 MB 18.3 and 22.6), rows that begin on lines or half lines show no
// gain that the runs agree on (n = 8 and 400 MB 72-75 against 69-74), and a
// column of fewer than four slot rows (n = 1, forward Euler) has none.
//
// Pairs against single intervals: pairs win (n = 2: 5.1 against 5.8 us at
// 20 MB, n = 1 under forward Euler: 8.3 against 13.0 at 40 MB), except where
// the whole output is in flight at once (n = 8: 5.7 against 4.8 at 20 MB,
// n = 16: 7.6 against 6.4 at 28 MB; forward Euler, with half the stores per
// cosine, up to a fifth of that).
inline JacPath jac_path(int64_t N, int n, int m, int slots, bool euler, uint64_t addr)
{
    const int64_t bytes = (int64_t)n * N * slots * 8;
    const int64_t line_wgs = (N + kLineDoubles - 1 + kJacLinesSpan - 1) / kJacLinesSpan * (n + m);
    const bool fills = line_wgs >= (euler ? 700 : 560);
    if (N % 2 != 0 || addr % 16 != 0) return fills ? kJacLines : kJacSingle;
    if (bytes <= std::min<int64_t>(28, n * (euler ? 1 : 5)) * kMiB) return kJacSingle;
    const bool halves = N % 8 == 0 && addr % 64 == 0;
    return !halves && fills && slots >= 4 && bytes > 32 * kMiB ? kJacLines : kJacPair;
}

// The quadrotor's Jacobian values (68 slots): whole lines evaluate each node's
// partials once, and gain from 500 workgroups on at any alignment once the
// output exceeds the L2s (N = 80,000: 10.2 -> 10.0 us, 80,001: 12.5 -> 10.1),
// and below that for rows off half lines (N = 30,001: 6.4 -> 6.0); fewer
// workgroups leave the chip idle (N = 10,000: 4.0 -> 4.7).  Pairs gain over
// single intervals from about 12 MiB on (N = 30,000: 5.2 against 5.8 us,
// 20,000: 5.1 against 4.7).
inline JacPath quad_jac_path(int64_t N, uint64_t addr)
{
    const int64_t bytes = 68 * N * 8;
    const bool fills = (N + kLineDoubles - 1 + kJacLinesSpan - 1) / kJacLinesSpan * 9 >= 500;
    const bool halves = N % 8 == 0 && addr % 64 == 0;
    if (fills && (!halves || bytes > 30 * kMiB)) return kJacLines;
    return halves && bytes > 12 * kMiB ? kJacPair : kJacSingle;
}

}  // namespace rules
}  // namespace ocp
