// Which kernel variant or tile shape a call takes, as plain functions of its
// sizes, so that they can be looked over and tested without a GPU.  Each
// comment says what was measured on both sides of the line (MI355X, 256 CUs).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

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

// Whether lane `tid` of a workgroup that evaluates nodes k = b span + tid, of
// which the next one's begin after `span`, stores node k: the last of N + 1
// nodes is the overlap's first where the workgroups end with the intervals.
constexpr bool owns_node(int tid, int64_t k, int64_t N, int span)
{
    return k <= N && (tid < span || (tid == span && k == N));
}

// Whether the adjoint of the coefficient gradient stores its `values` doubles
// past the caches: from 8 MiB on (n = 8, N = 100,000: 16.2 -> 13.5 us, n = 16,
// N = 1e6 258 -> 236, n = 12, N = 333,333 52.2 -> 50.8); a short call waits
// longer for such stores (n = 2, N = 1000 4.4 -> 4.6 us, n = 4, N = 50,001 6.7 ->
// 7.0, n = 8, N = 20,000 11.1 -> 11.4).
constexpr bool adjoint_nt(int64_t values) { return values * 8 > 8 * kMiB; }

// LDS doubles of one defect-row tile of KT intervals of the fused KKT values (n
// states, m controls, T Jacobian slots per row): states and cosines at KT+1
// nodes, the rows' regularization, the scaled coefficients, the output row block.
inline size_t kkt_defect_lds(int n, int m, int T, int KT)
{
    return 2 * (size_t)n * (KT + 1) + (size_t)n * KT + (size_t)n * (n + m) + (size_t)n + (size_t)KT * (T + 1);
}

// Intervals per defect-row tile: 16, 32 or 64, for the instances Ns evaluated
// together (one, or a batch).  Row blocks of 64 (T + 1) entries store the
// fewest lines in part (n = 16: 1.09 ms against 1.10 and 1.10 at N = 1e6,
// n = 6: 0.359 against 0.383 and 0.43 at N = 2e6), but a short grid needs
// smaller tiles to reach every CU, the sooner the more work a tile is: n = 3,
// N = 20,000 10.0 us with 64 and 11.0 with 16; n = 4, N = 5000 11.4, with 32
// 10.3; n = 8, N = 20,001 (forward Euler) 22.4, 19.8; n = 16, N = 20,000 55,
// with 32 43.0, with 16 45; n = 16, N = 20,001 (forward Euler) 50, 40.8, 38.0.
// Forward Euler stores half as much per cosine and per barrier and needs more
// workgroups per CU to hide them: its tile gets half the LDS (n = 16, N = 1e6:
// 0.719 ms with 32 intervals in 22 KB, 0.885 with 64 in 41 KB), and until 64 pay
// the trapezoidal one three quarters (n = 32, N = 33,000: 245 us with 32
// intervals in 62 KB, 225 with 16).  In a batch, a tile taller than its instance
// computes rows that it does not store (4096 instances of 16 intervals, n = 16:
// 327 us with 64, 229 with 16): the tile is halved while that saves a third of
// the rows.
constexpr size_t kDefectLdsMax = 64 * 1024;  // bytes of LDS a tile may take
inline int kkt_defect_kt(int n, int m, int T, bool euler, const int64_t *Ns, int64_t count)
{
    int64_t total = 0;
    for (int64_t i = 0; i < count; i++) total += Ns[i];
    auto rows = [&](int KT) {
        int64_t r = 0;
        for (int64_t i = 0; i < count; i++) r += (Ns[i] + KT - 1) / KT * KT;
        return r;
    };
    const int64_t k = total / 1024;
    const int T1 = T + 1;
    const int64_t from64 = T1 < 10 ? 16 : T1 < 17 ? 40 : 64, from32 = T1 < 10 ? 0 : T1 < 17 || !euler ? 16 : 32;
    const size_t lds = euler ? kDefectLdsMax / 2 : k >= 64 ? kDefectLdsMax : kDefectLdsMax / 4 * 3;
    auto fits = [&](int KT) { return kkt_defect_lds(n, m, T, KT) * sizeof(double) <= lds; };
    int KT = k >= from64 ? 64 : k >= from32 ? 32 : 16;
    while (KT > 16 && !fits(KT)) KT /= 2;
    // instances of an even number of 16s: half the tiles for the same rows
    if (count > 1 && KT == 16 && fits(32) && rows(32) == rows(16)) KT = 32;
    while (KT > 16 && 2 * rows(KT) >= 3 * rows(KT / 2)) KT /= 2;
    return KT;
}

// Jacobian tiles of a batch, one column of a run of intervals per workgroup:
//   kBatchDirect  one or two intervals per lane, stored directly
//   kBatchShort   one interval per lane in the kernel of the whole-line tiles,
//                 which more workgroups fit: an instance gives a tile one
//                 wavefront's work or little more, and only workgroups in flight
//                 hide its descriptors and loads
//   kBatchLines   whole lines of 2 `block` - 16 intervals (instances whose rows
//                 begin on lines stored directly among them)
// A whole-line tile takes its full time however few intervals it stores, so
// what counts is its wavefronts against those of the direct tiles (r): at
// N = 17, n = 6 (346 MB) whole lines take 2.4 times as long, at r = 1.1 and
// n = 6 1.2 times, n = 16 0.91 times, at r = 0.8 and 122 MB 1.15 times, at
// r = 0.6 0.8 times (n = 4 .. 24, 0.7 to 0.9 GB); below the size of the L2s
// direct stores merge there and win (n = 4, 26 MB: 8.4 against 9.0 us; n = 8,
// 54 MB: 16.5 against 14.5).  Forward Euler stores half as much per node:
// r = 0.75 and 96 MB still 1.12 times.  Rows that all begin on lines need none
// of it: direct (N = 384, n = 6: 33 against 37 us).
// kBatchShort against kBatchDirect: N in 10 .. 60, n = 6 57 against 64 us,
// forward Euler (n = 8) 83 against 115, N in 50 .. 200 37 against 42, but
// under the trapezoidal scheme N in 50 .. 200, n = 8, 56 against 50.
enum BatchJac { kBatchDirect = 0, kBatchShort, kBatchLines };

inline BatchJac batch_jac(const std::vector<int64_t> &Ns, int n, int slots, bool euler, bool pair, int block)
{
    const int64_t span = 2 * block - kLineDoubles, waves = block / 64, count = (int64_t)Ns.size();
    int64_t intervals = 0, direct = 0, lines = 0;  // and wavefronts of each form, per column
    bool on_lines = true;
    for (int64_t N : Ns) {
        intervals += N;
        on_lines = on_lines && N % kLineDoubles == 0;
        direct += (N + 63) / 64;
        lines += (N + kLineDoubles - 1 + span - 1) / span * waves;
    }
    const int64_t bytes = (int64_t)n * slots * intervals * 8;
    if (10 * direct <= 11 * count || (euler && intervals <= 128 * count)) return kBatchShort;
    if (!pair || on_lines) return kBatchDirect;
    // the largest r, in hundredths: higher for an output that no cache holds,
    // and then with many rows per column
    const bool large = bytes > 256 * kMiB;
    const int64_t r = euler ? (large && n >= 12 ? 80 : 70) : !large ? 78 : n >= 8 ? 110 : 85;
    return 100 * lines <= r * direct && bytes > (euler ? 48 : 40) * kMiB ? kBatchLines : kBatchDirect;
}

// Objective and gradient of a batch together: tiles that load each node once,
// unless one round of them leaves CUs idle that tiles of their own for each
// would use (256 instances of 50 to 200 intervals: n = 2 5.1 against 5.6 us,
// n = 24 13.2 against 15.9; 512 such: 5.7 against 5.8 and 19.8 against 17.6;
// 4096 of 10 to 60, n = 6: 24.5 against 13.8).
inline bool batch_obj_grad_once(const std::vector<int64_t> &Ns)
{
    int64_t tiles = 0;  // of 256 nodes
    for (int64_t N : Ns) tiles += N / 256 + 1;
    return tiles > 256;
}

// log2 of the constraint rows per tile of the assembly: 128 rows while their
// T + 1 entries each fit 64 KiB of LDS, else 64 or 32, and fewer where that
// leaves most CUs without a tile.  From 128 tiles on the taller ones win (128
// rows against 64 or 32: n = 4, N = 16,000 6.7 us and 7.5; n = 8, N = 4000 8.1
// and 8.4; n = 16, N = 1000 11.2 and 12.2; n = 2, N = 16,000 5.5 and 5.9),
// below that the shorter (n = 4, N = 1000: 5.4 and 5.1; n = 2, N = 4000: 5.3
// and 5.0).
inline int assembly_lg(int64_t N, int n, int T)
{
    int lg = 7;
    auto tiles = [&] { return ((N + (1 << lg) - 1) >> lg) * n; };
    while (lg > 5 && (((size_t)(T + 1) << lg) * sizeof(double) > 64 * 1024 || tiles() < 128)) lg--;
    return lg;
}

// log2 of the nodes per tile of the mapped assembly, for N1 nodes of `per_node`
// entries (and 2 n that overhang): as many as fit 16 KiB of values, 32 KiB
// (five workgroups per CU) where that leaves two tiles per CU, 4 nodes while
// those fit 62 KiB, and up to 8 (half a line of values) in 72 KiB while 250
// tiles are left, 400 with 8 nodes, to reach every CU.  n = 18, m = 10: 16.9 us
// with 8 nodes and 20.5 with 4 at N = 4000, 12.7 and 11.0 at N = 2000, 10.1 and
// 6.4 at N = 100.  Fewer than 4 nodes would gain on the shortest grids (n = 18,
// N = 100: one node 4.4 us), but a plan that a caller kept from a library with
// tiles of 4 would be too short for them, and its length is not passed.
constexpr int kMapCap = 9216;  // most values staged per workgroup (72 KiB, two workgroups per CU)
inline int map_lg(int64_t N1, int64_t per_node, int n)
{
    auto need = [&](int lg) { return ((int64_t)1 << lg) * per_node + 2 * n; };
    int lg = 0;
    while (lg < 10 && need(lg + 1) <= 2048) lg++;
    const bool many = (N1 >> (lg + 1)) >= 512;
    while (many && lg < 10 && need(lg + 1) <= 4096) lg++;
    while (lg < 2 && need(lg + 1) <= 7936) lg++;
    while (lg < 3 && need(lg + 1) <= kMapCap && (N1 >> (lg + 1)) >= (lg < 2 ? 250 : 400)) lg++;
    return lg;
}

}  // namespace rules
}  // namespace ocp
