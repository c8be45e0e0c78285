// Per-node device arithmetic shared by the single-instance kernels and the
// batched persistent kernel of the evaluation library (gfx950, wave64).
//
// Every evaluation maps one grid node (or one interval) to one lane, the SIMD
// structure of direct transcription (paper Sec. 3): the same few functions are
// evaluated at every node.  All arrays are structure-of-arrays with the node
// index fastest, so the lanes of a wavefront touch consecutive doubles.
//
// Formulas (component-major unknowns, h = 1/N, hh = h/2, p(i) = (i+1) mod n):
//   F_i(k)   = sum_j A_ij sin X_jk + sum_l B_il U_lk + gamma_i X_ik X_{p(i)k}
//   c_{ik}   = (X_{i,k+1} - X_ik) - hh (F_i(k) + F_i(k+1))         [Sec. 5]
//   f        = sum_k w_k (sum_j q_j X_jk^2 + sum_l r_l U_lk^2)     [Sec. 5]
//   dF_i/dX_j = A_ij cos X_j + gamma_i (delta_ij X_p(i) + delta_j,p(i) X_i)
//   Hessian of L = sigma f + y^T c at node k uses the node multiplier
//   yt_ik = y_{i,k-1} [k >= 1] + y_{ik} [k < N]  (node k is the right end of
//   interval k-1 and the left end of interval k).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ocp {
namespace dev {

typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));  // FP64 MFMA 16x16 accumulator

// pairs loaded from any element of an array
typedef double dbl2_any __attribute__((ext_vector_type(2), aligned(8)));
typedef int32_t int2_any __attribute__((ext_vector_type(2), aligned(4)));
constexpr int kAsmBatch = 4;  // pairs in flight per lane in the KKT assembly

constexpr int kBlock = 256;  // threads per workgroup of the single-instance kernels (4 waves)

// Kernel-side view of one problem: sizes and device coefficient pointers.
struct KP {
    int N;         // intervals
    int N1;        // nodes = N + 1
    int n, m, npair, T, S;
    int nnzk;      // KKT entries
    int NU;        // control nodes: N + 1 (trapezoidal) or N (forward Euler)
    int scheme;    // 0 trapezoidal, 1 forward Euler
    int nb;        // boundary rows after the n N defect rows
    double h, hh;
    const double *A;    // n x n row-major
    const double *B;    // n x m row-major
    const double *gam;  // n
    const double *q;    // n
    const double *r;    // m
    const double *AT;   // n columns of kLd: AT[j kLd + i] = A_ij (i < n), 0 (n <= i < kLd)
    const double *BT;   // m columns of kLd: BT[l kLd + i] = B_il (i < n), 0 (n <= i < kLd)
};

// Column stride of the padded copies AT and BT (the bound on n).  A kernel
// whose register bound NB <= kLd sums a column over all NB rows without a
// guard, the padding adding exact zeros; the column's entries are contiguous
// at offsets known at compile time, so a wavefront fetches them with a few
// wide scalar loads instead of one load per coefficient behind a branch.
constexpr int kLd = 32;

// Host side: the padded copies of one instance's A (n x n) and B (n x m),
// both row-major, into AT (n kLd doubles) and BT (m kLd doubles).
inline void pack_columns(int n, int m, const double *A, const double *B, double *AT, double *BT)
{
    for (int j = 0; j < n; j++)
        for (int i = 0; i < kLd; i++) AT[j * kLd + i] = i < n ? A[i * n + j] : 0.0;
    for (int l = 0; l < m; l++)
        for (int i = 0; i < kLd; i++) BT[l * kLd + i] = i < n ? B[i * m + l] : 0.0;
}

// Cost weight of node k: trapezoidal rule (end nodes h/2), or the forward
// Euler sum over nodes 0..N-1 (weight h, none at node N).
__device__ __forceinline__ double node_weight(const KP &P, int k)
{
    if (P.scheme) return k < P.N ? P.h : 0.0;
    return (k == 0 || k == P.N) ? P.hh : P.h;
}

__device__ __forceinline__ void st_nt(double *p, double v) { __builtin_nontemporal_store(v, p); }
// A store that is non-temporal when NT (the default for outputs), else an
// ordinary one.
template <bool NT>
__device__ __forceinline__ void st_out(double *p, double v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
__device__ __forceinline__ void st_nt2(double *p, dbl2 v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<dbl2 *>(p));
}

// ---------------------------------------------------------------------------
// Workgroups are dispatched round-robin over the chip's 8 XCDs, each with an
// L2 of its own.  xcd_order maps the dispatch index b of nb workgroups to a
// work index so that each XCD takes one contiguous run of the work (a
// bijection of [0, nb)): neighbouring tiles then share an L2, which merges the
// lines that two tiles each write (or read) a part of.
// ---------------------------------------------------------------------------
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t xcd_order(uint32_t b, uint32_t nb)
{
    const uint32_t x = b % kXcds, q = nb / kXcds, r = nb % kXcds;
    return x * q + (x < r ? x : r) + b / kXcds;
}

// ---------------------------------------------------------------------------
// A workgroup of BS lanes copies cnt doubles from LDS to out (position sh in
// its line), placed so that every wavefront's store begins on a
// 128-byte line of HBM: pure 3 GiB write streams reach 5.7-6.2 TB/s that way
// and 3.4-4.5 TB/s from anywhere else (8-byte lanes, 784-double runs), since
// each wavefront then completes its lines instead of leaving two of them to be
// merged with a neighbour's.  Non-temporal 8-byte stores: 16-byte ones measured
// the same or slower here, ordinary ones 10-30 % slower.
//
// Where an output begins within its line (0 .. 15 doubles) is a kernel
// argument, `al`, computed on the host by line_pos: a kernel that looks at an
// output's address itself loses the proof that its stores leave the
// coefficients alone, and loads those lane by lane instead of through the
// scalar cache.
// ---------------------------------------------------------------------------
constexpr int kLine = 16;  // doubles per 128-byte line
inline int line_pos(const double *p) { return (int)(((uintptr_t)p / sizeof(double)) % kLine); }
// The position of element i of an output that begins at position al.
__device__ __forceinline__ int line_pos_at(int al, int64_t i) { return (int)((al + i) & (kLine - 1)); }
// Intervals per workgroup of the kernels whose lanes exchange values with the
// next node's (kBlock nodes close kBlock - 1): a multiple of a line.
constexpr int kSpan = kBlock - kLine;
template <int BS>
__device__ __forceinline__ void copy_lines(double *__restrict__ out, int sh, const double *src, int cnt)
{
    int x = (int)threadIdx.x - sh;
    if (x >= 0 && x < cnt) st_nt(out + x, src[x]);
    for (x += BS; x < cnt; x += BS) st_nt(out + x, src[x]);
}

// Fixed-shape sums: over a wavefront (cross-lane shuffles, tree of halving
// offsets) and over a workgroup of BS lanes (wavefront sums, then the BS/64
// wave totals in order).  The order of additions never depends on timing.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

template <int BS>
__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double ws[BS / 64];
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) ws[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < BS / 64; i++) t += ws[i];
    }
    return t;  // valid in thread 0
}

// A reduction's second pass, one workgroup of kBlock lanes: lane t adds
// partials t, t + kBlock, ... in order, kSumBatch of them loaded at a time
// (one at a time, each addition waited for its own load), then the fixed tree.
// The result is valid in thread 0.
constexpr int kSumBatch = 8;
__device__ __forceinline__ double sum_partials(const double *__restrict__ partials, int count)
{
    double acc = 0.0;
    for (int i0 = threadIdx.x; i0 < count; i0 += kSumBatch * kBlock) {
        double v[kSumBatch];
#pragma unroll
        for (int u = 0; u < kSumBatch; u++) v[u] = i0 + u * kBlock < count ? partials[i0 + u * kBlock] : 0.0;
#pragma unroll
        for (int u = 0; u < kSumBatch; u++)
            if (i0 + u * kBlock < count) acc += v[u];
    }
    return block_sum<kBlock>(acc);
}

// ---------------------------------------------------------------------------
// Jacobian values, one column of the node-local variables at a time.  Column
// col < n is state column j: it writes slots 2j, 2j+1 (nodes k, k+1) of every
// row i under the trapezoidal scheme; col = n + l is control column l, the
// constants -hh B_il.  Forward Euler (paper Sec. 3): row i's slots, in
// ascending column order, are X_0..X_i at k (slots 0..i), X_i at k+1 (slot
// i+1), X_{i+1}..X_{n-1} at k (slots i+2..n), U_l at k (slot n+1+l), so state
// column j writes slot (j <= i ? j : j+1) of every row i and the +1 at slot
// j+1 of row j.
//
// The bilinear term touches only rows i = j (partner X_{j+1}) and i = j-1
// (factor X_{j-1}).  jac_entry is the state columns' value, the same bits
// wherever it is used: a = -w A_ij, c = cos X_j, id the identity's part,
// gj = -w gamma_j, gp = -w gamma_{j-1}, xn = X_{j+1}, xp = X_{j-1}, all at the
// slot's node.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double jac_entry(bool own, bool prev, double a, double c, double id, double gj, double gp,
                                            double xn, double xp)
{
#pragma clang fp contract(off)
    double v = a * c;
    if (own) v = __builtin_fma(a, c, __builtin_fma(gj, xn, id));
    const double lo = gp * xp;
    if (prev) v = lo + v;
    return v;
}

// One column at NPT intervals k .. k + NPT - 1 < N, stored directly.  NPT = 2
// stores a 16-byte pair per lane, so a wavefront's store is one contiguous KiB
// of a slot row: it needs an even N and 16-byte aligned rows (see jac_path for
// the choice).  The scheme is a template argument: with it read from P, the
// smallest calls took up to 15 % longer (N = 17, n = 32).
template <int NPT, bool EULER>
__device__ __forceinline__ void jac_column(const KP &P, const double *__restrict__ z, double *__restrict__ jac,
                                           int64_t k, int col)
{
    constexpr int kNodes = EULER ? NPT : NPT + 1;
    const int n = P.n, m = P.m, T = P.T;
    const int64_t N = P.N, N1 = P.N1;
    const double w = EULER ? P.h : P.hh;
    auto put = [](double *o, const double (&v)[NPT]) {
        if constexpr (NPT == 2) st_nt2(o, dbl2{v[0], v[1]});
        else st_nt(o, v[0]);
    };
    double v[NPT];
    if (col < n) {
        const int j = col;
        const int jn = (j + 1 == n) ? 0 : j + 1;
        const int jp = (j == 0) ? n - 1 : j - 1;
        const double gj = -w * P.gam[j], gp = -w * P.gam[jp];
        const double *xj = z + j * N1 + k, *xn = z + jn * N1 + k, *xp = z + jp * N1 + k;
        double cs[kNodes], vn[kNodes], vp[kNodes];
#pragma unroll
        for (int u = 0; u < kNodes; u++) {
            cs[u] = cos(xj[u]);
            vn[u] = xn[u];
            vp[u] = xp[u];
        }
        for (int i = 0; i < n; i++) {
            const double a = -w * P.A[i * n + j];
            const bool own = i == j, prev = i == jp;
            double v1[NPT];
#pragma unroll
            for (int u = 0; u < NPT; u++) {
                v[u] = jac_entry(own, prev, a, cs[u], -1.0, gj, gp, vn[u], vp[u]);
                if constexpr (!EULER) v1[u] = jac_entry(own, prev, a, cs[u + 1], 1.0, gj, gp, vn[u + 1], vp[u + 1]);
            }
            double *o = jac + ((int64_t)i * T + (!EULER ? 2 * j : j <= i ? j : j + 1)) * N + k;
            put(o, v);
            if constexpr (!EULER) put(o + N, v1);
        }
        if constexpr (EULER) {
#pragma unroll
            for (int u = 0; u < NPT; u++) v[u] = 1.0;
            put(jac + ((int64_t)j * T + j + 1) * N + k, v);
        }
    } else {
        const int l = col - n;
        for (int i = 0; i < n; i++) {
#pragma unroll
            for (int u = 0; u < NPT; u++) v[u] = -w * P.B[i * m + l];
            double *o = jac + ((int64_t)i * T + (EULER ? n + 1 + l : 2 * (n + l))) * N + k;
            put(o, v);
            if constexpr (!EULER) put(o + N, v);
        }
    }
}

// Slot rows stored in whole lines.  A workgroup of BS lanes takes a tile of
// lines_span(BS) = 2 BS - 16 intervals from k0 (a multiple of the span) of a
// slot row of N values, which begins at position al in its line, and stores the
// row's intervals [k0 - sh, k0 - sh + span), sh the position of interval k0: the
// 128-byte lines that begin there, so every wavefront's 16-byte stores fill
// whole lines whatever the row's address.
// val(x) is the value of interval k0 - 15 + x, 0 <= x < 2 BS - 1.  The tiles
// of a row are ceil((N + 15) / span).
constexpr int kHalo = kLine - 1;
constexpr int lines_span(int bs) { return 2 * bs - kLine; }
template <int BS, class F>
__device__ __forceinline__ void store_row_lines(double *__restrict__ row, int al, int64_t N, int64_t k0, F val)
{
    const int sh = line_pos_at(al, k0);
    const int x = 2 * (int)threadIdx.x;
    if (x >= lines_span(BS)) return;
    const int64_t k = k0 - sh + x;
    const double v0 = val(kHalo - sh + x), v1 = val(kHalo - sh + x + 1);
    if (k >= 0 && k + 1 < N) {
        st_nt2(row + k, dbl2{v0, v1});
    } else {
        if (k >= 0 && k < N) st_nt(row + k, v0);
        if (k + 1 >= 0 && k + 1 < N) st_nt(row + k + 1, v1);
    }
}

// One column of a tile of lines_span(BS) intervals from k0, stored in whole
// lines from 6 BS doubles of LDS (the cosines and the two bilinear factors at
// the tile's 2 BS nodes; each node is evaluated once).
template <int BS>
__device__ __forceinline__ void jac_column_lines(const KP &P, const double *__restrict__ z, double *__restrict__ jac,
                                                 int al, int64_t k0, int col, double *lds)
{
    const int n = P.n, m = P.m, T = P.T;
    const int64_t N = P.N, N1 = P.N1;
    const bool euler = P.scheme != 0;
    const double w = euler ? P.h : P.hh;
    auto put = [&](int64_t r, auto val) { store_row_lines<BS>(jac + r, line_pos_at(al, r), N, k0, val); };
    if (col < n) {
        const int j = col;
        const int jn = (j + 1 == n) ? 0 : j + 1;
        const int jp = (j == 0) ? n - 1 : j - 1;
        const double gj = -w * P.gam[j], gp = -w * P.gam[jp];
        double *cs = lds, *xn = lds + 2 * BS, *xp = lds + 4 * BS;
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int x = (int)threadIdx.x + u * BS;
            const int64_t k = min(max(k0 - kHalo + x, (int64_t)0), N);  // clamped: values past the ends are not stored
            cs[x] = cos(z[j * N1 + k]);
            xn[x] = z[jn * N1 + k];
            xp[x] = z[jp * N1 + k];
        }
        __syncthreads();
        for (int i = 0; i < n; i++) {
            const double a = -w * P.A[i * n + j];
            auto at = [&](int x, double id) {
                return jac_entry(i == j, i == jp, a, cs[x], id, gj, gp, i == j ? xn[x] : 0.0, i == jp ? xp[x] : 0.0);
            };
            const int64_t r = ((int64_t)i * T + (!euler ? 2 * j : j <= i ? j : j + 1)) * N;
            put(r, [&](int x) { return at(x, -1.0); });
            if (!euler) put(r + N, [&](int x) { return at(x + 1, 1.0); });
        }
        if (euler) put(((int64_t)j * T + j + 1) * N, [](int) { return 1.0; });
    } else {
        const int l = col - n;
        for (int i = 0; i < n; i++) {
            const double v = -w * P.B[i * m + l];
            const int64_t r = ((int64_t)i * T + (euler ? n + 1 + l : 2 * (n + l))) * N;
            put(r, [&](int) { return v; });
            if (!euler) put(r + N, [&](int) { return v; });
        }
    }
}

// ---------------------------------------------------------------------------
// Hessian-of-Lagrangian values at node k <= N.  NB >= n is a compile-time
// bound so the node's states and multipliers stay in registers; all loads are
// issued before the arithmetic, and the control slots (constants) and the
// bilinear slots (multipliers only) are stored before the state diagonals,
// so their stores leave while the sines are computed.
// NT selects non-temporal stores.  The single-instance trapezoidal kernel
// stores ordinarily: a node's values go to S slot rows, one 8-byte store per
// lane and row, and with non-temporal stores that pattern reaches 60 % of HBM
// with no arithmetic at all against 73 % with ordinary ones.  The lines are
// then written back during the next kernel (in an interior-point step the
// assembly, which reads these values).  The batched kernel and the forward
// Euler kernel keep non-temporal stores (with ordinary ones their steps
// measured the same or slower).
// ---------------------------------------------------------------------------
template <int NB, bool NT>
__device__ __forceinline__ void hess_node(const KP &P, const double *__restrict__ z,
                                          const double *__restrict__ y, double sigma,
                                          double *__restrict__ hv, int k)
{
    const int n = P.n, m = P.m;
    const int64_t N = P.N, N1 = P.N1;
    const double w = node_weight(P, k);
    double x[NB], yl[NB], yr[NB];
#pragma unroll
    for (int i = 0; i < NB; i++) {
        x[i] = yl[i] = yr[i] = 0.0;
        if (i < n) {
            x[i] = z[i * N1 + k];
            const double *yi = y + i * N + k;
            if (k >= 1) yl[i] = yi[-1];
            if (k < P.N) yr[i] = yi[0];
        }
    }
    const int64_t ub = (int64_t)(n + P.npair) * N1 + k;
    for (int l = 0; l < m; l++) st_out<NT>(hv + ub + l * N1, 2.0 * sigma * w * P.r[l]);
    double yt[NB];
#pragma unroll
    for (int i = 0; i < NB; i++) yt[i] = yl[i] + yr[i];
    if (n >= 3) {
#pragma unroll
        for (int i = 0; i < NB; i++)
            if (i < n) st_out<NT>(hv + (n + i) * N1 + k, -P.hh * yt[i] * P.gam[i]);
    } else if (n == 2) {
        st_out<NT>(hv + 2 * N1 + k, -P.hh * (yt[0] * P.gam[0] + yt[1] * P.gam[1]));
    }
#pragma unroll
    for (int j = 0; j < NB; j++) {
        if (j < n) {
            const double sx = sin(x[j]);
            const double *a = P.AT + j * kLd;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < NB; i++) s = __builtin_fma(yt[i], a[i], s);
            double v = 2.0 * sigma * w * P.q[j] + P.hh * sx * s;
            if (n == 1) v -= P.h * yt[0] * P.gam[0];
            st_out<NT>(hv + j * N1 + k, v);
        }
    }
}

// ---------------------------------------------------------------------------
// Dynamics at node k <= N: the node's states x[i] = X_ik and F_i(k) for every
// i < n (NB >= n, entries beyond n are zero).  F_i sums j ascending, then l
// ascending, then the bilinear term.  dyn_load loads the states of node k and
// the first MB controls of node ku, before any arithmetic, and clears F;
// dyn_eval adds the dynamics into F
// (further controls, when m > MB, loaded there); a caller that knows
// m <= MB < NB saves the registers of NB - MB controls.
// ---------------------------------------------------------------------------
template <int NB, int MB>
__device__ __forceinline__ void dyn_load(const KP &P, const double *__restrict__ z, int64_t k, int64_t ku,
                                         double (&x)[NB], double (&u)[MB], double (&F)[NB])
{
    static_assert(MB <= NB, "the control bound is at most the state bound");
    const double *U = z + (int64_t)P.n * P.N1;
#pragma unroll
    for (int i = 0; i < NB; i++) {
        x[i] = (i < P.n) ? z[i * (int64_t)P.N1 + k] : 0.0;
        if (i < MB) u[i] = (i < P.m) ? U[(int64_t)i * P.NU + ku] : 0.0;
        F[i] = 0.0;
    }
}

template <int NB, int MB>
__device__ __forceinline__ void dyn_eval(const KP &P, const double *__restrict__ z, int64_t ku,
                                         const double (&x)[NB], const double (&u)[MB], double (&F)[NB])
{
    const int n = P.n, m = P.m;
    const double *U = z + (int64_t)n * P.N1;
#pragma unroll
    for (int j = 0; j < NB; j++) {
        if (j < n) {
            const double s = sin(x[j]);
            const double *a = P.AT + j * kLd;
#pragma unroll
            for (int i = 0; i < NB; i++) F[i] = __builtin_fma(a[i], s, F[i]);
        }
    }
#pragma unroll
    for (int l = 0; l < MB; l++) {
        if (l < m) {
            const double *b = P.BT + l * kLd;
#pragma unroll
            for (int i = 0; i < NB; i++) F[i] = __builtin_fma(b[i], u[l], F[i]);
        }
    }
    for (int l = MB; l < m; l++) {
        const double ul = U[(int64_t)l * P.NU + ku];
        const double *b = P.BT + l * kLd;
#pragma unroll
        for (int i = 0; i < NB; i++) F[i] = __builtin_fma(b[i], ul, F[i]);
    }
#pragma unroll
    for (int i = 0; i < NB; i++) {
        if (i < n) {
            const double xp = (i + 1 < n) ? x[(i + 1) % NB] : x[0];
            F[i] = __builtin_fma(P.gam[i] * x[i], xp, F[i]);  // explicit: same bits in every kernel
        }
    }
}

template <int NB, int MB = NB>
__device__ __forceinline__ void dyn_node(const KP &P, const double *__restrict__ z, int64_t k,
                                         double (&x)[NB], double (&F)[NB])
{
    double u[MB];
    dyn_load<NB, MB>(P, z, k, k, x, u, F);
    dyn_eval<NB, MB>(P, z, k, x, u, F);
}

// Entry n-1 of a register array (n is a run-time value <= NB), by selects so
// the array stays in registers.
template <int NB>
__device__ __forceinline__ double last_of(const double (&a)[NB], int n)
{
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < NB; i++)
        if (i == n - 1) v = a[i];
    return v;
}

// ---------------------------------------------------------------------------
// Forward Euler Hessian-of-Lagrangian values at node k <= N: node k enters
// only the defect of interval k (multiplier y_k, factor h); node N enters no
// defect and carries no cost, so its entries are zero.  Control slots exist
// for k < N only, at (n+npair)(N+1) + l N + k.  NT as for hess_node.
// ---------------------------------------------------------------------------
template <int NB, bool NT>
__device__ __forceinline__ void hess_node_euler(const KP &P, const double *__restrict__ z,
                                                const double *__restrict__ y, double sigma,
                                                double *__restrict__ hv, int k)
{
    const int n = P.n, m = P.m;
    const int64_t N = P.N, N1 = P.N1;
    const double w = node_weight(P, k);
    const double h = P.h;
    double x[NB], yt[NB];
#pragma unroll
    for (int i = 0; i < NB; i++) {
        x[i] = yt[i] = 0.0;
        if (i < n) {
            x[i] = z[i * N1 + k];
            if (k < P.N) yt[i] = y[i * N + k];
        }
    }
    // the control and bilinear slots (no sines) are stored first, as in
    // hess_node, then the diagonals
    if (k < P.NU) {
        const int64_t ub = (int64_t)(n + P.npair) * N1 + k;
        for (int l = 0; l < m; l++) st_out<NT>(hv + ub + (int64_t)l * P.NU, 2.0 * sigma * w * P.r[l]);
    }
    if (n >= 3) {
#pragma unroll
        for (int i = 0; i < NB; i++)
            if (i < n) st_out<NT>(hv + (n + i) * N1 + k, -h * yt[i] * P.gam[i]);
    } else if (n == 2) {
        st_out<NT>(hv + 2 * N1 + k, -h * (yt[0] * P.gam[0] + yt[1] * P.gam[1]));
    }
#pragma unroll
    for (int j = 0; j < NB; j++) {
        if (j < n) {
            const double sx = sin(x[j]);
            const double *a = P.AT + j * kLd;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < NB; i++) s = __builtin_fma(yt[i], a[i], s);
            double v = 2.0 * sigma * w * P.q[j] + h * sx * s;
            if (n == 1) v -= 2.0 * h * yt[0] * P.gam[0];
            st_out<NT>(hv + j * N1 + k, v);
        }
    }
}

// Host-side launchers of the single-instance kernels (ocp_eval.hip,
// ocp_fused.hip); the batched path uses them for its per-instance mode.  Each
// covers the problem's boundary rows too.  launch_obj's `partials` holds
// min(4096, ceil((N+1) / 256)) doubles.
hipError_t launch_jac(const KP &P, const double *z, double *jac, hipStream_t stream);
hipError_t launch_hess(const KP &P, const double *z, const double *y, double sigma, double *hv,
                       hipStream_t stream);
hipError_t launch_obj(const KP &P, const double *z, double *partials, double *obj, hipStream_t stream);
hipError_t launch_grad(const KP &P, const double *z, double *g, hipStream_t stream);
// `scale`: null, or a device double that every value is multiplied by
hipError_t launch_cons(const KP &P, const double *z, double *c, const double *scale, hipStream_t stream);
hipError_t launch_eval_kkt(const KP &P, const double *z, const double *y, double sigma, const double *reg,
                           double *kkt, hipStream_t stream);

}  // namespace dev
}  // namespace ocp
