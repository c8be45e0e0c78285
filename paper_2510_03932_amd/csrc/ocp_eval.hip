// Device layer of the evaluation library, single-instance entry points: HIP
// kernels for gfx950 (CDNA4, wave64) and the C ABI functions that validate
// arguments and launch them.  The per-node arithmetic shared with the batched
// path lives in ocp_device.h.  The path is HBM-bound sparse evaluation, not a
// dense contraction: no MFMA.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>

#include "ocp_device.h"
#include "ocp_internal.h"
#include "ocp_problem.h"
#include "ocp_rules.h"
#include "ocp_quad.h"
#include "ocp_step_device.h"

using namespace ocp;
using namespace ocp::dev;

namespace {

// ---------------------------------------------------------------------------
// Jacobian values.  2-D grid: blockIdx.y is the column (state j < n, control
// n + l), blockIdx.x the tile: kBlock lanes of one or two intervals each,
// stored directly (jac_kernel), or lines_span(kBlock) intervals stored in whole
// lines (jac_lines_kernel).  Many short workgroups keep the write stream at the
// device's rate for slot rows, 5.5-5.8 TB/s.
// ---------------------------------------------------------------------------
// Boundary row b's single Jacobian entry (1.0), after the defect entries.  The
// boundary rows (at most 2 OCP_MAX_DIM = 64) ride in the first workgroup of
// the kernel that writes the defect rows: a launch of their own took 4-5 us.
// They come last in it: after a store the compiler no longer reads the
// coefficients through the scalar cache (stored first, the fused KKT's
// variable rows took 65 us instead of 53 at N = 333,333, n = 12, m = 5).
__device__ __forceinline__ void bnd_jac(const KP &P, double *__restrict__ jac, int64_t b)
{
    if (b < P.nb) jac[(int64_t)P.n * P.N * P.T + b] = 1.0;
}

template <int NPT, bool EULER>
__global__ __launch_bounds__(kBlock) void jac_kernel(KP P, const double *__restrict__ z, double *__restrict__ jac)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t * NPT < P.N) jac_column<NPT, EULER>(P, z, jac, t * NPT, blockIdx.y);
    bnd_jac(P, jac, blockIdx.y == 0 ? t : P.nb);
}

__global__ __launch_bounds__(kBlock) void jac_lines_kernel(KP P, int al, const double *__restrict__ z,
                                                           double *__restrict__ jac)
{
    __shared__ double lds[6 * kBlock];
    jac_column_lines<kBlock>(P, z, jac, al, (int64_t)blockIdx.x * lines_span(kBlock), blockIdx.y, lds);
    bnd_jac(P, jac, blockIdx.x == 0 && blockIdx.y == 0 ? threadIdx.x : P.nb);
}

// ---------------------------------------------------------------------------
// Hessian-of-Lagrangian values, one lane per node.
// ---------------------------------------------------------------------------
template <int NB>
__global__ __launch_bounds__(kBlock) void hess_kernel(KP P, const double *__restrict__ z,
                                                      const double *__restrict__ y, double sigma,
                                                      double *__restrict__ hv)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k > P.N) return;
    hess_node<NB, false>(P, z, y, sigma, hv, k);
}

// ---------------------------------------------------------------------------
// Defects.  Workgroup b evaluates the dynamics at kBlock nodes from b kSpan,
// one node per lane, and writes kSpan of the intervals they close.  With
//   c_ik = (X_{i,k+1} - hh F_i(k+1)) - (X_ik + hh F_i(k)),
// lane k keeps X_ik + hh F_i(k) in registers and publishes X_ik - hh F_i(k)
// in LDS for lane k-1, so every state value is read from HBM once.  kSpan is
// 240, not the 255 intervals the nodes close: a multiple of a line, so that
// where N is one too every wavefront stores whole lines.  `scale`: null, or a
// device double that multiplies every value (a backward pass).
// ---------------------------------------------------------------------------
// The boundary rows' values, by one workgroup.
__device__ __forceinline__ void bnd_cons(const KP &P, const double *__restrict__ z, double *__restrict__ c,
                                         const double *__restrict__ scale)
{
    const int b = threadIdx.x;
    if (b < P.nb) c[(int64_t)P.n * P.N + b] = bnd_value(P, z, b) * (scale ? *scale : 1.0);
}

template <int NB, int MB>
__global__ __launch_bounds__(kBlock) void cons_kernel(KP P, const double *__restrict__ z,
                                                      double *__restrict__ c, const double *__restrict__ scale)
{
    __shared__ double Ms[NB][kBlock];
    const int tid = threadIdx.x;
    const int64_t k = (int64_t)blockIdx.x * kSpan + tid;
    const int n = P.n;
    const int64_t N = P.N;
    double Pk[NB];
    if (k <= N) {
        double x[NB], F[NB];
        dyn_node<NB, MB>(P, z, k, x, F);
#pragma unroll
        for (int i = 0; i < NB; i++) {
            if (i < n) {
                Ms[i][tid] = __builtin_fma(-P.hh, F[i], x[i]);
                Pk[i] = __builtin_fma(P.hh, F[i], x[i]);
            }
        }
    }
    __syncthreads();
    if (tid < kSpan && k < N) {
        const double f = scale ? *scale : 1.0;
#pragma unroll
        for (int i = 0; i < NB; i++)
            if (i < n) st_nt(c + i * N + k, (Ms[i][tid + 1] - Pk[i]) * f);
    }
    if (blockIdx.x == 0) bnd_cons(P, z, c, scale);
}

// ---------------------------------------------------------------------------
// Forward-Euler defects: one lane per interval k < N,
//   c_ik = (X_{i,k+1} - X_ik) - h F_i(k)  (paper Sec. 3).
// The boundary rows have a workgroup of their own, the last: beside the defects
// they and *scale, loaded ahead, cost the sums scalar registers (N = 4e5,
// n = 32, m = 16 140 -> 135 us, n = 24, m = 10 103.8 -> 101.6; the trapezoidal
// kernel shows no such loss, and at N = 1000, n = 24, m = 10 takes 22.6 us with
// them beside the defects and 23.2 so).
// ---------------------------------------------------------------------------
template <int NB, int MB>
__global__ __launch_bounds__(kBlock) void cons_euler_kernel(KP P, const double *__restrict__ z,
                                                            double *__restrict__ c,
                                                            const double *__restrict__ scale)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if ((int64_t)blockIdx.x * kBlock >= P.N) {  // the workgroup of the boundary rows
        bnd_cons(P, z, c, scale);
        return;
    }
    if (k < P.N) cons_euler_interval<NB, MB>(P, z, c, k, scale);
}

template <int NB>
__global__ __launch_bounds__(kBlock) void hess_euler_kernel(KP P, const double *__restrict__ z,
                                                            const double *__restrict__ y,
                                                            double sigma, double *__restrict__ hv)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k > P.N) return;
    hess_node_euler<NB, true>(P, z, y, sigma, hv, k);
}

// ---------------------------------------------------------------------------
// Gradient: g = 2 w_k q_j X_jk, 2 w_k r_l U_lk.  blockIdx.y = component.
// Rows of N + 1 values start off the line nearly always, so each workgroup
// takes the nodes of whole lines of its row: 70 -> 64 us at N = 1e6, n = 16,
// m = 8 (6.0 TB/s), 18.0 -> 16.2 us at N = 333,333, n = 12, m = 5.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void grad_kernel(KP P, int al, const double *__restrict__ z,
                                                      double *__restrict__ g)
{
    grad_row(P, z, g, al, blockIdx.y, (int64_t)blockIdx.x * kBlock);
}

// ---------------------------------------------------------------------------
// Objective: deterministic two-pass sum.  Pass 1: min(ceil((N+1)/256), 4096)
// workgroups (so one node per lane up to 1M nodes), each lane summing its
// nodes in order, then a fixed-shape tree over the wavefront (cross-lane
// shuffles) and over the 4 waves; pass 2: one workgroup sums the partials in a
// fixed order.  The grid depends only on N, so the result is reproducible.
// ---------------------------------------------------------------------------
template <int NB>
__global__ __launch_bounds__(kBlock) void obj_partial_kernel(KP P, const double *__restrict__ z,
                                                             double *__restrict__ partials)
{
    const int64_t N1 = P.N1;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < N1; k += (int64_t)gridDim.x * kBlock)
        acc += obj_node<NB>(P, z, k);
    const double t = block_sum<kBlock>(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void obj_final_kernel(const double *__restrict__ partials,
                                                           int count, double *__restrict__ obj)
{
    const double t = sum_partials(partials, count);
    if (threadIdx.x == 0) obj[0] = t;
}

// ---------------------------------------------------------------------------
// KKT assembly.
//
// Jacobian part: the COO values are slot-major (node fastest) while the CSR
// rows of the constraint block are row-major, so the scatter is a transpose.
// Workgroup g < gj owns a tile of up to KT = 2^LG consecutive constraint rows
// of one state component i (intervals k0 .. k0+kn-1).  It reads the tile's T
// slot rows coalesced, drops each value into LDS at perm_j[e] - base, where
// [base, base + ext) is the tile's CSR range from rowptr, adds the tile's
// diagonals, and then writes the whole range in full lines.  A slot outside
// the range is stored directly.  If the values that landed in LDS do not cover
// the range exactly (a slot map other than the closed-form one), the tile is
// redone with direct stores, so the result is the same for any injective slot
// map.
//
// Reading bounds it: each slot row gives a tile KT 4-byte slots and KT values,
// which at an odd N start anywhere in a line.  So each lane takes two adjacent
// intervals of a slot row with one 16-byte and one 8-byte load at any
// alignment, kAsmBatch slot rows' loads are in flight per lane, and a tile is as
// tall as its LDS allows.  Against tiles of 64 rows, one slot row at a time and
// 8-byte loads at odd entries: 452 -> 339 us at N = 200,001, n = 16, m = 8
// (forward Euler), 718 -> 592 us at N = 333,333, n = 12, m = 5 (5.1 TB/s),
// 87 -> 81 us at N = 1e5, n = 8, m = 4, 2.95 -> 2.89 ms at N = 1e6, n = 16,
// m = 8 (5.8 TB/s).  Tiles of 256 rows leave too few workgroups per CU (4.0 ms
// at n = 16, m = 8); 512 lanes gain 1 % there and lose 12 % at N = 1e5.
//
// Hessian part: workgroups gj.. take nodes and scatter the S Hessian slots
// directly (rows of 1 to 3 entries, close to contiguous across lanes), adding
// reg on the variable diagonals in the same IEEE add; the loads of kHessBatch
// slots are issued before their stores.
// ---------------------------------------------------------------------------
constexpr int kHessBatch = 8;  // slots in flight per lane (Hessian part)

__global__ __launch_bounds__(kBlock) void assemble_kernel(
    KP P, int gj, int gh, int LG, int al, const int32_t *__restrict__ perm_j, const int32_t *__restrict__ perm_h,
    const int32_t *__restrict__ rowptr, const double *__restrict__ jv,
    const double *__restrict__ hv, const double *__restrict__ reg, double *__restrict__ kkt)
{
    extern __shared__ __align__(16) double tile[];
    __shared__ int filled;
    const int64_t N = P.N, N1 = P.N1;
    const int64_t nvar = (int64_t)P.n * N1 + (int64_t)P.m * P.NU;
    const uint32_t nnzk = (uint32_t)P.nnzk;  // slots outside [0, nnzk) are skipped
    const int T = P.T;
    if ((int)blockIdx.x < gj) {
        const int KT = 1 << LG;
        const int tiles_per_i = (P.N + KT - 1) >> LG;
        const int i = blockIdx.x / tiles_per_i;
        const int k0 = (blockIdx.x - i * tiles_per_i) << LG;
        const int kn = min(KT, P.N - k0);
        const int64_t r0 = nvar + (int64_t)i * N + k0;  // first KKT row of the tile
        const int32_t base = rowptr[r0];
        const int32_t ext = (int32_t)((uint32_t)rowptr[r0 + kn] - (uint32_t)base);
        const int cap = KT * (T + 1);
        // stage only a range inside [0, nnzk) (a corrupt rowptr falls back
        // to bounds-checked direct stores)
        const bool staged = ext >= 0 && ext <= cap && base >= 0 && (int64_t)base + ext <= (int64_t)nnzk;
        if (threadIdx.x == 0) filled = 0;
        // Zeros first (up to 2 % of the call): a map that names a slot twice
        // and another of the range never has the right count all the same, and
        // must not store what the LDS held.  An odd ext leaves room for its
        // pair: cap is even.
        if (staged)
            for (int x = 2 * threadIdx.x; x < ext; x += 2 * kBlock) *reinterpret_cast<dbl2 *>(tile + x) = dbl2{0.0, 0.0};
        __syncthreads();
        const int64_t e0 = (int64_t)i * T * N + k0;
        // Visit every (slot, value) of the tile; `put` decides where it goes.
        auto visit = [&](auto put) {
            const int total = T << (LG - 1);  // interval pairs of the tile's slot rows
            for (int w0 = threadIdx.x; w0 < total; w0 += kBlock * kAsmBatch) {
                int2_any q[kAsmBatch];
                dbl2_any v[kAsmBatch];
                int live[kAsmBatch];
#pragma unroll
                for (int u = 0; u < kAsmBatch; u++) {
                    const int w = w0 + u * kBlock;
                    const int kl = 2 * (w & (KT / 2 - 1));
                    const int64_t e = e0 + (int64_t)(w >> (LG - 1)) * N + kl;
                    live[u] = w < total ? min(kn - kl, 2) : 0;
                    if (live[u] == 2) {
                        q[u] = __builtin_nontemporal_load(reinterpret_cast<const int2_any *>(perm_j + e));
                        v[u] = __builtin_nontemporal_load(reinterpret_cast<const dbl2_any *>(jv + e));
                    } else if (live[u] == 1) {
                        q[u].x = perm_j[e];
                        v[u].x = jv[e];
                    }
                }
#pragma unroll
                for (int u = 0; u < kAsmBatch; u++) {
                    if (live[u] >= 1) put(q[u].x, v[u].x);
                    if (live[u] == 2) put(q[u].y, v[u].y);
                }
            }
            for (int x = threadIdx.x; x < kn; x += kBlock) {
                const int64_t d = r0 + x;
                put(rowptr[d + 1] - 1, reg ? reg[d] : 0.0);
            }
        };
        int mine = 0;
        visit([&](int32_t q, double v) {
            const uint32_t loc = (uint32_t)q - (uint32_t)base;
            if (staged && loc < (uint32_t)ext) {
                tile[loc] = v;
                mine++;
            } else if ((uint32_t)q < nnzk) {
                kkt[q] = v;
            }
        });
        if (mine) atomicAdd(&filled, mine);
        __syncthreads();
        if (!staged) return;
        if (filled == ext) {
            copy_lines<kBlock>(kkt + base, line_pos_at(al, base), tile, ext);
        } else {
            // not an exact cover: store this tile's values directly
            visit([&](int32_t q, double v) {
                if ((uint32_t)q < nnzk) kkt[q] = v;
            });
        }
    } else if ((int)blockIdx.x < gj + gh) {
        const int64_t k = (int64_t)(blockIdx.x - gj) * kBlock + threadIdx.x;
        if (k >= N1) return;
        const int n = P.n, np = P.npair, S = P.S;
        for (int s0 = 0; s0 < S; s0 += kHessBatch) {
            double v[kHessBatch], rg[kHessBatch];
            int32_t q[kHessBatch];
#pragma unroll
            for (int u = 0; u < kHessBatch; u++) {
                const int s = s0 + u;
                q[u] = -1;
                rg[u] = 0.0;
                if (s >= S) continue;
                int64_t e, row = -1;  // COO entry; KKT row of a diagonal entry
                if (s < n + np) {
                    e = (int64_t)s * N1 + k;
                    if (s < n) row = e;
                } else {
                    if (k >= P.NU) continue;  // control slots exist on NU nodes
                    const int64_t l = s - n - np;
                    e = (int64_t)(n + np) * N1 + l * P.NU + k;
                    row = (int64_t)n * N1 + l * P.NU + k;
                }
                q[u] = perm_h[e];
                v[u] = hv[e];
                if (reg && row >= 0) rg[u] = reg[row];
            }
#pragma unroll
            for (int u = 0; u < kHessBatch; u++) {
                const int s = s0 + u;
                const bool diag = s < n || s >= n + np;
                if ((uint32_t)q[u] < nnzk) kkt[q[u]] = reg && diag ? v[u] + rg[u] : v[u];
            }
        }
    } else {
        // boundary rows: their Jacobian entry and their diagonal
        const int b = (blockIdx.x - gj - gh) * kBlock + threadIdx.x;
        if (b >= P.nb) return;
        const int64_t e = (int64_t)P.n * N * T + b;
        const uint32_t q = (uint32_t)perm_j[e];
        if (q < nnzk) kkt[q] = jv[e];
        const int64_t d = nvar + (int64_t)P.n * N + b;
        const uint32_t dq = (uint32_t)(rowptr[d + 1] - 1);
        if (dq < nnzk) kkt[dq] = reg ? reg[d] : 0.0;
    }
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================

namespace ocp {
namespace dev {

// The three ways to store the slot rows; rules::jac_path says which and why.
static_assert(rules::kLineDoubles == kLine && rules::kJacLinesSpan == lines_span(kBlock), "jac_path's tiles");
hipError_t launch_jac(const KP &P, const double *z, double *jac, hipStream_t stream)
{
    const unsigned cols = (unsigned)(P.n + P.m);
    const bool euler = P.scheme != 0;
    const dim3 g1(blocks_for(P.N, kBlock), cols), g2(blocks_for(P.N / 2, kBlock), cols);
    switch (rules::jac_path(P.N, P.n, P.m, P.T, euler, (uintptr_t)jac)) {
    case rules::kJacLines:
        hipLaunchKernelGGL(jac_lines_kernel, dim3(blocks_for((int64_t)P.N + kHalo, lines_span(kBlock)), cols),
                           dim3(kBlock), 0, stream, P, line_pos(jac), z, jac);
        break;
    case rules::kJacPair:
        if (euler) hipLaunchKernelGGL((jac_kernel<2, true>), g2, dim3(kBlock), 0, stream, P, z, jac);
        else hipLaunchKernelGGL((jac_kernel<2, false>), g2, dim3(kBlock), 0, stream, P, z, jac);
        break;
    default:
        if (euler) hipLaunchKernelGGL((jac_kernel<1, true>), g1, dim3(kBlock), 0, stream, P, z, jac);
        else hipLaunchKernelGGL((jac_kernel<1, false>), g1, dim3(kBlock), 0, stream, P, z, jac);
    }
    return hipGetLastError();
}

template <int NB>
static void launch_hess_nb(const KP &P, const double *z, const double *y, double sigma, double *hv,
                           hipStream_t stream)
{
    const dim3 g((unsigned)((P.N1 + kBlock - 1) / kBlock));
    if (P.scheme == 0) hipLaunchKernelGGL(hess_kernel<NB>, g, dim3(kBlock), 0, stream, P, z, y, sigma, hv);
    else hipLaunchKernelGGL(hess_euler_kernel<NB>, g, dim3(kBlock), 0, stream, P, z, y, sigma, hv);
}

hipError_t launch_hess(const KP &P, const double *z, const double *y, double sigma, double *hv,
                       hipStream_t stream)
{
    if (P.n <= 4) launch_hess_nb<4>(P, z, y, sigma, hv, stream);
    else if (P.n <= 8) launch_hess_nb<8>(P, z, y, sigma, hv, stream);
    else if (P.n <= 16) launch_hess_nb<16>(P, z, y, sigma, hv, stream);
    else launch_hess_nb<32>(P, z, y, sigma, hv, stream);
    return hipGetLastError();
}

hipError_t launch_obj(const KP &P, const double *z, double *partials, double *obj, hipStream_t stream)
{
    const unsigned g = (unsigned)std::min<int64_t>(kObjBlocks, blocks_for(P.N1, kBlock));
    if (P.n <= 4) hipLaunchKernelGGL(obj_partial_kernel<4>, dim3(g), dim3(kBlock), 0, stream, P, z, partials);
    else if (P.n <= 8) hipLaunchKernelGGL(obj_partial_kernel<8>, dim3(g), dim3(kBlock), 0, stream, P, z, partials);
    else if (P.n <= 16) hipLaunchKernelGGL(obj_partial_kernel<16>, dim3(g), dim3(kBlock), 0, stream, P, z, partials);
    else hipLaunchKernelGGL(obj_partial_kernel<32>, dim3(g), dim3(kBlock), 0, stream, P, z, partials);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(obj_final_kernel, dim3(1), dim3(kBlock), 0, stream, partials, (int)g, obj);
    return hipGetLastError();
}

hipError_t launch_grad(const KP &P, const double *z, double *g, hipStream_t stream)
{
    dim3 grid(blocks_for((int64_t)P.N1 + kHalo, kBlock), P.n + P.m);
    hipLaunchKernelGGL(grad_kernel, grid, dim3(kBlock), 0, stream, P, line_pos(g), z, g);
    return hipGetLastError();
}

// The trapezoidal defect kernel for the state bound NB, with the controls'
// register array halved when m <= NB/2 (at n = 16, m = 8: 109 VGPRs instead
// of 125, 4 wavefronts per SIMD either way, 1-3 % faster at N = 1e6).  The
// sums run in the same order, so the values are the same bits.
template <int NB>
void launch_cons_trap(const KP &P, unsigned g, const double *z, double *c, const double *scale, hipStream_t stream)
{
    if (P.m <= NB / 2) hipLaunchKernelGGL((cons_kernel<NB, NB / 2>), dim3(g), dim3(kBlock), 0, stream, P, z, c, scale);
    else hipLaunchKernelGGL((cons_kernel<NB, NB>), dim3(g), dim3(kBlock), 0, stream, P, z, c, scale);
}

// The forward-Euler defect kernel, with the same control bound.
template <int NB>
void launch_cons_euler(const KP &P, unsigned g, const double *z, double *c, const double *scale, hipStream_t stream)
{
    if (P.m <= NB / 2) hipLaunchKernelGGL((cons_euler_kernel<NB, NB / 2>), dim3(g), dim3(kBlock), 0, stream, P, z, c, scale);
    else hipLaunchKernelGGL((cons_euler_kernel<NB, NB>), dim3(g), dim3(kBlock), 0, stream, P, z, c, scale);
}

hipError_t launch_cons(const KP &P, const double *z, double *c, const double *scale, hipStream_t stream)
{
    const int n = P.n;
    if (P.scheme == 0) {
        const unsigned g = blocks_for(P.N, kSpan);
        if (n <= 4) launch_cons_trap<4>(P, g, z, c, scale, stream);
        else if (n <= 8) launch_cons_trap<8>(P, g, z, c, scale, stream);
        else if (n <= 16) launch_cons_trap<16>(P, g, z, c, scale, stream);
        else launch_cons_trap<32>(P, g, z, c, scale, stream);
    } else {
        const unsigned g = blocks_for(P.N, kBlock) + (P.nb > 0);
        if (n <= 4) launch_cons_euler<4>(P, g, z, c, scale, stream);
        else if (n <= 8) launch_cons_euler<8>(P, g, z, c, scale, stream);
        else if (n <= 16) launch_cons_euler<16>(P, g, z, c, scale, stream);
        else launch_cons_euler<32>(P, g, z, c, scale, stream);
    }
    return hipGetLastError();
}

}  // namespace dev
}  // namespace ocp

extern "C" {

int ocp_create(int64_t N, int32_t n, int32_t m, const double *A, const double *B,
               const double *gamma, const double *q, const double *r, ocp_problem **out)
{
    return ocp_create_ex(N, n, m, nullptr, A, B, gamma, q, r, out);
}

int ocp_create_ex(int64_t N, int32_t n, int32_t m, const ocp_options *opt, const double *A,
                  const double *B, const double *gamma, const double *q, const double *r,
                  ocp_problem **out)
{
    clear_error();
    if (!out) return fail(OCP_ERR_ARG, "ocp_create: out is NULL");
    *out = nullptr;
    Dims d;
    int rc = make_dims_ex(N, n, m, opt ? opt->scheme : OCP_SCHEME_TRAPEZOIDAL,
                          opt ? opt->boundary : OCP_BOUNDARY_NONE, &d);
    if (rc) return rc;
    if (!A || !gamma || !q || (m > 0 && (!B || !r)))
        return fail(OCP_ERR_ARG, "ocp_create: coefficient pointer is NULL");
    for (int64_t x = 0; x < (int64_t)n * n; x++)
        if (!std::isfinite(A[x])) return fail(OCP_ERR_ARG, "ocp_create: A has a non-finite entry");

    ocp_problem *p = new (std::nothrow) ocp_problem();
    if (!p) return fail(OCP_ERR_ALLOC, "ocp_create: out of host memory");
    p->d = d;
    hipError_t e = hipGetDevice(&p->device);
    if (e != hipSuccess) { delete p; return hip_fail("ocp_create: hipGetDevice", e); }
    // locate this device's scratch array of the allocation-free entry point
    // now, outside any stream capture (a failure only disables that entry)
    (void)noalloc_scratch(p->device);
    static_assert(kLd == OCP_MAX_DIM, "padded coefficient columns hold up to OCP_MAX_DIM rows");
    const size_t nplain = (size_t)n * n + (size_t)n * m + 3 * (size_t)n + (size_t)m;
    const size_t ncoef = nplain + (size_t)(n + m) * kLd;
    e = hipMalloc(&p->coef, ncoef * sizeof(double));
    if (e != hipSuccess) { delete p; return fail(OCP_ERR_ALLOC, std::string("ocp_create: hipMalloc: ") + hipGetErrorString(e)); }
    e = hipMalloc(&p->partials, kObjBlocks * sizeof(double));
    if (e == hipSuccess)
        e = hipMalloc(&p->cpart, (size_t)n * (n + m + 1) * coef_blocks(d.N1) * sizeof(double));
    if (e != hipSuccess) {
        ocp_destroy(p);
        return fail(OCP_ERR_ALLOC, std::string("ocp_create: hipMalloc: ") + hipGetErrorString(e));
    }
    double *host = new (std::nothrow) double[ncoef];
    if (!host) { ocp_destroy(p); return fail(OCP_ERR_ALLOC, "ocp_create: out of host memory"); }
    size_t o = 0;
    std::memcpy(host + o, A, sizeof(double) * n * n); o += (size_t)n * n;
    if (m) std::memcpy(host + o, B, sizeof(double) * n * m); o += (size_t)n * m;
    std::memcpy(host + o, gamma, sizeof(double) * n); o += n;
    std::memcpy(host + o, q, sizeof(double) * n); o += n;
    if (m) std::memcpy(host + o, r, sizeof(double) * m);
    pack_columns(n, m, A, B, host + nplain, host + nplain + (size_t)n * kLd);
    e = hipMemcpy(p->coef, host, ncoef * sizeof(double), hipMemcpyHostToDevice);
    delete[] host;
    if (e != hipSuccess) { ocp_destroy(p); return hip_fail("ocp_create: hipMemcpy", e); }

    KP &kp = p->kp;
    kp.N = (int)d.N;
    kp.N1 = (int)d.N1;
    kp.n = n;
    kp.m = m;
    kp.npair = d.npair;
    kp.T = d.T;
    kp.S = d.S;
    kp.nnzk = (int)d.nnzk;
    kp.NU = (int)d.NU;
    kp.scheme = d.scheme;
    kp.nb = (int)d.nb;
    kp.h = 1.0 / (double)d.N;
    kp.hh = 0.5 * kp.h;
    kp.A = p->coef;
    kp.B = p->coef + (size_t)n * n;
    kp.gam = kp.B + (size_t)n * m;
    kp.q = kp.gam + n;
    kp.r = kp.q + n;
    kp.AT = p->coef + nplain;
    kp.BT = kp.AT + (size_t)n * kLd;
    *out = p;
    return OCP_OK;
}

void ocp_destroy(ocp_problem *p)
{
    if (!p) return;
    if (p->coef) (void)hipFree(p->coef);
    if (p->partials) (void)hipFree(p->partials);
    if (p->cpart) (void)hipFree(p->cpart);
    if (p->mplan) (void)hipFree(p->mplan);
    delete p;
}

int ocp_problem_sizes(const ocp_problem *p, ocp_sizes_t *out)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_problem_sizes")) return rc;
    if (!out) return fail(OCP_ERR_ARG, "ocp_problem_sizes: out is NULL");
    to_public(p->d, out);
    return OCP_OK;
}

int ocp_eval_obj(const ocp_problem *p, const double *z, double *obj, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_eval_obj")) return rc;
    if (!z || !obj) return fail(OCP_ERR_ARG, "ocp_eval_obj: null array");
    if (p->model == quad::kModel) return quad::eval_obj(p, z, obj, stream);
    const hipError_t e = launch_obj(p->kp, z, p->partials, obj, stream);
    if (e != hipSuccess) return hip_fail("ocp_eval_obj", e);
    return OCP_OK;
}

int ocp_eval_grad(const ocp_problem *p, const double *z, double *g, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_eval_grad")) return rc;
    if (!z || !g) return fail(OCP_ERR_ARG, "ocp_eval_grad: null array");
    if (p->model == quad::kModel) return quad::eval_grad(p, z, g, stream);
    const hipError_t e = launch_grad(p->kp, z, g, stream);
    if (e != hipSuccess) return hip_fail("ocp_eval_grad", e);
    return OCP_OK;
}

int ocp_eval_cons(const ocp_problem *p, const double *z, double *c, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_eval_cons")) return rc;
    if (!z || !c) return fail(OCP_ERR_ARG, "ocp_eval_cons: null array");
    if (p->model == quad::kModel) return quad::eval_cons(p, z, c, nullptr, stream);
    const hipError_t e = launch_cons(p->kp, z, c, nullptr, stream);
    if (e != hipSuccess) return hip_fail("ocp_eval_cons", e);
    return OCP_OK;
}

int ocp_eval_jac(const ocp_problem *p, const double *z, double *jvals, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_eval_jac")) return rc;
    if (!z || !jvals) return fail(OCP_ERR_ARG, "ocp_eval_jac: null array");
    if (p->model == quad::kModel) return quad::eval_jac(p, z, jvals, stream);
    const hipError_t e = launch_jac(p->kp, z, jvals, stream);
    if (e != hipSuccess) return hip_fail("ocp_eval_jac", e);
    return OCP_OK;
}

int ocp_eval_hess(const ocp_problem *p, const double *z, const double *y, double sigma,
                  double *hvals, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_eval_hess")) return rc;
    if (!z || !y || !hvals) return fail(OCP_ERR_ARG, "ocp_eval_hess: null array");
    if (!std::isfinite(sigma)) return fail(OCP_ERR_ARG, "ocp_eval_hess: sigma is not finite");
    if (p->model == quad::kModel) return quad::eval_hess(p, z, y, sigma, hvals, stream);
    const hipError_t e = launch_hess(p->kp, z, y, sigma, hvals, stream);
    if (e != hipSuccess) return hip_fail("ocp_eval_hess", e);
    return OCP_OK;
}

int ocp_assemble_kkt(const ocp_problem *p, const int32_t *perm_j, const int32_t *perm_h,
                     const int32_t *rowptr, const double *jvals, const double *hvals,
                     const double *reg, double *kkt, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_assemble_kkt")) return rc;
    if (!perm_j || !perm_h || !rowptr || !jvals || !hvals || !kkt)
        return fail(OCP_ERR_ARG, "ocp_assemble_kkt: null array");
    if (p->model == quad::kModel)
        return quad::assemble_kkt(p, perm_j, perm_h, rowptr, jvals, hvals, reg, kkt, stream);
    const int LG = rules::assembly_lg(p->d.N, p->d.n, p->d.T);
    const unsigned gj = (unsigned)(((p->d.N + (1 << LG) - 1) >> LG) * p->d.n);
    const unsigned gh = blocks_for(p->d.N1, kBlock);
    const unsigned gb = blocks_for(p->d.nb, kBlock);
    const size_t lds = ((size_t)(p->d.T + 1) << LG) * sizeof(double);
    hipLaunchKernelGGL(assemble_kernel, dim3(gj + gh + gb), dim3(kBlock), lds, stream, p->kp, (int)gj,
                       (int)gh, LG, line_pos(kkt), perm_j, perm_h, rowptr, jvals, hvals, reg, kkt);
    return check_launch("ocp_assemble_kkt");
}

}  // extern "C"
