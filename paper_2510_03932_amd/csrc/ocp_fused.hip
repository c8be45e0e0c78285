// Fused evaluation into the KKT matrix (ocp_eval_kkt): the Jacobian and the
// Hessian of the Lagrangian are evaluated straight into their slots of the
// lower CSR KKT matrix of ocp_build_kkt, with the regularization on the
// diagonal, skipping the COO value arrays.  An interior-point iteration that
// only needs the assembled matrix (paper Sec. 6) then moves the matrix once:
// the state rows, y and reg in, the KKT values out (about 7 GB at N = 1e6,
// n = 16, m = 8, against 23 GB for eval_jac + eval_hess + assemble_kkt).
//
// The values are the COO kernels' and the assembly's, except that the defect
// rows round each product of a state's partial derivative before it is added
// (defect_column), where the COO kernels fuse one into the sum: an entry at a
// row's own state or its bilinear partner may differ in the last bit.  The tile
// bodies (ocp_step_device.h) are shared with the batched evaluation.
//
// Defect rows: a workgroup owns KT = 16, 32 or 64 consecutive intervals
// (rules::kkt_defect_kt); each XCD takes a contiguous run of the tiles, so that the
// lines neighbouring tiles share (states read, rows stored) meet in one L2.
// It stages the states and their cosines at the KT+1 nodes, the rows'
// regularization and the scaled coefficients -hh A, -hh B, -hh gamma in LDS
// (a wavefront spans several slots of a row, so coefficient reads from global
// memory would be per-lane loads, each waited for); then, for each state
// component i, it computes the tile's KT rows (T Jacobian entries and the
// diagonal each) column by column into an LDS tile and writes the rows'
// contiguous CSR range with full-line stores.
// Variable rows: one lane per node computes the node's Hessian values (+ reg
// on the diagonals), as in eval_hess; each state block's rows of the
// workgroup's nodes are staged in LDS and written contiguously.
#include <hip/hip_runtime.h>

#include <cmath>
#include <string>

#include "ocp_device.h"
#include "ocp_problem.h"
#include "ocp_quad.h"
#include "ocp_rules.h"
#include "ocp_step_device.h"

using namespace ocp;
using namespace ocp::dev;

namespace {

__global__ __launch_bounds__(kBlock) void kkt_defect_kernel(KP P, KKTLayout Lo, int LG, int al,
                                                            const double *__restrict__ z,
                                                            const double *__restrict__ reg,
                                                            double *__restrict__ kkt)
{
    extern __shared__ double lds[];
    kkt_defect_tile<kBlock>(P, Lo, z, reg, kkt, al, (int64_t)xcd_order(blockIdx.x, gridDim.x) << LG, LG, lds);
}

template <int NB>
__global__ __launch_bounds__(kBlock) void kkt_var_kernel(KP P, KKTLayout Lo, int al, const double *__restrict__ z,
                                                         const double *__restrict__ y, double sigma,
                                                         const double *__restrict__ reg,
                                                         double *__restrict__ kkt)
{
    __shared__ double buf[3 * kBlock];  // one state block's rows of this workgroup (<= 3 entries each)
    kkt_var_tile<NB, kBlock>(P, Lo, z, y, sigma, reg, kkt, al, (int64_t)xcd_order(blockIdx.x, gridDim.x) * kBlock,
                             buf);
    // the boundary rows ride in the first workgroup, after its own
    if (blockIdx.x == 0 && (int)threadIdx.x < P.nb) kkt_bnd_row(P, Lo, reg, kkt, threadIdx.x);
}

template <int NB>
void launch_kkt_var(const KP &P, const KKTLayout &Lo, int al, const double *z, const double *y, double sigma,
                    const double *reg, double *kkt, hipStream_t stream)
{
    hipLaunchKernelGGL(kkt_var_kernel<NB>, dim3(blocks_for(P.N1, kBlock)), dim3(kBlock), 0, stream, P, Lo, al, z, y,
                       sigma, reg, kkt);
}

}  // namespace

namespace ocp {
namespace dev {

hipError_t launch_eval_kkt(const KP &P, const double *z, const double *y, double sigma, const double *reg,
                           double *kkt, hipStream_t stream)
{
    const KKTLayout Lo = kkt_layout(P.n);
    // defect-row tiles of KT = 2^LG intervals; LDS holds the tile's states,
    // their cosines, the rows' regularization, the scaled coefficients and the
    // output row block
    const int64_t N = P.N;
    const int KT = rules::kkt_defect_kt(P.n, P.m, P.T, P.scheme != 0, &N, 1);
    const int LG = __builtin_ctz((unsigned)KT), al = line_pos(kkt);
    const size_t lds = rules::kkt_defect_lds(P.n, P.m, P.T, KT) * sizeof(double);
    hipLaunchKernelGGL(kkt_defect_kernel, dim3(blocks_for(P.N, KT)), dim3(kBlock), lds, stream, P, Lo, LG, al, z,
                       reg, kkt);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (P.n <= 4) launch_kkt_var<4>(P, Lo, al, z, y, sigma, reg, kkt, stream);
    else if (P.n <= 8) launch_kkt_var<8>(P, Lo, al, z, y, sigma, reg, kkt, stream);
    else if (P.n <= 16) launch_kkt_var<16>(P, Lo, al, z, y, sigma, reg, kkt, stream);
    else launch_kkt_var<32>(P, Lo, al, z, y, sigma, reg, kkt, stream);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace ocp

extern "C" {

int ocp_eval_kkt(const ocp_problem *p, const double *z, const double *y, double sigma, const double *reg,
                 double *kkt, hipStream_t stream)
{
    clear_error();
    if (int rc = check_handle(p, "ocp_eval_kkt")) return rc;
    if (!z || !y || !kkt) return fail(OCP_ERR_ARG, "ocp_eval_kkt: null array");
    if (!std::isfinite(sigma)) return fail(OCP_ERR_ARG, "ocp_eval_kkt: sigma is not finite");
    if (p->model == quad::kModel) return quad::eval_kkt(p, z, y, sigma, reg, kkt, stream);
    const hipError_t e = launch_eval_kkt(p->kp, z, y, sigma, reg, kkt, stream);
    if (e != hipSuccess) return hip_fail("ocp_eval_kkt", e);
    return OCP_OK;
}

}  // extern "C"
