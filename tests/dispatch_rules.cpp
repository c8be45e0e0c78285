// The dispatch rules of the library (csrc/ocp_rules.h) behind C symbols, for
// tests/test_dispatch_rules.py.
#include "ocp_rules.h"

#include <vector>

using namespace ocp::rules;

extern "C" {

int jac_path_of(int64_t N, int n, int m, int slots, int euler, uint64_t addr)
{
    return jac_path(N, n, m, slots, euler != 0, addr);
}

int quad_jac_path_of(int64_t N, uint64_t addr) { return quad_jac_path(N, addr); }

int batch_jac_of(int64_t count, const int64_t *Ns, int n, int slots, int euler, int pair, int block)
{
    return batch_jac(std::vector<int64_t>(Ns, Ns + count), n, slots, euler != 0, pair != 0, block);
}

int kkt_defect_kt_of(int64_t count, const int64_t *Ns, int n, int m, int T, int euler)
{
    return kkt_defect_kt(n, m, T, euler != 0, Ns, count);
}

int adjoint_nt_of(int64_t values) { return adjoint_nt(values); }

// How often a grid of ceil(N / span) workgroups of `block` lanes stores each
// of the N + 1 nodes.
void node_owners(int64_t N, int block, int span, int *count)
{
    for (int64_t b = 0; b * span < N; b++)
        for (int tid = 0; tid < block; tid++)
            if (owns_node(tid, b * span + tid, N, span)) count[b * span + tid]++;
}

int batch_obj_grad_once_of(int64_t count, const int64_t *Ns)
{
    return batch_obj_grad_once(std::vector<int64_t>(Ns, Ns + count));
}

int assembly_lg_of(int64_t N, int n, int T) { return assembly_lg(N, n, T); }

int map_lg_of(int64_t N1, int64_t per_node, int n) { return map_lg(N1, per_node, n); }

}  // extern "C"
