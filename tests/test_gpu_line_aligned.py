"""Kernels whose stores are placed on 128-byte lines, at the sizes and output
addresses where that placement can go wrong: outputs at any 8-byte offset,
grids of any remainder, and each tile height.  Values against the oracle
(within 1e-12 * mu); the elements around the output stay untouched."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from tests.helpers import check_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PAD = 16  # doubles of a line: guard elements before and after an output


@pytest.fixture(scope="module")
def ocp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_03932_amd as ocp
    ocp.lib()
    return ocp


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda", 0))


class Guarded:
    """An output of `count` doubles at element `offset` past a 128-byte line,
    with a marker in the elements before and after it."""

    def __init__(self, count, offset):
        self.raw = torch.full((count + offset + 2 * PAD,), -7.25, dtype=torch.float64, device="cuda")
        assert self.raw.data_ptr() % (8 * PAD) == 0
        self.lo, self.hi = PAD + offset, PAD + offset + count
        self.out = self.raw[self.lo:self.hi]
        self.out.fill_(float("nan"))

    def values(self):
        a = self.raw.cpu().numpy()
        assert np.all(a[:self.lo] == -7.25) and np.all(a[self.hi:] == -7.25), "stored outside the output"
        return a[self.lo:self.hi]


# the fused KKT call's defect rows take tiles of 64 intervals from N = 65,536
# (n = 20, m = 10: 32, the LDS bound; forward Euler n = 13 is the last of its
# half bound at m = 3, n = 14 takes 32), 32 from 32,768, else 16
@pytest.mark.parametrize("N,n,m,scheme,bnd,offset", [
    (65536, 3, 1, 0, 0, 1), (65573, 2, 1, 0, 2, 15), (65599, 3, 2, 1, 1, 8), (65541, 20, 10, 0, 0, 3),
    (65541, 13, 3, 1, 0, 1), (65541, 14, 3, 1, 2, 6),
    (32768, 4, 0, 0, 1, 9), (32799, 3, 1, 1, 2, 0), (32767, 5, 2, 0, 0, 7), (17, 3, 1, 0, 0, 5), (1, 1, 1, 1, 2, 2)])
def test_fused_kkt_tiles(ocp, N, n, m, scheme, bnd, offset):
    print(f"[lines] fused N={N} n={n} m={m} scheme={scheme} bnd={bnd} offset={offset}", flush=True)
    inst = synth.make_instance(N, n, m, seed=71, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    s = prob.sizes
    rp, _, pj, ph = ocp.kkt_pattern(N, n, m, scheme=scheme, boundary=bnd)
    reg = np.random.default_rng(5).normal(size=s["dim"])
    out = Guarded(s["nnzk"], offset)
    prob.eval_kkt(_t(inst.z), _t(inst.y), 0.7, _t(reg), out=out.out)
    oj, mj = oracle.jac_ex(inst, scheme, bnd)
    oh, mh = oracle.hess_ex(inst, scheme, bnd, sigma=0.7)
    check_close(out.values(), oracle.assemble(rp, pj, oj, ph, oh, reg),
                oracle.assemble(rp, pj, mj, ph, mh, np.abs(reg)), what="kkt")
    prob.close()


# the assembly takes tiles of 128 rows from 512 of them, else 64 or 32; at
# n = m = 32 (T = 128) the LDS bound gives 32; N odd puts every other slot row
# off the 16-byte grid
@pytest.mark.parametrize("N,n,m,scheme,bnd,offset", [
    (65536, 1, 0, 0, 0, 0), (21845, 3, 1, 0, 1, 1), (21889, 3, 2, 1, 2, 15), (16384, 2, 1, 0, 0, 8),
    (10923, 3, 1, 0, 0, 3), (5500, 3, 1, 1, 0, 9), (97, 5, 2, 0, 2, 7), (2051, 32, 32, 0, 0, 5), (1, 1, 0, 0, 0, 2),
    (2, 2, 2, 1, 1, 4)])
def test_assembly_tiles(ocp, N, n, m, scheme, bnd, offset):
    print(f"[lines] assembly N={N} n={n} m={m} scheme={scheme} bnd={bnd} offset={offset}", flush=True)
    prob = ocp.Problem(N, n, m, np.zeros((n, n)), np.zeros((n, m)), np.zeros(n), np.ones(n), np.ones(m),
                       scheme=scheme, boundary=bnd)
    s = prob.sizes
    rng = np.random.default_rng(3)
    jv, hv, reg = (rng.normal(size=s[k]) for k in ("nnzj", "nnzh", "dim"))
    rp, _, pj, ph = prob.kkt_pattern()
    cross = pj.copy()  # an injective map whose tiles exchange slots: no tile covers its range
    cross[[0, -1 - bnd * n]] = cross[[-1 - bnd * n, 0]]
    for maps in (pj, cross):
        for r in (None, reg):
            out = Guarded(s["nnzk"], offset)
            # inputs at odd elements too: the paired loads take any alignment
            prob.assemble_kkt(_t(np.r_[np.int32(0), maps])[1:], _t(ph), _t(rp), _t(np.r_[0.0, jv])[1:], _t(hv),
                              None if r is None else _t(r), out=out.out)
            want = oracle.assemble(rp, maps, jv, ph, hv, r)
            assert np.array_equal(out.values().view(np.uint64), want.view(np.uint64))
    prob.close()


# slot rows are stored in whole lines above 32 MiB of output unless every row
# begins on a line; a tile holds 496 intervals and reaches 15 before its start
@pytest.mark.parametrize("N,n,m,scheme,bnd,offset", [
    (89280, 4, 2, 0, 0, 0), (89281, 4, 2, 0, 2, 1), (89265, 4, 2, 0, 0, 15), (178531, 4, 2, 1, 1, 7),
    (120011, 6, 1, 1, 2, 8), (524289, 2, 0, 0, 0, 3), (1048579, 1, 1, 0, 1, 4), (2100007, 1, 0, 1, 0, 9),
    (60000, 5, 3, 0, 0, 0), (60000, 5, 3, 0, 0, 16), (98000, 5, 3, 1, 0, 8), (8001, 16, 8, 0, 0, 2)])
def test_jacobian_lines(ocp, N, n, m, scheme, bnd, offset):
    print(f"[lines] jacobian N={N} n={n} m={m} scheme={scheme} bnd={bnd} offset={offset}", flush=True)
    inst = synth.make_instance(N, n, m, seed=72, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    out = Guarded(prob.sizes["nnzj"], offset)
    prob.jac(_t(inst.z), out=out.out)
    want, mu = oracle.jac_ex(inst, scheme, bnd)
    check_close(out.values(), want, mu, what="jac")
    prob.close()


@pytest.mark.parametrize("scheme,bnd", [(0, 0), (0, 1), (1, 2)])
def test_batched_jacobian_lines_match_per_instance(ocp, scheme, bnd):
    """Instances around a tile of 496 (256 lanes) or 240 (128 lanes) intervals,
    and ones whose rows begin on lines, at an output off the line."""
    Ns = [496, 481, 482, 480, 240, 225, 226, 1, 16, 15, 17, 2049, 992, 977]
    insts = synth.make_batch(len(Ns), 5, 2, seed=4, Ns=Ns, scheme=scheme, bnd=bnd)
    batch = ocp.Batch.from_instances(insts, scheme=scheme, boundary=bnd)
    z, _ = synth.pack(insts)
    z, total = _t(z), int(batch.offsets["jac"][-1])
    want = batch.eval(z, what=ocp.EVAL_JAC, mode="per_instance")[0].cpu().numpy()
    for block in (128, 256):
        for wgs in (0, 1):
            batch.config = {"block": block, "pair": 1, "wgs_per_cu": wgs, "order": 1}
            for offset in (0, 1, 8):
                out = Guarded(total, offset)
                batch.eval(z, jac=out.out, what=ocp.EVAL_JAC)
                assert np.array_equal(out.values().view(np.uint64), want.view(np.uint64))
    batch.close()


# the mapped assembly's tiles hold 32 KiB of values from 512 of them, else
# 16 KiB, and at least 8 nodes while those fit 72 KiB (more LDS than 64 KiB
# needs the kernel's attribute, also when the call is captured)
@pytest.mark.parametrize("N,n,m,scheme,bnd,offset", [
    (32767, 3, 1, 0, 0, 1), (32766, 3, 1, 0, 1, 0), (33001, 3, 1, 1, 2, 15), (100, 18, 10, 0, 2, 8),
    (37, 24, 20, 0, 0, 3), (50, 32, 32, 1, 1, 5), (4, 20, 0, 0, 2, 7)])
def test_mapped_assembly_tiles(ocp, N, n, m, scheme, bnd, offset):
    print(f"[lines] mapped N={N} n={n} m={m} scheme={scheme} bnd={bnd} offset={offset}", flush=True)
    prob = ocp.Problem(N, n, m, np.zeros((n, n)), np.zeros((n, m)), np.zeros(n), np.ones(n), np.ones(m),
                       scheme=scheme, boundary=bnd)
    s = prob.sizes
    rng = np.random.default_rng(3)
    jv, hv, reg = (rng.normal(size=s[k]) for k in ("nnzj", "nnzh", "dim"))
    maps = ocp.kkt_permute(*prob.kkt_pattern(), ocp.stage_order(N, n, m, scheme, bnd))[2:]
    want = oracle.assemble_mapped(s["nnzk"], maps[2], maps[0], jv, maps[1], hv, reg)
    dmaps, args = [_t(a) for a in maps], [_t(a) for a in (jv, hv, reg)]
    for plan in (None, prob.mapped_plan(*dmaps)):
        out = Guarded(s["nnzk"], offset)
        prob.assemble_kkt_mapped(*dmaps, *args, out=out.out, plan=plan)
        assert np.array_equal(out.values().view(np.uint64), want.view(np.uint64))
    graph, out = torch.cuda.CUDAGraph(), Guarded(s["nnzk"], offset)
    with torch.cuda.graph(graph):
        prob.assemble_kkt_mapped(*dmaps, *args, out=out.out, plan=plan)
    for _ in range(3):
        out.out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.values().view(np.uint64), want.view(np.uint64))
    prob.close()


# quadrotor: slot rows in whole lines (tiles of 496) above 32 MiB of Jacobian,
# defect rows of the fused KKT in tiles of 255 intervals, variable rows in
# tiles of 256 nodes, assembly tiles of 144 to 2048 rows
@pytest.mark.parametrize("N,bnd,offset", [(61681, 0, 0), (61682, 1, 1), (61504, 2, 15), (61505, 0, 8), (62000, 1, 3),
                                          (255, 1, 1), (256, 2, 8), (510, 0, 15), (511, 1, 5), (1, 2, 7),
                                          (2048, 0, 4), (2049, 2, 9)])
def test_quadrotor_tiles(ocp, N, bnd, offset):
    print(f"[lines] quadrotor N={N} bnd={bnd} offset={offset}", flush=True)
    q = synth.make_quadrotor(N, seed=73, bnd=bnd)
    prob = ocp.QuadrotorProblem.from_instance(q, torch.device("cuda", 0))
    s = prob.sizes
    z, y = _t(q.z), _t(q.y)
    rp, _, pj, ph = prob.kkt_pattern()
    reg = np.random.default_rng(5).normal(size=s["dim"])
    (oj, mj), (oh, mh) = oracle.quad_jac(q), oracle.quad_hess(q, sigma=0.7)
    jac = Guarded(s["nnzj"], offset)
    prob.jac(z, out=jac.out)
    check_close(jac.values(), oj, mj, what="jac")
    kkt = Guarded(s["nnzk"], offset)
    prob.eval_kkt(z, y, 0.7, _t(reg), out=kkt.out)
    check_close(kkt.values(), oracle.assemble(rp, pj, oj, ph, oh, reg),
                oracle.assemble(rp, pj, mj, ph, mh, np.abs(reg)), what="fused kkt")
    asm = Guarded(s["nnzk"], offset)
    prob.assemble_kkt(_t(np.r_[np.int32(0), pj])[1:], _t(ph), _t(rp), jac.out, _t(np.r_[0.0, oh])[1:], _t(reg),
                      out=asm.out)
    want = oracle.assemble(rp, pj, jac.values(), ph, oh, reg)
    assert np.array_equal(asm.values().view(np.uint64), want.view(np.uint64))
    prob.close()


# workgroups of the defect, J v and coefficient-adjoint kernels close 240
# intervals from 256 nodes; the Lagrangian's first pass takes one chunk of 255
# per workgroup up to 4096 of them; its controls' register bound halves when
# m <= half the state bound
@pytest.mark.parametrize("N,n,m,scheme,bnd", [
    (240, 4, 2, 0, 1), (241, 4, 3, 0, 0), (255, 8, 4, 0, 2), (256, 8, 5, 1, 1), (480, 3, 0, 0, 0), (479, 16, 8, 0, 1),
    (511, 16, 9, 1, 0), (1, 2, 1, 0, 2), (239, 20, 10, 0, 0), (1044480, 1, 1, 0, 0), (1044481, 1, 1, 0, 1)])
def test_node_spans(ocp, N, n, m, scheme, bnd):
    print(f"[lines] spans N={N} n={n} m={m} scheme={scheme} bnd={bnd}", flush=True)
    inst = synth.make_instance(N, n, m, seed=74, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    z, y = _t(inst.z), _t(inst.y)
    rng = np.random.default_rng(8)
    v = rng.normal(size=prob.sizes["nvar"])
    t = [rng.normal(size=sh) for sh in ((n, n), (n, m), (n,))]
    cons, jv = Guarded(prob.sizes["ncon"], 1), Guarded(prob.sizes["ncon"], 3)
    prob.cons(z, out=cons.out)
    check_close(cons.values(), *oracle.cons_ex(inst, scheme, bnd), what="cons")
    prob.jvp(z, _t(v), out=jv.out)
    check_close(jv.values(), *oracle.jvp_ex(inst, v, scheme, bnd), what="jvp")
    L = prob.lagrangian(z, y, 0.7).cpu().numpy()
    want, mu = oracle.lagrangian_ex(inst, scheme, bnd, sigma=0.7)
    check_close(L, np.atleast_1d(want), np.atleast_1d(mu), what="L")
    gz, gy = Guarded(prob.sizes["nvar"], 0), Guarded(prob.sizes["ncon"], 9)
    prob.coef_adjoint(z, y, *(_t(a) for a in t), out_z=gz.out, out_y=gy.out)
    (wz, wy), (mz, my) = oracle.coef_adjoint_ex(inst, *t, scheme, bnd)
    check_close(gz.values(), wz, mz, what="adjoint z")
    check_close(gy.values(), wy, my, what="adjoint y")
    prob.close()


@pytest.mark.parametrize("quad,bnd", [(False, 0), (False, 2), (True, 1)])
def test_scaled_backward_bits(ocp, quad, bnd):
    """The one-call backward equals the separate calls' values times the
    incoming gradient, bit for bit, with each kernel scaling its own stores."""
    inst = synth.make_quadrotor(777, seed=75, bnd=bnd) if quad else synth.make_instance(777, 5, 3, seed=75, bnd=bnd)
    prob = (ocp.QuadrotorProblem if quad else ocp.Problem).from_instance(inst, torch.device("cuda", 0))
    z, y = _t(inst.z), _t(inst.y)
    g = _t(np.array([-0.37]))
    gz, gy, coef = prob.lagrangian_backward(z, y, 0.7, g, want_coef=not quad)
    same = lambda a, b: torch.equal(a.view(torch.int64), b.view(torch.int64))  # noqa: E731
    assert same(gz, prob.lag_grad(z, y, 0.7) * g) and same(gy, prob.cons(z) * g)
    if not quad:
        assert all(same(a, b * g) for a, b in zip(coef, prob.coef_grad(z, y)))
    prob.close()


# the gradient's workgroups take 256 nodes of whole lines of a row; batched
# tiles take the objective's 256 nodes and the gradient from one load, more
# controls than the state bound in groups
@pytest.mark.parametrize("N,n,m,scheme,offset", [(255, 3, 1, 0, 1), (256, 4, 2, 1, 0), (241, 2, 7, 0, 15),
                                                 (240, 4, 9, 1, 8), (511, 8, 4, 0, 3), (497, 5, 0, 0, 7),
                                                 (1, 1, 1, 1, 2), (14, 1, 0, 0, 9)])
def test_gradient_lines(ocp, N, n, m, scheme, offset):
    print(f"[lines] gradient N={N} n={n} m={m} scheme={scheme} offset={offset}", flush=True)
    insts = synth.make_batch(3, n, m, seed=76, Ns=[N, N + 1, max(1, N - 1)], scheme=scheme)
    want, mu = oracle.grad_ex(insts[0], scheme, 0)
    prob = ocp.Problem.from_instance(insts[0], torch.device("cuda", 0))
    out = Guarded(prob.sizes["nvar"], offset)
    prob.grad(_t(insts[0].z), out=out.out)
    check_close(out.values(), want, mu, what="grad")
    prob.close()
    batch = ocp.Batch.from_instances(insts, scheme=scheme)
    z = _t(synth.pack(insts)[0])
    both = ocp.EVAL_OBJ | ocp.EVAL_GRAD
    ref = batch.step(z, what=both, mode="per_instance")
    for block in (128, 256):
        for wgs in (0, 1):
            batch.config = {"block": block, "pair": 1, "wgs_per_cu": wgs, "order": 1}
            for what in (both, ocp.EVAL_OBJ, ocp.EVAL_GRAD):
                g = Guarded(int(batch.offsets["z"][-1]), offset)
                got = batch.step(z, what=what, out={"grad": g.out})
                if what & ocp.EVAL_OBJ:
                    assert torch.equal(got["obj"].view(torch.int64), ref["obj"].view(torch.int64))
                if what & ocp.EVAL_GRAD:
                    assert np.array_equal(g.values().view(np.uint64), ref["grad"].cpu().numpy().view(np.uint64))
    batch.close()
