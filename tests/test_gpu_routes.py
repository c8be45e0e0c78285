"""Calls whose kernel variant or tile shape is chosen by their sizes, at sizes
on each side of the lines.  Values against the oracle (within 1e-12 * mu) or
bit for bit against another route; the elements around an output stay
untouched."""
from __future__ import annotations

from fractions import Fraction

import numpy as np
import pytest

import oracle
import synth
from tests.helpers import check_close
from tests.test_gpu_line_aligned import Guarded, _t, ocp  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# one interval per lane, two, and whole lines (the last of each group of three
# differs from the first in the grid or the address only); remainders of the
# 512 intervals of a workgroup of pairs; boundary rows beside each
@pytest.mark.parametrize("N,n,m,scheme,bnd,offset", [
    (374992, 1, 1, 0, 2, 0), (374992, 1, 1, 0, 1, 1), (374991, 1, 1, 0, 0, 2),
    (500002, 1, 1, 1, 2, 2), (500002, 1, 0, 1, 1, 0), (500001, 1, 1, 1, 0, 0),
    (9952, 16, 8, 1, 1, 0), (9954, 16, 8, 1, 2, 14), (9952, 16, 8, 1, 0, 3),
    (8194, 16, 8, 0, 2, 0), (2050, 32, 16, 0, 0, 2), (2048, 32, 16, 0, 1, 8),
    (512, 2, 1, 0, 2, 0), (514, 2, 1, 1, 2, 0), (2, 3, 1, 0, 1, 4), (30001, 2, 2, 0, 0, 0)])
def test_jacobian_paths(ocp, N, n, m, scheme, bnd, offset):
    print(f"[routes] jacobian N={N} n={n} m={m} scheme={scheme} bnd={bnd} offset={offset}", flush=True)
    inst = synth.make_instance(N, n, m, seed=81, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    out = Guarded(prob.sizes["nnzj"], offset)
    prob.jac(_t(inst.z), out=out.out)
    want, mu = oracle.jac_ex(inst, scheme, bnd)
    check_close(out.values(), want, mu, what="jac")
    prob.close()


@pytest.mark.parametrize("N,bnd,offset", [(27265, 1, 0), (27266, 2, 1), (27267, 0, 9), (30000, 1, 15),
                                          (30000, 2, 0), (25608, 1, 8), (512, 0, 1)])
def test_quadrotor_jacobian_paths(ocp, N, bnd, offset):
    print(f"[routes] quadrotor jacobian N={N} bnd={bnd} offset={offset}", flush=True)
    q = synth.make_quadrotor(N, seed=82, bnd=bnd)
    prob = ocp.QuadrotorProblem.from_instance(q, torch.device("cuda", 0))
    out = Guarded(prob.sizes["nnzj"], offset)
    prob.jac(_t(q.z), out=out.out)
    want, mu = oracle.quad_jac(q)
    check_close(out.values(), want, mu, what="jac")
    prob.close()


@pytest.mark.parametrize("N,bnd", [(1000, 1), (4097, 0), (30001, 2), (40000, 1)])
def test_quadrotor_fused_kkt_has_the_separate_calls_bits(ocp, N, bnd):
    """eval_kkt evaluates the expressions of jac and hess: without
    regularization its entries are theirs bit for bit, also where the two
    products of a partial derivative nearly cancel (one in 250 entries of such
    slots), on every path of the Jacobian."""
    print(f"[routes] quadrotor fused bits N={N} bnd={bnd}", flush=True)
    q = synth.make_quadrotor(N, seed=83, bnd=bnd)
    prob = ocp.QuadrotorProblem.from_instance(q, torch.device("cuda", 0))
    z, y = _t(q.z), _t(q.y)
    _, _, pj, ph = prob.kkt_pattern()
    kkt = prob.eval_kkt(z, y, 0.7).view(torch.int64)
    assert torch.equal(kkt[_t(pj).long()], prob.jac(z).view(torch.int64))
    assert torch.equal(kkt[_t(ph).long()], prob.hess(z, y, 0.7).view(torch.int64))
    prob.close()


# the forward-Euler defects' boundary rows have a workgroup of their own, after
# the 256 intervals of each of the others; also scaled, in a backward pass
@pytest.mark.parametrize("N,n,m,bnd", [(1, 2, 1, 2), (255, 3, 1, 1), (256, 3, 1, 2), (257, 32, 4, 2), (512, 17, 9, 1),
                                       (256, 5, 2, 0)])
def test_euler_boundary_rows(ocp, N, n, m, bnd):
    print(f"[routes] euler boundary N={N} n={n} m={m} bnd={bnd}", flush=True)
    inst = synth.make_instance(N, n, m, seed=86, bnd=bnd, scheme=1)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    z, y = _t(inst.z), _t(inst.y)
    out = Guarded(prob.sizes["ncon"], 1)
    prob.cons(z, out=out.out)
    want, mu = oracle.cons_ex(inst, 1, bnd)
    check_close(out.values(), want, mu, what="cons")
    gy = prob.lagrangian_backward(z, y, 0.7, _t(np.array([-3.0])))[1].cpu().numpy()
    assert np.array_equal(gy.view(np.uint64), (-3.0 * out.values()).view(np.uint64))
    prob.close()


# the adjoint of the coefficient gradient stores 8 MiB and less through the
# caches; both outputs, and each alone, which may take the other kernel
@pytest.mark.parametrize("N,n,m,scheme,bnd", [
    (149000, 3, 1, 0, 1), (150241, 3, 1, 0, 2), (62005, 8, 1, 1, 1), (33360, 16, 0, 0, 0), (15615, 32, 4, 0, 2),
    (239, 2, 2, 0, 2), (495, 20, 1, 0, 1)])
def test_coefficient_adjoint_stores(ocp, N, n, m, scheme, bnd):
    print(f"[routes] coefficient adjoint N={N} n={n} m={m} scheme={scheme} bnd={bnd}", flush=True)
    inst = synth.make_instance(N, n, m, seed=87, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    z, y = _t(inst.z), _t(inst.y)
    rng = np.random.default_rng(8)
    t = [rng.normal(size=shape) for shape in ((n, n), (n, m), (n,))]
    outs = [Guarded(prob.sizes[k], 3) for k in ("nvar", "ncon")]
    prob.coef_adjoint(z, y, *(_t(a) for a in t), out_z=outs[0].out, out_y=outs[1].out)
    (oz, oy), (mz, my) = oracle.coef_adjoint_ex(inst, *t, scheme, bnd)
    check_close(outs[0].values(), oz, mz, what="z")
    check_close(outs[1].values(), oy, my, what="y")
    for i in (0, 1):
        alone = prob.coef_adjoint(z, y, *(_t(a) for a in t), want_z=i == 0, want_y=i == 1)[i]
        assert torch.equal(alone.view(torch.int64), outs[i].out.view(torch.int64))
    prob.close()


def _fma(a, b, c):
    """a b + c of doubles, rounded once."""
    return np.array([float(Fraction(x) * Fraction(y) + Fraction(w)) for x, y, w in zip(a, b, c)])


@pytest.mark.parametrize("N", [1, 64, 4096])
def test_quadrotor_roll_rate_rounding(ocp, N):
    """d x7' / d x7 = (u3 cos x7 - u2 sin x7) sec x8: the second product is
    rounded, the first fused into the difference.  At x8 = 0 (sec = 1) and a
    step that is a power of two, the sine and cosine that the kernel used stand
    in other entries, so the values follow bit for bit."""
    print(f"[routes] quadrotor roll rate N={N}", flush=True)
    q = synth.make_quadrotor(N, seed=88, bnd=0)
    prob = ocp.QuadrotorProblem.from_instance(q, torch.device("cuda", 0))
    rng = np.random.default_rng(9)
    z = np.array(q.z)
    z[:9 * (N + 1)].reshape(9, N + 1)[7] = 0.0
    z[:9 * (N + 1)].reshape(9, N + 1)[6] = rng.uniform(-1.5, 1.5, N + 1)
    u2, u3 = z[9 * (N + 1):].reshape(4, N + 1)[1:3]
    u2[:], u3[:] = rng.uniform(-2, 2, (2, N + 1))
    slot = prob.jac(_t(z)).cpu().numpy().reshape(68, N)
    hh = -slot[66][0]  # d x9' / d u4 = 1
    assert np.log2(hh) == np.round(np.log2(hh))
    for side in (0, 1):  # node k, node k + 1 of the intervals
        s7, c7 = slot[52 + side] / hh, -slot[54 + side] / hh
        a, b = u2[side:N + side], u3[side:N + side]
        want = _fma(np.full(N, -hh), _fma(b, c7, -(a * s7)), np.full(N, 2.0 * side - 1.0))
        assert np.array_equal(slot[40 + side].view(np.uint64), want.view(np.uint64))
    prob.close()


# a batch's Jacobian tiles: one interval per lane (every instance within a
# wavefront), one or two (even lengths, at any 8-byte offset), and whole lines
# (from 40 MiB on)
@pytest.mark.parametrize("Ns,n,m,scheme,bnd", [
    ([1, 2, 16, 17, 63, 64, 33, 20], 5, 2, 0, 2), ([10, 60, 128, 1, 65], 5, 2, 1, 1),
    ([255, 256, 257, 512, 514, 70, 1, 300], 5, 2, 0, 1), ([512, 511, 2, 130, 1026, 700], 3, 0, 1, 2),
    ([2000, 2001, 2016, 1, 480, 497] * 20, 4, 2, 0, 1), ([2000, 2001, 2016, 1, 992, 4096] * 20, 6, 3, 1, 2)])
def test_batched_jacobian_paths(ocp, Ns, n, m, scheme, bnd):
    print(f"[routes] batched jacobian {Ns[:6]} x {len(Ns)} n={n} m={m} scheme={scheme} bnd={bnd}", flush=True)
    insts = synth.make_batch(len(Ns), n, m, seed=6, Ns=Ns, scheme=scheme, bnd=bnd)
    batch = ocp.Batch.from_instances(insts, scheme=scheme, boundary=bnd)
    z, total = _t(synth.pack(insts)[0]), int(batch.offsets["jac"][-1])
    want = batch.eval(z, what=ocp.EVAL_JAC, mode="per_instance")[0].view(torch.int64)
    for block, pair, wgs in ((256, 1, 0), (128, 1, 1), (256, 0, 1)):
        batch.config = {"block": block, "pair": pair, "wgs_per_cu": wgs, "order": 1}
        for offset in (0, 1, 2):
            out = Guarded(total, offset)
            batch.eval(z, jac=out.out, what=ocp.EVAL_JAC)
            out.values()
            assert torch.equal(out.out.view(torch.int64), want)
    batch.close()


# a batch's defect-row tiles of 16, 32 and 64 intervals over instances shorter
# and longer than a tile; the boundary rows ride in an instance's first tile
@pytest.mark.parametrize("Ns,n,m,scheme,bnd", [
    ([1, 15, 16, 17, 5], 6, 3, 0, 2), ([20] * 30 + [31, 32, 1], 6, 3, 1, 1), ([32, 64, 20, 30], 16, 8, 0, 2),
    ([200, 1, 63, 64, 65, 7000, 9000], 3, 1, 0, 2), ([2049, 64, 127, 15000, 1], 4, 2, 1, 2),
    ([40000, 25500, 65, 64, 1, 16], 12, 5, 0, 1), ([33000, 1, 32800, 5], 24, 10, 0, 2)])
def test_batched_kkt_tiles(ocp, Ns, n, m, scheme, bnd):
    print(f"[routes] batched kkt {Ns[:6]} x {len(Ns)} n={n} m={m} scheme={scheme} bnd={bnd}", flush=True)
    insts = synth.make_batch(len(Ns), n, m, seed=7, Ns=Ns, scheme=scheme, bnd=bnd)
    batch = ocp.Batch.from_instances(insts, scheme=scheme, boundary=bnd)
    z, y = (_t(a) for a in synth.pack(insts))
    reg = _t(np.random.default_rng(5).normal(size=int(batch.offsets["dim"][-1])))
    for r in (None, reg):
        want = batch.step(z, y, 0.7, r, what=ocp.EVAL_KKT, mode="per_instance")["kkt"].view(torch.int64)
        for block in (128, 256):
            batch.config = {"block": block, "pair": 1, "wgs_per_cu": 0, "order": 1}
            out = Guarded(int(batch.offsets["kkt"][-1]), 3)
            batch.step(z, y, 0.7, r, what=ocp.EVAL_KKT, out={"kkt": out.out})
            out.values()
            assert torch.equal(out.out.view(torch.int64), want)
    batch.close()


# the assembly's tiles of 32, 64 and 128 rows, and an injective map under which
# no tile covers its range: a row's entry in each run of 32 rows goes to the next
@pytest.mark.parametrize("N,n,m,scheme,bnd", [
    (1000, 4, 2, 0, 0), (1001, 8, 4, 0, 1), (2065, 8, 4, 1, 2), (16257, 1, 0, 0, 1), (700, 32, 32, 0, 2), (33, 3, 1, 1, 0)])
def test_assembly_without_a_covering_tile(ocp, N, n, m, scheme, bnd):
    print(f"[routes] assembly N={N} n={n} m={m} scheme={scheme} bnd={bnd}", flush=True)
    inst = synth.make_instance(N, n, m, seed=85, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    s = prob.sizes
    rng = np.random.default_rng(6)
    jv, hv, reg = (rng.normal(size=s[k]) for k in ("nnzj", "nnzh", "dim"))
    rp, _, pj, ph = prob.kkt_pattern()
    T = (s["nnzj"] - bnd * n) // (n * N)
    one = np.concatenate([i * T * N + np.arange(0, N, 32) for i in range(n)])  # slot row 0 of each component
    rotated = pj.copy()
    rotated[one] = np.roll(pj[one], 1)
    assert len(np.unique(rotated)) == len(rotated)
    for maps in (pj, rotated):
        for r in (None, reg):
            out = Guarded(s["nnzk"], 1)
            prob.assemble_kkt(_t(maps), _t(ph), _t(rp), _t(jv), _t(hv), None if r is None else _t(r), out=out.out)
            want = oracle.assemble(rp, maps, jv, ph, hv, r)
            assert np.array_equal(out.values().view(np.uint64), want.view(np.uint64))
    prob.close()


# the mapped assembly's tiles of 1, 2, 4 and 8 nodes, shorter on a short grid
@pytest.mark.parametrize("N,n,m,scheme,bnd", [
    (499, 18, 10, 0, 1), (997, 18, 10, 0, 2), (1001, 18, 10, 0, 0), (3201, 18, 10, 0, 2), (101, 12, 6, 0, 2),
    (1, 32, 32, 0, 2), (249, 32, 32, 0, 1), (503, 32, 32, 1, 0), (2, 24, 12, 1, 2)])
def test_mapped_assembly_on_short_grids(ocp, N, n, m, scheme, bnd):
    print(f"[routes] mapped N={N} n={n} m={m} scheme={scheme} bnd={bnd}", flush=True)
    inst = synth.make_instance(N, n, m, seed=84, bnd=bnd, scheme=scheme)
    prob = ocp.Problem.from_instance(inst, torch.device("cuda", 0))
    s = prob.sizes
    rng = np.random.default_rng(4)
    jv, hv, reg = (rng.normal(size=s[k]) for k in ("nnzj", "nnzh", "dim"))
    pj2, ph2, dg2 = ocp.kkt_permute(*prob.kkt_pattern(), ocp.stage_order(N, n, m, scheme, bnd))[2:]
    shuffled = rng.permutation(s["nnzk"]).astype(np.int32)
    for maps in ((pj2, ph2, dg2), tuple(shuffled[q] for q in (pj2, ph2, dg2))):
        dmaps = [_t(q) for q in maps]
        want = oracle.assemble_mapped(s["nnzk"], maps[2], maps[0], jv, maps[1], hv, reg)
        for plan in (None, prob.mapped_plan(*dmaps)):
            out = Guarded(s["nnzk"], 3)
            prob.assemble_kkt_mapped(*dmaps, _t(jv), _t(hv), _t(reg), out=out.out, plan=plan)
            assert np.array_equal(out.values().view(np.uint64), want.view(np.uint64))
    prob.close()


# objective and gradient: tiles of their own up to 256 tiles and for a mask of
# one, tiles that load each node once above; controls in groups of the state
# bound, with and after the states
@pytest.mark.parametrize("Ns,n,m,scheme", [
    ([255, 256, 1, 20] * 3, 3, 9, 0), ([255, 256, 1, 20] * 70, 3, 9, 0), ([511, 512, 7] * 60, 8, 4, 1),
    ([70000], 12, 5, 0), ([40, 300] * 90, 16, 17, 1), ([40, 257] * 90, 24, 10, 0)])
def test_batched_objective_and_gradient(ocp, Ns, n, m, scheme):
    print(f"[routes] batched obj+grad {Ns[:4]} x {len(Ns)} n={n} m={m} scheme={scheme}", flush=True)
    insts = synth.make_batch(len(Ns), n, m, seed=8, Ns=Ns, scheme=scheme)
    batch = ocp.Batch.from_instances(insts, scheme=scheme)
    z = _t(synth.pack(insts)[0])
    both = ocp.EVAL_OBJ | ocp.EVAL_GRAD
    ref = batch.step(z, what=both, mode="per_instance")
    for block in (128, 256):
        for wgs in (0, 1):
            batch.config = {"block": block, "pair": 1, "wgs_per_cu": wgs, "order": 1}
            for what in (both, ocp.EVAL_OBJ, ocp.EVAL_GRAD):
                g = Guarded(int(batch.offsets["z"][-1]), 5)
                got = batch.step(z, what=what, out={"grad": g.out})
                if what & ocp.EVAL_OBJ:
                    assert torch.equal(got["obj"].view(torch.int64), ref["obj"].view(torch.int64))
                if what & ocp.EVAL_GRAD:
                    g.values()
                    assert torch.equal(g.out.view(torch.int64), ref["grad"].view(torch.int64))
    batch.close()
