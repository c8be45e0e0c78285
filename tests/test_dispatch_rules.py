"""The rules that choose a kernel variant or a tile shape, on the CPU: each
test holds sizes on both sides of a line at which the variants were timed."""
from __future__ import annotations

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

SINGLE, PAIR, LINES = 0, 1, 2  # rules::JacPath


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rules") / "rules.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2510_03932_amd", "csrc"),
                           os.path.join(ROOT, "tests", "dispatch_rules.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    lib.jac_path_of.argtypes = [i64, i32, i32, i32, i32, ctypes.c_uint64]
    lib.quad_jac_path_of.argtypes = [i64, ctypes.c_uint64]
    lib.kkt_defect_kt_of.argtypes = [i64, ctypes.POINTER(i64), i32, i32, i32, i32]
    lib.batch_obj_grad_once_of.argtypes = [i64, ctypes.POINTER(i64)]
    lib.assembly_lg_of.argtypes = [i64, i32, i32]
    lib.map_lg_of.argtypes = [i64, i64, i32]
    lib.batch_jac_of.argtypes = [i64, ctypes.POINTER(i64), i32, i32, i32, i32, i32]
    return lib


@pytest.mark.parametrize("N,n,m,euler,offset,want", [
    # rows that take no pairs: whole lines once enough workgroups carry them
    (13009, 8, 4, 0, 0, SINGLE), (52081, 4, 2, 0, 0, LINES), (5457, 32, 16, 0, 0, LINES),
    (2049, 32, 16, 0, 0, SINGLE), (53569, 4, 2, 1, 0, SINGLE), (124993, 4, 2, 1, 0, LINES),
    (20000, 8, 4, 0, 1, SINGLE), (1, 1, 0, 0, 0, SINGLE),
    # an even grid: pairs past the smallest outputs, whole lines past the L2s
    (734000, 1, 1, 0, 0, PAIR), (978656, 1, 1, 1, 0, PAIR), (32768, 8, 4, 0, 0, PAIR),
    (2050, 32, 16, 0, 0, PAIR), (8194, 16, 8, 0, 0, PAIR), (58594, 8, 4, 0, 0, LINES),
    (13008, 8, 4, 0, 0, SINGLE), (4544, 16, 8, 0, 0, SINGLE), (9952, 16, 8, 1, 0, PAIR),
    (2500002, 1, 1, 1, 0, PAIR),
    # rows on lines or half lines: never whole lines
    (58600, 8, 4, 0, 0, PAIR), (65104, 16, 8, 0, 8, PAIR), (65104, 16, 8, 0, 4, LINES),
    (100000, 8, 4, 0, 0, PAIR), (1000000, 16, 8, 0, 0, PAIR)])
def test_jacobian_path(rules, N, n, m, euler, offset, want):
    slots = n + 1 + m if euler else 2 * (n + m)
    assert rules.jac_path_of(N, n, m, slots, euler, 1 << 20 | 8 * offset) == want


@pytest.mark.parametrize("N,offset,want", [
    (10000, 0, SINGLE), (20000, 0, SINGLE), (26000, 0, PAIR), (26001, 0, SINGLE), (26000, 1, SINGLE),
    (30001, 0, LINES), (30000, 0, PAIR), (30000, 4, LINES), (50000, 0, PAIR), (60000, 0, LINES), (1, 0, SINGLE)])
def test_quadrotor_jacobian_path(rules, N, offset, want):
    assert rules.quad_jac_path_of(N, 1 << 20 | 8 * offset) == want


DIRECT, SHORT, BATCH_LINES = 0, 1, 2  # rules::BatchJac


def _lengths(Ns):
    Ns = np.ascontiguousarray(Ns, np.int64)
    return len(Ns), Ns.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), Ns


@pytest.mark.parametrize("count,lo,hi,n,m,euler,pair,want", [
    # short horizons, as model-predictive control has them
    (4096, 10, 60, 4, 2, 0, 1, SHORT), (4096, 10, 60, 16, 8, 0, 1, SHORT), (23529, 17, 17, 6, 3, 0, 1, SHORT),
    (4096, 10, 60, 16, 8, 1, 1, SHORT), (1024, 50, 200, 8, 4, 1, 1, SHORT), (40, 20, 20, 4, 2, 0, 0, SHORT),
    # a wavefront or two more: direct, until whole lines pay
    (6153, 65, 65, 16, 8, 0, 1, DIRECT), (1024, 50, 200, 6, 3, 0, 1, DIRECT), (2072, 193, 193, 6, 3, 0, 1, DIRECT),
    (1024, 100, 300, 4, 2, 0, 1, DIRECT), (256, 100, 300, 6, 3, 1, 1, DIRECT), (2072, 193, 193, 16, 8, 0, 1, BATCH_LINES),
    (804, 497, 497, 4, 2, 0, 1, DIRECT), (1556, 257, 257, 6, 3, 0, 1, BATCH_LINES),
    # long instances: whole lines past the L2s
    (512, 200, 20000, 6, 3, 0, 1, BATCH_LINES), (512, 200, 20000, 6, 3, 0, 0, DIRECT),
    (9, 2001, 2001, 6, 3, 0, 1, DIRECT), (512, 100, 2000, 16, 8, 1, 1, BATCH_LINES), (402, 497, 497, 6, 3, 1, 1, DIRECT),
    (77, 257, 257, 16, 8, 0, 1, DIRECT), (520, 384, 384, 6, 3, 0, 1, DIRECT), (1, 1, 1, 1, 0, 0, 1, SHORT)])
def test_batched_jacobian_path(rules, count, lo, hi, n, m, euler, pair, want):
    slots = n + 1 + m if euler else 2 * (n + m)
    k, ptr, _keep = _lengths(np.random.default_rng(0).integers(lo, hi + 1, count))
    assert rules.batch_jac_of(k, ptr, n, slots, euler, pair, 256) == want


@pytest.mark.parametrize("count,lo,hi,n,m,euler,want", [
    # one instance: by its length and the work of a tile
    (1, 20000, 20000, 3, 1, 0, 64), (1, 10000, 10000, 2, 1, 0, 32), (1, 5000, 5000, 4, 2, 0, 16),
    (1, 20000, 20000, 4, 2, 0, 32), (1, 41000, 41000, 4, 2, 0, 64), (1, 20000, 20000, 16, 8, 0, 32),
    (1, 20001, 20001, 16, 8, 1, 16), (1, 10000, 10000, 12, 5, 0, 16), (1, 333333, 333333, 12, 5, 0, 64),
    (1, 1000000, 1000000, 16, 8, 0, 64), (1, 1000000, 1000000, 16, 8, 1, 32), (1, 33000, 33000, 32, 16, 0, 16),
    # a batch: by the length of its instances too
    (4096, 16, 16, 16, 8, 0, 16), (4096, 16, 16, 6, 3, 0, 16), (4096, 5, 5, 12, 5, 1, 16), (4096, 20, 20, 12, 5, 0, 32),
    (4096, 33, 33, 6, 3, 0, 64), (4096, 10, 60, 6, 3, 0, 64), (1024, 20, 20, 16, 8, 0, 32), (300, 200, 200, 4, 2, 1, 64),
    (300, 16, 16, 16, 8, 0, 16), (512, 200, 20000, 6, 3, 0, 64), (1, 1, 1, 1, 1, 1, 16)])
def test_kkt_defect_tile(rules, count, lo, hi, n, m, euler, want):
    T = n + 1 + m if euler else 2 * (n + m)
    k, ptr, _keep = _lengths(np.random.default_rng(0).integers(lo, hi + 1, count))
    assert rules.kkt_defect_kt_of(k, ptr, n, m, T, euler) == want


@pytest.mark.parametrize("count,N,once", [(1, 1, 0), (256, 255, 0), (256, 256, 1), (257, 1, 1), (1, 65535, 0),
                                          (1, 65536, 1), (512, 10000, 1)])
def test_batched_objective_and_gradient_tiles(rules, count, N, once):
    k, ptr, _keep = _lengths(np.full(count, N))
    assert rules.batch_obj_grad_once_of(k, ptr) == once


@pytest.mark.parametrize("N,n,m,euler,lg", [
    # short grids: tiles no taller than 4 nodes, and 16 KiB
    (50, 18, 10, 0, 2), (100, 18, 10, 1, 2), (500, 18, 10, 0, 2), (1000, 18, 10, 0, 2), (2000, 18, 10, 0, 2),
    (100, 12, 6, 0, 2), (2000, 12, 6, 0, 2), (100, 8, 4, 0, 3), (1, 1, 0, 0, 8), (100, 24, 12, 1, 2),
    (50, 32, 32, 0, 0), (100, 32, 32, 1, 1), (499, 32, 20, 0, 1),
    # long ones: half a line of values per slot row, as far as 72 KiB go
    (4000, 18, 10, 0, 3), (3500, 12, 6, 0, 3), (500, 32, 32, 0, 1), (100000, 8, 4, 0, 4), (100000, 32, 32, 0, 1),
    (100000, 32, 32, 1, 2), (1000000, 2, 1, 0, 7), (100000, 1, 0, 1, 8)])
def test_mapped_assembly_tile(rules, N, n, m, euler, lg):
    slots = n + 1 + m if euler else 2 * (n + m)
    pairs = 0 if n < 2 else (1 if n == 2 else n)
    per_node = n * slots + n + pairs + m + n
    assert rules.map_lg_of(N + 1, per_node, n) == lg
    assert (per_node << lg) + 2 * n <= 9216


def test_mapped_assembly_tiles_never_shrink(rules):
    """A caller may hold a plan made when the tiles were as many nodes as fit
    2048 values, at least 4 while those fit 7936: it has an entry for every
    tile as long as no tile is shorter than that."""
    for N in (1, 50, 300, 999, 4000, 100000):
        for per_node in list(range(4, 300, 7)) + list(range(300, 5000, 53)):
            n = min(32, max(1, per_node // 30))
            lg = 0
            while lg < 10 and (per_node << (lg + 1)) + 2 * n <= 2048:
                lg += 1
            while lg < 2 and (per_node << (lg + 1)) + 2 * n <= 7936:
                lg += 1
            assert rules.map_lg_of(N + 1, per_node, n) >= lg


@pytest.mark.parametrize("N,n,m,euler,lg", [
    # fewer than 128 tiles: shorter ones
    (1000, 4, 2, 0, 5), (4000, 2, 1, 0, 5), (1000, 8, 4, 0, 6), (300, 8, 4, 0, 5), (1, 1, 0, 0, 5), (992, 8, 4, 1, 6),
    # from there on as tall as 64 KiB allow
    (2000, 8, 4, 0, 7), (16000, 4, 2, 0, 7), (16000, 2, 1, 0, 7), (16257, 1, 0, 0, 7), (16256, 1, 0, 0, 6),
    (1000, 16, 8, 0, 7), (1000, 32, 16, 0, 6), (1000, 32, 32, 0, 5), (1000000, 24, 10, 0, 6)])
def test_assembly_tile(rules, N, n, m, euler, lg):
    T = n + 1 + m if euler else 2 * (n + m)
    assert rules.assembly_lg_of(N, n, T) == lg
    assert (T + 1) * 8 << lg <= 64 * 1024


@pytest.mark.parametrize("N", [1, 15, 239, 240, 241, 254, 255, 256, 479, 480, 481, 495, 496, 1000])
def test_one_workgroup_stores_a_node(rules, N):
    count = np.zeros(N + 256, np.int32)
    rules.node_owners(ctypes.c_int64(N), 256, 240, count.ctypes.data_as(ctypes.c_void_p))
    assert np.array_equal(count[:N + 1], np.ones(N + 1)) and not count[N + 1:].any()


@pytest.mark.parametrize("N,n,m,nt", [(1000, 2, 1, 0), (50001, 4, 2, 0), (20000, 8, 4, 0), (100000, 8, 4, 1),
                                      (333333, 12, 5, 1), (1, 1, 0, 0)])
def test_adjoint_stores(rules, N, n, m, nt):
    assert rules.adjoint_nt_of(ctypes.c_int64(n * (N + 1) + m * (N + 1) + n * N)) == nt


def test_assembly_clears_its_tile():
    """A slot map that names a slot twice is outside the contract, so no test
    runs one; the tile's places that it leaves empty have to be zeros all the
    same, not what the LDS held."""
    src = open(os.path.join(ROOT, "paper_2510_03932_amd", "csrc", "ocp_eval.hip")).read()
    kernel = src[src.index("void assemble_kernel("):]
    clear, barrier, put = (kernel.find(s) for s in ("(tile + x) = dbl2{0.0, 0.0}", "__syncthreads()", "tile[loc] = v"))
    assert 0 < clear < barrier < put


def test_kernels_look_at_no_address():
    """Addresses become integers on the host only (line_pos, the Jacobian's
    path): in a kernel they cost the coefficients the scalar cache."""
    csrc = os.path.join(ROOT, "paper_2510_03932_amd", "csrc")
    hits = [line.strip() for name in sorted(os.listdir(csrc)) if name.endswith((".hip", ".h"))
            for line in open(os.path.join(csrc, name)) if "uintptr_t" in line]
    allowed = ("inline int line_pos(const double *p)", "switch (rules::jac_path(", "switch (rules::quad_jac_path(")
    assert len(hits) == 3 and all(h.startswith(allowed) for h in hits), hits
