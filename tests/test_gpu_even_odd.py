"""CG on the even-odd reduced system (Schur complement over the even sites of
the red-black colouring) against the oracle's plain CG and against the
library's own plain-CG path (TIP_EO=0): same quadratures to the 1e-10 bar,
fewer iterations, and the plain path wherever the reduction does not apply."""

import os

import numpy as np
import pytest

from conftest import gpu_binding, to_dev
from oracle import exact
from oracle.estimator import trace_inv_probe as oracle_trace
from oracle.mask import MASK_NONE, MASK_Z2, MASK_Z4
from oracle.operators import Operator as OracleOp
from paper_1302_4018_amd import inputs

pytestmark = pytest.mark.gpu
REL = 1e-10


def _rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b)) / np.maximum(np.abs(np.asarray(b)), 1e-300)))


def _ops(tip, dims, kind, seed, coupled=True, field=True, mass=0.1):
    w = inputs.couplings(dims, seed=seed + 1) if coupled else None
    mf = inputs.mass_field(dims, seed=seed + 2) if field else None
    U = inputs.haar_links(dims, seed=seed + 3) if kind == 1 else None
    orc = OracleOp(dims, kind, mass=mass, mass_field=mf, coupling=w, links=U)
    gop = tip.Operator(dims, kind, mass=mass, mass_field=to_dev(mf), coupling=to_dev(w), links=to_dev(U))
    return orc, gop


def _plain(tip, gop, *args, **kw):
    os.environ["TIP_EO"] = "0"
    try:
        return tip.trace_inv_probe(gop, *args, **kw)
    finally:
        del os.environ["TIP_EO"]


@pytest.mark.parametrize("dims,kind,n,mask", [
    ([8, 8, 8, 8], 1, 8, MASK_Z4),        # covariant, several tiles
    ([4, 4, 4, 8], 1, 16, MASK_Z4),
    ([16, 16], 0, 32, MASK_Z2),           # 2-D scalar
    ([8, 4, 8], 0, 24, MASK_Z4),          # 3-D complex scalar, n not a power of two
    ([2, 2, 2, 2], 1, 16, MASK_NONE),     # smallest bipartite 4-D torus
])
def test_even_odd_matches_oracle_and_plain_cg(dims, kind, n, mask):
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, kind, seed=400 + kind)
    tol = 1e-12
    print(f"even-odd parity: dims {dims} kind {kind} n {n} mask {mask}", flush=True)
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=mask)
    est_p, q_p, st_p = _plain(tip, gop, n, tol, 4018, mask=mask)
    est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, mask)
    assert st["even_odd"] == 1 and st_p["even_odd"] == 0
    assert st["max_true_relres"] <= tol
    assert _rel(est, est_o) <= REL and _rel(q, q_o) <= REL
    assert _rel(est, est_p) <= REL
    assert st["total_iters"] < st_p["total_iters"]


def test_even_odd_exact_recovery():
    tip = gpu_binding()
    orc, gop = _ops(tip, [2, 2, 4, 2], 1, seed=410)
    est, q, st = tip.trace_inv_probe(gop, orc.V, 1e-12, 5)
    assert st["even_odd"] == 1
    tr = exact.dense_trace_inverse(orc.dense())
    assert abs(est[-1] - tr) <= 1e-10 * abs(tr)


@pytest.mark.parametrize("dims,kind,coupling_sign", [
    ([1, 8, 8], 0, 1.0),       # a side of 1: self-loops, not bipartite
    ([8, 8], 0, -1.0),         # a negative coupling: no positive-diagonal guarantee
])
def test_plain_cg_where_the_reduction_does_not_apply(dims, kind, coupling_sign):
    tip = gpu_binding()
    w = inputs.couplings(dims, seed=420)
    if coupling_sign < 0:
        w[0, 3] = -0.05
    mass = 2.0
    orc = OracleOp(dims, kind, mass=mass, coupling=w)
    gop = tip.Operator(dims, kind, mass=mass, coupling=to_dev(w))
    est, q, st = tip.trace_inv_probe(gop, 16, 1e-12, 7)
    est_o, q_o, _ = oracle_trace(orc, 16, 1e-12, 7, MASK_Z2)
    assert st["even_odd"] == 0
    assert _rel(est, est_o) <= REL


def test_even_odd_full_size_solution():
    """32^4 covariant workload: the solution of one probe (x = A^-1 b assembled
    from x_e and x_o) has a true FP64 residual within tol, computed here with
    the library's own operator application on the full lattice."""
    tip = gpu_binding()
    import torch
    dims = [32, 32, 32, 32]
    U = inputs.haar_links(dims)
    mf = inputs.mass_field(dims)
    gop = tip.Operator(dims, tip.KIND_COVARIANT, mass_field=to_dev(mf), links=to_dev(U))
    with tip.OpHandle(gop) as h:
        x, q, st = h.solve_probe(5, 1, 1e-10, 4018)
        assert st["even_odd"] == 1
    b = tip.tip_probe_vectors(dims, 3, tip.MASK_DEFAULT, 4018, 5, 1, 1)[0]
    bfull = torch.zeros((gop.V, 3), dtype=torch.complex128, device="cuda")
    bfull[:, 1] = b
    ax = tip.tip_apply_operator(gop, x.reshape(1, gop.V, 3))[0]
    rel = float(torch.linalg.vector_norm(bfull - ax) / torch.linalg.vector_norm(bfull))
    assert rel <= 1e-10
    assert abs(q - complex(torch.vdot(bfull.flatten(), x.flatten()))) <= 1e-12 * abs(q)


@pytest.mark.parametrize("dims,kind,n,mask", [
    ([8, 8, 8, 8], 1, 8, MASK_Z4),
    ([16, 16], 0, 32, MASK_Z2),
    ([4, 4, 4, 8], 1, 16, MASK_Z4),
])
def test_mixed_even_odd_matches_oracle(dims, kind, n, mask):
    """FP32 CG on the reduced system with FP64 reliable updates of r_e = b_hat - S x_e
    and the same FP64 acceptance: estimates at the 1e-10 bar, within the bound."""
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, kind, seed=430 + kind)
    tol = 1e-12
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=mask, precision=tip.PREC_MIXED)
    est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, mask)
    assert st["even_odd"] == 1 and st["reliable_updates"] > 0
    assert st["max_true_relres"] <= tol
    assert _rel(est, est_o) <= REL and _rel(q, q_o) <= REL
    assert np.all(np.abs(q - q_o) <= 2 * st["max_quad_err_bound"] + 1e-13 * np.abs(q_o))


def _with_env(name, value, fn):
    os.environ[name] = value
    try:
        return fn()
    finally:
        del os.environ[name]


@pytest.mark.parametrize("dims,kind,n,mask,prec", [
    ([8, 8, 8, 8], 1, 8, MASK_Z4, "fp64"),
    ([8, 8, 8, 8], 1, 8, MASK_Z4, "mixed"),
    ([16, 16], 0, 32, MASK_Z2, "fp64"),
    ([8, 4, 8], 0, 24, MASK_Z4, "mixed"),
])
def test_even_odd_restart_after_failed_true_residual(dims, kind, n, mask, prec):
    """TIP_FREEZE_SLACK = 10 freezes a solve once its recursive residual is below
    10 tol, so the FP64 true-residual check (two half-lattice passes) fails and
    CG restarts from x with r = p = the reduced residual: the estimates still
    match the oracle and the plain run, every solve meets tol, and the restarts
    are counted."""
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, kind, seed=450 + kind)
    tol = 1e-11
    precision = tip.PREC_MIXED if prec == "mixed" else tip.PREC_FP64
    print(f"even-odd restart: dims {dims} kind {kind} n {n} {prec}", flush=True)
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=mask, precision=precision)
    est_r, q_r, st_r = _with_env("TIP_FREEZE_SLACK", "10",
                                 lambda: tip.trace_inv_probe(gop, n, tol, 4018, mask=mask, precision=precision))
    est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, mask)
    assert st["even_odd"] == 1 and st_r["even_odd"] == 1
    assert st["restarts"] == 0 and st_r["restarts"] >= 1
    assert st_r["max_true_relres"] <= tol
    assert _rel(est_r, est_o) <= REL and _rel(q_r, q_o) <= REL
    assert _rel(est_r, est) <= REL


def test_even_odd_gradient_and_solution_assemble_x():
    """Only the gradient and solve_probe read x on the full lattice: with the
    half-lattice true residual both still see x_e and x_o in place."""
    tip = gpu_binding()
    import torch
    orc, gop = _ops(tip, [4, 4, 4, 8], 1, seed=460)
    with tip.OpHandle(gop) as h:
        x, qx, st = h.solve_probe(3, 2, 1e-12, 4018)
        assert st["even_odd"] == 1
        est, q, gm, gw, stg = h.trace_inv_probe_grad(4, 1e-12, 4018)
        assert stg["even_odd"] == 1
    from oracle.probing import rhs as oracle_rhs
    b = oracle_rhs(orc.dims, 3, 3, 2, 4018, MASK_Z4)
    ax = orc.apply(x.cpu().numpy().reshape(orc.V, 3))
    assert np.linalg.norm(ax - b) <= 1e-12 * np.linalg.norm(b) * 1.01
    assert np.all(gm.cpu().numpy() < 0)


@pytest.mark.parametrize("dims,n", [([16, 16, 16, 16], 16), ([8, 8, 8, 8], 12), ([8, 4, 8], 12)])
def test_mixed_two_rhs_per_thread_matches_one(dims, n):
    """In mixed precision with 32 rhs per block the covariant iteration's two
    hops load two rhs per thread (16-byte loads, 16 sites per tile).  Each rhs
    is computed as with one per thread, so against TIP_EO_PAIR=0 the
    quadratures agree to rounding and every solve meets tol; 4-D and 3-D
    lattices, several tiles."""
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, 1, seed=470)
    tol = 1e-11
    print(f"pair kernel: dims {dims} n {n}", flush=True)
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=MASK_Z4, precision=tip.PREC_MIXED, rhs_block=32)
    est_1, q_1, st_1 = _with_env("TIP_EO_PAIR", "0", lambda: tip.trace_inv_probe(
        gop, n, tol, 4018, mask=MASK_Z4, precision=tip.PREC_MIXED, rhs_block=32))
    assert st["even_odd"] == 1 and st_1["even_odd"] == 1
    assert st["max_true_relres"] <= tol and st_1["max_true_relres"] <= tol
    assert _rel(q, q_1) <= REL
    if orc.V <= 4096:
        est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, MASK_Z4)
        assert _rel(q, q_o) <= REL
    assert abs(st["total_iters"] - st_1["total_iters"]) <= 2 * st["solves"]


@pytest.mark.parametrize("dims,n,coupled", [([16, 16], 32, True), ([32, 32, 32], 32, True), ([8, 8, 8, 8], 24, False),
                                            ([8, 4, 8], 20, True)])
def test_fp64_scalar_two_rhs_per_thread_matches_one(dims, n, coupled):
    """FP64 real scalar operator, 32 rhs per block: the iteration's two hops
    load two rhs per thread (one 16-byte load per pair), couplings staged per
    tile.  Against TIP_EO_PAIR=0 the quadratures agree to rounding, and
    against the oracle to the 1e-10 bar; 2-D, 3-D and 4-D, several tiles."""
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, 0, seed=480, coupled=coupled)
    tol = 1e-12
    print(f"scalar pair kernel: dims {dims} n {n} coupled {coupled}", flush=True)
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=MASK_Z2, rhs_block=32)
    est_1, q_1, st_1 = _with_env("TIP_EO_PAIR", "0", lambda: tip.trace_inv_probe(
        gop, n, tol, 4018, mask=MASK_Z2, rhs_block=32))
    assert st["even_odd"] == 1 and st_1["even_odd"] == 1
    assert st["max_true_relres"] <= tol and st_1["max_true_relres"] <= tol
    assert _rel(q, q_1) <= REL
    assert abs(st["total_iters"] - st_1["total_iters"]) <= st["solves"]
    if orc.V <= 4096:
        est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, MASK_Z2)
        assert _rel(q, q_o) <= REL


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("dims,n", [([16, 16, 16, 16], 16), ([8, 4, 8], 12)])
def test_once_per_block_passes_in_512_threads_match_256(dims, n, prec):
    """The FP64 passes outside the iteration (reduced right-hand side, true
    residual, reliable updates) run in 256-thread workgroups by default;
    TIP_EO_WIDE_ONCE=1 puts them on 16-site tiles in 512 threads.  Each site
    is computed the same way, so the quadratures agree to rounding, in FP64
    and in the mixed solver, and both match the oracle."""
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, 1, seed=493)
    tol = 1e-12
    pr = tip.PREC_MIXED if prec == "mixed" else tip.PREC_FP64
    print(f"512-thread once-per-block passes: dims {dims} n {n} {prec}", flush=True)
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=MASK_Z4, rhs_block=32, precision=pr)
    est_1, q_1, st_1 = _with_env("TIP_EO_WIDE_ONCE", "1", lambda: tip.trace_inv_probe(
        gop, n, tol, 4018, mask=MASK_Z4, rhs_block=32, precision=pr))
    assert st["even_odd"] == 1 and st_1["even_odd"] == 1
    assert st["max_true_relres"] <= tol and st_1["max_true_relres"] <= tol
    assert _rel(q, q_1) <= REL
    if orc.V <= 4096:
        est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, MASK_Z4)
        assert _rel(q, q_o) <= REL and _rel(q_1, q_o) <= REL


@pytest.mark.parametrize("dims,n", [([16, 16, 16, 16], 16), ([8, 8, 8, 8], 12), ([8, 4, 8], 12)])
def test_fp64_covariant_512_thread_hops_match_256(dims, n):
    """FP64 covariant operator, 32 rhs per block: the iteration's two hops run
    in 512-thread workgroups (16 sites per tile, one rhs per lane).  Each site
    is computed as in the 256-thread kernel, so against TIP_EO_WIDE=0 the
    quadratures agree to rounding; 4-D and 3-D lattices, several tiles."""
    tip = gpu_binding()
    orc, gop = _ops(tip, dims, 1, seed=490)
    tol = 1e-12
    print(f"512-thread hops: dims {dims} n {n}", flush=True)
    est, q, st = tip.trace_inv_probe(gop, n, tol, 4018, mask=MASK_Z4, rhs_block=32)
    est_1, q_1, st_1 = _with_env("TIP_EO_WIDE", "0", lambda: tip.trace_inv_probe(
        gop, n, tol, 4018, mask=MASK_Z4, rhs_block=32))
    assert st["even_odd"] == 1 and st_1["even_odd"] == 1
    assert st["max_true_relres"] <= tol and st_1["max_true_relres"] <= tol
    assert _rel(q, q_1) <= REL
    assert abs(st["total_iters"] - st_1["total_iters"]) <= st["solves"]
    if orc.V <= 4096:
        est_o, q_o, _ = oracle_trace(orc, n, tol, 4018, MASK_Z4)
        assert _rel(q, q_o) <= REL


@pytest.mark.parametrize("slack", [None, "50"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind,dims", [(0, [8, 16]), (0, [8, 8, 16]), (1, [4, 4, 8]), (1, [8, 4, 4, 8])])
def test_grouped_directions_leave_nothing_outstanding(kind, dims, precision, slack, monkeypatch):
    """The block solver adds the x updates of three iterations together.  Masses
    whose iteration counts differ, so that right-hand sides stop at every place
    of a group, and restarts from an x that has to be complete; a block wider
    than its right-hand sides."""
    from oracle.general import trace_inv_probe as oracle_trace
    from oracle.mask import MASK_Z4
    from oracle.operators import Operator as OracleOp
    tip = gpu_binding()
    monkeypatch.setenv("TIP_RESIDENT", "0")
    monkeypatch.setenv("TIP_EO_GROUP", "1")                  # by itself only past the memory-side cache
    if slack:
        monkeypatch.setenv("TIP_FREEZE_SLACK", slack)
    prec = tip.PREC_MIXED if precision == "mixed" else tip.PREC_FP64
    U = inputs.haar_links(dims, seed=911) if kind else None
    iters = set()
    for m0 in (0.05, 0.2, 0.5, 1.1, 3.0):
        mf = inputs.mass_field(dims, m0=m0, seed=912)
        gop = tip.Operator(dims, kind, mass_field=to_dev(mf), links=to_dev(U))
        _, q, st = tip.trace_inv_probe(gop, 5, 1e-12, 4018, mask=MASK_Z4, precision=prec)
        _, q_o, _ = oracle_trace(OracleOp(dims, kind, mass_field=mf, links=U), 5, 1e-12, 4018, MASK_Z4)
        # a mass field with negative values (m0 = 0.05) leaves the even-odd reduction, and groups of one
        assert st["even_odd"] == (1 if mf.min() > 0 else 0) and st["stencil_launches"] > 1
        assert st["max_true_relres"] <= 1e-12
        assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= 1e-10, m0
        iters.add(st["stencil_launches"] % 3)
    assert len(iters) > 1
