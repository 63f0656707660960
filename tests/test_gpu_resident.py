"""The solvers that keep a system in LDS (one workgroup per even-odd system, a
cluster of workgroups per whole lattice) at the edges of their row counts,
against the oracle: systems of 2 rows to the largest, whole lattices just below
and above each change of shape, real and complex right-hand sides, with and
without couplings, clusters of 1 to 32 workgroups."""

import numpy as np
import pytest

from conftest import gpu_binding, to_dev
from oracle.general import trace_inv_probe as oracle_trace
from oracle.mask import MASK_Z2, MASK_Z4
from oracle.operators import Operator as OracleOp
from paper_1302_4018_amd import inputs

pytestmark = pytest.mark.gpu

REL = 1e-10      # both sides solve to 1e-12; a quadrature's error is second order in the residual


@pytest.mark.parametrize("dims", [
    # even-odd systems: V / 2 = 2, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384 rows
    [2, 2], [4, 8], [4, 4, 4], [8, 16], [16, 16], [8, 8, 8], [32, 32], [8, 4, 8, 8], [16, 16, 16], [32, 16, 16],
    [8, 8, 16, 16], [32, 32, 32],
    # whole lattices: 15, 256, 264, 1023, 1056, 2025, 2052, 4096, 4097, 8190, 8448, 20000 rows
    [3, 5], [16, 16, 1], [11, 24], [31, 33], [32, 33], [45, 45], [19, 12, 9], [64, 64, 1], [17, 241], [90, 91],
    [4, 8, 8, 33], [20, 40, 25],
])
@pytest.mark.parametrize("mask,weighted", [(MASK_Z2, True), (MASK_Z4, False)])
def test_resident_matches_oracle(dims, mask, weighted):
    tip = gpu_binding()
    w = inputs.couplings(dims, seed=900) if weighted else None
    mf = inputs.mass_field(dims, m0=0.4, seed=901)
    orc = OracleOp(dims, 0, mass_field=mf, coupling=w)
    gop = tip.Operator(dims, 0, mass_field=to_dev(mf), coupling=to_dev(w))
    n = min(orc.V, 5)
    est, q, st = tip.trace_inv_probe(gop, n, 1e-12, 4018, mask=mask)
    est_o, q_o, _ = oracle_trace(orc, n, 1e-12, 4018, mask)
    assert st["stencil_launches"] == 1, "not solved in LDS"
    assert st["max_true_relres"] <= 1e-12
    assert np.max(np.abs(est - est_o) / np.abs(est_o)) <= REL
    assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= REL


@pytest.mark.parametrize("dims", [
    # clusters of 2, 2, 3, 6 and 8 workgroups at the least, cut along each dimension in turn
    [3, 59, 113], [150, 9, 16], [30, 47, 31], [9, 101, 101], [48, 48, 48],
    # and lattices that fewer would hold, split over idle CUs
    [7, 11, 100], [12000, 1], [6, 5, 90, 3],
])
@pytest.mark.parametrize("n,weighted", [(1, True), (4, False)])
def test_cluster_matches_oracle(dims, n, weighted):
    tip = gpu_binding()
    w = inputs.couplings(dims, seed=902) if weighted else None
    mf = inputs.mass_field(dims, m0=0.5, seed=903)
    orc = OracleOp(dims, 0, mass_field=mf, coupling=w)
    gop = tip.Operator(dims, 0, mass_field=to_dev(mf), coupling=to_dev(w))
    est, q, st = tip.trace_inv_probe(gop, n, 1e-12, 4018, mask=MASK_Z2)
    est_o, q_o, _ = oracle_trace(orc, n, 1e-12, 4018, MASK_Z2)
    assert st["stencil_launches"] == 1 and st["max_true_relres"] <= 1e-12
    assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= REL
    assert np.array_equal(tip.trace_inv_probe(gop, n, 1e-12, 4018, mask=MASK_Z2)[1], q), "not reproducible"


@pytest.mark.parametrize("dims,launches", [
    # even-odd systems of 2, 8, 32, 64, 128, 256, 512, 1024 and 2048 rows, then one past the limit
    ([2, 2], 1), ([2, 2, 2, 2], 1), ([8, 8], 1), ([4, 4, 8], 1), ([4, 4, 4, 4], 1), ([8, 8, 8], 1), ([4, 8, 8, 4], 1),
    ([32, 64], 1), ([8, 8, 8, 8], 1), ([16, 16, 32], 2),
])
@pytest.mark.parametrize("weighted", [True, False])
def test_resident_covariant_matches_oracle(dims, launches, weighted):
    tip = gpu_binding()
    w = inputs.couplings(dims, seed=905) if weighted else None
    mf = inputs.mass_field(dims, m0=0.3, seed=906)
    U = inputs.haar_links(dims, seed=907)
    orc = OracleOp(dims, 1, mass_field=mf, coupling=w, links=U)
    gop = tip.Operator(dims, 1, mass_field=to_dev(mf), coupling=to_dev(w), links=to_dev(U))
    n = 3
    est, q, st = tip.trace_inv_probe(gop, n, 1e-12, 4018, mask=MASK_Z4)
    est_o, q_o, _ = oracle_trace(orc, n, 1e-12, 4018, MASK_Z4)
    assert (st["stencil_launches"] == 1) == (launches == 1) and st["even_odd"] == 1
    assert st["max_true_relres"] <= 1e-12
    assert np.max(np.abs(est - est_o) / np.abs(est_o)) <= REL
    assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= REL


def test_lattice_past_every_limit_uses_the_block_solver():
    tip = gpu_binding()
    dims = [83, 84, 85]                                      # three planes of 6972 sites do not fit one CU
    gop = tip.Operator(dims, 0, mass=2.0)
    _, q, st = tip.trace_inv_probe(gop, 1, 1e-12, 4018)
    _, q_o, _ = oracle_trace(OracleOp(dims, 0, mass=2.0), 1, 1e-12, 4018, MASK_Z2)
    assert st["stencil_launches"] > 1
    assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= REL


def test_batch_teams_take_several_packets_of_mixed_cluster_sizes():
    """Launches with more packets than teams (64 teams of 4 workgroups, 8 of 32),
    packets of one, two, four and eight workgroups per system behind one another,
    full and partly filled, at 15360 rows and just past them."""
    tip = gpu_binding()
    shapes = ([([48, 48, 48], 1)] * 7 + [([48, 48, 48], 5), ([40, 50, 45], 2)]        # 8 workgroups a system
              + [([30, 47, 31], 3), ([16, 30, 32], 3), ([16, 31, 31], 3)]             # 4, 1 and 2
              + [([4 + k % 3, 5, 6 + k % 7], 1 + k % 6) for k in range(66)])
    ops = [dict(mass=0.4 + 0.002 * k) for k in range(len(shapes))]
    ns = [n for _, n in shapes]
    gops = [tip.Operator(d, 0, **o) for (d, _), o in zip(shapes, ops)]
    out = tip.trace_inv_probe_batch(gops, ns, 1e-12, 4018, mask=MASK_Z2)
    again = tip.trace_inv_probe_batch(gops, ns, 1e-12, 4018, mask=MASK_Z2)
    for k, ((dims, n), (_, st)) in enumerate(zip(shapes, out)):
        assert st["max_true_relres"] <= 1e-12, (dims, n)
        q, q2 = (np.asarray(s["quadratures"]) for s in (st, again[k][1]))
        assert np.array_equal(q, q2), (dims, n, "not reproducible")
        if 1 <= k <= 6:                                      # a large lattice of the same shape as the first
            q_o = tip.trace_inv_probe(gops[k], n, 1e-12, 4018, mask=MASK_Z2)[1]
        else:
            q_o = oracle_trace(OracleOp(dims, 0, **ops[k]), n, 1e-12, 4018, MASK_Z2)[1]
        assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= REL, (dims, n)
