"""What calls keep when their lattices are solved in LDS: results complete when
a call returns, the same failures reported, the same arithmetic for a
right-hand side whichever run it belongs to, the same arrays allowed."""

import numpy as np
import pytest
import torch

from conftest import gpu_binding, to_dev
from oracle.mask import MASK_Z2, MASK_Z4
from oracle.operators import Operator as OracleOp
from oracle.general import rhs, trace_inv_probe as oracle_trace
from paper_1302_4018_amd import inputs

pytestmark = pytest.mark.gpu

# even-odd system, scalar and covariant; whole lattice on one CU and on several
LDS = [([16, 16, 16], 0), ([4, 4, 4, 8], 1), ([9, 7, 15], 0), ([30, 47, 31], 0)]


def _op(tip, dims, kind, seed, m0=0.3):
    w = inputs.couplings(dims, seed=seed)
    mf = inputs.mass_field(dims, m0=m0, seed=seed + 1)
    U = inputs.haar_links(dims, seed=seed + 2) if kind else None
    return (OracleOp(dims, kind, mass_field=mf, coupling=w, links=U),
            tip.Operator(dims, kind, mass_field=to_dev(mf), coupling=to_dev(w), links=to_dev(U)))


@pytest.mark.parametrize("dims,kind", LDS)
@pytest.mark.parametrize("own", [True, False])
def test_solve_probe_has_written_x_when_it_returns(dims, kind, own):
    """On a caller's stream nothing is left queued; on the null stream, where the
    library works on a stream of its own, x is read at once on another stream,
    and the handle may go.  A second call needs more workspace than the first."""
    tip = gpu_binding()
    orc, gop = _op(tip, dims, kind, 920)
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with tip.OpHandle(gop) as h:
        x, q, st = h.solve_probe(3, 0, 1e-11, 17, mask=MASK_Z4, stream=stream if own else None)
        if own:
            assert stream.query(), "work left on the caller's stream"
        with torch.cuda.stream(other):
            xg = x.cpu().numpy()
        assert st["stencil_launches"] == 1, "not solved in LDS"
        h.trace_inv_probe(min(orc.V, 16), 1e-6, 17, mask=MASK_Z4, stream=stream if own else None)
    again = x.cpu().numpy()
    assert np.array_equal(xg, again)
    b = rhs(orc.dims, orc.ncomp, 3, 0, 17, MASK_Z4)
    r = b - orc.apply(xg)
    assert np.linalg.norm(r) <= 2e-11 * np.linalg.norm(b)
    assert abs(q - np.vdot(b, xg)) <= 1e-12 * abs(q)


@pytest.mark.parametrize("dims,kind,resident", [([16, 16], 0, "1"), ([9, 7, 15], 0, "1"), ([8, 8, 8], 0, "0")])
def test_gradient_of_a_failed_run_leaves_nothing_queued(dims, kind, resident, monkeypatch):
    tip = gpu_binding()
    monkeypatch.setenv("TIP_RESIDENT", resident)
    _, gop = _op(tip, dims, kind, 930)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with tip.OpHandle(gop) as h:
        with pytest.raises(tip.TipError) as e:
            h.trace_inv_probe_grad(70, 1e-12, 17, max_iter=2, stream=stream)
        assert e.value.status == tip.TIP_ENOCONV
        assert stream.query(), "work left on the caller's stream"


@pytest.mark.parametrize("dims,kind,n", [([9, 7, 15], 0, 945), ([12, 5, 8], 0, 480),
                                         # one, four and eight waves a system
                                         ([16, 16], 0, 256), ([8, 16, 16], 0, 1500), ([16, 16, 16], 0, 800),
                                         ([4, 4, 4, 8], 1, 200), ([8, 8, 8, 8], 1, 160)])
@pytest.mark.parametrize("broken", [False, True])
def test_failure_is_the_first_in_probe_order(dims, kind, n, broken, monkeypatch):
    """More systems than run at once, stopped at an iteration that most finish
    before: the probe named, the status, the checkpoints and the residuals up to
    it follow from the iterations of each probe by itself, whatever class of the
    three-colouring it is of."""
    tip = gpu_binding()
    late_ones = 0
    for seed in (940, 941, 942, 943):
        _, gop = _op(tip, dims, kind, seed, m0=0.5)
        with tip.OpHandle(gop) as h:
            _, q, _ = h.trace_inv_probe(n, 1e-10, 4018, mask=MASK_Z2)
            iters = [h.trace_inv_probe(m + 1, 1e-10, 4018, mask=MASK_Z2, m_begin=m, quadratures=q)[2]["max_iters"]
                     for m in range(n)]
            # the stops whose first failure comes latest, and latest among the probes solved in real arithmetic
            first = {v: next(m for m in range(n) if iters[m] > v) for v in set(iters) if 0 < v < max(iters)}
            late = sorted(first, key=first.get)[-2:]
            real = sorted((v for v in first if first[v] % 3 == 0), key=first.get)[-1:]
            for stop in set(late + real):
                bad, kw = first[stop], {}
                if broken:
                    monkeypatch.setenv("TIP_FORCE_BREAKDOWN", str(stop + 1))
                else:
                    kw = {"max_iter": stop}
                est, _, st = h.trace_inv_probe(n, 1e-10, 4018, mask=MASK_Z2, raise_on_error=False, **kw)
                monkeypatch.delenv("TIP_FORCE_BREAKDOWN", raising=False)
                print(f"{dims} seed {seed} stop {stop} broken {broken}: probe {bad} of {n}", flush=True)
                assert st["status"] == (tip.TIP_EBREAKDOWN if broken else tip.TIP_ENOCONV)
                assert f"probe {bad} " in tip.tip_last_error()
                assert len(est) == bad.bit_length()                # checkpoints 1, 2, 4, .. up to bad probes
                assert not np.isnan(st["residuals"][:bad]).any() and np.isnan(st["residuals"][bad]).any()
                late_ones += bad >= 16
    assert late_ones or not any(d % 3 == 0 for d in dims)      # lattices with two classes have late ones


@pytest.mark.parametrize("kind,nrhs", [(0, 1), (0, 5), (1, 1), (1, 5)])
@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("array", ["mass_field", "coupling", "links"])
def test_output_may_overlap_the_operators_arrays(array, noalloc, kind, nrhs):
    """y lies over the beginning of one of them, which the call reads as it was.
    Without allocation a later vector sees a mass field or couplings that earlier
    results have overwritten, so there one vector."""
    import ctypes
    tip = gpu_binding()
    if array == "links" and kind == 0:
        pytest.skip("no links")
    if noalloc and array != "links":
        nrhs = 1
    orc, gop = _op(tip, [7, 6, 10], kind, 950)
    src = getattr(gop, array)
    rng = np.random.default_rng(951)
    shape = (nrhs, orc.V, 3) if kind else (nrhs, orc.V)
    x = rng.standard_normal(shape) + (1j * rng.standard_normal(shape) if kind else 0.0)
    xd = to_dev(x)
    flat = src.reshape(-1) if not src.is_complex() else torch.view_as_real(src).reshape(-1)
    n = x.size * (2 if kind else 1)
    mem = torch.zeros(max(n, flat.numel()), dtype=torch.float64, device="cuda")
    mem[:flat.numel()] = flat
    s = gop.c_struct()
    setattr(s, array, mem.data_ptr())
    fn = tip.lib.tip_apply_operator_noalloc if noalloc else tip.lib.tip_apply_operator
    torch.cuda.synchronize()
    assert fn(ctypes.byref(s), nrhs, ctypes.c_void_p(xd.data_ptr()), ctypes.c_void_p(mem.data_ptr()), None) == tip.TIP_OK
    y = mem[:n].cpu().numpy()
    y = (y.view(np.complex128) if kind else y).reshape(shape)
    for j in range(nrhs):
        want = orc.apply(x[j])
        # at most 2 (2 ndim + 1) products of 3 terms per component, each rounded once
        assert np.abs(y[j] - want).max() <= 64 * 2.0 ** -53 * 16 * np.abs(x[j]).max() * 3, j


def test_a_long_solve_in_a_batch_outlasts_no_wait(monkeypatch):
    """Clusters without a system wait for the whole solve of their team's others,
    here many times the limit that a single exchange has; the solve runs to
    max_iter and is reported as such, the other problems are whole."""
    tip = gpu_binding()
    dims = [9, 7, 15]
    rng = np.random.default_rng(960)
    w = 10.0 ** rng.uniform(-6, 6, size=(3, 945))
    hard = tip.Operator(dims, 0, mass=1e-9, coupling=to_dev(w))
    orc, easy = _op(tip, [7, 6, 11], 0, 961)
    ns = [2, 1, 6]
    tip.trace_inv_probe_batch([easy] * 3, ns, 1e-11, 4018, mask=MASK_Z2)                   # the kernel is on the device
    monkeypatch.setenv("TIP_CLUSTER_POLLS", "2048")
    out = tip.trace_inv_probe_batch([easy, hard, easy], ns, 1e-11, 4018, mask=MASK_Z2, max_iter=4000,
                                    raise_on_error=False)
    assert [st["status"] for _, st in out] == [tip.TIP_OK, tip.TIP_ENOCONV, tip.TIP_OK], tip.tip_last_error()
    assert out[1][1]["max_iters"] == 4000
    for k in (0, 2):
        q_o = oracle_trace(orc, ns[k], 1e-11, 4018, MASK_Z2)[1]
        assert np.max(np.abs(out[k][1]["quadratures"] - q_o) / np.abs(q_o)) <= 1e-10


@pytest.mark.parametrize("dims,mask", [([30, 47, 31], MASK_Z4), ([30, 47, 31], MASK_Z2)])
def test_clusters_that_cannot_run_together_leave_the_call_to_the_block_solver(dims, mask, monkeypatch):
    """A limit of one poll stands for CUs that something else holds: every kind of
    call is answered all the same."""
    tip = gpu_binding()
    orc, gop = _op(tip, dims, 0, 970, m0=0.6)
    n = 4
    _, q_o, _ = oracle_trace(orc, n, 1e-11, 4018, mask)
    with tip.OpHandle(gop) as h:
        _, q0, st0 = h.trace_inv_probe(n, 1e-11, 4018, mask=mask)
        _, _, gm0, gw0, _ = h.trace_inv_probe_grad(n, 1e-11, 4018, mask=mask)
        assert st0["stencil_launches"] == 1
        monkeypatch.setenv("TIP_CLUSTER_POLLS", "1")
        _, q, st = h.trace_inv_probe(n, 1e-11, 4018, mask=mask)
        _, _, gm, gw, _ = h.trace_inv_probe_grad(n, 1e-11, 4018, mask=mask)
        x, qx, stx = h.solve_probe(0, 0, 1e-11, 4018, mask=mask)
    assert st["stencil_launches"] > 1 and stx["stencil_launches"] > 1
    assert st["solves"] == st0["solves"] and st["status"] == tip.TIP_OK
    assert np.max(np.abs(q - q_o) / np.abs(q_o)) <= 1e-10
    assert abs(qx - q_o[0]) <= 1e-10 * abs(q_o[0])
    # two solutions of residual 1e-11 differ by at most 2e-11 sqrt(V) / min m, their squares by twice that times |x|
    lam = float(gop.mass_field.min())
    bound = 4 * (4e-11 * np.sqrt(orc.V) / lam) * np.sqrt(float(gm0.abs().max())) + 1e-20
    assert float((gm - gm0).abs().max()) <= bound and float((gw - gw0).abs().max()) <= 4 * bound
    # the batch's block solver counts its launches only while it times them: none in LDS
    out = tip.trace_inv_probe_batch([gop, gop], [n, 2], 1e-11, 4018, mask=mask)
    for (_, s), k in zip(out, (n, 2)):
        assert s["status"] == tip.TIP_OK and s["stencil_launches"] == 0
        assert np.max(np.abs(s["quadratures"] - q_o[:k]) / np.abs(q_o[:k])) <= 1e-10


@pytest.mark.parametrize("dims,n", [([21, 34, 15], 80), ([12000, 1], 60), ([12, 48, 48], 20)])
def test_arithmetic_of_a_right_hand_side_does_not_depend_on_its_run(dims, n):
    """A whole run, a resumed one and single solves of a lattice that more CUs
    would take when few systems are solved: the same quadratures bit for bit."""
    tip = gpu_binding()
    _, gop = _op(tip, dims, 0, 980, m0=0.5)
    with tip.OpHandle(gop) as h:
        _, q, st = h.trace_inv_probe(n, 1e-10, 4018, mask=MASK_Z4)
        assert st["stencil_launches"] == 1, "not solved in LDS"
        _, half, _ = h.trace_inv_probe(n // 2, 1e-10, 4018, mask=MASK_Z4)
        _, rest, _ = h.trace_inv_probe(n, 1e-10, 4018, mask=MASK_Z4, m_begin=n // 2, quadratures=half)
        assert np.array_equal(half, q[:n // 2]) and np.array_equal(rest, q)
        for m in (0, 1, n - 1):
            assert h.solve_probe(m, 0, 1e-10, 4018, mask=MASK_Z4)[1] == q[m], m


@pytest.mark.parametrize("resident", ["1", "0"])
def test_mixed_batch_restarts_where_fp64_breaks_down(resident, monkeypatch):
    """p^H A p <= 0 in a mixed batch, forced at iteration 3 and on an indefinite
    operator: a restart from the FP64 residual, and TIP_ENOCONV when the budget of
    restarts is spent; in FP64 a breakdown.  In LDS as in blocks."""
    tip = gpu_binding()
    monkeypatch.setenv("TIP_RESIDENT", resident)
    orc, gop = _op(tip, [7, 6, 11], 0, 990)
    neg = tip.Operator([9, 5, 6], 0, mass=-20.0)

    def run(precision):
        return tip.trace_inv_probe_batch([gop, neg], [6, 3], 1e-11, 4018, mask=MASK_Z2, precision=precision,
                                         raise_on_error=False)
    assert [s["status"] for _, s in run(tip.PREC_FP64)] == [tip.TIP_OK, tip.TIP_EBREAKDOWN]
    assert [s["status"] for _, s in run(tip.PREC_MIXED)] == [tip.TIP_OK, tip.TIP_ENOCONV]
    if resident == "0":
        return                                               # the batch's blocks have no forced breakdown
    monkeypatch.setenv("TIP_FORCE_BREAKDOWN", "3")
    assert [s["status"] for _, s in run(tip.PREC_FP64)] == [tip.TIP_EBREAKDOWN] * 2
    st = run(tip.PREC_MIXED)[0][1]
    assert st["status"] == tip.TIP_OK and st["restarts"] >= st["solves"] and st["max_true_relres"] <= 1e-11
    q_o = oracle_trace(orc, 6, 1e-11, 4018, MASK_Z2)[1]
    assert np.max(np.abs(st["quadratures"] - q_o) / np.abs(q_o)) <= 1e-10


@pytest.mark.parametrize("dims,kind,mixed", [([16, 16, 16], 0, False), ([4, 4, 4, 8], 1, False), ([9, 7, 15], 0, False),
                                             ([16, 16, 16], 0, True)])
def test_autotuning_does_not_leave_the_lds_solvers(dims, kind, mixed, tmp_path):
    """The fixed launch shapes it times are the block solver's, so what no shape
    fixes is among what it chooses from."""
    tip = gpu_binding()
    from paper_1302_4018_amd import autotune
    _, gop = _op(tip, dims, kind, 1000)
    prec = tip.PREC_MIXED if mixed else tip.PREC_FP64
    with tip.OpHandle(gop) as h:
        best, tried = h.autotune(1e-10, 4018, sample_vectors=16, precision=prec)
        assert sorted({t["rhs_block"] for t in tried}) == [16, 32, 64]
        assert best["seconds_per_solve"] <= min(t["seconds_per_solve"] for t in tried)
        if mixed:
            assert best in tried
            return
        assert best["rhs_block"] == best["round_tiles"] == 0
        kw = autotune.tuned(h, 1e-10, 4018, sample_vectors=16, path=str(tmp_path / "tune.json"))
        assert h.trace_inv_probe(16, 1e-10, 4018, **kw)[2]["stencil_launches"] == 1
        fixed, tried = h.autotune(1e-10, 4018, sample_vectors=16, rhs_block=16)
        assert fixed["rhs_block"] == 16 and fixed in tried


def test_batch_autotuning_of_lds_problems_is_not_noise():
    tip = gpu_binding()
    ops = [_op(tip, d, 0, 1010)[1] for d in ([9, 7, 15], [8, 8, 8])]
    best, tried = tip.tip_autotune_batch(ops, [8, 8], 1e-10, 4018, sample_vectors=8)
    assert len(tried) == 12 and len({t["seconds_per_solve"] for t in tried}) == 1
    assert (best["rhs_block"], best["item_sites"]) == (32, 512)


def test_gradient_keeps_a_bounded_number_of_solutions():
    """4096 probes of 32^3: 1 GiB of solutions if all were kept.  The sums over
    probes against the block solver's, which keeps one block."""
    tip = gpu_binding()
    _, gop = _op(tip, [32, 32, 32], 0, 1020)
    n, tol = 4096, 1e-10
    with tip.OpHandle(gop) as h:
        h.trace_inv_probe(4, tol, 4018)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        _, _, gm, gw, st = h.trace_inv_probe_grad(n, tol, 4018)
        used = before - torch.cuda.mem_get_info()[0]
        assert st["stencil_launches"] < 64, "not solved in LDS"
        assert used <= 512 << 20, used
        _, _, gm_b, gw_b, _ = h.trace_inv_probe_grad(n, tol, 4018, rhs_block=64)
    lam = float(gop.mass_field.min())
    from conftest import assert_gradient_entries
    assert_gradient_entries(gm.cpu().numpy(), gw.cpu().numpy(), gm_b.cpu().numpy(), gw_b.cpu().numpy(), tol, gop.V, lam)


def test_kept_memory_is_bounded_and_given_back():
    """Ten handles of some 77 MB each leave at most 512 MiB behind, which goes when it
    is asked for; 2000 small ones leave what they left, and calls go on."""
    tip = gpu_binding()
    U = inputs.haar_links([16, 16, 16, 16], seed=1030)
    big = tip.Operator([16, 16, 16, 16], 1, mass=0.5, links=to_dev(U))
    orc, small = _op(tip, [5, 3], 0, 1031)
    free = lambda: torch.cuda.mem_get_info()[0]
    tip.OpHandle(small).close()
    tip.tip_release_memory()
    before = free()
    hs = [tip.OpHandle(big) for _ in range(10)]
    for h in hs:
        h.close()
    assert 256 << 20 <= before - free() <= (512 << 20) + (8 << 20)
    q = None
    for _ in range(20):
        hs = [tip.OpHandle(small) for _ in range(100)]
        q = hs[-1].trace_inv_probe(4, 1e-11, 7, mask=MASK_Z2)[1]
        for h in hs:
            h.close()
    tip.tip_release_memory()
    assert before - free() <= 8 << 20
    assert np.max(np.abs(q - oracle_trace(orc, 4, 1e-11, 7, MASK_Z2)[1]) / np.abs(q)) <= 1e-10
    assert np.array_equal(tip.trace_inv_probe(small, 4, 1e-11, 7, mask=MASK_Z2)[1], q)


def test_time_of_a_batch_grows_with_its_problems_not_their_square():
    tip = gpu_binding()
    ops = [tip.Operator([5, 3, 4], 0, mass=0.5 + 0.0001 * k) for k in range(4000)]

    def seconds(n):
        return min(tip.trace_inv_probe_batch(ops[:n], [60] * n, 1e-10, 7)[0][1]["seconds"] for _ in range(4))
    seconds(4000)
    few, many = seconds(1000), seconds(4000)
    assert many <= 6.5 * few, (few, many)      # 4 when linear; the scan over all systems for each problem made it 9.4


def test_host_threads_share_kernels_and_kept_memory():
    """Threads with streams of their own, in lattices of different sizes for the
    same kernels, handles made and destroyed all along: every result is what the
    call alone gives, bit for bit."""
    import threading
    tip = gpu_binding()
    cases = [([48, 48, 48], 0), ([9, 7, 15], 0), ([16, 16, 16], 0), ([4, 4, 4, 8], 1)]
    ops = [_op(tip, d, k, 1040 + i)[1] for i, (d, k) in enumerate(cases)]

    def call(i, stream):
        with tip.OpHandle(ops[i], stream=stream) as h:
            q = h.trace_inv_probe(3, 1e-10, 7, mask=MASK_Z4, stream=stream)[1]
            x = h.solve_probe(1, 0, 1e-10, 7, mask=MASK_Z4, stream=stream)[0].cpu().numpy()
            # the block solver, which captures graphs
            m = h.trace_inv_probe(2, 1e-10, 7, mask=MASK_Z4, stream=stream, precision=tip.PREC_MIXED)[1]
        b = [s["quadratures"] for _, s in tip.trace_inv_probe_batch([ops[1], ops[0]][:1 + i % 2], [4, 2][:1 + i % 2],
                                                                    1e-10, 7, mask=MASK_Z2, stream=stream)]
        return q, x, m, *b
    want = [call(i, None) for i in range(len(cases))]
    wrong = []

    def work(t):
        stream = torch.cuda.Stream()
        try:
            for r in range(8):
                i = (t + r) % len(cases)
                if not all(np.array_equal(g, w) for g, w in zip(call(i, stream), want[i])):
                    wrong.append((t, r, cases[i]))
        except Exception as e:                                   # noqa: BLE001
            wrong.append((t, repr(e)))
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


def test_default_limit_of_iterations(monkeypatch):
    """10 V ncomp, as in blocks, for a covariant operator on which CG gets nowhere."""
    tip = gpu_binding()
    dims = [4, 4]
    w = 10.0 ** np.random.default_rng(1060).uniform(-9, 9, size=(2, 16))
    gop = tip.Operator(dims, 1, mass=1e-14, coupling=to_dev(w), links=to_dev(inputs.haar_links(dims, seed=1061)))
    runs = []
    for resident in ("1", "0"):
        monkeypatch.setenv("TIP_RESIDENT", resident)
        runs.append(tip.trace_inv_probe(gop, 1, 1e-14, 7, raise_on_error=False)[2])
    assert [st["status"] for st in runs] == [tip.TIP_ENOCONV] * 2
    assert [st["max_iters"] for st in runs] == [10 * gop.V * gop.ncomp] * 2


@pytest.mark.parametrize("dims,n,m0", [([32, 32, 32], 16500, 16300), ([27, 32, 64], 55296, 48000)])
def test_runs_longer_than_a_launch(dims, n, m0):
    """More than 16384 right-hand sides, of one class and of each of two."""
    tip = gpu_binding()
    _, gop = _op(tip, dims, 0, 1070, m0=2.0)
    with tip.OpHandle(gop) as h:
        _, q, st = h.trace_inv_probe(n, 1e-9, 4018, mask=MASK_Z2)
        _, tail, st2 = h.trace_inv_probe(n, 1e-9, 4018, mask=MASK_Z2, m_begin=m0, quadratures=q)
        _, some, _ = h.trace_inv_probe(300, 1e-9, 4018, mask=MASK_Z2)
    assert st["stencil_launches"] > 1 and st["status"] == tip.TIP_OK and st["solves"] + st["reused"] == n
    assert np.max(np.abs(tail - q) / np.abs(q)) <= 1e-12 and np.max(np.abs(some - q[:300]) / np.abs(some)) <= 1e-12


@pytest.mark.parametrize("dims", [[9, 7, 5], [6, 10]])
def test_solve_probe_refuses_complex_probes_in_real_arithmetic(dims, monkeypatch):
    """With a real mask x is real; the probes of the three-colouring's other columns
    are not.  Refused in blocks, so in LDS: not the solution of their real part."""
    tip = gpu_binding()
    _, gop = _op(tip, dims, 0, 1080)
    runs = []
    for resident in ("1", "0"):
        monkeypatch.setenv("TIP_RESIDENT", resident)
        with tip.OpHandle(gop) as h:
            _, q, _ = h.trace_inv_probe(24, 1e-11, 4018, mask=MASK_Z2)
            run = []
            for m in range(24):
                try:
                    qm = h.solve_probe(m, 0, 1e-11, 4018, mask=MASK_Z2)[1]
                    assert abs(qm - q[m]) <= 1e-10 * abs(q[m]), m
                    run.append(True)
                except tip.TipError as e:
                    assert e.status == tip.TIP_ENOCONV
                    run.append(False)
        runs.append(run)
    assert runs[0] == runs[1] and True in runs[0] and False in runs[0]


@pytest.mark.parametrize("seed", range(6))
def test_lds_and_block_solvers_agree_over_what_both_take(seed, monkeypatch):
    """Sides of 1 to 16 in two to four dimensions, every kind of probe and mask, with
    and without fields, negative couplings, resumed runs: status, counts and
    quadratures of the two routes.  Each solution's residual is at most 1e-12 of
    ||b||, so a quadrature's relative error at most 1e-12 times the condition number,
    which stays below 500 here (masses of 0.2 and more, weights up to 1.5)."""
    import random
    tip = gpu_binding()
    rng = random.Random(seed)
    for k in range(20):
        kind = rng.choice([0, 0, 0, 1])
        pow2 = rng.random() < 0.5
        while True:
            dims = [rng.choice([1, 2, 4, 8, 16]) if pow2 else rng.randint(1, 13) for _ in range(rng.choice([2, 3, 4]))]
            V = int(np.prod(dims))
            if 4 <= V <= (1024 if kind else 4096):
                break
        kinds = [tip.PROBE_HIERARCHICAL] * 3 + [tip.PROBE_RANDOM]
        if all(d & (d - 1) == 0 for d in dims):
            kinds += [tip.PROBE_NATURAL, tip.PROBE_STOPPED, tip.PROBE_FOURIER]
        probe = rng.choice(kinds)
        mask = rng.choice([1, 2] if probe == tip.PROBE_RANDOM else [0, 1, 2])
        n = min(V, rng.choice([1, 2, 5, 17, 40]))
        begin = rng.randint(0, n - 1) if rng.random() < 0.3 else 0
        negative = rng.random() < 0.25
        w = inputs.couplings(dims, seed=k) if negative or rng.random() < 0.6 else None
        if negative:
            w = w * np.where(np.random.default_rng(k).random(w.shape) < 0.1, -0.1, 1.0)
        U = inputs.haar_links(dims, seed=k) if kind else None
        gop = tip.Operator(dims, kind, mass=3.0 if negative else rng.choice([0.2, 1.0]), coupling=to_dev(w), links=to_dev(U),
                           mass_field=to_dev(inputs.mass_field(dims, m0=3.0 if negative else 0.5, seed=k))
                           if rng.random() < 0.5 else None)
        kw = dict(mask=mask, probe=probe, stop_levels=rng.randint(0, 4) if probe == tip.PROBE_STOPPED else 0)
        print(f"case {seed}.{k}: {dims} kind {kind} {kw} n {n} begin {begin} negative {negative}", flush=True)
        runs = []
        for resident in ("1", "0"):
            monkeypatch.setenv("TIP_RESIDENT", resident)
            with tip.OpHandle(gop) as h:
                first = h.trace_inv_probe(begin, 1e-12, 7, **kw)[1] if begin else None
                runs.append(h.trace_inv_probe(n, 1e-12, 7, m_begin=begin, quadratures=first, **kw))
        (est, q, st), (est_b, q_b, st_b) = runs
        assert all(st[f] == st_b[f] for f in ("status", "solves", "reused", "n_checkpoints_done"))
        assert st["max_true_relres"] <= 1e-12
        if kind == 0 or (not negative and all(d > 1 and d & (d - 1) == 0 for d in dims)):
            assert st["stencil_launches"] == 1, "not solved in LDS"
        assert np.max(np.abs(q - q_b) / np.abs(q_b)) <= 1e-9 and np.max(np.abs(est - est_b) / np.abs(est_b)) <= 1e-9
        assert np.array_equal(np.isnan(st["residuals"]), np.isnan(st_b["residuals"]))
