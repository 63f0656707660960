"""The block solvers on lattices that are solved in LDS by default.  They remain
the path of larger lattices, and their tests on small ones check them only with
the LDS solvers off: those tests again with TIP_RESIDENT=0, and every call shown
to have taken the blocks."""

import itertools

import pytest

import test_gpu_batch
import test_gpu_even_odd
import test_gpu_general
import test_gpu_graph
import test_gpu_trace
from conftest import gpu_binding

pytestmark = pytest.mark.gpu


def _cases(module, *names):
    """(test function, one set of its parameters) for all of each test's sets."""
    for name in names:
        fn = getattr(module, name)
        axes = []
        for mark in getattr(fn, "pytestmark", []):
            keys = [k.strip() for k in mark.args[0].split(",")]
            axes.append([dict(zip(keys, v if len(keys) > 1 else [v])) for v in mark.args[1]])
        for combo in itertools.product(*axes):
            kw = {k: v for part in combo for k, v in part.items()}
            yield pytest.param(fn, kw, id=name[5:] + "-" + "-".join(str(v).replace(" ", "") for v in kw.values()))


@pytest.mark.parametrize("fn,kw", [
    *_cases(test_gpu_graph, "test_graph_replays_match_eager"),
    *_cases(test_gpu_batch, "test_batch_forked_chains_equal_one_chain", "test_batch_stencil_per_dimension",
            "test_batch_equals_single_calls_and_oracle", "test_batch_mixing_kinds_masks_and_precisions",
            "test_batch_comparison_probe_kinds_against_oracle", "test_uneven_tori_batch_first_probes_against_oracle"),
    *_cases(test_gpu_even_odd, "test_even_odd_restart_after_failed_true_residual",
            "test_even_odd_matches_oracle_and_plain_cg", "test_fp64_scalar_two_rhs_per_thread_matches_one",
            "test_fp64_covariant_512_thread_hops_match_256", "test_even_odd_gradient_and_solution_assemble_x"),
    *_cases(test_gpu_general, "test_conjugate_f3_columns_reuse_their_partner", "test_gradient_on_an_odd_torus",
            "test_estimates_match_oracle"),
    *_cases(test_gpu_trace, "test_deterministic_and_resumable", "test_solve_probe_matches_dense_solve_and_trace",
            "test_non_power_of_two_vector_count_and_ragged_tiles", "test_scalar_masks_and_complex_path",
            "test_block_size_changes_only_rounding"),
])
def test_with_the_lds_solvers_off(fn, kw, monkeypatch):
    tip = gpu_binding()
    monkeypatch.setenv("TIP_RESIDENT", "0")
    calls = []

    def single(st):
        # a launch of the stencil for every iteration of a block; a whole solve in LDS is one
        assert st["stencil_launches"] >= st["max_iters"] > 1, "solved in LDS"
        calls.append(st)

    def batch(st):
        # the batch counts its blocks' launches only while it times them; those in LDS always
        assert st["stencil_launches"] == 0, "solved in LDS"
        calls.append(st)

    def spy(owner, name, stats, check):
        f = getattr(owner, name)

        def g(*a, **k):
            out = f(*a, **k)
            for st in stats(out):
                check(st)
            return out
        monkeypatch.setattr(owner, name, g)
    spy(tip, "trace_inv_probe", lambda out: [out[-1]], single)
    spy(tip, "trace_inv_probe_batch", lambda out: [st for _, st in out], batch)
    for name in ("trace_inv_probe", "trace_inv_probe_grad", "solve_probe"):
        spy(tip.OpHandle, name, lambda out: [out[-1]], single)
    kw = dict(kw)
    if "monkeypatch" in fn.__code__.co_varnames[:fn.__code__.co_argcount]:
        kw["monkeypatch"] = monkeypatch
    fn(**kw)
    assert calls
