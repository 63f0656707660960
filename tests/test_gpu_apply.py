"""The operator application on the caller's arrays: every count of right-hand
sides at which its split over lanes changes, and an output that overlaps the
input, against the oracle's operator."""

import numpy as np
import pytest
import torch

from conftest import gpu_binding, to_dev
from oracle.operators import Operator as OracleOp
from paper_1302_4018_amd import inputs

pytestmark = pytest.mark.gpu


def _case(tip, dims, kind, nrhs, weighted=True):
    w = inputs.couplings(dims, seed=911) if weighted else None
    mf = inputs.mass_field(dims, seed=912)
    U = inputs.haar_links(dims, seed=913) if kind == 1 else None
    orc = OracleOp(dims, kind, mass_field=mf, coupling=w, links=U)
    gop = tip.Operator(dims, kind, mass_field=to_dev(mf), coupling=to_dev(w), links=to_dev(U))
    rng = np.random.default_rng(914)
    shape = (nrhs, orc.V, 3) if kind == 1 else (nrhs, orc.V)
    x = rng.standard_normal(shape) + (1j * rng.standard_normal(shape) if kind == 1 else 0.0)
    return orc, gop, x


def _check(orc, x, y):
    # at most 2 (2 ndim + 1) products of 3 terms per component, each rounded once
    for j in range(x.shape[0]):
        want = orc.apply(x[j])
        assert np.abs(y[j] - want).max() <= 64 * 2.0 ** -53 * 16 * np.abs(x[j]).max() * 3, j


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("dims", [[5, 7, 3], [4, 4, 4, 8]])
def test_apply_every_split(kind, nrhs, dims):
    tip = gpu_binding()
    orc, gop, x = _case(tip, dims, kind, nrhs, weighted=nrhs % 2 == 1)
    _check(orc, x, tip.tip_apply_operator(gop, to_dev(x)).cpu().numpy())


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("noalloc", [False, True])
def test_apply_in_place(kind, noalloc):
    import ctypes
    tip = gpu_binding()
    orc, gop, x = _case(tip, [6, 5, 4], kind, 3)
    xd = to_dev(x)
    ptr = ctypes.c_void_p(xd.data_ptr())
    fn = tip.lib.tip_apply_operator_noalloc if noalloc else tip.lib.tip_apply_operator
    s = gop.c_struct()
    assert fn(ctypes.byref(s), 3, ptr, ptr, None) == tip.TIP_OK
    torch.cuda.synchronize()
    _check(orc, x, xd.cpu().numpy())
