"""Right-hand side and one step on meshes at the edges of the work split: one or
two elements per axis (an element that is its own neighbour), rows shorter than
a block, a last block with one element, walls on both sides of one element, and
orders whose face tasks take one pass of a block or two.  Against the FP64
reference with the tolerances of the parity tests."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2305_13847_amd import synth

pytestmark = pytest.mark.gpu

MESHES = [(2, order, n) for order in (1, 2, 3, 4, 5, 7) for n in ((1, 1), (2, 1), (3, 7), (17, 2), (1, 9))]
MESHES += [(3, order, n) for order in (1, 2, 3, 4) for n in ((1, 1, 1), (2, 1, 2), (3, 3, 1), (5, 2, 3))]


def _case(dim, order, n):
    return synth.moist_bubble(n=n, order=order, seed=31) if dim == 2 else synth.warm_rain_3d(n=n, order=order, seed=32)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 1e-4)])
@pytest.mark.parametrize("dim,order,n", MESHES)
def test_small_meshes_match_the_reference(dim, order, n, prec, tol):
    from paper_2305_13847_amd import lib
    c = _case(dim, order, n)
    dg = lib.for_case(c, precision=lib.DG_FP64 if prec == "fp64" else lib.DG_FP32_BULK)
    U = torch.tensor(c.U, dtype=dg.dtype, device="cuda").contiguous()
    Uin = U.double().cpu().numpy()
    o = O.Oracle.for_case(c)
    ref = o.rhs(Uin)
    got = dg.rhs(U).double().cpu().numpy()
    ref1, _ = o.rk(Uin, c.dt, 1)
    dg.rk_step(U, c.dt, 1)
    got1 = U.double().cpu().numpy()
    for v in range(c.nvars):
        assert np.abs(got[v] - ref[v]).max() <= tol * np.abs(ref[v]).max(), ("rhs", v)
        assert np.abs(got1[v] - ref1[v]).max() <= tol * np.abs(ref1[v]).max(), ("step", v)
    assert dg.stats()["status"] == 0
