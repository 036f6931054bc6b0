"""Rain in two dimensions, every order, on odd sizes: right-hand side, three steps,
and in FP64 the transposed derivative, against the FP64 reference (tolerances of
the parity and adjoint tests)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu


def _case(order):
    c = synth.moist_bubble(n=(9, 5), order=order, seed=131)
    X = synth.node_coords(c.mesh)
    rr = 2e-4 + 1e-3 * np.exp(-((X[0] - 9e3) ** 2 + (X[1] - 3e3) ** 2) / 4e6)
    c.U = np.concatenate([c.U[:2], rr[None], c.U[2:]])
    rho = (c.bg["rho_d"] + c.bg["rho_m"])[synth.height_index(c.mesh)]
    c.U[3] += 3.0 * rho                     # a wind, off the kink of |u|
    c.U[4] += 1.0 * rho
    c.nvars, c.rain, c.vr_const = 6, 1, 5.0
    return c


def _check(c, got, ref, tol, what):
    for v in range(c.nvars):
        assert np.abs(got[v] - ref[v]).max() <= tol * np.abs(ref[v]).max(), (what, v)


@pytest.mark.parametrize("prec,tol", [(lib.DG_FP64, 1e-11), (lib.DG_FP32_BULK, 1e-4)])
@pytest.mark.parametrize("order", [1, 2, 3, 4, 5, 6, 7])
def test_rain_2d_matches_the_reference(order, prec, tol):
    c = _case(order)
    dg = lib.for_case(c, precision=prec)
    U = torch.tensor(c.U, dtype=dg.dtype, device="cuda")
    Uin = U.double().cpu().numpy()
    o = O.Oracle.for_case(c)
    _check(c, dg.rhs(U).double().cpu().numpy(), o.rhs(Uin), tol, "rhs")
    if prec == lib.DG_FP64:
        rng = np.random.default_rng(132)
        V = rng.standard_normal(U.shape) * np.array([1e-4, 1e-5, 1e-6, 1e-2, 1e-2, 10.0])[:, None, None]
        W = rng.standard_normal(U.shape)
        bar = dg.rhs_vjp(U, torch.tensor(W, device="cuda")).cpu().numpy()
        assert np.sum(bar * V) == pytest.approx(np.sum(o.rhs_jvp(Uin, V)[1] * W), rel=1e-10)
    dg.rk_step(U, c.dt, 3)
    ref, _ = o.rk(Uin, c.dt, 3)
    _check(c, U.double().cpu().numpy(), ref, tol, "steps")
