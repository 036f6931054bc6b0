"""Artificial diffusion inside the Q3 stage kernel at the edges of its bricks:
one element per axis (periodic: its own neighbour and the only element around
each vertex; walled: vertices shared by one element), odd numbers of elements in
either horizontal direction, with and without rain, alone and as members of an
ensemble.  Right-hand side, and three steps (each stage reads the viscosity that
the one before it wrote), against the FP64 reference with the tolerances of the
parity tests."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2305_13847_amd import synth

pytestmark = pytest.mark.gpu

GAM = 0.3
MESHES = [(1, 1, 1), (2, 1, 2), (1, 2, 1), (3, 3, 1), (5, 2, 3), (2, 5, 2)]


def _case(kind, n):
    if kind == "periodic":
        return synth.periodic_smooth(n=n, order=3, dim=3, seed=52)
    c = synth.warm_rain_3d(n=n, order=3, seed=51)
    rho = (c.bg["rho_d"] + c.bg["rho_m"] + c.bg["rho_r"])[synth.height_index(c.mesh)]
    c.U[2 + c.rain] += 10.0 * rho   # a mean wind: viscosity of the size the rain runs use
    return c


def _check(c, got, ref, tol, what):
    for v in range(c.nvars):
        assert np.abs(got[v] - ref[v]).max() <= tol * np.abs(ref[v]).max(), (what, v)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 1e-4)])
@pytest.mark.parametrize("kind", ["rain", "periodic"])
@pytest.mark.parametrize("n", MESHES)
def test_brick_edges_match_the_reference(kind, n, prec, tol):
    from paper_2305_13847_amd import lib
    c = _case(kind, n)
    dg = lib.for_case(c, precision=lib.DG_FP64 if prec == "fp64" else lib.DG_FP32_BULK, sip_gamma=GAM)
    U = torch.tensor(c.U, dtype=dg.dtype, device="cuda").contiguous()
    Uin = U.double().cpu().numpy()
    o = O.Oracle.for_case(c, sip_gamma=GAM)
    _check(c, dg.rhs(U).double().cpu().numpy(), o.rhs(Uin), tol, "rhs")
    ref, _ = o.rk(Uin, c.dt, 3)
    dg.rk_step(U, c.dt, 3)
    _check(c, U.double().cpu().numpy(), ref, tol, "steps")
    assert dg.stats()["status"] == 0


def test_members_of_odd_sizes_match_single_runs():
    from paper_2305_13847_amd import lib
    cases = [_case("rain", n) for n in ((3, 2, 2), (2, 3, 3), (1, 1, 2), (4, 5, 1))]
    dg = lib.for_ensemble(cases, precision=lib.DG_FP64, sip_gamma=GAM)
    U = torch.cat([torch.tensor(c.U).reshape(c.nvars, -1) for c in cases], dim=1).contiguous().cuda()
    U = U.reshape(dg.shape)
    dg.rk_step(U, np.array([c.dt for c in cases]), 3)
    Uh = U.cpu().numpy().reshape(cases[0].nvars, -1)
    off = 0
    for c in cases:
        m = c.mesh.ne * c.mesh.npe
        ref, _ = O.Oracle.for_case(c, sip_gamma=GAM).rk(c.U, c.dt, 3)
        _check(c, Uh[:, off:off + m].reshape(c.U.shape), ref, 1e-11, c.mesh.n)
        off += m
