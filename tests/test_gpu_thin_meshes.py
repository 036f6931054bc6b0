"""Q3 hexahedra on columns and slabs: meshes of one element along x, along y, or
both, whose bricks are one element wide there, and an ensemble of such members with
a wider one, whose bricks are not.  Right-hand side and three steps against the
FP64 reference (tolerances of the parity tests), plain, in the Gauss basis and with
the artificial diffusion."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu

KINDS = {"plain": ("lobatto", {}), "gauss": ("gauss", {}), "diffusion": ("lobatto", dict(sip_gamma=0.6))}


def _case(n, basis, walls):
    c = synth.warm_rain_3d(n=n, order=3, seed=101, basis=basis)
    if walls:
        c = dataclasses.replace(c, mesh=dataclasses.replace(c.mesh, bc=[synth.WALL] * 3))
    return c


def _check(c, got, ref, tol, what):
    for v in range(c.nvars):
        assert np.abs(got[v] - ref[v]).max() <= tol * np.abs(ref[v]).max(), (what, v)


@pytest.mark.parametrize("prec,tol", [(lib.DG_FP64, 1e-11), (lib.DG_FP32_BULK, 1e-4)])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n", [(1, 1, 1), (1, 1, 5), (2, 1, 3), (5, 1, 2), (1, 2, 3), (1, 5, 2)])
def test_columns_and_slabs(n, kind, walls, prec, tol):
    basis, over = KINDS[kind]
    c = _case(n, basis, walls)
    dg = lib.for_case(c, precision=prec, **over)
    U = torch.tensor(c.U, dtype=dg.dtype, device="cuda")
    Uin = U.double().cpu().numpy()
    o = O.Oracle.for_case(c, **over)
    _check(c, dg.rhs(U).double().cpu().numpy(), o.rhs(Uin), tol, "rhs")
    dg.rk_step(U, c.dt, 3)
    ref, _ = o.rk(Uin, c.dt, 3)
    _check(c, U.double().cpu().numpy(), ref, tol, "steps")


@pytest.mark.parametrize("kind", list(KINDS))
def test_ensemble_of_thin_and_wide_members(kind):
    basis, over = KINDS[kind]
    cases = [_case(n, basis, False) for n in ((1, 1, 4), (3, 1, 2), (1, 2, 2), (3, 2, 2))]
    dg = lib.for_ensemble(cases, precision=lib.DG_FP64, **over)
    U = torch.cat([torch.tensor(c.U).reshape(c.nvars, -1) for c in cases], dim=1).contiguous().cuda().reshape(dg.shape)
    dg.rk_step(U, np.array([c.dt for c in cases]), 2)
    got, off = U.reshape(cases[0].nvars, -1).cpu().numpy(), 0
    for c in cases:
        n = c.mesh.ne * c.mesh.npe
        ref, _ = O.Oracle.for_case(c, **over).rk(c.U, c.dt, 2)
        _check(c, got[:, off:off + n].reshape(c.U.shape), ref, 1e-11, c.mesh.n)
        off += n
