"""Gauss basis on Q3 hexahedra in handles whose trace buffers outgrow 32-bit byte
offsets (96 FP64 values an element; 4 GiB): they take the block kernels.  A small
state repeated along x and y, right-hand side and two steps: every repeat has the
same bits, and they match the FP64 reference of the small state (tolerances of the
parity tests)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2305_13847_amd import lib, synth
from test_gpu_large_handles import _large, _repeat, _tiles

pytestmark = pytest.mark.gpu

ELEMENTS = (1 << 32) // (96 * 8) + 1


def _first_tile(x, c, rep):
    """The first repeat, after a check that all are its copies."""
    t = _tiles(x, c, rep)
    one = t[:, :, :1, :, :1]
    for v in range(c.nvars):
        assert bool((t[v] == one[v]).all()), (c.name, v)
    return one.reshape(c.U.shape).double().cpu().numpy()


def _check(c, got, ref, tol, what):
    for v in range(c.nvars):
        assert np.abs(got[v] - ref[v]).max() <= tol * np.abs(ref[v]).max(), (what, v)


@pytest.mark.parametrize("kind,prec,tol", [("rain", lib.DG_FP32_BULK, 1e-4), ("periodic", lib.DG_FP64, 1e-11)])
def test_block_kernels_of_large_handles(kind, prec, tol):
    c = (synth.warm_rain_3d(n=(4, 4, 2), order=3, seed=141, basis="gauss") if kind == "rain" else
         synth.periodic_smooth(n=(4, 4, 2), order=3, dim=3, seed=142, basis="gauss"))
    big, rep = _large(c, ELEMENTS * 64)
    ne, size = big.mesh.ne, 4 if prec == lib.DG_FP32_BULK else 8
    assert ne >= ELEMENTS and ne * 64 < (1 << 29)
    torch.cuda.empty_cache()
    need = ne * (64 * (8 * c.nvars * size + 8 * 8) + 96 * (2 * c.nvars * size + 4 * 8)) + (4 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %d GiB of free GPU memory" % (need >> 30))
    print(kind, big.mesh.n, c.digest(), flush=True)
    dg = lib.for_case(big, precision=prec)
    U = torch.tensor(c.U, dtype=dg.dtype, device="cuda")
    Uin = U.double().cpu().numpy()
    o = O.Oracle.for_case(c)
    X = _repeat(U, c, big, rep)
    R = torch.empty_like(X)
    _check(c, _first_tile(dg.rhs(X, out=R), c, rep), o.rhs(Uin), tol, "rhs")
    dg.rk_step(X, c.dt, 2)
    ref, _ = o.rk(Uin, c.dt, 2)
    _check(c, _first_tile(X, c, rep), ref, tol, "steps")
    dg.close()
