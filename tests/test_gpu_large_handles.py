"""FP32 handles of 2^29 nodes and more, whose FP64 arrays (T, rho_vs; 8 bytes per
node) pass 4 GiB.  The state is a small one repeated along the periodic axes, so
every result is the small handle's, bit for bit (the arithmetic of an element
does not depend on where it lies)."""
import dataclasses
import math

import pytest
import torch

from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu

SMALL = {
    "2d-q4": lambda: synth.moist_bubble(n=(16, 24), order=4, seed=51),
    "2d-q2": lambda: synth.moist_bubble(n=(16, 64), order=2, seed=52),
    "3d-q3": lambda: synth.warm_rain_3d(n=(4, 4, 2), order=3, seed=53),
    "3d-q2": lambda: synth.warm_rain_3d(n=(4, 4, 2), order=2, seed=54),
    "2d-q3-gauss": lambda: synth.moist_bubble(n=(16, 48), order=3, seed=55, basis="gauss"),
}


def _large(c, nodes):
    """The case c repeated along x (and y) to at least `nodes` nodes, without its
    state: (case, repeats per horizontal axis)."""
    d = c.mesh.dim
    need = nodes / (c.mesh.ne * c.mesh.npe)
    rep = [int(need) + 1] if d == 2 else [int(math.sqrt(need)) + 1] * 2
    n, hi = list(c.mesh.n), list(c.mesh.hi)
    for a, r in enumerate(rep):
        n[a] *= r
        hi[a] *= r
    return dataclasses.replace(c, mesh=dataclasses.replace(c.mesh, n=n, hi=hi)), rep


def _tiles(x, c, rep):
    """x of the repeated case as (variable, z, [y repeat, y,] x repeat, x, node)."""
    n = c.mesh.n
    mid = [rep[0], n[0]] if c.mesh.dim == 2 else [rep[1], n[1], rep[0], n[0]]
    return x.view(c.nvars, n[-1], *mid, c.mesh.npe)


def _repeat(x, c, big, rep):
    one = _tiles(x, c, [1] * len(rep))
    out = torch.empty((c.nvars, big.mesh.ne, c.mesh.npe), dtype=x.dtype, device=x.device)
    _tiles(out, c, rep).copy_(one.expand(_tiles(out, c, rep).shape))
    return out


def _same(got, want, c, rep):
    g, w = _tiles(got, c, rep), _tiles(want, c, [1] * len(rep))
    for v in range(c.nvars):
        assert bool((g[v] == w[v]).all()), (c.name, v)


def _handles(name, nodes=1 << 29, states=10):
    c = SMALL[name]()
    big, rep = _large(c, nodes)
    n = big.mesh.ne * big.mesh.npe
    assert nodes <= n < (1 << 30)
    torch.cuda.empty_cache()
    need = n * (states * c.nvars * 4 + 10 * 8) + (8 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %d GiB of free GPU memory" % (need >> 30))
    print(name, big.mesh.n, c.digest(), flush=True)
    return c, big, rep, lib.for_case(c, precision=lib.DG_FP32_BULK), lib.for_case(big, precision=lib.DG_FP32_BULK)


@pytest.mark.parametrize("name", ["2d-q4", "3d-q3"])
def test_rhs_vjp(name):
    c, big, rep, ds, db = _handles(name)
    U = torch.tensor(c.U, dtype=torch.float32, device="cuda")
    lam = torch.randn(U.shape, generator=torch.Generator().manual_seed(5)).cuda()
    want = ds.rhs_vjp(U, lam)
    got = db.rhs_vjp(_repeat(U, c, big, rep), _repeat(lam, c, big, rep))
    _same(got, want, c, rep)


@pytest.mark.parametrize("name", ["2d-q2", "2d-q4", "3d-q2", "3d-q3", "2d-q3-gauss"])
def test_rhs_and_step(name):
    c, big, rep, ds, db = _handles(name, states=14 if "gauss" in name else 9)
    U = torch.tensor(c.U, dtype=torch.float32, device="cuda")
    X = _repeat(U, c, big, rep)
    R = torch.empty_like(X)
    _same(db.rhs(X, out=R), ds.rhs(U), c, rep)
    db.rk_step(X, c.dt, 1)
    ds.rk_step(U, c.dt, 1)
    _same(X, U, c, rep)
