"""The split without iterations (series about one point of the saturation
curve) against the FP64 reference: temperatures over its whole range, states
at and on both sides of the branch point, iteration caps on both sides of the
one that switches it off, and steps whose temperature changes lie inside and
outside the series' range."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2305_13847_amd import synth

pytestmark = pytest.mark.gpu


def _case(seed, T_lo, T_hi, order=3, n=(5, 4)):
    """Random states at rest in a periodic box: T and the ratio of rho_m to the
    saturation density drawn per node, a third of the nodes within 1e-12 ...
    1e-3 of saturation."""
    rng = np.random.default_rng(seed)
    c = synth.periodic_smooth(n=n, order=order, seed=seed)
    shape = c.U.shape[1:]
    T = rng.uniform(T_lo, T_hi, shape)
    rvs = synth.paper_rho_vs(T)
    ratio = 10.0 ** rng.uniform(-1.0, 0.5, shape)
    near = rng.random(shape) < 0.33
    ratio = np.where(near, 1.0 + rng.choice([-1.0, 1.0], shape) * 10.0 ** rng.uniform(-12.0, -3.0, shape), ratio)
    rd = rng.uniform(0.3, 1.2, shape)
    rm = np.minimum(ratio * rvs, 0.05)
    rv = np.minimum(rm, rvs)
    E = synth.energy(rd, rv, rm - rv, 0.0, T)
    c.U = np.stack([rd - c.bg["rho_d"][0], rm - c.bg["rho_m"][0], 0.0 * T, 0.0 * T, E - c.bg["E"][0]])
    return c


@pytest.mark.parametrize("T_lo,T_hi", [(140.0, 220.0), (220.0, 320.0), (320.0, 420.0)])
@pytest.mark.parametrize("maxit", [8, 9, 30])
def test_split_over_temperatures_and_near_the_branch_point(T_lo, T_hi, maxit):
    from paper_2305_13847_amd import lib
    c = _case(11, T_lo, T_hi)
    dg = lib.for_case(c, precision=lib.DG_FP64, newton_maxit=maxit)
    ref = O.Oracle.for_case(c).split_field(c.U)
    U = torch.tensor(c.U, device="cuda").contiguous()
    T, rv, rc = (x.cpu().numpy().reshape(ref["T"].shape) for x in dg.saturation_split(U))
    if maxit < 30 and dg.stats()["status"] == lib.DG_ENOCONV:
        pytest.skip("the general path does not converge under this cap")
    # the tolerance of the split's parity tests: 1e-13 of the field's maximum
    assert np.abs(T - ref["T"]).max() <= 1e-13 * ref["T"].max()
    assert np.abs(rv - ref["rho_v"]).max() <= 1e-13 * ref["rho_v"].max()
    assert dg.stats()["status"] == 0


@pytest.mark.parametrize("factor", [1e-3, 1.0, 20.0])
def test_warm_steps_inside_and_outside_the_series_range(factor):
    # factor 20 (CFL 4, two steps): the stages change T by kelvins, beyond the series
    from paper_2305_13847_amd import lib
    c = synth.periodic_smooth(n=(6, 5), order=3, seed=12)
    dg = lib.for_case(c, precision=lib.DG_FP64)
    U = torch.tensor(c.U, device="cuda").contiguous()
    steps = 2 if factor > 1 else 10
    dg.rk_step(U, factor * c.dt, steps)
    ref, _ = O.Oracle.for_case(c).rk(c.U, factor * c.dt, steps)
    got = U.cpu().numpy()
    for v in range(c.nvars):
        assert np.linalg.norm(got[v] - ref[v]) <= 1e-11 * np.linalg.norm(ref[v]), v
