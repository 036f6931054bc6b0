"""newton_rtol and newton_maxit choose how the split is solved: below 1e-14, and
with a cap of 8 or less, by Newton iterations alone.  Both switches lead to the
same iterations, so results under either agree bit for bit (where the cap is not
reached), cold and warm, on boxes and on triangles; and the closed form keeps
within the smallest cap that allows it."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_split_paths import _case
from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu


def _box(c, steps, **over):
    dg = lib.for_case(c, precision=lib.DG_FP64, **over)
    U = torch.tensor(c.U, device="cuda")
    T, rv, rc = dg.saturation_split(U)
    dg.rk_step(U, c.dt, steps)
    assert dg.stats()["status"] == 0
    return T, rv, rc, U


@pytest.mark.parametrize("order,dim", [(1, 2), (3, 2), (2, 3), (3, 3)])
def test_a_tolerance_below_the_closed_form_iterates(order, dim):
    c = synth.periodic_smooth(n=(5, 4, 3)[:dim], order=order, dim=dim, seed=81)
    tight = _box(c, 2, newton_rtol=5e-15, newton_maxit=30)
    capped = _box(c, 2, newton_rtol=5e-15, newton_maxit=8)
    for a, b in zip(tight, capped):
        assert torch.equal(a, b)


def test_a_tolerance_below_the_closed_form_iterates_on_triangles():
    c = synth.tri_bubble(n=(5, 3), order=3, seed=82)
    out = []
    for maxit in (30, 8):
        dg = lib.for_tri_case(c, precision=lib.DG_FP64, newton_rtol=5e-15, newton_maxit=maxit)
        C = dg.state(c.point_state)
        dg.rk_step(C, c.dt, 2)
        assert dg.stats()["status"] == 0
        out.append(C)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("T_lo,T_hi", [(140.0, 220.0), (220.0, 320.0), (320.0, 420.0)])
def test_the_closed_form_needs_no_more_than_its_cap(T_lo, T_hi):
    # nine steps: the smallest cap that allows the closed form, and too few for
    # the iterations from scratch at some of these states.  Only what the closed
    # form leaves to them (below its range, 150 K) may reach the cap.
    c = _case(11, T_lo, T_hi)
    dg = lib.for_case(c, precision=lib.DG_FP64, newton_maxit=9)
    ref = O.Oracle.for_case(c).split_field(c.U)
    T, rv, _ = (x.cpu().numpy().reshape(ref["T"].shape) for x in dg.saturation_split(torch.tensor(c.U, device="cuda")))
    st, own = dg.stats(), ref["T"] > 150.5
    assert st["nonconverged"] <= np.count_nonzero(~own) and not st["nonfinite"]
    # (the hottest states hold no cloud: no saturated solve)
    cloud = np.any(ref["rho_v"] < c.bg["rho_m"][0] + c.U[1])
    assert (2 if cloud else 0) <= st["max_iters"] <= (9 if cloud else 0)
    assert np.abs(T - ref["T"])[own].max() <= 1e-13 * ref["T"].max()
    assert np.abs(rv - ref["rho_v"])[own].max() <= 1e-13 * ref["rho_v"].max()
