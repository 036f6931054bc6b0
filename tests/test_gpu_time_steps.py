"""The time steps of a call belong to that call: queued calls keep theirs whatever
is called next, and a launch captured by the caller keeps those it was captured
with.  `_sleep` holds the stream back so that every call is queued before the
first one runs."""
import numpy as np
import pytest
import torch

from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu

FACTORS = (1.0, 0.25, 0.6)


def _setup(members):
    cases = synth.ensemble(nmembers=members, order=2, seed=61, lo=2, hi=5)
    dg = lib.for_ensemble(cases, precision=lib.DG_FP64)
    U = torch.cat([torch.tensor(c.U).reshape(c.nvars, -1) for c in cases], dim=1).contiguous().cuda().reshape(dg.shape)
    return dg, U, np.array([c.dt for c in cases])


def _synchronised(dg, U0, dt, factors):
    U = U0.clone()
    for f in factors:
        dg.rk_step(U, dt * f, 1)
        torch.cuda.synchronize()
    return U


# 600 members: more than one launch takes as arguments
@pytest.mark.parametrize("members", [1, 3, 300, 600])
@pytest.mark.parametrize("graph", [False, True])
def test_queued_calls_keep_their_time_steps(members, graph):
    dg, U0, dt = _setup(members)
    want = _synchronised(dg, U0, dt, FACTORS)
    U = U0.clone()
    step = dg.rk_step_graph if graph else dg.rk_step
    step(U, dt, 1)                       # (the library's graph is captured here)
    U.copy_(U0)
    torch.cuda.synchronize()
    torch.cuda._sleep(200_000_000)
    for f in FACTORS:
        step(U, dt * f, 1)
    torch.cuda.synchronize()
    assert torch.equal(U, want)


@pytest.mark.parametrize("members", [1, 3, 300, 600])
def test_a_captured_call_keeps_its_time_steps(members):
    dg, U0, dt = _setup(members)
    want = _synchronised(dg, U0, dt, (0.5,))
    U, V = U0.clone(), U0.clone()
    dg.rk_step(U, dt, 1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dg.rk_step(U, dt * 0.5, 1)
    for f in FACTORS:
        V.copy_(U0)
        dg.rk_step(V, dt * f, 1)         # eager calls between the replays, other time steps
        torch.cuda.synchronize()
        U.copy_(U0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(U, want), f
