"""Gauss basis on Q3 hexahedra with a node so hot that the trace of T on one face
beside it is negative: that side has no wave speed, and both elements of the face
take the other side's (the maximum goes to the plus side unless the minus side is
the larger).  The lower element's upper face, each direction, every element: faces
inside the bricks and between them."""
import numpy as np
import pytest
import torch

from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [lib.DG_FP64, lib.DG_FP32_BULK])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_both_elements_see_one_flux(axis, prec):
    c = synth.warm_rain_3d(n=(3, 3, 2), order=3, seed=151, basis="gauss")
    n0, n1, n2 = c.mesh.n
    dg = lib.for_case(c, precision=prec)
    node = 2 * 4 ** axis                     # weight -0.81 on the upper face, 0.40 on the lower
    for e in range(c.mesh.ne):
        if axis == 2 and e // (n0 * n1) == n2 - 1:
            continue                         # the lid: both sides are the trace itself
        U = torch.tensor(c.U, dtype=dg.dtype, device="cuda")
        U[-1, e, node] += 6e5
        T = dg.saturation_split(U)[0].reshape(c.mesh.ne, 64)[e].cpu().numpy()
        line = T[[k * 4 ** axis for k in range(4)]]
        x, up = np.polynomial.legendre.leggauss(4)[0], 0.0
        for i in range(4):
            up += line[i] * np.prod([(1.0 - x[k]) / (x[i] - x[k]) for k in range(4) if k != i])
        assert up < -50.0                    # (the state is what the test is about)
        R = dg.rhs(U)
        assert bool(torch.isfinite(R).all()), (axis, e)
