"""The autotuner on Q3 hexahedra, whose stage kernels take bricks whatever the block
width and the persistent grid are: it leaves both alone (the split, the adjoint and
the diagnostics run with them) and chooses among the item orders."""
import pytest
import torch

from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("basis", ["lobatto", "gauss"])
@pytest.mark.parametrize("persist", [0, 1])
def test_only_the_item_order_is_tuned(basis, persist):
    c = synth.warm_rain_3d(n=(7, 6, 5), order=3, seed=121, basis=basis)
    for epb in (1, 3, 4):
        dg = lib.for_case(c, precision=lib.DG_FP32_BULK)
        dg.set_launch(epb, persist)
        U = torch.tensor(c.U, dtype=torch.float32, device="cuda")
        U0 = U.clone()
        rec = dg.autotune(U, c.dt, nsteps=2)
        assert torch.equal(U, U0)
        assert (rec["elems_per_block"], rec["persist_per_cu"]) == (epb, persist) == dg.get_launch()
        assert rec["item_order"] == dg.get_item_order() and rec["item_order"] in (0, 1, 2, 3)
        assert rec["ms_per_step"] > 0
