"""The table of work items: a handle allocates what its launch geometry needs, not
an item per element, and smaller blocks set later find a larger one, without a
change in results or in launches that were captured before."""
import pytest
import torch

from paper_2305_13847_amd import lib, synth

pytestmark = pytest.mark.gpu


def test_handle_memory_at_q1():
    # what a handle of twice the elements takes more (fixed costs, as of its
    # streams, are the same in both)
    c = synth.periodic_smooth(n=(4, 4), order=1, seed=91)
    lib.for_case(c, precision=lib.DG_FP32_BULK).close()      # (the library and the context are loaded)
    used = []
    for n in ((2048, 1024), (4096, 1024)):
        mesh = synth.Mesh(2, list(n), c.mesh.lo, c.mesh.hi, c.mesh.bc, 1)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        dg = lib.DG(mesh, 1, c.nvars, lib.params_for_case(c, lib.DG_FP32_BULK))
        used.append(free - torch.cuda.mem_get_info()[0])
        dg.close()
    ne, nodes = 2048 * 1024, 2048 * 1024 * 4
    # six states, eight FP64 fields, three partial sums an element, the table at
    # 64 elements an item; 2 MiB of granularity for each of some 40 allocations
    need = 6 * c.nvars * nodes * 4 + 8 * nodes * 8 + 24 * ne + ne
    assert abs(used[1] - used[0] - need) <= 80 << 20


def test_smaller_blocks_later():
    c = synth.moist_bubble(n=(24, 14), order=2, seed=92)
    dg = lib.for_case(c, precision=lib.DG_FP32_BULK)
    U0 = torch.tensor(c.U, dtype=torch.float32, device="cuda")
    want = dg.rk_step(U0.clone(), c.dt, 3)
    emax = dg.get_launch()[0]
    U = U0.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dg.rk_step(U, c.dt, 3)
    for epb in (emax // 2, 1, emax, 3, 1):
        dg.set_launch(epb, 0)
        assert dg.get_launch() == (epb, 0)
        assert torch.equal(dg.rk_step(U0.clone(), c.dt, 3), want), epb
        V = U0.clone()
        assert torch.equal(dg.rk_step_graph(V, c.dt, 3), want), epb
        U.copy_(U0)
        g.replay()
        assert torch.equal(U, want), epb
