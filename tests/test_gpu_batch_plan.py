"""Batches by the plan that creation chooses (no set_shape): column tiles of one instance split over several
XCDs, the fall-back of very long lists, FP64 batches above and below the fused line, walls in one instance.
Every instance's bits are those of its own single solve."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

PLANS = {
    # 4 M cells and more: FP64 runs fused; 50 column tiles and more in a chunk against 32 slots of an XCD
    "split_f64": ("f64", [(160, 160, 160), (40, 36, 70), (33, 17, 9)], None),
    "walls_f64": ("f64", [(160, 160, 160), (40, 36, 70), (33, 17, 9)], 1),
    # 162 column tiles against 64 slots
    "split_f32": ("f32", [(288, 288, 20), (31, 50, 130), (16, 16, 16)], None),
    # more than 20000 tiles: 64 planes without a search
    "long_list": ("f32", [(3232, 3232, 1), (20, 20, 70)], None),
    # FP64 of 4 M cells in planes, thin slabs and small grids stays per stage
    "planes_f64": ("f64", [(512, 512, 1)] * 17, None),
    "slabs_f64": ("f64", [(300, 180, 8)] * 10, None),
}


@pytest.mark.parametrize("plan", PLANS)
def test_batch_plan_matches_single_solves(plan):
    import paper_1803_01262_amd as pf
    dtype, shapes, walled = PLANS[plan]
    td = torch.float32 if dtype == "f32" else torch.float64
    dx = 1.0 / 64

    def walls(b):
        return (b == walled, False, b == walled)

    torch.manual_seed(7)
    groups = []
    for nx, ny, nz in shapes:
        f = [torch.rand((nz, ny, nx), dtype=td, device="cuda") for _ in range(4)]
        for t in f[1:]:
            t.sub_(0.5)
        groups.append(f)
    phis = [g[0].clone() for g in groups]
    batch = pf.BatchSolver([pf.make_params(s, dx, 0.8 * dx, 1.0, 0.1 * dx, dtype=dtype, walls=walls(b))
                            for b, s in enumerate(shapes)])
    print("batch", plan, flush=True)
    batch.step(phis, *[[g[k] for g in groups] for k in (1, 2, 3)], nsteps=3)
    torch.cuda.synchronize()
    batch.close()
    for b, (s, g) in enumerate(zip(shapes, groups)):
        one = pf.Solver(s, dx, 0.8 * dx, 1.0, 0.1 * dx, dtype=dtype, walls=walls(b))
        one.step(*g, nsteps=3)
        torch.cuda.synchronize()
        one.close()
        assert torch.equal(phis[b], g[0]), (plan, s)
