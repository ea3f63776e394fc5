"""The automatic variant on both sides of its lines (two-stage bricks, single-stage bricks, per-stage marches,
fused marches by tile): steps, kept stages and the adjoint, bit for bit those of the one-thread-per-cell kernel."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, grid, walls: two-stage bricks end at one per compute unit (256: 64 x 64 x 16 in 8x8x4), ...
    ("f32", (64, 64, 16), ""), ("f32", (64, 64, 17), ""), ("f64", (64, 64, 17), ""),
    # ... single-stage bricks at 12 in FP64 (3072: 128 x 128 x 96), at 15 with walls (3840: 128 x 120 x 128)
    ("f64", (128, 128, 96), ""), ("f64", (129, 128, 96), ""), ("f64", (128, 120, 128), "xz"), ("f32", (128, 120, 129), "xz"),
    # FP32 marches choose their tile above 108^3 cells, walled ones run fused from 144^3
    ("f32", (108, 108, 108), ""), ("f32", (108, 108, 109), ""), ("f32", (151, 173, 129), ""), ("f32", (250, 100, 75), ""),
    ("f32", (136, 141, 139), "xz"), ("f32", (144, 144, 144), "y"), ("f64", (128, 128, 128), ""),
]


@pytest.mark.parametrize("dtype,shape,walls", CASES)
def test_automatic_variant_matches_the_plain_kernel(dtype, shape, walls):
    import paper_1803_01262_amd as pf
    kd, td = (pf.PF_F32, torch.float32) if dtype == "f32" else (pf.PF_F64, torch.float64)
    nm = [pf.phasefield_variant_name(kd, v) for v in range(pf.phasefield_variant_count(kd))]
    nx, ny, nz = shape
    dx = 1.0 / max(shape)

    def fields(seed):
        rng = np.random.default_rng(seed)
        return [torch.tensor(rng.uniform(lo, hi, (nz, ny, nx)), dtype=td, device="cuda")
                for lo, hi in ((0.0, 1.0), (-0.5, 0.5), (-0.5, 0.5), (-0.5, 0.5))]

    res = []
    for variant in (nm.index("global"), -1):
        out = []
        for scheme in ("rk4", "rk2"):
            print("case", dtype, shape, walls, scheme, variant, flush=True)
            s = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, dtype=dtype, scheme=scheme, delta=1.0, variant=variant,
                          walls=tuple(a in walls for a in "xyz"))
            phi, *vel = fields(23)
            s.step(phi, *vel, nsteps=3)
            out.append(phi.clone())
            for nxt in (torch.empty_like(phi), None):
                ys = [torch.empty_like(phi) for _ in range(s.stage_count)]
                out += [s.step_stages(phi.clone(), *vel, 0.1, *ys, phi_next=nxt), *ys]
            lam = fields(24)[0]
            g = fields(25)[1:]
            s.adjoint_step(phi, *vel, 0.1, lam, *g)
            torch.cuda.synchronize()
            s.close()
            out += [lam, *g]
        res.append(out)
    for k, (a, b) in enumerate(zip(*res)):
        assert torch.equal(a, b), k
