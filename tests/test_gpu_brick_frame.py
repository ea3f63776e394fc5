"""The frame that the single-stage bricks share (pf_brick.h): bricks whose halo stays inside the plane and
bricks at its edges, the shortest axes of the one-period form and the longest of the general one, walls on
any axis. Every bit is the one-thread-per-cell kernel's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# 18 x 10 x 6 is the smallest grid of the one-period form (bricks of 16 x 8 x 4 with a halo of two); three
# bricks along x and y leave one whose halo stays inside the plane
SHAPES = [(18, 10, 6), (17, 10, 6), (18, 9, 6), (18, 10, 5), (48, 24, 12), (50, 26, 13), (67, 33, 9), (515, 11, 7)]


@pytest.fixture(scope="module")
def pf():
    assert torch.cuda.is_available()
    import paper_1803_01262_amd
    return paper_1803_01262_amd


def fields(shape, dtype, seed):
    rng = np.random.default_rng(seed)
    td = torch.float32 if dtype == "f32" else torch.float64
    nx, ny, nz = shape
    return [torch.tensor(rng.uniform(lo, hi, (nz, ny, nx)), dtype=td, device="cuda")
            for lo, hi in ((0.0, 1.0), (-0.5, 0.5), (-0.5, 0.5), (-0.5, 0.5))]


@pytest.mark.parametrize("walls", [(False, False, False), (True, False, True), (False, True, False), (True, True, True)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_stages_and_reverse_stages_match_the_plain_kernels(pf, dtype, walls):
    kd = pf.PF_F32 if dtype == "f32" else pf.PF_F64
    nm = [pf.phasefield_variant_name(kd, v) for v in range(pf.phasefield_variant_count(kd))]
    for shape in SHAPES:
        dx = 1.0 / max(shape)
        for scheme in ("rk4", "rk3", "rk2", "euler"):
            res = {}
            # the automatic variant's reverse stages run on bricks, the named one's stages
            for variant in ("global", "tiled_brick16x8x4", None):
                print("case", shape, dtype, walls, scheme, variant, flush=True)
                s = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, dtype=dtype, scheme=scheme, walls=walls, delta=1.0,
                              variant=-1 if variant is None else nm.index(variant))
                phi, *vel = fields(shape, dtype, 17)
                s.step(phi, *vel, nsteps=2)
                lam = fields(shape, dtype, 18)[0]
                g = fields(shape, dtype, 19)[1:]
                s.adjoint_step(phi, *vel, 0.1, lam, *g)
                torch.cuda.synchronize()
                s.close()
                res[variant] = [phi, lam, *g]
            for variant, got in res.items():
                for k, (a, b) in enumerate(zip(got, res["global"])):
                    assert torch.equal(a, b), (shape, scheme, variant, k)
