"""Fused sweeps on rows that are no whole number of 16-byte pieces, on tiles at and across the row's end, in
single grids and batches: the bits of the one-thread-per-cell kernel."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# every remainder of a piece, rows shorter than one piece, than a tile, of one tile and of two
ROWS = [1, 2, 3, 5, 6, 7, 29, 31, 33, 34, 35, 37, 63, 65, 66, 67, 131]


@pytest.fixture(scope="module")
def pf():
    assert torch.cuda.is_available()
    import paper_1803_01262_amd
    return paper_1803_01262_amd


def fields(shape, dtype, seed=5):
    rng = np.random.default_rng(seed)
    td = torch.float32 if dtype == "f32" else torch.float64
    nx, ny, nz = shape
    return [torch.tensor(rng.uniform(lo, hi, (nz, ny, nx)), dtype=td, device="cuda")
            for lo, hi in ((0.0, 1.0), (-0.5, 0.5), (-0.5, 0.5), (-0.5, 0.5))]


def names(pf, dtype):
    kd = pf.PF_F32 if dtype == "f32" else pf.PF_F64
    return [pf.phasefield_variant_name(kd, v) for v in range(pf.phasefield_variant_count(kd))]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx", ROWS)
def test_straddling_rows_match_the_plain_kernel(pf, nx, dtype):
    nm = names(pf, dtype)
    shape, dx = (nx, 17, 9), 1.0 / 32
    out = {}
    for v in ["global"] + [k for k in nm if k.startswith("fused_") and "x" in k and "brick" not in k]:
        for scheme in ("rk4", "rk2"):
            g = fields(shape, dtype)
            print("case", shape, dtype, v, scheme, flush=True)
            s = pf.Solver(shape, dx, 0.8 * dx, 1.0, 0.1 * dx, dtype=dtype, variant=nm.index(v), scheme=scheme)
            s.step(*g, t0=0.1, nsteps=3)
            torch.cuda.synchronize()
            s.close()
            ref = out.setdefault(scheme, g[0])
            assert torch.equal(g[0], ref), (v, scheme)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_batches_of_straddling_rows_match_single_solves(pf, dtype):
    shapes = [(nx, 19, 11 + 37 * (k % 4)) for k, nx in enumerate(ROWS)]  # one z-chunk and several
    dx = 1.0 / 32
    groups = [fields(s, dtype, seed=20 + k) for k, s in enumerate(shapes)]
    nm = names(pf, dtype)
    want = []
    for s, g in zip(shapes, groups):
        ref = g[0].clone()
        solver = pf.Solver(s, dx, 0.8 * dx, 1.0, 0.1 * dx, dtype=dtype, variant=nm.index("global"))
        solver.step(ref, *g[1:], nsteps=2)
        torch.cuda.synchronize()
        solver.close()
        want.append(ref)
    for shape in ("fused_32x16", "fused_64x8"):
        phis = [g[0].clone() for g in groups]
        b = pf.BatchSolver([pf.make_params(s, dx, 0.8 * dx, 1.0, 0.1 * dx, dtype=dtype) for s in shapes])
        b.set_shape(shape)
        print("batch", dtype, shape, flush=True)
        b.step(phis, [g[1] for g in groups], [g[2] for g in groups], [g[3] for g in groups], nsteps=2)
        torch.cuda.synchronize()
        b.close()
        for k, (got, ref) in enumerate(zip(phis, want)):
            assert torch.equal(got, ref), (shape, shapes[k])
