"""Brick and whole-step forms of small grids (stage_brick.hip, stage_brick1.hip, stage_plane.hip, adjoint_brick.hip): bit-identical to
the one-thread-per-cell kernel at the edges of their bricks, patches and halos, on every
boundary, and in every place a handle with the automatic variant takes them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 8), (9, 7, 5), (16, 8, 4), (12, 12, 12), (11, 13, 17), (20, 28, 12), (1, 3, 2), (2, 1, 9)]
PLANES = [(16, 16), (17, 15), (24, 20), (32, 32), (33, 31), (5, 70), (1, 40), (2, 3)]
WALLS = [(False, False, False), (True, True, True), (True, False, False), (False, True, False),
         (False, False, True)]


@pytest.fixture(scope="module")
def pf():
    assert torch.cuda.is_available()
    import paper_1803_01262_amd
    return paper_1803_01262_amd


def fields(shape, dtype, seed=11):
    rng = np.random.default_rng(seed)
    td = torch.float32 if dtype == "f32" else torch.float64
    nx, ny, nz = shape
    phi = rng.uniform(0.0, 1.0, (nz, ny, nx))
    vel = [rng.uniform(-0.5, 0.5, phi.shape) for _ in range(3)]
    return [torch.tensor(a, dtype=td, device="cuda") for a in (phi, *vel)]


def names(pf, dtype):
    kd = pf.PF_F32 if dtype == "f32" else pf.PF_F64
    return [pf.phasefield_variant_name(kd, v) for v in range(pf.phasefield_variant_count(kd))]


def stepped(pf, shape, dtype, variant, nsteps, **kw):
    g = fields(shape, dtype)
    dx = 1.0 / max(shape)
    s = pf.Solver(shape, dx, 0.8 * dx, 1.0, 0.1 * dx, dtype=dtype, variant=variant, **kw)
    print("case", shape, dtype, variant, kw, flush=True)
    s.step(*g, t0=0.1, nsteps=nsteps)
    torch.cuda.synchronize()
    s.close()
    return g[0]


@pytest.mark.parametrize("walls", WALLS)
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_bricks_match_the_plain_kernel(pf, dtype, walls):
    nm = names(pf, dtype)
    for shape in SHAPES:
        for scheme, nsteps in (("rk4", 3), ("rk3", 1), ("rk2", 2), ("euler", 2)):
            kw = dict(scheme=scheme, walls=walls, vel_mode=1, vel_T=0.7)
            ref = stepped(pf, shape, dtype, nm.index("global"), nsteps, **kw)
            for v in [k for k in nm if "brick" in k] + [None]:
                got = stepped(pf, shape, dtype, -1 if v is None else nm.index(v), nsteps, **kw)
                assert torch.equal(got, ref), (shape, scheme, v)


@pytest.mark.parametrize("walls", WALLS)
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_plane_step_matches_the_plain_kernel(pf, dtype, walls):
    nm = names(pf, dtype)
    for nx, ny in PLANES:
        for scheme, nsteps in (("rk4", 3), ("rk3", 2), ("rk2", 3), ("euler", 2)):
            kw = dict(scheme=scheme, walls=walls, vel_mode=1, vel_T=0.7)
            ref = stepped(pf, (nx, ny, 1), dtype, nm.index("global"), nsteps, **kw)
            for v in (nm.index("fused_plane"), -1):
                assert torch.equal(stepped(pf, (nx, ny, 1), dtype, v, nsteps, **kw), ref), (nx, ny, scheme, v)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("walls", WALLS[:2])
@pytest.mark.parametrize("shape", [(20, 12, 9), (16, 8, 4), (3, 2, 5), (24, 18, 1), (401, 363, 1)])
def test_stages_and_adjoint_take_bricks(pf, dtype, shape, walls):
    """step_stages (in and out of place), the adjoint's recompute and its reverse stages on a
    handle whose steps run in bricks: the bits of the plain kernels."""
    dx = 1.0 / max(shape)
    nm = names(pf, dtype)
    res = []
    for variant in (nm.index("global"), -1):
        s = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, dtype=dtype, variant=variant, walls=walls, delta=1.0)
        phi, u, v, w = fields(shape, dtype)
        out = []
        for in_place in (False, True):
            p, ys = phi.clone(), [torch.empty_like(phi) for _ in range(3)]
            nxt = None if in_place else torch.empty_like(phi)
            out += [s.step_stages(p, u, v, w, 0.1, *ys, phi_next=nxt), *ys]
        lam = fields(shape, dtype, seed=3)[0]
        g = [torch.zeros_like(lam) for _ in range(3)]
        s.adjoint_step(phi, u, v, w, 0.1, lam, *g)
        torch.cuda.synchronize()
        s.close()
        res.append(out + [lam, *g])
    # the plain adjoint sums as the tiled one does: all bits equal
    for k, (a, b) in enumerate(zip(*res)):
        assert torch.equal(a, b), k


@pytest.mark.parametrize("eps_mode", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("walls", WALLS[:3])
def test_stretched_bricks_match_the_march(pf, dtype, walls, eps_mode):
    """A non-uniform mesh: the automatic variant's bricks against a named variant's march."""
    nm = names(pf, dtype)
    for shape in [(16, 8, 4), (19, 13, 9), (3, 2, 5), (33, 9, 8)]:
        rng = np.random.default_rng(5)
        dx = 1.0 / max(shape)
        h = [dx * rng.uniform(0.7, 1.4, n) for n in shape]
        res = []
        for variant in (nm.index("tiled_32x4"), -1):
            g = fields(shape, dtype)
            s = pf.Solver(shape, dx, dx, 1.0, 0.03 * dx, dtype=dtype, variant=variant, walls=walls)
            s.set_spacing(*[list(a) for a in h], eps_mode=eps_mode)
            print("case", shape, dtype, walls, eps_mode, variant, flush=True)
            s.step(*g, nsteps=2)
            torch.cuda.synchronize()
            s.close()
            res.append(g[0])
        assert torch.equal(*res), shape


def test_bricks_replay_from_graphs(pf):
    """A stream of its own: whole graphs, odd remainders and eager work between the replays."""
    st = torch.cuda.Stream()
    shape, dtype = (24, 16, 20), "f32"
    nm = names(pf, dtype)
    g, r = fields(shape, dtype), fields(shape, dtype)
    a = pf.Solver(shape, 1 / 24, 1 / 24, 1.0, 0.1 / 24, dtype=dtype)
    b = pf.Solver(shape, 1 / 24, 1 / 24, 1.0, 0.1 / 24, dtype=dtype, variant=nm.index("global"), use_graph=False)
    torch.cuda.synchronize()
    for n in (8, 17, 3, 24):
        a.step(*g, nsteps=n, stream=st)
        st.synchronize()
        b.step(*r, nsteps=n)
        torch.cuda.synchronize()
        assert torch.equal(g[0], r[0]), n
    a.close()
    b.close()
