"""What a handle runs after tuning, from a tuning cache and with a variant named: a fused choice is one of whole
steps and leaves single stages and reverse stages to the rules, a per-stage choice runs them and lends its tile.
Bits are the plain kernel's either way."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BRICK = "tiled_brick16x8x4"
# name, given by, scheme -> whole steps, single stages, reverse stages on bricks (a 40 x 24 x 24 grid; FP32)
ROUTES = [
    ("fused_brick8x8x8", "cache", "rk4", ("fused_brick8x8x8", BRICK, True)),
    ("fused_brick8x8x8", "cache", "rk3", (BRICK, BRICK, True)),
    ("fused_64x8x32", "cache", "rk2", ("fused_64x8x32", BRICK, True)),
    ("fused_64x8x32", "cache", "euler", (BRICK, BRICK, True)),
    ("tiled_64x8x16", "cache", "rk4", ("tiled_64x8x16", "tiled_64x8x16", False)),
    ("fused_brick8x8x4", "param", "rk4", ("fused_brick8x8x4", BRICK, True)),
    ("fused_brick8x8x4", "param", "euler", (BRICK, BRICK, True)),
    (BRICK, "param", "rk4", (BRICK, BRICK, True)),
    ("fused_32x16", "param", "rk4", ("fused_32x16", "tiled_64x4", False)),
    ("fused_32x16", "param", "rk3", ("tiled_64x4", "tiled_64x4", False)),
    ("tiled_64x4", "param", "rk4", ("tiled_64x4", "tiled_64x4", False)),
    (None, None, "rk4", ("fused_brick8x8x4", BRICK, True)),
    (None, None, "rk3", (BRICK, BRICK, True)),
]


@pytest.fixture(scope="module")
def pf():
    import paper_1803_01262_amd
    return paper_1803_01262_amd


def names(pf):
    return [pf.phasefield_variant_name(pf.PF_F32, v) for v in range(pf.phasefield_variant_count(pf.PF_F32))]


def outputs(pf, s, shape):
    rng = np.random.default_rng(4)
    phi, *vel = [torch.tensor(rng.uniform(lo, 0.5, shape[::-1]), dtype=torch.float32, device="cuda")
                 for lo in (0.0, -0.5, -0.5, -0.5)]
    s.step(phi, *vel, nsteps=2)
    ys = [torch.empty_like(phi) for _ in range(s.stage_count)]
    nxt = s.step_stages(phi, *vel, 0.1, *ys, phi_next=torch.empty_like(phi))
    lam, *g = [torch.tensor(rng.uniform(-1, 1, shape[::-1]), dtype=torch.float32, device="cuda") for _ in range(4)]
    s.adjoint_step(phi, *vel, 0.1, lam, *g)
    torch.cuda.synchronize()
    return [phi, nxt, *ys, lam, *g]


@pytest.mark.parametrize("k", range(len(ROUTES)))
def test_routes(pf, tmp_path, monkeypatch, k):
    name, given, scheme, want = ROUTES[k]
    shape = (40, 24, 24 + k)  # a grid of its own: the cache lives as long as the process
    dx = 1.0 / 40
    if given == "cache":
        f = tmp_path / "tune.txt"
        f.write_text(f"{pf.PF_F32} {shape[0]} {shape[1]} {shape[2]} {name}\n")
        monkeypatch.setenv("PF_TUNE_CACHE", str(f))
    kw = dict(dtype="f32", scheme=scheme, delta=1.0)
    s = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, variant=names(pf).index(name) if given == "param" else -1, **kw)
    print("case", name, given, scheme, s.routes, flush=True)
    assert s.routes == want
    got = outputs(pf, s, shape)
    s.close()
    r = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, variant=names(pf).index("global"), **kw)
    for a, b in zip(got, outputs(pf, r, shape)):
        assert torch.equal(a, b)
    r.close()


def test_a_tuned_handle_keeps_its_rules(pf):
    shape, dx = (48, 24, 25), 1.0 / 48
    s = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, dtype="f32", delta=1.0)
    best, times = s.autotune(reps=1)
    name = names(pf)[best]
    assert s.variant_name == name != "fused_plane" and len(times) == len(names(pf))
    step, stage, bricks = s.routes
    assert step == name
    by_rule = "brick" in name or name.startswith("fused")
    assert (stage, bricks) == ((BRICK, True) if by_rule else (name, False))
    r = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, dtype="f32", delta=1.0, variant=names(pf).index("global"))
    for a, b in zip(outputs(pf, s, shape), outputs(pf, r, shape)):
        assert torch.equal(a, b)
    s.close()
    r.close()


def test_default_routes_of_larger_grids(pf):
    """The FP32 tile by the march, on a tie the one that pads fewer columns; one plane."""
    for shape, dtype, scheme, want in (((250, 200, 150), "f32", "rk4", "fused_64x8"), ((263, 268, 300), "f32", "rk2", "fused_32x16"),
                                       ((256, 256, 256), "f32", "rk4", "fused_64x8"), ((160, 160, 160), "f32", "rk2", "fused_32x16"),
                                       ((160, 160, 160), "f32", "rk3", "tiled_32x4"), ((128, 128, 128), "f64", "rk4", "fused_32x16"),
                                       ((64, 64, 1), "f64", "rk3", "fused_plane"), ((64, 64, 1), "f64", "euler", "tiled_32x4")):
        dx = 1.0 / max(shape)
        s = pf.Solver(shape, dx, dx, 1.0, 0.1 * dx, dtype=dtype, scheme=scheme)
        print("case", shape, dtype, scheme, s.variant_name, s.routes, flush=True)
        assert s.routes[0] == want, (shape, dtype, scheme)
        s.close()
