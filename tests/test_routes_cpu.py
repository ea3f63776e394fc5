"""Which grids the two-stage sweeps of a variant take: host logic that steps, kept stages and the adjoint's
recompute share, called by its C++ name (no device, no allocation)."""
import ctypes

import pytest

import paper_1803_01262_amd as pf

sweeps_take = getattr(pf.lib, "_ZN2pf11sweeps_takeERK9pf_paramsi")
sweeps_take.restype = ctypes.c_bool


@pytest.mark.parametrize("dtype,n", [("f32", (1024, 1024, 1023)), ("f64", (1024, 1024, 511))])
def test_walled_arrays_of_4_gib_run_single_stages(dtype, n):
    kd = pf.PF_F32 if dtype == "f32" else pf.PF_F64
    for v in range(pf.phasefield_variant_count(kd)):
        name = pf.phasefield_variant_name(kd, v)
        for planes, walls in ((0, False), (0, True), (1, False), (1, True)):  # one plane more: 4 GiB
            p = pf.make_params((n[0], n[1], n[2] + planes), 0.1, 0.1, 1.0, 0.01, dtype=dtype, walls=(False, walls, False))
            want = name.startswith("fused") and not (walls and planes)
            assert sweeps_take(ctypes.byref(p), v) == want, (name, planes, walls)
