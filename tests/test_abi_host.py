"""Host-only checks of the C ABI: the library loads, exports every symbol of include/pbsplit.h,
and rejects bad arguments / out-of-order calls before touching the GPU."""
import ctypes as C
import os
import re

import pytest

from paper_2504_00340_amd import inputs as I
from paper_2504_00340_amd import pbsplit as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    src = open(os.path.join(ROOT, "include", "pbsplit.h")).read()
    return sorted(set(re.findall(r"\b(pbs_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    L = B.lib()
    names = _declared()
    assert set(names) == set(B.EXPORTS), names
    for n in names:
        assert hasattr(L, n), n


def _create(grid, phys=None, prec=B.PBS_FP32):
    L = B.lib()
    ctx = C.c_void_p()
    rc = L.pbs_create(C.byref(B._mk(B.Grid, grid)), C.byref(B._mk(B.Physics, phys or I.PHYS)), prec, C.byref(ctx))
    return rc, ctx


def test_create_validates_grid_and_physics():
    g = I.config1()["grid"]
    rc, ctx = _create(g)
    assert rc == B.PBS_OK and ctx.value
    nb = C.c_size_t()
    assert B.lib().pbs_workspace_bytes(ctx, C.byref(nb)) == B.PBS_OK and nb.value > 0
    # state machine: everything before bind is ESTATE, bad bind is EINVAL
    L = B.lib()
    assert L.pbs_set_beam(ctx, C.byref(B._mk(B.Beam, I.beam(100.0)))) == B.PBS_ESTATE
    assert L.pbs_step_depth(ctx, 1, None) == B.PBS_ESTATE
    assert L.pbs_run_beam(ctx) == B.PBS_ESTATE
    assert L.pbs_bind(ctx, None, nb.value, None) == B.PBS_EINVAL
    assert L.pbs_bind(ctx, C.c_void_p(256 * 1024), nb.value - 1, None) == B.PBS_EINVAL
    assert L.pbs_bind(ctx, C.c_void_p(256 * 1024 + 8), nb.value, None) == B.PBS_EINVAL
    assert b"workspace" in L.pbs_last_error(ctx)
    # the schedule switch is host state: valid modes anytime, others EINVAL
    for mode in (B.PBS_SCHED_ONE_STREAM, B.PBS_SCHED_TWO_STREAMS, B.PBS_SCHED_AUTO):
        assert L.pbs_set_schedule(ctx, mode) == B.PBS_OK
    assert L.pbs_set_schedule(ctx, 3) == B.PBS_EINVAL and L.pbs_set_schedule(ctx, -1) == B.PBS_EINVAL
    L.pbs_destroy(ctx)
    for bad in [dict(g, nth=7), dict(g, nth=2), dict(g, ng=1), dict(g, nz=0), dict(g, ngen=0), dict(g, ngen=9),
                dict(g, dz=-0.1), dict(g, x_half=float("nan")), dict(g, e_hi=g["e_lo"]), dict(g, ny=300)]:
        rc, ctx = _create(bad)
        assert rc == B.PBS_EINVAL and not ctx.value, bad
    rc, _ = _create(dict(g, nth=14))
    assert rc == B.PBS_EUNSUPPORTED
    rc, _ = _create(g, dict(I.PHYS, bk_alpha=0.0))
    assert rc == B.PBS_EINVAL
    # stopping-power model: the two known values; the Bethe-Bloch form needs a floor >= 0.5 MeV
    for phys, want in ((dict(I.PHYS, stopping=B.PBS_STOP_BETHE), B.PBS_OK), (dict(I.PHYS, stopping=2), B.PBS_EINVAL),
                       (dict(I.PHYS, stopping=-1), B.PBS_EINVAL),
                       (dict(I.PHYS, stopping=B.PBS_STOP_BETHE, e_floor=0.4), B.PBS_EINVAL),
                       (dict(I.PHYS, stopping=B.PBS_STOP_BRAGG_KLEEMAN, e_floor=0.4), B.PBS_OK)):
        rc, ctx = _create(g, phys)
        assert rc == want, phys
        if ctx.value:
            B.lib().pbs_destroy(ctx)
    rc, _ = _create(g, prec=7)
    assert rc == B.PBS_EINVAL


def test_workspace_scales_with_precision_and_generations():
    g = I.config1()["grid"]
    sizes = {}
    for prec in (B.PBS_FP32, B.PBS_FP64):
        for ngen in (1, 2):
            rc, ctx = _create(dict(g, ngen=ngen), prec=prec)
            nb = C.c_size_t()
            B.lib().pbs_workspace_bytes(ctx, C.byref(nb))
            sizes[prec, ngen] = nb.value
            B.lib().pbs_destroy(ctx)
    assert sizes[B.PBS_FP64, 1] > sizes[B.PBS_FP32, 1]
    assert sizes[B.PBS_FP32, 2] > 2 * sizes[B.PBS_FP32, 1] - 1


def test_batch_create_validates_shape_class():
    L = B.lib()
    g1 = I.grid(10, 10, 16, 20, 4, 2, 1.0, 1.0, 0.15, 0.0, 40.0, 0.6)
    g2 = dict(g1, ng=33, nz=7, e_hi=50.0)
    bm = I.beam(30.0)
    grids = (B.Grid * 2)(B._mk(B.Grid, g1), B._mk(B.Grid, g2))
    beams = (B.Beam * 2)(B._mk(B.Beam, bm), B._mk(B.Beam, bm))
    h = C.c_void_p()
    assert L.pbs_batch_create(grids, beams, 2, C.byref(B._mk(B.Physics, I.PHYS)), 0, C.byref(h)) == B.PBS_OK
    nb = C.c_size_t()
    assert L.pbs_batch_workspace_bytes(h, C.byref(nb)) == B.PBS_OK and nb.value > 0
    assert L.pbs_batch_run(h) == B.PBS_ESTATE
    L.pbs_batch_destroy(h)
    bad = (B.Grid * 2)(B._mk(B.Grid, g1), B._mk(B.Grid, dict(g2, nx=11)))
    h = C.c_void_p()
    assert L.pbs_batch_create(bad, beams, 2, C.byref(B._mk(B.Physics, I.PHYS)), 0, C.byref(h)) == B.PBS_EINVAL
    small = (B.Grid * 1)(B._mk(B.Grid, dict(g1, nth=8)))
    assert L.pbs_batch_create(small, beams, 1, C.byref(B._mk(B.Physics, I.PHYS)), 0, C.byref(h)) == B.PBS_EUNSUPPORTED


def test_surrogate_and_network_argument_checks():
    import numpy as np

    L = B.lib()
    g = dict(I.config1()["grid"])           # ngen = 2
    rc, ctx = _create(g)
    nb0 = C.c_size_t()
    L.pbs_workspace_bytes(ctx, C.byref(nb0))
    # blobs: wrong magic, wrong size, NaN; then recording mode grows the workspace
    good = B.pack_weights(np.zeros(B.param_count(), dtype=np.float32), 0.01)
    bad_magic = b"XXXX" + good[4:]
    assert L.pbs_set_surrogate(ctx, bad_magic, len(bad_magic), 1e-2) == B.PBS_EINVAL
    assert L.pbs_set_surrogate(ctx, good, len(good) - 4, 1e-2) == B.PBS_EINVAL
    nanp = np.zeros(B.param_count(), dtype=np.float32)
    nanp[5] = np.nan
    nan_blob = B.pack_weights(nanp, 0.0)
    assert L.pbs_set_surrogate(ctx, nan_blob, len(nan_blob), 1e-2) == B.PBS_EINVAL
    assert L.pbs_set_surrogate(ctx, good, len(good), -1.0) == B.PBS_EINVAL
    assert L.pbs_set_surrogate(ctx, None, 0, 0.0) == B.PBS_OK
    nb1 = C.c_size_t()
    L.pbs_workspace_bytes(ctx, C.byref(nb1))
    assert nb1.value > nb0.value
    assert L.pbs_set_surrogate(ctx, good, len(good), 1e-2) == B.PBS_OK
    nb2 = C.c_size_t()
    L.pbs_workspace_bytes(ctx, C.byref(nb2))
    assert nb2.value > nb1.value
    out = (C.c_double * 8)()
    assert L.pbs_surrogate_report(ctx, out, 8) == B.PBS_ESTATE
    L.pbs_destroy(ctx)
    # the surrogate replaces generation 1 of a K = 1 grid only
    for bad in (dict(g, ngen=1), dict(g, ngen=3)):
        rc, ctx = _create(bad)
        assert L.pbs_set_surrogate(ctx, None, 0, 0.0) == B.PBS_EINVAL
        L.pbs_destroy(ctx)
    rc, ctx = _create(dict(g, ny=65))
    assert L.pbs_set_surrogate(ctx, None, 0, 0.0) == B.PBS_EUNSUPPORTED
    L.pbs_destroy(ctx)
    # network
    n = C.c_size_t()
    assert L.pbs_net_param_count(C.byref(n)) == B.PBS_OK and n.value == 21121
    h = C.c_void_p()
    assert L.pbs_net_create(64, 65, 4, C.byref(h)) == B.PBS_EINVAL
    assert L.pbs_net_create(64, 64, 0, C.byref(h)) == B.PBS_EINVAL
    assert L.pbs_net_create(64, 64, 4, C.byref(h)) == B.PBS_OK
    nb = C.c_size_t()
    assert L.pbs_net_workspace_bytes(h, C.byref(nb)) == B.PBS_OK and nb.value > 4 * 64 * 64 * 32 * 2 * 5
    p = np.zeros(n.value, dtype=np.float32)
    assert L.pbs_net_set_params(h, p.ctypes.data_as(C.POINTER(C.c_float)), p.size) == B.PBS_ESTATE
    assert L.pbs_net_forward(h, C.c_void_p(4096), C.c_void_p(4096), 1) == B.PBS_ESTATE
    assert L.pbs_net_bind(h, C.c_void_p(256 * 1024 + 8), nb.value, None) == B.PBS_EINVAL
    assert b"aligned" in L.pbs_net_last_error(h)
    L.pbs_net_destroy(h)


def test_physics_switches_are_validated():
    """Straggling, media other than water and their Bethe-Bloch requirement, scattering model, nuclear bands
    (count and increasing anchors); the batched path and the surrogate refuse straggling and bands."""
    import numpy as np

    L = B.lib()
    g = I.config1()["grid"]
    paper = I.paper_physics(I.MAT_BONE)
    bands = dict(I.PHYS, **I.NUC_BANDS)
    for phys, want in ((paper, B.PBS_OK), (dict(paper, stopping=B.PBS_STOP_BRAGG_KLEEMAN), B.PBS_EINVAL),
                       (dict(I.PHYS, material=I.MAT_BONE), B.PBS_EINVAL), (dict(I.PHYS, straggling=1), B.PBS_EINVAL),
                       (dict(paper, straggling=2), B.PBS_EINVAL), (dict(paper, material=3), B.PBS_EINVAL),
                       (dict(paper, scattering=2), B.PBS_EINVAL), (dict(I.PHYS, scattering=B.PBS_SCAT_RUTHERFORD),
                                                                   B.PBS_OK),
                       (bands, B.PBS_OK), (dict(bands, nuc_bands=5), B.PBS_EINVAL),
                       (dict(bands, nuc_e=[52.5, 104.3, 104.3, 207.9]), B.PBS_EINVAL),
                       (dict(bands, nuc_beta=[25.0, 0.0, 45.0, 55.0]), B.PBS_EINVAL),
                       (dict(bands, nuc_alpha=[0.5, 2.0, 2.2, 2.4]), B.PBS_EINVAL)):
        rc, ctx = _create(g, phys)
        assert rc == want, phys
        if ctx.value:
            L.pbs_destroy(ctx)
    # straggling and bands: single-beam path only, no surrogate
    g1 = I.grid(10, 10, 16, 20, 4, 2, 1.0, 1.0, 0.15, 0.0, 40.0, 0.6)
    grids = (B.Grid * 1)(B._mk(B.Grid, g1))
    beams = (B.Beam * 1)(B._mk(B.Beam, I.beam(30.0)))
    h = C.c_void_p()
    for phys in (I.paper_physics(), bands):
        assert L.pbs_batch_create(grids, beams, 1, C.byref(B._mk(B.Physics, phys)), 0, C.byref(h)) == \
            B.PBS_EUNSUPPORTED
        rc, ctx = _create(g, phys)
        assert L.pbs_set_surrogate(ctx, None, 0, 0.0) == B.PBS_EUNSUPPORTED
        L.pbs_destroy(ctx)
    # FP32 contexts with straggling take the FP32 source product: the split-BF16 modes are refused
    rc, ctx = _create(dict(g, nth=16), I.paper_physics())
    assert L.pbs_set_source_precision(ctx, B.PBS_SRC_BF16X1) == B.PBS_EUNSUPPORTED
    assert L.pbs_set_source_precision(ctx, B.PBS_SRC_FP32) == B.PBS_OK
    L.pbs_destroy(ctx)


def test_voxel_phantom_resampling_matches_the_batched_plan():
    """pbs_resample_phantom (the resampling of pbs_set_phantom_voxels) on the shared 128 x 128 x 400 phantom of
    the batched plan (0.1 x 0.1 x 0.0875 cm voxels) gives exactly the nearest-voxel densities the plan's input
    generator assigns each beam's 32 x 32 window; bad spacings and densities are refused; before bind the
    context call returns PBS_ESTATE."""
    import numpy as np

    cfg = I.config4(seed=0, nbeams=6)
    ph = cfg["phantom"]
    corner_of = lambda spot: (-12.8 / 2 - spot[0], -12.8 / 2 - spot[1])
    for b in cfg["beams"]:
        got = B.resample_phantom(b["grid"], ph, (0.0875, 0.1, 0.1), corner_of(b["spot"]))
        assert np.array_equal(got, b["rho"]), b["spot"]
    g = cfg["beams"][0]["grid"]
    with pytest.raises(B.PbsError):
        B.resample_phantom(g, ph, (0.0875, 0.0, 0.1), (0.0, 0.0))
    bad = ph[:4, :5, :6].copy()
    bad[1, 2, 3] = -1.0
    with pytest.raises(B.PbsError):
        B.resample_phantom(g, bad, (0.0875, 0.1, 0.1), (0.0, 0.0))
    rc, ctx = _create(g)
    v = np.ascontiguousarray(ph[:4, :5, :6])
    assert B.lib().pbs_set_phantom_voxels(ctx, v.ctypes.data_as(C.POINTER(C.c_double)), 4, 5, 6, 0.1, 0.1, 0.1,
                                          0.0, 0.0) == B.PBS_ESTATE
    B.lib().pbs_destroy(ctx)


# contexts of fewer than 128 angular unknowns just within the static scratch, as large as the unpadded product matrices
# allow (bytes: the tables' exact sizes are part of what fits)
@pytest.mark.parametrize("nx,ny,nth,ng,nz,ngen,prec,bands", [
    (16, 4, 8, 145, 18454, 2, B.PBS_FP64, True), (16, 4, 10, 96, 17019, 2, B.PBS_FP64, True),
    (16, 4, 12, 89, 10867, 2, B.PBS_FP64, True), (16, 4, 12, 133, 215, 2, B.PBS_FP64, True),
    (16, 4, 12, 124, 15763, 3, B.PBS_FP32, False), (16, 4, 12, 138, 18083, 2, B.PBS_FP32, True)])
def test_contexts_near_the_static_scratch_still_fit(nx, ny, nth, ng, nz, ngen, prec, bands):
    g = I.grid(nx, ny, nth, ng, nz, ngen, 4.0, 4.0, 0.15, 0.0, 160.0, 1.0)
    rc, ctx = _create(g, dict(I.PHYS, **I.NUC_BANDS) if bands else None, prec)
    assert rc == B.PBS_OK
    nb = C.c_size_t()
    assert B.lib().pbs_workspace_bytes(ctx, C.byref(nb)) == B.PBS_OK
    B.lib().pbs_destroy(ctx)
    assert nb.value <= B.PBS_STATIC_SCRATCH_BYTES
