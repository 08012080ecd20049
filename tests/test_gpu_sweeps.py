"""Sweep kernels at the sizes where a variant's edges lie, through the C ABI against the FP64 oracle.

Bounds: FP64 sub-steps 1e-12, FP32 ones 1e-5 of the largest value of the generation (the bounds of the other
sub-step tests: a few hundred rounding errors of 2^-53 / 2^-24 along a line)."""
import numpy as np
import pytest

from paper_2504_00340_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}


@pytest.fixture(scope="module")
def O():
    from oracle import oracle

    return oracle


def _setup(O, prec, shape, phys=None, src=None, seed=7):
    from paper_2504_00340_amd import pbsplit as P

    c = I.small(nz=2, seed=seed, **shape)
    if phys:
        c["phys"] = phys
    s = P.Solver(c["grid"], c["phys"], precision=prec)
    if src is not None and (shape["nth"] - 1) ** 2 >= 128 and prec == "fp32":
        s.set_source_precision(src)
    s.set_phantom(c["rho"])
    s.set_beam(c["beam"])
    st = I.random_state(s.state_shape, seed)
    st[:, :, 1] *= 0.3
    s.set_state(st)
    return s, O.Oracle(c["grid"], c["phys"]), c, st


def _check(got, ref, prec, what):
    for k in range(ref.shape[0]):
        e = np.abs(got[k] - ref[k])
        print(what, prec, "generation", k, "max error", e.max() / np.abs(ref[k]).max(), "at",
              np.unravel_index(e.argmax(), e.shape), flush=True)
        assert e.max() <= TOL[prec] * np.abs(ref[k]).max()


# group counts around the groups a chunk of the pipeline of waves holds (grids this small take it), angular counts whose
# last line group holds one line (nth 10: 81 = 8 * 10 + 1; nth 16: 225 = 8 * 28 + 1); the rings have a test of their own
@pytest.mark.parametrize("ng", [2, 3, 4, 5, 7])
@pytest.mark.parametrize("nth,prec", [(6, "fp32"), (10, "fp64"), (16, "fp64"), (16, "fp32"), (20, "fp32")])
def test_energy_step_around_the_group_ring(O, nth, prec, ng):
    print("case energy ring", nth, prec, ng, flush=True)
    # generation 1's one-product BF16 source has its own bound; the exact source modes are tested below
    s, o, c, st = _setup(O, prec, dict(nx=5, ny=7, nth=nth, ng=ng, ngen=2))
    ref = st.copy()
    o.energy_all(ref, np.ascontiguousarray(c["rho"][1].reshape(-1)), 0.02)
    s.apply(1, 1, 0.02)
    got = s.state()
    s.close()
    if prec == "fp32" and nth >= 16:
        _check(got[:1], ref[:1], prec, "ring")
        e = np.abs(got[1] - ref[1]).max() / np.abs(ref[1]).max()
        print("generation 1, BF16 source:", e, flush=True)
        assert e <= 1e-2
    else:
        _check(got, ref, prec, "ring")


# one lateral tile: an odd number of (tile, line) rows, the last block's second half repeats the last one
@pytest.mark.parametrize("ng,ngen", [(2, 2), (9, 3)])
@pytest.mark.parametrize("nth,prec", [(8, "fp32"), (12, "fp64"), (16, "fp64"), (16, "fp32")])
def test_energy_pipeline_of_one_tile(O, nth, prec, ng, ngen):
    print("case energy pipeline", nth, prec, ng, ngen, flush=True)
    s, o, c, st = _setup(O, prec, dict(nx=4, ny=5, nth=nth, ng=ng, ngen=ngen), phys=dict(I.PHYS, **I.NUC_BANDS))
    ref = st.copy()
    rho = np.ascontiguousarray(c["rho"][1].reshape(-1))
    o.energy_all(ref, rho, 0.02)
    s.apply(1, 1, 0.02)
    got = s.state()
    s.close()
    n = 1 if prec == "fp32" and nth >= 16 else ngen   # the BF16 source has its own bound
    _check(got[:n], ref[:n], prec, "pipeline")


def test_batched_ring_is_the_single_beam_pass():
    """The single beam takes the pipeline of waves, few batched beams the ring and many the plain pass: the same bits."""
    from paper_2504_00340_amd.pbsplit import Batch, Solver

    def beams(n):
        out = []
        for i in range(n):
            c = I.small(nx=16, ny=16, nth=16, ng=9 + i % 3, nz=3, ngen=2, e0=32.0, e_hi=40.0, depth=0.6, seed=40 + i)
            out.append(dict(grid=c["grid"], beam=c["beam"], rho=c["rho"]))
        return out

    few, many = beams(2), beams(40)   # 232 waves per beam: 464 and 9280, either side of the rule
    doses = []
    for bs in (few, many):
        b = Batch(bs, dict(I.PHYS))
        b.run()
        doses.append([b.dose(i) for i in range(2)])
        b.close()
    for i in range(2):
        s = Solver(few[i]["grid"], dict(I.PHYS), "fp32")
        s.set_phantom(few[i]["rho"])
        s.set_beam(few[i]["beam"])
        s.run()
        d = s.dose()
        s.close()
        assert np.array_equal(d, doses[0][i]) and np.array_equal(d, doses[1][i])


# widths around the lanes a plane takes in the packed transport (16, 32, 64, two planes in three operations, one in
# two), rows around the rows loaded ahead (4; FP64's wide forms 2), odd plane counts (the last wave's missing planes)
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 4), (4, 15), (5, 16), (7, 17), (8, 31), (9, 32), (12, 33), (2, 63), (10, 64),
                                   (3, 65), (4, 70), (6, 80), (7, 95), (9, 96), (11, 97), (5, 127), (13, 128), (3, 129)])
def test_transport_widths(O, nx, ny, prec):
    print("case transport", nx, ny, prec, flush=True)
    s, o, c, st = _setup(O, prec, dict(nx=nx, ny=ny, nth=6, ng=3, ngen=1))
    ref = st.copy()
    for k in range(ref.shape[0]):
        o.transport_cn(ref[k], 0.05)
    s.apply(2, 1, 0.05)
    got = s.state()
    s.close()
    _check(got, ref, prec, "transport")


# every number of 32-row waves of the small product (9, 25, 49, 81, 121 angles), one tile per block and, past 8192
# (half, group, tile) items, several (with a last block that is not full); the dose checks the reduction's slots
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nth,ng", [(3, 5, 4, 3), (5, 7, 6, 4), (6, 6, 8, 5), (9, 8, 10, 3), (4, 9, 12, 4),
                                          (67, 64, 4, 70), (65, 65, 6, 66)])
def test_small_source_product_and_dose(O, nx, ny, nth, ng, prec):
    print("case small source product", nx, ny, nth, ng, prec, flush=True)
    s, o, c, st = _setup(O, prec, dict(nx=nx, ny=ny, nth=nth, ng=ng, ngen=2))
    ref = st.copy()
    rho = np.ascontiguousarray(c["rho"][1].reshape(-1))
    dep = o.energy_all(ref, rho, 0.02)
    s.apply(1, 1, 0.02)
    got, dose = s.state(), s.dose()[1].reshape(-1)
    vol = o.dx * o.dy * c["grid"]["dz"]
    s.close()
    _check(got, ref, prec, "source")
    e = np.linalg.norm(dose - dep / (rho * vol)) / np.linalg.norm(dep / (rho * vol))
    print("dose", e, flush=True)
    # the oracle's deposit is a difference of energy contents, far larger than it
    assert e <= (1e-11 if prec == "fp64" else TOL[prec])


# the straggling sweeps around their ring of two groups, with and without a source and a next generation; a whole
# march takes every mode (open, fused pair, close) and the factors of both halves
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("ng,ngen", [(2, 1), (3, 2), (4, 3), (5, 2)])
def test_straggling_march_around_the_group_ring(O, ng, ngen, prec):
    from paper_2504_00340_amd import pbsplit as P

    print("case straggling ring", ng, ngen, prec, flush=True)
    c = I.small(nx=5, ny=9, nth=6, ng=ng, nz=3, ngen=ngen, e0=60.0, e_hi=70.0, depth=0.3, seed=9)
    c["phys"] = I.paper_physics(I.MAT_BONE)
    dref, fref = O.Oracle(c["grid"], c["phys"]).run(c["beam"], c["rho"])
    s = P.Solver(c["grid"], c["phys"], precision=prec)
    s.set_phantom(c["rho"])
    s.set_beam(c["beam"])
    s.run()
    d, f = s.dose(), s.state()
    s.close()
    e = np.linalg.norm(d - dref) / np.linalg.norm(dref)
    print("dose", e, flush=True)
    assert e <= (1e-12 if prec == "fp64" else 1e-4)
    for k in range(ngen):
        assert np.abs(f[k] - fref[k]).max() <= (1e-12 if prec == "fp64" else 1e-4) * np.abs(fref[k]).max(), k


# every angular grid (dense and parity-split matrix forms, vector form for 4 and 6), with a last tile that is not full
# and tile counts around the 8 that share an XCD group
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nth", [4, 6, 8, 10, 12, 16, 20, 24, 32])
@pytest.mark.parametrize("nx,ny", [(3, 7), (9, 30)])
def test_angular_step(O, nx, ny, nth, prec):
    print("case angular", nx, ny, nth, prec, flush=True)
    s, o, c, st = _setup(O, prec, dict(nx=nx, ny=ny, nth=nth, ng=2, ngen=2))
    ref = st.copy()
    rho = np.ascontiguousarray(c["rho"][1].reshape(-1))
    for k in range(ref.shape[0]):
        o.angular_cn(ref[k], rho, 0.3)
    s.apply(3, 1, 0.3)
    got = s.state()
    s.close()
    _check(got, ref, prec, "angular")


# T A T of a small slab in one launch (one stream) against its three passes (two streams), whose bits it has: every
# angular count it takes, one and two planes per 32 lanes, partly filled and several tiles, the fewest slabs and the most
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nth,ng,ngen", [(1, 1, 6, 48, 1), (3, 5, 8, 24, 2), (4, 4, 12, 50, 2), (2, 16, 10, 128, 2),
                                               (5, 16, 12, 64, 1), (3, 17, 8, 64, 4), (2, 32, 6, 50, 2), (9, 31, 6, 60, 2),
                                               (2, 30, 10, 48, 1), (1, 32, 12, 64, 2)])
def test_small_slabs_in_one_launch(nx, ny, nth, ng, ngen, prec):
    from paper_2504_00340_amd import pbsplit as P

    print("case one launch", nx, ny, nth, ng, ngen, prec, flush=True)
    c = I.small(nz=4, seed=3, nx=nx, ny=ny, nth=nth, ng=ng, ngen=ngen)
    out = []
    for mode in (P.PBS_SCHED_ONE_STREAM, P.PBS_SCHED_TWO_STREAMS):
        s = P.Solver(c["grid"], c["phys"], precision=prec)
        s.set_schedule(mode)
        s.set_phantom(c["rho"])
        s.set_beam(c["beam"])
        s.set_state(I.random_state(s.state_shape, 3))
        s.step(3)
        out.append((s.state(), s.dose()))
        s.close()
    assert np.isfinite(out[0][0]).all()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


# slabs of 1 GiB and more: the sweep by pointers.  A beam in the middle of a very long grid against the same beam
# on a short one of the same cells (nothing reaches either one's ends), so that no host copy of the fluence is needed.
@pytest.mark.parametrize("ny,long_nx", [(33, 8500), (20, 14000), (64, 8801)])
def test_transport_of_slabs_beyond_a_buffer_resource(ny, long_nx):
    from paper_2504_00340_amd import pbsplit as P

    print("case large slab", ny, long_nx, flush=True)
    doses = []
    for nx in (long_nx, 200 + long_nx % 2):
        g = I.grid(nx, ny, 32, 2, 2, 1, 0.05 * nx, 1.5, 0.1, 0.0, 40.0, 0.4)
        s = P.Solver(g, dict(I.PHYS), "fp32")
        s.set_phantom(I.water(g))
        s.set_beam(I.beam(30.0, y0=0.1, sigma_x=0.3, sigma_y=0.25))
        s.run()
        d = s.dose()
        s.close()
        lo = nx // 2 - 60
        doses.append(d[:, lo:lo + 120].copy())
    e = np.abs(doses[0] - doses[1]).max() / np.abs(doses[1]).max()
    print("difference", e, flush=True)
    assert np.isfinite(doses[0]).all() and e <= TOL["fp32"]


# the two-plane sweep that the passes take at 32 columns and whole groups of eight rows against the fused launch's
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,nth,ng,ngen", [(8, 6, 50, 2), (32, 6, 48, 2), (16, 8, 60, 1), (8, 10, 50, 2), (8, 12, 48, 2)])
def test_small_slabs_of_32_columns_in_one_launch(nx, nth, ng, ngen, prec):
    from paper_2504_00340_amd import pbsplit as P

    print("case one launch, 32 columns", nx, nth, ng, ngen, prec, flush=True)
    c = I.small(nz=4, seed=3, nx=nx, ny=32, nth=nth, ng=ng, ngen=ngen)
    out = []
    for mode in (P.PBS_SCHED_ONE_STREAM, P.PBS_SCHED_TWO_STREAMS):
        s = P.Solver(c["grid"], c["phys"], precision=prec)
        s.set_schedule(mode)
        s.set_phantom(c["rho"])
        s.set_beam(c["beam"])
        s.set_state(I.random_state(s.state_shape, 3))
        s.step(3)
        out.append((s.state(), s.dose()))
        s.close()
    assert np.isfinite(out[0][0]).all()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


# more than 800 blocks of 64 threads, so that the register rings run and not the pipeline of waves: one line per thread
# (fewer than 128 angles, FP64), four lines (FP32 from 128 on), and the plain four-line pass above 8192 waves; group counts
# with every remainder of the ring, with one law of nuclear data and with four bands
@pytest.mark.parametrize("bands", [False, True])
@pytest.mark.parametrize("nx,ny,nth,prec,ng", [
    (65, 65, 6, "fp32", 2), (65, 65, 6, "fp32", 3), (65, 65, 6, "fp32", 5), (65, 65, 6, "fp64", 3), (65, 65, 6, "fp64", 4),
    (20, 24, 16, "fp64", 5), (40, 32, 16, "fp32", 2), (40, 32, 16, "fp32", 3), (41, 33, 16, "fp32", 7), (20, 24, 24, "fp32", 5),
    (96, 97, 16, "fp32", 3)])
def test_energy_rings_above_the_pipeline(O, nx, ny, nth, prec, ng, bands):
    print("case ring", nx, ny, nth, prec, ng, bands, flush=True)
    phys = dict(I.PHYS, **I.NUC_BANDS) if bands else None
    s, o, c, st = _setup(O, prec, dict(nx=nx, ny=ny, nth=nth, ng=ng, ngen=2), phys=phys)
    ref, rho = st.copy(), np.ascontiguousarray(c["rho"][1].reshape(-1))
    o.energy_all(ref, rho, 0.02)
    s.apply(1, 1, 0.02)
    got = s.state()
    s.close()
    _check_modes(got, ref, prec, nth, "ring", o, st, rho)


def _check_modes(got, ref, prec, nth, what, o, st, rho):
    """All generations at the sub-step bound; those that take the one-product BF16 source within what its roundings
    (the matrix, the scans with their carried residue, the product: 2^-9 each) make of the source's part in them."""
    n = 1 if prec == "fp32" and nth >= 16 else len(ref)
    _check(got[:n], ref[:n], prec, what)
    for k in range(n, len(ref)):
        alone = np.zeros_like(st)   # no earlier generation, no source
        alone[k] = st[k]
        o.energy_all(alone, rho, 0.02)
        top = np.abs(ref[k]).max()
        tol = TOL[prec] + 2.0 ** -6 * np.abs(ref[k] - alone[k]).max() / top
        e = np.abs(got[k] - ref[k]).max() / top
        print(what, "generation", k, "BF16 source:", e, "of", tol, flush=True)
        assert e <= tol


# the exact source modes, every generation at the sub-step bound: FP32 scans (the one-line pipeline and ring) and three
# BF16 products of scans in two halves (the plain four-line pass; each term within 2^-15 of the source)
@pytest.mark.parametrize("ng", [2, 3, 4, 5, 7])
@pytest.mark.parametrize("nx,ny,nth,src", [(5, 7, 16, 0), (20, 24, 16, 0), (5, 7, 16, 1), (5, 7, 20, 1), (40, 32, 16, 1)])
def test_energy_step_with_an_exact_source(O, nx, ny, nth, src, ng):
    print("case exact source", nx, ny, nth, src, ng, flush=True)
    s, o, c, st = _setup(O, "fp32", dict(nx=nx, ny=ny, nth=nth, ng=ng, ngen=3), src=src)
    ref = st.copy()
    o.energy_all(ref, np.ascontiguousarray(c["rho"][1].reshape(-1)), 0.02)
    s.apply(1, 1, 0.02)
    got = s.state()
    s.close()
    _check(got, ref, "fp32", "exact source")


# the later generations of the pipeline, whose source is read in BF16
@pytest.mark.parametrize("bands", [False, True])
@pytest.mark.parametrize("nx,ny,ng,ngen", [(4, 5, 2, 2), (4, 5, 9, 3), (5, 7, 7, 4), (16, 16, 5, 2)])
def test_energy_pipeline_later_generations(O, nx, ny, ng, ngen, bands):
    print("case pipeline generations", nx, ny, ng, ngen, bands, flush=True)
    phys = dict(I.PHYS, **I.NUC_BANDS) if bands else None
    s, o, c, st = _setup(O, "fp32", dict(nx=nx, ny=ny, nth=16, ng=ng, ngen=ngen), phys=phys)
    ref, rho = st.copy(), np.ascontiguousarray(c["rho"][1].reshape(-1))
    o.energy_all(ref, rho, 0.02)
    s.apply(1, 1, 0.02)
    got = s.state()
    s.close()
    _check_modes(got, ref, "fp32", 16, "pipeline", o, st, rho)
