"""The schedule that a march takes by itself, seen from the launches that the kernel timing counts: on one stream a
step's transport is two launches for all generations, on two streams two for each."""
import pytest

from paper_2504_00340_amd import inputs as I

pytestmark = pytest.mark.gpu


def _streams(nx, ny, nth, ng, ngen, prec):
    from paper_2504_00340_amd import pbsplit as P

    print("case schedule", nx, ny, nth, ng, ngen, prec, flush=True)
    c = I.small(nz=3, seed=3, nx=nx, ny=ny, nth=nth, ng=ng, ngen=ngen)
    s = P.Solver(c["grid"], c["phys"], precision=prec)
    s.set_phantom(c["rho"])
    s.set_beam(c["beam"])
    s.profile(True)
    s.step(2)
    n = s.profile_read()["tpass"][1]
    s.close()
    assert n in (4, 4 * ngen)
    return 1 if n == 4 else 2


def test_timing_keeps_the_stream_of_the_march():
    # small slabs whose T A T is one launch stay on one stream, also while their passes are timed one by one
    assert _streams(32, 32, 6, 60, 2, "fp32") == 1


# short steps stay on one stream, long ones overlap, around the length that the second stream's events cost; from 1e6
# cells or 128 angles on always two, one generation always one
@pytest.mark.parametrize("nx,ny,nth,ng,ngen,prec,streams", [
    (10, 10, 8, 130, 2, "fp32", 2), (10, 40, 8, 24, 2, "fp32", 1), (10, 40, 6, 90, 2, "fp32", 2), (10, 40, 6, 60, 2, "fp32", 1),
    (4, 4, 4, 130, 2, "fp32", 1), (4, 4, 12, 130, 2, "fp32", 2), (10, 40, 8, 48, 3, "fp32", 2), (8, 20, 10, 60, 2, "fp64", 2),
    (8, 20, 10, 30, 2, "fp64", 1), (4, 4, 16, 16, 2, "fp32", 2), (40, 40, 12, 16, 2, "fp32", 2), (10, 40, 8, 130, 1, "fp32", 1)])
def test_second_stream_by_the_length_of_the_step(nx, ny, nth, ng, ngen, prec, streams):
    assert _streams(nx, ny, nth, ng, ngen, prec) == streams


# more slabs than CUs: T A T stays one launch on one stream except where the passes on two streams are faster
@pytest.mark.parametrize("nx,ny,nth,ng,ngen,prec,streams", [
    (16, 16, 8, 128, 2, "fp32", 1), (16, 20, 8, 100, 2, "fp32", 2), (16, 20, 8, 100, 3, "fp32", 2), (16, 20, 8, 60, 4, "fp32", 1),
    (24, 32, 6, 128, 2, "fp32", 1), (10, 16, 12, 129, 2, "fp32", 2), (10, 16, 12, 128, 2, "fp32", 2), (8, 16, 12, 128, 2, "fp32", 1),
    (4, 4, 12, 128, 2, "fp64", 2), (4, 4, 12, 64, 2, "fp64", 1), (4, 4, 12, 64, 4, "fp64", 1), (8, 20, 8, 128, 2, "fp64", 1)])
def test_second_round_of_small_slabs(nx, ny, nth, ng, ngen, prec, streams):
    assert _streams(nx, ny, nth, ng, ngen, prec) == streams
