"""The shapes the tuner times. CPU only: the list, not the timing."""
import ctypes as C

import pytest

from paper_2508_13867_amd import _abi as A


class Shape(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("cpt", "persistent", "nt", "layout", "pad", "bx", "fuse", "fty", "fwin")]

    def key(self):
        return tuple(getattr(self, n) for n, _ in self._fields_)


def problem(geometry, prec, nx, ny, **kw):
    spec = dict(geometry=geometry, precision=prec, nx=nx, ny=ny, nu=0.02, dists=[("nu", 0.015, 0.025)],
                rule=dict(kind="mc", N=8, seed=1), **kw)
    return A.make_problem(dict(spec, u0=0.03) if geometry == "tgv" else dict(spec, u_peak=0.05, ramp=10))


def candidates(p, S):
    fn = A.lib()["_ZN3uqi15tune_candidatesERK10uq_problemlPNS_9StepShapeEl"]
    fn.restype = C.c_int64
    out = (Shape * 512)()
    n = fn(C.byref(p), C.c_int64(S), out, C.c_int64(512))
    assert 0 < n <= 512
    return [out[k] for k in range(n)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("geometry, nx, ny, S", [
    ("tgv", 64, 64, 5), ("tgv", 64, 64, 64), ("tgv", 128, 128, 135), ("tgv", 160, 160, 64), ("tgv", 256, 192, 64),
    ("tgv", 300, 190, 100), ("tgv", 1024, 1024, 16), ("channel", 100, 41, 64), ("channel", 220, 41, 512),
    ("channel", 440, 82, 64), ("channel", 880, 164, 32)])
def test_the_untuned_shape_is_timed(prec, geometry, nx, ny, S):
    p, s = problem(geometry, prec, nx, ny), Shape()
    fn = A.lib()["_ZN3uqi14pipeline_shapeERK10uq_problemlPNS_9StepShapeE"]
    fn.restype = C.c_double
    # what a StepShape holds where the pipeline leaves it alone
    s.cpt, s.bx = 1, 64
    us = fn(C.byref(p), C.c_int64(S), C.byref(s))
    single = A.lib()["_ZN3uqi14single_step_usERK10uq_probleml"]
    single.restype = C.c_double
    keys = [c.key() for c in candidates(p, S)]
    # the pipeline, or one step per launch where the job takes that; the
    # single steps are there in either layout
    assert s.key() in keys or us >= single(C.byref(p), C.c_int64(S))
    assert {c[3] for c in keys if c[6] < 2} == {1, 2}


@pytest.mark.parametrize("nx", [160, 192, 256])
def test_double_precision_strips_are_timed(nx):
    # its rings hold no more than 4 steps over whole rows there
    got = {(c.fwin, c.fuse) for c in candidates(problem("tgv", "fp64", nx, nx), 64)}
    assert {(3, 6), (3, 8), (2, 4)} <= got and not any(w == 2 and n > 4 for w, n in got)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("nx, ny, S", [(64, 64, 5), (96, 96, 3), (128, 128, 8), (128, 128, 4096), (64, 64, 4096),
                                       (32, 32, 5000), (1024, 1024, 16)])
def test_nothing_is_timed_in_vain(prec, nx, ny, S):
    got = [c.key() for c in candidates(problem("tgv", prec, nx, ny), S)]
    assert len(set(got)) == len(got)
    # more tiles than the card takes, with a ring to compute around each
    if S * nx * ny > 1 << 20 and nx * ny > 1024:
        assert not any(c[8] == 4 for c in got)


def test_interpolated_channels_take_one_row():
    p = problem("channel", "fp32", 440, 80, cyl_bc="bouzidi", cyl_x=40.0, cyl_y=39.5, cyl_d=20.0, xbc="interp",
                layout="ab")
    assert {c.cpt for c in candidates(p, 11)} == {1}
