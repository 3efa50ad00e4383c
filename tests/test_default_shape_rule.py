"""Which jobs that nobody tuned run in a pipeline: those it makes faster. On
lattices of few rows and on channels of few nodes one step per launch is the
faster of the two."""
import ctypes as C

import pytest

from paper_2508_13867_amd import _abi as A

# geometry, precision, nx, ny, samples, us per step in single steps and in the pipeline (one MI355X)
MEASURED = [
    ("tgv", "fp32", 4096, 2, 512, 43.0, 59.8), ("tgv", "fp32", 4096, 4, 512, 92.9, 69.0),
    ("tgv", "fp32", 20000, 2, 32, 15.3, 18.6), ("tgv", "fp64", 20000, 2, 512, 542, 682),
    ("tgv", "fp64", 130, 100, 512, 239, 54.6), ("tgv", "fp16s", 4096, 4, 512, 43.4, 93.2),
    ("tgv", "fp16s", 4096, 16, 512, 232, 153), ("tgv", "fp32", 64, 8, 2, 2.4, 0.56),
    ("channel", "fp32", 400, 30, 2, 3.43, 4.17), ("channel", "fp32", 400, 30, 32, 8.37, 4.96),
    ("channel", "fp32", 1024, 8, 512, 45.7, 57.8), ("channel", "fp32", 4096, 3, 512, 71.1, 157),
    ("channel", "fp32", 4096, 16, 512, 437, 282), ("channel", "fp32", 100, 5, 512, 8.58, 3.56),
    ("channel", "fp64", 500, 60, 2, 4.21, 5.75), ("channel", "fp64", 500, 60, 32, 23.1, 15.1),
    ("channel", "fp32", 264, 49, 22, 7.32, 6.18), ("channel", "fp16s", 528, 98, 3, 4.8, 5.54),
    ("channel", "fp64", 64, 512, 2, 4.29, 6.26), ("channel", "fp64", 2, 427, 143, 54.7, 67.6),
    ("channel", "fp16s", 20000, 3, 512, 363, 832),
    ("channel", "fp16s", 129, 50, 2, 3.44, 4.81), ("channel", "fp16s", 500, 60, 512, 161, 114),
]


def problem(geometry, prec, nx, ny, n):
    spec = dict(geometry=geometry, precision=prec, nx=nx, ny=ny, nu=0.02, dists=[("nu", 0.015, 0.025)],
                rule=dict(kind="mc", N=n, seed=1))
    return dict(spec, u0=0.03) if geometry == "tgv" else dict(spec, u_peak=0.05, ramp=10, xbc="zouhe")


@pytest.mark.parametrize("geometry, prec, nx, ny, n, single, pipeline", MEASURED)
def test_the_faster_of_the_two(geometry, prec, nx, ny, n, single, pipeline):
    est = A.lib()["_ZN3uqi14single_step_usERK10uq_probleml"], A.lib()["_ZN3uqi14pipeline_shapeERK10uq_problemlPNS_9StepShapeE"]
    p, shape = A.make_problem(problem(geometry, prec, nx, ny, n)), C.create_string_buffer(256)
    for fn in est:
        fn.restype = C.c_double
    s = est[0](C.byref(p), C.c_int64(n))
    q = est[1](C.byref(p), C.c_int64(n), shape)
    assert (q < s) == (pipeline < single)


@pytest.mark.gpu
@pytest.mark.parametrize("geometry, prec, nx, ny, n, layout", [
    ("channel", "fp32", 400, 30, 2, 1), ("channel", "fp32", 400, 30, 32, 2), ("channel", "fp64", 64, 512, 2, 1),
    ("tgv", "fp32", 20000, 2, 32, 1), ("tgv", "fp32", 257, 64, 32, 2)])
def test_layout_taken(geometry, prec, nx, ny, n, layout):
    from paper_2508_13867_amd import Job

    print("case layout taken", geometry, prec, nx, ny, n, flush=True)
    with Job(problem(geometry, prec, nx, ny, n)) as job:
        assert job.info().layout == layout and bool(job.info().fused) == (layout == 2)
