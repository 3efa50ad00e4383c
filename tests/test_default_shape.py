"""The launch shape of jobs that nobody tuned and whose layout nobody fixed:
periodic lattices run in the row pipelines, bit for bit as one step per launch
in the AA layout, and keep to one slab where a second one finds no room."""
import ctypes as C

import numpy as np
import pytest

SHAPE_ENV = ("UQ_CPT", "UQ_PERSISTENT", "UQ_NT_STORE", "UQ_PLANE_PAD", "UQ_BX", "UQ_FUSE", "UQ_FUSE_TY",
             "UQ_FUSE_WINDOW", "UQ_LAYOUT")


def vortex(nx, ny, prec, n=2, **kw):
    return dict(geometry="tgv", precision=prec, nx=nx, ny=ny, u0=0.03, nu=0.02,
                dists=[("nu", 0.015, 0.025), ("u0", 0.02, 0.04)], rule=dict(kind="gl", n=n, order=1), **kw)


@pytest.fixture(autouse=True)
def no_shape_env(monkeypatch):
    for k in SHAPE_ENV:
        monkeypatch.delenv(k, raising=False)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("nx, ny", [(3, 2), (48, 9), (128, 40), (129, 7), (256, 33), (257, 21)])
def test_untuned_job_equals_single_steps(prec, nx, ny):
    from paper_2508_13867_amd import Job

    print("case default shape", prec, nx, ny, flush=True)
    got = {}
    for layout in (None, "aa"):
        with Job(vortex(nx, ny, prec, **({"layout": layout} if layout else {}))) as job:
            assert (job.info().fused >= 3) == (layout is None)
            for steps in (1, 16, 26):
                job.run(steps)
            got[layout] = [job.populations(s) for s in (0, 3)]
    assert np.array_equal(got[None], got["aa"])


@pytest.mark.gpu
def test_no_room_for_a_second_slab():
    import torch

    from paper_2508_13867_amd import Job
    from paper_2508_13867_amd import _abi as A

    print("case one slab only", flush=True)
    spec = vortex(96, 64, "fp32", n=4)
    slab = 16 * 9 * (64 * 128 + 64) * 4

    class OneSlab(A.TorchAllocator):
        def alloc(self, nbytes, ctx):
            if nbytes >= slab and any(t.numel() >= slab for t in self.live.values()):
                return None
            return super().alloc(nbytes, ctx)

    keep, dev = OneSlab(0), A.Device()
    dev.device = 0
    dev.stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    dev.alloc, dev.free = keep._alloc, keep._free
    h, p = C.c_void_p(), A.make_problem(spec)
    A.check(A.lib().uq_create(C.byref(p), C.byref(dev), C.byref(h)))
    inf, out = A.JobInfo(), np.zeros((9, 64, 96))
    A.check(A.lib().uq_job_get_info(h, C.byref(inf)))
    assert inf.layout == 1 and inf.fused == 0
    A.check(A.lib().uq_run(h, 20))
    A.check(A.lib().uq_populations(h, 5, out.ctypes.data))
    A.lib().uq_destroy(h)
    with Job(spec) as job:
        assert job.info().layout == 2 and job.info().fused
        job.run(20)
        assert np.array_equal(job.populations(5), out)
