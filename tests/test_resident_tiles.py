"""Resident tiles (fused window 4): one node per lane, n steps per launch.
Bit for bit the single-step result where tiles begin to split, where one or
both directions are whole periods, and where the last tile moves back."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("nx, ny, n", [(2, 2, 3), (32, 32, 16), (33, 32, 8), (32, 33, 5), (64, 16, 12), (64, 17, 8),
                                       (31, 90, 6), (100, 23, 8), (70, 61, 4), (257, 3, 7), (48, 48, 16)])
def test_tiles_equal_single_steps(prec, nx, ny, n, monkeypatch):
    from paper_2508_13867_amd import Job

    spec = dict(geometry="tgv", precision=prec, nx=nx, ny=ny, u0=0.03, nu=0.02, layout="ab",
                dists=[("nu", 0.015, 0.025), ("u0", 0.02, 0.04)], rule=dict(kind="gl", n=2, order=1))
    print("case tiles", prec, nx, ny, n, flush=True)
    monkeypatch.setenv("UQ_FUSE_WINDOW", "4")
    res = {}
    for fuse in (0, n):
        monkeypatch.setenv("UQ_FUSE", str(fuse))
        with Job(spec) as job:
            assert job.info().fused == fuse and (not fuse or job.info().fused_window == 4)
            job.run(2 * n + 5)  # pairs of launches, an odd one and single steps
            job.run(2 * n)
            res[fuse] = [job.populations(s) for s in (0, 3)]
    assert np.array_equal(res[0], res[n])
