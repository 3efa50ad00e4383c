"""One launch per step for interpolated boundaries: column chunks of 81 rows,
cylinder nodes of all samples side by side, bulk tiles. Where the chunks and
the node list end, against the FP64 oracle (its arithmetic agrees to rounding:
the bound of the other population tests, 1e-13)."""
import numpy as np
import pytest

import oracle as O
from test_gpu_cylinder_interp import SMALL, VARIANTS, oracle_f
from paper_2508_13867_amd import workloads as W


@pytest.mark.gpu
@pytest.mark.parametrize("nt", ["0", "1"])
@pytest.mark.parametrize("nx, ny, N, variant", [
    (30, 80, 3, "bouzidi+fd"), (30, 81, 7, "halfway+fd"), (65, 82, 13, "bouzidi+fd"), (64, 163, 2, "bouzidi+fd"),
    (31, 27, 40, "bouzidi+zouhe")])
def test_populations(nx, ny, N, variant, nt, monkeypatch):
    from paper_2508_13867_amd import Job

    monkeypatch.setenv("UQ_NT_STORE", nt)
    spec = W.scaled(SMALL, nx=nx, ny=ny, rule=dict(kind="mc", N=N, seed=5), ramp=5, **VARIANTS[variant])
    print("case interp step", nx, ny, N, variant, nt, flush=True)
    with Job(spec) as job:
        job.run(9)
        xi, _ = job.samples()
        for s in (0, N - 1):
            ref = oracle_f(spec, O.sample_params(spec, xi[s]), 9)["f"]
            assert np.abs(job.populations(s) - ref).max() < 1e-13
