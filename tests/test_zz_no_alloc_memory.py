"""What the statistics leave in a job's memory. uq_moments_noalloc promises to
leave all of it untouched; uq_moments may use the slab that does not hold the
state, and the steps after it must not notice, solid nodes included."""
import numpy as np
import pytest

from paper_2508_13867_amd import Job

CASES = {
    "vortex": dict(geometry="tgv", precision="fp32", nx=96, ny=96, u0=0.03, nu=0.02,
                   dists=[("nu", 0.015, 0.025)], rule=dict(kind="gl", n=3, order=2), layout="ab"),
    "cylinder": dict(geometry="channel", precision="fp64", nx=90, ny=41, u_peak=0.05, nu=0.05, D=12, cx=20, cy=20,
                     ramp=10, xbc="zouhe", dists=[("re", 16.0, 24.0)], rule=dict(kind="gl", n=2, order=1),
                     layout="ab"),
    "curved": dict(geometry="channel", precision="fp32", nx=90, ny=40, u_peak=0.06, nu=0.04, cyl_bc="bouzidi",
                   cyl_x=20.0, cyl_y=19.5, cyl_d=12.0, ramp=10, xbc="interp", dists=[("u_peak", 0.05, 0.07)],
                   rule=dict(kind="gl", n=2, order=1), layout="ab"),
}


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [16, 17])  # either slab holds the state
@pytest.mark.parametrize("name", list(CASES))
def test_noalloc_touches_nothing_of_the_job(name, steps):
    import torch

    print("case noalloc memory", name, steps, flush=True)
    with Job(CASES[name]) as job:
        job.run(steps)
        job.sync()
        before = {p: t.clone() for p, t in job._keep.live.items()}
        torch.cuda.synchronize()
        got = {q: job.moments(q, noalloc=True) for q in ("ke", "vel")}
        torch.cuda.synchronize()
        assert set(job._keep.live) == set(before)
        for p, t in before.items():
            assert torch.equal(t, job._keep.live[p])
        for q, g in got.items():
            want = job.moments(q)
            assert all(np.array_equal(g[k], want[k]) for k in want)


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [16, 17])
@pytest.mark.parametrize("name", ["cylinder", "curved"])
def test_steps_do_not_notice_the_statistics(name, steps):
    print("case watched channel", name, steps, flush=True)
    out = []
    for watch in (False, True):
        with Job(CASES[name]) as job:
            job.run(steps)
            if watch:
                job.moments("ke")
                job.qoi_samples("cd")
            job.run(9)
            out.append([job.populations(s) for s in (0, 1)] + [job.moments("cd")["mean"]])
    assert all(np.array_equal(a, b) for a, b in zip(*out))
