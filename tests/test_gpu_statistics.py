"""The split reductions of the statistics: nodes of a sample over chunks,
samples over waves. Against the same sums of the exported populations in
float64 on the host, compensated on neither side: a sum of n terms of one sign
is within n 2^-53 of itself there, and n stays below 10^6."""
import numpy as np
import pytest

CX = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1.0])
CY = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1.0])


def spec_of(nx, ny, N, layout):
    return dict(geometry="tgv", precision="fp64", nx=nx, ny=ny, u0=0.03, nu=0.02, layout=layout,
                dists=[("nu", 0.015, 0.025), ("u0", 0.02, 0.04)], rule=dict(kind="mc", N=N, seed=3))


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["aa", "ab"])
@pytest.mark.parametrize("nx, ny, N", [(2, 2, 2), (5, 3, 2), (31, 33, 2), (64, 17, 3), (33, 32, 9), (300, 41, 2),
                                       (8, 8, 129), (16, 9, 700), (70, 61, 17)])
def test_statistics_of_split_sums(nx, ny, N, layout):
    from paper_2508_13867_amd import Job

    print("case statistics", nx, ny, N, layout, flush=True)
    for steps in (2, 3):  # either slab holds the state
        with Job(spec_of(nx, ny, N, layout)) as job:
            job.run(steps)
            f = np.stack([job.populations(s) for s in range(N)])
            rho = f.sum(1)
            u = np.stack([np.tensordot(CX, f, (0, 1)), np.tensordot(CY, f, (0, 1))], 1) / rho[:, None]
            ke = 2 / (nx * ny * 0.03 ** 2) * (u ** 2).sum((1, 2, 3))
            # populations of 0.03-speed flow: j loses 1/0.03 to cancellation
            assert np.allclose(job.qoi_samples("ke")[:, 0], ke, rtol=1e-11, atol=1e-13)
            for q, v in (("ke", ke[:, None]), ("vel", u.reshape(N, -1)), ("rho", rho.reshape(N, -1))):
                m = job.moments(q)
                assert np.allclose(m["mean"], v.mean(0), rtol=1e-11, atol=1e-13)
                assert np.allclose(m["var_alt"], v.var(0), rtol=1e-9, atol=1e-13)
                assert np.allclose(m["var"], v.var(0, ddof=1), rtol=1e-9, atol=1e-13)
            job.run(3)  # the chunks' sums left nothing behind in the idle slab
            after = job.populations(N - 1)
        with Job(spec_of(nx, ny, N, layout)) as job:
            job.run(steps + 3)
            assert np.array_equal(after, job.populations(N - 1))
