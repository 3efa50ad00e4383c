"""The whole-row pipeline down column strips (fused window 3).

CPU: a model of the strips' columns. A work item's lanes take the columns
x0 - (N - 1) .. of the periodic lattice; a pull from beyond the outermost
lane brings in a wrong value (NaN here), so one more lane per level is wrong
on either side, and level N stores only the W lanes in the middle.

GPU: bit for bit the single-step result, at the widths where the strips
begin to split, on ragged and wrapping lattices, in every format.
"""
import numpy as np
import pytest

CX = [0, 1, 0, -1, 0, 1, -1, -1, 1]
CY = [0, 0, 1, 0, -1, 1, 1, -1, -1]
LANES = 128


def strips_of(nx, n):
    wmax = LANES - 2 * (n - 1)
    strips = -(-nx // wmax)
    return strips, -(-nx // strips)


@pytest.mark.parametrize("n", [3, 6, 8])
@pytest.mark.parametrize("nx", [1, 3, 114, 115, 128, 129, 300, 1024])
def test_strip_columns(nx, n):
    # every node stored with the value of n plain periodic steps; the "step"
    # mixes the pulled directions so that a wrong pull shows
    rng = np.random.default_rng(nx)
    ny, w = 4, rng.uniform(0.05, 0.15, (9, 9))
    src = rng.uniform(size=(9, ny, nx))

    def step(f, pull):
        return np.tensordot(w, np.stack([pull(f[i], i) for i in range(9)]), 1)

    want = src
    for _ in range(n):
        want = step(want, lambda v, i: np.roll(v, (CY[i], CX[i]), (0, 1)))

    def lane_pull(v, i):  # rows are whole; the outermost lane has no neighbour
        v = np.roll(v, (CY[i], CX[i]), (0, 1))
        if CX[i]:
            v[:, 0 if CX[i] > 0 else -1] = np.nan
        return v

    strips, W = strips_of(nx, n)
    assert W <= nx and W <= LANES - 2 * (n - 1)
    got = np.full((9, ny, nx), np.nan)
    for k in range(strips):
        x0 = min(k * W, nx - W)
        cols = (x0 - (n - 1) + np.arange(LANES)) % nx
        # level 1 pulls from the slab, at every lane's own column
        f = step(src, lambda v, i: np.roll(v, (CY[i], CX[i]), (0, 1)))[:, :, cols]
        for _ in range(n - 1):
            f = step(f, lane_pull)
        got[:, :, x0:x0 + W] = f[:, :, n - 1:n - 1 + W]
    assert np.array_equal(np.isnan(got), np.zeros_like(got, bool))
    assert np.abs(got - want).max() <= 1e-14 * np.abs(want).max()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("nx, ny, rows, n", [
    (114, 9, 8, 8), (115, 9, 8, 8), (300, 21, 8, 8), (700, 11, 64, 6), (257, 16, 8, 7), (122, 13, 8, 4),
    (130, 5, 8, 3), (126, 10, 16, 5), (3, 5, 8, 8)])
def test_strips_equal_single_steps(prec, nx, ny, rows, n, monkeypatch):
    from paper_2508_13867_amd import Job

    spec = dict(geometry="tgv", precision=prec, nx=nx, ny=ny, u0=0.03, nu=0.02, layout="ab",
                dists=[("nu", 0.015, 0.025), ("u0", 0.02, 0.04)], rule=dict(kind="gl", n=2, order=1))
    print("case strips", prec, nx, ny, rows, n, flush=True)
    monkeypatch.setenv("UQ_FUSE_WINDOW", "3")
    monkeypatch.setenv("UQ_FUSE_TY", str(rows))
    steps = 2 * n + 5  # pairs of launches, an odd one and single steps
    res = {}
    for fuse in (0, n):
        monkeypatch.setenv("UQ_FUSE", str(fuse))
        with Job(spec) as job:
            assert job.info().fused == fuse and (not fuse or job.info().fused_window == 3)
            job.run(steps)
            res[fuse] = [job.populations(s) for s in (0, 3)]
    assert np.array_equal(res[0], res[n])
