"""The ends of a channel in the strip pipeline (fused window 3): walls and
periodic ends, beside cylinders and the walls above and below.

CPU: a model of the rings in the order the kernel writes them (the lanes' first
columns pushed and bounced before their second ones, later rows over earlier
ones), against plain steps.

GPU: bit for bit the single-step result. A channel without an inlet starts at
rest and stays there, so the test fills the population slab itself (the library
takes its memory from the caller's allocator) before the first step.
"""
import ctypes as C

import numpy as np
import pytest

from test_channel_strips import CX, CY, GJ, OPP


class Ring:
    """One strip of one channel, as one workgroup runs it."""

    def __init__(self, nx, ny, solid, ends, lanes, seam_closed=True):
        self.nx, self.ny, self.solid, self.ends, self.L = nx, ny, solid, ends, lanes
        self.closed = ends == "walls" and seam_closed
        self.w = np.random.default_rng(7).uniform(0.05, 0.15, (9, 9))

    def source(self, i, y, x):  # of a pull: its node, or None for a wall
        sy, sx = y - CY[i], x - CX[i]
        if not 0 <= sy < self.ny:
            return None
        if not 0 <= sx < self.nx:
            if self.ends == "walls":
                return None
            sx %= self.nx
        return None if i and self.solid[sy, sx] else (sy, sx)

    def gather(self, g, y, x):
        src = [self.source(i, y, x) for i in range(9)]
        return np.array([g[(OPP[i], y, x)] if s is None else g[(i, *s)] for i, s in enumerate(src)])

    def plain(self, g):
        out = np.full_like(g, np.nan)
        for y in range(self.ny):
            for x in range(self.nx):
                if not self.solid[y, x]:
                    out[:, y, x] = self.w @ self.gather(g, y, x)
        return out

    def push_column(self, c, x, cx):
        if self.closed and ((cx > 0 and x == self.nx - 1) or (cx < 0 and x == 0)):
            return 0 if cx > 0 else self.L - 1
        return (c + cx) % self.L

    def strip(self, src, out, N, x0, W, yb, ye):
        L, RG = self.L, N - 1
        ring = np.full((N, 8, 3, L), np.nan)
        cols = [(x0 - RG + c) % self.nx for c in range(L)]
        pre = np.full((N + 1, L, 9), np.nan)
        for it in range(ye - yb + 3 * RG):
            done = []  # what this row step hands on, after every level has read
            for lvl in range(1, N + 1):
                span, y = RG - (lvl - 1), yb - RG - 2 * (lvl - 1) + it
                lo, hi = max(0, yb - span), min(self.ny, ye + span)
                if not (lo if lvl == 1 else lo - 1) <= y < hi:
                    continue
                f = {}
                for c in range(L):
                    if lvl == 1:
                        v = None if self.solid[y, cols[c]] else self.gather(src, y, cols[c])
                    else:
                        v = pre[lvl, c].copy()
                        for i in range(9):
                            if CY[i] < 0:
                                v[i] = ring[lvl - 2, (it + 2) % 3, GJ[i], c]
                            else:
                                slot = 3 + (it + 1) % 2 if CY[i] == 0 else 5 + (it + 1) % 3
                                pre[lvl, c, i] = ring[lvl - 2, slot, GJ[i], c]
                        if y < lo or self.solid[y, cols[c]]:
                            v = None
                    if v is not None:
                        f[c] = self.w @ v
                if lvl == N:
                    for c in range(RG, RG + W):
                        if c in f:
                            out[:, y, cols[c]] = f[c]
                else:
                    done.append((lvl, y, f))
            for lvl, y, f in done:
                for half in (range(L // 2), range(L // 2, L)):
                    mine = [c for c in half if c in f]
                    for c in mine:
                        for i in range(9):
                            slot = it % 3 if CY[i] < 0 else (3 + it % 2 if CY[i] == 0 else 5 + it % 3)
                            ring[lvl - 1, slot, GJ[i], self.push_column(c, cols[c], CX[i])] = f[c][i]
                    for c in mine:
                        for i in range(1, 9):
                            if self.source(i, y, cols[c]) is None:
                                slot = (it + 1) % 3 if CY[i] < 0 else (3 + it % 2 if CY[i] == 0 else 5 + (it + 2) % 3)
                                ring[lvl - 1, slot, GJ[i], c] = f[c][OPP[i]]


def both(nx, ny, N, H, ends, seam_closed=True):
    solid = np.zeros((ny, nx), bool)
    solid[ny // 2 - 1:ny // 2 + 1, nx // 3:nx // 3 + 2] = True
    lanes = 2 * (N - 1) + 8
    m = Ring(nx, ny, solid, ends, lanes, seam_closed)
    src = np.random.default_rng(nx).uniform(size=(9, ny, nx))
    want = src
    for _ in range(N):
        want = m.plain(want)
    got = np.full_like(src, np.nan)
    strips = -(-nx // 8)
    W = -(-nx // strips)
    for k in range(strips):
        for yb in range(0, ny, H):
            m.strip(src, got, N, min(k * W, nx - W), W, yb, min(ny, yb + H))
    fluid = np.broadcast_to(~solid, got.shape)
    return got[fluid], want[fluid]


@pytest.mark.parametrize("ends", ["walls", "periodic"])
@pytest.mark.parametrize("nx, ny, N, H", [(11, 9, 3, 9), (12, 10, 4, 4), (23, 8, 5, 8), (8, 7, 6, 3), (30, 12, 8, 6)])
def test_ring_ends(nx, ny, N, H, ends):
    got, want = both(nx, ny, N, H, ends)
    # sums of 9 N terms in another order
    assert np.abs(got - want).max() <= 1e-14 * np.abs(want).max()


def test_pushes_across_a_wall_would_show():
    got, want = both(23, 8, 5, 8, "walls", seam_closed=False)
    assert not np.abs(got - want).max() <= 1e-3


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("xbc", ["walls", "periodic"])
@pytest.mark.parametrize("nx, ny, rows, n", [
    (130, 16, 8, 6), (2, 7, 8, 3), (30, 12, 8, 7), (64, 21, 21, 5), (115, 24, 13, 7), (300, 33, 17, 7), (114, 9, 8, 4)])
def test_moving_channels_equal_single_steps(prec, xbc, nx, ny, rows, n, monkeypatch):
    import torch

    from paper_2508_13867_amd import _abi as A

    D = min(8, ny // 2, nx // 4)
    spec = dict(geometry="channel", precision=prec, nx=nx, ny=ny, u_peak=0.05, nu=0.02, D=D, cx=nx // 3,
                cy=ny // 2 - 1, xbc=xbc, layout="ab", dists=[("nu", 0.015, 0.025)],
                rule=dict(kind="gl", n=2, order=1))
    print("case moving channel", prec, xbc, nx, ny, rows, n, flush=True)
    dtype = dict(fp64=torch.float64, fp32=torch.float32, fp16s=torch.float16, bf16s=torch.bfloat16)[prec]
    monkeypatch.setenv("UQ_FUSE_WINDOW", "3")
    monkeypatch.setenv("UQ_FUSE_TY", str(rows))
    res = {}
    for fuse in (0, n):
        monkeypatch.setenv("UQ_FUSE", str(fuse))
        dev, keep = A.torch_device(0)
        h, p, info = C.c_void_p(), A.make_problem(spec), A.JobInfo()
        A.check(A.lib().uq_create(C.byref(p), C.byref(dev), C.byref(h)))
        A.check(A.lib().uq_job_get_info(h, C.byref(info)))
        assert info.fused == fuse and (not fuse or info.fused_window == 3)
        # the first slab holds the state of step 0: shifted populations of a few 1e-3
        bytes_ = info.S * 9 * (ny * info.pitch + info.plane_pad) * torch.empty(0, dtype=dtype).element_size()
        slabs = [t for t in keep.live.values() if t.numel() == bytes_]
        f = np.random.default_rng(5).normal(0.0, 2e-3, bytes_ // slabs[0].view(dtype).element_size())
        slabs[0].view(dtype).copy_(torch.from_numpy(f * 2.0 ** info.scale_exp).to(dtype))
        A.check(A.lib().uq_run(h, 2 * n + 5))  # pairs of launches, an odd one and single steps
        A.check(A.lib().uq_run(h, 2 * n))
        out = np.zeros((2, 9, ny, nx))
        for s in range(2):
            A.check(A.lib().uq_populations(h, s, out[s].ctypes.data))
        A.lib().uq_destroy(h)
        res[fuse] = out
    assert np.isfinite(res[0]).all()
    assert np.abs(res[0][0, 1, :, 0] - 1 / 9).max() > 1e-5  # it does move, at the ends too
    assert np.array_equal(res[0], res[n])


@pytest.mark.gpu
@pytest.mark.parametrize("nx", [300, 500, 900])
def test_served_channels_between_walls(nx):
    from paper_2508_13867_amd import Server

    print("case served walls", nx, flush=True)
    spec = dict(geometry="channel", precision="fp32", nx=nx, ny=20, u_peak=0.05, nu=0.02, xbc="walls",
                dists=[("nu", 0.015, 0.025)], rule=dict(kind="gl", n=2, order=1))
    with Server(memory_budget_gb=0.25, steps_per_tick=48, precision="fp32") as srv:
        got = srv.wait(srv.submit(spec, 101, "ke"))
    assert got["status"] == 0 and got["mean"] == 0.0  # at rest
