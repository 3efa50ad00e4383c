"""The channel pipeline down column strips (channel jobs, fused window 3).

CPU: a model of the rings with the bounce-back on the writing side: places,
slots and row steps as the kernel takes them, on lattices with walls, solid
nodes and open ends (whose pulls a rule overwrites: here with the node's own
column index), against plain steps.

GPU: bit for bit the single-step result, at the widths where the strips begin
to split, chunks that meet the walls and the cylinder, in every format.
"""
import numpy as np
import pytest

CX = [0, 1, 0, -1, 0, 1, -1, -1, 1]
CY = [0, 0, 1, 0, -1, 1, 1, -1, -1]
OPP = [0, 3, 4, 1, 2, 7, 8, 5, 6]
GJ = [0, 1, 0, 2, 0, 1, 2, 1, 2]


class Model:
    def __init__(self, nx, ny, solid, lanes):
        self.nx, self.ny, self.solid, self.lanes = nx, ny, solid, lanes
        self.w = np.random.default_rng(7).uniform(0.05, 0.15, (9, 9))

    def kind(self, i, y, x):  # of the pull of direction i at a fluid node
        sy, sx = y - CY[i], x - CX[i]
        if sy < 0 or sy >= self.ny:
            return "wall"
        if sx < 0 or sx >= self.nx:
            return "open"
        return "wall" if i and self.solid[sy, sx] else "in"

    def collide(self, f, x):
        return self.w @ f

    def gather(self, g, y, x):
        f = np.empty(9)
        for i in range(9):
            k = self.kind(i, y, x)
            f[i] = g[OPP[i], y, x] if k == "wall" else (x if k == "open" else g[i, y - CY[i], x - CX[i]])
        return f

    def plain(self, g):
        out = np.full_like(g, np.nan)
        for y in range(self.ny):
            for x in range(self.nx):
                if not self.solid[y, x]:
                    out[:, y, x] = self.collide(self.gather(g, y, x), x)
        return out

    def strip(self, src, out, N, x0, W, yb, ye):
        nx, ny, L, RG = self.nx, self.ny, self.lanes, N - 1
        ring = np.full((N, 8, 3, L), np.nan)
        cols = [(x0 - RG + c) % nx for c in range(L)]
        pre = {}
        for it in range(ye - yb + 3 * RG):
            reads, writes = set(), {}

            def read(lvl, slot, g, c):
                reads.add((lvl - 2, slot, g, c))
                return ring[lvl - 2, slot, g, c]

            def write(lvl, slot, g, c, v, c_own):
                k = (lvl - 1, slot, g, c)
                # only an edge lane's wrapped push may meet another write
                assert k not in writes or c in (0, L - 1), k
                writes[k] = v

            for lvl in range(1, N + 1):
                span = RG - (lvl - 1)
                lo, hi = max(0, yb - span), min(ny, ye + span)
                y = yb - RG - 2 * (lvl - 1) + it
                f = {}
                if lvl == 1:
                    if lo <= y < hi:
                        f = {c: self.gather(src, y, cols[c]) for c in range(L) if not self.solid[y, cols[c]]}
                elif lo - 1 <= y < hi:
                    for c in range(L):
                        v = np.empty(9)
                        new = np.empty(9)
                        for i in range(9):
                            if CY[i] < 0:
                                v[i] = read(lvl, (it + 2) % 3, GJ[i], c)
                            else:
                                v[i] = pre.get((lvl, c), np.full(9, np.nan))[i]
                                new[i] = read(lvl, 3 + (it + 1) % 2 if CY[i] == 0 else 5 + (it + 1) % 3, GJ[i], c)
                        pre[lvl, c] = new
                        if y >= lo and not self.solid[y, cols[c]]:
                            for i in range(9):
                                if self.kind(i, y, cols[c]) == "open":
                                    v[i] = cols[c]
                            f[c] = v
                for c, v in f.items():
                    v = self.collide(v, cols[c])
                    if lvl == N:
                        if RG <= c < RG + W:
                            out[:, y, cols[c]] = v
                        continue
                    for i in range(9):
                        slot = it % 3 if CY[i] < 0 else (3 + it % 2 if CY[i] == 0 else 5 + it % 3)
                        write(lvl, slot, GJ[i], (c + CX[i]) % L, v[i], c)
                    for i in range(1, 9):
                        if self.kind(i, y, cols[c]) == "wall":
                            slot = (it + 1) % 3 if CY[i] < 0 else (3 + it % 2 if CY[i] == 0 else 5 + (it + 2) % 3)
                            k = (lvl - 1, slot, GJ[i], c)
                            # whatever else lands there this step comes around the strip's edge
                            assert k not in writes or c in (0, L - 1), k
                            writes[k] = v[OPP[i]]
            assert not reads & set(writes)  # no place is read and written in one step
            for k, v in writes.items():
                ring[k] = v


@pytest.mark.parametrize("nx, ny, N, H", [(11, 9, 3, 9), (12, 10, 4, 4), (23, 8, 5, 8), (5, 7, 6, 3), (30, 12, 8, 6)])
def test_rings_with_bounce_on_the_writing_side(nx, ny, N, H):
    solid = np.zeros((ny, nx), bool)
    solid[ny // 2 - 1:ny // 2 + 1, nx // 3:nx // 3 + 2] = True
    solid[ny // 2, min(nx - 2, nx // 3 + 3)] = True  # a one-node gap between solids
    solid[0, nx // 2] = True
    lanes = 2 * (N - 1) + 8
    m = Model(nx, ny, solid, lanes)
    src = np.random.default_rng(nx).uniform(size=(9, ny, nx))
    want = src
    for _ in range(N):
        want = m.plain(want)
    got = np.full_like(src, np.nan)
    wmax = lanes - 2 * (N - 1)
    strips = -(-nx // wmax)
    W = -(-nx // strips)
    for k in range(strips):
        for yb in range(0, ny, H):
            m.strip(src, got, N, min(k * W, nx - W), W, yb, min(ny, yb + H))
    assert np.array_equal(np.isnan(got), np.broadcast_to(solid, got.shape))
    ok = ~np.isnan(got)
    assert np.abs(got[ok] - want[ok]).max() <= 1e-14 * np.abs(want[ok]).max()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s", "bf16s"])
@pytest.mark.parametrize("nx, ny, rows, n, over", [
    (114, 20, 8, 7, {}), (117, 9, 8, 6, {}), (300, 41, 21, 7, {}), (230, 33, 33, 5, {}), (64, 10, 8, 4, {}),
    (30, 12, 8, 3, {}), (116, 24, 24, 7, dict(xbc="periodic")), (130, 16, 8, 6, dict(xbc="walls")),
    (3, 9, 9, 6, dict(D=0)), (240, 26, 13, 8, {})])
def test_strips_equal_single_steps(prec, nx, ny, rows, n, over, monkeypatch):
    from paper_2508_13867_amd import Job

    if prec == "fp64" and n > 7:
        pytest.skip("double precision takes up to 7 steps")
    D = min(8, ny // 2, nx // 4)
    spec = dict(geometry="channel", precision=prec, nx=nx, ny=ny, u_peak=0.05, nu=0.02, D=D, cx=nx // 3, cy=ny // 2 - 1,
                ramp=13, xbc="zouhe", layout="ab", dists=[("re", 16.0, 24.0), ("u_peak", 0.045, 0.055)],
                rule=dict(kind="gl", n=2, order=1))
    spec.update(over)
    if not spec["D"]:
        spec["dists"] = [("nu", 0.015, 0.025), ("u_peak", 0.045, 0.055)]
    print("case channel strips", prec, nx, ny, rows, n, over, flush=True)
    monkeypatch.setenv("UQ_FUSE_WINDOW", "3")
    monkeypatch.setenv("UQ_FUSE_TY", str(rows))
    res = {}
    for fuse in (0, n):
        monkeypatch.setenv("UQ_FUSE", str(fuse))
        with Job(spec) as job:
            assert job.info().fused == fuse
            job.run(2 * n + 5)  # pairs of launches, an odd one and single steps
            job.run(2 * n)
            res[fuse] = [job.populations(s) for s in (0, 3)]
    assert np.isfinite(res[0]).all()
    assert np.array_equal(res[0], res[n])


@pytest.mark.gpu
@pytest.mark.parametrize("nx, ny, N", [(400, 30, 5), (800, 21, 3)])
def test_server_channels_in_strips(nx, ny, N):
    from paper_2508_13867_amd import Job, Server

    print("case served strips", nx, ny, N, flush=True)
    spec = dict(geometry="channel", precision="fp32", nx=nx, ny=ny, u_peak=0.05, nu=0.02, D=8, cx=nx // 3, cy=ny // 2,
                ramp=13, xbc="zouhe", dists=[("re", 16.0, 24.0)], rule=dict(kind="gl", n=N, order=1))
    with Server(memory_budget_gb=1.0, steps_per_tick=48, precision="fp32") as srv:
        got = srv.wait(srv.submit(spec, 119, "cd"))
    with Job(dict(spec, layout="aa")) as job:
        job.run(119)
        want = job.moments("cd")
    assert got["mean"] == pytest.approx(want["mean"][0], rel=1e-12)
    assert got["var"] == pytest.approx(want["var"][0], rel=1e-9)
