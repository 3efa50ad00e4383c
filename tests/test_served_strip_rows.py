"""Chunk heights of served vortex strips: few samples on wide lattices must not
leave the card idle. CPU: the height a group of jobs gets, by its work items.
GPU: served results against the job API in single steps, at widths where the
routes part (whole rows, strips, 16-bit whole rows, single steps)."""
import ctypes as C

import pytest

from paper_2508_13867_amd import _abi as A


def group_rows(jobs):  # (nx, ny, samples) each, 8 steps per launch
    strips = [-(-nx // 114) for nx, _, _ in jobs]
    items = (C.c_int64 * len(jobs))(*[s * S for s, (_, _, S) in zip(strips, jobs)])
    ny = (C.c_int * len(jobs))(*[h for _, h, _ in jobs])
    fn = A.lib()["_ZN3uqi10group_rowsEPKlPKiiii"]
    rows = fn(items, ny, len(jobs), 21, 2)
    return rows, sum(i * -(-h // rows) for i, h in zip(items, ny))


@pytest.mark.parametrize("jobs", [[(640, 256, 4)], [(384, 384, 4)], [(1024, 1024, 2)], [(1024, 128, 2)],
                                  [(300, 300, 2), (640, 256, 4)], [(768, 700, 8)], [(512, 512, 16)]])
def test_few_samples_fill_the_card(jobs):
    rows, work = group_rows(jobs)
    tallest = max(ny for _, ny, _ in jobs)
    assert 8 <= rows <= tallest
    # a workgroup for every CU, unless the chunks are as short as they get (two
    # rounds of the shortest chunks cost less than one of anything taller)
    assert work >= 256 or rows < 2 * 8
    assert rows <= 128


def test_many_samples_take_tall_chunks():
    rows, work = group_rows([(1024, 1024, 64), (384, 384, 256)])
    assert rows >= 100 and work > 2000


@pytest.mark.gpu
@pytest.mark.parametrize("prec, nx, ny, N", [
    ("fp32", 640, 90, 3), ("fp32", 300, 64, 2), ("fp16s", 384, 50, 3), ("bf16s", 512, 33, 2), ("fp16s", 640, 64, 2),
    ("fp32", 4100, 2, 9), ("fp16s", 4100, 4, 9)])
def test_served_equals_single_steps(prec, nx, ny, N):
    from paper_2508_13867_amd import Job, Server

    print("case served vortex", prec, nx, ny, N, flush=True)
    spec = dict(geometry="tgv", precision=prec, nx=nx, ny=ny, u0=0.03, nu=0.02,
                dists=[("nu", 0.015, 0.025), ("u0", 0.02, 0.04)], rule=dict(kind="gl", n=N, order=1))
    with Server(memory_budget_gb=1.0, steps_per_tick=48, precision=prec) as srv:
        tickets = [srv.submit(spec, steps, "ke") for steps in (119, 48)]
        got = [srv.wait(t) for t in tickets]
    for steps, g in zip((119, 48), got):
        with Job(dict(spec, layout="aa")) as job:
            job.run(steps)
            want = job.moments("ke")
        assert g["mean"] == pytest.approx(want["mean"][0], rel=1e-12)
        assert g["var"] == pytest.approx(want["var"][0], rel=1e-9)
