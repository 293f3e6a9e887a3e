"""More workers never cost the encoder time: their counters and brick ranges lie
in cache lines of their own.  In volumes of one or two bricks a row, eight to
sixteen workers' ranges would share a line, each storing into it for every row
of voxels, and four workers take several times as long as one."""
import os
import time

import numpy as np
import pytest

from paper_2504_04564_amd import _build, vdbc


@pytest.fixture(scope="module", autouse=True)
def lib():
    _build.ensure_built()
    return vdbc.load()


@pytest.mark.parametrize("shape", [(2048, 2048, 1), (512, 512, 40)])
@pytest.mark.parametrize("flags", [0, vdbc.BG_EXPLICIT])
def test_four_workers_are_not_slower_than_one(shape, flags):
    if len(os.sched_getaffinity(0)) < 4:
        pytest.skip("needs four CPUs")
    v = np.zeros(shape, np.float32)
    v[: shape[0] // 8] = 0.5
    best = {1: float("inf"), 4: float("inf")}
    bufs = {}
    for _ in range(6):
        for threads in best:
            t = time.perf_counter()
            bufs[threads], _ = vdbc.encode(v, 0.01, flags=flags, threads=threads)
            best[threads] = min(best[threads], time.perf_counter() - t)
    assert np.array_equal(bufs[1], bufs[4])
    assert best[4] < best[1], best
