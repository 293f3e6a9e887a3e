"""The encoder's background where its one-pass count of a sampled candidate
decides, and where it must not: candidates that are not the mode, ties, both
zeros, brick rows of one value beside mixed ones, and rows holding NaN."""
import numpy as np
import pytest

import oracle
from paper_2504_04564_amd import _build, vdbc


@pytest.fixture(scope="module", autouse=True)
def lib():
    _build.ensure_built()
    return vdbc.load()


def _volume(kind, shape):
    rng = np.random.default_rng(5)
    n = int(np.prod(shape))
    v = rng.random(n).astype(np.float32)
    at = [i * (n - 1) // 60 for i in range(61)]          # where the candidate is sampled
    if kind == "sampled value is rare":
        v[rng.random(n) < 0.3] = -2.0
        v[at] = 7.0
    elif kind == "mode in the sampled value's bucket":
        v[:] = np.float32(1.0)
        v[: n // 3] = np.nextafter(np.float32(1.0), np.float32(2.0))
        v[at] = np.nextafter(np.float32(1.0), np.float32(2.0))
    elif kind == "tie goes to the smallest":
        v = np.tile(np.array([3.0, -1.0], np.float32), (n + 1) // 2)[:n]
    elif kind == "both zeros":
        v[rng.random(n) < 0.35] = 0.0
        v[rng.random(n) < 0.35] = -0.0
    elif kind == "rows of one value":
        v = v.reshape(shape)
        v[:, ::2] = 0.5
        v[:, 1::4, :40] = -0.0
    elif kind == "one value":
        v[:] = -3.25
    return np.ascontiguousarray(v.reshape(shape))


@pytest.mark.parametrize("shape", [(33, 40, 70), (1, 1, 3), (5, 64, 64)])
@pytest.mark.parametrize("kind", ["sampled value is rare", "mode in the sampled value's bucket",
                                  "tie goes to the smallest", "both zeros", "rows of one value", "one value"])
@pytest.mark.parametrize("threads", [1, 5])
def test_buffer_is_the_oracles(shape, kind, threads):
    v = _volume(kind, shape)
    buf, st = vdbc.encode(v, 0.4, threads=threads)
    want, _ = oracle.encode(v, 0.4)
    assert st["background"] == np.float32(oracle.background(v))
    assert bytes(buf) == bytes(want)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_row_of_non_finite_values_is_refused(bad):
    v = np.zeros((9, 9, 70), np.float32)
    v[4, 4, 32:64] = bad
    with pytest.raises(vdbc.VdbcError):
        vdbc.encode(v, 0.4)
