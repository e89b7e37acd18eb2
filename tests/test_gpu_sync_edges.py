"""Preamble metric at the edges of its tiles, bit for bit against the oracle: the chip counts at which the matrix
product takes one more step of 64 (L + 15 = 64 k, 64 k + 1), and candidate counts around a row, a wavefront's 256
and a workgroup's 1024, with streams that end inside the window."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.test_gpu_sync import _check_find, rx  # noqa: E402,F401


@pytest.mark.parametrize("L", [1, 48, 49, 50, 113, 114, 511, 512, 1009, 1010])
@pytest.mark.parametrize("n_search", [1, 15, 17, 255, 257, 1023, 1025])
def test_metric_tile_edges(rx, L, n_search):  # noqa: F811
    print("[case] sync edges", L, n_search, flush=True)
    rng = np.random.default_rng([L, n_search])
    n = n_search + L // 2 + 1                      # the last windows run past the stream's end
    raw = rng.integers(-32768, 32768, size=(3, n + 5, 2)).astype(np.int16)
    raw[1] = rng.choice([-32768, 32767], size=(n + 5, 2))
    _check_find(rx, raw, rng.choice([-1, 1], size=L), n_search, n_samples=n)
