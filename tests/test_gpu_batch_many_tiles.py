"""A batch with more tiles than one launch holds (2^32 threads): 65536 frames of 257 symbols."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from rxgen import C2, make_frames  # noqa: E402
from tests.parity import as_complex, check_xhat  # noqa: E402


@pytest.fixture(scope="module")
def rx():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_1901_07499_amd import rx as mod
    return mod


def test_more_tiles_than_a_launch_holds(rx):
    n = 65536
    cfg = C2.replace(n_ant=1, fft_len=64, cp_len=0, n_used=4, n_sym=257, bits_per_sym=4, n_slots=1, snr_db=(30.0, 30.0))
    print("[case] batch tiles", n, cfg.n_sym, flush=True)
    fr = make_frames(cfg, n_slots=1)
    batch = rx.Batch([cfg] * n, [fr.pilot] * n)
    iq = torch.from_numpy(fr.iq.reshape(1, -1)).cuda().expand(n, -1).reshape(-1)
    out = batch.outputs(iq.device, want_H=False)
    out[1].fill_(float("nan"))
    out[2].fill_(0xAA)
    batch.process(iq, out)
    torch.cuda.synchronize()
    x, bits = out[1].view(n, cfg.n_sym - 1, cfg.n_used, 2), out[2].view(n, -1)
    check_xhat(as_complex(x[:1]), oracle.run_config(fr).xhat)
    assert (x == x[0]).all() and (bits == bits[0]).all()
    lat = batch.frame_latency_ms()
    assert np.all(lat > 0) and np.all(lat < 1e4)
