"""Batches at the default configuration (one pair of kernels over all FFT lengths) against the FP64 oracle:
4- and 8-wavefront workgroups, spectra inside and past the 5-register window, a single frame, and replays."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from rxgen import make_batch  # noqa: E402
from tests.test_gpu_batch import _check_frames  # noqa: E402


@pytest.fixture(scope="module")
def rx():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_1901_07499_amd import rx as mod
    return mod


# frames, seed, antennas, FFT lengths: short tiles only (4 wavefronts), long ones in a small batch (8), long ones
# that a larger batch hides (4); lengths 64 and 256 have wide spectra, the others narrow ones
@pytest.mark.parametrize("n,seed,antennas,lens", [
    (40, 51, (1, 5, 16), (64, 128, 256, 512)), (6, 52, (9, 33), (64, 128, 256, 512, 1024, 2048)),
    (1, 53, (7,), (2048,)), (1, 54, (130,), (64,)), (70, 55, (1, 2, 8), (64, 1024, 2048)),
    (120, 56, (4, 5), (2048,))])
def test_merged_batch_matches_oracle(rx, n, seed, antennas, lens):
    print("[case] merged batch", n, seed, antennas, lens, flush=True)
    bt = make_batch(n, seed, antennas=antennas, fft_lens=lens)
    batch = rx.Batch(bt.configs, [f.pilot for f in bt.frames])
    iq = torch.from_numpy(bt.iq).cuda()
    refs = [oracle.run_config(fr) for fr in bt.frames]
    out = batch.outputs(iq.device)
    first = None
    for rep in range(3):
        for o in out[:3]:
            o.fill_(float("nan") if o.is_floating_point() else 0xAA)
        batch.process(iq, out)
        torch.cuda.synchronize()
        _check_frames(batch, bt, *out[:3], refs=refs)
        lat = batch.frame_latency_ms()
        assert np.all(lat > 0) and np.all(lat < 1e4)
        if first is not None:
            assert torch.equal(out[1], first)
        first = out[1].clone()
    # the kernels per FFT length give the same samples of x-hat within the same bounds
    for m in sorted({c.fft_len for c in bt.configs}):
        batch.set_config(m, 4, 2, 0, 0)
    batch.process(iq, out)
    torch.cuda.synchronize()
    _check_frames(batch, bt, *out[:3], refs=refs)
