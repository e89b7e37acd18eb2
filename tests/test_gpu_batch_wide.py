"""Batches that hold frames of both merged kernel pairs (spectra inside and past the narrow register window) at every
FFT length, with 4- and with 8-wavefront demod workgroups, against the FP64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from rxgen import C2, make_frames  # noqa: E402
from tests.test_gpu_batch import _check_frames  # noqa: E402


@pytest.fixture(scope="module")
def rx():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_1901_07499_amd import rx as mod
    return mod


NARROW = {64: 52, 128: 108, 256: 220, 512: 300, 1024: 636, 2048: 1200}
WIDE = {64: 60, 128: 124, 256: 252, 512: 444, 1024: 900, 2048: 1700}


def _wide(c):
    """More registers per lane than the narrow kernels hold: 7 up to 256 points, 5 above."""
    lanes = c.fft_len // 16
    return -(-(c.n_used // 2 + 1) // lanes) > (7 if c.fft_len <= 256 else 5)


class _Frames:
    def __init__(self, configs):
        self.configs = configs
        self.frames = [make_frames(c) for c in configs]
        self.iq = np.concatenate([f.iq.reshape(-1) for f in self.frames])


# (antennas of the frames of each length, copies of the set, wavefronts): the longest tile past 8 transforms of 1024
# points in a small batch takes 8, tiles up to that length take 4
@pytest.mark.parametrize("ants,copies,waves", [((130, 3, 5, 9, 7, 6), 1, 8), ((3, 60, 31, 5, 6, 4), 2, 4)])
def test_narrow_and_wide_frames_in_one_batch(rx, ants, copies, waves):
    print("[case] batch wide", ants, copies, waves, flush=True)
    cfgs = []
    for k in range(copies):
        for i, (n, a) in enumerate(zip(NARROW, ants)):
            for used in (NARROW[n], WIDE[n]):
                cfgs.append(C2.replace(n_ant=a, fft_len=n, cp_len=n // 16 + (i + k) % 2, n_used=used, n_sym=3 + i % 3,
                                       bits_per_sym=(2, 4, 6)[i % 3], n_slots=1))
    longest = max(c.n_ant * c.fft_len for c in cfgs)
    tiles = sum(c.n_ant * c.fft_len * (c.n_sym - 1) for c in cfgs)
    assert waves == (8 if longest > 8 * 1024 and 5 * tiles <= 6 * longest * 256 else 4)
    assert {(c.fft_len, _wide(c)) for c in cfgs} == {(n, w) for n in NARROW for w in (False, True)}
    bt = _Frames(cfgs)
    refs = [oracle.run_config(fr) for fr in bt.frames]
    batch = rx.Batch(bt.configs, [f.pilot for f in bt.frames])
    iq = torch.from_numpy(bt.iq).cuda()
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
