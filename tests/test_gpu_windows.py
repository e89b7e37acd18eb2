"""Spectrum windows of 6, 7 and 8 registers in calls past the small-call paths, and in a batch, against the FP64
oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from rxgen import C2, make_frames  # noqa: E402
from tests.parity import as_complex, check_bits, check_H, check_xhat  # noqa: E402


@pytest.fixture(scope="module")
def rx():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_1901_07499_amd import rx as mod
    return mod


# the least and the greatest multiple of four subcarriers of each window
@pytest.mark.parametrize("N,U", [(64, 40), (64, 44), (64, 48), (64, 52), (64, 56), (64, 60), (128, 80), (128, 92),
                                 (128, 96), (128, 108), (128, 112), (128, 124), (256, 160), (256, 188), (256, 192),
                                 (256, 220), (256, 224), (256, 252), (512, 324), (512, 380), (512, 384), (512, 444), (1024, 644),
                                 (1024, 764), (1024, 768), (1024, 892), (2048, 1284), (2048, 1532), (2048, 1536), (2048, 1788)])
@pytest.mark.parametrize("A,cp_odd", [(3, 0), (10, 1)])
def test_wide_windows(rx, N, U, A, cp_odd):
    S = 700 if N < 512 else 90                     # past the split of a wavefront's slots over antennas
    cfg = C2.replace(n_ant=A, fft_len=N, cp_len=N // 16 + cp_odd, n_used=U, n_sym=4, bits_per_sym=4, n_slots=S)
    print("[case] window", N, U, A, cp_odd, flush=True)
    fr = make_frames(cfg, n_slots=2)
    src = np.arange(S) % 2
    iq = torch.from_numpy(fr.iq).cuda()[torch.from_numpy(src).cuda()].contiguous()
    plan = rx.Plan.from_config(cfg, fr.pilot)
    H, x, b = plan.process(iq, want_H=True)
    torch.cuda.synchronize()
    ref = oracle.process_frame(fr.iq, fr.pilot, n_ant=A, fft_len=N, cp_len=cfg.cp_len, n_used=U, n_sym=4,
                               bits_per_sym=4)
    check_H(as_complex(H), ref.H[src])
    check_xhat(as_complex(x), ref.xhat[src])
    check_bits(b.cpu().numpy(), ref.bits[src], ref.xhat[src], 4)
    batch = rx.Batch([cfg] * 2, [fr.pilot] * 2)
    out = batch.outputs(iq.device)
    batch.process(iq[:2].contiguous(), out)
    torch.cuda.synchronize()
    check_xhat(as_complex(out[1].view(2, 3, U, 2)), ref.xhat)
