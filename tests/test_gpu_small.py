"""Calls too small to fill the GPU: the one-kernel path, 8-wavefront workgroups per item, and transform
slots of a wavefront split over an item's antennas, against the FP64 oracle and against each other."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from rxgen import C2, make_frames  # noqa: E402
from tests.parity import as_complex, check_bits, check_xhat  # noqa: E402


@pytest.fixture(scope="module")
def rx():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_1901_07499_amd import rx as mod
    return mod


# (antennas, FFT length, subcarriers, symbols, slots): one antenna; one group of antennas, with idle transform
# slots, exactly full, and one past; several groups with an uneven last one; every spectrum window; the last small
# call and the first that is not (256 items); the split of a wavefront's slots with the antennas ending mid-job,
# with unaligned records (odd cyclic prefix), and with items ending mid-workgroup
CASES = [(1, 64, 52, 2, 1), (8, 64, 52, 11, 1), (128, 64, 16, 3, 1), (129, 64, 60, 3, 2), (16, 128, 72, 14, 3),
         (13, 512, 300, 8, 2), (17, 512, 120, 3, 1), (33, 512, 440, 3, 1), (64, 1024, 600, 14, 1),
         (37, 1024, 900, 14, 2), (9, 1024, 200, 3, 1), (41, 2048, 1200, 14, 1), (5, 2048, 400, 2, 1),
         (30, 2048, 1700, 5, 1), (3, 256, 180, 3, 128), (3, 256, 180, 2, 257), (21, 128, 72, 14, 37),
         (100, 64, 52, 14, 20), (35, 256, 92, 8, 41), (18, 512, 300, 8, 40)]


@pytest.mark.parametrize("A,N,U,T,S", CASES)
@pytest.mark.parametrize("cp_odd", [0, 1])
def test_small_calls(rx, A, N, U, T, S, cp_odd):
    cfg = C2.replace(n_ant=A, fft_len=N, cp_len=N // 16 + cp_odd, n_used=U, n_sym=T, bits_per_sym=6, n_slots=S)
    print("[case] small", A, N, U, T, S, cp_odd, flush=True)
    uniq = min(S, 3)
    fr = make_frames(cfg, n_slots=uniq)
    src = np.arange(S) % uniq
    iq = torch.from_numpy(fr.iq).cuda()[torch.from_numpy(src).cuda()].contiguous()
    plan = rx.Plan.from_config(cfg, fr.pilot)
    x = torch.full((S, T - 1, U, 2), float("nan"), device="cuda")
    b = torch.full((S, T - 1, plan.row_bytes), 0xAA, dtype=torch.uint8, device="cuda")
    ws = torch.full((plan.workspace_bytes(S) + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    plan.process(iq, out=(None, x, b), workspace=ws)
    _, xh, bh = plan.process(iq, want_H=True)      # the estimate for the caller: the two kernels
    torch.cuda.synchronize()
    assert (ws[plan.workspace_bytes(S):] == 0xFF).all()
    ref = oracle.process_frame(fr.iq, fr.pilot, n_ant=A, fft_len=N, cp_len=cfg.cp_len, n_used=U, n_sym=T,
                               bits_per_sym=6)
    for got, bits in ((x, b), (xh, bh)):
        check_xhat(as_complex(got), ref.xhat[src])
        check_bits(bits.cpu().numpy(), ref.bits[src], ref.xhat[src], 6)
