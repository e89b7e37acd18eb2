"""Calls on both sides of the lines at which the 128- and 256-point demod changes its register window, against the
FP64 oracle and with every slot of a call the same."""
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


# workgroups of 8 items (128 points) or 4 (256): 512 and 768, 769 and 1024, 1025
@pytest.mark.parametrize("N,U,per_group", [(128, 108, 8), (256, 180, 4), (256, 220, 4)])
@pytest.mark.parametrize("A", [31, 32])
def test_window_lines(rx, N, U, per_group, A):
    cfg = C2.replace(n_ant=A, fft_len=N, cp_len=N // 16, n_used=U, n_sym=2, bits_per_sym=4, n_slots=2)
    fr = make_frames(cfg)
    ref = oracle.process_frame(fr.iq, fr.pilot, n_ant=A, fft_len=N, cp_len=cfg.cp_len, n_used=U, n_sym=2,
                               bits_per_sym=4)
    plan = rx.Plan.from_config(cfg, fr.pilot)
    for groups in (512, 513, 768, 769, 1024, 1025):
        S = groups * per_group
        print("[case] window line", N, U, A, groups, flush=True)
        src = np.arange(S) % 2
        iq = torch.from_numpy(fr.iq).cuda()[torch.from_numpy(src).cuda()].contiguous()
        _, x, b = plan.process(iq)
        torch.cuda.synchronize()
        assert torch.equal(x[2:], x[:2].repeat(S // 2, 1, 1, 1)[2:]) and torch.equal(b[2:], b[:2].repeat(S // 2, 1, 1)[2:])
        check_xhat(as_complex(x[:2]), ref.xhat)
        check_bits(b[:2].cpu().numpy(), ref.bits, ref.xhat, 4)
