"""One call's forms against each other and the FP64 oracle.  Without H: x-hat and bits together, each alone, and the
call that allocates nothing give the same bits.  With H: the whole call and estimate followed by demod give the same
bits.  The two sides, which may sum in another order, both hold the oracle's bounds."""
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


def _noalloc(rx, plan, iq, want_xhat=True, want_bits=True):
    S, Td = iq.shape[0], plan.n_sym - 1
    x = torch.full((S, Td, plan.n_used, 2), float("nan"), device="cuda") if want_xhat else None
    b = torch.full((S, Td, plan.row_bytes), 0xAA, dtype=torch.uint8, device="cuda") if want_bits else None
    st = rx.rx_process_frame_noalloc(plan._plan, iq.data_ptr(), S, x.data_ptr() if want_xhat else None,
                                     b.data_ptr() if want_bits else None, torch.cuda.current_stream().cuda_stream)
    assert st == rx.RX_OK, st
    return x, b


# one group of antennas; several groups (subcarriers that end inside and at the end of a finishing workgroup's 256); the
# two kernels with 8 wavefronts; a call past the small ones; as many antennas as 4 wavefronts transform, and one more
@pytest.mark.parametrize("A,N,U,T,S", [(8, 64, 52, 11, 1), (17, 512, 300, 3, 1), (64, 1024, 600, 14, 1),
                                       (64, 1024, 512, 6, 2), (41, 2048, 1200, 5, 1), (24, 1024, 600, 14, 2),
                                       (12, 256, 180, 8, 60), (1, 2048, 1200, 5, 2), (2, 2048, 1700, 3, 1),
                                       (3, 2048, 1200, 3, 1)])
@pytest.mark.parametrize("zf,bits", [(0, 2), (0, 4), (1, 4), (0, 6), (1, 2)])
def test_forms_of_a_call(rx, A, N, U, T, S, zf, bits):
    cfg = C2.replace(n_ant=A, fft_len=N, cp_len=N // 16 + 1, n_used=U, n_sym=T, bits_per_sym=bits, n_slots=S)
    print("[case] forms", A, N, U, T, S, zf, bits, flush=True)
    uniq = min(S, 2)
    fr = make_frames(cfg, n_slots=uniq)
    src = np.arange(S) % uniq
    iq = torch.from_numpy(fr.iq).cuda()[torch.from_numpy(src).cuda()].contiguous()
    plan = rx.Plan.from_config(cfg, fr.pilot, zf)
    _, x, b = plan.process(iq)
    _, x1, _ = plan.process(iq, want_bits=False)
    _, _, b1 = plan.process(iq, want_xhat=False)
    xn, bn = _noalloc(rx, plan, iq)
    xn1, _ = _noalloc(rx, plan, iq, want_bits=False)
    _, bn1 = _noalloc(rx, plan, iq, want_xhat=False)
    H, xh, bh = plan.process(iq, want_H=True)
    _, xh1, _ = plan.process(iq, want_H=True, want_bits=False)
    H2 = plan.estimate(iq)
    x2, b2 = plan.demod(iq, H2)
    torch.cuda.synchronize()
    for other in (x1, xn, xn1):
        assert torch.equal(x, other)
    for other in (b1, bn, bn1):
        assert torch.equal(b, other)
    assert torch.equal(H, H2) and torch.equal(xh, x2) and torch.equal(xh, xh1) and torch.equal(bh, b2)
    ref = oracle.process_frame(fr.iq, fr.pilot, n_ant=A, fft_len=N, cp_len=cfg.cp_len, n_used=U, n_sym=T,
                               bits_per_sym=bits)
    check_H(as_complex(H), ref.H[src])
    for got, dec in ((x, b), (xh, bh)):
        check_xhat(as_complex(got), ref.xhat[src])
        check_bits(dec.cpu().numpy(), ref.bits[src], ref.xhat[src], bits)


# estimates of 39 MB a slot, so each slot is a chunk of its own: with antenna groups, and (comb pilot) the two kernels
@pytest.mark.parametrize("spacing", [1, 4])
def test_small_noalloc_call_in_chunks(rx, spacing):
    A, N, CP, U, T, S = 4096, 2048, 16, 1200, 3, 3
    print("[case] chunks", spacing, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    iq = torch.randint(-9000, 9001, (S, T, A, CP + N, 2), generator=gen, device="cuda", dtype=torch.int16)
    plan = rx.Plan(A, N, CP, U, T, 4, np.exp(2j * np.pi * np.random.default_rng(5).random(U)), pilot_spacing=spacing)
    assert 2 * A * U * 8 > rx.RX_NOALLOC_SCRATCH_BYTES >= A * U * 8
    _, x, b = plan.process(iq)
    xn, bn = _noalloc(rx, plan, iq)
    torch.cuda.synchronize()
    assert torch.equal(x, xn) and torch.equal(b, bn)
