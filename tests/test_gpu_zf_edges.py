"""ZF where the channel energy overflows or a channel is not finite, as its weights conj(H) / g have it: finite
channels give 0 once g overflows (also where the sum over the antennas would overflow too), a channel that is not
finite gives NaN, and an energy close below the overflow an ordinary quotient."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rx():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_1901_07499_amd import rx as mod
    return mod


def _iq(S, T, A, L, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-9000, 9001, (S, T, A, L, 2), generator=g, device="cuda", dtype=torch.int16)


def _spectra(iq, N, CP, U):
    """Used bins of every data symbol, complex128 [S][T-1][A][U] (tensors on the GPU in 64 bits)."""
    y = iq[:, 1:, :, CP:].double()
    bins = torch.cat([torch.arange(N - U // 2, N), torch.arange(1, U // 2 + 1)]).cuda()
    return torch.fft.fft(torch.complex(y[..., 0], y[..., 1]))[..., bins]


# an 8-wavefront workgroup per item; several items per workgroup: a transform slot per item, wavefronts that share
# an item, slots that share one; 4-wavefront workgroups of one- and two-wavefront transforms
SHAPES = [(3, 1024, 600, 5, 2), (1, 64, 52, 4, 900), (20, 128, 72, 5, 700), (20, 128, 72, 14, 25), (40, 1024, 600, 5, 70),
          (9, 2048, 1200, 5, 70)]


@pytest.mark.parametrize("A,N,U,T,S", SHAPES)
def test_zf_demod_channel_edges(rx, A, N, U, T, S):
    print("[case] zf edges", A, N, U, T, S, flush=True)
    CP = N // 16
    iq = _iq(S, T, A, N + CP, 7)
    plan = rx.Plan(A, N, CP, U, T, 2, np.ones(U), combiner=1)
    gen = torch.Generator(device="cuda").manual_seed(8)
    H = torch.randn((S, A, U, 2), generator=gen, device="cuda")
    kind = torch.arange(U, device="cuda") % 6
    H[:, :, kind == 1] *= 1e33                      # the sum over the antennas overflows with the energy
    H[:, :, kind == 2] *= 1e22                      # the energy alone
    H[:, A - 1, kind == 3, 1] = float("nan")
    H[:, A // 2, kind == 4, 0] = float("-inf")
    near = H[:, :, kind == 5].double()              # energies of 1.5e38, subnormal reciprocals
    H[:, :, kind == 5] = (near * torch.sqrt(1.5e38 / (near ** 2).sum((1, 3), keepdim=True))).float()
    x, b = plan.demod(iq, H)
    torch.cuda.synchronize()
    assert (x[:, :, (kind == 1) | (kind == 2)] == 0).all()
    assert torch.isnan(x[:, :, (kind == 3) | (kind == 4)]).all()
    fine = (kind == 0) | (kind == 5)
    Hc = torch.view_as_complex(H.double())[:, :, fine]
    Y = _spectra(iq, N, CP, U)[..., fine]
    ref = (Hc.conj()[:, None] * Y).sum(2) / (Hc.abs() ** 2).sum(1)[:, None]
    err = (torch.view_as_complex(x[:, :, fine].double()) - ref).abs()
    # FP32 products and sums of magnitudes at most sum |h| |y| / g, and an FFT within 1e-6 of its largest bin
    scale = (Hc.abs().sum(1)[:, None] * Y.abs().amax((2, 3), keepdim=True)[..., 0]) / (Hc.abs() ** 2).sum(1)[:, None]
    assert (err <= 1e-5 * scale).all()


@pytest.mark.parametrize("A,N,U,T,S", [(8, 64, 52, 11, 1), (64, 1024, 600, 14, 1), (64, 1024, 600, 14, 30)])
@pytest.mark.parametrize("want_H", [False, True])
@pytest.mark.parametrize("pilot,want", [(1e-26, 0.0), (1e-40, float("nan"))])
def test_zf_process_pilot_edges(rx, A, N, U, T, S, want_H, pilot, want):
    # a pilot this small makes the estimates so large that the energy overflows (1e-26) or that they overflow (1e-40)
    print("[case] zf pilot", A, N, U, T, S, want_H, pilot, flush=True)
    CP = N // 16
    iq = _iq(S, T, A, N + CP, 9)
    plan = rx.Plan(A, N, CP, U, T, 2, np.full(U, pilot), combiner=1)
    _, x, _ = plan.process(iq, want_H=want_H)
    torch.cuda.synchronize()
    assert torch.isnan(x).all() if np.isnan(want) else (x == want).all()
