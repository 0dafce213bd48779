"""The float32 convolution (forward, input gradient, kernel gradient) against
the float64 oracle at every length of the register transforms: odd batches (a
pair without its second row), several signals in one wave and blocks with empty
signal slots (L <= 512), several row pairs per kernel spectrum (the wide case),
rows of very different scale in one pair and a row whose maximum lies in a
single lane of its last wave."""
import numpy as np
import pytest
import torch

import oracle
from tests._util import check, f32dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h3():
    import paper_2212_14052_amd as h3
    h3.lib()
    return h3


@pytest.mark.parametrize("B,H,L", [(3, 70, 16), (2, 9, 32), (1, 5, 64), (5, 3, 128), (3, 3, 256), (5, 3, 512),
                                   (1, 2, 1024), (5, 2200, 1024), (3, 2, 2048), (5, 2, 4096), (3, 2, 8192)])
def test_conv_f32(h3, B, H, L):
    rng = np.random.default_rng(7 * L + B)
    k = (rng.standard_normal((H, L)) * np.exp(-np.arange(L) / (L / 3))).astype(np.float32)
    u = rng.standard_normal((B, H, L)).astype(np.float32)
    u *= (2.0 ** (6.0 * (np.arange(B) % 3) - 9)).astype(np.float32)[:, None, None]
    # the spike's response lies in the outputs kept: a transform's error is
    # relative to all 2L points, |err| <= c |u|_2 |k|_2 / sqrt(2L) with c about log2(2L)
    # half units, so a spike at L - 1, whose response is cut off after one
    # point, would be measured against 64 u (k_0 + D) however small that is
    u[0, :, L // 8 - 1] *= 64
    dy = rng.standard_normal((B, H, L)).astype(np.float32)
    D = rng.standard_normal(H).astype(np.float32)
    y = h3.fftconv(f32dev(u), f32dev(k), f32dev(D))
    du, dk, _ = h3.fftconv_bwd(f32dev(u), f32dev(k), f32dev(D), f32dev(dy))
    torch.cuda.synchronize()
    sel = np.unique(np.r_[0, H // 2, H - 1])
    u, dy, k, D = (a.astype(np.float64) for a in (u[:, sel], dy[:, sel], k[sel], D[sel]))
    # each radix-2 level of the 2L-point transforms rounds twice (twiddle
    # product, sum) and each value passes two transforms: 4 log2(2L) half units
    # of the rows' scale
    tol = 4 * np.log2(2 * L) * 2.0 ** -24
    check(y.cpu().numpy()[:, sel], oracle.causal_conv(u, k, D), tol)
    corr = oracle.causal_conv(dy[..., ::-1], k, D)[..., ::-1]
    check(du.cpu().numpy()[:, sel], corr, tol)
    N = 2 * L
    dkr = np.fft.irfft(np.conj(np.fft.rfft(u, N)) * np.fft.rfft(dy, N), N)[..., :L].sum(0)
    check(dk.cpu().numpy()[sel], dkr, tol)
