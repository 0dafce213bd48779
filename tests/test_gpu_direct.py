"""The convolution of 16-bit rows by direct summation (L = 256, 512, 1024) and
by the float32 transform at 4096, forward and as the input gradient, against
the float64 oracle: batches that leave a wave's rows or a workgroup's waves
unfilled, channel counts that split a channel over workgroups, few and many
rows per kernel spectrum at 4096, kernels and inputs far from 1."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests._util import check, f32dev, record, to_dev, to_np64

pytestmark = pytest.mark.gpu

# the output's own rounding, half a unit in the last place of the largest value
# (2^-11, 2^-8 halved), and a tenth for the sums
TOL = {workloads.F16: 1.1 * 2.0 ** -11, workloads.BF16: 1.1 * 2.0 ** -9 * 2}


@pytest.fixture(scope="module")
def h3():
    import paper_2212_14052_amd as h3
    h3.lib()
    return h3


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,H,L", [(1, 3, 256), (5, 2, 256), (2, 3, 512), (35, 2, 512), (1, 2, 1024), (3, 5, 1024),
                                   (16, 3, 1024), (33, 1, 1024), (1, 1280, 4096), (5, 256, 4096), (3, 426, 4096),
                                   (160, 8, 4096)])
def test_conv_direct(h3, dtype, B, H, L):
    w = workloads.conv_workload("t", B, H, L, dtype, seed=3 * B + L, m=4)
    A, Bm, C, dt = w.ssm.complex64()
    k = oracle.ssm_kernel(A, Bm, C, dt, L).astype(np.float32)
    u = to_dev(w.u, dtype)
    y = h3.fftconv(u, f32dev(k), f32dev(w.D))
    du, _, _ = h3.fftconv_bwd(None, f32dev(k), f32dev(w.D), u, want_dk=False, want_dD=False)
    torch.cuda.synchronize()
    sel = np.unique(np.r_[0, H // 2, H - 1])
    k64, D64 = k[sel].astype(np.float64), w.D[sel].astype(np.float64)
    x = np.ascontiguousarray(w.u64[:, sel])
    check(y[:, sel.tolist()], oracle.causal_conv(x, k64, D64), TOL[dtype], "y")
    ref = oracle.causal_conv(np.ascontiguousarray(x[..., ::-1]), k64, D64)[..., ::-1]
    check(du[:, sel.tolist()], np.ascontiguousarray(ref), TOL[dtype], "du")


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("ks,us", [(1e-6, 1.0), (300.0, 1.0), (1.0, 2.0 ** -9), (1.0, 256.0), (0.0, 1.0)])
def test_conv_direct_ranges(h3, dtype, ks, us):
    B, H, L = 3, 4, 1024
    rng = np.random.default_rng(5)
    u_s, u64 = workloads.round_to(rng.standard_normal((B, H, L)) * us, dtype)
    # taps over six decades within one kernel
    k = (rng.standard_normal((H, L)) * 10.0 ** rng.uniform(-6, 0, (H, L)) * ks).astype(np.float32)
    if dtype == workloads.F16 and ks < 1e-3:
        u_s, u64 = workloads.round_to(u64 * 1e3, dtype)   # outputs above fp16's subnormals
    y = h3.fftconv(to_dev(u_s, dtype), f32dev(k))
    torch.cuda.synchronize()
    check(y, oracle.causal_conv(u64, k.astype(np.float64), None), TOL[dtype], "y")


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("L", [256, 512, 1024])
def test_conv_direct_cancelling_taps(h3, dtype, L):
    """Taps that sum to nothing in threes against a constant row: what is left
    of them at every third output is the error of the taps and of the sums.
    An fp16 pair holds a tap to 2^-23 of itself and the sums round to 2^-24 per
    32 terms, together below 2^-22 sqrt(L) of the taps' rms, and the result is
    rounded once (bf16 pieces of a tap: 2^-17 of it)."""
    B, H = 3, 4
    rng = np.random.default_rng(L)
    a = rng.standard_normal((H, L // 3 + 1, 3))
    a[..., 2] = -a[..., 0] - a[..., 1]
    k = a.reshape(H, -1)[:, :L].astype(np.float32)
    D = np.full(H, 3.0, np.float32)
    k[:, 0] -= D                      # the skip weight is part of tap 0
    u = np.zeros((B, H, L)) + 1.0
    u_s, u64 = workloads.round_to(u, dtype)
    ud = to_dev(u_s, dtype)
    y = h3.fftconv(ud, f32dev(k), f32dev(D))
    du, _, _ = h3.fftconv_bwd(None, f32dev(k), f32dev(D), ud, want_dk=False, want_dD=False)
    torch.cuda.synchronize()
    kd = k.astype(np.float64)
    kd[:, 0] = (k[:, 0] + D).astype(np.float32)
    ref = np.cumsum(kd, axis=1)[:, 2::3]
    tol = 2.0 ** -22 * np.sqrt(L * np.mean(kd ** 2)) + np.abs(ref).max() * (2.0 ** -8 if dtype == workloads.BF16 else 2.0 ** -11)
    for what, v in (("y", y), ("du", torch.flip(du, (-1,)))):
        err = np.abs(to_np64(v)[..., 2::3] - ref).max()
        record(f"cancelling {what} {dtype} L={L}", err=float(err), tol=float(tol))
        assert err < tol, (what, err, tol)


@pytest.mark.parametrize("us", [2.0 ** -100, 2.0 ** 100])
def test_conv_direct_bf16_scales(h3, us):
    """bf16 rows far outside fp16's range, row by row, and one with an infinity,
    which leaves the other rows alone."""
    B, H, L = 5, 3, 512
    rng = np.random.default_rng(7)
    scale = us ** rng.uniform(0, 1, (B, H, 1))
    u_s, u64 = workloads.round_to(rng.standard_normal((B, H, L)) * scale, workloads.BF16)
    k = rng.standard_normal((H, L)).astype(np.float32)
    u = to_dev(u_s, workloads.BF16)
    u[1, 2, 100] = float("inf")
    y = to_np64(h3.fftconv(u, f32dev(k)))
    ref = oracle.causal_conv(u64, k.astype(np.float64), None)
    assert not np.isfinite(y[1, 2, 100:]).any()
    y[1, 2], ref[1, 2] = 1.0, 1.0
    n = np.abs(ref).max(axis=-1, keepdims=True)
    check(y / n, ref / n, TOL[workloads.BF16], "y")
