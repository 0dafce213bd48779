"""The layer's sequence mixing by direct summation (L = 256, 512, 1024) against
the float64 oracle: batches that leave a wave's rows unfilled or split a
channel over workgroups, few taps, no skips, both output-projection paths,
and gates far from 1 (G is scaled per row)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests._util import check, f32dev, record, to_dev, to_np64

pytestmark = pytest.mark.gpu

# Q, K, V, O and the output are rounded to 16 bits: five times half a unit in
# the last place of the largest value
TOL = {workloads.F16: 5 * 2.0 ** -12, workloads.BF16: 5 * 2.0 ** -9}


@pytest.fixture(scope="module")
def h3():
    import paper_2212_14052_amd as h3
    h3.lib()
    return h3


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,L,d,m_s,skips,vscale", [
    (1, 256, 128, 64, True, 1.0), (3, 256, 256, 1, False, 1.0), (2, 512, 128, 5, True, 1.0),
    (1, 1024, 256, 64, True, 1.0), (5, 1024, 128, 63, False, 1.0), (17, 1024, 128, 64, True, 1.0),
    (2, 1024, 256, 17, True, 2.0 ** -7), (1, 1024, 640, 64, True, 2.0 ** 6),
])
def test_layer_direct(h3, dtype, B, L, d, m_s, skips, vscale):
    w = workloads.layer_workload("t", B, L, d, dtype, seed=B + L + m_s, m=8, m_shift=m_s)
    A, Bm, C, dt = w.diag.complex64()
    k = oracle.ssm_kernel(A, Bm, C, dt, L).astype(np.float32)
    Wv, Wv64 = workloads.round_to(w.W["v"][1] * vscale, dtype)
    sD = np.linspace(-1, 1, d).astype(np.float32) if skips else None
    dD = w.diag_D if skips else None
    W = {n: to_dev(w.W[n][0], dtype) for n in "qko"}
    out = h3.layer_fwd(to_dev(w.x, dtype), W["q"], W["k"], to_dev(Wv, dtype), W["o"], f32dev(w.shift_C),
                       None if sD is None else f32dev(sD), f32dev(k), None if dD is None else f32dev(dD))
    torch.cuda.synchronize()
    ref = oracle.h3_layer(w.x64, w.W["q"][1], w.W["k"][1], Wv64, w.W["o"][1], w.shift_C.astype(np.float64),
                          k.astype(np.float64), None if dD is None else dD.astype(np.float64),
                          shift_D=None if sD is None else sD.astype(np.float64))
    check(out, ref, TOL[dtype], "out", rows=False)


@pytest.mark.parametrize("B,L", [(1, 256), (3, 1024)])
def test_layer_direct_tiny_gate(h3, B, L):
    """G = Kbar V near 2^-118, whose reciprocal is no float32; Q brings the
    output back into range."""
    d, dtype = 128, workloads.BF16
    w = workloads.layer_workload("t", B, L, d, dtype, seed=L, m=8, m_shift=64)
    A, Bm, C, dt = w.diag.complex64()
    k = oracle.ssm_kernel(A, Bm, C, dt, L).astype(np.float32)
    W = {n: workloads.round_to(w.W[n][1] * s, dtype)
         for n, s in (("q", 2.0 ** 30), ("k", 2.0 ** -10), ("v", 2.0 ** -110), ("o", 1.0))}
    out = h3.layer_fwd(to_dev(w.x, dtype), *(to_dev(W[n][0], dtype) for n in "qkvo"), f32dev(w.shift_C), None,
                       f32dev(k), f32dev(w.diag_D))
    torch.cuda.synchronize()
    ref = oracle.h3_layer(w.x64, *(W[n][1] for n in "qkvo"), w.shift_C.astype(np.float64), k.astype(np.float64),
                          w.diag_D.astype(np.float64))
    check(out, ref, TOL[dtype], "out", rows=False)


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("L", [256, 512, 1024])
@pytest.mark.parametrize("which", ["taps", "kernel"])
def test_layer_direct_cancelling(h3, dtype, L, which):
    """Q, K, V of ones and an output projection that changes nothing, so that
    the output is the running sum of the shift taps (the diagonal kernel a
    unit) or of the diagonal kernel (one tap of 1/3, so that G is no 16-bit
    value): in threes they sum to nothing, and every third output is the error
    of what the float32 parameters are held in and of the sums.  fp16 pairs are
    off by 2^-23, 2^-22 where the low halves' product is left out, at random:
    2^-24 sqrt(n) of the rms.  The partial sums, of 32 terms that split the
    threes, wander to sqrt(n / 32) rms and are rounded to 2^-24 of themselves
    3 n / 32 times: 2^-25 sqrt(3) n / 32, at n = 1024 as much.  Four deviations
    of the two are below 2^-21 sqrt(n) (the float32 transform: 3.6e-6 at L =
    1024 with its kernel of rms 0.38; bf16 pieces of a tap: 2^-18 sqrt(n)).  The
    output is rounded once."""
    B, d = 3, 128
    rng = np.random.default_rng(L)
    n = 63 if which == "taps" else L
    a = rng.standard_normal((d, n // 3 + 1, 3))
    a[..., 2] = -a[..., 0] - a[..., 1]
    p = a.reshape(d, -1)[:, :n].astype(np.float32)
    if which == "taps":
        taps, k = p, np.zeros((d, L), np.float32)
        k[:, 0] = 1.0
        unit = 1.0
    else:
        taps, k = np.full((d, 1), 1 / 3, np.float32), p
        unit = float(taps[0, 0])
    x = torch.zeros((B, L, d), device="cuda")
    x[..., 0] = 1.0
    one = torch.zeros((d, d), device="cuda")
    one[0] = 1.0
    t = torch.float16 if dtype == workloads.F16 else torch.bfloat16
    out = h3.layer_fwd(x.to(t), *(w.to(t) for w in (one, one, one, torch.eye(d, device="cuda"))), f32dev(taps), None,
                       f32dev(k), None)
    torch.cuda.synchronize()
    ref = np.cumsum(p.astype(np.float64), axis=1)[:, 2::3].T * unit
    err = np.abs(to_np64(out)[:, 2:n:3] - ref).max()
    tol = 2.0 ** -21 * np.sqrt(n * np.mean(p.astype(np.float64) ** 2)) * unit
    tol += np.abs(ref).max() * (2.0 ** -8 if dtype == workloads.BF16 else 2.0 ** -11)
    record(f"cancelling layer {which} {dtype} L={L}", err=float(err), tol=float(tol))
    assert err < tol, (err, tol)
