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
from tests._util import check, f32dev, to_dev

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
