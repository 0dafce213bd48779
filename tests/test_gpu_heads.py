"""The layer with heads where the convolution forms the outer products Kbar_i
V_j in its own loads (L = 256, 512, 1024 and 2048), against the float64 oracle:
every head dimension, odd batches (a pair without its second row, waves
without rows), the one- and two-channel forms at 2048 and a channel split over
workgroups (B = 16)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests._util import check, f32dev, to_dev

pytestmark = pytest.mark.gpu

# Q, K, V, Kbar, the products, their convolution and O are rounded to 16 bits
# on the way to the output, and it is: eight times half a unit in the last
# place of the largest value; the convolution at 2048 has fp16 operands
# (another two)
TOL = {workloads.F16: 10 * 2.0 ** -12, workloads.BF16: 10 * 2.0 ** -9}


@pytest.fixture(scope="module")
def h3():
    import paper_2212_14052_amd as h3
    h3.lib()
    return h3


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,L,d,dh", [(1, 256, 128, 2), (3, 512, 128, 4), (5, 1024, 128, 8), (2, 1024, 256, 2),
                                      (1, 2048, 128, 8), (3, 2048, 256, 2), (5, 2048, 128, 4), (16, 2048, 128, 2)])
def test_layer_heads_products_in_conv(h3, dtype, B, L, d, dh):
    w = workloads.layer_workload("t", B, L, d, dtype, seed=B + L + dh, m=8, m_shift=16)
    rng = np.random.default_rng(L + 10 * dh + B)
    ssm = workloads.make_diag_ssm(rng, d * dh, 8, 1e-3, 1e-1)
    k = oracle.ssm_kernel(*ssm.complex64(), L).astype(np.float32)
    dD = rng.standard_normal(d * dh).astype(np.float32)
    W = {n: to_dev(w.W[n][0], dtype) for n in "qkvo"}
    out = h3.layer_fwd_heads(to_dev(w.x, dtype), W["q"], W["k"], W["v"], W["o"], f32dev(w.shift_C), None, f32dev(k),
                             f32dev(dD), dh)
    torch.cuda.synchronize()
    ref = oracle.h3_layer(w.x64, w.W["q"][1], w.W["k"][1], w.W["v"][1], w.W["o"][1], w.shift_C.astype(np.float64),
                          k.astype(np.float64), dD.astype(np.float64), d_head=dh)
    check(out, ref, TOL[dtype], "out", rows=False)
