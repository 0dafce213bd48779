"""The direct kernel gradient (16-bit rows, L in 256 .. 8192) against the
float64 oracle, at the edges of its dispatch: every length, channel counts on
both sides of the split rules, batches on both sides of a stage of rows and of
the rows between two reductions."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests._util import check, f32dev, to_dev, to_np64

pytestmark = pytest.mark.gpu

# A result sums chains of 64 matrix instructions, each rounding its float32
# accumulator four times: as a random walk 2^-24 sqrt(256) = 1e-6 of the
# result, doubled for the sums over waves and chains.
TOL = 2e-6


@pytest.fixture(scope="module")
def h3():
    import paper_2212_14052_amd as h3
    h3.lib()
    return h3


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,H,L", [(1, 2, 256), (65, 3, 256), (5, 3, 512), (34, 2, 512), (4, 7, 1024), (17, 2, 1024),
                                   (3, 2, 2048), (9, 2, 2048), (5, 64, 4096), (2, 65, 4096), (1, 129, 4096),
                                   (1, 128, 8192), (3, 2, 8192), (2, 129, 8192)])
def test_wgrad_direct(h3, dtype, B, H, L):
    w = workloads.conv_workload("t", B, H, L, dtype, seed=B + L)
    g = workloads.conv_workload("g", B, H, L, dtype, seed=B + L + 1)
    u, dy, k = to_dev(w.u, dtype), to_dev(g.u, dtype), f32dev(np.zeros((H, L)))
    _, dk, dD = h3.fftconv_bwd(u, k, None, dy, want_du=False)
    _, dk_only, none_dD = h3.fftconv_bwd(u, k, None, dy, want_du=False, want_dD=False)
    _, none_dk, dD_only = h3.fftconv_bwd(u, k, None, dy, want_du=False, want_dk=False)
    torch.cuda.synchronize()
    assert none_dD is None and none_dk is None
    _, rdk, rdD = oracle.causal_conv_bwd(w.u64, np.zeros((H, L)), None, g.u64)
    check(dk, rdk, TOL, "dk")
    check(dD, rdD, TOL, "dD", rows=False)
    np.testing.assert_array_equal(to_np64(dk), to_np64(dk_only))
    np.testing.assert_array_equal(to_np64(dD), to_np64(dD_only))
