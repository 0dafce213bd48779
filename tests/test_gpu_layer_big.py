"""A layer whose activations pass 4 GiB (B L d > 2^31 values of 16 bits), each
way the projections read them: the last two sequences against the same two in
a call of their own, all others zero."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,d", [
    (5464, 1024, 384),    # 128-wide weight tiles, O read K-major
    (410, 2048, 2560),    # 320-wide, O gated in the convolution
    (342, 16384, 384),    # O token-major
])
def test_layer_past_4gib(B, L, d):
    import paper_2212_14052_amd as h3
    need = h3.workspace_size(h3.OP_LAYER, B, d, L, 4, 0, h3.F16) + 4 * B * L * d
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("needs 30 GB of GPU memory")
    assert B * L * d > 1 << 31
    g = torch.Generator(device="cuda")
    g.manual_seed(L)

    def rand(*shape, scale=1.0, dtype=torch.float16):
        return torch.randn(shape, generator=g, device="cuda", dtype=dtype) * scale

    W = [rand(d, d, scale=d ** -0.5) for _ in range(4)]
    shift, k = rand(d, 4, dtype=torch.float32), rand(d, L, scale=L ** -0.5, dtype=torch.float32)
    two = rand(2, L, d)
    x = torch.zeros((B, L, d), dtype=torch.float16, device="cuda")
    x[-2:] = two
    out = h3.layer_fwd(x, *W, shift, None, k, None)
    ref = h3.layer_fwd(two, *W, shift, None, k, None)
    assert torch.count_nonzero(out[:-2]) == 0
    # other tile widths and row pairings: 16-bit Q, K, V, G, O apart by an ulp here and there
    e = float((out[-2:].double() - ref.double()).norm() / ref.double().norm())
    del x, out
    torch.cuda.empty_cache()
    assert e < 2e-3, e
