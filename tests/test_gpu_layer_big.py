"""The projections' addresses: activations past 4 GiB (B L d > 2^31 values of 16
bits), each way they are read, and sums of more than 256 steps, each tile width."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,d", [
    (5464, 1024, 384),    # 128-wide weight tiles, O read K-major
    (410, 2048, 2560),    # 320-wide, O gated in the convolution
    (342, 16384, 384),    # O token-major
])
def test_layer_past_4gib(B, L, d):
    """The last two sequences against the same two in a call of their own, all
    others zero."""
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


@pytest.mark.parametrize("B,d", [(1, 8320), (5, 8448), (19, 8320)])   # weight tiles 128, 256 and 320 wide
def test_layer_many_steps(B, d):
    """More than 256 steps along the projections' sums: the operands' bases
    move on.  Against float64, the sequence mixing a unit (one tap, a unit
    kernel): out = (Q K V) Wo."""
    import paper_2212_14052_amd as h3
    L = 256
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    W = [torch.randn((d, d), generator=g, device="cuda", dtype=torch.float16) * d ** -0.5 for _ in range(4)]
    x = torch.randn((B, L, d), generator=g, device="cuda", dtype=torch.float16)
    k = torch.zeros((d, L), device="cuda")
    k[:, 0] = 1.0
    out = h3.layer_fwd(x, *W, torch.ones((d, 1), device="cuda"), None, k, None)
    q, kk, v = (x.double() @ w.double() for w in W[:3])
    ref = (q * kk * v) @ W[3].double()
    # Q, K, V, O and the output rounded to 2^-12 of themselves on average
    e = float((out.double() - ref).norm() / ref.norm())
    assert e < 5 * 2.0 ** -12, e
