"""One-pass state passing (16-bit rows, chunks 2048, 8192, 16384) against the
float64 recurrence and against the chunked float32 convolution path, at the
edges of its dispatch: one and many segments per row, a short last segment,
one to four waves per workgroup, few modes, and parameters that leave the
usual range."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests._util import check, cplx64, cplx_to_f32pairs, f32dev, record, to_dev, to_np64

pytestmark = pytest.mark.gpu

# fp16 tables and states: 2^-11 each, sums of 128 and 64 products around the
# largest term, then the output's rounding (bf16: 2^-8), against the tensor's
# and the row's maximum
TOL = {workloads.F16: 5e-3, workloads.BF16: 1e-2}
TOL_X = {workloads.F16: 3e-3, workloads.BF16: 1e-4}


@pytest.fixture(scope="module")
def h3():
    import paper_2212_14052_amd as h3
    h3.lib()
    return h3


def _run(h3, w, Ab, Bb, C, D, x0, chunk):
    y, xf = h3.statepass_conv(to_dev(w.u, w.dtype), f32dev(Ab), f32dev(Bb), f32dev(C),
                              None if D is None else f32dev(D), chunk, x0=None if x0 is None else f32dev(x0))
    torch.cuda.synchronize()
    return to_np64(y), cplx64(to_np64(xf))


def _ref(w, Ab, Bb, C, D, x0):
    return oracle.recurrence(w.u64, cplx64(Ab), cplx64(Bb), cplx64(C),
                             None if D is None else D.astype(np.float64), x0=None if x0 is None else cplx64(x0))


def _params(w):
    A, B, C, dt = w.ssm.complex64()
    Ab, Bb = oracle.zoh(A, B, dt)
    return cplx_to_f32pairs(Ab), cplx_to_f32pairs(Bb), w.ssm.C


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,H,L,chunk,m,x0", [
    (1, 1, 2048, 2048, 64, True),          # one step, one wave
    (1, 2, 2 * 2048, 2048, 1, False),      # one mode, two segments
    (3, 5, 7 * 2048, 2048, 33, True),      # one step per segment
    (1, 700, 5 * 2048, 2048, 8, True),     # three segments, the last one short
    (1, 1025, 2048, 2048, 4, True),        # rows past one per SIMD: one segment
    (2, 515, 2 * 2048, 2048, 16, False),   # two waves per workgroup
    (5, 210, 2048, 2048, 64, True),        # five items, the last workgroup not full
    (2, 3, 16384, 8192, 64, True),
    (1, 3, 32768, 16384, 64, False),
])
def test_scan_matches_recurrence(h3, dtype, B, H, L, chunk, m, x0):
    w = workloads.statepass_workload("t", B, H, L, chunk, dtype, seed=H + L, m=m, dt_lo=1e-3, dt_hi=1e-1,
                                     x0_scale=1.0 if x0 else 0.0)
    Ab, Bb, C = _params(w)
    y, xf = _run(h3, w, Ab, Bb, C, w.D, w.x0, chunk)
    ry, rx = _ref(w, Ab, Bb, C, w.D, w.x0)
    check(y, ry, TOL[dtype], "y")
    check(xf, rx, TOL_X[dtype], "x_final", rows=False)


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("case", ["no_skip", "zero_b", "zero_c", "growing", "decayed", "tiny_u", "large_u", "scaled_c"])
def test_scan_unusual_parameters(h3, dtype, case):
    B, H, L = 2, 6, 4 * 2048
    w = workloads.statepass_workload("t", B, H, L, 2048, dtype, seed=17, m=48, dt_lo=1e-3, dt_hi=1e-1, x0_scale=1.0)
    Ab, Bb, C = (np.array(v) for v in _params(w))
    D, x0 = w.D, np.array(w.x0)
    if case == "no_skip":
        D = None
    elif case == "zero_b":          # modes that the input does not reach
        Bb[:, ::3] = 0
    elif case == "zero_c":          # modes that the output does not see, with a large state
        C[:, ::3] = 0
        x0[:, :, ::3] *= 1e4
    elif case == "growing":         # |Abar| > 1 by a factor of three over the sequence
        a = cplx64(Ab)
        Ab = cplx_to_f32pairs(a / np.abs(a) * 3.0 ** (1.0 / L))
        Bb = Bb * 1e-2
    elif case == "decayed":         # modes gone within a few inputs, and Abar = 0
        a = cplx64(Ab)
        Ab = cplx_to_f32pairs(a * np.linspace(0.0, 0.5, a.shape[1]))
    elif case in ("tiny_u", "large_u"):
        # |y| reaches some 30 here: 2^12 times that leaves fp16 (65504)
        s = 2.0 ** -10 if case == "tiny_u" else 2.0 ** (12 if dtype == workloads.BF16 else 10)
        w.u, w.u64 = workloads.round_to(w.u64 * s, dtype)
        x0 = (x0 * s).astype(np.float32)
    elif case == "scaled_c":        # output weights far apart between channels
        f = (10.0 ** np.linspace(-12, 12, H)).astype(np.float32) if dtype == workloads.BF16 else \
            (10.0 ** np.linspace(-2, 3, H)).astype(np.float32)
        C = C * f[:, None, None]
        D = D * f
    y, xf = _run(h3, w, Ab, Bb, C, D, x0, 2048)
    ry, rx = _ref(w, Ab, Bb, C, D, x0)
    for h in range(H):
        check(np.ascontiguousarray(y[:, h]), np.ascontiguousarray(ry[:, h]), TOL[dtype], f"y{h}")
    check(xf, rx, TOL_X[dtype], "x_final", rows=False)
    if case == "decayed":
        return   # the general path takes Abar's logarithm, which Abar = 0 has not
    # the general path (float32 convolution of chunks of 512) on the same inputs
    y2, x2 = _run(h3, w, Ab, Bb, C, D, x0, 512)
    for h in range(H):
        check(np.ascontiguousarray(y[:, h]), np.ascontiguousarray(y2[:, h]), 2 * TOL[dtype], f"y{h} chunk 512")
    check(xf, x2, 2 * TOL_X[dtype], "x_final chunk 512", rows=False)


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,H,L", [(2, 6, 24 * 2048), (1, 1024, 16 * 2048)])   # one step per segment; one segment
def test_scan_zero_tail(h3, dtype, B, H, L):
    """A zero-padded sequence: the state decays through the smallest floats to
    zero, over steps that hold nothing else."""
    w = workloads.statepass_workload("t", B, H, L, 2048, dtype, seed=23, m=4, dt_lo=3e-3, dt_hi=1e-1)
    w.u[..., 2048:] = 0
    w.u64[..., 2048:] = 0
    Ab, Bb, C = _params(w)
    y, xf = _run(h3, w, Ab, Bb, C, w.D, None, 2048)
    assert np.isfinite(y).all() and np.isfinite(xf).all()
    sel = np.unique(np.r_[0, H // 3, H - 1])
    ry, rx = oracle.recurrence(np.ascontiguousarray(w.u64[:, sel]), *(cplx64(a[sel]) for a in (Ab, Bb, C)),
                               w.D[sel].astype(np.float64))
    check(np.ascontiguousarray(y[:, sel]), ry, TOL[dtype], "y")
    # (most final states lie below float32's range)
    assert np.abs(xf[:, sel] - rx).max() <= TOL_X[dtype] * np.abs(rx).max() + 1e-37


@pytest.mark.parametrize("dtype,chunk", [(workloads.F16, 2048), (workloads.BF16, 2048), (workloads.F16, 512)])
@pytest.mark.parametrize("B,H,L", [(1, 2, 2 * 2048), (3, 5, 8 * 2048), (2, 100, 13 * 2048), (1, 1040, 2048)])
def test_scan_state_in_place(h3, dtype, chunk, B, H, L):
    """x_final on x0's own buffer, as a program that carries one state along
    calls it: the rows cut into segments, and whole ones."""
    w = workloads.statepass_workload("t", B, H, L, chunk, dtype, seed=41 + H, m=24, dt_lo=1e-4, dt_hi=1e-2, x0_scale=4.0)
    Ab, Bb, C = (f32dev(v) for v in _params(w))
    u, D, x0 = to_dev(w.u, dtype), f32dev(w.D), f32dev(w.x0)
    y, xf = h3.statepass_conv(u, Ab, Bb, C, D, chunk, x0=x0)
    state = x0.clone()
    y2, xf2 = h3.statepass_conv_noalloc(u, Ab, Bb, C, D, chunk, x0=state, x_final=state)
    torch.cuda.synchronize()
    assert xf2.data_ptr() == state.data_ptr()
    assert torch.equal(y, y2) and torch.equal(xf, state)


@pytest.mark.parametrize("B,H,L", [(1, 1024, 1 << 18), (1, 1, 1 << 21)])   # 4096 blocks in one segment; 1024 segments
def test_scan_undamped_modes(h3, B, H, L):
    """Modes of modulus 1 over a long sequence, bf16 rows: the state's decay
    factor acts once per block or segment, and what its rounding leaves over
    must not add up.  The bf16 pairs hold the tables to 2^-17 and the state is
    rounded twice per block, as a random walk 2^-24 sqrt(2 L / 64): 1.2e-5
    together, relative to the norm (a float32 factor alone: 2^-25 L / 64 on
    average, 1e-4 here)."""
    m = 4
    rng = np.random.default_rng(31)
    a = cplx_to_f32pairs(np.exp(1j * rng.uniform(0, np.pi, (H, m))))
    b = cplx_to_f32pairs(rng.standard_normal((H, m)) + 1j * rng.standard_normal((H, m)))
    c = cplx_to_f32pairs((rng.standard_normal((H, m)) + 1j * rng.standard_normal((H, m))) / 8)
    a = a * (1 - 2.0 ** -24 * np.float32(rng.uniform(0, 1)))
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    u = torch.randn((B, H, L), generator=g, device="cuda", dtype=torch.bfloat16) * 2.0 ** -4
    _, xf = h3.statepass_conv(u, f32dev(a), f32dev(b), f32dev(c), None, 2048)
    torch.cuda.synchronize()
    xf = cplx64(to_np64(xf))
    sel = np.unique(np.r_[0, H // 3, H - 1])
    _, rx = oracle.recurrence(to_np64(u[:, sel.tolist()]), *(cplx64(v[sel].astype(np.float32)) for v in (a, b, c)), None)
    err = np.linalg.norm(xf[:, sel] - rx) / np.linalg.norm(rx)
    record(f"undamped L={L}", rel_err=float(err))
    assert err < 1.2e-5, err


@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
@pytest.mark.parametrize("B,H,mag", [(1, 3, 1.06), (1, 3, 2.0), (2, 520, 1.06)])   # four segments; one
def test_scan_growing_mode_without_input(h3, dtype, B, H, mag):
    """A mode outside the unit circle whose state is and stays zero (Bbar = 0,
    no initial state) is as good as absent."""
    w = workloads.statepass_workload("t", B, H, 4 * 2048, 2048, dtype, seed=3, m=4, dt_lo=1e-3, dt_hi=1e-1)
    Ab, Bb, C = _params(w)
    y, xf = _run(h3, w, Ab, Bb, C, w.D, None, 2048)
    one = np.zeros((H, 1, 2), np.float32)
    Ab2 = np.concatenate([Ab, one + np.float32([mag, 0.1])], axis=1)
    y2, xf2 = _run(h3, w, Ab2, np.concatenate([Bb, one], axis=1), np.concatenate([C, one + 1], axis=1), w.D, None, 2048)
    assert np.array_equal(y, y2) and np.array_equal(xf, xf2[:, :, :4]) and not xf2[:, :, 4].any()
