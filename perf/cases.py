"""The calls whose speed is measured: what a program that uses this package has it do.

Six kinds of call, each through the package's public entry points:

  conv       kernel generation and the fused convolution, one SSM pass of a
             forward step (ssm_kernel, fftconv);
  train      the fused convolution and its backward pass (fftconv, fftconv_bwd);
  layer      a whole H3 layer, the kernel laid out once (layer_fwd);
  heads      the same with heads of dimension d_head (layer_fwd_heads);
  statepass  a long prompt, chunk by chunk, with its final state (statepass_conv);
  step       generation from a carried state (ssm_step).

listed() holds fixed cases, draw() takes others from the same ranges.
Everything is drawn on the GPU from the seed: activations N(0, 1), S4D-Lin
modes, log-uniform step sizes, shift taps and weights scaled by their fan-in.
"""
from __future__ import annotations

import math

import torch

import paper_2212_14052_amd as h3

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


# ------------------------------------------------------------------ cases ---
def listed():
    return [
        # one long convolution at batch 1, the smallest call: latency
        dict(name="conv_f32_single", kind="conv", B=1, H=64, L=1024, m=64, dtype="f32"),
        # the float32 convolution of a wide batch, larger than the last-level cache
        dict(name="conv_f32_batch", kind="conv", B=8, H=4096, L=1024, m=64, dtype="f32"),
        # one SSM of a 125M-parameter layer, the ordinary training shape
        dict(name="conv_125m", kind="conv", B=8, H=768, L=2048, m=64, dtype="f16"),
        # between the two tuned lengths, odd batch and odd channel count
        dict(name="conv_l4096_odd", kind="conv", B=5, H=767, L=4096, m=64, dtype="bf16"),
        # the longest sequence of the paper's fused range
        dict(name="conv_l8192", kind="conv", B=16, H=256, L=8192, m=64, dtype="bf16"),
        # forward and backward at the ordinary training shape
        dict(name="train_125m", kind="train", B=8, H=768, L=2048, m=64, dtype="f16"),
        # forward and backward of long sequences, odd batch
        dict(name="train_l8192", kind="train", B=3, H=400, L=8192, m=64, dtype="bf16"),
        # a 125M-parameter layer's forward at the short training length
        dict(name="layer_125m_l1024", kind="layer", B=8, L=1024, d=768, m_s=64, m=64, dtype="f16"),
        # a 2.7B-parameter layer's forward
        dict(name="layer_2p7b", kind="layer", B=4, L=2048, d=2560, m_s=64, m=64, dtype="bf16"),
        # the same width with the pure H3 model's heads of dimension 8
        dict(name="layer_heads8", kind="heads", B=4, L=2048, d=2560, d_head=8, m_s=64, m=64, dtype="bf16"),
        # a 128K-token prompt past the fused limit
        dict(name="statepass_128k", kind="statepass", B=2, H=1024, L=131072, chunk=8192, m=64, x0=False,
             dtype="f16"),
        # one generated token for 64 sequences
        dict(name="step_decode", kind="step", B=64, H=768, T=1, m=64, dtype="f16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dtype(rng):
    return rng.choice(["f32", "f16", "f16", "bf16", "bf16"])


def draw(rng):
    kind = rng.choice(["conv", "conv", "conv", "train", "train", "layer", "layer", "heads", "statepass",
                       "statepass", "step"])
    m = rng.choice([16, 32, 64, 64])
    if kind == "conv":
        dtype = _dtype(rng)
        L = rng.choice([512, 1024, 2048, 4096, 8192] + ([16384] if dtype != "f32" else []))
        B = _log(rng, 1, 16)
        return dict(kind=kind, B=B, H=_log(rng, 64, max(64, min(4096, (32 << 20) // (B * L)))), L=L, m=m, dtype=dtype)
    if kind == "train":
        L = rng.choice([1024, 2048, 4096, 8192])
        B = _log(rng, 1, 16)
        return dict(kind=kind, B=B, H=_log(rng, 64, max(64, min(2048, (8 << 20) // (B * L)))), L=L, m=m,
                    dtype=_dtype(rng))
    if kind == "layer":
        L = rng.choice([1024, 2048, 4096, 8192])
        B = _log(rng, 1, 8)
        d = 128 * _log(rng, 2, max(2, min(20, (10 << 20) // (B * L * 128))))
        return dict(kind=kind, B=B, L=L, d=d, m_s=rng.choice([4, 64]), m=m, dtype=rng.choice(["f16", "bf16"]))
    if kind == "heads":
        L = rng.choice([1024, 2048])
        B = _log(rng, 1, 6)
        dh = rng.choice([2, 4, 8, 8])
        d = 128 * _log(rng, 2, max(2, min(20, (64 << 20) // (B * L * 128 * dh))))
        return dict(kind=kind, B=B, L=L, d=d, d_head=dh, m_s=64, m=m, dtype=rng.choice(["f16", "bf16"]))
    if kind == "statepass":
        dtype = _dtype(rng)
        chunk = rng.choice([2048, 4096, 8192, 8192] + ([16384] if dtype != "f32" else []))
        L = chunk * rng.randint(2, 16)
        B = _log(rng, 1, 4)
        most = (16 if dtype == "f32" or chunk < 8192 else 96) << 20
        return dict(kind=kind, B=B, H=_log(rng, 32, max(32, min(1024, most // (B * L)))), L=L, chunk=chunk, m=m,
                    x0=rng.random() < 0.5, dtype=dtype)
    B, T = _log(rng, 1, 128), _log(rng, 1, 32)
    return dict(kind="step", B=B, H=_log(rng, 64, max(64, min(2560, 100000 // (B * T) * 8))), T=T, m=m,
                dtype=_dtype(rng))


# ----------------------------------------------------------------- inputs ---
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (int(seed) + 1))
    return g


def _randn(g, shape, dtype=torch.float32, scale=1.0):
    t = torch.randn(shape, generator=g, device="cuda", dtype=dtype)
    return t if scale == 1.0 else t.mul_(scale)


def _ssm(g, H, m, lo, hi):
    """S4D-Lin modes A_n = -1/2 + i pi n, B = 1, C ~ CN(0, 1), dt log-uniform."""
    dt = torch.empty(H, device="cuda").uniform_(math.log(lo), math.log(hi), generator=g).exp_()
    A = torch.empty(H, m, 2, device="cuda")
    A[..., 0] = -0.5
    A[..., 1] = math.pi * torch.arange(m, device="cuda", dtype=torch.float32)
    B = torch.zeros(H, m, 2, device="cuda")
    B[..., 0] = 1.0
    return A, B, _randn(g, (H, m, 2), scale=math.sqrt(0.5)), dt


def _c128(t):
    return torch.view_as_complex(t.double().contiguous())


def _zoh(A, B, dt):
    """(Abar, Bbar) in complex128."""
    a = _c128(A)
    Ab = torch.exp(dt.double()[:, None] * a)
    return Ab, (Ab - 1) / a * _c128(B)


def _pair32(z):
    return torch.view_as_real(z).float().contiguous()


def _inputs(case, seed):
    """The tensors of a case, by name."""
    c, g = case, _gen(seed)
    kind, dtype, m = c["kind"], DTYPES[c["dtype"]], c["m"]
    s = {}
    if kind in ("conv", "train"):
        B, H, L = c["B"], c["H"], c["L"]
        s["u"] = _randn(g, (B, H, L), dtype)
        s["A"], s["Bc"], s["C"], s["dt"] = _ssm(g, H, m, 1e-3, 1e-1)
        s["D"] = _randn(g, (H,))
        if kind == "train":
            s["dy"] = _randn(g, (B, H, L), dtype)
            # a trained kernel held in float32
            s["k"] = _kernel64(*_zoh(s["A"], s["Bc"], s["dt"]), _c128(s["C"]), L).float()
    elif kind in ("layer", "heads"):
        B, L, d, dh = c["B"], c["L"], c["d"], c.get("d_head", 1)
        s["x"] = _randn(g, (B, L, d), dtype)
        for n in ("Wq", "Wk", "Wv", "Wo"):
            s[n] = _randn(g, (d, d), dtype, 1.0 / math.sqrt(d))
        s["shift_C"] = _randn(g, (d, c["m_s"]), scale=1.0 / math.sqrt(c["m_s"]))
        A, Bc, C, dt = _ssm(g, d * dh, m, 1e-3, 1e-1)
        s["diag_k"] = _kernel64(*_zoh(A, Bc, dt), _c128(C), L).float()
        s["diag_D"] = _randn(g, (d * dh,))
    elif kind == "statepass":
        B, H, L = c["B"], c["H"], c["L"]
        s["u"] = _randn(g, (B, H, L), dtype)
        A, Bc, s["C"], dt = _ssm(g, H, m, 1e-4, 1e-2)
        s["Abar"], s["Bbar"] = (_pair32(z) for z in _zoh(A, Bc, dt))
        s["D"] = _randn(g, (H,))
        s["x0"] = _randn(g, (B, H, m, 2)) if c["x0"] else None
    else:
        B, H, T = c["B"], c["H"], c["T"]
        s["u"] = _randn(g, (B, H, T), dtype)
        A, Bc, s["C"], dt = _ssm(g, H, m, 1e-3, 1e-1)
        s["Abar"], s["Bbar"] = (_pair32(z) for z in _zoh(A, Bc, dt))
        s["D"] = _randn(g, (H,))
        s["x"] = _randn(g, (B, H, m, 2))
    return s


def prepare(case, seed):
    """Inputs, parameters and weights on the GPU, and for the calls that take
    one a workspace, kept from call to call as a program would."""
    c = case
    s = _inputs(case, seed)
    s["case"] = dict(case)
    dt = {"f32": h3.F32, "f16": h3.F16, "bf16": h3.BF16}[c["dtype"]]
    kind = c["kind"]
    if kind == "conv":
        n = h3.workspace_size(h3.OP_FFTCONV, c["B"], c["H"], c["L"], 0, 0, dt)
    elif kind == "train":
        n = max(h3.workspace_size(op, c["B"], c["H"], c["L"], 0, 0, dt) for op in (h3.OP_FFTCONV, h3.OP_FFTCONV_BWD))
    elif kind == "layer":
        n = h3.workspace_size(h3.OP_LAYER, c["B"], c["d"], c["L"], c["m_s"], 0, dt)
    elif kind == "heads":
        n = h3.workspace_size(h3.OP_LAYER_HEADS, c["B"], c["d"], c["L"], c["m_s"], c["d_head"], dt)
    elif kind == "statepass":
        n = h3.workspace_size(h3.OP_STATEPASS, c["B"], c["H"], c["L"], c["m"], c["chunk"], dt)
    else:
        n = 0
    s["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------- pass ---
def run(s):
    kind, ws = s["case"]["kind"], s["ws"]
    if kind == "conv":
        k = h3.ssm_kernel(s["A"], s["Bc"], s["C"], s["dt"], s["case"]["L"])
        return {"k": k, "y": h3.fftconv(s["u"], k, s["D"], workspace=ws)}
    if kind == "train":
        y = h3.fftconv(s["u"], s["k"], s["D"], workspace=ws)
        du, dk, dD = h3.fftconv_bwd(s["u"], s["k"], s["D"], s["dy"], workspace=ws)
        return {"y": y, "du": du, "dk": dk, "dD": dD}
    if kind == "layer":
        return h3.layer_fwd(s["x"], s["Wq"], s["Wk"], s["Wv"], s["Wo"], s["shift_C"], None, s["diag_k"],
                            s["diag_D"], workspace=ws)
    if kind == "heads":
        return h3.layer_fwd_heads(s["x"], s["Wq"], s["Wk"], s["Wv"], s["Wo"], s["shift_C"], None, s["diag_k"],
                                  s["diag_D"], s["case"]["d_head"], workspace=ws)
    if kind == "statepass":
        y, xf = h3.statepass_conv(s["u"], s["Abar"], s["Bbar"], s["C"], s["D"], s["case"]["chunk"], x0=s["x0"],
                                  workspace=ws)
        return {"y": y, "x_final": xf}
    y = h3.ssm_step(s["u"], s["Abar"], s["Bbar"], s["C"], s["D"], s["x"])
    return {"y": y, "x": s["x"]}


# ------------------------------------------------------------------- work ---
def work(case):
    """Inputs read once and outputs written once; the FFT convolution's
    arithmetic (2.5 N log2 N per real transform of N = 2L points), the matrix
    products, and two real multiply-adds per mode, element and use of a state."""
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    kind, m = c["kind"], c["m"]

    def conv(rows, channels, L, transforms=2):
        n = 2 * L
        return (transforms * rows + channels) * 2.5 * n * math.log2(n) + 3 * n * rows

    if kind in ("conv", "train"):
        B, H, L = c["B"], c["H"], c["L"]
        io = B * H * L * e
        if kind == "conv":
            return {"bytes": 2 * io + 4 * H * L + 24 * H * m + 8 * H,
                    "flops": conv(B * H, H, L) + 4 * m * H * L}
        # forward: u, k in, y out; backward: dy in, du, dk, dD out
        return {"bytes": 4 * io + 8 * H * L + 8 * H, "flops": 2.5 * conv(B * H, H, L)}
    if kind in ("layer", "heads"):
        B, L, d, dh = c["B"], c["L"], c["d"], c.get("d_head", 1)
        return {"bytes": 2 * B * L * d * e + 4 * d * d * e + 4 * d * c["m_s"] + 4 * d * dh * (L + 1),
                "flops": 8 * B * L * d * d + 2 * c["m_s"] * B * L * d + conv(B * d * dh, d * dh, L)
                + 4 * B * L * d * dh}
    if kind == "statepass":
        B, H, L = c["B"], c["H"], c["L"]
        chunk = c["chunk"]
        return {"bytes": 2 * B * H * L * e + 24 * H * m + 4 * H + 8 * B * H * m * (2 if c["x0"] else 1),
                "flops": conv(B * H * (L // chunk), H, chunk) + 8 * m * B * H * L + 4 * m * H * chunk}
    B, H, T = c["B"], c["H"], c["T"]
    return {"bytes": 2 * B * H * T * e + 16 * B * H * m + 24 * H * m + 4 * H, "flops": 14 * m * B * H * T}


# -------------------------------------------------------------- tolerance ---
def tolerance(case):
    """About four times the largest error against 64 bits over the listed and
    some drawn cases: float32 sums, one 16-bit rounding after fp16 matrix-core
    operands, and for the layers the 16-bit Q, K, V, G and O between."""
    kind, dtype = case["kind"], case["dtype"]
    if kind in ("layer", "heads"):
        return {"rel": 3e-3 if dtype == "f16" else 2e-2, "max": 3e-2 if dtype == "f16" else 1.8e-1}
    return {"f32": {"rel": 1.5e-6, "max": 6e-5}, "f16": {"rel": 4e-3, "max": 4e-2},
            "bf16": {"rel": 8e-3, "max": 8e-2}}[dtype]


# ------------------------------------------------------------------ exact ---
def _kernel64(Ab, Bb, C, L):
    """2 Re sum_n C Bbar Abar^t for t < L, (H, L) float64: t = w a + b."""
    H, m = Ab.shape
    w = 1 << ((L.bit_length()) // 2)
    la = torch.log(Ab)
    out = torch.empty(H, L, dtype=torch.float64, device=Ab.device)
    b = torch.arange(w, dtype=torch.float64, device=Ab.device)
    a = torch.arange((L + w - 1) // w, dtype=torch.float64, device=Ab.device) * w
    for h in range(0, H, 512):
        z = la[h:h + 512, :, None]
        P = torch.exp(z * a) * (C * Bb)[h:h + 512, :, None]
        k = torch.matmul(P.transpose(1, 2).contiguous(), torch.exp(z * b))
        out[h:h + 512] = 2 * k.real.reshape(z.shape[0], -1)[:, :L]
    return out


def _conv64(u, k, D, corr=False):
    """Causal convolution (or correlation) of (B, H, L) float64 rows with (H, L), plus D u."""
    L = u.shape[-1]
    f = torch.fft.rfft(k, 2 * L)
    y = torch.fft.irfft(torch.fft.rfft(u, 2 * L) * (f.conj() if corr else f), 2 * L)[..., :L]
    return y + D[:, None] * u


def exact(case, seed):
    """run()'s outputs in 64 bits from the same inputs."""
    s, c = _inputs(case, seed), case
    kind, m = c["kind"], c["m"]
    if kind == "conv":
        k = _kernel64(*_zoh(s["A"], s["Bc"], s["dt"]), _c128(s["C"]), c["L"])
        y = torch.empty(s["u"].shape, dtype=torch.float64, device="cuda")
        for h in range(0, c["H"], 256):
            y[:, h:h + 256] = _conv64(s["u"][:, h:h + 256].double(), k[h:h + 256], s["D"][h:h + 256].double())
        return {"k": k, "y": y}
    if kind == "train":
        L = c["L"]
        out = {n: torch.empty(s["u"].shape, dtype=torch.float64, device="cuda") for n in ("y", "du")}
        out["dk"] = torch.empty(s["k"].shape, dtype=torch.float64, device="cuda")
        out["dD"] = torch.empty(c["H"], dtype=torch.float64, device="cuda")
        for h in range(0, c["H"], 128):
            e = slice(h, h + 128)
            u, dy, k, D = s["u"][:, e].double(), s["dy"][:, e].double(), s["k"][e].double(), s["D"][e].double()
            out["y"][:, e] = _conv64(u, k, D)
            out["du"][:, e] = _conv64(dy, k, D, corr=True)
            z = (torch.fft.rfft(u, 2 * L).conj() * torch.fft.rfft(dy, 2 * L)).sum(0)
            out["dk"][e] = torch.fft.irfft(z, 2 * L)[..., :L]
            out["dD"][e] = (u * dy).sum((0, 2))
        return out
    if kind in ("layer", "heads"):
        B, L, d, dh = c["B"], c["L"], c["d"], c.get("d_head", 1)
        x = s["x"].double().reshape(B * L, d)
        q, k, v = ((x @ s[n].double()).reshape(B, L, d).transpose(1, 2).contiguous() for n in ("Wq", "Wk", "Wv"))
        taps = s["shift_C"].double()
        kbar = torch.zeros_like(k)
        for j in range(c["m_s"]):
            kbar[..., j:] += taps[:, j, None] * k[..., :L - j]
        o = torch.empty_like(q)
        diag_k, diag_D = s["diag_k"].double().reshape(d, dh, L), s["diag_D"].double().reshape(d, dh)
        for h in range(0, d, 64):   # whole heads: dh divides 64
            e = slice(h, h + 64)
            heads = [t[:, e].reshape(B, 64 // dh, dh, L) for t in (q, kbar, v)]
            kv = heads[1][:, :, :, None] * heads[2][:, :, None]   # (B, head, i, j, L)
            S = _conv64(kv.reshape(B, 64 * dh, L), diag_k[e].reshape(64 * dh, L), diag_D[e].reshape(-1))
            o[:, e] = (heads[0][:, :, :, None] * S.reshape(B, 64 // dh, dh, dh, L)).sum(2).reshape(B, 64, L)
        return (o.transpose(1, 2).reshape(B * L, d) @ s["Wo"].double()).reshape(B, L, d)
    Ab, Bb, C, D = _c128(s["Abar"]), _c128(s["Bbar"]), _c128(s["C"]), s["D"].double()
    if kind == "statepass":
        B, H, L = c["B"], c["H"], c["L"]
        y = torch.empty(s["u"].shape, dtype=torch.float64, device="cuda")
        xf = torch.empty(B, H, m, dtype=torch.complex128, device="cuda")
        w = c["chunk"]
        t = torch.arange(w, dtype=torch.float64, device="cuda")
        for h in range(0, H, 32):
            e = slice(h, h + 32)
            u, la = s["u"][:, e].double(), torch.log(Ab[e])
            n = u.shape[1]
            y[:, e] = _conv64(u, _kernel64(Ab[e], Bb[e], C[e], L), D[e])
            # end states by chunk, then the sum over chunks
            P = torch.exp(la[:, None, :] * (w - 1 - t)[None, :, None]) * Bb[e][:, None, :]
            ends = torch.matmul(u.transpose(0, 1).reshape(n, -1, w).contiguous(),
                                torch.view_as_real(P).reshape(n, w, 2 * m))
            ends = torch.view_as_complex(ends.reshape(n, B, L // w, m, 2))
            left = torch.arange(L // w - 1, -1, -1, dtype=torch.float64, device="cuda") * w
            xf[:, e] = (ends * torch.exp(la[:, None, None, :] * left[:, None])).sum(2).transpose(0, 1)
            if s["x0"] is not None:
                x0 = _c128(s["x0"][:, e])
                xf[:, e] += x0 * torch.exp(la * L)
                y[:, e] += torch.stack([_kernel64(Ab[e], Ab[e], C[e] * x0[b], L) for b in range(B)])
        return {"y": y, "x_final": torch.view_as_real(xf)}
    x, y = _c128(s["x"]), torch.empty(s["u"].shape, dtype=torch.float64, device="cuda")
    for i in range(c["T"]):
        u = s["u"][..., i].double()
        x = Ab * x + Bb * u[..., None]
        y[..., i] = 2 * (C * x).sum(-1).real + D * u
    return {"y": y, "x": torch.view_as_real(x)}
