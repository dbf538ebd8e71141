"""Performance cases: the calls a diffusion UNet makes of this library.

Every case goes through the package's public entry points with preallocated
outputs and workspaces on the current stream, as a denoising loop calls them.
Sizes are those of the SD1.4 UNet at a 512x512 image (latent levels 64, 32,
16, 8 with head widths 40, 80, 160, 160; channels 320, 640, 1280, 1280; a
77-token text context; batch 2 for classifier-free guidance) and, in draw(),
other latent sides, batches and head counts around them.

Kinds of case:
  attn        one attention call: forward (fp16), or forward_ex where the case
              is bf16 or asks for the row statistics (L, S)
  block       a self-attention block: projections, attention, output projection
  block_kv    a cross-attention block at one denoising step, the text context's
              K and V computed once per prompt
  conv        a 3x3 convolution with kernels transformed once per layer
  norm_geglu  a level's group normalisation, and its gated activation
  twopass     the partially fused softmax in three calls (logits, row
              statistics, normalisation with the product by V)
"""
import math

import numpy as np
import torch

import paper_2304_11267_amd as sd

EPS = 1e-5
GROUPS = 32
TEXT = 77


def listed():
    return [
        # the 64x64 level's self-attention: most of a denoising step's attention time
        _attn("self64", 2, 8, 4096, 4096, 40),
        # the 32x32 level's self-attention
        _attn("self32", 2, 8, 1024, 1024, 80),
        # the 16x16 level's, with large logits (queries four times as long)
        _attn("self16_peaked", 2, 8, 256, 256, 160, q_mult=4.0),
        # cross-attention over the text at the 64x64 level
        _attn("cross64", 2, 8, 4096, TEXT, 40),
        # the smallest attention call of a step: the 8x8 middle block over the text
        _attn("cross8", 2, 8, 64, TEXT, 160),
        # a 66x60 latent without guidance, bf16, with the row statistics a caller
        # needs to merge key ranges
        _attn("self_ragged_stats", 1, 8, 3960, 3960, 40, dtype="bf16", stats=True),
        # a whole self-attention block of the 64x64 level
        _block("block64_self", 2, 4096, 320, 8, "f16"),
        # a cross-attention block of the 16x16 level at one denoising step
        _block_kv("block16_kv", 2, 256, TEXT, 1280, 8, "bf16"),
        # the convolutions of a residual block: few channels on a large map ...
        _conv("conv64", 2, 320, 320, 64, 64, "f16"),
        # ... and many on a small one
        _conv("conv16", 2, 1280, 1280, 16, 16, "bf16"),
        # normalisation and gated activation of the 64x64 level
        _norm("norm_geglu64", 2, 320, 64, 64, "f16"),
        # the 64x64 self-attention with its logits in memory
        _twopass("twopass64", 2, 8, 4096, 4096, 40, "f16"),
    ]


def _attn(name, B, H, Lq, Lk, D, dtype="f16", stats=False, q_mult=1.0):
    return _named(name, dict(kind="attn", B=B, H=H, Lq=Lq, Lk=Lk, D=D, dtype=dtype, stats=stats,
                             q_mult=q_mult))


def _block(name, B, L, C, H, dtype):
    return _named(name, dict(kind="block", B=B, Lq=L, C=C, H=H, dtype=dtype))


def _block_kv(name, B, Lq, Lk, C, H, dtype):
    return _named(name, dict(kind="block_kv", B=B, Lq=Lq, Lk=Lk, C=C, H=H, dtype=dtype))


def _conv(name, B, Ci, Co, h, w, dtype):
    return _named(name, dict(kind="conv", B=B, Ci=Ci, Co=Co, h=h, w=w, dtype=dtype))


def _norm(name, B, C, h, w, dtype):
    return _named(name, dict(kind="norm_geglu", B=B, C=C, h=h, w=w, dtype=dtype))


def _twopass(name, B, H, Lq, Lk, D, dtype):
    return _named(name, dict(kind="twopass", B=B, H=H, Lq=Lq, Lk=Lk, D=D, dtype=dtype))


def _named(name, case):
    return dict(case, name=name) if name else case


def draw(rng):
    """One more case: other images (latent sides), batches, heads and options."""
    most = [work(c) for c in listed()]
    flops, nbytes = max(w["flops"] for w in most), max(w["bytes"] for w in most)
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return case


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["attn"] * 5 + ["block", "block_kv"] + ["conv"] * 2 + ["norm_geglu", "twopass"])
    dtype = rng.choice(["f16", "f16", "bf16"])
    B = rng.choice([1, 2, 2, 4])
    if kind in ("attn", "twopass"):
        D = rng.choice([40, 40, 64, 80, 160])
        L = _log(rng, 64, 4096)
        H = rng.choice([5, 8, 8, 10])
        if kind == "twopass":
            return _twopass(None, B, H, L, L, D, dtype)
        Lk = rng.choice([L, L, L, TEXT, 2 * TEXT])
        return _attn(None, B, H, L, Lk, D, dtype, stats=rng.random() < 0.25,
                     q_mult=rng.choice([1.0, 1.0, 1.0, 4.0]))
    # a level of the UNet with another latent: height and width up to twice as
    # long or half as short
    side, C = rng.choice([(64, 320), (32, 640), (16, 1280), (8, 1280)])
    h, w = (max(4, _log(rng, side / 2, side * 1.4)) for _ in range(2))
    if kind == "block":
        return _block(None, B, h * w, C, 8, dtype)
    if kind == "block_kv":
        return _block_kv(None, B, h * w, TEXT, C, 8, dtype)
    if kind == "conv":
        # the decoder's convolutions read concatenated maps
        Ci = rng.choice([C, C, 2 * C, C + 320])
        return _conv(None, B, Ci, C, h, w, dtype)
    return _norm(None, B, C, h, w, dtype)


# ---------------------------------------------------------------- inputs

def _dtype(case):
    return {"f16": torch.float16, "bf16": torch.bfloat16}[case["dtype"]]


def _scale(D):
    return float(np.float32(1.0 / math.sqrt(D)))


def _inputs(case, seed):
    """The tensors a call reads, in the order run() and exact() take them."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = _dtype(case)

    def randn(*shape, sigma=1.0):
        return (torch.randn(*shape, device="cuda", generator=g) * sigma).to(dt)

    kind, B = case["kind"], case["B"]
    if kind in ("attn", "twopass"):
        H, Lq, Lk, D = case["H"], case["Lq"], case["Lk"], case["D"]
        return (randn(B, H, Lq, D, sigma=case.get("q_mult", 1.0)), randn(B, H, Lk, D),
                randn(B, H, Lk, D))
    if kind in ("block", "block_kv"):
        L, C, H = case["Lq"], case["C"], case["H"]
        x = randn(B, L, C)
        wq, wk, wv, wo = (randn(C, C, sigma=C ** -0.5) for _ in range(4))
        bo = randn(C, sigma=0.1)
        if kind == "block":
            return x, wq, wk, wv, wo, bo
        k, v = (randn(B, H, case["Lk"], C // H) for _ in range(2))
        return x, wq, k, v, wo, bo
    if kind == "conv":
        Ci, Co = case["Ci"], case["Co"]
        return (randn(B, Ci, case["h"], case["w"]), randn(Co, Ci, 3, 3, sigma=(9 * Ci) ** -0.5),
                randn(Co, sigma=0.1))
    # activations are not centred: every channel has its own mean and spread
    C, h, w = case["C"], case["h"], case["w"]
    mean = torch.randn(1, C, 1, 1, device="cuda", generator=g)
    spread = 0.2 + 1.8 * torch.rand(1, C, 1, 1, device="cuda", generator=g)
    x = (mean + spread * torch.randn(B, C, h, w, device="cuda", generator=g)).to(dt)
    gamma, beta = (1 + randn(C, sigma=0.2).float()).to(dt), randn(C, sigma=0.2)
    return x, gamma, beta, randn(B * h * w, 8 * C, sigma=1.5)


def prepare(case, seed):
    ins = _inputs(case, seed)
    dt, dev, kind, B = _dtype(case), ins[0].device, case["kind"], case["B"]
    st = dict(case=case, ins=ins, out=torch.empty_like(ins[0]))
    if kind in ("attn", "twopass"):
        H, Lq, Lk = case["H"], case["Lq"], case["Lk"]
        if kind == "twopass" or case["stats"]:
            st["ls"] = torch.empty(B, H, Lq, 2, dtype=torch.float32, device=dev)
        if kind == "twopass":
            st["a"] = torch.empty(B, H, Lq, Lk, dtype=dt, device=dev)
    elif kind in ("block", "block_kv"):
        n = sd.attention_block_workspace(B, case["Lq"], case["Lq"] if kind == "block" else 0,
                                         case["C"])
        st["ws"] = torch.empty(n, dtype=torch.uint8, device=dev)
    elif kind == "conv":
        x, w, bias = ins
        Ci, Co, h, wd = case["Ci"], case["Co"], case["h"], case["w"]
        u = torch.empty(36, Co, Ci, dtype=dt, device=dev)
        sd.winograd_weights(w, u)
        st["ins"] = (x, u, bias)
        st["out"] = torch.empty(B, Co, h, wd, dtype=dt, device=dev)
        st["ws"] = torch.empty(sd.conv3x3_workspace(B, Ci, Co, h, wd), dtype=torch.uint8, device=dev)
    else:
        h = ins[3]
        st["act"] = torch.empty(h.shape[0], h.shape[1] // 2, dtype=dt, device=dev)
    return st


def run(st):
    case, ins, out = st["case"], st["ins"], st["out"]
    kind = case["kind"]
    if kind == "attn":
        q, k, v = ins
        if case["stats"]:
            sd.forward_ex(q, k, v, out, _scale(case["D"]), ls=st["ls"])
            return out, st["ls"]
        if case["dtype"] == "f16":
            return sd.forward(q, k, v, out, _scale(case["D"]))
        return sd.forward_ex(q, k, v, out, _scale(case["D"]))
    if kind == "block":
        x, wq, wk, wv, wo, bo = ins
        return sd.attention_block(x, x, wq, wk, wv, wo, bo, out, st["ws"], case["H"],
                                  _scale(case["C"] // case["H"]))
    if kind == "block_kv":
        x, wq, k, v, wo, bo = ins
        return sd.attention_block_kv(x, wq, k, v, wo, bo, out, st["ws"],
                                     _scale(case["C"] // case["H"]))
    if kind == "conv":
        x, u, bias = ins
        return sd.conv3x3(x, u, out, st["ws"], bias=bias)
    if kind == "norm_geglu":
        x, gamma, beta, h = ins
        sd.group_norm(x, GROUPS, out, gamma, beta, EPS)
        return out, sd.geglu(h, st["act"])
    q, k, v = ins
    a, ls = st["a"], st["ls"]
    sd.logits(q, k, a, _scale(case["D"]))
    sd.softmax_rows(a.view(-1, case["Lk"]), ls.view(-1, 2))
    return sd.softmax_pv(a, ls, v, out), ls, a


# ---------------------------------------------------------------- work, tolerance, reference

def work(case):
    """Bytes: every input read once, every output written once (2-byte
    elements); the two-pass logits are an output of the first call and an input
    of the two others.  Flops: the definition's multiply-adds; a convolution's
    are those of its 36 products per 4x4 tile."""
    kind, B = case["kind"], case["B"]
    if kind in ("attn", "twopass"):
        H, Lq, Lk, D = case["H"], case["Lq"], case["Lk"], case["D"]
        nbytes = 4 * B * H * D * (Lq + Lk)
        if kind == "twopass":
            nbytes += 3 * 2 * B * H * Lq * Lk + 2 * 8 * B * H * Lq
        elif case["stats"]:
            nbytes += 8 * B * H * Lq
        return dict(bytes=nbytes, flops=4 * B * H * Lq * Lk * D)
    if kind in ("block", "block_kv"):
        L, C = case["Lq"], case["C"]
        if kind == "block":
            return dict(bytes=2 * (2 * B * L * C + 4 * C * C),
                        flops=8 * B * L * C * C + 4 * B * L * L * C)
        Lk = case["Lk"]
        return dict(bytes=2 * (2 * B * L * C + 2 * C * C + 2 * B * Lk * C),
                    flops=4 * B * L * C * C + 4 * B * L * Lk * C)
    if kind == "conv":
        Ci, Co, h, w = case["Ci"], case["Co"], case["h"], case["w"]
        tiles = B * ((h + 3) // 4) * ((w + 3) // 4)
        return dict(bytes=2 * (B * (Ci + Co) * h * w + 36 * Ci * Co), flops=2 * 36 * tiles * Ci * Co)
    C, n = case["C"], case["h"] * case["w"]
    # two reductions, a scale and a shift per value; about twenty for a gated value
    return dict(bytes=2 * (2 * B * C * n + 12 * B * C * n), flops=6 * B * C * n + 20 * 4 * B * C * n)


# Relative error (2-norm) of this path against exact(), by kind and type, times
# about four.
REL = {"attn": {"f16": 1.2e-3, "bf16": 1e-2}, "block": {"f16": 2e-3, "bf16": 1.6e-2},
       "block_kv": {"f16": 1.6e-3, "bf16": 1.2e-2}, "conv": {"f16": 1e-2, "bf16": 8e-2},
       "norm_geglu": {"f16": 8e-4, "bf16": 7e-3}, "twopass": {"f16": 2.4e-3, "bf16": 2e-2}}


def tolerance(case):
    return {"rel": REL[case["kind"]][case["dtype"]]}


def _attention(q, k, v, scale):
    """softmax(scale q k^T) v and the row statistics, one (batch, head) at a time."""
    B, H, Lq, D = q.shape
    out = torch.empty(B, H, Lq, D, dtype=torch.float64, device=q.device)
    ls = torch.empty(B, H, Lq, 2, dtype=torch.float64, device=q.device)
    for b in range(B):
        for h in range(H):
            a = (q[b, h] @ k[b, h].t().contiguous()) * scale
            top = a.amax(dim=1, keepdim=True)
            p = (a - top).exp()
            s = p.sum(dim=1, keepdim=True)
            out[b, h] = (p @ v[b, h]) / s
            ls[b, h] = torch.cat([top, s], dim=1)
    return out, ls


def _logits(q, k, scale):
    B, H, Lq, _ = q.shape
    a = torch.empty(B, H, Lq, k.shape[2], dtype=torch.float64, device=q.device)
    for b in range(B):
        for h in range(H):
            a[b, h] = (q[b, h] @ k[b, h].t().contiguous()) * scale
    return a


def exact(case, seed):
    kind, B = case["kind"], case["B"]
    ins = [t.double() for t in _inputs(case, seed)]
    if kind in ("attn", "twopass"):
        q, k, v = ins
        out, ls = _attention(q, k, v, _scale(case["D"]))
        if kind == "twopass":
            return out, ls, _logits(q, k, _scale(case["D"]))
        return (out, ls) if case["stats"] else out
    if kind in ("block", "block_kv"):
        L, C, H = case["Lq"], case["C"], case["H"]

        def heads(t):
            return t.view(B, -1, H, C // H).transpose(1, 2).contiguous()

        if kind == "block":
            x, wq, wk, wv, wo, bo = ins
            k, v = heads(x @ wk.t()), heads(x @ wv.t())
        else:
            x, wq, k, v, wo, bo = ins
        o, _ = _attention(heads(x @ wq.t()), k, v, _scale(C // H))
        return o.transpose(1, 2).reshape(B, L, C) @ wo.t() + bo
    if kind == "conv":
        x, w, bias = ins
        Co, h, wd = case["Co"], case["h"], case["w"]
        pad = torch.nn.functional.pad(x, (1, 1, 1, 1))
        y = bias.view(1, Co, 1, 1).repeat(B, 1, h, wd)
        for i in range(3):
            for j in range(3):
                m = w[:, :, i, j].contiguous()
                for b in range(B):
                    y[b] += (m @ pad[b, :, i:i + h, j:j + wd].reshape(case["Ci"], -1)).view(Co, h, wd)
        return y
    x, gamma, beta, hid = ins
    C, h, w = case["C"], case["h"], case["w"]
    xg = x.view(B, GROUPS, -1)
    mean = xg.mean(dim=2, keepdim=True)
    var = ((xg - mean) ** 2).mean(dim=2, keepdim=True)
    y = ((xg - mean) / (var + EPS).sqrt()).view(B, C, h, w)
    y = y * gamma.view(1, C, 1, 1) + beta.view(1, C, 1, 1)
    val, gate = hid[:, :4 * C], hid[:, 4 * C:]
    return y, val * (0.5 * gate * (1 + torch.erf(gate * math.sqrt(0.5))))
