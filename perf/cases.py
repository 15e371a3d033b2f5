"""Workloads for timing this library through its public entry points: what a program that serves or trains a model with
CLEAR local attention calls, over the range of sizes, data types and options the library is built for.

`listed()` names twelve of them, `draw(rng)` gives another of the same ranges, `prepare` makes what such a program holds
before the call (tensors, context), `run` is one call as it makes it, `work` the bytes and operations one pass cannot do
without, `tolerance` how far two correct implementations of the same precision may be apart.

A case is a dict: op ("forward", "prologue", "train", "band"), dtype, B, H, n_text, gridH, gridW, d, r, mask, shift and,
for a band, n_bands and band (gridH is then the whole image's)."""
import math

import torch

from paper_2412_16112_amd import clear_attn as ca
from paper_2412_16112_amd.autograd import clear_attention
from paper_2412_16112_amd.inputs import make_prologue_inputs

MASKS = {"disc": ca.CLEAR_MASK_DISC, "square": ca.CLEAR_MASK_SQUARE, "swin": ca.CLEAR_MASK_SWIN, "strided": ca.CLEAR_MASK_STRIDED}


def _case(op, B, H, n_text, gridH, gridW, d, r, dtype="bf16", mask="disc", shift=0, **more):
    return dict(op=op, dtype=dtype, B=B, H=H, n_text=n_text, gridH=gridH, gridW=gridW, d=d, r=r, mask=mask, shift=shift, **more)


def listed():
    return [
        # the smallest call: a unit test or a debugging session of a model, one head in fp32; launches and host work
        dict(_case("forward", 1, 1, 8, 16, 16, 64, 4, dtype="f32"), name="tiny-f32"),
        # a whole layer of SD3.5-Large geometry in fp32 (38 heads of 64 channels, 1024 x 1024 pixels): a reference run
        dict(_case("forward", 1, 38, 333, 64, 64, 64, 16, dtype="f32"), name="sd35l-1024-f32"),
        # a preview or thumbnail, 512 x 512 pixels, FLUX geometry: a fraction of the chip's CUs
        dict(_case("forward", 1, 24, 512, 32, 32, 128, 8), name="flux-512"),
        # the ordinary image, 1024 x 1024 pixels
        dict(_case("forward", 1, 24, 512, 64, 64, 128, 16), name="flux-1024"),
        # SD3.5-Large geometry with classifier-free guidance: two prompts in the batch, head_dim 64
        dict(_case("forward", 2, 38, 333, 64, 64, 64, 16), name="sd35l-1024-cfg"),
        # 1360 x 768 pixels and a short prompt: no size a multiple of a tile
        dict(_case("forward", 1, 24, 77, 48, 85, 128, 16), name="flux-ragged"),
        # a wide image at the large radius
        dict(_case("forward", 1, 24, 512, 192, 320, 128, 32), name="flux-4096-wide-r32"),
        # the largest: 8192 x 8192 pixels
        dict(_case("forward", 1, 24, 512, 512, 512, 128, 16), name="flux-8k"),
        # the attention of a block as inference runs it: raw projections in token-major storage, RMS norm, rotary
        # embedding and logit scale fused in, 2048 x 2048 pixels
        dict(_case("prologue", 1, 24, 512, 128, 128, 128, 16), name="flux-2048-prologue"),
        # one distillation step's attention, forward and backward through autograd, at the training resolution
        dict(_case("train", 1, 24, 512, 64, 64, 128, 16), name="flux-1024-train"),
        # one of eight row bands of the 8192 x 8192 image, with the merge of the text rows
        dict(_case("band", 1, 24, 512, 512, 512, 128, 16, n_bands=8, band=4), name="flux-8k-band"),
        # one of the compared local masks: shifted windows at 2048 x 2048 pixels
        dict(_case("forward", 1, 24, 512, 128, 128, 128, 16, mask="swin", shift=8), name="flux-2048-swin"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _draw_once(rng):
    op = rng.choices(["forward", "train", "prologue", "band"], [10, 5, 3, 2])[0]
    dtype = "f32" if op == "forward" and rng.random() < 0.2 else "bf16"
    d = 64 if dtype == "f32" or rng.random() < 0.35 else 128
    gridH = _log_int(rng, 12, {"train": 128, "prologue": 256}.get(op, 64 if dtype == "f32" else 512))
    gridW = max(12, min(512, round(gridH * math.exp(rng.uniform(-0.7, 0.7)))))
    if rng.random() < 0.5:  # image sides are often multiples of 128 pixels
        gridH, gridW = max(16, gridH // 8 * 8), max(16, gridW // 8 * 8)
    H = rng.choice([24, 38]) if rng.random() < 0.6 else _log_int(rng, 1, 40)
    B = rng.choice([1, 1, 1, 2, 4])
    n_text = rng.choice([77, 333, 512]) if rng.random() < 0.6 else rng.randint(0, 512)
    r = rng.choice([8, 16, 32]) if rng.random() < 0.7 else rng.randint(4, 32)
    c = _case(op, B, H, n_text, gridH, gridW, d, r, dtype=dtype)
    if op == "forward" and dtype == "bf16" and rng.random() < 0.25:
        c["mask"] = rng.choice(["square", "swin", "strided"])
        if c["mask"] == "swin":
            c["shift"] = rng.choice([0, r // 2])
        if c["mask"] == "strided":
            c["r"] = min(r, 16, gridH, gridW)
            c["shift"] = rng.randrange(c["r"] * c["r"])
    if op == "band":
        c["n_bands"] = rng.choice([2, 3, 4, 8])
        c["band"] = rng.randrange(c["n_bands"])
        c["gridH"] = max(gridH, c["n_bands"] * r)
    return c


def draw(rng):
    top = work(_case("forward", 1, 24, 512, 512, 512, 128, 16))
    top_f32 = work(_case("forward", 1, 38, 333, 64, 64, 64, 16, dtype="f32"))
    while True:
        c = _draw_once(rng)
        w, most = work(c), top_f32 if c["dtype"] == "f32" else top
        share = 1.0 if c["mask"] == "disc" and c["d"] == 128 else 0.4  # (these reach less of the matrix rate)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"] * share:
            return c


def _band_layout(c):
    y0, y1, top, bottom = ca.clear_attn_band_layout(c["gridH"], c["r"], c["n_bands"], c["band"])
    return y0, y1, top, top + (y1 - y0) + bottom  # owned rows, halo above, rows of the band's own grid


class State:
    """What run() gets: the case's plain values and the tensors and handles made for it."""

    def __init__(self, **have):
        self.__dict__.update(have)


def _normal(gen, shape, dtype, scale=1.0):
    x = torch.empty(shape, dtype=dtype, device="cuda")
    for b in range(shape[0]):
        x[b].normal_(generator=gen)
    return x if scale == 1.0 else x.mul_(scale)


def prepare(case, seed):
    op, B, H, n_text, d, r = (case[k] for k in ("op", "B", "H", "n_text", "d", "r"))
    gridH, gridW = case["gridH"], case["gridW"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    code = ca.CLEAR_F32 if case["dtype"] == "f32" else ca.CLEAR_BF16
    if op == "band":
        y0, y1, top, gridH = _band_layout(case)
    N = n_text + gridH * gridW
    token_major = op in ("train", "prologue")  # as the projections leave them: [B, N, H, d], passed as transposed views
    shape = (B, N, H, d) if token_major else (B, H, N, d)
    raw = 2.0 if op == "prologue" else 1.0  # raw projections are normalised by the call, the others were before it
    Q, K, V = (_normal(gen, shape, dtype, raw if t < 2 else 1.0) for t in range(3))
    # heads differ in how sharp their logits are
    sharp = (0.5 + 1.5 * torch.rand(H, generator=gen, device="cuda")).to(dtype)
    Q.mul_(sharp.view(1, 1, H, 1) if token_major else sharp.view(1, H, 1, 1))
    if token_major:
        Q, K, V = (t.transpose(1, 2) for t in (Q, K, V))
    s = State(op=op, Q=Q, K=K, V=V, n_text=n_text, gridH=gridH, gridW=gridW, r=r, mask=MASKS[case["mask"]], shift=case["shift"])
    if op == "train":
        s.dO = _normal(gen, shape, dtype).transpose(1, 2)
        for t in (Q, K, V):
            t.requires_grad_(True)
        return s
    s.ctx = ca.ClearAttn(n_text, gridH, gridW, d, r, code, s.mask, s.shift)
    s.ctx.reserve(B * H)
    if op == "prologue":
        s.q_gain, s.k_gain, s.rope_y, s.rope_x = make_prologue_inputs(gridH, gridW, d, int(seed) % (1 << 31), ntk_factor=10.0, device="cuda")
        s.O = torch.zeros(shape, dtype=dtype, device="cuda").transpose(1, 2)
        return s
    s.O = torch.zeros(shape, dtype=dtype, device="cuda")
    if op == "band":
        s.own = (top, top + (y1 - y0))
        # text rows: this band's result and what the other bands have sent
        s.text_o = [0.1 * torch.randn((B, H, n_text, d), generator=gen, device="cuda") for _ in range(case["n_bands"])]
        s.text_lse = [8.0 + 0.1 * torch.randn((B, H, n_text), generator=gen, device="cuda") for _ in range(case["n_bands"])]
        s.band = case["band"]
    return s


def run(state):
    s = state
    if s.op == "train":
        O = clear_attention(s.Q, s.K, s.V, s.n_text, s.gridH, s.gridW, s.r, s.mask, s.shift)
        return (O,) + torch.autograd.grad(O, (s.Q, s.K, s.V), s.dO)
    if s.op == "prologue":
        return s.ctx.forward_strided(s.Q, s.K, s.V, s.O, q_gain=s.q_gain, k_gain=s.k_gain, rope_y=s.rope_y, rope_x=s.rope_x, logit_scale=1.1)
    if s.op == "band":
        to, tl = s.text_o[s.band], s.text_lse[s.band]
        s.ctx.forward_band(s.Q, s.K, s.V, s.O, s.own[0], s.own[1], True, to, tl)
        if s.n_text == 0:
            return s.O
        ca.clear_attn_merge_text(s.text_o, s.text_lse, s.O, s.n_text, ca.CLEAR_MERGE_AVERAGE)
        return s.O, to, tl
    return s.ctx.forward(s.Q, s.K, s.V, s.O)


def _band_pairs(c):
    """(query, key) pairs of one band: its image queries, and the text queries over the text and the owned rows."""
    y0, y1, _, _ = _band_layout(c)
    n_text, W, r = c["n_text"], c["gridW"], c["r"]
    pairs = (y1 - y0) * W * n_text + n_text * (n_text + (y1 - y0) * W)
    for dy in range(-r + 1, r):
        rows = max(0, min(y1, c["gridH"] - dy) - max(y0, -dy))
        reach = math.isqrt(r * r - dy * dy - 1)  # the largest dx with dx^2 + dy^2 < r^2
        pairs += rows * sum(max(0, W - abs(dx)) for dx in range(-reach, reach + 1))
    return pairs


def work(case):
    c = case
    heads, d, size = c["B"] * c["H"], c["d"], 4 if c["dtype"] == "f32" else 2
    if c["op"] == "band":
        y0, y1, _, rows = _band_layout(c)
        pairs = _band_pairs(c)
        own, local = c["n_text"] + (y1 - y0) * c["gridW"], c["n_text"] + rows * c["gridW"]
        parts = 4 * c["n_text"] * (d + 1) * (1 + c["n_bands"])  # written for this band, read for all of them
        return {"bytes": heads * (2 * d * size * (own + local) + parts), "flops": 4.0 * pairs * d * heads}
    N = c["n_text"] + c["gridH"] * c["gridW"]
    pairs = ca.clear_attn_mask_count_masked(c["n_text"], c["gridH"], c["gridW"], c["r"], MASKS[c["mask"]], c["shift"])
    if c["op"] == "train":  # Q, K, V, dO in; O, dQ, dK, dV out; two products forward, five backward
        return {"bytes": 8 * heads * N * d * size, "flops": 14.0 * pairs * d * heads}
    return {"bytes": 4 * heads * N * d * size, "flops": 4.0 * pairs * d * heads}


def tolerance(case):
    # fp32: sums of a few thousand products and exponentials in fp32.  bf16: probabilities and outputs are rounded to
    # 8 bits, each half an ulp (2^-9 = 2e-3) of its own value.
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
