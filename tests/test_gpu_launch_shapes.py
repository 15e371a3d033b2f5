"""Sizes at which the host picks another launch shape or kernel variant: each is checked against the oracle on sampled
rows (corners, tile edges, text rows, random rows), so that every variant of a dispatch runs at its edges."""
import numpy as np
import pytest
import torch

from oracle import clear_oracle as orc
from paper_2412_16112_amd import clear_attn as ca
from paper_2412_16112_amd.inputs import make_qkv_shape
from tests.parity_util import TOL, error_metrics

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(n_text, gh, gw, seed, n=96):
    rng = np.random.default_rng(seed)
    img = {(y, x) for y in (0, 3, 4, 7, 8, 15, 16, gh - 1) for x in (0, 3, 4, 7, 8, 15, 16, gw - 1) if 0 <= y < gh and 0 <= x < gw}
    rows = [n_text + y * gw + x for y, x in img] + list(n_text + rng.integers(0, gh * gw, size=n))
    if n_text:
        rows += [0, n_text - 1] + list(rng.integers(0, n_text, size=24))
    return np.unique(np.array(rows, dtype=np.int64))


# BH workgroup counts on either side of the rule's lines: four, two and one waves per query patch (groups 4, 2, 1), text
# rows in one key range (written directly) and in several (merged), without text, tiles cut by both borders, every mask
@pytest.mark.parametrize("B,H,n_text,gh,gw,r,kind,shift", [
    (1, 1, 8, 16, 16, 4, ca.CLEAR_MASK_DISC, 0),      # groups 4
    (1, 3, 17, 37, 29, 9, ca.CLEAR_MASK_DISC, 0),     # groups 4, cut tiles
    (1, 6, 70, 44, 41, 8, ca.CLEAR_MASK_DISC, 0),     # groups 2, cut tiles
    (2, 6, 0, 36, 60, 5, ca.CLEAR_MASK_DISC, 0),      # groups 2, no text
    (1, 10, 333, 64, 61, 16, ca.CLEAR_MASK_DISC, 0),  # groups 1, several key ranges
    (1, 12, 33, 66, 50, 6, ca.CLEAR_MASK_SQUARE, 0),  # groups 1
    (1, 12, 64, 50, 66, 12, ca.CLEAR_MASK_SWIN, 5),   # groups 1, windows off every lattice
])
def test_f32_launch_shapes(B, H, n_text, gh, gw, r, kind, shift):
    print(f"[case] f32 B={B} H={H} n_text={n_text} grid={gh}x{gw} r={r} kind={kind}", flush=True)
    Q, K, V = make_qkv_shape(B, H, n_text, gh, gw, 64, "f32", seed=4000 + gh, device="cpu")
    ctx = ca.ClearAttn(n_text, gh, gw, 64, r, ca.CLEAR_F32, kind, shift)
    try:
        O = torch.full(Q.shape, float("nan"), device=DEV)
        ctx.forward(Q.to(DEV), K.to(DEV), V.to(DEV), O)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    O = O.cpu()
    assert torch.isfinite(O).all()
    rows = _rows(n_text, gh, gw, seed=gh)
    for b, h in ((0, 0), (B - 1, H - 1)):
        with orc.mask_kind(kind, shift):
            ref = orc.attention_rows(*(t[b, h].double().numpy() for t in (Q, K, V)), rows, n_text, gh, gw, r)
        mx, rms = error_metrics(O[b, h].numpy()[rows], ref)
        assert mx <= TOL["f32"][0] and rms <= TOL["f32"][1], (mx, rms)


# bf16: few workgroups (several waves per query patch, joined in LDS; text rows in one key range and written directly), about one per
# CU, and several (one wave per patch, text rows in key ranges and merged), text tiles of every filling, tiles cut by both
# borders, masks that depend on more than the offset
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B,H,n_text,gh,gw,r,kind,shift", [
    (1, 1, 8, 16, 16, 4, ca.CLEAR_MASK_DISC, 0),  # four waves per patch of text queries, two of them without a key in the last stage
    (1, 1, 31, 20, 20, 6, ca.CLEAR_MASK_DISC, 0),
    (1, 2, 512, 33, 31, 16, ca.CLEAR_MASK_DISC, 0),
    (2, 6, 65, 37, 45, 9, ca.CLEAR_MASK_DISC, 0),
    (1, 14, 97, 61, 50, 16, ca.CLEAR_MASK_DISC, 0),
    (1, 24, 200, 76, 68, 13, ca.CLEAR_MASK_DISC, 0),
    (1, 3, 0, 130, 120, 32, ca.CLEAR_MASK_DISC, 0),
    (1, 5, 40, 50, 66, 12, ca.CLEAR_MASK_SWIN, 5),
    (1, 9, 12, 43, 39, 7, ca.CLEAR_MASK_SQUARE, 0),
    (1, 2, 50, 38, 45, 5, ca.CLEAR_MASK_STRIDED, 17),
])
def test_bf16_launch_shapes(d, B, H, n_text, gh, gw, r, kind, shift):
    print(f"[case] bf16 d={d} B={B} H={H} n_text={n_text} grid={gh}x{gw} r={r} kind={kind}", flush=True)
    Q, K, V = make_qkv_shape(B, H, n_text, gh, gw, d, "bf16", seed=5000 + gh, device="cpu")
    ctx = ca.ClearAttn(n_text, gh, gw, d, r, ca.CLEAR_BF16, kind, shift)
    try:
        Qd, Kd, Vd = Q.to(DEV), K.to(DEV), V.to(DEV)
        O = torch.full(Q.shape, float("nan"), dtype=Q.dtype, device=DEV)
        ctx.forward(Qd, Kd, Vd, O)
        again = ctx.forward(Qd, Kd, Vd)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    assert torch.isfinite(O.float()).all() and torch.equal(O, again)
    O = O.float().cpu()
    rows = _rows(n_text, gh, gw, seed=gh)
    for b, h in ((0, 0), (B - 1, H - 1)):
        with orc.mask_kind(kind, shift):
            ref = orc.attention_rows(*(t[b, h].double().numpy() for t in (Q, K, V)), rows, n_text, gh, gw, r)
        mx, rms = error_metrics(O[b, h].numpy()[rows], ref)
        assert mx <= TOL["bf16"][0] and rms <= TOL["bf16"][1], (mx, rms)


# one key range of text queries whose last stage holds one key tile of two (or of four at 64 channels)
@pytest.mark.parametrize("B,H,n_text,gh,gw,r,d", [(1, 1, 8, 16, 16, 4, 128), (1, 1, 8, 16, 16, 4, 64), (1, 1, 31, 16, 16, 8, 128),
                                                   (1, 1, 128, 12, 12, 5, 128), (1, 1, 9, 20, 20, 6, 64), (2, 2, 100, 14, 14, 6, 128)])
def test_bf16_small_call_does_not_depend_on_what_ran_before(B, H, n_text, gh, gw, r, d):
    """Kernels leave their data in the LDS.  An fp32 call on every CU, with finite values of which every other 16 bits read
    as a bf16 NaN or infinity, in front of a small bf16 call: the same bits as without."""
    print(f"[case] B={B} H={H} n_text={n_text} grid={gh}x{gw} d={d}", flush=True)
    Q, K, V = make_qkv_shape(B, H, n_text, gh, gw, d, "bf16", seed=61, device=DEV)
    q32, k32, v32 = make_qkv_shape(1, 16, 64, 64, 64, 64, "f32", seed=62, device=DEV)
    ctx, ctx32 = ca.ClearAttn(n_text, gh, gw, d, r, ca.CLEAR_BF16), ca.ClearAttn(64, 64, 64, 64, 8, ca.CLEAR_F32)
    got = []
    try:
        for low in (0x0000, 0x7FC0, 0x7F80, 0x3F80):
            dirty = [((t.view(torch.int32) & -65536) | low).view(torch.float32) for t in (q32, k32, v32)]
            ctx32.forward(*dirty)
            got.append(ctx.forward(Q, K, V))
            torch.cuda.synchronize()
    finally:
        ctx.destroy()
        ctx32.destroy()
    assert torch.isfinite(got[0].float()).all()
    for O in got[1:]:
        assert torch.equal(O, got[0])


@pytest.mark.parametrize("H,n_text,gh,gw,range_keys", [(12, 77, 64, 44, 2893), (4, 64, 320, 320, 1664)])
def test_f32_text_rows_round_once_per_cell_of_keys(H, n_text, gh, gw, range_keys):
    """Relative error of the text rows, dense sums over key ranges of at most `range_keys`, against 64 bits.  A range is
    added up in steps of 16 keys: each step rounds the running sum by half an ulp of 2^-24 (root mean square below 2^-25), and as a sum of
    random terms grows like a root, k steps leave 2^-25 sqrt(k / 2) of the result.  12 such halves cover the rest (logits of 64
    products, exponentials, normalisation).  A rounding per key would leave 4 times the first part."""
    print(f"[case] f32 text rows H={H} n_text={n_text} grid={gh}x{gw}", flush=True)
    Q, K, V = make_qkv_shape(1, H, n_text, gh, gw, 64, "f32", seed=71, device=DEV)
    ctx = ca.ClearAttn(n_text, gh, gw, 64, 4, ca.CLEAR_F32)
    try:
        O = ctx.forward(Q, K, V)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    num = den = 0.0
    for h in range(H):
        ref = torch.softmax(Q[0, h, :n_text].double() @ K[0, h].double().T / 8, 1) @ V[0, h].double()
        num += ((O[0, h, :n_text].double() - ref) ** 2).sum().item()
        den += (ref ** 2).sum().item()
    rel = (num / den) ** 0.5
    assert rel <= 2.0 ** -25 * ((range_keys / 16 / 2) ** 0.5 + 12), rel


@pytest.mark.parametrize("n_text,gh,gw,r", [(40, 253, 251, 400), (7, 320, 320, 300)])
def test_bf16_window_of_the_size_of_the_grid(n_text, gh, gw, r):
    """Windows that hold the whole grid (the waves share one program, border masks do not depend on the offset), or about all of it
    (every query tile has programs of its own, tables of several MB copied piece by piece)."""
    print(f"[case] n_text={n_text} grid={gh}x{gw} r={r}", flush=True)
    Q, K, V = make_qkv_shape(1, 1, n_text, gh, gw, 128, "bf16", seed=81, device=DEV)
    ctx = ca.ClearAttn(n_text, gh, gw, 128, r, ca.CLEAR_BF16)
    try:
        O = ctx.forward(Q, K, V)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    rows = _rows(n_text, gh, gw, seed=r, n=64)
    ref = orc.attention_rows(*(t[0, 0].double().cpu().numpy() for t in (Q, K, V)), rows, n_text, gh, gw, r)
    mx, rms = error_metrics(O[0, 0].float().cpu().numpy()[rows], ref)
    assert mx <= TOL["bf16"][0] and rms <= TOL["bf16"][1], (mx, rms)


@pytest.mark.parametrize("n_text", [0, 928, 960, 991, 1024, 1056, 1100, 2975, 3040])
def test_bf16_64_channel_programs_around_64_words(n_text):
    """At 64 channels a wave fetches its program 64 words at a time.  A window that holds a 32 x 32 grid is 32 blocks to every wave, each 32 text keys
    are one more: programs of 63 to 67 and of 125 to 129 words, and of a few."""
    H, gh, gw, r = 64, 32, 32, 64
    print(f"[case] H={H} n_text={n_text} grid={gh}x{gw} r={r}", flush=True)
    Q, K, V = make_qkv_shape(1, H, n_text, gh, gw, 64, "bf16", seed=83, device=DEV)
    ctx = ca.ClearAttn(n_text, gh, gw, 64, r, ca.CLEAR_BF16)
    try:
        O = ctx.forward(Q, K, V)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    rows = _rows(n_text, gh, gw, seed=n_text, n=64)
    for h in (0, H - 1):
        ref = orc.attention_rows(*(t[0, h].double().cpu().numpy() for t in (Q, K, V)), rows, n_text, gh, gw, r)
        mx, rms = error_metrics(O[0, h].float().cpu().numpy()[rows], ref)
        assert mx <= TOL["bf16"][0] and rms <= TOL["bf16"][1], (h, mx, rms)


def test_f32_more_workgroups_than_a_launch_can_have():
    """2 050 heads of a 1 x 32 767 grid are 2^24 workgroups of 256 threads and more, which no single launch can have.  r = 1 without text: a
    token sees itself alone, so O = V."""
    H, gw = 2050, 32767
    print(f"[case] f32 H={H} grid=1x{gw}", flush=True)
    V = torch.empty((1, H, gw, 64), device=DEV)
    V.normal_(generator=torch.Generator(device=DEV).manual_seed(91))
    O = torch.empty_like(V)
    ctx = ca.ClearAttn(0, 1, gw, 64, 1, ca.CLEAR_F32)
    try:
        ctx.forward(V, V, V, O)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    assert all(torch.equal(O[0, h:h + 82], V[0, h:h + 82]) for h in range(0, H, 82))


def test_bf16_more_workgroups_than_a_launch_can_have():
    """Thin grids of many heads: 2 731 heads of 1 x 32 767 are more than 2^32 threads for the forward kernel (768 a workgroup, 2 048
    workgroups a head), 4 097 for the backward kernels (512 a workgroup).  r = 1 without text: a token sees itself alone, so O = V, dV = dO and
    dQ = dK = 0 but for what two fp32 sums of the same 64 products differ by, dP and delta: 2 x 64 x 2^-24 of the products' sizes, which add up to
    less than 100, times a key below 6 and the scale 1/8: 6e-4."""
    H, gw = 4097, 32767
    print(f"[case] bf16 H={H} grid=1x{gw}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(92)
    V, dO = (torch.empty((1, H, gw, 64), dtype=torch.bfloat16, device=DEV).normal_(generator=gen) for _ in range(2))
    ctx = ca.ClearAttn(0, 1, gw, 64, 1, ca.CLEAR_BF16)
    heads = [(h, min(h + 100, H)) for h in range(0, H, 100)]
    try:
        O, lse = ctx.forward_lse(V, V, V)
        torch.cuda.synchronize()
        assert all(torch.equal(O[0, a:b], V[0, a:b]) for a, b in heads)
        for a, b in heads:
            s = (V[0, a:b].float() ** 2).sum(-1) / 8
            assert ((lse[0, a:b] - s).abs() <= 1e-5 * (1 + s)).all()
        dQ, dK, dV = ctx.backward(V, V, V, O, dO, lse)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    assert all(torch.equal(dV[0, a:b], dO[0, a:b]) for a, b in heads)
    assert all(float(t[0, a:b].abs().max()) <= 6e-4 for t in (dQ, dK) for a, b in heads)


@pytest.mark.parametrize("B,H,n_text,gh,gw,r,kind,shift", [
    (1, 1, 8, 16, 16, 4, ca.CLEAR_MASK_DISC, 0),      # four waves per patch
    (1, 6, 70, 44, 41, 8, ca.CLEAR_MASK_DISC, 0),     # two, cut tiles
    (1, 10, 33, 64, 61, 16, ca.CLEAR_MASK_DISC, 0),   # one, several key ranges of the text rows
    (1, 2, 0, 37, 29, 5, ca.CLEAR_MASK_SQUARE, 0),
    (1, 3, 20, 50, 66, 12, ca.CLEAR_MASK_SWIN, 5),
])
def test_f32_non_finite_values_reach_only_the_queries_that_see_them(B, H, n_text, gh, gw, r, kind, shift):
    """An infinity and a NaN in V, at tokens inside the grid and in its last corner: queries whose window holds neither come out as
    if they were not there, the others as the plain sum has them."""
    print(f"[case] f32 non-finite V H={H} n_text={n_text} grid={gh}x{gw} r={r} kind={kind}", flush=True)
    Q, K, V = make_qkv_shape(B, H, n_text, gh, gw, 64, "f32", seed=95, device=DEV)
    spots = [(n_text + (gh // 2) * gw + gw // 3, 5, float("inf")), (n_text + gh * gw - 1, 40, float("nan"))]
    clean = V.clone()
    for token, ch, value in spots:
        V[:, :, token, ch] = value
    ctx = ca.ClearAttn(n_text, gh, gw, 64, r, ca.CLEAR_F32, kind, shift)
    try:
        O, ref = ctx.forward(Q, K, V), ctx.forward(Q, K, clean)
        torch.cuda.synchronize()
    finally:
        ctx.destroy()
    pos = torch.arange(gh * gw, device=DEV)
    y, x = pos // gw, pos % gw
    for token, ch, value in spots:
        ky, kx = (token - n_text) // gw, (token - n_text) % gw
        if kind == ca.CLEAR_MASK_DISC:
            sees = (y - ky) ** 2 + (x - kx) ** 2 < r * r
        elif kind == ca.CLEAR_MASK_SQUARE:
            sees = ((y - ky).abs() < r) & ((x - kx).abs() < r)
        else:
            sees = ((y + shift) // r == (ky + shift) // r) & ((x + shift) // r == (kx + shift) // r)
        sees = torch.cat([torch.ones(n_text, dtype=torch.bool, device=DEV), sees])
        got = O[..., ch]
        assert (torch.isnan(got) if value != value else torch.isinf(got))[..., sees].all()
        assert torch.isfinite(got[..., ~sees]).all()
    finite = torch.isfinite(O)
    assert int((~finite).sum()) < O.numel() // 20
    # the keys one by one in place of cells: two fp32 sums of at most some thousand terms, relative to values of order one
    assert (O - ref).abs()[finite].max() <= 2e-5
