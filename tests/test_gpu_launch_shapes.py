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
