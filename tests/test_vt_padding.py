"""The key padding of the transposed V rows (OmniCache §3.2.3): the attention
that stages keys by DMA multiplies whole 64-key tiles, so every position of
[0, lpad) has to be written by the projection, whatever the workspace held.
The cases are calls whose projection takes tiles of 96 or 160 rows, which end
32 positions short of lpad."""
import numpy as np
import pytest
import torch

from oc_synth import bf16_bits, small_workload
from oracle import oc_oracle as O
import paper_2607_23844_amd as oc

from parity import check_output_bars, dev_tensor, rel_err, to_f64, weights_dev, weights_f64

CASES = [   # heads, head dim, C, sequences, tokens, context; rows of the projection's tile
    (20, 64, 1280, 1, 1024, 77, 160),
    (13, 72, 936, 1, 1414, 0, 160),
    (12, 64, 768, 1, 2060, 0, 160),
    (10, 64, 640, 5, 480, 0, 160),
    (5, 64, 320, 20, 480, 0, 160),
    (4, 64, 256, 8, 1440, 0, 160),
    (16, 72, 1152, 3, 288, 0, 96),
    (16, 72, 1152, 1, 660, 0, 96),
]


@pytest.fixture
def cover(native):
    return native("vt_cover")


def test_every_position_is_written(cover):
    r = cover()
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("heads,dh,C,n_seq,L,n_ctx,tile", CASES)
def test_cases_reach_the_padding(cover, heads, dh, C, n_seq, L, n_ctx, tile):
    """The calls below take the tile they are meant for, whose rows end before
    lpad, and the attention that reads whole 64-key tiles."""
    rows, covered, lpad, dma = map(int, cover(heads, dh, C, n_seq, L, n_ctx).stdout.split())
    assert rows == tile and 0 < covered < lpad and dma == 1


@pytest.mark.gpu
@pytest.mark.parametrize("heads,dh,C,n_seq,L,n_ctx,tile", CASES)
def test_attention_on_any_workspace(heads, dh, C, n_seq, L, n_ctx, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"Vt padding heads={heads} dh={dh} C={C} {n_seq}x{L}+{n_ctx}", flush=True)
    wl = small_workload("token", F=1, H=4, W=4, C=C, heads=heads, head_dim=dh, dtype="bf16", seed=71)
    rng = np.random.default_rng(C * 100 + L)
    sh = oc.Shape(1, 4, 4, C, heads, dh, n_ctx, "bf16")
    xk = bf16_bits(rng.standard_normal((n_seq, L, C)).astype(np.float32))
    ctx = bf16_bits(rng.standard_normal((n_ctx, C)).astype(np.float32)) if n_ctx else None
    ws = torch.full((oc.attn_workspace_bytes(sh, n_seq, L),), 0x7f, dtype=torch.uint8, device="cuda:0")   # NaNs
    y, yc = oc.attn_reduced(dev_tensor(wl, xk), n_seq, L, weights_dev(wl), sh, ctx=dev_tensor(wl, ctx) if n_ctx else None,
                            ws=ws)
    torch.cuda.synchronize()
    y64, yc64 = O.attn_reduced(wl.f64(xk), wl.f64(ctx) if n_ctx else None, weights_f64(wl), heads, dh)
    e = rel_err(to_f64(y), y64, "bf16")
    if n_ctx:
        e = max(e, rel_err(to_f64(yc), yc64, "bf16"))
    print(f"  err {e:.3g}", flush=True)
    check_output_bars(e, 0.0, "bf16")
