"""Attention of few query tiles (GPU, against the CPU oracle, OmniCache
§3.2.3): the waves of a block share out the keys in tiles of 32 and merge.
Key counts around the tile and wave counts, every head dimension, context
rows, several sequences, and frames that keep varying numbers of tokens."""
import numpy as np
import pytest
import torch

from oc_synth import bf16_bits, small_workload
from oracle import oc_oracle as O
import paper_2607_23844_amd as oc

from parity import (check_output_bars, dev_tensor, layer_step_parity, rel_err, shapes, to_f64, weights_dev,
                    weights_f64)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,heads,n_seq,L,n_ctx", [
    (16, 2, 3, 65, 0),      # three tiles of 32 keys: three waves, the last tile one key
    (32, 1, 1, 96, 0),
    (48, 2, 1, 255, 0),     # eight waves, one key short of a full round
    (64, 1, 2, 256, 0),
    (64, 3, 1, 250, 7),     # 257 keys with the context: a second round of one key
    (72, 2, 2, 130, 0),     # zero-padded features
    (80, 1, 1, 521, 0),
    (96, 1, 2, 300, 0),
    (128, 2, 1, 600, 3),
    (64, 4, 1, 4000, 0),    # 500 query tiles: two rounds of blocks
    (32, 6, 1, 4001, 0),    # 756 query tiles, head dim 32
])
def test_few_tiles(dh, heads, n_seq, L, n_ctx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    C = 128
    print(f"attn split dh={dh} heads={heads} {n_seq}x{L}+{n_ctx}", flush=True)
    wl = small_workload("token", F=1, H=4, W=4, C=C, heads=heads, head_dim=dh, dtype="bf16", seed=31)
    rng = np.random.default_rng(dh * 10000 + L)
    sh = oc.Shape(1, 4, 4, C, heads, dh, n_ctx, "bf16")
    xk = bf16_bits(rng.standard_normal((n_seq, L, C)).astype(np.float32))
    ctx = bf16_bits(rng.standard_normal((n_ctx, C)).astype(np.float32)) if n_ctx else None
    # the workspace holds NaNs: padded keys must not reach the outputs
    ws = torch.full((oc.attn_workspace_bytes(sh, n_seq, L),), 0x7f, dtype=torch.uint8, device="cuda:0")
    y, yc = oc.attn_reduced(dev_tensor(wl, xk), n_seq, L, weights_dev(wl), sh,
                            ctx=dev_tensor(wl, ctx) if n_ctx else None, ws=ws)
    torch.cuda.synchronize()
    y64, yc64 = O.attn_reduced(wl.f64(xk), wl.f64(ctx) if n_ctx else None, weights_f64(wl), heads, dh)
    e = rel_err(to_f64(y), y64, "bf16")
    if n_ctx:
        e = max(e, rel_err(to_f64(yc), yc64, "bf16"))
    print(f"  err {e:.3g}", flush=True)
    # the rounding-adjusted bar (long uniform sequences: outputs whose peaks
    # are many times the RMS, whose own rounding exceeds the raw bar)
    check_output_bars(e, 0.0, "bf16")


@pytest.mark.parametrize("dh,k,H,W", [(32, 2, 12, 8), (72, 2, 16, 16), (128, 4, 16, 16)])
def test_varying_lengths(dh, k, H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"attn split, frame patches dh={dh} k={k} {H}x{W}", flush=True)
    wl = small_workload("frame", F=6, H=H, W=W, C=dh, heads=1, head_dim=dh, dtype="bf16", r_frame=0.34, patch_k=k,
                        frame_drift=0.3, n_steps=2, seed=41)
    sh, cf, osh, ocf = shapes(wl)
    dev = torch.device("cuda:0")
    ws, cache = oc.workspace(sh, cf, dev), oc.LayerCache(sh, dev)
    ws.fill_(0x7f)
    W_, W64 = weights_dev(wl), weights_f64(wl)
    ora, valid = None, False
    for s in range(2):
        res, _ = layer_step_parity(wl, wl.steps[s], sh, cf, osh, ocf, cache, ws, ora, valid, None, None, W_, W64,
                                   case="latte_spatial frame patches k2")
        ora, valid = res.y, True
