"""fp32 layers on fp32 MFMA tiles (GPU, against the CPU oracle, OmniCache
§3.2): edges of the 32 x 32 and 64 x 64 tiles and of the K chunks, every
16-element step count of the head dimension, key counts around the runs of
32 keys and the wave counts, and long descriptors."""
import numpy as np
import pytest
import torch

from oc_synth import small_workload
from oracle import oc_oracle as O
import paper_2607_23844_amd as oc

from parity import (check_output_bars, dev_tensor, layer_step_parity, rel_err, shapes, to_f64, weights_dev,
                    weights_f64)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,heads,C,n_seq,L,n_ctx", [
    (8, 1, 8, 1, 1, 0),          # one token, one K chunk of 8
    (8, 3, 24, 5, 17, 0),        # one wave, a query tile of one row past 16
    (24, 2, 40, 2, 33, 0),       # two waves, K not a multiple of 16
    (40, 1, 136, 1, 64, 1),      # K just past one chunk of 128; a context row
    (56, 2, 112, 1, 129, 0),     # eight waves, the last run one key
    (64, 2, 128, 3, 250, 0),
    (72, 2, 144, 1, 100, 5),     # four waves (wide heads)
    (104, 1, 104, 2, 40, 0),
    (120, 2, 240, 1, 257, 0),
    (128, 3, 384, 1, 300, 7),
    (64, 10, 640, 1, 1300, 0),   # 64 x 64 tiles in both projections
])
def test_attn_reduced_f32(dh, heads, C, n_seq, L, n_ctx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"attn f32 dh={dh} heads={heads} C={C} {n_seq}x{L}+{n_ctx}", flush=True)
    wl = small_workload("token", F=1, H=4, W=4, C=C, heads=heads, head_dim=dh, dtype="f32", seed=21)
    rng = np.random.default_rng(dh * 1000 + L)
    sh = oc.Shape(1, 4, 4, C, heads, dh, n_ctx, "f32")
    xk = rng.standard_normal((n_seq, L, C)).astype(np.float32)
    ctx = rng.standard_normal((n_ctx, C)).astype(np.float32) if n_ctx else None
    y, yc = oc.attn_reduced(dev_tensor(wl, xk), n_seq, L, weights_dev(wl), sh,
                            ctx=dev_tensor(wl, ctx) if n_ctx else None)
    torch.cuda.synchronize()
    y64, yc64 = O.attn_reduced(wl.f64(xk), wl.f64(ctx) if n_ctx else None, weights_f64(wl), heads, dh)
    e = rel_err(to_f64(y), y64)
    if n_ctx:
        e = max(e, rel_err(to_f64(yc), yc64))
    print(f"  err {e:.3g}", flush=True)
    check_output_bars(e, e, "f32")


@pytest.mark.parametrize("kw", [
    dict(gran="token", F=1, H=10, W=6, C=40, heads=1, head_dim=40, r=0.5),                 # one ragged tile
    dict(gran="token", F=1, H=64, W=40, C=136, heads=1, head_dim=16, r=0.5),               # 64 x 64 tiles
    dict(gran="token", F=3, H=16, W=16, C=72, heads=1, head_dim=72, r=0.6, patch_k=2),
    dict(gran="block", F=6, H=20, W=12, C=24, heads=3, head_dim=8, r=0.5),                 # segments of 24
    dict(gran="frame", F=6, H=12, W=8, C=48, heads=2, head_dim=24, r_frame=0.3, patch_k=2, frame_drift=0.3),
    dict(gran="frame_token", F=6, H=8, W=8, C=64, heads=1, head_dim=64, r=0.4, r_frame=0.34, planted=True),
], ids=lambda k: f"{k['gran']}_{k['H']}x{k['W']}_C{k['C']}")
def test_chain_f32(kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"f32 chain {kw}", flush=True)
    wl = small_workload(dtype="f32", n_steps=2, seed=77, **kw)
    sh, cf, osh, ocf = shapes(wl)
    dev = torch.device("cuda:0")
    ws, cache = oc.workspace(sh, cf, dev), oc.LayerCache(sh, dev)
    W, W64 = weights_dev(wl), weights_f64(wl)
    ora, valid = None, False
    for s in range(2):
        res, _ = layer_step_parity(wl, wl.steps[s], sh, cf, osh, ocf, cache, ws, ora, valid, None, None, W, W64,
                                   case="f32 chain")
        ora, valid = res.y, True
