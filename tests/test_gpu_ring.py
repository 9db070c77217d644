"""Projections on the ring-buffered tiles (GPU, against the CPU oracle,
OmniCache §3.2.3): a case per tile shape, K below the ring's depth and not a
multiple of 64, ragged rows, context rows in the middle of an instruction's
eight rows, listed rows, and V by rows for short sequences.  (The key padding
after tiles of 96 and 160 rows: test_vt_padding.py.)"""
import numpy as np
import pytest
import torch

from oc_synth import bf16_bits, small_workload
from oracle import oc_oracle as O
import paper_2607_23844_amd as oc

from parity import check_output_bars, dev_tensor, rel_err, to_f64, weights_dev, weights_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,dh,C,n_seq,L,n_ctx", [
    (24, 64, 320, 24, 125, 0),     # 256 x 256 tiles in the Q/K/V projection
    (24, 64, 520, 20, 105, 0),     # 256 x 192, K tail of 8
    (24, 64, 520, 15, 100, 0),     # 256 x 128
    (18, 64, 1536, 15, 100, 0),    # 128 x 192
    (24, 64, 64, 7, 100, 0),       # 128 x 128, one K step
    (18, 64, 320, 15, 100, 0),     # 128 x 192, two per compute unit
    (24, 64, 136, 10, 100, 0),     # 160 x 128
    (24, 64, 1024, 7, 100, 0),     # 128 x 64
    (1, 64, 64, 1, 70, 0),         # 96 x 128
    (1, 64, 72, 1, 70, 0),         # 64 x 64
    (3, 72, 8, 2, 67, 0),          # one K chunk of 8
    (4, 64, 136, 1, 301, 33),      # the context starts inside an instruction's rows
    (2, 64, 64, 1, 0, 77),         # context rows only
    (16, 72, 72, 50, 40, 0),       # short sequences: V by rows
    (8, 64, 1536, 60, 100, 0),     # 256 x 192 in the output projection
    (8, 64, 3072, 20, 100, 0),     # 256 x 128
])
def test_ring_shapes(heads, dh, C, n_seq, L, n_ctx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"ring heads={heads} dh={dh} C={C} {n_seq}x{L}+{n_ctx}", flush=True)
    wl = small_workload("token", F=1, H=4, W=4, C=C, heads=heads, head_dim=dh, dtype="bf16", seed=61)
    rng = np.random.default_rng(C * 100 + L)
    sh = oc.Shape(1, 4, 4, C, heads, dh, n_ctx, "bf16")
    xk = bf16_bits(rng.standard_normal((n_seq, L, C)).astype(np.float32))
    ctx = bf16_bits(rng.standard_normal((n_ctx, C)).astype(np.float32)) if n_ctx else None
    ws = torch.full((oc.attn_workspace_bytes(sh, n_seq, L),), 0x7f, dtype=torch.uint8, device="cuda:0")
    xd = dev_tensor(wl, xk) if L else torch.zeros((1, 1, C), dtype=torch.bfloat16, device="cuda:0")
    y, yc = oc.attn_reduced(xd, n_seq, L, weights_dev(wl), sh, ctx=dev_tensor(wl, ctx) if n_ctx else None, ws=ws)
    torch.cuda.synchronize()
    y64, yc64 = O.attn_reduced(wl.f64(xk), wl.f64(ctx) if n_ctx else None, weights_f64(wl), heads, dh)
    e = rel_err(to_f64(y), y64, "bf16") if L else 0.0
    if n_ctx:
        e = max(e, rel_err(to_f64(yc), yc64, "bf16"))
    print(f"  err {e:.3g}", flush=True)
    check_output_bars(e, 0.0, "bf16")
