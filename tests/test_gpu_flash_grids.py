"""The long-sequence attention on grids of its own (GPU, against 64-bit torch
and, for varying lengths, the CPU oracle; OmniCache §3.2.3).  Calls of few query
tiles take the kernel that shares out the keys; these have more than 768 tiles
of 32 queries, so that every head dimension meets the eight-wave blocks staged
by DMA, the eight- and four-wave ones staged through registers, the four-wave
DMA blocks (head dims 64 and 128) and sequences of varying length.  The
workspace holds NaNs."""
import math

import pytest
import torch

from oc_synth import small_workload
import paper_2607_23844_amd as oc

from parity import check_output_bars, layer_step_parity, rel_err, shapes, to_f64, weights_dev, weights_f64

pytestmark = pytest.mark.gpu
DIMS = [16, 32, 48, 64, 72, 80, 96, 128]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n_seq,L", [
    (9, 260),     # 810 tiles, eight-wave DMA blocks, four keys past a tile of 64
    (16, 130),    # 800 tiles, under 256 keys: eight-wave register-staged blocks
    (30, 130),    # 600 blocks of four waves
    (18, 260),    # four-wave DMA blocks for head dims 64 and 128
])
@pytest.mark.parametrize("dh", DIMS)
def test_grids(dh, n_seq, L):
    heads, C = 10, 64
    print(f"attention grid dh={dh} {n_seq}x{L}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(dh * 1000 + L + n_seq)
    x = torch.randn(n_seq, L, C, generator=g, device="cuda").bfloat16()
    hd = heads * dh
    w = {n: (torch.randn(hd, C, generator=g, device="cuda") / C ** 0.5).bfloat16() for n in ("wq", "wk", "wv")}
    w["wo"] = (torch.randn(C, hd, generator=g, device="cuda") / hd ** 0.5).bfloat16()
    sh = oc.Shape(1, 4, 4, C, heads, dh, 0, "bf16")
    ws = torch.full((oc.attn_workspace_bytes(sh, n_seq, L),), 0x7f, dtype=torch.uint8, device="cuda")
    y, _ = oc.attn_reduced(x, n_seq, L, w, sh, ws=ws)
    q, k, v = ((x.double() @ w[n].double().t()).view(n_seq, L, heads, dh).transpose(1, 2).contiguous()
               for n in ("wq", "wk", "wv"))
    p = torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(dh), dim=3)
    ref = torch.matmul(p, v).transpose(1, 2).reshape(n_seq * L, hd) @ w["wo"].double().t()
    e = rel_err(to_f64(y), ref.cpu().numpy(), "bf16")
    print(f"  err {e:.3g}", flush=True)
    check_output_bars(e, 0.0, "bf16")


@pytest.mark.parametrize("dh", DIMS)
def test_varying_lengths(dh):
    print(f"attention grid, frame patches dh={dh}", flush=True)
    wl = small_workload("frame", F=6, H=16, W=16, C=64, heads=17, head_dim=dh, dtype="bf16", r_frame=0.34, patch_k=2,
                        frame_drift=0.3, n_steps=2, seed=43)    # 816 tiles
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
