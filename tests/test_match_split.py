"""The K split of the Block Cache similarity (OmniCache §3.2.1): a split stays
inside one frame's channels, so with many frames over a middling number of
similarity tiles the whole frame is the longest split."""
import subprocess
import sys

import pytest
import torch

from oc_synth import small_workload
import paper_2607_23844_amd as oc

from parity import layer_step_parity, shapes, weights_dev, weights_f64

PLANS = """
import paper_2607_23844_amd as oc
for F, H, W, C, k in ((16, 32, 32, 1152, 1), (18, 16, 8, 192, 4), (32, 16, 16, 64, 2), (17, 32, 32, 128, 1),
                      (16, 16, 16, 1152, 1), (25, 24, 24, 320, 1)):
    sh, cf = oc.Shape(F, H, W, C, 1, 64, 0, "bf16"), oc.Cfg("block", r=0.5, patch_k=k)
    pl = oc.plan(sh, cf)
    # room for the partials of at most one split per frame and 64 channels
    most = F * C // 64 * pl.n_groups * pl.n_src_max * pl.n_dst_max * 4
    assert 0 < pl.workspace_bytes <= most + 64 * F * H * W * C + (1 << 20), (F, H, W, C, k)
"""


def test_plan_returns_for_many_frames():
    # in a child process: a split search without an end would not return
    r = subprocess.run([sys.executable, "-c", PLANS], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-800:]


@pytest.mark.gpu
@pytest.mark.parametrize("F,H,W,C,k", [(18, 16, 8, 192, 4), (17, 32, 32, 64, 1), (32, 16, 16, 64, 2)])
def test_chain_with_whole_frame_splits(F, H, W, C, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = small_workload("block", F=F, H=H, W=W, C=C, heads=1, head_dim=64, dtype="bf16", r=0.5, patch_k=k, n_steps=2,
                        seed=501)
    print(f"block split: F={F} {H}x{W} C={C} k={k}", flush=True)
    sh, cf, osh, ocf = shapes(wl)
    dev = torch.device("cuda:0")
    ws, cache = oc.workspace(sh, cf, dev), oc.LayerCache(sh, dev)
    W_, W64 = weights_dev(wl), weights_f64(wl)
    ora, valid = None, False
    for s in range(2):
        res, _ = layer_step_parity(wl, wl.steps[s], sh, cf, osh, ocf, cache, ws, ora, valid, None, None, W_, W64,
                                   case="block split")
        ora, valid = res.y, True
