"""Compaction over several blocks (GPU, bit-exact against the CPU oracle,
OmniCache §3.2.1, §3.2.3): partial last blocks, several frames, patch-local
groups and the second level, cold and warm maps; and tile norms of one block
per tile with 256 and 1024 threads."""
import pytest
import torch

from oc_synth import small_workload
import paper_2607_23844_amd as oc

from parity import layer_step_parity, shapes, weights_dev, weights_f64

pytestmark = pytest.mark.gpu

CASES = [
    ("block", dict(F=5, H=12, W=12, C=32, patch_k=2, r=0.5), {}),            # 144 positions: 2.25 blocks of 64
    ("block", dict(F=2, H=20, W=10, C=32, patch_k=5, r=0.7), {}),            # 200 positions, groups of 8
    ("block", dict(F=3, H=48, W=48, C=32, patch_k=4, r=0.25), {}),           # 36 blocks
    ("token", dict(F=2, H=48, W=44, C=32, patch_k=2, r=0.4), {}),            # 2112 tokens: 2 chunks and 64 tokens
    ("token", dict(F=3, H=8, W=8, C=32, patch_k=2, r=0.5), {}),              # one partial chunk per frame
    ("token", dict(F=1, H=48, W=48, C=32, patch_k=4, r=0.25), dict(coarse_k=2, r_coarse=0.2)),
    ("frame", dict(F=4, H=32, W=32, C=128, patch_k=2, r_frame=0.25, frame_drift=0.3), {}),   # tiles of 64 KB
    ("frame", dict(F=4, H=36, W=32, C=120, patch_k=2, r_frame=0.5, frame_drift=0.3), {}),    # just above
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_compaction_chain(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gran, kw, two = CASES[case]
    print(f"compaction {gran} {kw} {two}", flush=True)
    wl = small_workload(gran, heads=1, head_dim=32, dtype="bf16", n_steps=2, seed=600 + case, **kw)
    sh, cf, osh, ocf = shapes(wl, **two)
    dev = torch.device("cuda:0")
    ws, cache = oc.workspace(sh, cf, dev), oc.LayerCache(sh, dev)
    W, W64 = weights_dev(wl), weights_f64(wl)
    ora, valid = None, False
    for s in range(2):
        res, _ = layer_step_parity(wl, wl.steps[s], sh, cf, osh, ocf, cache, ws, ora, valid, None, None, W, W64,
                                   case="latte_spatial frame patches k2" if gran == "frame" else "")
        ora, valid = res.y, True
