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


@pytest.mark.parametrize("gran,F,H,W,k", [
    ("token", 2, 256, 128, 4),     # 32768 tokens: the blocks count the flags before their own
    ("token", 2, 256, 132, 2),     # 33792: from chunk counts
    ("token", 1, 260, 132, 2),     # 34320, the last chunk partial
    ("block", 3, 256, 128, 4),
    ("block", 2, 260, 132, 2),
    ("block", 1, 512, 256, 4),
])
def test_many_tokens(gran, F, H, W, k):
    """The selection of many tokens against its definition, on random
    similarities without ties."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"compaction of many tokens {gran} F={F} {H}x{W} k={k}", flush=True)
    sh, cf = oc.Shape(F, H, W, 8, 1, 16, 0, "bf16"), oc.Cfg(gran, r=0.4, patch_k=k)
    pl = oc.plan(sh, cf)
    G, S, N = pl.n_groups, pl.n_src_max, H * W
    g = torch.Generator(device="cuda").manual_seed(H)
    nm = (torch.randperm(G * S, generator=g, device="cuda").float() / (G * S)).contiguous()
    ni = torch.zeros(G * S, dtype=torch.int32, device="cuda")
    kept, cached, rmap = oc.select(nm, ni, sh, cf, oc.workspace(sh, cf, nm.device))
    # candidates of a patch: its tokens off the even rows and columns, ascending
    ids = torch.arange(N, device="cuda").view(H, W)
    ph, pw = H // k, W // k
    R = int(0.4 * ph * pw)
    Fg = F if gran == "token" else 1
    flag = torch.zeros(Fg, N, dtype=torch.bool, device="cuda")
    for f in range(Fg):
        for p in range(k * k):
            tile = ids[p // k * ph:(p // k + 1) * ph, p % k * pw:(p % k + 1) * pw]
            cand = tile.reshape(-1)
            cand = cand[((cand // W) % 2 == 1) | ((cand % W) % 2 == 1)]
            flag[f, cand[nm[(f * k * k + p) * S:][:S].topk(R).indices]] = True
    if gran == "token":
        want_kept = (~flag).reshape(-1).nonzero().reshape(-1)
        want_cached = flag.reshape(-1).nonzero().reshape(-1)
    else:
        pos = (~flag[0]).nonzero().reshape(-1)
        want_kept = (torch.arange(F, device="cuda")[None, :] * N + pos[:, None]).reshape(-1)
        want_cached = (torch.arange(F, device="cuda")[:, None] * N + flag[0].nonzero().reshape(-1)[None, :]).reshape(-1)
    want_map = torch.full((F * N,), -1, dtype=torch.int64, device="cuda")
    want_map[want_kept] = torch.arange(want_kept.numel(), device="cuda")
    assert torch.equal(kept.long(), want_kept)
    assert torch.equal(cached.long(), want_cached)
    assert torch.equal(rmap.long(), want_map)
