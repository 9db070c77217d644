"""Token similarity on the ring-buffered tiles (GPU, OmniCache §3.2.3, §3.3):
a case per tile shape, with one or several representative tiles per block, K
of a single 16-byte chunk and not a multiple of 64, ragged groups; and frame
pairs, whose groups hold more candidate tiles than the others, against the
CPU oracle.

The dot products are sums of exact products in fp32 (K <= 320 terms, an error
of 320 * 2^-24 of the norms' product at most), hence 2e-5 on a cosine."""
import pytest
import torch

from oc_synth import small_workload
import paper_2607_23844_amd as oc

from parity import dev_tensor, layer_step_parity, shapes, weights_dev, weights_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("F,H,W,C,k", [
    (16, 72, 72, 128, 1),    # 256 x 256 tiles, six per block
    (4, 76, 78, 136, 1),     # 256 x 256, two per block
    (5, 78, 72, 8, 1),       # 128 x 128, one K chunk, several tiles per block
    (5, 96, 64, 72, 1),      # 256 x 192, three per block
    (3, 74, 88, 72, 1),      # 256 x 128, ragged last tile
    (5, 82, 78, 8, 1),       # 128 x 192
    (1, 66, 72, 8, 1),       # 96 x 128
    (2, 76, 70, 16, 1),      # 128 x 128
    (3, 70, 82, 16, 1),      # 160 x 128
    (9, 64, 64, 64, 1),      # one step per tile
    (1, 76, 94, 16, 1),      # 64 x 64, several tiles per block
    (1, 4, 24, 8, 2),        # groups of 18 candidates and 6 representatives
    (11, 88, 88, 8, 2),      # 128 x 64
])
def test_token_match(F, H, W, C, k):
    print(f"match F={F} {H}x{W} C={C} k={k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(F * 1000 + C)
    x = torch.randn(F, H * W, C, generator=g, device="cuda").bfloat16()
    x[0, 3] = 0                                     # a zero-norm candidate
    x[F - 1, 0] = 0                                 # and a zero-norm representative
    sh, cf = oc.Shape(F, H, W, C, 1, 16, 0, "bf16"), oc.Cfg("token", r=0.5, patch_k=k)
    node_max, node_idx = oc.match(x, sh, cf, oc.workspace(sh, cf, x.device))
    pl = oc.plan(sh, cf)
    node_max, node_idx = node_max.view(F, k * k, pl.n_src_max), node_idx.view(F, k * k, pl.n_src_max).long()
    xd = x.double()
    u = xd / xd.norm(dim=2, keepdim=True).clamp_min(1e-300)
    ids = torch.arange(H * W, device="cuda").view(H, W)
    for f in range(F):
        for p in range(k * k):
            y0, x0 = (p // k) * (H // k), (p % k) * (W // k)
            tile = ids[y0:y0 + H // k, x0:x0 + W // k]
            reps = tile[::2, ::2].reshape(-1)
            cand = tile.reshape(-1)
            cand = cand[~torch.isin(cand, reps)]
            best = (u[f, cand] @ u[f, reps].t()).max(dim=1).values
            at = node_idx[f, p] - f * H * W
            assert bool(torch.isin(at, reps).all())
            mine = (u[f, cand] * u[f, at]).sum(dim=1)
            assert float((node_max[f, p].double() - best).abs().max()) < 2e-5
            assert float((best - mine).abs().max()) < 4e-5


@pytest.mark.parametrize("F,H,W,C,k,r_frame", [
    (9, 56, 48, 32, 1, 0.34),     # pairs of 4704 candidates beside frames of 2016
    (10, 20, 28, 48, 2, 0.5),     # patches, every odd frame paired
    (7, 16, 16, 32, 1, 0.0),      # no pairs
])
def test_frame_pairs(F, H, W, C, k, r_frame):
    print(f"pairs F={F} {H}x{W} C={C} k={k} r_frame={r_frame}", flush=True)
    wl = small_workload("frame_token", F=F, H=H, W=W, C=C, heads=C // 16, head_dim=16, dtype="bf16", r=0.4,
                        r_frame=r_frame, patch_k=k, n_steps=2, seed=77, planted=True)
    sh, cf, osh, ocf = shapes(wl)
    dev = torch.device("cuda:0")
    ws, cache = oc.workspace(sh, cf, dev), oc.LayerCache(sh, dev)
    ora, valid = None, False
    for s in range(2):
        res, st = layer_step_parity(wl, wl.steps[s], sh, cf, osh, ocf, cache, ws, ora, valid, None, None,
                                    weights_dev(wl), weights_f64(wl), case=f"pairs {F} {k}")
        print(f"  step {s}: {st}", flush=True)
        ora, valid = res.y, True


@pytest.mark.parametrize("F,H,W,C,k", [
    (4, 16, 24, 64, 1),      # one K step per segment
    (3, 32, 40, 128, 1),     # two, several representative tiles
    (5, 24, 16, 192, 2),     # three, patches
    (7, 64, 56, 64, 4),      # enough tiles that K is not split
    (2, 72, 96, 128, 1),     # 96 x 128 tiles, three per block, two segments of two steps
])
def test_blocks(F, H, W, C, k):
    print(f"blocks F={F} {H}x{W} C={C} k={k}", flush=True)
    wl = small_workload("block", F=F, H=H, W=W, C=C, heads=C // 64, head_dim=64, dtype="bf16", r=0.5, patch_k=k,
                        n_steps=2, seed=78)
    sh, cf, osh, ocf = shapes(wl)
    dev = torch.device("cuda:0")
    ws, cache = oc.workspace(sh, cf, dev), oc.LayerCache(sh, dev)
    ora, valid = None, False
    for s in range(2):
        res, st = layer_step_parity(wl, wl.steps[s], sh, cf, osh, ocf, cache, ws, ora, valid, None, None,
                                    weights_dev(wl), weights_f64(wl), case=f"blocks {F} {k}")
        print(f"  step {s}: {st}", flush=True)
        ora, valid = res.y, True


@pytest.mark.parametrize("F,H,W,C,k", [
    (2, 16, 24, 64, 1),      # one ragged tile of representatives
    (2, 40, 36, 72, 1),      # several tiles, the last one ragged
    (1, 32, 32, 64, 4),      # patches of 16 representatives
    (16, 72, 72, 128, 1),    # 256 x 256 tiles, six per block
])
def test_infinite_and_nan_candidates(F, H, W, C, k):
    """A candidate whose every product is -inf is matched to the first
    representative of its group (equal values: the smallest id), one whose
    products are NaN to none, and neither touches its neighbours."""
    print(f"match, infinite candidates F={F} {H}x{W} C={C} k={k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(F * 1000 + C)
    x = torch.randn(F, H, W, C, generator=g, device="cuda")
    x[:, ::2, ::2, 0] = -x[:, ::2, ::2, 0].abs() - 0.5      # every representative: a negative first channel
    sh, cf = oc.Shape(F, H, W, C, 1, 16, 0, "bf16"), oc.Cfg("token", r=0.5, patch_k=k)
    pl = oc.plan(sh, cf)
    ws = oc.workspace(sh, cf, x.device)
    clean = oc.match(x.bfloat16().view(F, H * W, C), sh, cf, ws)
    y = x.clone()
    y[F - 1, H - 1, W - 1, 0] = float("inf")                # the last candidate of the last group
    y[0, 0, 1, 0] = float("inf")                            # the first of the first
    y[0, 0, 3, 1] = float("nan")
    nm, ni = oc.match(y.bfloat16().view(F, H * W, C), sh, cf, ws)
    ni, was = ni.view(-1, pl.n_src_max), clean[1].view(-1, pl.n_src_max)
    ph, pw = H // k, W // k
    assert int(ni[0, 0]) == 0
    assert int(ni[-1, -1]) == (F - 1) * H * W + (k - 1) * ph * W + (k - 1) * pw
    assert int(ni[0, 1]) == -1
    changed = (ni != was).nonzero().tolist()
    assert all(c in ([0, 0], [0, 1], [ni.shape[0] - 1, pl.n_src_max - 1]) for c in changed), changed[:8]
