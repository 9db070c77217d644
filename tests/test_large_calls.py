"""Calls past 32-bit limits that the library accepts (GPU, against 64-bit
torch): batches of 2^31 elements and more at the attention entry point, and
launches of more than 2^32 threads (a grid's limit along one dimension)."""
import math

import pytest
import torch

import paper_2607_23844_amd as oc



def test_projections_fit_a_grid(native):
    """Half a billion rows of few columns: no tile shape is picked whose grid
    HIP would cut short."""
    r = native("launch_size")()
    assert r.returncode == 0, r.stdout


@pytest.fixture
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.empty_cache()


def _attn64(x, w, heads):
    """Attention of one sequence [L, C], projected by wo, in 64 bits."""
    q, k, v = (x.double() @ w[n].double().t() for n in ("wq", "wk", "wv"))
    d = q.shape[1] // heads
    o = torch.empty_like(q)
    for h in range(heads):
        s = slice(h * d, h * d + d)
        o[:, s] = torch.softmax(q[:, s] @ k[:, s].t() / math.sqrt(d), dim=1) @ v[:, s]
    return o @ w["wo"].double().t()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,dh,C,n_seq,L,dtype,tol", [
    # short sequences, a batch of 2^31 + 2.9e6 elements (bf16 outputs and fp16
    # intermediates: 1.7e-3 of the 2-norm, see perf/cases.py)
    (1, 64, 4096, 21000, 25, "bf16", 8e-3),
    # fp32 attention, 8.4 M blocks of 512 threads
    (64, 8, 8, 14600, 129, "f32", 1e-5),
])
def test_attention_batch(gpu, heads, dh, C, n_seq, L, dtype, tol):
    print(f"large batch heads={heads} dh={dh} C={C} {n_seq}x{L} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.empty(n_seq, L, C, dtype=dt, device="cuda").normal_(generator=g)
    hd = heads * dh
    w = {n: (torch.randn(hd, C, generator=g, device="cuda") / C ** 0.5).to(dt) for n in ("wq", "wk", "wv")}
    w["wo"] = (torch.randn(C, hd, generator=g, device="cuda") / hd ** 0.5).to(dt)
    y, _ = oc.attn_reduced(x, n_seq, L, w, oc.Shape(1, 4, 4, C, heads, dh, 0, dtype))
    y = y.view(n_seq, L, C)
    for s in (0, n_seq // 2, n_seq - 7, n_seq - 1):
        ref = _attn64(x[s], w, heads)
        err = float((y[s].double() - ref).norm() / ref.norm())
        assert err < tol, (s, err)


@pytest.mark.gpu
def test_f32_similarity_over_many_frames(gpu):
    # 192 x 64 tiles of 1400 frames, 17.2 M blocks of 256 threads
    F, H, W, C = 1400, 128, 128, 8
    print("f32 similarity, 1400 frames of 128 x 128", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(F, H * W, C, generator=g, device="cuda")
    sh, cf = oc.Shape(F, H, W, C, 1, 8, 0, "f32"), oc.Cfg("token", r=0.5)
    node_max, node_idx = oc.match(x, sh, cf, oc.workspace(sh, cf, x.device))
    ids = torch.arange(H * W, device="cuda").view(H, W)
    reps = ids[::2, ::2].reshape(-1)
    cand = ids.reshape(-1)
    cand = cand[~torch.isin(cand, reps)]
    node_max, node_idx = node_max.view(F, -1), node_idx.view(F, -1).long()
    for f in (0, 700, F - 1):
        u = x[f].double()
        u = u / u.norm(dim=1, keepdim=True)
        best = (u[cand] @ u[reps].t()).max(dim=1).values
        at = node_idx[f] - f * H * W
        assert bool(torch.isin(at, reps).all())
        # fp32 sums of 8 products and two norms: a few ulps of 1
        assert float((node_max[f].double() - best).abs().max()) < 2e-6
        assert float((best - (u[cand] * u[at]).sum(dim=1)).abs().max()) < 4e-6
