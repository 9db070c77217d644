"""Calls past 32-bit limits that the library accepts (GPU, against 64-bit
torch): batches of 2^31 elements and more at the attention entry point."""
import math

import pytest
import torch

import paper_2607_23844_amd as oc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
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


@pytest.mark.parametrize("heads,dh,C,n_seq,L,dtype,tol", [
    # short sequences, a batch of 2^31 + 2.9e6 elements (bf16 outputs and fp16
    # intermediates: 1.7e-3 of the 2-norm, see perf/cases.py)
    (1, 64, 4096, 21000, 25, "bf16", 8e-3),
])
def test_attention_batch(heads, dh, C, n_seq, L, dtype, tol):
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
