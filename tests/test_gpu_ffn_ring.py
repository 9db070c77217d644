"""The feed-forward sublayer on the ring-buffered tiles (GPU, against 64-bit
torch; OmniCache §4.2): large tiles with ragged rows and widths, one K step,
and row indices outside the tensor, whose rows are neither computed from
foreign memory nor stored.

H is rounded to fp16 and y to bf16: half an ulp of each, 2^-12 and 2^-9 of a
value, so 4e-3 of the outputs' 2-norm bounds a correct result."""
import pytest
import torch

import paper_2607_23844_amd as oc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,hidden,rows", [
    (4096, 1536, 6144, 2048),    # 256 x 256 up, 96 x 128 down
    (4096, 1536, 3072, 2500),    # ragged rows
    (2304, 640, 2560, 1153),
    (1024, 64, 128, 77),         # one K step up, two down
    (64, 128, 64, 64),
    (6000, 640, 1536, 6000),     # 256 x 192 up
    (4000, 64, 3072, 4000),      # 128 x 192 up
    (6000, 64, 1536, 6000),      # 160 x 128 up
    (6000, 1536, 512, 6000),     # 256 x 192 down
    (6000, 1536, 64, 6000),      # 160 x 128 down
    (6000, 2048, 64, 6000),      # 128 x 192 down
])
def test_ffn_ring(N, C, hidden, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"ffn N={N} C={C} hidden={hidden} rows={rows}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(C + rows)

    def randn(*s):
        return torch.randn(*s, generator=g, device="cuda")

    x = randn(1, N, C).bfloat16()
    w = dict(w1=(randn(hidden, C) / C ** 0.5).bfloat16(), w2=(randn(C, hidden) / hidden ** 0.5).bfloat16())
    idx = torch.randperm(N, generator=g, device="cuda")[:rows].to(torch.int32)
    bad = torch.tensor([0, rows // 2], device="cuda")
    idx[bad] = torch.tensor([-1, N], dtype=torch.int32, device="cuda")
    y = torch.full((1, N, C), 7.0, dtype=torch.bfloat16, device="cuda")
    sh = oc.Shape(1, 2, N // 2, C, C // 64, 64, 0, "bf16")
    oc.ffn_reduced(x, w, sh, kept_idx=idx, y=y)
    ok = torch.ones(rows, dtype=torch.bool, device="cuda")
    ok[bad] = False
    at = idx[ok].long()
    h = torch.nn.functional.gelu(x[0, at].double() @ w["w1"].double().t(), approximate="tanh")
    ref = h @ w["w2"].double().t()
    assert float((y[0, at].double() - ref).norm() / ref.norm()) < 4e-3
    rest = torch.ones(N, dtype=torch.bool, device="cuda")
    rest[at] = False
    assert bool((y[0, rest] == 7.0).all())
