"""The V projection's transposed rows where tiles cross sequences (GPU,
against the CPU oracle, OmniCache §3.2.3): sequence starts at every residue of
4 and of 16, K tails, the wide tiles, and the key padding."""
import numpy as np
import pytest
import torch

from oc_synth import bf16_bits, small_workload
from oracle import oc_oracle as O
import paper_2607_23844_amd as oc

from parity import check_output_bars, dev_tensor, rel_err, to_f64, weights_dev, weights_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,heads,C,n_seq,L", [
    (64, 2, 128, 5, 131),     # starts 0, 131, 262, ...: quads across sequences
    (72, 1, 72, 3, 66),       # K not a multiple of 64, starts 2 mod 4
    (32, 3, 64, 7, 100),      # starts 0 mod 4, not mod 16
    (64, 1, 64, 2, 272),      # starts 0 mod 16
    (64, 18, 64, 23, 133),    # 128 x 192 tiles (one round of them)
    (48, 2, 40, 9, 97),
    (48, 4, 192, 100, 65),    # padding that the attention masks and nobody zeroes
    (64, 6, 128, 20, 263),    # padding that the attention reads, staged by DMA
])
def test_vt_across_sequences(dh, heads, C, n_seq, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"Vt across sequences dh={dh} heads={heads} C={C} {n_seq}x{L}", flush=True)
    wl = small_workload("token", F=1, H=4, W=4, C=C, heads=heads, head_dim=dh, dtype="bf16", seed=51)
    rng = np.random.default_rng(L * 100 + dh)
    sh = oc.Shape(1, 4, 4, C, heads, dh, 0, "bf16")
    xk = bf16_bits(rng.standard_normal((n_seq, L, C)).astype(np.float32))
    ws = torch.full((oc.attn_workspace_bytes(sh, n_seq, L),), 0x7f, dtype=torch.uint8, device="cuda:0")
    y, _ = oc.attn_reduced(dev_tensor(wl, xk), n_seq, L, weights_dev(wl), sh, ws=ws)
    torch.cuda.synchronize()
    y64, _ = O.attn_reduced(wl.f64(xk), None, weights_f64(wl), heads, dh)
    e = rel_err(to_f64(y), y64, "bf16")
    print(f"  err {e:.3g}", flush=True)
    check_output_bars(e, 0.0, "bf16")
