"""GPU parity of GQA decode (bf16, hd 128, 2 to 8 query heads per kv-head), which runs on MFMAs with
the probabilities in two bf16 parts.

Bound per element: half an ulp of the bf16 output (2^-8 of the value), plus, times the largest
|v|, 2^-17 for what two bf16 parts leave of a probability and 128 * 2^-24 * |s| for the fp32 scores
(|s| < 8 here), rounded up to 1e-4. Probabilities rounded once to bf16 would miss it on the cases
with few keys (up to 2^-9 |v|).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34972_amd as dvl
from tests.gpu_helpers import cuda, f64, say

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Nv, q_pos0: single keys, edges of the 32-key tiles, ragged ends, every group size, no
# visual keys, and key counts that split over blocks (with the workspace) or run in one
CASES = [(1, 2, 1, 0, 0), (1, 4, 2, 1, 0), (2, 6, 2, 2, 1), (1, 8, 2, 31, 30), (3, 10, 2, 32, 31),
         (1, 12, 2, 33, 32), (2, 28, 4, 127, 5), (1, 16, 2, 257, 64), (4, 28, 4, 1000, 77),
         (1, 28, 4, 4099, 200), (65, 28, 4, 40, 9)]


@pytest.mark.parametrize("split", [True, False], ids=["ws", "nows"])
@pytest.mark.parametrize("spec", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_decode_gqa(spec, split):
    B, Hq, Hkv, Nv, q0 = spec
    hd, Nkt = 128, q0 + 3  # two free cache slots that must not be read
    say(f"[gqa decode {spec} split={split}]")
    g = torch.Generator().manual_seed(41)
    mk = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16)
    x = dict(Q=mk(B, 1, Hq, hd), Kv=mk(B, Hkv, Nv, hd), Vv=mk(B, Hkv, Nv, hd),
             Kt=mk(B, Hkv, Nkt, hd), Vt=mk(B, Hkv, Nkt, hd))
    x["Kt"][:, :, q0 + 1:] = float("nan")
    x["Vt"][:, :, q0 + 1:] = float("nan")
    xg = {k: cuda(v) for k, v in x.items()}
    n = dvl.text_visual_attention_workspace(B, Hq, Hkv, hd, Nv, 1, Nkt) if split else 0
    ws = torch.full((max(n, 16),), 0xFF, dtype=torch.uint8, device="cuda:0")
    O = torch.full_like(xg["Q"], float("nan"))
    dvl.text_visual_attention(xg["Q"], xg["Kv"], xg["Vv"], xg["Kt"], xg["Vt"], O, q_pos0=q0, ws=ws)
    torch.cuda.synchronize()
    ref = oracle.text_visual_attention(f64(x["Q"]), f64(x["Kv"]), f64(x["Vv"]), f64(x["Kt"]),
                                       f64(x["Vt"]), q0)
    vmax = max(float(np.abs(f64(x["Vt"])[:, :, :q0 + 1]).max()), float(np.abs(f64(x["Vv"])).max()) if Nv else 0.0)
    err = np.abs(f64(O) - ref)
    assert np.all(np.isfinite(f64(O)))
    worst = float(np.max(err - 2.0 ** -8 * np.abs(ref)) / vmax)
    say(f"  beyond half an ulp, over the largest |v|: {worst:.1e}")
    assert worst <= 1e-4
