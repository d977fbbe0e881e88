"""Infinite V entries (a cache whose projection overflowed): an output that gives such a key a positive
probability is that infinity, in every kernel that multiplies by more than the probability itself or pads a
key tile. GQA decode (probabilities in two bf16 parts, the second of either sign or zero) and the fp32
kernel for few rows (16-key tiles whose tail repeats the last key): keys at the edges of their tiles, the
last visual key and the last key of all, with and without a key split. All other outputs are finite and
meet the parity bar."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34972_amd as dvl
from tests.gpu_helpers import TOL, cuda, f64, say

pytestmark = pytest.mark.gpu

# dtype, B, Hq, Hkv, hd, Nv, q_pos0 (one query): the last two of each dtype split their keys given room
CASES = [("bf16", 1, 4, 2, 128, 40, 5), ("bf16", 2, 14, 2, 128, 0, 33), ("bf16", 1, 8, 1, 128, 1000, 70),
         ("bf16", 2, 28, 4, 128, 4099, 9),
         ("f32", 1, 9, 1, 64, 17, 5), ("f32", 2, 18, 2, 128, 0, 20), ("f32", 1, 16, 1, 64, 1000, 3),
         ("f32", 1, 10, 1, 128, 2003, 9)]


@pytest.mark.parametrize("split", [True, False], ids=["ws", "nows"])
@pytest.mark.parametrize("spec", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_infinite_values(spec, split):
    dt, B, Hq, Hkv, hd, Nv, q0 = spec
    say(f"[infinite values {spec} split={split}]")
    g = torch.Generator().manual_seed(29)
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    mk = lambda *s: torch.randn(*s, generator=g).to(tdt)
    Nkt = q0 + 1
    x = dict(Q=mk(B, 1, Hq, hd), Kv=mk(B, Hkv, Nv, hd), Vv=mk(B, Hkv, Nv, hd), Kt=mk(B, Hkv, Nkt, hd),
             Vt=mk(B, Hkv, Nkt, hd))
    inf = {}  # channel -> value; one key each
    keys = [("Vt", 0), ("Vt", q0)] + ([("Vv", 0), ("Vv", min(31, Nv - 1)), ("Vv", Nv // 2), ("Vv", Nv - 1)] if Nv else [])
    ref_in = {k: v.clone() for k, v in x.items()}
    for i, (name, key) in enumerate(keys):
        c = 7 + 9 * i
        inf[c] = float("-inf") if i % 2 else float("inf")
        x[name][:, :, key, c] = inf[c]
    xg = {k: cuda(v) for k, v in x.items()}
    n = dvl.text_visual_attention_workspace(B, Hq, Hkv, hd, Nv, 1, Nkt) if split else 0
    ws = torch.full((max(n, 16),), 0xFF, dtype=torch.uint8, device="cuda:0")
    O = torch.full_like(xg["Q"], float("nan"))
    dvl.text_visual_attention(xg["Q"], xg["Kv"], xg["Vv"], xg["Kt"], xg["Vt"], O, q_pos0=q0, ws=ws)
    torch.cuda.synchronize()
    out = f64(O)
    for c, v in inf.items():
        assert np.all(out[..., c] == v), f"channel {c}: {out[..., c].ravel()[:4]} instead of {v}"
    rest = [c for c in range(hd) if c not in inf]
    ref = oracle.text_visual_attention(*(f64(ref_in[k]) for k in ("Q", "Kv", "Vv", "Kt", "Vt")), q0)[..., rest]
    err = float(np.max(np.abs(out[..., rest] - ref)) / np.max(np.abs(ref)))
    assert np.isfinite(err) and err <= TOL[dt]
