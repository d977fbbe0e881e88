"""GPU parity of the bf16 build at the edges of its launch rules: token counts around one and two row
tiles of every kernel (waves whose rows all lie past the end compute nothing), few enough tiles for the
four-stage down projection and, in the last case, just too many, with a short last run of layers in the up
projection's blocks. Parity bar of the build tests (2e-2) against the fp64 oracle.

The recurrent adapter runs on at most the first 16 layers of a case: each layer rounds its operand and Z
to bf16 (rms 2^-9 / sqrt 3 of the value each) and the errors of all layers add up in the state, over l
layers to about sqrt(2 l) 2^-9 / sqrt 3 rms, 0.0064 at 16 layers and 0.013 at 70; the largest of 1e4
elements lies about four times the rms above it, over the bar at 70 layers and well inside it at 16
relative to the largest value (itself about four times the rms).
"""
import pytest
import torch

import oracle
import paper_2609_34972_amd as dvl
from paper_2609_34972_amd import configs, synth
from tests.gpu_helpers import DOWN_128, DOWN_DEEP, assert_close, cuda, down_tiles, f64, say, up_layers_per_block

pytestmark = pytest.mark.gpu

# T, d, L, r, Hkv, hd
CASES = [(1, 64, 1, 64, 1, 64), (63, 128, 3, 64, 2, 128), (64, 192, 2, 128, 2, 64), (65, 256, 5, 64, 3, 128),
         (129, 320, 17, 128, 2, 128), (193, 256, 9, 256, 4, 64), (257, 256, 11, 64, 4, 128),
         (320, 128, 70, 128, 1, 128), (577, 512, 7, 256, 2, 128),
         (385, 256, 65, 128, 1, 64)]


@pytest.mark.parametrize("spec", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_build_edges(spec):
    T, d, L, r, Hkv, hd = spec
    say(f"[build edges {spec}]")
    many = spec == CASES[-1]  # 260 tiles of 128 x 128; runs of two layers, the last of one
    assert down_tiles(T, L * r) == (DOWN_128 if many else DOWN_DEEP)
    assert up_layers_per_block(T, d, L) == (2 if many else 1) and (not many or L % 2 == 1)
    w = configs.Workload("edge", "bf16", d=d, L=L, r=r, Hq=Hkv, Hkv=Hkv, hd=hd, Nv=T, Nt=1, B=1)
    E, wts = synth.make_E(w, seed=3), synth.make_build_weights(w, seed=3)
    Eg, g = cuda(E), {k: cuda(v) for k, v in wts.items()}
    Z = torch.full((L, T, r), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    Kv = torch.full((L, 1, Hkv, T, hd), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    Vv = torch.full_like(Kv, float("nan"))
    dvl.build_visual_memory(Eg, g["Dw"], Z)
    dvl.project_visual_kv(Eg, Z, g["Uw"], g["gamma"], g["Wk"], g["Wv"], Kv, Vv, eps=1e-5)
    n = min(L, 16)
    Kr, Vr = torch.full_like(Kv[:n], float("nan")), torch.full_like(Kv[:n], float("nan"))
    dvl.recurrent_visual_kv(Eg, *(g[k][:n].contiguous() for k in ("Dw", "Uw", "gamma", "Wk", "Wv")), Kr, Vr, eps=1e-5)
    torch.cuda.synchronize()
    a = {k: f64(v) for k, v in wts.items()}
    Mr = oracle.memory_recurrent(f64(E), a["Dw"][:n], a["Uw"][:n], 0)
    Zr = oracle.down(f64(E), a["Dw"], 0)
    Me = oracle.memory(f64(E), Zr, a["Uw"])
    for l in sorted({0, n // 2, n - 1, L - 1}):
        assert_close(f64(Z[l]), Zr[l], "bf16", f"Z[{l}]")
        one = lambda M: None if l >= len(M) else oracle.visual_kv(M[l:l + 1], a["gamma"][l:l + 1], a["Wk"][l:l + 1],
                                         a["Wv"][l:l + 1], 1, T, Hkv, hd, 1e-5)
        for name, got, ref in [("K", (Kv, Vv), one(Me))] + [("recurrent K", (Kr, Vr), one(Mr))] * (l < n):
            assert_close(f64(got[0][l]), ref[0][0], "bf16", f"{name}[{l}]")
            assert_close(f64(got[1][l]), ref[1][0], "bf16", f"{name} values[{l}]")
