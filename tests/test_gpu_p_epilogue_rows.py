"""The projection's K/V epilogue where its walk over the rows of a 256-row tile changes sequence often or
part-way: sequences of 1 to 5 and of 85 tokens (tiles that hold many sequences, and one that ends inside a
sequence), head sizes 64 and 128, K/V widths that fill part of a 256-column tile, with and without each
step. Against the fp64 oracle with the bf16 bar of the other epilogue tests."""
import pytest
import torch

from paper_2609_34972_amd import configs, synth
from tests.gpu_helpers import assert_close, f64, say
from tests.test_gpu_e_epilogue import make_epi, oracle_kv, run

pytestmark = pytest.mark.gpu

FEATS = [(), ("rope",), ("bias", "norm"), ("bias", "norm", "rope")]


@pytest.mark.parametrize("feats", FEATS, ids=lambda f: "+".join(f) or "none")
@pytest.mark.parametrize("hd,Hkv", [(128, 1), (128, 3), (64, 3)])
@pytest.mark.parametrize("B,Nv", [(300, 1), (130, 2), (87, 3), (53, 5), (7, 85)])
def test_epilogue_rows(B, Nv, hd, Hkv, feats):
    say(f"[epilogue rows B {B} Nv {Nv} hd {hd} Hkv {Hkv} {feats}]")
    w = configs.QWEN25VL_VIDEO.with_(name="rows", d=256, L=2, r=64, Hq=Hkv, Hkv=Hkv, hd=hd, B=B, Nv=Nv,
                                     outlier_channels=())
    E, wts, ew = synth.make_E(w, 6), synth.make_build_weights(w, 6), synth.make_epilogue_weights(w)
    pos = torch.arange(B * 3 * Nv, dtype=torch.int32).view(B, 3, Nv) * 7 % 113
    sections = (hd // 8, hd // 8, hd // 4)
    Kv, Vv = run(w, E, wts, make_epi(w, feats, ew, pos, sections, 1e4))
    Kr, Vr = oracle_kv(w, E, wts, feats, ew, pos, sections, 1e4)
    for l in range(w.L):
        assert_close(f64(Kv[l]), Kr[l], w.dtype, f"Kv layer {l}")
        assert_close(f64(Vv[l]), Vr[l], w.dtype, f"Vv layer {l}")
