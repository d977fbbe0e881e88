"""GPU parity of the fp32 kernels for small calls: the build in 16 x 16 tiles (token counts around a tile,
reductions of less than one and of several batches of loads, several layers in a tile row) and attention in blocks of
16 rows whose waves share out 16-key tiles (fewer tiles than waves, ragged and masked tiles, no visual keys,
a chunk of a longer prompt, key splits). At or below the launch rule's line and just above it, where the
64 x 64-tile kernels run, and, for the build, both sides compared to the bit. Parity bar for fp32 (1e-4) against
the fp64 oracle; fp32 sums of a few hundred terms lie near 1e-6.
"""
import ctypes

import pytest
import torch

import oracle
import paper_2609_34972_amd as dvl
from paper_2609_34972_amd import configs, synth
from tests.gpu_helpers import assert_close, cuda, f64, launch_rule, say

pytestmark = pytest.mark.gpu

# T, d, L, r, Hkv, hd, act
BUILD = [(1, 64, 1, 16, 1, 64, 0), (15, 64, 3, 16, 2, 128, 1), (17, 128, 2, 48, 1, 64, 0), (64, 256, 4, 16, 4, 64, 1),
         (100, 704, 2, 80, 2, 128, 0), (130, 320, 5, 32, 1, 64, 1), (385, 192, 16, 64, 1, 64, 0)]


@pytest.mark.parametrize("spec", BUILD, ids=["x".join(map(str, c)) for c in BUILD])
def test_small_build(spec):
    T, d, L, r, Hkv, hd, act = spec
    say(f"[small fp32 build {spec}]")
    w = configs.Workload("small", "f32", d=d, L=L, r=r, Hq=Hkv, Hkv=Hkv, hd=hd, Nv=T, Nt=1, B=1, act=act)
    E, wts = synth.make_E(w, seed=5), synth.make_build_weights(w, seed=5)
    Eg, g = cuda(E), {k: cuda(v) for k, v in wts.items()}
    nan = lambda *s: torch.full(s, float("nan"), device="cuda:0")
    Z, Kv, Vv = nan(L, T, r), nan(L, 1, Hkv, T, hd), nan(L, 1, Hkv, T, hd)
    dvl.build_visual_memory(Eg, g["Dw"], Z, act=act)
    dvl.project_visual_kv(Eg, Z, g["Uw"], g["gamma"], g["Wk"], g["Wv"], Kv, Vv, eps=1e-5)
    torch.cuda.synchronize()
    a = {k: f64(v) for k, v in wts.items()}
    Zr = oracle.down(f64(E), a["Dw"], act)
    Kr, Vr = oracle.visual_kv(oracle.memory(f64(E), Zr, a["Uw"]), a["gamma"], a["Wk"], a["Wv"], 1, T, Hkv, hd, 1e-5)
    for name, got, ref in (("Z", Z, Zr), ("K", Kv, Kr), ("V", Vv, Vr)):
        say(f"  {name}: {assert_close(f64(got), ref, 'f32', name):.1e}")


def small(tiles, up=False):
    return launch_rule("_ZN2dv9small_f32Elb", ctypes.c_bool, (ctypes.c_int64, tiles), (ctypes.c_bool, up))


# T, d, L, r, Hkv, hd: the all-layer launches lie above the rule's line (which of down, up, K/V: the last
# entry), those of one layer, or of a few tokens, at or below it. 20 sums of squares a row, short and odd
# ranks, a last row tile of 4 to 44 tokens.
SIDES = [(300, 704, 6, 64, 2, 128, "uk"), (300, 192, 24, 64, 1, 64, "duk"), (100, 1280, 8, 80, 2, 128, "uk"),
         (68, 576, 14, 144, 2, 64, "uk"), (129, 320, 14, 48, 1, 128, "uk")]


@pytest.mark.parametrize("spec", SIDES, ids=["x".join(map(str, c)) for c in SIDES])
def test_same_bits_on_both_sides_of_the_rule(spec):
    """A layer's Z, K and V have the same bits whichever kernels its launch takes: the all-layer call, a
    workspace of one layer, a layer range, kept layers, one layer's weights alone, and the first tokens alone."""
    T, d, L, r, Hkv, hd, big = spec
    say(f"[fp32 bits {spec}]")
    c = lambda a, b: -(-a // b)
    rows, kvw = c(T, 64), 2 * Hkv * hd
    tiles = {"d": (c(L * r, 64) * rows, c(r, 64) * rows), "u": (d // 64 * rows * L, d // 64 * rows),
             "k": (kvw // 64 * rows * L, kvw // 64 * rows)}
    for k, (every, one) in tiles.items():
        assert small(one, k == "u") and (k not in big or not small(every, k == "u")), (k, every, one)
    w = configs.Workload("sides", "f32", d=d, L=L, r=r, Hq=Hkv, Hkv=Hkv, hd=hd, Nv=T, Nt=1, B=1, act=T % 2)
    Eg, g = cuda(synth.make_E(w, seed=5)), {k: cuda(v) for k, v in synth.make_build_weights(w, seed=5).items()}
    proj = [g[k] for k in ("Uw", "gamma", "Wk", "Wv")]
    nan = lambda *s: torch.full(s, float("nan"), device="cuda:0")
    need = lambda n: torch.empty(dvl.project_visual_kv_workspace(T, d, n, torch.float32), dtype=torch.uint8, device="cuda:0")

    def run(E, Dw, weights, n, **kw):
        Z, Kv, Vv = nan(n, len(E), r), nan(n, 1, Hkv, len(E), hd), nan(n, 1, Hkv, len(E), hd)
        dvl.build_visual_memory(E, Dw, Z, act=w.act)
        dvl.project_visual_kv(E, Z, *weights, Kv, Vv, eps=1e-5, **kw)
        torch.cuda.synchronize()
        return Z, Kv, Vv

    Z, Kv, Vv = run(Eg, g["Dw"], proj, L)
    assert all(torch.isfinite(x).all() for x in (Z, Kv, Vv))
    for name, x, y in zip(("Z", "K", "V"), (Z, Kv, Vv), run(Eg, g["Dw"], proj, L, ws=need(1))):
        assert torch.equal(x, y), f"one-layer workspace: {name}"
    Kr, Vr = torch.zeros_like(Kv), torch.zeros_like(Vv)
    dvl.project_visual_kv(Eg, Z, *proj, Kr, Vr, eps=1e-5, l0=2, nl=1, ws=need(1))
    torch.cuda.synchronize()
    assert torch.equal(Kr[2], Kv[2]) and torch.equal(Vr[2], Vv[2]), "layer range"
    keep = [l in (0, 3, 4) for l in range(L)]
    Kk, Vk = nan(3, 1, Hkv, T, hd), nan(3, 1, Hkv, T, hd)
    dvl.kept_visual_kv(Eg, g["Dw"], *proj, keep, Kk, Vk, eps=1e-5, act=w.act)
    torch.cuda.synchronize()
    assert torch.equal(Kk, Kv[[0, 3, 4]]) and torch.equal(Vk, Vv[[0, 3, 4]]), "kept layers"
    for name, x, y in zip(("Z", "K", "V"), (Z, Kv, Vv), run(Eg, g["Dw"][1:2], [x[1:2] for x in proj], 1)):
        assert torch.equal(x[1:2], y), f"one layer's weights: {name}"
    for name, x, y in zip(("Z", "K", "V"), (Z, Kv, Vv), run(Eg[:20], g["Dw"], proj, L)):
        assert torch.equal(x[..., :20, :], y), f"first tokens: {name}"


# B, Hq, Hkv, hd, Nv, Nq, q_pos0
ATTN = [(1, 1, 1, 64, 0, 1, 0), (1, 2, 2, 64, 3, 2, 0), (2, 4, 4, 64, 64, 16, 0), (1, 9, 1, 128, 17, 1, 5),
        (1, 6, 2, 64, 31, 5, 0), (1, 4, 2, 128, 100, 32, 9), (2, 2, 1, 64, 300, 17, 0), (1, 4, 1, 64, 1000, 16, 0),
        (1, 2, 2, 128, 2000, 64, 0), (1, 2, 1, 64, 33, 33, 2)]


@pytest.mark.parametrize("split", [True, False], ids=["ws", "nows"])
@pytest.mark.parametrize("spec", ATTN, ids=["x".join(map(str, c)) for c in ATTN])
def test_small_attention(spec, split):
    B, Hq, Hkv, hd, Nv, Nq, q0 = spec
    Nkt = q0 + Nq + 2  # two free cache slots that must not be read
    say(f"[small fp32 attention {spec} split={split}]")
    gen = torch.Generator().manual_seed(17)
    mk = lambda *s: torch.randn(*s, generator=gen)
    x = dict(Q=mk(B, Nq, Hq, hd), Kv=mk(B, Hkv, Nv, hd), Vv=mk(B, Hkv, Nv, hd), Kt=mk(B, Hkv, Nkt, hd),
             Vt=mk(B, Hkv, Nkt, hd))
    x["Kt"][:, :, q0 + Nq:] = float("nan")
    x["Vt"][:, :, q0 + Nq:] = float("nan")
    xg = {k: cuda(v) for k, v in x.items()}
    n = dvl.text_visual_attention_workspace(B, Hq, Hkv, hd, Nv, Nq, Nkt) if split else 0
    ws = torch.full((max(n, 16),), 0xFF, dtype=torch.uint8, device="cuda:0")
    O = torch.full_like(xg["Q"], float("nan"))
    dvl.text_visual_attention(xg["Q"], xg["Kv"], xg["Vv"], xg["Kt"], xg["Vt"], O, q_pos0=q0, ws=ws)
    torch.cuda.synchronize()
    ref = oracle.text_visual_attention(f64(x["Q"]), f64(x["Kv"]), f64(x["Vv"]), f64(x["Kt"]), f64(x["Vt"]), q0)
    say(f"  {assert_close(f64(O), ref, 'f32', 'O'):.1e}")
