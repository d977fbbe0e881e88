"""Performance cases of the visual-memory path, through the package's public entry points.

Each case is one thing a user's program does with the library on one GPU, at the sizes of the
workloads in ``paper_2609_34972_amd.configs`` (LLaVA-1.5-7B, LLaVA-NeXT, Qwen2.5-VL video, batched
decode, hybrid linear-attention backbones, the small fp32 workload) or of the same backbones at
other token counts:

  step       build + K/V projection + attention of every layer, the whole path in one pass
  build      build_visual_memory + project_visual_kv of every layer (once per image or video)
  skip       kept_visual_kv: the adapters of the first and last layers are skipped
  recurrent  recurrent_visual_kv: the recurrent adapter and K/V of every layer
  attention  text_visual_attention of `layers` layers over cached K/V, prefill or decode
  delta      delta_rule_write of `layers` linear-attention layers

Weights, caches and output buffers are what a serving program keeps; workspaces are left to the
binding, as in the README. Attention and delta cases walk several layers, each with its own cache
or inputs, since that is how a model meets them: a layer's K/V comes from memory, not from a cache
level that holds one layer.
"""
import math

import torch

import paper_2609_34972_amd as dv

# Backbones: hidden size, layers, query heads, key/value heads, head size.
BACKBONES = {
    "llava7b": dict(d=4096, L=32, Hq=32, Hkv=32, hd=128),
    "qwen25vl": dict(d=3584, L=28, Hq=28, Hkv=4, hd=128),
    "small64": dict(d=2048, L=24, Hq=32, Hkv=8, hd=64),
}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # The smallest whole path (fp32, GELU, 64-wide heads): six short launches, so launch
        # latency and the host's work per call are what a user sees.
        dict(name="tiny_step_f32", family="step", dtype="f32", d=256, L=4, r=16, Hq=4, Hkv=4,
             hd=64, B=1, Nv=64, Nt=16, act=dv.ACT_GELU, eps=1e-5),
        # One 576-token image of an interactive request, with the adapters of the first 5 and the
        # last 10 layers skipped.
        dict(name="image_skip", family="skip", backbone="llava7b", r=256, B=1, Nv=576, first=5,
             last=10),
        # A batch of four images: the benchmark's build.
        dict(name="image_batch_build", family="build", backbone="llava7b", r=256, B=4, Nv=576,
             epilogue=False),
        # Two high-resolution images of five tiles each.
        dict(name="tiles_build", family="build", backbone="llava7b", r=256, B=2, Nv=2880,
             epilogue=False),
        # A 64-frame video on a GQA backbone with projection biases and multimodal rotation.
        dict(name="video_build_rope", family="build", backbone="qwen25vl", r=512, B=1, Nv=16384,
             epilogue=True),
        # The recurrent adapter on the batch of four images.
        dict(name="image_batch_recurrent", family="recurrent", backbone="llava7b", r=256, B=4,
             Nv=576),
        # Prefill of 64 text tokens per image over all layers of the cached visual K/V.
        dict(name="image_prefill", family="attention", backbone="llava7b", layers=32, B=4, Nv=576,
             Nq=64, past=0),
        # Prefill of 128 text tokens over the video.
        dict(name="video_prefill", family="attention", backbone="qwen25vl", layers=28, B=1,
             Nv=16384, Nq=128, past=0),
        # One decode step of a batch of 64 image conversations with 512 earlier text tokens (two
        # layers: each reads 1.1 GB).
        dict(name="image_batch_decode", family="attention", backbone="llava7b", layers=2, B=64,
             Nv=576, Nq=1, past=512),
        # One decode step of four video conversations on the GQA backbone, all layers.
        dict(name="video_decode", family="attention", backbone="qwen25vl", layers=28, B=4,
             Nv=16384, Nq=1, past=200),
        # The visual write of a hybrid backbone, a batch of four images and one long video.
        dict(name="image_delta", family="delta", layers=24, B=4, N=576, Hk=16, Hv=32, dk=128,
             dv=128, dtype="bf16"),
        dict(name="video_delta", family="delta", layers=6, B=1, N=16384, Hk=16, Hv=32, dk=128,
             dv=128, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: 1 to 5760 tokens per call on the wide backbone, up to
    16384 on the GQA one, batches of 1 to 64, odd and ragged sizes among them."""
    family = rng.choice(["step", "build", "build", "skip", "recurrent", "prefill", "prefill",
                         "decode", "decode", "delta", "delta"])
    if family == "step":
        return dict(family="step", dtype="f32", d=64 * rng.randint(2, 12), L=rng.randint(2, 6),
                    r=16 * rng.randint(1, 4), Hq=rng.choice([4, 8]), Hkv=rng.choice([2, 4]),
                    hd=rng.choice([64, 64, 128]), B=rng.randint(1, 2), Nv=_log(rng, 16, 300),
                    Nt=_log(rng, 4, 64), act=rng.choice([dv.ACT_SILU, dv.ACT_GELU]), eps=1e-5)
    if family in ("build", "skip", "recurrent"):
        wide = family != "build" or rng.random() < 0.5
        most = 2304 if family == "recurrent" else (5760 if wide else 16384)
        B = rng.choice([1, 1, 1, 2, 3, 4])
        case = dict(family=family, backbone="llava7b" if wide else "qwen25vl",
                    r=rng.choice([128, 256, 256, 512]), B=B, Nv=_log(rng, 64, most // B))
        if family == "build":
            case["epilogue"] = rng.random() < 0.4
        if family == "skip":
            case["first"], case["last"] = rng.choice([(5, 10), (10, 10), (3, 8)])
        return case
    if family in ("prefill", "decode"):
        backbone = rng.choice(["llava7b", "llava7b", "qwen25vl", "qwen25vl", "small64"])
        b = BACKBONES[backbone]
        B = _log(rng, 1, 64) if family == "decode" else _log(rng, 1, 8)
        Nv = _log(rng, 64, 16384 if b["Hkv"] < 32 else 2880)
        past = _log(rng, 1, 1024) if family == "decode" else 0
        Nq = 1 if family == "decode" else _log(rng, 8, 256)
        # bounds on the bytes of one layer's caches and on the score work of one layer
        row = 2 * b["Hkv"] * b["hd"] * 2
        while B > 1 and (B * (Nv + past + Nq) * row > 1.2e9 or B * b["Hq"] * Nq * Nv > 1.2e8):
            B //= 2
        layers = max(1, min(b["L"], int(1.5e9 // (B * (Nv + past + Nq) * row))))
        return dict(family="attention", backbone=backbone, layers=layers, B=B, Nv=Nv, Nq=Nq,
                    past=past)
    B = rng.choice([1, 1, 2, 4])
    N = _log(rng, 64, 16384 // B)
    dk = rng.choice([128, 128, 128, 64])
    return dict(family="delta", layers=max(1, min(24, 100000 // (B * N))), B=B, N=N, Hk=16,
                Hv=rng.choice([16, 32, 32]), dk=dk, dv=dk, dtype="bf16")


# ------------------------------------------------------------------ inputs


def _sizes(case):
    s = dict(case)
    if "backbone" in case:
        s.update({k: v for k, v in BACKBONES[case["backbone"]].items() if k not in case})
        s.setdefault("dtype", "bf16")
        s.setdefault("act", dv.ACT_SILU)
        s.setdefault("eps", 1e-6 if case["backbone"] == "qwen25vl" else 1e-5)
    return s


class _Draw:
    """Seeded normals on the GPU, rounded to the call's dtype."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.dtype = dtype

    def __call__(self, *shape, std=1.0, shift=0.0, dtype=None):
        out = torch.empty(*shape, dtype=dtype or self.dtype, device="cuda")
        rows = out.view(shape[0], -1)
        for i in range(shape[0]):  # row by row: no fp32 copy of a whole weight stack
            rows[i] = torch.randn(rows.shape[1], generator=self.gen, device="cuda") * std + shift
        return out


def _build_inputs(s, draw):
    L, d, r, kv = s["L"], s["d"], s["r"], s["Hkv"] * s["hd"]
    T = s["B"] * s["Nv"]
    E = torch.randn(T, d, generator=draw.gen, device="cuda").to(draw.dtype)
    if s.get("backbone") == "llava7b":  # a few channels of the projector's output are large
        E[:, 211::512] *= 20.0
    return dict(E=E, Dw=draw(L, r, d, std=d ** -0.5), Uw=draw(L, d, r, std=r ** -0.5),
                gamma=draw(L, d, std=0.1, shift=1.0), Wk=draw(L, kv, d, std=d ** -0.5),
                Wv=draw(L, kv, d, std=d ** -0.5))


def _cache(s, L, dtype):
    shape = (L, s["B"], s["Hkv"], s["Nv"], s["hd"])
    return torch.empty(*shape, dtype=dtype, device="cuda"), torch.empty(*shape, dtype=dtype,
                                                                        device="cuda")


def _keep(s):
    return [s["first"] <= l < s["L"] - s["last"] for l in range(s["L"])]


def _positions(B, Nv):
    """(frame, row, column) ids of a grid of 16 x 16 tokens a frame, after 20 text tokens."""
    i = torch.arange(Nv, dtype=torch.int32)
    p = torch.stack([i // 256, (i // 16) % 16, i % 16], 0) + 20
    return p.unsqueeze(0).expand(B, 3, Nv).contiguous().cuda()


ROPE_SECTIONS = (16, 24, 24)
ROPE_THETA = 1e6


def prepare(case, seed):
    s = _sizes(case)
    draw = _Draw(seed, DTYPES[s["dtype"]])
    st = {"s": s}
    fam = s["family"]
    if fam in ("step", "build", "skip", "recurrent"):
        st.update(_build_inputs(s, draw))
        n = sum(_keep(s)) if fam == "skip" else s["L"]
        st["Kv"], st["Vv"] = _cache(s, n, draw.dtype)
        if fam in ("step", "build"):
            st["Z"] = torch.empty(s["L"], s["B"] * s["Nv"], s["r"], dtype=draw.dtype,
                                  device="cuda")
        if s.get("epilogue"):
            kv = s["Hkv"] * s["hd"]
            st["epilogue"] = dv.KVEpilogue(
                k_bias=draw(s["L"], kv, std=0.05), v_bias=draw(s["L"], kv, std=0.05),
                positions=_positions(s["B"], s["Nv"]), rope_sections=ROPE_SECTIONS,
                rope_theta=ROPE_THETA)
        if fam == "step":
            st["Q"] = draw(s["L"], s["B"], s["Nt"], s["Hq"], s["hd"])
            st["Kt"] = draw(s["L"], s["B"], s["Hkv"], s["Nt"], s["hd"])
            st["Vt"] = draw(s["L"], s["B"], s["Hkv"], s["Nt"], s["hd"])
            st["O"] = torch.empty_like(st["Q"])
    elif fam == "attention":
        n, B, Hkv, hd = s["layers"], s["B"], s["Hkv"], s["hd"]
        nkt = s["past"] + s["Nq"]
        st["Q"] = draw(n, B, s["Nq"], s["Hq"], hd)
        st["Kv"], st["Vv"] = draw(n, B, Hkv, s["Nv"], hd), draw(n, B, Hkv, s["Nv"], hd)
        st["Kt"], st["Vt"] = draw(n, B, Hkv, nkt, hd), draw(n, B, Hkv, nkt, hd)
        st["O"] = torch.empty_like(st["Q"])
    else:
        n, B, Hk, Hv, N, dk, dv_ = (s[k] for k in ("layers", "B", "Hk", "Hv", "N", "dk", "dv"))
        f32 = torch.float32
        k = draw(n, B, Hk, N, dk, dtype=f32)
        st["k"] = (k / k.norm(dim=-1, keepdim=True)).to(draw.dtype)  # the backbone normalises keys
        st["v"] = draw(n, B, Hv, N, dv_)
        z = draw(n, B, Hv, N, dtype=f32)
        st["alpha"] = torch.exp(-0.1 * torch.nn.functional.softplus(z))
        st["beta"] = torch.sigmoid(draw(n, B, Hv, N, dtype=f32))
        st["S"] = draw(n, B, Hv, dk, dv_, std=0.1, dtype=f32)
    return st


# ------------------------------------------------------------------ one pass


def run(st):
    s = st["s"]
    fam = s["family"]
    if fam in ("step", "build"):
        dv.build_visual_memory(st["E"], st["Dw"], st["Z"], act=s["act"])
        dv.project_visual_kv(st["E"], st["Z"], st["Uw"], st["gamma"], st["Wk"], st["Wv"],
                             st["Kv"], st["Vv"], eps=s["eps"], epilogue=st.get("epilogue"))
        if fam == "build":
            return [st["Kv"], st["Vv"]]
        for l in range(s["L"]):
            dv.text_visual_attention(st["Q"][l], st["Kv"][l], st["Vv"][l], st["Kt"][l],
                                     st["Vt"][l], st["O"][l])
        return [st["Kv"], st["Vv"], st["O"]]
    if fam == "skip":
        dv.kept_visual_kv(st["E"], st["Dw"], st["Uw"], st["gamma"], st["Wk"], st["Wv"], _keep(s),
                          st["Kv"], st["Vv"], eps=s["eps"], act=s["act"])
        return [st["Kv"], st["Vv"]]
    if fam == "recurrent":
        dv.recurrent_visual_kv(st["E"], st["Dw"], st["Uw"], st["gamma"], st["Wk"], st["Wv"],
                               st["Kv"], st["Vv"], eps=s["eps"], act=s["act"])
        return [st["Kv"], st["Vv"]]
    if fam == "attention":
        for l in range(s["layers"]):
            dv.text_visual_attention(st["Q"][l], st["Kv"][l], st["Vv"][l], st["Kt"][l],
                                     st["Vt"][l], st["O"][l], q_pos0=s["past"])
        return [st["O"]]
    for l in range(s["layers"]):
        dv.delta_rule_write(st["k"][l], st["v"][l], st["alpha"][l], st["beta"][l], st["S"][l])
    return [st["S"]]


# ------------------------------------------------------------------ work and tolerance


def work(case):
    s = _sizes(case)
    fam = s["family"]
    e = 4 if s["dtype"] == "f32" else 2
    nbytes = flops = 0.0
    if fam in ("step", "build", "skip", "recurrent"):
        T, d, r, kv = s["B"] * s["Nv"], s["d"], s["r"], s["Hkv"] * s["hd"]
        n = sum(_keep(s)) if fam == "skip" else s["L"]
        flops += n * T * (4.0 * d * r + 4.0 * d * kv)
        nbytes += e * (T * d + n * (2.0 * d * r + d + 2.0 * kv * d + 2.0 * T * kv))
    if fam in ("step", "attention"):
        n = s["L"] if fam == "step" else s["layers"]
        Nq, past = (s["Nt"], 0) if fam == "step" else (s["Nq"], s["past"])
        pairs = s["B"] * s["Hq"] * (Nq * (s["Nv"] + past) + Nq * (Nq + 1) / 2)
        flops += n * 4.0 * pairs * s["hd"]
        # in a whole step the visual K/V that the attention reads are the path's own output
        keys = (0 if fam == "step" else s["Nv"]) + past + Nq
        nbytes += n * e * (2.0 * s["B"] * Nq * s["Hq"] * s["hd"]
                           + 2.0 * s["B"] * s["Hkv"] * keys * s["hd"])
    if fam == "delta":
        n, B, Hk, Hv, N, dk, dv_ = (s[k] for k in ("layers", "B", "Hk", "Hv", "N", "dk", "dv"))
        flops = n * 6.0 * B * Hv * N * dk * dv_
        nbytes = n * (e * B * N * (Hk * dk + Hv * dv_) + 8.0 * B * Hv * N
                      + 8.0 * B * Hv * dk * dv_)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the error measured against exact(): 4e-7 in fp32; in bf16 0.0025 to 0.0029
    for the K/V of the embedding adapter, 0.0063 for the recurrent one (it grows over the layers),
    0.0017 to 0.0023 for attention and 0.003 for the delta-rule state."""
    s = _sizes(case)
    if s["dtype"] == "f32":
        return {"rel": 3e-6}
    return {"rel": {"build": 1e-2, "skip": 1e-2, "recurrent": 2.4e-2, "attention": 1e-2,
                    "delta": 1.2e-2}[s["family"]]}


# ------------------------------------------------------------------ 64-bit values


def _kv64(st, l, M):
    """K and V [B, Hkv, Nv, hd] of layer l from its memory M, in float64."""
    s = st["s"]
    B, Nv, Hkv, hd = s["B"], s["Nv"], s["Hkv"], s["hd"]
    X = M * torch.rsqrt(M.square().mean(1, keepdim=True) + s["eps"]) * st["gamma"][l].double()
    k, v = X @ st["Wk"][l].double().t(), X @ st["Wv"][l].double().t()
    epi = st.get("epilogue")
    if epi is not None:
        k, v = k + epi.k_bias[l].double(), v + epi.v_bias[l].double()
    k, v = (x.view(B, Nv, Hkv, hd).transpose(1, 2) for x in (k, v))
    if epi is not None:
        half = hd // 2
        j = torch.arange(half, device="cuda")
        c0, c1 = ROPE_SECTIONS[0], ROPE_SECTIONS[0] + ROPE_SECTIONS[1]
        axis = torch.where(j < c0, 0, torch.where(j < c1, 1, 2))
        pos = epi.positions.double()[:, axis, :].transpose(1, 2)  # [B, Nv, half]
        ang = (pos * ROPE_THETA ** (-j.double() / half)).unsqueeze(1)
        a, b = k[..., :half], k[..., half:]
        k = torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)
    return k, v


def _phi64(x, act):
    return torch.nn.functional.silu(x) if act == dv.ACT_SILU else torch.nn.functional.gelu(x)


def _attention64(q, kv, vv, kt, vt, past):
    """One layer: q [B, Nq, Hq, hd], keys [B, Hkv, *, hd], in float64."""
    B, Nq, Hq, hd = q.shape
    G = Hq // kt.shape[1]
    out = torch.empty(B, Nq, Hq, hd, dtype=torch.float64, device="cuda")
    Nv = kv.shape[2]
    n = Nv + past + Nq
    ok = torch.arange(n, device="cuda")[None, :] <= Nv + past + torch.arange(Nq, device="cuda")[:, None]
    for b in range(B):
        for g in range(kt.shape[1]):
            K = torch.cat([kv[b, g], kt[b, g, :past + Nq]], 0).double()
            V = torch.cat([vv[b, g], vt[b, g, :past + Nq]], 0).double()
            x = q[b, :, g * G:(g + 1) * G].double().transpose(0, 1).reshape(G * Nq, hd)
            p = (x @ K.t() * hd ** -0.5).view(G, Nq, n).masked_fill(~ok, -math.inf).softmax(-1)
            out[b, :, g * G:(g + 1) * G] = (p.view(G * Nq, n) @ V).view(G, Nq, hd).transpose(0, 1)
    return out


def exact(case, seed):
    st = prepare(case, seed)
    s = st["s"]
    fam = s["family"]
    f64 = torch.float64
    if fam in ("step", "build", "skip", "recurrent"):
        E = st["E"].double()
        keep = _keep(s) if fam == "skip" else [True] * s["L"]
        Kv, Vv = (torch.empty(st["Kv"].shape, dtype=f64, device="cuda") for _ in range(2))
        M, c = E, 0
        for l in range(s["L"]):
            if not keep[l]:
                continue
            X = M if fam == "recurrent" else E
            M = X + _phi64(X @ st["Dw"][l].double().t(), s["act"]) @ st["Uw"][l].double().t()
            Kv[c], Vv[c] = _kv64(st, l, M)
            c += 1
        if fam != "step":
            return [Kv, Vv]
        O = torch.stack([_attention64(st["Q"][l], Kv[l], Vv[l], st["Kt"][l], st["Vt"][l], 0)
                         for l in range(s["L"])], 0)
        return [Kv, Vv, O]
    if fam == "attention":
        return [torch.stack([_attention64(st["Q"][l], st["Kv"][l], st["Vv"][l], st["Kt"][l],
                                          st["Vt"][l], s["past"]) for l in range(s["layers"])], 0)]
    # The recurrence token by token, all layers, sequences and heads at once.
    G = s["Hv"] // s["Hk"]
    S = st["S"].double()
    for t in range(s["N"]):
        k = st["k"][..., t, :].double().repeat_interleave(G, 2)
        S *= st["alpha"][..., t].double()[..., None, None]
        u = st["v"][..., t, :].double() - (k.unsqueeze(-2) @ S).squeeze(-2)
        S += (st["beta"][..., t].double()[..., None] * k).unsqueeze(-1) * u.unsqueeze(-2)
    return [S]
