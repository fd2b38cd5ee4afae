"""Timed cases of the decode step: the MoE layer and the decode attention, through their
public entry points.

A case is one call of a serving engine's inner loop: one MoE decode step
(``MoEDecode.forward``, or ``moe_decode_forward_noalloc`` for callers without a handle)
or one step of decode attention over the paged KV cache (``AttnDecode.forward``).
``listed`` holds the sizes of this repository's layer and attention configurations, from
the smallest layer to the largest batch the interface takes; ``draw`` gives other batch
sizes, layer shapes, formats, layouts and context mixes of the same ranges.  Inputs follow
the distributions of ``workload.py`` and ``attn_workload.py``, drawn and quantised on the
GPU.
"""
import math

import numpy as np
import torch

from paper_2609_11133_amd import binding as B
from paper_2609_11133_amd.attn_workload import NAN_BF16, context_lengths

DEV = "cuda"
PAGE, HEAD_DIM = 16, 128
WFMT = {"fp8": B.MOE_WFMT_FP8_E4M3_B128, "mxfp4": B.MOE_WFMT_MXFP4_E2M1_B32, "nvfp4": B.MOE_WFMT_NVFP4_E2M1_B16}
E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


# ------------------------------------------------------------------ the cases


def moe(T, shape, fmt, packed=True, act="bf16", bias="", noalloc=False):
    H, E, k, I = shape
    return dict(op="moe", T=T, H=H, E=E, k=k, I=I, fmt=fmt, packed=packed, act=act, bias=bias, noalloc=noalloc)


def attn(batch, heads, mix, capacity, lengths=0):
    return dict(op="attn", batch=batch, Hq=heads[0], Hkv=heads[1], mix=mix, capacity=capacity, lengths=lengths)


# (hidden, experts, top-k, intermediate size) of configs.py
TINY, L235, L480, L480TP4 = (256, 8, 2, 128), (4096, 128, 8, 1536), (6144, 160, 8, 2560), (6144, 160, 8, 640)
# (query heads, key/value heads) of attn_workload.py
A235, A480TP4 = (64, 4), (24, 2)


def listed():
    return [
        # the smallest layer, fp32 activations, called without a handle: launches and latency
        dict(name="tiny-f32-T4", **moe(4, TINY, "fp8", packed=False, act="f32", noalloc=True)),
        # one sequence in flight: latency of a single-user decode step
        dict(name="fp8-235b-T1", **moe(1, L235, "fp8")),
        # the 235B decode lane's concurrency (24) on weights in their default, row-major layout
        dict(name="fp8-235b-rowmajor-T24", **moe(24, L235, "fp8", packed=False)),
        # the headline step of bench.py
        dict(name="fp8-480b-T64", **moe(64, L480, "fp8", bias="normal:0.5")),
        # one GPU's share of the 480B decode lane (TP4) at its concurrency
        dict(name="fp8-480b-tp4-T48", **moe(48, L480TP4, "fp8", bias="normal:0.5")),
        # a batch near the interface's limit of 1024 tokens, not a multiple of any tile
        dict(name="fp8-480b-T1000", **moe(1000, L480, "fp8", bias="normal:0.5")),
        # the 235B decode lane in NVFP4 at its concurrency
        dict(name="nvfp4-235b-T24", **moe(24, L235, "nvfp4")),
        # large batches with a few hot experts, in both 4-bit formats
        dict(name="nvfp4-235b-zipf-T256", **moe(256, L235, "nvfp4", bias="zipf:1.1")),
        dict(name="mxfp4-235b-zipf-T256", **moe(256, L235, "mxfp4", bias="zipf:1.1")),
        # attention of the 235B lane, chat contexts, block tables for 4K tokens
        dict(name="attn-235b-standard", **attn(24, A235, "standard", 4096)),
        # attention of the 480B lane's TP4 share, agent contexts, block tables for 32K tokens
        dict(name="attn-480b-tp4-agentic", **attn(48, A480TP4, "agentic", 32768)),
        # attention over long contexts
        dict(name="attn-235b-long32k", **attn(24, A235, "long:32768", 32768)),
    ]


def _spread(rng, lo, hi):
    """An integer of lo..hi, uniform over the logarithm."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    if rng.random() < 0.25:
        Hkv = rng.choice([1, 2, 4, 8])
        G = rng.choice([1, 4, 8, 12, 16])
        mix = rng.choice(["standard", "agentic", "long"])
        batch = _spread(rng, 1, 96)
        cap = rng.choice([4096, 32768])
        if mix == "long":
            # at most the tokens of the listed long case's cache (24 x 32768 x 4 heads)
            most = min(cap, 24 * 32768 * 4 // (batch * Hkv))
            mix = "long:%d" % _spread(rng, 512, max(512, most))
        return attn(batch, (G * Hkv, Hkv), mix, cap, lengths=rng.randrange(1, 1 << 20))
    fmt = rng.choice(["fp8", "fp8", "nvfp4", "nvfp4", "mxfp4"])
    act = "f32" if fmt != "nvfp4" and rng.random() < 0.15 else "bf16"
    shapes = [L235, L235, (2048, 64, 6, 1024), (256 * rng.randint(4, 16), rng.randint(16, 160), rng.randint(1, 8), 256 * rng.randint(1, 8))]
    if act == "bf16":
        shapes.append((6144, 160, 8, 2560))
    if fmt == "fp8":
        shapes.append((128 * rng.randint(4, 32), rng.randint(16, 128), rng.randint(1, 8), 128 * rng.randint(1, 16)))
        if act == "bf16":
            shapes.append(L480TP4)
    return moe(_spread(rng, 1, 1000), rng.choice(shapes), fmt, packed=rng.random() < 0.75, act=act,
               bias=rng.choice(["", "normal:0.5", "zipf:1.1"]))


# ------------------------------------------------------------------ inputs of the MoE layer


def _quantise_fp8(w):
    """[n, R, K] fp32 -> E4M3 codes [n, R*K] and fp32 scales of 128x128 blocks."""
    n, R, K = w.shape
    b = w.view(n, R // 128, 128, K // 128, 128)
    s = b.abs().amax(dim=(2, 4)) / 448.0
    s = torch.where(s > 0, s, torch.ones_like(s))
    q = (b / s[:, :, None, :, None]).to(torch.float8_e4m3fn)
    return q.view(torch.uint8).reshape(n, R * K), s.reshape(n, -1)


def _e2m1_codes(v):
    """fp32 -> E2M1 codes, two per byte, the even index in the low nibble."""
    mids = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], device=v.device)
    c = torch.bucketize(v.abs(), mids, out_int32=True).to(torch.uint8) | ((v < 0).to(torch.uint8) << 3)
    c = c.view(*c.shape[:-1], -1, 2)
    return c[..., 0] | (c[..., 1] << 4)


def _quantise_mxfp4(w):
    n, R, K = w.shape
    b = w.view(n, R, K // 32, 32)
    e = torch.frexp(b.abs().amax(dim=3))[1] - 3  # floor(log2 amax) - 2
    q = _e2m1_codes((b * torch.exp2(-e.float())[..., None]).view(n, R, K))
    return q.reshape(n, -1), (e + 127).to(torch.uint8).reshape(n, -1)


def _quantise_nvfp4(w):
    n, R, K = w.shape
    ts = w.abs().amax(dim=(1, 2)) / (6.0 * 448.0)
    b = w.view(n, R, K // 16, 16) / ts[:, None, None, None]
    s = (b.abs().amax(dim=3) / 6.0).clamp(2.0 ** -6).to(torch.float8_e4m3fn)
    q = _e2m1_codes((b / s.float()[..., None]).view(n, R, K))
    return q.reshape(n, -1), s.view(torch.uint8).reshape(n, -1), ts


def _experts(case, gen):
    """Row-major expert weights [E, bytes] and scales [E, ...], as moe_decode.h lays them out."""
    H, E, I, fmt = case["H"], case["E"], case["I"], case["fmt"]
    per = 3 * H * I if fmt == "fp8" else 3 * H * I // 2
    w = torch.empty(E, per, dtype=torch.uint8, device=DEV)
    sc = []
    step = max(1, (1 << 28) // (3 * H * I))
    for e in range(0, E, step):
        n = min(step, E - e)
        gu = torch.randn(n, 2 * I, H, generator=gen, device=DEV) * (H ** -0.5)
        dn = torch.randn(n, H, I, generator=gen, device=DEV) * (I ** -0.5)
        if fmt == "nvfp4":
            parts = [_quantise_nvfp4(m) for m in (gu[:, :I], gu[:, I:], dn)]
            head = torch.stack([p[2] for p in parts] + [torch.zeros_like(parts[0][2])], dim=1)
            sc.append(torch.cat([head.view(torch.uint8)] + [p[1] for p in parts], dim=1))
        else:
            parts = [(_quantise_fp8 if fmt == "fp8" else _quantise_mxfp4)(m) for m in (gu, dn)]
            sc.append(torch.cat([p[1] for p in parts], dim=1))
        w[e:e + n] = torch.cat([p[0] for p in parts], dim=1)
    return w, torch.cat(sc)


def _moe_inputs(case, seed):
    gen = torch.Generator(DEV).manual_seed(int(seed))
    dt = torch.bfloat16 if case["act"] == "bf16" else torch.float32
    T, H, E = case["T"], case["H"], case["E"]
    x = torch.randn(T, H, generator=gen, device=DEV).to(dt)
    rw = (torch.randn(E, H, generator=gen, device=DEV) * (H ** -0.5)).to(dt)
    bias = None
    if case["bias"]:
        kind, val = case["bias"].split(":")
        if kind == "normal":
            bias = torch.randn(E, generator=gen, device=DEV) * float(val)
        else:  # Zipf popularity: -s ln(rank), ranks in a random order
            bias = (-float(val) * torch.log(torch.randperm(E, generator=gen, device=DEV) + 1.0)).float()
    w, sc = _experts(case, gen)
    return x, rw, bias, w, sc


def _prepare_moe(case, seed):
    x, rw, bias, w, sc = _moe_inputs(case, seed)
    T, k = case["T"], case["k"]
    f32 = case["act"] == "f32"
    capacity = next(c for c in (64, 256, 1024) if c >= T)  # the batch the engine's handle is sized for
    dtype = B.MOE_DTYPE_F32 if f32 else B.MOE_DTYPE_BF16
    cfg = B.make_config(case["H"], case["E"], case["I"], k, capacity, act_dtype=dtype, router_dtype=dtype,
                        wfmt=WFMT[case["fmt"]],
                        weight_layout=B.MOE_WLAYOUT_TILED16 if case["packed"] else B.MOE_WLAYOUT_ROW_MAJOR)
    if case["packed"]:
        stream = torch.cuda.current_stream().cuda_stream
        pw, ps = torch.empty_like(w), (None if case["fmt"] == "fp8" else torch.empty_like(sc))
        B.moe_decode_pack_weights(cfg, stream, w, pw, case["E"], None if ps is None else sc, ps)
        w, sc = pw, (sc if ps is None else ps)
    return dict(cfg=cfg, layer=None if case["noalloc"] else B.MoEDecode(cfg, device=DEV), T=T, k=k, x=x, rw=rw,
                bias=bias, w=w, sc=sc, y=torch.empty_like(x),
                ids=torch.empty(T, k, dtype=torch.int32, device=DEV), wts=torch.empty(T, k, device=DEV))


# ------------------------------------------------------------------ inputs of the attention


def _lengths(case):
    return context_lengths(case["mix"], case["batch"], draw=case["lengths"])


def _attn_inputs(case, seed):
    gen = torch.Generator(DEV).manual_seed(int(seed))
    L = _lengths(case)
    pages = (L + PAGE - 1) // PAGE
    used = int(pages.sum())
    n_pages = used + used // 10 + 1
    perm = torch.randperm(n_pages, generator=gen, device=DEV).int()
    table = torch.zeros(case["batch"], case["capacity"] // PAGE, dtype=torch.int32, device=DEV)
    o = 0
    for b, n in enumerate(pages.tolist()):
        table[b, :n] = perm[o:o + n]
        o += n
    q = torch.randn(case["batch"], case["Hq"], HEAD_DIM, generator=gen, device=DEV).bfloat16()
    kc = torch.randn(n_pages, case["Hkv"], PAGE, HEAD_DIM, generator=gen, device=DEV, dtype=torch.bfloat16)
    vc = torch.randn(n_pages, case["Hkv"], HEAD_DIM, PAGE, generator=gen, device=DEV, dtype=torch.bfloat16)
    for c in (kc, vc):  # pages no sequence owns hold anything
        c.view(torch.int16)[perm[used:].long()] = NAN_BF16
    return q, kc, vc, table, torch.from_numpy(L).to(DEV)


def _prepare_attn(case, seed):
    q, kc, vc, table, ctx = _attn_inputs(case, seed)
    cfg = B.make_attn_config(case["Hq"], case["Hkv"], case["batch"], case["capacity"] // PAGE)
    return dict(attn=B.AttnDecode(cfg, device=DEV), q=q, kc=kc, vc=vc, table=table, ctx=ctx, batch=case["batch"],
                out=torch.empty_like(q))


# ------------------------------------------------------------------ one pass


def prepare(case, seed):
    return (_prepare_moe if case["op"] == "moe" else _prepare_attn)(case, seed)


def run(s):
    if "attn" in s:
        s["attn"].forward(s["q"], s["kc"], s["vc"], s["kc"].shape[0], s["table"], s["ctx"], s["batch"],
                          HEAD_DIM ** -0.5, s["out"])
        return s["out"]
    if s["layer"] is None:
        stream = torch.cuda.current_stream().cuda_stream
        B.moe_decode_forward_noalloc(s["cfg"], stream, s["x"], s["T"], s["rw"], s["bias"], s["w"], s["sc"], s["k"],
                                     s["y"], s["ids"], s["wts"])
    else:
        s["layer"].forward(s["x"], s["T"], s["rw"], s["bias"], s["w"], s["sc"], s["k"], s["y"], s["ids"], s["wts"])
    return s["y"], s["ids"], s["wts"]


# ------------------------------------------------------------------ what a pass cannot do without


def _active_experts(case):
    """Experts with at least one token, simulated: a logit is N(0, 1) plus the bias."""
    r = np.random.default_rng(7)
    T, E, k = case["T"], case["E"], case["k"]
    got = []
    for _ in range(4):
        bias = np.zeros(E)
        if case["bias"].startswith("normal"):
            bias = r.standard_normal(E) * float(case["bias"].split(":")[1])
        elif case["bias"]:
            bias = -float(case["bias"].split(":")[1]) * np.log(1.0 + r.permutation(E))
        got.append(len(np.unique(np.argpartition(-(r.standard_normal((T, E)) + bias), k - 1, axis=1)[:, :k])))
    return sum(got) / len(got)


def work(case):
    if case["op"] == "attn":
        tokens = int(_lengths(case).astype(np.int64).sum())
        qo = 2 * case["batch"] * case["Hq"] * HEAD_DIM * 2
        return {"bytes": tokens * case["Hkv"] * HEAD_DIM * 2 * 2 + tokens // PAGE * 4 + qo,
                "flops": 4 * tokens * case["Hq"] * HEAD_DIM}
    T, H, E, k, I, fmt = (case[n] for n in ("T", "H", "E", "k", "I", "fmt"))
    expert = {"fp8": 3 * H * I * (1 + 4 / 16384), "mxfp4": 3 * H * I * (0.5 + 1 / 32),
              "nvfp4": 3 * H * I * (0.5 + 1 / 16) + 16}[fmt]
    a = 2 if case["act"] == "bf16" else 4
    return {"bytes": _active_experts(case) * expert + E * H * a + 2 * T * H * a + T * k * 8,
            "flops": 6 * T * k * H * I + 2 * T * E * H}


# ------------------------------------------------------------------ what the results may be off by


def tolerance(case):
    # bf16 outputs, bf16 probabilities (attention) and bf16-exact activations (8-bit
    # mantissas after the two-term split, MoE): two orders and paths differ by some 2e-3.
    # Expert ids are whole numbers and never differ.
    return {"rel": 1e-2, "max": 0.1}


# ------------------------------------------------------------------ the same in 64 bits


def _dequant(case, w, sc):
    """One expert's row-major codes and scales -> gate/up [2I, H] and down [H, I] in fp64."""
    H, I, fmt = case["H"], case["I"], case["fmt"]
    if fmt == "fp8":
        v = w.view(torch.float8_e4m3fn).double()
        out, o, so = [], 0, 0
        for R, K in ((2 * I, H), (H, I)):
            s = sc[so:so + R * K // 16384].double().view(R // 128, 1, K // 128, 1)
            out.append((v[o:o + R * K].view(R // 128, 128, K // 128, 128) * s).view(R, K))
            o, so = o + R * K, so + R * K // 16384
        return out
    table = torch.tensor(E2M1 + tuple(-v for v in E2M1), dtype=torch.float64, device=w.device)
    v = table[torch.stack([w & 15, w >> 4], dim=1).view(-1).long()]
    if fmt == "mxfp4":
        s, blk = torch.exp2(sc.double() - 127.0), 32
    else:
        s, blk = sc[16:].view(torch.float8_e4m3fn).double(), 16
        s *= torch.repeat_interleave(sc[:12].view(torch.float32).double(), H * I // 16)
    v = (v.view(-1, blk) * s[:, None]).view(-1)
    return v[:2 * H * I].view(2 * I, H), v[2 * H * I:].view(H, I)


def _exact_moe(case, seed):
    x, rw, bias, w, sc = _moe_inputs(case, seed)
    T, k, I = case["T"], case["k"], case["I"]
    xd = x.double()
    logits = xd @ rw.double().T
    if bias is not None:
        logits += bias.double()
    top, ids = torch.sort(logits.float(), dim=1, descending=True, stable=True)  # ties: the lower index
    ids, wts = ids[:, :k], torch.softmax(top[:, :k].double(), dim=1)
    y = torch.zeros_like(xd)
    for e in torch.unique(ids).tolist():
        t, j = torch.nonzero(ids == e, as_tuple=True)
        gu, dn = _dequant(case, w[e], sc[e])
        h = xd[t] @ gu.T
        g = h[:, :I]
        y.index_add_(0, t, wts[t, j][:, None] * ((g / (1.0 + torch.exp(-g)) * h[:, I:]) @ dn.T))
    return y, ids.int(), wts


def _exact_attn(case, seed):
    q, kc, vc, table, ctx = _attn_inputs(case, seed)
    Hq, Hkv = case["Hq"], case["Hkv"]
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for b, n in enumerate(ctx.tolist()):
        pages = table[b, :(n + PAGE - 1) // PAGE].long()
        for g in range(Hkv):
            K = kc[pages, g].reshape(-1, HEAD_DIM)[:n].double()
            V = vc[pages, g].transpose(1, 2).reshape(-1, HEAD_DIM)[:n].double()
            heads = slice(g * Hq // Hkv, (g + 1) * Hq // Hkv)
            out[b, heads] = torch.softmax(q[b, heads].double() @ K.T * HEAD_DIM ** -0.5, dim=1) @ V
    return out


def exact(case, seed):
    return (_exact_moe if case["op"] == "moe" else _exact_attn)(case, seed)
