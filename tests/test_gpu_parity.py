"""Parity of the HIP decode layer (through the C ABI) with the fp64 oracle.

Routing must match bit-exactly (canonical logits and expert ids, ties to the lower
index); routing weights within 1e-6; outputs within max|err| <= 2e-2 * max|ref|.
Every token is compared, at full size too (the oracle computes tokens independently,
on 16 host threads); the 12-layer stack on sampled tokens of every layer."""
import os
import sys

import numpy as np
import pytest

import oracle
from paper_2609_11133_amd import configs as C
from paper_2609_11133_amd import workload as W
from paper_2609_11133_amd.configs import LayerConfig

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THREADS = min(16, os.cpu_count() or 1)
TOL = 2e-2


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_11133_amd import binding as B

    B.lib()  # fails loudly if the library is missing
    return torch.device("cuda:0")


class Run:
    def __init__(self, cfg, hl, dev, max_tokens, mfma_min_tokens=0, screen_min_tokens=0, weight_layout=0):
        from paper_2609_11133_amd import binding as B

        self.cfg, self.hl, self.dev = cfg, hl, dev
        bc = W.binding_config(cfg, max_tokens, mfma_min_tokens, screen_min_tokens, weight_layout)
        self.m = B.MoEDecode(bc, device=dev)
        self.rw = W.to_device(hl.router_w, dev)
        self.bias = W.to_device(hl.bias, dev)
        self.ew = W.to_device(hl.expert_w, dev)
        self.sc = W.to_device(hl.scales, dev)
        if weight_layout == 1:  # the library's own conversion of the row-major weights (and E2M1 scales)
            packed = torch.empty_like(self.ew)
            nv = cfg.wfmt != "fp8"
            psc = torch.empty_like(self.sc) if nv else None
            B.moe_decode_pack_weights(bc, torch.cuda.current_stream(dev).cuda_stream, self.ew, packed, cfg.n_experts,
                                      self.sc if nv else None, psc)
            torch.cuda.synchronize(dev)
            self.ew = packed
            if nv:
                self.sc = psc

    def forward(self, x, topk=None):
        k = topk or self.cfg.topk
        T = x.shape[0]
        xd = W.to_device(x, self.dev)
        y = W.empty_y(self.cfg, T, self.dev)
        ids = torch.full((T, k), -1, dtype=torch.int32, device=self.dev)
        wts = torch.zeros((T, k), dtype=torch.float32, device=self.dev)
        self.m.forward(xd, T, self.rw, self.bias, self.ew, self.sc, k, y, ids, wts)
        torch.cuda.synchronize(self.dev)
        return ids.cpu().numpy(), wts.cpu().numpy(), W.y_to_f64(y)

    def route(self, x, topk=None):
        k = topk or self.cfg.topk
        T = x.shape[0]
        xd = W.to_device(x, self.dev)
        lg = torch.empty((T, self.cfg.n_experts), dtype=torch.float32, device=self.dev)
        ids = torch.empty((T, k), dtype=torch.int32, device=self.dev)
        wts = torch.empty((T, k), dtype=torch.float32, device=self.dev)
        self.m.route(xd, T, self.rw, self.bias, k, lg, ids, wts)
        torch.cuda.synchronize(self.dev)
        return lg.cpu().numpy(), ids.cpu().numpy(), wts.cpu().numpy()


def check_layer(run, x, tokens=None, topk=None, label=""):
    cfg, hl = run.cfg, run.hl
    k = topk or cfg.topk
    say(f"[parity] {label} T={x.shape[0]} k={k} tokens={'all' if tokens is None else list(tokens)}")
    ids, wts, y = run.forward(x, topk=k)
    lo, io, wo, yo = oracle.forward(x, hl.router_w, hl.bias, hl.expert_w, hl.scales, k, cfg.inter, cfg.wfmt_id,
                                    tokens=tokens, threads=THREADS)
    sel = slice(None) if tokens is None else np.asarray(tokens)
    assert np.array_equal(ids[sel], io), f"{label}: expert selection differs"
    assert np.abs(wts[sel] - wo).max() <= 1e-6, f"{label}: routing weights differ"
    ref = yo
    err = np.abs(y[sel] - ref).max()
    scale = np.abs(ref).max()
    say(f"[parity] {label}: max|err|/max|ref| = {err / scale if scale else err:.3e}")
    if scale == 0:
        assert err == 0
    else:
        assert err <= TOL * scale, f"{label}: max|err| {err} > {TOL} * {scale}"
    return ids, wts, y


def check_routing(run, x, topk=None, label=""):
    cfg, hl = run.cfg, run.hl
    k = topk or cfg.topk
    say(f"[routing] {label} T={x.shape[0]} k={k}")
    lg, ids, wts = run.route(x, topk=k)
    for t in range(x.shape[0]):
        l_o, i_o, w_o, _ = oracle.route_token(x[t], hl.router_w, hl.bias, k)
        assert np.array_equal(lg[t].view(np.uint32), l_o.view(np.uint32)), f"{label}: logits of token {t} differ"
        assert np.array_equal(ids[t], i_o), f"{label}: selection of token {t} differs"
        assert np.abs(wts[t] - w_o).max() <= 1e-6
    return lg, ids, wts


# ---------------------------------------------------------------- small layers, every token

SMALL_FP8 = LayerConfig("small-fp8", 512, 16, 4, 256, "bf16", "bf16", "fp8", "normal:0.5", [])
SMALL_MX = LayerConfig("small-mxfp4", 512, 16, 4, 512, "bf16", "bf16", "mxfp4", "zipf:1.1", [])
SMALL_F32_MX = LayerConfig("small-f32-mxfp4", 256, 8, 2, 256, "f32", "f32", "mxfp4", None, [])
SMALL_NV = LayerConfig("small-nvfp4", 512, 16, 4, 256, "bf16", "bf16", "nvfp4", "normal:0.5", [])


@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
@pytest.mark.parametrize("T", [1, 5, 13, 32])
def test_small_fp8_layer(dev, T, screen):
    """Both routing paths: every logit exact, or screened (bf16 matrix-core brackets,
    exact logits only for the experts whose bracket can reach the top k)."""
    hl = W.host_layer(SMALL_FP8, seed=501)
    run = Run(SMALL_FP8, hl, dev, max_tokens=32, screen_min_tokens=screen)
    check_layer(run, W.host_x(SMALL_FP8, T, seed=501), label=f"small-fp8 T={T} screen={screen}")
    st, _ = run.m.stats()
    assert st.route_screened == (screen > 0)
    assert (st.n_exact_logits < T * SMALL_FP8.n_experts) if screen > 0 else (st.n_exact_logits == T * 16)


@pytest.mark.parametrize("T", [3, 13])
def test_small_mxfp4_layer(dev, T):
    hl = W.host_layer(SMALL_MX, seed=502)
    run = Run(SMALL_MX, hl, dev, max_tokens=16)
    check_layer(run, W.host_x(SMALL_MX, T, seed=502), label=f"small-mxfp4 T={T}")


@pytest.mark.parametrize("T", [1, 5, 13, 32])
def test_small_nvfp4_layer(dev, T):
    hl = W.host_layer(SMALL_NV, seed=541)
    run = Run(SMALL_NV, hl, dev, max_tokens=32, screen_min_tokens=13)
    check_layer(run, W.host_x(SMALL_NV, T, seed=541), label=f"small-nvfp4 T={T}")


# NVFP4 staged segments hold two 256-input blocks and the K loop takes four blocks
# per pass, then a tail of 0-3 blocks.  These (H, I) pairs give the gate/up and down
# projections every block count from 1 to 7; Zipf skew puts more than 16 tokens on
# some expert at T=32 (32-token tiles).
NV_SEG_SHAPES = [(1024, 768), (1280, 512), (1536, 1792), (256, 256)]


@pytest.mark.parametrize("shape", NV_SEG_SHAPES)
@pytest.mark.parametrize("T", [1, 7, 32])
def test_nvfp4_segments(dev, shape, T):
    H, I = shape
    cfg = LayerConfig(f"nvfp4-seg-{H}x{I}", H, 16, 4, I, "bf16", "bf16", "nvfp4", "zipf:1.1", [])
    hl = W.host_layer(cfg, seed=542)
    run = Run(cfg, hl, dev, max_tokens=32)
    check_layer(run, W.host_x(cfg, T, seed=542 + T), label=f"nvfp4-seg {H}x{I} T={T}")
    if T == 32:
        assert max(run.m.stats()[1]) > 16


def test_tiny_config(dev):
    cfg = C.TINY
    hl = W.host_layer(cfg)
    run = Run(cfg, hl, dev, max_tokens=4)
    check_layer(run, W.host_x(cfg, 4), label="tiny")
    check_routing(run, W.host_x(cfg, 4), label="tiny")


def test_fp32_mxfp4_layer(dev):
    hl = W.host_layer(SMALL_F32_MX, seed=503)
    run = Run(SMALL_F32_MX, hl, dev, max_tokens=8)
    check_layer(run, W.host_x(SMALL_F32_MX, 6, seed=503), label="f32-mxfp4")


def test_small_routing_bitwise(dev):
    hl = W.host_layer(SMALL_FP8, seed=504)
    run = Run(SMALL_FP8, hl, dev, max_tokens=32)
    check_routing(run, W.host_x(SMALL_FP8, 32, seed=504), label="small-fp8")


@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
@pytest.mark.parametrize("k", [1, 16])
def test_topk_extremes(dev, k, screen):
    cfg = LayerConfig("k-extreme", 512, 16, 16, 256, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=505)
    run = Run(cfg, hl, dev, max_tokens=8, screen_min_tokens=screen)
    check_layer(run, W.host_x(cfg, 5, seed=505), topk=k, label=f"k={k}")


@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
def test_single_expert_dense(dev, screen):
    """E = 1, k = 1: every token routes to expert 0 with weight 1 and the layer is one
    dense SwiGLU block (the degenerate case of the method)."""
    cfg = LayerConfig("one-expert", 512, 1, 1, 512, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=511)
    run = Run(cfg, hl, dev, max_tokens=40, screen_min_tokens=screen)
    ids, wts, _ = check_layer(run, W.host_x(cfg, 37, seed=511), label="E=1")
    assert np.all(ids == 0) and np.all(wts == 1.0)


@pytest.mark.parametrize("cfg,k", [
    (LayerConfig("wide-1024", 256, 1024, 64, 256, "bf16", "bf16", "fp8", "normal:0.5", []), 64),
    (LayerConfig("wide-600", 512, 600, 24, 512, "bf16", "bf16", "mxfp4", "zipf:1.1", []), 24),
], ids=["E1024-k64", "E600-k24"])
@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
def test_many_experts(dev, cfg, k, screen):
    """The largest expert counts and top-k the library accepts (16 keys per lane in
    the wave top-k, the widest grouping bitmasks)."""
    hl = W.host_layer(cfg, seed=512)
    run = Run(cfg, hl, dev, max_tokens=48, screen_min_tokens=screen)
    check_layer(run, W.host_x(cfg, 33, seed=512), topk=k, label=f"{cfg.name} k={k} screen={screen}")
    assert run.m.stats()[0].route_screened == (screen > 0)
    check_routing(run, W.host_x(cfg, 9, seed=513), topk=k, label=f"{cfg.name} k={k}")


def test_zero_input_and_ties(dev):
    """x = 0, no bias: every logit is +0, the selection is experts 0..k-1 with equal
    weights, and y = 0.  Duplicate router rows tie; the lower index wins."""
    hl = W.host_layer(SMALL_FP8, seed=506)
    hl.bias = None
    hl.router_w[9] = hl.router_w[2]
    hl.router_w[11] = hl.router_w[2]
    run = Run(SMALL_FP8, hl, dev, max_tokens=8)
    x = W.host_x(SMALL_FP8, 8, seed=506)
    x[3] = 0
    ids, wts, y = check_layer(run, x, label="zero+ties")
    assert list(ids[3]) == [0, 1, 2, 3] and np.all(wts[3] == 0.25) and np.all(y[3] == 0)
    check_routing(run, x, label="zero+ties")


@pytest.mark.parametrize("E,k,H,T,screen", [(300, 4, 1024, 256, 0), (257, 8, 512, 700, 0), (64, 17, 256, 1024, 1)],
                         ids=lambda v: str(v))
def test_screened_routing_large(dev, E, k, H, T, screen):
    """The screened kernels at large batches, on layers that they serve by default (more than
    256 experts) or when asked for (more than 16 choices)."""
    cfg = LayerConfig(f"screened-{E}-{k}", H, E, k, 128, "bf16", "bf16", "fp8", "normal:0.5", [])
    run = Run(cfg, W.host_layer(cfg, seed=522), dev, max_tokens=T, screen_min_tokens=screen)
    check_layer(run, W.host_x(cfg, T, seed=522), label=f"{cfg.name} T={T}")
    st = run.m.stats()[0]
    assert st.route_screened == 1 and st.n_exact_logits < T * E


def test_screened_routing_degenerate(dev):
    """The screened forward step brackets every logit with matrix-core sums and
    computes exactly only the experts that can reach the top k.  Degenerate inputs
    make every expert a candidate: a zero row (all logits +0), duplicate router rows
    (ties to the lower index), and logits on fp32 rounding midpoints (double-double
    fallback); the selection must still be the oracle's."""
    hl = W.host_layer(SMALL_FP8, seed=514)
    hl.bias = None
    hl.router_w[9] = hl.router_w[2]
    hl.router_w[11] = hl.router_w[2]
    run = Run(SMALL_FP8, hl, dev, max_tokens=64, screen_min_tokens=1)
    x = W.host_x(SMALL_FP8, 40, seed=514)
    x[3] = 0
    x[17] = 0
    ids, wts, y = check_layer(run, x, label="screened zero+ties")
    assert list(ids[3]) == [0, 1, 2, 3] and np.all(wts[3] == 0.25) and np.all(y[3] == 0)

    cfg = LayerConfig("midpoint-screened", 512, 16, 4, 256, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=515)
    one, tiny24, tiny80 = 0x3F80, 0x3380, 0x1780  # 1.0, 2^-24, 2^-80 in bf16
    hl.router_w[:] = 0
    hl.router_w[:, 0] = one
    hl.router_w[5, 1] = tiny24  # l = 1 + 2^-24: tie -> 1.0
    hl.router_w[6, 1] = tiny24  # l = 1 + 2^-24 + 2^-80: above the tie -> 1 + 2^-23
    hl.router_w[6, 2] = tiny80
    x = np.zeros((36, cfg.hidden), np.uint16)
    x[:, 0] = x[:, 1] = x[:, 2] = one
    run = Run(cfg, hl, dev, max_tokens=64, screen_min_tokens=1)
    ids, _, _ = check_layer(run, x, label="screened midpoint")
    assert np.all(ids[:, 0] == 6)
    st, _ = run.m.stats()
    assert st.route_screened and st.n_fallback >= 36 and st.n_exact_logits == 36 * 16


def test_exact_fallback_path(dev):
    """Logits whose exact value sits on (or within 2^-80 of) an fp32 rounding midpoint
    must take the double-double path and still equal the oracle bit for bit."""
    from paper_2609_11133_amd import binding as B

    cfg = LayerConfig("midpoint", 512, 16, 4, 256, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=507)
    one, tiny24, tiny80 = 0x3F80, 0x3380, 0x1780  # 1.0, 2^-24, 2^-80 in bf16
    hl.router_w[:] = 0
    hl.router_w[:, 0] = one
    hl.router_w[5, 1] = tiny24          # l = 1 + 2^-24: tie -> 1.0
    hl.router_w[6, 1] = tiny24          # l = 1 + 2^-24 + 2^-80: above the tie -> 1 + 2^-23
    hl.router_w[6, 2] = tiny80
    x = np.zeros((4, cfg.hidden), np.uint16)
    x[:, 0] = one
    x[:, 1] = one
    x[:, 2] = one
    run = Run(cfg, hl, dev, max_tokens=8)
    lg, ids, _ = check_routing(run, x, label="midpoint")
    assert lg[0, 5] == np.float32(1.0) and lg[0, 6] == np.float32(1.0 + 2.0**-23)
    assert ids[0, 0] == 6
    check_layer(run, x, label="midpoint")
    st, _ = run.m.stats()
    assert st.n_fallback >= 4


def tiled(cfg, T, k=None):
    """Whether a step of this size takes the tiled routing."""
    E, H = cfg.n_experts, cfg.hidden
    if T * E <= 6400 or E > 256 or (k or cfg.topk) > 16 or H % 256:
        return False
    if cfg.act != "bf16" or cfg.router != "bf16":
        return True
    return T >= 50 if H >= 3072 else T * E >= 10000 and T >= (256 if E > 192 and H >= 2048 else 128)


# (experts, top-k, hidden, activations, router, tokens on both sides of the switch to the
# tiled routing, or past one of its limits: 256 experts, 16 choices, inputs in 256s); token
# and expert tiles of 16 with remainders, 4 to 16 keys per lane, 1 to 4 slices of the inputs
TILED = [(256, 16, 256, "bf16", "bf16", (127, 128)), (130, 3, 512, "bf16", "f32", (49, 50)),
         (160, 8, 1280, "f32", "bf16", (40, 41)), (64, 1, 2048, "f32", "f32", (100, 101)),
         (65, 5, 768, "bf16", "bf16", (153, 154)), (16, 16, 512, "bf16", "bf16", (624, 625)),
         (200, 16, 1024, "bf16", "bf16", (127, 131)), (200, 4, 2048, "bf16", "bf16", (255, 256)),
         (136, 4, 3072, "bf16", "bf16", (49, 50)), (257, 2, 256, "bf16", "bf16", (130,)),
         (160, 17, 256, "bf16", "bf16", (130,)), (160, 8, 384, "bf16", "bf16", (130,))]


@pytest.mark.parametrize("E,k,H,act,router,tokens", TILED, ids=lambda v: str(v))
def test_tiled_routing(dev, E, k, H, act, router, tokens):
    """Bit-exact logits and selections on both sides of the switch to the tiled routing (and
    of its limits on experts, choices and inputs), with and without grouping; the screen
    asked for or not, which the tiled routing does not run."""
    cfg = LayerConfig(f"tiled-{E}-{k}-{H}", H, E, k, 256, act, router, "fp8", "normal:0.5", [])
    hl = W.host_layer(cfg, seed=517)
    assert [tiled(cfg, t) for t in tokens] == ([False, True] if len(tokens) == 2 else [False])
    for screen in (-1, 1):
        run = Run(cfg, hl, dev, max_tokens=max(tokens), screen_min_tokens=screen)
        for t in tokens:
            x = W.host_x(cfg, t, seed=517 + t)
            check_layer(run, x, label=f"{cfg.name} T={t} screen={screen}")
            st, _ = run.m.stats()
            screened = screen > 0 and act == "bf16" and router == "bf16" and H % 256 == 0 and not tiled(cfg, t)
            assert st.route_screened == screened
            if screened:
                assert st.n_exact_logits < t * E or k == E
            elif tiled(cfg, t):  # a few logits per token tile are uncertain, fewer matter
                assert 0.9 * t * E <= st.n_exact_logits <= t * E
            else:
                assert st.n_exact_logits == t * E
            if screen < 0:
                check_routing(run, x, label=f"{cfg.name} T={t}")


@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
def test_tiled_routing_degenerate(dev, screen):
    """The tiled routing on zero rows, ties (to the lower index) and logits on fp32 rounding
    midpoints, which no error bound certifies."""
    cfg = LayerConfig("tiled-midpoint", 512, 16, 4, 256, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=518)
    one, tiny24, tiny80 = 0x3F80, 0x3380, 0x1780  # 1.0, 2^-24, 2^-80 in bf16
    hl.router_w[:] = 0
    hl.router_w[:, 0] = one
    hl.router_w[5, 1] = tiny24  # l = 1 + 2^-24: tie -> 1.0
    hl.router_w[6, 1] = tiny24  # l = 1 + 2^-24 + 2^-80: above the tie -> 1 + 2^-23
    hl.router_w[6, 2] = tiny80
    T = 641
    assert tiled(cfg, T)
    x = np.zeros((T, cfg.hidden), np.uint16)
    x[:, 0] = x[:, 1] = x[:, 2] = one
    x[7] = 0
    x[400:] = 0
    run = Run(cfg, hl, dev, max_tokens=T, screen_min_tokens=screen)
    ids, _, _ = check_layer(run, x, label=f"tiled midpoint screen={screen}")
    assert np.all(ids[8:400, 0] == 6) and list(ids[7]) == [0, 1, 2, 3]
    st, _ = run.m.stats()
    assert st.n_fallback >= 399
    check_routing(run, x, label="tiled midpoint")


def _bf16(v):
    """fp32 values that are bf16 values -> their bits."""
    u = np.asarray(v, np.float32).view(np.uint32)
    assert not (u & 0xFFFF).any()
    return (u >> 16).astype(np.uint16)


@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
def test_tiled_routing_cancellation(dev, screen):
    """Logits whose products cancel: the fp64 sum's bound spans many fp32 steps there, and
    the top k has to come from the exact values.  Rows 0..15: equal zeros of different row
    norms (ties to the lower index); then a tiny positive logit next to certain zeros; then
    pairs of random products that cancel and leave tiny logits of either sign."""
    cfg = LayerConfig("tiled-cancel", 512, 16, 4, 256, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=519)
    T = 641
    assert tiled(cfg, T, 4)
    run = Run(cfg, hl, dev, max_tokens=T, screen_min_tokens=screen)

    def check(x, w, k, label):
        hl.router_w[:] = _bf16(w)
        run.rw = W.to_device(hl.router_w, dev)
        ids, _, _ = check_layer(run, _bf16(x), topk=k, label=f"tiled cancel {label} screen={screen}")
        left = T * 16 - run.m.stats()[0].n_exact_logits  # uncertain, but below the top k
        say(f"[route] {label}: {left} of {T * 16} logits left uncertain")
        assert left > 0 if label.startswith("pairs") else left == 0
        check_routing(run, _bf16(x[:633]), topk=k, label=f"tiled cancel {label}")
        return ids

    x, w = np.zeros((T, cfg.hidden)), np.zeros((16, cfg.hidden))
    x[:, :2] = 1.0
    w[:, 0] = 2.0 - np.arange(16) / 16
    w[:, 1] = -w[:, 0]
    assert np.all(check(x, w, 4, "zeros") == np.arange(4))

    x[:, :3] = 2.0 ** 24, 2.0 ** 24, 1.0
    w[:] = 0
    w[1, :3] = 1.0, -1.0, 2.0 ** -21
    assert np.all(check(x, w, 1, "tiny") == 1)

    r = np.random.default_rng(519)
    m = lambda n: (1 + r.integers(0, 128, n) / 128) * np.exp2(r.integers(-4, 5, n)) * r.choice([-1, 1], n)  # noqa: E731
    x = np.empty((T, cfg.hidden))
    x[:, 0::2] = m((T, cfg.hidden // 2))
    x[:, 1::2] = x[:, 0::2]
    w = np.empty((16, cfg.hidden))
    w[:, 0::2] = m((16, cfg.hidden // 2)) * np.exp2(r.integers(0, 12, 16))[:, None]  # norms of a wide range
    w[:, 1::2] = -w[:, 0::2]
    x[:, -1] = 2.0 ** -20
    x[:, -2] = 0
    for k in (1, 3, 4):
        check(x, w, k, f"pairs k={k}")


@pytest.mark.parametrize("E,k,T", [(128, 8, 131), (160, 16, 129), (20, 4, 505)], ids=lambda v: str(v))
@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
def test_tiled_routing_unordered_rows(dev, E, k, T, screen):
    """Tokens whose logits do not compare (NaN or infinite inputs) still get k different
    experts below E and leave the other tokens' results alone, on expert counts that fill the
    sixteen lanes and that do not."""
    cfg = LayerConfig(f"tiled-nan-{E}", 256, E, k, 256, "bf16", "bf16", "fp8", "normal:0.5", [])
    hl = W.host_layer(cfg, seed=520)
    run = Run(cfg, hl, dev, max_tokens=T, screen_min_tokens=screen)
    x = W.host_x(cfg, T, seed=520)
    assert tiled(cfg, T)
    ids0, wts0, y0 = check_layer(run, x, label=f"{cfg.name} clean")
    bad = [0, 17, 18, T - 1]
    x[0] = 0x7FC0        # NaN
    x[17, 3] = 0xFFC0    # one NaN, its sign bit set
    x[18, 5] = 0x7F80    # +inf
    x[T - 1, 7] = 0xFF80  # -inf
    ids, wts, y = run.forward(x)
    rids = run.route(x)[1]
    ok = np.setdiff1d(np.arange(T), bad)
    for i in (ids, rids):
        assert np.array_equal(i[ok], ids0[ok]) and i.min() >= 0 and i.max() < E
        assert all(len(set(i[t])) == k for t in bad)
    assert np.array_equal(wts[ok], wts0[ok])
    # an expert's tokens may fall into other columns, which changes no sum of a token
    assert np.array_equal(y[ok], y0[ok])


def test_tiled_routing_overflowing_logits(dev):
    """Finite inputs whose logits overflow fp32 to -inf: the finite ones first, then the
    infinite ones by index, none twice."""
    cfg = LayerConfig("tiled-overflow", 512, 16, 4, 256, "bf16", "bf16", "fp8", None, [])
    hl = W.host_layer(cfg, seed=521)
    T = 641
    assert tiled(cfg, T)
    run = Run(cfg, hl, dev, max_tokens=T, screen_min_tokens=-1)
    x, w = np.zeros((T, cfg.hidden)), np.zeros((16, cfg.hidden))
    x[:, 0] = 2.0 ** 100
    x[:, 1] = 1.0
    w[:, 0] = -(2.0 ** 100)
    w[[3, 9], 0] = 0
    w[[3, 9], 1] = 1.0, 2.0
    hl.router_w[:] = _bf16(w)
    run.rw = W.to_device(hl.router_w, dev)
    _, ids, wts = run.route(_bf16(x))
    assert np.all(ids == [9, 3, 0, 1])
    e = np.exp(-1.0)
    assert np.abs(wts - np.array([1 / (1 + e), e / (1 + e), 0, 0])).max() <= 1e-6


def test_bitwise_repeatable_and_permutation_equivariant(dev):
    hl = W.host_layer(SMALL_FP8, seed=508)
    run = Run(SMALL_FP8, hl, dev, max_tokens=32)
    x = W.host_x(SMALL_FP8, 29, seed=508)
    a = run.forward(x)
    for _ in range(3):
        b = run.forward(x)
        assert all(np.array_equal(p, q) for p, q in zip(a, b))
    perm = np.random.default_rng(0).permutation(29)
    c = run.forward(x[perm])
    assert np.array_equal(c[0], a[0][perm]) and np.array_equal(c[2], a[2][perm])


def test_zero_tokens_leaves_output_untouched(dev):
    hl = W.host_layer(SMALL_FP8, seed=509)
    run = Run(SMALL_FP8, hl, dev, max_tokens=8)
    y = torch.full((1, SMALL_FP8.hidden), 7.0, dtype=torch.bfloat16, device=dev)
    xd = torch.zeros((1, SMALL_FP8.hidden), dtype=torch.int16, device=dev)
    run.m.forward(xd, 0, run.rw, run.bias, run.ew, run.sc, 4, y)
    torch.cuda.synchronize(dev)
    assert torch.all(y == 7.0)


@pytest.mark.parametrize("screen", [-1, 1], ids=["exact", "screened"])
def test_max_tokens(dev, screen):
    cfg = LayerConfig("maxT", 512, 16, 4, 256, "bf16", "bf16", "fp8", "normal:0.5", [])
    hl = W.host_layer(cfg, seed=510)
    run = Run(cfg, hl, dev, max_tokens=1024, screen_min_tokens=screen)
    tokens = None if screen > 0 else [0, 511, 1023]  # the screened run: every token
    check_layer(run, W.host_x(cfg, 1024, seed=510), tokens=tokens, label=f"T=1024 screen={screen}")


# LDS-staged MFMA kernels (K spanning a multiple of four 128-input blocks; the down
# projection from 16 blocks): small layers whose I reaches them, with Zipf skew so that
# some expert holds more than 16 tokens (32-token tiles) and others a single one.
LDS_FP8 = LayerConfig("lds-fp8", 512, 16, 4, 2048, "bf16", "bf16", "fp8", "zipf:1.1", [])
LDS_MX = LayerConfig("lds-mxfp4", 1024, 16, 4, 2048, "bf16", "bf16", "mxfp4", "zipf:1.1", [])


@pytest.mark.parametrize("cfg", [LDS_FP8, LDS_MX], ids=["fp8", "mxfp4"])
@pytest.mark.parametrize("T", [1, 7, 32])
def test_lds_staged_kernels(dev, cfg, T):
    hl = W.host_layer(cfg, seed=530)
    run = Run(cfg, hl, dev, max_tokens=32)
    check_layer(run, W.host_x(cfg, T, seed=530 + T), label=f"{cfg.name} T={T}")
    st, counts = run.m.stats()
    say(f"[lds] {cfg.name} T={T}: tokens per expert {sorted(counts, reverse=True)[:4]}")
    if T == 32:
        assert max(counts) > 16


# Seeded random small layers across the accepted shapes: weight formats, activation
# and router dtypes, bias recipes, K extents that take the staged or the two-tile
# kernels, top-k up to 16 and ragged token counts.
# ---------------------------------------------------------------- packed 16-row tile layout

def pack_reference(expert_w, cfg):
    """Packed 16-row tiles from row-major expert weights (uint8 [E][bytes]), written
    from the layout's definition: per matrix [rows][K] and per (16-row tile, 128-input
    K block), lane l's operand bytes of row l%16 in lane order."""
    fp4 = cfg.wfmt != "fp8"
    H, I, E = cfg.hidden, cfg.inter, cfg.n_experts
    ew = expert_w.reshape(E, -1)
    out = np.empty_like(ew)
    for rows, K, off in ((2 * I, H, 0), (H, I, 2 * I * H // (2 if fp4 else 1))):
        rowb = K // 2 if fp4 else K
        m = ew[:, off: off + rows * rowb]
        if cfg.wfmt == "mxfp4":  # [E][tile][r][kb][g*16+i] -> [E][tile][kb][g][r][i]
            v = m.reshape(E, rows // 16, 16, K // 128, 4, 16).transpose(0, 1, 3, 4, 2, 5)
        elif cfg.wfmt == "nvfp4":  # 256-input blocks: [E][tile][r][kb][g*32+half*16+i] -> [..][kb][half][g][r][i]
            v = m.reshape(E, rows // 16, 16, K // 256, 4, 2, 16).transpose(0, 1, 3, 5, 4, 2, 6)
        else:  # [E][tile][r][kb][half*64+g*16+i] -> [E][tile][kb][half][g][r][i]
            v = m.reshape(E, rows // 16, 16, K // 128, 2, 4, 16).transpose(0, 1, 3, 4, 5, 2, 6)
        out[:, off: off + rows * rowb] = v.reshape(E, -1)
    return out.reshape(expert_w.shape)


def pack_scales_reference(scales, cfg):
    """Packed scales.  NVFP4 E4M3: per expert the 16 bytes of matrix scales, then per
    matrix [rows][K/16] and per (16-row tile, 256-input block) 256 bytes, lane l's
    scales [4g, 4g+4) of row l%16 at 4l; where K/256 is a multiple of four, per (16-row
    tile, group of four blocks) 1 KB, lane l's scales of each block of the group at 16l.
    MXFP4 E8M0: per matrix [rows][K/32] and per
    (16-row tile, group of four 128-input blocks) lane l's bytes (sub-block g of row l%16,
    blocks 4q..4q+3) at 4l (a last group of two blocks: 2l)."""
    H, I, E = cfg.hidden, cfg.inter, cfg.n_experts
    sc = scales.reshape(E, -1)
    out = sc.copy()
    if cfg.wfmt == "mxfp4":
        off = 0
        for rows, K in ((2 * I, H), (H, I)):
            KB = K // 128
            m = sc[:, off: off + rows * K // 32].reshape(E, rows // 16, 16, KB, 4)  # [E][tile][r][kb][g]
            parts = []
            for q0 in range(0, KB, 4):
                n = min(4, KB - q0)
                parts.append(m[:, :, :, q0: q0 + n, :].transpose(0, 1, 4, 2, 3).reshape(E, rows // 16, -1))
            out[:, off: off + rows * K // 32] = np.concatenate(parts, axis=2).reshape(E, -1)
            off += rows * K // 32
        return out.reshape(scales.shape)
    off = 16
    for rows, K in ((2 * I, H), (H, I)):
        KB = K // 256
        m = sc[:, off: off + rows * K // 16].reshape(E, rows // 16, 16, KB, 4, 4)  # [E][tile][r][kb][g][4]
        if KB % 4 == 0:  # [E][tile][group][g][r][block of the group][4]
            v = m.reshape(E, rows // 16, 16, KB // 4, 4, 4, 4).transpose(0, 1, 3, 5, 2, 4, 6)
        else:  # [E][tile][kb][g][r][4]
            v = m.transpose(0, 1, 3, 4, 2, 5)
        out[:, off: off + rows * K // 16] = v.reshape(E, -1)
        off += rows * K // 16
    return out.reshape(scales.shape)


PACK_MX_768 = LayerConfig("pk-mx-768", 768, 16, 4, 768, "bf16", "bf16", "mxfp4", None, [])


PACK_NV_G = LayerConfig("pk-nv-g", 2048, 8, 2, 1024, "bf16", "bf16", "nvfp4", None, [])


@pytest.mark.parametrize("cfg", [SMALL_FP8, SMALL_MX, PACK_MX_768, SMALL_NV, PACK_NV_G],
                         ids=["fp8", "mxfp4", "mxfp4-768", "nvfp4", "nvfp4-grouped"])
def test_pack_matches_layout_definition(dev, cfg):
    from paper_2609_11133_amd import binding as B

    hl = W.host_layer(cfg, seed=560)
    bc = W.binding_config(cfg, 8, weight_layout=1)
    src = W.to_device(hl.expert_w, dev)
    dst = torch.zeros_like(src)
    nv = cfg.wfmt != "fp8"
    ssrc = W.to_device(hl.scales, dev) if nv else None
    sdst = torch.zeros_like(ssrc) if nv else None
    B.moe_decode_pack_weights(bc, torch.cuda.current_stream(dev).cuda_stream, src, dst, cfg.n_experts, ssrc, sdst)
    torch.cuda.synchronize(dev)
    got = dst.cpu().numpy().view(np.uint8).reshape(hl.expert_w.view(np.uint8).shape)
    assert np.array_equal(got, pack_reference(hl.expert_w.view(np.uint8), cfg))
    if nv:
        gs = sdst.cpu().numpy().view(np.uint8).reshape(hl.scales.view(np.uint8).shape)
        assert np.array_equal(gs, pack_scales_reference(hl.scales.view(np.uint8), cfg))


# every kernel variant on packed weights: FP8 staged gate/up (H/128 a multiple of 4) and
# two-tile gate/up (H = 384), two-tile down (I/128 < 16) and staged down (I = 2048);
# E2M1 staged (H, I multiples of 512; three gate/up tiles per wave in eight-wave
# workgroups at I = 1536) and two-tile (H = I = 768) kernels
PACKED_CFGS = [
    LayerConfig("pk-fp8", 512, 16, 4, 256, "bf16", "bf16", "fp8", "normal:0.5", []),
    LayerConfig("pk-fp8-h384", 384, 16, 4, 2048, "bf16", "bf16", "fp8", None, []),
    LayerConfig("pk-mx", 512, 16, 4, 512, "bf16", "bf16", "mxfp4", "zipf:1.1", []),
    LayerConfig("pk-mx-768", 768, 16, 4, 768, "bf16", "bf16", "mxfp4", None, []),
    # E2M1 staged gate/up with three tiles per wave (I a multiple of 1536)
    LayerConfig("pk-mx-i1536", 1024, 16, 4, 1536, "bf16", "bf16", "mxfp4", "zipf:1.1", []),
    LayerConfig("pk-f32-mx", 256, 8, 2, 256, "f32", "f32", "mxfp4", None, []),
    LayerConfig("pk-nv", 512, 16, 4, 256, "bf16", "bf16", "nvfp4", "normal:0.5", []),
    LayerConfig("pk-nv-odd", 1280, 16, 4, 768, "bf16", "bf16", "nvfp4", "zipf:1.1", []),
    # grouped NVFP4 scales (K/256 a multiple of four): one group in both projections, and
    # three groups (gate/up) with two (down)
    LayerConfig("pk-nv-g4", 1024, 16, 4, 1024, "bf16", "bf16", "nvfp4", None, []),
    LayerConfig("pk-nv-g12", 3072, 8, 2, 2048, "bf16", "bf16", "nvfp4", "normal:0.5", []),
]


@pytest.mark.parametrize("cfg", PACKED_CFGS, ids=[c.name for c in PACKED_CFGS])
@pytest.mark.parametrize("T", [1, 13, 40])
def test_packed_layout_layers(dev, cfg, T):
    hl = W.host_layer(cfg, seed=561)
    run = Run(cfg, hl, dev, max_tokens=40, weight_layout=1)
    check_layer(run, W.host_x(cfg, T, seed=561), label=f"{cfg.name} packed T={T}")


PK_MX_SKEW = LayerConfig("pk-mx-skew", 1024, 8, 2, 512, "bf16", "bf16", "mxfp4", "zipf:1.1", [])
# three gate/up tiles per wave (I a multiple of 1536)
PK_MX_SKEW_I1536 = LayerConfig("pk-mx-skew-i1536", 512, 8, 2, 1536, "bf16", "bf16", "mxfp4", "zipf:1.1", [])


@pytest.mark.parametrize("cfg", [PK_MX_SKEW, PK_MX_SKEW_I1536], ids=lambda c: c.name)
@pytest.mark.parametrize("T", [20, 70, 150])
def test_packed_mxfp4_skewed_chunks(dev, cfg, T):
    """Packed MXFP4 weights on the staged kernels (four and three tiles per wave) with a
    Zipf-skewed small layer: the hot expert fits one chunk of two token tiles at T=20
    (17 and 13 tokens), takes two chunks at T=70 (more than 32) and three or four at
    T=150 (more than 64)."""
    hl = W.host_layer(cfg, seed=571)
    run = Run(cfg, hl, dev, max_tokens=150, weight_layout=1)
    check_layer(run, W.host_x(cfg, T, seed=571 + T), label=f"{cfg.name} T={T}")
    st, counts = run.m.stats()
    say(f"[skew] {cfg.name} T={T}: tokens per expert {sorted(counts, reverse=True)}")
    if T >= 70:
        assert max(counts) > 32
    if T == 150:
        assert max(counts) > 64


# The large-batch FP8 kernels (128-token chunks): K block counts of 6 and 5 (gate/up, down:
# tails of two and one blocks), and of 4 and 3.
WIDE_FP8 = [LayerConfig("wide-k6-5", 768, 16, 8, 640, "bf16", "bf16", "fp8", "zipf:1.1", []),
            LayerConfig("wide-k4-3", 512, 16, 8, 384, "f32", "bf16", "fp8", "zipf:1.1", [])]


def wide_from(cfg, packed):
    """The fewest tokens of a step that takes the wide kernels, on a layer of few work items
    (the rule of chunk_tokens)."""
    E, t13, t2 = cfg.n_experts, cfg.inter // 128, cfg.hidden // 256
    assert E * (t13 + t2) < 1024
    if cfg.wfmt == "fp8":
        pairs = max((20000 if packed else 26000) * E // cfg.inter + 1, -(-7680 // min(t13, t2)), 32 * E)
    else:
        pairs = max((13 if packed else 3) * E + 1, (13000 if packed else 7000) * E // cfg.inter + 1,
                    -(-(6144 if packed else 4608) // min(t13, t2)), (30 if packed else 16) * E)
    return -(-pairs // cfg.topk)


@pytest.mark.parametrize("cfg", WIDE_FP8, ids=lambda c: c.name)
@pytest.mark.parametrize("layout", [0, 1], ids=["rows", "packed"])
def test_wide_chunks(dev, cfg, layout):
    """FP8 layers on both sides of the switch to 128-token chunks.  The Zipf-skewed batches
    give chunks of few tokens, of every number of token-tile pairs (2, 4, 6, 8 tiles) and
    several chunks of one expert."""
    hl = W.host_layer(cfg, seed=611)
    first = wide_from(cfg, layout == 1)
    assert first < 640
    run = Run(cfg, hl, dev, max_tokens=700, weight_layout=layout)
    sizes = set()
    for T in (first - 1, first, 640, 700):
        check_layer(run, W.host_x(cfg, T, seed=611 + T), label=f"{cfg.name} T={T}")
        _, counts = run.m.stats()
        say(f"[wide] {cfg.name} T={T}: tokens per expert {sorted(counts, reverse=True)}")
        if T >= first:
            for c in counts:
                sizes |= {128} if c >= 128 else set()
                sizes |= {c % 128} - {0}
    assert max(counts) > 256
    for lo, hi in ((1, 32), (33, 64), (65, 96), (97, 128)):
        assert any(lo <= n <= hi for n in sizes), (lo, hi, sorted(sizes))


# The large-batch NVFP4 kernels (64-token chunks): K block counts of 5 and 3, 2 and 1, and 8
# and 4 (grouped packed scales in both projections).
WIDE_NV = [LayerConfig("nv-wide-k5-3", 1280, 16, 8, 768, "bf16", "bf16", "nvfp4", "zipf:1.1", []),
           LayerConfig("nv-wide-k2-1", 512, 16, 8, 256, "bf16", "bf16", "nvfp4", "zipf:1.1", []),
           LayerConfig("nv-wide-k8-4", 2048, 16, 8, 1024, "bf16", "bf16", "nvfp4", "zipf:1.1", [])]


@pytest.mark.parametrize("cfg", WIDE_NV, ids=lambda c: c.name)
@pytest.mark.parametrize("layout", [0, 1], ids=["rows", "packed"])
def test_nvfp4_wide_chunks(dev, cfg, layout):
    """NVFP4 layers on both sides of the switch to 64-token chunks; the Zipf-skewed batches
    give chunks of both token-tile counts and several chunks of one expert."""
    hl = W.host_layer(cfg, seed=621)
    first = wide_from(cfg, layout == 1)
    run = Run(cfg, hl, dev, max_tokens=first + 80, weight_layout=layout)
    sizes = set()
    for T in (first - 1, first, first + 80):
        check_layer(run, W.host_x(cfg, T, seed=621 + T), label=f"{cfg.name} T={T}")
        _, counts = run.m.stats()
        say(f"[wide] {cfg.name} T={T}: tokens per expert {sorted(counts, reverse=True)}")
        if T >= first:
            sizes |= {c % 64 for c in counts} | {64 * (c >= 64) for c in counts}
    assert max(counts) > 128
    assert any(1 <= n <= 32 for n in sizes) and any(33 <= n <= 64 for n in sizes)


# (layer, top-k, tokens): the down projection that combines, taken up to 8 pairs, and for FP8
# layers of I up to 2048 up to 8 tokens where its row blocks fill the CUs evenly (H 4096) or,
# packed, at least three quarters of them; K block counts from 1 to 16 around its ring of
# four, passes of up to eight tokens, and the token and pair counts next to its limits; NVFP4
# layers up to 12 tokens (or 8 pairs) in passes of four and eight, with each scale layout (K
# block counts 1, 3, 4 and 5)
OWN = [(LayerConfig("own-k1", 256, 8, 2, 128, "f32", "f32", "fp8", None, []), (1, 3, 4, 5)),
       (LayerConfig("own-k5", 640, 16, 4, 640, "bf16", "bf16", "fp8", "normal:0.5", []), (1, 2, 3)),
       (LayerConfig("own-mx-k6", 1024, 8, 1, 768, "bf16", "bf16", "mxfp4", "zipf:1.1", []), (1, 7, 8, 9)),
       (LayerConfig("own-mx-k4", 512, 4, 4, 512, "f32", "bf16", "mxfp4", "zipf:1.1", []), (1, 2)),
       (LayerConfig("own-h4096", 4096, 16, 4, 384, "bf16", "bf16", "fp8", "zipf:1.1", []), (3, 7, 8, 9)),
       (LayerConfig("own-h4096-k3", 4096, 24, 3, 1152, "f32", "bf16", "fp8", None, []), (8,)),
       (LayerConfig("own-h3072", 3072, 12, 4, 2048, "bf16", "bf16", "fp8", "zipf:1.1", []), (3, 8, 9)),
       (LayerConfig("own-h3968", 3968, 12, 2, 256, "f32", "f32", "fp8", None, []), (5, 8)),
       (LayerConfig("own-nv-k1", 256, 8, 2, 256, "bf16", "bf16", "nvfp4", None, []), (1, 3, 4, 5)),
       (LayerConfig("own-nv-k4", 3072, 16, 4, 1024, "bf16", "f32", "nvfp4", "zipf:1.1", []), (1, 2, 4, 5, 12, 13)),
       (LayerConfig("own-nv-h4096", 4096, 64, 3, 768, "bf16", "bf16", "nvfp4", "normal:0.5", []), (4, 10, 11, 12)),
       (LayerConfig("own-nv-k5", 1024, 4, 1, 1280, "bf16", "bf16", "nvfp4", "zipf:1.1", []), (7, 8, 9))]


@pytest.mark.parametrize("cfg,tokens", OWN, ids=lambda v: v.name if isinstance(v, LayerConfig) else "")
@pytest.mark.parametrize("layout", [0, 1], ids=["rows", "packed"])
def test_down_projection_with_combine(dev, cfg, tokens, layout):
    hl = W.host_layer(cfg, seed=631)
    run = Run(cfg, hl, dev, max_tokens=max(tokens), weight_layout=layout)
    for T in tokens:
        check_layer(run, W.host_x(cfg, T, seed=631 + T), label=f"{cfg.name} T={T}")
        x = W.host_x(cfg, T, seed=900 + T)
        a, b = run.forward(x), run.forward(x)
        assert all(np.array_equal(p, q) for p, q in zip(a, b)), "not repeatable"


PK_NV_WIDE = LayerConfig("pk-nv-wide", 1024, 16, 8, 1024, "bf16", "bf16", "nvfp4", "zipf:1.1", [])


@pytest.mark.parametrize("T", [127, 128, 140])
def test_nvfp4_eight_wave_gate_up(dev, T):
    """NVFP4 gate/up on either side of the eight-wave choice (from 1024 (token, expert)
    pairs per step: T=128 at top-8), with skewed routing so that chunks are full."""
    hl = W.host_layer(PK_NV_WIDE, seed=591)
    run = Run(PK_NV_WIDE, hl, dev, max_tokens=140, weight_layout=1)
    check_layer(run, W.host_x(PK_NV_WIDE, T, seed=591 + T), label=f"{PK_NV_WIDE.name} T={T}")


PK_NV_T16 = LayerConfig("pk-nv-t16", 512, 32, 2, 256, "bf16", "bf16", "nvfp4", "zipf:1.1", [])


@pytest.mark.parametrize("T", [1, 37, 100, 128, 129])
def test_nvfp4_one_tile_passes(dev, T):
    """Packed NVFP4 kernels in passes of one 16-token tile, used up to eight (token,
    expert) pairs per expert on average (T <= 128 at top-2 of 32 experts), and the
    two-tile kernels at T=129.  Zipf-skewed routing gives the hot expert 24 tokens at
    T=37 (one chunk, two passes) and 70 at T=100 (chunks of 32, 32 and 6)."""
    hl = W.host_layer(PK_NV_T16, seed=601)
    run = Run(PK_NV_T16, hl, dev, max_tokens=129, weight_layout=1)
    check_layer(run, W.host_x(PK_NV_T16, T, seed=601 + T), label=f"{PK_NV_T16.name} T={T}")
    st, counts = run.m.stats()
    say(f"[t16] {PK_NV_T16.name} T={T}: tokens per expert {sorted(counts, reverse=True)[:6]}")
    if T == 37:
        assert max(counts) > 16
    if T >= 100:
        assert max(counts) > 32


@pytest.mark.parametrize("T", [1, 64])
def test_full_235b_packed(dev, full_235b, T):
    """The 235B-shaped layer on packed weights (staged gate/up, the 12-block down)."""
    run = Run(C.QWEN3_235B, full_235b, dev, max_tokens=64, weight_layout=1)
    _full(run, C.QWEN3_235B, T, batch=T)


@pytest.mark.parametrize("T", C.QWEN3_480B.tokens)
def test_full_480b_packed(dev, full_480b, T):
    """The 480B-shaped layer on packed weights in the launch configuration the
    benchmark times (max_tokens = 128, the largest T of the sweep)."""
    run = Run(C.QWEN3_480B, full_480b, dev, max_tokens=128, weight_layout=1)
    _full(run, C.QWEN3_480B, T, batch=5 + T)


@pytest.mark.parametrize("T", [1, 64])
def test_full_235b_nvfp4_packed(dev, full_235b_nv, T):
    run = Run(C.QWEN3_235B_NVFP4, full_235b_nv, dev, max_tokens=64, weight_layout=1)
    _full(run, C.QWEN3_235B_NVFP4, T, batch=T)


def test_full_mxfp4_zipf_packed(dev):
    cfg = C.QWEN3_235B_MXFP4
    hl = W.host_layer(cfg)
    run = Run(cfg, hl, dev, max_tokens=256, weight_layout=1)
    _full(run, cfg, 256, batch=6)


def _random_layer(i):
    rng = np.random.default_rng(9000 + i)
    wfmt = ["fp8", "mxfp4"][i % 2]
    q = 128 if wfmt == "fp8" else 256
    H = q * int(rng.integers(1, 9))
    I = q * int(rng.integers(1, 9))
    E = int(rng.choice([2, 5, 16, 40, 96, 160]))
    k = int(min(E, rng.choice([1, 2, 4, 8, 16])))
    act = ["bf16", "f32"][int(rng.integers(0, 4)) == 0]
    router = ["bf16", "f32"][int(rng.integers(0, 4)) == 0]
    bias = [None, "normal:0.5", "zipf:1.1"][int(rng.integers(0, 3))]
    T = int(rng.integers(1, 70))
    return LayerConfig(f"rand{i}", H, E, k, I, act, router, wfmt, bias, []), T


@pytest.mark.parametrize("i", range(12))
def test_random_small_layers(dev, i):
    cfg, T = _random_layer(i)
    assert 4 * max(cfg.hidden, cfg.inter) * (2 if cfg.act == "bf16" else 4) <= 65536  # accepted shapes
    hl = W.host_layer(cfg, seed=700 + i)
    run = Run(cfg, hl, dev, max_tokens=T, mfma_min_tokens=[0, -1, 2][i % 3], screen_min_tokens=[1, -1][(i // 2) % 2])
    say(f"[random] {cfg}")
    check_layer(run, W.host_x(cfg, T, seed=700 + i), label=f"random {i}")


def _random_nvfp4_layer(i):
    rng = np.random.default_rng(9500 + i)
    H = 256 * int(rng.integers(1, 9))
    I = 256 * int(rng.integers(1, 9))
    E = int(rng.choice([2, 5, 16, 40, 96, 160]))
    k = int(min(E, rng.choice([1, 2, 4, 8, 16])))
    router = ["bf16", "f32"][int(rng.integers(0, 4)) == 0]
    bias = [None, "normal:0.5", "zipf:1.1"][int(rng.integers(0, 3))]
    T = int(rng.integers(1, 70))
    return LayerConfig(f"rand-nv{i}", H, E, k, I, "bf16", router, "nvfp4", bias, []), T


@pytest.mark.parametrize("i", range(6))
def test_random_nvfp4_layers(dev, i):
    cfg, T = _random_nvfp4_layer(i)
    hl = W.host_layer(cfg, seed=750 + i)
    run = Run(cfg, hl, dev, max_tokens=T, mfma_min_tokens=[0, -1, 2][i % 3], screen_min_tokens=[1, -1][i % 2])
    say(f"[random] {cfg}")
    check_layer(run, W.host_x(cfg, T, seed=750 + i), label=f"random nvfp4 {i}")


@pytest.mark.parametrize("i", range(10))
def test_random_packed_layers(dev, i):
    """Random shapes of all three weight formats on packed 16-row tiles (and packed E2M1
    scales), MFMA for every expert, screened routing forced on every other case."""
    cfg, T = _random_layer(100 + i) if i % 3 else _random_nvfp4_layer(100 + i)
    hl = W.host_layer(cfg, seed=780 + i)
    run = Run(cfg, hl, dev, max_tokens=T, mfma_min_tokens=1, screen_min_tokens=[1, -1][i % 2], weight_layout=1)
    say(f"[random packed] {cfg}")
    check_layer(run, W.host_x(cfg, T, seed=780 + i), label=f"random packed {i}")


# ---------------------------------------------------------------- full-size layers

@pytest.fixture(scope="module")
def full_235b(dev):
    say("[gen] qwen3-235b-a22b layer")
    return W.host_layer(C.QWEN3_235B)


@pytest.fixture(scope="module")
def full_480b(dev):
    say("[gen] qwen3-coder-480b-a35b layer")
    return W.host_layer(C.QWEN3_480B)


def _full(run, cfg, T, batch, screened=None):
    """Every token of a full-size step against the oracle: expert selection, routing
    weights and outputs."""
    x = W.host_x(cfg, T, batch=batch)
    check_layer(run, x, label=f"{cfg.name} T={T}")
    st = run.m.stats()[0]
    if screened is None:  # the library default: screened from T*E*H >= 2^26 multiply-adds
        screened = T * cfg.n_experts * cfg.hidden >= 1 << 26
    screened = screened and not tiled(cfg, T)
    say(f"[route] screened={st.route_screened} exact logits {st.n_exact_logits} of {T * cfg.n_experts}")
    assert st.route_screened == screened


@pytest.mark.parametrize("screen", [0, 1], ids=["default", "screened"])
@pytest.mark.parametrize("T", C.QWEN3_235B.tokens)
def test_full_235b(dev, full_235b, T, screen):
    run = Run(C.QWEN3_235B, full_235b, dev, max_tokens=max(C.QWEN3_235B.tokens), screen_min_tokens=screen)
    _full(run, C.QWEN3_235B, T, batch=T, screened=True if screen else None)


@pytest.mark.parametrize("T", C.QWEN3_480B.tokens)
def test_full_480b(dev, full_480b, T):
    run = Run(C.QWEN3_480B, full_480b, dev, max_tokens=max(C.QWEN3_480B.tokens))
    _full(run, C.QWEN3_480B, T, batch=T)


@pytest.mark.parametrize("T", [1, 48])
def test_full_480b_tp4_shard(dev, T):
    """One GPU's share of the 480B layer in a TP4 decode lane (I = 640, five 128-blocks):
    the down projection's K spans five blocks, the gate/up projection's 48."""
    cfg = C.QWEN3_480B_TP4
    say("[gen] qwen3-coder-480b-a35b tp4 shard")
    hl = W.host_layer(cfg)
    run = Run(cfg, hl, dev, max_tokens=max(cfg.tokens))
    _full(run, cfg, T, batch=T)


def test_stack_480b_back_to_back(dev, full_480b):
    """Twelve 480B-shaped layers decoded back to back at T=256 on one handle and one
    stream with no synchronisation between them: three distinct weight sets (router,
    bias and experts of layers 0, 1 and 2 of the seeded generator), layer li running
    set li % 3 from its own device copy (twelve distinct addresses), a distinct input
    batch per layer.  Every layer's outputs are checked after a single
    synchronisation, on eight sampled tokens each."""
    cfg = C.QWEN3_480B
    L, T = C.QWEN3_480B_X12.layers, max(C.QWEN3_480B_X12.tokens)
    hls = [full_480b] + [W.host_layer(cfg, layer=s) for s in (1, 2)]
    runs = [Run(cfg, hl, dev, max_tokens=T) for hl in hls]
    m = runs[0].m  # one handle for every layer
    ews = [runs[li % 3].ew if li < 3 else runs[li % 3].ew.clone() for li in range(L)]
    xs = [W.host_x(cfg, T, batch=200 + li) for li in range(L)]
    ys = [W.empty_y(cfg, T, dev) for _ in range(L)]
    ids = [torch.full((T, cfg.topk), -1, dtype=torch.int32, device=dev) for _ in range(L)]
    wts = [torch.zeros((T, cfg.topk), dtype=torch.float32, device=dev) for _ in range(L)]
    xd = [W.to_device(x, dev) for x in xs]
    say(f"[stack] {L} layers x T={T}, {L * runs[0].ew.numel() / 1e9:.1f} GB of expert weights, 3 weight sets")
    for li in range(L):
        r = runs[li % 3]
        m.forward(xd[li], T, r.rw, r.bias, ews[li], r.sc, cfg.topk, ys[li], ids[li], wts[li])
    torch.cuda.synchronize(dev)
    for li in range(L):
        hl = hls[li % 3]
        tokens = sorted({(37 * li + 29 * j) % T for j in range(8)})
        lo, io, wo, yo = oracle.forward(xs[li], hl.router_w, hl.bias, hl.expert_w, hl.scales, cfg.topk, cfg.inter,
                                        cfg.wfmt_id, tokens=tokens, threads=THREADS)
        got_ids = ids[li].cpu().numpy()[tokens]
        got_y = W.y_to_f64(ys[li])[tokens]
        assert np.array_equal(got_ids, io), f"layer {li}: selection differs"
        assert np.abs(wts[li].cpu().numpy()[tokens] - wo).max() <= 1e-6
        err, scale = np.abs(got_y - yo).max(), np.abs(yo).max()
        say(f"[stack] layer {li} (weight set {li % 3}) tokens {tokens}: max|err|/max|ref| = {err / scale:.3e}")
        assert err <= TOL * scale
    del runs, ews


def test_full_235b_mxfp4_zipf(dev):
    cfg = C.QWEN3_235B_MXFP4
    say("[gen] qwen3-235b-a22b mxfp4 layer")
    hl = W.host_layer(cfg)
    run = Run(cfg, hl, dev, max_tokens=256)
    _full(run, cfg, 256, batch=0)
    st, counts = run.m.stats()
    say(f"[zipf] active={st.n_active} max tokens/expert={max(counts)}")
    assert max(counts) > 4 * (256 * cfg.topk / st.n_active)  # skewed popularity


# ---------------------------------------------------------------- both expert paths

@pytest.mark.parametrize("mstar", [-1, 1, 2])
@pytest.mark.parametrize("cfg,T", [(SMALL_FP8, 13), (SMALL_MX, 13), (SMALL_FP8, 32), (C.TINY, 4), (SMALL_NV, 13)])
def test_expert_paths(dev, cfg, T, mstar):
    """mfma_min_tokens = -1 forces the GEMV path for every expert, 1 the MFMA path,
    2 mixes them within one step."""
    hl = W.host_layer(cfg, seed=520)
    run = Run(cfg, hl, dev, max_tokens=max(T, 32), mfma_min_tokens=mstar)
    check_layer(run, W.host_x(cfg, T, seed=520), label=f"{cfg.name} T={T} mstar={mstar}")
    st, counts = run.m.stats()
    if mstar == 1:
        assert st.n_active_mfma == st.n_active
    elif mstar == -1:
        assert st.n_active_mfma == 0
    say(f"[paths] mstar={mstar}: {st.n_active_mfma}/{st.n_active} experts on MFMA tiles")


@pytest.mark.parametrize("mstar", [-1, 1])
def test_full_235b_paths(dev, full_235b, mstar):
    cfg = C.QWEN3_235B
    run = Run(cfg, full_235b, dev, max_tokens=64, mfma_min_tokens=mstar)
    _full(run, cfg, 64, batch=3)


@pytest.mark.parametrize("mstar", [-1, 1])
def test_full_mxfp4_paths(dev, mstar):
    cfg = C.QWEN3_235B_MXFP4
    hl = W.host_layer(cfg)
    run = Run(cfg, hl, dev, max_tokens=256, mfma_min_tokens=mstar)
    _full(run, cfg, 256, batch=1)


@pytest.fixture(scope="module")
def full_235b_nv(dev):
    say("[gen] qwen3-235b-a22b nvfp4 layer")
    return W.host_layer(C.QWEN3_235B_NVFP4)


@pytest.mark.parametrize("T", C.QWEN3_235B_NVFP4.tokens)
def test_full_235b_nvfp4(dev, full_235b_nv, T):
    run = Run(C.QWEN3_235B_NVFP4, full_235b_nv, dev, max_tokens=max(C.QWEN3_235B_NVFP4.tokens))
    _full(run, C.QWEN3_235B_NVFP4, T, batch=T)


@pytest.mark.parametrize("mstar", [-1, 1])
def test_full_nvfp4_zipf_paths(dev, mstar):
    cfg = C.QWEN3_235B_NVFP4_ZIPF
    say("[gen] qwen3-235b-a22b nvfp4 zipf layer")
    hl = W.host_layer(cfg)
    run = Run(cfg, hl, dev, max_tokens=256, mfma_min_tokens=mstar)
    _full(run, cfg, 256, batch=2)
    st, counts = run.m.stats()
    say(f"[zipf] nvfp4 active={st.n_active} max tokens/expert={max(counts)}")
