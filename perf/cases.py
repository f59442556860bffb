"""Performance cases of the quantized-linear hot path, through its public entry points.

Each case is work that a program around a diffusion denoiser has this library do:

* ``linear``        one linear layer of a sampler step: the fp32 input quantized to the layer's
                    A8 format (static scales of a LUT, or each sample's own range), then the
                    mixed-format linear with searched weights (packed once, or compact);
* ``grouped``       the same layer with the DiT fork's group-scaled weights;
* ``conv``          the UNet's shortcut-fed 3x3 convolution on MXFP8 codes;
* ``search``        the per-channel weight search of a block's layers, packed for the GEMM;
* ``group_search``  the DiT (group size, format) search with its calibration energies;
* ``calibrate``     moments of a forward pass's layer inputs and the LUT built from them;
* ``step``          one sampler step over the four linears of a transformer block, still
                    calibrating while it runs.

Sizes are those of the SDXL-like and PixArt-like stacks (``synth.sdxl_block_layers``,
``synth.pixart_block_layers``), their single-step variant and the up-block convolution.
``exact`` redoes a case in plain torch from the formats' definitions, with binary64 sums.
"""
import math

import numpy as np
import torch

from paper_2609_33496_amd import cham, synth

DEV = "cuda"
W4, W8, DIT4 = cham.MASK_W4, cham.MASK_W8, cham.MASK_DIT_W4
ACT = {"int8": cham.A_INT8_ASYM, "e4m3": cham.A_FP8_E4M3, "e5m2": cham.A_FP8_E5M2, "mxfp8": cham.A_MXFP8,
       "mxint8": cham.A_MXINT8}
BUCKETS = 10


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------
def listed():
    return [
        # cross-attention K/V of the text tokens (2 x 120), each CFG half with its own range:
        # the smallest call, two rows of tiles and a long inner dimension
        dict(name="linear_text_kv", kind="linear", M=240, N=1152, K=4096, bits=4, act="int8", samples=2, packed=True, t=300),
        # attention output projection of a single-step sampler: few tiles, short inner dimension
        dict(name="linear_out_1024", kind="linear", M=1024, N=1280, K=1280, bits=4, act="e5m2", samples=0, packed=True, t=999),
        # GEGLU projection at width 1280, CFG batch 2: the widest output of the UNet stack
        dict(name="linear_geglu", kind="linear", M=2048, N=10240, K=1280, bits=4, act="e4m3", samples=0, packed=True, t=379),
        # feed-forward output with weights kept compact (0.6 B per weight resident): records
        # are derived in every call
        dict(name="linear_ff_compact", kind="linear", M=2048, N=1280, K=5120, bits=4, act="e5m2", samples=0, packed=False, t=700),
        # DiT MLP in W8A8 with per-sample dynamic scaling: the largest layer
        dict(name="linear_w8_fc1", kind="linear", M=8192, N=4608, K=1152, bits=8, act="int8", samples=2, packed=True, t=300),
        # 1x1 shortcut projection behind a skip concatenation (pinned to MXFP8), at an image
        # size that is not a power of two (2 x 50 x 81 pixels)
        dict(name="linear_mx_ragged", kind="linear", M=8100, N=640, K=1920, bits=4, act="mxfp8", samples=0, packed=True, t=500),
        # DiT QKV with group-scaled weights and per-sample dynamic FP8 inputs
        dict(name="grouped_qkv", kind="grouped", M=8192, N=3456, K=1152, act="e4m3", samples=2, t=300),
        # up-block resnet conv1 after the skip concatenation (1280 + 640 -> 640), CFG batch 2
        dict(name="conv_up_block", kind="conv", B=2, H=32, W=32, C=1920, Co=640, bits=4, act="mxfp8", t=500),
        # format search of one transformer block at width 1280, packed for the GEMM
        dict(name="search_block_w4", kind="search", d=1280, blocks=1, bits=4, ragged=0),
        # (group size, format) search of the DiT MLP from 2 x 4096 calibration rows
        dict(name="group_search_fc1", kind="group_search", M=8192, N=4608, K=1152, t=300),
        # moments of the inputs of two blocks' layers, and the LUT
        dict(name="calibrate_blocks", kind="calibrate", d=1280, M=2048, blocks=2, t=379),
        # a sampler step over one transformer block at width 640 (64 x 64 latents, CFG batch 2)
        dict(name="step_block_640", kind="step", d=640, M=8192, t=379),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear"] * 6 + ["grouped", "conv", "search", "group_search", "calibrate", "step"])
    t = rng.randrange(1000)
    if kind in ("linear", "grouped"):
        while True:
            M, N, K = _logint(rng, 200, 8192), _logint(rng, 320, 10240), 64 * _logint(rng, 10, 80)
            if M * N * K <= 8192 * 4608 * 1152:
                break
        samples = rng.choice([0, 1, 2]) if kind == "linear" else rng.choice([1, 2])
        M = max(2, M - M % max(1, samples))
        if kind == "grouped":
            return dict(kind=kind, M=M, N=N, K=K, act=rng.choice(["int8", "e4m3", "e5m2"]), samples=samples, t=t)
        act = rng.choice(["int8", "e4m3", "e5m2", "e4m3", "e5m2", "mxfp8", "mxint8"])
        return dict(kind=kind, M=M, N=N, K=K, bits=rng.choice([4, 4, 4, 8]), act=act, samples=samples,
                    packed=rng.random() < 0.8, t=t)
    if kind == "conv":
        H, W = rng.randrange(12, 41), rng.randrange(12, 41)
        return dict(kind=kind, B=rng.choice([1, 2]), H=H, W=W, C=64 * rng.randrange(8, 31), Co=32 * rng.randrange(10, 21) + rng.choice([0, 0, 3]),
                    bits=rng.choice([4, 4, 8]), act=rng.choice(["mxfp8", "mxfp8", "e4m3", "int8"]), t=t)
    if kind == "search":
        return dict(kind=kind, d=64 * rng.randrange(5, 21), blocks=1, bits=rng.choice([4, 4, 8]), ragged=rng.randrange(0, 40))
    if kind == "group_search":
        return dict(kind=kind, M=_logint(rng, 500, 8192), N=_logint(rng, 320, 4608), K=64 * rng.randrange(5, 19), t=t)
    if kind == "calibrate":
        return dict(kind=kind, d=64 * rng.randrange(5, 21), M=_logint(rng, 200, 2048), blocks=rng.choice([1, 2]), t=t)
    d = 64 * rng.randrange(5, 21)
    return dict(kind="step", d=d, M=_logint(rng, 256, max(300, min(8192, 8192 * 640 * 640 // (d * d)))), t=t)


def _mask(c):
    return W4 if c["bits"] == 4 else W8


def _block(c):
    """[(K, N)] of the layers of a search, calibration or step case; ragged takes some output
    channels off, as a pruned layer would have."""
    r = c.get("ragged", 0)
    return [(K, N - r) for _, K, N in synth.sdxl_block_layers(c["d"])] * c.get("blocks", 1)


def work(c):
    k = c["kind"]
    if k in ("linear", "grouped"):
        M, N, K, b = c["M"], c["N"], c["K"], c.get("bits", 4)
        return {"bytes": 4 * M * K + N * K * b / 8 + 4 * M * N, "flops": 2 * M * N * K}
    if k == "conv":
        M, K = c["B"] * c["H"] * c["W"], 9 * c["C"]
        return {"bytes": 4 * M * c["C"] + c["Co"] * K * c["bits"] / 8 + 4 * M * c["Co"], "flops": 2 * M * c["Co"] * K}
    if k == "search":
        n = sum(K * N for K, N in _block(c))
        f = 5 if c["bits"] == 4 else 3
        return {"bytes": n * (4 + c["bits"] / 8 + 0.09), "flops": n * f * 8}
    if k == "group_search":
        return {"bytes": 4 * c["M"] * c["K"] + c["N"] * c["K"] * 4.5 + c["N"] * c["K"] / 4,
                "flops": 2 * c["M"] * c["K"] + c["N"] * c["K"] * 15 * 8}
    n = sum(c["M"] * K for K, _ in _block(c))
    if k == "calibrate":
        return {"bytes": 4 * n, "flops": 9 * n}
    out = sum(c["M"] * N for _, N in _block(c))
    w = sum(K * N for K, N in _block(c))
    return {"bytes": 4 * n + 4 * out + n + w / 2, "flops": 2 * c["M"] * w + 9 * n}


def tolerance(c):
    """About four times the error measured against exact() (rounding levels to the GEMM's
    half-precision operand for 4-bit weights: 2e-4; binary32 sums for 8-bit weights: 1e-5)."""
    k = c["kind"]
    if k == "search":
        return "exact"
    if k == "calibrate":  # binary64 sums; the kurtosis amplifies their rounding
        return {"rel": 1e-9, "max": 1e-8, "differ": 0.0}
    if k == "group_search":  # binary64 sums, the energies rounded to binary32
        return {"rel": 2e-7, "max": 5e-7, "differ": 0.0}
    if c.get("bits", 4) == 8:
        return {"rel": 4e-5, "max": 4e-4, "differ": 0.0}
    return {"rel": 8e-4, "max": 6e-3, "differ": 0.0}


# ---------------------------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------------------------
def _seed(seed, *key):
    return int(np.random.SeedSequence([seed, *key]).generate_state(1)[0] >> 1)


def _acts(seed, layer, t, M, K, step=0):
    return synth.diffusion_acts_dev(_seed(seed, 1), layer, t, M, K, DEV, step)


def _weights(seed, layer, N, K):
    return synth.hetero_weights_dev(_seed(seed, 2, layer), N, K, DEV)


def _scale_zp(lo, hi, act):
    """ScaleZP of a range (binary32 0-d tensors)."""
    tiny = torch.finfo(torch.float32).tiny
    one, zero = torch.ones_like(lo), torch.zeros_like(lo)
    amax = torch.maximum(lo.abs(), hi.abs())
    if act == "int8":
        d = hi - lo
        flat = torch.where(lo != 0, lo.abs(), one)
        s = torch.where(d == 0, flat, _div(d, 255.0).clamp(min=tiny))
        return s, torch.round((-lo.double() / s.double()).float())
    if act == "e4m3":
        return _div(amax, 448.0).clamp(min=tiny), zero
    if act == "e5m2":
        return _div(amax, 57344.0).clamp(min=tiny), zero
    return one, zero


def _static(c, seed):
    """Static scale of a linear case: the range of a calibration batch of 256 rows."""
    cal = _acts(seed, 0, c["t"], 256, c["K"], step=1)
    s, z = _scale_zp(cal.min(), cal.max(), c["act"])
    return s.reshape(1), z.reshape(1)


def _lut_calibration(c, seed):
    """Calibration batches of a step's layers: (input, layer, bucket), 256 rows per bucket."""
    for layer, (K, _) in enumerate(_block(c)):
        for b in range(BUCKETS):
            t = (2 * b + 1) * 1000 // (2 * BUCKETS)
            yield _acts(seed, layer, t, 256, K, step=1), layer, b


def prepare(c, seed):
    k = c["kind"]
    st = {"case": c}
    if k in ("linear", "grouped"):
        M, N, K = c["M"], c["N"], c["K"]
        st["X"] = _acts(seed, 0, c["t"], M, K)
        st["aq"] = cham.alloc_aq(M, K, DEV, with_e8m0=c["act"].startswith("mx"), nsamples=max(1, c["samples"]))
        st["Y"] = torch.empty((M, N), dtype=torch.float32, device=DEV)
        W = _weights(seed, 0, N, K)
        if k == "grouped":
            energy = (_acts(seed, 0, c["t"], 256, K, step=2) ** 2).mean(0)
            st["wq"] = cham.select_group_formats(W, energy, want_packed=True)
        else:
            st["wq"] = cham.select_weight_formats(W, _mask(c), want_packed=c["packed"])
        if c["samples"] == 0:
            st["s"], st["z"] = _static(c, seed)
        # the workspaces that a serving program keeps
        st["ws_q"] = torch.empty(max(256, cham.workspace_bytes(cham.OP_QUANT_ACT, M, 0, K)), dtype=torch.uint8, device=DEV)
        st["ws"] = torch.empty(max(256, cham.workspace_bytes(cham.OP_LINEAR, M, N, K)), dtype=torch.uint8, device=DEV)
    elif k == "conv":
        M = c["B"] * c["H"] * c["W"]
        st["X"] = _acts(seed, 0, c["t"], M, c["C"])
        st["aq"] = cham.alloc_aq(M, c["C"], DEV, nsamples=1)
        st["wq"] = cham.select_weight_formats(_weights(seed, 0, c["Co"], 9 * c["C"]), _mask(c), want_packed=9 * c["C"] <= 8192)
        if 9 * c["C"] > 8192:
            st["wq"].packed = torch.empty(cham.packed_bytes(c["Co"], 9 * c["C"]), dtype=torch.uint8, device=DEV)
            cham.pack_weights_batch([st["wq"]])
        st["Y"] = torch.empty((M, c["Co"]), dtype=torch.float32, device=DEV)
        st["ws_q"] = torch.empty(max(256, cham.workspace_bytes(cham.OP_QUANT_ACT, M, 0, c["C"])), dtype=torch.uint8, device=DEV)
        nb = cham.lib().cham_conv3x3_workspace_bytes(c["B"], c["H"], c["W"], c["C"], c["Co"])
        st["ws"] = torch.empty(int(nb), dtype=torch.uint8, device=DEV)
    elif k == "search":
        st["Ws"] = [_weights(seed, i, N, K) for i, (K, N) in enumerate(_block(c))]
        st["outs"] = [cham.alloc_wq(W.shape[0], W.shape[1], _mask(c), DEV, want_packed=True) for W in st["Ws"]]
        st["batch"] = cham.SearchBatch(st["Ws"], st["outs"])
    elif k == "group_search":
        st["X"] = _acts(seed, 0, c["t"], c["M"], c["K"])
        st["W"] = _weights(seed, 0, c["N"], c["K"])
        st["colsq"] = torch.zeros(c["K"], dtype=torch.float64, device=DEV)
        st["gq"] = cham.alloc_gwq(c["N"], c["K"], DIT4, device=DEV, want_packed=True)
        st["ws_c"] = torch.empty(cham.workspace_bytes(cham.OP_COLSQ, c["M"], 0, c["K"]), dtype=torch.uint8, device=DEV)
        st["ws_g"] = torch.empty(cham.workspace_bytes(cham.OP_GSELECT, 0, c["N"], c["K"]), dtype=torch.uint8, device=DEV)
    elif k == "calibrate":
        lay = _block(c)
        st["Xs"] = [_acts(seed, i, c["t"], c["M"], K) for i, (K, _) in enumerate(lay)]
        st["stats"] = cham.alloc_stats(len(lay), BUCKETS, DEV)
        b = cham.bucket(c["t"], 1000, BUCKETS)
        st["batch"] = cham.StatsBatch(st["Xs"], range(len(lay)), [b] * len(lay), st["stats"])
        st["lut"] = _alloc_lut(len(lay))
    else:  # step
        lay = _block(c)
        cal = cham.alloc_stats(len(lay), BUCKETS, DEV)
        cham.act_stats_reset(cal)
        for X, layer, b in _lut_calibration(c, seed):
            cham.act_stats_accumulate(X, layer, b, cal)
        st["lut"] = cham.build_act_lut(cal).mirror()
        st["Xs"] = [_acts(seed, i, c["t"], c["M"], K) for i, (K, _) in enumerate(lay)]
        st["aqs"] = [cham.alloc_aq(c["M"], K, DEV) for K, _ in lay]
        st["wqs"] = cham.select_weight_formats_batch([_weights(seed, i, N, K) for i, (K, N) in enumerate(lay)], W4, want_packed=True)
        st["Ys"] = [torch.empty((c["M"], N), dtype=torch.float32, device=DEV) for _, N in lay]
        st["stats"] = cham.alloc_stats(len(lay), BUCKETS, DEV)
        st["quant"] = cham.QuantStatsBatch(st["Xs"], range(len(lay)), st["aqs"], st["lut"], st["stats"])
        st["next"] = _alloc_lut(len(lay))
        nb = max(cham.workspace_bytes(cham.OP_LINEAR, c["M"], N, K) for K, N in lay)
        st["ws"] = torch.empty(max(256, nb), dtype=torch.uint8, device=DEV)
    return st


def _alloc_lut(L):
    n = L * BUCKETS
    f32 = torch.float32
    return cham.LUT(L, BUCKETS, 1000, torch.empty(n, dtype=torch.uint8, device=DEV), torch.empty(n, dtype=f32, device=DEV),
                    torch.empty(n, dtype=f32, device=DEV), torch.empty(n, dtype=torch.float64, device=DEV))


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def _quantize(st):
    c = st["case"]
    ns = c.get("samples", 0)
    return cham.quantize_act(st["X"], ACT[c["act"]], dynamic=ns > 0 or c["kind"] == "conv", s=st.get("s"), z=st.get("z"),
                             out=st["aq"], ws=st["ws_q"], nsamples=max(1, ns))


def run(st):
    c = st["case"]
    k = c["kind"]
    if k == "linear":
        aq = _quantize(st)
        return {"Y": cham.mixed_linear(aq, st["wq"], st["Y"], st["ws"]), "codes": aq.codes}
    if k == "grouped":
        aq = _quantize(st)
        return {"Y": cham.mixed_linear_grouped(aq, st["wq"], st["Y"], st["ws"]), "codes": aq.codes}
    if k == "conv":
        aq = _quantize(st)
        return {"Y": cham.conv3x3_mixed(aq, c["B"], c["H"], c["W"], st["wq"], st["Y"], st["ws"]), "codes": aq.codes}
    if k == "search":
        st["batch"].run()
        return [{"fmt": o.fmt, "codes": o.codes, "scale": o.scale, "zero": o.zero, "absmax": o.nf4_absmax, "e8m0": o.e8m0,
                 "perm": o.perm, "group_off": o.group_off} for o in st["outs"]]
    if k == "group_search":
        st["colsq"].zero_()
        cham.act_colsq_accumulate(st["X"], st["colsq"], st["ws_c"])
        energy = (st["colsq"] / c["M"]).float()
        g = cham.select_group_formats(st["W"], energy, DIT4, out=st["gq"], ws=st["ws_g"])
        return {"energy": energy, "choice": g.choice, "fmt": g.fmt, "codes": g.codes, "gscale": g.gscale, "gzero": g.gzero, "err": g.err}
    if k == "calibrate":
        cham.act_stats_reset(st["stats"])
        st["batch"].run()
        lut = cham.build_act_lut(st["stats"], out=st["lut"])
        return _stats_out(st["stats"], lut)
    cham.act_stats_reset(st["stats"])
    st["quant"].run(c["t"])
    nxt = cham.build_act_lut(st["stats"], out=st["next"])
    Ys = [cham.mixed_linear(a, w, Y, st["ws"]) for a, w, Y in zip(st["aqs"], st["wqs"], st["Ys"])]
    return {"Y": Ys, "codes": [a.codes for a in st["aqs"]], **_stats_out(st["stats"], nxt)}


def _stats_out(s, lut):
    """Moments and LUT; the kurtosis of buckets without data is NaN, as defined."""
    return {"nS": s.nS, "lohi": s.lohi, "F": lut.F, "S": lut.S, "Z": lut.Z, "kappa": lut.kappa}


# ---------------------------------------------------------------------------------------------
# the same in plain torch: the formats' binary32 arithmetic, then binary64
# ---------------------------------------------------------------------------------------------
def _div(a, b):
    """Correctly rounded binary32 quotient."""
    return (a.double() / b).float()


def _rcp(s):
    return (1.0 / s.double()).float()


def _floor_log2(a):
    return torch.frexp(a)[1] - 1


def _mx_exp(amax, emax):
    return torch.where(amax > 0, (_floor_log2(amax) - emax).clamp(-127, 127), torch.full_like(amax, -127, dtype=torch.int32))


def _e2m1(y):
    a = y.abs()
    step = torch.where(a < 2, 0.5, torch.where(a < 4, 1.0, 2.0))
    return torch.copysign(torch.round(a / step) * step, y)


_NF4_BITS = (0xbf800000, 0xbf3239b1, 0xbf066b2e, 0xbeca329e, 0xbe91a24b, 0xbe3d353d, 0xbdba7869, 0x00000000, 0x3da2fb01,
             0x3e24cadf, 0x3e7c04da, 0x3ead0336, 0x3ee1a4b5, 0x3f1007a9, 0x3f3913b0, 0x3f800000)


def _nf4(y):
    lv = torch.tensor(np.array(_NF4_BITS, dtype=np.uint32).view(np.float32), device=y.device)
    mid = (lv[:-1].double() + lv[1:].double()) / 2
    return lv[torch.bucketize(y.double(), mid)]


def _group_quant(W, f):
    """Reconstruction (binary64), scale and zero point of W [..., g] in format f, with one set of
    parameters for the last dimension (an MX format: its block)."""
    tiny = torch.finfo(torch.float32).tiny
    lo, hi = W.amin(-1, keepdim=True), W.amax(-1, keepdim=True)
    amax = torch.maximum(lo.abs(), hi.abs())
    zero = torch.zeros_like(lo)
    if f in (cham.W_INT8_SYM, cham.W_INT4_SYM):
        Q = 127.0 if f == cham.W_INT8_SYM else 7.0
        s = _div(amax, Q).clamp(min=tiny)
        return torch.round(W * _rcp(s)).clamp(-Q, Q) * s, s, zero
    if f in (cham.W_INT8_ASYM, cham.W_INT4_ASYM):
        L = 255.0 if f == cham.W_INT8_ASYM else 15.0
        d = hi - lo
        s = torch.where(d == 0, torch.where(lo != 0, lo.abs(), torch.ones_like(lo)), _div(d, L).clamp(min=tiny))
        z = torch.round((-lo.double() / s.double()).float())
        return (((torch.round(W * _rcp(s)) + z).clamp(0.0, L)) - z) * s, s, z
    if f == cham.W_FP4:
        s = _div(amax, 6.0).clamp(min=tiny)
        return _e2m1((W * _rcp(s)).clamp(-6.0, 6.0)) * s, s, zero
    if f == cham.W_NF4:
        s = amax.clamp(min=tiny)
        return _nf4(W * _rcp(s)) * s, s, zero
    E = _mx_exp(amax, 2 if f == cham.W_MXFP4 else 0)
    if f == cham.W_MXFP4:
        return torch.ldexp(_e2m1(torch.ldexp(W.double(), -E).clamp(-6.0, 6.0)), E).float(), zero, zero
    F, Q = (6, 127.0) if f == cham.W_MXINT8 else (2, 7.0)
    return torch.ldexp(torch.round(torch.ldexp(W.double(), F - E)).clamp(-Q, Q), E - F).float(), zero, zero


def _search(W, mask):
    """Per channel: the format of the smallest squared error, its reconstruction and scales."""
    N, K = W.shape
    best = torch.full((N,), math.inf, dtype=torch.float64, device=W.device)
    fmt = torch.zeros(N, dtype=torch.int64, device=W.device)
    Wh = torch.zeros_like(W)
    scale, zero = torch.zeros(N, device=W.device), torch.zeros(N, device=W.device)
    absmax = torch.zeros((N, K // 64), device=W.device) if mask >> cham.W_NF4 & 1 else None
    for f in range(9):
        if not mask >> f & 1:
            continue
        mx = f in (cham.W_MXINT8, cham.W_MXINT4, cham.W_MXFP4)
        g = 64 if f == cham.W_NF4 else 32 if mx else K
        h, s, z = _group_quant(W.reshape(N, K // g, g), f)
        h = h.reshape(N, K)
        e = (W.double() - h.double()).square().sum(1)
        take = e < best
        best, fmt = torch.where(take, e, best), torch.where(take, f, fmt)
        Wh[take] = h[take]
        scalar = f not in (cham.W_NF4, cham.W_MXINT8, cham.W_MXINT4, cham.W_MXFP4)
        scale[take] = s.reshape(N, -1)[take, 0] if scalar else 0.0
        zero[take] = z.reshape(N, -1)[take, 0] if scalar else 0.0
        if absmax is not None:
            absmax[take] = s.reshape(N, -1)[take] if f == cham.W_NF4 else 0.0
    return fmt, Wh.double(), scale, zero, absmax


def _groups(W, f, g):
    """Group-scaled reconstruction and parameters [N, ceil(K / g)] (the last group may be short)."""
    N, K = W.shape
    k0 = K // g * g
    parts = [_group_quant(W[:, :k0].reshape(N, -1, g), f)] if k0 else []
    parts += [_group_quant(W[:, None, k0:], f)] if k0 < K else []
    h = torch.cat([p[0].reshape(N, -1) for p in parts], 1)
    return h.double(), torch.cat([p[1][..., 0] for p in parts], 1), torch.cat([p[2][..., 0] for p in parts], 1)


def _group_search(W, energy):
    err = torch.full((45,), -1.0, dtype=torch.float64, device=W.device)
    best, pick = math.inf, None
    for gi, g in enumerate(cham.GROUP_SIZES):
        for f in (cham.W_INT4_ASYM, cham.W_NF4, cham.W_FP4):
            h, _, _ = _groups(W, f, g)
            d = (W - h.float()).double()  # the difference of two binary32 values, in binary32
            err[gi * 9 + f] = e = (d.square() * energy.double()).sum()
            if float(e) < best:
                best, pick = float(e), (g, f)
    g, f = pick
    h, s, z = _groups(W, f, g)
    return err, pick, h, s, z


def _dequant_act(X, act, s, z):
    """Binary64 values of X [M, K] quantized with scale and zero point (broadcast over X)."""
    if act.startswith("mx"):
        B = X.reshape(X.shape[0], -1, 32)
        E = _mx_exp(B.abs().amax(-1, keepdim=True), 0)
        y = torch.ldexp(B.double(), -E)
        if act == "mxfp8":
            q = y.float().clamp(-448.0, 448.0).to(torch.float8_e4m3fn).double()
        else:
            q = torch.round(y * 64.0).clamp(-127.0, 127.0) / 64.0
        return torch.ldexp(q, E).reshape(X.shape)
    y = X * _rcp(s)
    if act == "int8":
        return ((torch.round(y) + z).clamp(0.0, 255.0).double() - z.double()) * s.double()
    m, dt = (448.0, torch.float8_e4m3fn) if act == "e4m3" else (57344.0, torch.float8_e5m2)
    return y.clamp(-m, m).to(dt).double() * s.double()


def _dequant_case(X, c, seed):
    if c["kind"] != "conv" and c["samples"] == 0:
        s, z = _static(c, seed)
        return _dequant_act(X, c["act"], s, z)
    halves = X.chunk(max(1, c.get("samples", 1)))
    return torch.cat([_dequant_act(h, c["act"], *_scale_zp(h.min(), h.max(), c["act"])) for h in halves])


def _moments(X):
    d = X.double().reshape(-1)
    return torch.stack([torch.tensor(float(d.numel()), dtype=torch.float64, device=DEV), d.sum(), (d ** 2).sum(), (d ** 3).sum(),
                        (d ** 4).sum()]), torch.stack([X.min(), X.max()])


def _route(nS, lohi):
    """(F, S, Z, kappa) of the accumulators [L * BUCKETS] under the default schedule."""
    r = np.sqrt(0.00085) + (np.sqrt(0.012) - np.sqrt(0.00085)) * np.arange(1000) / 999.0
    abar = np.cumprod(1.0 - r * r)
    n, s1, s2, s3, s4 = nS.unbind(1)
    mu, e2, e3, e4 = s1 / n, s2 / n, s3 / n, s4 / n
    m2 = e2 - mu * mu
    kap = (e4 - 4.0 * mu * e3 + 6.0 * mu * mu * e2 - 3.0 * mu ** 4) / (m2 * m2)
    F, S, Z = [], [], []
    for i, kp in enumerate(kap.tolist()):
        a = abar[(2 * (i % BUCKETS) + 1) * 1000 // (2 * BUCKETS)]
        snr = a / (1.0 - a)
        f = "e5m2" if kp > 5.0 or snr < 0.2 else "int8" if kp <= 3.0 and snr > 2.0 else "e4m3"
        s, z = _scale_zp(lohi[i, 0], lohi[i, 1], f if float(n[i]) else "none")
        F.append(f)
        S.append(s)
        Z.append(z)
    return F, torch.stack(S).double(), torch.stack(Z).double(), kap


def _empty_stats(L):
    nS = torch.zeros((L * BUCKETS, 5), dtype=torch.float64, device=DEV)
    return nS, torch.tensor([math.inf, -math.inf], device=DEV).repeat(L * BUCKETS, 1)


def _exact_stats(Xs, t):
    nS, lohi = _empty_stats(len(Xs))
    b = min(t * BUCKETS // 1000, BUCKETS - 1)
    for i, X in enumerate(Xs):
        nS[i * BUCKETS + b], lohi[i * BUCKETS + b] = _moments(X)
    _, S, Z, kap = _route(nS, lohi)
    return {"nS": nS, "lohi": lohi.double(), "F": None, "S": S, "Z": Z, "kappa": kap}


def exact(c, seed):
    k = c["kind"]
    if k in ("linear", "grouped"):
        W = _weights(seed, 0, c["N"], c["K"])
        if k == "grouped":
            Wh = _group_search(W, (_acts(seed, 0, c["t"], 256, c["K"], step=2) ** 2).mean(0))[2]
        else:
            Wh = _search(W, _mask(c))[1]
        return {"Y": _dequant_case(_acts(seed, 0, c["t"], c["M"], c["K"]), c, seed) @ Wh.T, "codes": None}
    if k == "conv":
        B, H, Wd, C, Co = c["B"], c["H"], c["W"], c["C"], c["Co"]
        Wh = _search(_weights(seed, 0, Co, 9 * C), _mask(c))[1]
        X = _dequant_case(_acts(seed, 0, c["t"], B * H * Wd, C), c, seed).reshape(B, H, Wd, C)
        P = torch.zeros((B, H + 2, Wd + 2, C), dtype=torch.float64, device=DEV)
        P[:, 1:-1, 1:-1] = X
        Y = torch.zeros((B * H * Wd, Co), dtype=torch.float64, device=DEV)
        for tap in range(9):
            y, x = divmod(tap, 3)
            Y += P[:, y:y + H, x:x + Wd].reshape(-1, C) @ Wh[:, tap * C:(tap + 1) * C].T
        return {"Y": Y, "codes": None}
    if k == "search":
        out = []
        for i, (K, N) in enumerate(_block(c)):
            _, _, s, z, a = _search(_weights(seed, i, N, K), _mask(c))
            out.append({"fmt": None, "codes": None, "scale": s.double(), "zero": z.double(),
                        "absmax": None if a is None else a.double(), "e8m0": None, "perm": None, "group_off": None})
        return out
    if k == "group_search":
        X = _acts(seed, 0, c["t"], c["M"], c["K"])
        e = X.double().square().sum(0) / c["M"]
        err, (g, f), _, s, z = _group_search(_weights(seed, 0, c["N"], c["K"]), e.float())
        pad = (0, c["K"] // 32 - s.shape[1])
        return {"energy": e, "choice": None, "fmt": None, "codes": None, "gscale": torch.nn.functional.pad(s, pad).double(),
                "gzero": torch.nn.functional.pad(z, pad).double(), "err": err}
    lay = _block(c)
    Xs = [_acts(seed, i, c["t"], c["M"], K) for i, (K, _) in enumerate(lay)]
    if k == "calibrate":
        return _exact_stats(Xs, c["t"])
    nS, lohi = _empty_stats(len(lay))
    for X, layer, b in _lut_calibration(c, seed):
        nS[layer * BUCKETS + b], lohi[layer * BUCKETS + b] = _moments(X)
    F, S, Z, _ = _route(nS, lohi)
    Ys = []
    b = min(c["t"] * BUCKETS // 1000, BUCKETS - 1)
    for i, (K, N) in enumerate(lay):
        j = i * BUCKETS + b
        Ys.append(_dequant_act(Xs[i], F[j], S[j].float(), Z[j].float()) @ _search(_weights(seed, i, N, K), W4)[1].T)
    return {"Y": Ys, "codes": [None] * len(lay), **_exact_stats(Xs, c["t"])}
