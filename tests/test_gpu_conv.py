"""GPU parity of the UNet path's 3x3 convolution on quantized activations (implicit GEMM,
stride 1, zero padding 1, channels last): every activation format, W4 and W8 weights,
ragged rows and channels, against the oracle's convolution; and an SDXL-like up-block
resnet conv1 fed by a shortcut concatenation, whose LUT entry is pinned to MXFP8 (Sec. 4.6),
on sampled outputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_33496_amd import cham, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def case(msg):
    print(f"[case] {msg}", flush=True)


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("mask", [oracle.MASK_W4, oracle.MASK_W8])
def test_conv3x3_small_every_format(mask):
    B, H, W, C, Co = 2, 5, 7, 64, 96
    g = np.random.default_rng(1)
    X = (g.standard_t(4, (B, H, W, C)) * np.exp(g.normal(0, 1, (1, 1, 1, C)))).astype(np.float32)
    Wt, _ = synth.hetero_weights(2, Co, 9 * C)
    wq = cham.select_weight_formats(torch.from_numpy(Wt).to(DEV), mask)
    wp = cham.select_weight_formats(torch.from_numpy(Wt).to(DEV), mask, want_packed=True)
    ref = oracle.select_weight_formats(Wt, mask, want_err=False, want_perm=False)
    Wh = oracle.dequant_weights(ref, 9 * C)
    for fmt in range(5):
        for ns in (1, B):
            case(f"conv3x3 B={B} H={H} W={W} C={C} Co={Co} mask={mask:#x} fmt={fmt} nsamples={ns}")
            xq = cham.quantize_act(torch.from_numpy(X.reshape(-1, C)).to(DEV), fmt, dynamic=True, nsamples=ns)
            Y = _np(cham.conv3x3_mixed(xq, B, H, W, wq)).astype(np.float64)
            Yp = _np(cham.conv3x3_mixed(xq, B, H, W, wp)).astype(np.float64)
            _, _, xh, _, _ = oracle.quantize_act_per_sample(X.reshape(-1, C), fmt, ns, want_xhat=True)
            Yr, Bm = oracle.conv3x3(xh.reshape(B, H, W, C), Wh)
            rel = np.abs(Y - Yr.reshape(-1, Co)) / np.maximum(Bm.reshape(-1, Co), 1e-300)
            assert rel.max() <= 1e-3, (fmt, ns, rel.max())
            assert np.array_equal(Y, Yp)


def test_conv3x3_shortcut_conv1_mxfp8_sampled():
    """An SDXL-like up-block resnet conv1 on a shortcut concatenation (1280 + 640 -> 640
    channels at 32 x 32, CFG batch 2): the LUT routes its input to MXFP8 in every bucket,
    the W4 weights are searched per channel, and sampled outputs match the oracle."""
    B, H, W, C, Co = 2, 32, 32, 1920, 640
    L, Bk = 2, 4
    st = cham.alloc_stats(L, Bk, DEV)
    cham.act_stats_reset(st)
    for b in range(Bk):
        for l in range(L):
            cham.act_stats_accumulate(torch.from_numpy(synth.diffusion_acts(3, l, 125 + 250 * b, 64, C)).to(DEV), l, b, st)
    lut = cham.build_act_lut(st, is_shortcut=torch.tensor([0, 1], dtype=torch.uint8, device=DEV)).mirror()
    assert np.all(lut.F_host.numpy().reshape(L, Bk)[1] == cham.A_MXFP8)
    X = synth.diffusion_acts(4, 1, 600, B * H * W, C)
    X[:, 1280:] *= np.float32(8.0)  # the concatenated skip half on another scale: wide tails
    xq = cham.quantize_act_lut(torch.from_numpy(X).to(DEV), lut, 1, 600)
    assert xq.fmt == cham.A_MXFP8
    Wt, _ = synth.hetero_weights(5, Co, 9 * C)
    wq = cham.select_weight_formats(torch.from_numpy(Wt).to(DEV), cham.MASK_W4, want_packed=True)
    case(f"conv3x3 shortcut conv1 B={B} H={H} W={W} C={C} Co={Co} MXFP8")
    Y = _np(cham.conv3x3_mixed(xq, B, H, W, wq))
    codes, e8, xh = oracle.quantize_act(X, oracle.A_MXFP8, want_xhat=True)
    assert np.array_equal(_np(xq.codes), codes)
    g = np.random.default_rng(6)
    S = 1500
    pix = g.integers(0, B * H * W, S)
    pix[:4] = [0, W - 1, H * W - 1, B * H * W - W]  # corners: padding on two sides
    nn = g.integers(0, Co, S)
    chans = np.unique(nn)
    ref = oracle.select_weight_formats(Wt[chans], cham.MASK_W4, want_err=False, want_perm=False)
    Wh = np.zeros((Co, 9 * C), np.float32)
    Wh[chans] = oracle.dequant_weights(ref, 9 * C)
    xp = np.zeros((B, H + 2, W + 2, C), np.float32)
    xp[:, 1:-1, 1:-1] = xh.reshape(B, H, W, C)
    b, rem = pix // (H * W), pix % (H * W)
    y, x = rem // W, rem % W
    cols = np.concatenate([xp[b, y + ky, x + kx] for ky in range(3) for kx in range(3)], axis=1)
    Yr, Bm = oracle.linear_pairs(cols, Wh, np.arange(S), nn)
    rel = np.abs(Y[pix, nn].astype(np.float64) - Yr) / np.maximum(Bm, 1e-300)
    assert rel.max() <= 1e-3, rel.max()


@pytest.mark.parametrize("fmt", [cham.A_MXFP8, cham.A_MXINT8, cham.A_INT8_ASYM])
@pytest.mark.parametrize("B,H,W,C,Co", [(1, 1, 1, 64, 5), (3, 1, 40, 128, 33), (2, 13, 3, 64, 130), (1, 20, 20, 192, 320),
                                         (2, 3, 300, 64, 40), (1, 1, 3100, 64, 5), (1, 2, 3072, 64, 3)])
def test_conv3x3_codes_decoded_while_staged(fmt, B, H, W, C, Co):
    """Images of one pixel, one line and narrow ones (tiles that straddle lines and images), lines
    longer than a tile, a k-split; block scales 2^24 apart within and between images; and zero points within and
    beyond +-1024 in one batch (INT8-asym), with the padding at zero for all."""
    g = np.random.default_rng(B + H + W + C)
    X = g.standard_t(4, (B, H, W, C)).astype(np.float32)
    if fmt == cham.A_INT8_ASYM:
        X[-1] = np.float32(300.0) + np.abs(X[-1]) / np.abs(X[-1]).max()  # last image: z about -76500
    else:
        X *= np.exp2(g.integers(-12, 13, (B, H, W, C // 32))).repeat(32, axis=3).astype(np.float32)
    Wt, _ = synth.hetero_weights(2, Co, 9 * C)
    wp = cham.select_weight_formats(torch.from_numpy(Wt).to(DEV), cham.MASK_W4, want_packed=True)
    ref = oracle.select_weight_formats(Wt, cham.MASK_W4, want_err=False, want_perm=False)
    case(f"conv3x3 staged decode B={B} H={H} W={W} C={C} Co={Co} fmt={fmt}")
    xq = cham.quantize_act(torch.from_numpy(X.reshape(-1, C)).to(DEV), fmt, dynamic=True, nsamples=B)
    Y = _np(cham.conv3x3_mixed(xq, B, H, W, wp)).astype(np.float64)
    _, _, xh, _, _ = oracle.quantize_act_per_sample(X.reshape(-1, C), fmt, B, want_xhat=True)
    Yr, Bm = oracle.conv3x3(xh.reshape(B, H, W, C), oracle.dequant_weights(ref, 9 * C))
    # 2^-11 per half-precision weight and, beyond +-1024, activation
    rel = np.abs(Y - Yr.reshape(-1, Co)) / np.maximum(Bm.reshape(-1, Co), 1e-300)
    assert rel.max() <= 1e-3, rel.max()


def test_conv3x3_int8_zero_point_with_a_fraction():
    """INT8-asym codes of another quantizer, whose zero point is no integer: q - z in binary32,
    rounded to half precision (2^-11 of it, beside 2^-11 of the weight: 1e-3 of the sum)."""
    B, H, W, C, Co = 2, 6, 5, 64, 40
    g = np.random.default_rng(11)
    codes = g.integers(0, 256, (B * H * W, C)).astype(np.uint8)
    s, z = np.array([0.02, 0.03], np.float32), np.array([127.375, 0.625], np.float32)
    Wt = np.abs(synth.hetero_weights(2, Co, 9 * C)[0])  # an error of z does not cancel over a channel
    wq = cham.select_weight_formats(torch.from_numpy(Wt).to(DEV), cham.MASK_W4, want_packed=True)
    Wh = oracle.dequant_weights(oracle.select_weight_formats(Wt, cham.MASK_W4, want_err=False, want_perm=False), 9 * C)
    aq = cham.AQ(B * H * W, C, cham.A_INT8_ASYM, torch.from_numpy(codes).to(DEV), None, torch.from_numpy(s).to(DEV),
                 torch.from_numpy(z).to(DEV), B)
    case(f"conv3x3 fractional zero points B={B} H={H} W={W} C={C} Co={Co}")
    Y = _np(cham.conv3x3_mixed(aq, B, H, W, wq)).astype(np.float64)
    xh = ((codes.reshape(B, -1).astype(np.float32) - z[:, None]) * s[:, None]).reshape(B, H, W, C)
    Yr, Bm = oracle.conv3x3(xh, Wh)
    rel = np.abs(Y - Yr.reshape(-1, Co)) / np.maximum(Bm.reshape(-1, Co), 1e-300)
    assert rel.max() <= 1e-3, rel.max()


T256, T128, T64 = (128, 256), (128, 128), (64, 128)


@pytest.mark.parametrize("B,H,W,C,Co,mask,tile,splits", [
    (2, 37, 41, 64, 4100, oracle.MASK_W4, T256, 1),
    (2, 50, 41, 64, 3333, oracle.MASK_W8, T256, 1),
    (2, 45, 41, 64, 2600, oracle.MASK_W4, T128, 1),
    (2, 20, 20, 448, 1290, oracle.MASK_W4, T128, 3),
    (2, 37, 41, 64, 777, oracle.MASK_W8, T64, 1),
])
@pytest.mark.parametrize("fmt", [cham.A_INT8_ASYM, cham.A_FP8_E4M3, cham.A_MXFP8, cham.A_MXINT8])
def test_conv3x3_tiles_sampled(B, H, W, C, Co, mask, tile, splits, fmt):
    """Every tile shape (the plan is the one named, on 256 CUs) with ragged rows and channels, a
    k-split; INT8-asym with one image's zero point within +-1024 and the other's beyond; block scales
    2^16 apart: sampled outputs, corners among them, against the oracle one by one."""
    M, K = B * H * W, 9 * C
    plan = cham.linear_plan(M, Co, K, 8 if mask == oracle.MASK_W8 else 4)
    assert [x["tile"] for x in plan["launches"]] == [tile] and plan["splits"] == splits, plan
    g = np.random.default_rng(M + Co)
    X = g.standard_t(4, (B, H * W * C)).astype(np.float32)
    if fmt == cham.A_INT8_ASYM:
        X[1] = np.float32(30.0) + X[1] / np.abs(X[1]).max()
    X = X.reshape(M, C)
    if fmt in (cham.A_MXFP8, cham.A_MXINT8):
        X *= np.exp2(g.integers(-8, 9, (M, C // 32))).repeat(32, axis=1).astype(np.float32)
    Wt, _ = synth.hetero_weights(8, Co, K)
    case(f"conv3x3 tiles B={B} H={H} W={W} C={C} Co={Co} mask={mask:#x} fmt={fmt}")
    wq = cham.select_weight_formats(torch.from_numpy(Wt).to(DEV), mask, want_packed=True)
    xq = cham.quantize_act(torch.from_numpy(X).to(DEV), fmt, dynamic=True, nsamples=B)
    Y = _np(cham.conv3x3_mixed(xq, B, H, W, wq))
    _, _, xh, _, z = oracle.quantize_act_per_sample(X, fmt, B, want_xhat=True)
    assert fmt != cham.A_INT8_ASYM or (abs(z[0]) < 1024 < abs(z[1]))
    S = 1200
    pix, nn = g.integers(0, M, S), g.integers(0, Co, S)
    pix[:4] = [0, W - 1, H * W - 1, M - W]  # corners: padding on two sides
    nn[4:6] = [Co - 1, 0]
    pix[6:8] = [M - 1, 0]
    chans = np.unique(nn)
    Wh = np.zeros((Co, K), np.float32)
    Wh[chans] = oracle.dequant_weights(oracle.select_weight_formats(Wt[chans], mask, want_err=False, want_perm=False), K)
    xp = np.zeros((B, H + 2, W + 2, C), np.float32)
    xp[:, 1:-1, 1:-1] = xh.reshape(B, H, W, C)
    b, rem = pix // (H * W), pix % (H * W)
    y, x = rem // W, rem % W
    cols = np.concatenate([xp[b, y + ky, x + kx] for ky in range(3) for kx in range(3)], axis=1)
    Yr, Bm = oracle.linear_pairs(cols, Wh, np.arange(S), nn)
    # 2^-11 per half-precision weight and, beyond +-1024, activation
    rel = np.abs(Y[pix, nn].astype(np.float64) - Yr) / np.maximum(Bm, 1e-300)
    assert rel.max() <= 1e-3, rel.max()
