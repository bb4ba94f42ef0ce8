"""GPU parity of the HIP path against the CPU oracle, through the C ABI.

Acceptance (readings of the paper's Sec. 3.4):
  * weight codes/scales and norm codes/scales: bit-exact;
  * fused SwiGLU re-quantization: bit-exact on the kernel's own fp32 h;
  * gate/up against the independent oracle (exact fp64 products): the
    kernel's fp32 h equals, element by element, SwiGLU of the oracle's
    operands under the measured model of the FP8 MFMA's accumulation
    (tests/mfma_model.c, itself checked against the hardware below) within a
    derived fp32 tolerance; every scale and code is explained by that h; the
    code mismatch fraction against the oracle is capped, every mismatch is
    one e4m3 step, and the scale ratio is capped (gpu_util.check_gateup_model);
  * down projection on the same operands: max row-normalised error <= 2e-3,
    bf16 store = RNE of the fp32 result, and the fp32 result within the MFMA
    model's tolerance element by element;
  * determinism: repeated calls give identical bytes;
  * no write lands outside an output or workspace (guard regions).
Full-size workloads run the whole GPU call and compare sampled rows (the FFN
is row-independent, so a row subset is an exact check).
"""

import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle.ffn as O
import paper_2607_16339_amd as lc
import synth
import mfma_model as MM
from gpu_util import (DEV, Layer, check_down_model, check_down_same_operands, check_gateup_explained,
                      check_gateup_model, check_norm_exact, check_requant_exact, dev_bf16, host, host_bf16,
                      mfma_dot_bound, run_stages)
from oracle import csweep
from oracle.bf16 import bf16_to_f32, rne_bf16

pytestmark = pytest.mark.gpu

TINY = synth.WORKLOADS["tiny_m64_h256_i768"]
BLOCK32 = synth.WORKLOADS["block32_h4096_i12288"]
SAR512 = synth.WORKLOADS["sar512_h4096_i12288"]
BATCH8K = synth.WORKLOADS["batch8x1024_h4096_i12288"]
STACK = synth.WORKLOADS["stack31_m512_h4096_i12288"]


def _say(msg):
    print(msg, flush=True)


@pytest.fixture(autouse=True)
def _auto_policy():
    prev = lc.lacache_set_path_policy(0)
    yield
    lc.lacache_set_path_policy(prev)


@pytest.fixture(scope="module")
def big_layer():
    return Layer(BLOCK32, layer=1)


# ---------------------------------------------------------------------------
# e4m3 encoder
# ---------------------------------------------------------------------------

def test_device_encoder_all_fp32_patterns():
    """The device encoder against the oracle's C encoder on all 2^32 patterns."""
    csweep.build_csweep()
    chunk = 1 << 28
    sub = 1 << 24
    codes = torch.empty(chunk, dtype=torch.uint8, device=DEV)
    total = 0
    firsts = []
    with ThreadPoolExecutor(max_workers=16) as ex:
        for c in range((1 << 32) // chunk):
            start = c * chunk
            bits = torch.arange(start, start + chunk, dtype=torch.int64, device=DEV).to(torch.int32)
            lc.lacache_encode_e4m3(bits.view(torch.float32), codes)
            h = codes.cpu().numpy()
            res = list(ex.map(lambda i: csweep.sweep_check(h[i * sub:(i + 1) * sub], start + i * sub),
                              range(chunk // sub)))
            total += sum(b for b, _ in res)
            firsts += [hex(f) for b, f in res if b]
            del bits
    assert total == 0, firsts[:4]


def test_device_encoder_ragged_lengths():
    for n in (1, 3, 5, 1027):
        v = torch.linspace(-500, 500, n, dtype=torch.float32, device=DEV)
        c = torch.full((n,), 0xAA, dtype=torch.uint8, device=DEV)
        lc.lacache_encode_e4m3(v, c)
        assert np.array_equal(host(c), csweep.encode_f32(host(v)))


# ---------------------------------------------------------------------------
# the FP8 MFMA's dot-product error model that the GEMM tolerances rest on
# ---------------------------------------------------------------------------

def _unit_scale_dot(A, B):
    """GPU result of every 128-term dot product A[m] . B[n] (unit scales)."""
    M, N = A.shape[0], B.shape[0]
    lc.lacache_set_path_policy(2)
    out = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    tap = torch.empty((M, N), dtype=torch.float32, device=DEV)
    # B is the weight argument: its codes go in the weight tile layout
    lc.lacache_down_proj(torch.from_numpy(A).to(DEV), torch.ones((1, M), device=DEV),
                         torch.from_numpy(lc.weight_codes_tiled(B)).to(DEV), torch.ones((N // 128, 1), device=DEV),
                         out, tap)
    torch.cuda.synchronize()
    return host(tap).astype(np.float64)


def test_mfma_error_model_holds():
    """|P_gpu - P_exact| <= chunk-truncation bound + fp32 rounding, on random and adversarial codes."""
    rng = np.random.default_rng(11)
    cases = []
    for lo, hi in ((0x00, 0x7E), (0x30, 0x50), (0x01, 0x3F)):
        a = rng.integers(lo, hi + 1, (64, 128)).astype(np.uint8) | (rng.integers(0, 2, (64, 128)).astype(np.uint8) << 7)
        b = rng.integers(lo, hi + 1, (256, 128)).astype(np.uint8) | (rng.integers(0, 2, (256, 128)).astype(np.uint8) << 7)
        cases.append((a, b))
    a = np.full((64, 128), 0x08, np.uint8)  # many small terms ...
    a[:, ::8] = 0x7E                        # ... sharing each chunk with a large one
    b = np.full((256, 128), 0x38, np.uint8)
    b[::3, :] = 0x7E
    cases.append((a, b))
    worst = 0.0
    for a, b in cases:
        got = _unit_scale_dot(a, b)
        exact = O.dequant_codes(a) @ O.dequant_codes(b).T
        bound = mfma_dot_bound(a, b)[0] + np.spacing(np.abs(exact).astype(np.float32)).astype(np.float64)
        err = np.abs(got - exact)
        assert np.all(err <= bound), float((err / bound).max())
        worst = max(worst, float((err / bound).max()))
    _say("MFMA error / model bound: worst %.3f" % worst)


def _mfma_model_cases():
    """Seeded operand sets: random codes over several ranges, probes of the
    chunk width and the cut (one large term among small ones), cancellation
    between chunks, and quantized normal rows like the FFN's operands."""
    rng = np.random.default_rng(2026)

    def rnd(lo, hi, shape):
        return rng.integers(lo, hi + 1, shape).astype(np.uint8) | (rng.integers(0, 2, shape).astype(np.uint8) << 7)

    def qnormal(shape, outl=0.0):
        v = rng.standard_normal(shape)
        if outl:
            v[:, rng.choice(shape[1], max(1, int(outl * shape[1])), replace=False)] *= 40
        from oracle.e4m3 import e4m3_encode
        return e4m3_encode((v / (np.abs(v).max(axis=1, keepdims=True) / 448)).astype(np.float32))

    cases = [(rnd(0x00, 0x7E, (128, 128)), rnd(0x00, 0x7E, (256, 128))),
             (rnd(0x30, 0x50, (128, 128)), rnd(0x30, 0x50, (256, 128))),
             (rnd(0x01, 0x3F, (128, 128)), rnd(0x01, 0x3F, (256, 128)))]
    a = np.full((128, 128), 0x08, np.uint8)
    a[np.arange(128), np.arange(128)] = 0x7E
    cases.append((a, np.full((128, 128), 0x38, np.uint8)))
    a = np.zeros((128, 128), np.uint8)
    a[:, 0] = 0x7E
    a[:, 1] = np.arange(128, dtype=np.uint8)
    a[127, 1] = 0
    a[64:, 1] |= 0x80
    cases.append((a, np.full((128, 128), 0x38, np.uint8)))
    a = rnd(0x01, 0x10, (128, 128))
    a[:, 0:8] = rnd(0x70, 0x7E, (128, 8))
    b = rnd(0x01, 0x10, (256, 128))
    b[:, 0:8] = rnd(0x70, 0x7E, (256, 8))
    cases.append((a, b))
    cases.append((qnormal((128, 128), 0.01), qnormal((256, 128))))
    return cases


def test_mfma_model_matches_hardware():
    """The MFMA model that the gate/up and down tolerances come from, against
    the hardware's unit-scale dot products: |P_gpu - P_model| <= 2^(Eg - 19)
    plus half an fp32 ulp, and on quantized normal operands (the FFN's)
    P_gpu == fp32(P_model) exactly."""
    exact = []
    for i, (a, b) in enumerate(_mfma_model_cases()):
        got = _unit_scale_dot(a, b)
        P, D = MM.dots(a, b)
        tol = D + np.spacing(np.abs(P).astype(np.float32)).astype(np.float64) / 2
        err = np.abs(got - P)
        assert np.all(err <= tol), (i, float((err / tol).max()))
        exact.append(float((got == P.astype(np.float32)).mean()))
    assert exact[-1] == 1.0, exact
    _say("MFMA model: fraction of bit-exact dot products per case %s" % exact)


# ---------------------------------------------------------------------------
# weight quantization (128x128 blocks)
# ---------------------------------------------------------------------------

def test_quant_weights_tiny_and_special_blocks():
    lay = Layer(TINY, layer=1)
    wq, ws = O.quant_weights(lay.wgu_bits)
    assert np.array_equal(lc.weight_codes_rowmajor(lay.wgu_q), wq) and np.array_equal(host(lay.wgu_s).view(np.uint32), ws.view(np.uint32))
    wq, ws = O.quant_weights(lay.bits["w_down"])
    assert np.array_equal(lc.weight_codes_rowmajor(lay.wd_q), wq) and np.array_equal(host(lay.wd_s).view(np.uint32), ws.view(np.uint32))
    # special blocks: zeros, negative zeros, bf16 subnormals, huge values, a single spike
    rng = np.random.default_rng(0)
    w = (rng.standard_normal((256, 384)) * 0.02).astype(np.float32)
    w[0:128, 0:128] = 0.0
    w[0:128, 128:256] = -0.0
    w[128:256, 0:128] = rng.standard_normal((128, 128)) * 1e-39
    w[128:256, 128:256] = rng.standard_normal((128, 128)) * 1e37
    w[0:128, 256:384] *= 1e-3
    w[5, 300] = 3.0
    bits = torch.from_numpy(w).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    gq, gs = lc.quantize_weights(dev_bf16(bits))
    wq, ws = O.quant_weights(bits)
    assert np.array_equal(lc.weight_codes_rowmajor(gq), wq) and np.array_equal(host(gs).view(np.uint32), ws.view(np.uint32))


def test_quant_weights_full_size_sampled_blocks(big_layer):
    rng = np.random.default_rng(1)
    gq = lc.weight_codes_rowmajor(big_layer.wgu_q)
    gs = host(big_layer.wgu_s)
    dq = lc.weight_codes_rowmajor(big_layer.wd_q)
    ds = host(big_layer.wd_s)
    for (bits, q, s) in ((big_layer.wgu_bits, gq, gs), (big_layer.bits["w_down"], dq, ds)):
        NB, KB = s.shape
        picks = [(0, 0), (NB - 1, KB - 1)] + [tuple(p) for p in np.stack([rng.integers(0, NB, 30), rng.integers(0, KB, 30)], 1)]
        for nb, kb in picks:
            blk = bits[nb * 128:(nb + 1) * 128, kb * 128:(kb + 1) * 128]
            rq, rs = O.quant_weights(np.ascontiguousarray(blk))
            assert np.array_equal(q[nb * 128:(nb + 1) * 128, kb * 128:(kb + 1) * 128], rq), (nb, kb)
            assert s[nb, kb] == rs[0, 0], (nb, kb)


@pytest.mark.parametrize("N,K", [(256, 384), (384, 640), (1536, 4096)])
def test_pack_weights_rowmajor_oracle_codes(N, K):
    """Row-major codes from another producer (the oracle's quant_weights)
    through the C ABI's repack give the same bytes as the library's own
    quantization in the tile layout."""
    rng = np.random.default_rng(N + K)
    bits = torch.from_numpy((rng.standard_normal((N, K)) * 0.02).astype(np.float32)).to(torch.bfloat16)
    bits = bits.view(torch.int16).numpy().view(np.uint16)
    oq, os_ = O.quant_weights(bits)
    packed = lc.pack_weights(torch.from_numpy(oq).to(DEV))
    own_q, own_s = lc.quantize_weights(dev_bf16(bits))
    torch.cuda.synchronize()
    assert torch.equal(packed, own_q)
    assert np.array_equal(host(own_s).view(np.uint32), os_.view(np.uint32))


def test_ffn_with_oracle_quantized_weights():
    """The FFN on weights quantized by the oracle (row-major codes, packed on
    the device) equals the FFN on the library's own quantization, bit for bit."""
    lay = Layer(TINY, layer=1)
    wgu_q, wgu_s = O.quant_weights(lay.wgu_bits)
    wd_q, wd_s = O.quant_weights(lay.bits["w_down"])
    x = dev_bf16(synth.make_x(TINY, layer=1))
    a = lc.ffn_fp8(x, lay.norm_w, lay.wgu_q, lay.wgu_s, lay.wd_q, lay.wd_s)
    b = lc.ffn_fp8(x, lay.norm_w, lc.pack_weights(torch.from_numpy(wgu_q).to(DEV)), torch.from_numpy(wgu_s).to(DEV),
                   lc.pack_weights(torch.from_numpy(wd_q).to(DEV)), torch.from_numpy(wd_s).to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


# ---------------------------------------------------------------------------
# fused RMSNorm + 1x128 quantization
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("M,H", [(64, 256), (1, 128), (3, 384), (33, 4096), (100, 1024), (513, 4096), (7, 16384)])
def test_rmsnorm_quant_bit_exact(M, H):
    _say("rmsnorm M=%d H=%d" % (M, H))
    rng = np.random.default_rng(M * 7 + H)
    x = rng.standard_normal((M, H)).astype(np.float32) * np.exp(rng.uniform(-4, 4, (M, 1))).astype(np.float32)
    x[:, rng.choice(H, max(1, H // 100), replace=False)] *= 40
    x[0, :] = 0.0 if M > 1 else x[0, :]        # a zero row: r = 1/sqrt(eps), all groups zero
    if M > 2:
        x[2, :] *= np.float32(1e-30)           # tiny row
    xb = torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    wb = torch.from_numpy((1 + 0.02 * rng.standard_normal(H)).astype(np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    xq = torch.full((M, H), 0xFF, dtype=torch.uint8, device=DEV)
    xs = torch.full((H // 128, M), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_rmsnorm_quant(dev_bf16(xb), dev_bf16(wb), xq, xs)
    torch.cuda.synchronize()
    check_norm_exact(xb, wb, host(xq), host(xs))


@pytest.mark.parametrize("M,H", [(5, 256), (9, 1024), (17, 2176), (64, 16384), (1030, 512), (1100, 4096)])
def test_add_rmsnorm_quant_bit_exact(M, H):
    """The AddNorm kernel at 1, 2 and 4 wavefronts per row (H = 256, 1024,
    >= 2048 at M <= 1024; 2176 leaves the last pass ragged) and at one
    wavefront per row (M > 1024, one and eight passes): resid = RNE(resid + y)
    in place, then the norm and quantization of the new resid, all
    bit-exact."""
    _say("add_rmsnorm M=%d H=%d" % (M, H))
    rng = np.random.default_rng(M * 11 + H)
    x = rng.standard_normal((M, H)).astype(np.float32) * np.exp(rng.uniform(-3, 3, (M, 1))).astype(np.float32)
    yv = rng.standard_normal((M, H)).astype(np.float32) * 0.5
    x[:, rng.choice(H, max(1, H // 100), replace=False)] *= 40
    to_bits = lambda a: torch.from_numpy(a).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    xb, yb = to_bits(x), to_bits(yv)
    wb = to_bits((1 + 0.02 * rng.standard_normal(H)).astype(np.float32))
    want = O.residual_add(xb, yb)
    r = dev_bf16(xb)
    xq = torch.full((M, H), 0xFF, dtype=torch.uint8, device=DEV)
    xs = torch.full((H // 128, M), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_add_rmsnorm_quant(r, dev_bf16(yb), dev_bf16(wb), xq, xs)
    torch.cuda.synchronize()
    assert np.array_equal(host_bf16(r), want)
    check_norm_exact(want, wb, host(xq), host(xs))


def test_rmsnorm_quant_full_batch_sampled_rows():
    lay = Layer(BATCH8K, layer=1, quantize=False)
    xb = synth.make_x(BATCH8K, layer=1, step=0)
    M, H = xb.shape
    xq = torch.empty((M, H), dtype=torch.uint8, device=DEV)
    xs = torch.empty((H // 128, M), dtype=torch.float32, device=DEV)
    lc.lacache_rmsnorm_quant(dev_bf16(xb), lay.norm_w, xq, xs)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(2).choice(M, 64, replace=False))
    check_norm_exact(xb[rows], lay.bits["norm_w"], host(xq)[rows], host(xs)[:, rows])


# ---------------------------------------------------------------------------
# GEMM stages
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("policy", [0, 2])
def test_stages_tiny(policy):
    """Tiny workload, every row: skinny (auto at M=64) and tiled kernels."""
    lc.lacache_set_path_policy(policy)
    lay = Layer(TINY, layer=1)
    xb = synth.make_x(TINY, layer=1)
    M, H, I = TINY.M, TINY.H, TINY.I
    t = run_stages(dev_bf16(xb), lay, M, H, I)
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    check_norm_exact(xb, lay.bits["norm_w"], host(t["xq"]), host(t["xs"]))
    check_requant_exact(host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    g = check_gateup_model(host(t["xq"]), host(t["xs"]), wgu_q, wgu_s, I, host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    # the worst-case envelope of the model (16-wide spans) as a secondary check
    check_gateup_explained(host(t["xq"]), host(t["xs"]), wgu_q, wgu_s, I, host(t["hq"]), host(t["hs"]))
    e = check_down_same_operands(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]), host_bf16(t["out"]))
    d = check_down_model(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]))
    _say("tiny policy=%d: gate/up %s; down same-operand error %.2e, %.3f of the model tolerance" % (policy, g, e, d))


@pytest.mark.parametrize("M,policy", [(1, 0), (17, 0), (33, 0), (64, 0), (65, 0), (200, 0), (50, 2), (1, 2)])
def test_stages_ragged_shapes(M, policy):
    """Ragged M on both kernel paths, H=512, I=768 (several tiles, partial tails)."""
    _say("ragged M=%d policy=%d" % (M, policy))
    lc.lacache_set_path_policy(policy)
    w = synth.Workload(90, "ragged", M, 512, 768, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xb = synth.make_x(w, layer=1)
    t = run_stages(dev_bf16(xb), lay, M, w.H, w.I)
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    check_norm_exact(xb, lay.bits["norm_w"], host(t["xq"]), host(t["xs"]))
    check_requant_exact(host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_gateup_model(host(t["xq"]), host(t["xs"]), wgu_q, wgu_s, w.I, host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_down_same_operands(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]), host_bf16(t["out"]))
    check_down_model(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]))


@pytest.mark.parametrize("policy", [0, 2])
def test_zero_rows_and_zero_blocks(policy):
    """The method's degenerate cases through the whole FFN, on both paths: an
    all-zero input row and an all-(-0) one (r = 1/sqrt(eps), every group
    scale 0 and every code 0x00, an all-zero h row and output row); a zero
    128-row block of W_gate and W_up (that h-group is 0 in every row, so its
    scale is 0 and its codes 0x00 come from the epilogue's zero-scale rule);
    a zero 128-row block of W_down (those output columns 0). Checked against
    the oracle like every other case, and the fused call equals the stages."""
    lc.lacache_set_path_policy(policy)
    M, H, I = 17, 256, 768
    w = synth.Workload(89, "degenerate", M, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1, quantize=False)
    b = lay.bits
    b["w_gate"][256:384] = 0
    b["w_up"][256:384] = 0
    b["w_down"][128:256] = 0
    lay.wgu_bits = np.concatenate([b["w_gate"], b["w_up"]], axis=0)
    lay.wgu_q, lay.wgu_s = lc.quantize_weights(dev_bf16(lay.wgu_bits))
    lay.wd_q, lay.wd_s = lc.quantize_weights(dev_bf16(b["w_down"]))
    xb = synth.make_x(w, layer=1)
    xb[3] = 0
    xb[M - 1] = 0x8000
    x = dev_bf16(xb)
    t = run_stages(x, lay, M, H, I)
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    xq, xs, hq, hs = host(t["xq"]), host(t["xs"]), host(t["hq"]), host(t["hs"])
    check_norm_exact(xb, b["norm_w"], xq, xs)
    check_requant_exact(host(t["h_tap"]), hq, hs)
    g = check_gateup_model(xq, xs, wgu_q, wgu_s, I, host(t["h_tap"]), hq, hs)
    check_down_same_operands(hq, hs, wd_q, wd_s, host(t["out_tap"]), host_bf16(t["out"]))
    check_down_model(hq, hs, wd_q, wd_s, host(t["out_tap"]))
    for r in (3, M - 1):
        assert np.all(xq[r] == 0) and np.all(xs[:, r] == 0)
        assert np.all(hq[r] == 0) and np.all(hs[:, r] == 0)
    assert np.all(hq[:, 256:384] == 0) and np.all(hs[2] == 0)
    out = host_bf16(t["out"])
    assert np.all(out[:, 128:256] & 0x7FFF == 0) and np.all(out[[3, M - 1]] & 0x7FFF == 0)
    fused = lc.ffn_fp8(x, lay.norm_w, lay.wgu_q, lay.wgu_s, lay.wd_q, lay.wd_s)
    assert np.array_equal(host_bf16(fused), out)
    _say("degenerate policy=%d: gate/up %s" % (policy, g))


@pytest.mark.parametrize("M,H,I", [(5, 256, 384), (32, 640, 1152), (16, 8192, 256), (32, 4096, 384),
                                   (17, 1152, 2304), (3, 128, 256), (2, 256, 128), (33, 512, 384),
                                   (48, 4096, 384), (64, 1152, 256), (64, 4096, 128), (9, 256, 16384),
                                   (32, 384, 12416)])
def test_skinny_k_parts(M, H, I):
    """Skinny kernels at K ranges that split unevenly over their K parts: fewer
    K-groups than parts (H = 256, I = 384; a single K-group at H = 128), a part
    one group longer than the others (H = 640), the longest K the gate/up
    kernel's LDS holds (H = 8192 at M = 16; 4096 at M = 32), I = 128 (8 slab
    pairs: the last workgroup has an idle pair), 33..64 rows, where the
    gate/up workgroups take one half of K each (odd K-group counts: H = 1152),
    and down K ranges past the 8-part kernel's 96 K-groups at up to 32 rows
    (I = 16384, and 12416: 97 groups over 4 parts)."""
    _say("skinny M=%d H=%d I=%d" % (M, H, I))
    lc.lacache_set_path_policy(1)
    w = synth.Workload(91, "kparts", M, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xb = synth.make_x(w, layer=1)
    t = run_stages(dev_bf16(xb), lay, M, H, I)
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    check_norm_exact(xb, lay.bits["norm_w"], host(t["xq"]), host(t["xs"]))
    check_requant_exact(host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_gateup_model(host(t["xq"]), host(t["xs"]), wgu_q, wgu_s, I, host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_down_same_operands(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]), host_bf16(t["out"]))
    check_down_model(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]))


@pytest.mark.parametrize("M,H,I", [(5, 384, 4224), (48, 2560, 4224), (20, 256, 8320), (33, 128, 8192),
                                   (64, 2048, 128), (64, 2176, 256), (48, 2688, 128)])
def test_skinny_slab_pairs_per_workgroup(M, H, I):
    """The gate/up kernel's other workgroup shapes: 2 slab pairs x 4 K parts
    (I = 4224, 8192), 3 x 4 with a partial last workgroup (I = 8320) and 1 x
    4 (I = 128, 256), at 33..64 rows with all of K in the LDS up to its
    largest (H = 2688 at 48 rows, 2048 at 64) and with two K halves just above
    (2176 at 64)."""
    _say("skinny pairs M=%d H=%d I=%d" % (M, H, I))
    lc.lacache_set_path_policy(1)
    w = synth.Workload(91, "pairs", M, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xb = synth.make_x(w, layer=1)
    t = run_stages(dev_bf16(xb), lay, M, H, I)
    wgu_q, wgu_s, _, _ = lay.host_weights()
    check_norm_exact(xb, lay.bits["norm_w"], host(t["xq"]), host(t["xs"]))
    check_requant_exact(host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_gateup_model(host(t["xq"]), host(t["xs"]), wgu_q, wgu_s, I, host(t["h_tap"]), host(t["hq"]), host(t["hs"]))


@pytest.mark.parametrize("M,H", [(5, 640), (32, 2048), (33, 640), (64, 2048)])
def test_skinny_gateup_does_not_depend_on_i(M, H):
    """An element's four K parts and the order they are walked and added in do
    not depend on how many slab pairs share a workgroup (1 at I = 384, 2 at
    4224, 3 at 8448): the same weight rows give the same bytes."""
    _say("skinny gate/up of several I, M=%d H=%d" % (M, H))
    lc.lacache_set_path_policy(1)
    wide = 8448
    w = synth.Workload(91, "narrow", M, H, wide, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xq = torch.empty((M, H), dtype=torch.uint8, device=DEV)
    xs = torch.empty((H // 128, M), dtype=torch.float32, device=DEV)
    lc.lacache_rmsnorm_quant(dev_bf16(synth.make_x(w, layer=1)), lay.norm_w, xq, xs)
    gu = dev_bf16(np.concatenate([lay.bits["w_gate"], lay.bits["w_up"]]))
    ref = None
    for I in (wide, 4224, 384):
        wq, ws = lc.quantize_weights(torch.cat([gu[:I], gu[wide:wide + I]]).contiguous())
        hq = torch.full((M, I), 0xFF, dtype=torch.uint8, device=DEV)
        hs = torch.full((I // 128, M), float("nan"), dtype=torch.float32, device=DEV)
        tap = torch.full((M, I), float("nan"), dtype=torch.float32, device=DEV)
        lc.lacache_gateup_swiglu_quant(xq, xs, wq, ws, hq, hs, tap)
        torch.cuda.synchronize()
        if ref is None:
            ref = (hq, hs, tap)
        assert torch.equal(tap.view(torch.int32), ref[2][:, :I].contiguous().view(torch.int32)), I
        assert torch.equal(hq, ref[0][:, :I]), I
        assert torch.equal(hs.view(torch.int32), ref[1][:I // 128].view(torch.int32)), I


def test_skinny_gateup_of_one_and_two_k_pieces():
    """33..64 rows: all of K in one workgroup (48 rows at H = 2560) and two K
    halves (64 rows) add an element's K parts in the same order."""
    H, I = 2560, 384
    lc.lacache_set_path_policy(1)
    w = synth.Workload(91, "pieces", 64, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    x = dev_bf16(synth.make_x(w, layer=1))
    taps = []
    for M in (48, 64):
        _say("skinny gate/up M=%d H=%d" % (M, H))
        taps.append(run_stages(x[:M].contiguous(), lay, M, H, I)["h_tap"])
    torch.cuda.synchronize()
    assert torch.equal(taps[0].view(torch.int32), taps[1][:48].view(torch.int32))


@pytest.mark.parametrize("M,H,I,ks", [(65, 128, 128, 1), (100, 384, 768, 1), (128, 256, 16384, 8),
                                      (129, 512, 1536, 1), (200, 1024, 4224, 2), (1000, 512, 1920, 1)])
def test_down_rows_of_64(M, H, I, ks):
    """The down GEMM with its weights in registers: one K-group, K-group counts
    that leave 1, 2, 3 and all of the last chunk of 4, 8 K splits and 2 of unequal
    length, last row tiles of 1, 8, 36, 40 and 64 rows, up to 16 row tiles."""
    _plan_is(M, H, I, (64, 128, ks, True))
    _say("down rows64 M=%d H=%d I=%d" % (M, H, I))
    lc.lacache_set_path_policy(2)
    w = synth.Workload(93, "rows64", M, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xb = synth.make_x(w, layer=1)
    t = run_stages(dev_bf16(xb), lay, M, H, I)
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    check_requant_exact(host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_down_same_operands(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]), host_bf16(t["out"]))
    check_down_model(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]))


def _plan_is(M, H, I, down=None, gateup=None, col_scales=False):
    """The tiled kernels take what the test is about: the down GEMM's (tile rows,
    columns, K splits, weights in registers) and the gate/up tile height. (The
    rule counts compute units; other devices than 256 run the sizes as they are.)"""
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        got = lc.lacache_tiled_plan(M, H, I, col_scales)
        assert (down is None or got[1:] == down) and gateup in (None, got[0]), got


def _random_down(M, H, I, seed):
    """Operands of a down GEMM: finite codes, scales within a few binades."""
    rng = np.random.default_rng(seed)
    codes = lambda n, k: (rng.integers(0, 0x78, (n, k)) | (rng.integers(0, 2, (n, k)) << 7)).astype(np.uint8)  # noqa: E731
    hq, wd = codes(M, I), codes(H, I)
    hs = np.exp2(rng.uniform(-6, -2, (I // 128, M))).astype(np.float32)
    ws = np.exp2(rng.uniform(-9, -7, (H // 128, I // 128))).astype(np.float32)
    dev = [torch.from_numpy(a).to(DEV) for a in (hq, hs, lc.weight_codes_tiled(wd), ws)]
    return (hq, hs, wd, ws), dev


@pytest.mark.parametrize("M,H,I,down", [
    (500, 4224, 128, (128, 256, 1, False)), (300, 4224, 12288, (128, 256, 5, False)),
    (333, 3072, 12288, (128, 256, 6, False)), (2000, 4224, 2048, (256, 256, 1, False)),
    (257, 8192, 384, (128, 128, 1, False)), (333, 3072, 8192, (128, 128, 3, False)),
    (200, 3072, 12288, (128, 128, 5, False)), (65, 3072, 12288, (64, 128, 5, True))])
def test_down_tile_shapes(M, H, I, down):
    """Every down tile shape with and without K splits, ragged last row tiles,
    partial column tiles of the 256-wide shapes (H = 4224: 128 valid columns, the
    second block scale falling back to the first), a single K-group (I = 128)."""
    _say("down M=%d H=%d I=%d %s" % (M, H, I, down))
    _plan_is(M, H, I, down)
    lc.lacache_set_path_policy(2)
    (hq, hs, wd, ws), dev = _random_down(M, H, I, M + H + I)
    out = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    tap = torch.full((M, H), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_down_proj(*dev, out, tap)
    torch.cuda.synchronize()
    assert torch.isfinite(tap).all().item()
    rows = np.unique([0, down[0] - 1, down[0] % M, M // 2, M - 1])
    check_down_same_operands(hq[rows], np.ascontiguousarray(hs[:, rows]), wd, ws, host(tap)[rows], host_bf16(out)[rows])
    check_down_model(hq[rows], np.ascontiguousarray(hs[:, rows]), wd, ws, host(tap)[rows])


@pytest.mark.parametrize("M,H,I,ks", [(129, 512, 1536, 1), (1000, 512, 1920, 1), (200, 1024, 4224, 2),
                                      (190, 3072, 8192, 3), (128, 256, 16384, 8)])
def test_down_weights_in_registers_give_the_tiled_kernels_bits(M, H, I, ks):
    """The down GEMM with its weights in registers against the tiled kernel's 64 x
    128 tiles over the same K splits (which calls with per-channel scales take;
    the scales are ones): the same bits."""
    _say("down registers against LDS M=%d H=%d I=%d" % (M, H, I))
    _plan_is(M, H, I, (64, 128, ks, True))
    _plan_is(M, H, I, (64, 128, ks, False), col_scales=True)
    lc.lacache_set_path_policy(2)
    _, dev = _random_down(M, H, I, M + H + I)
    res = []
    for f, extra in ((lc.lacache_down_proj, ()), (lc.lacache_down_proj_g, (torch.ones((H,), device=DEV),))):
        out = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
        tap = torch.full((M, H), float("nan"), dtype=torch.float32, device=DEV)
        f(*dev, *extra, out, tap)
        res.append((out, tap))
    torch.cuda.synchronize()
    assert torch.equal(res[0][1].view(torch.int32), res[1][1].view(torch.int32))
    assert torch.equal(res[0][0].view(torch.int16), res[1][0].view(torch.int16))


def _full_size_case(big_layer, w, step, rows_pick, policy):
    lc.lacache_set_path_policy(policy)
    xb = synth.make_x(w, layer=1, step=step)
    M, H, I = w.M, w.H, w.I
    t = run_stages(dev_bf16(xb), big_layer, M, H, I)
    rows = rows_pick(M)
    wgu_q, wgu_s, wd_q, wd_s = big_layer.host_weights()
    xq, xs = host(t["xq"])[rows], host(t["xs"])[:, rows]
    hq, hs = host(t["hq"])[rows], host(t["hs"])[:, rows]
    check_norm_exact(xb[rows], big_layer.bits["norm_w"], xq, xs)
    check_requant_exact(host(t["h_tap"])[rows], hq, hs)
    g = check_gateup_model(xq, xs, wgu_q, wgu_s, I, host(t["h_tap"])[rows], hq, hs)
    e = check_down_same_operands(hq, hs, wd_q, wd_s, host(t["out_tap"])[rows], host_bf16(t["out"])[rows])
    d = check_down_model(hq, hs, wd_q, wd_s, host(t["out_tap"])[rows])
    # every row was written
    assert np.all(host(t["hq"]) != 0xFF) and torch.isfinite(t["out"].float()).all().item()
    return g, e, d


@pytest.mark.parametrize("policy", [0, 2])
def test_block32_full(big_layer, policy):
    """One 32-token decode block at H=4096, I=12288: every row."""
    g, e, d = _full_size_case(big_layer, BLOCK32, 0, lambda M: np.arange(M), policy)
    _say("block32 policy=%d: gate/up %s; down error %.2e, %.3f of the model tolerance" % (policy, g, e, d))


def test_sar512_sampled(big_layer):
    rows = lambda M: np.sort(np.random.default_rng(3).choice(M, 12, replace=False))
    g, e, d = _full_size_case(big_layer, SAR512, 5, rows, 0)
    _say("sar512: gate/up %s; down error %.2e, %.3f of the model tolerance" % (g, e, d))


def test_batch8192_sampled(big_layer):
    rows = lambda M: np.concatenate([[0, M - 1], np.sort(np.random.default_rng(4).choice(M, 6, replace=False))])
    g, e, d = _full_size_case(big_layer, BATCH8K, 0, rows, 0)
    _say("batch8192: gate/up %s; down error %.2e, %.3f of the model tolerance" % (g, e, d))


def test_batch4096_sampled(big_layer):
    """M = 4096, the smallest M of the MFMA-bound range: 256-row tiles for both
    GEMMs (one round of 256 down tiles over all of K), sampled rows."""
    w = synth.WORKLOADS["batch4x1024_h4096_i12288"]
    rows = lambda M: np.concatenate([[0, M - 1], np.sort(np.random.default_rng(6).choice(M, 6, replace=False))])
    g, e, d = _full_size_case(big_layer, w, 0, rows, 0)
    _say("batch4096: gate/up %s; down error %.2e, %.3f of the model tolerance" % (g, e, d))


def test_bm256_partial_row_tile_sampled(big_layer):
    """M = 3000: 256-row tiles for both GEMMs with a last row tile of 184 rows
    (clamped activation rows, unstored outputs); sampled rows, all of the last
    tile's edge included."""
    M = 3000
    w = synth.Workload(93, "bm256_partial", M, 4096, 12288, act="outlier", outlier_ratio=0.01)
    rows = lambda m: np.unique(np.concatenate([[0, 255, 256, 2815, 2816, m - 2, m - 1],
                                               np.random.default_rng(M).choice(np.arange(1, 2815), 4, replace=False)]))
    _plan_is(M, 4096, 12288, (256, 256, 1, False), 256)
    g, e, d = _full_size_case(big_layer, w, 0, rows, 0)
    _say("bm256 partial M=%d: gate/up %s; down error %.2e, %.3f of the model tolerance" % (M, g, e, d))


@pytest.mark.parametrize("M,ks,down", [(200, 6, (64, 128, 2, True)), (320, 5, (128, 256, 5, False)),
                                       (400, 4, (128, 256, 4, False)), (576, 3, (128, 256, 3, False)),
                                       (700, 2, (128, 256, 2, False)), (1024, 2, (128, 128, 1, False))])
def test_split_k_down_sampled(big_layer, M, ks, down):
    """The tiled down GEMM at H = 4096, I = 12288: the K splits that its workspace
    has room for (ks) and the tile shape and splits that it takes, oracle-checked
    on sampled rows, the first and last included."""
    _say("split-K M=%d KS=%d" % (M, ks))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        # the workspace: the KS fp32 partials [KS][M][H], then xq [M][H] and
        # hq [M][3H] (I = 3H), i.e. (KS + 1) M H 4 bytes, plus the scales
        ws = lc.lacache_ffn_workspace_bytes(M, 4096, 12288)
        assert (ks + 1) * M * 4096 * 4 <= ws < (ks + 2) * M * 4096 * 4
    _plan_is(M, 4096, 12288, down)
    w = synth.Workload(94, "splitk", M, 4096, 12288, act="outlier", outlier_ratio=0.01)
    rows = lambda m: np.concatenate([[0, m - 1], np.sort(np.random.default_rng(M).choice(np.arange(1, m - 1), 6,
                                                                                          replace=False))])
    g, e, d = _full_size_case(big_layer, w, 0, rows, 0)
    _say("split-K M=%d: gate/up %s; down error %.2e, %.3f of the model tolerance" % (M, g, e, d))


@pytest.mark.parametrize("M,height,down", [(100, 64, (64, 128, 4, True)), (190, 96, (64, 128, 2, True)),
                                           (230, 128, (64, 128, 2, True)), (333, 192, (128, 256, 5, False)),
                                           (400, 256, (128, 256, 4, False))])
def test_tile_heights_sampled(big_layer, M, height, down):
    """Each gate/up tile height with a ragged last row tile, and the down tiles
    that these calls take, oracle-checked on sampled rows, the tile edges
    included."""
    _plan_is(M, 4096, 12288, down, height)
    w = synth.Workload(98, "heights", M, 4096, 12288, act="outlier", outlier_ratio=0.01)
    rows = lambda m: np.unique([r for r in (0, 63, 64, 95, 96, 191, 192, m - 1) if r < m])
    g, e, d = _full_size_case(big_layer, w, 0, rows, 0)
    _say("tile heights M=%d: gate/up %s; down error %.2e, %.3f of the model tolerance" % (M, g, e, d))


def test_gateup_bytes_do_not_depend_on_the_tile_height(big_layer):
    """An element's K-groups are added in the same order at every tile height,
    so the codes and scales of a row are the same bytes in calls of 65, 190,
    256, 333, 512 and 700 rows (heights 64, 96, 128, 192, 256 and 192)."""
    w = synth.Workload(98, "heights", 700, 4096, 12288, act="outlier", outlier_ratio=0.01)
    x = dev_bf16(synth.make_x(w, layer=1))
    ref = None
    for M, height in ((700, 192), (512, 256), (333, 192), (256, 128), (190, 96), (65, 64)):
        _plan_is(M, 4096, 12288, gateup=height)
        xq = torch.empty((M, 4096), dtype=torch.uint8, device=DEV)
        xs = torch.empty((32, M), dtype=torch.float32, device=DEV)
        hq = torch.full((M, 12288), 0xFF, dtype=torch.uint8, device=DEV)
        hs = torch.full((96, M), float("nan"), dtype=torch.float32, device=DEV)
        _say("gate/up M=%d" % M)
        lc.lacache_rmsnorm_quant(x[:M], big_layer.norm_w, xq, xs)
        lc.lacache_gateup_swiglu_quant(xq, xs, big_layer.wgu_q, big_layer.wgu_s, hq, hs)
        torch.cuda.synchronize()
        if ref is None:
            ref = (hq, hs)
        assert torch.equal(hq, ref[0][:M]), M
        assert torch.equal(hs.view(torch.int32), ref[1][:, :M].view(torch.int32)), M


@pytest.mark.parametrize("M,H,I", [(5, 16384, 1024), (5, 256, 65536)])
def test_maximum_h_and_i(M, H, I):
    """The largest H (16384) and the largest I (65536) the library takes, each
    with a small M: long K loops (128 K-groups in the gate/up, 512 in the
    down), and at I = 65536 the down GEMM's widest K split (32 workgroups per
    output tile). Every row against the oracle."""
    _say("max sizes M=%d H=%d I=%d" % (M, H, I))
    _plan_is(M, H, I, (64, 128, 32 if I == 65536 else 1, True))
    w = synth.Workload(92, "max_%d_%d" % (H, I), M, H, I, act="outlier", outlier_ratio=0.01)
    lay = Layer(w, layer=1)
    g, e, d = _full_size_case(lay, w, 0, lambda m: np.arange(m), 0)
    _say("max sizes H=%d I=%d: gate/up %s; down error %.2e, %.3f of the model tolerance" % (H, I, g, e, d))


def test_maximum_m():
    """M = 2^24, the largest M the library takes (H = I = 128): every stage
    over 16.8 M rows (the activations drawn on the GPU from a seeded
    generator), checked against the oracle on sampled rows, the first and
    last included."""
    M, H, I = 1 << 24, 128, 128
    _say("max M=%d" % M)
    w = synth.Workload(91, "max_m", 64, H, I)  # the weights' shapes only
    lay = Layer(w, layer=1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(20260716)
    x = torch.randn((M, H), generator=gen, device=DEV, dtype=torch.float32).to(torch.bfloat16)
    t = run_stages(x, lay, M, H, I, sentinel=False)
    rows = np.unique(np.concatenate([[0, 1, M // 2, M - 2, M - 1], np.random.default_rng(7).choice(M, 11, replace=False)]))
    ri = torch.from_numpy(rows).to(DEV)
    sel = lambda name: host(t[name].index_select(0, ri))
    selc = lambda name: host(t[name].index_select(1, ri))
    xb = host_bf16(x.index_select(0, ri))
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    xq, xs, hq, hs = sel("xq"), selc("xs"), sel("hq"), selc("hs")
    check_norm_exact(xb, lay.bits["norm_w"], xq, xs)
    check_requant_exact(sel("h_tap"), hq, hs)
    g = check_gateup_model(xq, xs, wgu_q, wgu_s, I, sel("h_tap"), hq, hs)
    e = check_down_same_operands(hq, hs, wd_q, wd_s, sel("out_tap"), host_bf16(t["out"].index_select(0, ri)))
    d = check_down_model(hq, hs, wd_q, wd_s, sel("out_tap"))
    # every row was written: the fp32 taps started as NaN
    assert torch.isfinite(t["h_tap"]).all().item() and torch.isfinite(t["out_tap"]).all().item()
    _say("max M: gate/up %s; down error %.2e, %.3f of the model tolerance" % (g, e, d))
    del t, x
    torch.cuda.empty_cache()


@pytest.mark.parametrize("M", [50, 130])
def test_tiled_partial_column_tile(M):
    """The tiled kernels at H = 640, a column count that is no multiple of 256,
    with few rows (the down GEMM takes 64 x 128 tiles; the 256-wide ones' partial
    column tile is in test_down_tile_shapes)."""
    _say("tiled H=640 M=%d" % M)
    lc.lacache_set_path_policy(2)
    w = synth.Workload(95, "h640", M, 640, 1152, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xb = synth.make_x(w, layer=1)
    t = run_stages(dev_bf16(xb), lay, M, w.H, w.I)
    wgu_q, wgu_s, wd_q, wd_s = lay.host_weights()
    check_norm_exact(xb, lay.bits["norm_w"], host(t["xq"]), host(t["xs"]))
    check_requant_exact(host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_gateup_model(host(t["xq"]), host(t["xs"]), wgu_q, wgu_s, w.I, host(t["h_tap"]), host(t["hq"]), host(t["hs"]))
    check_down_same_operands(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]), host_bf16(t["out"]))
    check_down_model(host(t["hq"]), host(t["hs"]), wd_q, wd_s, host(t["out_tap"]))


def test_bm256_partial_row_and_column_tiles():
    """Many rows of a narrow layer: M = 12000 at H = 640, I = 1152 takes 256-row
    gate/up tiles whose last holds 224 rows, and 128 x 128 down tiles whose last
    row tile holds 96 (256 x 256 down tiles with both tails are in
    test_down_tile_shapes). Sampled rows, the tails' rows included, against the
    oracle."""
    M, H, I = 12000, 640, 1152
    _say("bm256 partial row and column tiles M=%d H=%d" % (M, H))
    _plan_is(M, H, I, (128, 128, 1, False), 256)
    w = synth.Workload(97, "bm256_tails", M, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    pick = lambda m: np.unique(np.concatenate([[0, 255, 256, m - 224, m - 2, m - 1],
                                               np.random.default_rng(11).choice(m, 24, replace=False)]))
    g, e, d = _full_size_case(lay, w, 0, pick, 0)
    _say("bm256 tails: gate/up %s; down error %.2e, %.3f of the model tolerance" % (g, e, d))


@pytest.mark.parametrize("step", [0, 31])
def test_stack_layers_with_residual_adds(step):
    """Three consecutive layers of the 31-layer stack (own weights per layer)
    at the first and the last denoising step: each layer runs on the bf16
    state the previous layer and residual add produced. Every layer's stages
    are checked on sampled rows as in the single-layer cases, the fused call
    must equal the stages, and the residual add is bit-exact."""
    M, H, I = STACK.M, STACK.H, STACK.I
    rows = np.sort(np.random.default_rng(6 + step).choice(M, 8, replace=False))
    x = dev_bf16(synth.make_x(STACK, layer=1, step=step))
    for li in (1, 2, 3):
        _say("stack step %d layer %d" % (step, li))
        layer = Layer(STACK, layer=li)
        xb = host_bf16(x)
        t = run_stages(x, layer, M, H, I)
        wgu_q, wgu_s, wd_q, wd_s = layer.host_weights()
        xq, xs = host(t["xq"])[rows], host(t["xs"])[:, rows]
        hq, hs = host(t["hq"])[rows], host(t["hs"])[:, rows]
        check_norm_exact(xb[rows], layer.bits["norm_w"], xq, xs)
        check_requant_exact(host(t["h_tap"])[rows], hq, hs)
        check_gateup_model(xq, xs, wgu_q, wgu_s, I, host(t["h_tap"])[rows], hq, hs)
        check_down_same_operands(hq, hs, wd_q, wd_s, host(t["out_tap"])[rows], host_bf16(t["out"])[rows])
        check_down_model(hq, hs, wd_q, wd_s, host(t["out_tap"])[rows])
        y = lc.ffn_fp8(x, layer.norm_w, layer.wgu_q, layer.wgu_s, layer.wd_q, layer.wd_s)
        torch.cuda.synchronize()
        assert np.array_equal(host_bf16(y), host_bf16(t["out"]))
        lc.lacache_add_bf16(x, y)
        torch.cuda.synchronize()
        assert np.array_equal(host_bf16(x), O.residual_add(xb, host_bf16(y)))
        del layer, t, y


# ---------------------------------------------------------------------------
# whole-layer call, workspace variant, determinism, residual add, errors
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("M", [32, 64, 200, 512])
def test_fused_call_matches_stages_and_is_deterministic(big_layer, M):
    _say("fused M=%d" % M)
    w = synth.Workload(91, "fused", M, 4096, 12288, act="outlier", outlier_ratio=0.01)
    xb = synth.make_x(w, layer=1)
    x = dev_bf16(xb)
    t = run_stages(x, big_layer, M, 4096, 12288)
    a = lc.ffn_fp8(x, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s)
    b = lc.ffn_fp8(x, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s)
    ws = torch.empty(lc.lacache_ffn_workspace_bytes(M, 4096, 12288), dtype=torch.uint8, device=DEV)
    ws.fill_(0xA5)  # garbage: the call must not rely on a clean workspace
    c = torch.empty_like(a)
    lc.lacache_ffn_fp8_ws(x, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s, c, ws)
    torch.cuda.synchronize()
    ref = host_bf16(t["out"])
    assert np.array_equal(host_bf16(a), ref)
    assert np.array_equal(host_bf16(b), ref)
    assert np.array_equal(host_bf16(c), ref)


def test_skinny_and_tiled_paths_agree(big_layer):
    xb = synth.make_x(BLOCK32, layer=1)
    x = dev_bf16(xb)
    outs = []
    for policy in (1, 2):
        lc.lacache_set_path_policy(policy)
        outs.append(lc.ffn_fp8(x, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s).float())
    torch.cuda.synchronize()
    d = (outs[0] - outs[1]).abs().amax(dim=1) / outs[1].abs().amax(dim=1)
    # different accumulation orders; flips of top-binade h codes move outputs by a few 1e-3 of the row max
    assert d.max().item() < 2e-2, d.max().item()


@pytest.mark.parametrize("M", [1, 32, 200, 512])
def test_addnorm_fused_equals_add_then_ffn(big_layer, M):
    """The AddNorm entry points: resid = RNE(resid + y) in place, the norm of
    the new resid bit-exact against the oracle, and the fused FFN call equal,
    bit for bit, to the residual add followed by the plain FFN call."""
    _say("addnorm M=%d" % M)
    H, I = 4096, 12288
    w = synth.Workload(92, "addnorm", M, H, I, act="outlier", outlier_ratio=0.01)
    xb = synth.make_x(w, layer=1)
    yb = synth.make_x(w, layer=2, step=1)
    y = dev_bf16(yb)
    want = O.residual_add(xb, yb)
    r1 = dev_bf16(xb)
    xq = torch.full((M, H), 0xFF, dtype=torch.uint8, device=DEV)
    xs = torch.full((H // 128, M), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_add_rmsnorm_quant(r1, y, big_layer.norm_w, xq, xs)
    torch.cuda.synchronize()
    assert np.array_equal(host_bf16(r1), want)
    check_norm_exact(want, big_layer.bits["norm_w"], host(xq), host(xs))
    r2 = dev_bf16(xb)
    out2 = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    lc.lacache_ffn_fp8_addnorm(r2, y, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q,
                               big_layer.wd_s, out2)
    r3 = dev_bf16(xb)
    lc.lacache_add_bf16(r3, y)
    out3 = lc.ffn_fp8(r3, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s)
    torch.cuda.synchronize()
    assert np.array_equal(host_bf16(r2), want)
    assert np.array_equal(host_bf16(out2), host_bf16(out3))


CANARY = 0x5A


def _guarded(shape, dtype, pre=256, post=4096):
    """A tensor of `shape` inside a canary-filled byte buffer: `pre` bytes
    before it and `post` after it (pre keeps every alignment the ABI needs)."""
    n = int(np.prod(shape)) * torch.empty((), dtype=dtype).element_size()
    buf = torch.full((pre + n + post,), CANARY, dtype=torch.uint8, device=DEV)
    return {"buf": buf, "pre": pre, "n": n, "t": buf[pre:pre + n].view(dtype).view(shape)}


def _canaries_intact(g, name):
    b = host(g["buf"])
    before, after = b[:g["pre"]], b[g["pre"] + g["n"]:]
    assert np.all(before == CANARY), "%s: write before the buffer" % name
    assert np.all(after == CANARY), "%s: write past the end (first at +%d)" % (
        name, int(np.argmax(after != CANARY)))


@pytest.mark.parametrize("M,H,I,policy", [(17, 512, 768, 0), (33, 512, 384, 0), (64, 1152, 256, 0),
                                          (65, 512, 768, 0), (200, 512, 4096, 0), (50, 640, 1152, 2),
                                          (1, 256, 384, 2), (3, 128, 256, 0)])
def test_guard_regions(M, H, I, policy):
    """Canary bytes before and after every output of the stage calls and of
    the fused calls, and around a caller-owned workspace, at ragged M on both
    kernel paths (skinny one and two K halves, tiled, split-K tiled down,
    tiled with a partial column tile): nothing lands outside its buffer, and
    the results equal the unguarded calls'."""
    _say("guard M=%d H=%d I=%d policy=%d" % (M, H, I, policy))
    lc.lacache_set_path_policy(policy)
    w = synth.Workload(96, "guard", M, H, I, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    x = dev_bf16(synth.make_x(w, layer=1))
    ref = run_stages(x, lay, M, H, I, sentinel=False)
    g = {"xq": _guarded((M, H), torch.uint8), "xs": _guarded((H // 128, M), torch.float32),
         "hq": _guarded((M, I), torch.uint8), "hs": _guarded((I // 128, M), torch.float32),
         "h_tap": _guarded((M, I), torch.float32), "out": _guarded((M, H), torch.bfloat16),
         "out_tap": _guarded((M, H), torch.float32), "fused": _guarded((M, H), torch.bfloat16),
         "fused_ws": _guarded((M, H), torch.bfloat16),
         "ws": _guarded((lc.lacache_ffn_workspace_bytes(M, H, I),), torch.uint8)}
    lc.lacache_rmsnorm_quant(x, lay.norm_w, g["xq"]["t"], g["xs"]["t"])
    lc.lacache_gateup_swiglu_quant(g["xq"]["t"], g["xs"]["t"], lay.wgu_q, lay.wgu_s, g["hq"]["t"], g["hs"]["t"],
                                   g["h_tap"]["t"])
    lc.lacache_down_proj(g["hq"]["t"], g["hs"]["t"], lay.wd_q, lay.wd_s, g["out"]["t"], g["out_tap"]["t"])
    lc.lacache_ffn_fp8(x, lay.norm_w, lay.wgu_q, lay.wgu_s, lay.wd_q, lay.wd_s, g["fused"]["t"])
    g["ws"]["t"].fill_(0xA5)
    lc.lacache_ffn_fp8_ws(x, lay.norm_w, lay.wgu_q, lay.wgu_s, lay.wd_q, lay.wd_s, g["fused_ws"]["t"], g["ws"]["t"])
    torch.cuda.synchronize()
    for name, gg in g.items():
        _canaries_intact(gg, name)
    for name in ("xq", "xs", "hq", "hs", "h_tap", "out_tap"):
        assert torch.equal(g[name]["t"].view(torch.uint8), ref[name].view(torch.uint8)), name
    for name in ("out", "fused", "fused_ws"):
        assert torch.equal(g[name]["t"].view(torch.int16), ref["out"].view(torch.int16)), name


def test_residual_add_bit_exact():
    rng = np.random.default_rng(5)
    n = 1_000_003
    a = torch.from_numpy(rng.standard_normal(n).astype(np.float32) * 4).to(torch.bfloat16)
    b = torch.from_numpy(rng.standard_normal(n).astype(np.float32) * 0.3).to(torch.bfloat16)
    ab = a.view(torch.int16).numpy().view(np.uint16)
    bb = b.view(torch.int16).numpy().view(np.uint16)
    x = dev_bf16(ab)
    lc.lacache_add_bf16(x, dev_bf16(bb))
    torch.cuda.synchronize()
    assert np.array_equal(host_bf16(x), O.residual_add(ab, bb))


# bf16 NaNs of both signs, signalling and quiet, with payloads; infinities
SPECIAL = [0x7F81, 0xFF81, 0x7FC0, 0xFFC0, 0x7FFF, 0xFFD5, 0x7F80, 0xFF80]


def _add_with_nans(xb, yb):
    with np.errstate(invalid="ignore"):
        s = (bf16_to_f32(xb) + bf16_to_f32(yb)).astype(np.float32)
    nan = np.isnan(s)
    return np.where(nan, np.uint16(0x7FC0), rne_bf16(np.where(nan, np.float32(0), s)))


@pytest.mark.parametrize("H", [128, 1024, 4096])
def test_residual_add_of_nans_and_infinities(H):
    """A NaN sum is stored as the quiet NaN 0x7FC0, whatever its operands' sign
    and payload (inf - inf included), in the residual add and in the AddNorm;
    rows of any bits, subnormal values among them, round to nearest even."""
    _say("residual add of NaNs, H=%d" % H)
    rng = np.random.default_rng(H)
    M = 40
    xb = synth.to_bf16_bits(rng.standard_normal((M, H)).astype(np.float32))
    yb = synth.to_bf16_bits(rng.standard_normal((M, H)).astype(np.float32))
    for i, a in enumerate(SPECIAL):
        xb[i, rng.integers(0, H, 4)] = a
        yb[8 + i, rng.integers(0, H, 4)] = a
        for j, b in enumerate(SPECIAL):
            xb[16 + i, 5 + 9 * j], yb[16 + i, 5 + 9 * j] = a, b
    xb[24:32] = rng.integers(0, 1 << 16, (8, H))  # any bits, subnormal ones and sums among them
    yb[24:28] = rng.integers(0, 1 << 16, (4, H))
    yb[28:32] = xb[28:32] ^ rng.integers(0, 1 << 10, (4, H)).astype(np.uint16)
    xb[32], yb[32] = rng.integers(0, 0x200, H), rng.integers(0, 0x200, H) | 0x8000
    want = _add_with_nans(xb, yb)
    x = dev_bf16(xb)
    lc.lacache_add_bf16(x, dev_bf16(yb))
    r = dev_bf16(xb)
    xq = torch.full((M, H), 0xFF, dtype=torch.uint8, device=DEV)
    xs = torch.full((H // 128, M), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_add_rmsnorm_quant(r, dev_bf16(yb), dev_bf16(np.full(H, 0x3F80, dtype=np.uint16)), xq, xs)
    odd = dev_bf16(xb[16:24, :59].ravel()[:-1])  # 8 n - 1 values: the last ones one by one
    odd[-1] = float("nan")
    lc.lacache_add_bf16(odd, dev_bf16(yb[16:24, :59].ravel()[:-1]))
    torch.cuda.synchronize()
    assert np.array_equal(host_bf16(x), want)
    assert np.array_equal(host_bf16(r), want)
    assert np.array_equal(host_bf16(odd)[:-1], want[16:24, :59].ravel()[:-2]) and host_bf16(odd)[-1] == 0x7FC0


def test_zero_rows_is_a_no_op(big_layer):
    x = torch.empty((0, 4096), dtype=torch.bfloat16, device=DEV)
    out = torch.empty((0, 4096), dtype=torch.bfloat16, device=DEV)
    lc.lacache_ffn_fp8(x, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s, out)
    torch.cuda.synchronize()


def test_workspace_growth_and_stream_capture():
    """The library workspace under HIP graph capture: a captured call that
    would have to grow it returns LACACHE_ERR_CAPTURE and enqueues nothing;
    once an eager call has sized it, the call captures and replays; a later,
    larger eager call grows the workspace without freeing the buffer the
    graph holds, so the graph still replays to the eager result (checked on
    every replay, with eager work in between)."""
    lc.lacache_release_workspace()
    w = synth.Workload(97, "capture", 200, 512, 4096, act="outlier", outlier_ratio=0.02)
    lay = Layer(w, layer=1)
    xb = synth.make_x(w, layer=1)
    small, big = dev_bf16(xb[:16]), dev_bf16(xb)
    args = (lay.norm_w, lay.wgu_q, lay.wgu_s, lay.wd_q, lay.wd_s)
    out = torch.empty((16, 512), dtype=torch.bfloat16, device=DEV)
    status = []
    g0 = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g0):
        try:
            lc.lacache_ffn_fp8(small, *args, out)
        except lc.LacacheError as e:
            status.append(e.status)
    assert status == [lc.LACACHE_ERR_CAPTURE]
    del g0
    ref = lc.ffn_fp8(small, *args)  # eager: allocates the workspace
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lc.lacache_ffn_fp8(small, *args, out)
    for i in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)), i
        # eager work in between; the second one grows the workspace (200 rows, split-K partials)
        lc.ffn_fp8(big if i == 1 else small, *args)
        torch.cuda.synchronize()
    del g
    lc.lacache_release_workspace()


def test_forced_workspace_allocation_failure(big_layer):
    lc.lacache_release_workspace()
    os.environ["LACACHE_TEST_FAIL_ALLOC"] = "1"
    try:
        x = dev_bf16(synth.make_x(BLOCK32, layer=1))
        out = torch.full((32, 4096), 7.0, dtype=torch.bfloat16, device=DEV)
        with pytest.raises(lc.LacacheError) as ei:
            lc.lacache_ffn_fp8(x, big_layer.norm_w, big_layer.wgu_q, big_layer.wgu_s, big_layer.wd_q, big_layer.wd_s, out)
        assert ei.value.status == lc.LACACHE_ERR_ALLOC
        torch.cuda.synchronize()
        assert bool((out.float() == 7.0).all())
    finally:
        del os.environ["LACACHE_TEST_FAIL_ALLOC"]
