"""GPU parity of the coarse quantization granularities (Sec. 4, Table
fp8-granularities: per token with per-channel weights, per tensor) against
the oracle in oracle/granularity.py, through the C ABI.

Bit-exact: weight codes and row scales, the fp32 RMSNorm, activation codes
and scales (every K-group of a row carries the row's scale). Within a bound
derived from the arithmetic: the gate/up GEMM + SwiGLU (the per-group path's
MFMA error model with the row scales applied after the K sum) and, on the
same operands, the down GEMM (row-max-normalised 2e-3, bf16 = RNE of fp32).
The fused call equals its stages bit for bit, and the paper's finding holds
on the GPU's own outputs: per-group error < per-token < per-tensor.
"""

import numpy as np
import pytest
import torch

import oracle.ffn as O
import oracle.granularity as G
import paper_2607_16339_amd as lc
import synth
from gpu_util import DEV, SILU_LIP, dev_bf16, host, host_bf16, mfma_dot_bound
from oracle import csweep
from oracle.bf16 import bf16_to_f32, rne_bf16

pytestmark = pytest.mark.gpu
GRANS = [(lc.LACACHE_GRAN_TOKEN, G.GRAN_TOKEN), (lc.LACACHE_GRAN_TENSOR, G.GRAN_TENSOR)]


def _say(msg):
    print(msg, flush=True)


def _inputs(M, H, I, seed=7, outliers=True):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, H)).astype(np.float32)
    if outliers:
        x[:, rng.choice(H, max(1, H // 100), replace=False)] *= np.float32(40.0)
        x[::5] *= np.float32(6.0)
    nw = (1.0 + 0.02 * rng.standard_normal(H)).astype(np.float32)
    wgu = (0.02 * rng.standard_normal((2 * I, H))).astype(np.float32)
    wd = (0.02 * rng.standard_normal((H, I))).astype(np.float32)
    return tuple(synth.to_bf16_bits(a) for a in (x, nw, wgu, wd))


def _weights(bits, gran):
    w_q, w_s, w_rs = lc.quantize_weights_g(dev_bf16(bits), gran)
    torch.cuda.synchronize()
    return w_q, w_s, w_rs


@pytest.mark.parametrize("gran,ogran", GRANS)
def test_weight_codes_and_row_scales_bit_exact(gran, ogran):
    _, _, wgu, wd = _inputs(8, 256, 384)
    for bits in (wgu, wd):
        w_q, w_s, w_rs = _weights(bits, gran)
        rq, rrs = G.quant_weights_g(bits, ogran)
        gq = lc.weight_codes_rowmajor(w_q)  # the device holds the codes in tiles
        assert np.array_equal(gq, rq), "codes differ in %d places" % int((gq != rq).sum())
        assert np.array_equal(host(w_rs).view(np.uint32), rrs.view(np.uint32))
        assert np.all(host(w_s) == 1.0)


@pytest.mark.parametrize("M", [1, 37, 200])
def test_rmsnorm_f32_bit_exact(M):
    x, nw, _, _ = _inputs(M, 1024, 256)
    y = torch.full((M, 1024), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_rmsnorm_f32(dev_bf16(x), dev_bf16(nw), y)
    torch.cuda.synchronize()
    ry, _ = O.rmsnorm(x, nw)
    assert np.array_equal(host(y).view(np.uint32), ry.view(np.uint32))


@pytest.mark.parametrize("gran,ogran", GRANS + [(lc.LACACHE_GRAN_GROUP, None)])
@pytest.mark.parametrize("M,K", [(1, 256), (37, 1024), (200, 768)])
def test_quant_rows_bit_exact(gran, ogran, M, K):
    rng = np.random.default_rng(M + K)
    v = (rng.standard_normal((M, K)) * np.exp(rng.uniform(-4, 4, (M, 1)))).astype(np.float32)
    v[0, :] = 0.0  # an all-zero row
    if M > 2:
        v[2, 5] = np.float32(3e4)
    q = torch.full((M, K), 0xFF, dtype=torch.uint8, device=DEV)
    s_kgm = torch.full((K // 128, M), float("nan"), dtype=torch.float32, device=DEV)
    s_rows = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_quant_rows_g(torch.from_numpy(v).to(DEV), q, s_kgm, None if ogran is None else s_rows, gran)
    torch.cuda.synchronize()
    if ogran is None:
        rq, rs = O.requant(v)
        assert np.array_equal(host(q), rq)
        assert np.array_equal(host(s_kgm).view(np.uint32), rs.view(np.uint32))
        return
    rq, rs = G.quantize_rows(v, ogran)
    assert np.array_equal(host(q), rq), "codes differ in %d places" % int((host(q) != rq).sum())
    assert np.array_equal(host(s_rows).view(np.uint32), rs.view(np.uint32))
    assert np.array_equal(host(s_kgm).view(np.uint32), np.tile(rs, (K // 128, 1)).view(np.uint32))


@pytest.mark.parametrize("M,K", [(3, 2048), (3, 2176), (5, 4096), (4, 4224), (3, 8192), (2, 12288), (3, 16384),
                                 (37, 16512)])
def test_quant_rows_per_token_at_every_row_length(M, K):
    """One scale per row, held in 1, 2, 4 or 8 passes of a workgroup's registers
    (K <= 2048, 4096, 8192, 16384; full and partly filled last passes, the
    maximum in the last values of a row) and, above, in three kernels."""
    _say("per-token rows M=%d K=%d" % (M, K))
    rng = np.random.default_rng(M + K)
    v = (rng.standard_normal((M, K)) * np.exp(rng.uniform(-4, 4, (M, 1)))).astype(np.float32)
    v[0, :] = 0.0
    v[1, K - 1] = np.float32(-9e3)
    q = torch.full((M, K), 0xFF, dtype=torch.uint8, device=DEV)
    s_kgm = torch.full((K // 128, M), float("nan"), dtype=torch.float32, device=DEV)
    s_rows = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_quant_rows_g(torch.from_numpy(v).to(DEV), q, s_kgm, s_rows, lc.LACACHE_GRAN_TOKEN)
    torch.cuda.synchronize()
    rq, rs = G.quantize_rows(v, G.GRAN_TOKEN)
    assert np.array_equal(host(q), rq), "codes differ in %d places" % int((host(q) != rq).sum())
    assert np.array_equal(host(s_rows).view(np.uint32), rs.view(np.uint32))
    assert np.array_equal(host(s_kgm).view(np.uint32), np.tile(rs, (K // 128, 1)).view(np.uint32))


def _quantize_any(v):
    """Codes and scale of each set v[i] (NaN and infinite values included): the
    scale from the largest magnitude that is not NaN, a NaN quotient clipped to
    -448, every code 0 where the scale is 0."""
    with np.errstate(invalid="ignore", over="ignore"):
        s = (np.fmax.reduce(np.abs(v), axis=1, initial=np.float32(0)) / np.float32(448)).astype(np.float32)
        u = v / np.where(s == 0, np.float32(1), s)[:, None]
    u = np.where(np.isnan(u), np.float32(-448), np.clip(u, np.float32(-448), np.float32(448)))
    codes = csweep.encode_f32(np.ascontiguousarray(u.astype(np.float32)).ravel()).reshape(v.shape)
    return np.where((s == 0)[:, None], np.uint8(0), codes), s


@pytest.mark.parametrize("gran,K", [(lc.LACACHE_GRAN_GROUP, 1024), (lc.LACACHE_GRAN_TOKEN, 1024),
                                    (lc.LACACHE_GRAN_TOKEN, 12288), (lc.LACACHE_GRAN_TOKEN, 16512),
                                    (lc.LACACHE_GRAN_TENSOR, 1024)])
def test_quantizers_on_nans_and_infinities(gran, K):
    """NaNs are left out of the maximum and take the code of -448; an infinite
    value makes the scale infinite: itself the code of -448, the others zero.
    Scales below the fast quantizer's range and the largest magnitudes as well."""
    _say("quantizer %d on NaNs, K=%d" % (gran, K))
    csweep.build_csweep()
    rng = np.random.default_rng(K)
    M = 12
    v = rng.standard_normal((M, K)).astype(np.float32)
    v[1, 3], v[2, K - 1] = np.nan, np.inf
    v[3, 130], v[3, 131], v[4, :] = -np.inf, np.nan, np.nan
    v[5, ::7] = np.nan
    v[6, 64], v[6, 65] = np.float32(3.4e38), np.float32(-0.0)
    v[7] *= np.float32(1e-40)  # subnormal values and scale
    v[8] *= np.float32(1e-30)  # the scale is below 2^-100
    v[9] *= np.float32(1e-36)
    v[9, 9] = np.nan
    v.view(np.uint32)[10, 20:24] = [0x7F800001, 0xFF800001, 0xFFC12345, 0x7FFFFFFF]
    v[11] = np.float32(-0.0)
    sets = [v] if gran != lc.LACACHE_GRAN_TENSOR else [v, np.where(np.isinf(v), np.float32(2), v)]
    for x in sets:
        if gran == lc.LACACHE_GRAN_GROUP:
            rq, rs = _quantize_any(x.reshape(-1, 128))
            rq, kgm = rq.reshape(M, K), rs.reshape(M, K // 128).T
        elif gran == lc.LACACHE_GRAN_TOKEN:
            rq, rs = _quantize_any(x)
            kgm = np.tile(rs, (K // 128, 1))
        else:
            rq, rs = _quantize_any(x.reshape(1, -1))
            rq, kgm = rq.reshape(M, K), np.full((K // 128, M), rs[0], dtype=np.float32)
        q = torch.full((M, K), 0xAA, dtype=torch.uint8, device=DEV)
        s_kgm = torch.full((K // 128, M), float("nan"), dtype=torch.float32, device=DEV)
        s_rows = None if gran == lc.LACACHE_GRAN_GROUP else torch.full((M,), 7.0, dtype=torch.float32, device=DEV)
        lc.lacache_quant_rows_g(torch.from_numpy(x).to(DEV), q, s_kgm, s_rows, gran)
        torch.cuda.synchronize()
        assert np.array_equal(host(s_kgm).view(np.uint32), np.ascontiguousarray(kgm).view(np.uint32))
        bad = np.argwhere(host(q) != rq)
        assert not len(bad), (bad[:4], host(q)[tuple(bad[0])], rq[tuple(bad[0])])


def _row_gemm_bound(aq, a_rows, bq, b_rows, acc_abs):
    """|acc_gpu - acc_exact| for acc = (sum_kb P_kb a_s[m]) * b_s[n] in fp32:
    the MFMA chunk truncation of every group, the fp32 rounding of each group
    result, of the accumulation and of the final column scale."""
    KB = aq.shape[1] // 128
    dots = mfma_dot_bound(aq, bq)
    bound = np.zeros((aq.shape[0], bq.shape[0]))
    mag = np.zeros_like(bound)
    for kb in range(KB):
        cols = slice(kb * 128, (kb + 1) * 128)
        P = np.abs(O.dequant_codes(aq[:, cols]) @ O.dequant_codes(bq[:, cols]).T)
        bound += dots[kb] + 2.0 ** -24 * P
        mag += P
    s = np.abs(a_rows.astype(np.float64))[:, None] * np.abs(b_rows.astype(np.float64))[None, :]
    return s * (bound + (KB + 18) * 2.0 ** -24 * mag) + 2.0 ** -23 * acc_abs


@pytest.mark.parametrize("gran,ogran", GRANS)
@pytest.mark.parametrize("M,H,I", [(64, 256, 768), (200, 1024, 2048)])
def test_gemms_against_the_oracle(gran, ogran, M, H, I):
    x, nw, wgu, wd = _inputs(M, H, I, seed=M)
    _say("granularity %d M=%d H=%d I=%d" % (gran, M, H, I))
    wgu_q, wgu_s, wgu_rs = _weights(wgu, gran)
    wd_q, wd_s, wd_rs = _weights(wd, gran)
    y = torch.empty((M, H), dtype=torch.float32, device=DEV)
    xq = torch.empty((M, H), dtype=torch.uint8, device=DEV)
    xs = torch.empty((H // 128, M), dtype=torch.float32, device=DEV)
    xr = torch.empty((M,), dtype=torch.float32, device=DEV)
    h = torch.full((M, I), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_rmsnorm_f32(dev_bf16(x), dev_bf16(nw), y)
    lc.lacache_quant_rows_g(y, xq, xs, xr, gran)
    lc.lacache_gateup_swiglu_f32(xq, xs, wgu_q, wgu_s, wgu_rs, h)
    torch.cuda.synchronize()
    # gate/up + SwiGLU against the exact fp64 result of the GPU's own codes
    aq, ar, bq, br = host(xq), host(xr), lc.weight_codes_rowmajor(wgu_q), host(wgu_rs)
    acc = G.scaled_gemm(aq, ar, bq, br)
    dacc = _row_gemm_bound(aq, ar, bq, br, np.abs(acc))
    g, u, dg, du = acc[:, :I], acc[:, I:], dacc[:, :I], dacc[:, I:]
    h64 = O.silu(g) * u
    dh = SILU_LIP * dg * (np.abs(u) + du) + np.abs(O.silu(g)) * du
    dh = dh + 2.0 ** -20 * (np.abs(h64) + dh)
    hg = host(h).astype(np.float64)
    assert np.all(np.isfinite(hg))
    worst = float((np.abs(hg - h64) / np.maximum(dh, 1e-300)).max())
    _say("  h: worst err/bound %.3f" % worst)
    assert worst <= 1.0
    # re-quantization of the GPU's own h: bit-exact
    hq = torch.empty((M, I), dtype=torch.uint8, device=DEV)
    hs = torch.empty((I // 128, M), dtype=torch.float32, device=DEV)
    hr = torch.empty((M,), dtype=torch.float32, device=DEV)
    lc.lacache_quant_rows_g(h, hq, hs, hr, gran)
    out = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    tap = torch.full((M, H), float("nan"), dtype=torch.float32, device=DEV)
    lc.lacache_down_proj_g(hq, hs, wd_q, wd_s, wd_rs, out, tap)
    torch.cuda.synchronize()
    rq, rr = G.quantize_rows(host(h), ogran)
    assert np.array_equal(host(hq), rq) and np.array_equal(host(hr).view(np.uint32), rr.view(np.uint32))
    # down on the same operands: fp32 within 2e-3 of the row max, bf16 = RNE(fp32)
    out64 = G.scaled_gemm(host(hq), host(hr), lc.weight_codes_rowmajor(wd_q), host(wd_rs))
    o32 = host(tap).astype(np.float64)
    e = float((np.abs(o32 - out64) / np.maximum(np.abs(out64).max(axis=1, keepdims=True), 1e-300)).max())
    _say("  out: err %.2e" % e)
    assert e <= 2e-3
    assert np.array_equal(host_bf16(out), rne_bf16(host(tap)))


@pytest.mark.parametrize("gran", [lc.LACACHE_GRAN_TOKEN, lc.LACACHE_GRAN_TENSOR])
@pytest.mark.parametrize("M", [32, 200])
def test_fused_call_equals_its_stages(gran, M):
    H, I = 1024, 2048
    x, nw, wgu, wd = _inputs(M, H, I, seed=3)
    wgu_q, wgu_s, wgu_rs = _weights(wgu, gran)
    wd_q, wd_s, wd_rs = _weights(wd, gran)
    xd, nwd = dev_bf16(x), dev_bf16(nw)
    fused = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    lc.lacache_ffn_fp8_g(xd, nwd, wgu_q, wgu_s, wgu_rs, wd_q, wd_s, wd_rs, fused, gran)
    y = torch.empty((M, H), dtype=torch.float32, device=DEV)
    xq = torch.empty((M, H), dtype=torch.uint8, device=DEV)
    xs = torch.empty((H // 128, M), dtype=torch.float32, device=DEV)
    r = torch.empty((M,), dtype=torch.float32, device=DEV)
    h = torch.empty((M, I), dtype=torch.float32, device=DEV)
    hq = torch.empty((M, I), dtype=torch.uint8, device=DEV)
    hs = torch.empty((I // 128, M), dtype=torch.float32, device=DEV)
    staged = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    lc.lacache_rmsnorm_f32(xd, nwd, y)
    lc.lacache_quant_rows_g(y, xq, xs, r, gran)
    lc.lacache_gateup_swiglu_f32(xq, xs, wgu_q, wgu_s, wgu_rs, h)
    lc.lacache_quant_rows_g(h, hq, hs, r, gran)
    lc.lacache_down_proj_g(hq, hs, wd_q, wd_s, wd_rs, staged)
    again = torch.empty_like(fused)
    lc.lacache_ffn_fp8_g(xd, nwd, wgu_q, wgu_s, wgu_rs, wd_q, wd_s, wd_rs, again, gran)
    torch.cuda.synchronize()
    assert torch.equal(fused.view(torch.int16), staged.view(torch.int16))
    assert torch.equal(fused.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("M,H,I", [(3, 128, 16512), (40, 640, 2176), (33, 1536, 256), (40, 2176, 256),
                                   (40, 4096, 4224), (1100, 4096, 256), (1030, 1024, 256), (9, 8192, 8320),
                                   (5, 16384, 128)])
def test_per_token_call_equals_its_stages_at_every_row_length(M, H, I):
    """The one-kernel norm + per-token quantization at 1 to 32 passes, one, two
    and four wavefronts to a row (and one to a row above 1024 rows, four rows to
    a workgroup), and h rows of every length class: the fused call is the staged
    one bit for bit, whose norm and quantizer have oracles."""
    _say("per-token M=%d H=%d I=%d" % (M, H, I))
    gran = lc.LACACHE_GRAN_TOKEN
    x, nw, wgu, wd = _inputs(M, H, I, seed=M + H)
    x[0] = 0
    wgu_q, wgu_s, wgu_rs = _weights(wgu, gran)
    wd_q, wd_s, wd_rs = _weights(wd, gran)
    xd, nwd = dev_bf16(x), dev_bf16(nw)
    fused = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    lc.lacache_ffn_fp8_g(xd, nwd, wgu_q, wgu_s, wgu_rs, wd_q, wd_s, wd_rs, fused, gran)
    y = torch.empty((M, H), dtype=torch.float32, device=DEV)
    xq = torch.empty((M, H), dtype=torch.uint8, device=DEV)
    xs = torch.empty((H // 128, M), dtype=torch.float32, device=DEV)
    r = torch.empty((M,), dtype=torch.float32, device=DEV)
    h = torch.empty((M, I), dtype=torch.float32, device=DEV)
    hq = torch.empty((M, I), dtype=torch.uint8, device=DEV)
    hs = torch.empty((I // 128, M), dtype=torch.float32, device=DEV)
    staged = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    lc.lacache_rmsnorm_f32(xd, nwd, y)
    lc.lacache_quant_rows_g(y, xq, xs, r, gran)
    lc.lacache_gateup_swiglu_f32(xq, xs, wgu_q, wgu_s, wgu_rs, h)
    torch.cuda.synchronize()
    rows = np.unique([0, 1, M // 2, M - 1])
    rq, rs = G.quantize_rows(O.rmsnorm(x[rows], nw)[0], G.GRAN_TOKEN)
    assert np.array_equal(host(xq)[rows], rq) and np.array_equal(host(r)[rows].view(np.uint32), rs.view(np.uint32))
    lc.lacache_quant_rows_g(h, hq, hs, r, gran)
    lc.lacache_down_proj_g(hq, hs, wd_q, wd_s, wd_rs, staged)
    torch.cuda.synchronize()
    assert torch.equal(fused.view(torch.int16), staged.view(torch.int16))


def test_group_granularity_is_the_library_ffn():
    M, H, I = 64, 256, 768
    x, nw, wgu, wd = _inputs(M, H, I, seed=5)
    wgu_q, wgu_s, none1 = _weights(wgu, lc.LACACHE_GRAN_GROUP)
    wd_q, wd_s, none2 = _weights(wd, lc.LACACHE_GRAN_GROUP)
    assert none1 is None and none2 is None
    a = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
    b = torch.empty_like(a)
    lc.lacache_ffn_fp8_g(dev_bf16(x), dev_bf16(nw), wgu_q, wgu_s, None, wd_q, wd_s, None, a, lc.LACACHE_GRAN_GROUP)
    lc.lacache_ffn_fp8(dev_bf16(x), dev_bf16(nw), wgu_q, wgu_s, wd_q, wd_s, b)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_coarser_granularity_loses_more_accuracy_on_the_gpu():
    """Table fp8-granularities' ordering on the GPU's outputs: against the
    unquantized bf16 FFN of the same inputs, per-group < per-token < per-tensor."""
    M, H, I = 128, 1024, 2048
    x, nw, wgu, wd = _inputs(M, H, I, seed=11)
    I2 = I
    ref = O.ffn_bf16_reference(x, nw, wgu[:I2], wgu[I2:], wd)
    errs = {}
    for name, gran in (("group", lc.LACACHE_GRAN_GROUP), ("token", lc.LACACHE_GRAN_TOKEN),
                       ("tensor", lc.LACACHE_GRAN_TENSOR)):
        wgu_q, wgu_s, wgu_rs = _weights(wgu, gran)
        wd_q, wd_s, wd_rs = _weights(wd, gran)
        out = torch.empty((M, H), dtype=torch.bfloat16, device=DEV)
        lc.lacache_ffn_fp8_g(dev_bf16(x), dev_bf16(nw), wgu_q, wgu_s, wgu_rs, wd_q, wd_s, wd_rs, out, gran)
        torch.cuda.synchronize()
        got = bf16_to_f32(host_bf16(out)).astype(np.float64)
        errs[name] = float(np.sqrt(((got - ref) ** 2).mean() / (ref ** 2).mean()))
    _say("rms error vs the bf16 FFN: %s" % errs)
    assert errs["group"] < errs["token"] < errs["tensor"], errs
