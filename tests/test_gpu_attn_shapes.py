"""The prefill attention's launch shapes (attn_shape.h; the sizes below take
each of them on 256 CUs) against the oracle: every code format, ragged
lengths whose last tile and last workgroup are partial, the per-query window,
and full-precision V beyond the f16 range (each key group raises its own
reference scale before the groups are merged)."""
import numpy as np
import pytest

import gpu_common as gc
from oracle import hyq_oracle as orc
from paper_2608_27875_amd import gen

hyq = gc.hyq
pytestmark = pytest.mark.gpu

# kind: (B, Hq, Hkv, L), and where nothing quantized takes another kind (a test of
# the policy checks each).  32-row units in all -> split8: 5, 175 (110);
# split2: 924; half: 1520 (520); full: 2528
SHAPES = {"split8_tiny": (1, 1, 1, 131), "split8": (1, 5, 1, 1111), "split2": (2, 14, 2, 1051),
          "half": (1, 40, 8, 1201), "full": (1, 32, 8, 2501)}
DENSE_SHAPES = {"split8": (1, 5, 1, 700), "half": (1, 40, 8, 401)}
FORMATS = {"int8": (8, hyq.FMT_INT), "int4": (4, hyq.FMT_INT), "fp8": (8, hyq.FMT_FP8),
           "fp4": (4, hyq.FMT_FP4), "fp4q6": (4, hyq.FMT_FP4Q6), "bf16": (16, hyq.FMT_INT)}


def shape_for(kind, fmt):
    return DENSE_SHAPES.get(kind, SHAPES[kind]) if fmt == "bf16" else SHAPES[kind]


def _run(kind, fmt, W, band=False, big_v=()):
    B, Hq, Hkv, L = shape_for(kind, fmt)
    bits, f = FORMATS[fmt]
    d = gen.generate(5, 500 + L, B=B, Hq=Hq, Hkv=Hkv, L=L, D=128, W=W, plant=0.03)
    if big_v:
        x = gen.bf16_bits_to_f32(d["V"])
        for pos, ch, v in big_v:
            x[..., pos, ch] = v
        d["V"] = gen.f32_to_bf16_bits(x)
    shape = hyq.Shape(B=B, Hq=Hq, Hkv=Hkv, L=L, window=W, budget_ppm=50000, bits_kv=bits,
                      kv_format=f, window_mode=hyq.WIN_BAND if band else hyq.WIN_FIXED)
    t = tuple(gc.to_dev(d[n]) for n in ("Q", "K", "V"))
    b = hyq.alloc_buffers(shape, t[0].device)
    out = hyq.prefill(shape, *t, b).cpu().numpy()
    idx, _ = orc.select_vertical(d["Q"], d["K"], Hkv, W, 50000)
    np.testing.assert_array_equal(b["idx"].cpu().numpy(), idx)
    qz = orc.quantize(d["Q"], d["K"], d["V"], idx, W, bits,
                      fmt=gc.fmt_name(shape) if bits != 16 else "int")
    heads = [(0, 0), (B - 1, Hq - 1)] if Hq > 1 else [(0, 0)]
    rows = gc.sample_rows(L, W, 70, 1)
    rows = np.union1d(rows, [31, 32, 63, 64, 65, min(L - 1, 700)])
    O = orc.attention(d["Q"], d["K"], d["V"], W, bits, idx, qz, heads=heads, rows=rows,
                      window_mode="band" if band else "fixed")
    return np.stack([out[bb, h][rows] for bb, h in heads]), O


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("kind", SHAPES)
def test_shapes(kind, fmt):
    G, O = _run(kind, fmt, W=100)
    mx, mean = gc.attention_error(G, O)
    assert mx <= gc.TOL_MAX and mean <= gc.TOL_MEAN, (mx, mean)


@pytest.mark.parametrize("fmt", ["int8", "fp4q6"])
@pytest.mark.parametrize("kind", SHAPES)
def test_band(kind, fmt):
    G, O = _run(kind, fmt, W=90, band=True)
    mx, mean = gc.attention_error(G, O)
    assert mx <= gc.TOL_MAX and mean <= gc.TOL_MEAN, (mx, mean)


@pytest.mark.parametrize("fmt", ["int8", "bf16"])
@pytest.mark.parametrize("kind", ["split8", "split2", "half", "full"])
def test_v_beyond_f16(kind, fmt):
    L = shape_for(kind, fmt)[3]
    G, O = _run(kind, fmt, W=200, big_v=[(L - 170, 7, 1.0e5), (L - 60, 20, -3.0e6)])
    keep = ~np.isin(np.arange(128), [7, 20])
    mx, mean = gc.attention_error(G[..., keep], O[..., keep])
    assert gc.scaled_error(G, O) <= gc.TOL_MAX and mx <= gc.TOL_MAX and mean <= gc.TOL_MEAN


# V so large that the unnormalised row sum (weights of up to L nearly equal
# keys times V) leaves float32 although the output does not: every shape
# divides by the row sum before it scales by V's reference.  (FP8 V codes:
# with the reference at its largest, 2^100, block scales up to 2^107 keep
# 448 * 2^7 within f16, so V may reach 448 * 2^107 = 7e34; int8 codes, whose
# conversion adds 1152 * 2^e, end at 127 * 2^105 = 5e33.)
ROW_SUM = [("split8", 1, 5, 1, 700, "bf16", 1e36), ("split2", 2, 14, 2, 703, "bf16", 1e36),
           ("full", 1, 32, 8, 2501, "bf16", 1e36), ("split8", 1, 1, 1, 16384, "fp8", 3e34),
           ("split2", 1, 2, 1, 16384, "fp8", 3e34)]
ROW_SUM_W = 128


@pytest.mark.parametrize("kind,B,Hq,Hkv,L,fmt,v", ROW_SUM)
def test_row_sum_beyond_float32(kind, B, Hq, Hkv, L, fmt, v):
    bits, f = FORMATS[fmt]
    W = ROW_SUM_W
    d = gen.generate(6, 600 + L, B=B, Hq=Hq, Hkv=Hkv, L=L, D=128, W=W, plant=0.0)
    d["Q"] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(d["Q"]) * np.float32(2.0 ** -6))
    d["V"] = gen.f32_to_bf16_bits(np.float32(v) * (1 + np.float32(0.1) *
                                                   gen.bf16_bits_to_f32(d["V"])))
    shape = hyq.Shape(B=B, Hq=Hq, Hkv=Hkv, L=L, window=W, budget_ppm=10000, bits_kv=bits,
                      kv_format=f)
    assert v * 0.9 * L > float(np.finfo(np.float32).max)
    t = tuple(gc.to_dev(d[n]) for n in ("Q", "K", "V"))
    out = hyq.prefill(shape, *t, hyq.alloc_buffers(shape, t[0].device)).cpu().numpy()
    idx, _ = orc.select_vertical(d["Q"], d["K"], Hkv, W, 10000)
    qz = orc.quantize(d["Q"], d["K"], d["V"], idx, W, bits, fmt=gc.fmt_name(shape))
    heads = [(B - 1, Hq - 1)]
    rows = gc.sample_rows(L, W, 40, 1)
    O = orc.attention(d["Q"], d["K"], d["V"], W, bits, idx, qz, heads=heads, rows=rows)
    G = np.stack([out[b, h][rows] for b, h in heads])
    mx, mean = gc.attention_error(G.astype(np.float64) / v, O.astype(np.float64) / v)
    assert mx <= gc.TOL_MAX and mean <= gc.TOL_MEAN, (mx, mean)


# A future V row must not reach earlier rows, however large or undefined it
# is.  With 8 heads to a KV head a workgroup's rows end inside a 64-key tile
# (8 or 4 units are 32 rows, as is kSplit8's one), so the rows before p are
# bit for bit what they are with any other V from p on.
FUTURE_V = [("split8", 1, 8, 1, 500, "bf16"), ("split2", 1, 24, 3, 600, "bf16"),
            ("half", 1, 24, 3, 400, "bf16"), ("full", 2, 64, 8, 600, "bf16"),
            ("split8", 1, 8, 1, 500, "int8"), ("split2", 1, 24, 3, 1100, "int8"),
            ("half", 2, 32, 4, 600, "int8"), ("full", 2, 64, 8, 600, "int8")]
FUTURE_V_W = 200


@pytest.mark.parametrize("v", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("kind,B,Hq,Hkv,L,fmt", FUTURE_V)
def test_future_v_is_not_seen(kind, B, Hq, Hkv, L, fmt, v):
    bits, f = FORMATS[fmt]
    W = FUTURE_V_W
    d = gen.generate(7, 700 + L, B=B, Hq=Hq, Hkv=Hkv, L=L, D=128, W=W, plant=0.02)
    shape = hyq.Shape(B=B, Hq=Hq, Hkv=Hkv, L=L, window=W, budget_ppm=20000, bits_kv=bits,
                      kv_format=f)
    p = (L - 60) // 64 * 64 + 32   # in the window, the second half of a tile
    assert L - W <= p < L
    Q, K, V = (gc.to_dev(d[n]) for n in ("Q", "K", "V"))
    out = []
    for x in (1.0, v):
        V[:, :, p:] = x
        b = hyq.alloc_buffers(shape, V.device)
        out.append(hyq.prefill(shape, Q, K, V, b)[:, :, :p].cpu().numpy())
    assert np.isfinite(out[0]).all()
    np.testing.assert_array_equal(out[1].view(np.uint32), out[0].view(np.uint32))
