"""hyq_prefill shares launches between selection and quantization, the top-k
runs as one launch on short prefixes and on longer ones of many heads, and the
K/V quantizer finds its rows from the vertical list: each against the oracle or the three calls at
the sizes where it can go wrong."""
import numpy as np
import pytest

import gpu_common as gc
from oracle import hyq_oracle as orc
from paper_2608_27875_amd import gen

hyq = gc.hyq
pytestmark = pytest.mark.gpu

BUFS = ("kq_pos", "q_codes", "k_codes", "v_codes", "q_scale", "k_scale", "v_scale")


@pytest.mark.parametrize("bits,fmt", [(8, hyq.FMT_INT), (4, hyq.FMT_INT), (8, hyq.FMT_FP8),
                                      (4, hyq.FMT_FP4), (4, hyq.FMT_FP4Q6), (16, hyq.FMT_INT)])
@pytest.mark.parametrize("L,W,ppm,sel", [(65, 64, 20000, 0), (1000, 100, 50000, 0),
                                         (700, 64, 1000000, 0), (130, 64, 0, 0), (60, 64, 20000, 0),
                                         (1000, 100, 50000, 1)])
def test_prefill_equals_the_three_calls(bits, fmt, L, W, ppm, sel):
    import torch
    d = gen.generate(1, 300 + L, B=2, Hq=6, Hkv=2, L=L, D=128, W=W, plant=0.02)
    shape = hyq.Shape(B=2, Hq=6, Hkv=2, L=L, window=W, budget_ppm=ppm, bits_kv=bits, kv_format=fmt,
                      selector=sel)
    t = tuple(gc.to_dev(d[n]) for n in ("Q", "K", "V"))
    g = gc.run_gpu(shape, d, tensors=t)
    b = hyq.alloc_buffers(shape, t[0].device)
    out = hyq.prefill(shape, *t, b)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), g["out"].view(np.uint32))
    np.testing.assert_array_equal(b["idx"].cpu().numpy(), g["idx"])
    for n in BUFS if bits != 16 else ():
        np.testing.assert_array_equal(b[n].cpu().numpy().view(np.uint8), g[n].view(np.uint8),
                                      err_msg=n)


# block scales near the ends of the reciprocal's range, below it and above it
@pytest.mark.parametrize("bits,fmt", [(8, hyq.FMT_INT), (8, hyq.FMT_FP8), (4, hyq.FMT_FP4),
                                      (4, hyq.FMT_FP4Q6)])
@pytest.mark.parametrize("e", [-130, -100, -58, -50, 100, 122])
def test_codes_of_tiny_and_huge_blocks(bits, fmt, e):
    d = gen.generate(2, 77, B=1, Hq=2, Hkv=1, L=200, D=128, W=8, plant=0.0)
    for n in ("Q", "K", "V"):
        x = np.ldexp(gen.bf16_bits_to_f32(d[n]).astype(np.float64), e).astype(np.float32)
        d[n] = gen.f32_to_bf16_bits(x)
        d[n][..., 5] = 0x8000   # -0 keeps its sign in the floating-point formats
    shape = hyq.Shape(B=1, Hq=2, Hkv=1, L=200, window=8, budget_ppm=0, bits_kv=bits, kv_format=fmt)
    b = hyq.alloc_buffers(shape, "cuda")
    hyq.hyq_quantize(shape, *(gc.to_dev(d[n]) for n in ("Q", "K", "V")), b["idx"],
                     b["q_codes"], b["q_scale"], b["k_codes"], b["k_scale"], b["v_codes"],
                     b["v_scale"], b["kq_pos"])
    g = {n: b[n].cpu().numpy() for n in BUFS}
    g["sizes"] = b["sizes"]
    c = gc.canonical(shape, g)
    qz = orc.quantize(d["Q"], d["K"], d["V"], np.zeros((1, 1, 0), np.int32), 8, bits,
                      fmt=gc.fmt_name(shape))
    for n in BUFS:
        np.testing.assert_array_equal(c[n], qz[n], err_msg=n)


# vertical lists the evenly spread guess misses: runs longer than the staged
# span at either end and in the middle, everything but a few keys, every other
@pytest.mark.parametrize("kind", ["head", "tail", "middle", "most", "alternate"])
def test_partition_of_clustered_lists(kind):
    import torch
    L, W = 3000, 64
    P = L - W
    pos = {"head": np.arange(700), "tail": np.arange(P - 700, P),
           "middle": np.concatenate([[0, 5], np.arange(1000, 1698)]),
           "most": np.delete(np.arange(P), np.arange(3, P, 97)),
           "alternate": np.arange(0, P, 2)}[kind].astype(np.int32)
    k = len(pos)
    ppm = next(x for x in range(int(k * 1e6 // P) - 400, 1000001)
               if orc.sizes(L, W, x)["k"] == k)
    shape = hyq.Shape(B=1, Hq=1, Hkv=1, L=L, window=W, budget_ppm=ppm, bits_kv=8)
    d = gen.generate(3, 78, B=1, Hq=1, Hkv=1, L=L, D=128, W=W, plant=0.0)
    b = hyq.alloc_buffers(shape, "cuda")
    b["idx"].copy_(torch.from_numpy(pos).view(1, 1, k))
    hyq.hyq_quantize(shape, *(gc.to_dev(d[n]) for n in ("Q", "K", "V")), b["idx"],
                     b["q_codes"], b["q_scale"], b["k_codes"], b["k_scale"], b["v_codes"],
                     b["v_scale"], b["kq_pos"])
    want = np.setdiff1d(np.arange(P), pos)
    got = b["kq_pos"].cpu().numpy()
    np.testing.assert_array_equal(got[:len(want)], want)
    assert np.all(got[len(want):] == hyq.KQ_POS_PAD)


# the shortest prefixes, and both sides of a window of the final pass's bitmaps
@pytest.mark.timeout(300)
@pytest.mark.parametrize("P", [1, 63, 1024, 1025, 8192, 131072, 131073])
def test_topk_prefix_lengths(P):
    W = 16
    d = gen.generate(4, 79, B=1, Hq=1, Hkv=1, L=P + W, D=128, W=W, plant=0.01)
    shape = hyq.Shape(B=1, Hq=1, Hkv=1, L=P + W, window=W, budget_ppm=30000, bits_kv=8)
    b = hyq.alloc_buffers(shape, "cuda")
    hyq.hyq_select_vertical(shape, gc.to_dev(d["Q"]), gc.to_dev(d["K"]), b["idx"], None, b["ws"])
    idx, _ = orc.select_vertical(d["Q"], d["K"], 1, W, 30000)
    np.testing.assert_array_equal(b["idx"].cpu().numpy(), idx)


# the selection's workspace may lie in memory that the quantization or the
# attention writes afterwards
@pytest.mark.parametrize("over", ["q_codes", "q_scale", "k_codes", "out"])
@pytest.mark.parametrize("sel", [0, 1])
def test_prefill_with_the_workspace_in_a_later_buffer(over, sel):
    import torch
    d = gen.generate(1, 301, B=2, Hq=6, Hkv=2, L=1000, D=128, W=100, plant=0.02)
    shape = hyq.Shape(B=2, Hq=6, Hkv=2, L=1000, window=100, budget_ppm=50000, bits_kv=8,
                      selector=sel)
    t = tuple(gc.to_dev(d[n]) for n in ("Q", "K", "V"))
    g = gc.run_gpu(shape, d, tensors=t)
    b = hyq.alloc_buffers(shape, t[0].device)
    own = b[over].numel() * b[over].element_size()
    n = max(own, b["ws"].numel())
    mem = torch.zeros((n + 15) // 16 * 16, dtype=torch.uint8, device=t[0].device)
    b["ws"] = mem[:b["ws"].numel()]
    b[over] = mem[:own].view(b[over].dtype).view(b[over].shape)
    out = hyq.prefill(shape, *t, b)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), g["out"].view(np.uint32))
    np.testing.assert_array_equal(b["idx"].cpu().numpy(), g["idx"])
    for n in BUFS:
        np.testing.assert_array_equal(b[n].cpu().numpy().view(np.uint8), g[n].view(np.uint8),
                                      err_msg=n)


# both sides of the lines between the one-launch top-k and the classification:
# 24576 keys, then 1536 per head, from 48 heads on 131072.  The scores are
# checked elsewhere, here the choice among them.
@pytest.mark.parametrize("heads,P", [(1, 24576), (1, 24577), (17, 26112), (17, 26113), (48, 131072),
                                     (48, 131073)])
def test_topk_lines(heads, P):
    import torch
    W = 64
    shape = hyq.Shape(B=1, Hq=heads, Hkv=heads, L=P + W, window=W, budget_ppm=20000)
    gen_ = torch.Generator(device="cuda").manual_seed(9)
    Q, K = (torch.randn((1, heads, P + W, 128), generator=gen_, device="cuda",
                        dtype=torch.bfloat16) for _ in range(2))
    z = hyq.hyq_sizes_for(shape)
    idx = torch.empty((1, heads, z["k"]), dtype=torch.int32, device="cuda")
    scores = torch.empty((1, heads, P), device="cuda")
    ws = torch.empty(z["select_ws_bytes"], dtype=torch.uint8, device="cuda")
    hyq.hyq_select_vertical(shape, Q, K, idx, scores, ws)
    order = torch.sort(scores, dim=-1, descending=True, stable=True).indices[..., :z["k"]]
    assert torch.equal(idx.long(), order.sort().values)


# 2^21 query heads: eight tail-proxy workgroups each are 2^32 threads, more
# than one dimension of a launch holds
def test_select_over_very_many_heads():
    import torch
    B, g = 1 << 18, 8
    shape = hyq.Shape(B=B, Hq=g, Hkv=1, L=2, window=1, budget_ppm=1000000)
    gen_ = torch.Generator(device="cuda").manual_seed(8)
    Q = torch.randn((B, g, 2, 128), generator=gen_, device="cuda", dtype=torch.bfloat16)
    K = torch.randn((B, 1, 2, 128), generator=gen_, device="cuda", dtype=torch.bfloat16)
    z = hyq.hyq_sizes_for(shape)
    idx = torch.full((B, 1, z["k"]), -1, dtype=torch.int32, device="cuda")
    scores = torch.full((B, 1, z["P"]), float("nan"), device="cuda")
    ws = torch.empty(z["select_ws_bytes"], dtype=torch.uint8, device="cuda")
    hyq.hyq_select_vertical(shape, Q, K, idx, scores, ws)
    assert int(idx.abs().max()) == 0
    want = (Q[:, :, 1].double().sum(1) * K[:, 0, 0].double()).sum(-1)
    # 7 float32 additions per channel, 128 products, a tree of 7 levels
    bound = 15 * 2.0 ** -24 * (Q[:, :, 1].double().abs().sum(1) * K[:, 0, 0].double().abs()).sum(-1)
    assert bool(((scores[:, 0, 0].double() - want).abs() <= bound).all())
