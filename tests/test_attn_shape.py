"""Host-side launch shape of the prefill attention (`attn_shape.h`): every
shape covers every unit exactly, the policy's lines lie where its comment
puts them, and the inputs of the GPU tests take the shapes they are named
for.  Plain C++, compiled with g++: runs without a GPU."""
import os
import shutil
import subprocess

import pytest

import test_gpu_attn_shapes as gpu
from oracle import hyq_oracle as orc

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_27875_amd", "csrc")
FULL, HALF, SPLIT2, SPLIT8 = range(4)
UNITS = {FULL: 8, HALF: 4, SPLIT2: 4, SPLIT8: 1}   # per workgroup
CODED, DENSE, MIXED, LISTED, BANDED, WIDE, WHOLE = range(7)   # the last three: per-query windows
SHARE = {CODED: 0.05, DENSE: 1.0, MIXED: 0.5, LISTED: 1.0, BANDED: 0.5, WIDE: 0.9, WHOLE: 1.0}
MODE = {CODED: 0, DENSE: 1, MIXED: 0, LISTED: 0, BANDED: 2, WIDE: 2, WHOLE: 2}


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("shape") / "shape_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC,
                    os.path.join(HERE, "attn_shape_check.cpp"), "-o", exe], check=True)

    def run(cases):   # (units per head, heads, L, full, mode, CUs) -> (kind, grid, fold, keys)
        inp = "".join(" ".join(map(str, c)) + "\n" for c in cases)
        out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


def test_every_unit_has_one_workgroup(choose):
    cases = [(g * -(-L // 32), heads, L, int(share * L), mode, n_cu)
             for g in (1, 4, 5, 8) for heads in (1, 2, 8, 40, 300)
             for L in (1, 33, 500, 2000, 9000, 131072) for share, mode in
             ((0.02, 0), (0.5, 0), (1.0, 0), (1.0, 1), (0.5, 2), (0.9, 2), (1.0, 2)) for n_cu in (80, 256)]
    for (units, heads, L, full, mode, n_cu), (kind, grid, fold, _) in zip(cases, choose(cases)):
        assert grid % heads == 0
        n = grid // heads   # workgroups per KV head
        assert (n - 1) * UNITS[kind] < units <= n * UNITS[kind]
        if kind == HALF:   # the kernel's order: slots below fold descend, the rest ascend
            order = [n - 1 - s if s < fold else s - fold for s in range(n)]
            assert sorted(order) == list(range(n)) and grid <= 2 * n_cu


def test_key_classes(choose):
    cases = [(1, 1, 1000, full, mode, 256) for full, mode in
             ((0, 0), (399, 0), (400, 0), (619, 0), (620, 0), (1000, 0), (0, 1), (1000, 1),
              (0, 2), (749, 2), (750, 2), (969, 2), (970, 2))]
    assert [c[3] for c in choose(cases)] == [CODED, CODED, MIXED, MIXED, LISTED, LISTED, DENSE, DENSE,
                                             BANDED, BANDED, WIDE, WIDE, WHOLE]


def test_lines(choose):
    # units/head, KV heads, tiles, keys: the last case before a line and the first behind it
    want = [((256, 1, 1, CODED), SPLIT8), ((257, 1, 11, CODED), HALF), ((257, 1, 12, CODED), SPLIT2),
            ((257, 1, 15, CODED), SPLIT2), ((512, 1, 16, CODED), SPLIT8), ((513, 1, 16, CODED), SPLIT2),
            ((128, 8, 1, CODED), HALF), ((132, 8, 2, CODED), FULL), ((132, 8, 3, CODED), HALF),
            ((129, 8, 3, CODED), FULL), ((129, 8, 4, CODED), HALF),
            ((28, 73, 2, CODED), HALF),
            ((128, 8, 12, CODED), SPLIT2), ((129, 8, 95, CODED), HALF), ((129, 8, 96, CODED), SPLIT2),
            ((192, 8, 96, CODED), SPLIT2), ((193, 8, 127, CODED), HALF),
            ((193, 8, 128, CODED), SPLIT2), ((256, 8, 128, CODED), SPLIT2),
            ((256, 8, 127, CODED), HALF), ((257, 8, 128, CODED), FULL), ((4096, 8, 512, CODED), FULL),
            ((512, 1, 15, MIXED), SPLIT2), ((512, 1, 16, MIXED), SPLIT8), ((513, 1, 11, MIXED), HALF),
            ((513, 1, 12, MIXED), SPLIT2), ((129, 8, 3, MIXED), FULL), ((129, 8, 4, MIXED), HALF), ((192, 8, 23, MIXED), HALF), ((192, 8, 24, MIXED), SPLIT2),
            ((256, 8, 47, MIXED), HALF), ((256, 8, 48, MIXED), SPLIT2), ((257, 8, 48, MIXED), FULL),
            ((256, 1, 1, LISTED), SPLIT8), ((257, 1, 15, LISTED), SPLIT2),
            ((512, 1, 16, LISTED), SPLIT8), ((28, 73, 7, LISTED), HALF), ((128, 8, 4, LISTED), HALF),
            ((128, 8, 5, LISTED), SPLIT2),
            ((192, 8, 19, LISTED), FULL), ((191, 8, 19, LISTED), FULL), ((192, 8, 20, LISTED), SPLIT2),
            ((256, 8, 31, LISTED), FULL), ((256, 8, 32, LISTED), SPLIT2),
            ((256, 1, 11, DENSE), SPLIT8), ((256, 1, 12, DENSE), SPLIT2), ((257, 1, 7, DENSE), HALF),
            ((192, 8, 3, DENSE), FULL), ((192, 8, 4, DENSE), HALF),
            ((257, 1, 8, DENSE), SPLIT2), ((192, 8, 11, DENSE), HALF), ((192, 8, 12, DENSE), SPLIT2),
            ((256, 8, 23, DENSE), HALF), ((256, 8, 24, DENSE), SPLIT2), ((257, 8, 200, DENSE), FULL),
            ((129, 8, 1, BANDED), HALF), ((257, 1, 4, BANDED), HALF),
            ((257, 1, 5, BANDED), SPLIT2), ((192, 8, 95, BANDED), HALF), ((192, 8, 96, BANDED), SPLIT2),
            # full-precision lists: a second turn of kFull's workgroups, half workgroups that
            # spread no head further
            ((28, 73, 11, LISTED), HALF), ((28, 73, 12, LISTED), FULL), ((4, 128, 2, LISTED), FULL),
            ((5, 128, 2, LISTED), HALF), ((4, 128, 2, MIXED), HALF),
            ((128, 8, 4, WIDE), HALF), ((128, 8, 5, WIDE), SPLIT2), ((192, 8, 8, WIDE), HALF),
            ((192, 8, 9, WIDE), SPLIT2), ((256, 8, 13, WIDE), HALF), ((256, 8, 14, WIDE), SPLIT2),
            ((257, 8, 14, WIDE), FULL),
            ((4, 128, 2, WHOLE), FULL), ((128, 8, 4, WHOLE), HALF), ((128, 8, 5, WHOLE), SPLIT2),
            ((192, 8, 8, WHOLE), FULL), ((192, 8, 9, WHOLE), SPLIT2), ((256, 8, 17, WHOLE), FULL),
            ((256, 8, 18, WHOLE), SPLIT2), ((28, 73, 11, WHOLE), HALF), ((28, 73, 12, WHOLE), FULL)]
    got = choose([(u, heads, 64 * t, int(64 * t * SHARE[keys]), MODE[keys], 256)
                  for (u, heads, t, keys), _ in want])
    assert [(k, c[0]) for (k, _), c in zip(want, got)] == want


# shapes, formats and window modes of the GPU tests, on an MI355X's 256 CUs
def test_gpu_tests_run_the_shapes_they_name(choose):
    names = {"split8_tiny": SPLIT8, "split8": SPLIT8, "split2": SPLIT2, "half": HALF, "full": FULL}
    cases = [(kind, *gpu.shape_for(kind, fmt), W, 50000, int(fmt == "bf16"))
             for kind in gpu.SHAPES for fmt in gpu.FORMATS for W in (100, 200)]
    cases += [(kind, *gpu.SHAPES[kind], 90, 50000, 2) for kind in gpu.SHAPES]   # per-query window
    cases += [(*c[:5], gpu.ROW_SUM_W, 10000, int(c[5] == "bf16")) for c in gpu.ROW_SUM]
    cases += [(*c[:5], gpu.FUTURE_V_W, 20000, int(c[5] == "bf16")) for c in gpu.FUTURE_V]
    got = choose([(Hq // Hkv * -(-L // 32), B * Hkv, L, orc.sizes(L, W, ppm)["k"] + min(W, L), mode,
                   256) for _, B, Hq, Hkv, L, W, ppm, mode in cases])
    for c, g in zip(cases, got):
        assert g[0] == names[c[0]], c
