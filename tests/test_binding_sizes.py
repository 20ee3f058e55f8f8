"""The binding's memo of a shape's struct and sizes: by value, with fresh
dicts, and for integer-like fields that cannot be hashed."""
import numpy as np
import pytest

import paper_2608_27875_amd as hyq


def test_sizes_are_fresh_and_by_value():
    s = hyq.Shape(B=1, Hq=4, Hkv=2, L=300, window=64, budget_ppm=20000)
    a = hyq.hyq_sizes_for(s)
    a["k"] = -1
    assert hyq.hyq_sizes_for(s)["k"] == hyq.hyq_sizes_for(hyq.Shape(**vars(s)))["k"] == 5
    t = hyq.Shape(B=1, Hq=4, Hkv=2, L=np.array(301), window=64, budget_ppm=20000)
    assert hyq.hyq_sizes_for(t)["P"] == 237


def test_errors_are_raised_every_time():
    bad = hyq.Shape(B=1, Hq=4, Hkv=3, L=300)
    for _ in range(2):
        with pytest.raises(hyq.HyqError):
            hyq.hyq_sizes_for(bad)


def test_mutable_fields_are_read_on_every_call():
    import torch
    t = torch.tensor(300)   # hashes by identity
    s = hyq.Shape(B=1, Hq=4, Hkv=2, L=t, window=64, budget_ppm=20000)
    assert hyq.hyq_sizes_for(s)["P"] == 236
    t += 200
    assert hyq.hyq_sizes_for(s)["P"] == 436

    class Duck:             # anything with a c()
        L = 300

        def c(self):
            return hyq.Shape(B=1, Hq=4, Hkv=2, L=self.L, window=64, budget_ppm=20000).c()
    d = Duck()
    assert hyq.hyq_sizes_for(d)["P"] == 236
    d.L = 500
    assert hyq.hyq_sizes_for(d)["P"] == 436


def test_sizes_in_the_buffers_are_the_callers():
    s = hyq.Shape(B=1, Hq=4, Hkv=2, L=300, window=64, budget_ppm=20000)
    b = hyq.alloc_buffers(s, "cpu")
    b["sizes"].update(k=-1, select_ws_bytes=0)
    z = hyq.hyq_sizes_for(s)
    assert z["k"] == 5 and z["select_ws_bytes"] > 0
    assert hyq.alloc_buffers(s, "cpu")["sizes"] == z
