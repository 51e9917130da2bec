"""The error bound of the k-means search (csrc/kmeans.hip): a product of two FP32
values from bf16 parts, h h + h m + m h, against the constant that the kernel
uses, over significands up to the worst ones.  Runs on the CPU."""
import os
import re

import numpy as np
import torch

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_2202_10297_amd", "csrc", "kmeans.hip")


def _parts(x):
    t = torch.from_numpy(x)
    h = t.to(torch.bfloat16).float()
    m = (t - h).to(torch.bfloat16).float()
    return h.double().numpy(), m.double().numpy()


def test_bound_covers_the_products_left_out():
    src = re.search(r"kBeta = ([\d.]+)f \* 0x1p-18f \+ ([\d.]+)f \* \(16\.f \* KS \+ 16\.f\) \* 0x1p-23f",
                    open(SRC).read())
    c0, c1 = float(src.group(1)), float(src.group(2))
    # every significand just above 1 + 2^-8 (m and r largest against x), every
    # 2^-23 apart, and a sample of the others
    near = 1.0 + 2.0 ** -8 + np.arange(-1024, 1025) * 2.0 ** -23
    rest = 1.0 + np.random.default_rng(3).integers(0, 1 << 23, 2000) * 2.0 ** -23
    x = np.concatenate([near, rest]).astype(np.float32)
    h, m = _parts(x)
    xd = x.astype(np.float64)
    exact = np.outer(xd, xd)
    off = np.abs(exact - (np.outer(h, h) + np.outer(h, m) + np.outer(m, h))) / exact
    worst = off.max() * 2.0 ** 18
    assert 7.9 < worst <= 8.0 < c0
    for ks in (2, 4, 8, 16):  # rows of up to 16 ks dimensions
        D = 16 * ks
        assert worst * 2.0 ** -18 + 3 * D * 2.0 ** -23 < c0 * 2.0 ** -18 + c1 * (D + 16) * 2.0 ** -23
