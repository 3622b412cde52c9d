"""The margin of the matrix-core hash is a proof: the error of its fp16 terms, measured here on the host in exact arithmetic for
rows made to lose as much as they can, stays below what csrc/hash_margin.h allows for, and that plus the fp32 sums of the products
and of the defining chain stays below the margin."""
import json
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "hash_margin.h"
int main(int argc, char **argv) {
    const int d = atoi(argv[1]);
    const double x = argc > 2 ? atof(argv[2]) : sa::kSplitMin;
    printf("{\"theta\": %.17g, \"error\": %.17g, \"split\": %.17g, \"min\": %.17g, \"max\": %.17g, \"scale\": %.17g}\n", (double)sa::hash_theta(d),
           sa::hash_error(d), sa::hash_split_error(d, x), __builtin_sqrt((double)sa::kOrdinaryMin2), __builtin_sqrt((double)sa::kOrdinaryMax2),
           (double)sa::kColumnScale);
}
"""


@pytest.fixture(scope="module")
def margin(tmp_path_factory):
    at = tmp_path_factory.mktemp("margin")
    src, exe = at / "driver.cpp", at / "driver"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2306_06446_amd", "csrc"), str(src), "-o", str(exe)])
    return lambda d, *x: json.loads(subprocess.check_output([str(exe), str(d)] + ["%.17g" % v for v in x]))


def terms(v):
    """fp32 -> its two fp16 terms, as the kernel rounds them, in fp64."""
    up = v.astype(np.float16)
    return up.astype(np.float64), (v - up.astype(np.float32)).astype(np.float16).astype(np.float64)


def split_error(x, r, scale):
    """|x . r^ - (xh rh + xh rl + xl rh)| / (|x| |r^|) of rows x against columns r (both [n, d], fp32, the columns of norm 1)."""
    (xh, xl), (rh, rl) = terms(x), terms(r * np.float32(scale))
    z = (xh * rh + xh * rl + xl * rh).sum(-1) / scale
    x, r = x.astype(np.float64), r.astype(np.float64)
    return np.abs((x * r).sum(-1) - z) / (np.linalg.norm(x, axis=-1) * np.linalg.norm(r, axis=-1))


@pytest.mark.parametrize("d", [32, 64, 128])
def test_margin_covers_every_error(margin, d):
    m = margin(d)
    rng = np.random.default_rng(d)
    worst_low = 0.0
    for length in (m["min"], 0.5, 1.4, 60.0, m["max"]):
        # elements of equal size and column elements of the same signs: the errors of a row, made to be nearly half a unit of
        # the lower term all in one direction, add up.  And rows and columns as they come.
        sign = np.where(rng.random((200, d)) < 0.5, -1.0, 1.0)
        base = (length / np.sqrt(d) * (1.0 + 0.01 * rng.random((200, d)))).astype(np.float32)
        best = base.copy()
        loss = np.full(base.shape, -1.0)
        for _ in range(200):                               # of 200 neighbours of every element the one that loses most
            cand = (base * (1.0 + 1e-3 * rng.random(base.shape))).astype(np.float32)
            up, lo = terms(cand)
            lost = cand.astype(np.float64) - up - lo
            best, loss = np.where(lost > loss, cand, best), np.maximum(lost, loss)
        flat = np.full((200, d), 1.0 / np.sqrt(d), np.float32)
        plain = rng.standard_normal((200, d))
        plain = (plain * (length * 1.001 / np.linalg.norm(plain, axis=-1, keepdims=True))).astype(np.float32)
        col = rng.standard_normal((200, d))
        col = (col / np.linalg.norm(col, axis=-1, keepdims=True)).astype(np.float32)
        worst = max(split_error((best * sign).astype(np.float32), (flat * sign).astype(np.float32), m["scale"]).max(),
                    split_error(plain, col, m["scale"]).max())
        assert worst <= margin(d, length)["split"], (length, worst)
        worst_low = max(worst_low, worst)
    # the sums, from the number of their roundings alone: 3 d products (truncated), d steps of the chain (rounded)
    total = worst_low + 3 * d * 2.0 ** -23 + d * 2.0 ** -24
    assert total < m["theta"], (total, m["theta"])
    assert total < m["error"] < m["theta"]
