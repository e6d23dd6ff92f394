"""fp32 carry split into hi and lo operands (split 3): how much the sums add to the error.

Taps are multiples of 2^-10 and inputs multiples of 2^-21 below 1, so that the fp16 hi
and lo parts hold them exactly and all error is the rounding of sums.  It is given in
units of one rounding of the exact result to fp32.  The bounds are what instructions of
two input lines each (the form before four lines shared one) leave on these inputs,
rounded up in the second decimal."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp

pytestmark = pytest.mark.gpu

BOUND = {(1, "box"): 1.79, (1, "star"): 1.77, (3, "box"): 2.32, (3, "star"): 2.28}


def _taps(r, kind):
    k = 2 * r + 1
    m = np.zeros((k, k), bool)
    m[r, :] = m[:, r] = True
    if kind == "box":
        m[:] = True
    rng = np.random.default_rng(r)
    return np.where(m, rng.integers(1, 2048 // m.sum(), (k, k)), 0) / 1024.0, rng


@pytest.mark.parametrize("r,kind", sorted(BOUND))
def test_one_step(oracle_mod, r, kind):
    w, rng = _taps(r, kind)
    x = rng.integers(0, 1 << 21, (200, 300)) / 2.0 ** 21
    want = oracle_mod.apply(w, x, 1)
    one = want.astype(np.float32).astype(np.float64) - want
    plan = sp.Plan(w, x.shape, carry="f32", engine="sparse", split=3)
    xd = torch.from_numpy(x).float().to("cuda:0")
    y = torch.empty_like(xd)
    plan.apply(xd, y, 1)
    err = y.double().cpu().numpy() - want
    ratio = np.sqrt((err * err).mean() / (one * one).mean())
    assert ratio <= BOUND[r, kind], ratio


@pytest.mark.parametrize("time_block", [1, 2, 3])
def test_roundings_do_not_lean_one_way(oracle_mod, time_block):
    # 40 steps of an averaging stencil (sum of taps exactly 1): a rounding that leans to one
    # side by a tenth of its size adds up to 40 tenths, unbiased ones average out with the
    # values they are in; two lines per instruction leave 2.8
    w = np.array([[48, 112, 80], [128, 288, 112], [96, 80, 80]]) / 1024.0
    assert w.sum() == 1.0
    x = np.random.default_rng(40).integers(0, 1 << 21, (120, 260)) / 2.0 ** 21
    want = oracle_mod.apply(w, x, 40)
    one = want.astype(np.float32).astype(np.float64) - want
    plan = sp.Plan(w, x.shape, carry="f32", engine="sparse", split=3, time_block=time_block)
    xd = torch.from_numpy(x).float().to("cuda:0")
    y = torch.empty_like(xd)
    plan.apply(xd, y, 40)
    err = y.double().cpu().numpy() - want
    ratio = np.sqrt((err * err).mean() / (one * one).mean())
    assert ratio <= 2.8, ratio
