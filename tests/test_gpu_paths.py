"""Kernels chosen by a layer's sizes, at the sizes where each can go wrong:
tile edges, remainders, the smallest and largest of a rule's range, operands
off their natural alignment.  References and tolerances are the oracle's and
tests/parity.py's."""
import math

import numpy as np
import pytest
import torch

import oracle
from parity import NEVER, W_ABS, check_fire, check_potentials, gpu, np_
from paper_2301_13659_amd import spk
from paper_2301_13659_amd.workloads import random_times

pytestmark = pytest.mark.gpu


def _t(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def _off(a, dev, by):
    """The array on the device, `by` elements past an aligned address."""
    t = _t(a, dev)
    buf = torch.zeros(t.numel() + by, dtype=t.dtype, device=dev)
    buf[by:] = t.reshape(-1)
    return buf[by:].view(t.shape)


@pytest.mark.parametrize("B,I,O,T,theta,dens,dt,by", [
    (1, 1, 1, 1, 0.5, 1.0, "f32", 0),
    (5, 15, 31, 8, 2.0, 0.5, "f32", 1),       # less than a slice, four samples per tile
    (9, 16, 32, 15, 3.0, 0.5, "f16", 0),
    (3, 17, 33, 16, 3.0, 0.5, "f32", 1),      # one tap past a slice, one map past a tile
    (2, 129, 65, 17, 20.0, 0.4, "f16", 3),    # T = 17: one sample per tile
    (4, 1000, 97, 32, 150.0, 0.3, "f32", 1),
    (300, 1125, 211, 15, 60.0, 0.3, "f32", 1),  # two row tiles per block, an odd last one
    (40, 130, 64, 20, math.inf, 0.5, "f32", 1),
    (33, 40, 70, 254, math.inf, 0.5, "f16", 1),
])
def test_fc_fire_edges(B, I, O, T, theta, dens, dt, by):
    dev = gpu()
    rng = np.random.default_rng(B * 1000 + I + O)
    x = random_times(rng, (B, I), T, dens)
    w = rng.uniform(-0.1, 1.0, size=(O, I)).astype(np.float32)
    if dt == "f16":
        w = w.astype(np.float16).astype(np.float32)
    wd = _off(w.astype(np.float16) if dt == "f16" else w, dev, by)
    g_tf, g_vk = spk.spk_fc_fire(_off(x, dev, by), wd, T, theta)
    o_tf, o_vk, o_V = oracle.fc_fire(x, w, T, theta, potentials=True)
    if math.isinf(theta):
        assert np.all(np_(g_tf) == NEVER)
        check_potentials(np_(g_vk), o_vk, "readout v_key")
        return
    exc = (np.abs(o_V.astype(np.float64) - theta) <= 1e-4 * abs(theta)).any(axis=1)
    check_fire(np_(g_tf), np_(g_vk), o_tf, o_vk, exc)


@pytest.mark.parametrize("Co,Ci,K,B,H,k,hw", [
    (3, 57, 3, 4, 5, 2, False),      # 513 synapses: the first size split over blocks
    (4, 64, 3, 300, 6, 8, True),     # 2400 winner slots: a second round of the list
    (2, 250, 5, 40, 5, 1, False),    # 6250 synapses, most winners on one map
])
def test_stdp_split_synapses(Co, Ci, K, B, H, k, hw):
    dev = gpu()
    rng = np.random.default_rng(Ci + B)
    x = random_times(rng, (B, Ci, H, H), 15, 0.4)
    w = rng.uniform(0.1, 0.9, size=(Co, Ci, K, K)).astype(np.float32)
    win = np.zeros((B, k), oracle.WINNER_DTYPE)
    for f, hi in (("c", Co), ("y", H), ("x", H), ("t", 15)):
        win[f] = rng.integers(0, hi, size=(B, k))
    win["c"][rng.random((B, k)) < 0.5] = Co - 1
    n = rng.integers(0, k + 1, size=B).astype(np.int32)
    cfgs = [(0.004, -0.003, 0.0, 1.0, 1), (-0.0005, 0.004, 0.0, 1.0, 0)]
    wc = rng.integers(0, 2, size=(B, k)).astype(np.int32)
    # the change of a weight is a float sum of at most B*k terms below 0.004,
    # each rounded: small steps keep it below the weights' tolerance
    cfgs = [(a / B, m / B, lo, up, st) for a, m, lo, up, st in cfgs]
    wd = _t(w, dev)
    wh = wd.half() if hw else None
    winners = _t(win.view(np.int32).reshape(B, k, 5), dev)
    spk.spk_stdp_update(wd, _t(x, dev), winners, _t(n, dev), cfgs, 1, K // 2, winner_cfg=_t(wc, dev), w_f16=wh)
    ref = oracle.stdp_update(w, x, win, n, cfgs, 1, K // 2, winner_cfg=wc)
    assert np.abs(np_(wd) - ref).max() <= W_ABS
    if hw:
        np.testing.assert_array_equal(np_(wh), np_(wd).astype(np.float16))
