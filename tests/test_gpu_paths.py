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
