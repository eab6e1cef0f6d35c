"""Data that the device checks refuse, in the skip mode: NaN results and the status word, whatever the
times are, with a plan whose ranges stay within what the fold of the partial sums assumes."""

import math

import numpy as np
import pytest
import torch

import synth
import paper_2407_11349_amd as hk
from paper_2407_11349_amd import _lib

pytestmark = pytest.mark.gpu

TS, TB, MAX_GROUPS = 256, 512, 1024


def _times(form, n):
    rng = np.random.default_rng(n)
    if form == "reversed":
        return np.sort(rng.uniform(0, 1000, n))[::-1].copy()
    if form == "shuffled":
        return rng.uniform(0, 1000, n)
    if form == "nan":
        t = np.sort(rng.uniform(0, 1000, n))
        t[n // 3::701] = np.nan
        return t
    # tiles that begin late and end early, and one block that ends last of all: a range that starts
    # beyond the end of the next row group's
    t = np.full(n, 500.0)
    t[::TS] = 1000.0
    t[TS - 1::TS] = t[-1] = 0.0
    b = -(-n // TB) // 3
    t[(b + 1) * TB - 1] = 2000.0
    return t


def _cell_ranges(ws, n):
    """gchi and gclo of the last FP32 call's plan: first the staged records, then the blocks' tile bounds."""
    up = lambda v: (v + 255) // 256 * 256  # noqa: E731
    tiles, blocks = -(-n // TS), -(-n // TB)
    a = 256 + up(4 * TS * tiles) + up(24 * tiles) + 9 * 8 * TS * tiles + 2 * up(4 * blocks)
    raw = ws._buf[ws.offset + a:ws.offset + a + 8 * MAX_GROUPS].cpu().numpy().view(np.int32)
    return raw[:blocks], raw[MAX_GROUPS:MAX_GROUPS + blocks]


@pytest.mark.parametrize("n", [2000, 9000, 16000, 20001])
@pytest.mark.parametrize("form", ["reversed", "shuffled", "nan", "one late block"])
def test_unsorted_times_in_skip_mode(form, n):
    ev = synth.generate(synth.N2K, n=n, seed=3)
    t = _times(form, n)
    th = synth.theta_default()
    th[2] = 2.0
    dev = hk.DeviceEvents.from_arrays(t, ev.x, ev.y, ev.s)
    ws = hk.Workspace(n, "fp32_skip")
    print(f"data checks: {form} n={n}", flush=True)
    ll, g = hk.loglik_grad(dev, th, precision="fp32_skip", ws=ws)
    assert ws.status() == (_lib.HAWKES_EDATA if form == "nan" else _lib.HAWKES_EORDER)
    assert math.isnan(float(ll.item())) and torch.isnan(g).all()
    hi, lo = _cell_ranges(ws, n)
    assert np.all(lo >= 0) and np.all(lo <= hi)
    # the cells of a column group fall with the row group: the fold's range search rests on it
    assert np.all(hi[1:] + 1 - lo[:-1] > 0)
    lam, comp = hk.event_terms(dev, th, precision="fp32_skip", ws=ws)
    assert torch.isnan(lam).all() and torch.isnan(comp).all()
    part, _ = hk.loglik_grad(dev, th, precision="fp32_skip", ws=ws, rows=(n // 4, n // 2))
    assert math.isnan(float(part.item()))
    assert torch.isnan(hk.loglik_batch(dev, np.stack([th, th]), precision="fp32_skip", ws=ws)).all()
    # the workspace serves sorted times again
    good = hk.DeviceEvents.from_arrays(ev.t, ev.x, ev.y, ev.s)
    ll, _ = hk.loglik_grad(good, th, precision="fp32_skip", ws=ws)
    ref, _ = hk.loglik_grad(good, th, precision="fp32_skip")
    assert ws.status() == _lib.HAWKES_OK and float(ll.item()) == float(ref.item())
