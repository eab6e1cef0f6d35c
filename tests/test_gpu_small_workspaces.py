"""Workspaces from the smallest accepted one on: the passes before the last use the space that the row
values and the rescue list take only afterwards, so results are bitwise those of a single pass also where
rows are recomputed, for every call, at sizes where that space holds less than, as much as and more than
all cells; and a call there takes a few times as long, not hundreds of times (one cell a pass)."""

import numpy as np
import pytest
import torch

import synth
import paper_2407_11349_amd as hk
from paper_2407_11349_amd import _lib

pytestmark = pytest.mark.gpu


def _events(n):
    """With events so far from all others that their rates are recomputed."""
    ev = synth.generate(synth.N100K, n=n, seed=n)
    x = ev.x.copy()
    alone = np.arange(n) % 131 == 5
    x[alone] += 1e4 + 130.0 * np.arange(alone.sum())
    return hk.DeviceEvents.from_arrays(ev.t, x, ev.y, ev.s)


def _outputs(dev, th, prec, ws):
    n = dev.n
    out = list(hk.loglik_grad(dev, th, precision=prec, ws=ws))
    out.append(hk.loglik(dev, th, precision=prec, ws=ws))
    out += hk.event_terms(dev, th, precision=prec, ws=ws)
    out += hk.loglik_grad(dev, th, precision=prec, ws=ws, rows=(n // 3, n - n // 9))
    out.append(hk.loglik_batch(dev, np.stack([th, 1.05 * th, 0.97 * th]), precision=prec, ws=ws))
    torch.cuda.synchronize()
    assert ws.status() == _lib.HAWKES_OK
    return out


@pytest.mark.parametrize("prec", ["fp32", "fp32_skip", "fp64"])
@pytest.mark.parametrize("n", [1, 300, 513, 2000, 4097, 9001, 20000])
def test_results_at_small_workspaces(n, prec):
    dev, th = _events(n), synth.theta_default()
    ref = _outputs(dev, th, prec, hk.Workspace(n, prec))
    lo = hk.workspace_min_bytes(n, prec)
    cell = 8 * 512 * 9
    for extra in (0, 256, cell - 256, 2 * cell, 37 * cell + 512, 400 * cell, 1100 * cell):
        print(f"n={n} {prec} minimum + {extra} bytes", flush=True)
        for a, b in zip(ref, _outputs(dev, th, prec, hk.Workspace(n, prec, nbytes=lo + extra))):
            assert torch.equal(a, b), extra


@pytest.mark.parametrize("n", [2000, 9000, 20000])
def test_time_at_the_minimum_workspace(n):
    """Below 30 times the time in the default workspace (47, 206 and 403 times with one cell a pass)."""
    ev = synth.generate(synth.N100K, n=n, seed=5)
    dev, th = hk.DeviceEvents.from_arrays(ev.t, ev.x, ev.y, ev.s), synth.theta_default()
    ms = []
    for nbytes in (None, hk.workspace_min_bytes(n, "fp32")):
        ws, best = hk.Workspace(n, "fp32", nbytes=nbytes), np.inf
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            hk.loglik_grad(dev, th, precision="fp32", ws=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
    print(f"n={n}: {ms[0]:.3f} ms, at the minimum workspace {ms[1]:.3f} ms", flush=True)
    assert ms[1] < 30.0 * ms[0]
