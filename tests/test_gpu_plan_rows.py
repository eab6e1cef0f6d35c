"""Per-row rates of whole-set calls with the default plan, whose column groups are 32 to 512 sources
by the event count: against the FP64 oracle at block and tile edges and on both sides of each change of
width that it is quick at, and against the row sweep on both sides of the counts from which row groups share
the 512-source width (384 blocks) and hold several blocks (652)."""

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2407_11349_amd as hk

pytestmark = pytest.mark.gpu

TOL_EV = 5e-6  # a row's FP32 rate against the oracle


def _rows(dev, th, prec, **kw):
    lam, comp = hk.event_terms(dev, th, precision=prec, **kw)
    torch.cuda.synchronize()
    return lam.cpu().numpy(), comp.cpu().numpy()


# one cell per CU at most up to 2560 (32 sources), 3584 (64), 5120 (128) and 7680 (256) events, then 128
@pytest.mark.parametrize("n", [1, 2, 255, 257, 511, 512, 513, 1024, 1537, 2049, 2560, 2561, 3584, 3585, 5120, 5121,
                               7680, 7681, 20480, 20481])
@pytest.mark.parametrize("ties", [False, True])
def test_default_plan_per_row(n, ties):
    ev = synth.generate(synth.N2K, n=n, seed=1300 + n)
    th = synth.theta_default()
    th[2] = 1.5  # short background range in time: far tiles also at small n
    t = np.floor(ev.t / 3.0) * 3.0 if ties else ev.t
    _, _, lam_ref, comp_ref, _ = oracle.loglik(t, ev.x, ev.y, ev.s, th, per_row=True)
    dev = hk.DeviceEvents.from_arrays(t, ev.x, ev.y, ev.s)
    pos = lam_ref > 0
    for prec, tol in (("fp32", TOL_EV), ("fp32_skip", TOL_EV), ("fp64", 1e-11)):
        print(f"n={n} ties={ties} {prec}", flush=True)
        lam, comp = _rows(dev, th, prec)
        np.testing.assert_allclose(lam[pos], lam_ref[pos], rtol=tol)
        np.testing.assert_allclose(comp, comp_ref, rtol=1e-13, atol=1e-13)


# 49152: 256 sources, 49153: 512; 196608 and 333824 events are 384 and 652 blocks
@pytest.mark.parametrize("n", [49152, 49153, 196608, 196609, 333824, 333825])
def test_default_plan_against_the_row_sweep(n):
    ev = synth.generate(synth.N100K, n=n, seed=9)
    th = synth.theta_default()
    dev = hk.DeviceEvents.from_arrays(ev.t, ev.x, ev.y, ev.s)
    row, comp_row = _rows(dev, th, "fp32", symmetric_groups=-1)
    ll_row, g_row = hk.loglik_grad(dev, th, precision="fp32", symmetric_groups=-1)
    for prec in ("fp32", "fp32_skip"):
        print(f"n={n} {prec}", flush=True)
        lam, comp = _rows(dev, th, prec)
        # the order of FP32 background sums differs (a wave's 128 targets instead of 8 sources)
        np.testing.assert_allclose(lam, row, rtol=1e-6)
        assert np.array_equal(comp, comp_row)
        ll, g = hk.loglik_grad(dev, th, precision=prec)
        assert float(ll.item()) == pytest.approx(float(ll_row.item()), rel=1e-10)
        np.testing.assert_allclose(g.cpu().numpy(), g_row.cpu().numpy(), rtol=1e-7)
