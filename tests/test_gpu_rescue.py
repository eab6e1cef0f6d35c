"""Rows whose FP32 rates underflow are recomputed in FP64 by teams of 1 to 16 waves, after the length of
their list: rates against the FP64 oracle at list lengths around every change of the team, in the sums
and per row; and a small set with every row on the list takes a few times as long as one with none."""

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2407_11349_amd as hk

pytestmark = pytest.mark.gpu


# one workgroup of 16 waves per 256 rows: the teams depend on how many rows of the list are in flight at once
@pytest.mark.parametrize("n, alone", [(1, 1), (2, 2), (200, 1), (200, 2), (200, 3), (200, 4), (200, 5), (200, 8), (200, 9),
                                      (200, 16), (200, 17), (200, 200), (700, 3), (700, 4), (700, 48), (700, 49),
                                      (700, 700), (3001, 12), (3001, 13), (3001, 192), (3001, 193), (3001, 2500)])
def test_rescued_rows_by_list_length(n, alone):
    ev = synth.generate(synth.N2K, n=n, seed=77)
    x, y = ev.x.copy(), ev.y.copy()
    pick = np.linspace(0, n - 1, alone).astype(int)
    # the next one about 125 km (12.5 tau_x) away: exp(-78) and less
    x[pick] = 1125.0 + x.max() + 125.0 * np.arange(alone)
    th = synth.theta_default()
    _, _, lam_ref, _, _ = oracle.loglik(ev.t, x, y, ev.s, th, per_row=True)
    ref, g_ref = oracle.loglik(ev.t, x, y, ev.s, th)
    dev = hk.DeviceEvents.from_arrays(ev.t, x, y, ev.s)
    print(f"rescue: n={n}, {alone} rows", flush=True)
    lam, _ = hk.event_terms(dev, th, precision="fp32")
    lam = lam.cpu().numpy()
    # both in FP64: 1e-11 leaves the two orders of summation and exponents of up to 700 room; a rate below
    # the smallest normal number has no relative precision
    far = pick[lam_ref[pick] >= np.finfo(float).tiny]
    np.testing.assert_allclose(lam[far], lam_ref[far], rtol=1e-11)
    for rep in range(2):
        ll, g = hk.loglik_grad(dev, th, precision="fp32")
        assert abs(float(ll.item()) - ref) <= 1e-9 * abs(ref)
        np.testing.assert_allclose(g.cpu().numpy(), g_ref, rtol=1e-6, atol=1e-6 * np.abs(g_ref).max())
    l1 = hk.loglik(dev, th, precision="fp32")
    assert float(l1.item()) == float(ll.item())


@pytest.mark.parametrize("n", [100, 700, 2000])
def test_time_with_every_row_rescued(n):
    """At most 12 times a call without any (20 to 50 times with a workgroup of 16 waves for every row)."""
    ev = synth.generate(synth.N2K, n=n, seed=5)
    th, ms = synth.theta_default(), []
    for t in (ev.t, np.full(n, 3.0)):  # all times tied: no rate at all, every row is recomputed
        dev = hk.DeviceEvents.from_arrays(t, ev.x, ev.y, ev.s)
        ws, best = hk.Workspace(n, "fp32"), np.inf
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                hk.loglik(dev, th, precision="fp32", ws=ws)
            b.record()
            b.synchronize()
            best = min(best, 100.0 * a.elapsed_time(b))
        ms.append(best)
    print(f"n={n}: {ms[0]:.1f} us, every row rescued {ms[1]:.1f} us", flush=True)
    assert ms[1] < 12.0 * ms[0]
