"""The skip mode's ranges against their bound: over every row that is not recomputed, the background
terms that the sweep leaves out are together below 2^-60 of the row's rate, and so are the triggering
terms.  Which terms those are follows from the plan that a call leaves in its workspace (each target
block's first tile and gap, each tile's times); the terms themselves are formed here in FP64.

The event sets have a site that is active, goes quiet and gets one more event, whose background comes from
afar in time alone: its block's gap is wide, those of the dense early blocks narrow.  With omega of 1 and
more, triggering ends long before the background's range."""

import numpy as np
import pytest
import torch

import synth
import paper_2407_11349_amd as hk

pytestmark = pytest.mark.gpu

TS, TB = 256, 512
WORD = np.dtype([("first", "<f8"), ("last", "<f8"), ("klo", "<i4"), ("gap", "<f4")])


def _plan(ws, n):
    """The tile records of the last skip-mode call: after the status words (256 bytes) and the tie groups."""
    tiles = -(-n // TS)
    a = ws.offset + 256 + 4 * TS * tiles
    return ws._buf[a:a + WORD.itemsize * tiles].cpu().numpy().view(WORD)


def _quiet_site(n, dist, late, dense):
    """A site with events over days 0 to 100 and `dense` more at the end of them, one on day `late`; all others
    dist km away over days 0 to 400."""
    rng = np.random.default_rng(int(dist) + n)
    here = (n - dense) // 3
    t = np.concatenate([rng.uniform(0, 100, here), rng.uniform(99.9, 100, dense), [late],
                        rng.uniform(0, 400, n - here - dense - 1)])
    site = np.arange(n) > here + dense
    x = 0.2 * rng.normal(size=n) + dist * site
    y = 0.2 * rng.normal(size=n)
    x[here + dense] = y[here + dense] = 0.0
    order = np.argsort(t, kind="stable")
    return t[order], x[order], y[order], int(np.flatnonzero(order == here + dense)[0])


def _left_out(t, x, y, s, th, lam, plan, rows):
    """(background, triggering) terms left out of the rows' rates, as shares of them."""
    mu, tx, tt, xi, h0, om = th
    n = len(t)
    u = s ** -2
    blk = np.arange(n) // TB
    tile = np.arange(n) // TS
    first, last_block = t[blk * TB], t[np.minimum(blk * TB + TB, n) - 1]
    klo, gap, last_tile = plan["klo"][2 * blk], plan["gap"][2 * blk].astype(float), plan["last"][tile]
    worst = np.zeros(2)
    for i in rows:
        d2 = (x - x[i]) ** 2 + (y - y[i]) ** 2
        dt = t[i] - t
        b = mu / ((2 * np.pi) ** 1.5 * tx * tx * tt) * np.exp(-d2 / (2 * tx * tx) - dt * dt / (2 * tt * tt))
        e = np.where(dt > 0, xi * om / (2 * np.pi * h0 * h0) * u * np.exp(-u * d2 / (2 * h0 * h0) - om * np.abs(dt)), 0.0)
        width = np.maximum(gap[i], gap)
        early = last_tile < first[i]  # swept from the row's block
        out_early = early & ((tile < klo[i]) | (first[i] - last_tile > width))
        late = first > last_block[i]  # swept from the other event's block
        out_late = late & ((tile[i] < klo) | (first - last_tile[i] > width))
        worst = np.maximum(worst, [b[out_early | out_late].sum() / lam[i], e[early & (tile < klo[i])].sum() / lam[i]])
    return worst


@pytest.mark.parametrize("omega", [0.2, 1.0, 2.0])
@pytest.mark.parametrize("n, dist, late, dense", [(20000, 200.0, 236.0, 6000), (20000, 90.0, 245.0, 6000),
                                                  (33001, 150.0, 220.0, 12000)])
def test_a_late_event_keeps_its_far_background(n, dist, late, dense, omega):
    t, x, y, lone = _quiet_site(n, dist, late, dense)
    s = np.ones(n)
    th = np.array([0.5, 20.0, 14.0, 0.3, 2.0, omega])
    dev = hk.DeviceEvents.from_arrays(t, x, y, s)
    ws = hk.Workspace(n, "fp32_skip")
    lam, _ = hk.event_terms(dev, th, precision="fp32_skip", ws=ws)
    plan = _plan(ws, n)
    full, _ = hk.event_terms(dev, th, precision="fp32")
    exact = hk.event_terms(dev, th, precision="fp64")[0].cpu().numpy()
    lam, full = lam.cpu().numpy(), full.cpu().numpy()
    print(f"n={n} dist={dist} late={late} omega={omega}: lone row {lam[lone]:.6e}, full {full[lone]:.6e}, gap "
          f"{plan['gap'][2 * (lone // TB)]:.1f}, first tile at {plan['last'][plan['klo'][2 * (lone // TB)]]:.1f} d", flush=True)
    mu, tx, tt, xi, h0, om = th
    recomputed = n * 2.0 ** -126 * (mu / ((2 * np.pi) ** 1.5 * tx * tx * tt) + xi * om / (2 * np.pi * h0 * h0)) / 1e-12
    assert exact[lone] > 2 * recomputed  # else the row would not see its range
    rows = [i for i in sorted({lone, *range(0, n, 101)}) if exact[i] > 2 * recomputed]
    back, trig = _left_out(t, x, y, s, th, exact, plan, rows)
    print(f"left out: background {back:.2e}, triggering {trig:.2e} of the rate", flush=True)
    assert back <= 2.0 ** -60 and trig <= 2.0 ** -60
    # what is left in differs in the FP32 order of triggering terms beyond the background's range: the rounding
    # of 8-term sums for a row that has no others
    np.testing.assert_allclose(lam, full, rtol=4.8e-7)
    part, _ = hk.event_terms(dev, th, precision="fp32_skip", rows=(lone - 300, lone + 7), ws=ws)
    np.testing.assert_allclose(part.cpu().numpy(), lam[lone - 300:lone + 7], rtol=4.8e-7)
    ll, g = hk.loglik_grad(dev, th, precision="fp32_skip")
    ll_f, g_f = hk.loglik_grad(dev, th, precision="fp32")
    assert float(ll.item()) == pytest.approx(float(ll_f.item()), rel=1e-13)
    np.testing.assert_allclose(g.cpu().numpy(), g_f.cpu().numpy(), rtol=1e-10)
    for thetas in ([th], [th, th * np.array([1.1, 0.9, 1.1, 0.9, 1.1, 1.2])]):
        np.testing.assert_allclose(hk.loglik_batch(dev, thetas, precision="fp32_skip").cpu().numpy(),
                                   hk.loglik_batch(dev, thetas, precision="fp32").cpu().numpy(), rtol=1e-13)


@pytest.mark.parametrize("form", ["plain", "days", "outliers"])
@pytest.mark.parametrize("omega", [0.2, 1.0, 3.0])
def test_the_bound_holds_on_other_sets(form, omega):
    n = 20000
    ev = synth.generate(synth.N100K, n=n, seed=71)
    t, x, y, s = ev.t.copy(), ev.x.copy(), ev.y.copy(), ev.s.copy()
    th = synth.theta_default()
    th[5] = omega
    rng = np.random.default_rng(n)
    if form == "days":
        t = np.floor(t / 40.0) * 40.0
    elif form == "outliers":
        k = rng.choice(n, 200, replace=False)
        x[k] += rng.choice([60.0, 80.0, 100.0], 200)
    dev = hk.DeviceEvents.from_arrays(t, x, y, s)
    ws = hk.Workspace(n, "fp32_skip")
    hk.loglik_grad(dev, th, precision="fp32_skip", ws=ws)
    plan = _plan(ws, n)
    exact = hk.event_terms(dev, th, precision="fp64")[0].cpu().numpy()
    mu, tx, tt, xi, h0, om = th
    recomputed = n * 2.0 ** -126 * (mu / ((2 * np.pi) ** 1.5 * tx * tx * tt) + xi * om / (2 * np.pi * h0 * h0)) / 1e-12
    rows = [i for i in range(0, n, 67) if exact[i] > 2 * recomputed]
    back, trig = _left_out(t, x, y, s, th, exact, plan, rows)
    print(f"{form} omega={omega}: left out: background {back:.2e}, triggering {trig:.2e} of the rate", flush=True)
    assert back <= 2.0 ** -60 and trig <= 2.0 ** -60


@pytest.mark.parametrize("omega", [2.0, 5.0, 20.0])
@pytest.mark.parametrize("n, days", [(16600, 1200.0), (20000, 3000.0)])
def test_ranges_are_as_short_as_the_terms_allow(n, days, omega):
    """Where triggering is over long before the background's gaps (by hundreds of bits), no block visits a tile
    beyond its own and the tiles' gaps: also where a step from one tile to the next is more than an FP32
    exponential spans."""
    rng = np.random.default_rng(n)  # all at one place: every row has near neighbours, so that its gap is narrow
    t = np.sort(rng.uniform(0.0, days, n))
    x, y = rng.normal(size=(2, n))
    th = synth.theta_default()
    th[5] = omega
    dev = hk.DeviceEvents.from_arrays(t, x, y, np.ones(n))
    ws = hk.Workspace(n, "fp32_skip")
    hk.loglik_grad(dev, th, precision="fp32_skip", ws=ws)
    plan = _plan(ws, n)
    blocks = plan[::2]
    for b in range(len(blocks)):
        # beyond the block's gap, and every tile so far beyond its own
        reach = np.maximum.accumulate(plan["last"] + np.repeat(blocks["gap"], 2)[:len(plan)])
        beyond = (plan["last"] < blocks["first"][b] - float(blocks["gap"][b])) & (reach < blocks["first"][b])
        assert blocks["klo"][b] >= beyond.sum(), (b, beyond.sum())
    assert blocks["gap"][1:].max() < 0.9 * blocks["gap"][0]  # the first rows have no event before them
    print(f"gaps {blocks['gap'][0]:.1f}, then up to {blocks['gap'][1:].max():.1f}", flush=True)
