"""The event pass on ring blocks at the edges of its register caches, against the oracle.

Every shape of the cache (one or two events per wavefront, rings of rows, pixels of the longest row)
with ellipses that just fit it, on a grid that cuts many of them.

Tolerance of the image (relative L2): 2e-6 for the single-precision kernel (the exponent, at most 13 in
magnitude, carries a few roundings of 2^-24) plus three standard deviations of the fixed-point
rounding, 0.29 units of 2^-23 per (event, pixel) pair.  A single event's denominator: 1e-5 (all its
pixels may share the roundings of the event's constants, each up to 2^-24 of an exponent near 13).
Counts: exact.
"""

import math

import numpy as np
import pytest

import oracle
from jpet_synth.events import simulate_events
from jpet_synth.phantom import c1_phantom

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1502_07478_amd import jpet  # noqa: E402

DEV = "cuda"
PIXEL = 2.0
# (events per wavefront, rings, pixels of the longest row)
SHAPES = [(2, 1, 8), (2, 1, 12), (2, 1, 16), (2, 1, 24), (2, 2, 10), (2, 2, 14), (2, 2, 18), (2, 2, 22), (2, 2, 28),
          (2, 3, 14), (2, 3, 18), (2, 3, 22), (2, 3, 26), (1, 1, 32), (1, 1, 48), (1, 1, 64), (1, 2, 16), (1, 2, 22),
          (1, 2, 28), (1, 2, 36), (1, 2, 48), (1, 2, 64), (1, 3, 18), (1, 3, 24), (1, 3, 32), (1, 3, 44), (1, 3, 54),
          (1, 3, 64), (1, 4, 20), (1, 4, 28), (1, 4, 40), (1, 4, 54)]


def resolution(events, rings, length):
    """sigma_z and sigma_dl whose largest ellipse reaches 0.6 rows less than the rings hold (122.4 rows: what
    a region of 256 rows holds), with a longest row of `length` pixels."""
    half_rows = min((16 if events == 2 else 32) * rings - 0.6, 122.4)
    return (length - 0.5) * PIXEL * math.sqrt(2.0) / 6.0, half_rows * PIXEL / 1.5


def rel_l2(a, b):
    return float(np.linalg.norm(a.ravel() - b.ravel()) / max(np.linalg.norm(b.ravel()), 1e-300))


def check(kw, ev_np, rho_np, plan=0):
    g, go = jpet.geometry(**kw, plan=plan), oracle.geometry(**kw)
    ev = torch.from_numpy(ev_np).to(DEV)
    rho = torch.from_numpy(rho_np.astype(np.float32)).to(DEV)
    want, sto, D_want = oracle.mlem(go, ev_np, rho_np.astype(np.float32).astype(np.float64), 1, return_D=True)
    D = jpet.denominators(g, ev, rho).double().cpu().numpy()
    live = D_want > 0
    assert np.array_equal(D > 0, live)
    if live.any() and not kw.get("sigma_z_edge"):  # (with it, the library's D carry the centre's constant factor)
        assert np.max(np.abs(D[live] / D_want[live] - 1)) <= 1e-5
    st = jpet.mlem_iterate(g, ev, rho, 1, want_stats=True)
    got = rho.double().cpu().numpy()
    for key in ("n_valid", "n_dropped", "n_pairs", "n_zero_denominator", "n_kappa_nonpositive"):
        assert st[key] == sto[key], (key, st[key], sto[key])
    assert st["n_unplaced_rows"] == 0
    tol = 2e-6 + 3 * 0.29 * 2.0 ** -23 * math.sqrt(st["n_pairs"]) / max(np.linalg.norm(want), 1e-300)
    err = rel_l2(got, want)
    print(f"plan {jpet.launch_info(g, len(ev_np))['plan']}: rel L2 {err:.2e} (tolerance {tol:.2e})", flush=True)
    assert err <= tol, (err, tol)
    return D, st


@pytest.mark.parametrize("events,rings,length", SHAPES)
def test_every_cache_at_its_edge(events, rings, length):
    sz, sdl = resolution(events, rings, length)
    kw = dict(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=101, n_z=83)
    n = 257
    ev = simulate_events(c1_phantom(), 450.0, 500.0, sz, sdl, n, 11 + length, workers=1)
    rho = np.linspace(0.5, 1.5, 101 * 83).reshape(101, 83)
    g = jpet.geometry(**kw)
    # a plan of the pass on ring blocks with the expected number of events per wavefront
    plans = [c for c, _ in jpet.plan_candidates(g, n)
             if c & 4 and (c >> 12) == 0 and jpet.launch_info(jpet.with_plan(g, c), n)["events_per_batch"] == events]
    assert plans, "no plan"
    check(kw, ev, rho, plan=plans[0])


@pytest.mark.parametrize("n", [1, 2, 3, 255])
@pytest.mark.parametrize("shape", [(2, 1, 12), (2, 3, 22), (1, 3, 44)])
def test_few_events_and_small_grids(n, shape):
    sz, sdl = resolution(*shape)
    for n_y, n_z in ((1, 1), (2, 65), (64, 3), (33, 40)):
        kw = dict(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=n_y, n_z=n_z)
        ev = simulate_events(c1_phantom(), 450.0, 500.0, sz, sdl, n, 5 + n, workers=1)
        check(kw, ev, np.ones((n_y, n_z)))


@pytest.mark.parametrize("scale", [1e-25, 1e-31])
def test_small_denominators(scale):
    """Denominators below 1e-28 take the pass's other way; the step does not depend on the image's scale."""
    sz, sdl = resolution(2, 2, 14)
    kw = dict(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=64, n_z=64)
    ev = simulate_events(c1_phantom(), 450.0, 500.0, sz, sdl, 300, 3, workers=1)
    D, st = check(kw, ev, np.full((64, 64), scale))
    assert st["n_zero_denominator"] == 0 and D[D > 0].min() < 1e-3 * scale


@pytest.mark.parametrize("R,L,sz,sdl,pixel", [(130.0, 300.0, 10.0, 40.0, 4.0), (130.0, 300.0, 12.0, 30.0, 3.0),
                                              (90.0, 400.0, 10.0, 30.0, 3.0), (450.0, 1000.0, 15.0, 90.0, 4.0)])
@pytest.mark.parametrize("gamma,variant,edge", [(0.0, 0, 0.0), (3e-4, 1, 0.1)])
def test_polynomial_and_exact_rows(R, L, sz, sdl, pixel, gamma, variant, edge):
    """Narrow strips and wide angles: rows of both polynomial degrees and exact ones in one pass; every
    event's denominator against the oracle's."""
    n_y = 2 * int(0.45 * 2 * R / pixel / 2)
    kw = dict(R=R, L=L, sigma_z=sz, sigma_dl=sdl, pixel=pixel, n_y=min(n_y, 120), n_z=90, gamma=gamma,
              kernel_variant=variant, sigma_z_edge=edge)
    ev = simulate_events(c1_phantom(), R, L, sz, sdl, 700, 23, workers=1, sigma_z_edge=edge)
    rho = np.linspace(0.2, 2.0, kw["n_y"] * 90).reshape(kw["n_y"], 90)
    check(kw, ev, rho)
