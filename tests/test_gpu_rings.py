"""The event pass on ring blocks at the edges of its register caches, against the oracle.

Every shape of the cache (one or two events per wavefront, rings of rows, pixels of the longest row)
with ellipses that just fit it, on a grid that cuts many of them.

Tolerance of the image (relative L2): 2e-6 for the single-precision kernel (the exponent, at most 13 in
magnitude, carries a few roundings of 2^-24) plus three standard deviations of the fixed-point
rounding, 0.29 units of 2^-23 per (event, pixel) pair.  A single event's denominator: 1e-5 (all its
pixels may share the roundings of the event's constants, each up to 2^-24 of an exponent near 13).
Counts: exact.  Log-likelihood: the value relative 1e-6 and dl/drho relative L2 1e-5 (an event's denominator
divides every term of its back-projection); a sigma derivative, whose events may cancel, relative 1e-3 plus
1e-5 of n / sigma, the size of its terms.
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


@pytest.mark.parametrize("events,rings,length", SHAPES)
@pytest.mark.parametrize("gamma,variant", [(0.0, 0), (3e-4, 1)])
def test_log_likelihood_at_every_cache(events, rings, length, gamma, variant):
    """Value, all gradients and the value alone, the ellipses held at sigmas 1.1 times the kernel's."""
    mask = resolution(events, rings, length)
    gamma = min(gamma, 0.3 / (mask[0] * mask[1]))  # a correlation well inside the domain, |gamma| sigma sigma < 1
    kw = dict(R=450.0, L=500.0, sigma_z=mask[0] / 1.1, sigma_dl=mask[1] / 1.1, pixel=PIXEL, n_y=101, n_z=83,
              gamma=gamma, kernel_variant=variant)
    n = 257
    ev_np = simulate_events(c1_phantom(), 450.0, 500.0, kw["sigma_z"], kw["sigma_dl"], n, 31 + length, workers=1)
    check_log_likelihood(kw, ev_np, mask)


@pytest.mark.parametrize("R,L,sz,sdl,pixel", [(130.0, 300.0, 10.0, 40.0, 4.0), (90.0, 400.0, 10.0, 30.0, 3.0)])
def test_log_likelihood_of_polynomial_and_exact_rows(R, L, sz, sdl, pixel):
    n_y = min(2 * int(0.45 * R / pixel), 120)
    kw = dict(R=R, L=L, sigma_z=sz, sigma_dl=sdl, pixel=pixel, n_y=n_y, n_z=90, gamma=3e-4, kernel_variant=1)
    check_log_likelihood(kw, simulate_events(c1_phantom(), R, L, sz, sdl, 700, 23, workers=1), None)


def check_log_likelihood(kw, ev_np, mask):
    g, go, n = jpet.geometry(**kw), oracle.geometry(**kw), len(ev_np)
    ev = torch.from_numpy(ev_np).to(DEV)
    rho_np = np.linspace(0.5, 1.5, kw["n_y"] * kw["n_z"]).reshape(kw["n_y"], kw["n_z"]).astype(np.float32)
    rho = torch.from_numpy(rho_np).to(DEV)
    so = oracle.sensitivity(go)
    s = torch.from_numpy(so.astype(np.float32)).to(DEV)
    l, dz, dd, gr, sto, D_want = oracle.loglik_grad(go, ev_np, rho_np, s=so, sigma_mask=mask, return_D=True)
    res = jpet.loglik_grad(g, ev, rho, s=s, sigma_mask=mask, want_D=True, want_stats=True)
    for key in ("n_valid", "n_dropped", "n_pairs", "n_zero_denominator", "n_kappa_nonpositive"):
        assert res.stats[key] == sto[key], (key, res.stats[key], sto[key])
    D, live = res.D.double().cpu().numpy(), D_want > 0
    assert live.any() and np.array_equal(D > 0, live)
    value = res.value.cpu().numpy()
    errs = (abs(value[0] / l - 1), abs(value[1] - dz), abs(value[2] - dd),
            rel_l2(res.grad_rho.double().cpu().numpy(), gr), float(np.max(np.abs(D[live] / D_want[live] - 1))))
    print("errors " + " ".join(f"{e:.1e}" for e in errs), flush=True)
    assert errs[0] <= 1e-6 and errs[3] <= 1e-5 and errs[4] <= 1e-5, errs
    assert errs[1] <= 1e-3 * abs(dz) + 1e-5 * n / kw["sigma_z"], (value[1], dz)
    assert errs[2] <= 1e-3 * abs(dd) + 1e-5 * n / kw["sigma_dl"], (value[2], dd)
    alone = jpet.loglik_grad(g, ev, rho, s=s, sigma_mask=mask, value_only=True)
    assert alone.value[0].item() == pytest.approx(l, rel=1e-6)


@pytest.mark.parametrize("image", ["plain", "zero band", "tiny band", "bright spot"])
def test_large_items_take_their_units_from_the_bits(image):
    """Items of 128 events and more form their units without a conversion, but for regions with pixels outside
    the range that allows it, here a band of 1e-25 and a spot of 1e9: the same bounds hold for all."""
    sz, sdl = resolution(2, 1, 12)
    kw = dict(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=101, n_z=83)
    ev = simulate_events(c1_phantom(), 450.0, 500.0, sz, sdl, 140_000, 3, workers=4)
    assert jpet.launch_info(jpet.geometry(**kw), len(ev))["events_per_workgroup"] >= 128
    rho = np.linspace(0.5, 1.5, 101 * 83).reshape(101, 83)
    if image != "plain":
        rho[40:60] *= {"zero band": 0.0, "tiny band": 1e-25, "bright spot": 1.0}[image]
    if image == "bright spot":
        rho[50, 40] = 1e9
    check(kw, ev, rho)
