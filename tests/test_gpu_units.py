"""The accumulators' units seen in an image: ten iterations with the sensitivity on 256 x 256 pixels of 600/256 mm,
whose columns 0.39 mm inside the strips' ends (s = 5e-4) few events reach, against the oracle.

Tolerance (relative L2): every iteration adds the kernel's 2e-6 and three standard deviations of the fixed-point
rounding, 0.29 units per (event, pixel) pair divided by the pixel's sensitivity, in the plan's own units; errors
of earlier iterations are carried on, not amplified (the step's derivative has eigenvalues from 0 to 1), so ten
times that bounds the image."""

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
ITERATIONS = 10
KW = dict(R=450.0, L=500.0, sigma_z=10.0, sigma_dl=63.0, pixel=600.0 / 256, n_y=256, n_z=256)


def pairs_per_pixel(ev):
    """Events whose 3-sigma ellipse holds each pixel centre."""
    zu, zd, dl = ev.astype(np.float64).T
    t = (zu - zd) / (2 * KW["R"])
    c = np.sqrt(1 + t * t)
    y = -0.5 * dl / c
    z = 0.5 * (zu + zd + 2 * y * t)
    pix, n = KW["pixel"], KW["n_z"]
    edges = np.zeros((KW["n_y"], n + 1))
    for i in range(KW["n_y"]):
        dy = (i + 0.5 - 0.5 * KW["n_y"]) * pix - y
        rem = 9.0 - 4.0 * (c * dy / KW["sigma_dl"]) ** 2
        half = np.sqrt(np.maximum(rem, 0.0) * 0.5) * KW["sigma_z"]
        centre = z + t * dy
        lo = np.clip(np.ceil((centre - half) / pix + 0.5 * n - 0.5), 0, n).astype(int)
        hi = np.clip(np.floor((centre + half) / pix + 0.5 * n - 0.5) + 1, 0, n).astype(int)
        ok = (rem >= 0) & (hi > lo)
        np.add.at(edges[i], lo[ok], 1.0)
        np.add.at(edges[i], hi[ok], -1.0)
    return np.cumsum(edges, axis=1)[:, :n]


@pytest.mark.parametrize("n", [3000, 20_000])
def test_columns_beside_the_strips_ends(n):
    ev_np = simulate_events(c1_phantom(), KW["R"], KW["L"], KW["sigma_z"], KW["sigma_dl"], n, 17, workers=4)
    go, g = oracle.geometry(**KW), jpet.geometry(**KW)
    so = oracle.sensitivity(go)
    assert 0 < so[so > 0].min() < 1e-3
    want, sto = oracle.mlem(go, ev_np, oracle.initial_image(so), ITERATIONS, s=so)
    N = pairs_per_pixel(ev_np)
    assert abs(N.sum() - sto["n_pairs"]) <= 1e-4 * sto["n_pairs"]
    live = so > 0
    spread = math.sqrt(float(np.sum(N[live] / so[live] ** 2)))
    ev = torch.from_numpy(ev_np).to(DEV)
    s = jpet.sensitivity(g)
    alone, batched = (s > 0).to(torch.float32), (s > 0).to(torch.float32)
    jpet.mlem_iterate(g, ev, alone, ITERATIONS, s=s)
    jpet.BatchedMLEM([(g, ev, s, batched)]).iterate(ITERATIONS)
    unit = 2.0 ** -jpet.launch_info(g, n)["accumulator_shift"]
    tol = ITERATIONS * (2e-6 + 3 * 0.29 * unit * spread / np.linalg.norm(want))
    for name, image in (("single", alone), ("batched", batched)):
        got = image.double().cpu().numpy()
        err = float(np.linalg.norm(got - want) / np.linalg.norm(want))
        print(f"{name}, {n} events, unit {unit:.1e}: rel L2 {err:.2e} (tolerance {tol:.2e})", flush=True)
        assert err <= tol, (name, err, tol)
