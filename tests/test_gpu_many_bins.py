"""Grids with more bins than the blocks of the preparation's scan sum for themselves: one chunk of 1024 bins a block
(more than 65,536 bins) and several (more than 2,097,152), against the oracle.  Image relative L2 2e-6 plus three
standard deviations of the rounding to units, counts exact; preparing again gives the same counts."""

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
KW = dict(R=450.0, L=1000.0, sigma_z=5.0, sigma_dl=30.0, pixel=0.5, n_y=1024, n_z=1024)


@pytest.mark.parametrize("least,most", [(65_537, 130_000), (2_097_153, 4_000_000)])
def test_scan_of_many_bins(least, most):
    n = 3000
    g = jpet.geometry(**KW)
    plan = next(c for c, _ in jpet.plan_candidates(g, n)
                if c & 4 and least <= jpet.launch_info(jpet.with_plan(g, c), n)["bins"] <= most)
    g = jpet.with_plan(g, plan)
    ev_np = simulate_events(c1_phantom(), 450.0, 1000.0, 5.0, 30.0, n, 3, workers=1)
    rho_np = np.linspace(0.5, 1.5, 1024 * 1024, dtype=np.float32).reshape(1024, 1024)
    want, sto = oracle.mlem(oracle.geometry(**KW), ev_np, rho_np.astype(np.float64), 1)
    ev = torch.from_numpy(ev_np).to(DEV)
    info = jpet.launch_info(g, n)
    print(f"plan {plan}: {info['bins']} bins", flush=True)
    for _ in range(2):
        rho = torch.from_numpy(rho_np).to(DEV)
        st = jpet.mlem_iterate(g, ev, rho, 1, want_stats=True)
        for key in ("n_valid", "n_dropped", "n_pairs", "n_zero_denominator", "n_kappa_nonpositive"):
            assert st[key] == sto[key], (key, st[key], sto[key])
        assert st["n_unplaced_rows"] == 0
        tol = 2e-6 + 3 * 0.29 * 2.0 ** -info["accumulator_shift"] * math.sqrt(st["n_pairs"]) / np.linalg.norm(want)
        err = float(np.linalg.norm(rho.double().cpu().numpy() - want) / np.linalg.norm(want))
        print(f"rel L2 {err:.2e} (tolerance {tol:.2e})", flush=True)
        assert err <= tol
