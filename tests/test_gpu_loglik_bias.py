"""The resolution derivatives of the log-likelihood are sums over the events of terms of size 1 / sigma that cancel to
a few percent: an error that every event shares stays, while roundings of their own average out.

Tolerance, of n / sigma: 2^-26, half of what a constant rounded to single precision may be off, for what is shared
(constants are applied in double precision; a row's polynomial is within 1e-7 at its ends, a tenth of that in the
mean), and four roundings of 2^-24 an event, independent: over the square root of n."""

import math

import pytest

import oracle
from jpet_synth.events import simulate_events
from jpet_synth.phantom import c1_phantom

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1502_07478_amd import jpet  # noqa: E402

DEV = "cuda"
N = 20_000
# (L, sigma_z, sigma_dl, pixel, n_y, n_z, kernel variant, gamma): the events' resolution; the kernel's is 0.92 and
# 0.95 times it
SETTINGS = [(500.0, 14.11, 87.48, 7.949, 81, 82, 1, 0.0), (500.0, 5.52, 78.88, 2.4579, 289, 334, 0, 2e-4),
            (1000.0, 14.53, 57.39, 2.002, 298, 315, 0, 0.0), (500.0, 10.0, 63.0, 2.5, 200, 200, 0, 0.0)]


@pytest.mark.parametrize("L,sigma_z,sigma_dl,pixel,n_y,n_z,variant,gamma", SETTINGS)
def test_resolution_derivatives_have_no_shared_error(L, sigma_z, sigma_dl, pixel, n_y, n_z, variant, gamma):
    ev_np = simulate_events(c1_phantom(), 450.0, L, sigma_z, sigma_dl, N, 41, workers=4)
    sz, sd = 0.92 * sigma_z, 0.95 * sigma_dl
    kw = dict(R=450.0, L=L, sigma_z=sz, sigma_dl=sd, pixel=pixel, n_y=n_y, n_z=n_z, kernel_variant=variant, gamma=gamma)
    g, go = jpet.geometry(**kw), oracle.geometry(**kw)
    rho = (jpet.sensitivity(g) > 0).to(torch.float32)
    l, dz, dd, gr, sto = oracle.loglik_grad(go, ev_np, rho.cpu().numpy())
    value = jpet.loglik_grad(g, torch.from_numpy(ev_np).to(DEV), rho, want_grad_rho=False).value.cpu().numpy()
    n = sto["n_valid"]
    size = 2.0 ** -26 + 4 * 2.0 ** -24 / math.sqrt(n)
    off = abs(value[1] - dz) * sz / n, abs(value[2] - dd) * sd / n
    print(f"derivatives {dz * sz / n:.3f} and {dd * sd / n:.3f} of n / sigma, off by {off[0]:.1e} and {off[1]:.1e} "
          f"(tolerance {size:.1e})", flush=True)
    assert max(off) <= size
