"""jpet_mlem_iterate_noalloc with a list that its array holds on batches of rows only, against jpet_mlem_iterate
(on ring blocks): one iteration, relative L2 1e-5 (two layouts of the same step, each within 2e-6 and the rounding to
units of 2^-23), the same counts.  The default plan and a named one."""

import numpy as np
import pytest

from jpet_synth.events import simulate_events
from jpet_synth.phantom import c1_phantom

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1502_07478_amd import jpet  # noqa: E402

DEV = "cuda"


@pytest.mark.parametrize("n,plan", [(849_000, 0), (809_000, 2253)])
def test_list_beyond_the_ring_blocks_space(n, plan):
    g = jpet.geometry(R=450.0, L=500.0, sigma_z=19.8, sigma_dl=15.9, pixel=1.79, n_y=73, n_z=200, plan=plan)
    assert jpet.workspace_size(g, n) > jpet.NOALLOC_SCRATCH_BYTES
    ev = torch.from_numpy(simulate_events(c1_phantom(), 450.0, 500.0, 19.8, 15.9, n, 3, workers=4)).to(DEV)
    s = jpet.sensitivity(g)
    a, b = (s > 0).to(torch.float32), (s > 0).to(torch.float32)
    sa = jpet.mlem_iterate_noalloc(g, ev, a, 1, s=s, want_stats=True)
    sb = jpet.mlem_iterate(g, ev, b, 1, s=s, want_stats=True)
    assert sa == sb and sa["n_unplaced_rows"] == 0
    x, y = a.double().cpu().numpy(), b.double().cpu().numpy()
    assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(y)
