"""Plans (host code, no GPU).  The units of the 32-bit accumulators: a plan is chosen for its speed, never at the
price of coarser units than batches of rows give the same call.

UNITS holds, for a geometry and a number of events, the power of two a count was divided by when every plan
ran on batches of rows (32: the 64-bit accumulators' units): the call's own plan, and the one a batch takes.
"""

import math

import pytest

from paper_1502_07478_amd import jpet, tune

COUNTS = (1, 500, 3000, 5003, 10000, 20000, 66000, 131100, 263000, 264253, 700000, 10000000)
# (R, L, sigma_z, sigma_dl, pixel, n_y, n_z): units of a single call, units in a batch (None: the same)
UNITS = {
    (450, 500, 10, 63, 2, 400, 400): ((28, 28, 28, 28, 28, 28, 26, 25, 24, 24, 23, 23), None),
    (450, 500, 10, 63, 600 / 256, 256, 256): ((28, 28, 28, 28, 28, 27, 26, 25, 24, 23, 23, 23), None),
    (450, 500, 10, 63, 4, 64, 64): ((27, 27, 27, 27, 27, 27, 26, 25, 24, 24, 23, 23), None),
    (450, 500, 10, 63, 2.5, 200, 200): ((32, 28, 28, 28, 28, 27, 26, 25, 24, 23, 23, 23),
                                        (29, 28, 28, 28, 28, 27, 26, 25, 24, 23, 23, 23)),
    (450, 500, 8.7, 46, 600 / 128, 128, 128): ((26, 26, 26, 26, 26, 26, 25, 25, 24, 24, 23, 23), None),
    (450, 500, 14.2, 88, 600 / 512, 512, 512): ((29, 29, 29, 29, 28, 27, 25, 24, 23, 23, 23, 23), None),
    (450, 500, 10, 63, 4, 61, 77): ((27, 27, 27, 27, 27, 27, 26, 25, 24, 24, 23, 23), None),
    (450, 500, 10, 63, 2, 225, 257): ((28, 28, 28, 28, 28, 28, 26, 25, 24, 24, 23, 23), None),
    (130, 300, 10, 40, 4, 64, 76): ((26, 26, 26, 26, 26, 26, 25, 24, 23, 23, 23, 23), None),
    (450, 1000, 5, 30, 0.5, 1024, 1024): ((29, 29, 29, 29, 29, 28, 26, 25, 24, 24, 23, 23), None),
    (450, 500, 1.5, 26.3, 4, 106, 281): ((32, 26, 26, 26, 26, 26, 25, 25, 24, 24, 23, 32),
                                         (26, 26, 26, 26, 26, 26, 25, 25, 24, 24, 23, 23)),
    (450, 500, 2.1, 12.2, 3.7, 210, 737): ((26, 26, 26, 26, 26, 26, 25, 24, 23, 23, 23, 32),
                                           (26, 26, 26, 26, 26, 26, 25, 24, 23, 23, 23, 23)),
    (300, 700, 5.6, 84.7, 1.34, 401, 973): ((32, 32, 32, 29, 28, 28, 26, 25, 24, 24, 23, 23),
                                            (29, 29, 29, 29, 28, 28, 26, 25, 24, 24, 23, 23)),
}


def unit_of(info):
    return info["accumulator_shift"] if info["accumulator_bits"] == 32 else 32


@pytest.mark.parametrize("geo", list(UNITS))
def test_units_are_not_coarser_than_on_batches_of_rows(geo):
    g = jpet.geometry(*geo)
    single, batch = UNITS[geo]
    for n, want, want_batch in zip(COUNTS, single, batch or single):
        assert unit_of(jpet.launch_info(g, n)) >= want, n
        # a batch takes the first plan of the list that it can run
        listed = jpet.plan_candidates(g, n)
        code = next(c for c, _ in listed if tune.batchable(g, c, n))
        assert unit_of(jpet.launch_info(jpet.with_plan(g, code), n)) >= want_batch, n
        # the call's plan heads the list, whose figures rise
        assert listed[0][0] == jpet.launch_info(g, n)["plan"]
        assert all(a[1] <= b[1] for a, b in zip(listed, listed[1:]))


@pytest.mark.parametrize("geo", list(UNITS))
def test_named_plans_keep_their_units(geo):
    """Every plan code gives units at least as fine as its items on batches of rows: n / 1024 events, whole
    batches, at most 511."""
    g = jpet.geometry(*geo)
    rows = math.floor(3.0 * g.sigma_dl / g.pixel) + 1
    for n in COUNTS:
        for code, _ in jpet.plan_candidates(g, n):
            info = jpet.launch_info(jpet.with_plan(g, code), n)
            if info["accumulator_bits"] != 32:
                continue
            waves = 16 if code & 3 == 2 else 8
            per_batch = min(32, 64 * waves // (rows * info["row_segments"]))
            item = min(max(n // 1024, per_batch), 511) // per_batch * per_batch
            assert unit_of(info) >= 32 - item.bit_length(), (n, code)
            assert info["events_per_workgroup"] < 2 ** (32 - unit_of(info)), (n, code)


@pytest.mark.parametrize("n", [1, 100_000, 3_000_000])
def test_bins_of_the_finest_grids_are_counted(n):
    """32768 x 32768 pixels: a plan of more bins than 32 bits count has a negative number of them, and a workspace
    whose parts overlap."""
    for pixel, sz, sdl in ((0.025, 0.2, 1.0), (0.027, 0.05, 0.3)):
        g = jpet.geometry(R=450.0, L=1000.0, sigma_z=sz, sigma_dl=sdl, pixel=pixel, n_y=32768, n_z=32768)
        for code, _ in jpet.plan_candidates(g, n):
            named = jpet.with_plan(g, code)
            info = jpet.launch_info(named, n)
            rows, cols = -(-32768 // info["tile_rows"]), -(-32768 // info["tile_cols"])
            assert info["bins"] >= info["t_bins"] * rows * cols
            # the accumulators and the log-likelihood's image, and five words a bin
            assert jpet.workspace_size(named, n) > 16 * 32768 ** 2 + 16 * info["bins"]
