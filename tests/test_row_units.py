"""Host checks of how the row GEMMs' launches are cut into units and of their
workspace, over GPUs of any number of compute units (a partitioned one has 128,
64 or 32)."""
import random

import pytest

import row_units as R

KINDS = [1, 2, 3, 31, 32, 38, 64, 104, 128, 200, 255, 256, 304, 585]


@pytest.mark.parametrize("G", KINDS)
def test_workspace_holds_its_layout(G):
    """What a caller is asked for holds counters and pieces, so the workspace
    is used (K pieces, both products in one launch) and not passed over."""
    h = R.lib()
    assert h.fits(G)
    assert h.used(G) <= h.bytes(G)
    # arrival counters of both products below the queue counters
    assert 2 * h.max_cut(G) * 4 <= 4096


def test_workspace_size_is_the_interface_s():
    from paper_2606_11867_amd import load
    assert load().foremoe_ffn_workspace_size() in {R.lib().bytes(G) for G in range(1, 1025)}


def test_units_cover_every_tile_and_pieces_stay_in_their_slots():
    rng = random.Random(7)
    for _ in range(4000):
        rows = [int(rng.choice([0, 1, 64, 65, 128, 129, 256, rng.expovariate(1 / 400), rng.expovariate(1 / 4000)]))
                for _ in range(rng.randint(1, 40))]
        G, phases, ws = rng.choice(KINDS), rng.choice([1, 2, 3]), rng.random() < 0.7
        d, F = 128 * rng.randint(1, 60), 128 * rng.randint(1, 30)
        for fn in (R.forward, R.dgrad):
            u0, u1, t = fn(rows, d, F, phases=phases, G=G, ws=ws)
            assert t.full == sum(r // 256 + (r % 256 > 128) for r in rows)
            assert t.short == sum(64 < r % 256 <= 128 for r in rows)
            assert t.thin == sum(0 < r % 256 <= 64 for r in rows)
            for bit, u in ((1, u0), (2, u1)):
                tiles = (t.full + t.short + t.thin) * u.nt
                cut = tiles - u.plain
                assert 0 <= cut <= tiles and u.h in (1, 2) and 1 <= u.s <= 4
                assert u.full_cut == max(0, cut - u.small)
                assert u.s == 1 or ws and u.kt // u.s >= 8
                n = u.full_cut * u.h + cut - u.full_cut
                assert u.s == 1 or n * u.s <= R.lib().max_cut(G)
                assert u.s == 1 or u.full_cut == 0 or u.h == 2  # a piece fits 128 KiB
                assert u.total == (u.plain + n * u.s if phases & bit else 0)
