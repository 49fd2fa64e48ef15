"""The parts a batch with host outputs is built in: whole blocks of rows or
events, all rows once, no more parts than a call has room for, and none where
the model of the launches sees too little to gain."""
import itertools

import numpy as np
import pytest

from parts_util import Planner


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return Planner(tmp_path_factory.mktemp("plan"))


SIZES = [(50000,), (20000,) * 10, (10000,) * 4, (20481, 1, 30007, 10240), (20480,), (20479,), (0, 30000, 0), (5,) * 8000,
         (0,), (10240, 10240), (100000, 3, 7)]


@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: f"{len(s)}x{s[0]}")
def test_parts_are_whole_blocks_and_cover_every_row(plan, sizes):
    starts = np.concatenate([[0], np.cumsum(sizes)])
    for geo, cands, layers, pinned in itertools.product((0, 1, 2, 3), (1, 6, 8), (4, 10, 16), (True, False)):
        ends = plan.ends(sizes, [int(1.3 * n) for n in sizes], geo, cands, layers, pinned=pinned)
        assert 1 <= len(ends) <= plan.most and ends[-1] == sum(sizes)
        assert all(a < b for a, b in zip(ends, ends[1:]))
        for e in ends:   # a row that an event or one of its blocks ends at
            i = int(np.searchsorted(starts, e, side="right")) - 1
            assert e in starts or (e - starts[i]) % plan.block == 0
        for spi in (5, 8, 10, 16, 20, 32, 40, 64):
            items = [plan.items(sizes, e, spi) for e in ends]
            assert items[-1] == sum(-(-n // spi) for n in sizes)
            assert all(a < b for a, b in zip(items, items[1:]))
            # as many items as the whole items of the rows before it
            for e, k in zip(ends, items):
                assert k == sum(-(-min(n, max(0, e - s)) // spi) for n, s in zip(sizes, starts))


def test_what_splits_and_what_does_not(plan):
    assert len(plan.ends((50000,), (65000,))) > 1
    assert len(plan.ends((20000,) * 10, (22000,) * 10)) > 1
    assert len(plan.ends((10000,) * 4, (11000,) * 4, geo=1)) > 1
    assert plan.ends((5003,) * 4, (5503,) * 4, geo=2) == [20012]        # less than two blocks
    assert plan.ends((20000,) * 10, (22000,) * 10, us_per_row=0.0) == [200000]   # nothing to deliver
