"""The byte counts behind the benchmark's arm-domain figures follow the launches
that the kernels make, not one pass at a time."""
import itertools

import pytest

import bench


def test_pass_launches():
    assert bench.pass_launches((0, 1, 2, 3)) == [(0,), (1, 2), (3,)]
    assert bench.pass_launches((0, 2, 1, 3)) == [(0, 2), (1, 3)]
    assert bench.pass_launches((0, 1, 2, 3, 4, 5)) == [[0], [1, 2], [3, 4], [5]]
    assert bench.pass_launches((0, 2, 4, 1, 3, 5)) == [[0, 2, 4], [1, 3, 5]]
    for arms in (4, 6):
        for order in itertools.permutations(range(arms)):
            groups = bench.pass_launches(order)
            assert [a for g in groups for a in g] == list(order)
            assert 2 <= len(groups) <= (3 if arms == 4 else 4)
            assert not any(a ^ 1 in g for g in groups for a in g)      # no two opposite arms in a launch


def test_bytes_per_update():
    # square lattice, two orders in three: 2 x (4 read + 2 written); else 5 + 6 + 5
    assert bench.pass_bytes_per_update(4) == pytest.approx((2 / 3 * 12 + 1 / 3 * 16) / 4)
    # cubic: 6 planes per launch, one eta plane and one written plane per arm
    orders = list(itertools.permutations(range(6)))
    launches = sum(len(bench.pass_launches(o)) for o in orders) / len(orders)
    assert bench.pass_bytes_per_update(6) == pytest.approx((6 * launches + 12) / 6)
