"""The operations that bench.py prices the Hessian's matrix kernel on (host code, no GPU)."""
import pytest

import bench


@pytest.mark.parametrize("c,k", [(1, 2), (2, 2), (2, 3), (3, 3), (4, 1)])
def test_entries_by_tap_offsets_are_the_distinct_ones(c, k):
    # an entry is known from its taps' offset and its channels; turned round it is the same
    seen = set()
    for a in range(k * k):
        for b in range(k * k):
            dy, dx = b // k - a // k, b % k - a % k
            for i in range(c):
                for j in range(c):
                    seen.add(max((dy, dx, i, j), (-dy, -dx, j, i)))
    assert bench.hessian_entries_formed(c * k * k, c) == len(seen)
    assert bench.hessian_entries_formed(c * k * k) == c * k * k * (c * k * k + 1) / 2
