"""The rules that cut launches into workgroups, over the shapes that the entry points take (host code, no GPU)."""
import pytest

import paper_2509_05576_amd as fobq


# one image or a few, one row or a few of them, aligned or not, channels beyond what the maxima take along
@pytest.mark.parametrize("maxima", [0, 1])
@pytest.mark.parametrize("aligned", [0, 1])
@pytest.mark.parametrize("n,h,w,c,pad", [(1, 1, 100352, 256, 0), (1, 1, 100352, 512, 0), (1, 1, 1 << 18, 64, 1), (1, 4, 50000, 64, 1), (32, 1, 1500, 384, 0),
                                         (1, 2, 200000, 16, 2), (2, 1, 40000, 255, 1), (2, 3, 30000, 1500, 0), (1, 1, 1 << 20, 1, 0), (1, 1, 1, 8192, 0),
                                         (1, 1, 1 << 20, 2000, 64), (64, 56, 56, 128, 1), (1 << 16, 7, 7, 3, 3)])
def test_long_rows_are_cut_until_the_chip_is_full(n, h, w, c, pad, aligned, maxima):
    parts, wgs = fobq.fobq_debug_plan(fobq.PLAN_PAD, [n, h, w, c, pad, aligned, maxima], 2)
    rows = (n + 1) * (h + 2 * pad)
    assert 1 <= parts <= w and 1 <= wgs <= min(rows * parts, 2048)
    # a part is worth a workgroup's while, and no workgroup holds more than a few times its share of what two per compute unit would
    lane = 4 if aligned and c % 4 == 0 else 1
    assert parts == 1 or w * c // lane // parts >= 1024
    share = rows * (w + 2 * pad) * c / 512
    assert -(-rows * parts // wgs) * (w + 2 * pad) * c / parts <= max(3 * share, 3 * 1024 * lane, c)


def test_bad_plans_are_refused():
    for args in ([0, 1, 1, 1, 0, 1, 1], [1, 1, 1, 1, -1, 1, 1], [1, 1, 1 << 20, 4096, 0, 1, 1], [1, 1, 1]):
        with pytest.raises(fobq.FobqError):
            fobq.fobq_debug_plan(fobq.PLAN_PAD, args, 2)
