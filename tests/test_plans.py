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


PART_US, GROUP_US, PRODUCT_US = {1: 7.5, 2: 11.0, 4: 18.0}, 5.0, 3.4       # the rules' weights in us: a part of columns, a sum's own time, one of its products


def _queue_us(r, d, nr, n1, n2, n3):
    """What every workgroup of queues 2 and 3 has to do, and the chain."""
    t, ng = -(-d // 64), -(-r // 64)
    return t * ng * (8 // nr) * PART_US[nr] / n2, t * ng * (t / 2 * PRODUCT_US + GROUP_US) / n3, t * 15.3


# from one block to many, from one row to the most, and a smaller device
@pytest.mark.parametrize("cus", [256, 64])
@pytest.mark.parametrize("d", [1, 64, 65, 200, 256, 512, 1024, 4608])
@pytest.mark.parametrize("r", [1, 64, 300, 2000, 16000, 65535])
def test_no_queue_of_an_elimination_is_left_without_workgroups(r, d, cus):
    nr, n1, n2, n3 = fobq.fobq_debug_plan(fobq.PLAN_ELIMINATE, [cus, r, d], 4)
    assert min(n1, n2, n3) >= 1 and 1 + n1 + n2 + n3 <= cus
    parts, groups, chain = _queue_us(r, d, nr, n1, n2, n3)
    assert groups <= 2.0 * max(parts, chain) + 2 * GROUP_US, (parts, groups, chain)


@pytest.mark.parametrize("layers", [[(40000, 256), (1, 1)], [(65535, 64), (64, 64)], [(20000, 256)] + [(64, 64)] * 30, [(1024, 256)] * 6 + [(64, 100)] * 14,
                                    [(64, 256)] * 256])
def test_no_queue_of_a_batched_elimination_is_left_without_workgroups(layers):
    out = fobq.fobq_debug_plan(fobq.PLAN_ELIMINATE, [256] + [x for layer in layers for x in layer], 4 * len(layers))
    for l, (r, d) in enumerate(layers):
        nr, n1, n2, n3 = out[4 * l:4 * l + 4]
        assert min(n1, n2, n3) >= 1 and nr == out[0]
        parts, groups, chain = _queue_us(r, d, nr, n1, n2, n3)
        assert groups <= 1.5 * max(parts, chain) + 2 * GROUP_US, (r, d, parts, groups, chain)
    assert sum(1 + out[4 * l + 1] + out[4 * l + 2] + out[4 * l + 3] for l in range(len(layers))) <= 256 + 16 * len(layers)


# the wide tiles of the fp64 Hessian are for long calls: in short ones (an image, a small batch) they were 1.3 to 1.9 times as slow
@pytest.mark.parametrize("conv", [0, 1])
@pytest.mark.parametrize("d", list(range(120, 300, 3)) + [129, 160, 161, 257, 288, 289, 512, 2304, 8192])
def test_short_hessian_calls_take_the_small_tiles(d, conv):
    wide = 160 if 129 <= d <= 160 else 96 if 257 <= d <= 288 else 0
    for n in (1, 196, 2048, 4095, 4096, 8192, 24575, 24576, 400000, (1 << 31) - 65):
        tile, slabs, touched = fobq.fobq_debug_plan(fobq.PLAN_HESSIAN, [d, n, conv], 3)
        assert tile == wide if wide and n >= (4096 if wide == 160 else 24576) else tile in (64, 128)
        assert 1 <= touched <= slabs


# slabs grown by a first call are freed and taken again in it, 0.3 ms
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("c", list(range(64, 1025, 64)) + [2048, 32, 48, 100, 65, 3])
def test_a_first_call_by_tap_offsets_finds_its_slabs(c, k):
    if c * k * k > 32768:
        return
    reserved, wanted = fobq.fobq_debug_plan(fobq.PLAN_SLABS, [c, k], 2)
    assert reserved >= max(wanted, 1)
    if c % 64 or k not in (2, 3) or c * k * k < 384:
        assert wanted == 0
