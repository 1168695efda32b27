"""The dispatch rules of paper_2609_09095_amd/csrc/dispatch.hpp, on the CPU,
over the sizes that the entry points accept."""
import itertools

import paper_2609_09095_amd as oz
from routes import rules

PLENTY = 1 << 40  # bytes of room for the partial maxima
KS = (1, 63, 64, 65, 256, 1000, 1024, 1025, 4096, 8192, 32768, 65536, 65537, 131072, 262143, 262144, 262145, 1 << 19,
      1 << 20, 1 << 21, oz.MAX_K)


def k_pad(k):
    return -(-k // 128) * 128


def test_joint_deconstruction_key_reads_are_linear_in_k():
    """Every 32-column x 128-k block of the joint deconstruction of B reads the
    scan's partial maxima of its columns, four bytes each: wherever the joint
    launches are taken, at most 2048 per block and column (eight times the
    block's own FP64 bytes), however long k is."""
    L = rules()
    taken = 0
    for m, n, k in itertools.product((1, 16, 64, 512, 1024, 100000), (1, 16, 64, 128, 256, 4096), KS):
        if L.rule_both_at_once(m, n, k, k_pad(k), PLENTY):
            taken += 1
            reads = L.rule_scan_both_slabs(n, k) * 4
            assert reads <= 8 * 128 * 8, (m, n, k, reads)
    assert taken > 100


def test_joint_scan_grid_fits():
    """A launch holds fewer than 2^32 work-items: rows that the separate row
    scan (256 per row) just holds must not be sent to the joint one, whose
    grid has B's slabs beside them."""
    L = rules()
    for n, k in itertools.product((1, 2, 64, 65, 128), (1, 64, 1024, 1025, 4096)):
        for m in (1024, 1 << 20, (1 << 24) - 1000, (1 << 24) - 65, (1 << 24) - 2, (1 << 24) - 1, 1 << 24, 1 << 26):
            if L.rule_both_at_once(m, n, k, k_pad(k), PLENTY):
                assert L.rule_scan_both_blocks(m, n, k) * 256 < 1 << 32, (m, n, k)
    assert not L.rule_both_at_once((1 << 24) - 1, 1, 1025, k_pad(1025), PLENTY)
    assert L.rule_both_at_once((1 << 24) - 100, 1, 1025, k_pad(1025), PLENTY)


def test_tall_product_fills_its_rounds():
    """Moduli per block of the tall/skinny product: with either count a CU
    holds one block and an XCD (32 CUs) every eighth strip of 128 rows; a
    round with five moduli takes 4/3 of one with three.  The chosen count is
    never the slower one by that reckoning, and few strips take three."""
    L = rules()
    for m in [*range(1024, 60000, 97), 262144, 1 << 22, 1 << 24]:
        per = -(-(-(-m // 128)) // 8)
        cost = {g: (4 if g == 5 else 3) * -(-(15 // g) * per // 32) for g in (3, 5)}
        g = L.rule_fused_moduli(m)
        assert cost[g] == min(cost.values()), m
    assert [L.rule_fused_moduli(m) for m in (1024, 6144, 6145, 10241, 12288, 12289, 262144)] == [3, 3, 5, 3, 3, 5, 5]


def test_xcd_ranges_on_the_measured_side():
    """The block placement of the int8 product, at products measured both
    ways (tiles, stages of 128 k, splits): in ranges where that was faster,
    dealt in turn where it was not."""
    rule = rules().rule_xcd_ranges
    for c in ((16, 8, 1), (30, 5, 1), (36, 32, 1), (16, 313, 1), (30, 94, 1), (9, 64, 3), (25, 24, 2), (6, 235, 5), (8, 422, 2)):
        assert rule(*c), c
    for c in ((16, 3, 1), (4, 8, 2), (64, 128, 1), (4, 16, 4), (12, 313, 4), (6, 313, 5), (24, 128, 2), (256, 64, 1)):
        assert not rule(*c), c
