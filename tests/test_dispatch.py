"""The rules that choose a call's kernels, queried on the host (no GPU): each
choice is a launch the runtime accepts and the kernel's on-chip memory holds."""
import ctypes as C
import random

import pytest

import paper_2609_35800_amd as hg
from hgtest import GROUPS, SPLIT, SPREAD, kivi_plan, select_with_values

THREADS, BLOCK_TOKENS = 256, 128  # a workgroup of the quantize kernels


@pytest.mark.parametrize("n", [1, 128, 129, 1000])
@pytest.mark.parametrize("D", [64, 128, 256])
def test_selection_with_the_values_stays_under_the_launch_limit(n, D):
    """The launch of the values with the selection has one workgroup a slice more
    than the values alone; a launch of 2^32 work-items or more is refused."""
    per_slice = -(-n // BLOCK_TOKENS) + 1
    most = (2**32 - 1) // THREADS // per_slice
    assert select_with_values(most, n, D, 2) and not select_with_values(most + 1, n, D, 2)
    assert not select_with_values(2**23, n, D, 2) or 2**23 * per_slice * THREADS < 2**32


# Spans whose norms fit the LDS that the value tiles' occupancy leaves: 160 KiB over
# one workgroup more than stay per compute unit (6 at 2 bits, 5 at 3, 4 at 4 bits and
# at head_dim 256) and 512 bytes, less the selection's 1072 and, at head_dim 256, the
# staged loads' 16 KiB.
@pytest.mark.parametrize("D,bits,limit", [(64, 2, 5711), (128, 2, 5711), (128, 3, 6686), (128, 4, 8052),
                                          (256, 2, 3956), (256, 3, 3956), (256, 4, 3956)])
def test_longest_span_selected_among_the_values(D, bits, limit):
    waves = 4 if bits == 4 or D == 256 else 5 if bits == 3 else 6
    lds = 160 * 1024 // (waves + 1) + 512 - 1072 - (16384 if D == 256 else 0)
    assert limit == lds // 4
    assert select_with_values(8, limit, D, bits) and not select_with_values(8, limit + 1, D, bits)


@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 7, 10, 11, 20, 21, 26, 31, 54, 55, 63])
def test_selections_are_spread_over_the_chip(tiles):
    """Consecutive workgroups go to the 8 XCDs in turn, and those of an XCD to its 32
    compute units: with a slice's selecting workgroup and its `tiles` value tiles in
    one run, no XCD gets more than 1.25 and no compute unit more than 2 times its
    share of the selections (always first, a run of 8 would put all on one XCD)."""
    f = hg.library().hg_test_select_place
    f.argtypes, f.restype = [C.c_uint32, C.c_uint32], C.c_uint32
    run, xcd, cu, slices = tiles + 1, [0] * 8, [0] * 256, 16384
    for s in range(slices):
        at = f(s, run)
        assert at < run
        xcd[(s * run + at) % 8] += 1
        cu[(s * run + at) % 256] += 1
    assert max(xcd) <= 1.25 * slices / 8 and max(cu) <= 2 * slices / 256


# Dequantize with retention: (head_dim, tokens, retained, slices) where the rows were
# measured to be stored faster in the dequantize kernel, or by a launch of their own.
@pytest.mark.parametrize("D,n,k,slices,fused", [
    (128, 3328, 67, 8, True), (128, 1296, 78, 1144, True), (128, 1296, 26, 1432, True), (128, 3328, 50, 568, True),
    (128, 1296, 78, 1432, False), (128, 1296, 130, 1432, False), (128, 5000, 250, 384, False),
    (64, 1296, 26, 1720, False), (64, 1296, 26, 1144, True), (64, 5000, 250, 768, False), (64, 640, 38, 5544, False),
    (256, 1280, 77, 648, True), (256, 1296, 130, 640, True), (128, 1000, 257, 8, False), (128, 3328, 67, 2048, False)])
def test_retained_rows_in_the_dequantize_kernel(D, n, k, slices, fused):
    f = hg.library().hg_test_retain_in_dequantize
    f.argtypes, f.restype = [C.c_uint64, C.c_int64, C.c_int64, C.c_int], C.c_int
    assert bool(f(4 * slices * n * D, n, k, D)) == fused


# Slices past 32 workgroups' rows: spread groups or the split kernels, whichever was
# measured faster (D, rows, slices), 2 and 4 bits, quantize and one-pass.
@pytest.mark.parametrize("D,T,items", [(128, 98304, 5), (128, 100000, 5), (128, 160000, 3), (128, 200000, 5),
                                       (64, 100000, 3), (64, 100000, 5), (64, 400000, 5),
                                       (64, 400000, 17), (256, 25000, 17), (256, 100000, 4), (256, 100000, 5),
                                       (256, 100000, 8), (256, 100000, 17)])
def test_split_kernels_where_spread_groups_are_slower(D, T, items):
    assert kivi_plan(T, D, items)[0] == SPLIT


@pytest.mark.parametrize("D,T,items", [(128, 50000, 1), (128, 50000, 4), (128, 80000, 8), (128, 98304, 6),
                                       (128, 131072, 1), (128, 131072, 2), (128, 131072, 5), (128, 131072, 104),
                                       (128, 300000, 2), (64, 131072, 8), (64, 131072, 104), (64, 600000, 1),
                                       (256, 25000, 1), (256, 25000, 8), (256, 32768, 17), (256, 65536, 1),
                                       (256, 100000, 1), (256, 150000, 4)])
def test_spread_groups_where_they_are_faster(D, T, items):
    assert kivi_plan(T, D, items)[0] == SPREAD


def test_every_plan_fits_the_workspace():
    """The words a plan's launches use lie in the workspace hg_packed_sizes reports,
    and every row of a slice has a slot."""
    rng = random.Random(7)
    for _ in range(4000):
        D = rng.choice([64, 128, 256])
        T = int(2 ** rng.uniform(0, 21))
        L, B, H = rng.randint(1, 80), rng.randint(1, 64), rng.randint(1, 32)
        cfg = hg.make_config(L=L, B=B, H=H, T=T, D=D, img_start=0, img_len=T, bits=2, base="kivi", keys_only=1,
                             kivi_group=0)
        have = hg.hg_packed_sizes(cfg, [0] * (L * H))["workspace"]
        kind, parts, slots, groups, words, _ = kivi_plan(T, D, L * B * H, T, rng.choice([1, 8, 31, 64, 256, 304, 1024]))
        assert words * 8 <= have
        if kind in (GROUPS, SPREAD):
            assert -(-T // parts) <= slots * 8192 // D and (parts == 1 or have > 0)


@pytest.mark.parametrize("T,items,us", [(50000, 1, 24), (131072, 1, 33), (131072, 2, 48), (131072, 104, 1750)])
def test_a_busy_chip_delays_a_spread_call_by_its_own_time_at_most(T, items, us):
    """A poll takes about 1 us; `us`: the whole call measured alone."""
    kind, polls = kivi_plan(T, 128, items)[0::5]
    assert kind == SPREAD and 16 <= polls <= min(128, us)


@pytest.mark.parametrize("D", [64, 128, 256])
def test_the_shortest_form_has_no_wide_groups(D):
    """Groups of more than 8 partners, which exchange in another way, never have the
    form of 8 row slots: it is not built for them."""
    for T in range(8192 // D, 32 * 24 * 8192 // D + 2, 97):
        for items in (1, 9, 60, 1000):
            kind, parts, slots = kivi_plan(T, D, items)[:3]
            assert kind != GROUPS or parts <= 8 or slots > 8
