"""The 16-bit path's attention plan (csrc/plan.h) and launch rules (csrc/launch_rules.h), built with the host compiler: pieces cover every row tile's keys once, and no
row of the row space -- filler rows between users included -- is said to have more partial sums than the call lays out.  The
layer tail reads what the row's entry says even where it drops the values, so this cannot be seen in any output."""
import random

import pytest

import plan_util
from plan_util import check


@pytest.fixture(scope="module")
def shim():
    return plan_util.shim()


@pytest.mark.parametrize("L,heads,dh", [
    ([2574, 9519], 2, 64),             # pieces of 25 key tiles; the filler rows from position 9600 would be 7 pieces of a possible 6
    ([3953, 8010, 346, 1573], 2, 64),  # 21; 7 of 6
    ([3841], 8, 128), ([3968], 8, 128),   # 31; 3 of 2
])
def test_filler_rows_have_no_more_sums_than_the_call_lays_out(shim, L, heads, dh):
    got = check(shim, L, heads=heads, dh=dh)
    assert got["blocks"] == 1 and got["nsplit"] > 1 and got["filler"] >= 1


def test_two_splits_share_a_workgroup_where_every_row_has_an_even_number(shim):
    assert check(shim, [4096] * 16, [0] * 16, [512] * 16, [0] * 16) == {"blocks": 2, "nsplit": 1, "gs": 2, "items": 32, "filler": 0}


@pytest.mark.parametrize("L,S,M,heads,dh,sums,items", [
    # a launch that leaves half of the chip free is cut finer than eight key tiles
    ([512], [0], [64], 8, 64, 4, 4), ([1024], [0], [512], 8, 64, 8, 32), ([2048], [0], [64], 8, 64, 8, 8), ([200], [0], [64], 8, 64, 2, 2),
    ([2048], [0], [256], 4, 128, 8, 16), ([512] * 24, [0] * 24, [32] * 24, 4, 64, 2, 48),
    # and one that does not, is not
    ([2048] * 8, [16] * 8, [256] * 8, 2, 64, 5, 120), ([2048], [0], [512], 8, 128, 4, 16), ([2048], [0], [1024], 8, 64, 4, 32),
    # equal items are cut into no more pieces than the chip takes at a time (512 workgroups, 256 at d_head 128)
    ([4096] * 12, [0] * 12, [300] * 12, 4, 64, 3, 108), ([1024] * 40, [0] * 40, [128] * 40, 8, 64, 1, 40),
    ([512] * 40, [0] * 40, [32] * 40, 4, 64, 2, 80), ([512] * 40, [0] * 40, [33] * 40, 4, 64, 1, 40), ([512] * 65, [0] * 65, [32] * 65, 4, 64, 1, 65),
    ([4096] * 10, [0] * 10, [300] * 10, 8, 64, 2, 60), ([2048] * 8, [0] * 8, [256] * 8, 8, 128, 2, 32),
])
def test_pieces_of_equal_items_fit_the_chip_and_small_launches_are_cut_finer(shim, L, S, M, heads, dh, sums, items):
    got = check(shim, L, S, M, [0] * len(L), heads, dh)
    assert (got["nsplit"] * got["gs"], got["items"]) == (sums, items)


@pytest.mark.parametrize("L,M,computed,sums,last", [
    ([4096] * 16, [512] * 16, 0, 1, 1), ([8192] * 32, [1000] * 32, 0, 1, 1),   # two pieces of a row meet inside a workgroup; uncut
    ([64], [512], 0, 1, 1), ([256], [512], 0, 2, 2), ([384], [512], 0, 4, 4), ([512], [512], 0, 4, 4), ([520], [512], 0, 8, 8), ([4096], [512], 0, 8, 8),   # one user's candidates
    ([100, 384], [30, 30], 0, 4, 4), ([64, 256], [30, 30], 0, 2, 2),           # rows with different numbers
    ([4096], None, 1, 4, 1),                                                  # a pre-inference has no rows in its last layer
    ([64], [64], 1, 1, 1), ([600], [200], 1, 4, 2),
])
def test_layer_tail_has_as_many_sums_in_flight_as_its_rows_have(shim, L, M, computed, sums, last):
    """It loads that many of every row, needed or not: launches of one or two sums a row must not take the kernels for more."""
    assert plan_util.sums_in_flight(L, M, computed=[computed] * len(L)) == (sums, last)


@pytest.mark.parametrize("L,M,computed,heads,dh,sums", [
    ([600], None, 1, 4, 64, 3), ([1000] * 4, None, 4, 4, 64, 4), ([600] * 8, None, 8, 4, 64, 3), ([1000], None, 1, 8, 128, 4),    # up to 3/8 of the slots
    ([1000] * 4, None, 4, 8, 64, 2), ([1000] * 16, None, 16, 4, 64, 2), ([600] * 16, None, 16, 4, 64, 2), ([1000] * 2, None, 2, 8, 128, 2),
    ([600], [64], 1, 8, 64, 3), ([1000] * 4, [64] * 4, 1, 8, 64, 4), ([600], [64], 1, 8, 128, 3),                                 # with new rows 3/16
    ([1000] * 4, [256] * 4, 1, 8, 64, 2), ([1000] * 16, [128] * 16, 4, 4, 64, 2), ([1000] * 32, [64] * 32, 9, 4, 64, 2),
])
def test_lists_with_prefix_rows_are_cut_finer_only_while_they_are_small(shim, L, M, computed, heads, dh, sums):
    got = check(shim, L, None, M, [int(u < computed) for u in range(len(L))], heads=heads, dh=dh)
    assert got["nsplit"] == sums


@pytest.mark.parametrize("heads,dh", [(4, 32), (16, 32), (1, 128), (2, 64), (4, 64), (8, 64), (16, 64), (2, 128), (8, 128)])
def test_every_row_has_the_sums_its_pieces_write(shim, heads, dh):
    rng = random.Random(heads * 1000 + dh)
    for _ in range(300):
        n = rng.choice([1, 1, 2, 3, 5, 17])
        top = rng.choice([300, 3000, 20000 if n < 5 else 5000])

        def length(lo):
            return rng.choice([lo, rng.randint(lo, top), rng.randint(lo, top) // 64 * 64 + rng.choice([0, 1, 63]), rng.randint(lo, top) // 256 * 256 + rng.choice([0, 1, 127, 128, 129])])

        L = [length(0) for _ in range(n)]
        kind = rng.choice(["prefill", "rank", "full", "mixed"])
        S = M = None
        computed = [int(l > 0) for l in L]
        if kind != "prefill":
            S = [rng.choice([0, 0, rng.randint(1, 200)]) for _ in range(n)]
            M = [rng.choice([0, 1, 128, 129, rng.randint(1, 2000)]) for _ in range(n)]
            if kind == "rank":
                computed = [0] * n
            elif kind == "mixed":
                computed = [c and rng.randint(0, 1) for c in computed]
        if kind == "prefill":
            L = [max(1, l) for l in L]
            computed = [1] * n
        if sum(L) + sum(M or []) == 0:
            continue
        check(shim, L, S, M, computed, heads, dh, rng.choice([256, 256, 304, 64]), rng.choice([8, 8, 1, 2, 3, 5]))


@pytest.mark.parametrize("attention,L,M,computed,longest,shared", [
    ("silu", [4096], [512], 0, 8, False), ("silu", [4608], [512], 0, 9, False), ("silu", [5120], [512], 0, 10, True), ("silu", [16384], [100], 0, 32, True),
    ("softmax", [7680], [512], 0, 15, False), ("softmax", [8192], [512], 0, 16, True),
    ("silu", [16384] * 5, [512] * 5, 0, 86, False),              # more pieces than compute units
    ("silu", [512] * 16, [512] * 16, 0, 8, False),                  # 256-row items, one a unit; longer ones are paired by the plan
    ("silu", [8192], [64], 1, 35, False), ("silu", [8192], None, 1, 32, False),                      # lists with prefix rows
])
def test_long_pieces_of_few_128_row_items_are_shared(attention, L, M, computed, longest, shared):
    got = plan_util.shared_pieces(attention, L, None, M, [computed] * len(L))
    assert got == (longest, (16 if attention == "softmax" else 10) if shared else None)


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("heads,dh,n_cus", [(2, 64, 256), (8, 64, 256), (8, 64, 104), (4, 128, 256), (4, 32, 256)])
def test_a_users_pieces_in_a_small_call_do_not_depend_on_the_other_histories(attention, heads, dh, n_cus):
    """Up to slots / 16 (row tile, head) pairs.  The pieces and the groups that take them are the order in which a row's sums are added."""
    rng = random.Random(heads * dh)
    pairs = min(512, n_cus if dh == 128 else 2 * n_cus) // 16
    for _ in range(300):
        n = rng.randint(2, 4)
        M = [rng.randint(1, 300) for _ in range(n)]
        if sum((m + 127) // 128 for m in M) * heads > pairs:
            continue
        S = [0] * n
        own = rng.choice([rng.randint(0, 1500), rng.randint(0, 20000)])
        seen = {str(plan_util.user_pieces([own] + [rng.choice([rng.randint(0, 1500), rng.randint(0, 20000)]) for _ in range(n - 1)], S, M, 0, attention, heads, dh, n_cus))
                for _ in range(8)}
        assert len(seen) == 1, (own, M, seen)


@pytest.mark.parametrize("d,nblk,borders", [
    (128, 4, [(1, "64x64"), (2049, "64x128"), (12289, "stationary")]),
    (128, 2, [(1, "64x64"), (4097, "64x128"), (24577, "stationary")]),
    (256, 4, [(1, "64x64"), (1025, "64x128"), (6145, "128x128"), (8193, "128x128/3"), (12289, "stationary")]),
    (256, 2, [(1, "64x64"), (2049, "64x128"), (12289, "128x128"), (16385, "128x128/3"), (24577, "stationary")]),
    (512, 4, [(1, "64x64"), (513, "64x128"), (1025, "128x128"), (2049, "64x128"), (3073, "128x128"), (4097, "128x128/3"), (6145, "stationary")]),
    (512, 2, [(1, "64x64"), (1025, "64x128"), (2049, "128x128"), (4097, "64x128"), (6145, "128x128"), (8193, "128x128/3"), (12289, "stationary")]),
    (1024, 4, [(1, "64x64"), (257, "64x128"), (513, "128x128"), (1025, "64x128"), (1537, "256x128")]),
    (1024, 2, [(1, "64x64"), (513, "64x128"), (1025, "128x128"), (2049, "64x128"), (3073, "256x128")]),
])
def test_projection_tiles_by_rows(d, nblk, borders):
    """Where a projection launch changes its tile: a border that moves takes the GPU tests of that border with it."""
    tiles = [(rows, plan_util.projection_tile(d, rows, nblk)) for rows in range(1, 30001)]
    assert [t for t, before in zip(tiles, [(0, "")] + tiles) if t[1] != before[1]] == borders


@pytest.mark.parametrize("n_cus", [64, 104, 256, 304])
def test_projection_tiles_are_built_for_their_width(n_cus):
    built = {128: {"64x64", "64x128", "stationary", "256x128"}, 1024: {"64x64", "64x128", "128x128", "256x128"}}
    for d, tiles in built.items():
        for nblk in (2, 4):
            assert {plan_util.projection_tile(d, rows, nblk, n_cus) for rows in range(1, 40001, 63)} <= tiles
