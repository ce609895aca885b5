"""GPU parity where a launch changes its kernel or its shape: row counts at both sides of the edges of the layer tail's workgroups
(8, 16 and 32 rows, the partly filled last one) with few and with many partial sums a row, and of the projection's tiles (64 x 64,
64 x 128, 128 x 128 with four and with three stages, 256 x 128, the weight-stationary form), with prefix, suffix and candidate rows; and where a wavefront of the attention
stops at its rows' last key tile before the others of its workgroup do.  Every case ranks on the cached prefix
and by full recompute, against the CPU oracle; at d = 128 with the boosted weights, which let attention reach the scores there."""
import numpy as np
import pytest

import paper_2601_01712_amd as rg
import plan_util
import synth
from gpu_util import BOOST, Harness, build_case
from test_gpu_parity import run_three_routes

pytestmark = pytest.mark.gpu

#   d, heads, dtype, prefix lengths, suffix lengths, candidates
TAIL = [
    (256, 4, "bf16", [600], [0], [1]),            # one row of five pieces
    (512, 8, "bf16", [600], [3], [4]),            # 7 rows: a workgroup of 8 not full
    (512, 8, "fp16", [520], [0], [17]),           # 8 + 8 + 1
    (256, 4, "bf16", [600, 70], [0, 5], [1019, 0]),   # 1024 rows: the last launch of 8-row workgroups
    (256, 4, "fp16", [600, 70], [0, 5], [1020, 0]),   # 1025: the first one of 16-row workgroups, unequal pieces
    (512, 8, "bf16", [130], [1], [1033]),         # 16-row workgroups, few pieces
    (128, 2, "bf16", [100], [0], [33]),           # the d = 128 kernel: 32 + 1
    (1024, 8, "bf16", [70], [0], [33]),           # d = 1024: workgroups of 8, the last of one row (32: WIDE_TAIL)
]


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("case", range(len(TAIL)))
def test_layer_tail_edges(case, attention):
    d, heads, dtype, L, S, M = TAIL[case]
    run_three_routes(synth.ModelConfig(2, d, heads, dtype, attention=attention), 7100 + case, L, S, M, page_tokens=64, boost=BOOST if d == 128 else None)


#   d, heads, dtype, prefix lengths, suffix lengths, candidates; the cached ranking's rows a workgroup and sums in flight, and the most sums a row has
SUMS = [
    (512, 8, "bf16", [64], [0], [9], 8, 1, 1),
    (256, 4, "fp16", [200], [0], [300], 8, 2, 2),
    (512, 8, "fp16", [60, 250], [0, 1], [30, 75], 8, 4, 3),          # users with one and with three
    (256, 4, "bf16", [440], [3], [20], 8, 4, 4),
    (512, 8, "bf16", [512], [0], [9], 8, 4, 4),
    (512, 8, "bf16", [1024], [0], [33], 8, 8, 8),
    (256, 4, "bf16", [960], [9], [5], 8, 8, 8),
    (512, 8, "bf16", [60], [0], [1025], 16, 1, 1),
    (256, 4, "fp16", [250], [0], [1100], 16, 2, 2),
    (256, 4, "bf16", [440], [3], [1030], 16, 4, 4),
    (512, 8, "fp16", [330], [0], [1100], 16, 4, 3),
    (256, 4, "bf16", [4033], [0], [1030], 16, 8, 8),
    (128, 2, "bf16", [64], [0], [300], 32, 1, 1),
    (128, 2, "fp16", [250], [0], [300], 32, 2, 2),
    (128, 2, "bf16", [1100], [3], [290], 32, 8, 7),                  # (two at a time)
    (256, 4, "bf16", [65] * 17, [0] * 17, [250] * 17, 32, 1, 1),
    (512, 8, "bf16", [65] * 17, [0] * 17, [250] * 17, 32, 1, 1),
    (128, 2, "bf16", [65] * 25, [0, 3] * 12 + [0], [1000] * 25, 64, 1, 1),
    (256, 4, "fp16", [65] * 25, [0, 3] * 12 + [0], [1000] * 25, 64, 1, 1),
    (512, 8, "bf16", [65] * 25, [0, 3] * 12 + [0], [1000] * 25, 64, 1, 1),
    (256, 4, "bf16", [65] * 24 + [1500], [0] * 25, [1000] * 25, 64, 4, 3),   # (two at a time)
]


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("case", range(len(SUMS)))
def test_layer_tail_sums_in_flight(case, attention):
    d, heads, dtype, L, S, M, rows, sums, most = SUMS[case]
    assert plan_util.tail_rows(d, sum(S) + sum(M)) == rows
    cached = {"computed": [0] * len(L), "heads": heads, "dh": d // heads}
    assert plan_util.sums_in_flight(L, M, S, **cached) == (sums, sums)
    assert plan_util.check(plan_util.shim(), L, S, M, **cached)["nsplit"] == most
    run_three_routes(synth.ModelConfig(1 if sum(L) + sum(M) > 5000 else 2, d, heads, dtype, attention=attention), 7400 + case, L, S, M, page_tokens=64,
                     boost=BOOST if d == 128 else None)


#   d, heads, dtype, prefix lengths, suffix lengths, candidates; tiles of the launches of all four columns: cached ranking, full recompute
PROJECTION = [
    (128, 2, "bf16", [70], [3], [64], "64x64", "64x64"),              # two row tiles
    (128, 2, "fp16", [70, 0], [3, 1], [2100, 70], "64x128", "64x128"),
    (256, 4, "bf16", [70], [65], [959], "64x64", "64x128"),           # 1024 rows: the last launch of 64 x 64 tiles
    (256, 4, "fp16", [70], [65], [960], "64x128", "64x128"),          # 1025
    (256, 4, "bf16", [70], [70], [2010], "64x128", "64x128"),
    (256, 4, "bf16", [130], [65], [6079], "64x128", "128x128"),       # 6144
    (256, 4, "fp16", [700, 130], [65, 0], [6000, 80], "128x128", "128x128"),   # 6145; two users' prefixes with filler between them
    (256, 4, "bf16", [700, 130], [65, 0], [6000, 80], "128x128", "128x128"),
    (256, 4, "fp16", [300], [0], [8192], "128x128", "128x128/3"),     # 8192
    (256, 4, "bf16", [1100], [70], [8123], "128x128/3", "128x128/3"), # 8193
    (512, 8, "bf16", [130], [5], [507], "64x64", "64x128"),           # 512 rows: the last of 64 x 64
    (512, 8, "fp16", [130], [5], [508], "64x128", "64x128"),          # 513
    (512, 8, "bf16", [130], [5], [1020], "128x128", "128x128"),       # 1025
    (512, 8, "bf16", [1990], [5], [60], "64x64", "64x128"),           # recomputed prefix of 2048 rows with filler, V token-major
    (512, 8, "fp16", [1100], [70], [300], "64x64", "128x128"),        # 1650 rows with a prefix, one of the tiles half filler
    (512, 8, "bf16", [130], [5], [3068], "128x128", "128x128"),       # 3073: the second range of four stages
    (512, 8, "fp16", [70], [1], [4096], "128x128/3", "128x128/3"),    # 4097
    (512, 8, "bf16", [200, 4100], [0, 5], [9, 700], "64x128", "128x128/3"),   # two users' prefixes
    (1024, 8, "bf16", [70], [33], [223], "64x64", "64x128"),          # 256 rows: 64 x 64 with a ring
    (1024, 8, "fp16", [70], [33], [224], "64x128", "128x128"),        # 257
    (1024, 8, "bf16", [70], [65], [600], "128x128", "128x128"),
    (1024, 8, "bf16", [70], [65], [1480], "256x128", "256x128"),      # 1545
]


@pytest.mark.parametrize("case", range(len(PROJECTION)))
def test_projection_tiles(case):
    d, heads, dtype, L, S, M, cached, full = PROJECTION[case]
    tiles = plan_util.projection_tiles(d, L, S, M)
    assert (tiles["cached"], tiles["full"]) == (cached, full)
    run_three_routes(synth.ModelConfig(2, d, heads, dtype), 7200 + case, L, S, M, page_tokens=64, boost=BOOST if d == 128 else None)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("d,heads,users", [(128, 2, 97), (256, 4, 97), (512, 8, 49)])
def test_every_launch_takes_the_weight_stationary_projection(dtype, d, heads, users):
    """Pre-inference into the pool, its last layer's K and V alone, ranking on the cache and full recompute: prefixes with ragged last tiles
    and filler behind them, suffix rows scattered into suffix tiles, candidates, a last unit that ends inside a 64-row block."""
    L = [(1, 63, 64, 65, 128, 129, 255, 256)[u % 8] if u < 16 else 70 + u * 41 % 187 for u in range(users)]
    S = [(0, 0, 70, 3)[u % 4] for u in range(users)]
    M = [120 + u * 13 % 17 for u in range(users)]
    assert set(plan_util.projection_tiles(d, L, S, M).values()) == {"stationary"} and (sum(S) + sum(M)) % 64
    run_three_routes(synth.ModelConfig(2, d, heads, dtype), 7250 + d, L, S, M, page_tokens=64, boost=BOOST if d < 512 else None)


#   heads at d = 128, prefix lengths, suffix lengths, candidates
CAUSAL = [
    (2, [1, 63, 64, 65, 127, 128, 129], [1, 0, 65, 64, 3, 1, 0], [3, 1, 2, 1, 1, 2, 1]),   # 32 rows a wavefront
    (2, [255, 256, 257, 700], [70, 200, 1, 129], [40, 1, 2, 3]),   # suffix rows behind a ragged last prefix tile
    (4, [1, 65, 190, 257], [100, 0, 33, 1], [1, 3, 2, 2]),         # d_head 32
    (1, [1, 65, 190, 257], [100, 0, 33, 1], [1, 3, 2, 2]),         # d_head 128
    (2, [300] * 40 + [64, 129, 1000], [5] * 40 + [130, 0, 300], [2] * 43),   # 64 rows a wavefront
]


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("case", range(len(CAUSAL)))
def test_causal_wavefronts(case, attention):
    heads, L, S, M = CAUSAL[case]
    run_three_routes(synth.ModelConfig(2, 128, heads, "bf16", attention=attention), 7300 + case, L, S, M, page_tokens=64, boost=BOOST)


@pytest.mark.parametrize("heads", [1, 2, 4])
@pytest.mark.parametrize("first", [1, 3, 7, 8, 9, 33])
def test_rows_that_end_inside_an_octet(first, heads):
    """q and the new rows' k and v lie in groups of eight rows, the last one as large as what is left: a user whose rows start inside a group, suffix
    rows in the first and the last one, all new rows less than one group, the last group of one to eight rows (heads: d_head 128, 64, 32)."""
    run_three_routes(synth.ModelConfig(2, 128, heads, "bf16"), 7500 + first, [70, 9], [0, 3], [first, 2], page_tokens=64, boost=BOOST)
    run_three_routes(synth.ModelConfig(2, 128, heads, "fp16"), 7550 + first, [70], [first % 3], [first], page_tokens=64, boost=BOOST)


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_d_head_128_items_of_eight_wavefronts(dtype, attention):
    """64 users x 4 heads of 128 make 256-row work items: rows that end in the first, in the last and just behind a wavefront's 32, behind a whole
    item, suffix rows, key tiles that only some of an item's wavefronts see (causal rows of 1 to 300 keys), pieces of one key tile."""
    L = [(1, 63, 64, 65, 130, 191, 257, 300)[u % 8] for u in range(64)]
    S = [(0, 0, 3, 0, 65)[u % 5] for u in range(64)]
    M = [(1, 31, 33, 10, 97, 5, 64)[u % 7] for u in range(63)] + [257]
    assert plan_util.check(plan_util.shim(), L, S, M, [0] * 64, heads=4, dh=128)["blocks"] == plan_util.check(plan_util.shim(), L, heads=4, dh=128)["blocks"] == 2
    run_three_routes(synth.ModelConfig(2, 512, 4, dtype, attention=attention), 7700, L, S, M, page_tokens=64)


#   attention, dtype, prefix lengths, suffix lengths, candidates; pieces, the longest one's key tiles and the groups that take it (4 heads of 64)
GROUPS = [
    ("silu", "bf16", [4500], [0], [130], 64, 9, 1),            # too short
    ("silu", "fp16", [4900], [70], [130], 64, 10, 2),          # five tiles a group, the last piece one tile short
    ("silu", "bf16", [5300, 0, 60], [3, 0, 65], [129, 5, 0], 76, 11, 2),    # six and five tiles; users of one piece: no key, one tile and suffix tiles
    ("softmax", "bf16", [7300], [0], [33], 32, 15, 1),
    ("softmax", "fp16", [7700, 64], [9, 0], [33, 4], 36, 16, 2),
]


@pytest.mark.parametrize("case", range(len(GROUPS)))
def test_pieces_by_two_groups_of_wavefronts(case):
    """Launches of no more pieces than compute units: the two groups of a workgroup take the halves of a long piece and add them in LDS; pieces of odd
    lengths, and beside them short ones, which the first group takes alone, of one key tile and of none."""
    attention, dtype, L, S, M, pieces, longest, groups = GROUPS[case]
    plan = plan_util.check(plan_util.shim(), L, S, M, [0] * len(L), heads=4, dh=64)
    tiles = (max(L) + 63) // 64 + (S[0] + 63) // 64
    assert (plan["blocks"], plan["gs"], plan["items"] * 4, -(-tiles // plan["nsplit"])) == (1, 1, pieces, longest)
    assert plan_util.shared_pieces(attention, L, S, M, heads=4) == (longest, None if groups == 1 else 10 if attention == "silu" else 16)
    run_three_routes(synth.ModelConfig(2, 256, 4, dtype, attention=attention), 7800 + case, L, S, M, boost=BOOST)


@pytest.mark.parametrize("attention", ["silu", "softmax"])
def test_a_users_scores_do_not_depend_on_the_history_beside_it(attention):
    """Users whose pieces are short beside one whose pieces two groups of wavefronts share, and beside another short one: the same bits."""
    L, M = [2000, 1900, 8192, 700], [100, 90, 90, 40]
    cfg = synth.ModelConfig(2, 512, 8, "bf16", attention=attention)
    shared = [[p[2] for p in plan_util.user_pieces([L[u] for u in us], [0] * 3, [M[u] for u in us], 1, attention)] for us in ((0, 1, 3), (0, 2, 3))]
    assert not any(shared[0]) and all(shared[1]) and len(shared[1]) == 8
    weights, batch = build_case(cfg, 7850, L, [0] * 4, M)
    h = Harness(cfg, weights, batch, page_tokens=64)
    try:
        h.prefill()

        def scores(users):
            b = h.sub_batch(users)
            b.set_handles([h.handles[u] for u in users])
            return rg.relaygr_rank_with_cache(h.ctx, h.pool, b).cpu().numpy()

        short, long = scores([0, 1, 3]), scores([0, 2, 3])
        assert np.array_equal(short[:100], long[:100]) and np.array_equal(short[190:], long[190:])
    finally:
        h.close()


#   prefix lengths, suffix lengths, candidates; rows a workgroup
WIDE_TAIL = [
    ([600], [3], [4], 8),                              # 7 rows of five sums: a workgroup not full
    ([2100, 70], [0, 5], [520, 0], 8),                 # unequal numbers of sums
    ([70], [0], [1024], 8),
    ([600], [1], [1024], 16),                          # 1025: a workgroup of one row
    ([65] * 17, [0] * 17, [250] * 17, 32),             # 4250
    ([65] * 16 + [1500], [0] * 17, [241] * 17, 32),    # 4097, and 9729 in full recompute: a last workgroup of one row; one and three sums
]


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("case", range(len(WIDE_TAIL)))
def test_layer_tail_edges_at_width_1024(case, attention):
    L, S, M, rows = WIDE_TAIL[case]
    assert plan_util.tail_rows(1024, sum(S) + sum(M)) == rows
    run_three_routes(synth.ModelConfig(2, 1024, 8, "fp16" if case % 2 else "bf16", attention=attention), 7900 + case, L, S, M, page_tokens=64)
