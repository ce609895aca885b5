"""GPU parity where a launch changes its kernel or its shape: row counts at both sides of the edges of the layer tail's workgroups
(8, 16 and 32 rows, the partly filled last one) with few and with many partial sums a row.  Every case ranks on the cached prefix
and by full recompute, against the CPU oracle; at d = 128 with the boosted weights, which let attention reach the scores there."""
import pytest

import synth
from gpu_util import BOOST
from test_gpu_parity import run_three_routes

pytestmark = pytest.mark.gpu

#   d, heads, dtype, prefix lengths, suffix lengths, candidates
TAIL = [
    (256, 4, "bf16", [600], [0], [1]),            # one row of eight pieces
    (512, 8, "bf16", [600], [3], [4]),            # 7 rows: a workgroup of 8 not full
    (512, 8, "fp16", [520], [0], [17]),           # 8 + 8 + 1
    (256, 4, "bf16", [600, 70], [0, 5], [1019, 0]),   # 1024 rows: the last launch of 8-row workgroups
    (256, 4, "fp16", [600, 70], [0, 5], [1020, 0]),   # 1025: the first one of 16-row workgroups, unequal pieces
    (512, 8, "bf16", [130], [1], [1033]),         # 16-row workgroups, few pieces
    (128, 2, "bf16", [100], [0], [33]),           # the d = 128 kernel: 32 + 1
    (1024, 8, "bf16", [70], [0], [33]),           # the d = 1024 kernel: 32 + 1
]


@pytest.mark.parametrize("attention", ["silu", "softmax"])
@pytest.mark.parametrize("case", range(len(TAIL)))
def test_layer_tail_edges(case, attention):
    d, heads, dtype, L, S, M = TAIL[case]
    run_three_routes(synth.ModelConfig(2, d, heads, dtype, attention=attention), 7100 + case, L, S, M, page_tokens=64, boost=BOOST if d == 128 else None)
