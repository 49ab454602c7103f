"""Decode attention where its passes change form: record counts around the
merge's rounds.  Outputs are held to the per-element bound of
tests/attn_tolerance.py against the float64 oracle."""

import pytest

from tests.gpu_helpers import BM, LM
from tests.test_attention_gpu import run_case, say
from workloads import Geometry

pytestmark = pytest.mark.gpu


# one wave merges up to 8 records at head_dim 128 (16 at 64), a workgroup 32
# (64) a round
@pytest.mark.parametrize("dh,records", [(d, n) for d, ns in ((128, (1, 2, 7, 8, 9, 31, 32, 33, 65)),
                                                           (64, (1, 3, 15, 16, 17, 63, 64, 65)))
                                        for n in ns])
def test_merge_at_its_record_counts(dh, records):
    geom = Geometry("merge", 1, 2, dh, 16, "bfloat16")
    split = 16
    lens = [split * records, split * records - 5, max(1, split * records // 3)]
    say(f"merge: head_dim {dh}, {records} records")
    # 3 query heads' worth of a wave's four, and whole fours
    for hq in (2, 8):
        run_case(geom, (LM, BM)[records % 2], sum(-(-t // 16) for t in lens) + 3, lens, hq,
                 900 + records, split, host_lens=bool(hq == 8))
