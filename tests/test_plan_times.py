"""CPU: the plans that the library chooses, against measured times of every unit
and chunk (profiles/decode_plan_grid.jsonl: 36 bf16 batches of 1 to 32 prompts,
us a decode step; by_rows and by_thresholds are the times of two earlier rules
for the same batches).  The estimate behind the choice is good to some 10%,
and a ragged batch's lengths are not known to it; the bounds leave that room
and no more: the earlier rules are up to 1.4 times the best measured."""
import json
import math
import os

import numpy as np
import pytest

from paper_2609_05707_amd import _lib as L
from tests import plan_probe
from tests.test_abi import FAKE, valid_batch

GRID = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles", "decode_plan_grid.jsonl")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return plan_probe.build(str(tmp_path_factory.mktemp("plan")))


def pieces(ctx, chunk):
    return tuple(-(-n // chunk) for n in ctx)


def test_chosen_plans_are_near_the_best_measured(plans):
    worst, ratio, earlier, found = 0.0, [], [], 0
    for line in open(GRID):
        s = json.loads(line)
        hq, hk, d = s["heads"]
        q, ctx, cpi = s["q"], s["ctx"], s["cpi"]
        bt = valid_batch(dtype=L.IPPD_DTYPE_BF16, head_dim=d, num_prompts=len(ctx), num_questions=sum(q),
                         num_q_heads=hq, num_kv_heads=hk, max_ctx_len=max(ctx), max_questions=max(q),
                         ctx_pool_tokens=s["pool"], seg_capacity=(s["seg_max"] + 15) // 8 * 8)
        if cpi:
            bt.num_instr, bt.max_instr_len = -(-len(ctx) // cpi), s["instr"]
            bt.max_instr_questions = max(int(np.sum(q[i:i + cpi])) for i in range(0, len(ctx), cpi))
            bt.instr_start = bt.instr_off = bt.instr_len = FAKE
        p = plans.step(bt)
        rows = 16 * p["waves"] * p["rb"]
        # the same pieces of every context: the same units
        t = [us for k, us in s["us"].items() if int(k.split("/")[0]) == rows and
             pieces(ctx, int(k.split("/")[1])) == pieces(ctx, p["chunk"])]
        if not t:
            continue                                 # a chunk between the measured ones
        found += 1
        r = t[0] / min(s["us"].values())
        assert r <= 1.15, (s["heads"], ctx, q, rows, p["chunk"], t[0], min(s["us"].values()))
        ratio.append(math.log(r))
        earlier.append(math.log(t[0] / min(s["by_rows"], s["by_thresholds"])))
        worst = max(worst, r)
    assert found >= 30
    assert np.exp(np.mean(ratio)) <= 1.03 and np.exp(np.mean(earlier)) <= 0.98, (worst, np.mean(ratio), np.mean(earlier))
