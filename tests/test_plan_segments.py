"""CPU: every plan leaves each segment task's waves room for at least one
partial state in the unit's LDS; without one the kernel folds none of the
task's cached keys."""

import pytest

from paper_2609_05707_amd import _lib as L
from tests import plan_probe
from tests.test_abi import FAKE, valid_batch


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return plan_probe.build(str(tmp_path_factory.mktemp("plan")))


@pytest.mark.parametrize("g", range(1, 17))
def test_every_segment_task_has_a_state(plans, g):
    most = 0
    for dtype in (L.IPPD_DTYPE_F32, L.IPPD_DTYPE_BF16):
        for d in (64, 128):
            for hk in (1, 2, 8):
                for B in (1, 3, 8, 40, 200):
                    for q in (1, 6, 17, 64, 300, 1024):
                        for ctx in (8, 304, 2048, 16384):
                            for rows in (0, 16, 128):
                                for instr, chunk in ((0, 0), (1, 0), (0, 256)):
                                    bt = valid_batch(dtype=dtype, head_dim=d, num_prompts=B, num_questions=min(q * B, 60000),
                                                     num_q_heads=hk * g, num_kv_heads=hk, max_ctx_len=ctx, max_questions=q,
                                                     ctx_pool_tokens=B * ctx + 1000, seg_capacity=64, tile_rows=rows,
                                                     chunk_tokens=chunk)
                                    if instr:
                                        bt.num_instr, bt.max_instr_len, bt.max_instr_questions = 1, 1000, q * B
                                        bt.instr_start = bt.instr_off = bt.instr_len = FAKE
                                    p = plans.step(bt)
                                    e = 2 if dtype == L.IPPD_DTYPE_BF16 else 4
                                    lds = plans.lib.segment_lds(e, d, p["waves"], p["deep"])
                                    assert lds // (g * (d + 4) * 4) // p["seg_tpu"] >= 1, (dtype, d, hk, B, q, ctx, rows, p)
                                    assert p["seg_tpu"] <= p["waves"]
                                    most = max(most, p["seg_tpu"])
    assert most >= 4
