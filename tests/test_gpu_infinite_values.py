"""GPU: infinities in valid values at the end of a context (bf16).  The keys and
values a tile holds past its last token, and the tiles and halves that only
repeat another, have weight 0: an infinity among their values would turn the
output into NaN.  Contexts whose last 8-token block is whole and whose halves
and tiles end everywhere; the output is infinite in the dims where the values
are, with their sign, and unchanged elsewhere.

Tolerance 2e-2 in the finite dims: operands and weights are rounded to 8 bits."""
import numpy as np
import pytest
import torch

import workload as W
from oracle import prefill as P
from paper_2609_05707_amd.session import DecodeBatch
from tests.gpu_harness import load_layer, log, make_batch, oracle_steps, run_gpu

pytestmark = pytest.mark.gpu

CTX = [8, 24, 32, 40, 64, 72, 88, 96, 104, 120, 128, 136, 168, 192, 200, 256]


def check(got, ref):
    inf = np.isinf(ref)
    assert inf.any() and (got[inf] == ref[inf]).all()
    assert np.isfinite(got[~inf]).all() and np.abs(got[~inf] - ref[~inf]).max() <= 2e-2


def with_infinities(kv, st):
    """+inf and -inf in two dims of every context's last token."""
    v = kv.ctx_v.copy()
    for b in range(len(st.ctx_len)):
        v[st.ctx_start[b + 1] - 1, :, 3] = np.inf
        v[st.ctx_start[b + 1] - 1, :, 40] = -np.inf
    return v


@pytest.mark.parametrize("rows,d", [(64, 128), (128, 128), (256, 128), (128, 64)])
@pytest.mark.parametrize("lc", CTX)
def test_decode(lc, rows, d):
    log(f"case: infinite values decode lc={lc} rows={rows} D={d}")
    wl = W.custom_workload(wid=810, dtype="bf16", num_prompts=2, hq=8, hkv=2, head_dim=d, ctx_len=(lc, lc),
                           questions=(33, 33), seg_len=(1, 9), steps=1, value_std=0.5)
    st = W.make_structure(wl)
    kv = W.layer_kv(st)
    kv.ctx_v[...] = with_infinities(kv, st)
    db = make_batch(st, tile_rows=rows)
    load_layer(db, st, 0, kv)
    gpu = run_gpu(st, [0], [0], db=db, kv=kv, fused=True)
    with np.errstate(invalid="ignore"):
        out, _ = oracle_steps(st, kv, [0], [0])[0]
    check(gpu.out[0], out)
    assert gpu.err == 0


@pytest.mark.parametrize("rows,d", [(128, 128), (256, 128), (128, 64), (0, 64)])
@pytest.mark.parametrize("lc", CTX)
def test_prefill_questions(lc, rows, d):
    log(f"case: infinite values prefill lc={lc} rows={rows} D={d}")
    rng = np.random.default_rng([811, lc])
    ql = 8 * [11]

    def draw(n, h):
        return W.round_to_bf16(rng.standard_normal((n, h, d)).astype(np.float32) * np.float32(0.5))

    ck, cv, cq, sk, sv, sq = draw(lc, 1), draw(lc, 1), draw(lc, 4), draw(88, 1), draw(88, 1), draw(88, 4)
    cv[lc - 1, :, 3], cv[lc - 1, :, 40] = np.inf, -np.inf
    db = DecodeBatch([lc], [8], 4, 1, d, "bf16", 16, tile_rows=rows)
    db.load_context(0, ck, cv)
    db.load_segments(0, sk, sv, ql)
    q_ctx, q_seg = db.pack_prefill_queries(cq, sq, ql)
    oc, os_ = db.prefill_outputs()
    db.prefill(0, q_ctx, q_seg, oc, os_, 88)
    torch.cuda.synchronize()
    got = np.concatenate([os_[i, :n].cpu().numpy() for i, n in enumerate(ql)])
    with np.errstate(invalid="ignore"):
        _, ref = P.prefill_standard(ck, cv, cq, np.array([0, lc]), np.array([0, 8]), sk, sv, sq,
                                    np.concatenate([[0], np.cumsum(ql)]), 10000.0)
    check(got, ref)
    assert db.err_flag() == 0
