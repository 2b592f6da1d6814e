"""GPU: the bf16 prefill units at the edges of their tiles: contexts and
questions of one key, just under, at and just over a 32-key half, a 64-key
tile and the 128 keys of a step of the two-group unit; keys that keep growing
(the softmax offset is raised again and again); cache memory past every
region holding NaN.  Against the fp64 oracle.

Tolerances.  Against the oracle, which rounds nothing: the rotated operands and
the weights are rounded to bf16 (relative 2^-9 each), so a score is off by at
most ds = 2 * 2^-9 * scale * sum |q||k|, a weight by a factor within
exp(+-ds)(1 +- 2^-9), numerator and denominator alike: |out - ref| <= max|v| *
(2 ds + 2^-8), computed from the inputs.  That bound is wide, so the same is
compared with fp64 over the rounded operands, where only the weights' rounding
is left (rounded_reference.py): the queries are rounded there from fp64 and in
the kernel from fp32, which a few in 2^15 elements straddle, so all but one in
a thousand outputs have to lie within that bound.  test_prefill_edges_power.py
shows on the CPU that hiding one key at the edge of a tile is seen."""
import numpy as np
import pytest
import torch

from oracle import prefill as P
from paper_2609_05707_amd.session import DecodeBatch
from tests.gpu_harness import log, max_err
from tests.prefill_edges import CASES, inputs, reference
from tests.rounded_reference import beyond

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("standard", [False, True])
@pytest.mark.parametrize("rows", [0, 128, 256])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_prefill_edges(case, rows, standard):
    name, hq, hkv, d, lc, ql, grow = case
    if d == 64 and rows == 256:
        pytest.skip("256-row units are asked for at head_dim 128 only")
    log(f"case: prefill edges {name} tile_rows={rows} standard={standard}")
    qn = [n for p in ql for n in p]
    q_count = [len(p) for p in ql]
    ck, cv, cq, sk, sv, sq = inputs(case)
    db = DecodeBatch(lc, q_count, hq, hkv, d, "bf16", max(qn), tile_rows=rows)
    for x in (db.ctx_k[0], db.ctx_vt[0], db.seg_k[0], db.seg_vt[0]):
        x.fill_(float("nan"))
    db.load_context(0, ck, cv)
    db.load_segments(0, sk, sv, qn)
    q_ctx, q_seg = db.pack_prefill_queries(cq, sq, qn)
    oc, os_ = db.prefill_outputs(fill=-777.0)
    bound = max(sum(p) for p in ql)
    db.prefill(0, q_ctx, q_seg, oc, os_, bound, standard=standard)
    torch.cuda.synchronize()
    oc, os_ = oc.cpu().numpy(), os_.cpu().numpy()
    g_ctx = np.concatenate([oc[db.ctx_off[b]: db.ctx_off[b] + lc[b]] for b in range(len(lc))])
    g_seg = np.concatenate([os_[i, :n] for i, n in enumerate(qn)])
    starts = [np.concatenate([[0], np.cumsum(x)]) for x in (lc, q_count, qn)]
    r_ctx, r_seg = P.prefill_standard(ck, cv, cq, starts[0], starts[1], sk, sv, sq, starts[2], 10000.0)
    if standard:
        for b in np.flatnonzero(np.array(q_count) == 0):
            rows_b = slice(starts[0][b], starts[0][b + 1])
            assert (g_ctx[rows_b] == -777.0).all()
            r_ctx[rows_b] = np.nan
    # Cauchy-Schwarz over each head bounds sum |q||k| (rotation keeps the norms)
    qmax = max(np.sqrt((np.square(x).sum(-1))).max() for x in (cq, sq))
    kmax = max(np.sqrt((np.square(x).sum(-1))).max() for x in (ck, sk))
    ds = 2 * 2.0 ** -9 * qmax * kmax / np.sqrt(d)
    tol = max(np.abs(cv).max(), np.abs(sv).max()) * (2 * ds + 2.0 ** -8)
    e_ctx, e_seg = max_err(g_ctx, r_ctx), max_err(g_seg, r_seg)
    log(f"  max err ctx {e_ctx:.3e} questions {e_seg:.3e}, bound {tol:.3e}")
    assert np.isfinite(g_ctx).all() and np.isfinite(g_seg).all()
    assert e_ctx <= tol and e_seg <= tol
    assert db.err_flag() == 0
    # over the rounded keys of the cache
    kc = db.ctx_k[0].float().cpu().numpy()
    kc = np.concatenate([kc[:, db.ctx_off[b]: db.ctx_off[b] + lc[b]] for b in range(len(lc))], 1)
    ks = db.seg_k[0].float().cpu().numpy()
    ks = np.concatenate([ks[i, :, :n] for i, n in enumerate(qn)], 1)
    (o_ctx, b_ctx), (o_seg, b_seg) = reference(case, kc, ks)
    if standard:
        served = np.concatenate([np.full(n, c > 0) for n, c in zip(lc, q_count)])
        g_ctx, o_ctx, b_ctx = g_ctx[served], o_ctx[served], b_ctx[served]
    for what, g, o, e in (("ctx", g_ctx, o_ctx, b_ctx), ("questions", g_seg, o_seg, b_seg)):
        share, most = beyond(g, o, e)
        log(f"  {what}: {share:.2e} of the outputs beyond the weights' rounding, largest {most:.2f} times it")
        assert share <= 1e-3
