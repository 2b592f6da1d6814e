"""GPU: the bf16 prefill units at the edges of their tiles: contexts and
questions of one key, just under, at and just over a 32-key half, a 64-key
tile and the 128 keys of a step of the two-group unit; keys that keep growing
(the softmax offset is raised again and again); cache memory past every
region holding NaN.  Against the fp64 oracle.

Tolerance: the rotated operands and the weights are rounded to bf16 (relative
2^-9 each), so a score is off by at most ds = 2 * 2^-9 * scale * sum |q||k|,
a weight by a factor within exp(+-ds)(1 +- 2^-9), numerator and denominator
alike: |out - ref| <= max|v| * (2 ds + 2^-8), computed from the inputs."""
import numpy as np
import pytest
import torch

import workload as W
from oracle import prefill as P
from paper_2609_05707_amd.session import DecodeBatch
from tests.gpu_harness import log, max_err

pytestmark = pytest.mark.gpu

CASES = [
    # (name, hq, hkv, D, context lengths, question lengths per prompt, growth of the keys per token)
    ("one-key", 4, 1, 128, [1, 0, 31], [[1], [1, 32], [33]], 0.0),
    ("tile-edges", 8, 2, 128, [32, 33, 63, 64, 65], [[31], [64], [65, 1], [], [5, 0, 7]], 0.0),
    ("step-edges", 8, 1, 128, [127, 128, 129, 193, 260], [[3], [40, 40], [64], [1], [96, 33]], 0.0),
    ("growing", 4, 1, 128, [300, 97], [[70, 5], [33]], 0.05),
    ("g3", 6, 2, 128, [86, 170], [[85, 1], [43]], 0.0),
    ("d64", 4, 1, 64, [1, 64, 65, 129, 200], [[1], [32, 33], [], [64], [127]], 0.0),
    ("d64-growing-g16", 16, 1, 64, [150, 33], [[9, 17], [40]], 0.05),
]


@pytest.mark.parametrize("standard", [False, True])
@pytest.mark.parametrize("rows", [0, 128, 256])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_prefill_edges(case, rows, standard):
    name, hq, hkv, d, lc, ql, grow = case
    if d == 64 and rows == 256:
        pytest.skip("256-row units are asked for at head_dim 128 only")
    log(f"case: prefill edges {name} tile_rows={rows} standard={standard}")
    rng = np.random.default_rng([930, CASES.index(case)])
    qn = [n for p in ql for n in p]
    q_count = [len(p) for p in ql]
    nc, ns = sum(lc), sum(qn)

    def draw(n, h):
        return W.round_to_bf16(rng.standard_normal((n, h, d)).astype(np.float32) * np.float32(0.5))

    pos_c = np.concatenate([np.arange(n) for n in lc])
    pos_s = np.concatenate([lc[b] + np.arange(n) for b, p in enumerate(ql) for n in p])
    ck, cv, cq, sk, sv, sq = draw(nc, hkv), draw(nc, hkv), draw(nc, hq), draw(ns, hkv), draw(ns, hkv), draw(ns, hq)
    ck = W.round_to_bf16(ck * (1 + grow * pos_c)[:, None, None].astype(np.float32))
    sk = W.round_to_bf16(sk * (1 + grow * pos_s)[:, None, None].astype(np.float32))
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
