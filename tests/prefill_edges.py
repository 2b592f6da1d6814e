"""Cases of the prefill's tile edges: inputs, and fp64 outputs over rounded operands."""
import numpy as np

import workload as W
from tests.rounded_reference import attend, bf16, rotate

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


def inputs(case):
    """Raw keys, values and queries of the contexts and of the questions, packed."""
    _, hq, hkv, d, lc, ql, grow = case
    rng = np.random.default_rng([930, CASES.index(case)])
    qn = [n for p in ql for n in p]
    nc, ns = sum(lc), sum(qn)

    def draw(n, h):
        return W.round_to_bf16(rng.standard_normal((n, h, d)).astype(np.float32) * np.float32(0.5))

    pos_c, pos_s = positions(case)
    ck, cv, cq, sk, sv, sq = draw(nc, hkv), draw(nc, hkv), draw(nc, hq), draw(ns, hkv), draw(ns, hkv), draw(ns, hq)
    ck = W.round_to_bf16(ck * (1 + grow * pos_c)[:, None, None].astype(np.float32))
    sk = W.round_to_bf16(sk * (1 + grow * pos_s)[:, None, None].astype(np.float32))
    return ck, cv, cq, sk, sv, sq


def positions(case):
    lc, ql = case[4], case[5]
    return (np.concatenate([np.arange(n) for n in lc]),
            np.concatenate([lc[b] + np.arange(n) for b, p in enumerate(ql) for n in p]))


def reference(case, kc, ks, hide=None):
    """Outputs and their rounding bounds of context and question rows over the
    rotated, rounded keys kc, ks [hkv][tokens][d].  hide: a context token that
    no row sees (but for rows that see nothing else)."""
    _, hq, hkv, d, lc, ql, _ = case
    _, cv, cq, _, sv, sq = (x.astype(np.float64) for x in inputs(case))
    pos_c, pos_s = positions(case)
    c = np.log2(np.e) / np.sqrt(d)                 # the kernel rounds the query with the softmax scale in it
    qc, qs = bf16(rotate(cq, pos_c) * c), bf16(rotate(sq, pos_s) * c)
    out = [np.empty(qc.shape), np.empty(qs.shape)]
    bound = [np.empty(qc.shape), np.empty(qs.shape)]
    ln2 = np.log(2.0)
    c0 = s0 = 0
    for n, questions in zip(lc, ql):
        seen = np.ones(n, bool)
        if hide is not None and hide < n and n > 1:
            seen[hide] = False
        for h in range(hq):
            k, v = kc[h // (hq // hkv), c0:c0 + n], cv[c0:c0 + n, h // (hq // hkv)]
            if n:
                see = np.tri(n, dtype=bool) & seen
                see[~see.any(1)] = np.tri(n, dtype=bool)[~see.any(1)]
                out[0][c0:c0 + n, h], bound[0][c0:c0 + n, h], _ = attend(qc[c0:c0 + n, h] @ k.T * ln2, v, see)
            at = s0
            for m in questions:
                kk = np.concatenate([k, ks[h // (hq // hkv), at:at + m]])
                vv = np.concatenate([v, sv[at:at + m, h // (hq // hkv)]])
                see = np.concatenate([np.broadcast_to(seen, (m, n)), np.tri(m, dtype=bool)], 1)
                out[1][at:at + m, h], bound[1][at:at + m, h], _ = attend(qs[at:at + m, h] @ kk.T * ln2, vv, see)
                at += m
        c0 += n
        s0 += sum(questions)
    return (out[0], bound[0]), (out[1], bound[1])
