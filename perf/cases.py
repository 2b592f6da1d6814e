"""Performance cases of the library: what a serving program does with one
layer's attention, from filling the cache to the decode steps.

A case is a dict of plain values:
  kind      "decode": a stretch of the decode loop (fused steps, every layer
            in turn); "attend": the same stretch as separate append and
            attention calls; "prefill": the attention of every header token;
            "fill": rotating raw keys/values into the cache
  dtype, hq, hkv, d         element type and head shape
  prompts, ctx_lo, ctx_hi   prompts and their context lengths (uniform)
  q_lo, q_hi                questions per prompt
  seg_lo, seg_hi            tokens cached per question before the pass
  cpi, instr                contexts behind one instruction and its length
                            (0: one-level batch)
  steps, layers             decode steps and independent layer caches
  stopped                   share of questions finished before the first step
  graph                     decode: the stretch replayed from a captured graph
  lens                      seed of the lengths

Layer buffers are separate, as in a model: a layer's cache is not in the
data caches because the layer before it ran.
"""
import math

import numpy as np
import torch

from paper_2609_05707_amd import _lib as L
from paper_2609_05707_amd.driver import DecodeLoop
from paper_2609_05707_amd.session import DecodeBatch

ROPE_BASE = 10000.0
DEV = "cuda"


def _case(name, kind, dtype, heads, prompts, ctx, q, seg, cpi=0, instr=0, steps=1, layers=1, stopped=0.0,
          graph=False, lens=1):
    c = dict(kind=kind, dtype=dtype, hq=heads[0], hkv=heads[1], d=heads[2], prompts=prompts, ctx_lo=ctx[0],
             ctx_hi=ctx[1], q_lo=q[0], q_hi=q[1], seg_lo=seg[0], seg_hi=seg[1], cpi=cpi, instr=instr, steps=steps,
             layers=layers, stopped=stopped, graph=graph, lens=lens)
    if name:
        c["name"] = name
    return c


def listed():
    llama = (32, 8, 128)
    return [
        # The smallest step: one short fp32 prompt, 4 questions; launches and latency are all there is.
        _case("decode-tiny-f32", "decode", "f32", (4, 2, 64), 1, (256, 256), (4, 4), (24, 24), steps=16, graph=True),
        # One user's document with a handful of questions, Llama-3-8B head shape; 8 layers of it.
        _case("decode-lc4096-n16", "decode", "bf16", llama, 1, (4096, 4096), (16, 16), (32, 96), steps=4, layers=8,
              graph=True),
        # A serving batch of documents of all lengths with 4 to 32 questions each.
        _case("decode-ragged-b32", "decode", "bf16", llama, 32, (1024, 8192), (4, 32), (16, 96), steps=2, layers=2,
              lens=3),
        # A book: one very long context with many questions.
        _case("decode-lc32768-n64", "decode", "bf16", llama, 1, (32768, 32768), (64, 64), (16, 128), steps=2,
              layers=3),
        # A uniform batch in the middle of its answers: four in ten questions have stopped.
        _case("decode-b8-lc8192-n32", "decode", "bf16", llama, 8, (8192, 8192), (32, 32), (48, 112), steps=3,
              layers=3, stopped=0.4),
        # Contexts behind shared instructions (few-shot preambles), read once for all contexts behind them.
        _case("decode-two-level", "decode", "bf16", llama, 12, (1024, 1024), (8, 8), (16, 48), cpi=4, instr=2048,
              steps=4, layers=4, graph=True),
        # A program that keeps rotation and attention apart, 64-wide heads in groups of three, odd lengths.
        _case("attend-d64-g3", "attend", "bf16", (24, 8, 64), 5, (301, 3001), (1, 9), (5, 77), steps=2, layers=4,
              lens=5),
        # The header of one document with 16 questions of 32 tokens.
        _case("prefill-lc4096-n16", "prefill", "bf16", llama, 1, (4096, 4096), (16, 16), (32, 32)),
        # The headers of a ragged batch: the largest call.
        _case("prefill-ragged-b8", "prefill", "bf16", llama, 8, (1024, 8192), (4, 32), (8, 32), lens=2),
        # A short document of odd length: few blocks for the chip.
        _case("prefill-lc1021", "prefill", "bf16", llama, 1, (1021, 1021), (7, 7), (9, 31), lens=4),
        # Headers behind shared instructions.
        _case("prefill-two-level", "prefill", "bf16", llama, 8, (1024, 1024), (8, 8), (16, 16), cpi=4, instr=2048),
        # Projected keys and values of a ragged batch written into the cache: every new prompt pays this once.
        _case("fill-ragged-b8", "fill", "bf16", llama, 8, (1024, 8192), (4, 32), (8, 32), lens=2),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["decode", "decode", "decode", "attend", "prefill", "prefill", "fill"])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    heads = rng.choice([(32, 8, 128), (32, 8, 128), (24, 8, 64), (16, 16, 64), (8, 2, 128), (32, 2, 128)])
    ctx_hi = spread(250, 32768) if kind == "decode" and dtype == "bf16" else spread(250, 8192)
    if kind == "prefill" and dtype == "f32":
        ctx_hi = min(ctx_hi, 3000)
    ctx_lo = max(1, int(ctx_hi * rng.choice([0.15, 0.6, 1.0])))
    # tokens over all prompts within what the largest listed cases hold
    most = max(1, min(32 if kind != "prefill" else 8, (65536 if kind != "prefill" else 24576) // ctx_hi))
    if dtype == "f32" and kind == "prefill":
        most = max(1, most // 4)
    prompts = spread(1, most) if most > 1 else 1
    q_hi = spread(1, 64 if prompts < 4 else 32)
    q_lo = max(1, int(q_hi * rng.choice([0.2, 1.0])))
    seg_hi = spread(4, 128) if kind != "prefill" else spread(4, 48)
    seg_lo = max(1, int(seg_hi * rng.choice([0.25, 1.0])))
    two = prompts > 1 and rng.random() < 0.25
    decode = kind in ("decode", "attend")
    return _case("", kind, dtype, heads, prompts, (ctx_lo, ctx_hi), (q_lo, q_hi), (seg_lo, seg_hi),
                 cpi=rng.randint(2, 4) if two else 0, instr=spread(100, 2048) if two else 0,
                 steps=rng.randint(2, 4) if decode else 1, layers=rng.randint(1, 3) if decode else 1,
                 stopped=rng.choice([0.0, 0.0, 0.3, 0.7]) if decode else 0.0,
                 graph=kind == "decode" and rng.random() < 0.5, lens=rng.randint(1, 10 ** 6))


# ---------------------------------------------------------------- structure
class _Shape:
    """Lengths, question ranges and per-step active masks of a case."""

    def __init__(self, c):
        r = np.random.default_rng([77, c["lens"]])
        B = c["prompts"]
        self.B = B
        self.ctx = r.integers(c["ctx_lo"], c["ctx_hi"], size=B, endpoint=True)
        self.nq = r.integers(c["q_lo"], c["q_hi"], size=B, endpoint=True)
        self.qs = np.concatenate([[0], np.cumsum(self.nq)])
        self.nt = int(self.qs[-1])
        self.seg = r.integers(c["seg_lo"], c["seg_hi"], size=self.nt, endpoint=True)
        self.prompt = np.repeat(np.arange(B), self.nq)
        self.istart = np.array(list(range(0, B, c["cpi"])) + [B]) if c["cpi"] else None
        self.S = len(self.istart) - 1 if c["cpi"] else 0
        self.ilen = np.full(self.S, c["instr"])
        self.instr_of = np.searchsorted(self.istart, np.arange(B), side="right") - 1 if self.S else None
        # answers end one after another: each step a few more questions than the share at the start
        rank = r.permutation(self.nt)
        self.active = [rank >= int((c["stopped"] + 0.02 * t) * self.nt) if c["stopped"] else
                       np.ones(self.nt, dtype=bool) for t in range(c["steps"])]
        self.fed = np.sum(self.active, axis=0) if c["kind"] in ("decode", "attend") else np.zeros(self.nt, dtype=int)

    def lp(self, b):
        return int(self.ilen[self.instr_of[b]]) if self.S else 0


def _rand(gen, dtype, *shape):
    # projections of normalised activations: centred, about half a unit wide
    return (torch.randn(*shape, generator=gen, device=DEV) * 0.5).to(torch.float32 if dtype == "f32" else torch.bfloat16)


def _layer_inputs(c, s, gen):
    """Raw keys and values of one layer, packed: instructions, contexts, segments."""
    hk, d, dt = c["hkv"], c["d"], c["dtype"]
    return [(_rand(gen, dt, int(n), hk, d), _rand(gen, dt, int(n), hk, d))
            for n in (s.ilen.sum() if s.S else 0, s.ctx.sum(), s.seg.sum())]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _step_inputs(c, s, gen):
    return [(_rand(gen, c["dtype"], s.nt, c["hq"], c["d"]), _rand(gen, c["dtype"], s.nt, c["hkv"], c["d"]),
             _rand(gen, c["dtype"], s.nt, c["hkv"], c["d"])) for _ in range(c["steps"])]


def _prefill_inputs(c, s, gen):
    hq, d, dt = c["hq"], c["d"], c["dtype"]
    return [_rand(gen, dt, int(n), hq, d) for n in (s.ilen.sum() if s.S else 0, s.ctx.sum(), s.seg.sum())]


def _batch(c, s):
    db = DecodeBatch(s.ctx.tolist(), s.nq.tolist(), c["hq"], c["hkv"], c["d"], c["dtype"],
                     int(s.seg.max()) + c["steps"], rope_base=ROPE_BASE, layers=c["layers"], device=DEV,
                     instr_len=s.ilen.tolist() if s.S else None, instr_prompt_start=s.istart.tolist() if s.S else None)
    for bufs in (db.ctx_k, db.ctx_vt, db.seg_k, db.seg_vt):
        for x in bufs:
            x.zero_()
    db.out.zero_()
    db.lse.zero_()
    return db


def _pool_rows(db, s):
    """Pool row of each packed instruction and context token."""
    ins = [np.arange(o, o + n) for o, n in zip(db.instr_off, s.ilen)] if s.S else []
    return (torch.from_numpy(np.concatenate(ins)).to(DEV) if ins else None,
            torch.from_numpy(np.concatenate([np.arange(o, o + n) for o, n in zip(db.ctx_off, s.ctx)])).to(DEV))


def _seg_rows(s, cap):
    """Row question * cap + slot of each packed segment token."""
    return torch.from_numpy(np.concatenate([i * cap + np.arange(n) for i, n in enumerate(s.seg)])).to(DEV)


# ------------------------------------------------------------------ the pass
def prepare(case, seed):
    c, s = case, _Shape(case)
    gen = _gen(seed)
    db = _batch(c, s)
    st = dict(case=c, db=db)
    if c["kind"] == "fill":
        # raw projections in pool and segment rows, as the projection wrote them
        (ik, iv), (ck, cv), (sk, sv) = _layer_inputs(c, s, gen)
        ri, rc = _pool_rows(db, s)
        st["ctx"] = [torch.zeros(db.pool, c["hkv"], c["d"], dtype=ck.dtype, device=DEV) for _ in range(2)]
        st["seg"] = [torch.zeros(s.nt * db.seg_cap, c["hkv"], c["d"], dtype=ck.dtype, device=DEV) for _ in range(2)]
        for to, a, b in zip(st["ctx"], (ik, iv), (ck, cv)):
            if s.S:
                to[ri] = a
            to[rc] = b
        rs = _seg_rows(s, db.seg_cap)
        for to, a in zip(st["seg"], (sk, sv)):
            to[rs] = a
        st["init"] = torch.from_numpy(s.seg.astype(np.int32)).to(DEV)
        return st
    for layer in range(c["layers"]):
        (ik, iv), (ck, cv), (sk, sv) = _layer_inputs(c, s, gen)
        if s.S:
            db.load_instructions(layer, ik, iv)
        db.load_context(layer, ck, cv)
        db.load_segments(layer, sk, sv, s.seg)
    if c["kind"] == "prefill":
        iq, cq, sq = _prefill_inputs(c, s, gen)
        st["q"] = db.pack_prefill_queries(cq, sq, s.seg, instr_q=iq if s.S else None)
        st["out"] = db.prefill_outputs()
        st["most"] = int(max(s.seg[s.qs[b]:s.qs[b + 1]].sum() for b in range(s.B)))
        return st
    steps = _step_inputs(c, s, gen)
    act = [torch.from_numpy(a.astype(np.uint8)).to(DEV) for a in s.active]
    st["loop"] = DecodeLoop(db, [x[0] for x in steps], [x[1] for x in steps], [x[2] for x in steps], act)
    if c["graph"]:
        st["loop"].capture()
    return st


def run(state):
    c, db = state["case"], state["db"]
    if c["kind"] == "fill":
        stream = db.stream()
        ck, cv = state["ctx"]
        sk, sv = state["seg"]
        if db.S:
            L.ippd_load_instructions(db.batches[0], ck.data_ptr(), cv.data_ptr(), db.caches[0], stream)
        L.ippd_load_context(db.batches[0], ck.data_ptr(), cv.data_ptr(), db.caches[0], stream)
        L.ippd_load_segments(db.batches[0], sk.data_ptr(), sv.data_ptr(), state["init"].data_ptr(), db.caches[0], stream)
        return dict(ctx_k=db.ctx_k[0], ctx_vt=db.ctx_vt[0], seg_k=db.seg_k[0], seg_vt=db.seg_vt[0],
                    seg_len=db.seg_len[0], err=db.d_err)
    if c["kind"] == "prefill":
        oc, os_ = state["out"]
        db.prefill(0, state["q"][0], state["q"][1], oc, os_, state["most"])
        return dict(ctx=oc, seg=os_, err=db.d_err)
    loop = state["loop"]
    loop.reset()                                     # back to the state before step 0: a pass can be repeated
    if c["kind"] == "attend":
        for t in range(loop.steps):
            db.d_active.copy_(loop.active[t])
            for layer in range(db.layers):
                db.append(layer, loop.q[t], loop.k[t], loop.v[t])
                db.decode(layer)
    elif c["graph"]:
        loop.replay()
    else:
        loop.enqueue()
    return dict(out=db.out, lse=db.lse, seg_k=db.seg_k, seg_vt=db.seg_vt, seg_len=db.seg_len[:db.layers], err=db.d_err)


# ------------------------------------------------------------ necessary work
def work(case):
    c, s = case, _Shape(case)
    e, d, hq, hk = (4 if c["dtype"] == "f32" else 2), c["d"], c["hq"], c["hkv"]
    if c["kind"] == "fill":
        n = int(s.ctx.sum() + s.seg.sum() + s.ilen.sum())
        return dict(bytes=4.0 * n * hk * d * e, flops=3.0 * n * hk * d)
    if c["kind"] == "prefill":
        rows = int(s.ctx.sum() + s.seg.sum() + s.ilen.sum())
        pairs = sum(n * (n + 1) / 2.0 for n in s.ilen)
        for b in range(s.B):
            lp, lc = s.lp(b), float(s.ctx[b])
            pairs += lc * lp + lc * (lc + 1) / 2
            for n in s.seg[s.qs[b]:s.qs[b + 1]]:
                pairs += float(n) * (lp + lc) + n * (n + 1) / 2.0
        return dict(bytes=float(rows) * (2 * hk * d * e + hq * d * (e + 4)), flops=4.0 * d * hq * pairs)
    by = fl = 0.0
    seg = s.seg.copy()
    for a in s.active:
        for b in range(s.B):
            i = np.arange(s.qs[b], s.qs[b + 1])[a[s.qs[b]:s.qs[b + 1]]]
            if len(i) == 0:
                continue
            by += 2.0 * s.ctx[b] * hk * d * e
            by += float(np.sum(2 * seg[i] * hk * d * e + (hq + 2 * hk) * d * e + 2 * hk * d * e + (hq * d + hq) * 4))
            if c["kind"] == "attend":
                by += 2.0 * len(i) * hq * d * e      # the rotated queries, written and read
            fl += 4.0 * d * hq * float(np.sum(s.lp(b) + s.ctx[b] + seg[i] + 1))
        for k in range(s.S):
            q0, q1 = s.qs[s.istart[k]], s.qs[s.istart[k + 1]]
            if a[q0:q1].any():
                by += 2.0 * s.ilen[k] * hk * d * e
        seg = seg + a
    return dict(bytes=by * c["layers"], flops=fl * c["layers"])


def tolerance(case):
    # about four times what the calls are off the same sums in 64 bits: bf16 operands and probabilities are rounded to
    # 8 bits once (1.8e-3), fp32 sums run over a few thousand terms (3.4e-7).  The largest single difference is that of
    # the first context rows, whose few keys leave values far above the others' root mean square.
    return {"rel": 1.5e-6, "max": 6e-5} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 0.28}


# ------------------------------------------------- the same in 64 bits, plain
def _rope(x, pos):
    """Rotate-half embedding of x [n, heads, d] at pos [n]."""
    h = x.shape[-1] // 2
    th = torch.tensor([ROPE_BASE ** (-j / h) for j in range(h)], dtype=torch.float64, device=x.device)
    ang = torch.as_tensor(pos, dtype=torch.float64, device=x.device)[:, None] * th
    cs, sn = ang.cos()[:, None, :], ang.sin()[:, None, :]
    x = x.double()
    return torch.cat([x[..., :h] * cs - x[..., h:] * sn, x[..., h:] * cs + x[..., :h] * sn], -1)


def _attend(q, k, v, causal_from=None):
    """q [m, hq, d] over k, v [n, hkv, d]; row r sees keys 0 .. causal_from + r (all if None).  (out, lse)."""
    m, hq, d = q.shape
    n, hk, _ = k.shape
    g = hq // hk
    out = torch.empty(m, hq, d, dtype=torch.float64, device=q.device)
    lse = torch.empty(m, hq, dtype=torch.float64, device=q.device)
    kt = k.permute(1, 2, 0).contiguous()
    vv = v.double().permute(1, 0, 2).contiguous()
    blk = max(1, (1 << 26) // max(1, n))
    for h in range(hq):
        for r0 in range(0, m, blk):
            r1 = min(m, r0 + blk)
            top = n if causal_from is None else min(n, causal_from + r1)
            s = (q[r0:r1, h].contiguous() @ kt[h // g][:, :top]) / math.sqrt(d)
            if causal_from is not None:
                see = causal_from + torch.arange(r0, r1, device=q.device)
                s.masked_fill_(torch.arange(top, device=q.device)[None, :] > see[:, None], -math.inf)
            l = torch.logsumexp(s, -1)
            out[r0:r1, h] = torch.exp(s - l[:, None]) @ vv[h // g][:top]
            lse[r0:r1, h] = l
    return out, lse


def _blocked(v):
    """[.., n, hkv, d] values to [.., hkv, n / 8, d, 8] column blocks."""
    *lead, n, hk, d = v.shape
    x = v.reshape(*lead, n // 8, 8, hk, d)
    k = len(lead)
    return x.permute(*range(k), k + 2, k, k + 3, k + 1).contiguous()


def exact(case, seed):
    c, s = case, _Shape(case)
    gen = _gen(seed)
    hq, hk, d = c["hq"], c["hkv"], c["d"]
    ioff = np.concatenate([[0], np.cumsum(s.ilen)]).astype(int)
    coff = np.concatenate([[0], np.cumsum(s.ctx)]).astype(int)
    soff = np.concatenate([[0], np.cumsum(s.seg)]).astype(int)
    cap = (int(s.seg.max()) + c["steps"] + 7) // 8 * 8
    r8 = lambda n: (int(n) + 7) // 8 * 8  # noqa: E731

    def ins(b):
        k = s.instr_of[b]
        return slice(ioff[k], ioff[k + 1])

    if c["kind"] in ("fill", "prefill"):
        (ik, iv), (ck, cv), (sk, sv) = _layer_inputs(c, s, gen)
        pi = np.concatenate([np.arange(n) for n in s.ilen]) if s.S else np.zeros(0)
        pc = np.concatenate([s.lp(b) + np.arange(s.ctx[b]) for b in range(s.B)])
        ps = np.concatenate([s.lp(s.prompt[i]) + s.ctx[s.prompt[i]] + np.arange(s.seg[i]) for i in range(s.nt)])
        # rows of the pool: instructions first, then contexts, each padded to 8
        po = np.concatenate([[0], np.cumsum([r8(n) for n in list(s.ilen) + list(s.ctx)])]).astype(int)
        pool = int(po[-1])
        ri = [torch.arange(po[k], po[k] + s.ilen[k], device=DEV) for k in range(s.S)]
        rc = [torch.arange(po[s.S + b], po[s.S + b] + s.ctx[b], device=DEV) for b in range(s.B)]
        rs = _seg_rows(s, cap)
        kr = [_rope(a, torch.from_numpy(p).to(DEV)) for a, p in ((ik, pi), (ck, pc), (sk, ps))]

        def lay(n, rows_values, heads):
            to = torch.zeros(n, heads, d, dtype=torch.float64, device=DEV)
            for rows, val in rows_values:
                if len(rows):
                    to[rows] = val.double()
            return to

        ra, rb = (torch.cat(ri) if s.S else torch.zeros(0, dtype=torch.int64, device=DEV)), torch.cat(rc)
        if c["kind"] == "fill":
            return dict(ctx_k=lay(pool, [(ra, kr[0]), (rb, kr[1])], hk).permute(1, 0, 2).contiguous(),
                        ctx_vt=_blocked(lay(pool, [(ra, iv), (rb, cv)], hk)),
                        seg_k=lay(s.nt * cap, [(rs, kr[2])], hk).reshape(s.nt, cap, hk, d).permute(0, 2, 1, 3).contiguous(),
                        seg_vt=_blocked(lay(s.nt * cap, [(rs, sv)], hk).reshape(s.nt, cap, hk, d)),
                        seg_len=None, err=None)
        iq, cq, sq = _prefill_inputs(c, s, gen)
        qr = [_rope(a, torch.from_numpy(p).to(DEV)) for a, p in ((iq, pi), (cq, pc), (sq, ps))]
        oc = torch.zeros(pool, hq, d, dtype=torch.float64, device=DEV)
        og = torch.zeros(s.nt, cap, hq, d, dtype=torch.float64, device=DEV)
        for k in range(s.S):
            sl = slice(ioff[k], ioff[k + 1])
            oc[ri[k]] = _attend(qr[0][sl], kr[0][sl], iv[sl], 0)[0]
        for b in range(s.B):
            lp, sl = s.lp(b), slice(coff[b], coff[b + 1])
            k, v = kr[1][sl], cv[sl]
            if lp:
                k, v = torch.cat([kr[0][ins(b)], k]), torch.cat([iv[ins(b)], v])
            oc[rc[b]] = _attend(qr[1][sl], k, v, lp)[0]
            for i in range(s.qs[b], s.qs[b + 1]):
                ss = slice(soff[i], soff[i + 1])
                og[i, :s.seg[i]] = _attend(qr[2][ss], torch.cat([k, kr[2][ss]]), torch.cat([v, sv[ss]]),
                                           lp + int(s.ctx[b]))[0]
        return dict(ctx=oc, seg=og.reshape(s.nt, cap, hq, d), err=None)

    layers = [_layer_inputs(c, s, gen) for _ in range(c["layers"])]
    steps = _step_inputs(c, s, gen)
    segk, segv = [], []
    for (ik, iv), (ck, cv), (sk, sv) in layers:
        tk = torch.zeros(s.nt, cap, hk, d, dtype=torch.float64, device=DEV)
        tv = torch.zeros_like(tk)
        for i in range(s.nt):
            b, n = s.prompt[i], int(s.seg[i])
            when = [t for t in range(c["steps"]) if s.active[t][i]]
            raw = torch.cat([sk[soff[i]:soff[i + 1]]] + [steps[t][1][i][None] for t in when])
            val = torch.cat([sv[soff[i]:soff[i + 1]]] + [steps[t][2][i][None] for t in when])
            tk[i, :n + len(when)] = _rope(raw, s.lp(b) + s.ctx[b] + torch.arange(n + len(when), device=DEV))
            tv[i, :n + len(when)] = val.double()
        segk.append(tk)
        segv.append(tv)
    out = torch.zeros(s.nt, hq, d, dtype=torch.float64, device=DEV)
    lse = torch.zeros(s.nt, hq, dtype=torch.float64, device=DEV)
    (ik, iv), (ck, cv), _ = layers[-1]
    for b in range(s.B):
        i = [j for j in range(s.qs[b], s.qs[b + 1]) if s.fed[j]]
        if not i:
            continue
        lp, sl = s.lp(b), slice(coff[b], coff[b + 1])
        k, v = _rope(ck[sl], lp + torch.arange(s.ctx[b], device=DEV)), cv[sl]
        if lp:
            k = torch.cat([_rope(ik[ins(b)], torch.arange(lp, device=DEV)), k])
            v = torch.cat([iv[ins(b)], v])
        # the row of a question is that of the last step it was fed at
        q = torch.stack([steps[max(t for t in range(c["steps"]) if s.active[t][j])][0][j] for j in i])
        n = torch.tensor([int(s.seg[j] + s.fed[j]) for j in i], device=DEV)
        q = _rope(q, lp + int(s.ctx[b]) + n - 1)
        o1, l1 = _attend(q, k, v)
        g = hq // hk
        ks, vs = segk[-1][i].permute(0, 2, 1, 3), segv[-1][i].permute(0, 2, 1, 3)      # [m, hk, cap, d]
        sc = (q.reshape(len(i), hk, g, 1, d) * ks[:, :, None]).sum(-1) / math.sqrt(d)
        sc.masked_fill_((torch.arange(cap, device=DEV)[None, :] >= n[:, None])[:, None, None], -math.inf)
        l2 = torch.logsumexp(sc, -1)
        o2 = (torch.exp(sc - l2[..., None])[..., None] * vs[:, :, None]).sum(-2).reshape(len(i), hq, d)
        l2 = l2.reshape(len(i), hq)
        l = torch.logaddexp(l1, l2)
        out[i] = o1 * torch.exp(l1 - l)[..., None] + o2 * torch.exp(l2 - l)[..., None]
        lse[i] = l
    return dict(out=out, lse=lse, seg_k=[x.permute(0, 2, 1, 3).contiguous() for x in segk],
                seg_vt=[_blocked(x) for x in segv], seg_len=[None] * c["layers"], err=None)
