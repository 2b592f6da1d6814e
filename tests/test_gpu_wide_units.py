"""GPU: decode units of 256 and 128 rows (bf16, head dim 128; two wave groups
half a step apart over 64-key tiles, at 128 rows on every other tile) against the fp64 oracle at the edges of their
tiles: contexts of 1 to 5 tiles with empty, partial and whole halves, chunks
that end inside a tile, 1 to 16 heads per kv head (quads that do and do not
share a question), waves and a whole wave group without active rows, and
instruction units.  The caches hold NaN where nothing is loaded.  Tolerance
2e-2: operands and weights are rounded to 8 bits, as everywhere in bf16.  As
that hides a lost key of a long context, the outputs and log sums are also
compared with fp64 over the call's own rounded queries and cached keys, where
only the weights' rounding is left (rounded_reference.py): one key of n moves a
log sum by about 1 / n, the bound is 2^-9."""
import numpy as np
import pytest

import workload as W
from oracle import ippd as O
from paper_2609_05707_amd.session import DecodeBatch
from tests.gpu_harness import load_layer, log, make_batch, max_err, oracle_steps, run_gpu
from tests.rounded_reference import EPS, attend, beyond
from tests.test_gpu_twolevel import run_steps

pytestmark = pytest.mark.gpu

TOL = 2e-2


def poison(db):
    for bufs in (db.ctx_k, db.ctx_vt, db.seg_k, db.seg_vt):
        for x in bufs:
            x.fill_(float("nan"))


def check_rounded(db, st, gpu, t):
    """Step t's outputs against fp64 over its rotated queries, the cached keys and values."""
    si = W.step_inputs(st, t)
    kc, vc = db.ctx_k[0].double().cpu().numpy(), db.ctx_values(0).double().cpu().numpy()
    ks, vs = db.seg_k[0].double().cpu().numpy(), db.seg_values(0).double().cpu().numpy()
    n, g, d = st.seg_len_at(t + 1), db.hq // db.hkv, db.D
    share, most, off = [], 0.0, 0.0
    for b in range(len(st.ctx_len)):
        c = slice(int(db.ctx_off[b]), int(db.ctx_off[b] + st.ctx_len[b]))
        for i in range(st.q_start[b], st.q_start[b + 1]):
            if not si.active[i]:
                continue
            for k in range(db.hkv):
                key = np.concatenate([kc[k, c], ks[i, k, : n[i]]])
                val = np.concatenate([vc[k, :, c].T, vs[i, k, :, : n[i]].T])
                h = slice(k * g, k * g + g)
                out, bound, lse = attend(gpu.q_rot[t][i, h].astype(np.float64) @ key.T / np.sqrt(d), val)
                s, m = beyond(gpu.out[t][i, h], out, bound)
                share.append(s)
                most, off = max(most, m), max(off, float(np.abs(gpu.lse[t][i, h] - lse).max()))
    log(f"  step {t}: {np.mean(share):.1e} of the outputs beyond the weights' rounding, largest {most:.2f} times it; lse {off:.1e}")
    assert np.mean(share) == 0 and off <= EPS + 2e-5


CASES = [
    # hq, hkv, context lengths, questions, stop range, chunk tokens
    (8, 2, (1, 1), (3, 3), None, 0),
    (8, 2, (31, 33), (64, 70), (1, 2), 0),
    (8, 2, (64, 64), (9, 40), (1, 2), 0),
    (8, 2, (65, 97), (33, 33), (1, 2), 0),
    (8, 2, (200, 330), (60, 66), (1, 2), 96),
    (8, 2, (253, 320), (64, 64), (1, 2), 0),
    (8, 2, (900, 1100), (20, 32), (1, 2), 1024),
    (6, 2, (130, 200), (50, 90), (1, 2), 64),
    (16, 1, (300, 301), (14, 18), (1, 2), 0),
    (4, 4, (190, 193), (200, 257), (1, 2), 0),
]


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_wide_units(case, rows, fused):
    hq, hkv, ctx, qs, stop, chunk = CASES[case]
    log(f"case: {rows}-row units {CASES[case]} fused={fused}")
    wl = W.custom_workload(wid=700 + case, dtype="bf16", num_prompts=3, hq=hq, hkv=hkv, head_dim=128, ctx_len=ctx,
                           questions=qs, seg_len=(1, 9), steps=2, stop=stop, value_std=0.5)
    st = W.make_structure(wl)
    kv = W.layer_kv(st)
    db = make_batch(st, chunk_tokens=chunk, tile_rows=rows)
    poison(db)
    load_layer(db, st, 0, kv)
    gpu = run_gpu(st, [0, 1], [0, 1], db=db, kv=kv, fused=fused, sentinel=-555.0)
    ref = oracle_steps(st, kv, [0, 1], [0, 1])
    assert gpu.err == 0
    for t in (0, 1):
        act = W.step_inputs(st, t).active
        e = max_err(gpu.out[t][act], ref[t][0][act]), max_err(gpu.lse[t][act], ref[t][1][act])
        log(f"  step {t}: {int(act.sum())} active, max err {e[0]:.3e}, lse {e[1]:.3e}")
        assert np.isfinite(gpu.out[t]).all() and e[0] <= TOL and e[1] <= TOL
        assert (gpu.out[t][~act] == -555.0).all()
        check_rounded(db, st, gpu, t)


@pytest.mark.parametrize("mode", ["fused", "separate"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("hq,lp", [(8, (1, 40)), (8, (250, 330)), (6, (64, 130))])
def test_wide_instruction_units(hq, lp, rows, mode):
    log(f"case: {rows}-row instruction units hq={hq} instruction {lp} mode={mode}")
    wl = W.custom_workload(wid=720 + hq, dtype="bf16", num_prompts=6, hq=hq, hkv=2, head_dim=128, ctx_len=(20, 150),
                           questions=(8, 30), seg_len=(1, 9), steps=2, stop=(1, 2), value_std=0.5)
    st = W.make_structure(wl)
    ins = W.instructions(st, 3, lp)
    db = DecodeBatch(st.ctx_len.tolist(), st.q_count.tolist(), hq, 2, 128, "bf16", 16, instr_len=ins.lp.tolist(),
                     instr_prompt_start=ins.prompt_start.tolist(), tile_rows=rows)
    poison(db)
    kv = W.layer_kv(st)
    db.load_instructions(0, ins.k, ins.v)
    load_layer(db, st, 0, kv)
    got = run_steps(db, st, mode)
    instr = O.Instructions(ins.prompt_start, ins.tok_start, ins.k, ins.v)
    state = O.KVState.from_packed(kv.seg_k, kv.seg_v, st.seg_start)
    for t in (0, 1):
        si = W.step_inputs(st, t)
        ref, _ = O.decode_step_standard(kv.ctx_k, kv.ctx_v, st.ctx_start, st.q_start, state, si.q_new, si.k_new,
                                        si.v_new, si.active, wl.rope_base, instr=instr)
        state.append(si.k_new, si.v_new, si.active)
        e = max_err(got[t][si.active], ref[si.active])
        log(f"  step {t}: max err {e:.3e}")
        assert np.isfinite(got[t][si.active]).all() and e <= TOL
    assert db.err_flag() == 0


@pytest.mark.parametrize("mode", ["fused", "separate"])
@pytest.mark.parametrize("hkv,g,instr", [(8, 4, False), (8, 5, True), (4, 2, False), (1, 7, False)])
def test_segments_after_the_context_units(hkv, g, instr, mode):
    """Calls whose segment units do not fit the chip beside their 128-row
    context units, for kv heads 1 to 8 (eight tasks a unit are one to eight
    questions), with prompts without questions and stopped questions."""
    log(f"case: segments after the context units hkv={hkv} G={g} instr={instr} mode={mode}")
    B = 32 // hkv + 8
    wl = W.custom_workload(wid=760 + hkv + g, dtype="bf16", num_prompts=B, hq=hkv * g, hkv=hkv, head_dim=128,
                           ctx_len=(60, 400), questions=(0, 1024 // (hkv * B) + 40), seg_len=(1, 70), steps=2, stop=(1, 2),
                           value_std=0.5)
    st = W.make_structure(wl)
    kv = W.layer_kv(st)
    ins = W.instructions(st, 3, (30, 200)) if instr else None
    ikw = dict(instr_len=ins.lp.tolist(), instr_prompt_start=ins.prompt_start.tolist()) if instr else {}
    db = DecodeBatch(st.ctx_len.tolist(), st.q_count.tolist(), hkv * g, hkv, 128, "bf16", 72, tile_rows=128,
                     chunk_tokens=32, **ikw)
    poison(db)
    if instr:
        db.load_instructions(0, ins.k, ins.v)
    load_layer(db, st, 0, kv)
    got = run_steps(db, st, mode)
    kw = dict(instr=O.Instructions(ins.prompt_start, ins.tok_start, ins.k, ins.v)) if instr else {}
    state = O.KVState.from_packed(kv.seg_k, kv.seg_v, st.seg_start)
    for t in (0, 1):
        si = W.step_inputs(st, t)
        ref, _ = O.decode_step_standard(kv.ctx_k, kv.ctx_v, st.ctx_start, st.q_start, state, si.q_new, si.k_new,
                                        si.v_new, si.active, wl.rope_base, **kw)
        state.append(si.k_new, si.v_new, si.active)
        e = max_err(got[t][si.active], ref[si.active])
        log(f"  step {t}: {int(si.active.sum())} of {st.num_questions} active, max err {e:.3e}")
        assert np.isfinite(got[t][si.active]).all() and e <= TOL
        assert (got[t][~si.active] == -555.0).all()
    np.testing.assert_array_equal(db.seg_len[0][: st.num_questions].cpu().numpy(), st.seg_len_at(2))
    assert db.err_flag() == 0


@pytest.mark.parametrize("g", [14, 15])
def test_segment_tasks_of_wide_groups(g):
    """Head dim 64, 14 and 15 heads per kv head, more segment tasks than the
    chip holds beside the context units: a task keeps a wave's state in the
    unit's LDS however many tasks share the unit, and its cached keys count."""
    log(f"case: segment tasks D=64 G={g}")
    wl = W.custom_workload(wid=790 + g, dtype="bf16", num_prompts=6, hq=g, hkv=1, head_dim=64, ctx_len=(88, 96),
                           questions=(256, 256), seg_len=(2, 40), steps=1, value_std=0.5)
    st = W.make_structure(wl)
    kv = W.layer_kv(st)
    db = make_batch(st)
    poison(db)
    load_layer(db, st, 0, kv)
    gpu = run_gpu(st, [0], [0], db=db, kv=kv, fused=True)
    ask = list(range(0, st.num_questions, 23))
    out, lse = oracle_steps(st, kv, [0], [0], questions={0: ask})[0]
    e = max_err(gpu.out[0][ask], out[ask]), max_err(gpu.lse[0][ask], lse[ask])
    log(f"  {len(ask)} questions, max err {e[0]:.3e}, lse {e[1]:.3e}")
    assert gpu.err == 0 and e[0] <= TOL and e[1] <= TOL
