"""CPU: the chunk of a decode plan, read from the workspace size.  The
partial states of a plan number (context chunks + 1 + instruction chunks) *
questions * heads; a chunk below 256 tokens is taken only while they fit the
no-allocation step's scratch, so that no batch it took is refused."""
import ctypes
import random

import pytest

from paper_2609_05707_amd import _lib as L
from tests.test_abi import FAKE, lib, valid_batch  # noqa: F401


def states(lib, bt, fn="ippd_decode_workspace_bytes"):  # noqa: F811
    need = getattr(lib, fn)(ctypes.byref(bt))
    return need, need // ((bt.head_dim + 2) * 4)


def batch(**k):
    k.setdefault("ctx_pool_tokens", k["num_prompts"] * k["max_ctx_len"])
    return valid_batch(seg_capacity=64, **k)


@pytest.mark.parametrize("dtype,heads,d,ctx,q,chunks", [
    (L.IPPD_DTYPE_F32, (4, 2), 64, 256, 4, 8),          # 32 tokens: eight units per kv head instead of one
    (L.IPPD_DTYPE_BF16, (32, 8), 128, 512, 4, 8),       # 64 tokens
    (L.IPPD_DTYPE_BF16, (32, 8), 128, 32768, 64, 24),   # 256-row units: segment units resident beside them
])
def test_chunks(lib, dtype, heads, d, ctx, q, chunks):  # noqa: F811
    bt = batch(dtype=dtype, num_prompts=1, num_questions=q, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=d,
               max_ctx_len=ctx, max_questions=q)
    need, _ = states(lib, bt)
    r = lambda x: (x + 255) // 256 * 256  # noqa: E731
    n = (chunks + 1) * q * heads[0]
    assert need == r(n * d * 4) + r(n * 8)


def test_short_chunks_stay_within_the_scratch(lib):  # noqa: F811
    rng = random.Random(5)
    seen = 0
    for _ in range(4000):
        hk = rng.choice([1, 2, 4, 8, 32])
        g = rng.choice([1, 2, 3, 4, 8, 16])
        d = rng.choice([64, 128])
        B = rng.choice([1, 1, 2, 5, 12, 40, 200])
        ctx = 8 * rng.randint(1, 2 ** rng.randint(1, 11))
        q = rng.choice([1, 3, 16, 64, 300, 1024])
        two = rng.random() < 0.3
        k = dict(num_instr=1, max_instr_len=8 * rng.randint(1, 300), max_instr_questions=q * B, instr_start=FAKE,
                 instr_off=FAKE, instr_len=FAKE) if two else {}
        bt = batch(dtype=rng.choice([L.IPPD_DTYPE_F32, L.IPPD_DTYPE_BF16]), num_prompts=B, num_questions=q * B,
                   num_q_heads=hk * g, num_kv_heads=hk, head_dim=d, max_ctx_len=ctx, max_questions=q,
                   **dict(k, ctx_pool_tokens=B * ctx + k.get("max_instr_len", 0)))
        need, _ = states(lib, bt)
        if need <= L.IPPD_NOALLOC_SCRATCH_BYTES:
            continue
        seen += 1
        # refused: then it is refused at every chunk below 256 tokens' worth of the plan, i.e. the 256-token plan is too
        bt.chunk_tokens = 256
        assert states(lib, bt)[0] >= need
    assert seen > 100
