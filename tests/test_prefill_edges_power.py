"""CPU: the GPU test of the prefill's tile edges notices one lost key.  Outputs with
the first or last key of a half, tile or step hidden, rounded as the kernel
rounds, lie beyond the test's bound."""
import numpy as np
import pytest

from tests.prefill_edges import CASES, inputs, positions, reference
from tests.rounded_reference import beyond, bf16, rotate


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_a_hidden_key_is_seen(case):
    lc = case[4]
    ck, _, _, sk, _, _ = inputs(case)
    pos_c, pos_s = positions(case)
    kc, ks = (np.ascontiguousarray(bf16(rotate(k, p)).transpose(1, 0, 2)) for k, p in ((ck, pos_c), (sk, pos_s)))
    (o_ctx, b_ctx), (o_seg, b_seg) = reference(case, kc, ks)
    assert beyond(o_ctx, o_ctx, b_ctx) == (0.0, 0.0) and beyond(o_seg, o_seg, b_seg)[0] == 0.0
    for key in (0, 31, 32, 63, 64, 127, 128):
        if not any(n > key + 1 for n in lc):
            continue
        (h_ctx, _), (h_seg, _) = reference(case, kc, ks, hide=key)
        share = beyond(h_ctx, o_ctx, b_ctx)[0], beyond(h_seg, o_seg, b_seg)[0]
        assert max(share) > 1e-2, (key, share)      # ten times what the test allows
