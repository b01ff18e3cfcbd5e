"""Residual products whose row groups many workgroups share (k_gemm_paired_long): from just above four contributors a group to 32, K ranges whose parts end
inside and at the ends of groups, against the oracle, and with 32 rows bit for bit what 64 rows give."""
import numpy as np
import pytest

import fv_inputs as fi
from fv_inputs.shapes import ModelShape
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hidden,heads,ffn", [   # row groups of 64: hidden / 64, in 256 equal parts of the K range
    ("bf16", 1024, 8, 3328),      # 16 groups, 16 parts each
    ("bf16", 1152, 9, 3456),      # 18 groups, 14.2
    ("bf16", 2048, 16, 3328),     # 32 groups, 8 each: the plain form above 32 rows
    ("bf16", 3200, 25, 3328),     # 50 groups, 5.1
    ("bf16", 4096, 32, 3328),     # 64 groups, 4 each: the plain form
    ("f32", 512, 4, 1664),        # 8 groups, 32 each
    ("f32", 768, 6, 1680),        # 12 groups, 21.3, zeros behind the end of the K range
    ("f32", 1920, 15, 1664),      # 30 groups, 8.5
])
def test_many_contributors(dtype, hidden, heads, ffn):
    import paper_2412_12639_amd as fv
    s = ModelShape(f"long-{hidden}-{ffn}", 1, hidden, heads, heads, 128, ffn, 500, dtype)
    w = fi.gen_weights(s, seed=7, gain_jitter=0.1)
    case = H.planted_case(s, w, 20, 64, [6, 3, 2, 2, 1, 1], 3, seed=6)
    g = fv.FalconVerifier(s, max_seq=100, max_tree=64)
    g.init_weights(w)
    g.set_step_invariant(True)
    assert g.prefill(case["prefix"]) == case["root"]
    rows = []
    for n in (1, 32, 33, 64):
        g.rollback(20, case["root"])
        got = g.verify_tree(case["tokens"][:n], case["parent"][:n], case["depth"][:n])
        rows.append(g.logits(n).copy())
    H.check_step(g, case, got, H.tol_for(s))
    g.close()
    for r in rows:
        assert np.array_equal(r, rows[-1][:len(r)]), len(r)
