"""Products of small matrices for up to 64 tokens (k_gemm_small, k_gemm_small_split): from one K batch to the longest K range that each form takes and one
beyond, against the oracle, and with 32 rows bit for bit what 64 rows give, whose residual products the general kernel computes."""
import numpy as np
import pytest

import fv_inputs as fi
from fv_inputs.shapes import ModelShape
from tests import helpers as H

pytestmark = pytest.mark.gpu


SHAPES = [   # K batches of the hidden size and of ffn: 128 columns each in bf16, 64 in fp32
    ("bf16", 128, 2, 64, 1152),      # 1, 9
    ("bf16", 256, 2, 128, 1040),     # 2, 9 with zeros behind the end
    ("bf16", 384, 6, 64, 2048),      # 3, 16
    ("bf16", 640, 5, 128, 2176),     # 5, 17
    ("bf16", 1024, 8, 128, 2048),    # 8, 16
    ("bf16", 1152, 9, 128, 2176),    # 9, 17
    ("f32", 192, 3, 64, 528),        # 3, 9 with zeros behind the end
    ("f32", 512, 4, 128, 1024),      # 8, 16
    ("f32", 576, 9, 64, 1376),       # 9, 22
]


@pytest.mark.parametrize("dtype,hidden,heads,head_dim,ffn", SHAPES)
def test_small_matrices(dtype, hidden, heads, head_dim, ffn):
    import paper_2412_12639_amd as fv
    s = ModelShape(f"small-{hidden}-{ffn}", 2, hidden, heads, heads, head_dim, ffn, 500, dtype)
    w = fi.gen_weights(s, seed=3, gain_jitter=0.1)
    tol = H.tol_for(s)
    case = H.planted_case(s, w, 40, 64, [6, 3, 2, 2, 1, 1], 3, seed=4)
    g = fv.FalconVerifier(s, max_seq=120, max_tree=64)
    g.init_weights(w)
    g.set_step_invariant(True)
    assert g.prefill(case["prefix"]) == case["root"]
    tokens, parent, depth = case["tokens"], case["parent"], case["depth"]
    rows = []
    for n in (1, 20, 32, 33, 64):
        g.rollback(40, case["root"])
        got = g.verify_tree(tokens[:n], parent[:n], depth[:n])
        rows.append(g.logits(n).copy())
    H.check_step(g, case, got, tol)
    g.close()
    for r in rows:
        assert np.array_equal(r, rows[-1][:len(r)]), len(r)


@pytest.mark.parametrize("dtype,hidden,heads,head_dim,ffn", SHAPES)
def test_small_forms_give_the_direct_kernels_bits(dtype, hidden, heads, head_dim, ffn, monkeypatch):
    import paper_2412_12639_amd as fv
    s = ModelShape(f"small-{hidden}-{ffn}", 2, hidden, heads, heads, head_dim, ffn, 500, dtype)
    w = fi.gen_weights(s, seed=5, gain_jitter=0.1)
    parent, depth, _ = fi.gen_tree(5, 64, [6, 3, 2, 2, 1, 1])
    root, got = 7, []
    tokens = fi.trees.fill_tokens(5, parent, s.vocab, root)
    for switch in ("1", "0"):
        monkeypatch.setenv("FV_GEMM_SMALL", switch)
        g = fv.FalconVerifier(s, max_seq=120, max_tree=64)
        g.init_weights(w)
        g.prefill(fi.gen_prefix(1, 40, s.vocab))
        out = []
        for n in (1, 20, 32, 33, 64):
            g.rollback(40, root)
            a, _, _ = g.verify_tree(tokens[:n], parent[:n], depth[:n])
            out += [g.logits(n).copy(), g.features(a + 1).copy()]
        got.append(out + list(g.read_kv(1, 0, 41)))
        g.close()
    for x, y in zip(*got):
        assert np.array_equal(x, y)
