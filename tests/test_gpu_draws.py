"""The tokens that a non-greedy step draws, at recorded inputs.

A draw inverts a cumulative sum over the vocabulary.  Where the model is unsure, a token carries a share of about 1e-4 to 1e-5,
so some of many draws fall to a neighbour as soon as logits move by their last few bits -- which every change in the order of a sum does,
in the step itself or in the prompt whose K and V it reads.  The same inputs are to give the same draws, so the tokens are recorded here,
as a digest of 256 of them over a nearly uniform distribution.  A digest that changes says that a sum runs in another order, not
that a result is inaccurate (tests/test_gpu_sampled.py holds the draws to the device's own logits, test_gpu_parity.py the logits to the oracle)."""
import hashlib

import numpy as np
import pytest

import fv_inputs as fi
from fv_inputs.shapes import ModelShape

pytestmark = pytest.mark.gpu

CASES = [
    # prefix, nodes, FFN width, digest of the drawn tokens
    (333, 33, 272, "a978081561d439b4"),      # 256 rows of the prompt in a chunk of their own
    (700, 33, 6640, "dd3d9bf94e4d3737"),     # 512 rows and the last chunk at once, long K ranges
    (2048, 250, 272, "f088aacf0cbdebf1"),    # the attention of 256 (head, node block) items over 72 key blocks
    (40, 100, 11008, "4fa621aa28cbf483"),    # 172 row groups of gate and up in equal ranges over 256 workgroups
]


def draws(prefix_len, nodes, ffn, n=256):
    import paper_2412_12639_amd as fv
    s = ModelShape(f"draws-{ffn}", 2, 256, 32, 8, 64, ffn, 16384, "bf16")
    g = fv.FalconVerifier(s, max_seq=prefix_len + 264, max_tree=256)
    g.init_weights(fi.gen_weights(s, seed=ffn, gain_jitter=0.1))
    root = g.prefill(fi.gen_prefix(prefix_len, prefix_len, s.vocab))
    parent, depth, _ = fi.gen_tree(nodes, nodes, [8, 4, 2, 2, 1, 1])
    rng = np.random.Generator(np.random.Philox(nodes))
    tokens = rng.integers(0, s.vocab, nodes).astype(np.int32)
    out = []
    for _ in range(n):
        g.rollback(prefix_len, root)
        tokens[0] = root
        out.append(g.verify_tree_sampled(tokens, parent, depth, 1.0, rng.random(nodes), rng.random(nodes))[2])
    g.close()
    return np.array(out, dtype=np.int32)


@pytest.mark.parametrize("prefix_len,nodes,ffn,digest", CASES)
def test_draws_are_the_recorded_ones(prefix_len, nodes, ffn, digest):
    got = draws(prefix_len, nodes, ffn)
    assert len(set(got.tolist())) > 200      # spread over the vocabulary
    assert hashlib.sha256(got.tobytes()).hexdigest()[:16] == digest
