"""Non-greedy verification where its kernels change over: at the edges of the groups of 2048 tokens that the on-chip form is built for, and above the 32768
tokens that it takes.  Decisions are held to the oracle's rule on the logits the device produced, as in test_gpu_sampled.py."""
from dataclasses import replace

import numpy as np
import pytest

import fv_inputs as fi
from oracle import falcon_oracle as fo

pytestmark = pytest.mark.gpu

L, N = 20, 24


def _session(vocab, seed=7):
    import paper_2412_12639_amd as fv
    s = replace(fi.SHAPES["tiny"], name=f"tiny-v{vocab}", vocab=vocab)
    g = fv.FalconVerifier(s, max_seq=64, max_tree=32)
    w = fi.gen_weights(s, seed=seed)
    g.init_weights(w)
    return g, s, w, g.prefill(fi.gen_prefix(4, L, vocab))


def _step(rng, vocab, root):
    parent, depth, _ = fi.gen_tree(9, N, [12, 2, 2])
    tokens = rng.integers(0, vocab, N).astype(np.int32)
    tokens[0], tokens[1], tokens[2] = root, vocab - 1, vocab // 2
    return tokens, parent, depth


def _proposals(rng, vocab):
    import torch
    q = rng.random((N, vocab), dtype=np.float32) ** 3
    q = (q / q.sum(axis=1, keepdims=True, dtype=np.float64)).astype(np.float32)
    return q, torch.from_numpy(q).cuda()


@pytest.mark.parametrize("proposals", [False, True])
@pytest.mark.parametrize("vocab", [33, 2047, 2049, 4095, 4096, 4097, 8192, 8193, 8196, 16384, 16385, 16388])
def test_decisions_at_the_edges_of_groups(vocab, proposals):
    g, s, _, root = _session(vocab)
    rng = np.random.default_rng(vocab)
    checked = 0
    for _ in range(4):
        tokens, parent, depth = _step(rng, vocab, root)
        ua, us = rng.uniform(0.2, 1.0, N), rng.uniform(0.0, 0.999, N)
        q, qdev = _proposals(rng, vocab) if proposals else (None, None)
        got = g.verify_tree_sampled(tokens, parent, depth, 1.0, ua, us, qdev)
        logits = g.logits(N)
        assert list(g.argmax()) == [int(i) for i in np.argmax(logits, axis=1)]
        d = fo.sampled_accept(logits.astype(np.float64), tokens, parent, depth, L, np.float32(1.0), ua, us, q)
        g.rollback(L, root)
        if d["min_margin"] < 1e-7:      # a decision too close to its threshold to demand anything of it
            continue
        checked += 1
        assert got[0] == d["accepted_len"] and list(got[1]) == list(d["accepted_tokens"]) and got[2] == d["next_token"]
    assert checked >= 2
    g.close()
