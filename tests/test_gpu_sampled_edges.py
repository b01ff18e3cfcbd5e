"""Non-greedy verification where its kernels change over: at the edges of the groups of 2048 tokens that the on-chip form is built for, and above the 32768
tokens that it takes (there, struck tokens of point-mass proposals as well); equal and non-finite logits.  Decisions are held to the oracle's rule on the logits the device produced, as in test_gpu_sampled.py."""
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
@pytest.mark.parametrize("vocab", [33, 2047, 2049, 4095, 4096, 4097, 8192, 8193, 8196, 16384, 16385, 16388, 32768, 32769, 32772])
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


@pytest.mark.parametrize("proposals", [False, True])
@pytest.mark.parametrize("vocab", [1004, 8196, 32772])
def test_the_lowest_of_equal_logits_is_the_greedy_choice(vocab, proposals):
    """Head rows of the tokens that lead at some nodes, repeated at other tokens: in the same four, in other lanes, wavefronts and groups."""
    g, s, w, root = _session(vocab)
    rng = np.random.default_rng(vocab)
    tokens, parent, depth = _step(rng, vocab, root)
    ua, us = rng.uniform(0.2, 1.0, N), rng.random(N)
    qdev = _proposals(rng, vocab)[1] if proposals else None
    g.verify_tree_sampled(tokens, parent, depth, 1.0, ua, us, qdev)
    lead = list(dict.fromkeys(int(t) for t in g.argmax()))[:6]
    g.close()
    head = w["lm_head"].copy()
    free = [t for t in (0, 1, 2, 3, 7, 255, 256, 700, 1001, 1002, 1003, 2047, 2048, 4097, 8191, 8192, 8195, 20000, 32771, *range(300, 330)) if t < vocab and t not in lead]
    for k, t in enumerate(lead):
        for at in free[k::len(lead)][:4]:
            head[at] = head[t]
    w = dict(w, lm_head=head)
    import paper_2412_12639_amd as fv
    g = fv.FalconVerifier(s, max_seq=64, max_tree=32)
    g.init_weights(w)
    g.prefill(fi.gen_prefix(4, L, vocab))
    g.rollback(L, root)
    got = g.verify_tree_sampled(tokens, parent, depth, 1.0, ua, us, qdev)
    logits = g.logits(N)
    assert (np.sum(logits == logits.max(axis=1, keepdims=True), axis=1) > 1).sum() >= len(lead) // 2   # (rows of strips whose K range is split elsewhere add in another order)
    assert list(g.argmax()) == [int(i) for i in np.argmax(logits, axis=1)]
    assert 0 <= got[2] < vocab
    g.close()


@pytest.mark.parametrize("proposals", [False, True])
@pytest.mark.parametrize("vocab", [1003, 1004, 32769, 32772])
def test_non_finite_logits_on_the_path_are_an_error_and_off_it_are_not(vocab, proposals):
    """A NaN comes from a token whose embedding is NaN, an infinity from a head row that overflows fp32 where the normalised hidden state is above one at a
    feature; the session's prompt and the other nodes do not meet them.  The first and the last token of the vocabulary have the head rows (the last
    four of a row are read together, whether they are all tokens or not)."""
    import paper_2412_12639_amd as fv
    g, s, w, root = _session(vocab)
    rng = np.random.default_rng(vocab)
    tokens, parent, depth = _step(rng, vocab, root)
    prefix = fi.gen_prefix(4, L, vocab)
    poison = next(t for t in range(vocab) if t not in set(int(x) for x in prefix) | set(int(x) for x in tokens))
    ua, us = np.ones(N), rng.uniform(0.1, 0.9, N)
    q, qdev = _proposals(rng, vocab) if proposals else (None, None)

    def normed(n):
        x = g.activation("x", n).astype(np.float64)
        return x / np.sqrt((x * x).mean(axis=1, keepdims=True) + s.rms_eps) * w["g_final"]

    end = normed(L)[-1]                      # the prompt's last row, whose logits must stay finite
    g.verify_tree_sampled(tokens, parent, depth, 1.0, ua, us, qdev)
    rows = normed(N)
    at_root = rows[0]
    g.close()

    def session(changed):
        h = fv.FalconVerifier(s, max_seq=64, max_tree=32)
        h.init_weights(dict(w, **changed))
        h.prefill(prefix)
        h.rollback(L, root)
        return h

    def refused(h, toks):
        h.rollback(L, int(toks[0]))
        with pytest.raises(fv.FvError) as ei:
            h.verify_tree_sampled(toks, parent, depth, 1.0, ua, us, qdev)
        assert ei.value.status == -10 and h.state() == (L, int(toks[0]))
        assert h.argmax()[0] == -1

    embed = w["embed"].copy()
    embed[poison] = np.nan
    h = session({"embed": embed})
    bad = tokens.copy()
    bad[0] = poison
    refused(h, bad)
    h.close()
    for sign in (1.0, -1.0):
        f = next(i for i in np.argsort(-sign * at_root) if abs(end[i]) < 0.9)
        assert sign * at_root[f] > 1.2
        for t in (0, vocab - 1):
            head = w["lm_head"].copy()
            head[t] = 0.0
            head[t, f] = 3.3e38
            h = session({"lm_head": head})
            refused(h, tokens)
            assert h.logits(1)[0, t] == sign * np.inf
            h.close()

    # off the path: nodes whose logit overflows at a feature where the root and the prompt's last row are small; u_accept is one and proposals are
    # above one, so the root's children are rejected
    if proposals:
        q = q + np.float32(1.5)
        qdev += 1.5
    f = max((i for i in range(s.hidden) if abs(end[i]) < 0.9 and -0.9 < at_root[i] < 0.0), key=lambda i: np.abs(rows[1:, i]).max())
    for t in (0, vocab - 1):
        head = w["lm_head"].copy()
        head[t] = 0.0
        head[t, f] = 3.3e38
        h = session({"lm_head": head})
        got = h.verify_tree_sampled(tokens, parent, depth, 1.0, ua, us, qdev)
        logits = h.logits(N)
        bad = ~np.isfinite(logits).all(axis=1)
        assert not bad[0] and bad.any()
        assert list(h.argmax()) == [-1 if bad[i] else int(np.argmax(logits[i])) for i in range(N)]
        d = fo.sampled_accept(logits.astype(np.float64), tokens, parent, depth, L, np.float32(1.0), ua, us, q)
        assert not bad[d["path"]].any() and got[0] == d["accepted_len"]
        if d["min_margin"] >= 1e-7:
            assert list(got[1]) == list(d["accepted_tokens"]) and got[2] == d["next_token"]
        h.close()
