"""One-node steps, whose greedy choice, result and features come from one launch (k_finish_one): at the ends of what 256 and 1024 threads hold at
once and beyond, with the largest logit at the first, the last and two equal tokens, and with logits that are no numbers."""
import numpy as np
import pytest

import fv_inputs as fi
from fv_inputs.shapes import ModelShape

pytestmark = pytest.mark.gpu


def _session(vocab, dtype, edit=None):
    import paper_2412_12639_amd as fv
    s = ModelShape(f"one-{vocab}", 1, 256, 4, 4, 64, 272, vocab, dtype)
    w = fi.gen_weights(s, seed=vocab, gain_jitter=0.1)
    if edit:
        w["lm_head"] = edit(w["lm_head"].copy())
    g = fv.FalconVerifier(s, max_seq=64, max_tree=64)
    g.init_weights(w)
    return s, w, g


def _overflows_behind(root, s, w, token, nan):
    """The same weights but for the logit of `token`, which is infinite, or the difference of two infinities, in a node of token `root` and finite in all
    others: units that are zero but for the root's embedding, and 3e38 in the head there."""
    units = np.r_[0:8, 128:136]      # the two halves of the head's K range
    one, big = (0x3F80, 0x7F60) if s.dtype == "bf16" else (1.0, 2.9774e38)
    w = dict(w, embed=w["embed"].copy(), lm_head=w["lm_head"].copy())
    w["embed"][:, units] = 0
    w["embed"][root, units] = one
    for name in [n for n in w if n.split(".")[-1] in ("wo", "wd")]:
        w[name] = w[name].copy()
        w[name][units] = 0
    w["lm_head"][token] = 0
    w["lm_head"][token, units[:8]] = big
    w["lm_head"][token, units[8:]] = (big | 0x8000 if s.dtype == "bf16" else -big) if nan else 0
    return w


def _f32(a):
    return a if a.dtype == np.float32 else (a.astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab", [33, 1000, 8189, 8192, 8193, 32001, 32768, 32771])
def test_choice_and_features(vocab, dtype):
    s, w, g = _session(vocab, dtype)
    root = g.prefill(fi.gen_prefix(1, 9, s.vocab))
    a, acc, nxt = g.verify_tree([root], [-1], [0])
    logits, f = g.logits(1)[0], g.features(1)[0]
    assert (a, len(acc), nxt) == (0, 0, int(np.argmax(logits))) and g.argmax(1)[0] == nxt
    assert g.state() == (10, nxt) and [list(x) for x in g.kv_moves()] == [[0], [9]]
    ref = _f32(w["lm_head"]).astype(np.float64) @ f.astype(np.float64)
    # fp32: sums of 256 products; bf16: the head's input is the feature before its factor, rounded to 8 bits
    assert np.max(np.abs(logits - ref)) <= (1e-5 if dtype == "f32" else 2 ** -8) * np.max(np.abs(ref))
    g.close()


@pytest.mark.parametrize("vocab", [1000, 8193, 32001, 32771])
def test_equal_largest_logits(vocab):
    """Two rows of the head that are the same and larger than all others: the lower token is the choice; the last token alone is found too."""
    s, w, g = _session(vocab, "f32")
    root = g.prefill(fi.gen_prefix(1, 9, s.vocab))
    g.verify_tree([root], [-1], [0])
    row = g.features(1)[0]
    g.close()
    for tokens in ([vocab - 1], [0, vocab - 1], [vocab // 2, vocab // 2 + 1], [5, 4 * 256 + 5]):
        tokens = [t for t in tokens if t < vocab]

        def edit(head):
            head[tokens] = row
            return head
        s, w, g = _session(vocab, "f32", edit)
        root = g.prefill(fi.gen_prefix(1, 9, s.vocab))
        g.rollback(9, root)
        # the step's own token decides what its features are; the head's rows above are the features of the same step with the first head's token
        _, _, nxt = g.verify_tree([root], [-1], [0])
        logits = g.logits(1)[0]
        assert nxt == int(np.argmax(logits)) and (logits[tokens] == logits[tokens[0]]).all()
        g.close()


@pytest.mark.parametrize("vocab,token", [(1000, 999), (8193, 8192), (32001, 0), (32771, 32770)])
@pytest.mark.parametrize("nan", [False, True])     # a product that overflows, a NaN
def test_no_choice(vocab, token, nan):
    """One logit of the node is no number; the prompt before it has choices throughout."""
    s, w, g = _session(vocab, "bf16")
    g.init_weights(_overflows_behind(7, s, w, token, nan))
    g.prefill(fi.gen_prefix(1, 9, s.vocab) % 4)
    g.rollback(9, 7)
    with pytest.raises(Exception) as e:
        g.verify_tree([7], [-1], [0])
    assert e.value.status == -10 and g.argmax(1)[0] == -1 and g.state() == (9, 7)
    g.close()


@pytest.mark.parametrize("vocab,token", [(1000, 999), (8193, 8192), (32771, 5)])
def test_no_choice_in_the_step_itself(vocab, token):
    """A prompt whose choices are numbers, then a node whose embedding overflows."""
    s, w, g = _session(vocab, "bf16")
    w = dict(w, embed=w["embed"].copy())
    w["embed"][token] = 0x7FC0
    g.init_weights(w)
    g.prefill(fi.gen_prefix(1, 9, s.vocab) % 4)
    g.rollback(9, token)
    with pytest.raises(Exception) as e:
        g.verify_tree([token], [-1], [0])
    assert e.value.status == -10
    g.rollback(9, 1)
    a, _, nxt = g.verify_tree([1], [-1], [0])
    assert a == 0 and nxt == int(np.argmax(g.logits(1)[0]))
    g.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab,token", [(1000, 999), (8192, 0), (8193, 8192), (32001, 32000), (32768, 5), (32771, 32770)])
def test_features_stay_where_there_is_no_choice(vocab, token, dtype):
    """Features that a step exported are the last choice's until the next choice, as behind steps of more nodes."""
    import paper_2412_12639_amd as fv
    s, w, g = _session(vocab, dtype)
    for nan in (False, True):
        g.init_weights(_overflows_behind(7, s, w, token, nan))
        g.prefill(fi.gen_prefix(1, 9, s.vocab) % 4)
        g.rollback(9, 3)
        g.verify_tree([3], [-1], [0])
        at = fv.features_device_ptr(g) - g.arena.data_ptr()
        before = g.features(1)[0].copy()
        g.rollback(9, 7)
        with pytest.raises(Exception) as e:
            g.verify_tree([7], [-1], [0])
        assert e.value.status == -10
        assert np.array_equal(g.arena[at:at + 4 * s.hidden].cpu().numpy().view(np.float32), before)
        logits = g.logits(1)[0]
        assert np.isnan(logits[token]) if nan else np.isinf(logits[token])
        assert np.isfinite(np.delete(logits, token)).all()
        g.rollback(9, 3)
        g.verify_tree([3], [-1], [0])
        assert np.array_equal(g.features(1)[0], before)
    g.close()
