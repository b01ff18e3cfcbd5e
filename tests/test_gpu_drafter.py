"""Drafting phase on the GPU against oracle/drafter_oracle.py, through the C ABI.

Every phase row's predicted feature and logits are compared element by element; the integer work
(top lists, the tokens of the tree) is checked bit-exactly: a top list must be the oracle's top_m
applied to the device's own logits (the decision taken in the device's precision), and the tree's
tokens must be those lists expanded by the oracle's structure function.  The oracle runs its later
passes on the device's tokens, so that a near-tie cannot make the two sides drift apart."""
import numpy as np
import pytest

from fv_inputs.shapes import shape_by_name
from fv_inputs.trees import gen_tree, sibling_ranks
from fv_inputs.weights import gen_drafter_weights, gen_features, gen_weights, sub_model
from oracle import drafter_oracle as do

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)


def _make(shape_name, k, max_seq=160, seed=21, layers=None):
    import torch
    from paper_2412_12639_amd.binding import FalconDrafter, FalconVerifier
    s = shape_by_name(shape_name)
    if layers is not None:
        s = s.with_layers(layers)
    lw = gen_weights(s, seed=seed, gain_jitter=0.1)
    dw = gen_drafter_weights(s, seed=seed + 1, gain_jitter=0.1)
    tgt = FalconVerifier(s, max_seq, 64)
    tgt.init_weights(lw)
    dr = FalconDrafter(tgt, k)
    dr.init_weights(dw)
    return s, lw, dw, tgt, dr


def _oracle_weights(w):
    """bf16 bit patterns widened to fp32 once (exact), so that the oracle does not widen per product."""
    return {n: ((a.astype(np.uint32) << 16).view(np.float32) if a.dtype == np.uint16 else a) for n, a in w.items()}


def _rel(a, b):
    return float(np.max(np.abs(a - b)) / max(1e-30, np.max(np.abs(b))))


def _tol_of_pass(tol, p):
    """Rows of pass p (the commit's rows are pass 0) are computed from the outputs of pass p - 1: its predicted
    features and its LSTM states, two channels that carry the same rounding errors, so the errors of successive
    passes add up rather than average out (measured at the 7B width: 0.5e-2 of the largest logit per pass).
    The 2e-2 bar is kept for the commit's rows and the first tree pass and widened by 1e-2 per further pass
    (bf16 builds only; fp32 builds keep their flat tolerance)."""
    return tol if tol < 1e-3 else tol * max(1.0, (p + 1) / 2)


def _check_phase(s, dr, orc, n_chain, tokens_dev, parent, depth, rank, tol):
    """Rows of the open phase: features, logits, top lists, tree tokens."""
    _, n_rows, chain = dr.state()
    assert chain == n_chain and n_rows == len(orc.phase["f"])
    f_dev, l_dev = dr.rows("features", 0, n_rows), dr.rows("logits", 0, n_rows)
    f_ref, l_ref = np.array(orc.phase["f"]), np.array(orc.phase["logits"])
    pass_of = np.zeros(n_rows, dtype=int)
    if parent is not None:
        for bi, (a, _) in enumerate(orc.blocks):
            if bi > 0:
                pass_of[orc.rows_of[bi]] = depth[a] // orc.k
    for p in range(int(pass_of.max()) + 1):
        rows = np.nonzero(pass_of == p)[0]
        ef, el = _rel(f_dev[rows], f_ref[rows]), _rel(l_dev[rows], l_ref[rows])
        say(f"    pass {p}: {len(rows)} rows, features rel err {ef:.2e}, logits rel err {el:.2e} (tol {_tol_of_pass(tol, p):.2g})")
        assert ef <= _tol_of_pass(tol, p) and el <= _tol_of_pass(tol, p)
    tops = dr.top(0, n_rows)
    for r in range(n_rows):
        np.testing.assert_array_equal(tops[r], do.top_m(l_dev[r], tops.shape[1]), err_msg=f"top list of row {r}")
    if parent is None:
        return
    # the tree's tokens: the lists expanded by the oracle's structure function (history rows: the last k committed rows)
    blocks, gen = do.sar_structure(parent, depth, orc.k)
    hist = dr.top(256, orc.k)   # history slots (valid for the k-1 first ones)
    for i in range(1, len(parent)):
        bi, j = gen[i]
        if bi == 0:
            c = n_chain - 1 + j
            lst = hist[c] if c < orc.k - 1 else tops[c - (orc.k - 1)]
        else:
            lst = tops[orc.rows_of[bi][j]]
        assert tokens_dev[i] == lst[rank[i]], f"node {i}"


CASES = [("tiny", 2, 1e-4), ("tiny", 3, 1e-4), ("tiny", 1, 1e-4), ("tiny-bf16", 2, 2e-2), ("small-gqa", 2, 2e-2),
         ("small-gqa-f32", 4, 1e-4)]


@pytest.mark.parametrize("shape_name,k,tol", CASES)
def test_drafting_phases_elementwise(shape_name, k, tol):
    import torch
    s, lw, dw, tgt, dr = _make(shape_name, k)
    orc = do.DrafterOracle(s, lw, dw, k, 160)
    rng = np.random.default_rng(5)
    trees = [gen_tree(31, 40, [4, 3, 2, 2, 1, 1], 6), gen_tree(32, 25, [5, 2, 2, 1, 1, 1, 1, 1], 8), gen_tree(33, 12, [3, 2, 1], 3)]
    hist_ref = []                                           # top lists of all committed rows so far (oracle side, from device logits)
    for phase, (n_new, tree) in enumerate(zip([7, 1, 3], trees)):
        say(f"  {shape_name} k={k} phase {phase}: commit {n_new} pairs")
        feats = gen_features(100 + phase, n_new, s.hidden)
        toks = rng.integers(0, s.vocab, n_new)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        orc.commit(feats, toks)
        _check_phase(s, dr, orc, n_new, None, None, None, None, tol)
        kd, vd = dr.read_kv(orc.L - n_new, n_new)
        assert _rel(kd, orc.K[orc.L - n_new:orc.L]) <= tol and _rel(vd, orc.V[orc.L - n_new:orc.L]) <= tol
        parent, depth, _ = tree
        rank = sibling_ranks(parent)
        tokens_dev = dr.draft_tree(parent, depth, rank, int(toks[-1]))
        tokens_ref = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=tokens_dev)
        _check_phase(s, dr, orc, n_new, tokens_dev, parent, depth, rank, tol)
        # where the oracle's own pick is clear of its neighbours by more than the tolerance, it is the device's pick
        agree = int(np.sum(tokens_dev == tokens_ref))
        say(f"    tree of {len(parent)} nodes: {agree} tokens equal the oracle's own picks")
        assert tokens_dev[0] == toks[-1]
        assert agree >= len(parent) - 2
    dr.close()
    tgt.close()


def test_wide_pass_and_degenerate_trees():
    """A pass of more than 64 rows (the shared-activation GEMM kernel and its separate reduction launch),
    a tree no deeper than k (no pass at all: the commit's rows give every token) and the one-node tree."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny", 2, max_seq=400)
    orc = do.DrafterOracle(s, lw, dw, 2, 400)
    rng = np.random.default_rng(6)
    shapes = [gen_tree(41, 205, [4, 10, 2, 1], 0), gen_tree(42, 9, [4, 1], 2), (np.array([-1]), np.array([0]), None)]
    for phase, (n_new, tree) in enumerate(zip([4, 2, 1], shapes)):
        feats = gen_features(200 + phase, n_new, s.hidden)
        toks = rng.integers(0, s.vocab, n_new)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        orc.commit(feats, toks)
        parent, depth, _ = tree
        rank = sibling_ranks(parent)
        got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
        want = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
        say(f"  tree of {len(parent)} nodes: phase rows {dr.state()[1]}")
        _check_phase(s, dr, orc, n_new, got, parent, depth, rank, 1e-4)
        np.testing.assert_array_equal(got, want)
        if phase == 0:
            assert dr.state()[1] - n_new > 64
    dr.close()
    tgt.close()


def test_benchmark_width_drafter_rows():
    """The 7B width (hidden 4096, 32 heads, FFN 11008, vocabulary 32000) with k = 2 and a 64-node tree of
    depth 8: what the benchmark times.  The oracle runs in fp32 on weights widened once."""
    import torch
    s, lw, dw, tgt, dr = _make("7b", 2, max_seq=256, layers=1)
    orc = do.DrafterOracle(s, _oracle_weights(lw), _oracle_weights(dw), 2, 256, dtype=np.float32)
    rng = np.random.default_rng(9)
    trees = [gen_tree(51, 64, [8, 4, 2, 2, 1, 1, 1, 1], 8), gen_tree(52, 64, [6, 3, 2, 2, 2, 1, 1, 1], 8)]
    for phase, (n_new, tree) in enumerate(zip([5, 2], trees)):
        feats = gen_features(300 + phase, n_new, s.hidden)
        toks = rng.integers(0, s.vocab, n_new)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        say(f"  7b phase {phase}: commit {n_new} pairs {dr.last_ms():.3f} ms")
        orc.commit(feats, toks)
        parent, depth, _ = tree
        rank = sibling_ranks(parent)
        got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
        say(f"    tree: {dr.state()[1] - n_new} rows in {int(max(depth) + 1) // 2 - 1} passes, {dr.last_ms():.3f} ms")
        want = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
        _check_phase(s, dr, orc, n_new, got, parent, depth, rank, 2e-2)
        say(f"    {int(np.sum(got == want))} of {len(parent)} tokens equal the oracle's own picks")
        assert int(np.sum(got == want)) >= len(parent) - 3
    dr.close()
    tgt.close()


@pytest.mark.parametrize("head", ["ties", "zero"])
def test_top_lists_with_equal_logits(head):
    """Equal logits are ordered by token id: three LM-head rows made identical (and large, so that they
    often make the list), and an all-zero head (every logit equal: the list is 0, 1, 2, ...)."""
    import torch
    from paper_2412_12639_amd.binding import FalconDrafter, FalconVerifier
    s = shape_by_name("tiny")
    lw = gen_weights(s, seed=2)
    lw["lm_head"] = lw["lm_head"].copy()
    if head == "ties":
        lw["lm_head"][[100, 300]] = lw["lm_head"][7]
        lw["lm_head"][[7, 100, 300]] *= 6.0
    else:
        lw["lm_head"][:] = 0.0
    dw = gen_drafter_weights(s, seed=3)
    tgt = FalconVerifier(s, 64, 64)
    tgt.init_weights(lw)
    dr = FalconDrafter(tgt, 2)
    dr.init_weights(dw)
    feats = gen_features(4, 9, s.hidden)
    toks = np.random.default_rng(4).integers(0, s.vocab, 9)
    dr.commit(toks, torch.from_numpy(feats).cuda())
    logits, tops = dr.rows("logits", 0, 9), dr.top(0, 9)
    for r in range(9):
        np.testing.assert_array_equal(tops[r], do.top_m(logits[r], 32))
        if head == "zero":
            assert list(tops[r]) == list(range(32))
        else:
            assert logits[r][7] == logits[r][100] == logits[r][300]
            lst = tops[r].tolist()
            if 7 in lst and lst.index(7) + 2 < len(lst):     # the three equal logits are neighbours, in id order
                assert lst[lst.index(7):lst.index(7) + 3] == [7, 100, 300]
    parent, depth, _ = gen_tree(3, 20, [6, 3, 1], 0)
    got = dr.draft_tree(parent, depth, sibling_ranks(parent), int(toks[-1]))
    if head == "zero":
        np.testing.assert_array_equal(got[1:], sibling_ranks(parent)[1:])   # rank r takes token r everywhere
    dr.close()
    tgt.close()


def test_long_commit_in_pieces_and_errors():
    import torch
    from paper_2412_12639_amd.binding import FvError
    s, lw, dw, tgt, dr = _make("tiny", 2, max_seq=256)
    orc = do.DrafterOracle(s, lw, dw, 2, 256)
    n = 150                                                  # three pieces: 64 + 64 + 22
    feats = gen_features(7, n, s.hidden)
    toks = np.random.default_rng(8).integers(0, s.vocab, n)
    dr.commit(toks, torch.from_numpy(feats).cuda())
    _, l_ref = orc.commit(feats, toks)
    committed, n_rows, chain = dr.state()
    assert committed == n and chain == 22
    assert _rel(dr.rows("logits", 0, 22), l_ref[-22:]) <= 1e-4
    kd, vd = dr.read_kv(0, n)
    assert _rel(kd, orc.K[:n]) <= 1e-4 and _rel(vd, orc.V[:n]) <= 1e-4
    parent, depth, _ = gen_tree(3, 20, [3, 2, 2, 1], 4)
    rank = sibling_ranks(parent)
    with pytest.raises(FvError) as e:                        # rank beyond the list
        dr.draft_tree(parent, depth, np.full(20, 40), int(toks[-1]))
    assert e.value.status == -1
    with pytest.raises(FvError) as e:                        # a tree that is no tree
        dr.draft_tree(np.array([-1, 1, 0]), np.array([0, 1, 1]), np.zeros(3), int(toks[-1]))
    assert e.value.status == -2
    got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
    want = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
    assert int(np.sum(got == want)) >= 19
    with pytest.raises(FvError) as e:                        # one tree per phase
        dr.draft_tree(parent, depth, rank, int(toks[-1]))
    assert e.value.status == -8
    dr.reset()
    with pytest.raises(FvError) as e:                        # no committed pairs
        dr.draft_tree(parent, depth, rank, 1)
    assert e.value.status == -8
    dr.commit(toks[:1], torch.from_numpy(feats[:1]).cuda())
    with pytest.raises(FvError) as e:                        # fewer than k committed pairs
        dr.draft_tree(parent, depth, rank, int(toks[0]))
    assert e.value.status == -8
    dr.close()
    tgt.close()


def test_drafted_tree_goes_through_verification():
    """The drafted tokens are a valid tree for the verification step, fed by the features it exports."""
    import torch
    from paper_2412_12639_amd.binding import features_device_ptr
    s, lw, dw, tgt, dr = _make("small-gqa", 2, max_seq=200)
    prompt = np.random.default_rng(3).integers(0, s.vocab, 12)
    root = tgt.prefill(prompt)
    # stand-in features for the prompt pairs (the prefill does not export them); afterwards the real ones
    feats = gen_features(9, len(prompt), s.hidden)
    dr.commit(np.concatenate([prompt[1:], [root]]), torch.from_numpy(feats).cuda())
    parent, depth, _ = gen_tree(5, 30, [4, 2, 2, 1, 1, 1], 6)
    rank = sibling_ranks(parent)
    for step in range(3):
        tokens = dr.draft_tree(parent, depth, rank, root)
        a, acc, nxt = tgt.verify_tree(tokens, parent, depth)
        say(f"  step {step}: accepted {a}")
        new = list(acc[:a]) + [nxt]
        dr.commit(new, features_device_ptr(tgt))
        root = nxt
        assert dr.state()[0] == tgt.state()[0]
    dr.close()
    tgt.close()


def _lstm_oracle(s, lw, dw, k, max_seq):
    """The oracle in fp64; at wide hidden sizes in fp32 on matrices widened once (its error there is 1e-6, the bar 2e-2)."""
    if s.hidden <= 1024:
        return do.DrafterOracle(s, lw, dw, k, max_seq)
    return do.DrafterOracle(s, _oracle_weights(lw), _oracle_weights(dw), k, max_seq, dtype=np.float32)


# every built size of the kernels (2, 4, 8, 16 and 32 fragments a wavefront); 384 and 2560 do not fill theirs, and at 2560 and 4096 a
# quarter of the fragments is in LDS
@pytest.mark.parametrize("hidden,give_up", [(h, g) for g in (False, True) for h in (256, 384, 512, 1024)] + [(2048, False), (2560, False), (4096, False)])
def test_chain_launches(hidden, give_up, monkeypatch):
    """Commits whose rows go through the LSTM in one launch per layer: two rows (the shortest), an odd count, a whole piece and
    one row more (the second piece is a single row), at hidden sizes that fill a built kernel and some that do not.
    give_up: the launches' workgroups wait for one that does not exist and leave; the separate launches must take over and the
    call must not show it.  The launch counts say which of the two computed the rows."""
    import torch
    from dataclasses import replace
    from paper_2412_12639_amd.binding import FalconDrafter, FalconVerifier
    if give_up:
        monkeypatch.setenv("FV_EXCHANGE_TEST", "chain")
    s = replace(shape_by_name("tiny-bf16"), name=f"tiny-bf16-h{hidden}", hidden=hidden)
    lw, dw = gen_weights(s, seed=61, gain_jitter=0.1), gen_drafter_weights(s, seed=62, gain_jitter=0.1)
    tgt = FalconVerifier(s, 200, 64)
    tgt.init_weights(lw)
    dr = FalconDrafter(tgt, 2)
    dr.init_weights(dw)
    orc = _lstm_oracle(s, lw, dw, 2, 200)
    passes = 0
    for n in (2, 7, 65, 64, 1) if hidden <= 1024 else (2, 65):
        feats = gen_features(400 + n, n, s.hidden)
        toks = np.random.default_rng(n).integers(0, s.vocab, n)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        f_ref, l_ref = orc.commit(feats, toks)
        rows = dr.state()[2]
        assert rows == (n - 1) % 64 + 1
        ef, el = _rel(dr.rows("features", 0, rows), f_ref[-rows:]), _rel(dr.rows("logits", 0, rows), l_ref[-rows:])
        kd, vd = dr.read_kv(orc.L - n, n)
        ek, ev = _rel(kd, orc.K[orc.L - n:orc.L]), _rel(vd, orc.V[orc.L - n:orc.L])
        say(f"  hidden {hidden}, {n} pairs: features {ef:.2e}, logits {el:.2e}, k {ek:.2e}, v {ev:.2e}")
        assert max(ef, el, ek, ev) <= 2e-2       # the bar of every bf16 commit above: the same formats, other sums
        passes += n > 1                          # of 65 pairs the first 64 are one pass, the last one has a single row
        # after a give-up (which the second layer's launch does not wait for again) the next 16 calls go without
        assert dr.launches() == ((2, 1) if give_up else (2 * passes, 0))
    feats = np.full((3, s.hidden), 1.0, dtype=np.float32)
    feats[1, 5] = np.nan                         # a state that is no number goes through the exchange as one
    with pytest.raises(Exception) as e:
        dr.commit([1, 2, 3], torch.from_numpy(feats).cuda())
    assert e.value.status == -10
    dr.close()
    tgt.close()


@pytest.mark.parametrize("hidden,k,give_up", [(256, 4, False), (384, 3, False), (512, 4, True), (1024, 5, False), (2048, 4, False), (2560, 3, False)])
def test_level_launches(hidden, k, give_up, monkeypatch):
    """Tree passes whose LSTM levels run in one launch per layer: three to five levels (the exchange buffers and their phase are used
    again from the third on), blocks that drop out on the way, up to sixteen blocks and more (which go level by level)."""
    import torch
    from dataclasses import replace
    from paper_2412_12639_amd.binding import FalconDrafter, FalconVerifier
    if give_up:
        monkeypatch.setenv("FV_EXCHANGE_TEST", "chain")
    s = replace(shape_by_name("tiny-bf16"), name=f"tiny-bf16-h{hidden}", hidden=hidden)
    lw, dw = gen_weights(s, seed=71, gain_jitter=0.1), gen_drafter_weights(s, seed=72, gain_jitter=0.1)
    tgt = FalconVerifier(s, 300, 64)
    tgt.init_weights(lw)
    dr = FalconDrafter(tgt, k)
    dr.init_weights(dw)
    orc = _lstm_oracle(s, lw, dw, k, 300)
    rng = np.random.default_rng(hidden)
    trees = [gen_tree(81, 40, [3, 2, 1, 1, 2, 1, 1, 1, 1, 1, 1, 1], 12), gen_tree(82, 90, [6, 4, 1, 1, 1, 1, 1, 1, 1], 9), gen_tree(83, 14, [1] * 13, 13)]
    if give_up:   # single rows take no such launch: the first tree is the one that gives up
        for i in range(k):
            feats = gen_features(600 + i, 1, s.hidden)
            dr.commit([i], torch.from_numpy(feats).cuda())
            orc.commit(feats, [i])
    for phase, (n_new, tree) in enumerate(zip([1 if give_up else k + 1, 2, 1], trees)):
        feats = gen_features(500 + phase, n_new, s.hidden)
        toks = rng.integers(0, s.vocab, n_new)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        orc.commit(feats, toks)
        parent, depth, _ = tree
        rank = sibling_ranks(parent)
        before = dr.launches()
        got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
        taken, gave_up = (b - a for a, b in zip(before, dr.launches()))
        # (the second tree is too wide in all passes for some k; a tree that gives up waits in vain once, the ones behind it go without)
        assert (gave_up == 1 and taken >= 2 if phase == 0 else taken == 0) if give_up else (gave_up == 0 and (taken > 0 or phase == 1))
        orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
        _check_phase(s, dr, orc, n_new, got, parent, depth, rank, 2e-2)
    dr.close()
    tgt.close()


def test_give_up_makes_the_next_calls_go_without(monkeypatch):
    """One time-out, then 16 calls without one-launch passes, then one attempt, then 32 calls without: a long commit after a
    give-up does not try again in its later pieces either."""
    import torch
    monkeypatch.setenv("FV_EXCHANGE_TEST", "chain")
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=700)
    commit = lambda n: dr.commit(np.arange(n), torch.from_numpy(gen_features(n, n, s.hidden)).cuda())
    commit(330)                                   # pieces of 256, 64 and 10 rows
    assert dr.launches() == (2, 1)
    parent, depth, _ = gen_tree(83, 14, [1] * 13, 13)
    for i in range(16):
        if i % 4 == 3:
            dr.draft_tree(parent, depth, sibling_ranks(parent), 1)
        else:
            commit(2)
        assert dr.launches() == (2, 1)
    commit(2)
    assert dr.launches() == (4, 2)
    for _ in range(32):
        commit(2)
    assert dr.launches() == (4, 2)
    commit(2)
    assert dr.launches() == (6, 3)
    dr.close()
    tgt.close()


@pytest.mark.parametrize("n,stay", [
    (400, 0),       # the only wide pass leaves
    (1300, 2),      # the second of two, whose rows continue what the first left
])
def test_wide_pass_that_leaves(n, stay, monkeypatch):
    """Chain launches give up in a wide pass: its rows go in pieces, and nothing of it shows in state, outputs, K and V, a tree or a further commit."""
    import torch
    monkeypatch.setenv("FV_EXCHANGE_TEST", f"chain:{stay}")
    s, lw, dw, tgt, dr = _make("tiny-bf16", 3, max_seq=1400)
    orc = do.DrafterOracle(s, lw, dw, 3, 1400)
    parent, depth, _ = gen_tree(31, 30, [4, 2, 2, 1, 1, 1, 1, 1, 1, 1], 9)
    rank = sibling_ranks(parent)
    for rows in (n, 5):
        feats = gen_features(rows, rows, s.hidden)
        toks = np.random.default_rng(rows).integers(0, s.vocab, rows)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        orc.commit(feats, toks)
        assert dr.launches() == (stay + 2, 1)
        tail = (rows - 1) % 64 + 1
        assert dr.state() == (orc.L, tail, tail)
        f_ref, l_ref = np.array(orc.phase["f"]), np.array(orc.phase["logits"])
        assert _rel(dr.rows("features", 0, tail), f_ref[-tail:]) <= 2e-2 and _rel(dr.rows("logits", 0, tail), l_ref[-tail:]) <= 2e-2
        kd, vd = dr.read_kv(0, orc.L)
        assert _rel(kd, orc.K[:orc.L]) <= 2e-2 and _rel(vd, orc.V[:orc.L]) <= 2e-2
        got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
        ref = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
        assert sum(got[i] != ref[i] for i in range(len(parent)) if depth[i] <= 3) <= 1
    dr.close()
    tgt.close()


def test_wide_pass_that_leaves_behind_one_that_was_no_numbers(monkeypatch):
    """A wide pass that leaves runs its block on what the wide pass before it kept as states, here NaNs; the pieces that follow end inside a block of 32
    keys and must not read what that made of the slots behind them."""
    import torch
    monkeypatch.setenv("FV_EXCHANGE_TEST", "chain:6")      # two launches each: a wide pass, its first piece, three pairs
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=500)
    orc = do.DrafterOracle(s, lw, dw, 2, 500)
    bad = gen_features(1, 400, s.hidden)
    bad[5, 5] = np.nan
    with pytest.raises(Exception) as e:
        dr.commit(np.arange(400), torch.from_numpy(bad).cuda())
    assert e.value.status == -10 and dr.launches() == (4, 0)
    dr.reset()
    for n in (3, 400):
        feats = gen_features(n, n, s.hidden)
        toks = np.random.default_rng(n).integers(0, s.vocab, n)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        orc.commit(feats, toks)
    assert dr.launches() == (8, 1) and dr.state() == (403, 16, 16)
    f_ref, l_ref = np.array(orc.phase["f"]), np.array(orc.phase["logits"])
    assert _rel(dr.rows("features", 0, 16), f_ref[-16:]) <= 2e-2 and _rel(dr.rows("logits", 0, 16), l_ref[-16:]) <= 2e-2
    kd, vd = dr.read_kv(0, 403)
    assert _rel(kd, orc.K[:403]) <= 2e-2 and _rel(vd, orc.V[:403]) <= 2e-2
    dr.close()
    tgt.close()


def test_tree_that_leaves_behind_a_commit_that_was_no_numbers(monkeypatch):
    """Tree passes of 20 rows whose level launches leave run their block on what is left of the residual stream, here a failed commit's NaNs in rows that
    the commit behind it (of fewer rows) did not write.  The passes run again and must not read what that made of the later passes' slots."""
    import torch
    monkeypatch.setenv("FV_EXCHANGE_TEST", "chain:4")      # two launches each: the failed commit, four pairs
    s, lw, dw, tgt, dr = _make("tiny-bf16", 4, max_seq=300)
    orc = do.DrafterOracle(s, lw, dw, 4, 300)
    bad = gen_features(1, 20, s.hidden)
    bad[0, 5] = np.nan
    with pytest.raises(Exception) as e:
        dr.commit(np.arange(20), torch.from_numpy(bad).cuda())
    assert e.value.status == -10
    dr.reset()
    feats = gen_features(2, 4, s.hidden)
    toks = np.random.default_rng(2).integers(0, s.vocab, 4)
    dr.commit(toks, torch.from_numpy(feats).cuda())
    orc.commit(feats, toks)
    assert dr.launches() == (4, 0)
    parent, depth = [-1], [0]                               # five paths of twelve nodes
    for _ in range(5):
        for j in range(12):
            parent.append(len(parent) - 1 if j else 0)
            depth.append(j + 1)
    parent, depth = np.array(parent), np.array(depth)
    rank = sibling_ranks(parent)
    got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
    assert dr.launches()[1] == 1
    orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
    _check_phase(s, dr, orc, 4, got, parent, depth, rank, 2e-2)
    dr.close()
    tgt.close()


def test_long_bf16_commit_in_wide_pieces():
    """300 pairs: 256 rows in one piece (the ring GEMM and the chain launch over 256 rows), then the 44 that stay open."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=400)
    orc = do.DrafterOracle(s, lw, dw, 2, 400)
    n = 300
    feats = gen_features(7, n, s.hidden)
    toks = np.random.default_rng(8).integers(0, s.vocab, n)
    dr.commit(toks, torch.from_numpy(feats).cuda())
    _, l_ref = orc.commit(feats, toks)
    assert dr.state() == (n, 44, 44)
    assert _rel(dr.rows("logits", 0, 44), l_ref[-44:]) <= 2e-2
    kd, vd = dr.read_kv(0, n)
    assert _rel(kd, orc.K[:n]) <= 2e-2 and _rel(vd, orc.V[:n]) <= 2e-2
    dr.close()
    tgt.close()


@pytest.mark.parametrize("n,k", [
    (68, 4),     # four rows stay open: all that the first level of the tree comes from
    (67, 4),     # three: its first row comes from the last row of the piece before
    (325, 5),    # three pieces, the open one just long enough
])
def test_tree_behind_a_commit_in_pieces(n, k):
    """The tree drafted behind a long commit, at the number of open rows where the piece before stops being read."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", k, max_seq=400)
    orc = do.DrafterOracle(s, lw, dw, k, 400)
    feats = gen_features(n, n, s.hidden)
    toks = np.random.default_rng(n).integers(0, s.vocab, n)
    dr.commit(toks, torch.from_numpy(feats).cuda())
    orc.commit(feats, toks)
    tail = (n - 1) % 64 + 1
    assert dr.state() == (n, tail, tail)
    f_ref, l_ref = np.array(orc.phase["f"]), np.array(orc.phase["logits"])
    assert _rel(dr.rows("features", 0, tail), f_ref[-tail:]) <= 2e-2 and _rel(dr.rows("logits", 0, tail), l_ref[-tail:]) <= 2e-2
    kd, vd = dr.read_kv(0, n)
    assert _rel(kd, orc.K[:n]) <= 2e-2 and _rel(vd, orc.V[:n]) <= 2e-2
    parent, depth, _ = gen_tree(31, 40, [4, 3, 2, 2, 1, 1], 6)
    rank = sibling_ranks(parent)
    got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
    ref = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
    first = [i for i in range(len(parent)) if depth[i] <= k]     # what the committed rows' lists give
    assert sum(got[i] != ref[i] for i in first) <= 1             # a near-tie at most
    dr.close()
    tgt.close()


@pytest.mark.parametrize("n,k", [
    (65, 8),      # one pass of which a single row stays open; the rows in front of it are the history of the first levels
    (128, 8),     # the history lies in rows that the open ones move over
    (256, 1),     # the longest pass of its kind, no history
    (257, 8),     # the shortest wide pass, a single open row
    (1024, 3),    # the longest, 64 open rows
    (1089, 2),    # a wide pass, one of 65 rows behind it
    (1300, 4),    # two wide passes
])
def test_commits_of_more_rows_than_stay_open(n, k):
    """Commits whose open rows are the last of a pass that others precede: state, outputs of the open rows, K and V of all, and a tree, whose first k levels
    come from the last k rows.  A second phase continues the LSTM states that were kept."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", k, max_seq=1400)
    orc = do.DrafterOracle(s, lw, dw, k, 1400)
    parent, depth, _ = gen_tree(31, 30, [4, 2, 2, 1, 1, 1, 1, 1, 1, 1], 9)
    rank = sibling_ranks(parent)
    for rows in (n, 3):
        feats = gen_features(rows + k, rows, s.hidden)
        toks = np.random.default_rng(rows).integers(0, s.vocab, rows)
        dr.commit(toks, torch.from_numpy(feats).cuda())
        orc.commit(feats, toks)
        tail = (rows - 1) % 64 + 1
        assert dr.state() == (orc.L, tail, tail)
        f_ref, l_ref = np.array(orc.phase["f"]), np.array(orc.phase["logits"])
        assert _rel(dr.rows("features", 0, tail), f_ref[-tail:]) <= 2e-2 and _rel(dr.rows("logits", 0, tail), l_ref[-tail:]) <= 2e-2
        kd, vd = dr.read_kv(0, orc.L)
        assert _rel(kd, orc.K[:orc.L]) <= 2e-2 and _rel(vd, orc.V[:orc.L]) <= 2e-2
        got = dr.draft_tree(parent, depth, rank, int(toks[-1]))
        ref = orc.draft(parent, depth, rank, int(toks[-1]), force_tokens=got)
        first = [i for i in range(len(parent)) if depth[i] <= k]
        assert sum(got[i] != ref[i] for i in first) <= 1
    dr.close()
    tgt.close()


@pytest.mark.parametrize("n,row,committed", [
    (100, 5, 64),       # the piece of 64 rows in front of the open ones
    (100, 70, 100),     # an open one
    (400, 5, 256),      # a wide pass: the first piece of 256, ..
    (400, 300, 384),    # .. the 128 rows between it and the open ones
])
def test_a_value_that_is_no_number_ends_the_piece_it_lies_in(n, row, committed):
    """Passes with rows in front of the open ones that turn out to hold a NaN: pairs count as committed up to the end of the piece that has it, pieces
    being 256 rows, then what is left before the open ones."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=500)
    feats = gen_features(n, n, s.hidden)
    feats[row, 5] = np.nan
    with pytest.raises(Exception) as e:
        dr.commit(np.arange(n), torch.from_numpy(feats).cuda())
    assert e.value.status == -10 and dr.state()[0] == committed
    dr.close()
    tgt.close()


def _one_token_that_overflows(s, lw, dw):
    """Weights whose logit of token 17 is infinite, from finite states, K and V, in rows whose feature has a one at place 0: eight units that are zero
    but for it, and a row of the head that is 3e38 there."""
    h, units = s.hidden, np.arange(8)

    def put(w, key, rows, row_of):
        a = w[key].copy() if w[key].dtype != np.uint16 else (w[key].astype(np.uint32) << 16).view(np.float32)
        for r, u in zip(rows, units):
            a[r] = row_of(u, a.shape[1])
        w[key] = a if w[key].dtype != np.uint16 else (a.view(np.uint32) >> 16).astype(np.uint16)   # (the values put are exact in bf16)

    def zero(u, n):
        return np.zeros(n, dtype=np.float32)

    def only(col):
        def row(u, n):
            v = zero(u, n)
            v[col(u)] = 8.0
            return v
        return row

    for layer, col in ((0, lambda u: 0), (1, lambda u: u)):
        b = dw[f"lstm{layer}.b"].copy()
        for gate, bias in ((0, 10.0), (1, -100.0), (2, 0.0), (3, 10.0)):   # in and out open, nothing kept, candidate from one input
            b[gate * h + units] = bias
            put(dw, f"lstm{layer}.w_ih", gate * h + units, only(col) if gate == 2 else zero)
            put(dw, f"lstm{layer}.w_hh", gate * h + units, zero)
        dw[f"lstm{layer}.b"] = b
    put(dw, "d.wo", units, zero)
    put(dw, "d.wd", units, zero)
    head = lw["lm_head"].copy()
    head[17] = 0
    head[17, units] = 0x7F60 if head.dtype == np.uint16 else 2.9774e38
    lw["lm_head"] = head


@pytest.mark.parametrize("n,row,committed", [
    (100, 70, 100),     # the 64 rows in front of the open ones have none
    (100, 5, 64),
    (400, 260, 384),    # a wide pass: neither has the first piece of 256
    (400, 390, 400),
])
def test_pieces_in_front_of_one_that_is_no_number_end_between_key_blocks(n, row, committed):
    """The same behind three committed pairs: a piece ends inside a block of 32 keys, whose other slots must not hold what the big pass left there."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=500)
    dr.commit([1, 2, 3], torch.from_numpy(gen_features(1, 3, s.hidden)).cuda())
    feats = gen_features(n, n, s.hidden)
    feats[row, 5] = np.nan
    with pytest.raises(Exception) as e:
        dr.commit(np.arange(n), torch.from_numpy(feats).cuda())
    assert e.value.status == -10 and dr.state()[0] == 3 + committed
    dr.close()
    tgt.close()


@pytest.mark.parametrize("n,late", [(200, 195), (400, 270)])     # one pass of up to 256 rows, a wide one
def test_what_a_failed_commit_leaves_behind_its_pairs_is_not_read(n, late):
    """Infinite logits in the fourth pair (its K, V and states are finite) and a NaN in a later piece: the call ends with the first piece.  A caller that
    goes on without a reset gets bit for bit what it would have got without the NaN, which lay behind the committed pairs."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=500)
    from paper_2412_12639_amd.binding import FalconDrafter
    _one_token_that_overflows(s, lw, dw)
    tgt.init_weights(lw)
    other = FalconDrafter(tgt, 2)
    toks = np.random.default_rng(4).integers(0, s.vocab, n)
    more = gen_features(5, 4, s.hidden)
    more[:, 0] = 0.0
    rows = []
    for d, value in ((dr, np.nan), (other, 0.25)):
        d.init_weights(dw)
        feats = gen_features(4, n, s.hidden)
        feats[:, 0] = 0.0
        feats[3, 0] = 1.0
        feats[late, 5] = value
        with pytest.raises(Exception) as e:
            d.commit(toks, torch.from_numpy(feats).cuda())
        first = min(256, (n - 1) // 64 * 64)
        assert e.value.status == -10 and d.state()[0] == first
        d.commit(toks[:4], torch.from_numpy(more).cuda())
        assert d.state() == (first + 4, 4, 4)
        rows.append((d.rows("logits", 0, 4), d.rows("features", 0, 4)) + d.read_kv(first, 4))
    for a, b in zip(*rows):
        assert np.isfinite(a).all() and np.array_equal(a, b)
    for d in (dr, other, tgt):
        d.close()


@pytest.mark.parametrize("name", ["tiny-bf16", "tiny"])
def test_overflow_of_an_early_rows_logits_is_reported(name):
    """200 pairs of which the fourth alone has infinite logits, from finite states, K and V: eight units that are zero but for it, and a row
    of the head that is 3e38 there.  Nothing behind that row shows it, so it is found only if every row of every piece goes
    through block and head."""
    import torch
    s, lw, dw, tgt, dr = _make(name, 2, max_seq=300)
    _one_token_that_overflows(s, lw, dw)
    tgt.init_weights(lw)
    dr.init_weights(dw)
    feats = gen_features(4, 200, s.hidden)
    feats[:, 0] = 0.0
    toks = np.random.default_rng(4).integers(0, s.vocab, 200)
    dr.commit(toks, torch.from_numpy(feats).cuda())
    assert dr.state() == (200, 8, 8) and np.all(dr.rows("logits", 0, 8)[:, 17] == 0.0)
    dr.reset()
    feats[3, 0] = 1.0
    with pytest.raises(Exception) as e:
        dr.commit(toks, torch.from_numpy(feats).cuda())
    assert e.value.status == -10
    dr.close()
    tgt.close()


def test_reset_after_a_commit_that_was_no_numbers():
    """200 pairs with a NaN among them leave NaNs in the cache and, 256 rows wide, in the block's activations, where the padding of its
    FFN's K range (688 to 768) lies for 64 and 32 rows.  After a reset the drafter is bitwise a new one: a commit, a tree behind it."""
    import torch
    s, lw, dw, tgt, dr = _make("tiny-bf16", 2, max_seq=300)
    from paper_2412_12639_amd.binding import FalconDrafter
    fresh = FalconDrafter(tgt, 2)
    fresh.init_weights(dw)
    bad = gen_features(1, 200, s.hidden)
    bad[3, 5] = np.nan
    with pytest.raises(Exception) as e:
        dr.commit(np.arange(200), torch.from_numpy(bad).cuda())
    assert e.value.status == -10
    dr.reset()
    feats = torch.from_numpy(gen_features(2, 64, s.hidden)).cuda()
    toks = np.random.default_rng(3).integers(0, s.vocab, 64)
    parent, depth, _ = gen_tree(81, 20, [3, 2, 1, 1, 1, 1], 6)
    trees = []
    for d in (dr, fresh):
        d.commit(toks, feats)
        trees.append(d.draft_tree(parent, depth, sibling_ranks(parent), int(toks[-1])))
    assert np.array_equal(*trees) and dr.state() == fresh.state()
    rows = dr.state()[1]
    assert np.array_equal(dr.rows("logits", 0, rows), fresh.rows("logits", 0, rows))
    for d in (fresh, dr, tgt):
        d.close()
