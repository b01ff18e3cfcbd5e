"""Ancestor sets of trees that begin with a chain (a prompt is nothing else), at the word edges of a set and around the depth up to which
the table of ancestors by depth is filled."""
import numpy as np
import pytest

import fv_inputs as fi
from oracle import falcon_oracle as fo

pytestmark = pytest.mark.gpu

CASES = [(1, 1), (2, 30), (32, 2), (33, 31), (34, 1), (63, 1), (64, 0), (65, 63), (128, 40), (129, 127), (200, 56), (256, 0)]   # nodes of the chain, nodes behind it


@pytest.fixture(scope="module")
def session():
    import paper_2412_12639_amd as fv
    s = fi.SHAPES["tiny"]
    g = fv.FalconVerifier(s, max_seq=512, max_tree=256)
    g.init_weights(fi.gen_weights(s, seed=0))
    yield g, s
    g.close()


@pytest.mark.parametrize("chain,more", CASES)
def test_ancestor_sets_behind_a_chain(session, chain, more):
    g, s = session
    n = chain + more
    rng = np.random.Generator(np.random.Philox(n))
    parent = np.arange(-1, n - 1, dtype=np.int32)
    for i in range(chain, n):      # the first one does not follow its neighbour; the others anywhere, some of them chains again
        parent[i] = rng.integers(0, i - 1) if i == chain and i > 1 else i - 1 if rng.random() < 0.5 else rng.integers(0, i)
    depth = np.zeros(n, dtype=np.int32)
    for i in range(1, n):
        depth[i] = depth[parent[i]] + 1
    root = g.prefill(np.arange(5, dtype=np.int32))
    tokens = rng.integers(0, s.vocab, n).astype(np.int32)
    tokens[0] = root
    g.verify_tree(tokens, parent, depth)
    assert np.array_equal(g.tree_mask(n), fo.ancestor_mask(parent))
