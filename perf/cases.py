"""What the performance of this framework is measured on: the calls a decoding program makes, through the public
entry points of paper_2412_12639_amd, over the range of sizes that the shapes, tests and benchmark of this repository use.

A case is one of four kinds of work:

  verify   one tree-verification step (fv_verify_tree and its three variants) over a prefix that is in the cache
  decode   the same with a one-node tree: plain decoding of one token
  prompt   a request's start on the target's side: the prompt goes in, the first tree is verified
  draft    a phase of the drafter: committed pairs go in (a few after a verification step, the whole prompt at a request's
           start), a static tree of draft tokens comes out

Models are the repository's shapes, cut to fewer layers where the layers only repeat (every layer runs the same kernels on
other weights, and even two layers and the head of the large shapes are far larger than the caches).

Weights are drawn on the GPU: matrices N(0, 0.02) like fv_inputs.gen_weights, with two additions that give a random model
the clear choices of a trained one, so that decisions do not hang on the last bits of a sum: embedding rows are large
enough to stay visible in the residual stream, and the head's row of token succ[t] leans towards the embedding of t, so the
greedy continuation of t is succ[t].  Trees carry that continuation along one planted path, as a drafter that is right for
three tokens would.  The drafter's predicted features have a steady component (LSTM biases) on every eighth feature, and
sixteen tokens of the head answer to it in clear steps, as frequent tokens do."""
import functools

import numpy as np
import torch

import fv_inputs as fi
import paper_2412_12639_amd as fv

BRANCHING = [8, 4, 2, 2, 1, 1]               # bench.py's tree
DRAFT_BRANCHING = [8, 4, 2, 2, 1, 1, 1, 1]   # bench.py's static drafting tree (height 8)
PLANT = 3
TREE = 0                                     # seed of the drafter's tree: a static tree is fixed per model
LADDER = 16                                  # draft tokens the drafter's lists start with


def listed():
    v = dict(kind="verify", mode="greedy")
    return [
        # plain decoding of one token by a small model: launches and host time are all there is
        dict(v, name="decode-small", kind="decode", shape="small-gqa", layers=2, prefix=70, nodes=1),
        # a small tree in fp32, every kernel's fp32 form
        dict(v, name="verify-f32", shape="small-gqa-f32", layers=2, prefix=130, nodes=23),
        # one token per step at the 7B width: what speculation is compared with, and its fallback
        dict(v, name="decode-7b", kind="decode", shape="7b", layers=4, prefix=700, nodes=1),
        # the benchmark's step, all 32 layers
        dict(v, name="verify-7b", shape="7b", layers=32, prefix=512, nodes=64),
        # rows that must not depend on the step they are verified in (lossless decoding bit for bit), a ragged tree
        dict(v, name="verify-7b-invariant", mode="invariant", shape="7b", layers=4, prefix=1100, nodes=49),
        # non-greedy verification against the distributions the drafter drew from
        dict(v, name="verify-7b-sampled", mode="sampled", shape="7b", layers=4, prefix=333, nodes=33),
        # a tree above one matrix-core block of rows, long prefix, the 13B width
        dict(v, name="verify-13b-100", shape="13b", layers=2, prefix=4096, nodes=100),
        # the largest trees
        dict(v, name="verify-7b-250", shape="7b", layers=4, prefix=2048, nodes=250),
        # grouped-query heads at the 70B width
        dict(v, name="verify-70b", shape="70b", layers=2, prefix=2048, nodes=32),
        # a long prompt and the first tree
        dict(v, name="prompt-7b", kind="prompt", shape="7b", layers=4, prefix=2000, nodes=64),
        # the drafter's share of a decoding round: the pairs of one verification step in, a tree out
        dict(name="draft-7b", kind="draft", shape="7b", pairs=4, k=2, nodes=64),
        # the drafter's share of a request's start: the whole prompt in, the first tree out
        dict(name="draft-prompt-7b", kind="draft", shape="7b", pairs=500, k=2, nodes=64),
    ]


def draw(rng):
    """Another case of the same ranges; no drawn case does more work than the largest listed one."""
    def log_int(lo, hi):
        return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))

    if rng.random() < 0.2:
        shape = rng.choice(["small-gqa", "7b", "7b"])
        return dict(kind="draft", shape=shape, pairs=log_int(4, 450), k=rng.randint(1, 4), nodes=log_int(9, 100))
    shape = rng.choice(["small-gqa", "small-gqa-f32", "7b", "7b", "13b", "70b"])
    layers = 2 if shape != "7b" else rng.randint(2, 4)
    if rng.random() < 0.2:
        longest = {"7b": 1900, "13b": 1900, "70b": 450}.get(shape, 1900)
        return dict(kind="prompt", mode="greedy", shape=shape, layers=layers, prefix=log_int(60, longest), nodes=log_int(1, 64))
    nodes = log_int(1, 256)
    mode = rng.choice(["greedy", "greedy", "invariant", "sampled", "noalloc"])
    if nodes > 64 and mode in ("invariant", "noalloc") or shape == "70b" and mode == "noalloc":
        mode = "greedy"      # beyond these modes' limits
    return dict(kind="decode" if nodes == 1 else "verify", mode=mode, shape=shape, layers=layers, prefix=log_int(20, 4096), nodes=nodes)


# ------------------------------------------------------------------------------------------------ models

def _shape(case):
    return fi.SHAPES[case["shape"]].with_layers(1 if case["kind"] == "draft" else case["layers"])


class _Draws:
    """Tensors drawn on the GPU from one seed, handed over as the host arrays the library's upload takes."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = torch.bfloat16 if dtype == "bf16" else torch.float32

    def normal(self, shp, std=fi.weights.STD):
        return torch.empty(shp, device="cuda", dtype=torch.float32).normal_(0.0, std, generator=self.gen)

    def host(self, x):
        """A matrix in the model's storage type (bf16 as raw 16-bit patterns), in pinned memory: the upload is a plain copy."""
        h = torch.empty(x.shape, dtype=self.dtype, pin_memory=True)
        h.copy_(x.to(self.dtype))
        return h.view(torch.uint16).numpy() if self.dtype is torch.bfloat16 else h.numpy()


def _target_weights(s, seed, ladder_on):
    d = _Draws(seed, s.dtype)
    w = {}
    for name, shp in fi.weights._tensor_ids(s):
        if len(shp) == 1:
            w[name] = np.ones(shp, dtype=np.float32)
        elif name not in ("embed", "lm_head"):
            w[name] = d.host(d.normal(shp))
    size = 0.5 * (1 + 4 * s.n_layers) ** 0.5 * max(1.0, (s.hidden / 4096) ** 1.5)      # about half of what the layers add to the residual stream
    embed = d.normal((s.vocab, s.hidden), size)
    succ = torch.randperm(s.vocab, generator=d.gen, device="cuda")
    head = d.normal((s.vocab, s.hidden))
    head[succ] += embed * (32.0 / (size * s.hidden))
    if ladder_on:
        rungs = torch.randperm(s.vocab, generator=d.gen, device="cuda")[:LADDER]
        step = torch.arange(LADDER, 0, -1, device="cuda") * 15.0 + 50.0
        head[rungs, ::8] += step[:, None] / (0.7 * (s.hidden // 8))
    w["embed"], w["lm_head"] = d.host(embed), d.host(head)
    return w, succ.cpu().numpy()


def _drafter_weights(s, seed):
    d = _Draws(seed, s.dtype)
    w = {}
    for name, shp in fi.weights.drafter_tensor_ids(s):
        if name.endswith(".b"):
            w[name] = d.normal(shp, 0.1).cpu().numpy()
        elif len(shp) == 1:
            w[name] = np.ones(shp, dtype=np.float32)
        else:
            w[name] = d.host(d.normal(shp))
    b, h = w["lstm1.b"].reshape(4, s.hidden), s.hidden
    b[0, ::8] += 3.0      # input gate open, candidate near one, output gate open: a steady positive output
    b[2, ::8] += 3.0
    b[3, ::8] += 3.0
    w["lstm1.b"] = np.ascontiguousarray(b.reshape(4 * h))
    return w


# ------------------------------------------------------------------------------------------------ inputs

def _tree(rng, seed, n, vocab, root, succ):
    """Topology of bench.py's trees; one path carries the greedy continuation, no other node does."""
    plant = min(PLANT, n - 1)
    parent, depth, planted = fi.gen_tree(seed, n, BRANCHING, plant)
    on_path = {int(i) for i in planted[1:]}
    tokens = np.zeros(n, dtype=np.int32)
    tokens[0] = root
    used = {}
    for i in range(1, n):
        p = int(parent[i])
        taken = used.setdefault(p, {int(succ[tokens[p]])})
        t = int(succ[tokens[p]])
        while i not in on_path and t in taken:
            t = int(rng.integers(0, vocab))
        taken.add(t)
        tokens[i] = t
    return tokens, parent, depth


def _view(owner, address, rows, width):
    """fp32 rows that live in a session's device arena."""
    at = address - owner.arena.data_ptr()
    return owner.arena[at:at + rows * width * 4].view(torch.float32).view(rows, width)


def prepare(case, seed):
    s = _shape(case)
    rng = np.random.Generator(np.random.Philox(key=[seed, 8101]))
    st = {"case": case, "shape": s}
    w, succ = _target_weights(s, seed, case["kind"] == "draft")
    if case["kind"] == "draft":
        target = fv.FalconVerifier(s, max_seq=1024, max_tree=256)
        target.init_weights(w)
        drafter = fv.FalconDrafter(target, case["k"])
        drafter.init_weights(_drafter_weights(s, seed + 1))
        parent, depth, _ = fi.gen_tree(TREE, case["nodes"], DRAFT_BRANCHING, 0)
        gen = torch.Generator(device="cuda").manual_seed(seed + 2)
        feats = torch.empty((case["pairs"], s.hidden), device="cuda").normal_(generator=gen)
        st.update(target=target, drafter=drafter, parent=parent, depth=depth, rank=fi.sibling_ranks(parent), feats=feats,
                  tokens=rng.integers(0, s.vocab, case["pairs"]).astype(np.int32))
        return st
    L, n = case["prefix"], case["nodes"]
    gpu = fv.FalconVerifier(s, max_seq=L + 256 + 8, max_tree=256)
    gpu.init_weights(w)
    if case["mode"] == "invariant":
        gpu.set_step_invariant(True)
    prefix = rng.integers(0, s.vocab, L).astype(np.int32)
    root = gpu.prefill(prefix)
    tokens, parent, depth = _tree(rng, seed, n, s.vocab, root, succ)
    st.update(gpu=gpu, prefix=prefix, root=root, tokens=tokens, parent=parent, depth=depth)
    st["features"] = fv.features_device_ptr(gpu)
    if case["mode"] == "sampled":
        # the distributions a node's children were drawn from: spread over the vocabulary, the drawn tokens among the likely
        gen = torch.Generator(device="cuda").manual_seed(seed + 3)
        q = torch.empty((n, s.vocab), device="cuda").normal_(0.0, 2.0, generator=gen)
        if n > 1:
            q[torch.from_numpy(parent[1:].astype(np.int64)).cuda(), torch.from_numpy(tokens[1:].astype(np.int64)).cuda()] = 8.0
        st["q"] = torch.softmax(q, dim=-1).contiguous()
        st["u_accept"], st["u_sample"] = rng.uniform(0.05, 0.9, n), rng.uniform(0.05, 0.9, n)
    return st


# ------------------------------------------------------------------------------------------------ one pass

def run(st):
    case = st["case"]
    if case["kind"] == "draft":
        d = st["drafter"]
        d.reset()
        d.commit(st["tokens"], st["feats"])
        drafted = d.draft_tree(st["parent"], st["depth"], st["rank"], int(st["tokens"][-1]))
        committed, rows, chain = d.state()
        # the predicted features of every row of the phase are what the drafter computes
        return {"tokens": drafted, "features": d.rows("features", 0, rows), "state": np.array([committed, rows, chain])}
    gpu = st["gpu"]
    if case["kind"] == "prompt":
        root = gpu.prefill(st["prefix"])
    else:
        root = st["root"]
        gpu.rollback(case["prefix"], root)      # the same step again: a host-side counter
    if case["mode"] == "sampled":
        a, accepted, nxt = gpu.verify_tree_sampled(st["tokens"], st["parent"], st["depth"], 1.0, st["u_accept"], st["u_sample"], st["q"])
    else:
        a, accepted, nxt = gpu.verify_tree(st["tokens"], st["parent"], st["depth"], noalloc=case["mode"] == "noalloc")
    # the features of the accepted path stay on the device, where the drafter takes them from; the greedy choice at every
    # node is a few bytes (the logits themselves are megabytes that no decoding program fetches)
    return {"root": root, "accepted": a, "tokens": accepted, "next": nxt, "argmax": gpu.argmax(),
            "features": _view(gpu, st["features"], a + 1, st["shape"].hidden)}


# ------------------------------------------------------------------------------------------------ what a pass cannot do without

def _layer_params(s):
    return (s.weight_params() - s.vocab * s.hidden) // s.n_layers


def _attention_flops(s, pairs):
    return 4.0 * s.n_layers * s.n_q_heads * s.head_dim * pairs


@functools.lru_cache(maxsize=None)
def _draft_rows(nodes, k):
    """Rows the passes below the root block have: one block of up to k rows per node at a depth that is a multiple of k and has children."""
    parent, depth, _ = fi.gen_tree(TREE, nodes, DRAFT_BRANCHING, 0)
    reach = depth.copy()
    for i in range(len(parent) - 1, 0, -1):
        reach[parent[i]] = max(reach[parent[i]], reach[i])
    return sum(min(k, int(reach[i] - depth[i])) for i in range(len(parent)) if depth[i] > 0 and depth[i] % k == 0 and reach[i] > depth[i])


def work(case):
    s = _shape(case)
    e, h = s.elem_bytes(), s.hidden
    if case["kind"] == "draft":
        rows = case["pairs"] + _draft_rows(case["nodes"], case["k"])
        lstm, layer, head = (8 + 3 * 4) * h * h, _layer_params(s), s.vocab * h
        kv = 2 * rows * s.n_kv_heads * s.head_dim * e
        return {"bytes": (lstm + layer + head) * e + case["pairs"] * h * 4 + rows * (h * e + h * 4) + kv,
                "flops": 2.0 * (lstm + layer) * rows + 2.0 * head * (rows - case["pairs"] + case["k"]) + _attention_flops(s, rows * (rows + 1) / 2)}
    L, n = case["prefix"], case["nodes"]
    step_flops = 2.0 * s.weight_params() * n + _attention_flops(s, n * (L + 4))
    out = n * 4 + (1 + PLANT) * h * 4
    if case["kind"] == "prompt":
        # the prompt's rows through the layers and the head once for its last row, then the step; the weights once for both
        return {"bytes": s.step_bytes(L, n) + L * h * e + out,
                "flops": step_flops + 2.0 * _layer_params(s) * s.n_layers * L + 2.0 * s.vocab * h + _attention_flops(s, L * (L + 1) / 2)}
    extra = (1 + PLANT) * s.vocab * 4 if case["mode"] == "sampled" else 0      # the draft distributions along the path
    return {"bytes": s.step_bytes(L, n) + out + extra, "flops": step_flops}


def tolerance(case):
    """About four times what the features move by when the sums of the matrix products run in another order.  Measured with the
    library's other kernel and split for the same products: fp32 7e-8; bf16, where such a change moves some of the roundings that
    follow, 2.5e-3 to 3.7e-3 at one to four layers and 7.2e-3 at 32, single values four times that.  The choices are clear
    enough to stay (the smallest top-2 gap is a hundred times the error), so whole numbers are compared exactly."""
    if fi.SHAPES[case["shape"]].dtype == "f32":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    rel = 2.8e-2 if case.get("layers", 1) > 8 else 1.4e-2
    return {"rel": rel, "max": 5 * rel, "differ": 0.0}
