"""Timed cases of the tree-verification library: what a program that verifies draft trees asks of it.

Every case goes through the public entry points of ``paper_2606_00535_amd.dreams``.  The kinds of call are

    attn      one layer's tree attention: bf16 or fp32, parent array or mask bits, with or without row entropies
    step      a whole verify step of a model: the attention of every layer, greedy acceptance, the KV commit
    accept    greedy acceptance from the target's logits
    sampled   acceptance at temperature 1 from target and draft logits
    lm_head   greedy acceptance from the final hidden states (the LM head inside the call)
    prefill   the statistics of a prompt and the visual-token selection that follows from them

``listed()`` names the ones that stand for the range, ``draw()`` gives others of the same range.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_00535_amd import dreams
from paper_2606_00535_amd import workload as W

DEVICE = "cuda"


# ---------------------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: one fp32 layer of 4 heads over 640 prefix tokens, where launches and latency count
        dict(name="attn_tiny_f32", kind="attn", dtype="f32", batch=1, hq=4, hkv=4, d=64, lo=640, hi=640, nodes=16,
             depth=4, branch=3, mask=False, entropy=False),
        # an ordinary decode call at batch 1: one LLaVA-1.6-7B layer, 2880 image and 256 text tokens
        dict(name="attn_7b_layer", kind="attn", dtype="bf16", batch=1, hq=32, hkv=32, d=128, lo=3136, hi=3136,
             nodes=60, depth=6, branch=4, mask=False, entropy=False),
        # options and odd sizes: head_dim 64, grouped heads, mask bits in, row entropies out, ragged lengths
        dict(name="attn_d64_mask_entropy", kind="attn", dtype="bf16", batch=3, hq=24, hkv=8, d=64, lo=517, hi=2733,
             nodes=37, depth=5, branch=3, mask=True, entropy=True),
        # many long sequences over few KV heads, the largest attention call: the matrix cores' case
        dict(name="attn_gqa_long", kind="attn", dtype="bf16", batch=16, hq=28, hkv=4, d=128, lo=8192, hi=8192,
             nodes=128, depth=8, branch=6, mask=False, entropy=False),
        # a whole step of a 32-layer model at batch 1, captured once and replayed, as a serving loop runs it
        dict(name="step_7b_b1_graph", kind="step", batch=1, hq=32, hkv=32, d=128, layers=32, lo=3136, hi=3136,
             nodes=60, depth=6, branch=4, vocab=32000, graph=True),
        # the same model at batch 4 with ragged lengths, called eagerly
        dict(name="step_7b_b4", kind="step", batch=4, hq=32, hkv=32, d=128, layers=32, lo=2900, hi=4096, nodes=60,
             depth=6, branch=4, vocab=32000, graph=False),
        # greedy acceptance over the largest vocabulary and batch: a stream of logits
        dict(name="accept_gqa_long", kind="accept", batch=16, nodes=128, depth=8, branch=6, vocab=152064),
        # acceptance at temperature 1: one sequence of a 32000-entry vocabulary, and the largest batch
        dict(name="sampled_7b", kind="sampled", batch=1, nodes=60, depth=6, branch=4, vocab=32000),
        dict(name="sampled_gqa_long", kind="sampled", batch=16, nodes=128, depth=8, branch=6, vocab=152064),
        # the LM head inside the call: one tree (the weight is streamed), and 2048 rows (a matrix product)
        dict(name="lm_head_7b", kind="lm_head", batch=1, nodes=60, depth=6, branch=4, hidden=4096, vocab=32000),
        dict(name="lm_head_gqa_long", kind="lm_head", batch=16, nodes=128, depth=8, branch=6, hidden=3584,
             vocab=152064),
        # after a prefill: row statistics, the layer's entropy, Eq. 2 importance, the kept fifth of 2880 image tokens
        dict(name="prefill_select_7b", kind="prefill", batch=1, hq=32, hkv=32, d=128, lo=3136, hi=3136, vis_begin=35,
             vis=2880, keep=576),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tree_shape(rng, most):
    nodes = _log_int(rng, 1, most)
    depth = rng.randint(min(3, nodes - 1), min(8, nodes - 1)) if nodes > 1 else 0
    return dict(nodes=nodes, depth=depth, branch=rng.randint(4, 6) if nodes <= 60 else 6)


_HEADS = ((32, 32), (40, 40), (28, 4), (32, 8), (24, 8), (16, 16), (8, 2))


def draw(rng):
    """One more case of the listed kinds, its sizes spread over the range that they cover."""
    kind = rng.choice(("attn", "attn", "attn", "attn_f32", "step", "accept", "sampled", "lm_head", "prefill"))
    if kind == "attn":
        hq, hkv = rng.choice(_HEADS)
        hi = _log_int(rng, 64, 8192)
        # caches of at most 8 sequences of 40 KV heads and 4096 slots (one LLaVA-1.6-13B layer at batch 8)
        batch = min(_log_int(rng, 1, 16), max(1, 8 * 40 * 4096 // (hkv * hi)))
        return dict(kind="attn", dtype="bf16", batch=batch, hq=hq, hkv=hkv, d=rng.choice((64, 128, 128)),
                    lo=max(1, int(hi * rng.uniform(0.3, 1.0))), hi=hi, mask=rng.random() < 0.3,
                    entropy=rng.random() < 0.3, **_tree_shape(rng, 128))
    if kind == "attn_f32":
        hq, hkv = rng.choice(((4, 4), (4, 2), (6, 2), (3, 3), (8, 8)))
        hi = _log_int(rng, 64, 1300)
        return dict(kind="attn", dtype="f32", batch=rng.randint(1, 2), hq=hq, hkv=hkv, d=rng.choice((64, 128)),
                    lo=max(1, int(hi * rng.uniform(0.3, 1.0))), hi=hi, mask=rng.random() < 0.3,
                    entropy=rng.random() < 0.3, **_tree_shape(rng, 100))
    if kind == "step":
        hq, hkv = rng.choice(((32, 32), (40, 40), (28, 4), (32, 8)))
        hi = _log_int(rng, 512, 4096)
        return dict(kind="step", batch=rng.randint(1, 4), hq=hq, hkv=hkv, d=128, layers=rng.choice((16, 24) if hkv > 32 else (16, 24, 28, 32)),
                    lo=max(1, int(hi * rng.uniform(0.4, 0.7))), hi=hi, vocab=_log_int(rng, 1000, 152064),
                    graph=rng.random() < 0.5, **_tree_shape(rng, 60))
    if kind in ("accept", "sampled"):
        return dict(kind=kind, batch=_log_int(rng, 1, 16), vocab=_log_int(rng, 1000, 152064), **_tree_shape(rng, 128))
    if kind == "lm_head":
        return dict(kind="lm_head", batch=_log_int(rng, 1, 16), hidden=256 * rng.randint(4, 14),
                    vocab=_log_int(rng, 1000, 152064), **_tree_shape(rng, 128))
    hq, hkv = rng.choice(((32, 32), (28, 4), (32, 8), (8, 2)))
    hi = _log_int(rng, 256, 3500)
    begin = rng.randint(0, 35)
    vis = max(8, int((hi - begin) * rng.uniform(0.5, 0.95)))
    return dict(kind="prefill", batch=rng.randint(1, 2), hq=hq, hkv=hkv, d=rng.choice((64, 128, 128)),
                lo=max(1, int(hi * rng.uniform(0.5, 1.0))), hi=hi, vis_begin=begin, vis=vis,
                keep=max(1, int(vis * rng.uniform(0.1, 0.5))))


# ------------------------------------------------------------------------------------------------------- inputs
class _Inputs:
    """Seeded draws on the device (tensors) and the host (trees, lengths)."""

    def __init__(self, seed):
        self.host = np.random.default_rng(seed)
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(int(seed))

    def normal(self, shape, dtype=torch.bfloat16, std=1.0):
        x = torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, std, generator=self.gen)
        return x

    def uniform(self, shape):
        return torch.rand(shape, generator=self.gen, device=DEVICE)

    def ints(self, high, shape):
        return torch.randint(0, high, shape, generator=self.gen, device=DEVICE, dtype=torch.int32)

    def lengths(self, lo, hi, batch):
        """Prefix lengths lo..hi, the longest one present (a server sizes its bound by it)."""
        n = self.host.integers(lo, hi + 1, size=batch).astype(np.int32)
        n[int(self.host.integers(batch))] = hi
        return n

    def trees(self, case):
        return np.stack([W.random_tree(self.host, case["nodes"], case["depth"], case["branch"])
                         for _ in range(case["batch"])])

    def logits(self, case):
        x = torch.empty((case["batch"], case["nodes"], case["vocab"]), device=DEVICE)
        return x.normal_(0.0, 3.0, generator=self.gen)

    def draft_tokens(self, case, parent, target):
        """The greedy target's own token of the parent with probability 0.7, any token otherwise."""
        follow = torch.gather(target, 1, parent.clamp(min=0).long())
        hit = self.uniform(parent.shape) < 0.7
        hit[:, 0] = False
        return torch.where(hit, follow.int(), self.ints(case["vocab"], parent.shape)).contiguous()


def _device(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEVICE)


def _visible(parent):
    """[B, T, T] truth values: node j is node i or an ancestor of it."""
    batch, nodes = parent.shape
    see = np.zeros((batch, nodes, nodes), dtype=bool)
    for b in range(batch):
        for i in range(nodes):
            if i:
                see[b, i] = see[b, parent[b, i]]
            see[b, i, i] = True
    return see


def _mask_bits(parent):
    see = _visible(parent)
    batch, nodes, _ = see.shape
    words = (nodes + 63) // 64
    bits = np.zeros((batch, nodes, words * 64), dtype=np.uint8)
    bits[:, :, :nodes] = see
    return np.packbits(bits, axis=2, bitorder="little").view(np.int64).reshape(batch, nodes, words)


def _prepare_attn(case, seed):
    r = _Inputs(seed)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    batch, nodes, d = case["batch"], case["nodes"], case["d"]
    lengths, parent = r.lengths(case["lo"], case["hi"], batch), r.trees(case)
    capacity = (case["hi"] + nodes + 63) // 64 * 64
    cache = (batch, case["hkv"], capacity, d)
    tree = dict(tree_mask=_device(_mask_bits(parent))) if case["mask"] else dict(parent=_device(parent))
    q = r.normal((batch, case["hq"], nodes, d), dtype, 0.125 if case["dtype"] == "f32" else 1.0)
    return dict(kind="attn", case=case, lengths=lengths, tree=parent, max_kv_len=case["hi"],
                tensors=(q, r.normal(cache, dtype), r.normal(cache, dtype), _device(lengths)), topology=tree)


def _run_attn(s):
    if s["case"]["entropy"]:
        return dreams.tree_verify_attn_entropy(*s["tensors"], max_kv_len=s["max_kv_len"], **s["topology"])
    return dreams.tree_verify_attn(*s["tensors"], max_kv_len=s["max_kv_len"], **s["topology"])


def _prepare_step(case, seed):
    r = _Inputs(seed)
    batch, nodes, d, layers = case["batch"], case["nodes"], case["d"], case["layers"]
    lengths, parent = r.lengths(case["lo"], case["hi"], batch), r.trees(case)
    capacity = (case["hi"] + nodes + 63) // 64 * 64
    cache = (layers, batch, case["hkv"], capacity, d)
    logits, par = r.logits(case), _device(parent)
    s = dict(kind="step", case=case, lengths=lengths, tree=parent, max_kv_len=case["hi"], kv_len=_device(lengths),
             parent=par, q=r.normal((layers, batch, case["hq"], nodes, d)), k=r.normal(cache), v=r.normal(cache),
             logits=logits, tokens=r.draft_tokens(case, par, logits.argmax(dim=2)))
    s["out"] = torch.empty_like(s["q"])
    if case["graph"]:
        _capture_step(s)
    return s


def _step_calls(s, workspaces, accepted, kv_len_out):
    for layer in range(s["case"]["layers"]):
        dreams.tree_verify_attn(s["q"][layer], s["k"][layer], s["v"][layer], s["kv_len"], s["parent"],
                                out=s["out"][layer], with_lse=False, max_kv_len=s["max_kv_len"],
                                workspace=workspaces[0])
    length, path, token, _ = dreams.tree_accept(s["logits"], s["tokens"], s["parent"], outputs=accepted,
                                                workspace=workspaces[1])
    kept = dreams.kv_commit(s["k"], s["v"], s["kv_len"], path, length, kv_len_out=kv_len_out)
    return dict(out=s["out"], accept_len=length, accept_path=path, next_token=token, kv_len=kept, k=s["k"], v=s["v"])


def _capture_step(s):
    """The step in a HIP graph: its buffers are the state's own, and a replay runs it on what they hold."""
    case, batch = s["case"], s["case"]["batch"]
    desc = dreams.attn_desc(s["q"][0], s["k"][0], 0, s["max_kv_len"])
    sizes = (dreams.tree_verify_attn_workspace_size(desc),
             dreams.tree_accept_workspace_size(batch, case["nodes"], case["vocab"]))
    workspaces = [torch.zeros(max(n, 256), dtype=torch.uint8, device=DEVICE) for n in sizes]
    accepted = (torch.empty(batch, dtype=torch.int32, device=DEVICE),
                torch.empty((batch, case["nodes"]), dtype=torch.int32, device=DEVICE),
                torch.empty(batch, dtype=torch.int32, device=DEVICE), None)
    kv_len_out = torch.empty(batch, dtype=torch.int32, device=DEVICE)
    # every kernel once before the capture; a commit of the roots alone moves nothing
    dreams.tree_verify_attn(s["q"][0], s["k"][0], s["v"][0], s["kv_len"], s["parent"], out=s["out"][0],
                            with_lse=False, max_kv_len=s["max_kv_len"], workspace=workspaces[0])
    dreams.tree_accept(s["logits"], s["tokens"], s["parent"], outputs=accepted, workspace=workspaces[1])
    dreams.kv_commit(s["k"], s["v"], s["kv_len"], accepted[1], torch.zeros_like(accepted[0]), kv_len_out=kv_len_out)
    torch.cuda.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"]):
        s["result"] = _step_calls(s, workspaces, accepted, kv_len_out)
    s["held"] = (workspaces, accepted, kv_len_out)


def _run_step(s):
    if "graph" in s:
        s["graph"].replay()
        return s["result"]
    return _step_calls(s, (None, None), None, None)


def _prepare_accept(case, seed):
    r = _Inputs(seed)
    parent = _device(r.trees(case))
    logits = r.logits(case)
    return dict(kind="accept", logits=logits, parent=parent,
                tokens=r.draft_tokens(case, parent, logits.argmax(dim=2)))


def _run_accept(s):
    return dreams.tree_accept(s["logits"], s["tokens"], s["parent"], want_target_argmax=True)


def _prepare_sampled(case, seed):
    r = _Inputs(seed)
    tree = r.trees(case)
    target = r.logits(case)
    draft = torch.empty_like(target)
    tokens = r.ints(case["vocab"], tree.shape)
    for b in range(case["batch"]):
        # the draft approximates the target, and samples each child's token at its parent (Gumbel-max)
        torch.add(target[b], torch.empty_like(target[b]).normal_(0.0, 1.0, generator=r.gen), out=draft[b])
        if case["nodes"] > 1:
            up = torch.from_numpy(tree[b, 1:].astype(np.int64)).to(DEVICE)
            noise = -torch.log(torch.empty((len(up), case["vocab"]), device=DEVICE).exponential_(generator=r.gen))
            tokens[b, 1:] = (draft[b][up] + noise).argmax(dim=1).int()
    return dict(kind="sampled", target=target, draft=draft, tokens=tokens, parent=_device(tree),
                uniforms=r.uniform(tree.shape))


def _run_sampled(s):
    return dreams.tree_accept_sampled(s["target"], s["draft"], s["tokens"], s["parent"], s["uniforms"], 1.0)


def _prepare_lm_head(case, seed):
    r = _Inputs(seed)
    batch, nodes, hidden, vocab = case["batch"], case["nodes"], case["hidden"], case["vocab"]
    parent = _device(r.trees(case))
    weight = r.normal((vocab, hidden), std=1.0 / math.sqrt(hidden))
    # a trained model's state points at its next token: that token's logit stands clear of the N(0, 1) others
    target = r.ints(vocab, (batch, nodes))
    state = (8.0 * weight[target.long()].float() + r.normal((batch, nodes, hidden), torch.float32)).bfloat16()
    return dict(kind="lm_head", hidden=state.contiguous(), weight=weight, parent=parent,
                tokens=r.draft_tokens(case, parent, target.long()))


def _run_lm_head(s):
    return dreams.tree_accept_lm_head(s["hidden"], s["weight"], s["tokens"], s["parent"], want_target_argmax=True)


def _prepare_prefill(case, seed):
    r = _Inputs(seed)
    batch, d, rows = case["batch"], case["d"], case["hi"]
    lengths = r.lengths(case["lo"], rows, batch)
    capacity = (rows + 63) // 64 * 64
    # every query looks along one direction, and the keys lie along it by a token's own amount: attention is
    # concentrated on few tokens, as in a trained model, and importances spread over orders of magnitude
    along = torch.nn.functional.normalize(r.normal((d,), torch.float32), dim=0) * d ** 0.25
    q = r.normal((batch, case["hq"], rows, d), torch.float32) + along
    k = r.normal((batch, case["hkv"], capacity, d), torch.float32)
    k += r.normal((batch, 1, capacity, 1), torch.float32) * along
    cache = (q.bfloat16(), k.bfloat16(), _device(lengths))
    return dict(kind="prefill", case=case, lengths=lengths, tensors=cache, v=r.normal(k.shape))


def _run_prefill(s):
    case, (q, k, lengths) = s["case"], s["tensors"]
    lse, entropy = dreams.prefill_attn_stats(q, k, lengths)
    mean = dreams.prefill_attn_entropy_mean(entropy, lengths)
    importance = dreams.prefill_visual_importance(q, k, lengths, lse, case["vis_begin"], case["vis"])
    keep = dreams.visual_topk(importance, case["keep"])
    k_kept, v_kept = dreams.visual_gather(k, s["v"], case["vis_begin"], keep)
    return dict(lse=lse, entropy=entropy, mean=mean, importance=importance, keep=keep, k=k_kept, v=v_kept)


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return globals()["_run_" + state["kind"]](state)


# ------------------------------------------------------------------------------------------------- what it takes
#: Nodes that a sampled walk visits in a sequence: the root and the drafts that it accepts (two at these drafts).
_WALKED = 3


def work(case):
    kind = case["kind"]
    if kind in ("attn", "step"):
        size = 4 if case.get("dtype") == "f32" else 2
        keys = (case["lo"] + case["hi"]) / 2 + case["nodes"]
        rows = case["batch"] * case["hq"] * case["nodes"]
        layer = 2 * case["batch"] * case["hkv"] * keys * case["d"] * size + 2 * rows * case["d"] * size
        flops = 4.0 * rows * keys * case["d"]
        if kind == "attn":
            return dict(bytes=layer + rows * 4 * (2 if case["entropy"] else 1), flops=flops)
        logits = case["batch"] * case["nodes"] * case["vocab"] * 4
        return dict(bytes=case["layers"] * layer + logits, flops=case["layers"] * flops)
    if kind == "prefill":
        keys, heads = (case["lo"] + case["hi"]) / 2, case["batch"] * case["hq"]
        seen = heads * keys * keys / 2
        scored = heads * case["vis"] * max(keys - case["vis_begin"] - case["vis"] / 2, 0)
        read = case["batch"] * keys * case["d"] * 2 * (2 * case["hq"] + 2 * case["hkv"])
        kept = 4 * case["batch"] * case["hkv"] * case["keep"] * case["d"] * 2
        return dict(bytes=read + kept + 4 * heads * keys * 2, flops=2.0 * case["d"] * (seen + scored))
    rows = case["batch"] * case["nodes"]
    if kind == "accept":
        return dict(bytes=rows * case["vocab"] * 4, flops=0)
    if kind == "sampled":
        return dict(bytes=case["batch"] * min(_WALKED, case["nodes"]) * case["vocab"] * 8, flops=0)
    return dict(bytes=(case["vocab"] + rows) * case["hidden"] * 2, flops=2.0 * rows * case["vocab"] * case["hidden"])


def tolerance(case):
    kind = case["kind"]
    if kind in ("accept", "sampled"):
        return "exact"      # whole numbers from given logits
    if kind == "lm_head":
        return dict(differ=0.005)   # an argmax between two logits that are equal in fp32 but for the sums' order
    if kind == "attn" and case["dtype"] == "f32":
        return dict(rel=2e-6, max=5e-5)     # fp32 sums of a few thousand products in another order
    # bf16 outputs of fp32 sums: 1.7e-3 from the rounding of the result, as much again from the probabilities'
    return dict(rel=1e-2, max=0.1, differ=0.005)


# --------------------------------------------------------------------------------------- the same, in 64 bits
def _exact_attn(q, k, v, lengths, tree):
    """(out, lse, entropy) of one layer: a masked softmax over each sequence's prefix and tree slots."""
    batch, hq, nodes, d = q.shape
    hkv = k.shape[1]
    see = torch.from_numpy(_visible(tree)).to(q.device)
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    lse = torch.empty((batch, hq, nodes), dtype=torch.float64, device=q.device)
    entropy = torch.empty_like(lse)
    for b in range(batch):
        n = int(lengths[b])
        for g in range(hkv):
            heads = slice(g * (hq // hkv), (g + 1) * (hq // hkv))
            rows = q[b, heads].double().reshape(-1, d)
            keys, values = k[b, g, :n + nodes].double(), v[b, g, :n + nodes].double()
            z = (rows @ keys.t().contiguous()).reshape(-1, nodes, n + nodes) / math.sqrt(d)
            z[:, :, n:].masked_fill_(~see[b], -math.inf)
            top = torch.logsumexp(z, dim=2)
            p = torch.exp(z - top[:, :, None])
            out[b, heads] = (p.reshape(-1, n + nodes) @ values).reshape(-1, nodes, d)
            lse[b, heads] = top
            entropy[b, heads] = top - (p * z.masked_fill(p == 0, 0.0)).sum(dim=2)
    return out, lse, entropy


def _exact_prefill(s):
    case, (q, k, _) = s["case"], s["tensors"]
    batch, hq, rows, d = q.shape
    group = hq // k.shape[1]
    begin, vis = case["vis_begin"], case["vis"]
    lse = torch.full((batch, hq, rows), -math.inf, dtype=torch.float64, device=q.device)
    entropy = torch.zeros((batch, hq, rows), dtype=torch.float64, device=q.device)
    importance = torch.zeros((batch, vis), dtype=torch.float64, device=q.device)
    for b in range(batch):
        n = int(s["lengths"][b])
        later = torch.ones((n, n), dtype=torch.bool, device=q.device).triu(1)
        last = min(n, begin + vis)
        for h in range(hq):
            z = q[b, h, :n].double() @ k[b, h // group, :n].double().t().contiguous() / math.sqrt(d)
            z.masked_fill_(later, -math.inf)
            top = torch.logsumexp(z, dim=1)
            p = torch.exp(z - top[:, None])
            lse[b, h, :n] = top
            entropy[b, h, :n] = top - (p * z.masked_fill_(later, 0.0)).sum(dim=1)
            if last > begin:
                importance[b, :last - begin] += p[:, begin:last].sum(dim=0)
        importance[b] /= hq * n
    mean = entropy.sum().reshape(1) / (hq * int(s["lengths"].sum()))
    # the kept rows are copies that follow from whole numbers
    return dict(lse=lse, entropy=entropy, mean=mean, importance=importance, keep=None, k=None, v=None)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("accept", "sampled", "lm_head"):
        return None     # whole numbers only
    s = prepare(case, seed)
    if kind == "prefill":
        return _exact_prefill(s)
    if kind == "attn":
        out, lse, entropy = _exact_attn(*s["tensors"][:3], s["lengths"], s["tree"])
        return (out, lse, entropy) if case["entropy"] else (out, lse)
    layers = [_exact_attn(s["q"][i], s["k"][i], s["v"][i], s["lengths"], s["tree"])[0] for i in range(case["layers"])]
    # acceptance is whole numbers, and the commit moves rows bit for bit
    return dict(out=torch.stack(layers), accept_len=None, accept_path=None, next_token=None, kv_len=None, k=None,
                v=None)
