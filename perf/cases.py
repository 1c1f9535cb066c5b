"""The work that programs built on this library have it do, as timed cases.

Every case goes through `paper_2410_20488_amd.binding` the way a serving or training program does:
an engine over one model is kept, requests are prefilled and decoded with a static draft tree, or
the training forward of one prediction step is run.  Four kinds of pass:

  request   prefill of the prompts and `steps` decoding steps: a whole short request
  decode    `steps` decoding steps of sequences that are already running
  prefill   the prompts of a new batch up to their first tokens
  train     the training-stage forward of one prediction step on one sequence

Weights are random, but the model is not a model of noise: the head's row of a token contains, with
falling weight, the embeddings of the eight tokens it is likely to follow, so that, like a trained
model's, a row of logits prefers one token by a wide margin and ranks the next few, and two correct
implementations emit the same text and draft the same candidates.  With `drafting` the FIRP maps do
what trained maps are for (map i carries a token's hidden state to that of the i-th token after it,
a rotation of the embedding), so the draft tree is accepted; without it they rotate to other tokens,
every draft is wrong and a step emits one token.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2410_20488_amd import binding, synth

# How many generated tokens a decoding sequence may take before the program starts it anew.
ROOM = 3072
# Branching of the regular draft trees by number of prediction steps.
BRANCHING = {1: (8,), 2: (8, 4), 3: (8, 4, 2), 4: (4, 3, 2, 2)}


def _case(name, kind, shape, layers, dtype="bf16", k=3, nodes=64, tree="regular", anchors="root", batch=1, prompt=512,
          steps=16, drafting=False):
    c = dict(kind=kind, shape=shape, layers=layers, dtype=dtype, k=k, nodes=nodes, tree=tree, anchors=anchors, batch=batch,
             prompt=prompt, steps=steps, drafting=drafting)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # The correctness configuration: a 4-layer fp32 model, chain tree, prompt 64, 32 steps.
        # Nothing but launches and small kernels.
        _case("request_small_f32", "request", "tiny", 4, dtype="f32", nodes=4, tree="chain", prompt=64, steps=32),
        # The same in bf16: the latency of the whole step where no kernel has work to speak of.
        _case("request_small_bf16", "request", "tiny_bf16", 4, nodes=4, tree="chain", prompt=64, steps=32, drafting=True),
        # Three ragged requests side by side on a model with grouped KV heads and odd widths (FFN
        # 352, vocabulary 520), an irregular tree with every node an anchor.
        _case("request_ragged_gqa", "request", "tiny_gqa", 3, k=2, nodes=23, tree="irregular", anchors="all", batch=3,
              prompt=211, steps=16),
        # Ordinary greedy decoding, one row a step: the library without its maps.
        _case("greedy_7b", "decode", "7b", 32, k=0, nodes=1, prompt=512),
        # 7B shape with the 41-node tree, prompt 512.
        _case("decode_7b_41", "decode", "7b", 32, nodes=41, tree="full432", prompt=512),
        # The headline: 13B shape, 64-node tree, prompt 1024.
        _case("decode_13b_64", "decode", "13b", 40, prompt=1024),
        # Every node an anchor (the paper-complete setting, 256 rows), maps that draft well: several
        # tokens a step and a cache that is compacted.
        _case("decode_13b_all_anchors", "decode", "13b", 40, anchors="all", prompt=1024, steps=8, drafting=True),
        # Long context: attention over 8k tokens beside the weight stream.
        _case("decode_7b_ctx8k", "decode", "7b", 32, prompt=8192),
        # Four sequences of the grouped-KV 34B shape (268 rows; a quarter of the depth).
        _case("decode_34b_batch4", "decode", "34b", 12, batch=4, prompt=2048),
        # Time to the first token of an ordinary and of a long prompt.
        _case("prefill_13b_1k", "prefill", "13b", 40, prompt=1024),
        _case("prefill_7b_8k", "prefill", "7b", 32, prompt=8192),
        # Training-stage forward of prediction step 2 on 128 tokens (256 rows and their logits).
        _case("train_forward_13b", "train", "13b", 40, prompt=128, steps=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any of the shapes at any depth up to the listed one, prompts of 16 to
    8192 tokens, one to four sequences, 0 to 4 prediction steps, trees of 1 to 64 nodes."""
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "request", "train"])
    if kind == "request":
        shape = rng.choice(["tiny", "tiny_bf16", "tiny_gqa"])
    else:
        shape = rng.choice(["7b", "7b", "13b", "13b", "34b"])
    layers = _log_int(rng, 2, {"7b": 32, "13b": 40, "34b": 12}.get(shape, 4))
    if kind == "train":
        k = rng.randint(1, 4)
        return _case(None, kind, shape, layers, k=k, nodes=1, prompt=rng.randint(8, 128), steps=rng.randint(1, k))
    batch = rng.choice([1, 1, 2, 3, 4])
    k = rng.choice([0, 1, 2, 3, 3, 3, 4])
    nodes = 1 if k == 0 else min(_log_int(rng, 1, 64), 1 + sum(math.prod(BRANCHING[k][:i + 1]) for i in range(k)))
    tree = rng.choice(["regular", "regular", "irregular"])
    anchors = "all" if k > 0 and nodes * (k + 1) <= 256 and rng.random() < 0.3 else "root"
    longest = 512 if kind == "request" else 8192 // batch
    prompt = _log_int(rng, 16, longest)
    steps = rng.randint(4, 16)
    return _case(None, kind, shape, layers, dtype="f32" if shape == "tiny" else "bf16", k=k, nodes=nodes, tree=tree,
                 anchors=anchors, batch=batch, prompt=prompt, steps=steps, drafting=rng.random() < 0.5)


# ----------------------------------------------------------------------------------------------- inputs


def _config(case):
    base = synth.CONFIGS[case["shape"]]
    layers = case["layers"]
    return synth.scaled_config(base, layers, firp_layer=layers // 2, k=case["k"], dtype=case["dtype"])


def _tree(case):
    n, k, anchors = case["nodes"], case["k"], case["anchors"] if case["k"] else "none"
    if n == 1:
        return synth.chain_tree(0, anchors)
    if case["tree"] == "chain":
        return synth.chain_tree(n - 1, anchors)
    if case["tree"] == "full432":
        return synth.full_tree((4, 3, 2), anchors)
    if case["tree"] == "irregular":
        return synth.with_anchors(synth.random_tree(n, n, k, 8, 0.5), anchors)
    return synth.budget_tree(BRANCHING[k], n - 1, anchors)


def _prompt_lengths(case):
    # sequences of a batch are ragged: the first has the full length, each further one about a sixth less
    return [max(1, case["prompt"] - b * (case["prompt"] // 6)) for b in range(case["batch"])]


def _weights(cfg, drafting, gen, dev):
    d, v, f, L = cfg.d_model, cfg.vocab, cfg.d_ffn, cfg.n_layers
    qd, kvd = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim
    dt = cfg.torch_dtype

    def normal(*shape, std):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dt).mul_(std)

    # tokens come in groups of up to d: token j of a group carries the group's vector rotated by j,
    # and the tokens likely to follow it are j + 1 (the likeliest), j + 6, j + 11, ... of its group
    groups = (v + d - 1) // d
    base = normal(groups, d, std=2.0)
    ring = torch.cat([base, base], dim=1)
    embed = torch.cat([ring[g].as_strided((min(d, v - g * d), d), (1, 1), ring[g].storage_offset()) for g in range(groups)])
    head = normal(v, d, std=0.01)
    for r in range(8):
        before = torch.cat([torch.roll(torch.arange(g * d, min(v, (g + 1) * d), device=dev), 1 + 5 * r)
                            for g in range(groups)])
        head += embed[before] * (0.02 * (8 - r) / 8)
    out_std = 0.02 / math.sqrt(2 * L)          # the usual scale of matrices that write to the residual stream
    w = dict(embed=embed.contiguous(), lm_head=head, norm_final=1 + normal(d, std=0.1))
    for name, shape, std in (("wq", (qd, d), 0.02), ("wk", (kvd, d), 0.02), ("wv", (kvd, d), 0.02), ("wo", (d, qd), out_std),
                             ("w_gate", (f, d), 0.02), ("w_up", (f, d), 0.02), ("w_down", (d, f), out_std)):
        w[name] = [normal(*shape, std=std) for _ in range(L)]
    for name in ("norm_attn", "norm_mlp"):
        w[name] = [1 + normal(d, std=0.1) for _ in range(L)]
    w["proj_w"], w["proj_b"] = [], None
    rows = torch.arange(d, device=dev)
    for i in range(cfg.k):
        m = normal(d, d, std=0.02 / math.sqrt(d))
        m[rows, (rows + i + 1 + (0 if drafting else d // 3)) % d] += 1.0
        w["proj_w"].append(m)
    return w


def prepare(case, seed):
    """An engine that has served before (its weights are laid out), the tree and the prompts of the next
    requests; the sequences of a decoding case are prefilled."""
    dev = torch.device("cuda:0")
    cfg, tree = _config(case), _tree(case)
    gen = torch.Generator(device=dev).manual_seed(1000003 * seed + 17)
    weights = _weights(cfg, case["drafting"], gen, dev)
    host = np.random.default_rng(seed)
    lens = _prompt_lengths(case)
    prompts = [host.integers(0, cfg.vocab, n).astype(np.int32).tolist() for n in lens]
    rows = 2 * case["prompt"] if case["kind"] == "train" else tree.n_nodes + cfg.k * sum(tree.anchor)
    room = {"decode": ROOM, "request": case["steps"] * (cfg.k + 1) + 16}.get(case["kind"], 16)
    engine = binding.engine_for_config(cfg, weights, max_ctx=max(lens) + room, max_batch=case["batch"],
                                       max_nodes=tree.n_nodes, max_rows=max(128, rows), b_max=8, keep_logits=True)
    engine.prefill([[0]] * case["batch"])
    if case["kind"] == "decode":
        engine.prefill(prompts)
    elif case["kind"] == "train":
        engine.reset()
    return dict(kind=case["kind"], engine=engine, prompts=prompts, steps=case["steps"], k=cfg.k, max_ctx=max(lens) + room,
                tree=(list(tree.parent), list(tree.rank), list(tree.anchor)))


def run(state):
    """One pass: the tokens (or the loss terms) and the logits that the program has at its end."""
    eng = state["engine"]
    if state["kind"] == "train":
        loss, kl = eng.train_forward(state["prompts"][0], state["steps"])
        return dict(loss=float(loss), kl=kl, logits=eng.last_logits())
    if state["kind"] == "prefill":
        first = eng.prefill(state["prompts"])
        return dict(tokens=np.asarray(first), logits=eng.last_logits())
    need = state["steps"] * (state["k"] + 1)
    if state["kind"] == "request" or max(eng.ctx_len()) + need > state["max_ctx"]:
        first = eng.prefill(state["prompts"])      # a new request, or a sequence that has reached its end
    else:
        first = [-1] * len(state["prompts"])
    text = np.full((state["steps"], len(first), state["k"] + 1), -1, dtype=np.int32)
    for i in range(state["steps"]):
        for b, tokens in enumerate(eng.step(*state["tree"])):
            text[i, b, :len(tokens)] = tokens
    return dict(first=np.asarray(first), tokens=text, logits=eng.last_logits())


# ------------------------------------------------------------------------------------------- accounting


def _forward_work(cfg, batch, new_rows, ctx, head_rows, elt):
    """Bytes and operations of one pass of `new_rows` rows per sequence over the decoder: every weight
    once, the live cache of `ctx` tokens once and the new rows' K and V out and in, the logits out."""
    rows = batch * new_rows
    layer = cfg.layer_params()
    kv_row = 2 * cfg.n_kv_heads * cfg.head_dim * elt
    nbytes = elt * (cfg.n_layers * layer + cfg.vocab * cfg.d_model) + 4 * head_rows * cfg.vocab
    nbytes += batch * cfg.n_layers * kv_row * (ctx + 2 * new_rows)
    flops = 2.0 * (rows * cfg.n_layers * layer + head_rows * cfg.vocab * cfg.d_model)
    flops += 4.0 * rows * cfg.n_layers * cfg.n_q_heads * cfg.head_dim * (ctx + new_rows / 2)
    return float(nbytes), flops


def work(case):
    cfg, tree = _config(case), _tree(case)
    elt = 2 if case["dtype"] == "bf16" else 4
    d2 = cfg.d_model ** 2
    lens, B = _prompt_lengths(case), case["batch"]
    n_anchor = sum(tree.anchor)
    if case["kind"] == "train":
        n = case["prompt"]
        nbytes, flops = _forward_work(cfg, 1, 2 * n, 0, 2 * n, elt)
        flops -= 2.0 * n * (cfg.n_layers // 2) * cfg.layer_params()      # the mapped rows skip the lower half
        return dict(bytes=nbytes + elt * d2, flops=flops + 2.0 * n * d2)
    nbytes = flops = 0.0
    if case["kind"] in ("prefill", "request"):
        nbytes += elt * (cfg.n_layers * cfg.layer_params() + cfg.vocab * cfg.d_model + cfg.k * d2)
        for n in lens:
            by, fl = _forward_work(cfg, 1, n, 0, 1 + cfg.k, elt)
            nbytes += 2 * cfg.n_kv_heads * cfg.head_dim * elt * cfg.n_layers * n + 4 * (1 + cfg.k) * cfg.vocab
            flops += fl + 2.0 * cfg.k * d2
    if case["kind"] in ("decode", "request"):
        ctx = sum(lens) / B + case["steps"] / 2
        # pseudo rows exist from the middle of the decoder on
        rows = tree.n_nodes + cfg.k * n_anchor / 2
        by, fl = _forward_work(cfg, B, rows, ctx, 0, elt)
        head = B * (tree.n_nodes + cfg.k * n_anchor)
        by += elt * cfg.k * d2
        fl += 2.0 * (head * cfg.vocab * cfg.d_model + B * n_anchor * cfg.k * d2)
        nbytes += case["steps"] * by + 4 * head * cfg.vocab
        flops += case["steps"] * fl
    return dict(bytes=float(nbytes), flops=float(flops))


def tolerance(case):
    # About four times what the weight-streaming kernels and the plain fp32 ones (other order of every
    # sum) differ by on these cases, or the fp32 model and an fp64 evaluation: f32 1.2e-7 (max 5e-7); bf16
    # 7B and 13B up to 1.6e-4 (max 9e-4), 34B 9.6e-4 (5e-3), the training forward's 256 rows of random
    # text 4.6e-4 (3e-3).  What makes bf16 models differ is that an entry of the cache may round to the
    # neighbouring bf16 value; the small ones happen to show 4e-6 without such an entry, and one entry
    # there is worth up to 1e-4.
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    if case["shape"].startswith("tiny"):
        return {"rel": 1e-4, "max": 1e-3}
    if case["shape"] == "34b" or case["kind"] == "train":
        return {"rel": 4e-3, "max": 2e-2}
    return {"rel": 1e-3, "max": 5e-3}
