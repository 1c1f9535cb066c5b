"""Prefill in chunks of up to 1024 rows (bf16 models): prompt lengths at the edges of the chunk, of
the attention kernel's 256-row blocks (64 rows with four query heads per KV head) and of its 16-row
tiles, against the CPU oracle: the cache the prompt leaves, and the logits of the step behind it."""
import numpy as np
import pytest
import torch

from paper_2410_20488_amd import synth
from tests.gpu_common import compare_cache, make_engine
from tests.helpers import cpu_weights, make_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("name,length", [
    ("tiny_bf16", 2), ("tiny_bf16", 17), ("tiny_bf16", 18), ("tiny_bf16", 257), ("tiny_bf16", 258), ("tiny_bf16", 1025),
    ("tiny_bf16", 1026), ("tiny_bf16", 2100), ("tiny_gqa", 65), ("tiny_gqa", 66), ("tiny_gqa", 300), ("tiny_gqa", 1041)])
def test_prompt_lengths_at_chunk_and_tile_edges(name, length):
    """(A prompt of n tokens sends n - 1 rows through the chunks; its last token is the root of the
    first step.)  A short prompt before it leaves stale rows in every buffer."""
    cfg = synth.CONFIGS[name]
    w = synth.make_weights(cfg, DEV, with_bias=True)
    orc = make_oracle(cfg, cpu_weights(w), dtype=torch.float64)
    eng = make_engine(cfg, w, max_ctx=length + 40, max_nodes=10, max_rows=64)
    prompt = synth.prompt_tokens(cfg.seed + 11, length, cfg.vocab).tolist()
    eng.prefill([synth.prompt_tokens(3, min(length, 50), cfg.vocab).tolist()])
    assert eng.prefill([prompt]) == [orc.prefill(prompt)]
    compare_cache(eng, orc, cfg)
    tree = synth.full_tree((3, 2)[:cfg.k], "root")
    args = dict(parent=list(tree.parent), rank=list(tree.rank), anchor=list(tree.anchor))
    cand = synth.prompt_tokens(5, tree.n_nodes, cfg.vocab).tolist()
    r = orc.step(**args, node_tokens=cand)
    eng.step_with_candidates(args["parent"], args["rank"], args["anchor"], [cand])
    ref = r.logits.double().numpy()
    assert np.abs(eng.last_logits()[0] - ref).max() / ref.std() <= 2e-2
    # equal inputs give equal bits, whatever an engine did before
    other = make_engine(cfg, w, max_ctx=length + 40, max_nodes=10, max_rows=64)
    other.prefill([prompt])
    other.step_with_candidates(args["parent"], args["rank"], args["anchor"], [cand])
    assert np.array_equal(other.last_logits(), eng.last_logits())
