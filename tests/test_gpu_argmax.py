"""The greedy token and the draft lists against the step's own logits: ties go to the lower id, NaN is never
chosen, infinities order like numbers; vocabularies at the edges of the selection kernel's segments, of its
groups of four tokens and of the path for rows that are not 16-byte aligned."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2410_20488_amd import synth
from tests.gpu_common import make_engine

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _order(row):
    """Ids by larger logit, then lower id; NaN last."""
    v = np.where(np.isnan(row), -np.inf, row.astype(np.float64))
    ids = np.lexsort((np.arange(len(v)), -v))
    return [i for i in ids if not np.isnan(row[i]) and row[i] != -np.inf]


@pytest.mark.parametrize("name,vocab,b_max", [
    ("tiny", 8, 8), ("tiny", 33, 3), ("tiny", 1003, 8), ("tiny", 4099, 16), ("tiny_bf16", 8, 8), ("tiny_bf16", 1004, 16),
    ("tiny_bf16", 2052, 8), ("tiny_bf16", 8196, 8), ("tiny_bf16", 16400, 1)])
@pytest.mark.parametrize("special", [False, True])
def test_selection_follows_the_logits(name, vocab, b_max, special):
    cfg = dataclasses.replace(synth.CONFIGS[name], vocab=vocab)
    w = synth.make_weights(cfg, DEV)
    head = w["lm_head"]
    head[vocab // 2:vocab // 2 * 2] = head[:vocab // 2].clone()     # every logit at least twice
    if special:
        head[1::5] = 3e38                                           # infinities of either sign, and NaN
        head[2::7, 0] = float("nan")
    nodes = 24                                                      # 24 rows, then a row, of which each has its own scale
    eng = make_engine(cfg, w, max_ctx=80, max_nodes=nodes, max_rows=64, b_max=b_max)
    first = eng.prefill([synth.prompt_tokens(3, 30, vocab).tolist()])
    for step in range(2):
        logits = eng.last_logits()[0]
        real = logits.shape[0] - cfg.k
        if step == 0:
            assert first[0] == _order(logits[0])[0]
        drafts, _ = eng.drafts()
        if real == 1 and cfg.k:
            for i in range(cfg.k):
                want = _order(logits[real + i])[:b_max]
                assert drafts[0][i].tolist()[:len(want)] == want
        cand = synth.prompt_tokens(5, nodes, vocab).tolist()
        tree = synth.with_anchors(synth.random_tree(3, nodes, cfg.k, min(b_max, 4), 0.5), "root") if b_max >= 4 else None
        if tree is None:
            break
        got = eng.step_with_candidates(list(tree.parent), list(tree.rank), list(tree.anchor), [cand])[0]
        logits = eng.last_logits()[0]
        for node, token in zip(eng.last_path()[0], got):
            assert token == _order(logits[node])[0]
