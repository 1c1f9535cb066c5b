"""The first step of a prefill resumes at the first prediction layer where the chunks already hold the last
prompt token: first token, drafts, logits and cache against the CPU oracle for every place that layer can
have, lengths at which the step does and does not resume, and sequences of different lengths."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2410_20488_amd import synth
from tests.gpu_common import compare_cache, make_engine
from tests.helpers import cpu_weights, make_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(cfg, lengths):
    w = synth.make_weights(cfg, DEV, with_bias=cfg.k > 0)
    eng = make_engine(cfg, w, max_ctx=max(lengths) + 24, max_batch=len(lengths), max_nodes=1, max_rows=64)
    prompts = [synth.prompt_tokens(cfg.seed + n, n, cfg.vocab).tolist() for n in lengths]
    for _ in range(2):                          # the second time over the first one's buffers and cache
        first = eng.prefill(prompts)
        logits = eng.last_logits()
    for b, prompt in enumerate(prompts):
        orc = make_oracle(cfg, cpu_weights(w), dtype=torch.float64)
        assert orc.prefill(prompt) == first[b]
        assert np.isfinite(logits[b]).all()
        if b == 0 and len(prompts) == 1:
            compare_cache(eng, orc, cfg)
    # one more step from the state that the prefill left
    orcs = []
    for prompt in prompts:
        orc = make_oracle(cfg, cpu_weights(w), dtype=torch.float64)
        orc.prefill(prompt)
        orcs.append(orc.step(parent=[-1], rank=[0], anchor=[1 if cfg.k else 0]))
    got = eng.step([-1], [0], [1 if cfg.k else 0])
    logits = eng.last_logits()
    for b, r in enumerate(orcs):
        assert got[b] == r.tokens
        ref = r.logits.double().numpy()
        assert np.abs(logits[b] - ref).max() / ref.std() <= 2e-2


@pytest.mark.parametrize("layers", [(0, 0, 0), (1, 2, 4), (2, 2, 2), (3, 3, 3), (4, 4, 4), ()])
@pytest.mark.parametrize("length", [2, 16, 130, 256, 257, 300])
def test_resumed_first_step(layers, length):
    cfg = dataclasses.replace(synth.CONFIGS["tiny_bf16"], k=len(layers), firp_layers=layers or None)
    _check(cfg, [length])


@pytest.mark.parametrize("lengths", [(130, 17, 2), (300, 257, 40), (70, 1)])
def test_resumed_first_step_of_several_sequences(lengths):
    _check(synth.CONFIGS["tiny_gqa"], list(lengths))
