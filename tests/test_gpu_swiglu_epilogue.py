"""gate|up projections of more than 128 rows that apply SwiGLU themselves, at the edges of their tiles: the cache
that a prompt leaves and the logits of the step behind it, against the CPU oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2410_20488_amd import synth
from tests.gpu_common import compare_cache, make_engine
from tests.helpers import cpu_weights, make_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d_ffn,length", [
    (16, 130), (96, 194), (128, 257), (208, 258), (1040, 322), (2064, 514), (4112, 140),   # whole 16-column tiles
    (360, 300), (4, 200)])                                                                 # not: the separate kernel
def test_prompt_rows_through_the_swiglu_epilogue(d_ffn, length):
    cfg = dataclasses.replace(synth.CONFIGS["tiny_bf16"], d_ffn=d_ffn)
    w = synth.make_weights(cfg, DEV)
    orc = make_oracle(cfg, cpu_weights(w), dtype=torch.float64)
    eng = make_engine(cfg, w, max_ctx=length + 16, max_nodes=1, max_rows=64)
    prompt = synth.prompt_tokens(cfg.seed + 5, length, cfg.vocab).tolist()
    assert eng.prefill([prompt]) == [orc.prefill(prompt)]
    compare_cache(eng, orc, cfg)
    r = orc.step(parent=[-1], rank=[0], anchor=[1])
    assert eng.step([-1], [0], [1])[0] == r.tokens
    ref = r.logits.double().numpy()
    assert np.abs(eng.last_logits()[0] - ref).max() / ref.std() <= 2e-2
