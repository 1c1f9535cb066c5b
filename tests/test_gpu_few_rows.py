"""Layers of up to 16 rows run on projections that do the next elementwise step themselves (residual and
norm, SwiGLU, row scale): whole-step parity with the CPU oracle at the edges of their rows, of their
16-column tiles, of the tiles per workgroup and of K."""
import dataclasses

import pytest

from paper_2410_20488_amd import synth
from tests.gpu_common import compare_cache, run_lockstep

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# rows of a step with k pseudo rows: nodes, nodes + k from the FIRP layer on
CASES = [
    # one tile per workgroup; K of the down projection not a multiple of 64 (352)
    ("tiny_gqa", {}, 1), ("tiny_gqa", {}, 2), ("tiny_gqa", {}, 14),
    ("tiny_gqa", {}, 15),                                    # 15 rows, then 17: leaves these kernels midway
    ("tiny_gqa", {"d_ffn": 360}, 3),                         # gate rows end inside a tile: never on these kernels
    # two output tiles per workgroup, the last workgroup half empty: gate|up, lm-head, residual + norm
    ("tiny_bf16", {"d_ffn": 4112, "vocab": 4120}, 5), ("tiny_bf16", {"d_model": 4128, "d_ffn": 64}, 4),
    # more tiles per workgroup (gate|up 3 and 4, lm-head 3 to 8)
    ("tiny_bf16", {"d_ffn": 8208, "vocab": 8260}, 1), ("tiny_bf16", {"d_ffn": 12304, "vocab": 12308}, 4),
    ("tiny_bf16", {"vocab": 20500}, 13), ("tiny_bf16", {"vocab": 36004}, 4),
    ("tiny_bf16", {"n_q_heads": 72, "n_kv_heads": 36, "vocab": 16388}, 4),
]


@pytest.mark.parametrize("name,change,nodes", CASES)
def test_steps_of_few_rows(name, change, nodes):
    cfg = dataclasses.replace(synth.CONFIGS[name], **change)
    w = synth.make_weights(cfg, DEV, with_bias=True)
    tree = synth.with_anchors(synth.random_tree(nodes, nodes, cfg.k, 4, 0.5), "root") if nodes > 1 else synth.chain_tree(0, "root")
    rep, eng, orc = run_lockstep(cfg, w, tree, prompt_len=70, n_steps=6, tol=2e-2)
    assert rep.steps == 6
    compare_cache(eng, orc, cfg)
