"""Weights requested into LDS ahead of a stage's barrier: widths just over one round of blocks (a second round exists, its last
block is partial), residual rows in one and in two tiles, and passes whose rows just fit ahead of the early blocks (4 rows of
2064 columns, 8 of 1040, in 32 KB) and just do not (5 and 9 rows).  Self-speculative ids equal the one-row greedy ids, and
both the oracle's up to near-ties."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import same_until_near_tie

pytestmark = pytest.mark.gpu

SHAPES = {
    "bf16": dict(d_model=1040, ffn_dim=2064, n_q_heads=9, n_kv_heads=9, head_dim=128, dtype="bf16"),
    "bf16_hd64": dict(d_model=1040, ffn_dim=2064, n_q_heads=34, n_kv_heads=17, head_dim=64, dtype="bf16"),
    "two_tiles": dict(d_model=4112, ffn_dim=1040, n_q_heads=9, n_kv_heads=9, head_dim=128, dtype="bf16"),
    "f32": dict(d_model=528, ffn_dim=1040, n_q_heads=9, n_kv_heads=9, head_dim=64, dtype="f32"),
}


@pytest.mark.parametrize("name", SHAPES)
def test_early_blocks_keep_the_ids(name):
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name=name, n_layers=2, vocab=528, rope_base=10000.0, rms_eps=1e-5, **SHAPES[name])
    w = W.Workload(m, exit_layer=1, draft_len=3, n_prompt=20, n_new=24, resid_scale=0.1, gain_jitter=0.1)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(m, ws, np.float32, emulate_bf16_act=m.dtype == "bf16")
    ref = O.greedy_full(om, prompt, 8)
    gm = LsModel(m, ws, max_seq=w.n_prompt + w.n_new + 17)
    ar, _ = gm.generate(prompt, w.n_new, 0, 0)
    same_until_near_tie(ar[:8], ref.tokens, ref.margins)
    for d in (1, 3, 4, 7, 8, 15):
        toks, _ = gm.generate(prompt, w.n_new, 1, d)
        assert toks == ar, d
    gm.close()
