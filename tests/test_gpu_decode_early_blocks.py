"""Weights requested into LDS ahead of a stage's barrier: widths just over one round of blocks (a second round exists, its last
block is partial), residual rows in one and in two tiles (rounds of 2048 and 1536 16-bit columns), and passes whose rows just
fit ahead of the early blocks (4 rows of 2064 columns, 8 of 1040, 5 of 1552 and 1664 in two tiles, in 32 KB) and just do not
(5, 9 and 6 rows).  The early blocks of two tiles fill the LDS region of the input to its last byte.  Hidden states of one-row
greedy passes are the oracle's; self-speculative jobs leave the same ids and hidden states as they, bit for bit."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import rel_err_rows, same_until_near_tie

pytestmark = pytest.mark.gpu

SHAPES = {
    "bf16": dict(d_model=1040, ffn_dim=2064, n_q_heads=9, n_kv_heads=9, head_dim=128, dtype="bf16"),
    "bf16_hd64": dict(d_model=1040, ffn_dim=2064, n_q_heads=34, n_kv_heads=17, head_dim=64, dtype="bf16"),
    "two_tiles": dict(d_model=4112, ffn_dim=1040, n_q_heads=9, n_kv_heads=9, head_dim=128, dtype="bf16"),   # (one round of residual blocks)
    "two_tiles_two_rounds": dict(d_model=4112, ffn_dim=1552, n_q_heads=13, n_kv_heads=13, head_dim=128, dtype="bf16"),
    "f32": dict(d_model=528, ffn_dim=1040, n_q_heads=9, n_kv_heads=9, head_dim=64, dtype="f32"),
}


@pytest.mark.parametrize("name", SHAPES)
def test_early_blocks_keep_the_ids(name):
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name=name, n_layers=2, vocab=528, rope_base=10000.0, rms_eps=1e-5, **SHAPES[name])
    w = W.Workload(m, exit_layer=1, draft_len=3, n_prompt=20, n_new=24, resid_scale=0.1, gain_jitter=0.1)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(m, ws, np.float32, emulate_bf16_act=m.dtype == "bf16")
    ref = O.greedy_full(om, prompt, 8, want_hidden=True)
    gm = LsModel(m, ws, max_seq=w.n_prompt + w.n_new + 17)
    rows = w.n_prompt + w.n_new - 1                      # positions whose token the job has emitted or been given

    def job(exit_layer, d):
        cap = gm.debug_capture(True)
        toks, _ = gm.generate(prompt, w.n_new, exit_layer, d)
        h = cap.cpu().numpy()[:, :rows].copy()
        gm.debug_capture(False)
        return toks, h

    ar, want = job(0, 0)
    n = w.n_prompt + same_until_near_tie(ar[:8], ref.tokens, ref.margins) - 1
    for l in range(m.n_layers):
        assert rel_err_rows(want[l][:n], ref.hidden[l + 1][:n]) < (2e-2 if m.dtype == "bf16" else 1e-4), l
    for d in (1, 3, 4, 5, 7, 8, 15):
        toks, got = job(1, d)
        assert toks == ar, d
        assert np.array_equal(got, want), d
    gm.close()
