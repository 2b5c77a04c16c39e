"""A row of a 16-bit model that is wider than the LDS region of a stage's input (65536 columns) goes through a normalised
product in chunks, each with its own gains: a one-row pass leaves the hidden states that the same row has in a pass of
several rows bit for bit, and the oracle's."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import rel_err_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model", [65536, 65552, 131088])     # one chunk; the second just begun; two full ones and a third
def test_one_row_of_a_wide_model(d_model):
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name="wide_row", n_layers=2, n_q_heads=1, n_kv_heads=1, head_dim=64, d_model=d_model, ffn_dim=32,
                      vocab=32, rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    w = W.Workload(m, exit_layer=1, draft_len=3, n_prompt=2, n_new=4, resid_scale=1.0, gain_jitter=0.5)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    ref = O.greedy_full(O.OracleModel(m, ws, np.float32, emulate_bf16_act=True), prompt, 1, want_hidden=True)
    gm = LsModel(m, ws, max_seq=32)

    def hidden(ids):
        cap = gm.debug_capture(True)
        gm.prefill(ids)
        h = cap.cpu().numpy()[:, :len(ids)].copy()
        gm.debug_capture(False)
        return h

    one, two = hidden(prompt[:1]), hidden(prompt)
    assert np.array_equal(one[:, 0], two[:, 0])
    for l in range(m.n_layers):
        assert rel_err_rows(two[l], ref.hidden[l + 1][:2]) < 2e-2
    gm.close()
