"""Products of the prompt pass that are covered by two tiles (whole rounds of the larger, the rest in a launch of the
smaller): gate/up with 130 columns of 256 x 256 tiles of which 128 make four rounds, and Q/K/V with 99 of 256 x 128 of which 96
make three; ragged last tiles in rows and columns.  Reference: the CPU oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import rel_err_rows

pytestmark = pytest.mark.gpu


def _case(name, n_prompt, **kw):
    base = dict(n_layers=1, n_q_heads=2, n_kv_heads=1, head_dim=128, d_model=256, ffn_dim=320, vocab=1040,
                rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    base.update(kw)
    return W.Workload(W.ModelConfig(name=name, **base), exit_layer=1, draft_len=3, n_prompt=n_prompt, n_new=8,
                      resid_scale=0.1, gain_jitter=0.1)


@pytest.mark.parametrize("w", [_case("gate_up", 1999, ffn_dim=130 * 128 - 64), _case("qkv", 1999, n_q_heads=33, n_kv_heads=33)],
                         ids=lambda w: w.model.name)
def test_products_in_two_tiles_match_oracle(w):
    from paper_2404_16710_amd import LsModel
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(w.model, ws, np.float32, emulate_bf16_act=True)
    ref = O.greedy_full(om, prompt, 1, want_hidden=True)
    gm = LsModel(w.model, ws, max_seq=w.n_prompt + w.n_new + 17)
    cap = gm.debug_capture(True)
    gm.prefill(prompt)
    got = cap.cpu().numpy()[0, :w.n_prompt]
    assert rel_err_rows(got, ref.hidden[1][:w.n_prompt]) < 2e-2
    gm.close()
