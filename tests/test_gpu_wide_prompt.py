"""Prompts of 17 to 31 ids, which would be two 16-row passes, go through the layers together and leave what those passes
leave: first token and margin, state, cache (seen through the rounds that follow) and hidden states, bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_prompt", [17, 24, 31])
@pytest.mark.parametrize("heads", [(4, 2, 128), (6, 2, 64)])
def test_short_prompts_in_one_wide_pass(n_prompt, heads):
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name="short", n_layers=3, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=heads[2], d_model=512,
                      ffn_dim=1472, vocab=1040, rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    w = W.Workload(m, exit_layer=1, draft_len=4, n_prompt=n_prompt, n_new=20, resid_scale=0.3, gain_jitter=0.1)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(m, ws, max_seq=100)

    def passes(rows):
        gm.set_prompt_tiles(rows)
        cap = gm.debug_capture(True)
        gm.prefill(prompt)
        hidden = cap.cpu().numpy()[:, :n_prompt].copy()
        gm.debug_capture(False)
        out = [gm.get_state()]
        gm.draft(1, 4); gm.verify(1, 4)
        out.append(gm.peek_round(4))
        gm.draft(2, 3); gm.verify(2, 3)
        out.append(gm.peek_round(3))
        toks, st = gm.generate(prompt, w.n_new, 1, 4)
        first = toks[0]
        out += [toks, st.rounds, gm.generate(prompt, 1, 1, 4)[0], gm.generate(prompt, w.n_new, 1, 4, eos_id=first)[0],
                gm.generate_early_exit(prompt, 6, 2)[0]]
        return hidden, out

    want, got = passes(16), passes(0)
    assert np.array_equal(want[0], got[0])
    assert want[1] == got[1]
    gm.close()
