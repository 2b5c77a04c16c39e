"""The prompt pass's matrix products with tiles sent straight into LDS, at the sizes where they can go
wrong: one row past and one short of a tile height, ragged last tiles in rows and columns, heads of
both widths, products whose K is split over several workgroups, with a capture and without, and
row counts that reach the tallest tile.  Reference: the CPU oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import NEAR_TIE, NOISE_BAND, rel_err_rows, same_until_near_tie

pytestmark = pytest.mark.gpu


def _case(name, n_prompt, **kw):
    base = dict(n_layers=2, n_q_heads=4, n_kv_heads=2, head_dim=128, d_model=512, ffn_dim=1472, vocab=1040,
                rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    base.update(kw)
    return W.Workload(W.ModelConfig(name=name, **base), exit_layer=1, draft_len=3, n_prompt=n_prompt, n_new=8,
                      resid_scale=0.1, gain_jitter=0.1)


CASES = [_case("rows32", 32), _case("rows65", 65), _case("rows127", 127), _case("rows257", 257),
         _case("hd64", 100, n_q_heads=8, n_kv_heads=4, head_dim=64, d_model=320, ffn_dim=1344),
         # d_model and ffn that are multiples of 64 but of no wider tile
         _case("narrow", 161, n_q_heads=3, n_kv_heads=3, d_model=448, ffn_dim=1088),
         # 16384 SwiGLU columns: the tallest and widest tile, with a ragged last one in rows
         _case("tall", 1999, n_q_heads=2, n_kv_heads=1, d_model=256, ffn_dim=16384)]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.model.name)
def test_prompt_products_match_oracle(w):
    from paper_2404_16710_amd import LsModel
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(w.model, ws, np.float32, emulate_bf16_act=True)
    gm = LsModel(w.model, ws, max_seq=w.n_prompt + w.n_new + 17)
    L = w.model.n_layers
    ref = O.greedy_full(om, prompt, 3, want_hidden=True)
    cap = gm.debug_capture(True)
    gm.prefill(prompt)
    got = cap.cpu().numpy()[:, :w.n_prompt]
    gm.debug_capture(False)
    for l in range(L):
        assert rel_err_rows(got[l], ref.hidden[l + 1][:w.n_prompt]) < 2e-2, l
    gm.prefill(prompt)
    _, last, _ = gm.get_state()
    if ref.margins[0] >= NEAR_TIE:
        assert last == ref.tokens[0]
        gm.draft(L, 1)                                   # the full model's next step, on the cache of the prompt pass
        ids, _, margins, _, _ = gm.peek_round(1)
        if ref.margins[1] >= NOISE_BAND:                 # (rounding noise of a logit: below half the band)
            assert ids[0] == ref.tokens[1]
            assert abs(margins[0] - ref.margins[1]) < NOISE_BAND
    toks, _ = gm.generate(prompt, 3, 1, 2)
    same_until_near_tie(toks, ref.tokens, ref.margins)
    gm.close()


# One prompt pass with a capture of the hidden states and one without leave the same cache, bit for bit, also where the
# products' K is split (so that a captured job has the ids of the same job without it).
@pytest.mark.parametrize("n", [33, 129, 300])
def test_a_captured_prompt_pass_is_the_same_pass(n):
    from paper_2404_16710_amd import LsModel
    w = _case("capture", n, d_model=512, ffn_dim=4096)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(w.model, ws, max_seq=n + 17)
    margins = []
    for on in (False, True, False):
        gm.debug_capture(on)
        gm.prefill(prompt)
        gm.draft(w.model.n_layers, 6)
        ids, _, m, _, _ = gm.peek_round(6)
        margins.append((list(ids), [float(x) for x in m]))
    gm.debug_capture(False)
    gm.close()
    assert margins[0] == margins[1] == margins[2]
