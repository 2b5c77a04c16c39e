"""Scoring and the layer probe in wide passes give the bits of the decode kernels' 16-row passes: predictions, margins
and every layer's hidden states, over what decides the order of a sum there (items of one and of several attention
tiles, one and two tiles of residual rows to a workgroup, both head widths, query groups, an odd number of K steps) and over
what decides tiles here (ragged rows and columns, several chunks)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _case(name, n_prompt, **kw):
    base = dict(n_layers=3, n_q_heads=4, n_kv_heads=2, head_dim=128, d_model=512, ffn_dim=1472, vocab=1040,
                rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    base.update(kw)
    return W.Workload(W.ModelConfig(name=name, **base), exit_layer=1, draft_len=3, n_prompt=n_prompt, n_new=8,
                      resid_scale=0.3, gain_jitter=0.1)


CASES = [(_case("rows17", 17), 64), (_case("rows33", 33), 34), (_case("rows257", 257), 8192),
         # an item per tile / three tiles per item (40 heads of both kinds), head_dim 64
         (_case("hd64", 300, n_q_heads=8, n_kv_heads=8, head_dim=64, d_model=320, ffn_dim=1344), 400),
         (_case("heads", 700, n_layers=2, n_q_heads=40, n_kv_heads=40, head_dim=64, d_model=256, ffn_dim=320), 1100),
         (_case("items", 700, n_layers=2, n_q_heads=30, n_kv_heads=10, head_dim=128, d_model=256, ffn_dim=320), 3000),
         (_case("group4", 130, n_q_heads=4, n_kv_heads=1, vocab=5008), 8192),
         # more than four units of residual columns to a workgroup: two tiles, dealt out to two waves
         (_case("wide", 65, n_layers=2, d_model=5120, ffn_dim=448), 100),
         # two chunks of rows
         (_case("chunks", 2100, n_layers=2, n_q_heads=2, n_kv_heads=1, d_model=256, ffn_dim=448), 2200)]


@pytest.mark.parametrize("w,max_seq", CASES, ids=lambda x: x.model.name if hasattr(x, "model") else str(x))
def test_wide_passes_have_the_bits_of_16_row_passes(w, max_seq):
    from paper_2404_16710_amd import LsModel
    ws, text = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(w.model, ws, max_seq=max_seq)
    n, L = len(text), w.model.n_layers

    def passes(rows):
        gm.set_prompt_tiles(rows)
        cap = gm.debug_capture(True)
        ids, margins = gm.score(text)
        hidden = cap.cpu().numpy()[:, :n].copy()
        gm.debug_capture(False)
        return hidden, ids, margins, gm.score(text, 1), gm.probe_layers(text), gm.get_state()

    want, got = passes(16), passes(0)
    for l in range(L):
        assert np.array_equal(want[0][l], got[0][l]), l
    assert np.isfinite(want[2]).all()
    assert np.array_equal(want[1], got[1]) and np.array_equal(want[2], got[2])
    for a, b in zip(want[3] + want[4], got[3] + got[4]):
        assert np.array_equal(a, b)
    assert want[5] == got[5]
    gm.close()
