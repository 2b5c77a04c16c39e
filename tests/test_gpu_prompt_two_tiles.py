"""Products of the prompt pass that fill many rounds of workgroups: in one launch (gate/up with 130 columns of 256 x 256
tiles, Q/K/V with 99 of 128 x 128), and covered by two tiles, whole rounds of the larger and the rest in a launch of the
smaller.  The latter with every tile that the rest may have, ragged last tiles in rows and columns, and a Q/K/V product
whose columns change tile within V.  Reference: the CPU oracle; and for two tiles the same product in 64 x 64 tiles
alone, whose sums are the same, bit for bit."""
import ctypes

import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import rel_err_rows


def _case(name, n_prompt, **kw):
    base = dict(n_layers=1, n_q_heads=2, n_kv_heads=1, head_dim=128, d_model=256, ffn_dim=320, vocab=1040,
                rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    base.update(kw)
    return W.Workload(W.ModelConfig(name=name, **base), exit_layer=1, draft_len=3, n_prompt=n_prompt, n_new=8,
                      resid_scale=0.1, gain_jitter=0.1)


ONE = [_case("gate_up", 1999, ffn_dim=130 * 128 - 64), _case("qkv", 1999, n_q_heads=33, n_kv_heads=33)]
# the workload, and the tile of the rest (1: 256 x 128, 2: 128 x 128, 4: 64 x 128, 5: 64 x 64)
TWO = [(_case("gate_up_1", 1537, d_model=448, ffn_dim=11392), 1), (_case("gate_up_2", 1537, d_model=576, ffn_dim=7056), 2),
       (_case("gate_up_4", 900, d_model=448, ffn_dim=10320), 4), (_case("gate_up_5", 1537, d_model=512, ffn_dim=5072), 5),
       (_case("qkv_5", 1537, d_model=512, n_q_heads=48, n_kv_heads=16), 5)]
_id = lambda x: x.model.name if hasattr(x, "model") else ""


def _plan(w, n_cu):
    """(tile, splits, first, rest) of the product that the workload is named after."""
    from paper_2404_16710_amd import lib
    m, out = w.model, (ctypes.c_int32 * 4)()
    if m.name.startswith("gate_up"):
        lib().ls_mm_plan(w.n_prompt, m.ffn_dim, 2, m.d_model, 0, 0, 1, n_cu, 0, out)
    else:
        lib().ls_mm_plan(w.n_prompt, m.q_dim + 2 * m.kv_dim, 1, m.d_model, m.q_dim, m.kv_dim, 1, n_cu, 0, out)
    return list(out)


@pytest.mark.parametrize("w,rest", TWO + [(w, -1) for w in ONE], ids=_id)
def test_plans_take_the_tiles_they_are_named_after(w, rest):
    tile, splits, first, r = _plan(w, 256)
    m = w.model
    n_out = m.ffn_dim if m.name.startswith("gate_up") else m.q_dim + 2 * m.kv_dim
    assert (r, splits) == (rest, 1)
    assert (first == n_out) if rest < 0 else (0 < first < n_out and tile < rest)
    if m.name == "qkv_5":
        assert m.q_dim + m.kv_dim < first


def _hidden(gm, w, plan):
    gm.debug_prompt_plan(*plan)
    cap = gm.debug_capture(True)
    gm.prefill(W.make_prompt(w))
    h = cap.cpu().numpy()[0, :w.n_prompt].copy()
    gm.debug_capture(False)
    return h


@pytest.mark.gpu
@pytest.mark.parametrize("w", ONE + [w for w, _ in TWO], ids=_id)
def test_products_in_two_tiles_match_oracle(w):
    import torch
    from paper_2404_16710_amd import LsModel
    two = w not in ONE
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert (_plan(w, n_cu)[3] >= 0) == two
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(w.model, ws, np.float32, emulate_bf16_act=True)
    ref = O.greedy_full(om, prompt, 1, want_hidden=True)
    gm = LsModel(w.model, ws, max_seq=w.n_prompt + w.n_new + 17)
    got = _hidden(gm, w, (0, 1))
    assert rel_err_rows(got, ref.hidden[1][:w.n_prompt]) < 2e-2
    if two:
        assert np.array_equal(got, _hidden(gm, w, (6, 1)))
    gm.close()
