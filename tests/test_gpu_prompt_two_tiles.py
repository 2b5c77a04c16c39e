"""Products of the prompt pass that fill many rounds of workgroups: in one launch (gate/up with 130 columns of 256 x 256
tiles, Q/K/V with 99 of 128 x 128), and covered by two tiles, whole rounds of the larger and the rest in a launch of the
smaller.  The latter with every pair of tiles that the rule is known to take, ragged last tiles in rows and columns, and Q/K/V
products whose columns change tile within V and within K.  Reference: the CPU oracle; and for two tiles the same product in 64 x 64 tiles
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
# the workload, and its two tiles (0: 256 x 256, 1: 256 x 128, 2: 128 x 128, 3: 128 x 64, 5: 64 x 64)
TWO = [(_case("gate_up_01", 1537, d_model=704, ffn_dim=10608), (0, 1)), (_case("gate_up_02", 1537, d_model=960, ffn_dim=7024), (0, 2)),
       (_case("gate_up_03", 1537, d_model=576, ffn_dim=10320), (0, 3)), (_case("gate_up_05", 1537, d_model=960, ffn_dim=5040), (0, 5)),
       (_case("gate_up_15", 1537, d_model=1280, ffn_dim=2512), (1, 5)), (_case("gate_up_25", 257, d_model=2048, ffn_dim=11472), (2, 5)),
       (_case("qkv_05", 1537, d_model=960, n_q_heads=48, n_kv_heads=16), (0, 5)),
       (_case("qkv_15", 777, d_model=1280, n_q_heads=52, n_kv_heads=13), (1, 5))]
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


@pytest.mark.parametrize("w,tiles", TWO + [(w, None) for w in ONE], ids=_id)
def test_plans_take_the_tiles_they_are_named_after(w, tiles):
    tile, splits, first, rest = _plan(w, 256)
    m = w.model
    n_out = m.ffn_dim if m.name.startswith("gate_up") else m.q_dim + 2 * m.kv_dim
    assert splits == 1
    assert (rest < 0 and first == n_out) if tiles is None else ((tile, rest) == tiles and 0 < first < n_out)
    if m.name == "qkv_05":
        assert m.q_dim + m.kv_dim < first
    if m.name == "qkv_15":
        assert m.q_dim < first < m.q_dim + m.kv_dim


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
