"""Scoring and the layer probe in wide passes give the bits of the decode kernels' 16-row passes: predictions, margins
and every layer's hidden states, over what decides the order of a sum there (items of one and of several attention
tiles, one and two tiles of residual rows to a workgroup, both head widths, query groups, an odd number of K steps) and over
what decides tiles here (ragged rows and columns, several chunks, every tile in every product, products that two tiles
cover)."""
import ctypes

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


def _passes(gm, text, rows, tile=0):
    gm.set_prompt_tiles(rows)
    gm.debug_prompt_plan(tile, 0)
    cap = gm.debug_capture(True)
    ids, margins = gm.score(text)
    hidden = cap.cpu().numpy()[:, :len(text)].copy()
    gm.debug_capture(False)
    return hidden, ids, margins, gm.score(text, 1), gm.probe_layers(text), gm.get_state()


def _assert_same(want, got, what=""):
    for l, (a, b) in enumerate(zip(want[0], got[0])):
        assert np.array_equal(a, b), (l, what)
    assert np.isfinite(want[2]).all()
    assert np.array_equal(want[1], got[1]) and np.array_equal(want[2], got[2]), what
    for a, b in zip(want[3] + want[4], got[3] + got[4]):
        assert np.array_equal(a, b), what
    assert want[5] == got[5]


@pytest.mark.parametrize("w,max_seq", CASES, ids=lambda x: x.model.name if hasattr(x, "model") else str(x))
def test_wide_passes_have_the_bits_of_16_row_passes(w, max_seq):
    from paper_2404_16710_amd import LsModel
    ws, text = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(w.model, ws, max_seq=max_seq)
    _assert_same(_passes(gm, text, 16), _passes(gm, text, 0))
    gm.close()


# Every tile that takes such sums, in the four products of a layer and in the head.  Pairs of steps along K in Q/K/V, gate/up and
# head; O; down: 8, 8, 23; 7, 6, 18; 5, 4, 9, i.e. chains of none to three blocks, the last block whole and half; the
# 128 columns that a tile is wide divide the q and the k/v widths, and a ragged tile is left in rows, d_model, ffn and vocabulary.
@pytest.mark.parametrize("w", [_case("pairs8", 300), _case("pairs7", 300, n_layers=2, d_model=448, n_q_heads=3, n_kv_heads=3, ffn_dim=1152),
                               _case("pairs5", 270, n_layers=2, d_model=320, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn_dim=576)],
                         ids=lambda w: w.model.name)
def test_every_tile_has_the_bits_of_16_row_passes(w):
    from paper_2404_16710_amd import LsModel
    ws, text = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(w.model, ws, max_seq=320)
    want = _passes(gm, text, 16)
    for tile in range(2, 7):
        _assert_same(want, _passes(gm, text, 0, tile), tile)
    gm.close()


# gate/up in tiles of 256 x 128 and of 128 x 128 with 64 x 64 behind them; Q/K/V in 256 x 128 and 64 x 64, with the change within K
@pytest.mark.parametrize("w", [_case("gate_up_15", 1537, n_layers=1, d_model=1280, n_q_heads=2, n_kv_heads=1, ffn_dim=2560),
                               _case("gate_up_25", 257, n_layers=1, d_model=2048, n_q_heads=2, n_kv_heads=1, ffn_dim=11520),
                               _case("qkv_15", 777, n_layers=1, d_model=1280, n_q_heads=52, n_kv_heads=13, ffn_dim=320)],
                         ids=lambda w: w.model.name)
def test_two_tiles_have_the_bits_of_16_row_passes(w):
    import torch
    from paper_2404_16710_amd import LsModel, lib
    m, plan = w.model, (ctypes.c_int32 * 4)()
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if m.name.startswith("gate_up"):
        lib().ls_mm_plan(w.n_prompt, m.ffn_dim, 2, m.d_model, 0, 0, 1, n_cu, 1, plan)
    else:
        lib().ls_mm_plan(w.n_prompt, m.q_dim + 2 * m.kv_dim, 1, m.d_model, m.q_dim, m.kv_dim, 1, n_cu, 1, plan)
        assert m.q_dim < plan[2] < m.q_dim + m.kv_dim
    assert (plan[0], plan[3]) == tuple(map(int, m.name[-2:]))
    ws, text = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(m, ws, max_seq=w.n_prompt + 20)
    _assert_same(_passes(gm, text, 16), _passes(gm, text, 0))
    gm.close()
