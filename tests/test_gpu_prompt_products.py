"""The prompt pass's matrix products with tiles sent straight into LDS, at the sizes where they can go
wrong: one row past and one short of a tile height, ragged last tiles in rows and columns, heads of
both widths, products whose K is split over several workgroups, with a capture and without; the tiles that
the shapes choose by themselves, and every tile with every epilogue, forced.  Reference: the CPU oracle."""
import functools

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
         # 16384 SwiGLU columns: the tallest and widest tile for gate and up, with a ragged last one in rows
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


# Every tile in all three epilogues (rows and both kinds of paired columns): 65 and 300 rows and 513 (two full tiles of 256
# rows and one row of a third), column counts that leave a ragged last tile of every width except in Q/K/V, whose tiles
# divide the heads by construction (q and k/v widths of 512 and 256 take all six); and the sums into the residual rows on
# one, two and four workgroups (O: two at most, its K has 8 steps of 64 and a share at least 4).
@functools.lru_cache(maxsize=None)
def _plan_case(hd):
    w = _case(f"plan{hd}", 513, n_q_heads=512 // hd, n_kv_heads=256 // hd, head_dim=hd, d_model=448, ffn_dim=1088)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(w.model, ws, np.float32, emulate_bf16_act=True)
    ref = {}
    for n in (65, 300, 513):
        ref[n] = O.greedy_full(om, prompt[:n], 2, want_hidden=True)
    return w, ws, prompt, ref


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("tile", [1, 2, 3, 4, 5, 6])
def test_every_tile_and_split_matches_oracle(tile, hd):
    from paper_2404_16710_amd import LsModel
    w, ws, prompt, refs = _plan_case(hd)
    L = w.model.n_layers
    gm = LsModel(w.model, ws, max_seq=2048)                  # room for the partial sums of four splits at every n
    cap = gm.debug_capture(True)
    for n, ref in refs.items():
        by_split = []
        for splits in (1, 2, 4):
            print(f"[prompt plan] tile {tile} splits {splits} rows {n} head_dim {hd}", flush=True)
            gm.debug_prompt_plan(tile, splits)
            cap.zero_()
            gm.prefill(prompt[:n])
            got = cap.cpu().numpy()[:, :n].copy()
            for l in range(L):
                assert rel_err_rows(got[l], ref.hidden[l + 1][:n]) < 2e-2, (n, splits, l)
            by_split.append(got)
            _, last, _ = gm.get_state()
            if ref.margins[0] >= NOISE_BAND:
                assert last == ref.tokens[0]
                gm.draft(L, 1)                               # reads the K and V that the pass left in the cache
                ids, _, margins, _, _ = gm.peek_round(1)
                if ref.margins[1] >= NOISE_BAND:
                    assert ids[0] == ref.tokens[1]
                    assert abs(margins[0] - ref.margins[1]) < NOISE_BAND
        # (the splits were taken: the order of a sum shows in some of its last bits)
        assert not np.array_equal(by_split[0], by_split[1]) and not np.array_equal(by_split[1], by_split[2])
    gm.close()


def test_forced_plans_are_checked_and_released():
    from paper_2404_16710_amd import LsModel
    from paper_2404_16710_amd.binding import LsError
    w, ws, prompt, refs = _plan_case(128)
    gm = LsModel(w.model, ws, max_seq=128)
    for tile, splits in ((-1, 0), (7, 0), (0, -1), (0, 9)):
        with pytest.raises(LsError) as e:
            gm.debug_prompt_plan(tile, splits)
        assert e.value.code == -2
    cap = gm.debug_capture(True)
    gm.prefill(prompt[:65])
    want = cap.cpu().numpy().copy()
    gm.debug_prompt_plan(3, 8)                               # more splits than there is room for: as many as there is
    gm.prefill(prompt[:65])
    assert rel_err_rows(cap.cpu().numpy()[0, :65], refs[65].hidden[1][:65]) < 2e-2
    gm.debug_prompt_plan(0, 0)
    gm.prefill(prompt[:65])
    assert np.array_equal(cap.cpu().numpy(), want)
    gm.close()


# The room for partial sums comes from the workspace, so one prompt takes other splits in a large context than in one it
# just fits (down projection: 2 against 8 at 33 and 129 rows, 2 against 6 at 300): both against the oracle.
@pytest.mark.parametrize("n", [33, 129, 300])
def test_a_prompt_in_a_tight_and_in_a_large_context(n):
    from paper_2404_16710_amd import LsModel
    w = _case("room", n, d_model=512, ffn_dim=4096)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    om = O.OracleModel(w.model, ws, np.float32, emulate_bf16_act=True)
    ref = O.greedy_full(om, prompt, 2, want_hidden=True)
    for max_seq in (n + 17, 8192):
        gm = LsModel(w.model, ws, max_seq=max_seq)
        cap = gm.debug_capture(True)
        gm.prefill(prompt)
        got = cap.cpu().numpy()[:, :n]
        for l in range(w.model.n_layers):
            assert rel_err_rows(got[l], ref.hidden[l + 1][:n]) < 2e-2, (max_seq, l)
        if ref.margins[0] >= NEAR_TIE:
            assert gm.get_state()[1] == ref.tokens[0], max_seq
        gm.close()


# One prompt pass with a capture of the hidden states and one without leave the same workspace (cache, residual row and
# state of the decoder), bit for bit, also where the products' K is split, and so the same ids and margins after it.
@pytest.mark.parametrize("n", [33, 129, 300])
def test_a_captured_prompt_pass_is_the_same_pass(n):
    from paper_2404_16710_amd import LsModel
    w = _case("capture", n, d_model=512, ffn_dim=4096)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(w.model, ws, max_seq=n + 17)
    margins, left = [], []
    for on in (False, True, False):
        gm.debug_capture(on)
        gm.prefill(prompt)
        gm.get_state()                                       # (synchronises)
        left.append(gm.workspace.clone())
        gm.draft(w.model.n_layers, 6)
        ids, _, m, _, _ = gm.peek_round(6)
        margins.append((list(ids), [float(x) for x in m]))
    gm.debug_capture(False)
    gm.close()
    assert margins[0] == margins[1] == margins[2]
    # (the first pass finds a fresh workspace, the others the rows of the drafts behind the prompt)
    assert bool((left[1] == left[2]).all())
