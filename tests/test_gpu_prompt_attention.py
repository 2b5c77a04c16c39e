"""The prompt pass's attention for 16-bit models, in every split of its waves over queries and keys (which one
a prompt takes depends on the number of 32-row blocks and heads) and at the edges of its tiles.  Reference: the
same layer in passes of 16 rows, whose attention is another kernel (pinned to the oracle by the parity tests)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# rows, query heads, key/value heads, head_dim; which split a chunk takes on 256 compute units.  One wave of queries: few
# blocks (and a second chunk of 60 rows deep in the cache); two: 500 rows x 32 heads, 449 x 40; four: 1999 x 32 and
# 2041 x 28 (heads not a multiple of 8).  Second chunks after 2048 positions: 552 rows x 32 heads two, 652 x 28 two,
# 1953 x 32 four, each head width.
@pytest.mark.parametrize("n, nq, nkv, hd", [
    (32, 4, 4, 128), (33, 4, 1, 128), (127, 3, 3, 128), (129, 8, 2, 64), (2108, 2, 1, 64), (2108, 2, 2, 128),
    (500, 32, 8, 64), (449, 40, 40, 128), (1025, 32, 8, 64), (1999, 32, 8, 128), (2041, 28, 28, 64),
    (2600, 32, 32, 64), (2600, 32, 8, 128), (2700, 28, 7, 128), (4001, 32, 8, 64), (4001, 32, 8, 128)])
def test_prompt_attention_matches_the_row_passes(n, nq, nkv, hd):
    import torch
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name="attn", n_layers=1, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_model=256, ffn_dim=320,
                      vocab=528, rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    w = W.Workload(m, exit_layer=1, draft_len=1, n_prompt=n, n_new=2, resid_scale=1.0, gain_jitter=0.1)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    layer = ws["layers"][0]
    layer["w_down"] = np.zeros_like(layer["w_down"])     # the layer adds the projected attention output and nothing else
    layer["wq"] = layer["wq"] + np.uint16(2 << 7)        # x 4: attention concentrated on few keys
    embed = torch.from_numpy(ws["embed"].view(np.int16)).view(torch.bfloat16)[torch.from_numpy(prompt).long()].double().numpy()
    gm = LsModel(m, ws, max_seq=n + 3)

    def added():
        cap = gm.debug_capture(True)
        gm.prefill(prompt)
        got = cap.cpu().numpy()[0, :n].astype(np.float64) - embed
        gm.debug_capture(False)
        return got

    got = added()
    gm.set_prompt_tiles(16)
    want = added()
    gm.close()
    assert np.isfinite(got).all()
    # Both round the output to bf16 (relative 2^-9 per element each), and a few elements of q, k and v, from products
    # summed in another order, differ by a bf16 unit (2^-8): together below 2^-7 per row.
    err = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
    assert err.max() < 2.0 ** -7, (int(err.argmax()), float(err.max()))
