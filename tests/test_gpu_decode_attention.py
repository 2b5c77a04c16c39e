"""Decode attention with the queries of a KV head dealt out in blocks: 16 rows x 4 query heads per KV head in a
draft-and-verify job, at contexts where 64 queries go in blocks of 4, 8 and 16 and undivided (one item per workgroup at
most: 8 KV heads x items of a KV head x blocks <= 256 workgroups), against one-row passes of the same model, whose
queries are never divided that way.  A query's arithmetic does not depend on its block, so the ids are the same.

An item is one 64-position tile in the cache of the first test, four in that of the second (8192 positions), where the
running softmax goes over the tiles of an item and the undivided form requests K and V again for each 16 of its queries."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd, dtype", [(64, "bf16"), (128, "bf16"), (64, "f32")])
@pytest.mark.parametrize("n_prompt", [40, 110, 180, 230, 300, 500, 560])
def test_blocks_of_queries_give_the_ids_of_one_row_passes(n_prompt, hd, dtype):
    _same_ids(n_prompt, hd, dtype, n_prompt + 48 + 17)


# blocks of 4 up to 512 positions, of 8 up to 1024, of 16 up to 2048, undivided beyond; the jobs of 470, 990 and 2010 ids
# cross a limit
@pytest.mark.parametrize("hd, dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
@pytest.mark.parametrize("n_prompt", [300, 470, 990, 1500, 2010, 2300])
def test_blocks_of_queries_with_items_of_several_tiles(n_prompt, hd, dtype):
    _same_ids(n_prompt, hd, dtype, 8192)


def _same_ids(n_prompt, hd, dtype, max_seq):
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name="blocks", n_layers=2, n_q_heads=32, n_kv_heads=8, head_dim=hd, d_model=256, ffn_dim=320,
                      vocab=528, rope_base=10000.0, rms_eps=1e-5, dtype=dtype)
    w = W.Workload(m, exit_layer=1, draft_len=15, n_prompt=n_prompt, n_new=48, resid_scale=0.1, gain_jitter=0.1)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(m, ws, max_seq=max_seq)
    toks, st = gm.generate(prompt, w.n_new, 1, 15)
    ar, _ = gm.generate(prompt, w.n_new, 0, 0)
    assert toks == ar
    gm.close()
