"""The enqueue-only calls recorded into a HIP graph: every replay repeats the eager round, with other work of the
same model between the replays."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# 16-row passes, the prompt pass, and (widths that are multiples of 64) a short prompt's rows together and the prompt pass
@pytest.mark.parametrize("n_prompt, ffn_dim", [(20, 1040), (70, 1040), (20, 1088), (70, 1088)])
def test_replays_of_a_captured_round_repeat_it(n_prompt, ffn_dim):
    import torch
    from paper_2404_16710_amd import LsModel
    m = W.ModelConfig(name="graph", n_layers=3, n_q_heads=4, n_kv_heads=2, head_dim=128, d_model=384, ffn_dim=ffn_dim,
                      vocab=1040, rope_base=10000.0, rms_eps=1e-5, dtype="bf16")
    w = W.Workload(m, exit_layer=1, draft_len=5, n_prompt=n_prompt, n_new=8, resid_scale=0.1, gain_jitter=0.1)
    ws, prompt = W.make_weights(w), W.make_prompt(w)
    gm = LsModel(m, ws, max_seq=n_prompt + 64)

    def one_round():
        gm.prefill(prompt)
        gm.draft(w.exit_layer, w.draft_len)
        gm.verify(w.exit_layer, w.draft_len)

    one_round()
    want = gm.peek_round(w.draft_len)
    dev_prompt = gm._dev_i32(prompt)                         # the graph reads it again at every replay
    gm._dev_i32 = lambda ids: dev_prompt
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        one_round()
    del gm._dev_i32
    for _ in range(4):
        gm.generate(list(prompt)[::-1], 6, 0, 0)             # another job on the same counters, and a synchronisation
        graph.replay()
        torch.cuda.synchronize()
        assert gm.peek_round(w.draft_len) == want
    del graph
    gm.close()
