"""The library only enqueues work on the stream it is given: calls captured into a HIP graph must
replay to the eager results, every time, and independent problems on two streams must not disturb
each other (each has its own workspace)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2503_10325_amd import workloads as W

from gpu_util import ATTN_TOL, attn_rel_err, compare_accept, oracle_attn

pytestmark = pytest.mark.gpu
C = W.CONFIGS


@pytest.fixture(scope="module")
def rt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding, runner
    binding.lib()
    return runner


def test_graph_replay_matches_eager(rt):
    cfg = W.scaled(C["c4_llama70b_serving"], batch=6, n_q_heads=16, n_kv_heads=2, ctx=("lognormal", 400, 0.8, 20, 2500))
    a = W.make_attn_inputs(cfg, seed=2)
    ai = W.make_accept_inputs(cfg, seed=2, st=a.st)
    attn = rt.DeviceAttn(a)
    acc = rt.DeviceAccept(a.st, ai.target_logits, ai.draft_q, ai.q_row, ai.draft_tokens, ai.u_accept, ai.u_resample)
    attn.run(); acc.run()                                   # eager: reference results (and one-time set-up)
    torch.cuda.synchronize()
    out0, lse0 = attn.out.clone(), attn.lse.clone()
    res0 = {k: v.copy() for k, v in acc.results().items() if v is not None}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            attn.run(); acc.run()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(4):
        attn.out.zero_(); attn.lse.zero_(); acc.accept_len.fill_(-9); acc.out_tokens.fill_(-9)
        attn.workspace.fill_(0xEE)                          # partials of earlier runs must not be needed
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(attn.out, out0) and torch.equal(attn.lse, lse0), rep
        res = acc.results()
        for k, v in res0.items():
            assert np.array_equal(res[k], v, equal_nan=True), (rep, k)
    ref, _ = oracle_attn(a)
    assert attn_rel_err(out0.float().cpu().numpy(), ref) <= ATTN_TOL


def test_two_streams_do_not_interfere(rt):
    cfgs = [W.scaled(C["c2_tree_llama3_8b"], batch=3, n_q_heads=8, n_kv_heads=2, ctx=("fixed", 700), vocab=70000),
            W.scaled(C["c1_llama2_7b"], batch=5, n_q_heads=4, n_kv_heads=4, ctx=("fixed", 900))]
    probs = []
    for i, cfg in enumerate(cfgs):
        a = W.make_attn_inputs(cfg, seed=20 + i)
        ai = W.make_accept_inputs(cfg, seed=20 + i, st=a.st)
        probs.append((a, ai, rt.DeviceAttn(a),
                      rt.DeviceAccept(a.st, ai.target_logits, ai.draft_q, ai.q_row, ai.draft_tokens, ai.u_accept,
                                      ai.u_resample)))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for rep in range(3):
        for (a, ai, attn, acc), s in zip(probs, streams):
            attn.run(stream=s)
            acc.run(stream=s)
    torch.cuda.synchronize()
    for a, ai, attn, acc in probs:
        ref, _ = oracle_attn(a)
        assert attn_rel_err(attn.out.float().cpu().numpy(), ref) <= ATTN_TOL
        want = oracle.accept(a.st.node_offsets, a.st.parent, ai.draft_tokens, ai.target_logits, ai.draft_q, ai.q_row,
                             ai.u_accept, ai.u_resample)
        bad, ties, B = compare_accept(acc.results(), want, a.st.n)
        assert not bad


@pytest.mark.parametrize("rows_extra", [0, 150])       # up to and above 128 rows
def test_graph_replay_lm_head_then_accept(rt, rows_extra):
    """spec_lm_head + spec_accept_prestats captured into one HIP graph: every replay reproduces the eager
    logits, statistics and acceptance results, with stale bytes in all scratch memory in between."""
    cfg = W.scaled(C["c1_llama2_7b"], batch=6, vocab=9000, draft=("linear_uniform", 2, 6))
    st = W.make_structure(cfg, seed=3)
    rows = st.total + cfg.batch
    li = W.make_lm_head_inputs(rows + rows_extra, 256, cfg.vocab, seed=3)     # extra rows: hidden states nobody verifies
    ai = W.make_accept_inputs(cfg, seed=3, st=st)
    ws = torch.zeros(max(rt.sv.spec_accept_workspace_size(cfg.batch, st.total, ai.draft_q.shape[0], cfg.vocab),
                         rt.sv.spec_row_stats_size(rows + rows_extra, cfg.vocab)), dtype=torch.uint8, device="cuda")
    head = rt.DeviceLmHead(li, stats=ws)
    acc = rt.DeviceAccept(st, head.logits[:rows], ai.draft_q, ai.q_row, ai.draft_tokens, ai.u_accept, ai.u_resample)
    acc.workspace = ws
    head.run(); acc.run_prestats()
    torch.cuda.synchronize()
    logits0, stats0 = head.logits.clone(), ws[: rt.sv.spec_row_stats_size(rows, cfg.vocab)].clone()
    res0 = {k: v.copy() for k, v in acc.results().items() if v is not None}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            head.run(); acc.run_prestats()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        head.logits.zero_(); head.workspace.fill_(0xEE); ws.fill_(0xEE)
        acc.accept_len.fill_(-9); acc.out_tokens.fill_(-9)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(head.logits, logits0), rep
        assert torch.equal(ws[: stats0.numel()], stats0), rep
        res = acc.results()
        for k, v in res0.items():
            assert np.array_equal(res[k], v, equal_nan=True), (rep, k)
    # reference: the oracle's own pipeline on the same host inputs; requests whose drafted logits are
    # bf16 neighbours on the two sides (about one entry in ten thousand is) are exempt
    tl = oracle.lm_head(li.hidden[:rows], li.weight)["logits"]
    want = oracle.accept(st.node_offsets, st.parent, ai.draft_tokens, tl, ai.draft_q, ai.q_row, ai.u_accept,
                         ai.u_resample)
    gpu_bits = head.logits_bits()
    disagree = [b for b in range(cfg.batch)
                if any(gpu_bits[int(st.node_offsets[b]) + b + j, ai.draft_tokens[int(st.node_offsets[b]) + j]] !=
                       tl[int(st.node_offsets[b]) + b + j, ai.draft_tokens[int(st.node_offsets[b]) + j]]
                       for j in range(int(st.n[b])))]
    bad, ties, B = compare_accept(res0, want, st.n)
    assert set(bad) <= set(disagree) and len(disagree) <= 1 and ties <= 1
