"""Ragged batches of up to 128 query rows per KV head: every request runs the attention body of its own row count
(token-split with two-term bf16 weights up to 64 rows, row-split beyond), whatever the largest request of the batch or
the declared bound is; and a block table much wider than the longest request changes neither the result nor which
workspaces are accepted."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

from gpu_util import oracle_attn

pytestmark = pytest.mark.gpu

# 8, 32, 64 | 72, 112, 128 query rows per KV head; contexts that end inside a page, a tile and a chunk
NODES, CTX = [1, 4, 8, 9, 14, 16], [40, 3001, 1000, 2500, 129, 1777]


def structure(nodes, ctx, tree):
    n = np.asarray(nodes, dtype=np.int32)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    parent = np.concatenate([(np.arange(k) - 1) // 2 for k in n]).astype(np.int32) if tree else None
    if tree:                                       # a binary heap under two roots
        parent[np.isin(np.arange(parent.size), off[:-1])] = -1
    return W.DraftStructure(n, off, parent, np.asarray(ctx, dtype=np.int32))


def attention(nodes, ctx, head_dim, tree, seed=7, kv_heads=2):
    cfg = W.scaled(W.CONFIGS["c4_llama70b_serving"], batch=len(nodes), n_q_heads=8 * kv_heads, n_kv_heads=kv_heads,
                   head_dim=head_dim)
    return W.make_attn_inputs(cfg, seed=seed, st=structure(nodes, ctx, tree))


def run_fp32(a, max_q=None):
    """(descriptor's plan, fp32 result, natural-log sums) with the partial rows poisoned."""
    from paper_2503_10325_amd import runner
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    if max_q:
        dev.desc.max_q_per_req = max_q
        dev.workspace = torch.empty(max(256, sv.spec_verify_attn_workspace_size(dev.desc)), dtype=torch.uint8, device="cuda")
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    return sv.spec_describe_attn_plan(dev.desc), dev.out.cpu().numpy(), dev.lse.cpu().numpy()


def check(a, got, lse):
    ref, ref_lse = oracle_attn(a)
    assert np.abs(lse - ref_lse).max() < 1e-4
    for b in range(len(a.st.n)):
        o, e = int(a.st.node_offsets[b]), int(a.st.node_offsets[b + 1])
        rows = (e - o) * a.cfg.n_q_heads // a.cfg.n_kv_heads
        # weights of two bf16 terms: 2^-17 of sum p |v| <= max |v| = 5.5, and fp32 sums; of one fp16 term (truncated,
        # its mean put back): 2^-12 of the same
        assert e == o or np.abs(got[o:e] - ref[o:e]).max() < (5e-5 if rows <= 64 else 3e-3), (b, rows)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("tree", [False, True])
def test_little_mixed_batch_keeps_each_request_s_body(head_dim, tree):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a = attention(NODES, CTX, head_dim, tree)
    plan, got, lse = run_fp32(a)
    assert "attn_mixed_kernel" in plan
    check(a, got, lse)


@pytest.mark.parametrize("nodes,kernel", [([2, 11, 16] * 22, "attn_mixed_kernel"), ([2, 8, 5] * 22, "attn_stream_kernel")])
def test_little_batch_with_many_requests_stays_whole(nodes, kernel):
    """132 (request, KV head) pairs of up to 500 tokens: no request is cut, nothing is merged."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a = attention(nodes, [(77 * k) % 500 for k in range(66)], 128, False)
    plan, got, lse = run_fp32(a)
    assert kernel in plan and "at most 1 per request" in plan, plan
    check(a, got, lse)


def test_loose_bound_changes_no_body():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a = attention([1, 4, 8, 5], [40, 3001, 1000, 777], 128, False)
    _, got, lse = run_fp32(a, max_q=16)            # no request has more than 64 rows, the bound says 128
    check(a, got, lse)


def widened(a, pages):
    table = np.full((a.block_table.shape[0], pages), -1, dtype=np.int32)
    table[:, :a.max_pages] = a.block_table
    return dataclasses.replace(a, block_table=table, max_pages=pages)


# (nodes, contexts): up to 64 rows per KV head, and both bodies
WIDE = [([1, 4, 8, 5], [40, 9000, 1000, 777]), ([1, 9, 14, 8], [300, 129, 9000, 777])]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("nodes,ctx", WIDE)
def test_wide_block_table(head_dim, nodes, ctx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a = widened(attention(nodes, ctx, head_dim, False), 8192)
    plan, got, lse = run_fp32(a)
    tokens, chunks = int(plan.split("chunks of ")[1].split()[0]), int(plan.split("at most ")[1].split()[0])
    assert "list" not in plan and tokens * chunks < 9000, plan          # the longest request's chunks are lengthened
    check(a, got, lse)


@pytest.mark.parametrize("nodes,ctx", WIDE)
@pytest.mark.parametrize("pages", [564, 8192])
def test_workspace_sized_under_another_hint(nodes, ctx, pages):
    """The hint only steers the cut: a workspace asked for without it, or with one that calls for the work list, serves
    the same batch under its own hint."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    a = widened(attention(nodes, ctx, 128, False), pages)
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    hint = dev.desc.total_kv_tokens_hint
    for other in (0, 130 * 1024):
        dev.desc.total_kv_tokens_hint = other if other == 0 or other < 0.8 * 4 * pages * 16 else 0
        need = sv.spec_verify_attn_workspace_size(dev.desc)
        dev.desc.total_kv_tokens_hint = hint
        dev.workspace = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda") if need > 256 else None
        dev.out.fill_(float("nan"))
        dev.run()
        torch.cuda.synchronize()
        check(a, dev.out.cpu().numpy(), dev.lse.cpu().numpy())


def listed(a, pages=8192):
    """The batch with a table and a hint that call for the work list (lengths are ragged against the table, and the hint
    says that there is much work; it only steers the cut)."""
    from paper_2503_10325_amd import runner
    a = widened(a, pages)
    hint = int(0.8 * len(a.st.n) * pages * 16)
    dev = runner.DeviceAttn(a, out_dtype=torch.float32, kv_hint=hint)
    plan = sv.spec_describe_attn_plan(dev.desc)
    assert "attn_stream_list_kernel" in plan
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    check(a, dev.out.cpu().numpy(), dev.lse.cpu().numpy())
    return plan


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("nodes,ctx,kv_heads", [
    (NODES, CTX, 2),
    ([8, 3, 0, 1], [5000, 0, 200, 64], 2),                      # token-split body only; no nodes, no context
    ([16, 12, 9], [9000, 0, 700], 2),                           # row-split body only
    ([2, 11] * 50, [(77 * k) % 300 for k in range(100)], 8),    # 800 items on 512 workgroups: two rounds
])
def test_work_list(head_dim, tree, nodes, ctx, kv_heads):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    listed(attention(nodes, ctx, head_dim, tree, kv_heads=kv_heads))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("nodes,longest,item", [(8, 70000, 32 * 128), (9, 75000, 42 * 16 * 32 // 5)])
def test_work_list_most_chunks(head_dim, nodes, longest, item):
    """Contexts that 16 items do not hold (64 rows: of 32 units of 128 tokens, 65536 in all; 72 rows, row-split body, whose 32
    tokens count 5/16 of a unit: of 42 units, 68800): the chunks get longer."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert longest > 16 * item
    plan = listed(attention([nodes, 2, nodes], [longest, 100, 3000], head_dim, False))
    assert "at most 16 per request" in plan


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("nodes", [9, 16])        # 72 and 128 rows: three and four 32-row blocks
def test_work_list_chunks_beyond_the_page_table_of_the_row_split_body(head_dim, nodes):
    """A 16th of 140000 tokens is more than the 8192 whose page ids the row-split body holds: the token-split body takes the
    request, a wave per 32-row block, with its two-term bf16 weights."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    a = widened(attention([nodes, 2, 8], [140000, 100, 3000], head_dim, False), 9000)
    dev = runner.DeviceAttn(a, out_dtype=torch.float32, kv_hint=int(0.8 * 3 * 9000 * 16))
    plan = sv.spec_describe_attn_plan(dev.desc)
    assert "attn_stream_list_kernel" in plan and "at most 16 per request" in plan and 140000 > 16 * 8192
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    ref, ref_lse = oracle_attn(a)
    # 2^-17 of sum p |v| <= max |v| = 5.5, and fp32 sums; the row-split body's weights of one fp16 term would be off by more
    assert np.abs(dev.out.cpu().numpy() - ref).max() < 5e-5
    assert np.abs(dev.lse.cpu().numpy() - ref_lse).max() < 1e-4


@pytest.mark.parametrize("head_dim", [64, 128])
def test_work_list_in_a_workspace_sized_without_a_hint(head_dim):
    """32 rows per KV head, a table for 65536 tokens: the list has up to 16 chunks of 4096, the workspace holds the results of 13."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    a = widened(attention([4, 2, 4], [60000, 100, 5600], head_dim, False, kv_heads=8), 4096)
    need = runner.DeviceAttn(a, out_dtype=torch.float32, kv_hint=0).workspace.numel()
    dev = runner.DeviceAttn(a, out_dtype=torch.float32, kv_hint=3 * 52000)
    assert "list" in sv.spec_describe_attn_plan(dev.desc) and dev.workspace.numel() > need
    # (held in a larger block whose other bytes have to stay as they are)
    block = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    dev.workspace = block[:need]
    dev.run()
    torch.cuda.synchronize()
    assert (block[need:] == 0xFF).all()
    check(a, dev.out.cpu().numpy(), dev.lse.cpu().numpy())


# 96 pairs: 252, 279, 318, 348 items of 32 units; 211, 233, 264, 288 of 40; 196, 216, 244, 266 of 44
@pytest.mark.parametrize("hint_units,cut", [(68, True), (77, False), (90, False), (100, True)])
def test_work_list_items_follow_the_compute_units(hint_units, cut):
    """Requests of up to 39 units: cut into items of 32, whole in items of 40 or 44 (no partial result is written)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the numbers are those of 256 compute units")
    from paper_2503_10325_amd import runner
    a = widened(attention([4] * 12, [4900 - 37 * k for k in range(12)], 64, False, kv_heads=8), 2048)
    dev = runner.DeviceAttn(a, out_dtype=torch.float32, kv_hint=12 * 128 * hint_units)
    assert "attn_stream_list_kernel" in sv.spec_describe_attn_plan(dev.desc)
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    assert bool((dev.workspace != 0xFF).any()) == cut
    check(a, dev.out.cpu().numpy(), dev.lse.cpu().numpy())
