"""Launch plan of spec_verify_attn for ragged batches with little work: what it asks for follows the tokens, not the width
of the block table (a serving engine allocates that for the longest context its model allows).  Host calls only."""
import ctypes
import os

import pytest

from paper_2503_10325_amd import binding as sv

SPEC_ERR_WORKSPACE, SPEC_ERR_LAUNCH = -4, -6

pytestmark = pytest.mark.skipif(not os.path.exists(sv.LIB_PATH), reason="libspecverify.so not built")


@pytest.mark.parametrize("batch,heads,total_q,max_q,hint,pages", [
    (4, (64, 8), 40, 10, 8040, 8192),       # 80 rows per KV head
    (8, (64, 8), 56, 7, 16056, 2048),       # 56
    (1, (64, 8), 8, 8, 2008, 8192),         # one request
    (16, (32, 8), 80, 5, 32080, 8192),      # many pairs of request and KV head
    (5, (12, 4), 30, 9, 9000, 8192),
    (2, (16, 2), 16, 8, 1, 8192),           # the hint is an estimate and may be far off
])
def test_wide_block_tables_do_not_scale_the_launch(batch, heads, total_q, max_q, hint, pages):
    kw = dict(batch=batch, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=128, total_q=total_q, max_q_per_req=max_q,
              max_pages_per_req=pages)
    desc = sv.make_attn_desc(total_kv_tokens_hint=hint, **kw)
    plan, need = sv.spec_describe_attn_plan(desc), sv.spec_verify_attn_workspace_size(desc)
    chunks = int(plan.split("at most ")[1].split()[0])
    # the work list cuts a request into at most 16 chunks, of 44 tiles per wave (32 for up to 32 rows) and more
    rows = max_q * heads[0] // heads[1]
    tiles = pages * 16 // 32 // (4 if rows <= 32 else 2 if rows <= 64 else 1)
    assert chunks <= min(16, -(-tiles // (32 if rows <= 32 else 44))), plan
    assert chunks * batch * heads[1] <= 4096 or "list" in plan, plan
    assert need <= 256 + total_q * heads[0] * 16 * 130 * 4
    # a workspace sized without the hint holds the partial results of every hint
    unknown = sv.spec_verify_attn_workspace_size(sv.make_attn_desc(total_kv_tokens_hint=0, **kw))
    assert need <= unknown


def test_narrow_block_tables_are_cut_by_tokens():
    desc = sv.make_attn_desc(batch=5, num_q_heads=12, num_kv_heads=4, head_dim=64, total_q=30, max_q_per_req=9,
                             max_pages_per_req=189, total_kv_tokens_hint=9000)
    plan = sv.spec_describe_attn_plan(desc)
    assert "list" not in plan and "chunks of 512 tokens, at most 6 per request" in plan


@pytest.mark.parametrize("batch,heads,max_q,hint,pages,chunks", [
    (100, (32, 8), 29, 26000, 33, 1),       # 800 pairs, up to 116 rows: whole up to 1008 tokens, 528
    (100, (32, 8), 29, 30000, 64, 2),       # 1024
    (40, (32, 8), 8, 16000, 96, 1),         # up to 32 rows: 1536
    (40, (32, 8), 8, 16000, 97, 4),
    (40, (32, 8), 16, 16000, 48, 1),        # up to 64: 768
    (40, (32, 8), 16, 16000, 49, 2),
    (15, (32, 8), 8, 7000, 96, 3),          # 120 pairs: cut, whatever the length
])
def test_short_requests_of_batches_with_many_pairs_stay_whole(batch, heads, max_q, hint, pages, chunks):
    desc = sv.make_attn_desc(batch=batch, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=128, total_q=batch * max_q,
                             max_q_per_req=max_q, max_pages_per_req=pages, total_kv_tokens_hint=hint)
    assert f"at most {chunks} per request" in sv.spec_describe_attn_plan(desc), sv.spec_describe_attn_plan(desc)


def status_of_a_call(desc, workspace_bytes):
    """Status of spec_verify_attn with pointers to nothing: without a GPU a call that is not refused ends with the launch."""
    p = ctypes.c_void_p(4096)
    return sv.lib().spec_verify_attn(ctypes.byref(desc), p, p, p, p, p, p, None, p, None, p, workspace_bytes, None)


@pytest.mark.parametrize("batch,heads,total_q,max_q,pages,hints", [
    (109, (7, 1), 33, 2, 1568, (2176346,)),             # 14 rows, chunks of 5120 tokens without a hint, 4096 in the list
    (64, (64, 8), 200, 4, 1000, (300000, 500000, 850000)),
    (64, (32, 8), 400, 8, 1024, (300000, 850000)),
    (16, (8, 8), 100, 16, 4000, (600000, 850000)),
    (128, (32, 32), 500, 6, 2048, (100000, 3500000)),
    (64, (64, 8), 400, 8, 1000, (300000, 850000)),      # 64 rows
])
def test_a_workspace_sized_without_a_hint_serves_the_work_list(batch, heads, total_q, max_q, pages, hints):
    import torch
    if torch.cuda.is_available():
        pytest.skip("the pointers of these calls are not to be launched with")
    kw = dict(batch=batch, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=128, total_q=total_q, max_q_per_req=max_q,
              max_pages_per_req=pages)
    unknown = sv.spec_verify_attn_workspace_size(sv.make_attn_desc(total_kv_tokens_hint=0, **kw))
    for hint in hints:
        desc = sv.make_attn_desc(total_kv_tokens_hint=hint, **kw)
        assert "list" in sv.spec_describe_attn_plan(desc)
        assert status_of_a_call(desc, unknown) == SPEC_ERR_LAUNCH, (hint, unknown, sv.spec_verify_attn_workspace_size(desc))
        assert status_of_a_call(desc, 256) == SPEC_ERR_WORKSPACE
