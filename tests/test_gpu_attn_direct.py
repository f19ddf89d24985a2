"""Token-split attention body: one and two 32-row query blocks per wave, lengths around the edges of a page, a tile and a round
of tiles, unused cache slots that hold NaN."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import binding as sv

from gpu_util import oracle_attn
from test_gpu_attn_bodies import attention

pytestmark = pytest.mark.gpu


def poisoned(a):
    """The same inputs with NaN in every cache slot that no token of a request occupies."""
    used = np.zeros((a.k_pool.shape[0], 16), dtype=bool)
    for b in range(len(a.st.n)):
        length = int(a.st.ctx_len[b] + a.st.n[b])
        for t in range(length):
            used[a.block_table[b, t // 16], t % 16] = True
    pools = []
    for pool in (a.k_pool, a.v_pool):
        p = pool.copy()
        p.transpose(0, 2, 1, 3)[~used] = 0x7FC0
        pools.append(p)
    return dataclasses.replace(a, k_pool=pools[0], v_pool=pools[1])


# contexts that leave 1, 15, 16, 17, 31, 32, 33 tokens in the last tile, and numbers of tiles around one and two per wave
EDGES = [0, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 257, 513, 1025]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("nodes,requests", [(1, 14), (4, 14), (5, 14), (8, 14), (4, 140), (8, 140)])   # 8 to 64 rows; 28 and 280 workgroups
def test_edges_and_stale_slots(head_dim, nodes, requests):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    ctx = [EDGES[b % len(EDGES)] for b in range(requests)]
    a = poisoned(attention([nodes] * requests, ctx, head_dim, True))
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    ref, ref_lse = oracle_attn(a)
    # weights of two bf16 terms: 2^-17 of sum p |v| <= max |v| = 5.5, and fp32 sums
    assert np.abs(dev.out.cpu().numpy() - ref).max() < 5e-5, sv.spec_describe_attn_plan(dev.desc)
    assert np.abs(dev.lse.cpu().numpy() - ref_lse).max() < 1e-4


# 72, 128 (four waves), 232 (eight waves; with few requests sliced) and 800 rows (two mask words) per KV head
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("nodes,requests", [(9, 14), (16, 14), (29, 14), (29, 70), (100, 5)])
def test_row_split_edges_and_stale_slots(head_dim, nodes, requests):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    ctx = [EDGES[(3 * b + 1) % len(EDGES)] for b in range(requests)]
    a = poisoned(attention([nodes] * requests, ctx, head_dim, True))
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    ref, ref_lse = oracle_attn(a)
    # weights of one fp16 term (truncated, its mean put back): 2^-12 of sum p |v| <= max |v| = 5.5
    assert np.abs(dev.out.cpu().numpy() - ref).max() < 3e-3, sv.spec_describe_attn_plan(dev.desc)
    assert np.abs(dev.lse.cpu().numpy() - ref_lse).max() < 1e-4


# 384 tokens of a chunk: up to there a wave has one 32-row query block, then two (four-wave workgroups)
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("nodes", [5, 8])         # 40 and 64 rows
def test_one_and_two_query_blocks_per_wave(head_dim, tree, nodes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    ctx = [384 - nodes + k for k in (-33, -32, -31, -1, 0, 1, 15, 16, 17, 31, 32, 33)] * 12
    a = poisoned(attention([nodes] * len(ctx), ctx, head_dim, tree))
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    assert "attn_stream_kernel" in sv.spec_describe_attn_plan(dev.desc)
    dev.workspace.fill_(0xFF)
    dev.run()
    torch.cuda.synchronize()
    ref, ref_lse = oracle_attn(a)
    # as above: 2^-17 of max |v| = 5.5, and fp32 sums
    assert np.abs(dev.out.cpu().numpy() - ref).max() < 5e-5
    assert np.abs(dev.lse.cpu().numpy() - ref_lse).max() < 1e-4
