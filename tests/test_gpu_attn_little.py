"""Launches with little work (eight-wave workgroups of the token-split body, ragged batches cut by tokens instead of the
sorted work list): one and two 32-row query blocks per KV head, fewer tiles than waves, contexts that end inside a page, a
tile and a chunk, trees and chains, both head dimensions."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

from gpu_util import oracle_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("group,draft,ctx", [
    (1, ("linear", 1), ("fixed", 1)),                          # one row, one tile
    (3, ("linear_uniform", 3, 9), ("uniform", 40, 3001)),      # ragged, one block
    (4, ("linear_uniform", 8, 16), ("uniform", 500, 2600)),    # ragged, two blocks in some requests
    (8, ("tree", (3, 2), 8), ("fixed", 1023)),                 # two full blocks, masks over a chunk's edge
    (8, ("linear_uniform", 2, 14), ("uniform", 100, 4000)),    # ragged with 65 to 112 rows: the row-split body
])
def test_little_work(head_dim, group, draft, ctx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    cfg = W.scaled(W.CONFIGS["c1_llama2_7b"], batch=3, n_q_heads=2 * group, n_kv_heads=2, head_dim=head_dim, ctx=ctx, draft=draft)
    a = W.make_attn_inputs(cfg, seed=31)
    ref, ref_lse = oracle_attn(a)
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    assert "list" not in sv.spec_describe_attn_plan(dev.desc)
    dev.workspace.fill_(0xFF)                     # partial rows that were not written are NaN
    dev.run()
    torch.cuda.synchronize()
    # fp32 result of weights carried to 16 bits: 2^-17 of sum p |v| <= max |v| = 5.5, and fp32 sums; the row-split body
    # carries 11 bits (2^-12 of the weights, truncated)
    rows = int(a.st.n.max()) * group
    assert np.abs(dev.out.cpu().numpy() - ref).max() < (5e-5 if rows <= 64 else 3e-3)
    assert np.abs(dev.lse.cpu().numpy() - ref_lse).max() < 1e-4
