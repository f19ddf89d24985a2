"""Merging of context chunks: every number of lane groups per row the combine kernel is launched with, chunk counts
that are no multiple of what a group keeps in flight, and both head dimensions."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import workloads as W

from gpu_util import oracle_attn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding, runner
    binding.lib()
    return runner


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("batch,ctx", [(1, 700), (1, 1790), (1, 3333), (2, 6001), (1, 16000)])
def test_combine_merges_every_chunk_count(rt, head_dim, batch, ctx):
    cfg = W.scaled(W.CONFIGS["c1_llama2_7b"], batch=batch, n_q_heads=6, n_kv_heads=2, head_dim=head_dim,
                   ctx=("fixed", ctx), draft=("linear", 3))
    a = W.make_attn_inputs(cfg, seed=21)
    ref, ref_lse = oracle_attn(a)
    dev = rt.DeviceAttn(a, out_dtype=torch.float32)
    dev.workspace.fill_(0xFF)                     # partial rows that were not written are NaN
    dev.run()
    torch.cuda.synchronize()
    # fp32 result of weights carried to 16 bits: 2^-17 of sum p |v| <= max |v| = 5.5, and fp32 sums
    assert np.abs(dev.out.cpu().numpy() - ref).max() < 5e-5
    assert np.abs(dev.lse.cpu().numpy() - ref_lse).max() < 1e-4
