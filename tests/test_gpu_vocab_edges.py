"""Vocabulary-wide kernels at vocabularies that no vector width divides, around the kernels' 8-class groups, 4096-class
blocks and 8192-class segments, and at bases that are aligned to one element only: acceptance of linear drafts and greedy
verification against the oracle (bars of test_gpu_parity.py), averaged distributions against the oracle (2e-5, as there:
fp32 exponentials)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2503_10325_amd import workloads as W

from gpu_util import compare_accept, ratio_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding, runner
    binding.lib()
    return runner


def off_by_one(x):
    """The array on the GPU at an address that is one element past a 16-byte boundary."""
    t = W.bf16_bits_to_f32(x) if x.dtype == np.uint16 else x
    dt = torch.bfloat16 if x.dtype == np.uint16 else torch.float32
    buf = torch.empty(t.size + 1, dtype=dt, device="cuda")
    buf[1:] = torch.from_numpy(np.ascontiguousarray(t)).reshape(-1).to("cuda")
    return buf[1:].view(t.shape)


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("V", [3, 7, 8, 9, 15, 4095, 4096, 4097, 8191, 8193, 20483, 270001])
def test_accept_and_greedy(rt, V, fp32):
    cfg = W.scaled(W.CONFIGS["c4_llama70b_serving"], batch=5 if V < 100000 else 2, vocab=V, draft=("linear_uniform", 1, 5))
    ai = W.make_accept_inputs(cfg, seed=V)
    tl, dq = ai.target_logits, ai.draft_q
    if fp32:
        tl, dq = W.bf16_bits_to_f32(tl), W.bf16_bits_to_f32(dq)
    ref = oracle.accept(ai.st.node_offsets, None, ai.draft_tokens, tl, dq, ai.q_row, ai.u_accept, ai.u_resample)
    rg = oracle.accept_greedy(ai.st.node_offsets, None, ai.draft_tokens, tl)
    for place in (lambda x: x, off_by_one):
        dev = rt.DeviceAccept(ai.st, place(tl), place(dq), ai.q_row, ai.draft_tokens, ai.u_accept, ai.u_resample)
        dev.run()
        got = dev.results()
        bad, _, _ = compare_accept(got, ref, ai.st.n)
        assert not bad
        assert ratio_err(got["ratio"], ref["ratio"]) < 5e-6
        assert np.array_equal(np.isnan(got["ratio"]), np.isnan(ref["ratio"]))
        devg = rt.DeviceGreedy(ai.st, place(tl), ai.draft_tokens)
        devg.run()
        gotg = devg.results()
        for key in ("row_argmax", "accept_len", "stop_node", "out_tokens"):
            assert np.array_equal(gotg[key], rg[key]), key


@pytest.mark.parametrize("V", [32768, 32769, 65536, 65537, 98304, 98305, 131072])
@pytest.mark.parametrize("fp32", [False, True])
def test_linear_draw_blocks_per_workgroup(rt, V, fp32):
    """64 requests leave eight workgroups each on 256 compute units: one to four 4096-class blocks per workgroup, the last
    one full or with a single class."""
    from paper_2503_10325_amd import binding as sv
    cfg = W.scaled(W.CONFIGS["c4_llama70b_serving"], batch=64, vocab=V, draft=("linear", 1))
    ai = W.make_accept_inputs(cfg, seed=V)
    tl, dq = ai.target_logits, ai.draft_q
    if fp32:
        tl, dq = W.bf16_bits_to_f32(tl), W.bf16_bits_to_f32(dq)
    ref = oracle.accept(ai.st.node_offsets, None, ai.draft_tokens, tl, dq, ai.q_row, ai.u_accept, ai.u_resample)
    dev = rt.DeviceAccept(ai.st, tl, dq, ai.q_row, ai.draft_tokens, ai.u_accept, ai.u_resample)
    dev.run(tuning=sv.SpecAcceptTuning(path=3))
    bad, _, _ = compare_accept(dev.results(), ref, ai.st.n)
    assert not bad


@pytest.mark.parametrize("V,N", [(5, 3), (9, 1), (2047, 4), (2049, 5), (3001, 17), (140003, 2)])
def test_mixture(rt, V, N):
    from paper_2503_10325_amd import binding as sv
    cfg = W.scaled(W.CONFIGS["c3_fusion"], batch=2, vocab=V, draft=("linear", 3), q_src=("fusion", N, 1.5))
    f = W.make_accept_inputs(cfg, seed=V).fusion
    ref = oracle.fuse_drafts(f.k_len, f.conf, f.draft_tokens, f.draft_logits, temperature=1.3, mode=oracle.FUSE_MIXTURE)
    dev = rt.DeviceFuse(f, V, temperature=1.3, mode=sv.SPEC_FUSE_MIXTURE)
    dev.run()
    torch.cuda.synchronize()
    got = dev.fused_probs.cpu().numpy().astype(np.float64)
    assert (np.abs(got - ref["fused_probs"]) / (ref["fused_probs"] + 1e-12)).max() < 2e-5
