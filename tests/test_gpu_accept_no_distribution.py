"""Acceptance where a draft row is no distribution (every logit -inf, or one +inf): q is NaN, a token that the target gives mass
is accepted, and a rejection leaves the target distribution as it is.  The same on every path that can take the batch."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

from gpu_util import compare_accept, visited_pattern_agrees

pytestmark = pytest.mark.gpu

NEG_INF, POS_INF = 0xFF80, 0x7F80       # bf16


def run(cfg, ai, target, draft, tokens, tuning):
    from paper_2503_10325_amd import runner
    ref = oracle.accept(ai.st.node_offsets, ai.st.parent, tokens, target, draft, ai.q_row, ai.u_accept, ai.u_resample,
                        temperature=cfg.temperature)
    dev = runner.DeviceAccept(ai.st, target, draft, ai.q_row, tokens, ai.u_accept, ai.u_resample, temperature=cfg.temperature)
    dev.workspace.fill_(0xFF)
    dev.run(tuning=sv.SpecAcceptTuning(patience=-1, helpers=-1, **tuning))
    return dev.results(), ref


def spoiled(cfg, seed):
    """Odd requests: the draft row of the root is -inf throughout; even ones: its class 5 has +inf."""
    ai = W.make_accept_inputs(cfg, seed=seed)
    target, draft, tokens = ai.target_logits.copy(), ai.draft_q.copy(), ai.draft_tokens.copy()
    off = ai.st.node_offsets
    for b in range(cfg.batch):
        q = int(ai.q_row[off[b]])
        if b % 2:
            draft[q] = NEG_INF
        else:
            draft[q, 5] = POS_INF
    return ai, target, draft, tokens


# slices of 8192 logits that stay in registers, and rows read from LDS
CLUSTERS = [(65544, dict(path=2, levels=1, slices=9)), (65544, dict(path=2, levels=2, slices=9)),
            (4096, dict(path=2, levels=2, slices=1)), (4096, dict(path=2, levels=1, slices=1))]
WALKS = [(65544, dict(path=1)), (4096, dict(path=1))]


@pytest.mark.parametrize("vocab,tuning", CLUSTERS + WALKS)
def test_tree_accepts(vocab, tuning):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=6, vocab=vocab, draft=("tree", (3, 2), 9))
    ai, target, draft, tokens = spoiled(cfg, seed=3)
    got, ref = run(cfg, ai, target, draft, tokens, tuning)
    assert (ref["accept_len"] >= 1).all()
    bad, ties, _ = compare_accept(got, ref, ai.st.n)
    assert not bad and ties <= 1
    assert visited_pattern_agrees(got, ref, ai.st.node_offsets)


@pytest.mark.parametrize("vocab,path", [(65544, 3), (4096, 3), (4096, 1), (65544, 2)])
def test_chain_accepts(vocab, path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=6, vocab=vocab, draft=("linear", 4))
    ai, target, draft, tokens = spoiled(cfg, seed=4)
    got, ref = run(cfg, ai, target, draft, tokens, dict(path=path))
    assert (ref["accept_len"] >= 1).all()
    bad, ties, _ = compare_accept(got, ref, ai.st.n)
    assert not bad and ties <= 1


@pytest.mark.parametrize("vocab,tuning", CLUSTERS + WALKS)
def test_rejected_sibling_leaves_the_target_distribution(vocab, tuning):
    """The root's first child holds a token without target mass; its siblings are tested against the same distribution."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=6, vocab=vocab, draft=("tree", (3, 2), 9))
    ai, target, draft, tokens = spoiled(cfg, seed=5)
    off = ai.st.node_offsets
    for b in range(cfg.batch):
        row = int(off[b]) + b
        tokens[off[b]] = np.argmin(W.bf16_bits_to_f32(target[row]))       # (no sibling holds it)
        target[row, tokens[off[b]]] = NEG_INF
    got, ref = run(cfg, ai, target, draft, tokens, tuning)
    assert (ref["accept_len"] >= 1).all() and np.isinf(ref["ratio"][off[:-1] + 1]).all()
    bad, ties, _ = compare_accept(got, ref, ai.st.n)
    assert not bad and ties <= 1
    assert visited_pattern_agrees(got, ref, off)


@pytest.mark.parametrize("vocab", [65544, 50257, 4096, 1000])
def test_chain_accepts_in_one_launch(vocab):
    """The kernel that a small linear batch takes by itself."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=4, vocab=vocab, draft=("linear", 3))
    assert sv.spec_describe_accept_plan(4, vocab, 12, 3, False).startswith("accept_chain_kernel")
    ai, target, draft, tokens = spoiled(cfg, seed=4)
    got, ref = run(cfg, ai, target, draft, tokens, dict(path=0))
    assert (ref["accept_len"] >= 1).all()
    bad, ties, _ = compare_accept(got, ref, ai.st.n)
    assert not bad and ties <= 1
    ai.u_accept[ai.st.node_offsets[1:] - 1] = 1.0 - 2.0 ** -24        # the last node is rejected where the draft favours its token
    got, ref = run(cfg, ai, target, draft, tokens, dict(path=0))
    bad, ties, _ = compare_accept(got, ref, ai.st.n)
    assert not bad and ties <= 1
