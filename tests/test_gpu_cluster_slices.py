"""Acceptance of draft trees by clusters whose slices stay in registers (8192 logits each): many rejected siblings (the weights
of several residual levels), a residual without mass, a last slice of eight logits, trees with a chain of windows; the workgroup
that walks alone gives the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

from gpu_util import compare_accept, ratio_err

pytestmark = pytest.mark.gpu

MASKED = 0xFF80       # bf16 -inf


def inputs(vocab, seed):
    """Six requests of a 12,2,2 tree: 0, 1: draft rows equal to the target rows, the first three children of the root hold tokens
    that both rows exclude (their rejection leaves a residual without mass); 2, 3: draft rows that have nothing to do with
    the target, whose most probable tokens are drafted (most siblings are rejected); 4, 5: as drawn."""
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=6, vocab=vocab, draft=("tree", (12, 2, 2), 60))
    ai = W.make_accept_inputs(cfg, seed=seed)
    off, parent = ai.st.node_offsets, ai.st.parent
    target, draft, tokens = ai.target_logits.copy(), ai.draft_q.copy(), ai.draft_tokens.copy()
    rng = np.random.default_rng(seed)
    for b in range(4):
        for j in range(int(ai.st.n[b])):
            row, q = int(off[b]) + b + 1 + int(parent[off[b] + j]), int(ai.q_row[off[b] + j])
            sibling = int((parent[off[b]:off[b] + j] == parent[off[b] + j]).sum())
            if b < 2:
                draft[q] = target[row]
            elif sibling == 0:
                draft[q] = rng.permutation(draft[q])
            if b >= 2:
                tokens[off[b] + j] = np.argsort(-W.bf16_bits_to_f32(draft[q]), kind="stable")[sibling]
    for b in range(2):
        root, q = int(off[b]) + b, int(ai.q_row[off[b]])
        for j in range(3):
            target[root, tokens[off[b] + j]] = MASKED
            draft[q, tokens[off[b] + j]] = MASKED
    return cfg, ai, target, draft, tokens


@pytest.mark.parametrize("levels", [1, 2])
@pytest.mark.parametrize("vocab", [65544, 98304, 128256])        # 9 (the last of 8 logits), 12 and 16 slices
def test_slices_in_registers(vocab, levels):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    cfg, ai, target, draft, tokens = inputs(vocab, seed=vocab)
    ref = oracle.accept(ai.st.node_offsets, ai.st.parent, tokens, target, draft, ai.q_row, ai.u_accept, ai.u_resample,
                        temperature=cfg.temperature)
    assert (ref["accept_len"][:2] > 0).all() and (~np.isnan(ref["ratio"])).sum() > 36
    got = {}
    for patience in (-1, 0):
        dev = runner.DeviceAccept(ai.st, target, draft, ai.q_row, tokens, ai.u_accept, ai.u_resample,
                                  temperature=cfg.temperature)
        dev.workspace.fill_(0xFF)
        dev.run(tuning=sv.SpecAcceptTuning(path=2, levels=levels, slices=-(-vocab // 8192), patience=patience))
        got[patience] = dev.results()
    bad, ties, _ = compare_accept(got[-1], ref, ai.st.n)
    assert not bad and ties <= 1
    # the ratios carry the row sums' error (hardware 2^x, 1e-7) and, behind a rejection, that of the residual's mass
    assert ratio_err(got[-1]["ratio"], ref["ratio"]) < 5e-6 or ties
    for key in ("accept_len", "out_tokens", "stop_node"):
        assert np.array_equal(got[-1][key], got[0][key]), key
    assert np.array_equal(got[-1]["ratio"], got[0]["ratio"], equal_nan=True)


# first-child chains that end inside a window, next to siblings whose chains go on: leaf, leaf, chain of three; chain of two, leaf,
# chain of four; three leaves below a node below a leaf's sibling; no node
SHORT = [[-1, -1, -1, 2, 3], [-1, 0, -1, -1, 3, 4, 5], [-1, -1, 1, 1, 1, 4, 5, 6, 6, 8], [], [-1, -1, 0, 0, 1, 3, 5, 5, 7, 4]]


@pytest.mark.parametrize("levels", [2, 3, 4])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_chains_shorter_than_the_window(levels, seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    n = np.array([len(p) for p in SHORT], dtype=np.int32)
    st = W.DraftStructure(n, np.concatenate([[0], np.cumsum(n)]).astype(np.int32), np.concatenate(SHORT).astype(np.int32),
                          np.zeros(len(SHORT), dtype=np.int32))
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=len(SHORT), vocab=65536)
    ai = W.make_accept_inputs(cfg, seed=seed, st=st)
    draft = ai.draft_q.copy()
    rng = np.random.default_rng(seed)
    for q in range(0, len(draft), 2):             # every other draft row has nothing to do with the target
        draft[q] = rng.permutation(draft[q])
    ref = oracle.accept(st.node_offsets, st.parent, ai.draft_tokens, ai.target_logits, draft, ai.q_row, ai.u_accept, ai.u_resample,
                        temperature=cfg.temperature)
    dev = runner.DeviceAccept(st, ai.target_logits, draft, ai.q_row, ai.draft_tokens, ai.u_accept, ai.u_resample,
                              temperature=cfg.temperature)
    dev.workspace.fill_(0xFF)
    dev.run(tuning=sv.SpecAcceptTuning(path=2, levels=levels, slices=8))
    got = dev.results()
    bad, ties, _ = compare_accept(got, ref, n)
    assert not bad and ties <= 1
    assert ratio_err(got["ratio"], ref["ratio"]) < 5e-6 or ties
