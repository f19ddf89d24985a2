"""Accept decisions where p / q and the uniform number agree to 1e-15: the scalar arithmetic of every path is good to the last bits
of a double."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

pytestmark = pytest.mark.gpu

NEG_INF, ZERO = 0xFF80, 0x0000       # bf16

# (logit of the second of two classes, temperature, u): the first class has p = 1 / (1 + 2^(-d c)), c = log2(e) / T in fp32, and q = 1;
# u is the next fp32 number above p, by 0.95e-15 and 1.3e-15 of it: the token is rejected.  An error of 3e-15 in the power of
# two would accept it; the power itself, the sum, the quotient and the product are off by 2^-53 each, 4.4e-16 in all.
TIES = [(0.373046875, 1.1030224561691284, 0.5837542414665222), (0.482421875, 1.4146226644515991, 0.5844395160675049)]


@pytest.mark.parametrize("d,temperature,u", TIES)
@pytest.mark.parametrize("vocab,second,draft,tuning", [
    (65544, 9000, ("tree", (3, 2), 9), dict(path=2, levels=1, slices=9)),      # slices that stay in registers
    (65544, 9000, ("tree", (3, 2), 9), dict(path=2, levels=2, slices=9)),
    (4096, 3000, ("tree", (3, 2), 9), dict(path=2, levels=1, slices=2)),       # slices read from LDS
    (65544, 9000, ("tree", (3, 2), 9), dict(path=1)),
    (65544, 9000, ("linear", 4), dict(path=3)),
])
def test_last_bits(vocab, second, draft, tuning, d, temperature, u):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=4, vocab=vocab, draft=draft)
    ai = W.make_accept_inputs(cfg, seed=1)
    target, draft_q, tokens, off = ai.target_logits.copy(), ai.draft_q.copy(), ai.draft_tokens.copy(), ai.st.node_offsets
    u_accept = ai.u_accept.copy()
    for b in range(cfg.batch):
        row, q = int(off[b]) + b, int(ai.q_row[off[b]])
        target[row], draft_q[q] = NEG_INF, NEG_INF
        target[row, 7], draft_q[q, 7] = ZERO, ZERO
        target[row, second] = W.f32_to_bf16_bits(np.array([-d], dtype=np.float32))[0]
        tokens[off[b]:off[b + 1]] = 7
        u_accept[off[b]] = u
    dev = runner.DeviceAccept(ai.st, target, draft_q, ai.q_row, tokens, u_accept, ai.u_resample, temperature=temperature)
    dev.run(tuning=sv.SpecAcceptTuning(**tuning))
    got = dev.results()
    # behind the rejection the residual holds the second class alone
    assert (got["accept_len"] == 0).all() and (got["out_tokens"][:, 0] == second).all()
