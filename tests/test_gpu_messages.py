"""Messages between the workgroups of one launch carry the call's tag in a workspace that nothing clears.  A workspace full of messages
that an earlier call could have left, 2^32 tags before (only the upper bits of the tag tell), gives what a cleared
one gives: one-launch acceptance, one-launch averaging, the cluster walk.  Another stream keeps the compute units busy meanwhile, so that workgroups start
far apart and look for messages that have not been sent yet."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LOW = (1 << 32) - 1


def stale(ws, seen, bits=37):
    """Fills the workspace with words of random data whose tags are the next call's but for bits above the 32nd.  seen: a message
    word of each of the two calls before."""
    step = (seen[1] - seen[0]) & LOW
    assert 0 < step <= 1 << 16                     # (the tags of a process follow one another)
    tag = (((seen[1] >> 32) + 1) << 32 | (seen[1] + step & LOW)) & (1 << bits) - 1
    words = ws.view(torch.int64)
    words.copy_(torch.randint(0, 1 << 63 - bits, words.shape, device="cuda") << bits | tag)


def nonzero(ws):
    return [int(w) for w in ws.view(torch.int64)[ws.view(torch.int64) != 0].tolist()]


def beside_work(fn):
    a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(3):
            torch.mm(a, a)
    out = fn()
    torch.cuda.synchronize()
    return out


def same(a, b):
    assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_one_launch_acceptance():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    from test_gpu_accept_chain import inputs, run
    V = 131072                                     # 16 x 16 workgroups
    d = inputs(V, [15], torch.bfloat16, torch.bfloat16, False, 1)
    d["ua"].fill_(1.0 - 2.0 ** -24)                # the first workgroups, which look first, decide
    assert sv.spec_describe_accept_plan(1, V, d["total"], d["most"], False).startswith("accept_chain_kernel")
    call = lambda ws: [run(sv, d, None, ws)[k].nan_to_num(-1.0) for k in ("len", "tok", "stop", "ratio")]
    ws = torch.zeros(sv.spec_accept_workspace_size(1, d["total"], d["total"], V) // 8 * 8, dtype=torch.uint8, device="cuda")
    seen = []
    for _ in range(2):
        ws.zero_()
        ref = call(ws)
        seen.append(nonzero(ws)[0])
    for _ in range(10):
        stale(ws, seen)
        seen = [seen[1], 2 * seen[1] - seen[0]]
        same(beside_work(lambda: call(ws)), ref)


def test_one_launch_averaging():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    from test_gpu_fuse_once import call as fuse, make
    d = make(2, 3, 3, 32000, torch.bfloat16, 1)
    d["lens"].fill_(3)
    ws = torch.zeros(sv.spec_fuse_drafts_workspace_size(2, 3, 3, 32000, sv.SPEC_FUSE_MIXTURE) // 8 * 8, dtype=torch.uint8, device="cuda")
    seen = []
    for _ in range(2):
        ws.zero_()
        ref = fuse(sv, d, ws)[1]
        seen.append(nonzero(ws)[0])
    stale(ws, seen)
    assert torch.equal(beside_work(lambda: fuse(sv, d, ws)[1]), ref)


def test_cluster_walk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    from paper_2503_10325_amd import runner, workloads as W
    cfg = W.scaled(W.CONFIGS["c2_tree_llama3_8b"], batch=4, vocab=65544, draft=("tree", (3, 2), 9))
    ai = W.make_accept_inputs(cfg, seed=3)
    dev = runner.DeviceAccept(ai.st, ai.target_logits, ai.draft_q, ai.q_row, ai.draft_tokens, ai.u_accept, ai.u_resample,
                              temperature=cfg.temperature)
    tuning = sv.SpecAcceptTuning(path=2, patience=-1, helpers=-1)

    def call():
        dev.run(tuning=tuning)
        got = dev.results()
        return [torch.from_numpy(got[k].copy()) for k in ("accept_len", "out_tokens", "stop_node")]

    ws = dev.workspace[:dev.workspace.numel() // 8 * 8]
    seen = []
    for _ in range(2):
        ws.zero_()
        ref = call()
        seen.append(min(w & (1 << 37) - 1 for w in nonzero(ws)))       # a tag of round 1
    for _ in range(10):
        stale(ws, seen)
        seen = [seen[1], 2 * seen[1] - seen[0]]
        same(beside_work(call), ref)
