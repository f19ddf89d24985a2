"""accept_chain_kernel (linear drafts in one launch) against the statistics pass + accept_linear_kernel (path 3, which the oracle
tests cover): same lengths, tokens and stop nodes, ratios to the last bits of the fp64 sums.  Vocabularies at the edges
of 8-class groups, waves, 4096-class blocks and 8192-class segments; requests without nodes; every dtype; probability drafts;
target statistics from the caller; and patience 0, where every record that is not there yet is worked out by the
workgroup that misses it.  The workspace starts as garbage and is not cleared between the calls."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def inputs(V, n, tdt, qdt, probs, seed, T=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = np.asarray(n)
    off = np.concatenate([[0], np.cumsum(n)])
    B, total = len(n), int(n.sum())
    target = torch.randn((total + B, V), generator=g, device="cuda") * 2
    rows = torch.from_numpy(np.concatenate([off[b] + b + np.arange(k) for b, k in enumerate(n)] + [[]]).astype(np.int64)).cuda()
    draft = target[rows] + 0.7 * torch.randn((total, V), generator=g, device="cuda")
    e = torch.empty_like(draft).exponential_(generator=g)
    tokens = (torch.softmax(draft / T, 1) / e).argmax(1).int()
    draft = (torch.softmax(draft, 1) if probs else draft).to(qdt).contiguous()
    u = torch.randint(0, 1 << 24, (total + B,), generator=g, device="cuda").float() * 2.0 ** -24
    return dict(B=B, total=total, most=int(n.max()), off=torch.from_numpy(off.astype(np.int32)).cuda(), tokens=tokens,
                target=target.to(tdt).contiguous(), draft=draft, q_row=torch.arange(total, dtype=torch.int32, device="cuda"),
                ua=u[:total].contiguous(), ur=u[total:].contiguous(), probs=probs)


def run(sv, d, tuning, workspace, T=0.9, prestats=False):
    out = dict(len=torch.full((d["B"],), -7, dtype=torch.int32, device="cuda"),
               tok=torch.full((d["B"], d["most"] + 1), -7, dtype=torch.int32, device="cuda"),
               stop=torch.full((d["B"],), -7, dtype=torch.int32, device="cuda"),
               ratio=torch.full((max(1, d["total"]),), -7.0, device="cuda"))
    a = (d["B"], d["total"], d["most"], d["off"], None, d["tokens"], d["target"], d["draft"],
         sv.SPEC_Q_PROBS if d["probs"] else sv.SPEC_Q_LOGITS, d["q_row"], T, d["ua"], d["ur"], out["len"], out["tok"], out["stop"],
         out["ratio"], workspace)
    if prestats:
        sv.spec_accept_prestats(*a)
    else:
        sv.spec_accept_tuned(tuning, *a)
    return out


def same(a, b):
    for k in ("len", "tok", "stop"):
        assert torch.equal(a[k], b[k]), k
    assert torch.equal(a["ratio"].isnan(), b["ratio"].isnan())
    assert torch.allclose(a["ratio"].nan_to_num(1.0), b["ratio"].nan_to_num(1.0), rtol=1e-6, atol=0)


@pytest.mark.parametrize("V,n,tdt,qdt,probs", [
    (8, [2, 0, 3], torch.bfloat16, torch.bfloat16, False),
    (9, [1], torch.float32, torch.float32, False),
    (519, [4, 4], torch.bfloat16, torch.float32, False),
    (4095, [3, 1, 0, 2], torch.bfloat16, torch.bfloat16, False),
    (4097, [5], torch.float32, torch.bfloat16, False),
    (8191, [16, 2], torch.bfloat16, torch.bfloat16, False),
    (8193, [3, 3], torch.bfloat16, torch.bfloat16, False),
    (12289, [2, 6], torch.bfloat16, torch.float32, True),
    (32000, [8, 1, 8], torch.bfloat16, torch.float32, True),
    (8200, [70, 5], torch.float32, torch.float32, False),        # more nodes than lanes
    (50257, [8, 3], torch.float32, torch.float32, False),
    (131072, [5, 2, 0], torch.bfloat16, torch.bfloat16, False),   # 16 segments
    (140000, [4], torch.bfloat16, torch.bfloat16, False),         # 18: more than a group of 16 lanes merges at once
    (600000, [1], torch.bfloat16, torch.bfloat16, False),         # 74 segments, 147 blocks: more than one block per lane
    (20000, [0, 0], torch.bfloat16, torch.bfloat16, False),       # no drafts at all
])
def test_chain_matches_two_launches(V, n, tdt, qdt, probs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    plan = None
    for seed in range(3):
        d = inputs(V, n, tdt, qdt, probs, seed)
        code = {torch.bfloat16: sv.SPEC_BF16, torch.float32: sv.SPEC_F32}
        plan = sv.spec_describe_accept_plan(d["B"], V, d["total"], d["most"], False, target_dtype=code[tdt], q_dtype=code[qdt],
                                            q_kind=sv.SPEC_Q_PROBS if probs else sv.SPEC_Q_LOGITS)
        assert plan.startswith("accept_chain_kernel"), plan
        size = sv.spec_accept_workspace_size(d["B"], d["total"], d["draft"].shape[0], V)
        ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device="cuda")
        ref = run(sv, d, sv.SpecAcceptTuning(path=3), ws.clone())
        for _ in range(2):
            same(run(sv, d, None, ws), ref)
        same(run(sv, d, sv.SpecAcceptTuning(patience=0), ws), ref)


@pytest.mark.parametrize("probs", [False, True])
def test_chain_from_given_target_statistics(probs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    from paper_2503_10325_amd import runner, workloads as W
    V, n = 16424, [3, 0, 6, 2]
    d = inputs(V, n, torch.bfloat16, torch.float32 if probs else torch.bfloat16, probs, 5)
    li = W.make_lm_head_inputs(d["total"] + d["B"], 256, V, seed=3)
    dev = runner.DeviceLmHead(li, temperature=0.9)
    dev.run()
    d["target"] = dev.logits
    size = sv.spec_accept_workspace_size(d["B"], d["total"], d["draft"].shape[0], V)
    ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device="cuda")
    head = torch.empty(max(256, sv.spec_lm_head_workspace_size(*dev.hidden.shape, V)), dtype=torch.uint8, device="cuda")
    ref = run(sv, d, sv.SpecAcceptTuning(path=3), ws.clone())
    for _ in range(2):
        sv.spec_lm_head(dev.hidden, dev.weight, 0.9, dev.logits, ws, head)
        same(run(sv, d, None, ws, prestats=True), ref)


def test_chain_replays():
    """A captured call repeats its message tag: replays on new inputs in the same buffers must not see old messages."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    sets = [inputs(32000, [6, 3, 8], torch.bfloat16, torch.bfloat16, False, s) for s in range(4)]
    d = {k: (v.clone() if torch.is_tensor(v) else v) for k, v in sets[0].items()}
    ws = torch.empty(sv.spec_accept_workspace_size(d["B"], d["total"], d["total"], 32000), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(sv, d, None, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        out = run(sv, d, None, ws)
    for s in sets + sets:
        for k, v in s.items():
            if torch.is_tensor(v):
                d[k].copy_(v)
        graph.replay()
        torch.cuda.synchronize()
        same(out, run(sv, s, sv.SpecAcceptTuning(path=3), torch.empty_like(ws)))


def given_statistics(d, T, V):
    """The records that the projection hands over: per 8192-class segment the largest logit m and the sum of 2^((l - m) c)."""
    c = float(np.float32(1.4426950408889634) / np.float32(T))
    rec = []
    for x in d["target"].double().split(8192, 1):
        m = x.amax(1)
        z = torch.exp2((x - m.where(m.isfinite(), torch.zeros_like(m))[:, None]) * c).sum(1)
        rec.append(torch.stack([m.float().view(torch.int32).long(), z.view(torch.int64)], 1))
    return torch.stack(rec, 1).contiguous().view(torch.uint8).view(-1)


@pytest.mark.parametrize("accepted", [True, False])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("shift,T", [(-200.0, 1.0), (-20.0, 0.1), (90.0, 0.1)])
@pytest.mark.parametrize("V,dtype", [(1000, torch.bfloat16), (32000, torch.bfloat16), (50257, torch.float32)])
def test_chain_of_shifted_and_masked_rows(V, dtype, shift, T, masked, accepted):
    """Acceptance does not depend on where the logits lie, nor on classes without mass: rows far below and above zero, draft rows cut
    to their 40 best classes and target rows without 64 to 2048 classes in a row (of a thread's classes none, some or all are left),
    and vocabularies whose last segment leaves threads without classes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from gpu_util import compare_accept
    from paper_2503_10325_amd import binding as sv
    n = np.asarray([4, 0, 3])
    d = inputs(V, n, torch.float32, torch.float32, False, 11, T)
    if masked:
        least = d["draft"].topk(40, 1).values[:, -1:]
        held = torch.zeros_like(d["draft"], dtype=torch.bool).scatter_(1, d["tokens"].long()[:, None], True)
        d["draft"] = d["draft"].masked_fill((d["draft"] < least) & ~held, -float("inf"))
        run_of = 64 if V < 8192 else 2048
        gone = torch.arange(V, device="cuda") // run_of % 2 == 1
        kept = torch.zeros_like(d["target"], dtype=torch.bool).index_fill_(1, d["tokens"].long(), True)
        d["target"] = d["target"].masked_fill(gone & ~kept, -float("inf"))
    d["target"], d["draft"] = (d["target"] + shift).to(dtype), (d["draft"] + shift).to(dtype)
    d["ua"].fill_(0.0 if accepted else 1.0 - 2.0 ** -24)
    code = sv.SPEC_BF16 if dtype == torch.bfloat16 else sv.SPEC_F32
    assert sv.spec_describe_accept_plan(3, V, 7, 4, False, target_dtype=code, q_dtype=code).startswith("accept_chain_kernel")
    ws = torch.randint(0, 256, (sv.spec_accept_workspace_size(3, 7, 7, V),), dtype=torch.uint8, device="cuda")
    bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16) if dtype == torch.bfloat16 else t.cpu().numpy()
    for seed in range(8):             # (one set of rows, many draws)
        g = torch.Generator().manual_seed(seed)
        d["ur"].copy_(torch.randint(0, 1 << 24, (3,), generator=g).float() * 2.0 ** -24)
        ref = run(sv, d, sv.SpecAcceptTuning(path=3), ws.clone(), T)
        got = run(sv, d, None, ws, T)
        same(got, ref)
        same(run(sv, d, sv.SpecAcceptTuning(patience=0), ws, T), ref)
        if dtype == torch.bfloat16:
            rec = given_statistics(d, T, V)
            ws[:rec.numel()].copy_(rec)
            same(run(sv, d, None, ws, T, prestats=True), ref)
        want = oracle.accept(d["off"].cpu().numpy(), None, d["tokens"].cpu().numpy(), bits(d["target"]), bits(d["draft"]),
                             d["q_row"].cpu().numpy(), d["ua"].cpu().numpy(), d["ur"].cpu().numpy(), temperature=T)
        assert (want["accept_len"] == n).all() == accepted
        bad, ties, _ = compare_accept(dict(accept_len=got["len"].cpu().numpy(), out_tokens=got["tok"].cpu().numpy(),
                                           stop_node=got["stop"].cpu().numpy()), want, n)
        assert not bad and ties <= 1


@pytest.mark.parametrize("B,V,dtype,parent", [
    (4, 1000, torch.bfloat16, False), (4, 7, torch.bfloat16, False), (64, 128256, torch.bfloat16, False), (40, 32000, torch.float32, False),
    (4, 65545, torch.bfloat16, True), (3, 65544, torch.bfloat16, True),
])
def test_no_drafts_beside_draft_rows(B, V, dtype, parent):
    """No request has drafts, draft rows and a row number are there all the same (or are announced behind a null pointer): one token
    from every target row, on every path, whatever the workspace held, target statistics from the caller included."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    g = torch.Generator(device="cuda").manual_seed(3)
    target = (torch.randn((B, V), generator=g, device="cuda") * 2).to(dtype)
    draft = torch.randn((5, V), generator=g, device="cuda").to(dtype)
    one = torch.zeros(1, dtype=torch.int32, device="cuda")
    off, ur = torch.zeros(B + 1, dtype=torch.int32, device="cuda"), torch.rand(B, generator=g, device="cuda")
    ua = torch.zeros(1, device="cuda")
    # the token: the first class whose running sum passes u, in fp64; the next ones where u is within the sums' rounding of it
    c = float(np.float32(1.4426950408889634) / np.float32(0.9)) * np.log(2.0)
    cdf = torch.softmax(target.double() * c, 1).cumsum(1)
    lo, hi = ((cdf < (ur.double() + e)[:, None]).sum(1).clamp(max=V - 1) for e in (-1e-6, 1e-6))
    size = sv.spec_accept_workspace_size(B, 0, 5, V)
    for how in ("plain", "prestats", "null") if dtype == torch.bfloat16 else ("plain", "null"):
        ws = torch.randint(0, 256, (size,), dtype=torch.uint8, generator=g, device="cuda")
        if how == "prestats":
            rec = given_statistics(dict(target=target), 0.9, V)
            ws[:rec.numel()].copy_(rec)
        for _ in range(2):
            length = torch.full((B,), -7, dtype=torch.int32, device="cuda")
            tok, stop = torch.full((B, 1), -7, dtype=torch.int32, device="cuda"), torch.full((B,), -7, dtype=torch.int32, device="cuda")
            if how == "null":
                code = sv.SPEC_BF16 if dtype == torch.bfloat16 else sv.SPEC_F32
                rc = sv.lib().spec_accept(B, V, 0, 5, 0, off.data_ptr(), one.data_ptr() if parent else None, None, target.data_ptr(), code,
                                          None, code, sv.SPEC_Q_LOGITS, None, 0.9, None, ur.data_ptr(), length.data_ptr(), tok.data_ptr(), 1,
                                          stop.data_ptr(), None, ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
                assert rc == sv.SPEC_OK
            else:
                (sv.spec_accept_prestats if how == "prestats" else sv.spec_accept)(
                    B, 0, 0, off, one if parent else None, one, target, draft, sv.SPEC_Q_LOGITS, one, 0.9, ua, ur, length, tok, stop, None, ws)
            assert bool((length == 0).all()) and bool((stop == -1).all()), how
            assert bool(((tok[:, 0] >= lo) & (tok[:, 0] <= hi)).all()), how
