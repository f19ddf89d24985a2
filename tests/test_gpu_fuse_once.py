"""Averaging of the drafters' distributions in one launch (every drafter row read once) against fp64 torch and against the
three launches that a smaller workspace takes: one to six drafters, vocabularies at the edges of 8-class groups, waves and
4096-class segments, ragged draft lengths, a workspace of garbage that is not cleared between calls, and graph replays
on changed inputs (a captured call repeats its message tag).

Tolerance: a probability is a sum of fp32 exponentials (two roundings of the argument and one of the result: 4e-7
relative at |argument| <= 4, growing with the argument, 16 here) times an fp64 factor, rounded to fp32 once."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def make(B, k, N, V, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    logits = (2 * torch.randn((B * k * N, V), generator=g, device="cuda")).to(dtype)
    conf = torch.rand((B, k, N), generator=g, device="cuda")
    conf[0] = 0.0                                   # no confidence anywhere: equal weights
    toks = torch.randint(0, V, (B, k, N), generator=g, device="cuda").int()
    lens = torch.randint(0, k + 1, (B,), generator=g, device="cuda").int()
    lens[0] = k
    return dict(logits=logits, conf=conf, toks=toks, lens=lens)


def call(sv, d, ws, T=0.8, patience=None):
    B, k, N = d["conf"].shape
    V = d["logits"].shape[1]
    got = [torch.full((B, k), -9, dtype=torch.int32, device="cuda") for _ in range(3)]
    out = torch.full((B * k, V), -1.0, device="cuda")
    fuse = sv.spec_fuse_drafts if patience is None else lambda *a: sv.spec_fuse_drafts_tuned(patience, *a)
    fuse(d["lens"], d["conf"], d["toks"], d["logits"], T, sv.SPEC_FUSE_MIXTURE, *got, out, ws)
    return got, out


def exact(d, T=0.8):
    B, k, N = d["conf"].shape
    w = d["conf"].double()
    s = w.sum(-1, keepdim=True)
    w = torch.where(s > 0, w / s, torch.full_like(w, 1.0 / N)).view(B * k, N, 1)
    # (1/T as the library has it: log2(e) / T in fp32)
    c = float(np.float32(1.4426950408889634) / np.float32(T)) * np.log(2.0)
    p = torch.softmax(d["logits"].double() * c, 1).view(B * k, N, -1)
    return (w * p).sum(1)


@pytest.mark.parametrize("B,k,N,V,dtype", [
    (3, 2, 1, 5, torch.bfloat16), (2, 2, 2, 8, torch.float32), (2, 3, 3, 513, torch.bfloat16), (2, 2, 4, 4095, torch.float32),
    (2, 2, 5, 4097, torch.bfloat16), (3, 2, 6, 8193, torch.bfloat16), (2, 2, 6, 12290, torch.float32), (4, 6, 4, 32000, torch.bfloat16),
    (1, 3, 2, 131072, torch.bfloat16), (2, 2, 6, 65536, torch.bfloat16), (40, 8, 2, 9001, torch.bfloat16),
])
def test_mixture_in_one_launch(B, k, N, V, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    full = sv.spec_fuse_drafts_workspace_size(B, k, N, V, sv.SPEC_FUSE_MIXTURE)
    least = B * k * N * ((V + 8191) // 8192) * 16 + 256
    ws = torch.randint(0, 256, (max(full, least),), dtype=torch.uint8, device="cuda")
    for seed in range(3):
        d = make(B, k, N, V, dtype, seed)
        used = (torch.arange(k, device="cuda")[None] < d["lens"][:, None]).reshape(-1)
        ints, out = call(sv, d, ws)
        ref = exact(d)
        assert bool(((out.double() - ref).abs()[used] <= 2e-6 * ref[used]).all())
        assert bool((out[~used] == -1.0).all())                       # positions behind a draft's end stay as they were
        best = d["conf"].argmax(-1).int()
        assert torch.equal(ints[1].view(-1)[used], best.view(-1)[used]) and bool((ints[1].view(-1)[~used] == -1).all())
        other, three = call(sv, d, ws[:least].clone())
        assert all(torch.equal(a, b) for a, b in zip(ints, other))
        assert torch.allclose(out[used], three[used], rtol=2e-6, atol=0)


def test_mixture_in_one_launch_replays():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    shape = (3, 4, 3, 20000)
    sets = [make(*shape, torch.bfloat16, s) for s in range(4)]
    for s in sets:
        s["lens"].fill_(4)
    d = {k: v.clone() for k, v in sets[0].items()}
    ws = torch.empty(sv.spec_fuse_drafts_workspace_size(*shape, sv.SPEC_FUSE_MIXTURE), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(sv, d, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ints, out = call(sv, d, ws)
    for s in sets + sets:
        for k, v in s.items():
            d[k].copy_(v)
        graph.replay()
        torch.cuda.synchronize()
        ref, want = call(sv, s, torch.empty_like(ws))
        assert torch.equal(out, want) and all(torch.equal(a, b) for a, b in zip(ints, ref))


@pytest.mark.parametrize("T", [1.0, 0.05])
@pytest.mark.parametrize("B,k,N,V,dtype", [
    (2, 2, 3, 1000, torch.bfloat16), (2, 3, 4, 32000, torch.bfloat16), (2, 2, 6, 9001, torch.float32), (2, 2, 2, 50264, torch.float32),
])
def test_mixture_of_masked_rows_far_below_zero(B, k, N, V, dtype, T):
    """Drafters cut to a few classes (a thread's classes are all without mass in one drafter, not in another), rows whose largest
    logit over T overflows an exponential.  Tolerance: an argument of A binary places is rounded twice and the thread's
    maximum has an argument of its own, 2^-24 A each; 2^-21 is for the exponentials, the sums and the result."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    full = sv.spec_fuse_drafts_workspace_size(B, k, N, V, sv.SPEC_FUSE_MIXTURE)
    least = B * k * N * ((V + 8191) // 8192) * 16 + 256
    ws = torch.randint(0, 256, (max(full, least),), dtype=torch.uint8, device="cuda")
    for seed in range(2):
        d = make(B, k, N, V, dtype, seed)
        x = d["logits"].float()
        cut = x.topk(30, 1).values[:, -1:]
        odd = torch.arange(B * k * N, device="cuda")[:, None] % 2 == 1
        x = x.masked_fill(odd & (x < cut), -float("inf"))                        # every other drafter: 30 classes
        x = x.masked_fill(~odd & (torch.arange(V, device="cuda") // 512 % 3 == 0), -float("inf"))      # the others: runs of 512 gone
        d["logits"] = (x - (1500.0 if T == 1.0 else 60.0)).to(dtype)
        used = (torch.arange(k, device="cuda")[None] < d["lens"][:, None]).reshape(-1)
        c = float(np.float32(1.4426950408889634) / np.float32(T))
        lg = d["logits"].double()
        A = ((lg.amax(1, keepdim=True) - lg) * c).nan_to_num(0.0, posinf=0.0)
        w = d["conf"].double()
        s = w.sum(-1, keepdim=True)
        w = torch.where(s > 0, w / s, torch.full_like(w, 1.0 / N)).view(-1, N, 1)
        p = torch.softmax(lg * (c * np.log(2.0)), 1)
        ref = (w * p.view(-1, N, V)).sum(1)
        bound = (w * (p * (2.0 ** -21 + A * 2.0 ** -22)).view(-1, N, V)).sum(1) + 2.0 ** -125       # (below: no normal number)
        for room in (full, least):
            _, out = call(sv, d, ws[:room], T)
            assert bool(((out.double() - ref).abs() <= bound)[used].all()), room


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("B,k,N,V,dtype", [
    (2, 2, 2, 4097, torch.bfloat16), (2, 3, 4, 32000, torch.bfloat16), (2, 2, 6, 9001, torch.float32), (2, 2, 5, 12290, torch.bfloat16),
    (1, 3, 2, 131072, torch.bfloat16), (40, 8, 2, 9001, torch.bfloat16),
])
def test_mixture_without_waiting(B, k, N, V, dtype, masked):
    """Patience 0: a workgroup looks once and works out every record that is not there yet itself, with the same arithmetic in the
    same order: the same bits as with the records of its peers, a segment without any mass in some drafters among them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding as sv
    ws = torch.randint(0, 256, (sv.spec_fuse_drafts_workspace_size(B, k, N, V, sv.SPEC_FUSE_MIXTURE),), dtype=torch.uint8, device="cuda")
    for seed in range(3):
        d = make(B, k, N, V, dtype, seed)
        if masked:
            d["logits"][1::2, :4096] = -float("inf")
        want, ref = call(sv, d, ws)
        for _ in range(3):
            ints, out = call(sv, d, ws, patience=0)
            assert torch.equal(out, ref) and all(torch.equal(a, b) for a, b in zip(ints, want))
