"""Cases of the verification step that are timed and compared between two states of this repository.

A case is what a program that serves a target model with speculative drafts does once per decoding step, through
``paper_2503_10325_amd.binding``:

  step      attention of all draft tokens over the paged cache, token fusion where there are several drafters, and
            acceptance-rejection of the drafts;
  lm_head   the projection that makes the target logits, and the acceptance that starts from its statistics;
  mixture   weighted averaging of several drafters' distributions, and acceptance against the averaged distribution;
  greedy    greedy verification.

Sizes are those of ``workloads.CONFIGS`` and of the tests, and generic ones between them.  Values are drawn as
``workloads`` draws them (Q, K, V ~ N(0, 1), target logits ~ N(0, 3), draft logits = target + noise, drafted tokens
sampled from the very draft rows that are handed in), on the GPU.
"""
import math

import numpy as np
import torch

from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

PAGE = 16


def _step(name, batch, q_heads, kv_heads, head_dim, ctx, nodes, vocab, **more):
    c = {"path": "step", "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": head_dim,
         "ctx_kind": "fixed", "ctx": ctx, "ctx_max": ctx, "tree": "", "nodes_min": nodes, "nodes": nodes, "vocab": vocab,
         "logits": "bf16", "out": "bf16", "lse": False, "target_sd": 3.0, "noise": 1.0, "drafters": 1, "temperature": 1.0,
         "mix": 0}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one request, four drafts, a small model; launches and latency are all there is
        _step("step_tiny", 1, 8, 8, 64, 256, 4, 1000, target_sd=2.0, noise=2.0 * math.sqrt(2.0)),
        # an ordinary batch of a 7B-shaped model without grouped heads, eight drafts in a line
        _step("step_7b", 8, 32, 32, 128, 2048, 8, 32000),
        # draft trees on an 8B-shaped model: 256 query rows per KV head, a large vocabulary
        _step("step_tree", 16, 32, 8, 128, 4096, 64, 128256, tree="4,4,2,2"),
        # four drafters fused position by position, contexts of many lengths
        _step("step_fusion", 32, 32, 32, 128, 1024, 6, 32000, ctx_kind="uniform", ctx_max=4096, drafters=4, noise=1.5),
        # a 70B-shaped serving batch: ragged contexts, ragged drafts (adaptive speculation)
        _step("step_serving", 64, 64, 8, 128, 2048, 10, 128256, ctx_kind="lognormal", ctx_max=16384, nodes_min=2),
        # one user with a long document: few heads to spread over the chip, odd lengths
        _step("step_long", 1, 64, 8, 128, 15999, 7, 128256),
        # a small model with a vocabulary that no vector width divides, logits and output in fp32, a temperature
        _step("step_odd", 5, 12, 4, 64, 777, 9, 50257, ctx_kind="uniform", ctx_max=3001, nodes_min=3, logits="f32",
              out="f32", lse=True, temperature=0.8),
        # weighted averaging of four drafters (fp32 probabilities written and verified)
        _step("mixture", 32, 32, 32, 128, 1024, 6, 32000, path="mixture", drafters=4, noise=1.5),
        # greedy verification of draft trees with a large vocabulary
        _step("greedy_tree", 16, 32, 8, 128, 4096, 64, 128256, path="greedy", tree="4,4,2,2"),
        # the projection of an ordinary batch: bound by reading the weights
        _step("lm_head_7b", 8, 32, 32, 128, 2048, 8, 32000, path="lm_head"),
        # ... of the serving batch: 429 rows or so
        _step("lm_head_serving", 64, 64, 8, 128, 2048, 10, 128256, path="lm_head", nodes_min=2),
        # ... of the tree batch: 1040 rows, the most matrix work
        _step("lm_head_tree", 16, 32, 8, 128, 4096, 64, 128256, path="lm_head", tree="4,4,2,2"),
    ]


def _between(rng, lo, hi):
    """A whole number whose logarithm is uniform between those of lo and hi."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["step"] * 6 + ["lm_head"] * 3 + ["mixture", "greedy"])
    while True:
        c = _step("", _between(rng, 1, 64), 0, rng.choice([1, 2, 4, 8, 8, 16, 32]),
                  128 if path == "lm_head" else rng.choice([64, 128, 128]),
                  _between(rng, 64, 16384), rng.randint(1, 16), _between(rng, 1000, 131072), path=path, mix=rng.randrange(1 << 20))
        c["q_heads"] = c["kv_heads"] * rng.choice([1, 1, 2, 3, 4, 7, 8])
        c["ctx_kind"] = rng.choice(["fixed", "uniform", "lognormal"])
        c["ctx_max"] = c["ctx"] if c["ctx_kind"] == "fixed" else min(16384, c["ctx"] * rng.randint(2, 6))
        c["nodes_min"] = rng.randint(1, c["nodes"])
        c["temperature"] = rng.choice([1.0, 1.0, 0.8, 1.3])
        if path in ("mixture", "lm_head") or rng.random() < 0.75:      # most vocabularies are padded
            c["vocab"] = c["vocab"] // 64 * 64 + 64
        if path == "mixture" or (path == "step" and rng.random() < 0.2):
            c["drafters"], c["noise"], c["nodes_min"] = rng.randint(2, 6), 1.5, c["nodes"]
        elif rng.random() < 0.4:
            c["tree"], c["nodes"] = rng.choice([("4,4,2,2", rng.randint(20, 116)), ("2,2,2,2", rng.randint(8, 30)),
                                                ("3,2,2", rng.randint(6, 21)), ("8,4,2", rng.randint(16, 104))])
            c["nodes_min"] = c["nodes"]
        if path == "step":
            c["lse"] = rng.random() < 0.25
            c["out"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        if path in ("step", "greedy"):
            c["logits"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        w = work(c)
        rows = _target_rows(c)
        held = (rows + _draft_rows(c)) * c["vocab"] * (4 if c["logits"] == "f32" else 2)
        if path == "lm_head":
            if rows <= 1100 and 1e6 < w["bytes"] < 2.2e9 and w["flops"] < 9e11:
                return c
        elif held < 6e8 and 1e6 < w["bytes"] < 1.2e9 and w["flops"] < 1e11:
            return c


# ----------------------------------------------------------------------------------------------------------------
# sizes of a case
# ----------------------------------------------------------------------------------------------------------------
def _structure(c):
    """(context lengths, nodes per request, parent array of one request or None) of a case: its own, whatever the seed."""
    r = np.random.RandomState(c["mix"])
    B = c["batch"]
    if c["ctx_kind"] == "fixed":
        ctx = np.full(B, c["ctx"])
    elif c["ctx_kind"] == "uniform":
        ctx = r.randint(c["ctx"], c["ctx_max"] + 1, B)
    else:
        ctx = np.clip(np.rint(c["ctx"] * np.exp(0.8 * r.standard_normal(B))), min(512, c["ctx"]), c["ctx_max"])
    parent = W.tree_parents([int(x) for x in c["tree"].split(",")], c["nodes"]) if c["tree"] else None
    n = np.full(B, len(parent)) if parent is not None else r.randint(c["nodes_min"], c["nodes"] + 1, B)
    return ctx.astype(np.int64), n.astype(np.int64), parent


def _target_rows(c):
    _, n, _ = _structure(c)
    return int(n.sum()) + c["batch"]


def _draft_rows(c):
    _, n, parent = _structure(c)
    if parent is not None:
        return c["batch"] * len(set(parent.tolist()))
    return int(n.sum()) * c["drafters"]


def _walked_rows(c):
    """(target rows, draft rows) a walk reaches on average: a draft token is accepted with probability sum min(p, q),
    2 Phi(-s / 2) where the logarithm of the ratio p / q has standard deviation s; the rows behind the first rejection of
    a chain, and off the path of a tree, are not needed.  A further sibling is accepted about half as often as the
    first."""
    a = math.erfc(c["noise"] / c["temperature"] / 2 / math.sqrt(2.0))
    _, n, parent = _structure(c)
    t = q = 0.0
    for nb in n.tolist():
        if parent is None:
            q += sum(a ** j for j in range(nb))
            t += sum(a ** j for j in range(nb + 1))
        else:
            reach = 1.0
            for br in [int(x) for x in c["tree"].split(",")]:
                t += reach
                q += reach
                reach *= 1.0 - (1.0 - a) * (1.0 - a / 2) ** (br - 1)
            t += reach
    return t, q


def work(case):
    c = case
    ctx, n, _ = _structure(c)
    D, V, size = c["head_dim"], c["vocab"], 4 if c["logits"] == "f32" else 2
    rows = _target_rows(c)
    t, q = _walked_rows(c)
    if c["path"] == "step":
        L = ctx + n
        by = (2 * c["kv_heads"] * L * D * 2 + n * c["q_heads"] * D * (2 + (4 if c["out"] == "f32" else 2))).sum()
        return {"bytes": float(by + (t + q) * V * size), "flops": float((4 * n * c["q_heads"] * L * D).sum())}
    if c["path"] == "mixture":      # every position's averaged distribution is an output
        k = int(n.sum())
        return {"bytes": float(k * V * (c["drafters"] * 2 + 4) + t * V * 2), "flops": 0.0}
    if c["path"] == "greedy":       # the argmax of every row is an output
        return {"bytes": float(rows * V * size), "flops": 0.0}
    d = c["q_heads"] * D
    return {"bytes": float(V * d * 2 + rows * d * 2 + rows * V * 2 + q * V * 2), "flops": float(2 * rows * d * V)}


# Four times what the results are off by from the same operations in 64 bits, measured over the listed cases: attention
# with a bf16 output and the projection's logits 1.65e-3 to 1.67e-3 (2-norm) and 3.9e-3 to 4.6e-3 (largest), which is the
# rounding of the result to bf16; attention with an fp32 output 2e-6 with two-term bf16 weights and 2.4e-4 with fp16
# weights (many query rows per KV head); averaged distributions 5e-8 and 4e-7.  Whole numbers agree but for ties: a token
# drawn from a near-uniform distribution over 10^5 classes sits within one rounding of a class boundary now and then, and
# a logit that rounds the other way (3e-4 of them under another order of the sums) moves such a boundary.
def tolerance(case):
    if case["path"] == "greedy":
        return "exact"
    if case["path"] == "mixture":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.005}
    if case["path"] == "lm_head":
        return {"rel": 7e-3, "max": 2e-2, "differ": 0.01}
    if case["out"] == "f32":
        return {"rel": 1e-3, "max": 1e-2, "differ": 0.005}
    return {"rel": 7e-3, "max": 2e-2, "differ": 0.005}


# ----------------------------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------------------------
def _i32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def _uniforms(g, n):
    return torch.randint(0, 1 << 24, (n,), generator=g, device="cuda").float() * 2.0 ** -24


def _sample(g, logits, temperature, draws):
    """`draws` tokens per row by the Gumbel-max construction: [rows, draws] int32."""
    rows, V = logits.shape
    got = torch.empty((rows, draws), dtype=torch.int32, device="cuda")
    some = max(1, (1 << 26) // V)
    for i in range(0, rows, some):
        z = logits[i:i + some].float() / temperature
        for d in range(draws):
            u = torch.rand(z.shape, generator=g, device="cuda").clamp_(1e-20, 1.0 - 2.0 ** -24)
            got[i:i + some, d] = (z - torch.log(-torch.log(u))).argmax(1).int()
    return got


class _Attention:
    def __init__(self, c, g, seed, ctx, n, parent):
        B, H, D = c["batch"], c["kv_heads"], c["head_dim"]
        pages = (ctx + n + PAGE - 1) // PAGE
        total = int(pages.sum())
        perm = np.random.RandomState(seed % (1 << 32)).permutation(total)
        table = np.full((B, int(pages.max())), -1)
        at = 0
        for b in range(B):
            table[b, :pages[b]] = perm[at:at + pages[b]]
            at += int(pages[b])
        self.q = torch.randn((int(n.sum()), c["q_heads"], D), generator=g, device="cuda").bfloat16()
        self.k = torch.empty((total, H, PAGE, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
        self.v = torch.empty((total, H, PAGE, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
        self.table, self.ctx = _i32(table), _i32(ctx)
        self.offsets = _i32(np.concatenate([[0], np.cumsum(n)]))
        self.parent = None if parent is None else _i32(np.tile(parent, B))
        f32 = c["out"] == "f32"
        self.out = torch.empty(self.q.shape, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
        self.lse = torch.empty(self.q.shape[:2], dtype=torch.float32, device="cuda") if c["lse"] else None
        self.desc = sv.make_attn_desc(B, c["q_heads"], H, D, int(n.sum()), int(n.max()), table.shape[1],
                                      int((ctx + n).sum()), 0.0, sv.SPEC_F32 if f32 else sv.SPEC_BF16)
        self.workspace = torch.empty(max(256, sv.spec_verify_attn_workspace_size(self.desc)), dtype=torch.uint8, device="cuda")

    def run(self):
        sv.spec_verify_attn(self.desc, self.q, self.k, self.v, self.table, self.ctx, self.offsets, self.parent, self.out,
                            self.lse, self.workspace)


class _State:
    pass


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    ctx, n, parent = _structure(c)
    s = _State()
    s.path, s.temperature = c["path"], c["temperature"]
    B, V, N = c["batch"], c["vocab"], c["drafters"]
    s.B, s.total, s.most = B, int(n.sum()), int(n.max())
    s.attention = _Attention(c, g, seed, ctx, n, parent) if c["path"] == "step" else None
    offsets = np.concatenate([[0], np.cumsum(n)])
    s.offsets = _i32(offsets)
    s.parent = None if parent is None else _i32(np.tile(parent, B))
    dtype = torch.float32 if c["logits"] == "f32" else torch.bfloat16

    # target rows: local row 0 of a request is the distribution after its committed prefix, row 1 + j the one after node j
    rows = s.total + B
    if c["path"] == "lm_head":
        d = c["q_heads"] * c["head_dim"]
        s.hidden = torch.randn((rows, d), generator=g, device="cuda").bfloat16()
        s.weight = torch.empty((V, d), dtype=torch.bfloat16, device="cuda").normal_(0.0, c["target_sd"] / math.sqrt(d), generator=g)
        s.target = torch.empty((rows, V), dtype=torch.bfloat16, device="cuda")
        known = torch.matmul(s.hidden, s.weight.t())
        s.head_workspace = torch.empty(max(256, sv.spec_lm_head_workspace_size(rows, d, V)), dtype=torch.uint8, device="cuda")
    else:
        s.target = torch.empty((rows, V), dtype=dtype, device="cuda").normal_(0.0, c["target_sd"], generator=g)
        known = s.target

    # draft rows: one per node (times the drafters), or one per node of a tree that has children
    first = torch.from_numpy(np.repeat(offsets[:-1] + np.arange(B), n)).cuda()     # first target row of a node's request
    local = torch.from_numpy(np.concatenate([np.arange(k) if parent is None else parent + 1 for k in n])).cuda()
    source = first + local                                                        # target row a node is tested against
    kids = 1
    if parent is None:
        of_row = source.repeat_interleave(N)
        s.q_row = torch.arange(s.total, dtype=torch.int32, device="cuda")
    else:
        of_row, inverse = torch.unique(source, return_inverse=True)
        s.q_row = inverse.int()
        kids = int(np.bincount(parent + 1).max())
    s.draft = known[of_row]
    noise = torch.empty_like(s.draft)
    s.draft = (s.draft + noise.normal_(0.0, c["noise"], generator=g)).contiguous()
    del noise
    if c["path"] == "greedy":
        tokens = torch.topk(s.draft, kids, dim=1).indices.int()               # a drafter's best, then its next ones
    else:
        tokens = _sample(g, s.draft, c["temperature"], kids)
    if parent is None:
        s.tokens = tokens.reshape(-1).contiguous()
    else:       # the j-th child of a node holds the j-th token of its row
        order = [int((parent[:i] == p).sum()) for i, p in enumerate(parent)]
        s.tokens = tokens[s.q_row.long(), torch.from_numpy(np.tile(order, B)).cuda()].contiguous()
    if c["path"] == "lm_head":
        del known
    s.u_accept, s.u_resample = _uniforms(g, s.total), _uniforms(g, B)
    s.accept_len = torch.empty(B, dtype=torch.int32, device="cuda")
    s.stop = torch.empty(B, dtype=torch.int32, device="cuda")
    s.out_tokens = torch.empty((B, s.most + 1), dtype=torch.int32, device="cuda")
    s.q_kind, s.fuse, s.mixed = sv.SPEC_Q_LOGITS, N > 1, None
    if s.fuse:
        s.candidates = s.tokens.view(B, s.most, N)
        s.conf = _beta22(g, (B, s.most, N))
        s.lengths = _i32(n)
        s.tokens = torch.empty((B, s.most), dtype=torch.int32, device="cuda")
        s.winner = torch.empty((B, s.most), dtype=torch.int32, device="cuda")
        s.q_row = torch.empty((B, s.most), dtype=torch.int32, device="cuda")
        s.mode = sv.SPEC_FUSE_ARGMAX
        if c["path"] == "mixture":
            s.mode, s.q_kind = sv.SPEC_FUSE_MIXTURE, sv.SPEC_Q_PROBS
            s.mixed = torch.zeros((B * s.most, V), dtype=torch.float32, device="cuda")
        s.fuse_workspace = torch.empty(max(256, sv.spec_fuse_drafts_workspace_size(B, s.most, N, V, s.mode)), dtype=torch.uint8, device="cuda")
    draft_rows = (s.mixed if s.mixed is not None else s.draft).shape[0]
    if c["path"] == "greedy":
        s.row_argmax = torch.empty(rows, dtype=torch.int32, device="cuda")
        ws = sv.spec_accept_greedy_workspace_size(B, s.total, V)
    else:
        ws = sv.spec_accept_workspace_size(B, s.total, draft_rows, V)
    s.workspace = torch.empty(max(256, ws), dtype=torch.uint8, device="cuda")
    return s


def _beta22(g, shape):
    """Beta(2, 2): the median of three uniforms."""
    u = torch.rand(shape + (3,), generator=g, device="cuda")
    return u.median(-1).values.contiguous()


def run(state):
    s = state
    got = {}
    if s.attention is not None:
        s.attention.run()
        got["attention"] = s.attention.out
        if s.attention.lse is not None:
            got["lse"] = s.attention.lse
    if s.path == "lm_head":
        sv.spec_lm_head(s.hidden, s.weight, s.temperature, s.target, s.workspace, s.head_workspace)
        got["logits"] = s.target
    if s.fuse:
        sv.spec_fuse_drafts(s.lengths, s.conf, s.candidates, s.draft, s.temperature, s.mode, s.tokens, s.winner, s.q_row,
                            s.mixed, s.fuse_workspace)
        got["fused"], got["winner"] = s.tokens, s.winner
        if s.mixed is not None:
            got["mixed"] = s.mixed
    if s.path == "greedy":
        sv.spec_accept_greedy(s.B, s.total, s.most, s.offsets, s.parent, s.tokens, s.target, s.accept_len, s.out_tokens,
                              s.stop, s.row_argmax, s.workspace)
        got["row_argmax"] = s.row_argmax
    else:
        accept = sv.spec_accept_prestats if s.path == "lm_head" else sv.spec_accept
        accept(s.B, s.total, s.most, s.offsets, s.parent, s.tokens, s.target, s.mixed if s.mixed is not None else s.draft,
               s.q_kind, s.q_row, s.temperature, s.u_accept, s.u_resample, s.accept_len, s.out_tokens, s.stop, None,
               s.workspace)
    got["accept_len"], got["out_tokens"], got["stop_node"] = s.accept_len, s.out_tokens, s.stop
    return got
