"""Performance cases of the verify step: what a serving loop or a scheduler
study asks of this library, through its C ABI (paper_2505_17074_amd.binding).

Four kinds of call ("path"):
  verify   spec_verify: attention and acceptance of one round
  attn     spec_verify_attn: the attention of one model layer (an engine calls
           it once per layer and round)
  accept   spec_accept: acceptance and the final sample of one round
  lm_head  spec_lm_head_accept: the LM head with the acceptance behind it

A case holds sizes and options only.  Per-request lengths and tree shapes come
from the case (its "mix"), values from the seed of prepare().
"""
import math

import numpy as np
import torch

from paper_2505_17074_amd import binding as B

_DEV = "cuda"
_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
_SPEC = {"bf16": B.SPEC_BF16, "f32": B.SPEC_F32}


def _case(name, path, batch, draft, k, **kw):
    c = {"path": path, "batch": batch, "draft": draft, "k": k, "mix": 0}
    if name:
        c["name"] = name
    if path in ("verify", "attn"):
        c.update(ctx="uniform", ctx_lo=512, ctx_hi=2048, hq=32, hkv=8, d=128, qkv="bf16", page=0)
    if path != "attn":
        c.update(vocab=32000, logits="f32", rule="independent")
    if path == "lm_head":
        c.update(hidden=4096)
    c.update(kw)
    return c


def listed():
    return [
        # one interactive request (the paper serves one at a time): LLaMA-7B heads,
        # a kilotoken of context, four drafts.  Latency and launches count.
        _case("step_b1", "verify", 1, "const", 4, ctx_lo=1000, ctx_hi=1000, hkv=32),
        # the benchmark's round: many ragged GQA requests with adaptive draft lengths
        _case("step_ragged_b128", "verify", 128, "uniform", 8, ctx="lognormal", ctx_lo=32, ctx_hi=8192),
        # token-tree rounds: 15-node binary trees over 2048 cached tokens
        _case("step_tree15_b64", "verify", 64, "tree", 15, ctx_lo=2048, ctx_hi=2048),
        # one layer of the paper's target model (MHA) over a mid-size batch
        _case("attn_mha7b_b32", "attn", 32, "const", 4, hkv=32),
        # the ragged batch over a paged KV cache (64-token pages, shuffled)
        _case("attn_paged_ragged_b128", "attn", 128, "uniform", 8, ctx="lognormal", ctx_lo=32, ctx_hi=8192, page=64),
        # long contexts, wide GQA groups, eight drafts
        _case("attn_long_b8", "attn", 8, "const", 8, ctx_lo=16384, ctx_hi=32768, hq=64),
        # fp32 attention: the fp32 model's heads at the mid-size batch's contexts
        _case("attn_f32_b32", "attn", 32, "const", 4, hq=8, hkv=8, d=64, qkv="f32"),
        # acceptance over a large bf16 vocabulary, few requests
        _case("accept_long_b8", "accept", 8, "const", 8, vocab=128256, logits="bf16"),
        # sequential sibling verification of token trees
        _case("accept_seq_tree_b64", "accept", 64, "tree", 15, rule="sequential"),
        # the LM head of a few interactive requests (20 rows: bound by the weights)
        _case("lm_head_b4", "lm_head", 4, "const", 4),
        # the LM head of the ragged batch (several hundred rows: bound by the matrix cores)
        _case("lm_head_ragged_b128", "lm_head", 128, "uniform", 8),
        # a wide model's head over a large vocabulary, bf16 logits
        _case("lm_head_long_b8", "lm_head", 8, "const", 8, vocab=128256, hidden=8192, logits="bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["verify", "attn", "attn", "accept", "lm_head", "lm_head"])
    draft = rng.choice(["const", "uniform", "uniform", "tree", "trees"])
    k = rng.randint(1, 8) if draft in ("const", "uniform") else rng.randint(3, 24)
    batch = _log_int(rng, 1, 128)
    kw = {"mix": rng.randint(1, 1 << 20)}
    if path in ("verify", "attn"):
        hq, hkv, d = rng.choice([(32, 32, 128), (32, 8, 128), (64, 8, 128), (32, 4, 128), (12, 12, 64), (16, 4, 64)])
        hi = _log_int(rng, 64, 32768)
        qkv = rng.choice(["bf16", "bf16", "bf16", "f32"])
        if qkv == "f32":
            hq, hkv, d, hi = 8, 8, 64, min(hi, 4096)
        while batch > 1 and batch * hi * hkv * d * (8 if qkv == "f32" else 4) > 600e6:
            batch = max(1, batch // 2)
        kw.update(ctx=rng.choice(["uniform", "lognormal"]), ctx_lo=max(1, hi // rng.choice([1, 2, 4, 16])), ctx_hi=hi,
                  hq=hq, hkv=hkv, d=d, qkv=qkv, page=rng.choice([0, 0, 32, 64]) if qkv == "bf16" else 0)
    if path != "attn":
        logits = rng.choice(["f32", "bf16"])
        vocab = rng.choice([32000, 128256, _log_int(rng, 1000, 128256)])
        while batch > 1 and batch * (k + 1) * vocab > 31e6:
            batch = max(1, batch // 2)
        rule = rng.choice(["independent", "sequential"]) if draft in ("tree", "trees") else "independent"
        kw.update(logits=logits, vocab=vocab, rule=rule)
    if path == "lm_head":
        hidden = rng.choice([1024, 2048, 4096, 5120, 8192])
        while batch > 1 and 2.0 * batch * (k + 1) * hidden * vocab > 180e9:
            batch = max(1, batch // 2)
        kw.update(hidden=hidden)
    return _case("", path, batch, draft, k, **kw)


# ---- shapes of a case ------------------------------------------------------
def _shape(c):
    """Per-request contexts and verify trees (chains too, as parent arrays)."""
    rng = np.random.default_rng([c["mix"], c["batch"], c["k"]])
    n = c["batch"]
    if "ctx" not in c:
        ctx = np.zeros(n, np.int64)
    elif c["ctx"] == "lognormal":       # median: an eighth of the longest, as in the ragged batch
        ctx = np.clip(np.rint(rng.lognormal(math.log(max(c["ctx_hi"] / 8, 1)), 1.0, n)), c["ctx_lo"], c["ctx_hi"])
    else:
        ctx = rng.integers(c["ctx_lo"], c["ctx_hi"] + 1, n)
    parents = []
    for _ in range(n):
        if c["draft"] == "const":
            par = np.arange(-1, c["k"])
        elif c["draft"] == "uniform":
            par = np.arange(-1, int(rng.integers(1, c["k"] + 1)))
        elif c["draft"] == "tree":      # binary, breadth first
            par = (np.arange(c["k"]) - 1) // 2
        else:                           # one random tree per request
            m = int(rng.integers(2, c["k"] + 1))
            par = np.array([-1] + sorted(int(rng.integers(0, j)) for j in range(1, m)))
            par[1:] = np.minimum(par[1:], np.arange(m - 1))
        parents.append(par.astype(np.int32))
    return ctx.astype(np.int32), parents


def _inner(par):
    return sorted(set(int(x) for x in par[1:]))


def _ancestors(par):
    m = np.eye(len(par), dtype=bool)
    for j in range(1, len(par)):
        m[j] |= m[par[j]]
    return m


def work(case):
    ctx, parents = _shape(case)
    nq = sum(len(p) for p in parents)
    by, fl = 0, 0
    if "hq" in case:
        s, rows = (4 if case["qkv"] == "f32" else 2), int(ctx.sum()) + nq
        by += rows * case["hkv"] * case["d"] * 2 * s + nq * case["hq"] * case["d"] * (s + 4)
        fl += 4 * case["d"] * case["hq"] * sum(int(c) * len(p) + int(_ancestors(p).sum()) for c, p in zip(ctx, parents))
    if "vocab" in case:
        s, v, b = (4 if case["logits"] == "f32" else 2), case["vocab"], case["batch"]
        ids = (nq - b) * (4 + s) + nq * 4 + 12 * b
        if case["path"] == "lm_head":
            h = case["hidden"]
            by += (nq * h + v * h) * 2 + nq * v * s + b * v * s + ids
            fl += 2 * nq * h * v
        else:
            # rows whose normalisers the tests need, and one draft row per request
            rows = sum(len(_inner(p)) for p in parents) + b
            by += min(rows, nq) * v * s + b * v * s + ids
            fl += 4 * rows * v
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # Four times the distance measured from 64 bits: 2.5e-6 for bf16 attention
    # (probabilities carried in two bf16 parts), 5e-7 for fp32 attention, 4e-7
    # for fp32 logits.  bf16 logits are 1.7e-3 from 64 bits by their storage;
    # two correct sums differ by one rounding step where they straddle a
    # boundary, about 5e-5 in all.  Tokens differ only at ties.
    t = {"differ": 0.01, "rel": 0.0}
    if case["path"] in ("verify", "attn"):
        t["rel"] = 1e-5 if case["qkv"] == "bf16" else 2e-6
    elif case["path"] == "lm_head":
        t.update({"rel": 2e-6} if case["logits"] == "f32" else {"rel": 2e-4, "max": 1e-2})
    return t


# ---- inputs and calls ------------------------------------------------------
class _Step:
    """One batch's device tensors, its argument structs, workspace and ring of
    pinned staging buffers (a buffer is rewritten once the stream has passed
    the calls that used it; one event covers eight calls)."""

    RING, EVERY = 32, 8

    def __init__(self, case, seed):
        self.case = case
        g = torch.Generator(device=_DEV)
        g.manual_seed(int(seed) * 7919 + 17)
        self.ctx, self.parents = _shape(case)
        self.nq = [len(p) for p in self.parents]
        self.q0 = np.concatenate([[0], np.cumsum(self.nq)])
        par0 = self.parents[0]
        if case["draft"] in ("const", "uniform"):
            self.req = B.make_requests(self.ctx, [n - 1 for n in self.nq])
        elif case["draft"] == "tree":
            self.req = B.make_requests(self.ctx, None, par0)
        else:
            self.req = B.make_requests(self.ctx, tree_parents=self.parents)
        self.attn = self.acc = self.lm = None
        if "hq" in case:
            self._attention(g)
        if "vocab" in case:
            self._acceptance(g)
        size = (B.spec_lm_head_workspace_bytes(self.req, self.lm, self.acc) if self.lm is not None
                else B.spec_workspace_bytes(self.req, self.attn, self.acc))
        B.check(size[0], "workspace size")
        self.ws_bytes, self.host_bytes = size[1], size[2]
        self._ws = torch.empty(self.ws_bytes + 256, dtype=torch.uint8, device=_DEV)
        self.ws = (self._ws.data_ptr() + 255) // 256 * 256
        slot = (self.host_bytes + 255) // 256 * 256
        self._staging = torch.empty(self.RING * slot + 256, dtype=torch.uint8, pin_memory=True)
        base = (self._staging.data_ptr() + 255) // 256 * 256
        self.slots = [base + i * slot for i in range(self.RING)]
        self.events = [None] * (self.RING // self.EVERY)
        self.calls = 0

    def _attention(self, g):
        c = self.case
        dt, hq, hkv, d = _DTYPE[c["qkv"]], c["hq"], c["hkv"], c["d"]
        rows = self.ctx.astype(np.int64) + self.nq
        self.kv0 = np.concatenate([[0], np.cumsum(rows)])
        self.q = torch.randn((int(self.q0[-1]), hq, d), generator=g, device=_DEV, dtype=dt)
        self.out = torch.empty((int(self.q0[-1]), hq, d), dtype=torch.float32, device=_DEV)
        a = self.attn = B.SpecAttnArgs()
        a.num_q_heads, a.num_kv_heads, a.head_dim, a.dtype = hq, hkv, d, _SPEC[c["qkv"]]
        a.q, a.out = self.q.data_ptr(), self.out.data_ptr()
        a.q_stride_tok, a.q_stride_head = hq * d, d
        a.kv_stride_tok, a.kv_stride_head = hkv * d, d
        if c["page"]:
            pages = -(-rows // c["page"])
            total = int(pages.sum())
            order = torch.randperm(total + 3, generator=g, device=_DEV)[:total].to(torch.int32)
            first = np.concatenate([[0], np.cumsum(pages)])
            self.table = torch.zeros((c["batch"], int(pages.max())), dtype=torch.int32, device=_DEV)
            for i in range(c["batch"]):
                self.table[i, :int(pages[i])] = order[int(first[i]):int(first[i + 1])]
            n = (total + 3) * c["page"]
            a.block_table, a.block_stride = self.table.data_ptr(), self.table.shape[1]
            a.page_tokens, a.num_pages = c["page"], total + 3
        else:
            n = int(rows.sum())
        self.k = torch.randn((n, hkv, d), generator=g, device=_DEV, dtype=dt)
        self.v = torch.randn((n, hkv, d), generator=g, device=_DEV, dtype=dt)
        a.k, a.v = self.k.data_ptr(), self.v.data_ptr()

    def _acceptance(self, g):
        c = self.case
        dt, V, nq, b = _DTYPE[c["logits"]], c["vocab"], int(self.q0[-1]), c["batch"]
        stride = -(-V // 8) * 8                     # 16-byte rows
        rng = np.random.default_rng([c["mix"], 99])
        sigma = np.repeat(rng.uniform(0.3, 2.5, b), self.nq).astype(np.float32)
        sigma = torch.from_numpy(sigma).to(_DEV)[:, None]
        self.logits = torch.zeros((nq, stride), dtype=dt, device=_DEV)
        if c["path"] == "lm_head":
            h = c["hidden"]
            self.hidden = torch.randn((nq, h), generator=g, device=_DEV, dtype=torch.bfloat16)
            self.weight = torch.randn((V, h), generator=g, device=_DEV, dtype=torch.bfloat16)
            self.weight *= 2.0 / math.sqrt(h)       # logits with a deviation of about 2
            base = torch.matmul(self.hidden, self.weight.t()).float()
        else:
            base = 2.0 * torch.randn((nq, V), generator=g, device=_DEV)
            self.logits[:, :V] = (base + sigma * torch.randn((nq, V), generator=g, device=_DEV)).to(dt)
        # draft rows of the nodes with children; each node's token from its parent's row
        inner, src, d0 = [], [], 0
        for i, par in enumerate(self.parents):
            own = _inner(par)
            inner += [int(self.q0[i]) + x for x in own]
            src += [d0 + own.index(int(x)) for x in par[1:]]
            d0 += len(own)
        if c["path"] == "lm_head":
            rows = torch.tensor(inner, device=_DEV)
            z = base[rows] + sigma[rows] * torch.randn((len(inner), V), generator=g, device=_DEV)
        else:
            z = base[torch.tensor(inner, device=_DEV)]
        self.probs = torch.zeros((len(inner), stride), dtype=dt, device=_DEV)
        self.probs[:, :V] = torch.softmax(z, -1).to(dt)
        at = torch.tensor(src, device=_DEV)
        tokens = torch.empty(len(src), dtype=torch.int32, device=_DEV)
        for s in range(0, len(src), 256):
            tokens[s:s + 256] = torch.multinomial(self.probs[at[s:s + 256], :V].float(), 1, generator=g)[:, 0].int()
        self.tokens, self.inner = tokens, inner
        self.uniforms = torch.randint(0, 1 << 24, (nq,), generator=g, device=_DEV).float() * 2.0 ** -24
        self.accepted, self.next, self.node = (torch.empty(b, dtype=torch.int32, device=_DEV) for _ in range(3))
        a = self.acc = B.SpecAcceptArgs()
        a.vocab, a.dtype = V, _SPEC[c["logits"]]
        a.target_logits, a.logits_stride = self.logits.data_ptr(), stride
        a.draft_probs, a.probs_stride = self.probs.data_ptr(), stride
        a.draft_tokens, a.uniforms = self.tokens.data_ptr(), self.uniforms.data_ptr()
        a.accepted_len, a.next_token, a.accepted_node = (x.data_ptr() for x in (self.accepted, self.next, self.node))
        a.tree_rule = B.SPEC_TREE_SEQUENTIAL if c["rule"] == "sequential" else B.SPEC_TREE_INDEPENDENT
        if c["path"] == "lm_head":
            m = self.lm = B.SpecLmHeadArgs()
            m.hidden_dim = m.hidden_stride = m.weight_stride = c["hidden"]
            m.hidden, m.weight = self.hidden.data_ptr(), self.weight.data_ptr()

    def call(self):
        s = self.calls % self.RING
        group = s // self.EVERY
        if s % self.EVERY == 0 and self.events[group] is not None:
            self.events[group].synchronize()
        self.calls += 1
        stream = torch.cuda.current_stream().cuda_stream
        rest = (self.ws, self.ws_bytes, self.slots[s], self.host_bytes, stream)
        path = self.case["path"]
        if path == "verify":
            st = B.spec_verify(self.req, self.attn, self.acc, *rest)
        elif path == "attn":
            st = B.spec_verify_attn(self.req, self.attn, *rest)
        elif path == "accept":
            st = B.spec_accept(self.req, self.acc, *rest)
        else:
            st = B.spec_lm_head_accept(self.req, self.lm, self.acc, *rest)
        B.check(st, path)
        if s % self.EVERY == self.EVERY - 1:
            self.events[group] = torch.cuda.Event()
            self.events[group].record()

    def outputs(self):
        r = {}
        if self.attn is not None:
            r["out"] = self.out
        if self.lm is not None:
            r["logits"] = self.logits[:, :self.case["vocab"]]
        if self.acc is not None:
            r.update(accepted_len=self.accepted, next_token=self.next, accepted_node=self.node)
        return r


def prepare(case, seed):
    return _Step(case, seed)


def run(state):
    state.call()
    return state.outputs()


# ---- the same outputs in 64 bits -------------------------------------------
def _attention64(s):
    c = s.case
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    out = torch.empty((int(s.q0[-1]), hq, d), dtype=torch.float64, device=_DEV)
    for i, par in enumerate(s.parents):
        n, length = len(par), int(s.ctx[i]) + len(par)
        if c["page"]:
            t = torch.arange(length, device=_DEV)
            rows = s.table[i].long()[t // c["page"]] * c["page"] + t % c["page"]
        else:
            rows = torch.arange(int(s.kv0[i]), int(s.kv0[i]) + length, device=_DEV)
        k, v = s.k[rows], s.v[rows]
        seen = torch.ones((n, length), dtype=torch.bool, device=_DEV)
        seen[:, int(s.ctx[i]):] = torch.from_numpy(_ancestors(par)).to(_DEV)
        q = s.q[int(s.q0[i]):int(s.q0[i + 1])].double()
        for h in range(hq):
            kh, vh = k[:, h // (hq // hkv)].double(), v[:, h // (hq // hkv)].double()
            x = torch.mm(q[:, h].contiguous(), kh.t().contiguous()) / math.sqrt(d)
            p = torch.softmax(x.masked_fill(~seen, -math.inf), -1)
            out[int(s.q0[i]):int(s.q0[i + 1]), h] = torch.mm(p, vh.contiguous())
    return out


def _sample(w, u):
    """The smallest id whose cumulative weight exceeds u * total."""
    cum = torch.cumsum(w, 0)
    over = torch.nonzero(cum > u * cum[-1])
    return int(over[0]) if len(over) else int(torch.nonzero(w > 0)[-1])


def _accept64(s):
    V = s.case["vocab"]
    got, d0 = [], 0
    tokens, uniforms = s.tokens.tolist(), s.uniforms.double().tolist()
    for i, par in enumerate(s.parents):
        n, q0, own = len(par), int(s.q0[i]), _inner(par)
        p = torch.softmax(s.logits[q0:q0 + n, :V].double(), -1)
        q = s.probs[d0:d0 + len(own), :V].double()
        d0 += len(own)
        tok = [0] + tokens[q0 - i:q0 - i + n - 1]
        u, depth = uniforms[q0:q0 + n], [0] * n
        for j in range(1, n):
            depth[j] = depth[int(par[j])] + 1
        kids = {x: [j for j in range(1, n) if par[j] == x] for x in range(n)}
        if s.case["rule"] == "sequential":
            node = 0
            while True:
                w, step = p[node], -1
                for j in kids[node]:
                    row = q[own.index(node)]
                    if u[j - 1] * float(row[tok[j]]) < float(w[tok[j]]):
                        step = j
                        break
                    rest = (w - row).clamp_min(0)
                    w = rest / rest.sum() if float(rest.sum()) > 0 else w
                if step < 0:
                    break
                node = step
        else:
            live, node = {0}, 0
            for j in range(1, n):
                x = int(par[j])
                if x in live and u[j - 1] * float(q[own.index(x)][tok[j]]) < float(p[x][tok[j]]):
                    live.add(j)
                    node = j if depth[j] > depth[node] else node
            w = p[node]
            if node in own:
                rest = (w - q[own.index(node)]).clamp_min(0)
                w = rest if float(rest.sum()) > 0 else w
        got.append((depth[node], _sample(w, u[n - 1]), node))
    t = torch.tensor(got, dtype=torch.int32)
    return {"accepted_len": t[:, 0].clone(), "next_token": t[:, 1].clone(), "accepted_node": t[:, 2].clone()}


def exact(case, seed):
    s = _Step(case, seed)
    r = {}
    if s.attn is not None:
        r["out"] = _attention64(s)
    if s.lm is not None:
        # whole numbers follow from the stored logits, which the path rounds
        r.update(accepted_len=None, next_token=None, accepted_node=None)
        h = s.hidden.double()
        r["logits"] = torch.cat([torch.mm(h, s.weight[v:v + 8192].double().t().contiguous())
                                 for v in range(0, case["vocab"], 8192)], 1)
    elif s.acc is not None:
        r.update(_accept64(s))
    return r
