"""Batches of fewer streams than the device has slots: the plan cuts them into
short pieces and a separate combine follows, and small steps stay on the
caller's stream.  Attention against fp64 within a derived bound at the rule's
edges (streams just under and over its shortest cut, one to five waves, more
pieces than the combine takes in one pass), the whole step against the
attention and acceptance calls alone on both sides of the stream rule, and the
no-allocation call's coarser plan."""
import numpy as np
import pytest
import torch

import parity_util as U
from paper_2505_17074_amd import binding as B
from paper_2505_17074_amd import workload as W
from paper_2505_17074_amd.batch import DeviceBatch, PagedKV, Verifier
from test_gpu_f32_attn import reference_and_bound

# bf16 probabilities are carried in two bf16 parts (a relative 2^-17)
P_REL = 2.0 ** -17
CASES = [
    ("uncut_238", dict(ctx=[233, 3], k=[4, 4], Hq=4, Hkv=4)),
    ("cut_239", dict(ctx=[234, 3], k=[4, 4], Hq=4, Hkv=4)),
    ("k0_one_row", dict(ctx=[700], k=[0], Hq=2, Hkv=2)),
    ("two_waves", dict(ctx=[1000], k=[4], Hq=8, Hkv=2)),
    ("three_waves_d64", dict(ctx=[515, 65], k=[8, 2], Hq=8, Hkv=2, d=64)),
    ("four_waves_tree", dict(ctx=[2000], tree_parent=W.full_binary_tree_parents(2, 4), Hq=8, Hkv=2)),
    ("five_waves", dict(ctx=[1500, 90], k=[8, 8], Hq=16, Hkv=2)),
    ("half_the_slots", dict(ctx=[600, 300] * 16, k=[4] * 32, Hq=32, Hkv=8)),
    ("over_half_the_slots", dict(ctx=[600, 300] * 16 + [500], k=[4] * 33, Hq=32, Hkv=8)),
    ("many_pieces", dict(ctx=[34000], k=[2], Hq=4, Hkv=1)),
    ("f32_uncut_151", dict(ctx=[146], k=[4], Hq=2, Hkv=2, d=64, qkv=W.F32)),
    ("f32_cut_152", dict(ctx=[147], k=[4], Hq=2, Hkv=2, d=64, qkv=W.F32)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,kw", CASES, ids=[c[0] for c in CASES])
def test_short_pieces(gpu_lib, name, kw):
    print(f"[small] {name}", flush=True)
    pool = U.custom_pool(**kw, seed=U.case_seed(name))
    b = DeviceBatch(pool, "cuda")
    f32 = pool.qkv_dtype == W.F32
    ref, bound = reference_and_bound(pool, 0.0 if f32 else P_REL)
    v = Verifier(b)
    b.out.fill_(float("nan"))
    v.run("attn")
    out = v.results()["out"]
    assert (np.abs(out - ref) <= bound).all(), float((np.abs(out - ref) / bound).max())
    if not f32:
        b.out.fill_(float("nan"))
        pk = PagedKV(b, 32)              # holds the page pools while they are read
        paged = Verifier(b, attn=pk.attn_args())
        paged.run("attn")
        assert np.array_equal(paged.results()["out"], out)


# requests, context, drafts, vocabulary, whether two streams run: the rule's line at
# 165 MiB of K/V (8 KB a key here) and 1.2 times the logits, few and many of them
STEPS = [
    ("kv_163", 8, 5200, 3, 5000, False),
    ("kv_169", 8, 5400, 3, 5000, True),
    ("logits_little", 16, 1500, 8, 32000, False),     # 94 MiB of K/V, 20 of logits
    ("logits_much", 16, 1500, 8, 128256, True),       # and 78
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,n,ctx,k,V,two", STEPS, ids=[c[0] for c in STEPS])
def test_step_on_one_or_two_streams(gpu_lib, name, n, ctx, k, V, two):
    print(f"[small] step {name}", flush=True)
    pool = U.custom_pool(ctx=[ctx] * n, k=[k] * n, Hq=8, Hkv=8, V=V, seed=5)
    b = DeviceBatch(pool, "cuda")
    v = Verifier(b)
    v.run("attn")
    v.run("accept")
    want = v.results()
    for t in (b.out, b.accepted_len, b.next_token, b.accepted_node):
        t.zero_()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()                      # creates the handles
    v.attn.event_end, v.acc.event_begin = ev[0].cuda_event, ev[1].cuda_event
    v.run("verify")
    got = v.results()
    for key in want:
        assert np.array_equal(want[key], got[key]), key
    # on one stream the acceptance begins once the attention has ended
    assert (ev[0].elapsed_time(ev[1]) < 0) == two


@pytest.mark.gpu
@pytest.mark.parametrize("qkv", [W.BF16, W.F32], ids=["bf16", "f32"])
def test_workspace_kept_from_another_batch(gpu_lib, qkv):
    """A workspace and a staging buffer that hold four pieces per stream (fp32: six;
    the longer pieces are of half the rows an item), not those the automatic
    split cuts: longer ones run in them, and nothing is written past their
    ends."""
    print(f"[small] kept workspace {qkv}", flush=True)
    f32 = qkv == W.F32
    pool = U.custom_pool(ctx=[3000], k=[4] if not f32 else [15], Hq=32, Hkv=8, seed=9, qkv=qkv)
    b = DeviceBatch(pool, "cuda")
    ref, bound = reference_and_bound(pool, 0.0 if f32 else P_REL)
    a = b.attn_args()
    a.split_kv = 768 if not f32 else 512
    req = b.requests()
    st, dev, host = B.spec_workspace_bytes(req, a, None)
    B.check(st, "workspace of four pieces")
    a.split_kv = 0
    st, dev0, host0 = B.spec_workspace_bytes(req, a, None)
    B.check(st, "workspace of the automatic split")
    assert dev < dev0 and host < host0
    ws = torch.full((dev + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    staging = torch.full((host + 4096,), 0xA5, dtype=torch.uint8, pin_memory=True)
    assert ws.data_ptr() % 256 == 0
    b.out.fill_(float("nan"))
    stream = torch.cuda.current_stream().cuda_stream
    B.check(B.spec_verify_attn(req, a, ws.data_ptr(), dev, staging.data_ptr(), host, stream), "kept workspace")
    torch.cuda.synchronize()
    assert (np.abs(b.out.cpu().numpy() - ref) <= bound).all()
    assert bool((ws[dev:] == 0xA5).all()) and bool((staging[host:] == 0xA5).all())


@pytest.mark.gpu
def test_noalloc_runs_the_longer_pieces(gpu_lib):
    """A step whose automatic split does not fit the static scratch beside the
    acceptance's statistics of a 4M-entry vocabulary, and whose longer pieces
    do: attention against fp64 for some of the requests, the acceptance as
    spec_accept gives it."""
    print("[small] noalloc, longer pieces", flush=True)
    n, k, ctx, V, d, Hq = 100, 9, 12000, 4000000, 128, 8
    nq = n * (k + 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)
    q, kk, vv = normal(nq, Hq, d), normal(n * (ctx + k + 1), 1, d), normal(n * (ctx + k + 1), 1, d)
    out = torch.full((nq, Hq, d), float("nan"), device="cuda")
    logits, probs = normal(nq, V), torch.empty((n * k, V), dtype=torch.bfloat16, device="cuda")
    for r in range(0, n * k, 50):
        probs[r:r + 50] = torch.softmax(2 * normal(min(50, n * k - r), V).float(), -1).bfloat16()
    tokens = torch.randint(0, V, (n * k,), generator=g, device="cuda", dtype=torch.int32)
    uniforms = torch.rand(nq, generator=g, device="cuda") * 0.5
    req = B.make_requests(np.full(n, ctx), np.full(n, k))
    a = B.SpecAttnArgs()
    a.num_q_heads, a.num_kv_heads, a.head_dim, a.dtype = Hq, 1, d, B.SPEC_BF16
    a.q, a.k, a.v, a.out = q.data_ptr(), kk.data_ptr(), vv.data_ptr(), out.data_ptr()
    a.q_stride_tok, a.q_stride_head, a.kv_stride_tok, a.kv_stride_head = Hq * d, d, d, d
    acc = []
    for _ in range(2):
        o = [torch.full((n,), -5, dtype=torch.int32, device="cuda") for _ in range(3)]
        c = B.SpecAcceptArgs()
        c.vocab, c.dtype, c.logits_stride, c.probs_stride = V, B.SPEC_BF16, V, V
        c.target_logits, c.draft_probs = logits.data_ptr(), probs.data_ptr()
        c.draft_tokens, c.uniforms = tokens.data_ptr(), uniforms.data_ptr()
        c.accepted_len, c.next_token, c.accepted_node = (x.data_ptr() for x in o)
        acc.append((c, o))
    st, dev, _ = B.spec_workspace_bytes(req, a, acc[0][0])
    assert st == B.SPEC_OK and dev > B.SPEC_NOALLOC_SCRATCH_BYTES
    h = torch.cuda.current_stream().cuda_stream
    B.check(B.spec_verify_noalloc(req, a, acc[0][0], h), "spec_verify_noalloc")
    st, dev, host = B.spec_workspace_bytes(req, None, acc[1][0])
    B.check(st, "workspace")
    ws = torch.empty(dev + 256, dtype=torch.uint8, device="cuda")
    staging = torch.empty(host, dtype=torch.uint8, pin_memory=True)
    B.check(B.spec_accept(req, acc[1][0], (ws.data_ptr() + 255) // 256 * 256, dev, staging.data_ptr(), host, h), "accept")
    torch.cuda.synchronize()
    for x, y in zip(acc[0][1], acc[1][1]):
        assert torch.equal(x, y)
    assert int(acc[0][1][1].min()) >= 0
    L = ctx + k + 1
    see = torch.ones((k + 1, L), dtype=torch.bool, device="cuda")
    see[:, ctx:] = torch.tril(see[:, ctx:])
    for i in (0, 1, 57, n - 1):
        K, V_ = kk[i * L:(i + 1) * L, 0].double(), vv[i * L:(i + 1) * L, 0].double()
        for hh in range(Hq):
            qq = q[i * (k + 1):(i + 1) * (k + 1), hh].double()
            s = (qq @ K.t().contiguous()) / d ** 0.5
            p = torch.softmax(s.masked_fill(~see, -float("inf")), -1)
            # scores off by (d + 4) 2^-24 sum|q k| / sqrt(d), as test_gpu_f32_attn.py derives
            ds = (qq.abs() @ K.abs().t().contiguous() / d ** 0.5).max(-1).values * (d + 4) * 2.0 ** -24
            bound = (2 * ds[:, None] + (L + 16) * 2.0 ** -24 + P_REL) * (p @ V_.abs())
            got = out[i * (k + 1):(i + 1) * (k + 1), hh].double()
            assert bool(((got - p @ V_).abs() <= bound).all()), (i, hh)


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up device pointers: only where nothing can be launched")
def test_noalloc_plans_coarser_before_it_refuses():
    """A step whose automatic split needs more than the static scratch, and
    whose longer pieces fit it, is not refused for its size."""
    n, k = 100, 9
    req = B.make_requests(np.full(n, 12000), np.full(n, k))
    a = B.SpecAttnArgs()
    a.num_q_heads, a.num_kv_heads, a.head_dim, a.dtype = 8, 1, 128, B.SPEC_BF16
    a.q = a.k = a.v = a.out = 1 << 20
    a.q_stride_tok, a.q_stride_head, a.kv_stride_tok, a.kv_stride_head = 1024, 128, 128, 128
    c = B.SpecAcceptArgs()
    c.vocab, c.dtype = 4000000, B.SPEC_F32
    c.target_logits = c.draft_probs = c.draft_tokens = c.uniforms = 1 << 20
    c.accepted_len = c.next_token = 1 << 20
    c.logits_stride = c.probs_stride = c.vocab
    st, dev, _ = B.spec_workspace_bytes(req, a, c)
    assert st == B.SPEC_OK and dev > B.SPEC_NOALLOC_SCRATCH_BYTES
    assert B.spec_verify_noalloc(req, a, c, 0) == B.SPEC_ERR_HIP        # past the size check, no device here
