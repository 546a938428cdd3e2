"""Values at the ends of the types' ranges: masks made of the lowest finite
value over whole chunks and tiles, scores that overflow to minus infinity,
infinities in V.  Attention against fp64 within the bounds of the finite tests,
acceptance and the LM head's decision against the acceptance oracle."""
import numpy as np
import pytest

import parity_util as U
from oracle import verify_accept
from paper_2505_17074_amd import binding as B
from paper_2505_17074_amd import workload as W
from paper_2505_17074_amd.batch import DeviceBatch, LmHeadVerifier, Verifier, pad_vocab_rows
from test_gpu_f32_attn import reference_and_bound
from test_gpu_small_batch import P_REL

pytestmark = pytest.mark.gpu

ATTN = [  # dtype, head dim, query heads, split_kv
    (W.F32, 64, 4, 0), (W.F32, 128, 4, 96), (W.BF16, 64, 4, 64), (W.BF16, 128, 4, 0), (W.BF16, 128, 16, 160),
]


@pytest.mark.parametrize("dtype,d,Hq,split", ATTN)
@pytest.mark.parametrize("mask", [-1e36, -2e38], ids=["finite", "overflow"])
def test_attention_of_masked_keys(gpu_lib, dtype, d, Hq, split, mask):
    """Positive queries; the first 700 of 1000 cached keys (whole tiles and, in
    a cut stream, whole pieces) hold the mask in every element, so their scores
    are about -1e37 or overflow to minus infinity and their weights are 0.  The
    reference is the attention over the other keys alone."""
    print(f"[extreme] {dtype} d {d} heads {Hq} split {split} mask {mask}", flush=True)
    pool = U.custom_pool(ctx=[1000, 701, 40], k=[4, 2, 3], Hq=Hq, Hkv=2, d=d, qkv=dtype, seed=d + Hq)
    pool.q = W.storage(np.abs(W.as_f32(pool.q, dtype)) + 0.25, dtype)
    low = W.storage(np.full(1, mask, np.float32), dtype)[0]
    keep = []                            # the keys of the reference's shorter contexts
    for i, c in enumerate((1000, 701, 40)):
        kv0, n_masked = int(pool.kv_start[i]), min(700, c - 1)
        pool.k[kv0:kv0 + n_masked] = low
        keep.append(np.arange(kv0 + n_masked, kv0 + c + int(pool.n_q[i])))
    short = U.custom_pool(ctx=[300, 1, 1], k=[4, 2, 3], Hq=Hq, Hkv=2, d=d, qkv=dtype)
    keep = np.concatenate(keep)
    short.q, short.k, short.v = pool.q, pool.k[keep], pool.v[keep]
    # P_REL: the roundings of bf16 probabilities
    ref, bound = reference_and_bound(short, 0.0 if dtype == W.F32 else P_REL)
    v = Verifier(DeviceBatch(pool, "cuda"), split_kv=split)
    v.batch.out.fill_(float("nan"))
    v.run("attn")
    out = v.results()["out"].astype(np.float64)
    # + 16 u of the weights' sum: the masked keys' zero terms enter running sums of 700 more
    bound = bound + 716 * 2.0 ** -24 * np.abs(W.as_f32(pool.v, dtype)).max()
    assert np.isfinite(out).all() and (np.abs(out - ref) <= bound).all(), float((np.abs(out - ref) / bound).max())


@pytest.mark.parametrize("dtype,d,split", [(W.F32, 64, 0), (W.F32, 128, 96), (W.BF16, 128, 0), (W.BF16, 64, 64)])
def test_attention_of_an_infinite_value(gpu_lib, dtype, d, split):
    """One infinity in V at a cached position: its column of its KV head's
    query heads is infinite in every row, every other element is as without.
    bf16 probabilities are carried in two parts, the second of either sign or
    zero, so there the column is infinite or NaN."""
    print(f"[extreme] infinite V {dtype} d {d} split {split}", flush=True)
    pool = U.custom_pool(ctx=[500, 90], k=[4, 6], Hq=4, Hkv=2, d=d, qkv=dtype, seed=d)
    b = DeviceBatch(pool, "cuda")
    v = Verifier(b, split_kv=split)
    v.run("attn")
    plain = v.results()["out"]
    b.v[int(pool.kv_start[1]) + 37, 1, 5] = float("inf")
    v.run("attn")
    out = v.results()["out"]
    hit = np.zeros(out.shape, bool)
    hit[int(pool.q_start[1]):, 2:, 5] = True
    assert (np.isposinf(out[hit]) if dtype == W.F32 else ~np.isfinite(out[hit])).all()
    assert np.array_equal(out[~hit], plain[~hit])


@pytest.mark.parametrize("logit", [W.F32, W.BF16])
@pytest.mark.parametrize("V,kw,rule", [
    (20000, dict(k=[4, 0, 8]), "independent"), (20000, dict(tree_parent=[-1, 0, 0, 1, 1, 2]), "independent"),
    (20000, dict(tree_parent=[-1, 0, 0, 1, 1, 2]), "sequential"), (140000, dict(tree_parent=[-1, 0, 0, 0]), "independent"),
    (140000, dict(tree_parent=[-1, 0, 0, 0]), "sequential"),
], ids=["chain", "tree", "tree_seq", "tree35chunks", "tree35chunks_seq"])
def test_acceptance_with_lowest_value_masks(gpu_lib, V, kw, rule, logit):
    """The first two chunks of 4096 entries, and the last ones, masked by the
    logit type's lowest finite value, in every row."""
    print(f"[extreme] accept V {V} {logit} {rule} {kw}", flush=True)
    pool = U.custom_pool(ctx=[1] * 3, Hq=1, Hkv=1, d=64, V=V, logit=logit, sigma=0.5, seed=7, **kw)
    lowest = np.float32(np.finfo(np.float32).min) if logit == W.F32 else np.uint16(0xFF7F)
    pool.target_logits[:, :8192] = lowest
    pool.target_logits[:, 16384:] = lowest
    b = DeviceBatch(pool, "cuda")
    pad_vocab_rows(b)
    v = Verifier(b)
    if rule == "sequential":
        v.acc.tree_rule = B.SPEC_TREE_SEQUENTIAL
    v.run("accept")
    got = v.results()
    ref = verify_accept(pool.target_logits, pool.draft_probs, pool.draft_tokens, pool.uniforms, pool.n_q,
                        dtype=logit, tree_parent=pool.tree_parent, tree_rule=rule)
    bad, ties = U.compare_accept(got, ref, pool)
    assert not bad and ties <= 1, (bad, ties)
    assert all(8192 <= int(t) < 16384 for t in got["next_token"])


@pytest.mark.parametrize("name,batch", [("mha7b_b32", 3), ("ragged_gqa_b128", 16), ("ragged_gqa_b128", 128)])
def test_lm_head_with_masked_entries(gpu_lib, name, batch):
    """Whole 128- and 256-entry tiles of the vocabulary masked through one
    weight column times a constant hidden feature (logits of about -3e38, near
    the lowest finite value), at low and tall tiles."""
    V = 3000
    print(f"[extreme] LM head {name} batch {batch}", flush=True)
    pool = W.make_lm_head_pool(W.CONFIG_BY_NAME[name], 1, batch=batch, hidden_dim=256, vocab=V)
    pool.hidden[:, 3] = W.storage(np.ones(1, np.float32), W.BF16)[0]
    pool.weight[:, 3] = 0
    masked = np.r_[0:512, 1024:1300, 2816:V]
    pool.weight[masked, 3] = W.storage(np.full(1, -3e38, np.float32), W.BF16)[0]
    lmv = LmHeadVerifier(pool, "cuda")
    lmv.batch.logits.fill_(float("nan"))
    lmv.run()
    fused, logits = lmv.results(), lmv.logits()
    x = W.as_f32(logits, pool.logit_dtype)
    free = np.setdiff1d(np.arange(V), masked)
    assert np.isfinite(x).all() and (x[:, masked] < -1e38).all() and (np.abs(x[:, free]) < 1e3).all()
    ref = verify_accept(logits, pool.draft_probs, pool.draft_tokens, pool.uniforms, pool.n_q,
                        dtype=pool.logit_dtype, tree_parent=pool.tree_parent)
    bad, ties = U.compare_accept(fused, ref, pool)
    assert not bad and ties <= U.max_near_ties(batch), (bad, ties)
    assert np.isin(fused["next_token"], free).all()
