"""The decision's folds over vocabulary chunks at their edges (one, 16 / 17, 32
/ 33 and 64 / 65 chunks of 4096 entries: lanes per row, held statistics, chunk
masses per pass) and at 1, 16, 17 and 32 verify positions, chains and trees,
against the acceptance oracle: bit-exact except counted near ties."""
import pytest

import parity_util as U
from oracle import verify_accept
from paper_2505_17074_amd import binding as B
from paper_2505_17074_amd import workload as W
from paper_2505_17074_amd.batch import DeviceBatch, Verifier, pad_vocab_rows

pytestmark = pytest.mark.gpu
K = [0, 1, 15, 16, 4, 2]
CASES = [
    (4096, W.F32, dict(k=K)), (4097, W.BF16, dict(k=K)), (65536, W.F32, dict(k=[3, 0, 5])),
    (65537, W.F32, dict(k=[3, 0, 5])), (131073, W.BF16, dict(k=[4, 0, 8])), (262144, W.F32, dict(k=[3, 0])),
    (262145, W.F32, dict(k=[3, 0, 2])), (300000, W.BF16, dict(k=[2, 0, 4])),
    (9000, W.F32, dict(tree_parent=W.full_binary_tree_parents(2, 5).tolist() + [15])),
    (9000, W.F32, dict(tree_parents=[[-1] + [0] * 16, [-1] + list(range(31)), [-1], [-1, 0, 0, 2, 2, 1]])),
]


@pytest.mark.parametrize("V,logit,kw", CASES)
def test_chunk_folds(gpu_lib, V, logit, kw):
    print(f"[chunks] V {V} {logit} {kw}", flush=True)
    n = len(kw["tree_parents"]) if "tree_parents" in kw else len(kw["k"]) if "k" in kw else 3
    for sigma in (0.2, 2.0):          # mostly accepted, mostly rejected
        pool = U.custom_pool(ctx=[1] * n, Hq=1, Hkv=1, d=64, V=V, logit=logit, sigma=sigma, seed=V % 97, **kw)
        b = DeviceBatch(pool, "cuda")
        pad_vocab_rows(b)
        v = Verifier(b)
        v.run("accept")
        ref = verify_accept(pool.target_logits, pool.draft_probs, pool.draft_tokens, pool.uniforms, pool.n_q,
                            dtype=logit, tree_parent=pool.tree_parent, tree_parents=pool.tree_parents)
        bad, ties = U.compare_accept(v.results(), ref, pool)
        assert not bad and ties <= 1, (bad, ties)


@pytest.mark.parametrize("V,logit,parents", [(65537, W.F32, [-1, 0, 0, 1, 1]), (131073, W.BF16, [-1, 0, 0, 0]),
                                             (6000, W.F32, W.full_binary_tree_parents(2, 5).tolist() + [15])])
def test_sequential_chunk_folds(gpu_lib, V, logit, parents):
    """The sequential walk's folds: 17 and 33 chunks, 32 verify positions."""
    print(f"[chunks] sequential V {V} {logit} {len(parents)} nodes", flush=True)
    pool = U.custom_pool(ctx=[1] * 3, Hq=1, Hkv=1, d=64, V=V, logit=logit, sigma=2.0, seed=V % 97, tree_parent=parents)
    b = DeviceBatch(pool, "cuda")
    pad_vocab_rows(b)
    v = Verifier(b)
    v.acc.tree_rule = B.SPEC_TREE_SEQUENTIAL
    v.run("accept")
    ref = verify_accept(pool.target_logits, pool.draft_probs, pool.draft_tokens, pool.uniforms, pool.n_q,
                        dtype=logit, tree_parent=pool.tree_parent, tree_rule="sequential")
    bad, ties = U.compare_accept(v.results(), ref, pool)
    assert not bad and ties <= 1, (bad, ties)
