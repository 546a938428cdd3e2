"""fp32 verify attention (fp32 matrix cores) against fp64, within a derived
bound, at the kernel's edges: one to four waves per work-group (16, 17, 33 and
64 rows), both head dims (32- and 16-key tiles), contexts around the tile and
piece edges, chains, a shared tree and per-request trees, forced splits, and a
key/value layout with padded strides."""
import numpy as np
import pytest
import torch

from paper_2505_17074_amd import workload as W
from paper_2505_17074_amd.batch import DeviceBatch, Verifier
import parity_util as U

pytestmark = pytest.mark.gpu

UNIT = 2.0 ** -24      # fp32 unit roundoff
CASES = [
    ("one_wave_d64", dict(ctx=[0, 1, 31, 32, 33, 500], k=[0, 4, 16, 3, 15, 4], Hq=4, Hkv=4, d=64), 0),
    ("two_waves_d64", dict(ctx=[63, 64, 65, 700], k=[16, 8, 2, 16], Hq=2, Hkv=2, d=64), 64),
    ("three_waves_d64", dict(ctx=[30, 257], k=[10, 10], Hq=6, Hkv=2, d=64), 96),
    ("four_waves_d64", dict(ctx=[900, 15], k=[15, 7], Hq=8, Hkv=2, d=64), 0),
    ("groups_d64", dict(ctx=[100, 40], k=[16, 1], Hq=8, Hkv=1, d=64), 32),
    ("one_wave_d128", dict(ctx=[0, 15, 16, 17, 1300], k=[1, 4, 15, 3, 8], Hq=2, Hkv=2, d=128), 0),
    ("two_waves_d128", dict(ctx=[47, 48, 49], k=[16, 3, 8], Hq=4, Hkv=2, d=128), 32),
    ("four_waves_d128", dict(ctx=[600, 3], k=[15, 8], Hq=8, Hkv=2, d=128), 160),
    ("tree_d64", dict(ctx=[50, 0, 95], tree_parent=[-1, 0, 0, 1, 1, 2, 5, 5], Hq=4, Hkv=2, d=64), 0),
    ("trees_d128", dict(ctx=[20, 64], tree_parents=[[-1, 0, 0, 0, 2], [-1] + list(range(31))], Hq=4, Hkv=2, d=128), 0),
]


def reference_and_bound(pool, p_rel=0.0):
    """fp64 output and, per row, a first-order bound of an fp32 evaluation:
    scores off by (d + 4) u scale sum|q k|, the exponentials by twice that
    (numerator and denominator) plus their own and the running sums' roundings,
    (L + 16) u of sum p |v|, plus p_rel of it (a rounding of p itself)."""
    def t(x):
        return torch.from_numpy(W.as_f32(x, pool.qkv_dtype).astype(np.float64))
    Hq, Hkv, d = pool.num_q_heads, pool.num_kv_heads, pool.head_dim
    q, k, v = t(pool.q), t(pool.k), t(pool.v)
    ref, bound = torch.empty(q.shape, dtype=torch.float64), torch.empty(q.shape, dtype=torch.float64)
    for i in range(pool.batch):
        n, c = int(pool.n_q[i]), int(pool.ctx_len[i])
        par = pool.parents_of(i)
        par = W.chain_parents(n) if par is None else par
        see = torch.eye(n, dtype=torch.bool)
        for j in range(1, n):
            see[j] |= see[int(par[j])]
        see = torch.cat([torch.ones((n, c), dtype=torch.bool), see], 1)
        q0, kv0 = int(pool.q_start[i]), int(pool.kv_start[i])
        for h in range(Hq):
            qq, kk, vv = q[q0:q0 + n, h], k[kv0:kv0 + c + n, h // (Hq // Hkv)], v[kv0:kv0 + c + n, h // (Hq // Hkv)]
            s = (qq @ kk.T) / d ** 0.5
            ds = ((qq.abs() @ kk.abs().T) / d ** 0.5 * (d + 4) * UNIT).masked_fill(~see, 0).max(-1).values
            p = torch.softmax(s.masked_fill(~see, -np.inf), -1)
            ref[q0:q0 + n, h] = p @ vv
            bound[q0:q0 + n, h] = (2 * ds[:, None] + (c + n + 16) * UNIT + p_rel) * (p @ vv.abs())
    return ref.numpy(), bound.numpy()


@pytest.mark.parametrize("name,kw,split", CASES, ids=[c[0] for c in CASES])
def test_f32_attention(gpu_lib, name, kw, split):
    print(f"[f32] {name}", flush=True)
    pool = U.custom_pool(**kw, qkv=W.F32, seed=U.case_seed(name))
    b = DeviceBatch(pool, "cuda")
    ref, bound = reference_and_bound(pool)
    for pad in (0, 4):
        v = Verifier(b, split_kv=split)
        if pad:                      # token rows and heads with gaps between them
            hs = pool.head_dim + pad
            ts = pool.num_kv_heads * hs + pad
            wide = []
            for src in (b.k, b.v):
                w = torch.full((src.shape[0], ts), float("nan"), device="cuda")
                w.as_strided(src.shape, (ts, hs, 1)).copy_(src)
                wide.append(w)
            v.attn.k, v.attn.v = wide[0].data_ptr(), wide[1].data_ptr()
            v.attn.kv_stride_tok, v.attn.kv_stride_head = ts, hs
        b.out.fill_(float("nan"))
        v.run("attn")
        out = v.results()["out"].astype(np.float64)
        assert (np.abs(out - ref) <= bound).all(), float((np.abs(out - ref) / bound).max())
