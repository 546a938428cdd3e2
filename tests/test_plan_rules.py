"""The attention planner's choices, read off spec_workspace_bytes on a host
without a GPU (the rules then assume 256 compute units): a plan that cuts no
stream needs no partial rows, one that cuts every stream in n pieces at least
n partial rows of d + 2 floats per query row and head."""
import numpy as np
import pytest

from paper_2505_17074_amd import binding as B


def sizes(ctx, k, hq, hkv, d, dtype=B.SPEC_BF16, split=0):
    """(device bytes, bytes of one partial row per query row and head)."""
    ctx = np.asarray(ctx)
    req = B.make_requests(ctx, np.full(len(ctx), k))
    a = B.SpecAttnArgs()
    a.num_q_heads, a.num_kv_heads, a.head_dim, a.dtype, a.split_kv = hq, hkv, d, dtype, split
    a.q = a.k = a.v = a.out = 1 << 20
    a.q_stride_tok, a.q_stride_head, a.kv_stride_tok, a.kv_stride_head = hq * d, d, hkv * d, d
    st, dev, _ = B.spec_workspace_bytes(req, a, None)
    B.check(st, "spec_workspace_bytes")
    return dev, len(ctx) * (k + 1) * hq * (d + 2) * 4


# requests, keys, k, query heads, KV heads, d; measured whole and cut in us
WHOLE = [
    (16, 261, 7, 64, 8, 128),      # 64 rows: 15.6 whole, 22.9 in two pieces
    (16, 409, 8, 64, 8, 128),      # 72 rows: 19.6, 26.3
    (16, 600, 7, 64, 8, 64),       # d = 64: 17.1, 20.5
    (16, 300, 4, 32, 8, 64),       # 20 rows: 11.8, 16.8
    (32, 1000, 8, 64, 8, 128),     # 256 streams: 36.7, 45.4
    (60, 1000, 8, 64, 8, 128),     # 480 streams, few of which have a free slot: 49, 57
    (1, 200, 4, 32, 8, 128),       # one request: 13.9, 14.3
]
CUT = [
    (1, 1000, 4, 32, 8, 128, 8),   # 34.1 whole, 16.2 in eight pieces
    (16, 4000, 7, 64, 8, 128, 2),  # 101, 66
    (32, 4000, 4, 32, 8, 64, 2),
    (1, 64000, 4, 8, 1, 128, 40),  # one stream: 43 us in 63 pieces, 37 in 125
]


@pytest.mark.parametrize("n,keys,k,hq,hkv,d", WHOLE)
def test_short_streams_run_whole(n, keys, k, hq, hkv, d):
    dev, row = sizes([keys - k - 1] * n, k, hq, hkv, d)
    assert dev < row                                  # the plan's tables alone


@pytest.mark.parametrize("n,keys,k,hq,hkv,d,pieces", CUT)
def test_long_streams_are_cut(n, keys, k, hq, hkv, d, pieces):
    dev, row = sizes([keys - k - 1] * n, k, hq, hkv, d)
    assert dev >= pieces * row


# the line the GPU tests of short pieces run on both sides of (test_gpu_small_batch.py)
EDGES = [
    ([233, 3], 4, 4, 128, B.SPEC_BF16, False),
    ([234, 3], 4, 4, 128, B.SPEC_BF16, True),
    ([146], 2, 2, 64, B.SPEC_F32, False),
    ([147], 2, 2, 64, B.SPEC_F32, True),
]


@pytest.mark.parametrize("ctx,hq,hkv,d,dtype,cut", EDGES)
def test_shortest_cut(ctx, hq, hkv, d, dtype, cut):
    dev, _ = sizes(ctx, 4, hq, hkv, d, dtype)
    one = 5 * hq * (d + 2) * 4                        # a partial row of the first request's rows and heads
    assert (dev >= 2 * one) == cut


def test_one_stream_is_not_cut_into_more_pieces_than_pay():
    """64000 keys on one KV head: 125 pieces 37 us, 500 (as many as there are
    slots) 66, since the combine walks a row's pieces in turn."""
    dev, row = sizes([64000 - 5], 4, 8, 1, 128)
    assert dev < 256 * row


# requests, keys, k, query heads, KV heads, d; fused combine by default (its
# arrival counters take workspace)
FUSED = [
    (24, 1500, 4, 8, 8, 128, True),     # 192 streams, two pieces, 5 rows: 37.2 us fused, 39.0 separate
    (24, 1500, 4, 32, 8, 128, True),    # 20 rows, two pieces
    (32, 2000, 4, 32, 8, 128, True),    # 256 streams, two pieces
    (16, 2000, 4, 32, 8, 128, False),   # 128 streams
    (1, 350, 7, 64, 8, 128, False),     # 8 streams in two pieces: 19.1 us fused, 16.5 separate
    (1, 1000, 4, 32, 8, 128, False),
]


@pytest.mark.parametrize("n,keys,k,hq,hkv,d,fused", FUSED)
def test_combine_inside_the_split_kernel(monkeypatch, n, keys, k, hq, hkv, d, fused):
    args = ([keys - k - 1] * n, k, hq, hkv, d)
    monkeypatch.delenv("SPEC_FUSED_COMBINE_MAX_BYTES", raising=False)
    dev, row = sizes(*args)
    assert dev >= 2 * row
    monkeypatch.setenv("SPEC_FUSED_COMBINE_MAX_BYTES", "0")
    assert (dev > sizes(*args)[0]) == fused


# (requests, longest context) whose sizes a caller allocated, those it is then
# used for, query heads, KV heads, d, type: shapes whose first batch is now cut
# less or by other rows than the second one's longer pieces assume
KEPT = [
    (16, 15080, 32, 384, 32, 32, 64, B.SPEC_F32),
    (16, 24482, 8, 26762, 32, 32, 128, B.SPEC_F32),
    (32, 32438, 128, 163, 64, 8, 128, B.SPEC_F32),
    (64, 26852, 128, 129, 32, 8, 128, B.SPEC_F32),
    (8, 3516, 4, 1171, 32, 32, 128, B.SPEC_BF16),
    (64, 23812, 64, 8799, 16, 4, 64, B.SPEC_BF16),
    (2, 18799, 32, 2103, 32, 8, 128, B.SPEC_BF16),
]


def batch_args(n, ctx, hq, hkv, d, dtype):
    req = B.make_requests(np.linspace(max(1, ctx // 16), ctx, n).astype(np.int32), np.full(n, 4))
    a = B.SpecAttnArgs()
    a.num_q_heads, a.num_kv_heads, a.head_dim, a.dtype = hq, hkv, d, dtype
    a.q = a.k = a.v = a.out = 1 << 20
    a.q_stride_tok, a.q_stride_head, a.kv_stride_tok, a.kv_stride_head = hq * d, d, hkv * d, d
    return req, a


def longer_pieces_bytes(n, ctx, hq, hkv, d, dtype):
    """Device and staging bytes of the plan of few, long pieces: 512 slots,
    pieces of max(40 rows, 256) keys (3584 where there are as many streams as
    slots), the widest item 80 rows (fp32: 4096 / d).  One k for all requests."""
    req, _ = batch_args(n, ctx, hq, hkv, d, dtype)
    L, nq, G = [int(req.ctx_len[i]) + 5 for i in range(n)], 5, hq // hkv
    ng = -(-G // max(1, (80 if dtype == B.SPEC_BF16 else 4096 // d) // nq))
    hpg = -(-G // ng)
    mult, rows = hkv * -(-G // hpg), hpg * nq
    pieces = [1] * n
    if mult * n >= 512:
        pieces = [-(-x // 3584) for x in L]
    else:
        lo, total = -(-max(40 * rows, 256) // 32) * 32, mult * n
        while True:
            i = max(range(n), key=lambda j: (-(-L[j] // pieces[j]), j))
            if (L[i] + pieces[i]) // (pieces[i] + 1) < lo or total + mult > 512:
                break
            pieces[i] += 1
            total += mult
    up = lambda x: -(-x // 256) * 256
    length = [-(-(-(-x // p)) // 32) * 32 for x, p in zip(L, pieces)]
    pieces = [-(-x // y) for x, y in zip(L, length)]
    items = sum(pieces) * mult
    part = sum(p for p in pieces if p > 1) * nq * hq
    tables = up(32 * n) + up(4 * nq * n) + up(64 * items)
    return tables + up(part * d * 4) + up(part * 8), tables


@pytest.mark.parametrize("na,ca,nb,cb,hq,hkv,d,dtype", KEPT)
def test_a_kept_workspace_is_not_refused(na, ca, nb, cb, hq, hkv, d, dtype):
    """The sizes cover the plan of long pieces for the same batch, and a call
    takes any workspace that holds its own: no device here, so it then fails
    later (SPEC_ERR_HIP), not for its size."""
    import torch
    req, a = batch_args(na, ca, hq, hkv, d, dtype)
    st, dev, host = B.spec_workspace_bytes(req, a, None)
    B.check(st, "spec_workspace_bytes")
    need = longer_pieces_bytes(na, ca, hq, hkv, d, dtype)
    assert dev >= need[0] and host >= need[1]
    if torch.cuda.is_available():
        return                           # made-up device pointers: only where nothing can be launched
    need = longer_pieces_bytes(nb, cb, hq, hkv, d, dtype)
    extra = 16384                        # arrival counters (8 bytes a stream) and the claim word
    if dev < need[0] + extra or host < need[1]:
        return
    req, a = batch_args(nb, cb, hq, hkv, d, dtype)
    staging = np.zeros(host + 256, np.uint8)
    assert B.spec_verify_attn(req, a, 1 << 20, dev, (staging.ctypes.data + 255) // 256 * 256, host, 0) == B.SPEC_ERR_HIP


# ---- the LM head's tiles (sv_rules.h compiled by itself) ----------------------
@pytest.fixture(scope="module")
def geometry(tmp_path_factory):
    import ctypes as C
    import os
    import subprocess
    src = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_17074_amd", "csrc")
    d = tmp_path_factory.mktemp("rules")
    (d / "g.cpp").write_text('#include "sv_rules.h"\nextern "C" void geo(int M, int V, int K, int cus, int* o) {\n'
                             '  const auto g = sv::lmh_geometry(M, V, K, cus);\n  o[0] = g.rb; o[1] = g.low_wr;'
                             ' o[2] = g.tile_rows; o[3] = g.m_tiles; o[4] = g.nt;\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", src, str(d / "g.cpp"),
                    "-o", str(d / "g.so")], check=True)
    lib = C.CDLL(str(d / "g.so"))

    def geo(M, V, K, cus=256):
        o = (C.c_int * 5)()
        lib.geo(M, V, K, cus, o)
        return tuple(o)
    return geo


# rows, vocabulary, hidden width, low tiles; measured low / tall (weights from
# HBM or, where a third of the cache holds them, from there)
TILES = [
    (20, 32000, 4096, True),      # 0.75
    (72, 128256, 8192, True),     # 0.93 at 80 rows
    (95, 50304, 1024, False),     # 57 / 42 us
    (190, 50304, 4096, False),    # 147 / 126
    (68, 111175, 5120, False),    # 280 / 247
    (95, 128256, 2048, False),    # 161 / 142
    (20, 50304, 4096, True),
    (190, 78071, 4096, True),     # 0.96
    (190, 32000, 8192, True),     # 0.89
    (95, 32000, 1024, False),     # 39 / 33, cached
    (95, 32000, 2048, True),      # 54 / 59
    (125, 16000, 8192, True),     # 0.80
    (125, 16000, 4096, False),    # 1.08, cached
    (190, 16000, 4096, False),    # 85 / 80
]


@pytest.mark.parametrize("M,V,K,low", TILES)
def test_lm_head_tiles(geometry, M, V, K, low):
    assert (geometry(M, V, K)[1] > 0) == low


def test_lm_head_tiles_cover_the_rows(geometry):
    """Every shape gets a build that exists and tiles that hold its rows."""
    rng = np.random.default_rng(3)
    for _ in range(20000):
        M, V, K = int(2 ** rng.uniform(0, 14)), int(2 ** rng.uniform(0, 20)), 32 * int(rng.integers(1, 512))
        rb, wr, rows, mt, nt = geometry(M, V, K, int(rng.choice([1, 64, 256, 304])))
        assert mt >= 1 and mt == -(-M // rows) and 4096 % nt == 0
        if wr:
            assert nt == 128 and mt == 1 and M <= 16 * rb * wr
            assert (wr == 1 and 1 <= rb <= 6) or (wr == 2 and 4 <= rb <= 6)
        else:
            assert nt == 256 and 1 <= rb <= 6 and rows <= 64 * rb


def test_lm_tile_cases_launch_every_build(geometry):
    """The GPU test's cases select every build of both kernels, and each tall
    one over more slices than its ring holds as well."""
    import test_gpu_lm_tiles as T
    got = {(g[1], g[0]) for g in (geometry(M, V, K) for M, V, K, _ in T.CASES)}
    assert got == {(1, rb) for rb in range(1, 7)} | {(2, rb) for rb in range(4, 7)} | {(0, rb) for rb in range(1, 7)}
    long = {g[0] for g in (geometry(M, V, K) for M, V, K, _ in T.CASES if K > 4 * 64) if g[1] == 0}
    assert {1, 2, 3} <= long
