"""The LM head's tile shapes at their edges: rows around each tile height (the
low tiles' 16-row blocks, 96 / 97 and 192 / 193 rows, 64-row steps of the tall
tiles, several row tiles; every build, which test_plan_rules.py checks),
vocabularies around the 128- and 256-entry tiles, hidden widths of a partial,
one, two and three slices and of more than the rings hold, rotated starts, padded row strides, fp32 and bf16 logits.  Logits against fp64 within
the bound of fp32 accumulation of exact bf16 products (K 2^-23 sum |h w|, plus
half a bf16 ulp, 2^-8 |x|, where stored in bf16); tokens against spec_accept on
the stored logits (the sampled values are fixed by the seed, away from ties)."""
import numpy as np
import pytest
import torch

from paper_2505_17074_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [  # rows, vocabulary, hidden width, bf16 logits
    (1, 129, 32, False), (3, 1, 96, False), (16, 127, 64, True), (17, 128, 128, False), (33, 4097, 160, True),
    (64, 300, 192, False), (65, 33000, 96, False), (80, 33024, 512, True), (96, 32900, 64, False),
    (97, 32900, 96, True), (128, 33001, 192, False), (161, 32800, 320, False), (192, 32769, 32, True),
    (193, 1000, 64, False), (256, 257, 192, True), (257, 5000, 96, False), (320, 32900, 128, False),
    (385, 32000, 64, True), (449, 32000, 32, False), (716, 32100, 320, False), (960, 32000, 96, True),
    # low tiles of 65 to 192 rows (weights too long for the cache), 21 and 21.5 slices
    (66, 32700, 1344, False), (80, 32700, 1344, True), (96, 32640, 1376, False), (97, 32700, 1344, True),
    (130, 32700, 1344, False), (161, 32700, 1376, True), (192, 32640, 1344, False),
    # tall tiles of 64, 128 and 192 rows over more slices than their rings hold
    # (7 and 8, also 6.5 and 7.5; 5 would start every tile at slice 0)
    (100, 1000, 512, False), (70, 5000, 480, True), (193, 32000, 448, False), (256, 32000, 416, True),
    (240, 32000, 448, True), (257, 32000, 416, False), (320, 32000, 448, True), (384, 32000, 448, False),
]


def _run(fn, req, acc, size, *args):
    st, dev, host = size
    B.check(st, "workspace size")
    ws = torch.empty(dev + 256, dtype=torch.uint8, device="cuda")
    staging = torch.empty(max(host, 1), dtype=torch.uint8, pin_memory=True)
    B.check(fn(req, *args, acc, (ws.data_ptr() + 255) // 256 * 256, dev, staging.data_ptr(), host,
               torch.cuda.current_stream().cuda_stream), "call")
    torch.cuda.synchronize()


@pytest.mark.parametrize("M,V,K,bf16", CASES)
def test_tiles(gpu_lib, M, V, K, bf16):
    print(f"[lm tiles] M {M} V {V} K {K} bf16 {bf16}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 31 + V)
    dt = torch.bfloat16 if bf16 else torch.float32
    # rows of K values inside wider rows whose padding is NaN: never read
    hid = torch.full((M, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    wgt = torch.full((V, K + 16), float("nan"), dtype=torch.bfloat16, device="cuda")
    hid[:, :K] = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    wgt[:, :K] = (torch.randn((V, K), generator=g, device="cuda") * 2 / K ** 0.5).bfloat16()
    Vp = -(-V // 8) * 8
    logits = torch.full((M, Vp), float("nan"), dtype=dt, device="cuda")
    k = min(7, M - 1)
    chain = [k] * (M // (k + 1)) + ([M % (k + 1) - 1] if M % (k + 1) else [])
    req = B.make_requests(np.zeros(len(chain)), np.array(chain))
    nd = max(sum(chain), 1)
    probs = torch.zeros((nd, Vp), dtype=dt, device="cuda")
    probs[:, :V] = torch.softmax(2 * torch.randn((nd, V), generator=g, device="cuda"), -1).to(dt)
    tokens = torch.multinomial(probs[:, :V].float(), 1, generator=g)[:, 0].int()
    uni = torch.rand(M, generator=g, device="cuda") * 0.999
    outs = []
    for _ in range(2):
        o = [torch.full((len(chain),), -5, dtype=torch.int32, device="cuda") for _ in range(3)]
        a = B.SpecAcceptArgs()
        a.vocab, a.dtype = V, B.SPEC_BF16 if bf16 else B.SPEC_F32
        a.target_logits, a.logits_stride, a.draft_probs, a.probs_stride = logits.data_ptr(), Vp, probs.data_ptr(), Vp
        a.draft_tokens, a.uniforms = tokens.data_ptr(), uni.data_ptr()
        a.accepted_len, a.next_token, a.accepted_node = (x.data_ptr() for x in o)
        outs.append((a, o))
    lm = B.SpecLmHeadArgs()
    lm.hidden_dim, lm.hidden, lm.hidden_stride = K, hid.data_ptr(), K + 8
    lm.weight, lm.weight_stride = wgt.data_ptr(), K + 16
    (a, fused), (a2, plain) = outs
    _run(B.spec_lm_head_accept, req, a, B.spec_lm_head_workspace_bytes(req, lm, a), lm)
    h, w = hid[:, :K].double(), wgt[:, :K].double().t().contiguous()
    ref, bound = torch.mm(h, w), torch.mm(h.abs(), w.abs()) * K * 2.0 ** -23
    if bf16:
        bound = bound + 2.0 ** -8 * ref.abs()
    err = (logits[:, :V].double() - ref).abs()
    assert bool((err <= bound).all()), float((err / bound.clamp_min(1e-30)).max())
    if Vp > V:
        assert bool(torch.isnan(logits[:, V:]).all())     # nothing written past the vocabulary
    _run(B.spec_accept, req, a2, B.spec_workspace_bytes(req, None, a2))
    for x, y in zip(fused, plain):
        assert torch.equal(x, y)
