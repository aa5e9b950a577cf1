"""Stage-level parity: the MFMA GEMM, the fused LM-head log-softmax-gather and the shared-prefix
attention, each against a plain float64 statement of the same operation."""
import math

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from oracle import atts_oracle as O
from synth import hash_uniform, stream_id
from util import announce, dev, ws

pytestmark = pytest.mark.gpu


def _rand(shape, seed, dtype, scale=1.0):
    n = int(np.prod(shape))
    return (hash_uniform(stream_id(seed, 1), n) * scale).view(*shape).to(dtype)


# ------------------------------------------------------------------------------------ GEMM
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", [(1, 1, 8), (33, 70, 72), (300, 200, 136), (257, 513, 1000), (128, 128, 64),
                                   (3584, 3600, 264),
                                   # aligned bf16 shapes with more 384-row tiles than compute units: workgroups walk two or
                                   # three tiles each, some one fewer than others (680 and 700 tiles)
                                   (1536, 43520, 768), (768, 89600, 832),
                                   # at most 16 rows: the weight-streaming kernel (bf16), ragged columns and k-step counts
                                   (1, 1, 32), (4, 100, 96), (7, 4608, 256), (16, 33, 2080), (16, 530, 3584), (3, 48, 18944)])
def test_gemm_nt_matches_float64_matmul(dtype, shape):
    import paper_2509_15148_amd as A
    M, N, Kd = shape
    announce("gemm", dtype, shape)
    a, w = _rand((M, Kd), 11, dtype), _rand((N, Kd), 12, dtype)
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_gemm_nt(a.cuda(), w.cuda(), c)
    torch.cuda.synchronize()
    ref = a.double().numpy() @ w.double().numpy().T
    assert np.allclose(c.cpu().numpy(), ref, rtol=1e-5, atol=2e-5 * math.sqrt(Kd))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", [
    (31, 33, 8), (32, 32, 16), (33, 65, 24), (64, 96, 40), (20, 31, 136),      # edges of 32 x 32 tiles; K from one step to ragged quarters
    (1024, 768, 72), (1024, 769, 72),                                          # bf16: 768 small tiles, and one column of tiles more
    (1024, 2048, 72), (1024, 2049, 72),                                        # fp32: 2048 small tiles, and more: 128 x 128 tiles
    (1024, 1920, 264), (1024, 1921, 264),                                      # fp32, longer sums: 1920
    (130, 33000, 40), (17, 66000, 24)])                                        # two and three rounds of 128 x 128 tiles
def test_gemm_small_products(dtype, shape):
    """Shapes at the edges of the kernel for products of few tiles and of the rule that chooses it, against the float64
    product.  Bound: a sum of K products rounds at most K times to 2^-24 of its absolute sum (here a few per cent of that)."""
    import paper_2509_15148_amd as A
    M, N, Kd = shape
    announce("gemm small", dtype, shape)
    a, w = _rand((M, Kd), 51, dtype), _rand((N, Kd), 52, dtype)
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_gemm_nt(a.cuda(), w.cuda(), c)
    torch.cuda.synchronize()
    ref = a.double().numpy() @ w.double().numpy().T
    bound = Kd * 2.0 ** -24 * (np.abs(a.double().numpy()) @ np.abs(w.double().numpy()).T) + 1e-30
    assert (np.abs(c.cpu().numpy() - ref) <= bound).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", [(1, 8, 1), (32, 40, 64), (33, 24, 65), (70, 72, 6145), (300, 72, 9001)])
def test_lmhead_small_products(dtype, shape):
    """The LM head where its product has few tiles: row and vocabulary counts at the edges of 32 x 64 tiles, and a
    vocabulary that takes larger tiles.  The logits are sums of K products (error at most K 2^-24 of their absolute sum)
    and the log-sum-exp adds a few roundings of values below 2^4."""
    import paper_2509_15148_amd as A
    B, d, V = shape
    announce("lmhead small", dtype, shape)
    x, w = _rand((B, d), 61, dtype, scale=2.0), _rand((V, d), 62, dtype, scale=4.0 / math.sqrt(d))
    tgt = torch.from_numpy(np.random.default_rng(4).integers(0, V, B).astype(np.int32))
    tgt[0], tgt[-1] = V - 1, 0
    lp = torch.full((B,), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_lmhead_logprobs(x.cuda(), w.cuda(), tgt.cuda(), lp, ws(A.atts_lmhead_workspace_bytes(B, V)))
    lp2 = torch.full((B,), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_lmhead_logprobs_static(x.cuda(), w.cuda(), tgt.cuda(), lp2)
    torch.cuda.synchronize()
    ref = torch.log_softmax(x.double() @ w.double().t(), dim=-1).gather(1, tgt.long()[:, None])[:, 0].numpy()
    most = float((x.double().abs() @ w.double().abs().t()).max())
    assert (np.abs(lp.cpu().numpy() - ref) <= 2 * d * 2.0 ** -24 * most + 32 * 2.0 ** -20).all()
    assert torch.equal(lp, lp2)


@pytest.mark.parametrize("V", [2304, 6144])
@pytest.mark.parametrize("B", [1, 7, 8, 9, 127, 128, 129, 255, 257, 300, 519])
def test_lmhead_exchanged_takes_any_number_of_rows(B, V):
    """Vocabulary entries as tile rows, scoring rows as columns read in place: one to 128 rows (128-column tiles) and more
    (256-column tiles), the last column tile filled by one, seven and eight rows and all but one.  The scoring rows end
    where their allocation does.  The smaller vocabulary goes to small tiles from 129 to 320 rows.  Bound as in
    test_lmhead_small_products."""
    import paper_2509_15148_amd as A
    d = 832
    announce("lmhead exchanged rows", B, V)
    _, route = A.atts_gemm_routes(torch.bfloat16, B, V, d)
    if V == 2304 and 128 < B <= 320:
        assert route.kernel == A.KERNEL_SMALL
    else:
        assert (route.kernel, route.tile_rows) == (A.KERNEL_EXCHANGED, 256 if B <= 128 else 384)
    x, w = _rand((B, d), 71, torch.bfloat16, scale=2.0), _rand((V, d), 72, torch.bfloat16, scale=4.0 / math.sqrt(d))
    tgt = torch.from_numpy(np.random.default_rng(5).integers(0, V, B).astype(np.int32))
    tgt[0], tgt[-1] = 0, V - 1
    lp = torch.full((B + 8,), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_lmhead_logprobs(x.cuda(), w.cuda(), tgt.cuda(), lp[:B], ws(A.atts_lmhead_workspace_bytes(B, V)))
    lp2 = torch.full((B,), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_lmhead_logprobs_static(x.cuda(), w.cuda(), tgt.cuda(), lp2)
    torch.cuda.synchronize()
    ref = torch.log_softmax(x.double() @ w.double().t(), dim=-1).gather(1, tgt.long()[:, None])[:, 0].numpy()
    most = float((x.double().abs() @ w.double().abs().t()).max())
    assert (np.abs(lp[:B].cpu().numpy() - ref) <= 2 * d * 2.0 ** -24 * most + 32 * 2.0 ** -20).all()
    assert torch.equal(lp[:B], lp2) and torch.isnan(lp[B:]).all()


@pytest.mark.parametrize("shape,tail", [((4608, 11008, 768), 128), ((2304, 14592, 1024), 256)])
def test_gemm_aligned_last_tile_rows_in_a_second_launch(shape, tail):
    """12 x 43 tiles of 384 x 256 = 516 = two rounds of 256 and four tiles over: the aligned bf16 path gives the last tile row to
    a launch of its own with 128-row tiles; 6 x 57 = 342: the last two to one with 256-row tiles.  Every element against
    the float64 product."""
    import paper_2509_15148_amd as A
    M, N, Kd = shape
    route, _ = A.atts_gemm_routes(torch.bfloat16, M, N, Kd)
    assert (route.kernel, route.tile_rows, route.tail_rows) == (A.KERNEL_ALIGNED, 384, tail) and 0 < route.head_rows < M
    announce("gemm tail launch", (M, N, Kd))
    a, w = _rand((M, Kd), 21, torch.bfloat16), _rand((N, Kd), 22, torch.bfloat16)
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_gemm_nt(a.cuda(), w.cuda(), c)
    torch.cuda.synchronize()
    ref = a.double().numpy() @ w.double().numpy().T
    assert np.allclose(c.cpu().numpy(), ref, rtol=1e-5, atol=2e-5 * math.sqrt(Kd))


@pytest.mark.parametrize("shape,tile,tail,seam", [((1280, 14336, 832), 256, 128, 51 * 256), ((3072, 12544, 832), 384, 256, 32 * 256)])
def test_gemm_aligned_last_columns_in_a_second_launch(shape, tile, tail, seam):
    """Tall tiles over the first columns, lower ones over the last.  Every element against the float64 product."""
    import paper_2509_15148_amd as A
    M, N, Kd = shape
    route, _ = A.atts_gemm_routes(torch.bfloat16, M, N, Kd)
    assert (route.kernel, route.tile_rows, route.head_rows, route.tail_rows, route.head_cols) == (A.KERNEL_ALIGNED, tile, 0, tail, seam)
    announce("gemm last columns", shape)
    a, w = _rand((M, Kd), 31, torch.bfloat16), _rand((N, Kd), 32, torch.bfloat16)
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_gemm_nt(a.cuda(), w.cuda(), c)
    torch.cuda.synchronize()
    ref = a.double().numpy() @ w.double().numpy().T
    assert np.allclose(c.cpu().numpy(), ref, rtol=1e-5, atol=2e-5 * math.sqrt(Kd))


def test_gemm_aligned_shapes_sweep():
    """Seeded sweep over shapes the aligned bf16 kernel takes (rows a multiple of 256, columns of 256, inner
    dimension of 64 from 768 up): tile counts below and above the number of compute units, partly filled last rounds of
    the tile walk, all tile heights, second launches.  Every element against the float64 product."""
    import paper_2509_15148_amd as A
    rng, heights = np.random.default_rng(15148), set()
    for case in range(12):
        M = int(rng.choice([256, 512, 768, 1024, 1280, 1536, 2304, 3072, 3840]))
        N = 256 * int(rng.integers(1, 90))
        Kd = 64 * int(rng.choice([12, 13, 16, 24, 31]))
        announce("gemm aligned", case, (M, N, Kd))
        route, _ = A.atts_gemm_routes(torch.bfloat16, M, N, Kd)
        assert route.kernel == A.KERNEL_ALIGNED
        heights |= {route.tile_rows, -route.tail_rows}
        a, w = _rand((M, Kd), 300 + case, torch.bfloat16), _rand((N, Kd), 400 + case, torch.bfloat16)
        c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        A.atts_gemm_nt(a.cuda(), w.cuda(), c)
        torch.cuda.synchronize()
        ref = a.double().numpy() @ w.double().numpy().T
        assert np.allclose(c.cpu().numpy(), ref, rtol=1e-5, atol=2e-5 * math.sqrt(Kd)), (M, N, Kd)
    assert heights == {128, 256, 384, 0, -128, -256}


def test_gemm_few_rows_random_shapes():
    """Seeded sweep over the shapes the weight-streaming kernel serves (1..16 rows, any column count, inner
    dimension a multiple of 32 up to several K slices), against the float64 product."""
    import paper_2509_15148_amd as A
    rng = np.random.default_rng(2509)
    for case in range(24):
        M = int(rng.integers(1, 17))
        N = int(rng.choice([1, 15, 16, 17, 31, 32, 33, 100, 255, 256, 1000, 3584, 4608]))
        Kd = 32 * int(rng.choice([1, 2, 3, 7, 8, 9, 16, 17, 63, 112, 129]))
        announce("gemm few rows", case, (M, N, Kd))
        a, w = _rand((M, Kd), 100 + case, torch.bfloat16), _rand((N, Kd), 200 + case, torch.bfloat16)
        c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        A.atts_gemm_nt(a.cuda(), w.cuda(), c)
        torch.cuda.synchronize()
        ref = a.double().numpy() @ w.double().numpy().T
        assert np.allclose(c.cpu().numpy(), ref, rtol=1e-5, atol=2e-5 * math.sqrt(Kd)), (M, N, Kd)


def test_gemm_rejects_unaligned_k():
    import paper_2509_15148_amd as A
    a = torch.zeros(4, 12, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(A.AttsError) as e:
        A.atts_gemm_nt(a, a, torch.zeros(4, 4, device="cuda"))
    assert e.value.code == A.ERR_SHAPE


# ------------------------------------------------------------------------------------ LM head
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-4), (torch.bfloat16, 1e-3)])
@pytest.mark.parametrize("shape", [(1, 16, 7), (37, 128, 1000), (256, 128, 1024), (130, 264, 5003), (4096, 256, 19008),
                                   # scoring rows a multiple of 256, vocabulary of 384, inner dimension of 64 from 768 up: the
                                   # bf16 product is taken with the operands exchanged (vocabulary entries as rows); 300 and 30
                                   # tiles, the second with a single column of tiles
                                   (1280, 768, 23040), (256, 1344, 11520)])
def test_lmhead_logprobs_matches_log_softmax_gather(dtype, tol, shape):
    """lp = z[target] - logsumexp(z) without materialising z; logits scaled to a spread of several
    units so that the running-max logic matters."""
    import paper_2509_15148_amd as A
    B, d, V = shape
    announce("lmhead", dtype, shape)
    x = _rand((B, d), 21, dtype, scale=2.0)
    w = _rand((V, d), 22, dtype, scale=4.0 / math.sqrt(d))
    tgt = torch.from_numpy(np.random.default_rng(3).integers(0, V, B).astype(np.int32))
    tgt[0], tgt[-1] = V - 1, 0
    lp = torch.full((B,), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_lmhead_logprobs(x.cuda(), w.cuda(), tgt.cuda(), lp, ws(A.atts_lmhead_workspace_bytes(B, V)))
    torch.cuda.synchronize()
    z = x.double().numpy() @ w.double().numpy().T
    ref = O.log_softmax(z)[np.arange(B), tgt.numpy()]
    got = lp.cpu().numpy()
    assert np.abs(got - ref).max() <= tol, np.abs(got - ref).max()
    assert np.all(got <= 1e-6)


@pytest.mark.parametrize("B,d,V,tail", [(129, 3584, 384 * 396, 256), (256, 3584, 384 * 396, 256), (385, 768, 384 * 396, 128),
                                        (513, 768, 384 * 262, 128), (1025, 768, 384 * 64, 128)])
def test_lmhead_with_a_second_launch(B, d, V, tail):
    """The vocabulary's last entries in smaller tiles (ragged and whole column tiles of scoring rows); targets on both sides of the
    seam, at both ends and inside.  bf16 products summed in fp32, the reference in float64: 1e-3 as above."""
    import paper_2509_15148_amd as A
    announce("lmhead, second launch", B, d, V, tail)
    _, route = A.atts_gemm_routes(torch.bfloat16, B, V, d)
    assert route.kernel == A.KERNEL_EXCHANGED and route.tail_rows == tail
    g = torch.Generator(device="cuda").manual_seed(B)
    x = (torch.randn(B, d, device="cuda", generator=g) * 2).to(torch.bfloat16)
    w = (torch.randn(V, d, device="cuda", generator=g) * (2 / math.sqrt(d))).to(torch.bfloat16)
    tgt = torch.randint(0, V, (B,), dtype=torch.int32, device="cuda", generator=g)
    seam = route.head_rows
    tgt[:6] = torch.tensor([0, V - 1, seam - 1, seam, seam + tail - 1, min(seam + tail, V - 1)])
    tgt[-1] = seam
    lp = torch.full((B,), float("nan"), dtype=torch.float32, device="cuda")
    A.atts_lmhead_logprobs(x, w, tgt, lp, ws(A.atts_lmhead_workspace_bytes(B, V)))
    torch.cuda.synchronize()
    z = x.double() @ w.double().t()
    ref = torch.log_softmax(z, dim=1).gather(1, tgt[:, None].long())[:, 0]
    assert (lp.double() - ref).abs().max().item() <= 1e-3


# ------------------------------------------------------------------------------------ attention
def _tree_attention_reference(qkv, P, K, T, nq, nkv, hd):
    """K independent causal sequences [prefix ; draft k] through torch's float64 SDPA."""
    R = P + K * T
    q, k, v = qkv.double().split([nq * hd, nkv * hd, nkv * hd], -1)
    out = torch.zeros(R, nq * hd, dtype=torch.float64)

    def run(rows):
        n = len(rows)
        o = F.scaled_dot_product_attention(q[rows].view(n, nq, hd).transpose(0, 1)[None],
                                           k[rows].view(n, nkv, hd).transpose(0, 1)[None],
                                           v[rows].view(n, nkv, hd).transpose(0, 1)[None],
                                           is_causal=True, enable_gqa=True)
        return o[0].transpose(0, 1).reshape(n, nq * hd)

    pre = torch.arange(P)
    out[:P] = run(pre)
    for kk in range(K):
        rows = torch.cat([pre, P + kk * T + torch.arange(T)])
        out[P + kk * T: P + (kk + 1) * T] = run(rows)[P:]
    return out.numpy()


@pytest.mark.parametrize("dtype,shape,tol", [
    (torch.float32, (64, 8, 32, 4, 4, 32), 2e-5),          # the tiny workload's shape
    (torch.float32, (5, 3, 7, 6, 2, 16), 2e-5),
    (torch.bfloat16, (9, 2, 5, 4, 2, 64), 1.5e-2),         # simple kernel in bf16
    (torch.bfloat16, (70, 3, 45, 4, 2, 128), 1.5e-2),      # MFMA kernel, nothing aligned
    (torch.bfloat16, (1, 4, 1, 2, 1, 128), 1.5e-2),
    (torch.bfloat16, (130, 5, 17, 8, 8, 128), 1.5e-2),     # several drafts inside one query tile
    (torch.bfloat16, (512, 4, 256, 7, 1, 128), 1.5e-2),    # aligned, GQA group 7
    (torch.bfloat16, (200, 0, 1, 2, 2, 128), 1.5e-2),      # prefix only
    (torch.bfloat16, (512, 16, 256, 28, 4, 128), 1.5e-2),  # the 7B step's launch: 256-row query tiles, 504 workgroups
    (torch.bfloat16, (200, 21, 200, 16, 2, 128), 1.5e-2),  # the same kernel (288 workgroups), drafts and prefix not aligned to its tiles
])
def test_shared_prefix_attention(dtype, shape, tol):
    _attention_case(dtype, shape, tol)


# Bounds of the general kernel: fp32 as above (probabilities and sums round to 2^-24 of values below 3); bf16 outputs round to
# 2^-9 of values below 3.
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-5), (torch.bfloat16, 1.5e-2)])
@pytest.mark.parametrize("hd", [8, 16, 24, 40, 64, 72, 136, 256])
@pytest.mark.parametrize("offset", [0, 1])
def test_general_attention_head_sizes(dtype, tol, hd, offset):
    """Head sizes below, at and above a wavefront's lanes (several keys per pass, one, several passes), key counts around
    whole groups of keys, and a buffer that does not start at a multiple of 16 bytes."""
    _attention_case(dtype, (21, 3, 14, 4, 2, hd), tol, offset)


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-5), (torch.bfloat16, 1.5e-2)])
@pytest.mark.parametrize("hd", [8, 16, 32, 64, 80, 256])
@pytest.mark.parametrize("P,K,T", [(1, 2, 9), (131, 2, 77), (64, 1, 200)])
def test_general_attention_key_counts(dtype, tol, hd, P, K, T):
    """Whole batches of eight keys a group and every remainder, in the prefix and in the draft, for one to eight groups."""
    _attention_case(dtype, (P, K, T, 2, 1, hd), tol)


@pytest.mark.parametrize("P,K,T,nq,nkv", [
    (1, 1, 1, 1, 1), (5, 1, 26, 2, 1), (5, 1, 27, 2, 1), (5, 1, 28, 2, 2),            # 7 rows below .. above one query tile of 32
    (224, 1, 32, 3, 1), (225, 2, 16, 3, 1), (250, 3, 8, 4, 4),                         # eight key tiles, one more, drafts inside a tile
    (480, 1, 32, 16, 2), (480, 1, 33, 16, 2),                                           # 256 workgroups, and one row more (128-row tiles)
    (1500, 1, 36, 8, 1), (1400, 3, 100, 9, 3),                                          # 384 and 486 workgroups with a long context
    (1400, 3, 100, 10, 5),                                                              # 540: too many
])
def test_attention_with_few_query_rows(P, K, T, nq, nkv):
    """Edges of the kernel for few query rows (keys divided among the wavefronts) and of the rule that takes it."""
    _attention_case(torch.bfloat16, (P, K, T, nq, nkv, 128), 1.5e-2)


# (query heads, rows): 3 and 10 workgroups of 32 rows with the keys divided; 128 rows a workgroup; 256 rows a workgroup
DOMINANT_SHAPES = [(1, 96), (1, 300), (32, 300), (8, 1100), (64, 1100)]


def _uniform_queries(nq, rows, key_values, v):
    """qkv for one key head: every query element 4, key j's elements key_values[j] (scores 45.25 times that), values v."""
    hd = v.shape[1]
    qkv = torch.zeros(rows, (nq + 2) * hd, dtype=torch.bfloat16)
    qkv[:, :nq * hd] = 4.0
    for j, x in key_values.items():
        qkv[j, nq * hd:(nq + 1) * hd] = x
    qkv[:, (nq + 1) * hd:] = v
    return qkv.cuda()


def _run_attention(qkv, nq, rows):
    import paper_2509_15148_amd as A
    out = torch.empty(rows, nq * 128, dtype=torch.bfloat16, device="cuda")
    A.atts_attention_shared_prefix(qkv, out, rows - 40, 1, 40, nq, 1, 128, ws(A.atts_attention_workspace_bytes(torch.bfloat16, rows, 1, 128)))
    torch.cuda.synchronize()
    return out.cpu().double().view(rows, nq, 128)


@pytest.mark.parametrize("nq,rows", DOMINANT_SHAPES)
@pytest.mark.parametrize("key", [3, 8, 21, 30, 47, 61])
def test_mfma_attention_one_dominant_key(nq, rows, key):
    """One key whose score stands 181 above all others (exp of the difference overflows fp32): every later row must return its
    value alone, whichever lane of the score tile holds it, and the rows before it the mean of theirs."""
    announce("attention, dominant key", nq, rows, key)
    v = torch.randn(rows, 128, generator=torch.Generator().manual_seed(key)).to(torch.bfloat16)
    got = _run_attention(_uniform_queries(nq, rows, {key: 4.0}, v), nq, rows)
    want = v.double().cumsum(0) / torch.arange(1, rows + 1)[:, None]
    want[key:] = v[key].double()
    assert (got - want[:, None]).abs().max().item() <= 1.5e-2


@pytest.mark.parametrize("nq,rows", DOMINANT_SHAPES)
@pytest.mark.parametrize("key", [5, 12, 70, 78])          # lower and upper half of the lanes, first and second tile
@pytest.mark.parametrize("x", [0.09375, 0.6640625, 0.97265625, 0.984375, 1.109375])
def test_mfma_attention_reference_left_behind(nq, rows, key, x):
    """One key 4.2 (2^6.1), 30, 44.0 (2^63.5), 44.5 (2^64.3) and 50 above all others: where the softmax reference just stays
    and just moves, for either half of the lanes.  Against the weighted mean in float64: the probabilities and the output are
    rounded to bf16, 2^-8 of a value each."""
    announce("attention, reference", nq, rows, key, x)
    v = torch.randn(rows, 128, generator=torch.Generator().manual_seed(key)).to(torch.bfloat16)
    got = _run_attention(_uniform_queries(nq, rows, {key: x}, v), nq, rows)
    w = torch.ones(rows, dtype=torch.float64)
    w[key] = math.exp(128 * 4 * x / math.sqrt(128))
    want = (w[:, None] * v.double()).cumsum(0) / w.cumsum(0)[:, None]
    assert (got - want[:, None]).abs().max().item() <= 2.0 ** -7 * v.double().abs().max().item()


@pytest.mark.parametrize("nq,rows", DOMINANT_SHAPES)
def test_mfma_attention_probabilities_stay_bounded(nq, rows):
    """Values of 2^60 with a key of the lower lanes 2^5.9 and one of the upper lanes 2^69 above the keys of the tile before.  With
    probabilities of at most 2^64 the sums are finite (2^124).  Tolerance as above."""
    announce("attention, bounded", nq, rows)
    v = torch.randn(rows, 128, generator=torch.Generator().manual_seed(nq)).clamp(-2, 2).to(torch.bfloat16)
    x = {66: 0.09033203125, 75: 1.0546875}                 # scores 4.088 (2^5.9) and 47.73 (2^68.9)
    got = _run_attention(_uniform_queries(nq, rows, x, v * 2.0 ** 60), nq, rows) / 2.0 ** 60
    w = torch.ones(rows, dtype=torch.float64)
    for j, c in x.items():
        w[j] = math.exp(128 * 4 * c / math.sqrt(128))
    want = (w[:, None] * v.double()).cumsum(0) / w.cumsum(0)[:, None]
    assert (got - want[:, None]).abs().max().item() <= 2.0 ** -7 * v.double().abs().max().item()


def _attention_case(dtype, shape, tol, offset=0):
    import paper_2509_15148_amd as A
    P, K, T, nq, nkv, hd = shape
    announce("attention", dtype, shape)
    R = P + K * T
    qkv = _rand((R, (nq + 2 * nkv) * hd), 31, dtype, scale=1.5)
    out = torch.full((R, nq * hd), float("nan"), dtype=dtype, device="cuda")
    wsb = A.atts_attention_workspace_bytes(dtype, R, nkv, hd)
    room = torch.empty(qkv.numel() + offset, dtype=dtype, device="cuda")
    room[offset:].copy_(qkv.flatten())
    A.atts_attention_shared_prefix(room[offset:].view(qkv.shape), out, P, K, T, nq, nkv, hd, ws(wsb) if wsb else None)
    torch.cuda.synchronize()
    ref = _tree_attention_reference(qkv, P, K, T, nq, nkv, hd)
    err = np.abs(out.float().cpu().numpy() - ref).max()
    assert err <= tol, err
