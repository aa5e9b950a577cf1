"""End-to-end parity of atts_score_drafts with the oracle (K independent fp64 causal forwards)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import atts_oracle as O
from synth import WORKLOADS, ModelConfig, make_token_ids, make_weights
from util import announce, dev, dirty_ws, tight_ws, weights_to_numpy, ws

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-4, "bf16": 2e-2}      # absolute, per-token log-prob


def _run_gpu(A, cfg, w_dev, prefix, drafts, lens=None, mode=0, want_lp=True):
    model = A.Model(cfg, w_dev)
    K, T = drafts.shape
    lp = torch.full((K, T), float("nan"), dtype=torch.float32, device="cuda") if want_lp else None
    sc = torch.full((K,), float("nan"), dtype=torch.float32, device="cuda")
    wsp = ws(A.atts_workspace_bytes(model, len(prefix), K, T))
    A.atts_score_drafts(model, dev(prefix), dev(drafts), None if lens is None else dev(lens), mode, lp, sc, wsp)
    torch.cuda.synchronize()
    flag = A.atts_model_check(model)
    return (None if lp is None else lp.cpu().numpy()), sc.cpu().numpy(), flag


def _case(cfg, P, K, T, seed, n_layers=None):
    w_dev = make_weights(cfg, seed, device="cuda", n_layers=n_layers)
    prefix, drafts = make_token_ids(cfg.vocab, P, K, T, seed)
    return w_dev, prefix.numpy(), drafts.numpy()


def test_generator_is_identical_on_cpu_and_gpu():
    cfg = ModelConfig(1, 64, 4, 2, 16, 96, 300, "bf16")
    a, b = make_weights(cfg, 9, "cpu"), make_weights(cfg, 9, "cuda")
    for k in a:
        for x, y in zip(a[k] if isinstance(a[k], list) else [a[k]], b[k] if isinstance(b[k], list) else [b[k]]):
            assert torch.equal(x, y.cpu()), k


@pytest.mark.parametrize("mode", [O.MEAN_NLL, O.SUM_NLL])
def test_tiny_workload_fp32(mode):
    import paper_2509_15148_amd as A
    wl = WORKLOADS["tiny"]
    announce("score tiny fp32 mode", mode)
    w_dev, prefix, drafts = _case(wl.model, wl.P, wl.K, wl.T, wl.seed)
    lp, sc, flag = _run_gpu(A, wl.model, w_dev, prefix, drafts, mode=mode)
    ref_lp, ref_s = O.score_drafts(weights_to_numpy(w_dev), wl.model, prefix, drafts, mode=mode)
    assert flag == 0
    assert np.abs(lp - ref_lp).max() <= TOL["fp32"], np.abs(lp - ref_lp).max()
    assert np.allclose(sc, ref_s, rtol=0, atol=TOL["fp32"] * (wl.T if mode == O.SUM_NLL else 1))


@pytest.mark.parametrize("cfg,P,K,T", [
    (ModelConfig(2, 256, 4, 2, 128, 520, 2003, "bf16"), 70, 3, 45),     # MFMA attention, ragged everywhere
    (ModelConfig(3, 128, 8, 2, 16, 264, 777, "bf16"), 33, 5, 9),        # simple attention in bf16
    (ModelConfig(1, 72, 6, 6, 12, 40, 100, "fp32"), 1, 1, 1),           # smallest call
    (ModelConfig(2, 96, 4, 1, 24, 200, 515, "fp32"), 19, 4, 23),
])
def test_small_models_ragged_shapes(cfg, P, K, T):
    import paper_2509_15148_amd as A
    announce("score small", cfg, P, K, T)
    w_dev, prefix, drafts = _case(cfg, P, K, T, seed=P * 1000 + K)
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, drafts)
    ref_lp, ref_s = O.score_drafts(weights_to_numpy(w_dev), cfg, prefix, drafts)
    assert flag == 0
    assert np.abs(lp - ref_lp).max() <= TOL[cfg.dtype], np.abs(lp - ref_lp).max()
    assert np.abs(sc - ref_s).max() <= TOL[cfg.dtype]
    # scores only (token_logprobs = NULL) gives the same scores, bit for bit: calls with this few rows split the K range
    # of some projections over workgroups, whose partial sums are added in a fixed order
    _, sc2, _ = _run_gpu(A, cfg, w_dev, prefix, drafts, want_lp=False)
    assert np.array_equal(sc, sc2)


@pytest.mark.parametrize("P,K,T", [(2, 1, 128), (44, 2, 128), (45, 3, 115), (8, 4, 128), (6, 3, 257), (160, 4, 250), (100, 6, 250)])
def test_row_counts_between_tiles(P, K, T):
    """130 to 1600 rows of an aligned bf16 model, most of them ending in a partly filled tile of 128 or 256 rows, with the narrow
    projections cut along K and an LM head of 128 to 1500 scoring rows.  Repeated runs agree bit for bit."""
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, 1024, 8, 2, 128, 4096, 2304, "bf16")
    announce("score rows", P, K, T)
    w_dev, prefix, drafts = _case(cfg, P, K, T, seed=P * 1000 + K)
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, drafts)
    ref_lp, ref_s = O.score_drafts(weights_to_numpy(w_dev), cfg, prefix, drafts)
    assert flag == 0
    assert np.abs(lp - ref_lp).max() <= TOL["bf16"], np.abs(lp - ref_lp).max()
    assert np.abs(sc - ref_s).max() <= TOL["bf16"]
    _, sc2, _ = _run_gpu(A, cfg, w_dev, prefix, drafts, want_lp=False)
    assert np.array_equal(sc, sc2)


ALIGNED, EXCHANGED = 4, 5      # atts.h: ATTS_KERNEL_*


@pytest.mark.parametrize("cfg,P,K,T,rope", [
    (ModelConfig(3, 64, 3, 1, 4, 36, 100, "fp32"), 5, 2, 3, 1),     # heads of 4 columns, 20 of a tile's 32
    (ModelConfig(2, 100, 5, 1, 8, 44, 130, "fp32"), 33, 3, 10, 1),  # inner dimension of 100: the last step of K half filled
    (ModelConfig(2, 36, 3, 3, 16, 260, 70, "fp32"), 31, 1, 2, 1),   # 33 rows: one past a tile
    (ModelConfig(2, 128, 4, 2, 32, 512, 1024, "fp32"), 1, 1, 31, 1),    # 32 rows
    (ModelConfig(2, 132, 2, 1, 64, 72, 90, "fp32"), 17, 2, 9, 0),   # heads of two tiles: the rotation stays a pass of its own
    (ModelConfig(2, 60, 5, 5, 12, 40, 100, "fp32"), 9, 2, 7, 0),    # ... and heads that are no power of two
])
def test_small_fp32_models_norms_and_rotation_in_the_products(cfg, P, K, T, rope):
    """Norms inside the projections that read them and rotary embedding inside the QKV projection, at the edges of their tiles.
    Cold scoring, and through a prefix handle (rows that do not start at 0); residual stream scaled to rows of unlike size.  The routes
    say which passes ride along, and the launches of the stages bear it out."""
    import paper_2509_15148_amd as A
    L = cfg.n_layers
    for kind in (A.PASS_SCORE, A.PASS_SCORE_CACHED):
        r = A.atts_pass_routes(cfg, kind, P, K, T)
        assert (r.rope_in_qkv, r.norm_in_gate_up, r.qkv_fused) == (rope, 1, 0)
    announce("small fp32", cfg, P, K, T)
    w, prefix, drafts = _case(cfg, P, K, T, seed=7)
    scale = torch.logspace(-3, 3, cfg.vocab, device="cuda")[:, None]
    w["tok_embed"] = (w["tok_embed"] * scale).contiguous()
    ref, _ = O.score_drafts(weights_to_numpy(w), cfg, prefix, drafts)
    model = A.Model(cfg, w)
    lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    A.atts_profile_enable(True)
    A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, lp, sc, dirty_ws(A.atts_workspace_bytes(model, P, K, T)))
    launches = {n: A.atts_profile_read(A.STAGES.index(n))[1] for n in ("norm", "rope")}
    A.atts_profile_enable(False)
    assert launches == ({"norm": 0, "rope": 0} if rope else {"norm": L - 1, "rope": L})
    assert np.abs(lp.cpu().numpy() - ref).max() <= TOL["fp32"]
    pre = A.Prefix(model, P)
    A.atts_prefix_extend(pre, dev(prefix), dirty_ws(A.atts_prefix_extend_workspace_bytes(pre, P)))
    lp.fill_(float("nan"))
    A.atts_score_drafts_cached(pre, dev(drafts), None, 0, lp, sc, dirty_ws(A.atts_workspace_bytes(model, P, K, T)))
    assert np.abs(lp.cpu().numpy() - ref).max() <= TOL["fp32"]


@pytest.mark.parametrize("cfg,P,K,T,product,tile,tail", [
    (ModelConfig(1, 1024, 8, 2, 128, 12288, 768, "bf16"), 7, 24, 32, "gate_up", 256, 128),
    (ModelConfig(1, 768, 6, 2, 128, 16384, 768, "bf16"), 8, 50, 37, "gate_up", 384, 256),
    (ModelConfig(1, 8192, 6, 2, 128, 1024, 768, "bf16"), 8, 150, 32, "down", 384, 256),
])
def test_last_columns_in_a_second_launch(cfg, P, K, T, product, tile, tail):
    """Tall tiles over the first columns, lower ones over the last (SwiGLU, whose gate and up rows lie apart, and the residual
    update): a wrong column shows in every row.  Oracle: the first, a middle and the last draft."""
    import paper_2509_15148_amd as A
    announce("last columns", cfg, P, K, T)
    r = getattr(A.atts_pass_routes(cfg, A.PASS_SCORE, P, K, T), product)
    assert (r.kernel, r.tile_rows, r.head_rows, r.tail_rows) == (ALIGNED, tile, 0, tail)
    w, prefix, drafts = _case(cfg, P, K, T, seed=K)
    model = A.Model(cfg, w)
    lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, lp, sc, dirty_ws(A.atts_workspace_bytes(model, P, K, T)))
    lp, sc, w_np = lp.cpu().numpy(), sc.cpu().numpy(), weights_to_numpy(w)
    assert np.isfinite(lp).all() and np.isfinite(sc).all()
    for k in (0, K // 2, K - 1):
        ref = O.token_logprobs(w_np, cfg, prefix, drafts[k])
        assert np.abs(lp[k] - ref).max() <= TOL["bf16"], (k, np.abs(lp[k] - ref).max())


@pytest.mark.parametrize("cfg,P,K,T,expected", [
    # product -> (kernel, rows of a tile, cut along K, rows of a tile of the second launch)
    (ModelConfig(1, 768, 6, 2, 128, 16384, 768, "bf16"), 8, 96, 16, {"gate_up": (ALIGNED, 384, False, 128), "down": (ALIGNED, 128, True, 0)}),
    (ModelConfig(1, 1024, 8, 2, 128, 8192, 768, "bf16"), 8, 64, 32, {"gate_up": (ALIGNED, 384, False, 256), "down": (ALIGNED, 256, True, 0)}),
    (ModelConfig(1, 2048, 16, 4, 128, 8192, 768, "bf16"), 8, 32, 32, {"o": (ALIGNED, 256, True, 0), "gate_up": (ALIGNED, 384, False, 0)}),
    (ModelConfig(1, 2048, 16, 4, 128, 8192, 768, "bf16"), 8, 64, 40, {"down": (ALIGNED, 384, True, 0), "lm_head": (ALIGNED, 256, False, 0)}),
    (ModelConfig(1, 8192, 6, 2, 128, 1024, 768, "bf16"), 8, 64, 64, {"o": (ALIGNED, 384, False, 0), "down": (ALIGNED, 384, False, 256)}),
    (ModelConfig(1, 768, 6, 2, 128, 768, 65536, "bf16"), 8, 49, 16, {"lm_head": (ALIGNED, 384, False, 128)}),
    (ModelConfig(1, 1024, 8, 2, 128, 768, 44032, "bf16"), 8, 27, 19, {"lm_head": (ALIGNED, 384, False, 256)}),
    (ModelConfig(1, 768, 6, 2, 128, 768, 98304, "bf16"), 8, 13, 23, {"lm_head": (EXCHANGED, 384, False, 0)}),
])
def test_tile_heights_second_launches_and_orientations(cfg, P, K, T, expected):
    """Every tile height of every product, cut along K and not, the last rows in a second launch of 128- and 256-row tiles
    (SwiGLU, residual update and LM head, whose targets, partials and logits then start further on) and both orientations of the
    LM head.  Oracle: the first and the last draft and those on either side of where a second launch begins."""
    import paper_2509_15148_amd as A
    announce("score routes", cfg, P, K, T)
    routes = A.atts_pass_routes(cfg, A.PASS_SCORE, P, K, T)
    sampled = {0, K - 1}
    for name, want in expected.items():
        r = getattr(routes, name)
        assert (r.kernel, r.tile_rows, r.slices > 1, r.tail_rows) == want, (name, r.kernel, r.tile_rows, r.slices, r.tail_rows)
        if r.tail_rows:
            first = r.head_rows if name == "lm_head" else r.head_rows - P
            sampled |= {(first - 1) // T, first // T, min(first // T + 1, K - 1)}
    w, prefix, drafts = _case(cfg, P, K, T, seed=K)
    model = A.Model(cfg, w)
    lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, lp, sc, dirty_ws(A.atts_workspace_bytes(model, P, K, T)))
    lp, sc, w_np = lp.cpu().numpy(), sc.cpu().numpy(), weights_to_numpy(w)
    assert np.isfinite(lp).all() and np.isfinite(sc).all()
    for k in sorted(sampled):
        ref = O.token_logprobs(w_np, cfg, prefix, drafts[k])
        assert np.abs(lp[k] - ref).max() <= TOL["bf16"], (k, np.abs(lp[k] - ref).max())
        assert abs(sc[k] - O.conformity_score(ref)) <= TOL["bf16"], k


@pytest.mark.parametrize("cfg,P,K,T", [
    (ModelConfig(1, 2304, 4, 2, 16, 64, 50, "fp32"), 5, 2, 3),          # embedding rows longer than a thread block keeps in registers
    (ModelConfig(1, 4352, 4, 2, 16, 64, 50, "bf16"), 5, 2, 3),
    (ModelConfig(0, 264, 4, 2, 16, 64, 50, "bf16"), 9, 3, 4),           # no layer, no first norm
    (ModelConfig(2, 4352, 4, 2, 128, 1024, 768, "bf16"), 3, 2, 5),      # the same for the residual update that adds K slices:
    (ModelConfig(2, 4352, 4, 2, 128, 1024, 768, "bf16"), 10, 5, 12),    # 13, 70 and 610 rows
    (ModelConfig(2, 4352, 4, 2, 128, 1024, 768, "bf16"), 10, 5, 120),
])
def test_start_of_a_pass_row_lengths(cfg, P, K, T):
    import paper_2509_15148_amd as A
    announce("score start", cfg, P, K, T)
    w_dev, prefix, drafts = _case(cfg, P, K, T, seed=77)
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, drafts)
    ref_lp, ref_s = O.score_drafts(weights_to_numpy(w_dev), cfg, prefix, drafts)
    assert flag == 0
    assert np.abs(lp - ref_lp).max() <= TOL[cfg.dtype], np.abs(lp - ref_lp).max()
    assert np.abs(sc - ref_s).max() <= TOL[cfg.dtype]


@pytest.mark.parametrize("d", [1024, 4352])
def test_first_norm_has_the_bits_of_the_norm_kernel(d):
    """A first layer whose two output projections are zero hands the embeddings on unchanged, so the layer after it must
    see the norm (taken by the norm kernel there, with the embedding gather in a model without that layer) bit for bit."""
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, d, 8, 2, 128, 256, 768, "bf16")
    announce("score first norm", d)
    w, prefix, drafts = _case(cfg, 100, 6, 250, seed=5)
    longer = {k: (v + v if isinstance(v, list) else v) for k, v in w.items()}
    for name in ("wo", "w_down"):
        longer[name] = [torch.zeros_like(w[name][0]), w[name][0]]
    lp, sc, _ = _run_gpu(A, cfg, w, prefix, drafts)
    lp2, sc2, _ = _run_gpu(A, dataclasses.replace(cfg, n_layers=2), longer, prefix, drafts)
    assert np.array_equal(lp, lp2) and np.array_equal(sc, sc2)


def test_workspace_of_the_largest_call_serves_smaller_ones():
    """A loop allocates once for its longest drafts.  Shorter ones, whose projections are cut along K where the longest's are
    not, run in that workspace, and give the same bits as in one of their own size."""
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, 3584, 28, 4, 128, 18944, 2304, "bf16")
    w, prefix, drafts = _case(cfg, 512, 16, 256, seed=3)
    model = A.Model(cfg, w)
    largest = dirty_ws(A.atts_workspace_bytes(model, 512, 16, 256))
    pre = A.Prefix(model, capacity=512)
    A.atts_prefix_extend(pre, dev(prefix), largest)
    cut = set()
    for T in (256, 216, 200, 48, 8, 1):
        need = A.atts_workspace_bytes(model, 512, 16, T)
        assert need <= largest.numel()
        for kind in (A.PASS_SCORE, A.PASS_SCORE_CACHED):
            announce("score in the largest call's workspace", T, kind)
            route = A.atts_pass_routes(cfg, kind, 512, 16, T)
            assert need == route.workspace_bytes
            cut |= {(T, kind)} if route.down.slices > 1 else set()
            out = []
            for space in (largest, dirty_ws(need)):
                lp, sc = (torch.full(shape, float("nan"), device="cuda") for shape in ((16, T), (16,)))
                if kind == A.PASS_SCORE:
                    A.atts_score_drafts(model, dev(prefix), dev(drafts[:, :T]), None, 0, lp, sc, space)
                else:
                    A.atts_score_drafts_cached(pre, dev(drafts[:, :T]), None, 0, lp, sc, space)
                out.append((lp, sc))
                largest.fill_(255)
            assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
            assert bool(torch.isfinite(out[0][0]).all()) and bool(torch.isfinite(out[0][1]).all())
    assert (216, A.PASS_SCORE_CACHED) in cut and (48, A.PASS_SCORE) in cut and (256, A.PASS_SCORE) not in cut


@pytest.mark.parametrize("P,K,T", [(8, 8, 14), (9, 9, 12)])
def test_partial_sums_in_little_room(P, K, T):
    """Many heads over a narrow model: the buffers that hold the K slices of the output projection are small for it, so fewer
    slices are taken than the shape allows.  The oracle's bound; NaN in the workspace."""
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, 768, 128, 4, 128, 64, 768, "bf16")
    announce("score little room", P, K, T)
    few, many = (A.atts_pass_routes(c, A.PASS_SCORE, P, K, T).o.slices for c in (cfg, dataclasses.replace(cfg, d_ffn=16384)))
    assert 2 <= few < many
    w, prefix, drafts = _case(cfg, P, K, T, seed=P)
    model = A.Model(cfg, w)
    lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, lp, sc, dirty_ws(A.atts_workspace_bytes(model, P, K, T)))
    ref_lp, ref_s = O.score_drafts(weights_to_numpy(w), cfg, prefix, drafts)
    assert np.abs(lp.cpu().numpy() - ref_lp).max() <= TOL["bf16"] and np.abs(sc.cpu().numpy() - ref_s).max() <= TOL["bf16"]


@pytest.mark.parametrize("heads,P,K,T,tile", [((8, 2), 1, 1, 128, 128), ((8, 2), 100, 6, 250, 128), ((24, 8), 1, 8, 192, 256), ((24, 8), 1, 24, 128, 384),
                                              ((24, 8), 2, 24, 128, 384), ((24, 8), 6, 24, 128, 384), ((24, 8), 3, 30, 150, 384)])
def test_the_pass_reads_nothing_past_its_workspace(heads, P, K, T, tile):
    """The workspace ends where its allocation ends, its last buffer is the rotary table, and the last row of tiles of the fused
    QKV projection holds one to six rows, or some waves' worth: waves past the last row take the table's last row."""
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, 1024, *heads, 128, 256, 768, "bf16")
    announce("score tight workspace", heads, P, K, T, tile)
    route = A.atts_pass_routes(cfg, A.PASS_SCORE, P, K, T)
    assert route.qkv_fused and route.qkv.tile_rows == tile
    w, prefix, drafts = _case(cfg, P, K, T, seed=9)
    model = A.Model(cfg, w)
    need = A.atts_workspace_bytes(model, P, K, T)
    out = []
    for space in (tight_ws(need), ws(need + (8 << 20))):
        lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
        A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, lp, sc, space)
        torch.cuda.synchronize()
        out.append(lp)
    assert torch.equal(*out) and bool(torch.isfinite(out[0]).all())


def test_more_rows_than_one_launch_has_threads_for():
    """11.5 million rows, head_dim 256: a workgroup for each row and for 256 rotary pairs each would be 4.4e9 threads, and a
    launch has at most 2^32.  No layers, so that the scores follow from a table over pairs of tokens."""
    import paper_2509_15148_amd as A
    cfg = ModelConfig(0, 8, 1, 1, 256, 8, 16, "bf16")
    P, K, T = 3, 720000, 16
    announce("score many rows", P, K, T)
    w = make_weights(cfg, 5, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(7)
    ids = lambda *shape: torch.randint(0, cfg.vocab, shape, dtype=torch.int32, device="cuda", generator=g)
    prefix, drafts = ids(P), ids(K, T)
    model = A.Model(cfg, w)
    lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    A.atts_score_drafts(model, prefix, drafts, None, 0, lp, sc, ws(A.atts_workspace_bytes(model, P, K, T)))
    assert A.atts_model_check(model) == 0
    h = w["tok_embed"].double()
    x = h * torch.rsqrt((h * h).mean(dim=1, keepdim=True) + cfg.rms_eps) * w["final_norm"].double()
    table = torch.log_softmax(x @ w["lm_head"].double().t(), dim=1)
    before = torch.cat([prefix[-1:].expand(K, 1), drafts[:, :-1]], dim=1).long()
    ref = table[before, drafts.long()]
    assert float((lp - ref).abs().max()) <= TOL["bf16"] and float((sc + ref.mean(dim=1)).abs().max()) <= TOL["bf16"]


def test_variable_draft_lengths_and_padding_ids():
    import paper_2509_15148_amd as A
    cfg = ModelConfig(2, 256, 4, 2, 128, 512, 1000, "bf16")
    announce("score draft_lens")
    w_dev, prefix, drafts = _case(cfg, 40, 4, 30, seed=5)
    lens = np.array([30, 1, 17, 29], dtype=np.int32)
    padded = drafts.copy()
    for k in range(4):
        padded[k, lens[k]:] = -12345                      # garbage ids in the padding are ignored
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, padded, lens=lens)
    ref_lp, ref_s = O.score_drafts(weights_to_numpy(w_dev), cfg, prefix, drafts, draft_lens=lens)
    assert flag == 0
    assert np.abs(lp - ref_lp).max() <= TOL["bf16"]
    for k in range(4):
        assert np.all(lp[k, lens[k]:] == 0)
    assert np.abs(sc - ref_s).max() <= TOL["bf16"]


def test_out_of_range_token_id_sets_the_flag_and_does_not_fault():
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, 64, 4, 2, 16, 96, 50, "fp32")
    announce("score bad id")
    w_dev, prefix, drafts = _case(cfg, 6, 2, 4, seed=1)
    bad = drafts.copy()
    bad[1, 2] = 50
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, bad)
    assert flag == 1 and np.all(np.isfinite(lp))
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, drafts)
    assert flag == 0


def test_workspace_and_argument_errors():
    import paper_2509_15148_amd as A
    cfg = ModelConfig(1, 64, 4, 2, 16, 96, 50, "fp32")
    w_dev, prefix, drafts = _case(cfg, 6, 2, 4, seed=1)
    model = A.Model(cfg, w_dev)
    need = A.atts_workspace_bytes(model, 6, 2, 4)
    sc = torch.empty(2, device="cuda")
    with pytest.raises(A.AttsError) as e:
        A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, None, sc, ws(need)[: need - 256])
    assert e.value.code == A.ERR_WORKSPACE
    with pytest.raises(A.AttsError) as e:
        A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 5, None, sc, ws(need))
    assert e.value.code == A.ERR_INVALID_ARG
    with pytest.raises(A.AttsError) as e:
        A.atts_score_drafts(model, dev(prefix)[:0], dev(drafts), None, 0, None, sc, ws(need))
    assert e.value.code == A.ERR_INVALID_ARG


def _full_width_case(name, n_layers, k_sample, shape=None):
    """GPU: the whole workload (all K drafts) in the benchmark's launch configuration (or the same model at
    another (P, K, T)).  Oracle: the drafts in `k_sample` (an index, a list of indices or "all"), each alone as one
    plain causal sequence; every draft's first token against the prediction from the last prefix position."""
    import paper_2509_15148_amd as A
    wl = WORKLOADS[name]
    cfg = wl.model
    P, K, T = shape if shape else (wl.P, wl.K, wl.T)
    sample = list(range(K)) if k_sample == "all" else ([k_sample] if isinstance(k_sample, int) else list(k_sample))
    announce("score full width", name, "layers", n_layers, "shape", (P, K, T), "sample drafts", sample)
    w_dev, prefix, drafts = _case(cfg, P, K, T, wl.seed, n_layers=n_layers)
    lp, sc, flag = _run_gpu(A, cfg, w_dev, prefix, drafts)
    assert flag == 0 and np.all(np.isfinite(lp)) and np.all(lp <= 0)
    if shape is not None:      # run-to-run bit-stability, also where projections split their K range over workgroups
        lp2, sc2, _ = _run_gpu(A, cfg, w_dev, prefix, drafts)
        assert np.array_equal(lp, lp2) and np.array_equal(sc, sc2)
    w_np = weights_to_numpy(w_dev)
    del w_dev
    torch.cuda.empty_cache()
    worst = 0.0
    for k in sample:
        ref = O.token_logprobs(w_np, cfg, prefix, drafts[k])
        err = np.abs(lp[k] - ref).max()
        worst = max(worst, float(err))
        assert err <= TOL["bf16"], (k, err)
        assert abs(sc[k] - O.conformity_score(ref)) <= TOL["bf16"], k
    print(f"[score full width {name} L={n_layers} {(P, K, T)}] max |dlogp| over drafts {sample} = {worst:.3e}", flush=True)
    # all drafts share the prediction of their first token from the last prefix position
    first = O.log_softmax(O.logits_from_hidden(w_np, cfg, O.decoder_hidden(w_np, cfg, prefix)[-1:]))[0]
    assert np.abs(lp[:, 0] - first[drafts[:, 0]]).max() <= TOL["bf16"]


@pytest.mark.timeout(900)
def test_7b_shape_two_layer_slice():
    """The benchmark's launch configuration at 7B width, two layers: EVERY one of the 16 drafts element by element."""
    _full_width_case("7b", n_layers=2, k_sample="all")


@pytest.mark.parametrize("shape", [(16, 16, 8), (300, 5, 67), (1, 2, 3), (700, 3, 100)])
def test_7b_width_few_and_ragged_rows(shape):
    """Row counts that are not whole 256-row tiles, at full model width: the decode-like shape that bench.py
    times (144 rows: projections with few tiles split their K range over several workgroups), a ragged
    multi-tile one, a handful of rows, and 1000 rows (four tile rows, still few enough tiles to split K).  All drafts
    are compared, and a second run must reproduce the first bit for bit."""
    _full_width_case("7b", n_layers=2, k_sample="all", shape=shape)


@pytest.mark.timeout(900)
def test_7b_full_model_sampled_draft():
    """The 7B-class workload exactly as bench.py runs it (28 layers, K = 16 drafts of 256 tokens after a
    512-token prefix); the oracle scores one sampled draft as a plain causal sequence (~1 minute of CPU)."""
    _full_width_case("7b", n_layers=None, k_sample=11)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name", ["32b", "70b"])
def test_large_models_two_layer_slice(name):
    """Full width, full row count (34,816 / 9,216 rows: 64-bit offsets in the FFN activation), two layers (the
    residual epilogue -> norm -> next layer hand-off at these widths); the oracle scores the first and the last
    draft (the last one ends in the last, ragged row tile)."""
    K = WORKLOADS[name].K
    _full_width_case(name, n_layers=2, k_sample=(3, K - 1))
