"""Projections of a few rows with weights streamed by about a tile a compute unit (SwiGLU up to 128 rows, narrow ones up to 64), inside a one-layer pass against the
oracle.  The down projection picks single features, one of every block of 16 in turn, so that each block reaches the logits by itself."""
import numpy as np
import pytest
import torch

import paper_2509_15148_amd as A
from oracle import atts_oracle as O
from synth import ModelConfig, make_token_ids, make_weights
from util import announce, dev, dirty_ws, weights_to_numpy

D = 768


@pytest.mark.parametrize("d_ffn,streamed", [(8192, False), (8320, True), (12288, True), (12416, True), (18944, True), (22016, True), (27648, True),
                                            (28672, False)])
def test_route_of_a_few_rows(d_ffn, streamed):
    """From F = 8193 on (96 weight rows a tile, three quarters of a tile's traffic with few rows), and while the aligned kernel's tiles
    of 128 features leave more than an eighth of the compute units without work."""
    cfg = ModelConfig(1, 3584, 28, 4, 128, d_ffn, 2304, "bf16")
    for rows in (2, 16, 17, 128, 129):
        r = A.atts_pass_routes(cfg, A.PASS_SCORE, 1, 1, rows - 1).gate_up
        assert (r.kernel == A.KERNEL_STREAMED) == (streamed and rows <= 128), rows


NARROW = ModelConfig(1, 3584, 28, 4, 128, 9216, 768, "bf16")       # tiles of 64 columns; of 128 for down from 33 rows on
WIDE = ModelConfig(1, 5568, 42, 2, 128, 4096, 768, "bf16")         # tiles of 128 columns, the last half filled


@pytest.mark.parametrize("cfg,rows,slices", [(NARROW, 16, (3, 4, 4)), (NARROW, 33, (3, 4, 9)), (WIDE, 17, (5, 5, 5)), (WIDE, 64, (5, 5, 5)),
                                             (ModelConfig(1, 8192, 64, 8, 128, 28672, 768, "bf16"), 20, (None, 4, 4)),
                                             (ModelConfig(1, 768, 6, 2, 128, 1024, 768, "bf16"), 20, (None, None, None))])
def test_route_of_narrow_projections(cfg, rows, slices):
    """QKV, O and down up to 64 rows where the tiles and slices fill three quarters of the chip; the bound of their sums holds for fewer rows."""
    r = A.atts_pass_routes(cfg, A.PASS_SCORE, 1, 1, rows - 1)
    for product, s in zip((r.qkv, r.o, r.down), slices):
        assert (product.kernel == A.KERNEL_STREAMED) == (s is not None) and (s is None or product.slices == s)
    r = A.atts_pass_routes(cfg, A.PASS_SCORE, 1, 1, 64)
    assert A.KERNEL_STREAMED not in (r.qkv.kernel, r.o.kernel, r.down.kernel)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,rows", [(NARROW, 2), (NARROW, 16), (NARROW, 17), (NARROW, 32), (NARROW, 33), (NARROW, 64), (WIDE, 5), (WIDE, 32), (WIDE, 50), (WIDE, 64)])
def test_partial_sums_of_a_few_rows(cfg, rows):
    """One and two blocks of rows, whole and not, slices of unequal length, a partly filled last tile; against the oracle, and against the same
    draft scored several times in one call of more than 64 rows, which other kernels serve."""
    announce("streamed partial sums", cfg.d_model, rows)
    w = make_weights(cfg, seed=rows, device="cuda")
    prefix, drafts = [x.numpy() for x in make_token_ids(cfg.vocab, 1, 1, rows - 1, seed=rows)]
    model = A.Model(cfg, w)

    def score(K):
        lp, sc = torch.full((K, rows - 1), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
        space = dirty_ws(A.atts_workspace_bytes(model, 1, K, rows - 1))
        A.atts_score_drafts(model, dev(prefix), dev(np.repeat(drafts, K, axis=0)), None, 0, lp, sc, space)
        return lp.cpu().numpy()
    lp, ref = score(1), O.score_drafts(weights_to_numpy(w), cfg, prefix, drafts)[0]
    assert np.abs(lp - ref).max() <= 2e-2                             # bf16 log-probabilities
    more = score(max(2, 64 // (rows - 1) + 1))                        # other orders of sums and attention tiles: half the tolerance
    assert np.abs(more - lp).max() <= 1e-2
    model.close()


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,rows", [(NARROW, 2), (NARROW, 16), (NARROW, 33), (NARROW, 64), (WIDE, 17), (WIDE, 64)])
@pytest.mark.parametrize("values_alone", [False, True])
def test_every_block_of_columns(cfg, rows, values_alone):
    """Partial sums column by column: the LM head takes single features of the last hidden state, one of every 32 in turn, each as the target of
    one row.  O and down as they are; and with O the identity, so that the values (the last columns of QKV) reach the features by themselves."""
    announce("streamed columns", cfg.d_model, rows, values_alone)
    d, T = cfg.d_model, rows - 1
    w = make_weights(cfg, seed=rows, device="cuda")
    if values_alone:
        w["wo"][0].copy_(torch.eye(d, cfg.n_q_heads * cfg.head_dim))
        w["w_down"][0].zero_()
    ids = np.random.default_rng(rows).permutation(cfg.vocab).astype(np.int32)
    prefix, drafts = ids[:1], ids[1:rows]                             # every row has a target of its own
    host = weights_to_numpy(w)
    hidden = O.rmsnorm(O.decoder_hidden(host, cfg, ids[:rows]), host["final_norm"], cfg.rms_eps)[:T]
    model, space = A.Model(cfg, w), None
    for first in range(0, d // 32, T):
        blocks = np.arange(first, first + T) % (d // 32)
        columns = 32 * blocks + (5 * blocks + rows) % 32
        head = torch.zeros(cfg.vocab, d)
        head[drafts, columns] = 2.0
        w["lm_head"].copy_(head)
        lp, sc = torch.full((1, T), float("nan"), device="cuda"), torch.full((1,), float("nan"), device="cuda")
        space = dirty_ws(A.atts_workspace_bytes(model, 1, 1, T)) if space is None else space
        A.atts_score_drafts(model, dev(prefix), dev(drafts[None]), None, 0, lp, sc, space)
        z = np.zeros((T, cfg.vocab))
        z[:, drafts] = 2.0 * hidden[:, columns]
        ref = O.log_softmax(z)[np.arange(T), drafts]
        # features up to 5 stored in bf16, twice: 2 x 5 x 2^-9 = 0.02, half as much again for the roundings ahead; another column's feature is 2 off
        assert np.abs(lp.cpu().numpy()[0] - ref).max() <= 3e-2, first
    model.close()


@pytest.mark.gpu
@pytest.mark.parametrize("d_ffn,rows", [(8320, 2), (8320, 33), (8320, 128), (12416, 16), (12416, 64), (12416, 65), (18944, 4), (18944, 32), (18944, 63),
                                        (18944, 100), (22016, 17), (22016, 48), (22016, 127), (27648, 31), (27648, 64), (27648, 128)])
def test_every_block_of_features(d_ffn, rows):
    """3 to 7 blocks a tile with a partly filled last tile (and a whole one), 1, 2 and 4 blocks of rows, whole and not."""
    cfg = ModelConfig(1, D, 6, 2, 128, d_ffn, 768, "bf16")
    P, K, T = 1, 1, rows - 1
    assert A.atts_pass_routes(cfg, A.PASS_SCORE, P, K, T).gate_up.kernel == A.KERNEL_STREAMED
    w = make_weights(cfg, seed=rows, device="cuda")
    prefix, drafts = [x.numpy() for x in make_token_ids(cfg.vocab, P, K, T, seed=d_ffn)]
    blocks = d_ffn // 16
    space = dirty_ws(A.atts_pass_routes(cfg, A.PASS_SCORE, P, K, T).workspace_bytes)
    for first in range(0, blocks, D):
        announce("streamed swiglu", d_ffn, rows, first)
        pick = torch.zeros(D, d_ffn)
        for i, b in enumerate(range(first, min(first + D, blocks))):
            pick[i, 16 * b + (5 * b + first // D) % 16] = 2.0
        w["w_down"][0].copy_(pick)
        model = A.Model(cfg, w)
        lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
        A.atts_score_drafts(model, dev(prefix), dev(drafts), None, 0, lp, sc, space)
        ref_lp, ref_s = O.score_drafts(weights_to_numpy(w), cfg, prefix, drafts)
        # bf16 log-probabilities (2e-2); a block taken from another place moves its logits by about 2 x 0.5 / sqrt(768) each
        assert np.abs(lp.cpu().numpy() - ref_lp).max() <= 2e-2
        model.close()
