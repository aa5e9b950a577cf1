"""The end of a scoring pass: final norm, LM head, log-probabilities and scores, in the launches that the sizes choose."""
import numpy as np
import pytest
import torch

import paper_2509_15148_amd as A
from oracle import atts_oracle as O
from synth import ModelConfig, make_token_ids, make_weights
from util import announce, dev, dirty_ws, weights_to_numpy

pytestmark = pytest.mark.gpu

SMALL = ModelConfig(1, 128, 4, 4, 32, 256, 1000, "fp32")           # scoring rows gathered and normalised inside the LM head's product
BF16 = ModelConfig(1, 768, 6, 2, 128, 256, 2304, "bf16")


@pytest.mark.parametrize("cfg,P,K,T", [(SMALL, 1, 1, 1), (SMALL, 3, 5, 1), (SMALL, 40, 3, 15), (SMALL, 7, 4, 16), (SMALL, 2, 9, 17), (SMALL, 5, 2, 32),
                                       (SMALL, 6, 2, 33), (SMALL, 4, 1, 70), (BF16, 1, 2, 8), (BF16, 9, 3, 32), (BF16, 4, 2, 33)])
@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("mode", [A.SCORE_MEAN_NLL, A.SCORE_SUM_NLL])
def test_log_probabilities_and_scores(cfg, P, K, T, cached, mode):
    """Drafts of at most 32 tokens take their scores with their log-probabilities; lengths from none to all tokens and outside of that, ids
    outside the vocabulary past a draft's length; the first tokens' hidden state from the tree and from a prefix handle."""
    announce("pass tail", cfg.dtype, P, K, T, cached, mode)
    w = make_weights(cfg, seed=K, device="cuda")
    prefix, drafts = [x.numpy() for x in make_token_ids(cfg.vocab, P, K, T, seed=T)]
    lens = np.random.default_rng(T).integers(1, T + 1, K).astype(np.int32)
    lens[0] = T
    for k, out_of_range in ((1, 0), (2, T + 5), (3, -2)):             # no token, and lengths that are read as all and as none
        if k < K:
            lens[k] = out_of_range
    padded, given, lens = drafts.copy(), lens, np.clip(lens, 0, T)
    for k in range(K):
        padded[k, lens[k]:] = -5 if k % 2 else cfg.vocab + 7
    model = A.Model(cfg, w)
    lp, sc = torch.full((K, T), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    space = dirty_ws(A.atts_workspace_bytes(model, P, K, T))
    if cached:
        pre = A.Prefix(model, P)
        A.atts_prefix_extend(pre, dev(prefix), dirty_ws(A.atts_prefix_extend_workspace_bytes(pre, P)))
        A.atts_score_drafts_cached(pre, dev(padded), dev(given), mode, lp, sc, space)
    else:
        A.atts_score_drafts(model, dev(prefix), dev(padded), dev(given), mode, lp, sc, space)
    no_lp, again = None, torch.full((K,), float("nan"), device="cuda")
    if not cached:                                                    # scores alone
        A.atts_score_drafts(model, dev(prefix), dev(padded), dev(given), mode, no_lp, again, space)
        assert torch.equal(again, sc)
    ref_lp = O.score_drafts(weights_to_numpy(w), cfg, prefix, drafts)[0]
    live = np.arange(T)[None, :] < lens[:, None]
    got, tol = lp.cpu().numpy(), 1e-4 if cfg.dtype == "fp32" else 2e-2
    assert np.abs(got - ref_lp * live).max() <= tol and (got[~live] == 0).all()
    total = -(ref_lp * live).sum(axis=1)
    want = total / np.maximum(lens, 1) if mode == A.SCORE_MEAN_NLL else total
    assert np.abs(sc.cpu().numpy() - want).max() <= tol * (1 if mode == A.SCORE_MEAN_NLL else T)
