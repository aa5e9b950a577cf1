"""Attention by one wavefront per (row, head) with keys, values and scores in registers, against 64 bits, and the general kernel for what it
does not serve."""
import math

import pytest
import torch

import paper_2509_15148_amd as A
from util import announce

pytestmark = pytest.mark.gpu


def _reference(qkv, P, K, T, nq, nkv, hd):
    x = qkv.double().cpu()
    R = x.shape[0]
    row, key = torch.arange(R)[:, None], torch.arange(R)[None, :]
    seg = torch.where(row < P, torch.zeros_like(row), P + (row - P) // max(T, 1) * max(T, 1))
    hidden = ~((key <= row) & ((key < P) | (key >= seg)))
    out = torch.empty(R, nq * hd, dtype=torch.float64)
    for h in range(nq):
        g = h // (nq // nkv)
        q, k, v = (x[:, c * hd:(c + 1) * hd] for c in (h, nq + g, nq + nkv + g))
        z = (q @ k.t()) / math.sqrt(hd)
        out[:, h * hd:(h + 1) * hd] = torch.softmax(z.masked_fill(hidden, -math.inf), dim=-1) @ v
    return out


def _run(qkv, P, K, T, nq, nkv, hd, out=None):
    out = torch.full((qkv.shape[0], nq * hd), float("nan"), dtype=qkv.dtype, device="cuda") if out is None else out
    A.atts_attention_shared_prefix(qkv, out, P, K, T, nq, nkv, hd, None)
    torch.cuda.synchronize()
    return out.double().cpu()


HEADS = [(torch.float32, 16), (torch.float32, 32), (torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 32), (torch.bfloat16, 64),
         (torch.bfloat16, 256)]


@pytest.mark.parametrize("dtype,hd", HEADS)
@pytest.mark.parametrize("P,K,T", [(1, 1, 1), (30, 2, 3), (32, 1, 2), (63, 2, 2), (126, 3, 4), (255, 1, 3), (250, 2, 9), (5, 3, 130), (300, 2, 40)])
def test_contexts_around_the_batches(dtype, hd, P, K, T):
    """Contexts of one key, around the 32, 64, 128 and 256 rows that are requested together, and of several batches; a draft's keys begin
    inside a batch and inside a load; two query heads a key head."""
    announce("attention rows", dtype, hd, P, K, T)
    g = torch.Generator().manual_seed(P + hd)
    nq, nkv = 4, 2
    qkv = torch.randn(P + K * T, (nq + 2 * nkv) * hd, generator=g).to(dtype).cuda()
    err = (_run(qkv, P, K, T, nq, nkv, hd) - _reference(qkv, P, K, T, nq, nkv, hd)).abs().max().item()
    assert err <= (2e-5 if dtype == torch.float32 else 1.5e-2), err


@pytest.mark.parametrize("dtype,hd", HEADS)
@pytest.mark.parametrize("order", ["rising", "falling", "spikes"])
def test_running_maximum(dtype, hd, order):
    """Scores that rise or fall by thousands from batch to batch, and single keys far above the others: the maximum moves between
    batches or never again, and everything before it vanishes."""
    announce("attention rows maximum", dtype, hd, order)
    P, K, T, nq, nkv = 600, 1, 7, 2, 1
    R = P + K * T
    g = torch.Generator().manual_seed(hd)
    qkv = torch.randn(R, (nq + 2 * nkv) * hd, generator=g)
    size = {"rising": torch.arange(R) * 4.0, "falling": (R - torch.arange(R)) * 4.0,
            "spikes": torch.where(torch.arange(R) % 97 == 5, 3000.0 + torch.arange(R), torch.zeros(R))}[order]
    qkv[:, :nq * hd] = 1.0 / math.sqrt(hd)
    qkv[:, nq * hd:(nq + nkv) * hd] = size[:, None]
    qkv = qkv.to(dtype).cuda()
    got = _run(qkv, P, K, T, nq, nkv, hd)
    err = (got - _reference(qkv, P, K, T, nq, nkv, hd)).abs().max().item()
    # scores up to 1.3e4 in fp32 carry 1e-3, which moves a probability by as much where two keys' scores are near
    assert torch.isfinite(got).all() and err <= (1e-2 if dtype == torch.float32 else 3e-2), err


@pytest.mark.parametrize("dtype,hd", HEADS)
@pytest.mark.parametrize("P,K,T", [(1, 1, 1), (7, 2, 3), (64, 1, 5), (300, 2, 40)])
def test_infinite_values(dtype, hd, P, K, T):
    """An infinite value reaches the rows that see its key, the key's own row (whose last key it is) among them, and no others."""
    announce("attention rows infinities", dtype, hd, P, K, T)
    nq, nkv, R = 4, 2, P + K * T
    qkv = torch.randn(R, (nq + 2 * nkv) * hd, generator=torch.Generator().manual_seed(hd + R)).to(dtype)
    ref = _reference(qkv, P, K, T, nq, nkv, hd)                       # with finite values
    row = torch.arange(R)
    seg = torch.where(row < P, torch.zeros_like(row), P + (row - P) // T * T)
    for i, key in enumerate(sorted({0, P // 2, P - 1, P, P + T - 1, R - 1})):
        sees = (row >= key) & ((key < P) | (seg <= key))
        qkv[key, (nq + nkv) * hd + i] = qkv[key, (nq + 2 * nkv - 1) * hd + i] = -math.inf if i % 2 else math.inf
        for h in range(nq):
            ref[sees, h * hd + i] = -math.inf if i % 2 else math.inf
    got = _run(qkv.cuda(), P, K, T, nq, nkv, hd)
    infinite = torch.isinf(ref)
    assert torch.equal(got[infinite], ref[infinite])
    assert (got[~infinite] - ref[~infinite]).abs().max().item() <= (2e-5 if dtype == torch.float32 else 1.5e-2)


@pytest.mark.parametrize("dtype,hd", [(torch.float32, 32), (torch.bfloat16, 64), (torch.float32, 20), (torch.float32, 8), (torch.bfloat16, 24), (torch.bfloat16, 16)])
def test_other_heads_and_addresses(dtype, hd):
    """Heads of other sizes, and rows that do not start at 16 bytes, stay with the general kernel; outputs may start anywhere."""
    announce("attention rows others", dtype, hd)
    P, K, T, nq, nkv = 70, 2, 20, 4, 2
    R, cols = P + K * T, (nq + 2 * nkv) * hd
    flat = torch.randn(R * cols + 8, generator=torch.Generator().manual_seed(hd)).to(dtype).cuda()
    room = torch.empty(R * nq * hd + 8, dtype=dtype, device="cuda")
    ref = None
    for at, to in ((0, 0), (1, 0), (0, 1), (4, 4)):
        qkv = flat[at:at + R * cols].view(R, cols)
        if at == 0 or ref is None:
            src = qkv
        else:
            qkv.copy_(src.clone())
        ref = _reference(qkv, P, K, T, nq, nkv, hd)
        err = (_run(qkv, P, K, T, nq, nkv, hd, room[to:to + R * nq * hd].view(R, nq * hd)) - ref).abs().max().item()
        assert err <= (2e-5 if dtype == torch.float32 else 1.5e-2), (at, to, err)


@pytest.mark.parametrize("dtype,hd", HEADS)
def test_output_at_any_address(dtype, hd):
    """An output that does not start at 16 bytes is served by the same kernel: the same bits, and nothing beside it is written."""
    announce("attention rows output address", dtype, hd)
    P, K, T, nq, nkv = 70, 2, 20, 4, 2
    R, size = P + K * T, (P + K * T) * nq * hd
    qkv = torch.randn(R, (nq + 2 * nkv) * hd, generator=torch.Generator().manual_seed(hd)).to(dtype).cuda()
    ref = _run(qkv, P, K, T, nq, nkv, hd)
    for to in (1, 3, 4):
        room = torch.full((size + 8,), 7.0, dtype=dtype, device="cuda")
        assert torch.equal(_run(qkv, P, K, T, nq, nkv, hd, room[to:to + size].view(R, nq * hd)), ref)
        assert (room[:to] == 7).all() and (room[to + size:] == 7).all()
