"""B = 128: the softmax references of a row are taken from its first 96 keys, so that the largest of their probabilities is 1 and
enters the row's sum without rounding to bf16, wherever among them its key stands."""
import pytest
import torch

from paper_2603_06274_amd import binding as sb

import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("key", [3, 70, 95])
def test_largest_of_the_first_probabilities_is_exact(d, key, wide, monkeypatch):
    """One key scores 9 to 11 above all others (with a reference from those others it would stay below the line for a move),
    so the sum is 1 and at most 3 * 128 e^-9 = 0.05 of the others, rounded by 2^-9 of that: 1e-4.  A probability of e^10
    rounded to bf16 instead is off by up to 2^-9 = 2e-3."""
    if wide:
        pu.widen_attention(monkeypatch)
    B, T, H = 128, 3 * 128, 4
    dev = torch.device("cuda:0")
    g = torch.Generator().manual_seed(1)
    q = (0.9 + 0.2 * torch.rand(T, H, 1, generator=g)).expand(T, H, d).to(torch.bfloat16)
    k = torch.zeros(T, H, d)
    k[key] = 10.0 / d ** 0.5
    k, v = k.to(torch.bfloat16), torch.randn(T, H, d, generator=g).to(torch.bfloat16)
    scores = torch.einsum("thd,shd->hts", q.double(), k.double()) * d ** -0.5
    want = torch.logsumexp(scores.masked_fill(torch.ones(T, T).triu(1).bool(), float("-inf")), dim=2)
    assert scores[:, :, key].min() > 8.9 and scores[:, :, key].max() < 11.09          # below e^11.09 = 2^16: no move
    q, k, v = (x.contiguous().to(dev) for x in (q, k, v))
    counts = torch.tensor([1, 2, 3], dtype=torch.int32, device=dev).repeat(H, 1)
    idx = torch.tensor([0, 1, 2], dtype=torch.int32, device=dev).repeat(H, 3, 1)
    out, lse = torch.empty_like(q), torch.empty(H, T, device=dev)
    sb.stem_sparse_attn(sb.Shape.from_tensors(q, k, B, [0, T]), q, k, v, counts, idx, 3, d ** -0.5, out, lse)
    err = (lse.cpu().double() - want).abs()[:, key:].max().item()
    print("case", d, key, wide, "error", err, flush=True)
    assert err <= 1e-4 + 2 ** -18 * 11
