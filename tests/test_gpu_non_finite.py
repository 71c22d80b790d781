"""A NaN or inf in one row of Q, K or V reaches the output rows that attend to it and no other one: stage 3 with and
without such rows, at places where other queries share a wave, a 32-query tile, a matrix product's column or a list
with them.  Everything else has to come out as without them: to the bit, unless a query among them, or one that they
replace, moves the softmax reference of its wave (a 16-query tile shares that decision)."""
import numpy as np
import pytest
import torch

from oracle import stem_oracle as so
from paper_2603_06274_amd import binding as sb

pytestmark = pytest.mark.gpu

HQ, HKV = 4, 2


def make(B, d, moving):
    # last blocks of 16 tokens (their last query is copied into the tile's unused lanes), of 31 and of B
    lens = [2 * B + 16, 3 * B + 31, 4 * B]
    cu = [0] + np.cumsum(lens).tolist()
    g = torch.Generator().manual_seed(23)
    T = cu[-1]
    ramp = 1.0 + 7.0 * moving * torch.arange(T).float() / T   # moving: the softmax reference does
    q = torch.randn(T, HQ, d, generator=g)
    k = torch.randn(T, HKV, d, generator=g) * ramp[:, None, None]
    v = torch.randn(T, HKV, d, generator=g)
    r = np.random.default_rng(7)
    R, nbmax = so.total_rows(cu, B)
    counts, idx = np.zeros((HQ, R), np.int32), np.full((HQ, R, nbmax), -1, np.int32)
    for (_, _, nb, row0) in so.sequence_table(cu, B):
        for i in range(nb):
            for h in range(HQ):
                before = [x for x in range(i) if r.random() < 0.8]
                pick = [i] + before if h % 2 else before + [i]   # the diagonal block masked key by key, or at the end
                counts[h, row0 + i], idx[h, row0 + i, :len(pick)] = len(pick), pick
    return cu, [x.to(torch.bfloat16) for x in (q, k, v)], counts, idx


def attend(B, d, cu, qkv, counts, idx):
    dev = torch.device("cuda:0")
    q, k, v = (x.to(dev) for x in qkv)
    shape = sb.Shape.from_tensors(q, k, B, cu)
    out = torch.full_like(q, 7.0)
    lse = torch.full((HQ, q.shape[0]), 7.0, dtype=torch.float32, device=dev)
    sb.stem_sparse_attn(shape, q, k, v, torch.from_numpy(counts).to(dev), torch.from_numpy(idx).to(dev), idx.shape[2],
                        d ** -0.5, out, lse)
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), lse.cpu().numpy()


def rows_with(B, cu, counts, idx, token, kv_head, causal):
    """[T, HQ]: the queries whose list holds the key's block, and of the key's own block the ones from it on if causal."""
    hit = np.zeros((cu[-1], HQ), bool)
    s = int(np.searchsorted(cu, token, side="right")) - 1
    row0, j = so.sequence_table(cu, B)[s][3], (token - cu[s]) // B
    for i in range(j, -(-(cu[s + 1] - cu[s]) // B)):
        lo, hi = cu[s] + i * B, min(cu[s] + (i + 1) * B, cu[s + 1])
        for h in range(HQ):
            if h // (HQ // HKV) == kv_head and j in idx[h, row0 + i, :counts[h, row0 + i]]:
                hit[max(lo, token) if causal and i == j else lo:hi, h] = True
    return hit


def same(got, want, rows, vmax, moving):
    """out and lse of `rows` as without the rows put in.  With another reference every bf16 probability may round the other
    way: 2^-8 of it before and after, so lse differs by 2^-7 at most and the output by 2^-7 of the values' distance from it;
    its own rounding adds 2^-8 of it on both sides."""
    (out, lse), (o, l) = [(x[rows], y.T[rows]) for x, y in (got, want)]
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    if moving:
        big = np.abs(o).max()
        assert np.abs(out - o).max() <= 2 ** -7 * (vmax + 2 * big) and np.abs(lse - l).max() <= 2 ** -7 + 1e-5
    else:
        assert np.array_equal(out, o) and np.array_equal(lse, l)


BAD = [float("nan"), float("inf"), float("-inf")]


@pytest.mark.parametrize("moving", [False, True])
@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("B,d", [(128, 128), (64, 128), (128, 64), (64, 64), (128, 256), (64, 256)])
def test_non_finite_rows_reach_only_what_attends_to_them(B, d, bad, moving):
    print("case", B, d, bad, moving, flush=True)
    cu, qkv, counts, idx = make(B, d, moving)
    vmax = qkv[2].abs().max().item()
    want = attend(B, d, cu, qkv, counts, idx)
    assert np.isfinite(want[0]).all() and np.isfinite(want[1]).all()

    # queries: the last of a tile that is not full, both halves of a tile, a block of one, the last of a sequence
    q = qkv[0].clone()
    hit = np.zeros((cu[-1], HQ), bool)
    for token, h in ((cu[1] - 1, 0), (cu[1] - 1, 1), (cu[1] + 5, 0), (cu[1] + B + 21, 2), (cu[2] + B + 33, 3),
                     (cu[2], 0), (cu[2] - 1, 3), (cu[3] - 1, 1)):
        q[token, h] = bad
        hit[token, h] = True
    got = attend(B, d, cu, [q] + qkv[1:], counts, idx)
    same(got, want, ~hit, vmax, moving)
    if np.isnan(bad):
        assert np.isnan(got[0][hit]).all()

    # keys and values of one KV head each, in the middle of a diagonal tile, at its ends, in an earlier block of later rows
    for token, g in ((cu[1] - 1, 0), (cu[1] + B + 20, 1), (cu[2] + 32, 0), (cu[2] + 3 * B + 63, 1)):
        k, v = qkv[1].clone(), qkv[2].clone()
        k[token, g] = bad
        hit = rows_with(B, cu, counts, idx, token, g, causal=True)
        got = attend(B, d, cu, [qkv[0], k, qkv[2]], counts, idx)
        same(got, want, ~hit, vmax, moving)
        if np.isnan(bad):
            assert np.isnan(got[0][hit]).all()
        v[token, g] = bad
        got = attend(B, d, cu, qkv[:2] + [v], counts, idx)
        same(got, want, ~rows_with(B, cu, counts, idx, token, g, causal=False), vmax, moving)
        assert np.array_equal(got[1], want[1])         # values do not enter lse

