"""The diagonal block of a row is left out of both products where a wave's queries cannot see it when it stands at the
end of a list, and masked key by key anywhere else.  Lists that hold it last, first, in the middle, twice, alone or not
at all, with the softmax reference moved by it or not, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import stem_oracle as so
from paper_2603_06274_amd import binding as sb

import parity_util as pu

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


PLACES = {
    "last": lambda before, i: before + [i],
    "first": lambda before, i: [i] + before,
    "twice": lambda before, i: before[:1] + [i] + before[1:] + [i],
    "middle": lambda before, i: before[:1] + [i] + before[1:],
    "alone": lambda before, i: [i],
    "absent": lambda before, i: before,
}


@pytest.mark.parametrize("place", sorted(PLACES))
@pytest.mark.parametrize("B,d", [(128, 128), (64, 128), (128, 64), (64, 64), (128, 256), (64, 256)])
def test_diagonal_block_wherever_it_stands(B, d, place):
    # the last block of a sequence holds 1, 31, 33, B - 1 and B tokens: a wave without queries, with one, with all but one
    lens = [3 * B + 1, B + 31, 2 * B + 33, 4 * B - 1, 5 * B, 1]
    cu = [0] + np.cumsum(lens).tolist()
    Hq, Hkv, T = 4, 2, sum(lens)
    g = torch.Generator().manual_seed(17)
    q, k, v = (torch.randn(T, h, d, generator=g) for h in (Hq, Hkv, Hkv))
    spike = torch.ones(T)
    for s, n in enumerate(lens):                       # every second sequence: a key in its last block's own tiles that
        if s % 2 and n > B:                            # overflows the reference set by the blocks before
            spike[cu[s + 1] - max(1, n % B // 2):cu[s + 1]] = 40.0
    k = k * spike[:, None, None]
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    qkv = tuple(x.float().numpy() for x in (q, k, v))
    R, nbmax = so.total_rows(cu, B)
    counts, idx = np.zeros((Hq, R), np.int32), np.full((Hq, R, nbmax + 1), -1, np.int32)
    want_c, want_i = counts.copy(), idx.copy()
    r = np.random.default_rng(3)
    for (_, _, nb, row0) in so.sequence_table(cu, B):
        for i in range(nb):
            for h in range(Hq):
                before = [x for x in range(i) if r.random() < 0.7]
                pick = PLACES[place](before, i)
                counts[h, row0 + i], idx[h, row0 + i, :len(pick)] = len(pick), pick
                want_c[h, row0 + i], want_i[h, row0 + i, :len(pick)] = len(pick), sorted(pick)
    dev = torch.device("cuda:0")
    qd, kd, vd = (x.to(dev) for x in (q, k, v))
    shape = sb.Shape.from_tensors(qd, kd, B, cu)
    say("case", place, B, d)
    out = torch.full_like(qd, float("nan"))
    lse = torch.zeros((Hq, T), dtype=torch.float32, device=dev)
    sb.stem_sparse_attn(shape, qd, kd, vd, torch.from_numpy(counts).to(dev), torch.from_numpy(idx).to(dev),
                        idx.shape[2], d ** -0.5, out, lse)
    torch.cuda.synchronize()
    o_out, o_lse = so.sparse_attention(*qkv, cu, B, want_c, want_i, d ** -0.5)
    pu.check_output(out, o_out, place, say, pu.ListedKeys(qkv, cu, B, want_c, want_i, d ** -0.5))
    got, seen = lse.cpu().numpy(), np.isfinite(o_lse)
    assert np.array_equal(seen, np.isfinite(got)) and not np.isnan(got).any()
    assert (np.abs(got[seen] - o_lse[seen]) / np.maximum(1.0, np.abs(o_lse[seen]))).max() <= 5e-3


@pytest.mark.parametrize("B,d", [(128, 128), (64, 128), (128, 64), (64, 64), (128, 256), (64, 256)])
def test_row_of_the_diagonal_block_alone(B, d):
    """A row whose only block is the diagonal one takes the same reference, and so the same bf16 probabilities, whether
    that block ends its list or an entry follows that nothing is done with.  Left is the order of the sum's additions: a
    few 2^-24 of it, which move one in some 10^4 outputs across a rounding boundary 2^-8 wide."""
    Hq, lens = 4, [B] * 9 + [B - 1, B // 2 + 1]
    cu, T = [0] + np.cumsum(lens).tolist(), sum(lens)
    g = torch.Generator().manual_seed(29)
    dev = torch.device("cuda:0")
    q, k, v = (torch.randn(T, Hq, d, generator=g).to(torch.bfloat16).to(dev) for _ in range(3))
    shape = sb.Shape.from_tensors(q, k, B, cu)
    idx = torch.tensor([0, -1], dtype=torch.int32, device=dev).repeat(Hq, len(lens), 1).contiguous()
    got = []
    for n in (1, 2):
        out, lse = torch.full_like(q, float("nan")), torch.zeros((Hq, T), dtype=torch.float32, device=dev)
        sb.stem_sparse_attn(shape, q, k, v, torch.full((Hq, len(lens)), n, dtype=torch.int32, device=dev), idx, 2,
                            d ** -0.5, out, lse)
        torch.cuda.synchronize()
        got.append((out.float().cpu().numpy(), lse.cpu().numpy()))
    (a, la), (b, lb) = got
    differ = (a != b).mean()
    say("case alone", B, d, "entries that differ", differ)
    assert differ <= 1e-3 and np.abs(la - lb).max() <= 2 ** -20 * max(1.0, np.abs(lb).max())
