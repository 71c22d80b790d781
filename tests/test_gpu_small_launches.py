"""Attention in launches around the number of workgroups that the chip takes at a time, every instantiation:
one-entry lists, unusable entries, an empty list and logits that make the softmax reference move in every block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,Hq,Hkv", [
    # Hq x 25 rows (B = 64) or 13 rows (B = 128)
    (64, 128, 4, 2), (64, 128, 16, 2), (64, 128, 44, 2),
    (64, 64, 10, 1), (64, 64, 20, 1), (64, 64, 43, 1),
    (64, 256, 10, 2), (128, 256, 10, 1),
    (128, 128, 18, 3), (128, 128, 22, 2),
    (128, 64, 4, 1), (128, 64, 24, 2),
])
def test_small_launches(B, d, Hq, Hkv):
    import torch
    import parity_util as pu
    from oracle import stem_oracle as so
    from paper_2603_06274_amd import binding as sb
    torch.manual_seed(8)
    T, G = 1536, Hq // Hkv
    cu = [0, 1000, T]
    q = torch.randn(T, Hq, d) * 3.0
    k = torch.randn(T, Hkv, d)
    v = torch.randn(T, Hkv, d)
    ramp = 1.0 + 6.0 * torch.arange(T).float() / T                     # later keys score higher
    ramp[40::97] *= 3.0                                                # spikes inside blocks
    k = k * ramp[:, None, None] + 0.5 * q.view(T, Hkv, G, d).mean(2) * ramp[:, None, None]
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    qkv = tuple(x.float().numpy() for x in (q, k, v))
    scale = d ** -0.5
    R, nbmax = so.total_rows(cu, B)
    clean_c, clean_i = np.zeros((Hq, R), np.int32), np.full((Hq, R, nbmax + 8), -1, np.int32)
    counts, idx = clean_c.copy(), clean_i.copy()
    r = np.random.default_rng(5)
    for (_, _, nb, row0) in so.sequence_table(cu, B):
        for i in range(nb):
            for h in range(Hq):
                pick = sorted(set(r.integers(0, i + 1, size=1 + int(r.integers(0, 2 * i + 2))).tolist()) | {i})
                junk = [-3, i + 1 + int(r.integers(0, 50)), 2 ** 30][:int(r.integers(0, 4))]
                dirty = junk[2:] + pick[:len(pick) // 2] + junk[:1] + pick[len(pick) // 2:] + junk[1:2]
                for c, ix, entries in ((clean_c, clean_i, pick), (counts, idx, dirty)):
                    c[h, row0 + i] = len(entries)
                    ix[h, row0 + i, :len(entries)] = entries
    counts[:, R - 1] = 0                                               # an empty list: zeros and -inf
    idx[:, R - 1] = -1
    dev = torch.device("cuda:0")
    qd, kd, vd = (x.to(dev) for x in (q, k, v))
    shape = sb.Shape.from_tensors(qd, kd, B, cu)
    heads = [0, Hq - 1]
    for name, c, ix in (("clean", clean_c, clean_i), ("with unusable entries", counts, idx)):
        print("case B %d d %d Hq %d: %s" % (B, d, Hq, name), flush=True)
        last = T if name == "clean" else T - (T - 1000 - 1) % B - 1    # without the row whose list is empty
        o_out, o_lse = so.sparse_attention(*qkv, cu, B, clean_c, clean_i, scale, heads=heads)
        o_out[last:], o_lse[:, last:] = np.nan, np.nan
        runs = []
        for _ in range(2):
            out = torch.full_like(qd, float("nan"))
            lse = torch.full((Hq, T), float("nan"), dtype=torch.float32, device=dev)
            sb.stem_sparse_attn(shape, qd, kd, vd, torch.from_numpy(c).to(dev), torch.from_numpy(ix).to(dev),
                                ix.shape[2], scale, out, lse)
            torch.cuda.synchronize()
            runs.append((out, lse))
        assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
        assert not torch.isnan(out).any().item() and not torch.isnan(lse).any().item()
        if last < T:
            assert not out[last:].any().item() and torch.isneginf(lse[:, last:]).all().item()
        pu.check_output(out, o_out, name, print, pu.ListedKeys(qkv, cu, B, clean_c, clean_i, scale))
        known = ~np.isnan(o_lse)
        err = np.abs(lse.cpu().numpy() - o_lse)[known] / np.maximum(1.0, np.abs(o_lse[known]))
        assert err.max() <= 5e-3
