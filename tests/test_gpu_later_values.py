"""A NaN or inf among the values of keys that come after a query.  Where the diagonal block ends a row's list, the 32-key
tiles that begin after a wave's queries are left out of the second product, so that such a value reaches the queries from its
tile on and none before; anywhere else in the list it has a weight of zero in the whole block."""
import numpy as np
import pytest
import torch

from oracle import stem_oracle as so

import parity_util as pu
import test_gpu_non_finite as nf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("B,d", [(128, 128), (64, 128), (128, 64), (64, 64), (128, 256), (64, 256)])
def test_values_of_later_tiles_stay_out(B, d, wide, monkeypatch):
    print("case", B, d, wide, flush=True)
    if wide:
        pu.widen_attention(monkeypatch)
    cu, qkv, counts, idx = nf.make(B, d, False)
    want = nf.attend(B, d, cu, qkv, counts, idx)
    rows = so.sequence_table(cu, B)
    g, G = 1, nf.HQ // nf.HKV
    for s, block, offset in ((2, 3, 33), (2, 0, 63), (1, 2, B - 1), (2, 3, B - 32), (1, 3, 30)):
        token = cu[s] + block * B + offset
        for bad in (float("nan"), float("inf")):
            v = qkv[2].clone()
            v[token, g] = bad
            hit = nf.rows_with(B, cu, counts, idx, token, g, causal=False)
            lo = cu[s] + block * B
            for h in range(g * G, (g + 1) * G):
                r = rows[s][3] + block
                if idx[h, r, counts[h, r] - 1] == block:
                    hit[lo:lo + offset // 32 * 32, h] = False
            got = nf.attend(B, d, cu, qkv[:2] + [v], counts, idx)
            nf.same(got, want, ~hit, 0.0, False)
            assert np.array_equal(got[1], want[1])
            visible = nf.rows_with(B, cu, counts, idx, token, g, causal=True)
            assert not np.isfinite(got[0][visible]).any()
