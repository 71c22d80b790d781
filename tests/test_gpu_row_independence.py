"""Stage 3 sums a row in one order, whatever else its call holds: rows asked for in a chunk, without the
sequences they were packed with, or by fewer heads come out as the same bits of output and lse."""
import numpy as np
import pytest
import torch

from oracle import stem_oracle as so
from paper_2603_06274_amd import binding as sb

pytestmark = pytest.mark.gpu


class Call:
    """Inputs and lists of a packed call on the device, and parts of it as calls of their own."""

    def __init__(self, B, d, Hq, Hkv, lens, longest_list, shared=False, wide=0):
        self.B, self.d, self.Hq, self.Hkv, self.G = B, d, Hq, Hkv, Hq // Hkv
        self.cu = [0] + np.cumsum(lens).tolist()
        T = self.cu[-1]
        dev = torch.device("cuda:0")
        g = torch.Generator().manual_seed(9)
        ramp = 1.0 + 3.0 * torch.arange(T).float() / T                 # the softmax reference moves
        q = 2.0 * torch.randn(T, Hq, d, generator=g)
        k = torch.randn(T, Hkv, d, generator=g) * ramp[:, None, None]
        self.q = q.to(torch.bfloat16).to(dev)
        self.kv = []
        for x in (k, torch.randn(T, Hkv, d, generator=g)):
            rows = torch.empty(T, Hkv, d + wide, dtype=torch.bfloat16, device=dev)
            rows[:, :, :d] = x.to(torch.bfloat16).to(dev)
            self.kv.append(rows[:, :, :d])
        r = np.random.default_rng(5)
        self.table = so.sequence_table(self.cu, B)
        R, lists = so.total_rows(self.cu, B)[0], Hkv if shared else Hq
        self.shared = shared
        counts = np.zeros((lists, R), np.int32)
        indices = np.full((lists, R, longest_list), -1, np.int32)
        for (_, _, nb, row0) in self.table:
            for i in range(nb):
                for h in range(lists):
                    n = min(i + 1, int(r.integers(1, longest_list + 1)))
                    pick = np.sort(np.append(r.permutation(i)[:n - 1], i))
                    counts[h, row0 + i] = n
                    indices[h, row0 + i, :n] = pick
        self.counts, self.indices = torch.from_numpy(counts).to(dev), torch.from_numpy(indices).to(dev)

    def attend(self, seqs, chunk=None, kv_heads=None):
        """out and lse of the sequences `seqs` (chunk: block range of each, (lo, hi)), of the first kv_heads
        KV heads, as one call; and the token rows of the whole call that they are."""
        kv_heads = kv_heads or self.Hkv
        heads = kv_heads * self.G
        B, cu, starts, ends = self.B, [0], [], []
        tokens, keys, rows = [], [], []
        for x, s in enumerate(seqs):
            lo, hi, nb, row0 = self.table[s]
            a, b = chunk[x] if chunk else (0, nb)
            starts.append(a * B)
            ends.append(min(b * B, hi - lo))
            cu.append(cu[-1] + hi - lo)
            keys.append(torch.arange(lo, hi))
            tokens.append(torch.arange(lo + starts[-1], lo + ends[-1]))
            rows.append(torch.arange(row0 + a, row0 + b))
        tokens, keys, rows = torch.cat(tokens), torch.cat(keys), torch.cat(rows)
        q = self.q[tokens][:, :heads].contiguous()
        if seqs == list(range(len(self.table))):
            k, v = (x[:, :kv_heads] for x in self.kv)
        else:
            k, v = (x[keys][:, :kv_heads].contiguous() for x in self.kv)
        lists = kv_heads if self.shared else heads
        counts, indices = (x[:lists, rows].contiguous() for x in (self.counts, self.indices))
        shape = sb.Shape.from_tensors(q, k, B, cu, (starts, ends) if chunk else None)
        out = torch.full_like(q, float("nan"))
        lse = torch.full((heads, q.shape[0]), float("nan"), dtype=torch.float32, device=q.device)
        sb.stem_sparse_attn(shape, q, k, v, counts, indices, indices.shape[2], self.d ** -0.5, out, lse,
                            lists_per_kv_head=self.shared)
        torch.cuda.synchronize()
        assert not torch.isnan(out).any().item() and not torch.isnan(lse).any().item()
        return out, lse, tokens

    def check_part(self, whole, seqs, chunk=None, kv_heads=None):
        out, lse, tokens = self.attend(seqs, chunk, kv_heads)
        print("part: sequences", seqs, "blocks", chunk, "kv heads", kv_heads or self.Hkv, flush=True)
        assert torch.equal(out, whole[0][tokens][:, :out.shape[1]])
        assert torch.equal(lse, whole[1][:lse.shape[0], tokens])


@pytest.mark.parametrize("B,d,shared,wide", [
    (64, 128, False, 0), (64, 64, True, 0), (64, 256, False, 0),
    (128, 128, True, 0), (128, 64, False, 0), (128, 256, False, 0), (128, 128, False, 24),
])
def test_parts_of_a_call_by_themselves(B, d, shared, wide):
    """A call with more (head, row) pairs than the chip takes at a time, and parts of it that
    leave most of the chip idle, down to one row of one group of heads."""
    blocks = 110 if B == 64 else 80
    c = Call(B, d, 16, 4, (blocks * B - 5, 20 * B, 3 * B + 1), 70, shared, wide)
    whole = c.attend([0, 1, 2])
    c.check_part(whole, [1])
    c.check_part(whole, [0, 1, 2], [(blocks - 12, blocks), (9, 9), (2, 4)])
    c.check_part(whole, [0], [(blocks - 30, blocks - 26)])
    c.check_part(whole, [0], [(blocks - 1, blocks)], 1)
    c.check_part(whole, [1, 0], None, 1)


@pytest.mark.parametrize("d,blocks", [(128, 300), (64, 600), (256, 200)])
def test_rows_of_a_call_of_several_rounds(d, blocks):
    """B = 64 and more keys than an XCD's L2 holds: the rows that run late in a call of several rounds of
    workgroups, against a call of their own (in which they run first), and packed with another sequence."""
    c = Call(64, d, 8, 1, (blocks * 64 - 7, 11 * 64), 100)
    whole = c.attend([0, 1])
    c.check_part(whole, [0])
    c.check_part(whole, [0], [(blocks // 3, blocks // 3 + 40)])
    c.check_part(whole, [0, 1], [(blocks // 2, blocks // 2 + 60), (11, 11)])


@pytest.mark.parametrize("B,d,heads,lens", [
    (128, 128, (16, 4), (1500, 70, 900, 1300, 0, 400, 1500, 129, 2000, 64)),
    (64, 64, (24, 3), (1500, 70, 900, 1300, 0, 400, 1500, 65, 2000, 64)),
])
def test_rows_of_a_batch_in_another_order(B, d, heads, lens):
    """A batch whose rows are handed out longest sequence first: sequences by themselves, in another order
    (ascending, as they come) and with chunks."""
    c = Call(B, d, *heads, lens, 20)
    whole = c.attend(list(range(len(lens))))
    c.check_part(whole, [2])
    c.check_part(whole, sorted(range(len(lens)), key=lambda s: lens[s]))
    c.check_part(whole, [8, 1, 0], [(9, 12), (0, 1), (2, 5)])


@pytest.mark.parametrize("B,d,heads,line", [(64, 128, 8, 2.0), (64, 64, 8, 2.0), (128, 128, 4, 0.75), (128, 64, 4, 1.0),
                                            (64, 256, 8, 2.0), (128, 256, 4, 1.0)])
def test_rows_on_both_sides_of_the_line_between_wave_shapes(B, d, heads, line):
    """Calls of at most `line` rows per CU run with half as many queries per wave: a call just above the line, the same rows
    in one on it, and one row of it."""
    blocks = int(line * torch.cuda.get_device_properties(0).multi_processor_count) // heads
    c = Call(B, d, heads, 2, ((blocks + 1) * B - 3,), 40)
    whole = c.attend([0])
    c.check_part(whole, [0], [(1, blocks + 1)])
    c.check_part(whole, [0], [(blocks, blocks + 1)])


@pytest.mark.parametrize("B,rows_per_cu,kmax", [(128, 16, 10), (64, 16, 10), (64, 6, 20)])
def test_rows_on_both_sides_of_the_lines_between_wave_shapes_at_d_256(B, rows_per_cu, kmax):
    """Head size 256, lists with room for `kmax` blocks: a call just above `rows_per_cu` rows per CU, the same rows in one
    on it; and with room for one block more, where the wider shape starts."""
    blocks = rows_per_cu * torch.cuda.get_device_properties(0).multi_processor_count // 32
    c = Call(B, 256, 32, 4, ((blocks + 1) * B - 3,), kmax)
    whole = c.attend([0])
    c.check_part(whole, [0], [(1, blocks + 1)])
    c.indices = torch.cat([c.indices, torch.full_like(c.indices[:, :, :1], -1)], dim=2)
    c.check_part(whole, [0], [(1, blocks + 1)])


@pytest.mark.parametrize("B,d,rows_per_cu,kmax,late", [
    # the whole prompt's rows on the line and one block more of every head, or, late, the last rows of a longer one
    (128, 128, 1, 40, True), (128, 128, 2, 60, False), (128, 64, 1, 40, True), (128, 64, 2, 60, False),
    (64, 64, 2.75, 11, True), (64, 64, 3, 12, True), (64, 64, 4, 80, False),
    (64, 128, 2, 11, True), (64, 128, 3, 12, True), (64, 128, 3, 80, True), (64, 128, 4, 80, False),
    (64, 256, 1, 51, True), (64, 256, 3, 50, True), (64, 256, 3, 80, False), (128, 256, 16, 8, True),
])
def test_rows_on_both_sides_of_each_line(B, d, rows_per_cu, kmax, late):
    """Every line of the rule for the number of queries per wave: a call on it and one a block per head above it."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    heads = 32 if rows_per_cu == 16 else 8
    blocks = int(rows_per_cu * cus) // heads
    first = blocks if late else 0
    c = Call(B, d, heads, 2, ((first + blocks + 1) * B - 3,), kmax)
    above = c.attend([0], [(first, first + blocks + 1)])
    out, lse, tokens = c.attend([0], [(first, first + blocks)])
    print("case", B, d, blocks, kmax, late, flush=True)
    assert torch.equal(out, above[0][:out.shape[0]]) and torch.equal(lse, above[1][:, :lse.shape[1]])
    c.indices = torch.cat([c.indices, torch.full_like(c.indices[:, :, :1], -1)], dim=2)   # and with room for one block more
    out, lse, tokens = c.attend([0], [(first, first + blocks)])
    assert torch.equal(out, above[0][:out.shape[0]]) and torch.equal(lse, above[1][:, :lse.shape[1]])
