"""Packed batches in orders that the hand-out of query-block rows has to untangle (longest sequence first,
rows of a sequence from the last to the first) or leaves as they come, with empty, equal and one-token sequences,
for head counts that take either mapping of heads to XCDs; every row of every sequence against the oracle."""
import pytest

from paper_2603_06274_amd import workloads as wl

from test_gpu_parity import run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,heads,lens,k", [
    (128, (4, 2), (64, 700, 0, 700, 1300, 1), 4),              # ascending with a tie, an empty and a short end
    (64, (3, 3), (0, 900, 130, 0, 64, 65), 4),                 # an empty head, descending; 3 KV heads
    (64, (4, 2), (300, 0, 500), 4),                            # the most sequences looked at one after the other
    (64, (4, 2), (0, 300, 500, 64), 4),                        # the fewest counted by a ballot
    (64, (8, 1), tuple(37 * ((7 * x) % 64) for x in range(64)), 4),   # the most sequences a call takes, one empty
    # handed out longest first: 64 sequences of at most 5 blocks, 8 x 189 rows; 10 sequences, 24 x 35 rows
    (64, (8, 1), tuple(5 * ((7 * x) % 64) for x in range(64)), 4),
    (128, (24, 3), (700, 64, 0, 1300, 129, 700, 1, 640, 0, 257), 11),
    # as they come: nine sequences; ascending; lists of at most 5 of 11 blocks
    (128, (24, 3), (700, 64, 0, 1300, 129, 700, 1, 640, 257), 11),
    (128, (24, 3), (0, 1, 64, 64, 129, 300, 300, 640, 700, 1300), 11),
    (128, (24, 3), (700, 64, 0, 1300, 129, 700, 1, 640, 0, 257), 5),
])
def test_sequence_orders(B, heads, lens, k):
    w = wl.small("orders_%d_%d" % (B, len(lens)), seed=68, num_q_heads=heads[0], num_kv_heads=heads[1], seq_lens=lens,
                 block_size=B, k_start=tuple(min(k, max(1, -(-n // B))) for n in lens), n_sink=1, n_local=1,
                 outliers=tuple(1 if n else 0 for n in lens))
    run_both(w)
