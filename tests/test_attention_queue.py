"""stem_sparse_attn_queued: the last rows of a long call are claimed by the workgroups instead of handed out by their
ids.  Every row once, the same bits as stem_sparse_attn, whatever the scratch held; refused arguments; calls of several
streams side by side; a captured graph."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_06274_amd import binding as sb
from paper_2603_06274_amd.prefill import StemPrefill


def test_queue_arguments():
    shape = sb.Shape(4, 2, 128, 128, [0, 1024], (4 * 128, 128), (2 * 128, 128))
    L, fake = sb.lib(), 4096
    n = ctypes.c_size_t(1)
    assert L.stem_attn_queue_bytes(shape.ref(), 8, ctypes.byref(n)) == sb.STEM_OK and n.value == 0   # 32 rows: a short call
    assert L.stem_attn_queue_bytes(shape.ref(), 0, ctypes.byref(n)) == sb.STEM_ERR_INVALID_ARG
    assert L.stem_attn_queue_bytes(shape.ref(), 8, None) == sb.STEM_ERR_INVALID_ARG

    def call(queue, size, kmax=8, out=fake):
        return L.stem_sparse_attn_queued(shape.ref(), fake, fake, fake, fake, fake, kmax, 0, 0.1, out, None, queue,
                                         size, None)
    assert call(fake, 1023) == sb.STEM_ERR_WORKSPACE
    assert call(fake + 4, 1024) == sb.STEM_ERR_INVALID_ARG
    assert call(fake, 1024, kmax=0) == sb.STEM_ERR_INVALID_ARG and call(None, 0, out=None) == sb.STEM_ERR_INVALID_ARG


# heads, d, B, lengths: KV heads that share the XCDs evenly (8, 4, 1) and not (3, 16), rows that the XCDs of a
# head cannot share equally, several sequences, group-shared lists, a chunk
CASES = [
    dict(hq=32, hkv=8, d=128, B=128, lens=(33100,)),
    dict(hq=28, hkv=4, d=128, B=128, lens=(20000, 901, 16385)),
    dict(hq=20, hkv=1, d=64, B=128, lens=(70001,)),
    dict(hq=24, hkv=3, d=64, B=64, lens=(50001, 77)),
    dict(hq=32, hkv=16, d=256, B=128, lens=(18000,)),
    dict(hq=32, hkv=8, d=128, B=64, lens=(24000,), share="max"),
    dict(hq=32, hkv=8, d=128, B=128, lens=(65536,), chunk=24576),
    dict(hq=28, hkv=4, d=128, B=128, lens=(24000, 12001), keep=1.0),   # lists that grow with the row: a quarter is claimed
]


def make(hq, hkv, d, B, lens, share=None, chunk=0, keep=0.3, seed=3):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(seed)
    cu = [0] + np.cumsum(lens).tolist()
    q, k, v = (torch.randn(cu[-1], h, d, generator=g, device=dev).to(torch.bfloat16) for h in (hq, hkv, hkv))
    pf = StemPrefill(q[chunk:].contiguous(), k, v, cu, B, [keep * -(-n // B) for n in lens], n_sink=2, n_local=2, want_lse=True,
                     group_share=share, chunk=([chunk], [lens[0]]) if chunk else None)
    if chunk:                                          # the earlier keys are not pooled: lists that the budget alone makes
        pf.workspace.zero_()
    pf.estimate()
    pf.select()
    return pf


def check_queue(pf, queue):
    """What a call left in its scratch, a count of claims for each XCD every 128 bytes: each of them went through all the rows
    that its XCD had to claim, and every workgroup that claims has claimed at least once and no queue more than once
    beyond its end."""
    R, Hq, Hkv = pf.rows, pf.q.shape[1], pf.k.shape[1]
    share = 4 if pf.kmax > pf.nbmax // 2 else 8
    if 8 % Hkv == 0:                                   # m XCDs take turns at a KV head's rows
        m = 8 // Hkv
        rows = [len(range(x % m, R, m)) * (Hq // Hkv) for x in range(8)]
    else:                                              # contiguous ranges of all rows
        items = -(-Hq * R // 8)
        rows = [min(items, Hq * R - x * items) for x in range(8)]
    claimed = max(rows) // share
    to_claim = [max(0, r - (max(rows) - claimed)) for r in rows]
    claimers = 8 * (claimed + -(-claimed // 4))
    taken = queue.view(torch.int32)[::32].tolist()
    assert sum(to_claim) > 0 and len(taken) == 8
    assert all(n >= rows for n, rows in zip(taken, to_claim)), (taken, to_claim)
    assert all(n <= rows + claimers for n, rows in zip(taken, to_claim)), (taken, to_claim)
    assert claimers <= sum(taken) <= sum(to_claim) + 8 * claimers


def plain(pf):
    pf.out.fill_(float("nan"))
    sb.stem_sparse_attn(pf.shape, pf.q, pf.k, pf.v, pf.counts, pf.indices, pf.kmax, pf.softmax_scale, pf.out, pf.lse,
                        lists_per_kv_head=bool(pf.group_share))
    torch.cuda.synchronize()
    return pf.out.clone(), pf.lse.clone()


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES)))
def test_claimed_rows_give_the_same_bits(case):
    print("case", CASES[case], flush=True)
    pf = make(**CASES[case])
    assert pf.queue_bytes == 1024                      # the case is one that claims
    out, lse = plain(pf)
    assert not out.isnan().any()
    for fill in (0, 255, 77):                          # what the scratch holds does not matter
        queue = torch.full((1024,), fill, dtype=torch.uint8, device=pf.q.device)
        pf.out.fill_(float("nan"))
        pf.lse.fill_(0.0)
        sb.stem_sparse_attn_queued(pf.shape, pf.q, pf.k, pf.v, pf.counts, pf.indices, pf.kmax, pf.softmax_scale, pf.out,
                                   pf.lse, queue, lists_per_kv_head=bool(pf.group_share))
        torch.cuda.synchronize()
        assert torch.equal(pf.out.view(torch.int16), out.view(torch.int16)) and torch.equal(pf.lse, lse)
        check_queue(pf, queue)


@pytest.mark.gpu
def test_claiming_calls_on_two_streams_and_in_a_graph():
    a, b = make(**CASES[0]), make(**dict(CASES[1], seed=5))
    want = [plain(x) for x in (a, b)]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def check(what):
        for x, (out, lse) in zip((a, b), want):
            assert torch.equal(x.out.view(torch.int16), out.view(torch.int16)) and torch.equal(x.lse, lse), what

    for x in (a, b):
        x.out.fill_(float("nan"))
    torch.cuda.synchronize()
    for _ in range(4):                                 # the same object on both streams as well: each call has its own scratch
        for s, x in zip(streams, (a, b)):
            with torch.cuda.stream(s):
                x.attend()
        with torch.cuda.stream(streams[0]):
            b.attend()
    torch.cuda.synchronize()
    check("streams")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.attend()
        b.attend()
    for turn in range(4):
        for x in (a, b):
            x.out.fill_(float("nan"))
        b.lse.zero_()
        graph.replay()
        torch.cuda.synchronize()
        check("replay %d" % turn)
        a.attend()                                     # eager work between the replays
        torch.cuda.synchronize()
        check("eager %d" % turn)
