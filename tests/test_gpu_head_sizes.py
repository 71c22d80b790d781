"""Head sizes 64 and 256 through the whole path against the oracle (128 is what every other GPU
test runs): the pooling, score and fused kernels take the head size as a parameter, and the attention
kernel is one template over the block size and the head size, instantiated for all six combinations."""
import pytest

from paper_2603_06274_amd import workloads as wl

from test_gpu_parity import run_both

pytestmark = pytest.mark.gpu


def cases(d):
    return {
        # ragged single sequence, GQA 2:1, B = 64
        "ragged_b64": wl.small("ragged_b64_d%d" % d, seed=61, num_q_heads=4, num_kv_heads=2, seq_lens=(1000,),
                               block_size=64, k_start=(6,), n_sink=1, n_local=1, outliers=(2,), head_dim=d),
        # packed batch with an empty and a sub-block sequence, GQA 4:1, B = 128
        "packed_b128": wl.small("packed_b128_d%d" % d, seed=62, num_q_heads=8, num_kv_heads=2,
                                seq_lens=(700, 0, 1536, 130, 50), block_size=128, k_start=(3, 1, 5, 2, 1),
                                n_sink=1, n_local=2, outliers=(1, 0, 2, 1, 1), head_dim=d),
        # more than 64 blocks: several score tiles per row, B = 128, MHA
        "long_b128": wl.small("long_b128_d%d" % d, seed=63, num_q_heads=2, num_kv_heads=2, seq_lens=(9000,),
                              block_size=128, k_start=(12,), n_sink=2, n_local=2, outliers=(6,), head_dim=d),
        # a start budget of zero: every row keeps exactly its forced windows
        "forced_only_b64": wl.small("forced_only_b64_d%d" % d, seed=64, num_q_heads=2, num_kv_heads=1,
                                    seq_lens=(2000, 300), block_size=64, k_start=(0, 0), n_sink=2, n_local=3,
                                    outliers=(1, 1), head_dim=d),
    }


@pytest.mark.parametrize("name", ["ragged_b64", "packed_b128", "long_b128", "forced_only_b64"])
@pytest.mark.parametrize("d", [64, 256])
def test_head_size_whole_path(d, name):
    run_both(cases(d)[name])


@pytest.mark.parametrize("d,ad_stride", [(64, 1), (256, 2)])
def test_head_size_fused_above_1024_blocks(d, ad_stride):
    """The fused stage 1-2 with more than 1024 key blocks per row (128 KiB bands) at the other head
    sizes: dumped scores and lists against the oracle."""
    import torch
    import parity_util as pu
    w = wl.small("many_blocks_d%d" % d, seed=65, num_q_heads=2, num_kv_heads=1, seq_lens=(1100 * 64 + 5,),
                 block_size=64, k_start=(30,), n_sink=2, n_local=2, outliers=(8,), head_dim=d)
    data = wl.generate(w)
    qkv = pu.host_arrays(data)
    pf = pu.device_prefill(w, data, ad_stride=ad_stride)
    assert pf.nbmax > 1024
    dump = torch.full_like(pf.scores, float("nan"))
    pf.estimate_select(dump)
    torch.cuda.synchronize()
    scores = pu.oracle_estimate(w, qkv, ad_stride)[3]
    pu.check_scores(dump.cpu().numpy(), scores)
    _, counts, indices = pu.oracle_select(w, scores)
    same = pu.check_lists(w, pf.counts.cpu().numpy(), pf.indices.cpu().numpy(), counts, indices, scores, print)
    assert same.mean() > 0.99


@pytest.mark.parametrize("blocks,chunk_blocks", [(1024, 0), (1025, 0), (2048, 40), (2049, 41), (4096, 23)])
def test_fused_band_shapes_at_their_edges(blocks, chunk_blocks):
    """The three band shapes of the fused stage 1-2 at the first and last number of key blocks each
    serves, next to a short sequence (bands of one row): the dumped scores against the unfused score
    kernel's, the lists against the unfused selection on the dumped scores, which must be identical."""
    import torch
    import parity_util as pu
    w = wl.small("bands_%d" % blocks, seed=66, num_q_heads=2, num_kv_heads=1, seq_lens=(blocks * 64 - 3, 70),
                 block_size=64, k_start=(30, 2), n_sink=2, n_local=2, outliers=(8, 1), head_dim=64)
    data = wl.generate(w)
    dev = torch.device("cuda:0")
    q, k, v = (data[x].to(dev) for x in "qkv")
    ws = chunk = None
    args = (w.cu_seqlens, w.block_size, w.k_start_blocks, w.mu, w.k_min, w.n_sink, w.n_local)
    if chunk_blocks:                                   # the last rows only, as in chunked prefill
        n = blocks * 64 - 3
        start = (blocks - chunk_blocks) * 64
        earlier = pu.StemPrefill(torch.cat([q[:start], q[n:n + 64]]), k, v, *args, chunk=([0, 0], [start, 64]))
        q = torch.cat([q[start:n], q[n + 64:]])
        chunk = ([start, 64], [n, 70])
        pf = pu.StemPrefill(q, k, v, *args, chunk=chunk, fill_scores=True)
        ws = torch.empty(max(earlier.workspace.numel(), pf.workspace.numel()), dtype=torch.uint8, device=dev)
        earlier.workspace = pf.workspace = ws
        earlier.pool()
    else:
        pf = pu.StemPrefill(q, k, v, *args, fill_scores=True)
    assert pf.nbmax == blocks
    dump = torch.full_like(pf.scores, float("nan"))
    pf.estimate_select(dump)
    counts, indices = pf.counts.clone(), pf.indices.clone()
    pf.estimate()
    torch.cuda.synchronize()
    assert torch.equal(torch.isinf(dump), torch.isinf(pf.scores))
    seen = ~torch.isinf(dump)
    # both sum 64 products in fp32, in another order: 64 roundings of 2^-24 of the largest partial sum
    bound = 64 * 2.0 ** -24 * float(pf.scores[seen].abs().max()) * 2
    assert float((dump[seen] - pf.scores[seen]).abs().max()) <= bound
    pf.scores.copy_(dump)
    pf.select()
    torch.cuda.synchronize()
    assert torch.equal(counts, pf.counts) and torch.equal(indices, pf.indices)


@pytest.mark.parametrize("d", [64, 128, 256])
def test_several_rounds_of_long_lists(d):
    """B = 64, enough rows for several rounds of workgroups on each XCD and lists of more than the 64
    entries a wave holds at a time, against the oracle."""
    w = wl.small("rounds_d%d" % d, seed=67, num_q_heads=8, num_kv_heads=1, seq_lens=(600 * 64 - 5,),
                 block_size=64, k_start=(90,), n_sink=2, n_local=2, outliers=(20,), head_dim=d)
    run_both(w, rows=range(3, 600, 17), heads=[0, 5])
