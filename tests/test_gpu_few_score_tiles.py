"""Block scores of calls with few 64 x 64 tiles (up to half a tile per CU), which are worked on in quarters: the same bits as in
a call of more heads, which is not."""
import pytest
import torch

from paper_2603_06274_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,S,chunk", [
    (64, 64, 1, False), (64, 128, 4, True), (128, 64, 1, True), (128, 128, 1, False), (128, 64, 2, False),
    (256, 64, 1, True), (256, 64, 16, False),
])
def test_few_tiles_give_the_scores_of_many(d, B, S, chunk):
    blocks = [97, 0, 1, 33, 64, 65]                    # edges of tiles and of their quarters
    lens = [max(0, n * B - (5 if n % 2 else 0)) for n in blocks]
    starts, ends = [(n // 3) * B for n in blocks], lens
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(3)
    Hq, Hkv = 32, 8
    tokens = torch.cat([torch.arange(cu[x] + (starts[x] if chunk else 0), cu[x + 1]) for x in range(len(lens))]).to(dev)
    q = torch.randn(cu[-1], Hq, d, generator=g, device=dev).to(torch.bfloat16)[tokens]
    k, v = (torch.randn(cu[-1], Hkv, d, generator=g, device=dev).to(torch.bfloat16) for _ in range(2))

    def scores(heads, kv_heads):
        qq, kk, vv = q[:, :heads].contiguous(), k[:, :kv_heads].contiguous(), v[:, :kv_heads].contiguous()
        shape = sb.Shape.from_tensors(qq, kk, B, cu, (starts, ends) if chunk else None)
        rows, widest = sb.stem_rows(shape)
        ws = torch.zeros(sb.stem_workspace_bytes(shape, S), dtype=torch.uint8, device=dev)
        if chunk:                                      # the earlier positions' pooled keys
            at = sb.stem_workspace_layout(shape, S)[1]
            full = sb.Shape.from_tensors(torch.zeros(cu[-1], heads, d, dtype=torch.bfloat16, device=dev), kk, B, cu, None)
            ws_full = torch.zeros(sb.stem_workspace_bytes(full, S), dtype=torch.uint8, device=dev)
            sb.stem_pool(full, torch.zeros(cu[-1], heads, d, dtype=torch.bfloat16, device=dev), kk, vv, S, ws_full)
            n = 4 * kv_heads * sum(blocks) * S * d
            at_full = sb.stem_workspace_layout(full, S)[1]
            ws[at:at + n] = ws_full[at_full:at_full + n]
        out = torch.full((heads, rows, widest), 7.0, device=dev)
        sb.stem_estimate(shape, qq, kk, vv, 0.2, 0.5, S, out, ws, False)
        torch.cuda.synchronize()
        return out

    many, few = scores(Hq, Hkv), scores(Hq // Hkv, 1)
    print("d", d, "B", B, "S", S, "chunk", chunk, "rows", many.shape[1], flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    row_tiles = [-(-(n - (s // B if chunk else 0)) // 64) for n, s in zip(blocks, starts)]
    assert 2 * Hq * sum(row_tiles) > cus and not torch.isnan(many).any().item()
    assert torch.equal(few, many[:Hq // Hkv])


@pytest.mark.parametrize("d,B,S,chunk", [
    (64, 64, 1, False), (64, 128, 4, True), (128, 64, 1, True), (128, 128, 1, False), (128, 64, 2, False),
    (256, 64, 1, True), (256, 64, 16, False),
])
def test_the_calls_compared_lie_on_both_sides_of_the_line(d, B, S, chunk):
    """The comparison above says something only if its small call is worked on in quarters, that is has at most half a causal
    64 x 64 tile per CU, and its large one more."""
    tiles = 0
    for n in (97, 0, 1, 33, 64, 65):
        first = n // 3 if chunk else 0                 # block index of the call's first row of the sequence
        for i0 in range(0, n - first, 64):             # a row tile sees the blocks up to its last row's, in the call up to 97
            tiles += -(-min(first + i0 + 64, 97) // 64)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert 2 * 4 * tiles <= cus < 2 * 32 * tiles
