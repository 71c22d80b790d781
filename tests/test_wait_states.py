"""The checker of hand-placed wait states: does it flag what it must, and does the attention
kernel's assembly pass it?  (CPU only: hipcc cross-compiles.)"""
import os
import shutil

import pytest

from paper_2603_06274_amd import build, wait_states

HEAD = "_Z1kv:                                  ; @_Z1kv\n"
TAIL = "\ts_endpgm\n.Lfunc_end0:\n"
S_TILE = "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], a[0:3], v[0:15]\n"
ROW_SUM = "\tv_mfma_f32_4x4x4_16b_bf16 v[40:43], v[36:37], v[44:45], v[40:43]\n"
FILLER = "\ts_add_i32 s1, s1, 1\n"


def broken(body):
    return wait_states.check_kernel(HEAD + body + TAIL, "_Z1kv")


def test_vector_read_of_a_matrix_result():
    read = "\tv_mul_f32_e32 v30, v31, v7\n"
    assert broken(S_TILE + FILLER * 11 + read)
    assert not broken(S_TILE + FILLER * 12 + read)
    assert broken(S_TILE + "\ts_nop 10\n" + read)
    assert not broken(S_TILE + "\ts_nop 11\n" + read)
    assert not broken(S_TILE + "\tv_mul_f32_e32 v30, v31, v16\n")      # another register


def test_accumulation_follows_at_once_but_a_shifted_result_does_not():
    assert not broken(S_TILE + S_TILE)
    shifted = "\tv_mfma_f32_32x32x16_bf16 v[8:23], v[24:27], a[0:3], v[8:23]\n"
    assert broken(S_TILE + FILLER * 9 + shifted)
    assert not broken(S_TILE + FILLER * 10 + shifted)
    # results that overlap without a read in between are ordered by the pipe itself
    assert not broken(S_TILE + "\tv_mfma_f32_32x32x16_bf16 v[8:23], v[24:27], a[0:3], 0\n")
    as_operand = "\tv_mfma_f32_32x32x16_bf16 v[48:63], v[0:3], a[0:3], v[48:63]\n"
    assert broken(S_TILE + FILLER * 11 + as_operand)
    assert not broken(S_TILE + FILLER * 12 + as_operand)


def test_accumulator_registers_are_tracked_too():
    o_tile = "\tv_mfma_f32_32x32x16_bf16 a[16:31], v[20:23], v[24:27], a[16:31]\n"
    read = "\tv_accvgpr_read_b32 v1, a17\n"
    assert broken(o_tile + FILLER * 3 + read)
    assert not broken(o_tile + "\ts_nop 15\n" + read)


def test_row_sum_instruction():
    read = "\tv_add_f32_e32 v1, v2, v40\n"
    assert broken(ROW_SUM + FILLER * 4 + read)
    assert not broken(ROW_SUM + FILLER * 5 + read)
    assert broken(ROW_SUM + FILLER + ROW_SUM)
    assert not broken(ROW_SUM + FILLER * 2 + ROW_SUM)


def test_four_pass_instruction():
    row_sum = "\tv_mfma_f32_16x16x32_bf16 v[40:43], v[36:39], v[44:47], v[40:43]\n"
    read = "\tv_add_f32_e32 v1, v2, v40\n"
    assert broken(row_sum + FILLER * 7 + read)
    assert not broken(row_sum + FILLER * 8 + read)
    assert not broken(row_sum + row_sum)
    shifted = "\tv_mfma_f32_16x16x32_bf16 v[42:45], v[36:39], v[48:51], v[42:45]\n"
    assert broken(row_sum + FILLER * 5 + shifted)
    assert not broken(row_sum + FILLER * 6 + shifted)


def test_products_of_the_compiler_keep_the_same_distances():
    """A function with a product in inline assembly beside one that the compiler placed: both are held to 8 and 6."""
    by_hand = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 v[0:3], v[36:39], v[44:47], v[0:3]\n\t;;#ASMEND\n"
    placed = "\tv_mfma_f32_16x16x32_bf16 v[40:43], v[36:39], v[44:47], 0\n"
    for product, at in ((by_hand, 0), (placed, 40)):
        other = by_hand if product is placed else ""
        read = "\tv_cmp_nge_f32_e64 s[8:9], s7, v%d\n" % at
        assert broken(other + product + FILLER * 7 + read)
        assert not broken(other + product + FILLER * 8 + read)
        shifted = "\tv_mfma_f32_16x16x32_bf16 v[%d:%d], v[36:39], v[48:51], v[%d:%d]\n" % (at + 2, at + 5, at + 2, at + 5)
        assert broken(other + product + FILLER * 5 + shifted)
        assert not broken(other + product + FILLER * 6 + shifted)
    # over the branches around a block that is rarely taken, as in the check of a half block
    jump = "\ts_cmp_lg_u32 s1, 0\n\ts_cbranch_scc1 .LBB0_2\n" + FILLER * 9 + ".LBB0_2:\n"
    read = "\tv_cmp_nge_f32_e64 s[8:9], s7, v40\n"
    assert broken(by_hand + placed + jump + FILLER * 5 + read)
    assert not broken(by_hand + placed + jump + FILLER * 6 + read)


def test_matrix_read_after_vector_write():
    write = "\tv_accvgpr_write_b32 a2, v9\n"
    assert broken(write + FILLER + S_TILE)
    assert not broken(write + "\ts_nop 1\n" + S_TILE)
    assert broken("\tv_cvt_pk_bf16_f32 v45, v1, v2\n" + ROW_SUM)
    assert broken("\tv_permlane32_swap_b32_e32 v9, v21\n" + S_TILE)


def test_branch_targets_are_followed():
    read = "\tv_mul_f32_e32 v30, v31, v7\n"
    body = S_TILE + "\ts_cbranch_scc0 .LBB0_2\n" + FILLER * 12 + "\ts_branch .LBB0_3\n.LBB0_2:\n" + read + ".LBB0_3:\n"
    assert broken(body)
    # a second branch on the way
    body = (S_TILE + "\ts_cbranch_scc0 .LBB0_2\n" + FILLER * 12 + "\ts_branch .LBB0_4\n.LBB0_2:\n" + FILLER * 2 +
            "\ts_cbranch_scc1 .LBB0_3\n" + FILLER * 12 + "\ts_branch .LBB0_4\n.LBB0_3:\n" + read + ".LBB0_4:\n")
    assert broken(body)
    # after an unconditional branch nothing falls through
    assert not broken(S_TILE + "\ts_branch .LBB0_3\n.LBB0_2:\n" + read + ".LBB0_3:\n" + FILLER * 12)


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="needs hipcc to produce the kernel's assembly")
def test_attention_kernel_assembly_passes():
    os.makedirs(build.OBJ, exist_ok=True)
    build.check_wait_states()                      # raises with the offending lines
    with open(os.path.join(build.OBJ, "stem_attn.s")) as f:
        asm = f.read()
    hand_placed = [k for k in wait_states.kernels(asm, "sparse_attn_kernel") if "ELi256ELi2E" in k]
    assert len(hand_placed) == 2
    for k in hand_placed:                          # the check did look at hand-placed instructions
        body = asm[asm.index(k + ":"):]
        assert "v_mfma_f32_16x16x32_bf16 a[" in body[:body.index(".Lfunc_end")]


@pytest.mark.parametrize("found", [build.ATTENTION_KERNELS - 1, build.ATTENTION_KERNELS + 1])
def test_an_instantiation_that_is_not_expected_fails_the_build(found, tmp_path, monkeypatch):
    """One that is missing in the assembly was not checked, one too many is not known to be."""
    (tmp_path / "stem_attn.s").write_text("")
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "hipcc", lambda: "true")
    monkeypatch.setattr(wait_states, "kernels", lambda asm, name: ["_Z%d" % x for x in range(found)])
    monkeypatch.setattr(wait_states, "check_kernel", lambda asm, name: [])
    with pytest.raises(RuntimeError, match="found %d" % found):
        build.check_wait_states()


def test_addresses_of_the_largest_buffers_are_immediate_offsets():
    """B = 128, d = 256: 128 KiB of LDS.  A read's address is a base that several reads share and an immediate offset there too,
    as at B = 64; formed anew for every read of a half block it took two vector instructions more, 180 in the loop."""
    build.check_wait_states()
    with open(os.path.join(build.OBJ, "stem_attn.s")) as f:
        asm = f.read()

    def additions(B, tiles):
        name, = [k for k in wait_states.kernels(asm, "sparse_attn_kernel") if "ILi%dELi256ELi%dE" % (B, tiles) in k]
        body = asm[asm.index(name + ":"):]
        body = body[:body.index(".Lfunc_end")]
        return body.count("\tv_add_u32") + body.count("\tv_or_b32")

    for tiles in (1, 2):
        assert additions(128, tiles) <= additions(64, tiles) + 64


def test_every_attention_kernel_has_products_in_inline_assembly():
    """All twelve issue O^T from inline assembly; what the check above accepts has looked at those."""
    build.check_wait_states()
    with open(os.path.join(build.OBJ, "stem_attn.s")) as f:
        asm = f.read()
    names = wait_states.kernels(asm, "sparse_attn_kernel")
    assert len(names) == build.ATTENTION_KERNELS
    for name in names:
        body = asm[asm.index(name + ":"):]
        inside = [part.split("ASMEND")[0] for part in body[:body.index(".Lfunc_end")].split("ASMSTART")[1:]]
        assert sum("v_mfma_f32_16x16x32_bf16" in x for x in inside) >= 16
