"""Rows that the small calls of other tests cover with 16 queries per wave, once more in launches with 32: list entries that
cannot be used, empty lists, the diagonal block anywhere, a softmax reference that moves or is not there yet, rows that are not
finite.  Their heads are repeated until the launch is above the line, and every copy has the bits of the small call."""
import pytest

import parity_util as pu
import test_gpu_diagonal_block as diagonal
import test_gpu_non_finite as non_finite
import test_gpu_parity as parity

pytestmark = pytest.mark.gpu

SIZES = [(128, 128), (64, 128), (128, 64), (64, 64), (128, 256), (64, 256)]


@pytest.fixture(autouse=True)
def wide(monkeypatch):
    pu.widen_attention(monkeypatch)


@pytest.mark.parametrize("place", sorted(diagonal.PLACES))
@pytest.mark.parametrize("B,d", SIZES)
def test_diagonal_block(B, d, place):
    diagonal.test_diagonal_block_wherever_it_stands(B, d, place)


@pytest.mark.parametrize("B,d", SIZES)
def test_diagonal_block_alone(B, d):
    diagonal.test_row_of_the_diagonal_block_alone(B, d)


@pytest.mark.parametrize("B,d", SIZES)
def test_rows_without_a_usable_entry(B, d):
    parity.test_rows_without_a_usable_entry_give_zeros_and_minus_infinity(B, d)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("B,d", SIZES)
def test_reference_moves_and_unusable_entries(B, d, sign):
    parity.test_attention_reference_moves_and_unusable_entries(B, d, sign)


@pytest.mark.parametrize("moving", [False, True])
@pytest.mark.parametrize("bad", non_finite.BAD)
@pytest.mark.parametrize("B,d", SIZES)
def test_non_finite_rows(B, d, bad, moving):
    non_finite.test_non_finite_rows_reach_only_what_attends_to_them(B, d, bad, moving)
