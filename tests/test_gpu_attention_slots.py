"""Graph attention rows that a wave takes four at a time (groups of four rows and more), beside rows that it takes alone, that a
workgroup shares and that are split: the row lengths and the bar of the other row tests, groups that end inside four."""
import pytest

from test_gpu_attention_rows import test_row_lengths as _row_lengths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,cut,kw", [
    (2, 160, 80, dict(rows_per_group=4)), (2, 161, 97, dict(rows_per_group=5)), (1, 191, 30, dict(rows_per_group=7)),
    (2, 192, 64, dict(rows_per_group=16, long_nnz=16, part_nnz=16)), (2, 193, 100, dict(rows_per_group=6, long_nnz=40, part_nnz=17)),
    (1, 160, 33, dict(rows_per_group=32, long_nnz=64, part_nnz=65)), (2, 163, 3, dict(rows_per_group=3)),
])
def test_slots(T, N, cut, kw):
    _row_lengths(T, N, cut, kw)
