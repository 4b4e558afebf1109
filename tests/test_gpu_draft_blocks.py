"""The draft step around the block of 16 rows its attention works at a time: 8 queries (one wave sums q) and 9, 15, 16 (two), key counts
of one row, one past a step and one past a wave's share of it, drafted rows that begin and end inside a 16-key block.  The step, the
oracle and the bounds of test_gpu_prepared.py, which compares the plain entry point as well."""
import pytest

from test_gpu_prepared import test_prepared_step_matches_the_oracle as step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_true,T,H,G", [
    (1, 1, 0, 4, 4), (8, 31, 9, 4, 4), (9, 1, 0, 4, 2), (15, 129, 0, 4, 4), (16, 85, 40, 4, 4), (16, 257, 5, 2, 2), (7, 161, 64, 4, 1),
    (16, 0, 33, 4, 2), (2, 4100, 37, 32, 8), (4, 2000, 21, 32, 8),     # grouped: eight and sixteen rows of several heads
])
def test_step_around_a_block_of_rows(M, n_true, T, H, G):
    step(M, n_true, T, H, G, 512)
