"""Packed draft steps that rotate their queries, at the depths of the query projection that change its kernel: the launch writes the rotary
table too.  Up to five and up to eight macro-steps of 128 k for each of eight waves with up to 8 rows, up to five with 9 to 16, more
beyond.  The step, the oracle and the bounds of test_gpu_rope.py."""
import pytest

from test_gpu_rope import test_bf16_draft_step_on_packed_weights_rotates_the_queries as step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,rows,H,G,D,explicit", [
    (3, 300, 4, 4, 5120, True),      # five, 8 rows
    (16, 300, 4, 2, 5120, True),     # five, 16 rows
    (5, 200, 4, 4, 6144, True),      # six of eight
    (8, 130, 4, 1, 8192, False),     # eight
    (7, 200, 4, 4, 8320, True),      # one wave with a ninth: the kernel with a ring
    (12, 200, 4, 4, 5248, True),     # one wave with a sixth, past 8 rows: the same
])
def test_rotated_step_at_strip_depths(M, rows, H, G, D, explicit):
    step(M, rows, H, G, D, explicit)
