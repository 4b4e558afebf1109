"""The draft step of 17 to 32 queries at hidden up to 512, whose queries come as a single slice although the weights are not packed.  The steps,
the oracle and the bounds of test_gpu_tree_decode.py and test_gpu_rope.py; and, on the CPU, that the kernel which asks for one slice is there."""
import pytest

from test_gpu_rope import test_bf16_draft_step_rotates_the_queries as rotated
from test_gpu_tree_decode import test_bf16_tree_step as step
from test_mfma_in_place import library, pytestmark as needs_objdump  # noqa: F401


@pytest.mark.gpu
@pytest.mark.parametrize("M,n_true,T,H,G,D", [(17, 500, 40, 4, 4, 512), (24, 1, 0, 2, 2, 256), (32, 1000, 33, 8, 4, 512), (25, 129, 7, 3, 1, 64)])
def test_step(M, n_true, T, H, G, D):
    step(M, n_true, T, H, G, D)


@pytest.mark.gpu
@pytest.mark.parametrize("M,rows,H,G,D,explicit", [(17, 300, 4, 4, 512, True), (32, 700, 4, 2, 256, False)])
def test_rotated_step(M, rows, H, G, D, explicit):
    rotated(M, rows, H, G, D, explicit)


@needs_objdump
def test_the_kernel_of_one_slice_is_there(library):  # noqa: F811
    assert [n for n in library[1] if "decode_attn_kernelILi1ELi1ELb0EE" in n]
