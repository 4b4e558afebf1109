"""The draft block in float at a width whose output and down projections take tiles of 32 rows, which add the residual: the block, the oracle
and the bounds of test_gpu_block.py."""
import pytest

from test_gpu_block import test_fp32_block as block

pytestmark = pytest.mark.gpu
S, D, H, FFN = 550, 1540, 16, 1348


def test_wide_block():
    block(dict(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=4, block_size=8), FFN, True)
