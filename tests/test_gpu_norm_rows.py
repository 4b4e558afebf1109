"""The backward of the normalisation at row widths that take each number of register vectors per thread (256 threads of 16 bytes), a
width past them, and more rows than workgroups: the gradients of whole draft blocks against the float64 oracle, within the bounds of
test_gpu_block.py (the bf16 LSE is not among them: its bound there is for scores of 512 channels)."""
import pytest

import test_gpu_block as block
from gpu_harness import rel_fro, run_block
from paper_2505_24544_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [2112, 4160, 6208, 8256])        # 2, 3, 4 vectors, and past them
def test_bf16_widths(hidden):
    cfg = synth.CONFIGS["c2"].with_(seed_base=73, batch=1, seq_q=40, seq_kv=40, hidden=hidden, n_q_heads=1, n_kv_heads=1)
    bi = synth.make_block_inputs(cfg, 64)
    ref = block._oracle(cfg, bi, True)
    _, gr = run_block(cfg, bi, 64, block.RMS_EPS, True)
    for n in block.GRADS + tuple("d" + g for g in block.BLOCK_G):
        assert rel_fro(gr[n], ref[n]) <= block.BF16_GRAD_FRO, (n, rel_fro(gr[n], ref[n]))


@pytest.mark.parametrize("kw", [
    dict(seq_q=24, seq_kv=24, hidden=1028, n_q_heads=2, n_kv_heads=2),
    dict(seq_q=24, seq_kv=24, hidden=2052, n_q_heads=2, n_kv_heads=2),
    dict(seq_q=24, seq_kv=24, hidden=4096, n_q_heads=2, n_kv_heads=2),
    dict(seq_q=24, seq_kv=24, hidden=4100, n_q_heads=2, n_kv_heads=2),
    dict(batch=5, seq_q=517, seq_kv=517, hidden=64, n_q_heads=1, n_kv_heads=1),       # 2585 rows: two and three per workgroup
])
def test_fp32_widths(kw):
    block.test_fp32_block(kw, 64, True)
