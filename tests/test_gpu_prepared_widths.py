"""The strip projections around the depths that change their kernel: up to four, five and eight macro-steps of 128 k for each of eight
waves with up to 8 rows, four and five with up to 16, more beyond.  The steps, references and bounds of the two files imported."""
import pytest

import gpu_harness as gh
from test_gpu_block_draft import OUT_FRO, _problem, _ref, _run_prepared
from test_gpu_prepared import test_prepared_step_matches_the_oracle as step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,H,G,D", [
    (1, 32, 8, 1024),            # the whole of four macro-steps, one row; the merge rides in the projection
    (8, 33, 11, 128),            # one wave with a fifth; a single macro-step, one wave's
    (3, 41, 41, 640),            # one wave with a sixth
    (4, 64, 8, 512),             # eight everywhere
    (2, 65, 13, 512),            # one wave with a ninth
    (16, 40, 8, 5120),           # all of LDS: sixteen rows, five macro-steps everywhere
    (9, 41, 41, 640),            # one wave with a sixth, past 8 rows
])
def test_step_at_strip_depths(M, H, G, D):
    step(M, 200, 0, H, G, D)


@pytest.mark.parametrize("M,D,ffn", [(5, 4608, 256), (12, 4608, 5120), (7, 6144, 384)])
def test_block_step_at_strip_depths(M, D, ffn):
    """RMSNorm's row factor, the residuals and the down projection through the same kernels.  Against the oracle alone: next to the plain
    entry point, two independent sets of roundings (6e-3 each at 5120 of feed-forward, by either kernel) are sqrt(2) times that apart.  The LSE's bound is the one of 4096 channels, 4e-3, times the width: a
    score is off by the roundings' 2^-9 of |q| |k|, and both are sums over the width of terms of the same size."""
    cfg, bi, kc, vc = _problem("bf16", M, 150, 4, 2, D, 128, ffn, 241 + M)
    ref = _ref(cfg, bi, kc, vc, True, None, None)
    h, lse, _ = _run_prepared(cfg, bi, kc, vc, ffn, True, None, None)
    assert gh.rel_fro(h, ref["h"]) <= OUT_FRO, gh.rel_fro(h, ref["h"])
    assert gh.max_abs(lse, ref["lse"]) <= 4e-3 * D / 4096, gh.max_abs(lse, ref["lse"])
