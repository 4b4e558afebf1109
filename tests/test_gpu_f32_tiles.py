"""The float kernels around the edges of their tiles: 16 queries or keys, 128 keys to a round of eight waves, 16 x 32,
16 x 64 or 32 x 64 of a GEMM, 256 of a contraction to a round, 512 tiles to the launches that request ahead.  The step, the reference and the bound
of test_gpu_f32_kernels.py; test_f32_plan.py says on the CPU which GEMM kernel each launch of a row takes."""
import pytest

from test_gpu_f32_kernels import test_step_against_float64 as step

pytestmark = pytest.mark.gpu


STEPS = [
    (15, 17, 20, 2, 1, 20, 3, 1),              # a row less, a key more than a tile; one chunk of 20
    (16, 16, 64, 1, 1, 32, 1, 0),              # whole tiles of one wave
    (17, 129, 64, 2, 2, 64, 2, 1),             # one key past a round
    (128, 128, 256, 4, 4, 64, 4, 0),           # the reference problem
    (145, 272, 548, 4, 2, 68, 4, 3),           # three rounds of the contraction, the last of four; four channels in the third block
    (529, 600, 260, 4, 2, 44, 8, 5),           # up to 479 tiles in a launch, the last ones ending inside, in rows and columns
    (600, 300, 900, 12, 2, 60, 8, 3),          # every launch past 512 tiles of 16 rows: rows, columns and chunks end inside, both segments
    (45, 97, 1028, 20, 5, 52, 4, 2),           # 16 x 32: 225 and 99 tiles, 16 and 4 columns in the last; deep ones of 32 chunks and a ragged one
    (130, 140, 1540, 16, 4, 100, 4, 1),        # 32 rows alone on a CU, 16 ahead and in pairs, 32 in pairs: 2 and 12 rows in the last
    (777, 600, 1540, 16, 4, 100, 4, 1),        # every launch on tiles of 32 rows alone on a CU: 9 and 24 rows in the last, 4 and 16 columns, chunks of 4 - 28
    (512, 1024, 1024, 16, 16, 64, 16, 0),      # the same, whole everywhere
]


@pytest.mark.parametrize("S,L,D,H,G,hd,k,eps", STEPS)
def test_step_at_tile_edges(S, L, D, H, G, hd, k, eps):
    step(S, L, D, H, G, hd, k, eps)
