"""Which tiles the launches of the float GEMM take (csrc/f32_plan.h, compiled for the host): the wide problems' tiles of 32 rows where
tiles of 16 were up to 8 % slower than what was there before them, those of 16 where they are the faster ones.  And that the GPU tests of
the float kernels reach the launches they are there for."""
import os
import shutil
import subprocess

import pytest

import test_gpu_block_f32_wide as block
import test_gpu_f32_tiles as tiles

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "f32_plan_driver")
    subprocess.run([cxx, "-std=c++17", os.path.join(HERE, "f32_plan_driver.cpp"), "-o", exe], check=True)

    def lines(text):
        return subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout.splitlines()

    def run(*launches):
        out = lines("".join("%d %s\n" % (len(l), " ".join("%d %d %d" % p for p in l)) for l in launches))
        return [dict(rows=int(r), tiles=int(t), ahead=a == "1") for r, t, a in (l.split() for l in out)]
    run.grid = lambda *g: [int(v) for v in lines("0 %d %d %d\n" % g)[0].split()]
    return run


def _chunks(*ks):
    return sum(-(-k // 32) for k in ks)


def step(S, L, D, H, G, hd):
    """The four GEMM launches of a training step."""
    q, k = H * hd, G * hd
    return ([(S, q, _chunks(D)), (L, k, _chunks(D)), (L, k, _chunks(D))],
            [(S, D, _chunks(q))],
            [(S, q, _chunks(D)), (q, D, _chunks(S))],
            [(L, D, _chunks(k, k)), (S, D, _chunks(q)), (D, q, _chunks(S)), (D, k, _chunks(L)), (D, k, _chunks(L))])


@pytest.mark.parametrize("shape,rows", [
    ((128, 128, 256, 4, 4, 64), (16, 16, 16, 16)),                # the reference problem
    ((200, 200, 512, 4, 4, 128), (16, 16, 16, 16)),
    ((16, 16, 4096, 32, 32, 128), (16, 16, 16, 16)),              # one chunk of rows: nothing to share B with
    ((128, 128, 4096, 32, 32, 128), (32, 32, 32, 32)),            # the steps that had become slower
    ((512, 512, 2048, 16, 16, 128), (32, 32, 32, 32)),
    ((1024, 1024, 4096, 32, 32, 128), (32, 32, 32, 32)),
    ((1000, 1000, 5120, 40, 40, 128), (32, 32, 32, 32)),
    ((2048, 2048, 4096, 32, 8, 128), (32, 32, 32, 32)),
])
def test_tiles_of_a_step(plan, shape, rows):
    assert tuple(l["rows"] for l in plan(*step(*shape))) == rows


@pytest.mark.parametrize("queries", [1, 16, 40])
def test_projections_of_a_draft_step_keep_the_narrow_tiles(plan, queries):
    assert [(l["rows"], l["ahead"]) for l in plan([(queries, 4096, 128)], [(queries, 5120, 160)])] == [(16, True)] * 2


def test_the_steps_of_the_gpu_tests_reach_every_kernel(plan):
    got = {s[:6]: plan(*step(*s[:6])) for s in tiles.STEPS}
    assert all(l["ahead"] for l in got[(529, 600, 260, 4, 2, 44)])
    assert all(l["rows"] == 16 and l["tiles"] > 512 and not l["ahead"] for l in got[(700, 333, 772, 12, 2, 60)])
    assert all(l["rows"] == 32 for s in ((777, 600, 1540, 16, 4, 100), (512, 1024, 1024, 16, 16, 64)) for l in got[s])


def test_the_long_step_beside_them(plan):
    """The last row of test_gpu_f32_kernels.py."""
    got = plan(*step(1200, 1200, 2048, 2, 1, 64))
    assert [(l["rows"], l["ahead"]) for l in got] == [(32, False), (16, False), (16, True), (32, False)]


def test_the_wide_block_adds_its_residuals_on_tiles_of_32_rows(plan):
    S, D, q, f = block.S, block.D, block.H * 64, block.FFN
    assert [l["rows"] for l in plan([(S, D, _chunks(q))], [(S, D, _chunks(f))])] == [32, 32]


@pytest.mark.parametrize("rows,n0,n1", [
    (4, 8, 8), (1, 1, 1),
    (32, 1 << 18, 3), (32, (1 << 18) + 7, 1 << 18),               # 2^22 rows of 32 heads: more than one launch of queries
    (1, 1, 1 << 25), (3, (1 << 23) - 1, 5),                       # many keys; a part that ends a block past a launch
    (65535 * 64, 1024, 1),                                        # packed entries, one of them long: more blocks than 32 bits count
])
def test_long_grids_go_in_launches_that_hip_takes(plan, rows, n0, n1):
    """HIP refuses a launch of 2^32 threads and more in a dimension; workgroups have 512."""
    got, at = plan.grid(rows, n0, n1), 0
    for first, blocks, right in zip(got[::3], got[1::3], got[2::3]):
        assert first == at and 0 < blocks * 512 < 1 << 32 and right == 1
        at += blocks
    assert at == rows * (n0 + 2 * n1)
