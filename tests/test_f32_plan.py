"""Which tiles the launches of the float GEMM take (csrc/f32_plan.h, compiled for the host): 32 rows for the wide problems and 32 columns for
a few rows, where tiles of 16 x 64 were up to 8 and 10 % slower than what was there before them.  And that the GPU tests of the float
kernels reach the launches they are there for."""
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
        return [dict(tile=(int(r), int(c)), tiles=int(t), ahead=a == "1", alone=o == "1") for r, c, t, a, o in (l.split() for l in out)]
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


def kinds(launches):
    """n: 16 x 32; a, p: 16 x 64, a chunk ahead or workgroups in pairs; w, v: 32 x 64, alone on a CU or in pairs"""
    return "".join("n" if l["tile"] == (16, 32) else ("a" if l["ahead"] else "p") if l["tile"] == (16, 64) else
                   {(32, 64): "w" if l["alone"] else "v"}[l["tile"]] for l in launches)


@pytest.mark.parametrize("shape,want", [
    ((128, 128, 256, 4, 4, 64), "nnna"),                          # the reference problem
    ((200, 200, 512, 4, 4, 128), "anap"),
    ((16, 16, 4096, 32, 32, 128), "anvv"),                        # one chunk of rows
    ((128, 128, 4096, 32, 32, 128), "wwvv"),                      # the steps that had become slower
    ((512, 512, 2048, 16, 16, 128), "wwww"),
    ((1024, 1024, 4096, 32, 32, 128), "wwww"),
    ((1000, 1000, 5120, 40, 40, 128), "wwww"),
    ((2048, 2048, 4096, 32, 8, 128), "wwww"),
])
def test_tiles_of_a_step(plan, shape, want):
    assert kinds(plan(*step(*shape))) == want


@pytest.mark.parametrize("rows,D,want", [(1, 4096, "n"), (16, 5120, "n"), (16, 8192, "n"), (32, 4096, "n"), (40, 4096, "a"), (16, 8256, "a")])
def test_projections_of_a_few_rows(plan, rows, D, want):
    assert kinds(plan([(rows, D, _chunks(D))])) == want


def test_the_steps_of_the_gpu_tests_reach_every_kernel(plan):
    got = {s[:6]: kinds(plan(*step(*s[:6]))) for s in tiles.STEPS}
    assert got[(17, 129, 64, 2, 2, 64)] == "nnnn" and got[(45, 97, 1028, 20, 5, 52)] == "nnpp"
    assert got[(529, 600, 260, 4, 2, 44)] == "aaaa"
    assert got[(600, 300, 900, 12, 2, 60)] == "pppp"
    assert got[(777, 600, 1540, 16, 4, 100)] == got[(512, 1024, 1024, 16, 16, 64)] == "wwww"
    assert got[(130, 140, 1540, 16, 4, 100)] == "wapv"
    assert kinds(plan(*step(1200, 1200, 2048, 2, 1, 64))) == "wvav"        # the last row of test_gpu_f32_kernels.py


def test_the_wide_block_adds_its_residuals_on_tiles_of_32_rows(plan):
    S, D, q, f = block.S, block.D, block.H * 64, block.FFN
    assert kinds(plan([(S, D, _chunks(q))], [(S, D, _chunks(f))])) == "ww"


def test_the_long_append_is_more_than_one_launch(plan):
    n = (1 << 27) + 160
    assert plan([(n, 4, 1), (n, 4, 1)])[0]["tiles"] * 512 >= 1 << 32


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
