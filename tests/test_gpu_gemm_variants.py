"""Every instantiation of the GEMM kernels has a whole step against float32 that runs it: tile size, storage orders of
the operands (nn: X W, nt: X W^T, tn: X^T Y) and output type; tiles of 128 x 128 over up to 16 slices of 64 k ("shallow") have a
kernel of their own.  Which tiles a launch takes is computed here from the cost rule
that gemm_bf16.hip states, so that the sizes are known to reach what they are listed for."""
import heapq

import pytest

import test_gpu_gemm_tiles as whole

# (BM, BN, workgroups of a round, us per round, us per slice of 64 k, and the share of it that grows with how full the round is)
COSTS = ((256, 256, 256, 7.0, 0.91, 0.46), (256, 128, 256, 6.7, 0.45, 0.38), (128, 256, 256, 6.7, 0.45, 0.38),
         (128, 128, 256, 5.9, 0.29, 0.21), (128, 128, 512, 2.7, 0.285, 0.66))
CUT_US = 8.0
SHALLOW = 16
up = lambda a, b: -(-a // b)


def _uneven(at_once, fixed, each, fuller, tiles, depths):
    """Makespan of tiles of different depth, dealt out in order to whichever place is free first."""
    fill = min(1.0, sum(tiles) / at_once)
    free = [0.0] * at_once
    end = 0.0
    for t, d in zip(tiles, depths):
        for _ in range(t):
            at = heapq.heappop(free) + fixed + d * (each + fuller * fill)
            heapq.heappush(free, at)
            end = max(end, at)
    return end


def _choose(group):
    """group: (M, N, depths of the k segments) of every product of the launch -> ((BM, BN) or "shallow", microseconds)."""
    best = None
    for bm, bn, at_once, fixed, each, fuller in COSTS:
        tiles = [up(m, bm) * up(n, bn) for m, n, _ in group]
        depth = sum(t * sum(up(k, 64) for k in ks) for t, (_, _, ks) in zip(tiles, group)) / sum(tiles)
        if at_once == 512 and depth > SHALLOW:
            continue
        full, rest = divmod(sum(tiles) / at_once, 1.0)
        us = full * (fixed + depth * (each + fuller)) + (fixed + depth * (each + fuller * rest) if rest else 0.0)
        depths = [sum(up(k, 64) for k in ks) for _, _, ks in group]
        if len(set(depths)) > 1 and sum(tiles) <= 4096:
            us = _uneven(at_once, fixed, each, fuller, tiles, depths)
        if best is None or us < best[1]:
            best = ("shallow" if at_once == 512 else (bm, bn), us)
    return best


def _launches(group, rows_contiguous):
    """Tile sizes of the one or two launches that a group becomes."""
    tile, us = _choose(group)
    total = sum(up(m, 256) * up(n, 256) for m, n, _ in group)
    excess = total % 256
    if tile != (256, 256) or total < 256 or excess == 0 or excess > 128:
        return [tile]
    best, found = us - CUT_US, [tile]
    for i, (m, n, ks) in enumerate(group):
        rows, r = up(m, 256), up(excess, up(n, 256))
        if r >= rows or (rows_contiguous and m % 256):
            continue
        kept = (rows - r) * 256
        a, b = _choose(group[:i] + [(kept, n, ks)] + group[i + 1:]), _choose([(m - kept, n, ks)])
        if a[1] + b[1] < best:
            best, found = a[1] + b[1], [a[0], b[0]]
    return found


def _variants(S, D, H, G, wf32):
    """{(tile, orders, output type)} of a step's launches (dWk, dWv not in halves at these sizes)."""
    W, V = 128 * H, 128 * G
    assert up(D, 256) * (up(W, 256) + 2 * up(V, 256)) < 256
    nn, nt = [[(S, W, (D,)), (S, V, (D,)), (S, V, (D,))], [(S, D, (W,))]], [[(S, W, (D,))], [(S, D, (V, V)), (S, D, (W,))]]
    tn = [[(W, D, (S,))], [(D, W, (S,)), (D, V, (S,)), (D, V, (S,))]]
    out = set()
    for orders, groups in (("nn", nn), ("nt", nt), ("tn", tn)):
        for g in groups:
            out |= {(t, orders, "f32" if orders == "tn" and wf32 else "bf16") for t in _launches(g, orders == "tn")}
    return out


SHAPES = [
    (200, 1408, 8, 8, False),      # odd multiples of 128 channels: shallow weight gradients ...
    (200, 1408, 8, 8, True),       # ... in both output types
    (200, 2176, 16, 16, False),
    (200, 2560, 13, 1, True),
    (1152, 2688, 24, 8, False),    # an odd multiple of 128 rows: forward projections and input gradients on 128 x 256
    (700, 3072, 8, 4, False),
    (1024, 2048, 15, 15, False),   # forward projections on 256 x 128
    (60, 256, 2, 1, False),        # all shallow: less than a tile of rows
    (1030, 1024, 8, 2, False),     # shallow forward and dO, weight gradients over 17 slices: just past it
    (1030, 1024, 8, 2, True),
    (1030, 320, 29, 29, False),    # dWo on 128 x 256
    (1030, 320, 30, 30, True),
    (900, 2112, 6, 6, False),      # input gradients on 256 x 128
    (1030, 448, 23, 23, True),     # dWq, dWk, dWv on 256 x 128
    (1600, 256, 24, 24, False),    # 256 x 256 of few steps: forward projections ...
    (1600, 320, 24, 24, False),    # ... and dO, whose steps end inside a period of four
    (1030, 3776, 3, 1, False),     # input gradients on 256 x 256, two segments of 128
    (200, 1984, 19, 19, False),    # weight gradients on 256 x 256, an odd number of steps ...
    (200, 1984, 19, 19, True),     # ... in both output types
]


def test_shapes_reach_every_variant():
    tiles = [(bm, bn) for bm, bn, *_ in COSTS[:4]] + ["shallow"]
    want = {(tile, o, t) for tile in tiles for o, t in (("nn", "bf16"), ("nt", "bf16"), ("tn", "bf16"), ("tn", "f32"))}
    assert want <= set().union(*(_variants(*s) for s in SHAPES)), want - set().union(*(_variants(*s) for s in SHAPES))


@pytest.mark.gpu
@pytest.mark.parametrize("S,D,H,G,wf32", SHAPES)
def test_step_on_the_variant(S, D, H, G, wf32):
    whole.test_step_against_float32(S, D, H, G, wf32)


@pytest.mark.gpu
@pytest.mark.parametrize("S,D,H", [(70, 2048, 16), (130, 1088, 9)])       # past 16 slices on tiles of 128 x 128: with a residual
def test_residual_on_the_variant(S, D, H):
    whole.test_residual_operand(S, D, H)
