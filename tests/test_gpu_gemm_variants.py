"""Every instantiation of the GEMM kernels has a whole step against float32 that runs it: tile size, storage orders of
the operands (nn: X W, nt: X W^T, tn: X^T Y), output type and, where that makes a kernel of its own, a residual; tiles of 128 x 128 over
up to 16 slices of 64 k ("shallow") have a kernel of their own.  Which tiles a launch takes is computed here from the cost rule
that gemm_bf16.hip states, so that the sizes are known to reach what they are listed for."""
import heapq

import pytest
import torch

import test_gpu_gemm_tiles as whole
from paper_2505_24544_amd import binding as bx

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


# ---- with a residual (square tiles: a kernel of their own): y = o Wo + e and h = m W_down + y of the block's forward (nn), and without
# gains its backward's dy = du W_gate^T + dw W_up^T + dh and de = dq Wq^T + dy (nt), the latter in a launch with dK Wk^T + dV Wv^T
RESIDUAL_ON_128 = [(70, 2048, 16), (130, 1088, 9)]             # past 16 slices
RESIDUAL_NT = [(70, 512, 4, 128), (3500, 4096, 2, 128), (4100, 4096, 2, 768)]      # shallow, 256 x 256, and that with rows apart


def _nn(S, D, H):
    return _launches([(S, D, (128 * H,))], False)


def _nt(S, D, F):
    return _launches([(S, D, (F, F))], False)


def test_residuals_reach_what_they_are_listed_for():
    assert [_nn(*s) for s in whole.RESIDUAL] == [["shallow"], [(256, 128)], [(256, 256)], [(128, 256)], [(256, 256), (128, 128)]]
    assert all(_launches([(S, D, (128,))], False) == ["shallow"] for S, D, _ in whole.RESIDUAL)
    assert [_nn(*s) for s in RESIDUAL_ON_128] == [[(128, 128)]] * 2
    assert [_nt(S, D, F) for S, D, _, F in RESIDUAL_NT] == [["shallow"], [(256, 256)], [(256, 256), (128, 128)]]


def test_cut_launches_are_cut():
    """The rows of test_step_against_float32 whose comments say so: a second launch for the last tile rows of one product."""
    assert _launches([(5000, 2048, (3328,)), (5000, 1024, (3328,)), (5000, 1024, (3328,))], False) == [(256, 256), (128, 128)]
    assert _launches([(5000, 3328, (1024, 1024)), (5000, 3328, (2048,))], False) == [(256, 256), (128, 128)]
    assert _launches([(4360, 2560, (3072, 3072)), (4360, 2560, (3072,))], False) == [(256, 256), (128, 256)]
    assert _launches([(2560, 3072, (4360,))] * 3, True) == [(256, 256), (256, 128)]


@pytest.mark.gpu
@pytest.mark.parametrize("S,D,H", RESIDUAL_ON_128)
def test_residual_on_the_variant(S, D, H):
    whole.test_residual_operand(S, D, H)


def _block_reference(t, w, S, H, k):
    """Float32 autograd over Eq. 1 without normalisation; every product is a plain matrix product of contiguous operands."""
    e, hs = t["e"].float().requires_grad_(), t["hs"].float()
    w = {n: x.float() for n, x in w.items()}
    q, kk, v = e @ w["wq"], hs @ w["wk"], hs @ w["wv"]
    pos = torch.arange(S, device="cuda")
    see = pos[None, :] < (pos // k * k)[:, None]
    out = []
    for h in range(H):
        cols = slice(h * whole.HEAD, (h + 1) * whole.HEAD)
        s = (q[:, cols] @ kk[:, cols].t().contiguous()) / whole.HEAD ** 0.5
        out.append(torch.softmax(s.masked_fill(~see, -1e30), -1) * see @ v[:, cols])
    y = torch.cat(out, 1) @ w["wo"] + e
    (torch.nn.functional.silu(y @ w["w_gate"]) * (y @ w["w_up"]) @ w["w_down"] + y).backward(t["dh"].float())
    return e.grad


@pytest.mark.gpu
@pytest.mark.parametrize("S,D,H,F", RESIDUAL_NT)
def test_residual_of_the_input_gradient(S, D, H, F):
    gen = torch.Generator(device="cuda").manual_seed(S + F)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    W, k = H * whole.HEAD, 4
    w = dict(wq=r(D, W, std=0.02), wk=r(D, W, std=0.02), wv=r(D, W, std=0.02), wo=r(W, D, std=0.02), w_gate=r(D, F, std=0.02),
             w_up=r(D, F, std=0.02), w_down=r(F, D, std=0.02))
    t = dict(e=r(S, D), hs=r(S, D), dh=r(S, D))
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=H, head_dim=whole.HEAD, block_size=k,
                     flags=bx.BEAGLE_FLAG_NEED_DXKV)
    nan = lambda *s, dt=torch.bfloat16: torch.full(s, float("nan"), dtype=dt, device="cuda")
    sv = dict(q=nan(S, W), k=nan(S, W), v=nan(S, W), o=nan(S, W), lse=nan(H, S, dt=torch.float32), y=nan(S, D), u=nan(S, F), w=nan(S, F),
              m=nan(S, F))
    g = dict(de=nan(S, D), dhs=nan(S, D), **{"d" + n: nan(*x.shape) for n, x in w.items()})
    ws = lambda which: torch.empty(max(1, bx.beagle_xattn_block_workspace_bytes(d, F, which)), dtype=torch.uint8, device="cuda")
    p, saved = bx.make_block_params(F, 1e-5, **w), bx.make_block_saved(**sv)
    bx.beagle_xattn_block_fwd(d, p, t["e"], t["hs"], nan(S, D), saved, ws(bx.BEAGLE_WS_BLOCK_FWD))
    bx.beagle_xattn_block_bwd(d, p, t["dh"], t["e"], t["hs"], saved, bx.make_block_grads(**g), ws(bx.BEAGLE_WS_BLOCK_BWD))
    # the bound of the other gradients (roundings of 2^-9 between the inputs and here); the last tile rows by themselves too, which a
    # launch of their own may have written
    ref = _block_reference(t, w, S, H, k)
    assert whole.rel(g["de"], ref) <= 3e-2
    assert whole.rel(g["de"][S // 256 * 256:], ref[S // 256 * 256:]) <= 3e-2
