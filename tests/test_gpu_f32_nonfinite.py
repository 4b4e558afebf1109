"""Infinities and NaN in the float path: what the mask hides from a query (or a query from a key) does not reach it, also where
the two share a tile, and a contraction that ends inside a chunk of 32 adds nothing behind its end."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")
S, D, H, G, K, EPS = 150, 64, 4, 2, 5, 2


def _step(t, d, hd):
    e = lambda *s: torch.full(s, NAN, device="cuda")
    ws = lambda which: torch.empty(bx.beagle_xattn_workspace_bytes(d, which), dtype=torch.uint8, device="cuda")
    y, lse, q, k, v, o = e(S, D), e(H, S), e(S, H * hd), e(S, G * hd), e(S, G * hd), e(S, H * hd)
    dxq, dxkv = e(S, D), e(S, D)
    bx.beagle_xattn_fwd(d, t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], y, lse, q, k, v, o, ws(bx.BEAGLE_WS_FWD))
    bx.beagle_xattn_bwd(d, t["dy"], t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], q, k, v, o, lse, dxq, dxkv, e(D, H * hd),
                        e(D, G * hd), e(D, G * hd), e(H * hd, D), ws(bx.BEAGLE_WS_BWD))
    return y, lse, dxq, dxkv


def _close(got, ref):
    assert bool(torch.isfinite(got).all())
    # the rows of a tile are added one by one instead of two at a time: other roundings of the same float sums
    assert float((got - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("hd", [36, 64, 128])
@pytest.mark.parametrize("row", [33, 70, S - 1])       # inside a tile of 32, at the end of the last one
@pytest.mark.parametrize("what,bad", [("xkv", INF), ("xkv", NAN), ("xq", NAN), ("dy", -INF)])
def test_hidden_rows_stay_hidden(hd, row, what, bad):
    gen = torch.Generator(device="cuda").manual_seed(hd + row)
    r = lambda *s, std=1.0: torch.randn(*s, generator=gen, device="cuda") * std
    t = dict(xq=r(S, D), xkv=r(S, D), wq=r(D, H * hd, std=0.1), wk=r(D, G * hd, std=0.1), wv=r(D, G * hd, std=0.1),
             wo=r(H * hd, D, std=0.1), dy=r(S, D))
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=hd, block_size=K, block_offset=EPS,
                     io_dtype=bx.BEAGLE_F32, flags=bx.BEAGLE_FLAG_NEED_DXKV)
    clean = _step(t, d, hd)
    t[what] = t[what].clone()
    t[what][row] = bad
    y, lse, dxq, dxkv = _step(t, d, hd)
    pos = torch.arange(S, device="cuda")
    start = torch.where(pos < EPS, 0, EPS + (pos - EPS) // K * K)           # a query sees the keys below its window's start
    sees = pos[None, :] < start[:, None]
    if what == "xkv":
        mine = ~sees[:, row]                                                # queries that do not see the row
        assert not bool(torch.isfinite(y[~mine]).all(1).any())
        _close(y[mine], clean[0][mine])
        assert torch.equal(lse[:, mine].isfinite(), clean[1][:, mine].isfinite())
        _close(dxq[mine], clean[2][mine])
    else:
        mine = ~sees[row]                                                   # keys that the row does not see
        assert not bool(torch.isfinite(dxkv[~mine]).all(1).any())
        _close(dxkv[mine], clean[3][mine])
        _close(dxq[pos != row], clean[2][pos != row])


def test_contraction_that_ends_inside_a_chunk():
    hd, W = 36, 36
    gen = torch.Generator(device="cuda").manual_seed(1)
    r = lambda *s, std=1.0: torch.randn(*s, generator=gen, device="cuda") * std
    wo = r(W, D)
    wo[W - 1, 5] = INF
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=1, n_kv_heads=1, head_dim=hd, block_size=1, io_dtype=bx.BEAGLE_F32)
    e = lambda *s: torch.full(s, NAN, device="cuda")
    y, o = e(S, D), e(S, W)
    ws = torch.empty(bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_FWD), dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_fwd(d, r(S, D), r(S, D), r(D, W), r(D, W), r(D, W), wo, y, e(1, S), e(S, W), e(S, W), e(S, W), o, ws)
    assert torch.equal(y[1:, 5], torch.sign(o[1:, W - 1]) * INF)
    rest = [c for c in range(D) if c != 5]
    assert bool(torch.isfinite(y[:, rest]).all())
