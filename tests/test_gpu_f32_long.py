"""Float problems whose grids hold 2^32 threads and more, which go in several launches: rows of a GEMM, queries of the forward, (batch, head)
pairs of the backward.  Against float64; 1e-5 of the largest value, as in test_gpu_f32_kernels.py, and four times that for sums of 32768
terms (sixteen times as many)."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu


def _rand(seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *s: torch.randn(*s, generator=gen, device="cuda")


def _nan(*s):
    return torch.full(s, float("nan"), device="cuda")


def _ws(d, which):
    return torch.empty(max(bx.beagle_xattn_workspace_bytes(d, which), 256), dtype=torch.uint8, device="cuda")


def _close(name, got, ref, tol=1e-5):
    assert float((got.double() - ref).abs().max()) <= tol * float(ref.abs().max()), name


def test_append_of_a_row_block_past_one_launch():
    n = (1 << 27) + 160                                  # 2 x 4194309 tiles of 32 rows
    r = _rand(1)
    x, wk, wv = r(n, 4), r(4, 4), r(4, 4)
    d = bx.make_desc(batch=1, seq_q=n, seq_kv=n, hidden=4, n_q_heads=1, n_kv_heads=1, head_dim=4, io_dtype=bx.BEAGLE_F32)
    k, v = _nan(n, 4), _nan(n, 4)
    bx.beagle_xattn_kv_append(d, x, wk, wv, k, v, 0, _ws(d, bx.BEAGLE_WS_APPEND))
    torch.cuda.synchronize()
    x64 = x.double()
    _close("k", k, x64 @ wk.double())
    _close("v", v, x64 @ wv.double())


def test_forward_of_more_queries_than_one_launch():
    S, L, k = (1 << 27) + 20, 16, 4                      # 2^23 + 2 blocks of queries
    r = _rand(2)
    xq, xkv, wq, wk, wv, wo = r(S, 4), r(L, 4), r(4, 4), r(4, 4), r(4, 4), r(4, 4)
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=L, hidden=4, n_q_heads=1, n_kv_heads=1, head_dim=4, block_size=k, io_dtype=bx.BEAGLE_F32)
    y, lse, q, o, kk, vv = _nan(S, 4), _nan(S), _nan(S, 4), _nan(S, 4), _nan(L, 4), _nan(L, 4)
    bx.beagle_xattn_fwd(d, xq, xkv, wq, wk, wv, wo, y, lse, q, kk, vv, o, _ws(d, bx.BEAGLE_WS_FWD))
    torch.cuda.synchronize()
    assert not bool(torch.isnan(lse).any()) and bool(torch.isfinite(y).all())
    rows = torch.cat([torch.arange(4096), torch.arange(S - 4096, S), torch.randint(0, S, (4096,))]).cuda()
    q64, k64, v64 = xq[rows].double() @ wq.double(), xkv.double() @ wk.double(), xkv.double() @ wv.double()
    see = torch.arange(L, device="cuda")[None] < (rows // k * k)[:, None]
    s = (q64 @ k64.t()) / 2.0
    lse64 = torch.logsumexp(s.masked_fill(~see, float("-inf")), -1)
    p = torch.softmax(s.masked_fill(~see, -1e300), -1) * see
    _close("y", y[rows], (p @ v64) @ wo.double())
    seen = torch.isfinite(lse64)
    assert torch.equal(seen, torch.isfinite(lse[rows]))
    _close("lse", lse[rows][seen], lse64[seen])


def test_backward_of_more_heads_than_one_launch():
    B, S, H, D, k = 2048, 16, 4096, 4, 3                 # 2^23 blocks of queries and as many of keys
    r = _rand(3)
    xq, xkv, dy = r(B, S, D), r(B, S, D), r(B, S, D)
    w = {n: 0.5 * r(D, 4 * H) for n in ("wq", "wk", "wv")}
    w["wo"] = 0.5 * r(4 * H, D)
    d = bx.make_desc(batch=B, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=H, head_dim=4, block_size=k, block_offset=1,
                     io_dtype=bx.BEAGLE_F32, flags=bx.BEAGLE_FLAG_NEED_DXKV)
    y, lse = _nan(B, S, D), _nan(B, H, S)
    q, kk, v, o = (_nan(B, S, H, 4) for _ in range(4))
    bx.beagle_xattn_fwd(d, xq, xkv, w["wq"], w["wk"], w["wv"], w["wo"], y, lse, q, kk, v, o, _ws(d, bx.BEAGLE_WS_FWD))
    g = dict(dxq=_nan(B, S, D), dxkv=_nan(B, S, D), **{"d" + n: torch.full_like(t, float("nan")) for n, t in w.items()})
    bx.beagle_xattn_bwd(d, dy, xq, xkv, w["wq"], w["wk"], w["wv"], w["wo"], q, kk, v, o, lse, g["dxq"], g["dxkv"], g["dwq"],
                        g["dwk"], g["dwv"], g["dwo"], _ws(d, bx.BEAGLE_WS_BWD))
    torch.cuda.synchronize()
    del q, kk, v, o
    p = {n: t.double().requires_grad_() for n, t in dict(w, xq=xq, xkv=xkv).items()}
    pos = torch.arange(S, device="cuda")
    see = pos[None, :] < torch.where(pos < 1, 0, 1 + (pos - 1) // k * k)[:, None]
    for b in range(0, B, 64):
        heads = lambda x, n: (p[x][b:b + 64] @ p[n]).view(64, S, H, 4).transpose(1, 2)
        s = (heads("xq", "wq") @ heads("xkv", "wk").transpose(2, 3)) / 2.0
        out = (torch.softmax(s.masked_fill(~see, -1e300), -1) * see) @ heads("xkv", "wv")
        y64 = out.transpose(1, 2).reshape(64, S, 4 * H) @ p["wo"]
        y64.backward(dy[b:b + 64].double())
        _close("y", y[b:b + 64], y64.detach(), 4e-5)
    for n, t in p.items():
        _close("d" + n, g["d" + n], t.grad, 4e-5)
