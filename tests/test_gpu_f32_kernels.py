"""The float path where its kernels can go wrong: contractions and head widths that end inside a 32-wide chunk, rows and
columns that end inside a tile, one and many chunks per wave, all GEMM tile sizes.  Against float64 PyTorch on the card;
1e-5 of the largest value, the float path's bound (sums of up to 2048 terms: sqrt(n) 6e-8, through five of them)."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,L,D,H,G,hd,k,eps", [
    (1, 1, 4, 1, 1, 4, 1, 0),                  # smallest of everything
    (33, 33, 36, 3, 1, 12, 2, 1),              # one past a tile; chunk of 32 plus 4; head width inside a block
    (129, 129, 68, 2, 2, 36, 5, 3),            # second 32-channel block of four channels
    (140, 140, 96, 2, 1, 72, 4, 1),            # three blocks, the last of eight channels
    (97, 200, 64, 2, 2, 96, 4, 0),             # three whole blocks
    (200, 200, 256, 4, 2, 100, 4, 2),          # four blocks, the last of four channels
    (150, 97, 128, 2, 1, 128, 3, 0),           # more queries than keys
    (97, 290, 96, 2, 2, 64, 8, 7),             # more keys than queries, three key blocks per wave
    (1200, 1200, 2048, 2, 1, 64, 4, 0),        # 32 x 64 GEMM tiles, but for dO, dWo (16 x 64)
])
def test_step_against_float64(S, L, D, H, G, hd, k, eps):
    gen = torch.Generator(device="cuda").manual_seed(S + D)
    r = lambda *s, std=1.0: torch.randn(*s, generator=gen, device="cuda") * std
    t = dict(xq=r(S, D), xkv=r(L, D), wq=r(D, H * hd, std=0.05), wk=r(D, G * hd, std=0.05), wv=r(D, G * hd, std=0.05),
             wo=r(H * hd, D, std=0.05), dy=r(S, D))
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=L, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=hd, block_size=k, block_offset=eps,
                     io_dtype=bx.BEAGLE_F32, flags=bx.BEAGLE_FLAG_NEED_DXKV)
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    y, lse, q, kk, v, o = nan(S, D), nan(H, S), nan(S, H * hd), nan(L, G * hd), nan(L, G * hd), nan(S, H * hd)
    g = dict(dxq=nan(S, D), dxkv=nan(L, D), dwq=nan(D, H * hd), dwk=nan(D, G * hd), dwv=nan(D, G * hd), dwo=nan(H * hd, D))
    ws = lambda which: torch.empty(bx.beagle_xattn_workspace_bytes(d, which), dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_fwd(d, t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], y, lse, q, kk, v, o, ws(bx.BEAGLE_WS_FWD))
    bx.beagle_xattn_bwd(d, t["dy"], t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], q, kk, v, o, lse, g["dxq"], g["dxkv"],
                        g["dwq"], g["dwk"], g["dwv"], g["dwo"], ws(bx.BEAGLE_WS_BWD))

    p = {n: t[n].double().requires_grad_() for n in ("xq", "xkv", "wq", "wk", "wv", "wo")}
    q64, k64, v64 = p["xq"] @ p["wq"], p["xkv"] @ p["wk"], p["xkv"] @ p["wv"]
    pos = torch.arange(S, device="cuda")
    see = torch.arange(L, device="cuda")[None, :] < torch.where(pos < eps, 0, eps + (pos - eps) // k * k)[:, None]
    out, ls = [], []
    for h in range(H):
        gi = h // (H // G)
        s = (q64[:, h * hd:(h + 1) * hd] @ k64[:, gi * hd:(gi + 1) * hd].t()) / hd ** 0.5
        ls.append(torch.logsumexp(s.masked_fill(~see, float("-inf")), -1))
        out.append((torch.softmax(s.masked_fill(~see, -1e300), -1) * see) @ v64[:, gi * hd:(gi + 1) * hd])
    y64 = torch.cat(out, 1) @ p["wo"]
    y64.backward(t["dy"].double())
    lse64 = torch.stack(ls).detach()
    seen = torch.isfinite(lse64)
    assert torch.equal(seen, torch.isfinite(lse))

    def close(name, got, ref):
        big = float(ref.abs().max()) if ref.numel() else 0.0
        assert float((got.double() - ref).abs().max()) <= 1e-5 * max(big, 1e-30), name
    close("y", y, y64.detach())
    close("lse", lse[seen], lse64[seen]) if bool(seen.any()) else None
    for n, x in p.items():
        close("d" + n, g["d" + n], x.grad)
