"""The backward's row sums delta = rowsum(dO * O), as the dQ kernel leaves them in the workspace behind dO, dQ, dK and dV
([B, H, S] floats): one sign on both storage types, since the simulation step's band kernels of both read them there."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io,hd", [(bx.BEAGLE_F32, 64), (bx.BEAGLE_BF16, 128)])
def test_row_sums_in_the_workspace(io, hd):
    S, D, H, G = 130, 256, 4, 2
    dt = torch.float32 if io == bx.BEAGLE_F32 else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).to(dt)
    t = dict(xq=r(S, D), xkv=r(S, D), wq=r(D, H * hd, std=0.06), wk=r(D, G * hd, std=0.06), wv=r(D, G * hd, std=0.06),
             wo=r(H * hd, D, std=0.06))
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=hd, block_size=3, io_dtype=io)
    e = lambda *s, dtype=dt: torch.empty(*s, dtype=dtype, device="cuda")
    y, lse, q, k, v, o = e(S, D), e(H, S, dtype=torch.float32), e(S, H, hd), e(S, G, hd), e(S, G, hd), e(S, H, hd)
    ws = lambda which: torch.empty(bx.beagle_xattn_workspace_bytes(d, which), dtype=torch.uint8, device="cuda")
    w = ws(bx.BEAGLE_WS_BWD)
    bx.beagle_xattn_fwd(d, t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], y, lse, q, k, v, o, ws(bx.BEAGLE_WS_FWD))
    bx.beagle_xattn_bwd(d, r(S, D), t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], q, k, v, o, lse, e(S, D), None,
                        e(D, H * hd), e(D, G * hd), e(D, G * hd), e(H * hd, D), w)
    up = lambda n: (n + 255) // 256 * 256
    esz = y.element_size()
    at = 2 * up(S * H * hd * esz) + 2 * up(S * G * hd * esz)
    delta = w[at:at + 4 * H * S].view(torch.float32).reshape(H, S).double()
    dO = w[:S * H * hd * esz].view(dt).reshape(S, H, hd)
    ref = (dO.double() * o.double()).sum(-1).t()
    assert float(ref.abs().max()) > 0.1
    # hd float products and sums
    assert float((delta - ref).abs().max()) <= hd * 2.0 ** -24 * float((dO.double() * o.double()).abs().sum(-1).max())
