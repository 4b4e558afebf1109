"""The backward on less workspace than reported: from what its tensors need (key tiles whole) over a part of the shares to all of
them, with half-precision states behind the tensors, and nothing written past the bytes that were given."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu
up = lambda n: (n + 255) // 256 * 256


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("S,H,G", [(450, 8, 1), (600, 16, 2)])
def test_backward_on_less_workspace(S, H, G, f16):
    D, W, V = 256, H * 128, G * 128
    gen = torch.Generator(device="cuda").manual_seed(S)
    r = lambda *s, std=1.0: torch.randn(*s, generator=gen, device="cuda") * std
    b = lambda *s, std=1.0: r(*s, std=std).bfloat16()
    xkv = r(S, D).half() if f16 else b(S, D)
    t = dict(xq=b(S, D), wq=b(D, W, std=0.06), wk=b(D, V, std=0.06), wv=b(D, V, std=0.06), wo=b(W, D, std=0.06), dy=b(S, D))
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=128, block_size=4,
                     flags=bx.BEAGLE_FLAG_NEED_DXKV | (bx.BEAGLE_FLAG_STATES_F16 if f16 else 0))
    e = lambda *s, dt=torch.bfloat16: torch.empty(*s, dtype=dt, device="cuda")
    y, lse, q, k, v, o = e(S, D), e(H, S, dt=torch.float32), e(S, W), e(S, V), e(S, V), e(S, W)
    fw = torch.empty(bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_FWD), dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_fwd(d, t["xq"], xkv, t["wq"], t["wk"], t["wv"], t["wo"], y, lse, q, k, v, o, fw)
    reported = bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_BWD)
    need = 2 * up(S * W * 2) + 2 * up(S * V * 2) + 2 * up(H * S * 4) + (up(S * D * 2) if f16 else 0)
    share = (S + 127) // 128 * G * 2 * 128 * 128 * 4             # one chunk of every key tile
    assert reported >= need + 3 * share
    runs = []
    for n in (need, need + 2 * share - 1, need + 2 * share, need + 3 * share + 256, reported):
        ws = torch.full((n + 4096,), 0xff, dtype=torch.uint8, device="cuda")      # NaN: a share that nobody wrote would show
        g = [e(S, D), e(S, D), e(D, W), e(D, V), e(D, V), e(W, D)]
        bx.beagle_xattn_bwd(d, t["dy"], t["xq"], xkv, t["wq"], t["wk"], t["wv"], t["wo"], q, k, v, o, lse, *g, ws, workspace_bytes=n)
        assert bool((ws[n:] == 0xff).all()), n
        runs.append([x.float() for x in g])
    assert all(torch.equal(x, y) for x, y in zip(runs[0], runs[1]))               # no room for two chunks: tiles whole
    assert not torch.equal(runs[0][1], runs[2][1])                                # two chunks: other order of the same sums
    for run in runs[1:]:
        for x, ref in zip(run, runs[0]):
            # other roundings of dK, dV, and of what is formed from them: 2^-9 each
            assert float((x - ref).norm()) <= 2.0 ** -8 * float(ref.norm())
