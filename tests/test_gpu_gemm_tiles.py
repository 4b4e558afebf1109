"""The projection GEMMs at sizes that take each of their tile sizes (128 x 128, 128 x 256, 256 x 128, 256 x 256; with every
storage order and output type: test_gpu_gemm_variants.py): a whole
forward + backward against plain float32 PyTorch on the same inputs, rows that end inside a tile, weight gradients over
row counts that end inside a k slice, both output types; and a residual operand on the large and the small tiles."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu
HEAD = 128


def rel(a, ref):
    a, ref = a.float().reshape(-1), ref.float().reshape(-1)
    return float((a - ref).norm() / ref.norm())


def reference(t, S, D, H, G, k):
    """Float32 autograd over the dense mask; every product is a plain matrix product of contiguous operands."""
    p = {n: t[n].float().requires_grad_() for n in ("xq", "xkv", "wq", "wk", "wv", "wo")}
    q, kk, v = p["xq"] @ p["wq"], p["xkv"] @ p["wk"], p["xkv"] @ p["wv"]
    pos = torch.arange(S, device="cuda")
    see = pos[None, :] < (pos // k * k)[:, None]
    out = []
    for h in range(H):
        g = h // (H // G)
        s = (q[:, h * HEAD:(h + 1) * HEAD] @ kk[:, g * HEAD:(g + 1) * HEAD].t().contiguous()) / HEAD ** 0.5
        out.append(torch.softmax(s.masked_fill(~see, -1e30), -1) * see @ v[:, g * HEAD:(g + 1) * HEAD])
    y = torch.cat(out, 1) @ p["wo"]
    y.backward(t["dy"].float())
    return y.detach(), {n: x.grad for n, x in p.items()}


# (rows, D, H, G): tiles taken by [q, k, v] | output | dO | dWo | [dXkv, dXq] | [dWq, dWk, dWv] (s: 128 x 128 by four waves of 64 x 64)
@pytest.mark.parametrize("S,D,H,G,wf32", [
    (60, 256, 2, 1, False),          # s throughout, less than one tile of rows
    (700, 1024, 16, 4, True),        # s | 128 | s | s | 128 | s, ragged rows and k slices
    (1024, 2048, 16, 16, False),     # 256 x 128 | 128 | 128 | s | 128 | 256
    (1300, 1024, 32, 8, True),       # s | 128 | s | 128 | 128 | 256 x 128
    (900, 3072, 24, 12, False),      # 256 x 128 | 128 | 128 | 256 | 256 x 128 | s
    (513, 4096, 8, 2, True),         # 128 | s | 128 | s | s | s
    (4200, 4352, 32, 2, False),      # 128 x 256 | 128 x 256 | 128 x 256 | 256 x 128 | 256 x 128 | 256 x 128, more than a round of each
    (4200, 4352, 32, 2, True),
    (5000, 3328, 16, 8, False),      # forward and input gradients on 256 with the tile rows past whole rounds in a second launch
    (4360, 2560, 24, 24, False),     # the same of input and weight gradients (rows of X cut off) ...
    (4360, 2560, 24, 24, True),      # ... with float output
])
def test_step_against_float32(S, D, H, G, wf32):
    gen = torch.Generator(device="cuda").manual_seed(S + D)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    t = dict(xq=r(S, D, std=0.5), xkv=r(S, D), wq=r(D, H * HEAD, std=0.02), wk=r(D, G * HEAD, std=0.02), wv=r(D, G * HEAD, std=0.02),
             wo=r(H * HEAD, D, std=0.02), dy=r(S, D))
    k = 4
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=HEAD, block_size=k,
                     flags=bx.BEAGLE_FLAG_NEED_DXKV | (bx.BEAGLE_FLAG_WGRAD_F32 if wf32 else 0))
    nan = lambda *s, dt=torch.bfloat16: torch.full(s, float("nan"), dtype=dt, device="cuda")
    wdt = torch.float32 if wf32 else torch.bfloat16
    y, lse, q, kk, v, o = nan(S, D), nan(H, S, dt=torch.float32), nan(S, H * HEAD), nan(S, G * HEAD), nan(S, G * HEAD), nan(S, H * HEAD)
    g = dict(dxq=nan(S, D), dxkv=nan(S, D), dwq=nan(D, H * HEAD, dt=wdt), dwk=nan(D, G * HEAD, dt=wdt), dwv=nan(D, G * HEAD, dt=wdt),
             dwo=nan(H * HEAD, D, dt=wdt))
    ws = lambda which: torch.empty(bx.beagle_xattn_workspace_bytes(d, which), dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_fwd(d, t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], y, lse, q, kk, v, o, ws(bx.BEAGLE_WS_FWD))
    bx.beagle_xattn_bwd(d, t["dy"], t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], q, kk, v, o, lse, g["dxq"], g["dxkv"],
                        g["dwq"], g["dwk"], g["dwv"], g["dwo"], ws(bx.BEAGLE_WS_BWD))
    # one rounding of a float32 sum: at most 2^-8 of an element, 0.72 * 2^-8 / sqrt(3) = 1.6e-3 in the mean square
    assert rel(q, t["xq"].float() @ t["wq"].float()) <= 2.0 ** -9
    assert rel(kk, t["xkv"].float() @ t["wk"].float()) <= 2.0 ** -9
    ref_dwo = o.float().t().contiguous() @ t["dy"].float()
    assert rel(g["dwo"], ref_dwo) <= (1e-5 if wf32 else 2.0 ** -9)
    # the chain: five roundings of 2^-9 between inputs and gradients, as in the other bf16 tests
    yr, gr = reference(t, S, D, H, G, k)
    assert rel(y, yr) <= 1e-2
    for n in ("xq", "xkv", "wq", "wk", "wv", "wo"):
        assert rel(g["d" + n], gr[n]) <= 3e-2, n


# y takes 128 x 128 (s), 256 x 128, 256 x 256, 128 x 256, and 256 x 256 with the last tile rows apart; h always s
RESIDUAL = [(70, 512, 4), (1500, 4096, 32), (2900, 4096, 8), (4200, 4096, 32), (4100, 4096, 12)]


@pytest.mark.parametrize("S,D,H", RESIDUAL)
def test_residual_operand(S, D, H):
    """y = o Wo + e of the block's forward, from its own saved o: the residual is added before the one rounding."""
    gen = torch.Generator(device="cuda").manual_seed(S)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    F, W = 128, H * HEAD
    w = dict(wq=r(D, W, std=0.02), wk=r(D, W, std=0.02), wv=r(D, W, std=0.02), wo=r(W, D, std=0.02), w_gate=r(D, F, std=0.02),
             w_up=r(D, F, std=0.02), w_down=r(F, D, std=0.02))
    d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=H, head_dim=HEAD, block_size=4)
    e, hs = r(S, D), r(S, D)
    nan = lambda *s, dt=torch.bfloat16: torch.full(s, float("nan"), dtype=dt, device="cuda")
    sv = dict(q=nan(S, W), k=nan(S, W), v=nan(S, W), o=nan(S, W), lse=nan(H, S, dt=torch.float32), y=nan(S, D), u=nan(S, F), w=nan(S, F),
              m=nan(S, F))
    h = nan(S, D)
    ws = torch.empty(max(1, bx.beagle_xattn_block_workspace_bytes(d, F, bx.BEAGLE_WS_BLOCK_FWD)), dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_block_fwd(d, bx.make_block_params(F, 1e-5, **w), e, hs, h, bx.make_block_saved(**sv), ws)
    assert rel(sv["y"], sv["o"].float() @ w["wo"].float() + e.float()) <= 2.0 ** -9
    assert rel(h, sv["m"].float() @ w["w_down"].float() + sv["y"].float()) <= 2.0 ** -9
