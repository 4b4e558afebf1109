"""Head grouping together with queries that arrive in several k slices (plain weights, hidden above 512), up to the eight that are
requested at once and past them (hidden above 4096), with and without rotary angles, at every way of summing the slices (one, two
and four waves); on exactly the reported workspace.  Against float64 PyTorch on the card."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx
from test_gpu_tree_decode import BF16_OUT_ABS, BF16_OUT_FRO, LSE_TOL

pytestmark = pytest.mark.gpu
HD = 128


def _rotate(x, pos, base=10000.0):
    """x [n, heads, 128] turned by pos * base^(-2c/128) in channel pairs (c, c + 64)."""
    ang = pos.double()[:, None] * base ** (-2.0 * torch.arange(64, device="cuda", dtype=torch.float64) / HD)[None]
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    return torch.cat([x[..., :64] * c - x[..., 64:] * s, x[..., 64:] * c + x[..., :64] * s], -1)


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("M,L,D,H,G", [
    (1, 2500, 1024, 32, 8),      # two slices, four heads of one row
    (1, 4096, 4096, 32, 8),      # eight slices
    (5, 2049, 4096, 32, 8),      # four heads of eight rows, three of them padding
    (8, 1300, 4096, 32, 8),
    (9, 4200, 4096, 32, 8),      # two heads of sixteen rows
    (16, 2600, 1024, 32, 16),
    (4, 3000, 4608, 32, 8),      # nine slices: a second trip
    (12, 2300, 5120, 40, 8),     # ten; five heads per group: alone
    (3, 1700, 5120, 32, 4),
])
def test_grouped_heads_with_sliced_queries(M, L, D, H, G, rope):
    gen = torch.Generator(device="cuda").manual_seed(M + L + D)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    x, kc, vc = r(M, D), r(L, G, HD), r(L, G, HD)
    wq, wo = r(D, H * HD, std=D ** -0.5), r(H * HD, D, std=0.02)
    where = torch.tensor([L + 3 * i for i in range(M)], dtype=torch.int32, device="cuda") if rope else None
    d = bx.make_desc(batch=1, seq_q=M, seq_kv=L, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=HD,
                     flags=bx.BEAGLE_FLAG_ROPE if rope else 0, rope_positions=where)
    y, lse = torch.full((M, D), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.full((H, M), float("nan"), device="cuda")
    n = bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_DRAFT)
    ws = torch.full((n + 4096,), 0xff, dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_draft_step(d, x, kc, vc, wq, wo, y, lse, ws, workspace_bytes=n)
    assert bool((ws[n:] == 0xff).all())

    q = (x.double() @ wq.double()).reshape(M, H, HD)
    if rope:
        q = _rotate(q, where)
    o = []
    for h in range(H):
        s = q[:, h] @ kc[:, h // (H // G)].double().t() / HD ** 0.5
        assert float((lse[h].double() - torch.logsumexp(s, -1)).abs().max()) <= LSE_TOL, h
        o.append(torch.softmax(s, -1) @ vc[:, h // (H // G)].double())
    ref = torch.cat(o, 1) @ wo.double()
    assert float((y.double() - ref).abs().max()) <= BF16_OUT_ABS
    assert float((y.double() - ref).norm() / ref.norm()) <= BF16_OUT_FRO
