"""Appending more states than the streaming projections take, whose rows leave the small tiles past L2: one, two and many tiles of each
kind, ragged rows, a head count that leaves a wide tile half empty.  Against float64 on the bf16 inputs; the normalised states and the
rows round once each, 2^-9 of a value: 1e-2 in the norm, as the draft step's bounds have it.  Rows around the new ones stay as they were."""
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,G,D", [(65, 1, 2048), (129, 3, 1152), (300, 8, 4096), (700, 32, 1088), (1013, 5, 2048)])
def test_append_of_a_prompt(n, G, D):
    g = torch.Generator(device="cuda").manual_seed(n)
    R = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    w = dict(wk=R(D, G * 128, std=0.02), wv=R(D, G * 128, std=0.02), g_kv=1 + R(D, std=0.1))
    x, L = R(n, D, std=3.0), n + 40
    d = bx.make_desc(batch=1, seq_q=n, seq_kv=L, hidden=D, n_q_heads=G, n_kv_heads=G, head_dim=128)
    kc, vc = (torch.full((L, G, 128), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    ws = torch.empty(bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_BLOCK_APPEND), dtype=torch.uint8, device="cuda")
    bx.beagle_xattn_block_kv_append(d, bx.make_block_params(256, 1e-5, **w), x, kc, vc, 17, ws)
    torch.cuda.synchronize()
    x64 = x.double()
    x64 = x64 / (x64.square().mean(1, keepdim=True) + 1e-5).sqrt() * w["g_kv"].double()
    for c, m in ((kc, w["wk"]), (vc, w["wv"])):
        assert bool((c[:17] == 7).all()) and bool((c[17 + n:] == 7).all())
        ref = x64 @ m.double()
        assert float((c[17:17 + n].reshape(n, -1).double() - ref).norm() / ref.norm()) <= 1e-2
