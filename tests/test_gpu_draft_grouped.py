"""The draft step where several query heads of a key/value head share a workgroup: one, two, four and eight heads, query counts at
and between powers of two (padded rows), ranges of one step and more, a short last range, drafted rows under a mask, rotary
angles; next to it shapes where heads stay alone (three per group, more than 32 rows).  Same oracle and tolerances as the plain
step: the grouping changes which workgroup works on a row, not its arithmetic."""
import numpy as np
import pytest

from oracle import beagle_oracle as orc
from paper_2505_24544_amd import binding as bx
from gpu_harness import run_draft_prepared, run_draft_tree, max_abs, rel_fro
from test_gpu_tree_decode import _problem, BF16_OUT_ABS, BF16_OUT_FRO, LSE_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_true,T,H,G", [
    (1, 2500, 0, 32, 8),     # four heads of one row, 20 ranges of one step
    (1, 1500, 0, 32, 8),     # one step less does not pay for the merge's launch: heads alone
    (2, 1500, 33, 32, 8), (3, 4200, 0, 32, 8),
    (5, 2049, 40, 32, 8),    # four heads of eight rows, three of them padding
    (8, 4096, 0, 32, 8), (9, 1300, 31, 32, 8), (16, 2600, 0, 32, 16),
    (4, 1200, 0, 64, 8),     # eight heads
    (17, 1500, 0, 32, 8),    # 34 rows at two heads: alone
    (6, 1500, 20, 24, 8),    # three per group: alone
    (7, 3000, 0, 24, 4),     # six per group: two
])
def test_heads_that_share_a_workgroup(M, n_true, T, H, G):
    rng = np.random.default_rng(M + n_true)
    cfg, inp, kc, vc = _problem("bf16", M, n_true + T, H, G, 128, 128, 4100 + M)
    tm = rng.random((M, T)) < 0.5
    ref = orc.draft_step_tree(inp["xq"][0], kc, vc, inp["wq"], inp["wo"], n_true=n_true, tree_mask=tm, n_q_heads=H, n_kv_heads=G)
    runs = [run_draft_tree(cfg, inp["xq"][0], kc, vc, inp["wq"], inp["wo"], n_true, tm)]
    if M <= 16:
        runs.append(run_draft_prepared(cfg, inp["xq"][0], kc, vc, inp["wq"], inp["wo"], n_true, tm)[:2])
    for y, lse in runs:
        assert np.isfinite(y).all() and np.isfinite(lse).all()
        assert max_abs(y, ref["y"]) <= BF16_OUT_ABS and rel_fro(y, ref["y"]) <= BF16_OUT_FRO, rel_fro(y, ref["y"])
        assert max_abs(lse, ref["lse"]) <= LSE_TOL


def test_rotary_angles_of_padded_rows():
    """Every head's rows take the angles of their own query: equal heads on equal keys give equal rows."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).bfloat16()
    M, L, D, H, G = 5, 2100, 256, 32, 8
    x, kc, vc, wq1, wo = r(M, D), r(L, G, 128), r(L, G, 128), r(D, 128, std=0.06), r(H * 128, D, std=0.02)
    kc[:], vc[:] = kc[:, :1].clone(), vc[:, :1].clone()
    wq = wq1.repeat(1, H).contiguous()
    where = torch.tensor([L + 7 * i * i for i in range(M)], dtype=torch.int32, device="cuda")
    lses = {}
    for heads, groups in ((H, G), (H, H)):                   # grouped, and every head with rows of its own
        d = bx.make_desc(batch=1, seq_q=M, seq_kv=L, hidden=D, n_q_heads=heads, n_kv_heads=groups, head_dim=128,
                         flags=bx.BEAGLE_FLAG_ROPE, rope_positions=where)
        y, lse = torch.empty(M, D, dtype=torch.bfloat16, device="cuda"), torch.empty(heads, M, device="cuda")
        ws = torch.empty(bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_DRAFT), dtype=torch.uint8, device="cuda")
        k, v = (t[:, :1].expand(L, groups, 128).contiguous() for t in (kc, vc))
        bx.beagle_xattn_draft_step(d, x, k, v, wq, wo, y, lse, ws)
        lses[groups] = lse.double().cpu().numpy()
        assert np.array_equal(lses[groups], np.broadcast_to(lses[groups][:1], lses[groups].shape))
    assert np.abs(lses[G] - lses[H]).max() <= 1e-4           # float sums over ranges of other lengths
