"""Rotary embedding of projected rows against the rows the same call leaves without it, rotated in float64: head counts below,
at and above what one pass of the streaming kernel covers, contractions shorter than the append's eight waves, positions in
the millions.  A rotated row rounds once more: bf16 keeps eight significant bits, so by at most 2^-8 of a value, which is at
most the pair's length."""
import numpy as np
import pytest
import torch

from paper_2505_24544_amd import binding as bx

pytestmark = pytest.mark.gpu
HD = 128


def rotate(x, pos, base=10000.0):
    """x [rows, heads, 128] float64, pos [rows]"""
    c = np.arange(HD // 2)
    ang = pos[:, None] * base ** (-2.0 * c / HD)
    cs, sn = np.cos(ang)[:, None], np.sin(ang)[:, None]
    a, b = x[..., :HD // 2], x[..., HD // 2:]
    return np.concatenate([a * cs - b * sn, b * cs + a * sn], -1)


def close(got, ref):
    got, ref = got.reshape(ref.shape), ref
    pair = np.hypot(ref[..., :HD // 2], ref[..., HD // 2:])
    err = np.maximum(np.abs(got - ref)[..., :HD // 2], np.abs(got - ref)[..., HD // 2:])
    assert (err <= 2.0 ** -8 * pair + 1e-12).all(), float((err / np.maximum(pair, 1e-9)).max())


@pytest.mark.parametrize("S,H,G", [(70, 1, 1), (130, 32, 8), (33, 40, 40)])
def test_training_rows(S, H, G):
    gen = torch.Generator(device="cuda").manual_seed(S)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    D = 64
    t = dict(xq=r(S, D), xkv=r(S, D), wq=r(D, H * HD, std=0.1), wk=r(D, G * HD, std=0.1), wv=r(D, G * HD, std=0.1), wo=r(H * HD, D, std=0.1))
    out = {}
    for flag in (0, bx.BEAGLE_FLAG_ROPE):
        d = bx.make_desc(batch=1, seq_q=S, seq_kv=S, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=HD, block_size=4, flags=flag)
        e = lambda *s, dt=torch.bfloat16: torch.empty(*s, dtype=dt, device="cuda")
        y, lse, q, k, v, o = e(S, D), e(H, S, dt=torch.float32), e(S, H, HD), e(S, G, HD), e(S, G, HD), e(S, H, HD)
        bx.beagle_xattn_fwd(d, t["xq"], t["xkv"], t["wq"], t["wk"], t["wv"], t["wo"], y, lse, q, k, v, o)
        out[flag] = {n: x.double().cpu().numpy() for n, x in dict(q=q, k=k, v=v).items()}
    pos = np.arange(S, dtype=np.float64)
    for n in ("q", "k"):
        close(out[bx.BEAGLE_FLAG_ROPE][n], rotate(out[0][n], pos))
    assert np.array_equal(out[bx.BEAGLE_FLAG_ROPE]["v"], out[0]["v"])


@pytest.mark.parametrize("n,D,G,given", [(1, 128, 1, False), (8, 384, 2, True), (9, 640, 3, True), (16, 4096, 8, False)])
def test_append_on_packed_weights(n, D, G, given):
    gen = torch.Generator(device="cuda").manual_seed(D)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).bfloat16()
    x, w = r(n, D), dict(wk=r(D, G * HD, std=0.05), wv=r(D, G * HD, std=0.05))
    pk = {k + "_pk": torch.empty_like(v) for k, v in w.items()}
    L, at = n + 5, 3
    where = torch.tensor([7 + 1000003 * i for i in range(n)], dtype=torch.int32, device="cuda") if given else None
    rows = {}
    for flag in (0, bx.BEAGLE_FLAG_ROPE):
        d = bx.make_desc(batch=1, seq_q=n, seq_kv=L, hidden=D, n_q_heads=G, n_kv_heads=G, head_dim=HD, flags=flag,
                         rope_positions=where if flag else None)
        bx.beagle_xattn_prepare_weights(d, **w, **pk)
        kc, vc = (torch.full((L, G, HD), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        bx.beagle_xattn_kv_append_prepared(d, x, pk["wk_pk"], pk["wv_pk"], kc, vc, at)
        rows[flag] = kc[at:at + n].double().cpu().numpy(), vc[at:at + n].double().cpu().numpy()
        rest = torch.cat([kc[:at], kc[at + n:], vc[:at], vc[at + n:]])
        assert bool((rest == 7.0).all())
    pos = where.double().cpu().numpy() if given else at + np.arange(n, dtype=np.float64)
    close(rows[bx.BEAGLE_FLAG_ROPE][0], rotate(rows[0][0], pos))
    assert np.array_equal(rows[bx.BEAGLE_FLAG_ROPE][1], rows[0][1])
    plain = (x.float() @ w["wv"].float()).double().cpu().numpy()
    assert np.linalg.norm(rows[0][1].reshape(n, -1) - plain) <= 2.0 ** -8 * np.linalg.norm(plain)
