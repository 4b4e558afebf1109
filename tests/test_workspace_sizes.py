"""Workspace sizes on the host: the bytes reported for a program's largest call serve its smaller ones, and a call needs no more
than its tensors do.  Nothing is enqueued: the simulation step checks its step number behind the workspace, so that a negative
one tells whether the workspace would have done."""
import pytest

from paper_2505_24544_amd import binding as bx

A = 0x1000                                             # any aligned address: never read
up = lambda n: (n + 255) // 256 * 256


def _desc(batch, seq, H=32, G=8, D=4096, flags=0):
    return bx.make_desc(batch=batch, seq_q=seq, seq_kv=seq, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=128, block_size=4, flags=flags)


def _accepts(d, n):
    """Whether n bytes get a simulation step's backward past the workspace check."""
    st = bx.beagle_xattn_bwd_sim(d, *([A] * 15), -1, *([A] * 7), A, stream=0, workspace_bytes=n, check=False)
    assert st in (2, 4)
    return st == 2


def _tensors(batch, seq, H, G, D):
    """dO, dQ, dK, dV, delta and the scaled LSE, and the float halves of dWk, dWv where those are split."""
    q, k, f = up(batch * seq * H * 128 * 2), up(batch * seq * G * 128 * 2), up(batch * H * seq * 4)
    return 2 * q + 2 * k + 2 * f, up(4 * D * G * 128 * 4)


SHAPES = [(1, 300), (1, 777), (1, 1300), (1, 4096), (1, 4100), (1, 7300), (2, 2048), (4, 1024), (4, 1025), (8, 512)]


@pytest.mark.parametrize("H,G,D", [(32, 8, 4096), (32, 32, 4096), (40, 40, 5120), (16, 1, 2048)])
@pytest.mark.parametrize("sim", [False, True])
def test_largest_call_serves_the_smaller_ones(H, G, D, sim):
    which = bx.BEAGLE_WS_BWD_SIM if sim else bx.BEAGLE_WS_BWD
    size = lambda b, s: bx.beagle_xattn_workspace_bytes(_desc(b, s, H, G, D), which)
    block = lambda b, s: bx.beagle_xattn_block_workspace_bytes(_desc(b, s, H, G, D), 11008,
                                                               bx.BEAGLE_WS_BLOCK_BWD_SIM if sim else bx.BEAGLE_WS_BLOCK_BWD)
    for b, s in SHAPES:
        for b2, s2 in SHAPES:
            if b <= b2 and s <= s2:
                assert size(b, s) <= size(b2, s2) and block(b, s) <= block(b2, s2), ((b, s), (b2, s2))


@pytest.mark.parametrize("batch,seq", SHAPES)
@pytest.mark.parametrize("H,G,D", [(32, 8, 4096), (32, 32, 4096)])
def test_backward_needs_no_more_than_its_tensors(batch, seq, H, G, D):
    d = _desc(batch, seq, H, G, D)
    own, halves = _tensors(batch, seq, H, G, D)
    own += 2 * up(batch * seq * G * 128 * 2)           # dKp, dVp
    reported = bx.beagle_xattn_workspace_bytes(d, bx.BEAGLE_WS_BWD_SIM)
    assert not _accepts(d, own - 1) and _accepts(d, reported)
    assert _accepts(d, own) or _accepts(d, own + halves)
    assert own <= reported <= own + halves + (64 << 20)


def _draft(M, L, H=32, G=8, D=4096):
    return bx.make_desc(batch=1, seq_q=M, seq_kv=L, hidden=D, n_q_heads=H, n_kv_heads=G, head_dim=128)


@pytest.mark.parametrize("H,G,D", [(32, 8, 4096), (32, 32, 4096), (64, 8, 1024), (40, 40, 5120), (24, 4, 128)])
@pytest.mark.parametrize("L", [128, 619, 1024, 1300, 4096, 9000])
def test_widest_draft_step_serves_the_narrower_ones(L, H, G, D):
    size = [bx.beagle_xattn_workspace_bytes(_draft(M, L, H, G, D), bx.BEAGLE_WS_DRAFT) for M in range(1, 130)]
    assert all(a <= b for a, b in zip(size, size[1:]))
    # queries in k slices of 512, partial rows padded to 32, merged rows, output slices, rotary table: heads that share a
    # workgroup take no more than heads alone
    steps = (L + 127) // 128
    rng = -(-steps // min(256 // H, steps))
    for M in (1, 6, 8, 9, 16, 33, 64, 129):
        m = min(M, 64)
        rows = H * -(-steps // rng) * ((m + 31) // 32 * 32)
        need = (up(-(-D // 512) * m * H * 512) + up(rows * 512) + up(rows * 8) + up(m * H * 256) + up(-(-H * 128 // 512) * m * D * 4) +
                up(M * 512))
        assert size[M - 1] == need
