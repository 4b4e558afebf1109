"""Forward and dQ on whole key tiles per wave and on half tiles (two waves per 32 queries, merged): the two sides of the choice by
the number of workgroups, at tile edges, with ragged and unseen tiles, offsets, entries of other lengths, and scores so far
apart that the halves' running maxima differ.  Same oracle and tolerances as the packed and parity tests."""
import numpy as np
import pytest

import gpu_harness as gh
from oracle import beagle_oracle as orc
from paper_2505_24544_amd import synth
from test_gpu_packed import _pack, _ref, _run, OUT_ABS, OUT_FRO, LSE_TOL, GRAD_FRO, GRADS

pytestmark = pytest.mark.gpu
MANY = dict(hidden=64, n_q_heads=96, n_kv_heads=96)          # 3 entries: more than 256 workgroups, whole tiles
FEW = dict(hidden=64, n_q_heads=4, n_kv_heads=2)


@pytest.mark.parametrize("heads", [MANY, FEW])
@pytest.mark.parametrize("lens,k,eps", [
    ([129, 64, 1], 4, None),
    ([200, 97, 33], 3, [0, 2, 1]),
    ([65, 32, 31], 8, [5, 0, 7]),
])
def test_packed_entries_on_either_side(heads, lens, k, eps):
    cfg = synth.CONFIGS["c2"].with_(batch=3, seq_q=max(lens), seq_kv=max(lens), block_size=k, seed_base=701, **heads)
    pk, cu_q, cu_kv = _pack(cfg, synth.make_inputs(cfg, peaked_queries=True), lens, lens)
    ref = _ref(cfg, pk, cu_q, cu_kv, eps)
    fw, gr = _run(cfg, pk, cu_q, cu_kv, eps_list=eps)
    assert gh.max_abs(fw["y"], ref["y"]) <= OUT_ABS * max(1.0, np.abs(ref["y"]).max()) and gh.rel_fro(fw["y"], ref["y"]) <= OUT_FRO
    fin = np.isfinite(ref["lse"])
    assert np.array_equal(np.isneginf(fw["lse"]), ~fin)
    assert gh.max_abs(fw["lse"][fin], ref["lse"][fin]) <= LSE_TOL * max(1.0, np.abs(ref["lse"][fin]).max())
    for n in GRADS:
        assert gh.rel_fro(gr[n], ref[n]) <= GRAD_FRO, (n, gh.rel_fro(gr[n], ref[n]))


@pytest.mark.parametrize("S,L,H,scale_mul", [
    (130, 130, 200, 32.0), (130, 130, 4, 32.0),              # whole and half tiles, maxima tens of nats apart
    (1100, 1100, 32, 1.0), (1000, 1000, 34, 1.0),            # 288 workgroups: half tiles on the long chain, whole on the short
    (300, 90, 3, 1.0), (90, 300, 3, 1.0),                    # keys end inside a tile's second half; queries end first
])
def test_attention_core_on_either_side(S, L, H, scale_mul):
    from test_gpu_attn_core import _check
    cfg = synth.CONFIGS["c2"].with_(batch=1, seq_q=S, seq_kv=L, hidden=64, n_q_heads=H, n_kv_heads=H, seed_base=733)
    inp = synth.make_inputs(cfg, with_dy=False)
    scale = scale_mul / np.sqrt(cfg.head_dim)
    _, fw = gh.run_fwd(cfg, inp, scale=scale)
    _check(fw, orc.dense_mask(S, L, cfg.block_size, cfg.block_offset), scale, heads=sorted({0, H - 1}))
