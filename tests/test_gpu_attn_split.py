"""dK / dV with a key tile's (head, query tile) pairs shared by several workgroups: chunks that cross heads, the last chunk
short, tiles with a single chunk next to tiles with many, keys that nobody sees (packed: test_gpu_attn_split_packed.py)."""
import numpy as np
import pytest

import gpu_harness as gh
from oracle import beagle_oracle as orc
from paper_2505_24544_amd import binding as bx, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(batch=1, seq_q=64, seq_kv=64, n_q_heads=16, n_kv_heads=1, block_size=4),                   # one tile, one pair per head
    dict(batch=1, seq_q=450, seq_kv=450, n_q_heads=8, n_kv_heads=1, block_size=3, block_offset=2),  # ragged last tiles
    dict(batch=2, seq_q=385, seq_kv=385, n_q_heads=8, n_kv_heads=2, block_size=8, block_offset=5),
    dict(batch=1, seq_q=190, seq_kv=500, n_q_heads=6, n_kv_heads=1, block_size=4),                  # last key tiles unseen
])
def test_shared_key_tiles(kw):
    cfg = synth.CONFIGS["c3"].with_(hidden=256, seed_base=371, **kw)
    inp = synth.make_inputs(cfg, peaked_queries=True)
    mask = orc.dense_mask(cfg.seq_q, cfg.seq_kv, cfg.block_size, cfg.block_offset)
    ref = orc.xattn_backward(inp["dy"], inp["xq"], inp["xkv"], inp["wq"], inp["wk"], inp["wv"], inp["wo"],
                             n_q_heads=cfg.n_q_heads, n_kv_heads=cfg.n_kv_heads, mask=mask)
    dev, _ = gh.run_fwd(cfg, inp)
    _, gr = gh.run_bwd(cfg, inp, dev)
    for n in ("dxkv", "dwk", "dwv", "dwq", "dxq"):
        assert np.isfinite(gr[n]).all() and gh.rel_fro(gr[n], ref[n]) <= 3e-2, (n, gh.rel_fro(gr[n], ref[n]))
    _, again = gh.run_bwd(cfg, inp, dev)
    for n in ("dxkv", "dwk", "dwv"):
        assert np.array_equal(gr[n], again[n]), n
    unseen = ~mask.any(0)
    assert (gr["dxkv"][:, unseen] == 0).all()
