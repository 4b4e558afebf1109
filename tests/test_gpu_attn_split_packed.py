"""Shared key tiles on packed batches: the chunk length follows from the longest entry, the number of chunks of a tile from its own
entry and offset, in the kernel that writes the shares and in the one that adds them.  The workspace starts out as NaN, so that a
share that is read and was not written shows."""
import numpy as np
import pytest
import torch

import gpu_harness as gh
import test_gpu_packed as packed
from paper_2505_24544_amd import binding as bx, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,lens_q,lens_kv,eps_list", [
    # chunks of four pairs, four heads per group: the second entry's only query tile is one chunk, the third ends in a short one
    (dict(batch=3, seq_q=700, seq_kv=700, n_q_heads=8, n_kv_heads=2, block_size=4), [700, 50, 333], [700, 50, 333], [1, 0, 3]),
    # windows as long as a query tile with offsets far apart: first queries of a key tile in different tiles per entry
    (dict(batch=3, seq_q=450, seq_kv=450, n_q_heads=8, n_kv_heads=1, block_size=70), [130, 450, 64], [130, 450, 64], [69, 3, 40]),
    # more queries than keys and the other way round; an entry of one row
    (dict(batch=4, seq_q=500, seq_kv=300, n_q_heads=16, n_kv_heads=1, block_size=3), [500, 1, 90, 257], [300, 2, 260, 129], [0, 2, 1, 2]),
])
def test_shares_of_packed_entries(kw, lens_q, lens_kv, eps_list, monkeypatch):
    def poisoned(desc, which):
        return torch.full((bx.beagle_xattn_workspace_bytes(desc, which),), 0xff, dtype=torch.uint8, device=gh.DEV)
    monkeypatch.setattr(gh, "workspace", poisoned)
    cfg = synth.CONFIGS["c3"].with_(hidden=256, seed_base=381, **kw)
    pk, cu_q, cu_kv = packed._pack(cfg, synth.make_inputs(cfg, peaked_queries=True), lens_q, lens_kv)
    f, g = packed._run(cfg, pk, cu_q, cu_kv, eps_list=eps_list)
    ref = packed._ref(cfg, pk, cu_q, cu_kv, eps_list=eps_list)
    assert gh.rel_fro(f["y"], ref["y"]) <= packed.OUT_FRO
    for n in packed.GRADS:
        assert np.isfinite(g[n]).all() and gh.rel_fro(g[n], ref[n]) <= packed.GRAD_FRO, (n, gh.rel_fro(g[n], ref[n]))
    _, again = packed._run(cfg, pk, cu_q, cu_kv, eps_list=eps_list)
    for n in packed.GRADS:
        assert np.array_equal(g[n], again[n]), n
