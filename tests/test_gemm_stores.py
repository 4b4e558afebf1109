"""The bf16 GEMM kernels as they are compiled: the rows of a tile leave through global stores.  Flat ones count on the LDS counter as well,
and the waits for the patches that the rows are read from would wait for them."""
from test_mfma_in_place import kernels, library, pytestmark  # noqa: F401


def test_tiles_leave_through_global_stores(kernels):  # noqa: F811
    gemm = {n: c for n, c in kernels.items() if "gemm_bf16" in n}
    assert len(gemm) == 24
    ops = {n: {i.op for i in c if "_store_" in i.op or "_load_" in i.op} for n, c in gemm.items()}
    assert all(any(o.startswith("global_store") for o in v) for v in ops.values())
    assert {n: sorted(o for o in v if o.startswith("flat")) for n, v in ops.items() if any(o.startswith("flat") for o in v)} == {}
