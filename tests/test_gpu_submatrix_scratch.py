"""Device memory of the submatrix method beside its batches: P and one row sum
per block row of every block, no second copy of H's values."""
import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def test_row_sums_are_small(monkeypatch):
    need_gpu()
    import torch
    from paper_2003_03868_amd import bsm
    monkeypatch.setenv("BSM_SUB_BATCH_BYTES", str(64 << 20))
    n, b = 100_000, 32                          # diagonal blocks: 0.8 GB of values
    g = torch.Generator(device="cuda").manual_seed(2)
    v = 0.01 * torch.randn(n, b, b, generator=g, device="cuda", dtype=torch.float64)
    v = v + v.mT + torch.eye(b, device="cuda", dtype=torch.float64)
    sizes = np.full(n, b, dtype=np.int32)
    ptr = torch.arange(n + 1, device="cuda")
    torch.cuda.synchronize()
    h = bsm.Matrix(bsm.bsm_create(n, n, sizes, sizes, n, ptr, ptr[:n].to(torch.int32), v, 1), sizes, sizes)
    o = bsm.bsm_sign_opts_default()
    o.eps_filter, o.tol = 0.0, 1e-8
    before = torch.cuda.mem_get_info()[0]
    st, ph, _ = bsm.bsm_submatrix_density(h.handle, 0.0, o)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]     # freed scratch stays with the library
    p = bsm.Matrix(ph, sizes, sizes)
    assert st == bsm.OK and bsm.bsm_get_info(p.handle).nnzb == n
    print(f"{used / 2**30:.2f} GiB for {v.numel() * 8 / 2**30:.2f} GiB of values")
    assert used < 1.5 * v.numel() * 8
