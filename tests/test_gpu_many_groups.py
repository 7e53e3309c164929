"""More 4 x 4 groups of C blocks than one launch may have workgroups (2^32
threads): every group holds one C block of an outer product over block rows
and columns 0, 4, 8, ...  Whole-number values, so that results are exact."""
import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu
COLS = 32768


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _outer(rows, s, rest, prec):
    """C = A B for one block column of A and one block row of B, blocks of s
    at every fourth row and column, the rows and columns between of size
    `rest` and empty; C's values and those of a dense product."""
    import torch
    from paper_2003_03868_amd import bsm
    g = torch.Generator(device="cuda").manual_seed(rows)
    val = lambda *n: torch.randint(-7, 8, n, generator=g, device="cuda").double()
    a, b = val(rows, s, s), val(COLS, s, s)
    used = lambda n: np.where(np.arange(4 * n) % 4 == 0, s, rest).astype(np.int32)
    rs, ks, cs = used(rows), np.array([s], dtype=np.int32), used(COLS)
    a_ptr = (torch.arange(4 * rows + 1, device="cuda") + 3) // 4
    b_ptr = torch.tensor([0, COLS], device="cuda")
    a_col = torch.zeros(rows, dtype=torch.int32, device="cuda")
    b_col = 4 * torch.arange(COLS, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    ma = bsm.Matrix(bsm.bsm_create(4 * rows, 1, rs, ks, rows, a_ptr, a_col, a, 1), rs, ks)
    mb = bsm.Matrix(bsm.bsm_create(1, 4 * COLS, ks, cs, COLS, b_ptr, b_col, b, 1), ks, cs)
    mc = bsm.Matrix.empty_like(rs, cs)
    bsm.bsm_multiply(1.0, ma.handle, mb.handle, 0.0, mc.handle, 0.0, 0, prec)
    name = bsm.bsm_last_smm_kernel()
    n = rows * COLS
    inf = bsm.bsm_get_info(mc.handle)
    assert inf.nnzb == n and inf.nvalues == n * s * s
    ptr = torch.empty(4 * rows + 1, dtype=torch.int64, device="cuda")
    col = torch.empty(n, dtype=torch.int32, device="cuda")
    got = torch.empty(n * s * s, dtype=torch.float64, device="cuda")
    bsm.bsm_export(mc.handle, ptr, col, got, 1)
    torch.cuda.synchronize()
    assert torch.equal(ptr, a_ptr * COLS)
    assert torch.equal(col.view(rows, COLS), b_col.expand(rows, COLS))
    dense = a.reshape(rows * s, s) @ b.permute(1, 0, 2).reshape(s, COLS * s)
    want = dense.view(rows, s, COLS, s).permute(0, 2, 1, 3)
    return name, bool(torch.equal(got.view(rows, COLS, s, s), want))


def test_uniform(monkeypatch):
    monkeypatch.setenv("BSM_QUAD_MIN_REUSE", "0")
    name, same = _outer(129, 4, 4, 0)          # 1024 threads per group: 2^22 of them
    assert "k_smm_f64_tile" in name and same


def test_mixed(monkeypatch):
    monkeypatch.setenv("BSM_MIXED_TILE", "1")
    name, same = _outer(257, 2, 1, 0)          # 512 threads: 2^23
    assert "k_smm_f64_mtile" in name and same


def test_reduced_precision(monkeypatch):
    monkeypatch.setenv("BSM_LOWP_QUAD", "1")
    name, same = _outer(257, 5, 5, 1)
    assert "k_lowp_tile" in name and same


def test_reduced_precision_many_operand_blocks(monkeypatch):
    """An operand of 2^26 + 65,536 blocks of 5: more than one launch may have
    workgroups of 64 to pack them."""
    import torch
    from paper_2003_03868_amd import bsm
    monkeypatch.setenv("BSM_LOWP_QUAD", "1")
    nb, nk, s = 8200, 8192, 5
    g = torch.Generator(device="cuda").manual_seed(5)
    a = torch.empty(nb, nk, s, s, dtype=torch.float64, device="cuda").random_(0, 8, generator=g)
    b = torch.empty(2, s, s, dtype=torch.float64, device="cuda").random_(0, 8, generator=g)
    rows = [3, nk - 1]                         # B's blocks, in its only block column
    size = lambda n: np.full(n, s, dtype=np.int32)
    a_ptr = torch.arange(nb + 1, device="cuda") * nk
    a_col = torch.arange(nk, dtype=torch.int32, device="cuda").repeat(nb)
    b_ptr = torch.zeros(nk + 1, dtype=torch.int64, device="cuda")
    b_ptr[rows[0] + 1:] = 1
    b_ptr[nk] = 2
    b_col = torch.zeros(2, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    ma = bsm.Matrix(bsm.bsm_create(nb, nk, size(nb), size(nk), nb * nk, a_ptr, a_col, a, 1), size(nb), size(nk))
    mb = bsm.Matrix(bsm.bsm_create(nk, 1, size(nk), size(1), 2, b_ptr, b_col, b, 1), size(nk), size(1))
    mc = bsm.Matrix.empty_like(size(nb), size(1))
    bsm.bsm_multiply(1.0, ma.handle, mb.handle, 0.0, mc.handle, 0.0, 0, bsm.FP32)
    assert "k_lowp_tile" in bsm.bsm_last_smm_kernel()
    got = torch.from_numpy(mc.export()[2]).cuda()
    want = sum(a[:, r].reshape(-1, s) @ b[q] for q, r in enumerate(rows))
    assert torch.equal(got, want.reshape(-1))
