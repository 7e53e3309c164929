"""The per-class kernels of mixed sizes {5, 13, 23, 26}: stacks around the 64
products that a wave reads at once, inner sizes outside the set, and the rule
that chooses between them and the 4 x 4 groups (the same sums in the same
order, so the same bits)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import TOL_FP64_MULTIPLY, assert_same_matrix, from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _sizes(rng, n, of):
    return rng.choice(np.array(of, dtype=np.int32), n).astype(np.int32)


def _multiply(da, db, a, b):
    from paper_2003_03868_amd import bsm
    dc = bsm.Matrix.empty_like(a.row_blk_size, b.col_blk_size)
    bsm.bsm_multiply(1.0, da.handle, db.handle, 0.0, dc.handle, 0.0)
    return from_dev(dc), bsm.bsm_last_smm_kernel()


@pytest.mark.parametrize("nk", [1, 63, 64, 65, 129])
def test_class_stacks_around_a_chunk(monkeypatch, nk):
    rng = np.random.default_rng(nk)
    m, k, n = (_sizes(rng, q, (5, 13, 23, 26)) for q in (9, nk, 11))
    m[:4] = n[:4] = (5, 13, 23, 26)
    a, b = synth.random_bsr(9, nk, m, k, 1.0, rng), synth.random_bsr(nk, 11, k, n, 0.98, rng)
    da, db = to_dev(a), to_dev(b)
    monkeypatch.setenv("BSM_MIXED_TILE", "0")
    one, name = _multiply(da, db, a, b)
    assert "class" in name
    monkeypatch.setenv("BSM_MIXED_TILE", "1")
    groups, _ = _multiply(da, db, a, b)
    assert np.array_equal(one.values, groups.values)


@pytest.mark.parametrize("m,n,k", [(13, 23, 9), (5, 5, 1), (26, 26, 25), (23, 13, 4)])
def test_class_kernel_other_inner_size(orc, m, n, k):
    """A uniform product that the tuning table sends to the class kernel with
    an inner size that has no compile-time path."""
    from paper_2003_03868_amd import bsm
    rng = np.random.default_rng(m + k)
    a = synth.random_bsr(7, 70, np.full(7, m), np.full(70, k), 0.95, rng)
    b = synth.random_bsr(70, 6, np.full(70, k), np.full(6, n), 0.95, rng)
    bsm.bsm_set_smm_table([((m, n, k), (2, 1, 1))])
    try:
        got, name = _multiply(to_dev(a), to_dev(b), a, b)
    finally:
        bsm.bsm_set_smm_table(None)
    assert "class" in name
    assert_same_matrix(got, orc.multiply(1.0, a, b), TOL_FP64_MULTIPLY, "class")


@pytest.mark.parametrize("sizes,blocks,groups", [((5, 13, 23, 26), 80, True), ((5, 13), 80, False),
                                                 ((13, 23), 56, True), ((5, 13, 23, 26), 110, True),
                                                 ((13, 23), 80, True)])
def test_default_rule(monkeypatch, sizes, blocks, groups):
    """Few products per class, or many per C block: groups."""
    monkeypatch.delenv("BSM_MIXED_TILE", raising=False)
    rng = np.random.default_rng(blocks)
    s = _sizes(rng, blocks, sizes)
    dens = 0.95 if blocks == 110 else 0.99 if sizes == (13, 23) else 0.75
    a = synth.random_bsr(blocks, blocks, s, s, dens, rng)
    da = to_dev(a)
    got, name = _multiply(da, da, a, a)
    assert ("mtile" in name) == groups, name
    monkeypatch.setenv("BSM_MIXED_TILE", "0" if groups else "1")
    want, _ = _multiply(da, da, a, a)
    assert np.array_equal(got.values, want.values)
