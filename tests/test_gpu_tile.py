"""The 4 x 4 tile kernel of the FP64 block products at the sizes where it can
go wrong: entry counts around its chunks of 64, partial groups, operands at
the end of their allocation, blocks holding NaN and Inf."""
import numpy as np
import pytest

import synth
from tests.gpu_util import TOL_FP64_MULTIPLY, assert_same_matrix, from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _mult(alpha, a, b, beta=0.0, c=None):
    from paper_2003_03868_amd import bsm
    da = to_dev(a)
    db = da if b is a else to_dev(b)
    dc = to_dev(c) if c is not None else bsm.Matrix.empty_like(a.row_blk_size, b.col_blk_size)
    try:
        bsm.bsm_multiply(alpha, da.handle, db.handle, beta, dc.handle)
    except bsm.BsmError as e:
        assert e.status == bsm.ENONFINITE
    return from_dev(dc), bsm.bsm_last_smm_kernel()


@pytest.mark.parametrize("b", [4, 5, 6, 7, 9, 12, 13, 14, 16, 17, 18, 22, 23, 24, 25, 26, 29, 31, 32])
@pytest.mark.parametrize("nbr,nbk,nbc,dens", [
    (1, 1, 1, 1.0), (4, 1, 4, 1.0), (5, 2, 3, 1.0), (4, 63, 4, 1.0), (3, 64, 5, 1.0),
    (4, 65, 4, 0.7), (7, 128, 9, 0.5), (4, 129, 8, 1.0), (6, 131, 6, 0.4)])
def test_tile_kernel(orc, monkeypatch, b, nbr, nbk, nbc, dens):
    """Against the oracle, and bit for bit against the kernel of one C block
    per wave (the same products in the same order; sizes without a
    compile-time one: the run-time-shape kernel of 4 x 4 x 4 steps)."""
    monkeypatch.setenv("BSM_QUAD_MIN_REUSE", "0")
    monkeypatch.setenv("BSM_QUAD_GROUP", "4")
    rng = np.random.default_rng(1000 * nbk + 10 * nbr + b)
    size = lambda n: np.full(n, b)
    a = synth.random_bsr(nbr, nbk, size(nbr), size(nbk), dens, rng)
    bm = synth.random_bsr(nbk, nbc, size(nbk), size(nbc), dens, rng)
    c = synth.random_bsr(nbr, nbc, size(nbr), size(nbc), 0.5, rng)
    for alpha, beta, cc in [(1.0, 0.0, None), (-0.5, 1.5, c)]:
        got, kernel = _mult(alpha, a, bm, beta, cc)
        assert "k_smm_f64_tile" in kernel
        assert_same_matrix(got, orc.multiply(alpha, a, bm, beta, cc), TOL_FP64_MULTIPLY, "tile")
        monkeypatch.setenv("BSM_SMM_VARIANT", "2" if b in (5, 6, 13, 23, 26, 32) else "1")
        one, _ = _mult(alpha, a, bm, beta, cc)
        monkeypatch.delenv("BSM_SMM_VARIANT")
        assert np.array_equal(got.values, one.values)


@pytest.mark.parametrize("b", [9, 13, 23, 32])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_tile_kernel_nonfinite(monkeypatch, b, bad):
    """A block of NaN or Inf reaches the C blocks of its own products and no
    other (what the padding of a block reads is never stored)."""
    monkeypatch.setenv("BSM_QUAD_MIN_REUSE", "0")
    monkeypatch.setenv("BSM_QUAD_GROUP", "4")
    rng = np.random.default_rng(7)
    a = synth.random_bsr(9, 9, np.full(9, b), np.full(9, b), 0.6, rng)
    off = a.block_offsets()
    for t in (0, 1, a.nnzb // 2, a.nnzb - 1):
        a.values[off[t]:off[t + 1]][:: 1 + t % 3] = bad
    got, _ = _mult(1.0, a, a)
    monkeypatch.setenv("BSM_SMM_VARIANT", "2" if b != 9 else "1")
    one, _ = _mult(1.0, a, a)
    assert np.isfinite(one.values).any() and not np.isfinite(one.values).all()
    assert np.array_equal(got.values, one.values, equal_nan=True)


SIZES = {"basis": (5, 13, 23, 26), "other": (1, 2, 4, 7, 9, 16, 17, 22, 31, 32), "large": (31, 32),
         "all32": (32, 32)}


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("nbr,nbk,nbc,dens", [
    (2, 1, 2, 1.0), (4, 3, 4, 1.0), (5, 64, 3, 0.6), (6, 65, 7, 1.0), (9, 131, 10, 0.4),
    (17, 40, 21, 0.2)])
def test_mixed_tile_kernel(orc, monkeypatch, sizes, nbr, nbk, nbc, dens):
    """Mixed sizes (entries of more than one stage among them: four rows and
    columns of 32 with k = 32) against the oracle, and bit for bit against
    the run-time-shape kernel of 4 x 4 x 4 steps."""
    monkeypatch.setenv("BSM_MIXED_TILE", "1")
    rng = np.random.default_rng(100 * nbk + nbr)
    rs, ks, cs = (rng.choice(SIZES[sizes], n) for n in (nbr, nbk, nbc))
    rs[0], cs[0] = SIZES[sizes][0], SIZES[sizes][-1]
    if sizes == "all32":
        rs[-1] = 5                         # not uniform, one group of 32s only
    a = synth.random_bsr(nbr, nbk, rs, ks, dens, rng)
    b = synth.random_bsr(nbk, nbc, ks, cs, dens, rng)
    c = synth.random_bsr(nbr, nbc, rs, cs, 0.5, rng)
    for alpha, beta, cc in [(1.0, 0.0, None), (-0.5, 1.5, c)]:
        got, kernel = _mult(alpha, a, b, beta, cc)
        uniform = len(set(rs)) == len(set(ks)) == len(set(cs)) == 1
        assert uniform or "k_smm_f64_mtile" in kernel
        assert_same_matrix(got, orc.multiply(alpha, a, b, beta, cc), TOL_FP64_MULTIPLY, "mixed tile")
        monkeypatch.setenv("BSM_SMM_VARIANT", "1")
        one, _ = _mult(alpha, a, b, beta, cc)
        monkeypatch.delenv("BSM_SMM_VARIANT")
        assert np.array_equal(got.values, one.values)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_mixed_tile_kernel_nonfinite(monkeypatch, bad):
    monkeypatch.setenv("BSM_MIXED_TILE", "1")
    rng = np.random.default_rng(11)
    s = rng.choice([3, 5, 13, 14, 26, 32], 13)
    a = synth.random_bsr(13, 13, s, s, 0.6, rng)
    off = a.block_offsets()
    for t in (0, 1, a.nnzb // 2, a.nnzb - 1):
        a.values[off[t]:off[t + 1]][:: 1 + t % 3] = bad
    got, _ = _mult(1.0, a, a)
    monkeypatch.setenv("BSM_SMM_VARIANT", "1")
    one, _ = _mult(1.0, a, a)
    assert np.isfinite(one.values).any() and not np.isfinite(one.values).all()
    assert np.array_equal(got.values, one.values, equal_nan=True)
