"""Transpose and compaction of blocks at the sizes where their kernels can go
wrong: rows around the sort's workgroup and tile, runs of blocks around a
wave's share, the smallest and the largest blocks."""
import numpy as np
import pytest

import synth
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("nbr,nbc,sizes,dens", [
    (1, 1, (32,), 1.0), (256, 3, (1, 2), 1.0), (257, 2, (2, 5), 1.0), (2049, 2, (1, 3), 1.0),
    (4500, 1, (1, 2), 0.9), (40, 37, (1, 7, 16, 31, 32), 0.5), (3, 300, (13, 26), 0.3)])
def test_transpose(orc, nbr, nbc, sizes, dens):
    """Data movement: bit for bit."""
    from paper_2003_03868_amd import bsm
    rng = np.random.default_rng(nbr + nbc)
    a = synth.random_bsr(nbr, nbc, rng.choice(sizes, nbr), rng.choice(sizes, nbc), dens, rng)
    da = to_dev(a)
    got = from_dev(bsm.Matrix(bsm.bsm_transpose(da.handle), a.col_blk_size, a.row_blk_size))
    ref = orc.transpose(a)
    assert np.array_equal(got.row_ptr, ref.row_ptr) and np.array_equal(got.col_idx, ref.col_idx)
    assert np.array_equal(got.values, ref.values)


@pytest.mark.parametrize("nblk", [1, 2, 15, 16, 17, 31, 63, 64, 65, 127, 129])
@pytest.mark.parametrize("size", [1, 6, 11, 12, 32])
def test_filter_keeps_blocks(nblk, size):
    """The kept blocks of a row of blocks, bit for bit, with none, some and all
    of a run dropped."""
    from paper_2003_03868_amd import bsm
    rng = np.random.default_rng(31 * nblk + size)
    a = synth.random_bsr(2, nblk, np.full(2, size), np.full(nblk, size), 1.0, rng)
    keep = rng.random(a.nnzb) < 0.5
    if nblk >= 16:
        keep[:16] = False
        keep[-16:] = True
    blocks = a.values.reshape(a.nnzb, -1)
    blocks[~keep] *= 1e-9
    blocks[keep] += np.where(blocks[keep] < 0, -1.0, 1.0)
    d = to_dev(a)
    bsm.bsm_filter(d.handle, 1e-3)
    got = from_dev(d)
    rows = a.block_rows()[keep]
    assert np.array_equal(got.row_ptr, np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=2))]))
    assert np.array_equal(got.col_idx, a.col_idx[keep])
    assert np.array_equal(got.values, blocks[keep].ravel())


@pytest.mark.parametrize("nbr,nbc,long_rows", [(3, (1 << 24) + 9, ()), (30000, 5, (1, 4)), (70001, 7, (0,))])
def test_transpose_of_any_row_length(nbr, nbc, long_rows):
    """Results with more block rows than one launch may have workgroups of
    256 threads, and with rows of tens of thousands of blocks beside short
    ones."""
    import torch
    from paper_2003_03868_amd import bsm
    rng = np.random.default_rng(nbr)
    pairs = {(int(i), int(j)) for i, j in zip(rng.integers(0, nbr, 500), rng.integers(0, nbc, 500))}
    pairs |= {(0, 0), (nbr - 1, nbc - 1)}
    pairs |= {(i, j) for j in long_rows for i in range(nbr)}
    r, c = np.array(sorted(pairs)).T
    val = rng.standard_normal(len(r))
    ptr = lambda idx, n: np.concatenate([[0], np.cumsum(np.bincount(idx, minlength=n))])
    ones = lambda n: np.ones(n, dtype=np.int32)
    a = bsm.Matrix.from_arrays(ones(nbr), ones(nbc), ptr(r, nbr), c, val)
    t = bsm.Matrix(bsm.bsm_transpose(a.handle), ones(nbc), ones(nbr))
    got_ptr, got_col, got_val = t.export()
    o = np.lexsort((r, c))
    assert np.array_equal(got_ptr, ptr(c, nbc)) and np.array_equal(got_col, r[o])
    assert np.array_equal(got_val, val[o])


@pytest.mark.parametrize("nblk", [8191, 8192, 8193, 9001])
@pytest.mark.parametrize("size", [1, 6])
def test_filter_of_many_small_blocks(nblk, size):
    """Around the number of blocks from which a wave takes sixteen of them."""
    from paper_2003_03868_amd import bsm
    rng = np.random.default_rng(nblk + size)
    a = synth.random_bsr(2, nblk, np.full(2, size), np.full(nblk, size), 1.0, rng)
    keep = rng.random(a.nnzb) < 0.5
    keep[:64] = False
    keep[-64:] = True
    blocks = a.values.reshape(a.nnzb, -1)
    blocks[~keep] *= 1e-9
    blocks[keep] += np.where(blocks[keep] < 0, -1.0, 1.0)
    d = to_dev(a)
    bsm.bsm_filter(d.handle, 1e-3)
    got = from_dev(d)
    assert np.array_equal(got.col_idx, a.col_idx[keep])
    assert np.array_equal(got.values, blocks[keep].ravel())
