"""Reduced-precision products over 4 x 4 groups of C blocks against the
one-C-block-per-wave kernel, bit for bit (the same FP32 block products, added
into FP64 in the same order): partial groups, more than one 64-entry chunk of
a group's list, more than one entry per stage with a remainder, chunked row
ranges, a plan replayed with new values, and the rule that chooses between
the two."""
import numpy as np
import pytest

import synth
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _square_or_product(rng, nbr, nbk, nbc, b, density, square):
    a = synth.random_bsr(nbr, nbk, np.full(nbr, b), np.full(nbk, b), density, rng)
    if square:
        return a, a
    return a, synth.random_bsr(nbk, nbc, np.full(nbk, b), np.full(nbc, b), density, rng)


@pytest.mark.parametrize("prec", [1, 2, 3], ids=["fp32", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("b", [5, 13, 23, 26, 32])
@pytest.mark.parametrize("shape", [(4, 1, 4, 1.0), (5, 2, 3, 0.9), (7, 67, 6, 0.8), (30, 131, 9, 0.2)])
def test_groups_give_the_one_block_bits(monkeypatch, prec, b, shape):
    from paper_2003_03868_amd import bsm
    nbr, nbk, nbc, density = shape
    rng = np.random.default_rng(17 * b + nbk)
    a, bm = _square_or_product(rng, nbr, nbk, nbc, b, density, False)
    da, db = to_dev(a), to_dev(bm)
    out = {}
    for groups in ("0", "1"):
        monkeypatch.setenv("BSM_LOWP_QUAD", groups)
        dc = bsm.Matrix.empty_like(a.row_blk_size, bm.col_blk_size)
        bsm.bsm_multiply(1.0, da.handle, db.handle, 0.0, dc.handle, 0.0, 0, prec)
        assert ("tile" in bsm.bsm_last_smm_kernel()) == (groups == "1")
        out[groups] = from_dev(dc)
    assert np.array_equal(out["0"].col_idx, out["1"].col_idx)
    assert np.array_equal(out["0"].values, out["1"].values)


@pytest.mark.parametrize("prec", [1, 2, 3], ids=["fp32", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("b,square", [(5, True), (23, True), (23, False), (32, True)])
def test_group_plans_replay_new_values(monkeypatch, prec, b, square):
    """A plan made with groups packs both operands anew on every replay, also
    when A and B are one matrix (their images differ)."""
    from paper_2003_03868_amd import bsm
    monkeypatch.setenv("BSM_LOWP_QUAD", "1")
    rng = np.random.default_rng(b)
    a, bm = _square_or_product(rng, 21, 21, 21, b, 0.4, square)
    da = to_dev(a)
    db = da if square else to_dev(bm)
    dc = bsm.Matrix.empty_like(a.row_blk_size, bm.col_blk_size)
    plan, _ = bsm.bsm_multiply_plan(1.0, da.handle, db.handle, dc.handle, 0.0, 0, prec)
    try:
        first = from_dev(dc).values
        a2 = synth.BSR(a.row_blk_size, a.col_blk_size, a.row_ptr, a.col_idx, 2.0 * a.values[::-1].copy())
        b2 = a2 if square else bm
        da2 = to_dev(a2)
        db2 = da2 if square else db
        for x, y in ((da2, db2), (da, db), (da2, db2)):
            bsm.bsm_plan_execute(plan, x.handle, y.handle, dc.handle)
            dw = bsm.Matrix.empty_like(a.row_blk_size, bm.col_blk_size)
            bsm.bsm_multiply(1.0, x.handle, y.handle, 0.0, dw.handle, 0.0, 0, prec)
            assert np.array_equal(from_dev(dc).values, from_dev(dw).values)
        assert not np.array_equal(from_dev(dc).values, first)
    finally:
        bsm.bsm_plan_destroy(plan)


@pytest.mark.parametrize("prec,b,blocks,groups", [(3, 23, 60, False), (3, 32, 100, True),
                                                  (2, 23, 110, True), (1, 32, 100, True),
                                                  (1, 23, 100, True), (1, 23, 60, False)])
def test_default_rule(monkeypatch, prec, b, blocks, groups):
    """Whichever kernel the default picks, the bits are those of the other."""
    from paper_2003_03868_amd import bsm
    monkeypatch.delenv("BSM_LOWP_QUAD", raising=False)
    rng = np.random.default_rng(blocks)
    a, _ = _square_or_product(rng, blocks, blocks, blocks, b, 0.75, True)
    da = to_dev(a)
    got = bsm.Matrix.empty_like(a.row_blk_size, a.col_blk_size)
    bsm.bsm_multiply(1.0, da.handle, da.handle, 0.0, got.handle, 0.0, 0, prec)
    assert ("tile" in bsm.bsm_last_smm_kernel()) == groups
    monkeypatch.setenv("BSM_LOWP_QUAD", "0" if groups else "1")
    want = bsm.Matrix.empty_like(a.row_blk_size, a.col_blk_size)
    bsm.bsm_multiply(1.0, da.handle, da.handle, 0.0, want.handle, 0.0, 0, prec)
    assert np.array_equal(from_dev(got).values, from_dev(want).values)
