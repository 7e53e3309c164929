"""Groups of C blocks where neighbouring block rows and columns have much in
common, one C block per wave where they have not: the same band of blocks in
order and with its rows and columns renumbered at random.  Whichever kernel
the default picks, the bits are those of the other."""
import numpy as np
import pytest

from synth import BSR
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu
BASIS, OTHER = (5, 13, 23, 26), (4, 9, 13, 18, 22, 31)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _band(n, w, sizes, perm, rng):
    p = rng.permutation(n) if perm else np.arange(n)
    r = np.repeat(np.arange(n), w)
    c = (r + np.tile(np.arange(w) - w // 2, n)) % n
    r, c = p[r], p[c]
    o = np.lexsort((c, r))
    r, c = r[o], c[o]
    s = rng.choice(np.array(sizes, dtype=np.int32), n).astype(np.int32)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int64)
    return BSR(s, s, ptr, c.astype(np.int32), rng.standard_normal(int((s[r].astype(int) * s[c]).sum())))


# two million products and more (fewer for mixed sizes); enough per C block
@pytest.mark.parametrize("prec,sizes,n,w,groups,force", [
    (0, (23,), 1300, 33, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (13,), 800, 65, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (5,), 900, 151, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (32,), 800, 65, "k_smm_f64_quad", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (4,), 1500, 33, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (9,), 1300, 33, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (31,), 800, 33, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    # more block columns than a pass over the bitmap that counts entries has,
    # with at most and more than 256 blocks per row group
    (0, (4,), 66000, 33, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, (4,), 66000, 65, "k_smm_f64_tile", ("BSM_QUAD_MIN_REUSE", "0", "1e9")),
    (0, OTHER, 2000, 9, "k_smm_f64_mtile", ("BSM_MIXED_TILE", "1", "0")),
    (0, BASIS, 1000, 9, "k_smm_f64_mtile", ("BSM_MIXED_TILE", "1", "0")),
    (0, BASIS, 900, 151, "k_smm_f64_mtile", ("BSM_MIXED_TILE", "1", "0")),
    (1, (5,), 1300, 33, "k_lowp_tile", ("BSM_LOWP_QUAD", "1", "0")),
    (1, (32,), 800, 33, "k_lowp_tile", ("BSM_LOWP_QUAD", "1", "0")),
    (2, (13,), 800, 33, "k_lowp_tile", ("BSM_LOWP_QUAD", "1", "0")),
    (3, (23,), 800, 33, "k_lowp_tile", ("BSM_LOWP_QUAD", "1", "0"))])
@pytest.mark.parametrize("perm", [False, True])
def test_order_decides(monkeypatch, prec, sizes, n, w, groups, force, perm):
    from paper_2003_03868_amd import bsm
    for k in ("BSM_QUAD_MIN_REUSE", "BSM_MIXED_TILE", "BSM_LOWP_QUAD", "BSM_SMM_VARIANT", "BSM_QUAD_GROUP"):
        monkeypatch.delenv(k, raising=False)
    rng = np.random.default_rng(n + w)
    a = _band(n, w, sizes, perm, rng)
    da = to_dev(a)
    out = []
    for forced in (False, True):
        if forced:
            monkeypatch.setenv(force[0], force[1] if perm else force[2])
        dc = bsm.Matrix.empty_like(a.row_blk_size, a.col_blk_size)
        bsm.bsm_multiply(1.0, da.handle, da.handle, 0.0, dc.handle, 0.0, 0, prec)
        name = bsm.bsm_last_smm_kernel()
        # in order by default, at random when forced; size 13 then has quads
        assert (groups in name or "quad" in name) == (perm == forced), name
        out.append(from_dev(dc).values)
    assert np.array_equal(out[0], out[1])
