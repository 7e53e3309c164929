"""Product stacks around the 64 products that a wave reads at once: the
one-C-block-per-wave kernels of uniform sizes against the group kernels (the
same sums in the same order, so the same bits)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("prec", [0, 1, 2, 3], ids=["fp64", "fp32", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("b,nk", [(5, 63), (5, 64), (5, 65), (13, 127), (13, 128), (13, 129),
                                  (23, 200), (26, 65), (32, 64)])
def test_stacks_around_a_chunk(monkeypatch, prec, b, nk):
    from paper_2003_03868_amd import bsm
    rng = np.random.default_rng(1000 * b + nk)
    a = synth.random_bsr(3, nk, np.full(3, b), np.full(nk, b), 1.0, rng)
    bm = synth.random_bsr(nk, 5, np.full(nk, b), np.full(5, b), 0.97, rng)
    da, db = to_dev(a), to_dev(bm)
    out = []
    for env in ({"BSM_SMM_VARIANT": "2", "BSM_LOWP_QUAD": "0"}, {"BSM_SMM_VARIANT": "6", "BSM_LOWP_QUAD": "1"}):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        dc = bsm.Matrix.empty_like(a.row_blk_size, bm.col_blk_size)
        bsm.bsm_multiply(1.0, da.handle, db.handle, 0.0, dc.handle, 0.0, 0, prec)
        out.append(from_dev(dc).values)
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("b,blocks,groups", [(5, 100, False), (5, 130, True), (13, 130, True),
                                             (26, 100, False), (32, 130, True)])
def test_default_rule(monkeypatch, b, blocks, groups):
    """Whichever FP64 kernel the default picks, the bits are those of the other."""
    from paper_2003_03868_amd import bsm
    monkeypatch.delenv("BSM_SMM_VARIANT", raising=False)
    rng = np.random.default_rng(b)
    a = synth.random_bsr(blocks, blocks, np.full(blocks, b), np.full(blocks, b), 0.75, rng)
    da = to_dev(a)
    out = []
    for variant in (None, "2" if groups else "6"):
        if variant:
            monkeypatch.setenv("BSM_SMM_VARIANT", variant)
        dc = bsm.Matrix.empty_like(a.row_blk_size, a.col_blk_size)
        bsm.bsm_multiply(1.0, da.handle, da.handle, 0.0, dc.handle, 0.0)
        name = bsm.bsm_last_smm_kernel()
        assert ("fixed" not in name) == (groups if variant is None else not groups), name
        out.append(from_dev(dc).values)
    assert np.array_equal(out[0], out[1])
