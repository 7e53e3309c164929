"""Where the lists of groups or the operand images do not fit, the multiply is
done with one C block per wave: the same bits, C untouched by the first try."""
import numpy as np
import pytest

import synth
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu
FORCE = (("BSM_QUAD_MIN_REUSE", "0"), ("BSM_MIXED_TILE", "1"), ("BSM_LOWP_QUAD", "1"))


@pytest.fixture(autouse=True)
def _forced(monkeypatch):
    need_gpu()
    for k, v in FORCE:
        monkeypatch.setenv(k, v)


def _operands(sizes, seed):
    rng = np.random.default_rng(seed)
    m, k, n = (rng.choice(np.array(sizes, dtype=np.int32), q) for q in (21, 30, 19))
    return (synth.random_bsr(21, 30, m, k, 0.6, rng), synth.random_bsr(30, 19, k, n, 0.6, rng),
            synth.random_bsr(21, 19, m, n, 0.4, rng))


@pytest.mark.parametrize("prec,sizes,group", [
    (0, (23,), "k_smm_f64_tile"), (0, (5,), "k_smm_f64_quad"), (0, (9,), "k_smm_f64_tile"),
    (0, (5, 13, 23, 26), "k_smm_f64_mtile"), (0, (4, 9, 31), "k_smm_f64_mtile"),
    (1, (13,), "k_lowp_tile"), (3, (23,), "k_lowp_tile")])
@pytest.mark.parametrize("cap", ["64", "3000"])
def test_multiply(monkeypatch, prec, sizes, group, cap):
    from paper_2003_03868_amd import bsm
    a, b, c = _operands(sizes, len(sizes))
    da, db = to_dev(a), to_dev(b)
    out = []
    for limit in (None, cap):
        if limit:
            monkeypatch.setenv("BSM_GROUP_BYTES", limit)
        dc = to_dev(c)
        bsm.bsm_multiply(-0.5, da.handle, db.handle, 1.5, dc.handle, 0.0, 0, prec)
        name = bsm.bsm_last_smm_kernel()
        assert (group in name) == (limit is None), name
        out.append(from_dev(dc))
    assert np.array_equal(out[0].col_idx, out[1].col_idx)
    assert np.array_equal(out[0].values, out[1].values)


@pytest.mark.parametrize("prec,size", [(0, 23), (3, 13)])
def test_plan(monkeypatch, prec, size):
    from paper_2003_03868_amd import bsm
    a, b, _ = _operands((size,), 7)
    da, db = to_dev(a), to_dev(b)
    want = bsm.Matrix.empty_like(a.row_blk_size, b.col_blk_size)
    bsm.bsm_multiply(1.0, da.handle, db.handle, 0.0, want.handle, 0.0, 0, prec)
    monkeypatch.setenv("BSM_GROUP_BYTES", "64")
    dc = bsm.Matrix.empty_like(a.row_blk_size, b.col_blk_size)
    plan, _ = bsm.bsm_multiply_plan(1.0, da.handle, db.handle, dc.handle, 0.0, 0, prec)
    try:
        for _ in range(2):
            bsm.bsm_plan_execute(plan, da.handle, db.handle, dc.handle)
        assert np.array_equal(from_dev(dc).values, from_dev(want).values)
    finally:
        bsm.bsm_plan_destroy(plan)


def test_screening_has_groups_only(monkeypatch):
    from paper_2003_03868_amd import bsm
    a, b, c = _operands((13,), 9)
    da, db, dc = to_dev(a), to_dev(b), to_dev(c)
    monkeypatch.setenv("BSM_GROUP_BYTES", "64")
    with pytest.raises(bsm.BsmError) as e:
        bsm.bsm_multiply_screened(1.0, da.handle, db.handle, 0.0, dc.handle, 0.0, 0, 1e-3)
    assert e.value.status == bsm.ENOMEM
    assert np.array_equal(from_dev(dc).values, c.values)


@pytest.mark.parametrize("graph", [0, 1])
def test_sign(monkeypatch, graph):
    from paper_2003_03868_amd import bsm
    h = synth.neighbour_hamiltonian(96, 13, cutoff=4.5, seed=4)
    out = []
    for limit in (None, "64"):
        if limit:
            monkeypatch.setenv("BSM_GROUP_BYTES", limit)
        d = to_dev(h)
        o = bsm.bsm_sign_opts_default()
        o.eps_filter, o.tol, o.use_graph = 1e-6, 1e-8, graph
        st, xh, stats = bsm.bsm_sign_iterate(d.handle, 0.0, o)
        assert st == bsm.OK, bsm.bsm_last_error()
        out.append(from_dev(bsm.Matrix(xh, h.row_blk_size, h.col_blk_size)))
        assert limit is None or stats.graph_replays == 0
    assert np.array_equal(out[0].col_idx, out[1].col_idx)
    assert np.array_equal(out[0].values, out[1].values)
