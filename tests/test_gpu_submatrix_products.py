"""The submatrix method's dense products at the edges of their tiles, for a
matrix that equals its transpose (half of each product computed), one that
does not, and one that misses it by one bit of one element.

Every block is stored, so each submatrix is the whole matrix; the reference
is the same iteration in numpy float64.  Both stop at ||X^2 - I||_F / n <
1e-12, which bounds ||X - sign||_F by n tol / 2 <= 1e-10 (n <= 200), rounding
adds about n 2^-52 times the iteration's amplification of a few: 1e-9."""
import numpy as np
import pytest

from synth import BSR
from tests.gpu_util import from_dev, need_gpu, to_dev

pytestmark = pytest.mark.gpu

TOL = 1e-9


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _density(t):
    x = t / np.abs(t).sum(1).max()
    for _ in range(100):
        y = x @ x
        if np.linalg.norm(y - np.eye(len(t))) / len(t) < 1e-12:
            return 0.5 * (np.eye(len(t)) - x)
        x = 1.5 * x - 0.5 * x @ y
    raise AssertionError("reference iteration did not converge")


def _blocks(d, nb, b):
    vals = d.reshape(nb, b, nb, b).transpose(0, 2, 1, 3).reshape(-1)
    sizes = np.full(nb, b, dtype=np.int32)
    return BSR(sizes, sizes, np.arange(nb + 1, dtype=np.int64) * nb,
               np.tile(np.arange(nb, dtype=np.int32), nb), np.ascontiguousarray(vals))


# edges: 1, below and at the k depth, one past 32 and 64, 32 over a tile, the
# largest with four tiles, more than 64 block columns
@pytest.mark.parametrize("nb,b", [(1, 1), (3, 5), (1, 16), (2, 16), (11, 3), (4, 16), (5, 13),
                                  (4, 24), (8, 16), (25, 8), (70, 2)])
@pytest.mark.parametrize("kind", ["symmetric", "general", "one bit"])
def test_dense_products_at_tile_edges(nb, b, kind):
    from paper_2003_03868_amd import bsm
    n = nb * b
    rng = np.random.default_rng(1000 * nb + b)
    d = rng.standard_normal((n, n)) / (4.0 * np.sqrt(n))
    if kind != "general":
        d = 0.5 * (d + d.T)
    if kind == "one bit" and n > 1:
        d[n - 1, 0] = np.nextafter(d[n - 1, 0], 2.0)
    d[np.arange(n), np.arange(n)] += np.where(rng.random(n) < 0.3, -1.5, 1.5)
    h = to_dev(_blocks(d, nb, b))
    o = bsm.bsm_sign_opts_default()
    o.eps_filter, o.tol, o.max_iter = 0.0, 1e-12, 100
    st, ph, stats = bsm.bsm_submatrix_density(h.handle, 0.0, o)
    assert st == bsm.OK, bsm.bsm_last_error()
    sizes = np.full(nb, b, dtype=np.int32)
    p = from_dev(bsm.Matrix(ph, sizes, sizes))
    ref = _blocks(_density(d), nb, b)
    assert np.array_equal(p.row_ptr, ref.row_ptr) and np.array_equal(p.col_idx, ref.col_idx)
    err = np.abs(p.values - ref.values).max()
    print(f"n {n} {kind}: err {err:.2e}, {stats.max_iterations} iterations")
    assert err < TOL
