"""The coarsest level's explicit inverse at the edges of its blocks of 32 pivots, strips of 64
columns and groups of 32 rows (single-level hierarchies, the inverse of the level-0 operator
with quadratic, nonsymmetric rows): against numpy's, max |got - want| over max |want| 1e-12, the
bound of test_gpu_parity."""
import numpy as np
import pytest

import workloads as W
from oracle import solve

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,n", [(4, 4, 8), (4, 6, 16), (5, 4, 18), (4, 10, 32), (4, 11, 36), (6, 5, 48),
                                     (5, 9, 63), (6, 6, 64), (5, 10, 72), (6, 10, 128), (8, 8, 192),
                                     (9, 9, 315)])
def test_inverse_at_block_edges(nx, nz, n):
    print(f"[case] dense inverse of {n}", flush=True)
    shape = W.Shape.cylinder(1.0, 2.0)
    _, H = solve.build(shape, nx, nx, nz, W.VARIANT_QUAD)
    G = sa.setup(sa.domain_for(shape, nx, nx, nz), W.VARIANT_QUAD, sa.default_options())
    rows, inv = sa.coarse_inverse(G)
    sa.destroy(G)
    assert H.levels[-1].n == n and np.array_equal(rows, H.levels[-1].lin)
    want = np.linalg.inv(H.levels[-1].A.toarray())
    assert np.abs(inv - want).max() <= 1e-12 * np.abs(want).max()
