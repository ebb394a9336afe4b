"""GPU parity of the Galerkin product of level 0 where most aggregates have only interior rows
around them and take one column formed for all: patches of 9 nodes that straddle
the 64-node words of the masks, both storages (symmetric and full), open ends.  Every coefficient of every coarse level against the
oracle's, max |got - want| over max |want| 1e-12, the bound of test_gpu_parity.  The boxes of
33,748 and 33,120 aggregates take the shared column, the small one (fewer than 32,768) does not."""
import numpy as np
import pytest

import workloads as W
from oracle import amg, solve

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu

CYL, ELL = W.Shape.cylinder(1.0, 2.0), W.Shape.ellipse(1.0, 0.6, 2.0)


def _coef(lv):
    mx, my, mz = lv.dims
    c = amg.coarse_box_coords(lv)
    A = lv.A.tocoo()
    d = c[A.col] - c[A.row]
    k = (d[:, 0] + 1) + 3 * (d[:, 1] + 1) + 9 * (d[:, 2] + 1)
    out = np.zeros((27, mz, my, mx))
    out[k, c[A.row, 2], c[A.row, 1], c[A.row, 0]] = A.data
    return out


@pytest.mark.parametrize("shape,nx,ny,nz,variant,open_ends", [
    (CYL, 75, 40, 22, W.VARIANT_LIN, False),
    (ELL, 76, 31, 353, W.VARIANT_LIN, False),
    (CYL, 134, 24, 274, W.VARIANT_QUAD, True),
])
def test_coarse_operators_with_interior_aggregates(shape, nx, ny, nz, variant, open_ends):
    print(f"[case] galerkin {shape.name} {nx}x{ny}x{nz} variant {variant}", flush=True)
    sys_, H = solve.build(shape, nx, ny, nz, variant, robin=open_ends)
    dom = sa.domain_for(shape, nx, ny, nz, open_ends=open_ends)
    G = sa.setup(dom, variant, sa.default_options())
    assert sa.hierarchy_info(G)["n_levels"] == len(H.levels)
    for l, lv in enumerate(H.levels):
        got, want = sa.level_coefficients(G, l, lv.dims), _coef(lv)
        assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max(), l
    sa.destroy(G)
