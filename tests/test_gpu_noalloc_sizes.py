"""The allocation-free solve serves the boxes it served before its level-0 kernels took blocks of
their own: with long slabs asked for (32 planes), a box whose work vectors leave 4,720 bytes of
the 64 MiB array free has 484 stroke blocks where the step kernels would have 130, and their
partial sums may take no room of their own.  The result is saamg_solve's, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu


def test_a_box_that_fills_the_array():
    nx, ny, nz = 110, 129, 62
    print(f"[case] allocation-free solve of {nx}x{ny}x{nz}", flush=True)
    m = np.zeros((nz, ny, nx), dtype=np.uint8)
    m[1:-1, 1:-1, 1:-1] = 1
    e = np.zeros(0)
    G = sa.setup(sa.HostDomain(m, (1.0, 1.0, 1.0), e, e, e), sa.VARIANT_CONST,
                 sa.default_options(l0_planes=32, l0_tile_x=2))
    b = torch.from_numpy(np.random.default_rng(1).uniform(0, 1, m.size)).cuda()
    x, y = torch.zeros_like(b), torch.full_like(b, 7.0)
    want = sa.solve(G, b, x)
    got = sa.solve_noalloc(G, b, y)
    assert got["status"] == 0 and got["iterations"] == want["iterations"]
    assert torch.equal(x, y)
    sa.destroy(G)
