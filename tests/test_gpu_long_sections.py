"""Solves on boxes whose cross-section (x, y) is longer than 65,536 tiles of a fused level-0 kernel
along x or 32,768 along y.

The box is full (unknowns everywhere but on the faces), with the constant wall rule and unit
spacings, so the system is the 7-point Laplacian with 6 on the diagonal: the true residual is
formed here from shifted arrays, on every node.  A solve to 1e-8 that leaves no line out meets
1e-8 (plus the rounding of the check, 1e-12) and takes the iterations of a shorter box of
the same section, up to two."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu


def solve(nx, ny, nz, precision):
    m = np.zeros((nz, ny, nx), dtype=np.uint8)
    m[1:-1, 1:-1, 1:-1] = 1
    e = np.zeros(0)
    G = sa.setup(sa.HostDomain(m, (1.0, 1.0, 1.0), e, e, e), sa.VARIANT_CONST,
                 sa.default_options(precision=precision))
    g = torch.Generator("cuda")
    g.manual_seed(1)
    b = torch.rand((nz, ny, nx), dtype=torch.float64, device="cuda", generator=g)
    x = torch.zeros_like(b)
    res = sa.solve(G, b, x, tol=1e-8)
    sa.destroy(G)
    inner = (slice(1, -1),) * 3
    r = b[inner] - 6.0 * x[inner]
    for axis in range(3):
        for o in (0, 2):
            sl = [slice(1, -1)] * 3
            sl[axis] = slice(o, x.shape[axis] - 2 + o)
            r += x[tuple(sl)]
    return res, float(r.norm() / b[inner].norm())


@pytest.mark.parametrize("precision", [sa.FP64, sa.MIXED])
@pytest.mark.parametrize("dims,short", [((5, 196700, 5), (5, 3001, 5)), ((4100001, 5, 5), (3001, 5, 5))])
def test_every_tile_of_a_long_section_is_solved(dims, short, precision):
    print(f"[case] long section {dims} precision={precision}", flush=True)
    want, _ = solve(*short, precision)
    res, rel = solve(*dims, precision)
    print(f"iterations {res['iterations']} ({want['iterations']} at {short}), residual {rel:.2e}", flush=True)
    assert res["status"] == 0 and rel <= 1e-8 + 1e-12
    assert abs(res["iterations"] - want["iterations"]) <= 2
