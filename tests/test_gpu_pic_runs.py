"""Particle coupling where its work is split: runs of equal cells at the edges of the chunks of
sorted particles, run sums kept by cell or by particle, particles in every cell up to the
walls and open ends, and outside, against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import grid, pic

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu

# fp64 sums of up to a few thousand terms in another order than the oracle's
TOL = 1e-12


def _points(kind, n, g, rng):
    nl = np.array(g.lattice)
    lo, h = np.array(g.origin), np.array(g.h)
    if kind == "cell":        # one cell in the middle
        u = nl // 2 + rng.uniform(0.0, 1.0, (n, 3))
    elif kind == "few":       # runs of about 90 in cells of the first and the last row
        u = rng.uniform(0.0, 1.0, (n, 3))
        u[:, 0] += rng.integers(0, nl[0] - 1, n)
        u[n // 2:, 1:] += nl[1:] - 2
    else:                     # everywhere, a shell outside included
        u = rng.uniform(-1.0, 1.0, (n, 3)) * (nl + 1) / 2 + (nl - 1) / 2
        u[: n // 8] = np.floor(u[: n // 8])  # on lattice nodes and planes
    return lo + h * u


@pytest.mark.parametrize("robin", [False, True])
@pytest.mark.parametrize("kind,n,cap", [
    ("cell", 1, 1), ("cell", 256, 256), ("cell", 257, 100_000), ("cell", 4000, 4000),
    ("few", 3000, 3000), ("few", 3000, 100_000),
    ("all", 255, 300), ("all", 20_000, 20_000), ("all", 20_000, 100_000),
])
def test_deposit_and_gather_where_the_work_is_split(kind, n, cap, robin):
    nx, ny, nz = 18, 23, 29
    print(f"[case] pic split {kind} n={n} cap={cap} robin={robin}", flush=True)
    shape = W.Shape.ellipse(1.0, 0.6, 4.0)
    dom = sa.domain_for(shape, nx, ny, nz, open_ends=robin)
    origin = (-shape.a, -shape.b, -0.5 * shape.length)
    og = grid.from_shape(shape, nx, ny, nz, robin=robin)
    g = pic.Grid((og.nx, og.ny, og.nz), int(robin), origin, og.h, og.robin_d)
    rng = np.random.default_rng(n + cap)
    pts = _points(kind, n, g, rng)
    P = sa.pic_create(dom, origin, cap)
    dev = torch.device("cuda:0")
    pos = torch.from_numpy(pts).to(dev)
    rho = torch.full((dom.mask.size,), np.nan, dtype=torch.float64, device=dev)
    sa.pic_deposit(P, pos, -0.37, rho)
    got, want = rho.cpu().numpy(), pic.deposit(g, pts, -0.37).reshape(-1)
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    assert not got[want == 0.0].any()
    phi = rng.standard_normal(dom.mask.size)
    E = torch.full_like(pos, np.nan)
    sa.pic_gather(P, torch.from_numpy(phi).to(dev), pos, E)
    want = pic.gather(g, phi.reshape(og.mask.shape), og.mask, pts)
    assert np.abs(E.cpu().numpy() - want).max() <= TOL * np.abs(want).max()
