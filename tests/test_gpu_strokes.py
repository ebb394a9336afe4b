"""GPU parity of the fused level-0 strokes of the V-cycle where their tiling can go wrong.

A stroke's block takes 57 (down) or 60 (up) columns and 6, 18 or 42 lines of the lattice and
marches slabs of a multiple of 3 planes with 3 (2) halo nodes on every side, and keeps a
line's stencil rows from plane to plane while the line does not change.  The cases put the
lattice's edges on, one before and one after those of the tiles, and the "runs" domains change
their cross-section along z after 1, 2, 3 and more planes, without cut walls (planes of a run
share their rows, up to the end planes' missing neighbours) and with a different fraction at
every wall node (no plane shares its rows).  Their coarse levels, whose strokes take tiles of 6^3
nodes, have edges on, before and after those of the tiles as well.

One V-cycle against the oracle's, element by element, max |got - want| over max |want|: fp64
1e-11 and mixed 1e-4, the bounds of the V-cycle in test_gpu_parity (summation order, and fp32
rounding carried through every level).
"""
import numpy as np
import pytest

import workloads as W
from oracle import amg, grid, operator, solve

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu

CYL, ELL, BOX = W.Shape.cylinder(1.0, 2.0), W.Shape.ellipse(1.0, 0.6, 2.0), W.Shape.boxbore(0.8, 4.0)
PIPES = {
    "57x18x54": (ELL, 57, 18, 54, W.VARIANT_QUAD, False),
    "58x19x55": (CYL, 58, 19, 55, W.VARIANT_LIN, False),
    "60x43x57_open": (ELL, 60, 43, 55, W.VARIANT_QUAD, True),
    "61x6x60": (CYL, 61, 6, 60, W.VARIANT_CONST, False),
    "115x42x9": (ELL, 115, 42, 9, W.VARIANT_LIN, False),
    "121x44x31_box": (BOX, 121, 44, 31, W.VARIANT_LIN, False),
    "30x30x31_box_open": (BOX, 30, 30, 31, W.VARIANT_QUAD, True),
}


def emax(got, want):
    return np.abs(got - want).max() / max(np.abs(want).max(), 1e-300)


def check(dom, sys_, H, G, precision, name):
    r = W.random_box_vector((dom.nx, dom.ny, dom.nz), 5) * dom.mask
    want = amg.vcycle(H, sys_.gather(r))
    z = torch.zeros(r.size, dtype=torch.float64, device="cuda:0")
    sa.precond_apply(G, torch.from_numpy(r.reshape(-1)).to("cuda:0"), z)
    zc = z.cpu().numpy()
    e = emax(sys_.gather(zc), want)
    print(f"[{name}] precision={precision} vcycle emax={e:.2e}", flush=True)
    assert np.all(zc.reshape(dom.nz, dom.ny, dom.nx)[~dom.mask] == 0)
    assert e <= (1e-11 if precision == sa.FP64 else 1e-4)


@pytest.mark.parametrize("name", PIPES)
def test_vcycle_at_the_edges_of_the_tiles(name):
    shape, nx, ny, nz, variant, open_ends = PIPES[name]
    print(f"[case] strokes {name}", flush=True)
    sys_, H = solve.build(shape, nx, ny, nz, variant, robin=open_ends)
    for precision in (sa.FP64, sa.MIXED):
        G = sa.setup(sa.domain_for(shape, nx, ny, nz, open_ends), variant,
                     sa.default_options(precision=precision))
        check(sys_.dom, sys_, H, G, precision, name)
        sa.destroy(G)


def runs_domain(cut: bool) -> W.MaskDomain:
    """A pipe whose elliptic cross-section changes after runs of 1, 2, 3, 4, 1, 1, 2, ... planes."""
    nx, ny, runs = 64, 24, [1, 2, 3, 4, 1, 1, 2, 5, 3, 1, 2, 2, 6, 1]
    nz = sum(runs) + 2
    y, x = np.meshgrid(np.linspace(-1, 1, ny), np.linspace(-1, 1, nx), indexing="ij")
    m = np.zeros((nz, ny, nx), dtype=bool)
    z = 1
    for k, n in enumerate(runs):
        m[z:z + n] = x * x + y * y < (0.95 - 0.11 * (k % 4)) ** 2
        z += n
    e = np.zeros(0)
    node, d, s = W._wall_entries(m, np.random.default_rng(3), 0.3, 0.9) if cut else (
        e.astype(np.int64), e.astype(np.uint8), e)
    return W.MaskDomain((nx, ny, nz), (0.05, 0.06, 0.07), m, node, d, s)


@pytest.mark.parametrize("variant", [W.VARIANT_LIN, W.VARIANT_QUAD])
@pytest.mark.parametrize("cut", [False, True])
def test_vcycle_where_the_cross_section_changes_along_z(cut, variant):
    print(f"[case] strokes runs cut={cut} variant={variant}", flush=True)
    md = runs_domain(cut)
    nx, ny, nz = md.dims
    frac = np.ones((6, nz, ny, nx))
    frac[md.wall_dir.astype(np.int64), md.wall_node // (nx * ny), (md.wall_node // nx) % ny,
         md.wall_node % nx] = md.wall_s
    dom = grid.Domain(nx, ny, nz, md.h, md.mask.copy(), frac)
    sys_ = operator.assemble(dom, variant)
    H = amg.setup(sys_.As, md.dims, sys_.idx)
    for precision in (sa.FP64, sa.MIXED):
        G = sa.setup(sa.HostDomain(md.mask.astype(np.uint8), md.h, md.wall_node, md.wall_dir, md.wall_s),
                     variant, sa.default_options(precision=precision))
        check(dom, sys_, H, G, precision, f"runs cut={cut}")
        sa.destroy(G)


def test_solve_with_the_cg_passes_by_columns():
    """Narrow boxes from 600 thousand unknowns on take the CG passes whose blocks cover 62 columns,
    12 lines and 6 or 12 planes; lines of 2 * 62 + 1 nodes, 9 * 12 + 1 lines and a ragged last
    slab.  Bounds of the solves in test_gpu_parity: fp64 1e-8 with iterations +-1, mixed 1e-6
    against the oracle's 1e-13 solution."""
    shape, dims = W.Shape.ellipse(1.0, 0.9, 1.5), (125, 109, 77)
    print("[case] CG by columns, open ellipse", dims, flush=True)
    sys_, H = solve.build(shape, *dims, W.VARIANT_QUAD, robin=True)
    assert sys_.n >= 600000
    b = W.rhs(W.small(shape, *dims, W.VARIANT_QUAD, robin=True))
    o = solve.solve(sys_, H, b, tol=1e-8)
    tight = operator.unscale(sys_, solve.solve(sys_, H, b, tol=1e-13).x)
    want = operator.unscale(sys_, o.x)
    bt = torch.from_numpy(b.reshape(-1)).to("cuda:0")
    for precision in (sa.FP64, sa.MIXED):
        G = sa.setup(sa.domain_for(shape, *dims, True), W.VARIANT_QUAD, sa.default_options(precision=precision))
        x = torch.zeros_like(bt)
        res = sa.solve(G, bt, x, tol=1e-8)
        xg = x.cpu().numpy().reshape(sys_.dom.mask.shape)
        ref, lim = (want, 1e-8) if precision == sa.FP64 else (tight, 1e-6)
        err = np.linalg.norm(sys_.gather(xg) - ref) / np.linalg.norm(ref)
        print(f"precision={precision} oracle it={o.iterations} gpu it={res['iterations']} err={err:.2e}", flush=True)
        assert res["status"] == 0 and np.all(xg[~sys_.dom.mask] == 0) and err <= lim
        if precision == sa.FP64:
            assert abs(res["iterations"] - o.iterations) <= 1
        sa.destroy(G)


@pytest.mark.parametrize("precision", [sa.FP64, sa.MIXED])
def test_solve_by_columns_goes_on_from_the_true_residual(precision):
    """The recursive residual falls below a tolerance that the true one cannot meet: the solve
    forms the true residual (with the update x is still owed, in one pass), goes on from it, and
    ends at the iteration limit with the x of a solve to 1e-11: within 1e-8, that tolerance times
    a condition number below 1e3."""
    shape, dims = W.Shape.ellipse(1.0, 0.9, 1.5), (125, 109, 77)
    print("[case] CG by columns past the reachable tolerance", precision, flush=True)
    dom = sa.domain_for(shape, *dims)
    rng = np.random.default_rng(11)
    b = torch.from_numpy(np.where(dom.mask.reshape(-1) > 0, rng.uniform(0, 1, dom.mask.size), 0.0)).to("cuda:0")
    G = sa.setup(dom, W.VARIANT_LIN, sa.default_options(precision=precision))
    x, y = torch.zeros_like(b), torch.zeros_like(b)
    assert sa.solve(G, b, x, tol=1e-11)["status"] == 0
    with_limit = sa.solve(G, b, y, tol=1e-17, max_iter=60)
    print({k: with_limit[k] for k in ("iterations", "status", "replacements", "rel_res_true")}, flush=True)
    assert with_limit["replacements"] >= 1
    assert torch.isfinite(y).all()
    assert (x - y).norm() <= 1e-8 * x.norm()
    assert np.all(y.cpu().numpy()[dom.mask.reshape(-1) == 0] == 0)
    sa.destroy(G)
