"""GPU parity of the level-0 strokes in the blocks that large boxes take: 8 and 16 wavefronts (18 and 42
lines of outputs) and slabs of up to 57 planes, element by element, where lines keep their rows
from end to end and where they change after runs of planes (several changes inside a slab).

The boxes are too large for the oracle's setup, so one V-cycle is put together, in fp64, from the
component entry points, whose level-0 kernels work step by step and not by strokes, and which
the parity tests hold to the oracle on small boxes: with S(f) the smoother from zero,
  x = S(f); x += P V(P^T (f - A x)); x += S(f - A x)
on each level and the coarsest operator's inverse at the end.  Bounds: max |got - want| over max
|want|, fp64 1e-11 and mixed 1e-4, as for the V-cycle in the parity tests.

`tile` repeats the choice of a stroke's block, so that a case whose block changes is noticed; that
strokes ran shows in the kernel timer (2 launches of class 0 per launch of class 3)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu


def section(nx, ny, size):
    y, x = np.meshgrid(np.linspace(-1, 1, ny), np.linspace(-1, 1, nx), indexing="ij")
    m = np.abs(x) ** 6 + np.abs(y) ** 6 < size
    m[0] = m[-1] = m[:, 0] = m[:, -1] = False
    return m


def live(sec, columns, lines):
    """Tiles of the cross-section that hold an unknown."""
    ny, nx = sec.shape
    p = np.zeros((-(-ny // lines) * lines, -(-nx // columns) * columns), dtype=bool)
    p[:ny, :nx] = sec
    return int(p.reshape(p.shape[0] // lines, lines, -1, columns).any(axis=(1, 3)).sum())


def tile(sec, nz, precision, up):
    """Wavefronts of a block and planes of a slab."""
    fp32 = precision == sa.MIXED
    a, b = (0.38, 0.20) if fp32 else (0.15, 0.36)
    best = None
    for w in (4, 8, 16) if fp32 else (4, 8):
        per_cu, n = (16 if fp32 else 8) // w, live(sec, 60 if up else 57, 3 * (w - 2))
        for s in range(3, 58, 3):
            full, rest = divmod(n * -(-nz // s), 256 * per_cu)
            t = full * (a + b * w / 4 * per_cu) + (a + b * w / 4 * -(-rest // 256) if rest else 0.0)
            if best is None or 4.0 + (s + 6) * t < best[0]:
                best = (4.0 + (s + 6) * t, w, s)
    return best[1:]


def domain(nx, ny, nz, runs):
    """A pipe whose radius and wall fractions are those of a run of planes."""
    run = np.repeat(np.arange(nz), np.resize(runs, nz))[:nz]
    sections = [section(nx, ny, size) for size in (0.97, 0.85, 0.92)]
    m = np.zeros((nz, ny, nx), dtype=bool)
    for z in range(1, nz - 1):
        m[z] = sections[run[z] % 3]
    frac = np.random.default_rng(1).uniform(0.2, 0.95, (4, 7, nx * ny))
    node, dr, s = [], [], []
    for d in range(4):
        n = np.flatnonzero(m & ~np.roll(m, 1 if d % 2 == 0 else -1, axis=2 - d // 2))
        node.append(n)
        dr.append(np.full(n.size, d, dtype=np.uint8))
        s.append(frac[d, run[n // (nx * ny)] % 7, n % (nx * ny)])
    node, dr, s = map(np.concatenate, (node, dr, s))
    o = np.argsort(8 * node + dr)
    return sa.HostDomain(m, (0.05, 0.06, 0.07), node[o], dr[o], s[o]), sections[0]


def vcycle(G, info, l, f):
    dims = [d[::-1] for d in info["dims"]]
    if l == info["n_levels"] - 1:
        rows, inv = sa.coarse_inverse(G)
        x = np.zeros(f.size)
        x[rows] = inv @ f.reshape(-1)[rows]
        return x.reshape(dims[l])
    op = lambda kind, v, out: sa.level_apply(G, l, kind, v, dims[out], sa.FP64)
    x = op(sa.capi.OP_PRESMOOTH, f, l)
    fc = op(sa.capi.OP_RESTRICT, f - op(sa.capi.OP_APPLY, x, l), l + 1)
    x += op(sa.capi.OP_PROLONG, vcycle(G, info, l + 1, fc), l)
    x += op(sa.capi.OP_PRESMOOTH, f - op(sa.capi.OP_APPLY, x, l), l)
    return x


STRAIGHT, SHORT, LONG = [100000], [2, 9, 14, 5, 20, 1, 3], [24, 40, 17, 31]
BOTH, MIXED = (sa.FP64, sa.MIXED), (sa.MIXED,)
# box, runs of planes, precisions, {precision: tiles (wavefronts, planes) of the down- and up-stroke}
CASES = {
    "119x127x311": ((119, 127, 311), STRAIGHT, BOTH, {sa.MIXED: [(16, 12), (8, 9)], sa.FP64: [(8, 27), (8, 18)]}),
    "119x127x311 runs": ((119, 127, 311), SHORT, BOTH, {sa.MIXED: [(16, 12), (8, 9)], sa.FP64: [(8, 27), (8, 18)]}),
    "62x170x685 runs": ((62, 170, 685), SHORT, BOTH, {sa.MIXED: [(8, 27), (8, 27)], sa.FP64: [(8, 54), (8, 51)]}),
    "240x127x390": ((240, 127, 390), STRAIGHT, BOTH, {sa.MIXED: [(16, 24), (16, 21)], sa.FP64: [(8, 57), (8, 45)]}),
    "240x127x390 runs": ((240, 127, 390), LONG, BOTH, {sa.MIXED: [(16, 24), (16, 21)], sa.FP64: [(8, 57), (8, 45)]}),
    "115x211x690 runs": ((115, 211, 690), SHORT, MIXED, {sa.MIXED: [(16, 30), (16, 30)]}),
    "256x256x768 runs": ((256, 256, 768), LONG, MIXED, {sa.MIXED: [(16, 54), (16, 54)]}),
}


@pytest.mark.parametrize("name", CASES)
def test_vcycle_in_the_blocks_of_large_boxes(name):
    dims, runs, precisions, tiles = CASES[name]
    dom, sec = domain(*dims, runs)
    for precision in precisions:
        print(f"[case] strokes {name} precision={precision}", flush=True)
        assert [tile(sec, dims[2], precision, up) for up in (False, True)] == tiles[precision]
        G = sa.setup(dom, W.VARIANT_QUAD, sa.default_options(precision=precision))
        r = W.random_box_vector(dims, 5) * dom.mask
        z = torch.zeros(r.size, dtype=torch.float64, device="cuda")
        for k in ("l0_cheb", "l0_prolong"):
            sa.capi.timer_enable(k, True)
        sa.capi.timer_reset()
        sa.precond_apply(G, torch.from_numpy(r.reshape(-1)).cuda(), z)
        n = [sa.capi.timer_read(k)[1] for k in ("l0_cheb", "l0_prolong")]
        for k in ("l0_cheb", "l0_prolong"):
            sa.capi.timer_enable(k, False)
        sa.capi.timer_reset()
        got = z.cpu().numpy().reshape(r.shape)
        want = vcycle(G, sa.hierarchy_info(G), 0, r)
        sa.destroy(G)
        err = np.abs(got - want).max() / np.abs(want).max()
        print(f"launches {n}, error {err:.2e}", flush=True)
        assert n[0] == 2 * n[1] == 2
        assert np.all(got[dom.mask == 0] == 0)
        assert err <= (1e-11 if precision == sa.FP64 else 1e-4)


# iterations of the solves to 1e-8 with the V-cycle step by step (its level-0 kernels before the
# strokes; both precisions the same)
ITERATIONS = {"ell128": 17, "ell256_mixed": 22, "ell256_lin_mixed": 22, "cyl192_mixed": 17}


@pytest.mark.parametrize("precision", [sa.FP64, sa.MIXED])
@pytest.mark.parametrize("name", ITERATIONS)
def test_large_solves_take_the_iterations_of_the_step_kernels(name, precision):
    print(f"[case] iterations {name} precision={precision}", flush=True)
    w = W.by_name(name)
    b = torch.from_numpy(W.rhs(w).reshape(-1)).cuda()
    x = torch.zeros_like(b)
    G = sa.setup(sa.domain_for(w.shape, w.nx, w.ny, w.nz), w.variant, sa.default_options(precision=precision))
    res = sa.solve(G, b, x, tol=1e-8)
    sa.destroy(G)
    print(f"iterations {res['iterations']}", flush=True)
    assert res["status"] == 0 and abs(res["iterations"] - ITERATIONS[name]) <= 1
