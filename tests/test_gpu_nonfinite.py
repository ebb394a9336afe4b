"""Non-finite values stay inside the domain, and inside their call.

The fused level-0 kernels multiply the zero coefficients of nodes that are no unknowns with
their neighbours' values, so an Inf or NaN reaches those nodes of the work vectors.  What a
caller gets back holds 0 there all the same, and the next call on the hierarchy gives, bit
for bit, what a hierarchy without that history gives.  Boxes on one-node lanes below and above
the size from which the CG passes run by columns (600 thousand unknowns), and on 16-byte
lanes."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu

SHAPE = W.Shape.ellipse(1.0, 0.9, 1.5)
BOXES = {"small": (61, 49, 57), "columns": (125, 109, 77), "wide": (132, 60, 50)}


def setup(name, precision):
    dom = sa.domain_for(SHAPE, *BOXES[name])
    if name == "columns":
        assert dom.n_unknowns >= 600000
    G = sa.setup(dom, W.VARIANT_QUAD, sa.default_options(precision=precision))
    assert sa.hierarchy_info(G)["l0_wide"] == int(name == "wide")
    rng = np.random.default_rng(2)
    b = np.where(dom.mask.reshape(-1) > 0, rng.uniform(0.5, 1.0, dom.mask.size), 0.0)
    return G, torch.from_numpy(b).cuda(), torch.from_numpy(dom.mask.reshape(-1) == 0).cuda()


def clean(name, precision):
    G, b, _ = setup(name, precision)
    z, x = torch.zeros_like(b), torch.zeros_like(b)
    sa.precond_apply(G, b, z)
    assert sa.solve(G, b, x)["status"] == 0
    sa.destroy(G)
    return z, x


@pytest.mark.parametrize("precision", [sa.FP64, sa.MIXED])
@pytest.mark.parametrize("name", BOXES)
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_preconditioner(name, precision, value):
    print(f"[case] preconditioner of {value}, {name} precision={precision}", flush=True)
    G, b, out = setup(name, precision)
    r = b.clone()
    r[torch.nonzero(~out)[int((~out).sum()) // 3]] = value
    z = torch.full_like(b, 7.0)
    sa.precond_apply(G, r, z)
    assert not torch.isfinite(z[~out]).all()
    assert torch.all(z[out] == 0)
    z2, x2 = clean(name, precision)
    z, x = torch.zeros_like(b), torch.zeros_like(b)
    sa.precond_apply(G, b, z)
    assert torch.equal(z, z2)
    sa.precond_apply(G, r, z)
    assert sa.solve(G, b, x)["status"] == 0
    assert torch.equal(x, x2)
    sa.destroy(G)


@pytest.mark.parametrize("name", BOXES)
def test_a_residual_beyond_fp32(name):
    print(f"[case] residual beyond fp32, {name}", flush=True)
    G, b, out = setup(name, sa.MIXED)
    x = torch.full_like(b, 7.0)
    res = sa.solve(G, 1e150 * b, x)  # finite in fp64, its fp32 copy is not
    assert res["status"] == sa.capi.NONFINITE
    assert torch.all(x[out] == 0)
    z2, x2 = clean(name, sa.MIXED)
    assert sa.solve(G, b, x)["status"] == 0
    assert torch.equal(x, x2)
    sa.destroy(G)


@pytest.mark.parametrize("name", BOXES)
@pytest.mark.parametrize("ring", [0, 2])
def test_x_holds_the_last_iterate_of_a_solve_that_breaks_down(name, ring):
    """The first step has no finite length, so the last iterate is the initial guess: 0, or x0 up to
    the rounding of its scaling and back."""
    print(f"[case] last iterate, {name} ring={ring}", flush=True)
    dom = sa.domain_for(SHAPE, *BOXES[name])
    G = sa.setup(dom, W.VARIANT_QUAD, sa.default_options(precision=sa.MIXED, cg_ring=ring))
    inside = torch.from_numpy(dom.mask.reshape(-1) > 0).cuda()
    b = 1e150 * inside.double()
    x = torch.full_like(b, 7.0)
    assert sa.solve(G, b, x)["status"] == sa.capi.NONFINITE
    assert torch.all(x == 0)
    x0 = 0.75 * inside.double()
    assert sa.solve(G, b, x, x0=x0)["status"] == sa.capi.NONFINITE
    assert (x - x0).abs().max() <= 4 * 2.0 ** -53 * 0.75
    sa.destroy(G)
