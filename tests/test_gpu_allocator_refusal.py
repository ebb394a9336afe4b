"""A setup that refuses a domain has not asked the caller's allocator for anything, however large the
domain (those of 16384 wall entries and more are otherwise checked on the device), and one
that takes it builds the hierarchy that the library's own pool gives, bit for bit."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu

SHAPE, DIMS = W.Shape.cylinder(1.0, 2.0), (51, 51, 114)


def domain(open_ends=False):
    d = sa.domain_for(SHAPE, *DIMS, open_ends=open_ends)
    assert d.wall_node.size >= 16384
    return d


def face(d):
    d.mask[d.nz // 2, d.ny // 2, 0] = 1


def fraction(d):
    d.wall_s[-1] = 0.0


def node(d):
    d.wall_node[-1] = -1


def twice(d):
    d.wall_node[-1], d.wall_dir[-1] = d.wall_node[-2], d.wall_dir[-2]


@pytest.mark.parametrize("spoil,message", [(face, "face of the box"), (fraction, "wall fraction"),
                                           (node, "out of range"), (twice, "duplicate")])
def test_nothing_is_allocated_for_a_refused_domain(spoil, message):
    print(f"[case] refused domain and the caller's allocator: {message}", flush=True)
    al = sa.TorchAllocator()
    dom = domain()
    spoil(dom)
    with pytest.raises(sa.SaamgError, match=message):
        sa.setup(dom, W.VARIANT_QUAD, sa.default_options(allocator=al))
    assert (al.n_alloc, al.n_free) == (0, 0)


@pytest.mark.parametrize("options,message", [({"l0_wide": 2}, "multiple of 4"), ({"l0_tile_x": 2}, "exceeds")])
def test_nothing_is_allocated_for_an_option_that_does_not_fit_the_box(options, message):
    print(f"[case] refused option and the caller's allocator: {message}", flush=True)
    dom, bad = domain(), domain()
    face(bad)
    for alloc in (sa.TorchAllocator(), None):
        with pytest.raises(sa.SaamgError, match=message):
            sa.setup(dom, W.VARIANT_QUAD, sa.default_options(allocator=alloc, **options))
        with pytest.raises(sa.SaamgError, match="face of the box"):  # the domain's errors come first
            sa.setup(bad, W.VARIANT_QUAD, sa.default_options(allocator=alloc, **options))
        if alloc is not None:
            assert (alloc.n_alloc, alloc.n_free) == (0, 0)


@pytest.mark.parametrize("open_ends", [False, True])
def test_the_hierarchy_is_that_of_the_pool(open_ends):
    print(f"[case] the caller's allocator, open={open_ends}", flush=True)
    al = sa.TorchAllocator()
    dom = domain(open_ends)
    got = []
    for alloc in (al, None):
        G = sa.setup(dom, W.VARIANT_QUAD, sa.default_options(allocator=alloc))
        dims = sa.hierarchy_info(G)["dims"]
        got.append([sa.level_coefficients(G, l, q) for l, q in enumerate(dims)])
        sa.destroy(G)
    assert al.n_alloc > 0 and al.outstanding_bytes == 0
    for a, b in zip(*got):
        assert np.array_equal(a, b)
