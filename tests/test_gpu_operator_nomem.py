"""saamg_set_operator that runs out of memory at any of its allocations reports it, leaves nothing
behind, and later solves iterate either with the operator that was set before or with the
hierarchy's own."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu


class Limited(sa.TorchAllocator):
    """torch's allocator, failing from the given allocation on (None: never)."""

    left = None

    def _alloc(self, ctx, nbytes, stream):
        if self.left is not None:
            if self.left == 0:
                return None
            self.left -= 1
        return super()._alloc(ctx, nbytes, stream)


@pytest.mark.parametrize("dims", [(35, 29, 37), (61, 49, 161)])  # prepared on the host, on the device
@pytest.mark.parametrize("precision", [sa.FP64, sa.MIXED])
def test_every_allocation_of_an_operator(dims, precision):
    print(f"[case] operator out of memory {dims} precision={precision}", flush=True)
    first, second, third = (sa.domain_for(W.Shape.ellipse(1.0, 0.6, z), *dims) for z in (4.0, 4.3, 4.6))
    al = Limited()
    G = sa.setup(first, W.VARIANT_QUAD, sa.default_options(allocator=al, precision=precision))
    b = torch.rand(first.mask.size, dtype=torch.float64, device="cuda")

    def solution():
        x = torch.zeros_like(b)
        assert sa.solve(G, b, x)["status"] == 0
        return x

    own = solution()
    sa.set_operator(G, second)
    with_second = solution()
    assert not torch.equal(own, with_second)
    sa.refresh(G, first)
    assert torch.equal(solution(), own)
    held = al.outstanding_bytes
    k = 0
    while True:  # no operator set: H stays as it is
        al.left = k
        try:
            sa.set_operator(G, second)
        except sa.SaamgError as e:
            al.left = None
            assert e.status == sa.capi.NOMEM
            assert al.outstanding_bytes == held
            assert torch.equal(solution(), own)
        else:
            break
        k += 1
    al.left = None
    assert k > 5 and torch.equal(solution(), with_second)
    print(f"{k} allocations", flush=True)
    for j in range(k - 3):  # one set: it stays, or H's own comes back
        al.left = j
        with pytest.raises(sa.SaamgError):
            sa.set_operator(G, third)
        al.left = None
        x = solution()
        assert torch.equal(x, with_second) or torch.equal(x, own)
        sa.set_operator(G, second)
    sa.destroy(G)
    assert al.outstanding_bytes == 0
