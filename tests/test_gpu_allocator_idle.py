"""The allocator's free callback gets a block back only once no queued work uses it: whenever the
library frees during a setup, a re-setup and a change of the operator, the stream of
the call has nothing left to run."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
sa = pytest.importorskip("paper_0907_4863_amd")

pytestmark = pytest.mark.gpu


class Watch(sa.TorchAllocator):
    """torch's allocator, noting for each block freed whether the watched stream was idle."""

    def __init__(self, stream):
        super().__init__()
        self.stream = stream
        self.idle = []

    def _free(self, ctx, ptr, stream):
        self.idle.append(bool(self.stream.query()))
        super()._free(ctx, ptr, stream)


@pytest.mark.parametrize("precision", [sa.FP64, sa.MIXED])
@pytest.mark.parametrize("dims,variant", [((61, 49, 161), W.VARIANT_QUAD), ((132, 60, 90), W.VARIANT_LIN)])
def test_blocks_are_freed_on_an_idle_stream(dims, variant, precision):
    print(f"[case] frees on an idle stream {dims} variant={variant} precision={precision}", flush=True)
    stream = torch.cuda.Stream()
    al = Watch(stream)
    shape = lambda k: W.Shape.ellipse(1.0, 0.6, 4.0 + 0.3 * k)
    dom = [sa.domain_for(shape(k), *dims) for k in range(4)]
    b = torch.rand(dom[0].mask.size, dtype=torch.float64, device="cuda:0")
    x = torch.zeros_like(b)
    torch.cuda.synchronize()
    seen = {}

    def note(what):
        seen[what] = (len(al.idle), len(al.idle) - sum(al.idle))
        al.idle.clear()

    s = stream.cuda_stream
    G = sa.setup(dom[0], variant, sa.default_options(allocator=al, precision=precision), stream=s)
    note("setup")
    sa.refresh(G, dom[1], stream=s)
    note("refresh")
    sa.set_operator(G, dom[2], stream=s)
    note("operator")
    sa.set_operator(G, dom[3], stream=s)
    note("operator again")
    assert sa.solve(G, b, x, stream=s)["status"] == 0
    sa.refresh(G, dom[1], stream=s)
    note("refresh with an operator")
    sa.destroy(G)
    print({k: f"{n} frees, {busy} early" for k, (n, busy) in seen.items()}, flush=True)
    assert all(n > 0 and busy == 0 for n, busy in seen.values())
    assert al.outstanding_bytes == 0
