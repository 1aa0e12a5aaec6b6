"""A captured whmc_apply_MdagM replayed after eager calls on more right-hand sides, which need larger scratch:
the replays give the eager results, and write nothing but their own buffers."""
import pytest
import torch

from paper_1805_03560_amd import synth, whmc

from gpu_util import make_ctx

pytestmark = pytest.mark.gpu


# the direction-split kernels, and the sweep kernels (V_h = 32768)
@pytest.mark.parametrize("dims", [(6, 4, 6, 8), (16, 16, 16, 16)])
@pytest.mark.parametrize("eo", [True, False])
@pytest.mark.parametrize("n", [1, 3])
def test_replay_after_larger_calls(dims, eo, n):
    stream = torch.cuda.Stream()
    ctx = whmc.Context(dims, stream=stream)
    gen = torch.Generator(device="cuda").manual_seed(9500)
    size = (24 if eo else 48) * ctx.Vh
    x = torch.randn(16 * size, dtype=torch.float64, device="cuda", generator=gen)
    U = make_ctx(dims, synth.smooth_links(dims, 9501, width=0.8)).export_gauge()
    torch.cuda.synchronize()
    kappas = [0.10 + 0.002 * r for r in range(16)]
    with torch.cuda.stream(stream):
        ctx.load_gauge(U, unitarity_tol=0.0)
        ref = ctx.apply_MdagM(x[:n * size], kappas[:n], eo=eo).clone()
        out = torch.zeros_like(ref)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        ctx.apply_MdagM(x[:n * size], kappas[:n], out=out, eo=eo)
    for m in (n + 1, 16):
        with torch.cuda.stream(stream):
            big = ctx.apply_MdagM(x[:m * size], kappas[:m], eo=eo)
        other = torch.full((8 * size,), 7.0, dtype=torch.float64, device="cuda")
        for _ in range(2):
            out.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
        assert torch.equal(big[:n * size], ref) and bool((other == 7.0).all())
