"""FP64 solves on one right-hand side take 18-real links for every value of `links` that is not 12 or 8 (a
parameter struct of zeros), on lattices of either kind of kernel."""
import pytest
import torch

from paper_1805_03560_amd import synth, whmc

from gpu_util import make_ctx, pack_half

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [None, 0])   # 0: one thread per site
@pytest.mark.parametrize("links", [0, 5])
def test_other_link_values_are_18_real(links, schedule):
    dims = (4, 4, 6, 6)
    ctx = make_ctx(dims, synth.smooth_links(dims, 9510))
    if schedule is not None:
        ctx.set_option(whmc.OPT_HOP_SCHEDULE, schedule)
    b = pack_half(ctx, synth.gaussian_spinor(ctx.Vh, 9511))
    ref, st = ctx.cg_solve(b, [0.14], whmc.cg_params(tol=1e-12))
    x, st1 = ctx.cg_solve(b, [0.14], whmc.cg_params(tol=1e-12, links=links))
    assert st1[0]["converged"] and st1[0]["iters"] == st[0]["iters"] and torch.equal(x, ref)
