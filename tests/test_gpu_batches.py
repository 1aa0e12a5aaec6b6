"""Several masses at once with streamed links, and the solver whose update of p is part of the next hop, on lattices of
more than one XCD's blocks with part of a block."""
import pytest
import torch

from paper_1805_03560_amd import synth, whmc

from gpu_util import make_ctx, rel_err

pytestmark = pytest.mark.gpu


def _fields(ctx, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n * 24 * ctx.Vh, dtype=torch.float64, device="cuda", generator=gen)


# V_h = 32768 (16 masses a pass) and 35280 (14, the last of 128 sites short)
@pytest.mark.parametrize("dims,n", [((16, 16, 16, 16), 18), ((18, 14, 14, 20), 5)])
def test_streamed_mdagm_of_several_masses(dims, n):
    ctx = make_ctx(dims, synth.smooth_links(dims, 9560, width=0.8))
    kappas = [0.10 + 0.002 * r for r in range(n)]
    x = _fields(ctx, n, 9561)
    cached = ctx.apply_MdagM(x, kappas).clone()
    ctx.set_option(whmc.OPT_STREAM_THRESHOLD, 0)
    out = ctx.apply_MdagM(x, kappas)
    assert torch.equal(out, cached)
    for r in (0, n - 1):
        one = ctx.apply_MdagM(x.chunk(n)[r].clone(), [kappas[r]])
        assert torch.equal(out.chunk(n)[r], one), r
    assert torch.equal(ctx.apply_MdagM_noalloc(x, kappas, torch.full_like(x, float("nan"))), out)


# V_h = 7560 (119 blocks) and 1080; the bounds are those of the solves against the oracle at the same tolerances
@pytest.mark.parametrize("prec,links,n,tol,bound", [(whmc.F64, whmc.L18, 1, 1e-12, 1e-10), (whmc.F64, whmc.L12, 7, 1e-12, 1e-10),
                                                    (whmc.F32, whmc.L12, 1, 1e-10, 1e-8), (whmc.F32, whmc.L8, 6, 1e-10, 1e-8),
                                                    (whmc.F16, whmc.L12, 1, 1e-10, 1e-8), (whmc.F16, whmc.L12, 6, 1e-10, 1e-8)])
@pytest.mark.parametrize("check_every", [2, 7])
def test_fused_update_of_p_on_ragged_lattices(prec, links, n, tol, bound, check_every):
    dims = (18, 6, 10, 14) if n != 7 else (6, 6, 6, 10)
    U = synth.smooth_links(dims, 9570, width=0.8)
    ctx, thread = make_ctx(dims, U), make_ctx(dims, U)
    thread.set_option(whmc.OPT_HOP_KERNEL, 1)
    kappas = [(0.13, 0.10, 0.12)[r % 3] for r in range(n)]
    b = _fields(ctx, n, 9571)
    if n > 1:
        b.chunk(n)[1].zero_()
    prm = dict(tol=tol, prec=prec, links=links, delta=0.1, check_every=check_every)
    x, st = ctx.cg_solve(b, kappas, whmc.cg_params(**prm))
    block = dict(rhs_block=1, rhs_lanes=1) if n > 1 else {}
    ref, _ = thread.cg_solve(b, kappas, whmc.cg_params(**prm, **block))
    for r in range(n):
        assert st[r]["converged"] and st[r]["true_residual"] <= tol
        got, want = (v.chunk(n)[r].cpu().numpy() for v in (x, ref))
        assert not got.any() if n > 1 and r == 1 else rel_err(got, want) < bound, r
