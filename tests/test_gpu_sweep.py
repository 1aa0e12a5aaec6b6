"""The kernels that take a block of sites through all right-hand sides with each link read once: hops bit for
bit those of one thread per site (an explicit blocking), solves and M^dag M against theirs."""
import pytest
import torch

from paper_1805_03560_amd import synth, whmc

from gpu_util import make_ctx, rel_err

pytestmark = pytest.mark.gpu

# Vh = 32768 (the smallest lattice), 35280 (a tail of 80 of 128 sites), 34496 (a tail of exactly one half
# block), 36864 (slices of 9 blocks, padded to the XCDs)
DIMS = [(16, 16, 16, 16), (18, 14, 14, 20), (22, 14, 14, 16), (32, 12, 16, 12)]


def _fields(ctx, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n * 24 * ctx.Vh, dtype=torch.float64, device="cuda", generator=gen)


@pytest.mark.parametrize("streamed", [False, True])
@pytest.mark.parametrize("dims", DIMS)
def test_hops_are_bit_identical(dims, streamed):
    ctx = make_ctx(dims, synth.smooth_links(dims, 9400, width=0.8))
    if streamed:
        ctx.set_option(whmc.OPT_STREAM_THRESHOLD, 0)
    for prec, links, n in [(whmc.F64, whmc.L18, 2), (whmc.F64, whmc.L18, 3), (whmc.F64, whmc.L12, 3),
                           (whmc.F64, whmc.L8, 3), (whmc.F32, whmc.L12, 9), (whmc.F32, whmc.L8, 16)]:
        x = ctx.convert_spinor(_fields(ctx, n, 9401), whmc.F64, prec, n)
        for par, dag in [(0, False), (0, True), (1, False), (1, True)]:
            out = ctx.apply_H_multi(x, par, n, dagger=dag, prec=prec, links=links)
            ref = ctx.apply_H_multi(x, par, n, dagger=dag, prec=prec, links=links, rhs_block=1, rhs_lanes=1)
            assert torch.equal(out, ref), (prec, links, n, par, dag)


# one rhs of zeros (done before the first step) and unequal masses (stopped at different iterations); the
# bounds are those of the solves against the oracle at the same masses and tolerances
@pytest.mark.parametrize("prec,links,n,tol,bound", [(whmc.F64, whmc.L18, 4, 1e-12, 1e-10),
                                                    (whmc.F64, whmc.L8, 3, 1e-12, 1e-10),
                                                    (whmc.F32, whmc.L12, 9, 1e-10, 1e-8)])
@pytest.mark.parametrize("dims", DIMS[1:])
def test_solves_match_a_thread_per_site(dims, prec, links, n, tol, bound):
    ctx = make_ctx(dims, synth.smooth_links(dims, 9410, width=0.8))
    kappas = [(0.13, 0.10, 0.12)[r % 3] for r in range(n)]
    b = _fields(ctx, n, 9411)
    b.chunk(n)[1].zero_()
    prm = dict(tol=tol, prec=prec, links=links, delta=0.1, check_every=7)
    x, st = ctx.cg_solve(b, kappas, whmc.cg_params(**prm))
    ref, st1 = ctx.cg_solve(b, kappas, whmc.cg_params(rhs_block=1, rhs_lanes=1, **prm))
    for r in range(n):
        assert st[r]["converged"] and st[r]["true_residual"] <= tol
        if r != 1:
            got, want = (v.chunk(n)[r].cpu().numpy() for v in (x, ref))
            assert rel_err(got, want) < bound, r
    assert st[1]["iters"] == 0 and not x.chunk(n)[1].any()
    assert st[0]["iters"] != st[2]["iters"]


# a batch of the largest size, and what is left of it
@pytest.mark.parametrize("dims,n", [(DIMS[0], 18), (DIMS[1], 4), (DIMS[2], 5), (DIMS[3], 3)])
def test_mdagm_of_several_masses(dims, n):
    ctx = make_ctx(dims, synth.smooth_links(dims, 9420, width=0.8))
    kappas = [0.10 + 0.002 * r for r in range(n)]
    x = _fields(ctx, n, 9421)
    out = ctx.apply_MdagM(x, kappas).chunk(n)
    for r, one in enumerate(x.chunk(n)):
        assert torch.equal(out[r], ctx.apply_MdagM(one, [kappas[r]])), r
    noalloc = ctx.apply_MdagM_noalloc(x, kappas, torch.full_like(x, float("nan")))
    assert torch.equal(noalloc, torch.cat(out))
