"""The stencil and CG kernels of small lattices (a site's eight directions in one workgroup) against the
kernels with one thread per site, which an explicit schedule selects: hops bit for bit in every format,
solves to the tolerance, on lattices with less than a block, ragged tails and several blocks per XCD."""
import numpy as np
import pytest
import torch

from oracle import dirac
from oracle.lattice import Lattice
from oracle.solve import cg
from paper_1805_03560_amd import synth, whmc

from gpu_util import make_ctx, pack_half, rel_err, unpack_half

pytestmark = pytest.mark.gpu

# Vh = 8 (part of a block), 128, 288 (a tail of 32), 1728, 7560 (ragged, 119 blocks over the XCDs)
DIMS = [(2, 2, 2, 2), (4, 4, 4, 4), (4, 4, 6, 6), (6, 4, 12, 12), (18, 6, 10, 14)]
FORMATS = [(whmc.F64, whmc.L18), (whmc.F64, whmc.L12), (whmc.F64, whmc.L8), (whmc.F32, whmc.L18),
           (whmc.F32, whmc.L12), (whmc.F32, whmc.L8), (whmc.F16, whmc.L12), (whmc.F16, whmc.L8)]


def _pair(dims, seed):
    U = synth.smooth_links(dims, seed, width=0.8)
    split, thread = make_ctx(dims, U), make_ctx(dims, U)
    thread.set_option(whmc.OPT_HOP_SCHEDULE, 0)
    return U, split, thread


@pytest.mark.parametrize("dims", DIMS)
def test_hops_are_bit_identical(dims):
    U, split, thread = _pair(dims, 9300)
    x = pack_half(split, synth.gaussian_spinor(split.Vh, 9301))
    for prec, links in FORMATS:
        xp = split.convert_spinor(x, whmc.F64, prec)
        for par in (0, 1):
            for dag in (False, True):
                a, b = (c.apply_H(xp, par, dagger=dag, prec=prec, links=links) for c in (split, thread))
                assert torch.equal(a, b), (prec, links, par, dag)
    assert torch.equal(split.apply_Moo(x, 0.15), thread.apply_Moo(x, 0.15))
    assert torch.equal(split.apply_MdagM(x, [0.15]), thread.apply_MdagM(x, [0.15]))


@pytest.mark.parametrize("dims", DIMS[1:])
@pytest.mark.parametrize("prec,links", [(whmc.F64, whmc.L18), (whmc.F32, whmc.L12), (whmc.F16, whmc.L12)])
def test_multi_hops_are_those_of_each_rhs(dims, prec, links):
    U, split, thread = _pair(dims, 9310)
    n = 3
    xs = pack_half(split, np.stack([synth.gaussian_spinor(split.Vh, 9311 + r) for r in range(n)]))
    xp = split.convert_spinor(xs, whmc.F64, prec, n)
    out = split.apply_H_multi(xp, 1, n, prec=prec, links=links).chunk(n)
    for r, one in enumerate(xp.chunk(n)):
        assert torch.equal(out[r], thread.apply_H(one, 1, prec=prec, links=links)), r


# one rhs of zeros (done before the first step), unequal masses (stopped at different iterations), an odd
# number of iterations per host check (the scalars end in either buffer)
@pytest.mark.parametrize("prec,links,tol,bound", [(whmc.F64, whmc.L18, 1e-12, 1e-10), (whmc.F64, whmc.L8, 1e-12, 1e-10),
                                                  (whmc.F32, whmc.L12, 1e-10, 1e-8), (whmc.F16, whmc.L12, 1e-10, 1e-8)])
@pytest.mark.parametrize("check_every", [1, 7])
def test_solves_match_the_oracle(prec, links, tol, bound, check_every):
    dims = (6, 4, 6, 8)
    lat = Lattice(dims)
    U, split, _ = _pair(dims, 9320)
    kappas = [0.13, 0.10, 0.12]
    bs = np.stack([synth.gaussian_spinor(lat.Vh, 9321), np.zeros((lat.Vh, 4, 3), complex),
                   synth.gaussian_spinor(lat.Vh, 9322)])
    prm = whmc.cg_params(tol=tol, prec=prec, links=links, delta=0.1, check_every=check_every)
    x, st = split.cg_solve(pack_half(split, bs), kappas, prm)
    got = unpack_half(split, x, 3)
    for r in (0, 2):
        ref = cg(lambda v: dirac.apply_MooDagMoo(lat, U, v, kappas[r]), bs[r], tol=1e-14)[0]
        assert st[r]["converged"] and st[r]["true_residual"] <= tol and rel_err(got[r], ref) < bound
        one, st1 = split.cg_solve(pack_half(split, bs[r]), [kappas[r]], prm)
        assert st1[0]["converged"] and rel_err(unpack_half(split, one), ref) < bound
    assert st[1]["iters"] == 0 and not got[1].any()
    assert st[0]["iters"] != st[2]["iters"]


# M^dag M for several masses in one call against one call each: the
# direction-split kernels, and the multi-RHS kernels (streamed links make the lattice a large one), with
# the batches that 19 right-hand sides make
@pytest.mark.parametrize("eo", [True, False])
@pytest.mark.parametrize("dims,large,n", [((2, 2, 2, 2), False, 3), ((4, 4, 4, 4), False, 19), ((6, 4, 6, 8), False, 19),
                                          ((6, 4, 6, 8), True, 7), ((4, 12, 16, 16), True, 5)])
def test_mdagm_of_several_masses(dims, large, n, eo):
    lat = Lattice(dims)
    U, ctx, thread = _pair(dims, 9330)
    if large:
        ctx.set_option(whmc.OPT_STREAM_THRESHOLD, 0)
    kappas = [0.10 + 0.003 * r for r in range(n)]
    sites, parity = (lat.Vh, 1) if eo else (lat.V, -1)
    x = ctx.pack_spinor(torch.from_numpy(np.stack([synth.gaussian_spinor(sites, 9331 + r) for r in range(n)])).cuda(), parity)
    out = ctx.apply_MdagM(x, kappas, eo=eo).chunk(n)
    for r, one in enumerate(x.chunk(n)):
        ref = thread.apply_MdagM(one, [kappas[r]], eo=eo)
        assert float((out[r] - ref).abs().max() / ref.abs().max()) < 1e-14
        if not large:
            assert torch.equal(out[r], ref)
    if not large:
        noalloc = ctx.apply_MdagM_noalloc(x, kappas, torch.full_like(x, float("nan")), eo=eo)
        assert torch.equal(noalloc, torch.cat(out))


def test_mdagm_under_capture_keeps_to_the_scratch_there_is():
    dims = (6, 4, 6, 8)
    _, ctx, _ = _pair(dims, 9340)
    x = pack_half(ctx, np.stack([synth.gaussian_spinor(ctx.Vh, 9341 + r) for r in range(3)]))
    ref = [ctx.apply_MdagM(one, [0.12]).clone() for one in x.chunk(3)]   # scratch for one right-hand side
    stream = torch.cuda.Stream()
    ctx2 = whmc.Context(dims, stream=stream)
    with torch.cuda.stream(stream):
        ctx2.load_gauge(ctx.export_gauge(), unitarity_tol=0.0)
        ctx2.apply_MdagM(x.chunk(3)[0], [0.12])
        out = torch.zeros_like(x)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        ctx2.apply_MdagM(x, [0.12] * 3, out=out)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, torch.cat(ref))
