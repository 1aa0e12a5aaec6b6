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
