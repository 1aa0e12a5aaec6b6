"""The orders in which the force kernels take blocks of sites, and their address widths: lattices whose z planes are
whole 128-site blocks (each XCD takes columns of its planes through time) against the oracle, and the gauge force
on a link array beyond 4 GiB against that of the small lattice whose periodic copies fill it."""
import numpy as np
import pytest
import torch

from oracle import force, gauge
from oracle.lattice import Lattice
from paper_1805_03560_amd import synth, whmc

from gpu_util import algebra_to_numpy, make_ctx, oracle_cached, pack_half, rel_err

pytestmark = pytest.mark.gpu

# planes of 2, 2 and 4 blocks, 2, 4 and 2 planes per XCD
DIMS = [(2, 16, 16, 32), (2, 32, 32, 16), (2, 16, 32, 32)]


# ... and lattices without columns: one plane per XCD, and both sides of V_h = 4096, up to which a workgroup is one
# wavefront, with part of a block
@pytest.mark.parametrize("dims", DIMS + [(2, 8, 16, 32), (6, 2, 6, 6), (16, 8, 8, 8), (18, 6, 6, 14)])
def test_gauge_force_orders(dims):
    U = synth.smooth_links(dims, 9530, width=0.8)
    ctx = make_ctx(dims, U)
    F = ctx.force(None, 0, 0, 0, 0.15, 5.6, flags=whmc.FORCE_GAUGE)
    assert rel_err(algebra_to_numpy(ctx, F), gauge.gauge_force(Lattice(dims), U, 5.6)) < 1e-12


@pytest.mark.parametrize("kernel", [0, 1])   # a thread per link (in columns), a thread per site
@pytest.mark.parametrize("dims", DIMS[:2])
def test_pair_force_in_columns(dims, kernel):
    lat = Lattice(dims)
    U = synth.smooth_links(dims, 9531)
    phi = synth.gaussian_spinor(lat.Vh, 9532)
    ctx = make_ctx(dims, U)
    ctx.set_option(whmc.OPT_FORCE_KERNEL, kernel)
    F = ctx.force(pack_half(ctx, phi), 0, 0, 0, 0.12, 5.6, solver=whmc.cg_params(tol=1e-14))
    ref = oracle_cached(("pf_force_eo", dims, 9531, 9532, 0.12),
                        lambda: force.pf_force_eo(lat, U, phi, 0.12, tol=1e-14))
    assert rel_err(algebra_to_numpy(ctx, F), ref) < 1e-12


def test_gauge_force_with_64_bit_offsets():
    if torch.cuda.mem_get_info()[1] < 200 << 30:
        pytest.skip("takes about 105 GB of device memory")
    small, dims = (4, 4, 4, 4), (64, 64, 128, 116)
    U = torch.from_numpy(synth.smooth_links(small, 9540, width=0.8)).cuda()
    one = whmc.Context(small)
    one.load_gauge(U, unitarity_tol=1e-11)
    ref = one.unpack_algebra(one.force(None, 0, 0, 0, 0.15, 5.6, flags=whmc.FORCE_GAUGE))
    ctx = whmc.Context(dims)
    assert ctx.Vh * 144 > 1 << 32
    ctx.load_gauge(U.repeat(*[d // s for d, s in zip(dims, small)], 1, 1, 1), unitarity_tol=0.0)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    F = ctx.unpack_algebra(ctx.force(None, 0, 0, 0, 0.15, 5.6, flags=whmc.FORCE_GAUGE))
    F = F.view(16, 4, 16, 4, 32, 4, 29, 4, 4, 8)
    worst = max(float((part - ref.view(4, 1, 4, 1, 4, 1, 4, 4, 8)).abs().max()) for part in F)
    assert worst <= 1e-14 * float(ref.abs().max())
    ctx.close()
    torch.cuda.empty_cache()
