"""WHMC_OPT_HOP_KERNEL: a schedule or cap selects one thread per site on small lattices, and the option takes that
back.  The two kinds of kernels sum an FP64 solve's scalar products in different orders, so the bits of a solution tell
which ran; a hop's bits are the same."""
import pytest
import torch

from paper_1805_03560_amd import synth, whmc

from gpu_util import make_ctx, pack_half

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("option,value", [(whmc.OPT_HOP_SCHEDULE, 0), (whmc.OPT_HOP_SCHEDULE, 1),
                                          (whmc.OPT_HOP_WG_PER_CU, 0), (whmc.OPT_HOP_WG_PER_CU, 2)])
def test_schedules_and_caps_can_be_taken_back(option, value):
    dims = (8, 8, 16, 16)
    ctx = make_ctx(dims, synth.smooth_links(dims, 9550, width=0.6))
    b = pack_half(ctx, synth.gaussian_spinor(ctx.Vh, 9551))
    prm = whmc.cg_params(tol=1e-9)
    default, hop = ctx.cg_solve(b, [0.14], prm)[0].clone(), ctx.apply_H(b, 0).clone()
    assert ctx.get_option(whmc.OPT_HOP_KERNEL) == 0
    before = [(o, ctx.get_option(o)) for o in (whmc.OPT_HOP_SCHEDULE, whmc.OPT_HOP_WG_PER_CU, whmc.OPT_HOP_KERNEL)]
    ctx.set_option(option, value)
    assert ctx.get_option(whmc.OPT_HOP_KERNEL) == 1
    per_site = ctx.cg_solve(b, [0.14], prm)[0].clone()
    assert not torch.equal(per_site, default) and torch.equal(ctx.apply_H(b, 0), hop)
    for o, v in before:
        ctx.set_option(o, v)
    assert ctx.get_option(whmc.OPT_HOP_KERNEL) == 0
    assert torch.equal(ctx.cg_solve(b, [0.14], prm)[0], default)
    ctx.set_option(whmc.OPT_HOP_KERNEL, 1)
    assert not torch.equal(ctx.cg_solve(b, [0.14], prm)[0], default)
    ctx.set_option(whmc.OPT_HOP_KERNEL, 0)
    ctx.autotune_hop()
    assert ctx.get_option(whmc.OPT_HOP_KERNEL) == 0
    assert torch.equal(ctx.cg_solve(b, [0.14], prm)[0], default)


@pytest.mark.parametrize("bad", [-1, 2])
def test_other_values_are_refused(bad):
    ctx = whmc.Context((4, 4, 4, 4))
    with pytest.raises(whmc.WhmcError) as e:
        ctx.set_option(whmc.OPT_HOP_KERNEL, bad)
    assert e.value.status == 1 and ctx.get_option(whmc.OPT_HOP_KERNEL) == 0
