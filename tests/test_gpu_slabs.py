"""Sweeps of grids whose arrays exceed the Infinity Cache: the z and y passes run
slab by slab (256 planes in slabs of 86, 86 and 84; a walled z axis).  Every
stored node against one step from the node before it, which runs whole passes."""
import pytest
import torch

from paper_1204_5434_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc,prec", [((256, 192, 256), (0, 0, 0), B.PFT_C128), ((256, 256, 128), (0, 0, 1), B.PFT_C128),
                                       ((256, 256, 256), (0, 0, 0), B.PFT_C64)], ids=["ragged", "walls", "c64"])
def test_slabs_equal_whole_passes(n, bc, prec):
    print("slabs", n, bc, prec, flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    w = [0.3 * torch.randn(n, dtype=torch.complex128, device="cuda", generator=g) for _ in range(2)]
    ctx = B.Context(B.Params(*n, *[0.08 * a for a in n], 3, 0.4, 15.0, 2.0, prec, 0, B.PFT_DIBLOCK, 0.0, 0, bc))
    ctx.pft_set_fused_planes(0)
    ctx.pft_propagate(*w)
    tol = 1e-13 if prec == B.PFT_C128 else 1e-6
    node, got, want = (torch.empty(n, dtype=torch.complex128, device="cuda") for _ in range(3))
    for which in (0, 1):
        for j in range(ctx.K):
            ctx.pft_get_slice(which, j, node)
            ctx.pft_get_slice(which, j + 1, got)
            ctx.pft_apply_step(j if which == 0 else ctx.K - 1 - j, node, want)
            assert (got - want).abs().max().item() <= tol * want.abs().max().item(), (which, j)
    ctx.close()


@pytest.mark.parametrize("storage,model", [(B.PFT_STORE_BOTH, 0), (B.PFT_STORE_Q, 0), (B.PFT_STORE_BOTH, 1)],
                         ids=["both", "q", "edwards"])
def test_slabs_where_both_sweeps_run_at_once(storage, model):
    """Only sweeps that share the device run in slabs: the launches of one evaluation."""
    n, ns = (256, 256, 256), 3
    print("slab launches", storage, model, flush=True)
    w = [torch.zeros(n, dtype=torch.complex128, device="cuda") for _ in range(2)]
    ctx = B.Context(B.Params(*n, *[0.08 * a for a in n], ns, 0.4, 15.0, 2.0, B.PFT_C64, 0, model, 1.0, storage))
    sweeps = 1 if model else 2
    for together in ((True, False) if storage == B.PFT_STORE_BOTH and not model else (False,)):
        if not model and storage == B.PFT_STORE_BOTH:
            ctx.pft_set_concurrent_sweeps(together)
        ctx.pft_profile_begin()
        ctx.pft_propagate(w[0], None if model else w[1])
        k = ctx.pft_profile_end()
        slabs = 2 if together else 1  # arrays of 128 MiB in slabs of 64
        assert k["zpass"][1] == sweeps * slabs * (ctx.K + 1)
        assert k["ypass"][1] == sweeps * slabs * 2 * ctx.K
        assert k["xpass"][1] == sweeps * ctx.K
    ctx.close()
