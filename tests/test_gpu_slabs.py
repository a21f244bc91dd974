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
