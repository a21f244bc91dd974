"""Grids with few planes of 80, 96 and 128 points a side start on the axis
schedule; both sides of the line, one and two sweeps, equal to the fused pass."""
import pytest
import torch

from paper_1204_5434_amd import binding as B

pytestmark = pytest.mark.gpu
CASES = [(B.PFT_C64, 128, 0, 64, 96), (B.PFT_C64, 128, 1, 128, 192), (B.PFT_C64, 96, 0, 32, 40), (B.PFT_C64, 80, 1, 32, 40),
         (B.PFT_C128, 80, 0, 64, 80), (B.PFT_C128, 80, 1, 96, 128)]


@pytest.mark.parametrize("prec,side,model,few,enough", CASES)
def test_schedule_by_number_of_planes(prec, side, model, few, enough):
    tol = 1e-10 if prec == B.PFT_C128 else 2e-5
    for nx in (few, enough):
        n = (nx, side, side)
        print("planes", n, prec, model, flush=True)
        g = torch.Generator(device="cuda").manual_seed(nx)
        w = [0.2 * torch.randn(n, dtype=torch.complex128, device="cuda", generator=g) for _ in range(2)]
        ctx = B.Context(B.Params(*n, *[0.1 * a for a in n], 4, 0.5, 14.0, 1.0, prec, 0, model, 1.0))
        assert ctx.pft_fused_planes() == (0 if nx == few else 1)
        out = []
        for fused in (0, 1):
            ctx.pft_set_fused_planes(fused)
            out.append(ctx.evaluate(w[0], None if model else w[1])["phiA"].clone())
        ctx.close()
        assert (out[0] - out[1]).abs().max() <= tol * out[0].abs().max()


# the plain split step's lines: (precision, side, model, largest count on the axis schedule, next count)
SPLIT2 = [(B.PFT_C64, 128, 0, 48, 64), (B.PFT_C64, 128, 1, 128, 192), (B.PFT_C64, 96, 0, 24, 32), (B.PFT_C64, 96, 1, 24, 32),
          (B.PFT_C64, 80, 0, None, 8), (B.PFT_C64, 80, 1, None, 8), (B.PFT_C128, 80, 0, 48, 64), (B.PFT_C128, 80, 1, 96, 128)]


@pytest.mark.parametrize("prec,side,model,few,enough", SPLIT2)
def test_schedule_of_the_plain_split_step(prec, side, model, few, enough):
    tol = 1e-10 if prec == B.PFT_C128 else 2e-5
    for nx in filter(None, (few, enough)):
        n = (nx, side, side)
        print("planes of the plain split step", n, prec, model, flush=True)
        g = torch.Generator(device="cuda").manual_seed(nx)
        w = [0.2 * torch.randn(n, dtype=torch.complex128, device="cuda", generator=g) for _ in range(2)]
        ctx = B.Context(B.Params(*n, *[0.1 * a for a in n], 4, 0.5, 14.0, 1.0, prec, B.PFT_SPLIT2, model, 1.0))
        assert ctx.pft_fused_planes() == (0 if nx == few else 1)
        out = []
        for fused in (0, 1):
            ctx.pft_set_fused_planes(fused)
            out.append(ctx.evaluate(w[0], None if model else w[1])["phiA"].clone())
        ctx.close()
        assert (out[0] - out[1]).abs().max() <= tol * out[0].abs().max()
