"""Rounding of the diffusions that does not average out.  The mean of q is what Q
is made of, so an error with the same sign at every site of every pass grows
linearly with the contour steps in Q (a rounded 1/N as the k = 0 factor, or the
smallest matrix entries rounding away against the mean), while every short
comparison at the bars of the other tests passes.

Without fields a step is the diffusion D_h alone, of both schemes, and the sum of
D_h q over the sites is the product of the axes' sums D_h 1 with q (1 on periodic
axes and between reflecting walls), taken here in extended precision.  Averaged
over sites and fresh random q, what is left of the difference is the systematic
part of the rounding.

Bar, with u the unit roundoff: u/4 a step.  A rounded 1/N with N = 3 or 5 times a
power of two is off by u/2, an ordinary rounding error averages over at least a
thousand lines to less than u/30, and a table of rounded entries between
absorbing walls, each within u/2 and at random, to less than u/10.  Complex
double multiplies the Richardson combination by the rounded 1/3, u/2 more.
Absorbing walls are held to it on the matrix passes of complex float only, whose
entries are rounded once: in complex double the entries carry the roundings of
the sums they come from, and the line transforms keep no mode exactly there."""
import numpy as np
import pytest
import torch

from paper_1204_5434_amd import binding as B

pytestmark = pytest.mark.gpu
U = {B.PFT_C128: 2.0 ** -53, B.PFT_C64: 2.0 ** -24}
P, R, A = B.PFT_PERIODIC, B.PFT_REFLECTING, B.PFT_ABSORBING
# grids whose passes are line transforms on some axes, with the matrix passes beside them:
# single passes, one launch per plane, square planes (both schedules), walls of both kinds
GRIDS = [((80, 96, 40), (P, P, R)), ((24, 192, 96), (P, P, P)), ((96, 20, 192), (P, P, P)), ((24, 96, 16), (P, R, P)),
         ((20, 16, 96), (P, P, R)), ((192, 12, 20), (R, P, P)), ((8, 80, 80), (P, P, P)), ((12, 96, 96), (P, P, P)),
         ((16, 32, 32), (P, P, P)), ((12, 64, 64), (P, P, P)), ((20, 48, 48), (P, P, P)), ((48, 24, 40), (P, P, P)),
         ((16, 24, 40), (R, R, P)), ((12, 20, 48), (P, R, R)), ((24, 80, 64), (P, R, R)), ((16, 48, 20), (P, A, P)),
         ((20, 24, 40), (A, P, R)), ((16, 64, 80), (P, A, A))]
CASES = [(n, bc, scheme, prec, 20, 0.12) for n, bc in GRIDS for scheme in (B.PFT_SPLIT2, B.PFT_RQM4)
         for prec in (B.PFT_C128, B.PFT_C64) if A not in bc or prec == B.PFT_C64]
# a step and spacing at which matrix products that added up to the mean of q, instead of
# to its variation, would lose their smallest entries: 0.45 u a step for each axis of 64 points
CASES += [(n, bc, B.PFT_RQM4, B.PFT_C64, 50, 6 / 64) for n, bc in [
    ((64, 64, 64), (P, P, P)), ((16, 64, 64), (P, P, P)), ((64, 16, 12), (P, P, P)), ((16, 64, 12), (P, P, P)),
    ((16, 12, 64), (P, P, P)), ((64, 64, 80), (P, P, R)), ((16, 64, 12), (P, A, P)), ((12, 16, 64), (P, P, A))]]


def axis_sums(n, L, h, wall):
    """D_h applied to the constant 1 along one axis of n points."""
    one = np.ones(n, dtype=np.longdouble)
    if wall != A:
        return one
    x = (np.arange(n, dtype=np.longdouble) + np.longdouble(0.5)) / n
    pi = np.longdouble("3.14159265358979323846264338327950288")
    out = np.zeros(n, dtype=np.longdouble)
    for m in range(1, n + 1):
        s = np.sin(pi * m * x)
        out += s * (s.sum() / (s * s).sum()) * np.exp(-(pi * m / np.longdouble(L)) ** 2 * np.longdouble(h))
    return out


@pytest.mark.parametrize("n,bc,scheme,prec,ns,dx", CASES, ids=[
    f"{n}-{bc}-{'split2' if s else 'rqm4'}-{'c64' if p else 'c128'}-{ns}" for n, bc, s, p, ns, _ in CASES])
def test_the_mean_does_not_drift(n, bc, scheme, prec, ns, dx):
    print("mean of q", n, bc, scheme, prec, ns, flush=True)
    L = tuple(dx * a for a in n)
    ctx = B.Context(B.Params(*n, *L, ns, 0.5, 15.0, 2.0, prec, scheme, B.PFT_DIBLOCK, 0.0, 0, bc))
    zero = torch.zeros(n, dtype=torch.complex128, device="cuda")
    ctx.pft_propagate(zero, zero)
    v = [axis_sums(a, l, 1.0 / ns, w) for a, l, w in zip(n, L, bc)]
    g = torch.Generator().manual_seed(sum(n))
    out = torch.empty_like(zero)
    fused = [ctx.pft_fused_planes()]
    if n[1] == n[2] and (n[1] > 64 or bc[1] == P):
        fused.append(1 - fused[0])  # both schedules of a square plane
    for on in fused:
        if on != ctx.pft_fused_planes():
            ctx.pft_set_fused_planes(on)
        got = want = np.longdouble(0)
        for _ in range(max(4, -(-1_000_000 // zero.numel()))):
            q = (1.0 + 0.1 * torch.randn(n, generator=g, dtype=torch.float64)).to(
                torch.float32 if prec == B.PFT_C64 else torch.float64)
            ctx.pft_apply_step(0, q.to(torch.complex128).cuda(), out)
            x = q.double().numpy().astype(np.longdouble)
            want += (((x * v[2]).sum(2) * v[1]).sum(1) * v[0]).sum()
            got += out.real.cpu().numpy().astype(np.longdouble).sum()
        drift = float((got - want) / want)
        print(f"  fused {on}: drift {drift / U[prec]:+.3f} u a step", flush=True)
        third = 0.5 if prec == B.PFT_C128 and scheme == B.PFT_RQM4 else 0.0
        assert abs(drift) <= (0.25 + third) * U[prec]
    ctx.close()
