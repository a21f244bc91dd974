"""Line diffusions on the matrix cores (the axis passes, and the fused yz pass of
square planes up to 64): every x length beside a plane, uneven grids and walls
of both kinds on each axis length, both precisions,
against the oracle, with a junction sub-step; both sweeps in shared launches
equal to sweeps one after the other; the same x pass by line transforms.

Bars: those of the other passes (complex double |dphi| <= 1e-10 and Q 1e-11
relative; complex float 2e-5)."""
import numpy as np
import pytest
import torch

from paper_1204_5434_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
LENGTHS = {B.PFT_C128: (8, 12, 16, 20, 24, 32, 40, 48, 64, 80), B.PFT_C64: (8, 12, 16, 20, 24, 32, 40, 48, 64, 80, 96)}
CASES = [(prec, nx) for prec in LENGTHS for nx in LENGTHS[prec]]


def evaluate(ctx, wp, wm):
    return {k: v.cpu().numpy() for k, v in ctx.evaluate(wp, wm).items()}


@pytest.mark.parametrize("prec,nx", CASES, ids=[f"{'c128' if p == 0 else 'c64'}-{n}" for p, n in CASES])
def test_every_x_length(orc, prec, nx):
    side = (12, 20, 24, 8)[nx // 4 % 4]  # planes that share a workgroup, and ones that do not
    n, L, ns, f = (nx, side, side), (0.12 * nx, 0.13 * side, 0.1 * side), 9, 0.37
    print("matrix passes", prec, n, flush=True)
    r = np.random.default_rng(nx)
    wp, wm = (0.4 * r.standard_normal(n) + 0.1j * r.standard_normal(n) for _ in range(2))
    ref = orc.evaluate(orc.Params(*n, *L, ns, f, 15.0, 2.0, 0, False), wp, wm)
    gp, gm = torch.from_numpy(wp).to(DEV), torch.from_numpy(wm).to(DEV)
    ctx = B.Context(B.Params(*n, *L, ns, f, 15.0, 2.0, prec, 0))
    assert ctx.pft_fused_planes() == 1
    got = evaluate(ctx, gp, gm)
    ctx.pft_set_concurrent_sweeps(False)
    alone = evaluate(ctx, gp, gm)
    ctx.pft_set_variant(0, 0)
    lines = evaluate(ctx, gp, gm)
    ctx.close()
    tol, tq = (1e-10, 1e-11) if prec == B.PFT_C128 else (2e-5, 2e-5)
    for key in ("phiA", "phiB", "Q"):
        assert np.array_equal(got[key], alone[key]), key
    for o in (got, lines):
        for key in ("phiA", "phiB"):
            assert np.abs(o[key] - ref[key]).max() <= tol * max(1.0, np.abs(ref[key]).max()), key
        assert abs(o["Q"][0] - ref["Q"]) <= tq * abs(ref["Q"])


# uneven grids: every length once along y and along z, walls of both kinds
UNEVEN = [((16, 8, 12), (0, 0, 0), 0), ((12, 16, 8), (1, 2, 1), 0), ((8, 20, 16), (0, 1, 2), 0),
          ((24, 12, 20), (2, 0, 0), 1), ((20, 32, 24), (1, 1, 0), 0), ((8, 24, 32), (0, 2, 1), 0),
          ((12, 48, 40), (2, 1, 2), 0), ((40, 8, 48), (1, 0, 2), 0), ((8, 40, 64), (0, 2, 1), 1),
          ((8, 64, 80), (0, 1, 2), 0), ((80, 12, 16), (2, 2, 1), 0), ((8, 80, 96), (0, 0, 0), 0), ((48, 96, 8), (1, 0, 1), 0)]


@pytest.mark.parametrize("prec", [B.PFT_C128, B.PFT_C64])
@pytest.mark.parametrize("n,bc,scheme", UNEVEN, ids=[f"{n}-{bc}" for n, bc, _ in UNEVEN])
def test_uneven_grids_and_walls(orc, n, bc, scheme, prec):
    L, ns, f = tuple(0.11 * a for a in n), 7, 0.41
    print("matrix axis passes", prec, n, bc, scheme, flush=True)
    r = np.random.default_rng(sum(n))
    wp, wm = (0.4 * r.standard_normal(n) + 0.1j * r.standard_normal(n) for _ in range(2))
    ref = orc.evaluate(orc.Params(*n, *L, ns, f, 15.0, 2.0, scheme, False, bc), wp, wm)
    gp, gm = torch.from_numpy(wp).to(DEV), torch.from_numpy(wm).to(DEV)
    ctx = B.Context(B.Params(*n, *L, ns, f, 15.0, 2.0, prec, scheme, B.PFT_DIBLOCK, 0.0, 0, bc))
    got = evaluate(ctx, gp, gm)
    ctx.pft_set_concurrent_sweeps(False)
    alone = evaluate(ctx, gp, gm)
    ctx.close()
    tol, tq = (1e-10, 1e-11) if prec == B.PFT_C128 else (2e-5, 2e-5)
    for key in ("phiA", "phiB", "Q"):
        assert np.array_equal(got[key], alone[key]), key
    for key in ("phiA", "phiB"):
        assert np.abs(got[key] - ref[key]).max() <= tol * max(1.0, np.abs(ref[key]).max()), key
    assert abs(got["Q"][0] - ref["Q"]) <= tq * abs(ref["Q"])


# lengths that meet in one yz launch: rows and columns of one strip and of several,
# the remainder of a strip, the largest pair that fits, walls on either axis
PAIRS = [((8, 40, 24), (0, 0, 0)), ((8, 24, 40), (0, 1, 0)), ((8, 48, 40), (0, 0, 2)), ((8, 40, 48), (0, 2, 1)),
         ((8, 8, 48), (0, 0, 1)), ((8, 12, 8), (0, 0, 0)), ((8, 32, 32), (0, 1, 1)), ((8, 20, 48), (0, 0, 0))]


@pytest.mark.parametrize("prec", [B.PFT_C128, B.PFT_C64])
@pytest.mark.parametrize("n,bc", PAIRS, ids=[f"{n}-{bc}" for n, bc in PAIRS])
def test_yz_pass_of_uneven_planes(n, bc, prec):
    r = np.random.default_rng(sum(n))
    wp, wm = (torch.from_numpy(0.4 * r.standard_normal(n) + 0.1j * r.standard_normal(n)).to(DEV) for _ in range(2))
    ctx = B.Context(B.Params(*n, *[0.12 * a for a in n], 7, 0.4, 15.0, 2.0, prec, 0, B.PFT_DIBLOCK, 0.0, 0, bc))
    got = evaluate(ctx, wp, wm)
    ctx.pft_set_concurrent_sweeps(False)
    alone = evaluate(ctx, wp, wm)
    ctx.pft_set_variant(1, 0)  # z and y passes apart, y by line transforms
    apart = evaluate(ctx, wp, wm)
    ctx.close()
    tol = 1e-10 if prec == B.PFT_C128 else 2e-5
    for key in ("phiA", "phiB", "Q"):
        assert np.array_equal(got[key], alone[key]), key
        assert np.abs(got[key] - apart[key]).max() <= tol * np.abs(apart[key]).max(), key


@pytest.mark.parametrize("prec", [B.PFT_C128, B.PFT_C64])
def test_constant_and_nonfinite_fields(prec):
    """A uniform field leaves q uniform (its closed form, Eq. (5)); a field
    that is not finite at one site reaches the status flag."""
    n, ns, w = (16, 32, 32), 12, 0.7
    ctx = B.Context(B.Params(*n, 2.0, 4.0, 4.0, ns, 0.5, 15.0, 1.0, prec, 0))
    wp = torch.zeros(n, dtype=torch.complex128, device=DEV)
    wm = torch.full(n, w, dtype=torch.complex128, device=DEV)
    out = ctx.evaluate(wp, wm)
    # w_A = -w, w_B = w, f = 1/2: Q = 1 and phi_A = 1/2
    tol = 1e-13 if prec == B.PFT_C128 else 2e-6
    assert abs(out["Q"].item() - 1.0) <= tol
    assert ctx.pft_status_flags() == 0
    for bad in (float("inf"), float("nan")):
        c2 = B.Context(B.Params(*n, 2.0, 4.0, 4.0, ns, 0.5, 15.0, 1.0, prec, 0))
        w2 = wm.clone()
        w2[3, 5, 7] = -bad
        c2.evaluate(wp, w2)
        assert c2.pft_status_flags() & 1
        c2.close()
    ctx.close()


# which passes of large grids run by line transforms, on both sides of each line:
# (grid, walls, precision, scheme, axis, by lines)
LINES = [((128, 48, 128), (0, 0, 0), 1, 0, 1, True), ((96, 48, 128), (0, 0, 0), 1, 0, 1, False),
         ((128, 40, 128), (0, 0, 0), 1, 0, 1, False), ((96, 64, 192), (0, 0, 0), 1, 0, 1, False), ((128, 96, 128), (0, 0, 0), 1, 1, 1, True),
         ((64, 128, 128), (0, 0, 0), 1, 0, 0, True), ((80, 192, 128), (0, 0, 0), 1, 0, 0, False),
         ((128, 64, 128), (0, 2, 0), 1, 0, 1, True), ((128, 80, 128), (0, 1, 0), 1, 0, 1, False),
         ((96, 96, 80), (0, 0, 1), 1, 0, 2, True), ((96, 96, 64), (0, 0, 2), 1, 0, 2, False), ((96, 96, 64), (0, 0, 2), 1, 1, 2, True),
         ((96, 96, 48), (0, 0, 0), 0, 0, 2, True), ((24, 20, 48), (0, 0, 0), 0, 0, 2, False), ((96, 96, 40), (0, 0, 0), 0, 0, 2, False),
         ((128, 128, 64), (0, 0, 0), 0, 0, 2, False), ((192, 96, 64), (0, 0, 0), 0, 0, 2, True), ((96, 80, 64), (0, 0, 0), 0, 1, 2, True)]


@pytest.mark.parametrize("n,bc,prec,scheme,axis,lines", LINES)
def test_passes_of_large_grids(n, bc, prec, scheme, axis, lines):
    """The pass an axis runs by default equals the line transforms' bit for bit
    where it is one, and otherwise agrees with it to rounding."""
    print("passes of large grids", n, bc, prec, scheme, axis, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n[axis])
    w = [0.2 * torch.randn(n, dtype=torch.complex128, device=DEV, generator=g) for _ in range(2)]
    ctx = B.Context(B.Params(*n, *[0.1 * a for a in n], 3, 0.5, 14.0, 1.0, prec, scheme, B.PFT_DIBLOCK, 0.0, 0, bc))
    assert ctx.pft_fused_planes() == 0
    got = ctx.evaluate(*w)["phiA"]
    ctx.pft_set_variant(axis, 0)
    ref = ctx.evaluate(*w)["phiA"]
    ctx.close()
    assert torch.equal(got, ref) == lines
    assert (got - ref).abs().max() <= (1e-12 if prec == B.PFT_C128 else 2e-5) * ref.abs().max()


def launches(ctx, wp, wm):
    ctx.pft_profile_begin()
    ctx.pft_propagate(wp, wm)
    k = ctx.pft_profile_end()
    return tuple(k[name][1] for name in ("yzpass", "zpass", "ypass", "xpass"))


# (grid, walls, precision, yz or axis passes, shared by both sweeps): square planes, planes of one
# launch, planes too long for one, and the sizes next to the limits of either
SHARED = [((16, 32, 32), (0, 0, 0), 0, "yz", True), ((64, 64, 64), (0, 0, 0), 1, "yz", True), ((64, 64, 64), (0, 0, 0), 0, "yz", False),
          ((8, 40, 24), (0, 0, 0), 0, "yz", True), ((8, 40, 48), (0, 2, 1), 1, "yz", True), ((8, 32, 32), (0, 1, 1), 0, "yz", True),
          ((20, 48, 40), (1, 0, 0), 1, "yz", True), ((8, 48, 48), (0, 0, 1), 0, "axis", True), ((8, 64, 80), (0, 1, 0), 0, "axis", True),
          ((8, 80, 96), (0, 0, 0), 1, "axis", True), ((8, 96, 80), (0, 0, 0), 0, "axis", False), ((80, 80, 64), (0, 0, 0), 1, "axis", True),
          ((96, 96, 64), (0, 0, 0), 1, "axis", False)]


@pytest.mark.parametrize("n,bc,prec,kind,shared", SHARED, ids=[f"{n}-{bc}-{'c64' if p else 'c128'}" for n, bc, p, _, _ in SHARED])
def test_which_launches_run(n, bc, prec, kind, shared):
    """The passes of one propagation by name and number: one launch for both sweeps
    where they share it, twice as many with the sweeps one after the other, and no
    yz pass once an axis of an uneven plane is a line transform."""
    print("launches", n, bc, prec, flush=True)
    wp, wm = (torch.zeros(n, dtype=torch.complex128, device=DEV) for _ in range(2))
    ctx = B.Context(B.Params(*n, *[0.1 * a for a in n], 6, 0.4, 15.0, 2.0, prec, 0, B.PFT_DIBLOCK, 0.0, 0, bc))
    K = ctx.K

    def passes(kind, sweeps):
        return (sweeps * (K + 1), 0, 0, sweeps * K) if kind == "yz" else (0, sweeps * (K + 1), sweeps * 2 * K, sweeps * K)

    assert launches(ctx, wp, wm) == passes(kind, 1 if shared else 2)
    ctx.pft_set_concurrent_sweeps(False)
    assert launches(ctx, wp, wm) == passes(kind, 2)
    ctx.pft_set_concurrent_sweeps(True)
    ctx.pft_set_variant(1, 0)  # y by line transforms: nothing shared but a square plane's own pass
    assert launches(ctx, wp, wm) == passes("yz" if kind == "yz" and n[1] == n[2] and not any(bc) else "axis",
                                           1 if shared and n[1] == n[2] and not any(bc) else 2)
    ctx.close()
