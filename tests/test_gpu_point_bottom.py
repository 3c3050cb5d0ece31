"""Whole hierarchies in the bottom launch: level 0 of at most 4096 cells in LDS with the rest.

Two stochastic cycles (two components, given state) against the oracle on the same Philox
streams: FP64 every value within 1e-12 of the largest, FP32-refined within 1e-4 relative RMS; the
same cycles with the bottom kernel off (a launch per pass) to 1e-12 / 1e-5, the sums of the two
routes being in different orders; and a solve (a right-hand side on level 0) whose residual the
oracle's stencil confirms.

Shapes: the largest (16^3; 64x32x2, which one plane of blocks covers), fewer sites than lanes
(8x8x4), odd colour rows (22x12x8), an odd wall axis and extents that are no powers of two
(12x20x14), a smoothing-only single level, a wide coarsest draw between two launches (16^3, two
levels: 512 unknowns), and sweeps of (1, 0), (0, 1) and (2, 1).
"""
import numpy as np
import pytest

from oracle.mg import StochasticMG
from oracle.operator import apply_A

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    ((16, 16, 16), dict(levels=3)),
    ((64, 32, 2), dict(levels=2)),
    ((8, 8, 4), dict(levels=2)),
    ((22, 12, 8), dict(levels=2)),
    ((12, 20, 14), dict(levels=2)),
    ((16, 12, 8), dict(levels=1, coarsest="smooth")),
    ((16, 16, 8), dict(levels=2, coarsest="smooth")),
    ((16, 16, 16), dict(levels=2)),
    ((16, 8, 12), dict(levels=2, nu1=1, nu2=0)),
    ((16, 8, 12), dict(levels=2, nu1=0, nu2=1)),
    ((16, 8, 12), dict(levels=2, nu1=2, nu2=1)),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("dims,kw", CASES)
def test_cycles(dims, kw, precision):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] point bottom %s %s %s" % (dims, kw, precision), flush=True)
    H = Hierarchy(*dims, ncomp=2, kT=1.3, precision=precision, **kw)
    got = H.sample(2, 41, first_cycle=3)[0].cpu().numpy().reshape(2, 2, -1)
    H.set_bottom_kernel(False)
    off = H.sample(2, 41, first_cycle=3)[0].cpu().numpy().reshape(2, 2, -1)
    mg = StochasticMG(*dims, kT=1.3, **kw)
    ref, _ = mg.sample_chain(2, 41, first_cycle=3, ncomp=2)
    ref = ref.reshape(got.shape)
    print("  vs oracle %.2e, vs launches %.2e" % (np.max(np.abs(got - ref)) / np.max(np.abs(ref)),
                                                  np.max(np.abs(got - off)) / np.max(np.abs(ref))),
          flush=True)
    if precision == "fp64":
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
        assert np.max(np.abs(got - off)) <= 1e-12 * np.max(np.abs(ref))
    else:
        assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
        assert np.linalg.norm(got - off) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("dims,levels", [((16, 16, 16), 3), ((22, 12, 8), 2), ((16, 16, 16), 2)])
def test_solve(dims, levels, precision):
    from paper_1003_2680_amd.api import Hierarchy
    from paper_1003_2680_amd.inputs import gaussian_field
    print("[gpu-case] point bottom solve %s %s" % (dims, precision), flush=True)
    H = Hierarchy(*dims, ncomp=2, levels=levels, precision=precision)
    f = gaussian_field(H.shape, 5)
    u, cycles, relres = H.solve(torch.from_numpy(f).cuda(), rtol=1e-10)
    u = u.cpu().numpy()
    r = max(np.linalg.norm(f[c].ravel() - apply_A(u[c], *dims)) / np.linalg.norm(f[c])
            for c in range(2))
    assert relres <= 1e-10 and r <= 1.01e-10 and cycles <= 16
