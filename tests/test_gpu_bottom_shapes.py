"""The LDS-resident bottom of the V-cycle at the shapes where its lane layouts change.

Two stochastic cycles from the zero start, two components, against the oracle on the same Philox
streams: FP64 every value within 1e-12 of the largest (the parity bar of every sampler; the two
sides differ by summation order alone, about 1e-15), FP32-refined within 1e-4 relative RMS.

Shapes, by the first bottom level: flat levels whose colours exceed the work-group (64x32x2 and
32x20x6: several rounds per pass), the largest that still fill it once (16x16x16 and 32x32x4),
levels whose colours fill at most a quarter of it (8x8x8, 8x8x4) and just more (12x8x8), rings of
four cells (4x4x8), extents that are no powers of two, a single block layer (nz 2), and a
smoothed coarsest level.
"""
import numpy as np
import pytest

from oracle.mg import StochasticMG
from oracle.philox import PhiloxNoise

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [
    ((128, 64, 4), 2, "smooth"),
    ((128, 64, 4), 3, "cholesky"),
    ((64, 40, 12), 3, "cholesky"),
    ((32, 32, 32), 4, "cholesky"),
    ((64, 64, 8), 4, "cholesky"),
    ((16, 16, 16), 3, "cholesky"),
    ((16, 16, 8), 4, "cholesky"),
    ((24, 16, 16), 3, "cholesky"),
    ((8, 8, 16), 3, "cholesky"),
    ((16, 8, 24), 2, "smooth"),
    ((24, 40, 20), 3, "cholesky"),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("dims,levels,coarsest", SHAPES)
def test_bottom_shape_against_oracle(dims, levels, coarsest, precision):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] bottom %s L=%d %s %s" % (dims, levels, coarsest, precision), flush=True)
    H = Hierarchy(*dims, ncomp=2, kT=1.3, levels=levels, coarsest=coarsest, precision=precision)
    got = H.sample(2, 41, first_cycle=3)[0].cpu().numpy().reshape(2, 2, -1)
    mg = StochasticMG(*dims, kT=1.3, levels=levels, coarsest=coarsest)
    ref, _ = mg.sample_chain(2, 41, first_cycle=3, ncomp=2)
    ref = ref.reshape(got.shape)
    if precision == "fp64":
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
    else:
        assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)


# Coarsest levels drawn by a launch of their own (192 unknowns and more): below a block level, alone
# under level 0, sizes that are no multiple of the 16 rows of a work-group (216, 525, 2160), and
# component counts below, at and just above groups of four (eight and more share the factors).
@pytest.mark.parametrize("dims,levels,ncomp", [
    ((32, 32, 32), 3, 1), ((32, 32, 32), 3, 9), ((48, 48, 48), 4, 8), ((30, 14, 10), 2, 11),
    ((36, 20, 24), 2, 2), ((16, 16, 12), 2, 3),
])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
def test_wide_coarsest_against_oracle(dims, levels, ncomp, precision):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] wide coarsest %s L=%d nc=%d %s" % (dims, levels, ncomp, precision), flush=True)
    H = Hierarchy(*dims, ncomp=ncomp, kT=0.7, levels=levels, coarsest_max=4096,
                  precision=precision)
    got = H.sample(2, 7, first_cycle=1)[0].cpu().numpy().reshape(2, ncomp, -1)
    mg = StochasticMG(*dims, kT=0.7, levels=levels, coarsest_max=4096)
    zero = np.zeros(mg.levels[0].n)
    for c in sorted({0, ncomp // 2, ncomp - 1}):
        x = zero.copy()
        for k in range(2):
            x = mg.vcycle(x, zero, PhiloxNoise(7), 1 + k, c)
            if precision == "fp64":
                assert np.max(np.abs(got[k, c] - x)) <= 1e-12 * np.max(np.abs(x)), (c, k)
            else:
                assert np.linalg.norm(got[k, c] - x) <= 1e-4 * np.linalg.norm(x), (c, k)
    f = torch.randn(H.shape, dtype=torch.float64, device=H.device,
                    generator=torch.Generator(device=H.device).manual_seed(5))
    u, cycles, relres = H.solve(f, rtol=1e-12)
    ref, _, _ = mg.solve(f[-1].cpu().numpy().ravel(), rtol=1e-13)
    # both relative residuals are at most 1e-12: the solutions differ by the operator's condition
    # number (lambda from 12 / h^2 down to that of the lowest mode) times their sum
    cond = 12.0 / (4.0 * np.sin(np.pi / (2 * dims[2])) ** 2)
    assert np.linalg.norm(u[-1].cpu().numpy().ravel() - ref) <= 2e-12 * cond * np.linalg.norm(ref)
