"""The two-dimensional sampler's strip launches and LDS-resident bottom at the sizes where they
change shape, against the 2D oracle on the same Philox streams (every value within 1e-12 of the
largest: the parity bar of every FP64 sampler).

Strips: one and several per grid, a ragged last strip, rows whose noise calls straddle two rows
(nx not a multiple of four), odd row counts (smoothing only), sweep counts above two (several
launches per leg), zero, and grids too wide for a strip.  Bottom: a whole colour per pass (64x64),
several rounds per pass (72x60), a single block row (nz 2), a coarsest draw in the bottom, alone
(wide) between its halves, and a smoothed coarsest level; emission every second cycle.
"""
import numpy as np
import pytest

from oracle import mg2d
from oracle.philox import PhiloxNoise

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    ((128, 128), dict()), ((144, 120), dict()), ((64, 4), dict(levels=2, coarsest="smooth")),
    ((18, 16), dict(levels=2)), ((34, 21), dict(levels=1, coarsest="smooth")),
    ((32, 36), dict(levels=2, nu1=3, nu2=5)), ((32, 48), dict(levels=3, nu1=0, nu2=1)),
    ((48, 32), dict(levels=3, nu1=1, nu2=0)), ((40, 44), dict(levels=2)),
    ((1024, 8), dict(levels=2)), ((80, 72), dict(coarsest_max=64)),
]


@pytest.mark.parametrize("dims,kw", CASES)
def test_chain(dims, kw):
    from paper_1003_2680_amd.grid2d import Hierarchy2D
    print("[gpu-case] 2D strips %s %s" % (dims, kw), flush=True)
    nx, nz = dims
    H = Hierarchy2D(nx, nz, ncomp=3, kT=0.9, stride=2, **kw)
    mg = mg2d.StochasticMG2D(nx, nz, kT=0.9, **kw)
    out, state = H.sample(2, 23, first_cycle=1)
    got = out.cpu().numpy().reshape(2, 3, -1)
    assert torch.equal(out[-1], state)
    zero = np.zeros(nx * nz)
    for c in range(3):
        x = zero.copy()
        for k in range(4):
            x = mg.vcycle(x, zero, PhiloxNoise(23), 1 + k, c)
            if k % 2:
                assert np.max(np.abs(got[k // 2, c] - x)) <= 1e-12 * np.max(np.abs(x)), (c, k)


@pytest.mark.parametrize("dims", [(128, 128), (144, 120), (2048, 8), (18, 16)])
def test_solve(dims):
    from paper_1003_2680_amd.grid2d import Hierarchy2D
    print("[gpu-case] 2D strips solve %s" % (dims,), flush=True)
    H = Hierarchy2D(*dims, ncomp=2, levels=0 if dims[0] < 2048 else 3)
    f = torch.randn(H.shape, dtype=torch.float64, device=H.device,
                    generator=torch.Generator(device=H.device).manual_seed(2))
    u, cycles, relres = H.solve(f, rtol=1e-11)
    A = mg2d.StochasticMG2D(*dims, kT=1.0, levels=1, coarsest="smooth").levels[0].A
    for c in range(2):
        r = f[c].cpu().numpy().ravel() - A @ u[c].cpu().numpy().ravel()
        # the library's norm of the same residual, apart from the rounding of A u
        assert np.linalg.norm(r) <= 1.1e-11 * np.linalg.norm(f[c].cpu().numpy())
