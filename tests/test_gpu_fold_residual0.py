"""The folded level-0 residual restriction where its tiles end, against the oracle's P^T (b - A x).

A work-group takes 32 x 8 or 16 x 16 coarse columns (whichever covers the level with fewer) and 2 to
16 coarse layers; a lane holds two columns, so an odd number of them takes the window-sum kernel.
Every value within 1e-12 of the largest, the parity bar of the transfers.  The last shapes make the
layer count per work-group 2, 4 and 16 with a ragged last one.
"""
import numpy as np
import pytest

from oracle.mg import StochasticMG

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,ncomp", [
    ((4, 4, 2), 1),       # two columns, one layer: both walls in it
    ((4, 12, 6), 2),
    ((22, 8, 10), 2),     # eleven columns: window sums
    ((36, 32, 8), 1),     # 16 x 16 columns, the second column tile ragged
    ((64, 16, 20), 2),    # 32 x 8 columns exactly
    ((68, 20, 4), 1),     # 32 x 8 with two columns beyond, ragged rows
    ((64, 64, 36), 5),    # 18 layers, 4 a work-group
    ((64, 64, 44), 33),   # 22 layers, 16 a work-group
])
def test_fold(dims, ncomp):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] folded restriction %s x %d" % (dims, ncomp), flush=True)
    # the coarse level is smoothed where it can be, else drawn
    smooth = dims[0] % 8 == 0 and dims[1] % 8 == 0 and dims[2] % 4 == 0
    kw = dict(levels=2, coarsest="smooth") if smooth else dict(levels=2, coarsest_max=4096)
    H = Hierarchy(*dims, ncomp=ncomp, **kw)
    mg = StochasticMG(*dims, **kw)
    P, A = mg.levels[0].P, mg.levels[0].A
    rng = np.random.default_rng(3)
    N = dims[0] * dims[1] * dims[2]
    x, b = rng.standard_normal((2, ncomp, N))
    shape = (ncomp,) + tuple(reversed(dims))
    for use_b in (False, True):
        out = torch.empty((ncomp, N // 8), dtype=torch.float64, device="cuda")
        H.debug_restrict_residual(0, torch.from_numpy(x.reshape(shape)).cuda(),
                                  torch.from_numpy(b.reshape(shape)).cuda() if use_b else None, out)
        got = out.cpu().numpy()
        for c in (0, ncomp - 1):
            ref = P.T @ ((b[c] if use_b else 0.0) - A @ x[c])
            assert np.max(np.abs(got[c] - ref)) <= 1e-12 * np.max(np.abs(ref))


@pytest.mark.parametrize("dims,ncomp", [
    ((8, 8, 4), 1),       # level 1 of 4 x 4 x 2: one lane is a whole row, both walls in a layer
    ((72, 40, 24), 2),    # 36 x 20 x 12: 16 x 16 columns, ragged in x and y
    ((128, 32, 40), 1),   # 64 x 16 x 20: 32 x 8 columns exactly, a layer a work-group
    ((136, 16, 8), 3),    # 68 x 8 x 4: two columns beyond the second tile
    ((64, 64, 40), 60),   # 32 x 32 x 20 x 60: several layers a work-group, the last run short
    ((64, 64, 64), 170),  # 32 x 32 x 32 x 170: two items a lane
])
def test_fold_block_level(dims, ncomp):
    """The same on level 1 (a block level), whose tiles also come with 512 or 256 lanes."""
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] folded block-level restriction %s x %d" % (dims, ncomp), flush=True)
    # level 2 is smoothed where it can be, else drawn
    smooth = dims[0] % 16 == 0 and dims[1] % 16 == 0 and dims[2] % 8 == 0
    kw = dict(levels=3, coarsest="smooth") if smooth else dict(levels=3, coarsest_max=4096)
    H = Hierarchy(*dims, ncomp=ncomp, **kw)
    mg = StochasticMG(*dims, **kw)
    L, C = mg.levels[1], mg.levels[2]
    x, b = np.random.default_rng(4).standard_normal((2, ncomp, L.n))
    shape = (ncomp,) + tuple(reversed(L.dims))
    out = torch.empty((ncomp, C.n), dtype=torch.float64, device="cuda")
    H.debug_restrict_residual(1, torch.from_numpy(x.reshape(shape)).cuda(),
                              torch.from_numpy(b.reshape(shape)).cuda(), out)
    got = out.cpu().numpy()
    for c in (0, ncomp - 1):
        ref = L.P.T @ (b[c] - L.A @ x[c])
        assert np.max(np.abs(got[c] - ref)) <= 1e-12 * np.max(np.abs(ref))
