"""The wall transforms of the SELM projection at the edges of their tiles, against the oracle.

A lane carries 8, 4, 2 or 1 layers (the most that divides nz) and reads four entries of a row of
S at a time; a work-group takes 64 columns and four layer tiles.  Tolerance as for any projection
from a solve to rtol: |P u - P* u| <= 2 rtol sqrt(lambda_max) / lambda_min |D u|.
"""
import numpy as np
import pytest

from oracle import selm as oselm

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    (10, 6, 5),      # one layer a lane, a row of S that four does not divide
    (4, 4, 2),       # two layers, fewer columns than a wave
    (12, 12, 36),    # four layers, nine tiles: three waves of the last work-group without one
    (10, 14, 40),    # eight layers, columns that a wave does not divide
])
def test_projection_tiles(dims):
    from paper_1003_2680_amd.selm import SELM
    print("[gpu-case] SELM wall transform %s" % (dims,), flush=True)
    nx, ny, nz = dims
    S = SELM(nx, ny, nz, h=0.8)
    u = np.random.default_rng(11).standard_normal((3, nz, ny, nx))
    pu = S.project(torch.from_numpy(u).cuda(), rtol=1e-12).cpu().numpy()
    ref = oselm.apply_projection(u.ravel(), nx, ny, nz, h=0.8)
    D = oselm.divergence_matrix(nx, ny, nz, h=0.8)
    lmin = 4 / 0.64 * np.sin(np.pi / (2 * nz)) ** 2
    lmax = 12 / 0.64
    tol = 2e-12 * np.sqrt(lmax) / lmin * np.linalg.norm(D @ u.ravel())
    err = np.linalg.norm(pu.ravel() - ref)
    print("  |Pu - P*u| %.2e (bound %.2e)" % (err, tol), flush=True)
    assert err <= tol
