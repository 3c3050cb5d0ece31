"""Rounding of the two-dimensional level-0 pass on a large smooth field.

A noise-free red-black sweep (kT = 0, one level) from a field of values near 1000 that vary by about
pi/nz of themselves from row to row: a cell's new value is its old one plus a small correction formed
from exact differences, so it is the mean of its neighbours to half an ulp of its own and a little more
for the correction's rounding (its size is at most a tenth of the value away from the walls, a few
times the value beside them): 0.75 ulp.  The mean by a sum of four neighbours is off by up to 1.25.
The reference takes the neighbours that the pass had (the second colour reads the first's new
values, which the result holds) in 80-bit arithmetic.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz", [(32, 244), (64, 128), (20, 97)])
def test_sweep_rounding(nx, nz):
    from paper_1003_2680_amd.grid2d import Hierarchy2D
    print("[gpu-case] 2D sweep rounding %d x %d" % (nx, nz), flush=True)
    H = Hierarchy2D(nx, nz, kT=0.0, levels=1, coarsest="smooth", nu1=1, nu2=0)
    rng = np.random.default_rng(2)
    z, x = np.arange(nz)[:, None], np.arange(nx)[None, :]
    u = 1000.0 * np.sin(np.pi * (z + 0.5) / nz) * (1.0 + 0.1 * np.sin(2 * np.pi * x / nx))
    u *= 1.0 + 1e-3 * rng.standard_normal(u.shape)
    got = H.sample(1, 3, state=torch.from_numpy(u[None]).cuda())[0][0, 0].cpu().numpy()
    red = (x + z) % 2 == 0
    worst = 0.0
    for colour, field in ((red, u), (~red, got)):
        f = field.astype(np.longdouble)
        s = np.roll(f, 1, 1) + np.roll(f, -1, 1)
        s[1:] += f[:-1]
        s[:-1] += f[1:]
        d = np.full((nz, 1), 4.0)
        d[0] += 1.0
        d[-1] += 1.0
        err = np.abs(got - s / d) / np.spacing(np.abs(got))
        worst = max(worst, float(err[colour].max()))
    print("  worst %.3f ulp" % worst, flush=True)
    assert worst <= 0.75
