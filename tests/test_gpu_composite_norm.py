"""The norm that ends a composite solve, against the residual that a separate kernel forms.

The norm kernel takes one cell a thread, and four from 2^21 base and fine cells on; the last
work-group of the fine cells is ragged in every mesh here (their number is no multiple of 256).  A
solve is stopped early (rtol 1e-2), so the reported relative residual is far above rounding, and
compared with the norm of the residual entry point's fields (zero on covered cells) over that of the
right-hand side's.  Both form a cell's residual by the same operations and add squares, each sum to
a relative error of at most some tens of eps: 1e-12.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("base,box", [
    ((32, 32, 16), (9, 22, 7, 20, 0, 5)),          # 16384 + 6760 cells
    ((64, 32, 32), (20, 41, 8, 23, 3, 12)),        # an interior box
    ((128, 128, 112), (40, 85, 31, 76, 0, 17)),    # 1835008 + 275400 cells: four a thread
])
def test_reported_residual(base, box, precision):
    from paper_1003_2680_amd.composite import CompositeSampler
    print("[gpu-case] composite norm %s %s %s" % (base, box, precision), flush=True)
    S = CompositeSampler(*base, box, precision=precision)
    g = torch.Generator(device="cuda").manual_seed(9)
    rn = lambda shape: torch.randn(shape, generator=g, dtype=torch.float64, device="cuda")
    fc, ff = rn((base[2], base[1], base[0])), rn(S.fine_shape)
    # larger values where a work-group's last cells are, so that a lost tail shows
    fc.view(-1)[-200:] *= 40.0
    ff.view(-1)[-200:] *= 40.0
    uc, uf, info = S.solve(fc, ff, rtol=1e-2)

    def norm2(xc, xf):
        rc, rf = S.residual(xc, xf, fc, ff)
        return (rc.double().square().sum() + rf.double().square().sum()).item()

    z = S.zeros()
    want = (norm2(uc, uf) / norm2(*z)) ** 0.5
    print("  reported %.6e recomputed %.6e" % (info.relres, want), flush=True)
    assert 0.0 < info.relres <= 1e-2
    assert abs(info.relres - want) <= 1e-12 * want
