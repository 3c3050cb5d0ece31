"""The folded restrictions in FP32, through the refined solve's first cycle.

From u = 0 a cycle returns V(f): one FP32 V-cycle (all of its restrictions folded, since a solve has no
noise) against the FP64 one on the same right-hand side.  FP32 rounding moves a value by some 1e-5
of the largest (twenty passes of sums of up to 125 terms, 6e-8 each, in random signs), a wrong tap,
lane or edge by 1e-2 and more of it: every value within 1e-4.  Each shape runs with the bottom in LDS
and with every level's restriction a launch of its own; shapes as for the FP64 folds: ragged tiles of
16 x 16 and 32 x 8 columns, a lane that is a whole row, one or several layers a work-group, 256 and
512 lanes.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,ncomp,kw", [
    ((8, 8, 4), 1, dict(levels=2)),
    ((16, 16, 8), 2, dict(levels=3)),
    ((36, 32, 8), 1, dict(levels=2)),
    ((68, 20, 4), 1, dict(levels=2)),
    ((72, 40, 24), 2, {}),
    ((136, 16, 8), 3, {}),
    ((128, 32, 40), 1, {}),
    ((64, 64, 36), 5, dict(levels=2, coarsest="smooth")),
    ((64, 64, 40), 33, {}),
    ((64, 64, 64), 40, {}),
])
def test_first_cycle(dims, ncomp, kw):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] float folds %s x %d %s" % (dims, ncomp, kw), flush=True)
    kw = dict(dict(coarsest_max=4096) if "levels" in kw else {}, **kw)
    H64 = Hierarchy(*dims, ncomp=ncomp, **kw)
    H32 = Hierarchy(*dims, ncomp=ncomp, precision="fp32_refined", **kw)
    g = torch.Generator(device="cuda").manual_seed(6)
    f = torch.randn(H64.shape, generator=g, dtype=torch.float64, device="cuda")
    one = lambda H: H.solve(f, rtol=1e-30, max_cycles=1, raise_on_notconv=False)[0]
    ref = one(H64)
    for bottom in (True, False):
        H32.set_bottom_kernel(bottom)
        got = one(H32)
        err = ((got - ref).abs().amax() / ref.abs().amax()).item()
        print("  bottom %d: %.2e" % (bottom, err), flush=True)
        assert err <= 1e-4
