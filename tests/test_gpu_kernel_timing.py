"""Timing the level-0 colour passes of hierarchies whose level 0 is in the bottom launch.

While "fine_pass" is timed those passes are launches of their own, counted one by one (two a sweep),
and the bottom begins one level lower; the samples are those of the untimed call bit for bit.  Shapes:
three levels, a wide coarsest draw between two bottom launches (16^3, two levels: 512 unknowns), level 0
over the coarsest level alone, and a smoothing-only single level.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [((16, 16, 16), dict(levels=3)), ((16, 16, 16), dict(levels=2)),
          ((8, 8, 4), dict(levels=2)), ((16, 12, 8), dict(levels=1, coarsest="smooth"))]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("dims,kw", SHAPES)
def test_fine_pass_timing(dims, kw, precision):
    from paper_1003_2680_amd.api import Hierarchy, batch_run
    print("[gpu-case] fine pass timing %s %s %s" % (dims, kw, precision), flush=True)
    H = Hierarchy(*dims, ncomp=2, nu1=2, nu2=1, precision=precision, **kw)
    ref = H.sample(3, 7)[0]
    H.kernel_timing(True, "fine_pass")
    got = H.sample(3, 7)[0]
    torch.cuda.synchronize()
    count, ms = H.kernel_timing_read()
    batch = torch.empty_like(ref)
    batch_run([dict(H=H, op="sample", n=3, seed=7, state=H.new_state(), out=batch)])
    f = torch.ones(H.shape, dtype=torch.float64, device=H.device)
    u, cycles, relres = H.solve(f, rtol=1e-10, max_cycles=400)
    H.kernel_timing(False, "fine_pass")
    v, cycles0, _ = H.solve(f, rtol=1e-10, max_cycles=400)
    again = H.sample(3, 7)[0]
    torch.cuda.synchronize()
    assert count == 3 * 3 * 2 and ms > 0.0
    assert torch.equal(got, batch) and torch.equal(again, ref)
    assert torch.equal(got, ref)
    assert relres <= 1e-10 and cycles == cycles0


@pytest.mark.parametrize("dims,kw", SHAPES[:2])
def test_bottom_timing(dims, kw):
    """The bottom of a cycle counts once, however many launches it takes."""
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] bottom timing %s %s" % (dims, kw), flush=True)
    H = Hierarchy(*dims, ncomp=2, **kw)
    H.kernel_timing(True, "bottom")
    H.sample(3, 7)
    torch.cuda.synchronize()
    count, ms = H.kernel_timing_read()
    assert count == 3 and ms > 0.0
