"""A hierarchy of at most 4096 cells gives the same bits whether its level 0 runs in the LDS-resident
bottom or in launches of its own: those take over while its passes are timed, and where many chains
and sweeps make its normals too large for the workspace (csrc/plan.cpp), so that a chain's samples do
not depend on the chains beside it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# level-0 rows of whole and of odd pairs (the colour passes' two forms), an odd number of coarse
# columns (the restriction's two), walls next to each other, one smoothed level with an odd wall axis
SHAPES = [((16, 16, 16), {}), ((8, 12, 20), {}), ((12, 8, 16), {}), ((20, 12, 14), {}),
          ((4, 8, 2), dict(levels=2)), ((36, 4, 28), {}), ((12, 20, 2), dict(levels=2)),
          ((10, 6, 7), dict(levels=1, coarsest="smooth")), ((8, 6, 9), dict(levels=1, coarsest="smooth"))]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("kT,h,nu", [(1.0, 1.0, (2, 2)), (0.7, 0.6, (1, 3)), (0.0, 0.6, (0, 1))])
@pytest.mark.parametrize("dims,opt", SHAPES)
def test_same_bits_in_bottom_and_launches(dims, opt, kT, h, nu, precision):
    from paper_1003_2680_amd.api import Hierarchy
    res = []
    for timed in (False, True):
        H = Hierarchy(*dims, ncomp=3, h=h, kT=kT, nu1=nu[0], nu2=nu[1], precision=precision,
                      coarsest_max=128, **opt)
        if timed:
            H.kernel_timing(True, "fine_pass")
        g = torch.Generator("cuda").manual_seed(11)
        x = torch.randn(H.shape, dtype=torch.float64, device="cuda", generator=g)
        f = torch.randn(H.shape, dtype=torch.float64, device="cuda", generator=g)
        out, _ = H.sample(3, seed=5, state=x)
        u = H.solve(f, rtol=1e-6, max_cycles=4, raise_on_notconv=False)[0]
        torch.cuda.synchronize()
        if timed:
            assert H.kernel_timing_read()[0] > 0
        res.append((out, x, u))
    for a, b in zip(*res):
        assert torch.equal(a, b)


def test_chain_among_many_has_the_bits_of_one_alone():
    from paper_1003_2680_amd.api import Hierarchy
    many = Hierarchy(16, 16, 16, ncomp=128, nu1=8, nu2=8)
    one = Hierarchy(16, 16, 16, ncomp=1, nu1=8, nu2=8)
    out = torch.empty((2,) + many.shape, dtype=torch.float64, device="cuda")
    many.sample_batch(2, seeds=list(range(128)), first_cycles=[0] * 128, state=many.new_state(),
                      out=out)
    for k in (0, 77):
        ref, _ = one.sample(2, seed=k)
        assert torch.equal(out[:, k:k + 1], ref)
