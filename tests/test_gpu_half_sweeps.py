"""Several block colours per launch against one colour per launch, bit for bit.

A half-sweep launch (four colours, out of place) and a two-colour launch draw every cell by the
arithmetic of the single-colour pass from the same inputs, so chains and solves agree exactly:
rings of four cells, one and odd numbers of block rows and layers, a single layer (nz 2 on the
level), the widest rows, odd numbers of sweeps (a half-sweep sweep ends in the other field), and
component counts on both sides of the rule that picks the form (9 * 2^15 lanes FP64, 13 * 2^15
FP32; 2^16 a component at 64^3).
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [
    ((8, 8, 8), 2, 2, (2, 2)), ((16, 8, 4), 2, 1, (2, 2)), ((40, 24, 20), 2, 3, (2, 2)),
    ((72, 40, 24), 2, 2, (2, 2)), ((64, 88, 12), 2, 1, (3, 1)), ((256, 16, 8), 2, 1, (2, 2)),
    ((32, 32, 32), 3, 2, (1, 2)), ((64, 64, 64), 3, 7, (2, 1)), ((128, 64, 64), 3, 8, (2, 2)),
    ((128, 64, 64), 3, 15, (1, 1)),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("dims,levels,ncomp,nu", SHAPES)
def test_forms_agree_bitwise(dims, levels, ncomp, nu, precision):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] sweep forms %s L=%d nc=%d nu=%s %s" % (dims, levels, ncomp, nu, precision),
          flush=True)
    outs = []
    for pairs in (True, False):
        H = Hierarchy(*dims, ncomp=ncomp, kT=1.1, levels=levels, nu1=nu[0], nu2=nu[1],
                      coarsest_max=4096, coarsest="smooth", precision=precision)
        H.set_bottom_kernel(False)
        H.set_block_pairs(pairs)
        x, state = H.sample(2, 19, first_cycle=3)
        f = torch.randn(H.shape, dtype=torch.float64, device=H.device,
                        generator=torch.Generator(device=H.device).manual_seed(4))
        u, _, _ = H.solve(f, rtol=1e-30, max_cycles=2, raise_on_notconv=False)
        torch.cuda.synchronize()
        outs.append((x, state, u))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
