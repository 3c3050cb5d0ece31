"""Refined chains without noise (kT = 0) keep the order of additions of the chains with noise.

A chain whose kT is so small that its FP32 normals round to zero (1e-200: their factor sqrt(kT) is
below the smallest float) runs the passes of a noisy chain and adds nothing, so a kT = 0 chain from
the same state has its bits.  Shapes: level 0 in the bottom launch, block levels in half-sweep and
in two-colour launches, in single-colour launches (rows over 128 cells), a split bottom, flat levels;
alone, and in one batch call beside a noisy chain.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [((16, 16, 16), 1, {}), ((22, 12, 8), 2, dict(levels=2)), ((32, 32, 72), 2, {}),
          ((64, 64, 64), 3, {}), ((64, 64, 64), 56, dict(nu1=1, nu2=2)), ((272, 16, 8), 1, {}),
          ((40, 24, 28), 2, {}), ((16, 12, 8), 2, dict(levels=1, coarsest="smooth"))]


def _start(H):
    g = torch.Generator(device=H.device).manual_seed(11)
    return torch.randn(H.shape, dtype=torch.float64, device=H.device, generator=g)


@pytest.mark.parametrize("dims,ncomp,kw", SHAPES)
def test_still_chain_bits(dims, ncomp, kw):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] still chain %s x %d %s" % (dims, ncomp, kw), flush=True)
    outs = []
    for kT in (0.0, 1e-200):
        H = Hierarchy(*dims, ncomp=ncomp, kT=kT, precision="fp32_refined", **kw)
        outs.append(H.sample(2, 5, state=_start(H))[0])
    torch.cuda.synchronize()
    assert torch.equal(*outs)


def test_still_chain_in_batch():
    from paper_1003_2680_amd.api import Hierarchy, batch_run
    print("[gpu-case] still chains in a batch", flush=True)
    shapes = [((32, 32, 72), 0.0), ((64, 64, 64), 0.0), ((16, 16, 16), 0.0), ((48, 48, 24), 1.0),
              ((64, 32, 32), 0.0)]
    Hs = [Hierarchy(*d, kT=kT, precision="fp32_refined") for d, kT in shapes]
    alone = [H.sample(2, 5, state=_start(H))[0] for H in Hs]
    items, got = [], []
    for H in Hs:
        out = torch.empty((2,) + H.shape, dtype=torch.float64, device=H.device)
        items.append(dict(H=H, op="sample", n=2, seed=5, state=_start(H), out=out))
        got.append(out)
    batch_run(items)
    torch.cuda.synchronize()
    for a, b in zip(alone, got):
        assert torch.equal(a, b)
