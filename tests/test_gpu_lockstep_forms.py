"""Block sweeps of several hierarchies in shared launches, bit for bit those of each one alone.

Odd sweep counts (a half-sweep sweep ends in the other field and is copied back), items of different
counts in one call, and lanes that only together exceed the rule that picks two-colour launches (9 *
2^15 FP64, 13 * 2^15 FP32; 8192 a component at 64^3, so 163840 of each item here and 491520 in all).
One block level is above the bottom, two at 128x64x64, none at 32^3 (whose level 1 is the bottom).
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIXES = [
    [((48, 40, 24), 2, (1, 2)), ((64, 64, 32), 1, (1, 2)), ((96, 48, 48), 1, (1, 2))],
    [((48, 40, 24), 1, (3, 1)), ((64, 64, 32), 2, (3, 1)), ((128, 64, 64), 2, (2, 1))],
    [((48, 40, 24), 1, (1, 2)), ((64, 64, 32), 2, (3, 1)), ((128, 64, 64), 1, (2, 3)),
     ((32, 32, 32), 3, (1, 1))],
    [((64, 64, 64), 20, (1, 2)), ((64, 64, 64), 20, (3, 1)), ((64, 64, 64), 20, (2, 2))],
]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("mix", range(len(MIXES)))
def test_batch_equals_alone(mix, precision):
    from paper_1003_2680_amd.api import Hierarchy, batch_run
    print("[gpu-case] lockstep forms %d %s" % (mix, precision), flush=True)
    Hs = [Hierarchy(*d, ncomp=nc, kT=0.9, nu1=nu[0], nu2=nu[1], precision=precision)
          for d, nc, nu in MIXES[mix]]
    new = lambda H: torch.empty((2,) + H.shape, dtype=torch.float64, device=H.device)
    alone = [H.sample(2, 31 + k)[0] for k, H in enumerate(Hs)]
    got = [new(H) for H in Hs]
    batch_run([dict(H=H, op="sample", n=2, seed=31 + k, state=H.new_state(), out=got[k])
               for k, H in enumerate(Hs)])
    torch.cuda.synchronize()
    for a, b in zip(alone, got):
        assert torch.equal(a, b)
    # solves (without noise, and in FP32 by the other order of additions)
    g = torch.Generator(device="cuda").manual_seed(3)
    fs = [torch.randn(H.shape, generator=g, dtype=torch.float64, device=H.device) for H in Hs]
    alone = [H.solve(f, rtol=1e-30, max_cycles=2, raise_on_notconv=False)[0]
             for H, f in zip(Hs, fs)]
    us = [torch.empty_like(f) for f in fs]
    batch_run([dict(H=H, op="solve", f=f, u=u, rtol=1e-30, max_cycles=2)
               for H, f, u in zip(Hs, fs, us)])
    torch.cuda.synchronize()
    for a, b in zip(alone, us):
        assert torch.equal(a, b)
