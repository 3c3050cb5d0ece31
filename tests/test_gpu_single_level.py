"""Smoothing-only single levels of at most 4096 cells with an odd wall axis, in the bottom launch.

6x6x57: 2052 cells, whose pregenerated normals take 257 threads (2052 / 8 rounded up), one more than a
work-group; 10x6x7: 420 cells, no multiple of 8, so the colours' calls meet inside a thread's four; a
single layer.  Two stochastic cycles against the oracle on the same Philox streams: FP64 every value
within 1e-12 of the largest, FP32-refined within 1e-4 relative RMS.
"""
import numpy as np
import pytest

from oracle.mg import StochasticMG

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
@pytest.mark.parametrize("dims", [(6, 6, 57), (10, 6, 7), (12, 10, 1)])
def test_chain(dims, precision):
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] single level %s %s" % (dims, precision), flush=True)
    kw = dict(levels=1, coarsest="smooth")
    H = Hierarchy(*dims, ncomp=3, kT=1.2, precision=precision, **kw)
    got = H.sample(2, 17, first_cycle=2)[0].cpu().numpy().reshape(2, 3, -1)
    ref, _ = StochasticMG(*dims, kT=1.2, **kw).sample_chain(2, 17, first_cycle=2, ncomp=3)
    ref = ref.reshape(got.shape)
    if precision == "fp64":
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
    else:
        assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
