"""Hierarchies that the allocation-free entry point (64 MiB of scratch) takes.

A hierarchy of at most 4096 cells keeps its level-0 normals, (nu1 + nu2) fields of every component,
in its workspace only while that leaves it within the scratch.  The cases hold 17 to 34 MiB of
fields and tables and would hold 65 to 103 MiB with the normals; the last one, 62 MiB, keeps them.
"""
import ctypes

import pytest

abi = pytest.importorskip("paper_1003_2680_amd.abi")

CASES = [
    ((16, 16, 16), 192, 4, "fp64"),
    ((16, 16, 16), 128, 8, "fp64"),
    ((16, 16, 16), 255, 4, "fp32_refined"),
    ((12, 20, 14), 255, 6, "fp64"),
    ((16, 16, 16), 255, 2, "fp64"),
]


@pytest.mark.parametrize("dims,ncomp,nu,precision", CASES)
def test_workspace_fits(dims, ncomp, nu, precision):
    lib = abi.load()
    desc = abi.GridDesc(*dims, ncomp, 1.0, 1.0)
    prec = abi.SMG_FP64 if precision == "fp64" else abi.SMG_FP32_REFINED
    prm = abi.CycleParams(0, nu, nu, 512, abi.SMG_COARSEST_CHOLESKY, prec, 1, 0)
    hd = ctypes.c_void_p()
    abi.check(lib.smg_create_hierarchy(ctypes.byref(desc), ctypes.byref(prm), ctypes.byref(hd)))
    try:
        info = abi.Info()
        abi.check(lib.smg_hierarchy_info(hd, ctypes.byref(info)))
        print("workspace %.1f MiB" % (info.workspace_bytes / 2**20))
        assert info.workspace_bytes <= abi.SMG_STATIC_SCRATCH_BYTES
    finally:
        lib.smg_destroy_hierarchy(hd)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,ncomp,nu,precision", [CASES[1], CASES[2]])
def test_static_call_runs(dims, ncomp, nu, precision):
    """The call gives the bits of the ordinary entry point, and its first component is the oracle's
    chain (FP64 to 1e-12 of the largest value, FP32-refined to 1e-4 relative RMS)."""
    torch = pytest.importorskip("torch")
    import numpy as np
    from oracle.mg import StochasticMG
    from paper_1003_2680_amd.api import Hierarchy
    print("[gpu-case] static limit %s x %d V(%d,%d) %s" % (dims, ncomp, nu, nu, precision),
          flush=True)
    H = Hierarchy(*dims, ncomp=ncomp, nu1=nu, nu2=nu, precision=precision)
    ref, st_ref = H.sample(2, 7)
    out, st = torch.empty_like(ref), H.new_state()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    abi.check(abi.load().smg_sample_field_static(
        H._h, 2, 7, 0, ptr(st), ptr(out), abi.SMG_OUT_F64,
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and torch.equal(st, st_ref)
    want, _ = StochasticMG(*dims, nu1=nu, nu2=nu, coarsest_max=512).sample_chain(2, 7)
    want = np.asarray(want).reshape(2, -1)
    got = out[:, 0].cpu().numpy().reshape(2, -1)
    if precision == "fp64":
        assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want))
    else:
        assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
