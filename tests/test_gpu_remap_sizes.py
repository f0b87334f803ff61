"""Kernel functions and channel remap against the FP64 oracle at the lattice
sizes where their launches change: rows of 1, 2, 4, 8 and 16 lanes, the direct
gather (up to 12 momenta) and every tile shape of the tiled kernel above it,
with workgroup counts that do and do not divide over the XCDs.

Tolerances: sums of at most nine terms of size one (1e-13 relative in
complex128, a few ulp of FP32 in complex64) and means of up to 64 values."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import parquet as P
from workloads import ModelParams, lambda_box_parts, random_phi

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def T(x, dtype=torch.complex128):
    return torch.from_numpy(np.ascontiguousarray(x)).to(device=DEV, dtype=dtype)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("lx,ly,nv,box", [(1, 1, 2, False), (1, 1, 10, True), (1, 2, 6, False), (1, 3, 4, False), (1, 5, 4, True),
                                          (3, 3, 4, False), (2, 6, 4, True), (13, 1, 4, False), (4, 4, 4, True),
                                          (17, 1, 2, False), (4, 5, 4, True), (23, 1, 2, False), (5, 5, 2, True),
                                          (3, 9, 2, False), (8, 4, 2, False), (3, 11, 2, True), (5, 7, 4, False),
                                          (39, 1, 2, False), (8, 5, 2, True), (9, 5, 2, False), (7, 7, 2, True),
                                          (51, 1, 2, False), (11, 5, 2, False), (7, 8, 2, True), (8, 8, 4, False)])
def test_kernels_and_remap_sizes(prec, lx, ly, nv, box):
    print("CASE remap sizes", prec, lx, ly, nv, box, flush=True)
    from paper_1510_03330_amd.ops import Stage
    p = ModelParams(Lx=lx, Ly=ly, Nv=nv, U=1.2, beta=3.0, tp=-0.1)
    g = P.Grid(lx, ly, nv, 2)
    phi = random_phi(g.Nq, g.n, seed=23, scale=0.5)
    if prec == "fp32":
        phi = phi.astype(np.complex64).astype(np.complex128)
    st = Stage(p, prec)
    k1 = torch.empty(st.k1_shape, dtype=torch.complex128, device=DEV)
    k2 = torch.empty(st.k2_shape, dtype=torch.complex128, device=DEV)
    dphi = T(phi, st.vdtype)
    st.kernel_extract(dphi, k1, k2)
    K1, K2 = P.kernel_functions(g, phi, 2)
    torch.cuda.synchronize()
    assert np.max(np.abs(k1.cpu().numpy() - K1)) < 1e-14
    assert np.max(np.abs(k2.cpu().numpy() - K2)) < 1e-14
    lam, lam_box = P.pa_lambda(p.U), None
    if box:
        a, b = lambda_box_parts(nv, seed=5)
        lam = np.stack([a, b, 0.5 * a, 0.25 * b])
        lam_box = T(lam)
    gamma = torch.full(st.vshape, float("nan"), dtype=st.vdtype, device=DEV)
    st.channel_remap(P.pa_lambda(p.U), dphi, k1, k2, gamma, lam_box=lam_box)
    ref = P.remap(g, phi, K1, K2, lam)
    torch.cuda.synchronize()
    err = np.max(np.abs(gamma.cpu().numpy() - ref)) / np.max(np.abs(ref))
    assert err < (1e-13 if prec == "fp64" else 1e-6), err
