"""The box part of the Schwinger-Dyson stage with two rows k per wave and more than
one chunk of 512 values k', at sizes that fill neither: n = 576 (a second chunk of
64) and n = 630 (a second chunk of 118, a last workgroup of six rows). The vertex
is a seeded low-rank field that the oracle evaluates point by point; compared at
the first row and the last ones.

Tolerances: those of the full-size iteration. Complex128 differs by summation
order (1e-9 of the vertex part, 1e-11 of the whole), complex64 also by the rounding
of Phi (1e-4 of the vertex part, 1e-6 of the whole)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from lowrank_vertex import FullVertex, LowRankVertex
from oracle import parquet as P
from workloads import ModelParams, lowrank_phi_factors, random_sigma

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module", params=[(6, 6, 16), (5, 7, 18)])
def ref(request):
    lx, ly, nv = request.param
    print("CASE sigma rows oracle", lx, ly, nv, flush=True)
    p = ModelParams(Lx=lx, Ly=ly, Nv=nv, U=2.0, beta=5.0, tp=-0.2, mu_mode=0, mu_fixed=0.1, alpha=0.6)
    g = P.Grid(lx, ly, nv, p.f_ext)
    u, v = lowrank_phi_factors(g.Nq, g.n, g.Nk, g.Nv, 41)
    phi = LowRankVertex(u, v)
    mu = P.find_mu(p, g, None)
    G = P.dyson(p, g, random_sigma(g.Nve, g.Nk, 31, scale=0.1), mu)
    K1, K2 = P.kernel_functions(g, phi, p.kernel_level, p.edge_rule)
    top, last = nv // 2 - 1, g.Nk - 1
    pts = [(top, last), (top, last - 4), (-nv // 2, 0)]
    s1 = P.sigma_tilde1(p, g, G, mu)
    base = np.array([s1[g.eidx(n), K] for n, K in pts])
    vertex = P.sigma_tilde2(p, g, G, K1, K2, k_list=pts)
    vertex = vertex + P.sigma_box(p, g, G, FullVertex(g, phi, K1, K2, P.pa_lambda(p.U)), K1, K2, k_list=pts)
    return p, g, u, v, mu, G, K1, K2, pts, base, vertex


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_box_rows(ref, prec):
    p, g, u, v, mu, G, K1, K2, pts, base, vertex = ref
    print("CASE sigma rows", prec, g.n, flush=True)
    from paper_1510_03330_amd.ops import Stage
    st = Stage(p, prec)
    assert st.d.NW * st.d.n >= 8 * 1024 and st.d.n > 512             # the rows and chunks meant above
    phi = torch.empty(st.vshape, dtype=st.vdtype, device=DEV)
    for r in range(4):
        ur = torch.from_numpy(u[r]).to(device=DEV, dtype=st.vdtype)
        vr = torch.from_numpy(np.ascontiguousarray(v[r].transpose(0, 2, 1))).to(device=DEV, dtype=st.vdtype)
        torch.bmm(ur, vr, out=phi[r])

    def T(x, dtype=torch.complex128):
        return torch.from_numpy(np.ascontiguousarray(x)).to(device=DEV, dtype=dtype)

    out = torch.empty(st.sigma_shape, dtype=torch.complex128, device=DEV)
    st.sigma_sde(phi, T(K1), T(K2), T(G), T(np.array([mu]), torch.float64), out)
    torch.cuda.synchronize()
    sig = out.cpu().numpy()
    got = np.array([sig[g.eidx(n), K] for n, K in pts])
    whole = np.max(np.abs(got - base - vertex)) / np.max(np.abs(base + vertex))
    part = np.max(np.abs(got - base - vertex)) / np.max(np.abs(vertex))
    print(f"   whole {whole:.2e}, vertex part {part:.2e}", flush=True)
    assert whole < (1e-11 if prec == "fp64" else 1e-6)
    assert part < (1e-9 if prec == "fp64" else 1e-4)
    del phi
    torch.cuda.empty_cache()
