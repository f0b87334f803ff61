"""Dyson stage with the filling condition against the FP64 oracle at the sizes
where its launch shape changes (self-energy values per lattice: up to 128, 256,
512, 1024, 2048, 4096 and above) and around them, with self-energies of the
size an iteration meets and much larger ones.

Tolerance: both sides bisect to a bracket of 1e-14; the density's rounding
(1e-15 of order-one terms, divided by its slope, above 0.02 here) moves the
result by less than 1e-12."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import parquet as P
from workloads import ModelParams, random_sigma

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("scale", [0.1, 1.0])
@pytest.mark.parametrize("lx,ly,nv,f", [(2, 1, 2, 1), (4, 4, 4, 2), (3, 3, 8, 2), (4, 4, 8, 2), (4, 4, 16, 2), (5, 7, 14, 2),
                                        (8, 8, 8, 2), (8, 8, 16, 2), (8, 8, 10, 3), (8, 8, 32, 2), (8, 8, 14, 5),
                                        (7, 7, 34, 5)])
def test_filling_sizes(lx, ly, nv, f, scale):
    print("CASE dyson sizes", lx, ly, nv, f, scale, flush=True)
    from paper_1510_03330_amd.ops import Stage
    p = ModelParams(Lx=lx, Ly=ly, Nv=nv, U=1.5, beta=4.0, tp=-0.2, f_ext=f, filling=0.87, mu_mode=1)
    g = P.Grid(lx, ly, nv, f)
    sig = random_sigma(g.Nve, g.Nk, seed=9, scale=scale)
    sig = 0.5 * (sig + np.conj(sig[::-1]))
    sig.imag = -np.sign(g.nu(g.fext(), p.beta))[:, None] * np.abs(sig.imag)     # a causal sign: one root
    mu_ref = P.find_mu(p, g, sig)
    G_ref = P.dyson(p, g, sig, mu_ref)
    st = Stage(p, "fp64")
    G = torch.empty(st.g_shape, dtype=torch.complex128, device=DEV)
    mu = torch.empty(1, dtype=torch.float64, device=DEV)
    st.dyson_update(torch.from_numpy(sig).to(DEV), G, mu)
    torch.cuda.synchronize()
    assert abs(float(mu[0]) - mu_ref) < 1e-12
    assert np.max(np.abs(G.cpu().numpy() - G_ref)) / np.max(np.abs(G_ref)) < 1e-11


def test_filling_of_overflowing_and_nan_self_energy():
    """Values beyond the square range leave the density finite (their part is zero); NaN reaches G."""
    from paper_1510_03330_amd.ops import Stage
    p = ModelParams(Lx=2, Ly=2, Nv=4, U=1.5, beta=3.0, tp=-0.1, filling=0.9, mu_mode=1)
    g = P.Grid(2, 2, 4, 2)
    st = Stage(p, "fp64")
    G = torch.empty(st.g_shape, dtype=torch.complex128, device=DEV)
    mu = torch.empty(1, dtype=torch.float64, device=DEV)
    sig = random_sigma(g.Nve, g.Nk, seed=2, scale=0.1)
    sig[3, 1] = 1e200 - 1e200j
    sig[4, 1] = 1e200 + 1e200j
    st.dyson_update(torch.from_numpy(sig).to(DEV), G, mu)
    torch.cuda.synchronize()
    assert np.isfinite(G.cpu().numpy()).all() and abs(float(mu[0])) < 10
    sig[3, 1] = np.nan
    st.dyson_update(torch.from_numpy(sig).to(DEV), G, mu)
    torch.cuda.synchronize()
    assert np.isnan(G.cpu().numpy()).any()
