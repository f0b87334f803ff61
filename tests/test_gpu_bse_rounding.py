"""Rounding of the complex128 diagonal-block inversion P where A = 1 - s Gamma X is
near one and its entries repeat over the momenta, as at weak coupling: Phi is then
what is left of F after Gamma, and the error of P's diagonal is all of Phi's.

One panel (n = 64). Three of the four frequencies have columns Gamma(f, f') equal
over the momenta; a column of the last one holds a single 1, in row j of the first,
so that Phi there is column j of P - 1. Gamma and X have few bits: A is exact.

Tolerance (RMS over P's diagonal): an entry near one is rounded twice for each of the
15 other pivots of its 16-wide tile, once for each of the two other tiles with
coupling, and about three times in its pivot's reciprocal: 35 roundings, each at
most half an ulp of [1, 2), 0.64e-16 RMS, together 3.8e-16; 4.5e-16 leaves the spread
of an RMS over 768 entries. (Rounded with every term of the other tiles it
is 97 of them, 6.3e-16, and more where equal terms round alike.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from workloads import ModelParams

DEV = "cuda:0"
NK, NF, N = 16, 4, 64


def blocks(count, seed):
    """Gamma [count][64][64] and X [count][64], products exact in a double."""
    rng = np.random.default_rng(seed)
    g = np.zeros((count, N, N), dtype=np.complex128)
    x = np.zeros((count, N), dtype=np.complex128)
    for b in range(count):
        gf = rng.integers(512, 1536, (NF, NF - 1)) / 1024 + 1j * rng.integers(-128, 128, (NF, NF - 1)) / 1024
        xf = rng.integers(2 ** 7, 2 ** 9, NF) / 2 ** 20 + 1j * rng.integers(-2 ** 7, 2 ** 7, NF) / 2 ** 20
        g[b, :, :N - NK] = np.kron(gf, np.ones((NK, NK)))
        g[b, np.arange(NK), N - NK + np.arange(NK)] = 1.0
        x[b] = np.repeat(xf * rng.choice([-1.0, 1.0]), NK)
    return g, x


def inverse(a):
    """of [count][n][n] in extended precision, one pivot at a time"""
    a = a.astype(np.clongdouble)
    for c in range(a.shape[-1]):
        p = 1 / a[:, c, c]
        col, row = a[:, :, c].copy(), a[:, c, :] * p[:, None]
        row[:, c] = p
        a[:, :, c] = 0
        a -= col[:, :, None] * row[:, None, :]
        a[:, c, :] = row
    return a


@pytest.mark.gpu
@pytest.mark.parametrize("channel", [0, 2])
def test_inverse_near_one(channel):
    print("CASE bse rounding", channel, flush=True)
    from paper_1510_03330_amd.ops import Stage
    st = Stage(ModelParams(Lx=4, Ly=4, Nv=4, U=1.0, beta=2.0, mu_mode=0, alpha=0.5), "fp64")
    assert (st.d.n, st.d.Nk) == (N, NK)
    g, x = blocks(st.d.Nq, 3 + channel)
    p = inverse(np.eye(N) - (-1 if channel == 2 else 1) * g * x[:, None, :])
    G, X = torch.from_numpy(g).to(DEV), torch.from_numpy(x).to(DEV)
    phi = torch.zeros_like(G)
    st.bse_solve(channel, G, X, phi, alpha=1.0)
    torch.cuda.synchronize()
    j = np.arange(NK)
    err = (phi.cpu().numpy()[:, j, N - NK + j] + np.longdouble(1) - p[:, j, j]).real
    rms = float(np.sqrt(np.mean(err ** 2)))
    print(f"   rms {rms:.2e}", flush=True)
    assert rms < 4.5e-16
