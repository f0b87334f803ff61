// Regulated Schwinger-Dyson self-energy (high-frequency regulation subsection
// of the paper, Eq. PA_Sigma with the auxiliary vertex):
//
//   Sigma(k) = Sigma~_1(k) + Sigma~_2(k) + [k in box] Sigma_box(k)
//
// Sigma~_1 is the second-order diagram -U^2 G(r)^2 G(-r) over all Matsubara
// frequencies. G is split into its non-interacting pole part (transformed to
// imaginary time analytically, anti-periodic) and a correction supported on
// the extended box (a finite Fourier sum); the tau integral is analytic on
// [0, beta] and is done by Fejer's quadrature rule, momenta by direct
// lattice Fourier sums.
//
// Sigma~_2 and Sigma_box are evaluated in "native" variables: every term of
// F - F~ (resp. F~ - Lambda) is a reducible vertex P_r(k, b; p) at its own
// argument triple, so substituting (k', q) -> (b, p) turns both sums into
//   C sum_{p in bosonic box} sum_b { A1 [P_d W16 - P_m (W16 + 2 W25)] + A3 (P_s + P_t) W34 }
// with A1 = G(k+p) G(b+p) G(b), A3 = G(p-b) G(p-k) G(b), C = -U T^2 / 4N^2 and
// integer indicator weights W that encode which original (k', q) lie in the
// summation domain. The box part then only streams Phi (no Gamma, no
// gathers), and the kernel part only needs contiguous rows of K2.
#include <math.h>

#include <algorithm>
#include <mutex>

#include "pq_internal.h"

namespace pq {

namespace {

constexpr int kThreads = 256;
constexpr int kPoles = 128;   // semicircle pole representation (Gauss-Chebyshev)

__device__ inline double nu_of(int n, double beta) { return (2 * n + 1) * M_PI / beta; }

__device__ inline double pole_tau(double e, double tau, double tauc, double beta) {
  // imaginary-time transform of 1/(i nu - e), 0 < tau < beta, tauc = beta - tau
  if (e >= 0.0) return -exp(-e * tau) / (1.0 + exp(-beta * e));
  return -exp(e * tauc) / (exp(beta * e) + 1.0);
}

__device__ inline void semicircle_pole(int l, double D, double* e, double* c) {
  double th = (l + 1) * M_PI / (kPoles + 1);
  double s = sin(th);
  *e = D * cos(th);
  *c = 2.0 * s * s / (kPoles + 1);
}

__device__ inline double eps_of(int K, const Dims& d, double t, double tp) {
  int kx = K / d.Ly, ky = K - (K / d.Ly) * d.Ly;
  double cx = cos(2.0 * M_PI * kx / d.Lx), cy = cos(2.0 * M_PI * ky / d.Ly);
  return -2.0 * t * (cx + cy) - 4.0 * tp * cx * cy;
}

// exp(+2 pi i (kx rx / Lx + ky ry / Ly)) from the two one-dimensional phase
// tables tx[Lx], ty[Ly] of a workgroup
__device__ inline double2 lattice_phase(int K, int R, const Dims& d, const double2* tx, const double2* ty) {
  const int kx = K / d.Ly, ky = K - kx * d.Ly, rx = R / d.Ly, ry = R - rx * d.Ly;
  return cmul(tx[(kx * rx) % d.Lx], ty[(ky * ry) % d.Ly]);
}

__device__ inline void phase_tables(const Dims& d, double2* tx, double2* ty) {
  for (int i = threadIdx.x; i < d.Lx + d.Ly; i += blockDim.x) {
    const bool x = i < d.Lx;
    const int m = x ? i : i - d.Lx;
    double sn, cs;
    sincospi(2.0 * m / (x ? d.Lx : d.Ly), &sn, &cs);
    (x ? tx[m] : ty[m]) = mk(cs, sn);
  }
}

constexpr int kMaxNk = 64;     // momenta of the largest lattice

__host__ __device__ inline int pow2_ge(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

struct S1Args {
  Dims d;
  double beta, U, t, tp, D;
  int local;
  const double2* g;      // [NG][Nk]
  const double* mu;
  double2* srt;          // [ntau][Nk] w_j U^2 G(R, tau_j)^2 G(-R, beta - tau_j)
  double2* out;          // [Nve][Nk]
};

// Quadrature of the tau integral: Fejer's first rule on [0, beta] (Chebyshev
// points, L. Fejer 1933; weights in closed form, J. Waldvogel, BIT 46, 2006),
//   tau_j = beta sin^2(theta_j / 2),  theta_j = (j + 1/2) pi / N,
//   w_j = (beta / N) [1 - 2 sum_{k=1}^{N/2} cos(2 k theta_j) / (4 k^2 - 1)],
// symmetric (tau_{N-1-j} = beta - tau_j exactly). The integrand has the
// frequencies up to 4 nu_max and exponentials exp(-3 E tau): its Chebyshev
// coefficients fall off beyond degree 2 pi f Nv + O(beta E), which N = 8 f Nv +
// 64 + 4 beta E exceeds. (Gauss-Legendre nodes are exact to twice the degree but
// need N-long serial recurrences per Newton step: 103-223 us a call measured,
// against a few cosines per node here.)
//
// One workgroup per pair (j, N-1-j) (N is even), so that G(R, tau_j) and G(-R, beta - tau_j)
// meet in one workgroup: dG = G - G_pole on the extended box, the imaginary-time
// sums over its frequencies (exp(-i nu (beta - tau)) = -exp(i nu tau): one phase
// serves both nodes), the lattice transform and the product, which kernels of
// their own did before with one thread per output and a sincos per term (4x4,
// Nv = 16: 19 + 9 us; one momentum, Nv = 32: 67 + 84 us for the pole sums).
// Latency-bound: a few hundred operations per thread, N / 2 workgroups; at one
// momentum the pole sums (64 divisions per frequency) on four lanes each, 14.2 ->
// 12.0 us at Nv = 32.
template <int N>
__global__ __launch_bounds__(kThreads) void s1_tau_kernel(Many<S1Args, N> m) {
  const S1Args& a = m.a[N == 1 ? 0 : blockIdx.z];
  if ((int)blockIdx.x >= a.d.ntau / 2) return;           // an instance of fewer nodes than the launch's most
  __shared__ double2 ph[kThreads];
  __shared__ double2 red[2][kThreads];
  __shared__ double2 gk[2][kMaxNk];
  __shared__ double2 tx[kMaxNk], ty[kMaxNk];
  __shared__ double pe[kPoles], pc[kPoles];
  __shared__ double rsum[kThreads];
  __shared__ double gl[kThreads];                        // one momentum: sum of the poles per frequency
  const Dims& d = a.d;
  const int t = threadIdx.x, nt = d.ntau, j = blockIdx.x, Nk = d.Nk;
  const double sj = sinpi((j + 0.5) / (2.0 * nt)), cj = cospi((j + 0.5) / (2.0 * nt));
  const double u = sj * sj;                              // tau_j / beta
  const double tau = a.beta * u, tauc = a.beta * (cj * cj);
  double ws = 0.0;
  for (int k = 1 + t; k <= nt / 2; k += kThreads) {
    const long long r = ((long long)k * (2 * j + 1)) % (2 * nt);
    ws += cospi((double)r / nt) / (4.0 * k * k - 1.0);
  }
  phase_tables(d, tx, ty);
  if (a.local)
    for (int l = t; l < kPoles; l += kThreads) {
      semicircle_pole(l, a.D, &pe[l], &pc[l]);
    }
  const double w = (a.beta / nt) * (1.0 - 2.0 * block_sum(ws, rsum));
  // G(K, tau_j) and G(K, beta - tau_j): momentum K = t % NkP, a slice of the frequencies each
  const int NkP = pow2_ge(Nk), nsl = kThreads / NkP, K = t % NkP, sl = t / NkP;
  const bool live = K < Nk;
  const double xi = live && !a.local ? eps_of(K, d, a.t, a.tp) - *a.mu : 0.0;
  double2 acc0 = mk(0, 0), acc1 = mk(0, 0);
  for (int e0 = 0; e0 < d.Nve; e0 += kThreads) {
    __syncthreads();
    if (e0 + t < d.Nve) {                                // exp(-i nu_e tau_j)
      double sn, cs;
      sincospi((2 * (e0 + t - d.Nve / 2) + 1) * u, &sn, &cs);
      ph[t] = mk(cs, -sn);
    }
    if (a.local) {                                       // poles come in pairs +-e_l; 4 lanes a frequency
      const int cn = min(kThreads, d.Nve - e0);
      for (int x = t; x < 4 * cn; x += kThreads) {
        const double nu = nu_of(e0 + (x >> 2) - d.Nve / 2, a.beta);
        double s = 0.0;
        for (int l = x & 3; l < kPoles / 2; l += 4) s += pc[l] / (nu * nu + pe[l] * pe[l]);
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        if ((x & 3) == 0) gl[x >> 2] = -2.0 * nu * s;
      }
    }
    __syncthreads();
    if (live)
      for (int e = e0 + sl; e < min(d.Nve, e0 + kThreads); e += nsl) {
        const int n = e - d.Nve / 2;
        const double nu = nu_of(n, a.beta);
        double2 gp;
        if (a.local) {
          gp = mk(0.0, gl[e - e0]);
        } else {
          gp = crecip(mk(-xi, nu));
        }
        const double2 dg = csub(a.g[(size_t)(n + d.NG / 2) * Nk + K], gp);
        const double2 p = ph[e - e0];
        acc0 = cadd(acc0, cmul(dg, p));
        acc1 = csub(acc1, cmul(dg, mk(p.x, -p.y)));
      }
  }
  red[0][t] = acc0;
  red[1][t] = acc1;
  double pole0 = 0.0, pole1 = 0.0;
  if (a.local) {
    double s0 = 0.0, s1 = 0.0;
    for (int l = t; l < kPoles; l += kThreads) {
      s0 += pc[l] * pole_tau(pe[l], tau, tauc, a.beta);
      s1 += pc[l] * pole_tau(pe[l], tauc, tau, a.beta);
    }
    pole0 = block_sum(s0, rsum);
    pole1 = block_sum(s1, rsum);
  } else if (live) {
    pole0 = pole_tau(xi, tau, tauc, a.beta);
    pole1 = pole_tau(xi, tauc, tau, a.beta);
  }
  __syncthreads();
  for (int st = nsl / 2; st > 0; st >>= 1) {
    if (sl < st) {
      red[0][t] = cadd(red[0][t], red[0][t + st * NkP]);
      red[1][t] = cadd(red[1][t], red[1][t + st * NkP]);
    }
    __syncthreads();
  }
  if (t < Nk) {
    gk[0][t] = mk(pole0 + red[0][t].x / a.beta, red[0][t].y / a.beta);
    gk[1][t] = mk(pole1 + red[1][t].x / a.beta, red[1][t].y / a.beta);
  }
  __syncthreads();
  // G(R, tau) = (1/N) sum_K e^{i K R} G(K, tau), a slice of the momenta per thread
  acc0 = acc1 = mk(0, 0);
  if (live)
    for (int k = sl; k < Nk; k += nsl) {
      const double2 p = lattice_phase(k, K, d, tx, ty);
      acc0 = cadd(acc0, cmul(p, gk[0][k]));
      acc1 = cadd(acc1, cmul(p, gk[1][k]));
    }
  red[0][t] = acc0;
  red[1][t] = acc1;
  __syncthreads();
  for (int st = nsl / 2; st > 0; st >>= 1) {
    if (sl < st) {
      red[0][t] = cadd(red[0][t], red[0][t + st * NkP]);
      red[1][t] = cadd(red[1][t], red[1][t + st * NkP]);
    }
    __syncthreads();
  }
  if (t < Nk) {
    const int rx = t / d.Ly, ry = t - rx * d.Ly;
    const int mR = ((d.Lx - rx) % d.Lx) * d.Ly + (d.Ly - ry) % d.Ly;
    const double f = a.U * a.U * w / ((double)Nk * Nk * Nk);
    const double2 g0 = red[0][t], g1 = red[1][t];
    a.srt[(size_t)j * Nk + t] = cscale(cmul(cmul(g0, g0), red[1][mR]), f);
    a.srt[(size_t)(nt - 1 - j) * Nk + t] = cscale(cmul(cmul(g1, g1), red[0][mR]), f);
  }
}

// Sigma~_1(K, e) = sum_R e^{-i K R} sum_j e^{i nu_e tau_j} srt[j][R]: one
// workgroup per frequency e, a slice of the nodes per thread (the sums over the
// nodes ran serially in one thread per output before: 103-200 us).
constexpr int kRowThreads = 1024;
template <int N>
__global__ __launch_bounds__(kRowThreads) void s1_row_kernel(Many<S1Args, N> m) {
  const S1Args& a = m.a[N == 1 ? 0 : blockIdx.z];
  __shared__ double2 ph[kRowThreads];
  __shared__ double2 red[kRowThreads];
  __shared__ double2 tx[kMaxNk], ty[kMaxNk];
  const Dims& d = a.d;
  const int t = threadIdx.x, nt = d.ntau, e = blockIdx.x, Nk = d.Nk;
  const int NkP = pow2_ge(Nk), nsl = kRowThreads / NkP, R = t % NkP, sl = t / NkP;
  phase_tables(d, tx, ty);
  double2 acc = mk(0, 0);
  for (int j0 = 0; j0 < nt; j0 += kRowThreads) {
    __syncthreads();
    if (j0 + t < nt) {
      const double s = sinpi((j0 + t + 0.5) / (2.0 * nt));
      double sn, cs;
      sincospi((2 * (e - d.Nve / 2) + 1) * (s * s), &sn, &cs);
      ph[t] = mk(cs, sn);
    }
    __syncthreads();
    if (R < Nk) {
      const int hi = min(nt, j0 + kRowThreads);
#pragma unroll 4
      for (int j = j0 + sl; j < hi; j += nsl) acc = cadd(acc, cmul(ph[j - j0], a.srt[(size_t)j * Nk + R]));
    }
  }
  for (int pass = 0; pass < 2; ++pass) {        // the sum over the nodes, then over R
    red[t] = acc;
    __syncthreads();
    for (int st = nsl / 2; st > 0; st >>= 1) {
      if (sl < st) red[t] = cadd(red[t], red[t + st * NkP]);
      __syncthreads();
    }
    if (pass == 1) break;
    acc = mk(0, 0);
    if (R < Nk)
      for (int k = sl; k < Nk; k += nsl) {
        const double2 p = lattice_phase(R, k, d, tx, ty);
        acc = cadd(acc, cmul(mk(p.x, -p.y), red[k]));
      }
    __syncthreads();
  }
  if (t < Nk) a.out[(size_t)e * Nk + t] = red[t];
}

// ------------------------------------------------------------- Sigma~_2
// Re-indexed to native variables (transfer p = (m_p, P), second fermionic
// argument b = (n_b, B)), every term is a product of a G factor of (k, p), the
// indicator weights e16, e25, e34 of the summation domain, which depend on the
// frequencies (n_k, m_p, n_b) only, and momentum-dependent factors of (p, b).
// The momentum sums are therefore done first, once per (p, n_b):
//   U1 = sum_B G(b+p) G(b),  U3 = sum_B G(p-b) G(b),
//   V1d, V1m = sum_B G(b+p) G(b) K2_{d,m}(b;p),  V3st = sum_B G(p-b) G(b) (K2_s + K2_t)(b;p)
// (the V's for b in the box), then the sums over n_b once per (n_k, p),
//   A16 = sum e16 U1,  A25 = sum e25 U1,  A34 = sum e34 U3,
//   B1 = sum [e16 V1d - (e16 + 2 e25) V1m],  B3 = sum e34 V3st,
// and for every k
//   s16 = G(k+p) A16,  s25 = G(k+p) A25,  s34 = G(p-k) A34,  sk = G(k+p) B1 + G(p-k) B3.
struct S2Args {
  Dims d;
  int level;
  const double2* g;
  const double2* k1;     // [4][Nq]
  const double2* k2;     // [4][Nq][n]
  double2* tab;          // [Nve][5][Nq]  A16, A25, A34, B1, B3 per (n_k, p)
};

__device__ inline double ind(bool b) { return b ? 1.0 : 0.0; }

__device__ inline double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

constexpr int kS2Chunk = 256;    // frequencies n_b whose U, V lie in LDS at a time (20 KB)
constexpr int kS2Sl = 8;         // lanes that share a sum over n_b

// One workgroup per transfer p (of few transfers: per p and 32 n_k, up to 1024
// workgroups): U and V of a chunk of frequencies into LDS (sw
// lanes, the power of two >= Nk, per n_b, over the momentum B), then the sums over
// n_b, kS2Sl lanes for each of 32 n_k at a time. A box of more than kS2Chunk
// frequencies forms its chunks again for every 32 n_k. Bound by its integer and
// weight arithmetic (about 150 instructions per (n_k, n_b, p)), which a kernel with
// one workgroup per k did for every momentum K of k before. With the sums over p
// (sigma2_kernel), before -> now: 4x4, Nv = 16: 40 -> 24 us, 8x8, Nv = 8: 66 -> 57,
// one momentum, Nv = 32: 16 -> 15; 16 lanes a sum 25, 60, 13 us, 32 lanes 36, 83, 13.
template <int N>
__global__ __launch_bounds__(kThreads) void s2_sums_kernel(Many<S2Args, N> m, int sw) {
  const S2Args& a = m.a[N == 1 ? 0 : blockIdx.z];
  __shared__ double2 tab[5][kS2Chunk];
  const Dims& d = a.d;
  const int qi = blockIdx.x, t = threadIdx.x;
  const int jm = qi / d.Nk, P = qi - jm * d.Nk, mp = jm - (d.Nv / 2 - 1);
  const int hF = d.Nve / 2, hBe = d.Nve / 2 - 1, hG = d.NG / 2;
  const size_t n = d.n;
  const int sl = t % kS2Sl;
  constexpr int EK = kThreads / kS2Sl;
  bool formed = false;
  for (int ek0 = blockIdx.y * EK; ek0 < d.Nve; ek0 += gridDim.y * EK) {
    const int ek = ek0 + t / kS2Sl, nk = ek - hF;
    const bool kbox = in_fbox(nk, d.Nv);
    const int nkp = nk + mp;
    const bool Ye = nkp >= -hF && nkp <= hF - 1;
    const bool Yb = in_fbox(nkp, d.Nv);
    int lo = min(-hF, min(nk - hBe, -mp - nk - 1 - hBe));
    int hi = max(hF - 1, max(nk + hBe, -mp - nk - 1 + hBe));
    lo = max(lo, -hG);
    hi = ek < d.Nve ? min(hi, hG - 1) : lo - 1;
    double2 a16 = mk(0, 0), a25 = mk(0, 0), a34 = mk(0, 0), b1 = mk(0, 0), b3 = mk(0, 0);
    for (int c0 = 0; c0 < d.NG; c0 += kS2Chunk) {
      if (!formed || d.NG > kS2Chunk) {
        formed = true;
        __syncthreads();
        const int lane = t & (sw - 1), cn = min(kS2Chunk, d.NG - c0);
        for (int x = t / sw; x < cn; x += kThreads / sw) {        // uniform over the sw lanes
          const int nb = c0 + x - hG;
          const bool r1 = nb + mp >= -hG && nb + mp < hG, r3 = mp - nb - 1 >= -hG && mp - nb - 1 < hG;
          const bool kb2 = in_fbox(nb, d.Nv) && a.level >= 2;
          double v[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
          if (lane < d.Nk) {
            const int B = lane;
            const double2 gb = a.g[(size_t)(nb + hG) * d.Nk + B];
            const double2 g1 = r1 ? a.g[(size_t)(nb + mp + hG) * d.Nk + kadd(B, P, d.Lx, d.Ly)] : mk(0, 0);
            const double2 g3 = r3 ? a.g[(size_t)(mp - nb - 1 + hG) * d.Nk + ksub(P, B, d.Lx, d.Ly)] : mk(0, 0);
            const double2 u1 = cmul(g1, gb), u3 = cmul(g3, gb);
            double2 w1d = mk(0, 0), w1m = mk(0, 0), w3 = mk(0, 0);
            if (kb2) {
              const size_t bidx = (size_t)(nb + d.Nv / 2) * d.Nk + B;
              w1d = cmul(u1, a.k2[((size_t)0 * d.Nq + qi) * n + bidx]);
              w1m = cmul(u1, a.k2[((size_t)1 * d.Nq + qi) * n + bidx]);
              w3 = cmul(u3, cadd(a.k2[((size_t)2 * d.Nq + qi) * n + bidx], a.k2[((size_t)3 * d.Nq + qi) * n + bidx]));
            }
            v[0] = u1.x; v[1] = u1.y; v[2] = u3.x; v[3] = u3.y;
            v[4] = w1d.x; v[5] = w1d.y; v[6] = w1m.x; v[7] = w1m.y; v[8] = w3.x; v[9] = w3.y;
          }
          for (int o = sw >> 1; o > 0; o >>= 1) {
#pragma unroll
            for (int i = 0; i < 10; ++i) v[i] += __shfl_xor(v[i], o, 64);
          }
          if (lane == 0)
            for (int i = 0; i < 5; ++i) tab[i][x] = mk(v[2 * i], v[2 * i + 1]);
        }
        __syncthreads();
      }
      const int last = min(hi, c0 + kS2Chunk - 1 - hG);
      for (int nb = max(lo, c0 - hG) + sl; nb <= last; nb += kS2Sl) {
        const bool bFe = nb >= -hF && nb <= hF - 1;
        const bool bFb = in_fbox(nb, d.Nv);
        const int x1 = mp + nk + nb + 1, x2 = nb - nk, x3 = mp - nk - nb - 1;
        double e16 = bFe ? 1.0 + ind(x1 >= -hBe && x1 <= hBe) : 0.0;
        double e25 = Ye ? ind(x2 >= -hBe && x2 <= hBe) + ind(x1 >= -hBe && x1 <= hBe) : 0.0;
        double e34 = bFe ? 1.0 + ind(x3 >= -hBe && x3 <= hBe) : 0.0;
        if (kbox && bFb) {
          e16 -= 1.0 + ind(in_bbox(x1, d.Nv));
          e25 -= Yb ? ind(in_bbox(x2, d.Nv)) + ind(in_bbox(x1, d.Nv)) : 0.0;
          e34 -= 1.0 + ind(in_bbox(x3, d.Nv));
        }
        if (e16 == 0.0 && e25 == 0.0 && e34 == 0.0) continue;
        const int x = nb + hG - c0;
        const double2 u1 = tab[0][x], u3 = tab[1][x];
        a16 = cadd(a16, cscale(u1, e16));
        a25 = cadd(a25, cscale(u1, e25));
        a34 = cadd(a34, cscale(u3, e34));
        if (bFb && a.level >= 2) {
          b1 = cadd(b1, csub(cscale(tab[2][x], e16), cscale(tab[3][x], e16 + 2.0 * e25)));
          b3 = cadd(b3, cscale(tab[4][x], e34));
        }
      }
    }
    double v[10] = {a16.x, a16.y, a25.x, a25.y, a34.x, a34.y, b1.x, b1.y, b3.x, b3.y};
#pragma unroll
    for (int o = kS2Sl / 2; o > 0; o >>= 1)
#pragma unroll
      for (int i = 0; i < 10; ++i) v[i] += __shfl_xor(v[i], o, 64);
    if (sl == 0 && ek < d.Nve)
      for (int i = 0; i < 5; ++i) a.tab[((size_t)ek * 5 + i) * d.Nq + qi] = mk(v[2 * i], v[2 * i + 1]);
  }
}

struct CombineArgs {
  Dims d;
  double cfac;
  int has_s2;
  const double2* s1;
  const double2* partial;
  const double2* lam_part;   // nullable: the box-Lambda term per box k
  double2* out;
};

// The sum of the pieces, one workgroup per k point of the extended box:
// Sigma~_1 plus the Schwinger-Dyson constant times the kernel part (threads over
// the transfers p), the box part's sums over the bosonic index, and the box Lambda.
template <int N>
__global__ __launch_bounds__(kThreads) void sigma2_kernel(Many<S2Args, N> m2, Many<CombineArgs, N> mc) {
  const S2Args& a = m2.a[N == 1 ? 0 : blockIdx.z];
  const CombineArgs& c_ = mc.a[N == 1 ? 0 : blockIdx.z];
  __shared__ double red[kThreads];
  const Dims& d = a.d;
  const int kid = blockIdx.x;
  const int ek = kid / d.Nk, K = kid - ek * d.Nk;
  const int nk = ek - d.Nve / 2;
  const bool kbox = in_fbox(nk, d.Nv);
  const int kbi = kbox ? (nk + d.Nv / 2) * d.Nk + K : 0;
  const int hBb = d.Nv / 2 - 1, hG = d.NG / 2;
  const size_t n = d.n, nq = d.Nq;
  double tr = 0.0, ti = 0.0;
  for (int qi = threadIdx.x; c_.has_s2 && qi < d.Nq; qi += kThreads) {
    const int jm = qi / d.Nk, P = qi - jm * d.Nk;
    const int mp = jm - hBb;
    double2 c[4];
    for (int r = 0; r < 4; ++r) {
      c[r] = a.k1[(size_t)r * d.Nq + qi];
      if (kbox && a.level >= 2) c[r] = cadd(c[r], a.k2[((size_t)r * d.Nq + qi) * n + kbi]);
    }
    const int nkp = nk + mp;
    const double2 g_kp = a.g[(size_t)(nkp + hG) * d.Nk + kadd(K, P, d.Lx, d.Ly)];
    const double2 g_pk = a.g[(size_t)(mp - nk - 1 + hG) * d.Nk + ksub(P, K, d.Lx, d.Ly)];
    const double2* t = a.tab + (size_t)ek * 5 * nq + qi;
    const double2 s16 = cmul(g_kp, t[0]), s25 = cmul(g_kp, t[nq]), s34 = cmul(g_pk, t[2 * nq]);
    const double2 sk = cadd(cmul(g_kp, t[3 * nq]), cmul(g_pk, t[4 * nq]));
    double2 contrib = cmul(c[0], s16);
    contrib = csub(contrib, cmul(c[1], cadd(s16, cscale(s25, 2.0))));
    contrib = cadd(contrib, cmul(cadd(c[2], c[3]), s34));
    contrib = cadd(contrib, sk);
    tr += contrib.x;
    ti += contrib.y;
  }
  if (kbox) {
    for (int j = threadIdx.x; j < d.NW; j += blockDim.x) {
      const double2 v = c_.partial[(size_t)kbi * d.NW + j];
      tr += v.x;
      ti += v.y;
    }
    if (c_.lam_part && threadIdx.x == 0) {
      tr += c_.lam_part[kbi].x;
      ti += c_.lam_part[kbi].y;
    }
  }
  tr = block_sum(tr, red);
  ti = block_sum(ti, red);
  if (threadIdx.x == 0) {
    const double2 s = c_.s1[kid];
    c_.out[kid] = mk(s.x + c_.cfac * tr, s.y + c_.cfac * ti);
  }
}

// ------------------------------------------------------------ Sigma_box
template <typename C>
struct SBArgs {
  Dims d;
  const C* phi;          // [4][Nq][n][n]
  const double2* g;
  double2* partial;      // [n][NW]
};

// 16-byte streaming loads of E consecutive complex values (E = 2 complex64,
// 1 complex128): Phi is read exactly once, so the loads bypass the caches'
// retention (non-temporal), which lets the read stream run closer to the HBM
// read rate.
typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
template <typename C> struct Row16;
template <> struct Row16<float2> {
  static constexpr int E = 2;
  __device__ static void load(const float2* p, double2 (&o)[2]) {
    const f4v v = __builtin_nontemporal_load((const f4v*)p);
    o[0] = mk(v.x, v.y);
    o[1] = mk(v.z, v.w);
  }
};
template <> struct Row16<double2> {
  static constexpr int E = 1;
  __device__ static void load(const double2* p, double2 (&o)[1]) {
    const d2v v = __builtin_nontemporal_load((const d2v*)p);
    o[0] = mk(v.x, v.y);
  }
};

// The box part of Eq. PA_Sigma at the bosonic index m = blockIdx.x for 4 RPW
// rows k (RPW per wave) of the four channels, summed over Q and k'. HBM-bound:
// Phi is streamed once. The products G(k'+q) G(k') and G(q-k') G(k') do not
// depend on k: they are formed once per (q, k') and workgroup in LDS (in chunks
// of kBoxChunk), and G(k+q), G(q-k) multiply the rows' sums, so an element
// costs two multiply-adds per product (one row per workgroup with every product
// formed per element took 6.1 ms on the 8x8, Nv = 16 complex64 box, 5.3 TB/s,
// against 4.8 ms, 6.7 TB/s, now). Each lane takes E consecutive k' per 16-byte load
// (n is even, rows start 16-byte aligned).
constexpr int kBoxChunk = 512;

template <typename C, int RPW>
__global__ __launch_bounds__(kThreads) void sigmab_kernel(SBArgs<C> a) {
  __shared__ double2 u1[kBoxChunk], u3[kBoxChunk];
  __shared__ short bf[kBoxChunk];                  // frequency of k'
  using L16 = Row16<C>;
  constexpr int E = L16::E;
  const Dims& d = a.d;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int jm = blockIdx.x, mp = jm - (d.Nv / 2 - 1), hG = d.NG / 2;
  const size_t n = d.n, nn = (size_t)d.n * d.n, chan = (size_t)d.cs;
  int row[RPW], nk[RPW], K[RPW];
  double2 acc[RPW];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    row[r] = min((int)(blockIdx.y * 4 + wave) * RPW + r, d.n - 1);
    nk[r] = row[r] / d.Nk - d.Nv / 2;
    K[r] = row[r] % d.Nk;
    acc[r] = mk(0, 0);
  }
  for (int P = 0; P < d.Nk; ++P) {
    double2 s1[RPW], s3[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) s1[r] = s3[r] = mk(0, 0);
    const C* base = a.phi + (size_t)(jm * d.Nk + P) * nn;
    for (int b0 = 0; b0 < d.n; b0 += kBoxChunk) {
      const int nb_ = min(kBoxChunk, d.n - b0);
      __syncthreads();
      for (int i = t; i < nb_; i += kThreads) {
        const int b = b0 + i, f = b / d.Nk, B = b - f * d.Nk, nb = f - d.Nv / 2;
        const double2 gb = a.g[(size_t)(nb + hG) * d.Nk + B];
        u1[i] = cmul(a.g[(size_t)(nb + mp + hG) * d.Nk + kadd(B, P, d.Lx, d.Ly)], gb);
        u3[i] = cmul(a.g[(size_t)(mp - nb - 1 + hG) * d.Nk + ksub(P, B, d.Lx, d.Ly)], gb);
        bf[i] = (short)nb;
      }
      __syncthreads();
      for (int i = lane * E; i < nb_; i += 64 * E) {
        double2 pv[RPW][4][E];
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
          for (int c = 0; c < 4; ++c) L16::load(base + c * chan + (size_t)row[r] * n + b0 + i, pv[r][c]);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const double2 w1 = u1[i + e], w3 = u3[i + e];
          const int nb = bf[i + e];
#pragma unroll
          for (int r = 0; r < RPW; ++r) {
            const bool i1 = in_bbox(mp + nk[r] + nb + 1, d.Nv), i2 = in_bbox(nb - nk[r], d.Nv);
            const bool i3 = in_bbox(mp - nk[r] - nb - 1, d.Nv), Yb = in_fbox(nk[r] + mp, d.Nv);
            const double c16 = 1.0 + ind(i1);
            const double c25 = Yb ? ind(i2) + ind(i1) : 0.0;
            const double c34 = 1.0 + ind(i3);
            const double2 t1 = csub(cscale(pv[r][0][e], c16), cscale(pv[r][1][e], c16 + 2.0 * c25));
            const double2 t3 = cscale(cadd(pv[r][2][e], pv[r][3][e]), c34);
            s1[r] = cadd(s1[r], cmul(w1, t1));
            s3[r] = cadd(s3[r], cmul(w3, t3));
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const double2 g_kp = a.g[(size_t)(nk[r] + mp + hG) * d.Nk + kadd(K[r], P, d.Lx, d.Ly)];
      const double2 g_pk = a.g[(size_t)(mp - nk[r] - 1 + hG) * d.Nk + ksub(P, K[r], d.Lx, d.Ly)];
      acc[r] = cadd(acc[r], cadd(cmul(g_kp, s1[r]), cmul(g_pk, s3[r])));
    }
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const double2 v = mk(wave_sum(acc[r].x), wave_sum(acc[r].y));
    const int k = (int)(blockIdx.y * 4 + wave) * RPW + r;
    if (lane == 0 && k < d.n) a.partial[(size_t)k * d.NW + jm] = v;
  }
}

// rows per wave: two where that still fills the chip (the LDS products are then
// shared by eight rows), one for smaller boxes
template <typename C>
void launch_sigmab(const SBArgs<C>& a, hipStream_t s) {
  const Dims& d = a.d;
  if ((long long)d.NW * d.n >= 8 * 1024)
    hipLaunchKernelGGL((sigmab_kernel<C, 2>), dim3(d.NW, (d.n + 7) / 8), dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((sigmab_kernel<C, 1>), dim3(d.NW, (d.n + 3) / 4), dim3(kThreads), 0, s, a);
}

// ------------------------------------------------- local Lambda in the box
// A box Lambda that differs from (U, -U, 2U, 0) adds to Sigma_box the
// Schwinger-Dyson sum of dLambda over the box, with dLambda_dm = Lambda_d -
// Lambda_m - 2U and dLambda_st = Lambda_s + Lambda_t - 2U at (m; n, n'). Since
// Lambda is local, the momentum sums factor through two bubble-like tables
//   B1(n', m; Q) = sum_K' G(n'+m, K'+Q) G(n', K'),
//   B2(n', m; Q) = sum_K' G(m-n'-1, Q-K') G(n', K'),
// and Sigma_box(n, K) gains
//   sum_{n', m} [dLambda_dm sum_Q G(n+m, K+Q) B1 + dLambda_st sum_Q G(m-n-1, Q-K) B2]
// (times the Schwinger-Dyson constant, applied in sigma2_kernel).
struct LamArgs {
  Dims d;
  double U;
  const double2* g;
  const double2* lam;     // [4][NW][Nv][Nv]
  double2* b1;            // [Nv][NW][Nk]
  double2* b2;
  double2* out;           // [n] (box k)
};

__device__ inline double2 g_at(const LamArgs& a, int nu, int K) {
  return a.g[(size_t)(nu + a.d.NG / 2) * a.d.Nk + K];
}

__global__ __launch_bounds__(kThreads) void lam_tables_kernel(LamArgs a) {
  const Dims& d = a.d;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= d.Nv * d.NW * d.Nk) return;
  const int Q = idx % d.Nk, jm = (idx / d.Nk) % d.NW, i2 = idx / (d.Nk * d.NW);
  const int n2 = i2 - d.Nv / 2, m = jm - (d.Nv / 2 - 1);
  double2 s1 = mk(0, 0), s2 = mk(0, 0);
  for (int Kp = 0; Kp < d.Nk; ++Kp) {
    const double2 gk = g_at(a, n2, Kp);
    s1 = cadd(s1, cmul(g_at(a, n2 + m, kadd(Kp, Q, d.Lx, d.Ly)), gk));
    s2 = cadd(s2, cmul(g_at(a, m - n2 - 1, ksub(Q, Kp, d.Lx, d.Ly)), gk));
  }
  a.b1[idx] = s1;
  a.b2[idx] = s2;
}

// one workgroup per box k = (n, K); threads over (n', m)
__global__ __launch_bounds__(kThreads) void lam_sigma_kernel(LamArgs a) {
  __shared__ double red[2][kThreads];
  const Dims& d = a.d;
  const int kbi = blockIdx.x, i1 = kbi / d.Nk, K = kbi - (kbi / d.Nk) * d.Nk;
  const int n = i1 - d.Nv / 2;
  const size_t cs = (size_t)d.NW * d.Nv * d.Nv;
  double sr = 0.0, si = 0.0;
  for (int pr = threadIdx.x; pr < d.Nv * d.NW; pr += blockDim.x) {
    const int i2 = pr / d.NW, jm = pr - (pr / d.NW) * d.NW;
    const int m = jm - (d.Nv / 2 - 1);
    const size_t li = ((size_t)jm * d.Nv + i1) * d.Nv + i2;
    const double2 ldm = csub(csub(a.lam[li], a.lam[cs + li]), mk(2.0 * a.U, 0.0));
    const double2 lst = csub(cadd(a.lam[2 * cs + li], a.lam[3 * cs + li]), mk(2.0 * a.U, 0.0));
    double2 t1 = mk(0, 0), t2 = mk(0, 0);
    const double2* b1 = a.b1 + ((size_t)i2 * d.NW + jm) * d.Nk;
    const double2* b2 = a.b2 + ((size_t)i2 * d.NW + jm) * d.Nk;
    for (int Q = 0; Q < d.Nk; ++Q) {
      t1 = cadd(t1, cmul(g_at(a, n + m, kadd(K, Q, d.Lx, d.Ly)), b1[Q]));
      t2 = cadd(t2, cmul(g_at(a, m - n - 1, ksub(Q, K, d.Lx, d.Ly)), b2[Q]));
    }
    const double2 v = cadd(cmul(ldm, t1), cmul(lst, t2));
    sr += v.x;
    si += v.y;
  }
  red[0][threadIdx.x] = sr;
  red[1][threadIdx.x] = si;
  __syncthreads();
  for (int st = kThreads / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      red[0][threadIdx.x] += red[0][threadIdx.x + st];
      red[1][threadIdx.x] += red[1][threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) a.out[kbi] = mk(red[0][0], red[1][0]);
}

// ------------------------------------ second order without the regulation
// Eq. PA_Sigma at F = Lambda with both sums truncated to the box (the Sigma~_1
// term of the plain, unregulated equation):
//   -(U^2 T^2 / 2N^2) sum_{q in box} [G(k+q) S_ph(q) + G(q-k) S_pp(q)],
//   S_ph(q) = sum_{k' in box} G(k'+q) G(k'),  S_pp(q) = sum_{k' in box} G(q-k') G(k').
struct S2BoxArgs {
  Dims d;
  double cfac;             // -U^2 T^2 / (2 N^2)
  const double2* g;
  double2* sq;             // [Nq][2]  S_ph, S_pp
  double2* out;            // [Nve][Nk]
};

// one wave per transfer q, lanes over k'
__global__ __launch_bounds__(kThreads) void s2box_tables_kernel(S2BoxArgs a) {
  const Dims& d = a.d;
  const int qi = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (qi >= d.Nq) return;
  const int jm = qi / d.Nk, Q = qi - jm * d.Nk, m = jm - (d.Nv / 2 - 1), hG = d.NG / 2;
  double v[4] = {0, 0, 0, 0};
  for (int kp = lane; kp < d.n; kp += 64) {
    const int n2 = kp / d.Nk - d.Nv / 2, K2 = kp - (kp / d.Nk) * d.Nk;
    const double2 gk = a.g[(size_t)(n2 + hG) * d.Nk + K2];
    const double2 ph = cmul(a.g[(size_t)(n2 + m + hG) * d.Nk + kadd(K2, Q, d.Lx, d.Ly)], gk);
    const double2 pp = cmul(a.g[(size_t)(m - n2 - 1 + hG) * d.Nk + ksub(Q, K2, d.Lx, d.Ly)], gk);
    v[0] += ph.x; v[1] += ph.y; v[2] += pp.x; v[3] += pp.y;
  }
  for (int i = 0; i < 4; ++i) v[i] = wave_sum(v[i]);
  if (lane == 0) {
    a.sq[(size_t)qi * 2] = mk(v[0], v[1]);
    a.sq[(size_t)qi * 2 + 1] = mk(v[2], v[3]);
  }
}

// one workgroup per k (f = 1: the extended box is the box), threads over q
__global__ __launch_bounds__(kThreads) void s2box_kernel(S2BoxArgs a) {
  __shared__ double red[kThreads];
  const Dims& d = a.d;
  const int kid = blockIdx.x, e = kid / d.Nk, K = kid - e * d.Nk;
  const int nk = e - d.Nve / 2, hG = d.NG / 2;
  double tr = 0.0, ti = 0.0;
  for (int qi = threadIdx.x; qi < d.Nq; qi += blockDim.x) {
    const int jm = qi / d.Nk, Q = qi - jm * d.Nk, m = jm - (d.Nv / 2 - 1);
    const double2 gkq = a.g[(size_t)(nk + m + hG) * d.Nk + kadd(K, Q, d.Lx, d.Ly)];
    const double2 gqk = a.g[(size_t)(m - nk - 1 + hG) * d.Nk + ksub(Q, K, d.Lx, d.Ly)];
    const double2 v = cadd(cmul(gkq, a.sq[(size_t)qi * 2]), cmul(gqk, a.sq[(size_t)qi * 2 + 1]));
    tr += v.x;
    ti += v.y;
  }
  tr = block_sum(tr, red);
  ti = block_sum(ti, red);
  if (threadIdx.x == 0) a.out[kid] = mk(a.cfac * tr, a.cfac * ti);
}

struct WsLayout {
  size_t srt, s1, tab, part, lb1, lb2, lpart, sq, total;
};

WsLayout ws_layout(const Dims& d) {
  WsLayout L{};
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
  L.srt = take(sizeof(double2) * (size_t)d.ntau * d.Nk);
  L.s1 = take(sizeof(double2) * d.Nve * d.Nk);
  L.tab = take(sizeof(double2) * 5 * (size_t)d.Nve * d.Nq);
  L.part = take(sizeof(double2) * (size_t)d.n * d.NW);
  L.lb1 = take(sizeof(double2) * (size_t)d.Nv * d.NW * d.Nk);
  L.lb2 = take(sizeof(double2) * (size_t)d.Nv * d.NW * d.Nk);
  L.lpart = take(sizeof(double2) * (size_t)d.n);
  L.sq = take(sizeof(double2) * 2 * (size_t)d.Nq);
  L.total = off;
  return L;
}

inline unsigned nblk(size_t total) { return (unsigned)((total + kThreads - 1) / kThreads); }

S1Args s1_args(const pq_params& p, const Dims& d, const double2* g, const double* mu, double2* out, char* ws) {
  return S1Args{d, p.beta, p.U, p.t, p.tp, p.D, d.Nk == 1 ? 1 : 0, g, mu, (double2*)(ws + ws_layout(d).srt), out};
}

template <typename G>
hipError_t run_sigma1(G&& args, int count, hipStream_t s) {
  launch_groups<S1Args>(count, args, [&](const auto& m, int, int n) {
    constexpr int N = sizeof(m.a) / sizeof(m.a[0]);
    int nt = 0;
    for (int i = 0; i < n; ++i) nt = std::max(nt, m.a[i].d.ntau);
    hipLaunchKernelGGL(s1_tau_kernel<N>, dim3(nt / 2, 1, n), dim3(kThreads), 0, s, m);
    hipLaunchKernelGGL(s1_row_kernel<N>, dim3(m.a[0].d.Nve, 1, n), dim3(kRowThreads), 0, s, m);
  });
  return hipGetLastError();
}

}  // namespace

size_t sigma_scratch_bytes(const Dims& d) { return ws_layout(d).total; }

// Above the scratch by what an earlier form of the stage kept beside it (two arrays
// of nodes, one of ntau Nk and three of Nve Nk values, a table over NG frequencies):
// callers see this size, and sigma_sde_no_alloc's limit is one on it.
size_t sigma_ws_bytes(const Dims& d) {
  const size_t row = sizeof(double2) * (size_t)d.Nk, tab = sizeof(double2) * 5 * (size_t)d.Nq;
  return ws_layout(d).total + 2 * align256(sizeof(double) * d.ntau) + align256(row * d.ntau) + 3 * align256(row * d.Nve) +
         align256(tab * d.NG) - align256(tab * d.Nve);
}

// ------------------------------------------------------ static scratch
// Workspace of sigma_sde_no_alloc: a file-scope device array, one copy per
// device that loads the library, held until the process ends. Host code never
// uses the array's name as an address (on the host it is a stand-in symbol):
// the device address is looked up once per device with hipGetSymbolAddress,
// with that device current, and kept.
namespace {
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// The second-order term: over all frequencies (Sigma~_1 of the regulation) or,
// without the regulation, truncated to the box.
static hipError_t run_second_order(const pq_params& p, const Dims& d, const double2* g, const double* mu,
                                   double2* out, char* ws, hipStream_t s) {
  if (p.regulation != 0) {
    return run_sigma1([&](int) { return s1_args(p, d, g, mu, out, ws); }, 1, s);
  }
  const WsLayout L = ws_layout(d);
  const double T = 1.0 / p.beta;
  S2BoxArgs a{d, -p.U * p.U * T * T / (2.0 * d.Nk * (double)d.Nk), g, (double2*)(ws + L.sq), out};
  const unsigned wpb = kThreads / 64;
  hipLaunchKernelGGL(s2box_tables_kernel, dim3((d.Nq + wpb - 1) / wpb), dim3(kThreads), 0, s, a);
  hipLaunchKernelGGL(s2box_kernel, dim3(d.Nve * d.Nk), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_sigma1(const pq_params& p, const Dims& d, const double2* g, const double* mu,
                         double2* sigma_out, void* ws, hipStream_t s) {
  return run_second_order(p, d, g, mu, sigma_out, (char*)ws, s);
}

namespace {

CombineArgs combine_args(const pq_params& p, const Dims& d, const double2* s1, const double2* part,
                         const double2* lpart, double2* sigma_out) {
  const double T = 1.0 / p.beta;
  return CombineArgs{d, -p.U * T * T / (4.0 * d.Nk * (double)d.Nk), p.kernel_level > 0 ? 1 : 0, s1, part, lpart,
                     sigma_out};
}

template <typename G>
void run_s2_sums(const Dims& d, G&& args, int count, hipStream_t s) {
  const int parts = std::max(1, std::min(1024 / (d.Nq * count), (d.Nve * kS2Sl + kThreads - 1) / kThreads));
  launch_groups<S2Args>(count, args, [&](const auto& m, int, int n) {
    hipLaunchKernelGGL((s2_sums_kernel<sizeof(m.a) / sizeof(m.a[0])>), dim3(d.Nq, parts, n), dim3(kThreads), 0, s, m,
                       pow2_ge(d.Nk));
  });
}

template <typename G2, typename GC>
void run_sigma2(const Dims& d, G2&& args, GC&& combine, int count, hipStream_t s) {
  launch_groups<S2Args>(count, args, [&](const auto& m, int first, int n) {
    constexpr int N = sizeof(m.a) / sizeof(m.a[0]);
    static_assert(sizeof(Many<S2Args, N>) + sizeof(Many<CombineArgs, N>) <= 4096, "arguments of a launch");
    Many<CombineArgs, N> mc;
    for (int i = 0; i < N; ++i) mc.a[i] = combine(first + (i < n ? i : 0));
    hipLaunchKernelGGL(sigma2_kernel<N>, dim3(d.Nve * d.Nk, 1, n), dim3(kThreads), 0, s, m, mc);
  });
}

}  // namespace

// The stage of several instances of a box: a launch of each kernel over them, but
// for the box part, whose one instance fills the chip. Without the regulation (the
// second-order term in the box) one after another.
hipError_t launch_sigma_many(const StageIn* x, int count, hipStream_t s) {
  bool each = count == 1;
  for (int i = 0; i < count; ++i) each = each || x[i].p->regulation == 0;
  if (each) {
    for (int i = 0; i < count; ++i) {
      const hipError_t e = launch_sigma(*x[i].p, *x[i].d, x[i].phi, x[i].k1, x[i].k2, nullptr, x[i].g, x[i].mu,
                                        x[i].sigma_new, x[i].sig_ws, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const Dims& d = *x[0].d;
  auto ws = [&](int i, size_t WsLayout::*part) {
    return (double2*)((char*)x[i].sig_ws + ws_layout(*x[i].d).*part);
  };
  auto a2 = [&](int i) {
    return S2Args{*x[i].d, x[i].p->kernel_level, x[i].g, x[i].k1, x[i].k2, ws(i, &WsLayout::tab)};
  };
  const hipError_t e = run_sigma1(
      [&](int i) { return s1_args(*x[i].p, *x[i].d, x[i].g, x[i].mu, ws(i, &WsLayout::s1), (char*)x[i].sig_ws); }, count,
      s);
  if (e != hipSuccess) return e;
  bool has_s2 = false;
  for (int i = 0; i < count; ++i) has_s2 = has_s2 || x[i].p->kernel_level > 0;
  if (has_s2) run_s2_sums(d, a2, count, s);          // an instance without kernels does not read its own
  for (int i = 0; i < count; ++i) {
    if (x[i].p->storage == PQ_STORE_C64)
      launch_sigmab(SBArgs<float2>{*x[i].d, (const float2*)x[i].phi, x[i].g, ws(i, &WsLayout::part)}, s);
    else
      launch_sigmab(SBArgs<double2>{*x[i].d, (const double2*)x[i].phi, x[i].g, ws(i, &WsLayout::part)}, s);
  }
  run_sigma2(
      d, a2,
      [&](int i) {
        return combine_args(*x[i].p, *x[i].d, ws(i, &WsLayout::s1), ws(i, &WsLayout::part), nullptr, x[i].sigma_new);
      },
      count, s);
  return hipGetLastError();
}

hipError_t launch_sigma(const pq_params& p, const Dims& d, const void* phi, const double2* k1,
                        const double2* k2, const double2* lam_box, const double2* g, const double* mu,
                        double2* sigma_out, void* wsv, hipStream_t s) {
  char* ws = (char*)wsv;
  WsLayout L = ws_layout(d);
  double2* s1 = (double2*)(ws + L.s1);
  double2* part = (double2*)(ws + L.part);
  hipError_t e = run_second_order(p, d, g, mu, s1, ws, s);
  if (e != hipSuccess) return e;
  auto a2 = [&](int) { return S2Args{d, p.kernel_level, g, k1, k2, (double2*)(ws + L.tab)}; };
  if (p.kernel_level > 0) run_s2_sums(d, a2, 1, s);
  if (p.storage == PQ_STORE_C64)
    launch_sigmab(SBArgs<float2>{d, (const float2*)phi, g, part}, s);
  else
    launch_sigmab(SBArgs<double2>{d, (const double2*)phi, g, part}, s);
  double2* lpart = nullptr;
  if (lam_box) {
    lpart = (double2*)(ws + L.lpart);
    LamArgs al{d, p.U, g, lam_box, (double2*)(ws + L.lb1), (double2*)(ws + L.lb2), lpart};
    hipLaunchKernelGGL(lam_tables_kernel, dim3(nblk((size_t)d.Nv * d.NW * d.Nk)), dim3(kThreads), 0, s, al);
    hipLaunchKernelGGL(lam_sigma_kernel, dim3(d.n), dim3(kThreads), 0, s, al);
  }
  run_sigma2(d, a2, [&](int) { return combine_args(p, d, s1, part, lpart, sigma_out); }, 1, s);
  return hipGetLastError();
}

}  // namespace pq
