// Single-particle kernels: Dyson equation with the filling condition, the
// bubbles X_ph / X_pp of the Bethe-Salpeter equations, and linear mixing of
// Sigma with its convergence norm. All FP64.
#include <math.h>

#include <algorithm>

#include "pq_internal.h"

namespace pq {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxNk = 64;          // momenta of the largest lattice (one wave)

struct DysonArgs {
  Dims d;
  double beta, t, tp, D, filling, mu_fixed, U;
  int mu_mode, local;
  const double2* sigma;
  double2* g;
  double* mu_out;
};

__device__ inline double eps_of(int K, const Dims& d, double t, double tp) {
  int kx = K / d.Ly, ky = K - (K / d.Ly) * d.Ly;
  double cx = cos(2.0 * M_PI * kx / d.Lx), cy = cos(2.0 * M_PI * ky / d.Ly);
  return -2.0 * t * (cx + cy) - 4.0 * tp * cx * cy;
}

__device__ inline double nu_of(int n, double beta) { return (2 * n + 1) * M_PI / beta; }

// Sigma on the G grid: stored on the extended box, zero beyond.
__device__ inline double2 sigma_at(const DysonArgs& a, int n, int K) {
  const int h = a.d.Nve / 2;
  if (n < -h || n > h - 1) return mk(0.0, 0.0);
  return a.sigma[(size_t)(n + h) * a.d.Nk + K];
}

// Lattice G at mu for G-grid row g and momentum K.
__device__ inline double2 g_lattice(const DysonArgs& a, const double* eps, double mu, int gi, int K) {
  int n = gi - a.d.NG / 2;
  double nu = nu_of(n, a.beta);
  double2 s = sigma_at(a, n, K);
  double2 z = mk(mu - eps[K] - s.x, nu - s.y);
  return crecip(z);
}

// 1 / v of a normal v: the hardware estimate and two Newton steps (about 1 ulp)
__device__ inline double rcp_nr(double v) {
  double r = __builtin_amdgcn_rcp(v);
  r = fma(r, fma(-v, r, 1.0), r);
  return fma(r, fma(-v, r, 1.0), r);
}

// One value of the self-energy as the density needs it: a = eps + Re Sigma and
// y^2 = (nu - Im Sigma)^2, with eps and nu^2 of the same G without Sigma. Beyond
// 1e75 the value is held at 1e75 (its part of the density is zero there in any
// case, and the products of density_term stay finite); NaN stays NaN.
struct DElem {
  double a, y2, e, nu2;
};
__device__ inline DElem d_elem(const DysonArgs& p, const double* eps, int idx) {
  const int row = idx / p.d.Nk, K = idx - row * p.d.Nk;
  const double nu = nu_of(row - p.d.Nve / 2, p.beta);
  const double2 s = p.sigma[idx];
  DElem v;
  v.e = eps[K];
  v.nu2 = nu * nu;
  v.a = v.e + s.x;
  v.a = v.a > 1e75 ? 1e75 : (v.a < -1e75 ? -1e75 : v.a);
  const double y = nu - s.y, y2 = y * y;
  v.y2 = y2 > 1e150 ? 1e150 : y2;
  return v;
}

// Re [G - G(Sigma = 0)] at mu, with x = mu - a and z = mu - eps:
// x / (x^2 + y^2) - z / (z^2 + nu^2) over one common denominator
__device__ inline double density_term(const DElem& v, double mu) {
  const double x = mu - v.a, z = mu - v.e;
  const double d1 = fma(x, x, v.y2), d2 = fma(z, z, v.nu2);
  return fma(x, d2, -z * d1) * rcp_nr(d1 * d2);
}

// Dyson equation in one workgroup. The filling is a chain of about 52 bisection
// steps, so the kernel is bound by the latency of one density, not by its work.
// The density per spin is that of Sigma = 0, (1/N) sum_K f(xi_K) in closed form,
// plus T/N sum Re (G - G_0) over the extended box (Sigma is zero beyond it), one
// reciprocal per value; the values stay in registers. 2^LV - 1 points of the
// bisection tree below the present bracket are evaluated at once, each by LP
// lanes, and the path through them is the one bisection takes: LV steps per
// pass. A pass costs the values of every point plus a fixed part per wave (the
// Fermi function, the sum, the barrier), so few values take many points on few
// lanes, many values one point on every lane. Measured before (256 threads, one
// point at a time, three divisions per value of the whole grid, tail sums per
// step): 213 us at 4x4, Nv = 8, 490 us at 8x8, Nv = 16; now 26 and 45 us.
constexpr int dyson_threads(int lv, int lp) { return (((1 << lv) - 1) * lp + 63) / 64 * 64; }

template <int LV, int LP, int RE, int N>
__global__ __launch_bounds__(dyson_threads(LV, LP)) void dyson_kernel(Many<DysonArgs, N> m) {
  const DysonArgs& a = m.a[N == 1 ? 0 : blockIdx.z];
  constexpr int NC = (1 << LV) - 1;                  // points per pass
  constexpr int LG = LP < 64 ? LP : 64;              // lanes of one partial sum
  constexpr int W = LP / LG;                         // partial sums per point
  __shared__ double eps[kMaxNk];
  __shared__ double part[2][NC * W];
  const Dims& d = a.d;
  const int t = threadIdx.x, lane = t & 63;
  if (t < d.Nk) eps[t] = a.local ? 0.0 : eps_of(t, d, a.t, a.tp);
  __syncthreads();
  double mu = a.mu_fixed;
  if (!a.local && a.mu_mode == 1) {
    double emin = eps[min(lane, d.Nk - 1)], emax = emin;
    for (int o = 32; o > 0; o >>= 1) {
      emin = fmin(emin, __shfl_xor(emin, o, 64));
      emax = fmax(emax, __shfl_xor(emax, o, 64));
    }
    const int c = t / LP + 1, pl = t % LP;           // this lane's point (heap index) and place in it
    const int total = d.Nve * d.Nk, cnt = (total + LP - 1) / LP;
    DElem v[RE];
#pragma unroll
    for (int q = 0; q < RE; ++q) {
      const int idx = q * LP + pl;
      if (q < cnt && idx < total) v[q] = d_elem(a, eps, idx);
      else v[q] = DElem{0.0, 1.0, 0.0, 1.0};        // contributes zero
    }
    const double tn = 1.0 / (a.beta * d.Nk);
    double lo = emin - 10.0 - fabs(a.U), hi = emax + 10.0 + fabs(a.U);
    bool done = false;
    for (int it = 0, pass = 0; it < 200 && !done; ++pass) {
      double l = lo, h = hi, m = 0.5 * (l + h);     // the point of heap index c below the bracket
      for (int b = 30 - __clz(c); b >= 0; --b) {
        if ((c >> b) & 1) l = m; else h = m;
        m = 0.5 * (l + h);
      }
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < RE; ++q) s += density_term(v[q], m);
      for (int idx = RE * LP + pl; idx < total; idx += LP) s += density_term(d_elem(a, eps, idx), m);
      s *= tn;
      for (int K = pl; K < d.Nk; K += LP) s += 1.0 / (d.Nk * (exp(a.beta * (eps[K] - m)) + 1.0));
      s = group_total<LG>(s);
      if (c <= NC && lane % LG == LG - 1) part[pass & 1][t / LG] = s;
      __syncthreads();
      // bit i: the density at point i + 1 is above the filling
      double nn = 0.0;
      for (int w = 0; w < W; ++w) nn += part[pass & 1][(lane % NC) * W + w];
      const unsigned long long above = __ballot(2.0 * nn > a.filling);
      int node = 1;
      for (int k = 0; k < LV && it < 200 && !done; ++k, ++it) {
        const double mid = 0.5 * (lo + hi);
        const bool ab = (above >> (node - 1)) & 1;
        if (ab) hi = mid; else lo = mid;
        node = 2 * node + (ab ? 0 : 1);
        done = hi - lo < 1e-14;
      }
    }
    mu = 0.5 * (lo + hi);
  }
  for (int idx = t; idx < d.NG * d.Nk; idx += blockDim.x) {
    int gi = idx / d.Nk, K = idx - gi * d.Nk;
    double2 gv;
    if (a.local) {
      int n = gi - d.NG / 2;
      double nu = nu_of(n, a.beta);
      double sg = nu > 0 ? 1.0 : (nu < 0 ? -1.0 : 0.0);
      double c = 2.0 / (a.D * a.D);
      double2 g0 = mk(0.0, c * (nu - sg * sqrt(nu * nu + a.D * a.D)));
      double2 s = sigma_at(a, n, K);
      gv = crecip(csub(crecip(g0), s));
    } else {
      gv = g_lattice(a, eps, mu, gi, K);
    }
    a.g[idx] = gv;
  }
  if (t == 0) *a.mu_out = a.local ? 0.0 : mu;
}

struct BubbleArgs {
  Dims d;
  double T;
  const double2* g;
  double2* xph;
  double2* xpp;
};

template <int N>
__global__ __launch_bounds__(kThreads) void bubble_kernel(Many<BubbleArgs, N> ms) {
  const BubbleArgs& a = ms.a[N == 1 ? 0 : blockIdx.z];
  const Dims& d = a.d;
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)d.Nq * d.n) return;
  int qi = (int)(idx / d.n), ki = (int)(idx - (size_t)qi * d.n);
  int jm = qi / d.Nk, Q = qi - jm * d.Nk;
  int m = jm - (d.Nv / 2 - 1);
  int in = ki / d.Nk, K = ki - in * d.Nk;
  int n = in - d.Nv / 2;
  const int h = d.NG / 2;
  double2 gk = a.g[(size_t)(n + h) * d.Nk + K];
  double2 gkq = a.g[(size_t)(n + m + h) * d.Nk + kadd(K, Q, d.Lx, d.Ly)];
  double2 gqk = a.g[(size_t)(m - n - 1 + h) * d.Nk + ksub(Q, K, d.Lx, d.Ly)];
  a.xph[idx] = cscale(cmul(gk, gkq), a.T / d.Nk);
  a.xpp[idx] = cscale(cmul(gk, gqk), a.T / (2.0 * d.Nk));
}

template <int N>
__global__ __launch_bounds__(kThreads) void mix_kernel(int count, Many<MixIn, N> m, double alpha) {
  const MixIn& x = m.a[N == 1 ? 0 : blockIdx.z];
  const double2* snew = x.snew;
  double2* sio = x.sio;
  double *dnorm = x.dnorm, *smax = x.smax, *host = x.host;
  __shared__ double red[kThreads];
  double mx = 0.0, bad = 0.0, sm = 0.0;
  for (int i = threadIdx.x; i < count; i += blockDim.x) {
    double2 a = snew[i], b = sio[i];
    double dr = a.x - b.x, di = a.y - b.y;
    double dd = hypot(dr, di);
    if (!isfinite(a.x) || !isfinite(a.y)) bad = 1.0;
    mx = fmax(mx, dd);
    const double2 c = mk(alpha * a.x + (1.0 - alpha) * b.x, alpha * a.y + (1.0 - alpha) * b.y);
    sio[i] = c;
    sm = fmax(sm, hypot(c.x, c.y));
  }
  mx = block_max(mx, red);
  bad = block_max(bad, red);
  sm = block_max(sm, red);
  if (threadIdx.x == 0) {
    *dnorm = bad > 0.0 ? __builtin_nan("") : mx;
    if (smax) *smax = sm;
    if (host) {                       // dnorm[1 .. 4]: the BSE summary, dnorm[6]: mu~
      host[0] = *dnorm;
      for (int i = 1; i < 5; ++i) host[i] = dnorm[i];
      host[5] = sm;
      host[6] = dnorm[6];
    }
  }
}

// storage conversion of a vertex array (complex64 <-> complex128, or a copy)
template <typename S, typename D>
__global__ __launch_bounds__(kThreads) void convert_kernel(const S* src, D* dst, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x) {
    const S v = src[i];
    D w;
    w.x = v.x;
    w.y = v.y;
    dst[i] = w;
  }
}

// F = Gamma + Phi over a vertex array (Eq. PA_F_G)
template <typename C>
__global__ __launch_bounds__(kThreads) void vertex_sum_kernel(const C* a, const C* b, C* f, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x) {
    const C x = a[i], y = b[i];
    C z;
    z.x = x.x + y.x;
    z.y = x.y + y.y;
    f[i] = z;
  }
}

}  // namespace

hipError_t launch_vertex_sum(const void* a, const void* b, void* f, int storage, size_t count, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<size_t>(16384, (count + kThreads - 1) / kThreads);
  if (storage == PQ_STORE_C64)
    hipLaunchKernelGGL((vertex_sum_kernel<float2>), dim3(blocks), dim3(kThreads), 0, s, (const float2*)a,
                       (const float2*)b, (float2*)f, count);
  else
    hipLaunchKernelGGL((vertex_sum_kernel<double2>), dim3(blocks), dim3(kThreads), 0, s, (const double2*)a,
                       (const double2*)b, (double2*)f, count);
  return hipGetLastError();
}

hipError_t launch_convert(const void* src, int src_storage, void* dst, int dst_storage, size_t count,
                          hipStream_t s) {
  const unsigned blocks = (unsigned)std::min<size_t>(8192, (count + kThreads - 1) / kThreads);
  if (count == 0) return hipSuccess;
  if (src_storage == PQ_STORE_C64 && dst_storage == PQ_STORE_C128)
    hipLaunchKernelGGL((convert_kernel<float2, double2>), dim3(blocks), dim3(kThreads), 0, s,
                       (const float2*)src, (double2*)dst, count);
  else if (src_storage == PQ_STORE_C128 && dst_storage == PQ_STORE_C64)
    hipLaunchKernelGGL((convert_kernel<double2, float2>), dim3(blocks), dim3(kThreads), 0, s,
                       (const double2*)src, (float2*)dst, count);
  else if (src_storage == PQ_STORE_C64)
    hipLaunchKernelGGL((convert_kernel<float2, float2>), dim3(blocks), dim3(kThreads), 0, s,
                       (const float2*)src, (float2*)dst, count);
  else
    hipLaunchKernelGGL((convert_kernel<double2, double2>), dim3(blocks), dim3(kThreads), 0, s,
                       (const double2*)src, (double2*)dst, count);
  return hipGetLastError();
}

static_assert(sizeof(Many<DysonArgs, kMany>) <= 4096, "arguments of a launch");

hipError_t launch_dyson_many(const StageIn* x, int count, hipStream_t s) {
  const Dims& d = *x[0].d;
  if (d.Nk > kMaxNk) return hipErrorInvalidValue;
  auto args = [&](int i) {
    const pq_params& p = *x[i].p;
    return DysonArgs{*x[i].d, p.beta, p.t, p.tp, p.D, p.filling, p.mu_fixed, p.U, p.mu_mode, d.Nk == 1 ? 1 : 0,
                     x[i].sigma, x[i].g, x[i].mu};
  };
  // points per pass and lanes per point by the number of self-energy values, the
  // shape whose pass costs least per bisection step (256 values: 16 lanes
  // per point 26 us, a wave per point 33; 1024: 3 steps on 128 lanes per point 48,
  // 2 on 256 lanes 35; 2048: 2 on 256 lanes 58, 1 on 1024 lanes 50, on 512 45)
  const int values = d.Nve * d.Nk;
#define PQ_DYSON(LV, LP, RE)                                                                                      \
  launch_groups<DysonArgs>(count, args, [&](const auto& m, int, int n) {                                          \
    hipLaunchKernelGGL((dyson_kernel<LV, LP, RE, sizeof(m.a) / sizeof(m.a[0])>), dim3(1, 1, n),                   \
                       dim3(dyson_threads(LV, LP)), 0, s, m);                                                     \
  })
  if (values <= 16 * 8) PQ_DYSON(4, 16, 8);
  else if (values <= 16 * 16) PQ_DYSON(4, 16, 16);
  else if (values <= 128 * 4) PQ_DYSON(2, 128, 4);
  else if (values <= 256 * 4) PQ_DYSON(2, 256, 4);
  else if (values <= 512 * 4) PQ_DYSON(1, 512, 4);
  else if (values <= 1024 * 4) PQ_DYSON(1, 1024, 4);
  else PQ_DYSON(1, 1024, 8);
#undef PQ_DYSON
  return hipGetLastError();
}

hipError_t launch_dyson(const pq_params& p, const Dims& d, const double2* sigma, double2* g,
                        double* mu_out, hipStream_t s) {
  StageIn x{};
  x.p = &p;
  x.d = &d;
  x.sigma = sigma;
  x.g = g;
  x.mu = mu_out;
  return launch_dyson_many(&x, 1, s);
}

hipError_t launch_bubbles_many(const StageIn* x, int count, hipStream_t s) {
  auto args = [&](int i) { return BubbleArgs{*x[i].d, 1.0 / x[i].p->beta, x[i].g, x[i].xph, x[i].xpp}; };
  const size_t total = (size_t)x[0].d->Nq * x[0].d->n;
  const unsigned blocks = (unsigned)((total + kThreads - 1) / kThreads);
  launch_groups<BubbleArgs>(count, args, [&](const auto& m, int, int n) {
    hipLaunchKernelGGL((bubble_kernel<sizeof(m.a) / sizeof(m.a[0])>), dim3(blocks, 1, n), dim3(kThreads), 0, s, m);
  });
  return hipGetLastError();
}

hipError_t launch_bubbles(const pq_params& p, const Dims& d, const double2* g, double2* xph,
                          double2* xpp, hipStream_t s) {
  StageIn x{};
  x.p = &p;
  x.d = &d;
  x.g = const_cast<double2*>(g);
  x.xph = xph;
  x.xpp = xpp;
  return launch_bubbles_many(&x, 1, s);
}

hipError_t launch_mix_many(const Dims& d, const MixIn* x, int count, double alpha, hipStream_t s) {
  launch_groups<MixIn>(count, [&](int i) { return x[i]; }, [&](const auto& m, int, int n) {
    hipLaunchKernelGGL((mix_kernel<sizeof(m.a) / sizeof(m.a[0])>), dim3(1, 1, n), dim3(kThreads), 0, s, d.Nve * d.Nk, m,
                       alpha);
  });
  return hipGetLastError();
}

hipError_t launch_mix(const Dims& d, const double2* snew, double2* sio, double alpha,
                      double* dnorm, hipStream_t s, double* smax, double* host) {
  const MixIn x{snew, sio, dnorm, smax, host};
  return launch_mix_many(d, &x, 1, alpha, s);
}

}  // namespace pq

// ------------------------------------------------------ HBM streaming probes
// Reference rates for the memory-bound stages: float4 grid-stride streams,
// eight 16-byte accesses in flight per thread and iteration, non-temporal
// loads (and stores for the copy), up to 16384 workgroups: the fastest of the
// shapes tried on this device (unroll 4, 8, 16; 1024 to 16384 workgroups;
// with and without the non-temporal hint).
namespace pq {
namespace {

constexpr int kHbmUnroll = 8;
typedef float hf4 __attribute__((ext_vector_type(4)));

__device__ inline hf4 nt_ld(const hf4* p) { return __builtin_nontemporal_load(p); }

__global__ __launch_bounds__(256) void hbm_copy_kernel(const hf4* __restrict__ src, hf4* __restrict__ dst,
                                                       size_t count) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + (kHbmUnroll - 1) * stride < count; i += kHbmUnroll * stride) {
    hf4 v[kHbmUnroll];
#pragma unroll
    for (int u = 0; u < kHbmUnroll; ++u) v[u] = nt_ld(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < kHbmUnroll; ++u) __builtin_nontemporal_store(v[u], dst + i + u * stride);
  }
  for (; i < count; i += stride) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void hbm_read_kernel(const hf4* __restrict__ src, size_t count,
                                                       float* __restrict__ out) {
  __shared__ float red[256];
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  float acc = 0.f;
  for (; i + (kHbmUnroll - 1) * stride < count; i += kHbmUnroll * stride) {
    hf4 v[kHbmUnroll];
#pragma unroll
    for (int u = 0; u < kHbmUnroll; ++u) v[u] = nt_ld(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < kHbmUnroll; ++u) acc += (v[u].x + v[u].y) + (v[u].z + v[u].w);
  }
  for (; i < count; i += stride) acc += (src[i].x + src[i].y) + (src[i].z + src[i].w);
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void hbm_write_kernel(hf4* __restrict__ dst, size_t count, float value) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const hf4 v = {value, value, value, value};
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) dst[i] = v;
}

}  // namespace

hipError_t launch_hbm_stream(int mode, const void* src, void* dst, size_t bytes, hipStream_t s) {
  const size_t count = bytes / 16;
  const unsigned blocks = (unsigned)std::max<size_t>(1, std::min<size_t>(kHbmStreamBlocks, (count + 255) / 256));
  if (mode == 0)
    hipLaunchKernelGGL(hbm_copy_kernel, dim3(blocks), dim3(256), 0, s, (const hf4*)src, (hf4*)dst, count);
  else if (mode == 1)
    hipLaunchKernelGGL(hbm_read_kernel, dim3(blocks), dim3(256), 0, s, (const hf4*)src, count, (float*)dst);
  else
    hipLaunchKernelGGL(hbm_write_kernel, dim3(blocks), dim3(256), 0, s, (hf4*)dst, count, 1.0f);
  return hipGetLastError();
}

}  // namespace pq
