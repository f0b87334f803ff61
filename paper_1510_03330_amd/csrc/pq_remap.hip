// Kernel functions (two-level kernel approximation) and the channel remap of
// the parquet equations (Eqs. PA_Gamma_dm, PA_Gamma_st).
//
// Remap data flow. Every term of Gamma_r at (q, k, k') reads a reducible
// vertex whose first fermionic argument is the output's k. For fixed k and a
// fixed pair of output frequencies (m, n') the Nk x Nk momentum tile (Q, K')
// of a term is a permutation of one Nk x Nk source tile (Q_p, K_b) of
// Phi_r[p][k][b] at one frequency pair (m_p, n_b):
//   ph-bar  (d,m):  m_p = n'-n,       n_b = n+m      Q_p = K'-K,    K_b = K+Q
//   pp      (s,t):  m_p = n+n'+m+1,   n_b = n'       Q_p = K+K'+Q,  K_b = K'
//   st-1    (d,m):  m_p = n'-n,       n_b = m-n'-1   Q_p = K'-K,    K_b = Q-K'
//   st-2    (d,m):  m_p = m-n-n'-1,   n_b = n'       Q_p = Q-K-K',  K_b = K'
// (frequency shifts of ferm+bos, ferm-ferm, ferm+ferm+bos, bos-ferm, bos-ferm-ferm
// sums). A workgroup owns one (k, m) output plane, loads each source tile once
// through LDS with coalesced row reads, and applies the permutation from LDS.
// Source tiles outside the fermionic box are kernel-filled
// (K1(p) + K2(k;p), constant along K_b); transfers outside the bosonic box
// contribute nothing.
#include "pq_internal.h"

namespace pq {

namespace {

constexpr int kThreads = 256;
constexpr int kDirectNk = 12;

// ------------------------------------------------------- kernel functions
template <typename C>
struct KxArgs {
  Dims d;
  int level, edge_rule;
  const C* phi;
  double2* k1;
  double2* k2;
};

// Row means over the momenta of the edge columns: LPR lanes (a power of two, at
// most 16) read a row's strip of Nk values, 64 / LPR rows per wave at a time and
// kXU of those in flight, so that the strips stream at memory rate whatever the
// lattice; the lanes' sums meet on the vector unit. (One wave per row, one row in
// flight and shuffles through the LDS crossbar: 1.3 ms on the 8x8, Nv = 16
// complex64 box, 216 us at 5x7, Nv = 10 complex128; now 0.45 ms and 106 us.)
constexpr int kXU = 4;

template <int LPR>
__device__ inline double row_total(double v) {       // in the last lane of each group of LPR
  if (LPR >= 2) v = dpp_add<0x111, 0xf>(v);
  if (LPR >= 4) v = dpp_add<0x112, 0xf>(v);
  if (LPR >= 8) v = dpp_add<0x114, 0xf>(v);
  if (LPR >= 16) v = dpp_add<0x118, 0xf>(v);
  return v;
}

template <typename C, int LPR>
__global__ __launch_bounds__(kThreads) void kernel_extract_kernel(KxArgs<C> a) {
  extern __shared__ double2 srow[];   // [2][n]
  const Dims& d = a.d;
  const int r = blockIdx.x / d.Nq, qi = blockIdx.x - (blockIdx.x / d.Nq) * d.Nq;
  const int m = qi / d.Nk - (d.Nv / 2 - 1);
  const size_t n = d.n;
  const size_t ko = (size_t)r * d.Nq + qi;
  if (a.level == 0) {
    for (int k = threadIdx.x; k < d.n; k += blockDim.x) a.k2[ko * n + k] = mk(0, 0);
    if (threadIdx.x == 0) a.k1[ko] = mk(0, 0);
    return;
  }
  const int top = d.Nv / 2 - 1, bot = -d.Nv / 2;
  int e0, e1 = 0, ne = 1;
  if (a.edge_rule == 1) {
    e0 = bot;
  } else if (m == 0) {
    e0 = top; e1 = bot; ne = 2;
  } else if (r < 2) {
    e0 = m > 0 ? top : bot;
  } else {
    e0 = m > 0 ? bot : top;
  }
  const C* blk = a.phi + (size_t)r * d.cs + (size_t)qi * n * n;
  constexpr int RPB = kThreads / LPR;                 // rows the workgroup reads at a time
  const int row = threadIdx.x / LPR, l = threadIdx.x % LPR;
  for (int ei = 0; ei < ne; ++ei) {
    const int e = ei == 0 ? e0 : e1;
    const C* col = blk + (size_t)(e + d.Nv / 2) * d.Nk;
    for (int k0 = 0; k0 < d.n; k0 += RPB * kXU) {
      double2 sum[kXU];
#pragma unroll
      for (int u = 0; u < kXU; ++u) sum[u] = mk(0, 0);
      for (int K = l; K < d.Nk; K += LPR)
#pragma unroll
        for (int u = 0; u < kXU; ++u)
          sum[u] = cadd(sum[u], to_d(col[(size_t)min(k0 + u * RPB + row, d.n - 1) * n + K]));
#pragma unroll
      for (int u = 0; u < kXU; ++u) {
        const double2 v = mk(row_total<LPR>(sum[u].x), row_total<LPR>(sum[u].y));
        const int k = k0 + u * RPB + row;
        if (l == LPR - 1 && k < d.n) srow[ei * n + k] = mk(v.x / d.Nk, v.y / d.Nk);
      }
    }
  }
  __syncthreads();
  __shared__ double2 k1s;
  if (threadIdx.x < 64) {                             // Nk <= 64: a lane per momentum of the edge rows
    double2 s = mk(0, 0);
    if (threadIdx.x < d.Nk)
      for (int ei = 0; ei < ne; ++ei)
        s = cadd(s, srow[ei * n + (size_t)((ei == 0 ? e0 : e1) + d.Nv / 2) * d.Nk + threadIdx.x]);
    const double2 v = mk(group_total<64>(s.x), group_total<64>(s.y));
    if (threadIdx.x == 63) {
      k1s = mk(v.x / d.Nk / ne, v.y / d.Nk / ne);
      a.k1[ko] = k1s;
    }
  }
  __syncthreads();
  const double2 K1v = k1s;
  for (int k = threadIdx.x; k < d.n; k += blockDim.x) {
    double2 v = mk(0, 0);
    if (a.level >= 2) {
      double2 s = srow[k];
      if (ne == 2) s = cadd(s, srow[n + k]);
      v = csub(cscale(s, 1.0 / ne), K1v);
    }
    a.k2[ko * n + k] = v;
  }
}

// ------------------------------------------------------------------ remap
template <typename C>
struct RemapArgs {
  Dims d;
  double lam[4];
  const double2* lam_box;   // nullable: local Lambda_r(m; n, n') on the box, [4][NW][Nv][Nv]
  const C* phi;
  const double2* k1;
  const double2* k2;
  C* gamma;
};

template <typename C> __device__ inline C czero();
template <> __device__ inline float2 czero<float2>() { return make_float2(0.f, 0.f); }
template <> __device__ inline double2 czero<double2>() { return make_double2(0.0, 0.0); }

// non-temporal store of one complex value (Gamma is not read again here)
__device__ inline void st_stream(float2* p, float2 v) {
  typedef float v2 __attribute__((ext_vector_type(2)));
  const v2 w = {v.x, v.y};
  __builtin_nontemporal_store(w, (v2*)p);
}
__device__ inline void st_stream(double2* p, double2 v) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 w = {v.x, v.y};
  __builtin_nontemporal_store(w, (v2*)p);
}

// Whether Gamma goes out with streaming stores: not for complex64 rows that
// start inside a 64-byte sector whose parts the caches
// must join first (5x7, Nv = 10: 0.98 ms streaming, 0.78 not; complex128 the
// other way round, 1.41 and 1.44)
template <typename C> __device__ inline bool stream_rows(int Nk) {
  return sizeof(C) > sizeof(float2) || Nk * sizeof(C) % 64 == 0;
}

template <typename C, typename R>
__device__ inline C axpy(C acc, R c, C v) {
  acc.x += c * v.x;
  acc.y += c * v.y;
  return acc;
}

// Coefficients of the eight terms into the two output channels of a pass
// (pass 0 -> d, m; pass 1 -> s, t), Eqs. PA_Gamma_dm and PA_Gamma_st. Term
// order within a pass: pass 0: d ph-bar, m ph-bar, s pp, t pp; pass 1:
// d st-1, m st-1, d st-2, m st-2.
__constant__ float kCoef[2][4][2] = {
    {{-0.5f, -0.5f}, {-1.5f, 0.5f}, {0.5f, -0.5f}, {1.5f, 0.5f}},
    {{0.5f, -0.5f}, {-1.5f, -0.5f}, {0.5f, 0.5f}, {-1.5f, 0.5f}}};

// One workgroup of NT threads per (k, m) output plane walks the Nv x 2 x 4 (n',
// pass, term) source tiles in a fixed order, TPS of them (1, the two channels of
// a geometry, or the four terms of a pass) per step. The permutation of each
// geometry depends only on (K, Q, K'), so its LDS offsets are tabulated once per
// workgroup; a kernel-filled tile is written into LDS across all its columns so
// that the same offsets apply. The next step's global loads are issued before
// the current tiles are consumed from LDS, so TPS tiles per workgroup are always
// in flight; small tiles need several per step to cover the two barriers and the
// memory latency (5x7, Nv = 10: 1.57 -> 1.30 ms complex128, complex64 with the
// kernel functions 1.22 -> 0.81 ms; 8x8, Nv = 16, complex64 stays at one tile per
// step, 13 to 14 ms).
template <typename C, int EPT, int NT, int TPS>
__global__ __launch_bounds__(NT) void remap_kernel(RemapArgs<C> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  using R = decltype(C().x);
  const Dims& d = a.d;
  const int Nk = d.Nk, Nk2 = Nk * Nk, ld = Nk + 1;
  C* tile = (C*)smem;                                              // TPS x Nk rows, padded stride ld
  unsigned short* offs = (unsigned short*)(smem + sizeof(C) * TPS * Nk * ld);   // [4][Nk2]

  // block -> (k, m); consecutive logical blocks (same k) stay on one XCD
  const int lin = xcd_linear();
  const int kbi = lin / d.NW, jm = lin - (lin / d.NW) * d.NW;
  const int nk = kbi / Nk - d.Nv / 2, K = kbi - (kbi / Nk) * Nk;
  const int m = jm - (d.Nv / 2 - 1);
  const size_t n = d.n, nn = (size_t)d.n * d.n, chan = (size_t)d.cs;
  const int t = threadIdx.x;

  // output element e = Q Nk + K' reads source (Qp, Kb):
  //   g0 ph-bar: (K'-K, K+Q)  g1 pp: (K+K'+Q, K')  g2 st-1: (K'-K, Q-K')  g3 st-2: (Q-K-K', K')
  for (int e = t; e < Nk2; e += NT) {
    const int Q = e / Nk, Kp = e - (e / Nk) * Nk;
    const int Lx = d.Lx, Ly = d.Ly;
    const int kpk = ksub(Kp, K, Lx, Ly);
    offs[0 * Nk2 + e] = (unsigned short)(kpk * ld + kadd(K, Q, Lx, Ly));
    offs[1 * Nk2 + e] = (unsigned short)(kadd(kadd(K, Kp, Lx, Ly), Q, Lx, Ly) * ld + Kp);
    offs[2 * Nk2 + e] = (unsigned short)(kpk * ld + ksub(Q, Kp, Lx, Ly));
    offs[3 * Nk2 + e] = (unsigned short)(ksub(ksub(Q, K, Lx, Ly), Kp, Lx, Ly) * ld + Kp);
  }

  // tile index s = (n' index, pass, term) -> source tile
  auto info = [&](int s, int& geo, int& src, int& jmp, int& nb, bool& valid) {
    const int in2 = s >> 3, pass = (s >> 2) & 1, term = s & 3;
    const int n2 = in2 - d.Nv / 2;
    geo = pass * 2 + (term >> 1);                    // 0 ph-bar, 1 pp, 2 st-1, 3 st-2
    src = pass == 0 ? term : (term & 1);
    int mp;
    if (geo == 0) { mp = n2 - nk; nb = nk + m; }
    else if (geo == 1) { mp = nk + n2 + m + 1; nb = n2; }
    else if (geo == 2) { mp = n2 - nk; nb = m - n2 - 1; }
    else { mp = m - nk - n2 - 1; nb = n2; }
    valid = in_bbox(mp, d.Nv);
    jmp = mp + d.Nv / 2 - 1;
  };
  const bool lines = stream_rows<C>(Nk);
  C buf[TPS][EPT];
  auto fetch = [&](int s) {
#pragma unroll
    for (int j = 0; j < TPS; ++j) {
      int geo, src, jmp, nb;
      bool valid;
      info(s * TPS + j, geo, src, jmp, nb, valid);
      if (!valid) continue;
      if (in_fbox(nb, d.Nv)) {
        const C* base = a.phi + src * chan + (size_t)kbi * n + (size_t)(nb + d.Nv / 2) * Nk;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          const int idx = min(t + i * NT, Nk2 - 1);
          const int Qp = idx / Nk, Kb = idx - (idx / Nk) * Nk;
          buf[j][i] = base[(size_t)(jmp * Nk + Qp) * nn + Kb];
        }
      } else {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          const int idx = min(t + i * NT, Nk2 - 1);
          const size_t qo = (size_t)src * d.Nq + jmp * Nk + idx / Nk;
          buf[j][i] = from_d<C>(cadd(a.k1[qo], a.k2[qo * n + kbi]));
        }
      }
    }
  };
  const int nsteps = d.Nv * 8 / TPS;
  fetch(0);
  C acc0[EPT], acc1[EPT];
  for (int s = 0; s < nsteps; ++s) {
    bool valid[TPS], any = false;
#pragma unroll
    for (int j = 0; j < TPS; ++j) {
      int geo, src, jmp, nb;
      info(s * TPS + j, geo, src, jmp, nb, valid[j]);
      any = any || valid[j];
    }
    const int in2 = s * TPS >> 3, pass = (s * TPS >> 2) & 1, term0 = s * TPS & 3;
    if (term0 == 0) {
      // Lambda of the two output channels at (m; n, n'): constant over the
      // momentum plane, since the fully irreducible vertex is local
      C l0 = czero<C>(), l1 = czero<C>();
      if (a.lam_box) {
        const size_t cs = (size_t)d.NW * d.Nv * d.Nv;
        const size_t li = ((size_t)jm * d.Nv + kbi / Nk) * d.Nv + in2;
        const double2 v0 = a.lam_box[(size_t)(2 * pass) * cs + li];
        const double2 v1 = a.lam_box[(size_t)(2 * pass + 1) * cs + li];
        l0.x = (R)v0.x;
        l0.y = (R)v0.y;
        l1.x = (R)v1.x;
        l1.y = (R)v1.y;
      } else {
        l0.x = (R)a.lam[2 * pass];
        l1.x = (R)a.lam[2 * pass + 1];
      }
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        acc0[i] = l0;
        acc1[i] = l1;
      }
    }
    if (any) {                                     // uniform across the block
      __syncthreads();
#pragma unroll
      for (int j = 0; j < TPS; ++j)
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          const int idx = t + i * NT;
          if (valid[j] && idx < Nk2) tile[j * Nk * ld + (idx / Nk) * ld + idx % Nk] = buf[j][i];
        }
      __syncthreads();
    }
    if (s + 1 < nsteps) fetch(s + 1);              // in flight while these tiles are consumed
#pragma unroll
    for (int j = 0; j < TPS; ++j) {
      if (!valid[j]) continue;
      const int term = term0 + j;
      const R c0 = (R)kCoef[pass][term][0], c1 = (R)kCoef[pass][term][1];
      const unsigned short* og = offs + (pass * 2 + (term >> 1)) * Nk2;
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const int e = min(t + i * NT, Nk2 - 1);
        const C v = tile[j * Nk * ld + og[e]];
        acc0[i] = axpy(acc0[i], c0, v);
        acc1[i] = axpy(acc1[i], c1, v);
      }
    }
    if (term0 + TPS == 4) {
      C* o0 = a.gamma + (size_t)(2 * pass) * chan;
      C* o1 = a.gamma + (size_t)(2 * pass + 1) * chan;
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const int e = t + i * NT;
        if (e < Nk2) {
          const int Q = e / Nk, Kp = e - (e / Nk) * Nk;
          const size_t off = (size_t)(jm * Nk + Q) * nn + (size_t)kbi * n + (size_t)in2 * Nk + Kp;
          if (lines) {                                 // written once, read by a later stage
            st_stream(o0 + off, acc0[i]);
            st_stream(o1 + off, acc1[i]);
          } else {
            o0[off] = acc0[i];
            o1[off] = acc1[i];
          }
        }
      }
    }
  }
}

// The remap of a lattice of few momenta, without the LDS tiles: one workgroup
// per (k, m) as above, a thread per output (n', Q, K') with K' fastest, its eight
// source values gathered straight from memory. The tile of a term is then at
// most a few KB, which L1 holds, and all Nv tiles of all terms are in flight at
// once, where the tiled kernel walks its 8 Nv tiles with two barriers each and
// Nk^2 of its 512 threads busy. The sums run in the tiled kernel's order (same
// bits). One momentum, Nv = 32: 307 -> 6 us.
template <typename C>
__global__ __launch_bounds__(kThreads) void remap_direct_kernel(RemapArgs<C> a) {
  using R = decltype(C().x);
  const Dims& d = a.d;
  const int Nk = d.Nk, Lx = d.Lx, Ly = d.Ly, hv = d.Nv / 2;
  const int lin = xcd_linear();
  const int kbi = lin / d.NW, jm = lin - (lin / d.NW) * d.NW;
  const int nk = kbi / Nk - hv, K = kbi - (kbi / Nk) * Nk;
  const int m = jm - (hv - 1);
  const size_t n = d.n, nn = (size_t)d.n * d.n, chan = (size_t)d.cs, row = (size_t)kbi * n;
  const size_t lcs = (size_t)d.NW * d.Nv * d.Nv;
  const int total = d.Nv * Nk * Nk;
  const bool lines = stream_rows<C>(Nk);
  for (int i = threadIdx.x; i < total; i += kThreads) {
    const int r_ = i / Nk, Kp = i - r_ * Nk, in2 = r_ / Nk, Q = r_ - in2 * Nk, n2 = in2 - hv;
    // geometries: ph-bar, pp, st-1, st-2
    const int kpk = ksub(Kp, K, Lx, Ly), kq = kadd(K, Q, Lx, Ly);
    const int mp[4] = {n2 - nk, nk + n2 + m + 1, n2 - nk, m - nk - n2 - 1};
    const int nb[4] = {nk + m, n2, m - n2 - 1, n2};
    const int P[4] = {kpk, kadd(kq, Kp, Lx, Ly), kpk, ksub(ksub(Q, K, Lx, Ly), Kp, Lx, Ly)};
    const int B[4] = {kq, Kp, ksub(Q, Kp, Lx, Ly), Kp};
    C v[4][2];
    bool ok[4], in[4];
    size_t p[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {                 // clamped addresses: every load is in bounds
      ok[g] = in_bbox(mp[g], d.Nv);
      in[g] = in_fbox(nb[g], d.Nv);
      p[g] = ok[g] ? (size_t)((mp[g] + hv - 1) * Nk + P[g]) : 0;
      const C* src = a.phi + (g == 1 ? 2 * chan : 0) + p[g] * nn + row + (in[g] ? (nb[g] + hv) * Nk + B[g] : 0);
      v[g][0] = src[0];
      v[g][1] = src[chan];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (ok[g] && !in[g]) {                      // (ph-bar and st-1 only)
        const size_t q0 = (g == 1 ? 2 * d.Nq : 0) + p[g], q1 = q0 + d.Nq;
        v[g][0] = from_d<C>(cadd(a.k1[q0], a.k2[q0 * n + kbi]));
        v[g][1] = from_d<C>(cadd(a.k1[q1], a.k2[q1 * n + kbi]));
      }
    }
    C* out = a.gamma + (size_t)(jm * Nk + Q) * nn + row + (size_t)in2 * Nk + Kp;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      C acc[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        acc[c] = czero<C>();
        if (a.lam_box) {
          const double2 l = a.lam_box[(size_t)(2 * pass + c) * lcs + ((size_t)jm * d.Nv + kbi / Nk) * d.Nv + in2];
          acc[c].x = (R)l.x;
          acc[c].y = (R)l.y;
        } else {
          acc[c].x = (R)a.lam[2 * pass + c];
        }
#pragma unroll
        for (int term = 0; term < 4; ++term) {
          const int g = 2 * pass + (term >> 1);
          if (ok[g]) acc[c] = axpy(acc[c], (R)kCoef[pass][term][c], v[g][term & 1]);
        }
        C* o = out + (size_t)(2 * pass + c) * chan;
        if (lines) st_stream(o, acc[c]);
        else *o = acc[c];
      }
    }
  }
}

template <typename C, int EPT, int NT, int TPS>
hipError_t run_remap(const RemapArgs<C>& a, hipStream_t s) {
  const Dims& d = a.d;
  const size_t lds = align256(sizeof(C) * TPS * d.Nk * (d.Nk + 1) + 4 * sizeof(unsigned short) * d.Nk * d.Nk);
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)remap_kernel<C, EPT, NT, TPS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((remap_kernel<C, EPT, NT, TPS>), dim3(d.n * d.NW), dim3(NT), lds, s, a);
  return hipGetLastError();
}

template <typename C>
hipError_t dispatch_remap(const Dims& d, const double lam[4], const double2* lam_box, const void* phi,
                          const double2* k1, const double2* k2, void* gamma, hipStream_t s) {
  const RemapArgs<C> a{d, {lam[0], lam[1], lam[2], lam[3]}, lam_box, (const C*)phi, k1, k2, (C*)gamma};
  const int Nk2 = d.Nk * d.Nk;
  constexpr bool c64 = sizeof(C) == sizeof(float2);
  // Up to 12 momenta gather directly (2x3, Nv = 16, complex128 with the kernel
  // functions: 32 us, tiled 75; 3x4, Nv = 24, complex64: 645 against 674); at 16
  // the tiles win (4x4, Nv = 16, complex64: 271 against 314). The
  // tiles per step are what the LDS of two workgroups or more holds.
  if (d.Nk <= kDirectNk) {
    hipLaunchKernelGGL(remap_direct_kernel<C>, dim3(d.n * d.NW), dim3(kThreads), 0, s, a);
    return hipGetLastError();
  }
  if (Nk2 <= 256) return run_remap<C, 1, 256, 4>(a, s);
  if (Nk2 <= 2 * 256) return run_remap<C, 2, 256, 4>(a, s);
  if (Nk2 <= 3 * 256) return run_remap<C, 3, 256, 4>(a, s);
  if (Nk2 <= 4 * 256) return run_remap<C, 4, 256, c64 ? 4 : 2>(a, s);
  if (Nk2 <= 3 * 512) return run_remap<C, 3, 512, c64 ? 4 : 2>(a, s);
  if (Nk2 <= 4 * 512) return run_remap<C, 4, 512, c64 ? 2 : 1>(a, s);
  if (Nk2 <= 5 * 512) return run_remap<C, 5, 512, c64 ? 2 : 1>(a, s);
  if (Nk2 <= 6 * 512) return run_remap<C, 6, 512, c64 ? 2 : 1>(a, s);
  if (Nk2 <= 8 * 512) return run_remap<C, 8, 512, 1>(a, s);
  return hipErrorInvalidValue;
}

// Lambda_r = (U, -U, 2U, 0) at every point of a [4][NW][Nv][Nv] box array
__global__ __launch_bounds__(kThreads) void lambda_fill_kernel(double2* lam, size_t per_channel, double U) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 4 * per_channel) return;
  const int r = (int)(i / per_channel);
  const double v = r == 0 ? U : r == 1 ? -U : r == 2 ? 2.0 * U : 0.0;
  lam[i] = mk(v, 0.0);
}

}  // namespace

template <typename C>
static void run_extract(const KxArgs<C>& a, size_t lds, hipStream_t s) {
  const dim3 grid(4 * a.d.Nq);
  if (a.d.Nk > 8) hipLaunchKernelGGL((kernel_extract_kernel<C, 16>), grid, dim3(kThreads), lds, s, a);
  else if (a.d.Nk > 4) hipLaunchKernelGGL((kernel_extract_kernel<C, 8>), grid, dim3(kThreads), lds, s, a);
  else if (a.d.Nk > 2) hipLaunchKernelGGL((kernel_extract_kernel<C, 4>), grid, dim3(kThreads), lds, s, a);
  else if (a.d.Nk > 1) hipLaunchKernelGGL((kernel_extract_kernel<C, 2>), grid, dim3(kThreads), lds, s, a);
  else hipLaunchKernelGGL((kernel_extract_kernel<C, 1>), grid, dim3(kThreads), lds, s, a);
}

hipError_t launch_kernel_extract(const pq_params& p, const Dims& d, const void* phi, double2* k1,
                                 double2* k2, hipStream_t s) {
  size_t lds = 2 * sizeof(double2) * (size_t)d.n;
  if (lds > 64 * 1024) return hipErrorInvalidValue;
  if (p.storage == PQ_STORE_C64)
    run_extract(KxArgs<float2>{d, p.kernel_level, p.edge_rule, (const float2*)phi, k1, k2}, lds, s);
  else
    run_extract(KxArgs<double2>{d, p.kernel_level, p.edge_rule, (const double2*)phi, k1, k2}, lds, s);
  return hipGetLastError();
}

hipError_t launch_remap(const pq_params& p, const Dims& d, const double lam[4], const double2* lam_box,
                        const void* phi, const double2* k1, const double2* k2, void* gamma, hipStream_t s) {
  if (d.Nk > 64) return hipErrorInvalidValue;
  if (p.storage == PQ_STORE_C64) return dispatch_remap<float2>(d, lam, lam_box, phi, k1, k2, gamma, s);
  return dispatch_remap<double2>(d, lam, lam_box, phi, k1, k2, gamma, s);
}

hipError_t launch_lambda_fill(const Dims& d, double U, double2* lam_box, hipStream_t s) {
  const size_t per = (size_t)d.NW * d.Nv * d.Nv;
  hipLaunchKernelGGL(lambda_fill_kernel, dim3((unsigned)((4 * per + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                     lam_box, per, U);
  return hipGetLastError();
}

}  // namespace pq
