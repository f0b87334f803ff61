// Device-side helpers shared by the parquet kernels: complex arithmetic on
// float2/double2, compound-index and momentum arithmetic, block reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "parquet.h"

namespace pq {

// ----------------------------------------------------------------- sizes
struct Dims {
  int Lx, Ly, Nk, Nv, NW, f, Nve, NWe, NG, n, Nq, ntau;
  // elements between the channel arrays of a vertex (Phi, Gamma): Nq n^2 for
  // one instance's [4][Nq][n][n]; K Nq n^2 in a batch of K instances of one
  // box, whose vertices are stored [4][K][Nq][n][n]
  long long cs;
};

// ------------------------------------------------------------- complex
template <typename T> struct cplx_of;
template <> struct cplx_of<float> { using type = float2; };
template <> struct cplx_of<double> { using type = double2; };

__host__ __device__ inline double2 mk(double r, double i) { return make_double2(r, i); }
__host__ __device__ inline float2 mkf(float r, float i) { return make_float2(r, i); }

__device__ inline double2 cadd(double2 a, double2 b) { return mk(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return mk(a.x - b.x, a.y - b.y); }
__device__ inline double2 cmul(double2 a, double2 b) {
  return mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double2 cscale(double2 a, double s) { return mk(a.x * s, a.y * s); }
__device__ inline double2 cdiv(double2 a, double2 b) {
  // Smith's algorithm
  if (fabs(b.x) >= fabs(b.y)) {
    double r = b.y / b.x, d = b.x + b.y * r;
    return mk((a.x + a.y * r) / d, (a.y - a.x * r) / d);
  } else {
    double r = b.x / b.y, d = b.x * r + b.y;
    return mk((a.x * r + a.y) / d, (a.y * r - a.x) / d);
  }
}
__device__ inline double2 crecip(double2 b) { return cdiv(mk(1.0, 0.0), b); }

__device__ inline float2 cadd(float2 a, float2 b) { return mkf(a.x + b.x, a.y + b.y); }
__device__ inline float2 csub(float2 a, float2 b) { return mkf(a.x - b.x, a.y - b.y); }
__device__ inline float2 cmul(float2 a, float2 b) {
  return mkf(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline float2 cscale(float2 a, float s) { return mkf(a.x * s, a.y * s); }
__device__ inline float2 cdiv(float2 a, float2 b) {
  if (fabsf(b.x) >= fabsf(b.y)) {
    float r = b.y / b.x, d = b.x + b.y * r;
    return mkf((a.x + a.y * r) / d, (a.y - a.x * r) / d);
  } else {
    float r = b.x / b.y, d = b.x * r + b.y;
    return mkf((a.x * r + a.y) / d, (a.y * r - a.x) / d);
  }
}

__device__ inline double2 to_d(float2 a) { return mk((double)a.x, (double)a.y); }
__device__ inline double2 to_d(double2 a) { return a; }
template <typename C> __device__ inline C from_d(double2 a);
template <> __device__ inline double2 from_d<double2>(double2 a) { return a; }
template <> __device__ inline float2 from_d<float2>(double2 a) { return mkf((float)a.x, (float)a.y); }

__device__ inline double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }

// ------------------------------------------------ index arithmetic
// Fermionic box index of n (caller checks range): n + Nv/2.
__device__ inline bool in_fbox(int n, int Nv) { return n >= -Nv / 2 && n <= Nv / 2 - 1; }
__device__ inline bool in_bbox(int m, int Nv) { return m >= -(Nv / 2 - 1) && m <= Nv / 2 - 1; }
__device__ inline int kx_of(int K, int Ly) { return K / Ly; }
__device__ inline int ky_of(int K, int Ly) { return K - (K / Ly) * Ly; }
__device__ inline int kadd(int a, int b, int Lx, int Ly) {
  int ax = a / Ly, ay = a - ax * Ly, bx = b / Ly, by = b - bx * Ly;
  int x = ax + bx; if (x >= Lx) x -= Lx;
  int y = ay + by; if (y >= Ly) y -= Ly;
  return x * Ly + y;
}
__device__ inline int ksub(int a, int b, int Lx, int Ly) {
  int ax = a / Ly, ay = a - ax * Ly, bx = b / Ly, by = b - bx * Ly;
  int x = ax - bx; if (x < 0) x += Lx;
  int y = ay - by; if (y < 0) y += Ly;
  return x * Ly + y;
}

// ------------------------------------------------------ reductions
// Sum over each group of L = 16, 32 or 64 lanes of a wave, left in the group's
// last lane: row shifts and row broadcasts on the vector unit (a shuffle per
// step goes through the LDS crossbar, several times the latency). All lanes
// must be active.
template <int CTRL, int ROWS>
__device__ inline double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
template <int L>
__device__ inline double group_total(double v) {
  static_assert(L == 16 || L == 32 || L == 64, "rows of 16 lanes");
  v = dpp_add<0x111, 0xf>(v);                   // row_shr 1, 2, 4, 8
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  if (L >= 32) v = dpp_add<0x142, 0xa>(v);      // row_bcast 15 into rows 1 and 3
  if (L >= 64) v = dpp_add<0x143, 0xc>(v);      // row_bcast 31 into rows 2 and 3
  return v;
}

template <int CTRL, int ROWS>
__device__ inline double dpp_max(double v) {         // lanes without a source keep their own
  const int l = __double2loint(v), h = __double2hiint(v);
  return fmax(v, __hiloint2double(__builtin_amdgcn_update_dpp(h, h, CTRL, ROWS, 0xf, false),
                                  __builtin_amdgcn_update_dpp(l, l, CTRL, ROWS, 0xf, false)));
}

// Deterministic block reductions of doubles: in the wave's registers, then one
// exchange (a tree in LDS, with a barrier per level, took about 1 us a call in
// kernels of 5 to 15 us that make two to five of them). blockDim.x must be a
// multiple of 64, at most 1024; `red` is LDS of blockDim.x / 64 doubles or more.
__device__ inline double block_sum(double v, double* red) {
  v = group_total<64>(v);
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r += red[w];
  __syncthreads();
  return r;
}

__device__ inline double block_max(double v, double* red) {
  v = dpp_max<0x111, 0xf>(v);
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);
  v = dpp_max<0x143, 0xc>(v);
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, red[w]);
  __syncthreads();
  return r;
}

// Work-item order for a 2-D grid on the 8 XCDs of the chip. Workgroups are
// dealt to the XCDs round-robin by linear id; this returns the logical id so
// that the workgroups one XCD receives are consecutive in logical order (the
// first eighth of the work goes to XCD 0, and so on), which keeps the operands
// that neighbouring work items share in that XCD's own L2. A tail that does
// not divide by 8 keeps the identity order.
__device__ inline unsigned xcd_linear() {
  const unsigned total = gridDim.x * gridDim.y;
  const unsigned lin = blockIdx.y * gridDim.x + blockIdx.x;
  const unsigned per = total >> 3;
  return lin < (per << 3) ? (lin & 7u) * per + (lin >> 3) : lin;
}

}  // namespace pq
