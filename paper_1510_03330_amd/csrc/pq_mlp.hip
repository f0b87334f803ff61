// Learned warm start: the small multilayer perceptron that maps model
// parameters to kernel functions (forward, backward, Adam), the factorised
// output head (an orthonormal basis of the training solutions, built by
// Gram-Schmidt, and the expansion of predicted coefficients in it), and the
// reducible vertex rebuilt from kernel values (second-level kernel
// approximation, Sec. "Two-level kernel approximations": Phi ~ K1(q) +
// K2(k;q) + K2(k';q)).
//
// Network: hidden layers h_l = tanh(h_{l-1} W_l^T + b_l), linear output.
// Parameters packed layer by layer as [W_l (out x in, row-major), b_l (out)].
// Every product runs on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16) with
// FP32 accumulation: the weights enter as their bf16 copy (round to nearest
// even), the FP32 activations and gradients as two bf16 terms hi + lo, which
// carries them to about 2^-16 relative, so the products match FP32 operands
// with bf16 weights. Biases, activations and accumulation are FP32.
// Loss: mean squared error over all outputs.
#include <algorithm>
#include <utility>
#include <vector>

#include "pq_internal.h"

namespace pq {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ---- products -------------------------------------------------------------
// At the sizes of the warm start (batches of tens to hundreds, widths of a few
// hundred) a product is latency: one 32 x 32 tile per workgroup, whose eight
// waves bring kKC of K into LDS at once (an activation or gradient as hi + lo, a
// weight as its bf16 value) in the matrix cores' operand order; one wave then
// runs the chain of products over K in order (two per 16 of K: about 0.5 us for
// 512), so every output is one FP32 accumulation over ascending k. The weight
// gradient (K is the batch, both operands FP32, lo x lo dropped) reads its
// operands straight into registers, a tile per wave. 64 x 512 x 512 forward:
// 6.3 us, against 59 us with 64 x 64 tiles staged 32 of K at a time (8
// workgroups, two barriers per round); the whole step at batch 64 63 us
// against 520, at batch 65536 20 ms against 112.
constexpr int kSW = 8;                       // waves per workgroup
constexpr int kSThreads = 64 * kSW;
constexpr int kKG = 64, kKC = 8 * kKG;       // K staged at a time, in groups of 8
constexpr int kGU = 2;                       // steps in flight of the weight gradient

// this lane's 8 consecutive k of one row or column; VEC: k contiguous, K a
// multiple of 8 and 16-byte aligned rows; values past K (or of a row past the
// matrix, ok = false) are zero
template <bool VEC>
__device__ inline void load8(const float* p, long sk, int k, int K, bool ok, float (&v)[8]) {
  if constexpr (VEC) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    f4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    if (ok && k < K) {
      a = *(const f4*)(p + k);
      b = *(const f4*)(p + k + 4);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = a[e];
      v[4 + e] = b[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ok && k + e < K ? p[(long)(k + e) * sk] : 0.f;
  }
}
template <bool VEC>
__device__ inline bf16x8 load8(const __bf16* p, long sk, int k, int K, bool ok) {
  bf16x8 v;
  if constexpr (VEC) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.f;
    if (ok && k < K) v = *(const bf16x8*)(p + k);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ok && k + e < K ? p[(long)(k + e) * sk] : (__bf16)0.f;
  }
  return v;
}

__device__ inline void split(const float (&v)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    hi[e] = (__bf16)v[e];
    lo[e] = (__bf16)(v[e] - (float)hi[e]);
  }
}

// The gradient at the outputs, d = 2 (y - t) / count, formed where it is read
// (t = nullptr: p holds d itself).
struct GradSrc {
  const float* p;
  const float* t;
  float count;
  __device__ float at(size_t i) const {
    const float v = p[i];
    return t ? 2.f * (v - t[i]) / count : v;
  }
  // 8 consecutive values of a row of n from column k (VEC as in load8)
  template <bool VEC>
  __device__ void row8(size_t row, int k, int n, bool ok, float (&v)[8]) const {
    load8<VEC>(p + row, 1, k, n, ok, v);
    if (t) {
      float u[8];
      load8<VEC>(t + row, 1, k, n, ok, u);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = 2.f * (v[e] - u[e]) / count;
    }
  }
};

// The staged operands of a 32 x 32 tile: row or column r, k group g
struct Stage {
  bf16x8 ah[32][kKG + 1], al[32][kKG + 1], b[32][kKG + 1];
};

// C[m][n] = sum_k A(m, k) B(k, n) over the staged operands, by the first wave;
// la(row, k, v[8]) and lb(col, k) give 8 consecutive k (zero outside the
// matrices), f(row, col, sum) takes the elements, spread over the workgroup.
template <class LA, class LB, class F>
__device__ inline void tile_product(Stage& st, float (*out)[64], int K, LA la, LB lb, F f) {
  constexpr int GPT = 32 * kKG / kSThreads;  // groups per thread and operand
  const int t = threadIdx.x, lane = t & 63;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  for (int k0 = 0; k0 < K; k0 += kKC) {
    float av[GPT][8];
    bf16x8 bv[GPT];
#pragma unroll
    for (int i = 0; i < GPT; ++i) {
      const int e = t + i * kSThreads, r = e / kKG, k = k0 + 8 * (e % kKG);
      la(r, k, av[i]);
      bv[i] = lb(e, k0);
    }
    if (k0 > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < GPT; ++i) {
      const int e = t + i * kSThreads, r = e / kKG, g = e % kKG;
      split(av[i], st.ah[r][g], st.al[r][g]);
      lb.put(st, e, bv[i]);
    }
    __syncthreads();
    if (t < 64) {
      const int steps = (min(K - k0, kKC) + 15) / 16;
#pragma unroll 4
      for (int s = 0; s < steps; ++s) {
        const int r = lane & 31, g = 2 * s + (lane >> 5);
        const bf16x8 b = st.b[r][g];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.al[r][g], b, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.ah[r][g], b, acc, 0, 0, 0);
      }
    }
  }
  if (t < 64)
#pragma unroll
    for (int v = 0; v < 16; ++v) out[v][lane] = acc[v];
  __syncthreads();
  for (int e = t; e < 1024; e += kSThreads) {
    const int v = e >> 6, l = e & 63;
    f(8 * (v >> 2) + 4 * (l >> 5) + (v & 3), l & 31, out[v][l]);
  }
}

// weights as the forward product reads them: column n = output o, k along the row W[o][k]
template <bool VEC>
struct WRows {
  const __bf16* W;
  int n0, out, in;
  __device__ bf16x8 operator()(int e, int k0) const {
    const int n = n0 + e / kKG;
    return load8<VEC>(W + (size_t)min(n, out - 1) * in, 1, k0 + 8 * (e % kKG), in, n < out);
  }
  __device__ void put(Stage& st, int e, bf16x8 v) const { st.b[e / kKG][e % kKG] = v; }
};
// and as the input gradient reads them: column n = input i, k = output o down the
// rows; lanes take neighbouring i of one group of rows
struct WCols {
  const __bf16* W;
  int n0, out, in;
  __device__ bf16x8 operator()(int e, int k0) const {
    const int n = n0 + e % 32;
    return load8<false>(W + min(n, in - 1), in, k0 + 8 * (e / 32), out, n < in);
  }
  __device__ void put(Stage& st, int e, bf16x8 v) const { st.b[e % 32][e / 32] = v; }
};

// The tiles of a launch over the grid's two dimensions: a dimension takes fewer
// than 2^32 work items, which 2^23 workgroups of 512 reach (8192 outputs of a batch
// of 2^20). Workgroups past the last tile exit.
constexpr size_t kGridX = size_t(1) << 22;
constexpr size_t kMaxTiles = size_t(1) << 30;        // (4 TB of outputs)
inline dim3 tile_grid(size_t tiles) {
  const size_t x = std::min(tiles, kGridX);
  return dim3((unsigned)x, (unsigned)((tiles + x - 1) / x));
}
__device__ inline unsigned tile_index() { return blockIdx.y * gridDim.x + blockIdx.x; }

// y[b][o] = act(sum_i h[b][i] W[o][i] + bias[o])
template <bool VEC>
__global__ __launch_bounds__(kSThreads) void mlp_forward_kernel(int B, int out, int in, const float* h,
                                                                const __bf16* W, const float* bias, float* y,
                                                                int tanh_act) {
  __shared__ Stage st;
  __shared__ float res[16][64];
  const unsigned nt = (out + 31) / 32, id = tile_index();
  const int m0 = (int)(id / nt) * 32, n0 = (int)(id % nt) * 32;
  if (m0 >= B) return;
  tile_product(
      st, res, in,
      [&](int r, int k, float (&v)[8]) {
        load8<VEC>(h + (size_t)min(m0 + r, B - 1) * in, 1, k, in, m0 + r < B, v);
      },
      WRows<VEC>{W, n0, out, in},
      [&](int r, int c, float s) {
        const int b = m0 + r, o = n0 + c;
        if (b < B && o < out) {
          s += bias[o];
          y[(size_t)b * out + o] = tanh_act ? tanhf(s) : s;
        }
      });
}

// One layer of the backward pass in one launch, by workgroup index:
//   [0, ndn):  dn[b][i] = (sum_o d[b][o] W[o][i]) (1 - hin[b][i]^2), a 32 x 32 tile each
//   [ndn, ndn + ngw): gW[o][i] = sum_b d[b][o] hin[b][i], eight 32 x 32 tiles (one per
//              wave, 32 outputs x 256 inputs) each
//   [ndn + ngw, + ngb): gb[o] = sum_b d[b][o], one output per thread
//   the last one (d.t given): loss = mean (y - t)^2
template <bool VEC>
__global__ __launch_bounds__(kSThreads) void mlp_backward_kernel(int B, int out, int in, GradSrc d, const float* hin,
                                                                 const __bf16* W, float* gW, float* gb, float* dn,
                                                                 float* loss, int ndn, int ngw, int ngb) {
  __shared__ Stage st;
  __shared__ float res[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int id = (int)tile_index();
  if (id >= ndn + ngw + ngb + (d.t ? 1 : 0)) return;
  if (id < ndn) {
    const int nt = (in + 31) / 32, m0 = (id / nt) * 32, n0 = (id - (id / nt) * nt) * 32;
    tile_product(
        st, res, out,
        [&](int r, int k, float (&v)[8]) {
          d.row8<VEC>((size_t)min(m0 + r, B - 1) * out, k, out, m0 + r < B, v);
        },
        WCols{W, n0, out, in},
        [&](int r, int c, float s) {
          const int b = m0 + r, i = n0 + c;
          if (b < B && i < in) {
            const float e = hin[(size_t)b * in + i];
            dn[(size_t)b * in + i] = s * (1.f - e * e);
          }
        });
    return;
  }
  id -= ndn;
  if (id < ngw) {
    const int l32 = lane & 31, kk = 8 * (lane >> 5);
    const int nt = (in + 32 * kSW - 1) / (32 * kSW), m0 = (id / nt) * 32;
    const int n0 = ((id - (id / nt) * nt) * kSW + w) * 32;
    if (n0 >= in) return;                         // no barrier below
    const int m = m0 + l32, n = n0 + l32;
    const bool mok = m < out, nok = n < in;
    const int mc = mok ? m : 0, nc = nok ? n : 0;
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int k0 = 0; k0 < B; k0 += 16 * kGU) {
      float av[kGU][8], bv[kGU][8];
#pragma unroll
      for (int u = 0; u < kGU; ++u) {
        const int k = k0 + 16 * u + kk;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool in_b = k + e < B;
          av[u][e] = mok && in_b ? d.at((size_t)(k + e) * out + mc) : 0.f;
          bv[u][e] = nok && in_b ? hin[(size_t)(k + e) * in + nc] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < kGU; ++u) {
        bf16x8 ah, al, bh, bl;
        split(av[u], ah, al);
        split(bv[u], bh, bl);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int o = m0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      if (o < out && nok) gW[(size_t)o * in + n] = acc[v];
    }
    return;
  }
  id -= ngw;
  if (id < ngb) {
    const int o = id * kSThreads + (int)threadIdx.x;
    if (o >= out) return;
    float s = 0.f;
#pragma unroll 8
    for (int b = 0; b < B; ++b) s += d.at((size_t)b * out + o);
    gb[o] = s;
    return;
  }
  // the loss
  const int cnt = B * out;
  float part[8] = {};
  for (int i0 = threadIdx.x; i0 < cnt; i0 += 8 * kSThreads) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = min(i0 + u * kSThreads, cnt - 1);
      const float e = i0 + u * kSThreads < cnt ? d.p[i] - d.t[i] : 0.f;
      part[u] += e * e;
    }
  }
  float* rs = &res[0][0];
  rs[threadIdx.x] = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
  __syncthreads();
  for (int st_ = kSThreads / 2; st_ > 0; st_ >>= 1) {
    if (threadIdx.x < st_) rs[threadIdx.x] += rs[threadIdx.x + st_];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = rs[0] / d.count;
}

constexpr size_t kSLoss = 65536;             // loss terms one workgroup sums beside the last layer

inline bool vec8(const void* p, int K) { return K % 8 == 0 && (uintptr_t)p % 16 == 0; }

// d = 2 (y - t) / count and loss = mean (y - t)^2, in two passes with a fixed
// summation order (deterministic): each workgroup of the first pass sums a
// fixed grid-stride subset into part[blockIdx.x], the second (one workgroup)
// sums the parts.
__device__ inline float block_sum256(float v, float* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  return red[0];
}

__global__ __launch_bounds__(256) void mse_partial_kernel(size_t count, const float* y, const float* t, float* d,
                                                          float* part) {
  __shared__ float red[256];
  float s = 0.f;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x) {
    const float e = y[i] - t[i];
    d[i] = 2.f * e / (float)count;
    s += e * e;
  }
  const float b = block_sum256(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

__global__ __launch_bounds__(256) void mse_final_kernel(int nparts, const float* part, size_t count, float* loss) {
  __shared__ float red[256];
  float s = 0.f;
  for (int i = threadIdx.x; i < nparts; i += blockDim.x) s += part[i];
  const float b = block_sum256(s, red);
  if (threadIdx.x == 0) *loss = b / (float)count;
}

__global__ __launch_bounds__(256) void adam_kernel(size_t count, float* p, __bf16* pb, float* m, float* v,
                                                   const float* g, float lr, float b1, float b2, float eps,
                                                   float c1, float c2) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float w = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = w;
  pb[i] = (__bf16)w;
}

__global__ __launch_bounds__(256) void to_bf16_kernel(size_t count, const float* p, __bf16* pb) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) pb[i] = (__bf16)p[i];
}

template <typename C>
__global__ __launch_bounds__(256) void phi_from_kernels_kernel(Dims d, const double2* k1, const double2* k2,
                                                               C* phi) {
  const size_t n = d.n, total = 4 * (size_t)d.Nq * n * n;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const size_t kp = i % n, k = (i / n) % n, rq = i / (n * n);      // rq = r Nq + q
    const size_t r = rq / d.Nq, q = rq - r * d.Nq;
    const double2 a = k1[rq], b = k2[rq * n + k], c = k2[rq * n + kp];
    phi[r * d.cs + (q * n + k) * n + kp] = from_d<C>(mk(a.x + b.x + c.x, a.y + b.y + c.y));
  }
}

// ---- factorised output head: orthonormal basis of the training outputs ----
// Rows y_i (i < rows, len floats each) are centred on their mean and
// orthonormalised in order by classical Gram-Schmidt with one
// re-orthogonalisation pass; sample i is then y_i = mean + sum_{j<=i} c_ij q_j.
// Dot products accumulate in FP64 over kParts fixed segments of the row and are
// summed in a fixed order (deterministic).

__device__ inline double block_sum256d(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// mean[x] = (1 / rows) sum_i Y[i][x]; Y[i][x] -= mean[x]
__global__ __launch_bounds__(256) void center_kernel(float* Y, int rows, size_t len, float* mean) {
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < len; x += (size_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int i = 0; i < rows; ++i) s += Y[(size_t)i * len + x];
    const float mu = (float)(s / rows);
    mean[x] = mu;
    for (int i = 0; i < rows; ++i) Y[(size_t)i * len + x] -= mu;
  }
}

// part[j][b] = sum over segment b of Q_j[x] y[x] for j < nq, and of y[x]^2 for j = nq
__global__ __launch_bounds__(256) void dots_kernel(const float* Q, int nq, size_t len, const float* y,
                                                   double* part) {
  __shared__ double red[256];
  const size_t per = (len + gridDim.x - 1) / gridDim.x;
  const size_t lo = (size_t)blockIdx.x * per, hi = lo + per < len ? lo + per : len;
  for (int j = 0; j <= nq; ++j) {
    const float* q = j < nq ? Q + (size_t)j * len : y;
    double acc = 0.0;
    for (size_t x = lo + threadIdx.x; x < hi; x += blockDim.x) acc += (double)q[x] * (double)y[x];
    const double b = block_sum256d(acc, red);
    if (threadIdx.x == 0) part[(size_t)j * gridDim.x + blockIdx.x] = b;
  }
}

// r[j] = sum_b part[j][b] (in order), j <= nq
__global__ __launch_bounds__(256) void dots_reduce_kernel(const double* part, int nparts, int nq, double* r) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j > nq) return;
  double s = 0.0;
  for (int b = 0; b < nparts; ++b) s += part[(size_t)j * nparts + b];
  r[j] = s;
}

// y[x] -= sum_{j < nq} r[j] Q_j[x]
__global__ __launch_bounds__(256) void project_out_kernel(const float* Q, int nq, size_t len, const double* r,
                                                          float* y) {
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < len; x += (size_t)gridDim.x * blockDim.x) {
    double v = y[x];
    for (int j = 0; j < nq; ++j) v -= r[j] * (double)Q[(size_t)j * len + x];
    y[x] = (float)v;
  }
}

// Row i done: c[i][j] = r1[j] + r2[j] (j < i), c[i][i] = |y_i| after both
// passes; the row is kept (scaled to unit norm) when that norm exceeds 1e-6 of
// the centred row's, else it is dropped (set to zero: no new direction).
__global__ void basis_row_kernel(int i, int rows, const double* r1, const double* r2, const double* r3,
                                 double* c, double* rinv) {
  const int j = threadIdx.x + blockIdx.x * blockDim.x;
  const double nrm = sqrt(r3[0]), orig = sqrt(r1[i]);
  const bool keep = nrm > 1e-6 * orig && nrm > 0.0;
  if (j < rows) c[(size_t)i * rows + j] = j < i ? r1[j] + r2[j] : (j == i && keep ? nrm : 0.0);
  if (j == 0) *rinv = keep ? 1.0 / nrm : 0.0;
}

__global__ __launch_bounds__(256) void scale_row_kernel(float* y, size_t len, const double* rinv) {
  const double a = *rinv;
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < len; x += (size_t)gridDim.x * blockDim.x)
    y[x] = (float)(a * y[x]);
}

// scale = root mean square of c (rows x rows); out[i ld + j] = c[i][j] / scale
__global__ __launch_bounds__(256) void basis_coef_kernel(const double* c, int rows, float* out, int ld,
                                                         float* scale) {
  __shared__ double red[256];
  const size_t cnt = (size_t)rows * rows;
  double s = 0.0;
  for (size_t e = threadIdx.x; e < cnt; e += blockDim.x) s += c[e] * c[e];
  const double tot = block_sum256d(s, red);
  const double rms = tot > 0.0 ? sqrt(tot / (double)cnt) : 1.0;
  for (size_t e = threadIdx.x; e < cnt; e += blockDim.x)
    out[(e / rows) * (size_t)ld + e % rows] = (float)(c[e] / rms);
  if (threadIdx.x == 0) *scale = (float)rms;
}

// out[x] = mean[x] + scale sum_j coef[j] Q_j[x] (FP64 output)
__global__ __launch_bounds__(256) void expand_kernel(const float* Q, int rows, size_t len, const float* mean,
                                                     const float* coef, const float* scale, double* out) {
  const double sc = *scale;
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < len; x += (size_t)gridDim.x * blockDim.x) {
    double v = 0.0;
    for (int j = 0; j < rows; ++j) v += (double)coef[j] * (double)Q[(size_t)j * len + x];
    out[x] = (double)mean[x] + sc * v;
  }
}

constexpr int kBasisParts = 1024;

inline unsigned stream_blocks(size_t len) {
  return (unsigned)std::max<size_t>(1, std::min<size_t>(8192, (len + 255) / 256));
}

}  // namespace

size_t mlp_count(const int32_t* w, int nl) {
  size_t c = 0;
  for (int l = 0; l < nl; ++l) c += (size_t)w[l + 1] * w[l] + w[l + 1];
  return c;
}

hipError_t launch_mlp_forward(const int32_t* w, int nl, const void* pb, const float* p, const float* x, float* acts,
                              int B, hipStream_t s) {
  size_t off = 0, aoff = 0;
  const float* h = x;
  for (int l = 0; l < nl; ++l) {
    const int in = w[l], out = w[l + 1];
    float* y = acts + aoff;
    const __bf16* W = (const __bf16*)pb + off;
    const size_t tiles = (size_t)((out + 31) / 32) * ((B + 31) / 32);
    if (tiles > kMaxTiles) return hipErrorInvalidConfiguration;
    auto kernel = vec8(h, in) && vec8(W, in) ? mlp_forward_kernel<true> : mlp_forward_kernel<false>;
    hipLaunchKernelGGL(kernel, tile_grid(tiles), dim3(kSThreads), 0, s, B, out, in, h, W, p + off + (size_t)out * in, y,
                       l < nl - 1 ? 1 : 0);
    off += (size_t)out * in + out;
    aoff += (size_t)B * out;
    h = y;
  }
  return hipGetLastError();
}

hipError_t launch_mlp_backward(const int32_t* w, int nl, const void* pb, const float* x, const float* acts,
                               const float* target, float* grad, float* loss, float* scratch, int B, hipStream_t s) {
  int maxw = 0;
  for (int l = 0; l <= nl; ++l) maxw = w[l] > maxw ? w[l] : maxw;
  std::vector<size_t> poff(nl), aoff(nl);
  size_t po = 0, ao = 0;
  for (int l = 0; l < nl; ++l) {
    poff[l] = po;
    aoff[l] = ao;
    po += (size_t)w[l + 1] * w[l] + w[l + 1];
    ao += (size_t)B * w[l + 1];
  }
  float* d = scratch;
  float* dn = scratch + (size_t)B * maxw;
  const size_t nout = (size_t)B * w[nl];
  GradSrc g{acts + aoff[nl - 1], target, (float)nout};
  if (nout > kSLoss) {                          // more than one workgroup's worth of loss terms
    const int np = (int)std::min<size_t>({(size_t)1024, (nout + 255) / 256, (size_t)B * maxw});
    hipLaunchKernelGGL(mse_partial_kernel, dim3(np), dim3(256), 0, s, nout, acts + aoff[nl - 1], target, d, dn);
    hipLaunchKernelGGL(mse_final_kernel, dim3(1), dim3(256), 0, s, np, (const float*)dn, nout, loss);
    g = GradSrc{d, nullptr, 0.f};
  }
  for (int l = nl - 1; l >= 0; --l) {
    const int in = w[l], out = w[l + 1];
    const size_t tdn = l > 0 ? (size_t)((B + 31) / 32) * ((in + 31) / 32) : 0;
    const size_t tgw = (size_t)((out + 31) / 32) * ((in + 32 * kSW - 1) / (32 * kSW));
    if (tdn + tgw > kMaxTiles) return hipErrorInvalidConfiguration;
    const int ndn = (int)tdn, ngw = (int)tgw;
    float* gW = grad + poff[l];
    const float* hin = l == 0 ? x : acts + aoff[l - 1];
    const bool vec = vec8(g.p, out) && (!g.t || vec8(g.t, out));
    auto kernel = vec ? mlp_backward_kernel<true> : mlp_backward_kernel<false>;
    const int ngb = (out + kSThreads - 1) / kSThreads;
    hipLaunchKernelGGL(kernel, tile_grid((size_t)ndn + ngw + ngb + (g.t ? 1 : 0)), dim3(kSThreads), 0, s, B, out, in, g, hin,
                       (const __bf16*)pb + poff[l], gW, gW + (size_t)out * in, dn, loss, ndn, ngw, ngb);
    g = GradSrc{dn, nullptr, 0.f};
    std::swap(d, dn);
  }
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* p, void* pb, float* m, float* v, const float* g, size_t count, float lr, float b1,
                           float b2, float eps, int step, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count, p, (__bf16*)pb, m,
                     v, g, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_mlp_to_bf16(const float* p, void* pb, size_t count, hipStream_t s) {
  hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count, p, (__bf16*)pb);
  return hipGetLastError();
}

hipError_t launch_phi_from_kernels(const pq_params& p, const Dims& d, const double2* k1, const double2* k2,
                                   void* phi, hipStream_t s) {
  const size_t total = 4 * (size_t)d.Nq * d.n * d.n;
  const unsigned blocks = (unsigned)std::min<size_t>(65536, (total + 255) / 256);
  if (p.storage == PQ_STORE_C64)
    hipLaunchKernelGGL((phi_from_kernels_kernel<float2>), dim3(blocks), dim3(256), 0, s, d, k1, k2, (float2*)phi);
  else
    hipLaunchKernelGGL((phi_from_kernels_kernel<double2>), dim3(blocks), dim3(256), 0, s, d, k1, k2, (double2*)phi);
  return hipGetLastError();
}

size_t mlp_basis_ws_bytes(int rows) {
  return sizeof(double) * ((size_t)(rows + 1) * kBasisParts + 3 * (size_t)(rows + 1) + (size_t)rows * rows + 1);
}

hipError_t launch_mlp_basis(float* Y, int rows, size_t len, float* mean, float* coef, int ld, float* scale, void* ws,
                            hipStream_t s) {
  double* part = (double*)ws;
  double* r1 = part + (size_t)(rows + 1) * kBasisParts;
  double* r2 = r1 + rows + 1;
  double* r3 = r2 + rows + 1;
  double* c = r3 + rows + 1;
  double* rinv = c + (size_t)rows * rows;
  const unsigned nb = stream_blocks(len);
  const unsigned parts = (unsigned)std::min<size_t>(kBasisParts, (len + 255) / 256);
  hipLaunchKernelGGL(center_kernel, dim3(nb), dim3(256), 0, s, Y, rows, len, mean);
  for (int i = 0; i < rows; ++i) {
    float* y = Y + (size_t)i * len;
    const unsigned rb = (unsigned)((i + 1 + 255) / 256);
    hipLaunchKernelGGL(dots_kernel, dim3(parts), dim3(256), 0, s, (const float*)Y, i, len, (const float*)y, part);
    hipLaunchKernelGGL(dots_reduce_kernel, dim3(rb), dim3(256), 0, s, (const double*)part, (int)parts, i, r1);
    hipLaunchKernelGGL(project_out_kernel, dim3(nb), dim3(256), 0, s, (const float*)Y, i, len, (const double*)r1, y);
    hipLaunchKernelGGL(dots_kernel, dim3(parts), dim3(256), 0, s, (const float*)Y, i, len, (const float*)y, part);
    hipLaunchKernelGGL(dots_reduce_kernel, dim3(rb), dim3(256), 0, s, (const double*)part, (int)parts, i, r2);
    hipLaunchKernelGGL(project_out_kernel, dim3(nb), dim3(256), 0, s, (const float*)Y, i, len, (const double*)r2, y);
    hipLaunchKernelGGL(dots_kernel, dim3(parts), dim3(256), 0, s, (const float*)Y, 0, len, (const float*)y, part);
    hipLaunchKernelGGL(dots_reduce_kernel, dim3(1), dim3(256), 0, s, (const double*)part, (int)parts, 0, r3);
    hipLaunchKernelGGL(basis_row_kernel, dim3((rows + 255) / 256), dim3(256), 0, s, i, rows, (const double*)r1,
                       (const double*)r2, (const double*)r3, c, rinv);
    hipLaunchKernelGGL(scale_row_kernel, dim3(nb), dim3(256), 0, s, y, len, (const double*)rinv);
  }
  hipLaunchKernelGGL(basis_coef_kernel, dim3(1), dim3(256), 0, s, (const double*)c, rows, coef, ld, scale);
  return hipGetLastError();
}

hipError_t launch_mlp_expand(const float* Q, int rows, size_t len, const float* mean, const float* coef,
                             const float* scale, double* out, hipStream_t s) {
  hipLaunchKernelGGL(expand_kernel, dim3(stream_blocks(len)), dim3(256), 0, s, Q, rows, len, mean, coef, scale, out);
  return hipGetLastError();
}

}  // namespace pq
