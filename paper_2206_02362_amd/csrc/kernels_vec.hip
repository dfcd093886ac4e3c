// Vector kernels of the variable-projection solver: the linear
// conjugate-gradient iteration on the normal equation of eq. vp.obj needs
// inner products, the two updates of the iterate and residual, the new search
// direction and the diagonal regularization term eps^2 D* D.
//
// All of them are bandwidth-bound streams over [nh][nx][nz] or data-sized
// FP32 arrays.  Inner products accumulate in FP64 over a fixed grid and are
// reduced in a fixed order, so a result does not depend on scheduling.
#include "internal.h"

#include <algorithm>

namespace fw {

constexpr int kDotBlocks = 1024;
constexpr int kDotThreads = 256;

// out = a - b
__global__ void k_sub(const float *a, const float *b, float *out, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    out[i] = a[i] - b[i];
}

// part[block] = sum over this block's strided share of x[i] * y[i], in FP64
__global__ void __launch_bounds__(kDotThreads) k_dot_part(const float *x, const float *y, long n, double *part) {
  __shared__ double red[kDotThreads];
  double acc = 0.0;
  for (long i = (long)blockIdx.x * kDotThreads + threadIdx.x; i < n; i += (long)kDotBlocks * kDotThreads)
    acc += (double)x[i] * (double)y[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = kDotThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// *out = sum of the partials in a fixed tree order (one workgroup)
__global__ void __launch_bounds__(kDotThreads) k_dot_final(const double *part, double *out) {
  __shared__ double red[kDotThreads];
  double acc = 0.0;
  for (int i = threadIdx.x; i < kDotBlocks; i += kDotThreads) acc += part[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = kDotThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// p += alpha s;  r -= alpha q
__global__ void k_cg_step(float *p, float *r, const float *s, const float *q, float alpha, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    p[i] = fmaf(alpha, s[i], p[i]);
    r[i] = fmaf(-alpha, q[i], r[i]);
  }
}

// s = r + beta s
__global__ void k_cg_dir(float *s, const float *r, float beta, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    s[i] = fmaf(beta, s[i], r[i]);
}

// q[h] += e2d2[h] * s[h] for each offset plane h (plane = nx nz cells)
__global__ void k_add_diag(float *q, const float *s, const float *e2d2, long plane, int nh) {
  const long n = plane * nh;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    q[i] = fmaf(e2d2[i / plane], s[i], q[i]);
}

static unsigned stream_blocks(long n) {
  const long b = (n + 255) / 256;
  return (unsigned)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

hipError_t launch_sub(const float *a, const float *b, float *out, long n, hipStream_t st) {
  k_sub<<<stream_blocks(n), 256, 0, st>>>(a, b, out, n);
  return hipGetLastError();
}

hipError_t launch_dot(const float *x, const float *y, long n, double *part, double *out, hipStream_t st) {
  k_dot_part<<<kDotBlocks, kDotThreads, 0, st>>>(x, y, n, part);
  k_dot_final<<<1, kDotThreads, 0, st>>>(part, out);
  return hipGetLastError();
}

int dot_partials() { return kDotBlocks; }

hipError_t launch_cg_step(float *p, float *r, const float *s, const float *q, float alpha, long n, hipStream_t st) {
  k_cg_step<<<stream_blocks(n), 256, 0, st>>>(p, r, s, q, alpha, n);
  return hipGetLastError();
}

hipError_t launch_cg_dir(float *s, const float *r, float beta, long n, hipStream_t st) {
  k_cg_dir<<<stream_blocks(n), 256, 0, st>>>(s, r, beta, n);
  return hipGetLastError();
}

hipError_t launch_add_diag(float *q, const float *s, const float *e2d2, long plane, int nh, hipStream_t st) {
  k_add_diag<<<stream_blocks(plane * nh), 256, 0, st>>>(q, s, e2d2, plane, nh);
  return hipGetLastError();
}

// y = a x + b y (x may alias y)
__global__ void k_axpby(const float *x, float a, float *y, float b, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = fmaf(a, x[i], b * y[i]);
}

hipError_t launch_axpby(const float *x, float a, float *y, float b, long n, hipStream_t st) {
  k_axpby<<<stream_blocks(n), 256, 0, st>>>(x, a, y, b, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// L-BFGS direction from inner products.  The two-loop recursion only ever
// needs the inner products of its vectors s_i, y_i and g, so one pass forms
// them all, the recursion runs on numbers on the host, and a second pass forms
// the direction as one linear combination: two launches and one
// synchronization, where the recursion on the vectors took 3 k + 1 dots, each
// two launches, a copy and a synchronization (5 pairs of 5985: 330 us, nothing
// but round trips).
// ---------------------------------------------------------------------------
// Inner products of rows s_0 .. s_{k-1}, y_0 .. y_{k-1} with columns y_0 ..
// y_{k-1}, g.  One wavefront per workgroup; blockIdx.y takes four rows and all
// columns, so an element of a column is read once for four products, and
// blockIdx.x a strided share of the elements.  The 64 sums of a lane are
// reduced over the wavefront by halving: each exchange adds half of them from
// the other half of the lanes, and lane l ends with the total of product
// [l / 16][l % 16], stored to out[(blockIdx.y gridDim.x + blockIdx.x) 64 + l]
// (host memory).  FP64, fixed order.
__global__ void __launch_bounds__(64) k_lbfgs_gram(const LbfgsVectors v, long n, double *out) {
  constexpr int C = kLbfgsGramPairs + 1;
  static_assert(C == 16, "four rows of sixteen products");
  const int lane = threadIdx.x;
  const int r0 = 4 * blockIdx.y;
  double acc[64];
#pragma unroll
  for (int i = 0; i < 64; ++i) acc[i] = 0.0;
  for (long e = (long)blockIdx.x * 64 + lane; e < n; e += (long)gridDim.x * 64) {
    float row[4], col[C];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = min(r0 + r, 2 * v.k - 1);            // rows past the last repeat it
      row[r] = q < v.k ? v.s[q][e] : v.y[q - v.k][e];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) col[c] = c < v.k ? v.y[min(c, kLbfgsGramPairs - 1)][e] : c == v.k ? v.g[e] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < C; ++c) acc[r * C + c] = fma((double)row[r], (double)col[c], acc[r * C + c]);
  }
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) {
    const bool up = lane & h;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const double keep = up ? acc[i + h] : acc[i], give = up ? acc[i] : acc[i + h];
      acc[i] = keep + __shfl_xor(give, h);
    }
  }
  out[((long)blockIdx.y * gridDim.x + blockIdx.x) * 64 + lane] = acc[0];
}

// d = cg g + sum_i cs[i] s_i + cy[i] y_i in FP64, rounded once (d may be g)
__global__ void __launch_bounds__(256) k_lbfgs_combine(const LbfgsVectors v, const LbfgsCoefs c, long n, float *d) {
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    double x = c.g * (double)v.g[e];
    for (int i = 0; i < v.k; ++i) x = fma(c.s[i], (double)v.s[i][e], fma(c.y[i], (double)v.y[i][e], x));
    d[e] = (float)x;
  }
}

int lbfgs_gram_blocks(int k, long n) {
  const long groups = (2 * k + 3) / 4;
  return (int)std::max(1L, std::min((n + 511) / 512, kLbfgsGramBlocks / groups));
}

hipError_t launch_lbfgs_gram(const LbfgsVectors &v, long n, double *out, hipStream_t st) {
  const dim3 grid((unsigned)lbfgs_gram_blocks(v.k, n), (unsigned)((2 * v.k + 3) / 4));
  k_lbfgs_gram<<<grid, 64, 0, st>>>(v, n, out);
  return hipGetLastError();
}

hipError_t launch_lbfgs_combine(const LbfgsVectors &v, const LbfgsCoefs &c, long n, float *d, hipStream_t st) {
  k_lbfgs_combine<<<stream_blocks(n), 256, 0, st>>>(v, c, n, d);
  return hipGetLastError();
}

}  // namespace fw
