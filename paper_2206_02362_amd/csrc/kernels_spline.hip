// Linear spline operator S and its adjoint S* (Section 2: the velocity model
// is held on a coarse spline grid and mapped onto the finite-difference grid
// by linear spline interpolation; gradients come back through S*).
//
// S is the tensor product of two 1D hat-function interpolations: the fine
// point at depth iz*dz lies in spline cell kz (node kz <= iz*dz < node kz+1,
// the last cell closed) with weight tz for node kz+1 and 1 - tz for node kz;
// likewise along x.  Per axis a table kernel finds every fine point's cell by
// binary search over the node coordinates (in FP64) and, for every node j,
// the first fine point whose cell is at least j.  The same tables, evaluated
// at the nodes of a finer spline grid, move a model to that grid.  Because the cell index never
// decreases along the axis, the fine points of cell j form the range
// [start[j], start[j+1]), so the adjoint is a deterministic gather: node j
// collects the points of cell j - 1 with weight t and those of cell j with
// weight 1 - t, in ascending order.
//
// Layouts: fine fields [nx][nz], node values [nxn][nzn], z fastest.  All
// kernels are bandwidth-bound streams; the node arrays are small and stay in
// cache.
#include "internal.h"

namespace fw {

static unsigned spline_blocks(long n) {
  const long b = (n + 255) / 256;
  return (unsigned)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

// cell[i], wt[i] for target points i = 0..nf-1 at coordinate pts[i], or at
// i*h without pts (the finite-difference grid); nn >= 2 nodes
__global__ void k_spline_axis(const double *nodes, int nn, const double *pts, int nf, double h, int *cell,
                              float *wt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nf) return;
  const double p = pts ? pts[i] : i * h;
  int lo = 0, hi = nn - 2;                     // the cell is in [lo, hi]
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (nodes[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  double t = (p - nodes[lo]) / (nodes[lo + 1] - nodes[lo]);
  t = fmin(fmax(t, 0.0), 1.0);
  cell[i] = lo;
  wt[i] = (float)t;
}

// start[j] = first fine point whose cell is >= j, for j = 0..nn
__global__ void k_spline_starts(const int *cell, int nf, int nn, int *start) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j > nn) return;
  int lo = 0, hi = nf;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (cell[mid] >= j) hi = mid;
    else lo = mid + 1;
  }
  start[j] = lo;
}

// out[ix][iz] = sum over the four surrounding nodes of their bilinear weights
__global__ void k_spline_apply(const float *__restrict__ mc, int nzn, const int *__restrict__ cz,
                               const float *__restrict__ tz, const int *__restrict__ cx,
                               const float *__restrict__ tx, int nz, long n, float *__restrict__ out) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int ix = (int)(i / nz), iz = (int)(i - (long)ix * nz);
    const int kz = cz[iz], kx = cx[ix];
    const float wz = tz[iz], wx = tx[ix];
    const float *m0 = mc + (long)kx * nzn + kz;
    const float *m1 = m0 + nzn;
    const float a = (1.0f - wz) * m0[0] + wz * m0[1];
    const float b = (1.0f - wz) * m1[0] + wz * m1[1];
    out[i] = (1.0f - wx) * a + wx * b;
  }
}

// tmp[ix][jz] = sum over fine iz of A_z[iz][jz] f[ix][iz]
__global__ void k_spline_adj_z(const float *__restrict__ f, int nz, const float *__restrict__ tz,
                               const int *__restrict__ sz, int nzn, long n, float *__restrict__ tmp) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int ix = (int)(i / nzn), jz = (int)(i - (long)ix * nzn);
    const float *row = f + (long)ix * nz;
    float acc = 0.0f;
    if (jz > 0)
      for (int iz = sz[jz - 1]; iz < sz[jz]; ++iz) acc += tz[iz] * row[iz];
    for (int iz = sz[jz]; iz < sz[jz + 1]; ++iz) acc += (1.0f - tz[iz]) * row[iz];
    tmp[i] = acc;
  }
}

// out[jx][jz] = sum over fine ix of A_x[ix][jx] tmp[ix][jz]
__global__ void k_spline_adj_x(const float *__restrict__ tmp, int nzn, const float *__restrict__ tx,
                               const int *__restrict__ sx, long n, float *__restrict__ out) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int jx = (int)(i / nzn), jz = (int)(i - (long)jx * nzn);
    float acc = 0.0f;
    if (jx > 0)
      for (int ix = sx[jx - 1]; ix < sx[jx]; ++ix) acc += tx[ix] * tmp[(long)ix * nzn + jz];
    for (int ix = sx[jx]; ix < sx[jx + 1]; ++ix) acc += (1.0f - tx[ix]) * tmp[(long)ix * nzn + jz];
    out[i] = acc;
  }
}

hipError_t launch_spline_tables(const double *nodes, int nn, const double *pts, int nf, double h, int *cell,
                                float *wt, int *start, hipStream_t st) {
  k_spline_axis<<<(nf + 255) / 256, 256, 0, st>>>(nodes, nn, pts, nf, h, cell, wt);
  k_spline_starts<<<(nn + 1 + 255) / 256, 256, 0, st>>>(cell, nf, nn, start);
  return hipGetLastError();
}

hipError_t launch_spline_apply(const float *mc, int nzn, const int *cz, const float *tz, const int *cx,
                               const float *tx, int nz, int nx, float *out, hipStream_t st) {
  const long n = (long)nx * nz;
  k_spline_apply<<<spline_blocks(n), 256, 0, st>>>(mc, nzn, cz, tz, cx, tx, nz, n, out);
  return hipGetLastError();
}

hipError_t launch_spline_adjoint(const float *f, int nz, int nx, const float *tz, const int *sz, int nzn,
                                 const float *tx, const int *sx, int nxn, float *tmp, float *out, hipStream_t st) {
  const long n1 = (long)nx * nzn, n2 = (long)nxn * nzn;
  k_spline_adj_z<<<spline_blocks(n1), 256, 0, st>>>(f, nz, tz, sz, nzn, n1, tmp);
  k_spline_adj_x<<<spline_blocks(n2), 256, 0, st>>>(tmp, nzn, tx, sx, n2, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// S and S* in one launch each, for node sets that fit the kernel arguments.
// At the size of an inversion (35 x 171 nodes on 300 x 1700) both operators
// move 2 MB, 0.4 us at the copy rate, and a call was all round trips: two node
// uploads, two synchronizations, four table launches and up to two more (49
// us).  Here the node coordinates travel with the launch and every workgroup
// forms the part of the tables it needs in LDS, so a call is one launch: what
// bounds it is that launch and, inside it, one chain of memory reads.
// ---------------------------------------------------------------------------
// cell of coordinate p (last node at or before it, at most nn - 2), as in
// k_spline_axis
__device__ __forceinline__ int spline_cell(const double *nodes, int nn, double p) {
  int lo = 0, hi = nn - 2;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (nodes[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ float spline_weight(const double *nodes, int cell, double p) {
  const double t = (p - nodes[cell]) / (nodes[cell + 1] - nodes[cell]);
  return (float)fmin(fmax(t, 0.0), 1.0);
}
// first of the nf fine points whose cell is at least j, as in k_spline_starts
__device__ __forceinline__ int spline_start(const double *nodes, int nn, int nf, double h, int j) {
  if (j <= 0) return 0;
  if (j > nn - 2) return nf;
  int lo = 0, hi = nf;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (nodes[j] <= mid * h) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// out[ix][iz] for the workgroup's kSplineCols columns
__global__ void __launch_bounds__(256) k_spline_apply1(const SplineNodes s, int nz, int nx, double dz, double dx,
                                                       const float *__restrict__ mc, float *__restrict__ out) {
  __shared__ double nodes[kSplineNodes];
  __shared__ int cz[kSplineRows];
  __shared__ float tz[kSplineRows];
  for (int i = threadIdx.x; i < s.nzn + s.nxn; i += 256) nodes[i] = s.n[i];
  __syncthreads();
  for (int i = threadIdx.x; i < nz; i += 256) {
    cz[i] = spline_cell(nodes, s.nzn, i * dz);
    tz[i] = spline_weight(nodes, cz[i], i * dz);
  }
  __syncthreads();
  const int x0 = blockIdx.x * kSplineCols, x1 = min(nx, x0 + kSplineCols);
  for (int ix = x0; ix < x1; ++ix) {
    const int kx = spline_cell(nodes + s.nzn, s.nxn, ix * dx);
    const float wx = spline_weight(nodes + s.nzn, kx, ix * dx);
    for (int iz = threadIdx.x; iz < nz; iz += 256) {
      const float wz = tz[iz];
      const float *m0 = mc + (long)kx * s.nzn + cz[iz];
      const float *m1 = m0 + s.nzn;
      const float a = (1.0f - wz) * m0[0] + wz * m0[1];
      const float b = (1.0f - wz) * m1[0] + wz * m1[1];
      out[(long)ix * nz + iz] = (1.0f - wx) * a + wx * b;
    }
  }
}

// out[jx][jz] for one node column jx: the fine columns of its two cells go
// through the z gather into LDS, as many at a time as fit, and thread jz adds
// them in ascending order (k_spline_adj_z and k_spline_adj_x in one)
__global__ void __launch_bounds__(256) k_spline_adjoint1(const SplineNodes s, int nz, int nx, double dz, double dx,
                                                         const float *__restrict__ f, float *__restrict__ out) {
  __shared__ double nodes[kSplineNodes];
  __shared__ float tz[kSplineRows];
  __shared__ int sz[kSplineNodes + 1];
  __shared__ float tmp[kSplineTmp];
  const int jx = blockIdx.x, nzn = s.nzn;
  for (int i = threadIdx.x; i < nzn + s.nxn; i += 256) nodes[i] = s.n[i];
  __syncthreads();
  const double *xn = nodes + nzn;
  for (int i = threadIdx.x; i < nz; i += 256) tz[i] = spline_weight(nodes, spline_cell(nodes, nzn, i * dz), i * dz);
  for (int j = threadIdx.x; j <= nzn; j += 256) sz[j] = spline_start(nodes, nzn, nz, dz, j);
  const int xa = jx > 0 ? spline_start(xn, s.nxn, nx, dx, jx - 1) : 0;   // cell jx - 1: weight t
  const int xm = spline_start(xn, s.nxn, nx, dx, jx);                    // cell jx: weight 1 - t
  const int xe = spline_start(xn, s.nxn, nx, dx, jx + 1);
  const int cols = kSplineTmp / nzn;                  // fine columns at a time
  float acc[(kSplineNodes + 255) / 256];
#pragma unroll
  for (int q = 0; q < (kSplineNodes + 255) / 256; ++q) acc[q] = 0.0f;
  for (int xc = jx > 0 ? xa : xm; xc < xe; xc += cols) {
    const int n = min(cols, xe - xc);
    __syncthreads();                                  // tables ready; the last columns are read
    for (int p = threadIdx.x; p < n * nzn; p += 256) {
      const int c = p / nzn, jz = p - c * nzn;
      const float *row = f + (long)(xc + c) * nz;
      float a = 0.0f;
      if (jz > 0)
        for (int iz = sz[jz - 1]; iz < sz[jz]; ++iz) a += tz[iz] * row[iz];
      for (int iz = sz[jz]; iz < sz[jz + 1]; ++iz) a += (1.0f - tz[iz]) * row[iz];
      tmp[p] = a;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < (kSplineNodes + 255) / 256; ++q) {
      const int jz = threadIdx.x + 256 * q;
      if (jz >= nzn) break;
      for (int c = 0; c < n; ++c) {
        const int ix = xc + c;
        const float t = spline_weight(xn, ix < xm ? jx - 1 : min(jx, s.nxn - 2), ix * dx);
        acc[q] += (ix < xm ? t : 1.0f - t) * tmp[c * nzn + jz];
      }
    }
  }
#pragma unroll
  for (int q = 0; q < (kSplineNodes + 255) / 256; ++q)
    if (threadIdx.x + 256 * q < nzn) out[(long)jx * nzn + threadIdx.x + 256 * q] = acc[q];
}

hipError_t launch_spline_apply1(const SplineNodes &s, int nz, int nx, double dz, double dx, const float *mc,
                                float *out, hipStream_t st) {
  k_spline_apply1<<<(nx + kSplineCols - 1) / kSplineCols, 256, 0, st>>>(s, nz, nx, dz, dx, mc, out);
  return hipGetLastError();
}

hipError_t launch_spline_adjoint1(const SplineNodes &s, int nz, int nx, double dz, double dx, const float *f,
                                  float *out, hipStream_t st) {
  k_spline_adjoint1<<<s.nxn, 256, 0, st>>>(s, nz, nx, dz, dx, f, out);
  return hipGetLastError();
}

}  // namespace fw
