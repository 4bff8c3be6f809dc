// Restarted GMRES(m) on the device (right preconditioning), for nonsymmetric operators.
//
// Fig. 4 compares GMRES with CG and BiCGStab on the assembled system.  One Arnoldi
// step here: the Givens rotations of the step before, v_j = w / h_{j,j-1} and z = M^-1 v_j (one
// launch), w = A z (the library's operator), then classical Gram-Schmidt run twice (the second
// pass restores the orthogonality that one classical pass loses in floating point) in three
// launches: the dots of pass 1; w -= V c_1 with the dots of pass 2, which need only the lane's own
// new entries of w; w -= V c_2 with ||w||^2.  Every workgroup sums the partials of the launch
// before by itself, so nothing waits for a reduction launch (four launches a step and the operator
// in place of nine; with 15 vectors at 32^3 FP64 27 us of launches in place of 50).  All dot products are FP64 and summed in a fixed order.
// Iteration kernels return at once after a stop; the cycle-end kernels (triangular solve,
// x += M^-1 V y) always run.

#include <cmath>

#include "fe_internal.hpp"
#include "fe_device.hpp"

namespace fe {

namespace {

constexpr int KB = 256;  // threads per workgroup of every GMRES kernel

// Sum of part[0..np) by the whole workgroup, in fixed order; valid in every lane.
__device__ double group_sum(const double* part, int np, double* sh) {
  double v = 0;
  for (int i = threadIdx.x; i < np; i += KB) v += part[i];
  v = wave_sum_last(v);
  __syncthreads();
  if ((threadIdx.x & 63) == WAVE_LAST) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0;
#pragma unroll
  for (int w = 0; w < KB / 64; ++w) t += sh[w];
  __syncthreads();
  return t;
}

__device__ __forceinline__ bool is_finite(double v) { return v == v && v - v == 0.0; }

// z = M^-1 r for the three dofs of one node: node-block inverse (blk = 1; 6 words per
// node: xx, yy, zz, yz, xz, xy) or inverted point diagonal (blk = 0); blk = 2 (ILU(0),
// applied by its own sweeps afterwards) copies r.
template <typename T>
__device__ __forceinline__ void precond_node(const T* M, int blk, int64_t node, const T r[3], T z[3]) {
  if (blk == 2) {
#pragma unroll
    for (int c = 0; c < 3; ++c) z[c] = r[c];
  } else if (blk) {
    const T* m = M + 6 * node;
    z[0] = m[0] * r[0] + m[5] * r[1] + m[4] * r[2];
    z[1] = m[5] * r[0] + m[1] * r[1] + m[3] * r[2];
    z[2] = m[4] * r[0] + m[3] * r[1] + m[2] * r[2];
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c) z[c] = M[3 * node + c] * r[c];
  }
}

// x = 0, w = b, point diagonal inverted in place; controls reset.
template <typename T>
__global__ __launch_bounds__(KB) void gm_setup_kernel(int64_t n, const T* b, T* x, T* w, T* dinv, int blk,
                                                      GmresDev* dev, double rtol, int max_it, int m) {
  for (int64_t i = (int64_t)blockIdx.x * KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
    x[i] = 0;
    w[i] = b[i];
    if (!blk) dinv[i] = T(1) / dinv[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    GmresCtrl& c = dev->ctrl;
    c.rtol = rtol;
    c.tol = 0;
    c.bb = -1;  // set by the first cycle start
    c.res_est = 0;
    c.status = CG_RUNNING;
    c.iters = 0;
    c.max_it = max_it;
    c.k = 0;
    c.m = m;
    c.cycles = 0;
  }
}

// part[blockIdx] = this workgroup's share of (v, w).
template <typename T>
__global__ __launch_bounds__(KB) void gm_dot_kernel(int64_t n, const T* v, const T* w, double* part, const int* stop) {
  if (stop && *stop) return;
  __shared__ double sh[KB / 64];
  double acc = 0;
  for (int64_t d = (int64_t)blockIdx.x * KB + threadIdx.x; d < n; d += (int64_t)gridDim.x * KB)
    acc += (double)v[d] * (double)w[d];
  acc = wave_sum_last(acc);
  if ((threadIdx.x & 63) == WAVE_LAST) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0;
#pragma unroll
    for (int q = 0; q < KB / 64; ++q) t += sh[q];
    part[blockIdx.x] = t;
  }
}

// One launch of the Gram-Schmidt of step j over nv vectors:
//   PASS 0: the dots c_1 = V^T w                            -> part_out
//   PASS 1: w -= V c_1, then the dots c_2 = V^T w           -> part_out
//   PASS 2: w -= V c_2, then ||w||^2                        -> part_out
// c comes from the np partials per vector of the launch before, summed in a fixed order by every
// workgroup (16 lanes per vector).  A lane's entries of up to GT vectors are requested before that
// and stay in registers for both the update and the dots: V is read once a launch, and its latency
// hides behind the sums.  Workgroup 0 records the Hessenberg entries (pass 2 adds the
// re-orthogonalisation coefficients).
constexpr int GB = 512;  // lanes: one dof each up to 512 workgroups, then a loop
constexpr int GT = 32;   // vectors held in registers

template <typename T, int PASS>
__global__ __launch_bounds__(GB) void gm_pass_kernel(int64_t n, const T* __restrict__ V, int nv, T* w, GmresDev* dev,
                                                     int j, const double* part_in, int np, double* part_out,
                                                     const int* stop) {
  __shared__ double cs[GM_MAXM + GT + 1];
  __shared__ double sh[GM_MAXM + 1][GB / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int stopped = *stop;
  const int nt = min(nv, GT);
  T v[GT];
  auto request = [&](int64_t d, bool in, int i0, int cnt) {  // entries d of V_{i0} .. V_{i0 + cnt - 1}
#pragma unroll
    for (int b = 0; b < GT; b += 8) {
      if (b < cnt) {  // (uniform: whole groups of 8; past the end the last vector is read again, with c = 0)
#pragma unroll
        for (int u = 0; u < 8; ++u) v[b + u] = in ? V[(int64_t)(i0 + min(b + u, cnt - 1)) * n + d] : T(0);
      }
    }
  };
  int64_t d = (int64_t)blockIdx.x * GB + tid;
  request(d, d < n, 0, nt);
  double wd = d < n ? (double)w[d] : 0.0;
  if (stopped) return;
  if (PASS > 0) {
    for (int i = tid; i < GM_MAXM + GT + 1; i += GB)
      if (i >= nv) cs[i] = 0.0;
    for (int i = tid >> 4; i < nv; i += GB / 16) {
      double c = 0;
#pragma unroll 4
      for (int q = tid & 15; q < np; q += 16) c += part_in[(int64_t)i * np + q];
      c = dpp_add<0x111, 0xf>(c);  // row_shr 1, 2, 4, 8: the 16 lanes' sum in the last of them
      c = dpp_add<0x112, 0xf>(c);
      c = dpp_add<0x114, 0xf>(c);
      c = dpp_add<0x118, 0xf>(c);
      if ((tid & 15) == 15) cs[i] = c;
    }
    __syncthreads();
    if (blockIdx.x == 0)
      for (int i = tid; i < nv; i += GB) dev->H[j][i] = PASS == 1 ? cs[i] : dev->H[j][i] + cs[i];
  }
  double acc[GT], nrm = 0;
#pragma unroll
  for (int u = 0; u < GT; ++u) acc[u] = 0;
  bool first = true;
  for (; d - tid < n; d += (int64_t)gridDim.x * GB) {
    const bool in = d < n;
    if (!first) {
      request(d, in, 0, nt);
      wd = in ? (double)w[d] : 0.0;
    }
    first = false;
    if (PASS > 0) {
      double t = wd;
#pragma unroll
      for (int b = 0; b < GT; b += 8)
        if (b < nt)
#pragma unroll
          for (int u = 0; u < 8; ++u) t -= cs[b + u] * (double)v[b + u];
      for (int i = GT; i < nv; ++i) t -= cs[i] * (double)(in ? V[(int64_t)i * n + d] : T(0));
      const T tv = T(t);
      if (in) w[d] = tv;
      wd = (double)tv;
      if (PASS == 2) nrm += wd * wd;
    }
    if (PASS < 2)
#pragma unroll
      for (int b = 0; b < GT; b += 8)
        if (b < nt)
#pragma unroll
          for (int u = 0; u < 8; ++u) acc[b + u] += (double)v[b + u] * wd;
  }
  if (PASS == 2) {
    nrm = wave_sum_last(nrm);
    if (lane == WAVE_LAST) sh[0][wave] = nrm;
    __syncthreads();
    if (tid == 0) {
      double t = 0;
#pragma unroll
      for (int q = 0; q < GB / 64; ++q) t += sh[0][q];
      part_out[blockIdx.x] = t;
    }
    return;
  }
#pragma unroll
  for (int b = 0; b < GT; b += 8)
    if (b < nt)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double t = wave_sum_last(acc[b + u]);
        if (lane == WAVE_LAST) sh[b + u][wave] = t;
      }
  for (int i0 = GT; i0 < nv; i0 += GT) {  // longer restarts: the other vectors, w from memory (own entries)
    const int cnt = min(nv - i0, GT);
#pragma unroll
    for (int u = 0; u < GT; ++u) acc[u] = 0;
    for (d = (int64_t)blockIdx.x * GB + tid; d - tid < n; d += (int64_t)gridDim.x * GB) {
      const bool in = d < n;
      request(d, in, i0, cnt);
      const double x = in ? (double)w[d] : 0.0;
#pragma unroll
      for (int b = 0; b < GT; b += 8)
        if (b < cnt)
#pragma unroll
          for (int u = 0; u < 8; ++u) acc[b + u] += (double)v[b + u] * x;
    }
#pragma unroll
    for (int b = 0; b < GT; b += 8)
      if (b < cnt)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const double t = wave_sum_last(acc[b + u]);
          if (lane == WAVE_LAST && b + u < cnt) sh[i0 + b + u][wave] = t;
        }
  }
  __syncthreads();
  for (int i = tid; i < nv; i += GB) {
    double t = 0;
#pragma unroll
    for (int q = 0; q < GB / 64; ++q) t += sh[i][q];
    part_out[(int64_t)i * gridDim.x + blockIdx.x] = t;
  }
}

// Start of a cycle (one workgroup): beta = ||r|| from the partials of the residual in w;
// g = beta e_1; the first cycle also sets ||b|| and the tolerance.
__global__ __launch_bounds__(KB) void gm_beta_kernel(const double* part, int np, GmresDev* dev) {
  __shared__ double sh[KB / 64];
  GmresCtrl& c = dev->ctrl;
  if (c.status) return;
  const double beta = std::sqrt(group_sum(part, np, sh));
  if (threadIdx.x != 0) return;
  if (c.bb < 0) {
    c.bb = beta * beta;
    c.tol = c.rtol * beta;
  }
  c.k = 0;
  c.cycles += 1;
  c.res_est = beta;
  for (int i = 0; i <= c.m; ++i) dev->g[i] = 0;
  dev->g[0] = beta;
  if (!is_finite(beta)) {
    c.status = FE_ERR_NONFINITE;
  } else if (beta <= c.tol) {
    c.status = CG_CONVERGED;
  } else if (c.iters >= c.max_it) {
    c.status = FE_ERR_NOT_CONVERGED;
  }
}

// End of Arnoldi step j (one lane): h_{j+1,j} = ||w||, rotations on column j, new rotation, g
// update, stopping tests.
__device__ void givens_step(GmresDev* dev, int j, double hn) {
  GmresCtrl& c = dev->ctrl;
  double* h = dev->H[j];
  h[j + 1] = hn;
  if (!is_finite(hn)) {
    c.status = FE_ERR_NONFINITE;
    return;
  }
  double t = h[0];  // the running entry of the column stays in a register
  for (int i = 0; i < j; ++i) {
    const double a = dev->cs[i], b = dev->sn[i], hi = h[i + 1];
    h[i] = a * t + b * hi;
    t = -b * t + a * hi;
  }
  const double rho = std::hypot(t, hn);
  if (rho == 0.0) {
    c.status = FE_ERR_BREAKDOWN;
    return;
  }
  const double cj = t / rho, sj = hn / rho, gj = dev->g[j];
  dev->cs[j] = cj;
  dev->sn[j] = sj;
  h[j] = rho;
  h[j + 1] = 0.0;
  dev->g[j + 1] = -sj * gj;
  dev->g[j] = cj * gj;
  const int iters = c.iters + 1;
  c.iters = iters;
  c.k = j + 1;
  const double res = std::fabs(sj * gj);
  c.res_est = res;
  if (res <= c.tol) c.status = CG_CONVERGED;
  else if (iters >= c.max_it) c.status = FE_ERR_NOT_CONVERGED;
}

__global__ __launch_bounds__(KB) void gm_givens_kernel(const double* part, int np, GmresDev* dev, int j,
                                                       const int* stop) {
  __shared__ double sh[KB / 64];
  if (stop && *stop) return;
  const double hn = std::sqrt(group_sum(part, np, sh));
  if (threadIdx.x == 0) givens_step(dev, j, hn);
}

// v_j = w / ||w|| (stored as basis vector j) and z = M^-1 v_j, one node per lane; w is
// cleared for the operator, which adds its face contributions atomically.  ||w|| is summed from
// the np partials of the launch before; with givens, workgroup 0 first closes Arnoldi step j - 1
// (a stop found there takes effect at the next launch: this one only fills vectors that a stopped
// cycle does not read).
template <typename T>
__global__ __launch_bounds__(KB) void gm_basis_kernel(int64_t n_nodes, T* w, T* vj, T* z, const T* M, int blk,
                                                      const double* part, int np, GmresDev* dev, int j, int givens,
                                                      const int* stop) {
  __shared__ double sh[KB / 64];
  if (*stop) return;
  const double hn = std::sqrt(group_sum(part, np, sh));
  if (givens && blockIdx.x == 0 && threadIdx.x == 0) givens_step(dev, j - 1, hn);
  const T s = T(1.0 / hn);
  for (int64_t nd = (int64_t)blockIdx.x * KB + threadIdx.x; nd < n_nodes; nd += (int64_t)gridDim.x * KB) {
    T v[3], zz[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      v[c] = w[3 * nd + c] * s;
      vj[3 * nd + c] = v[c];
      w[3 * nd + c] = 0;
    }
    precond_node(M, blk, nd, v, zz);
#pragma unroll
    for (int c = 0; c < 3; ++c) z[3 * nd + c] = zz[c];
  }
}

// y = R^-1 g over the k finished columns (one wave; k <= GM_MAXM = 64: lane i holds entry i, column
// by column from the last).
__global__ __launch_bounds__(64) void gm_solve_kernel(GmresDev* dev) {
  static_assert(GM_MAXM <= 64, "one lane per entry");
  const int k = dev->ctrl.k, i = threadIdx.x;
  double g = i < k ? dev->g[i] : 0.0;
  const double d = i < k ? dev->H[i][i] : 1.0;
  for (int q = k - 1; q >= 0; --q) {
    const double h = i < q ? dev->H[q][i] : 0.0;
    const double yq = __shfl(g / d, q, 64);
    if (i == q) g = yq;
    else g -= h * yq;
  }
  if (i < k) dev->y[i] = g;
}

// x += M^-1 (sum_{i<k} y_i V_i), one node per lane (blk = 2: t = sum_i y_i V_i goes to
// tz instead, for the ILU sweeps and GM_ADD_Z); w is cleared for the operator application
// that starts the next cycle.
template <typename T>
__global__ __launch_bounds__(KB) void gm_combine_kernel(int64_t n_nodes, const T* V, int64_t n, T* x, T* w,
                                                        T* tz, const T* M, int blk, const GmresDev* dev) {
  __shared__ double ys[GM_MAXM];
  const int k = dev->ctrl.k;
  for (int i = threadIdx.x; i < k; i += KB) ys[i] = dev->y[i];
  __syncthreads();
  for (int64_t nd = (int64_t)blockIdx.x * KB + threadIdx.x; nd < n_nodes; nd += (int64_t)gridDim.x * KB) {
    T t[3], z[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) w[3 * nd + c] = 0;
    if (k == 0) continue;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double a = 0;
      for (int i = 0; i < k; ++i) a += ys[i] * (double)V[(int64_t)i * n + 3 * nd + c];
      t[c] = T(a);
    }
    if (blk == 2) {
#pragma unroll
      for (int c = 0; c < 3; ++c) tz[3 * nd + c] = t[c];
      continue;
    }
    precond_node(M, blk, nd, t, z);
#pragma unroll
    for (int c = 0; c < 3; ++c) x[3 * nd + c] += z[c];
  }
}

// x += z
template <typename T>
__global__ __launch_bounds__(KB) void gm_add_kernel(int64_t n, const T* z, T* x) {
  for (int64_t d = (int64_t)blockIdx.x * KB + threadIdx.x; d < n; d += (int64_t)gridDim.x * KB) x[d] += z[d];
}

// w = b - w (w holds A x) and partial ||w||^2 for the next cycle start.
template <typename T>
__global__ __launch_bounds__(KB) void gm_residual_kernel(int64_t n, const T* b, T* w, double* part) {
  __shared__ double sh[KB / 64];
  double nrm = 0;
  for (int64_t d = (int64_t)blockIdx.x * KB + threadIdx.x; d < n; d += (int64_t)gridDim.x * KB) {
    const T t = b[d] - w[d];
    w[d] = t;
    nrm += (double)t * (double)t;
  }
  nrm = wave_sum_last(nrm);
  if ((threadIdx.x & 63) == WAVE_LAST) sh[threadIdx.x >> 6] = nrm;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0;
#pragma unroll
    for (int q = 0; q < KB / 64; ++q) t += sh[q];
    part[blockIdx.x] = t;
  }
}

template <typename T> T* basis(const fe_problem* p, int i) { return static_cast<T*>(p->w_gm) + (int64_t)i * p->n_dof; }
template <typename T> T* work_w(const fe_problem* p) { return basis<T>(p, p->gm_cap + 1); }
template <typename T> T* work_z(const fe_problem* p) { return basis<T>(p, p->gm_cap + 2); }

// Workgroups of the Gram-Schmidt launches (each of them sums all partials of the one before).
int gs_grid(const fe_problem* p) { return (int)std::max<int64_t>(1, std::min<int64_t>((p->n_dof + GB - 1) / GB, GM_GRID)); }

int node_grid(const fe_problem* p) {
  return (int)std::min<int64_t>((p->n_nodes + KB - 1) / KB, 4 * GM_GRID);
}

template <typename T>
hipError_t gm_step_t(const fe_problem* p, int stage, int j, const void* b, void* x, hipStream_t s, int open_step) {
  const int64_t n = p->n_dof;
  const int* stop = &p->gm_dev->ctrl.status;
  const T* M = static_cast<const T*>(pc_buffer(p));
  switch (stage) {
    case GM_BASIS:  // ||w|| and, after the cycle's first step, the rotations of step j - 1 if still open
      hipLaunchKernelGGL(gm_basis_kernel<T>, dim3(node_grid(p)), dim3(KB), 0, s, p->n_nodes, work_w<T>(p),
                         basis<T>(p, j), work_z<T>(p), M, p->precond, p->gm_part, j == 0 ? GM_GRID : gs_grid(p),
                         p->gm_dev, j, open_step, stop);
      break;
    case GM_ORTHO: {  // two classical Gram-Schmidt passes, then ||w||^2
      const int G = gs_grid(p);
      double* part2 = p->gm_part + (int64_t)(GM_MAXM + 1) * GM_GRID;
      const T* V = basis<T>(p, 0);
      T* w = work_w<T>(p);
      hipLaunchKernelGGL((gm_pass_kernel<T, 0>), dim3(G), dim3(GB), 0, s, n, V, j + 1, w, p->gm_dev, j,
                         (const double*)nullptr, 0, p->gm_part, stop);
      hipLaunchKernelGGL((gm_pass_kernel<T, 1>), dim3(G), dim3(GB), 0, s, n, V, j + 1, w, p->gm_dev, j,
                         (const double*)p->gm_part, G, part2, stop);
      hipLaunchKernelGGL((gm_pass_kernel<T, 2>), dim3(G), dim3(GB), 0, s, n, V, j + 1, w, p->gm_dev, j,
                         (const double*)part2, G, p->gm_part, stop);
      break;
    }
    case GM_GIVENS:  // closes step j where no basis launch follows at once
      hipLaunchKernelGGL(gm_givens_kernel, dim3(1), dim3(KB), 0, s, p->gm_part, gs_grid(p), p->gm_dev, j, stop);
      break;
    case GM_START:  // w holds the residual: ||w|| -> beta, g = beta e_1
      hipLaunchKernelGGL(gm_dot_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, work_w<T>(p), work_w<T>(p), p->gm_part,
                         (const int*)nullptr);
      hipLaunchKernelGGL(gm_beta_kernel, dim3(1), dim3(KB), 0, s, p->gm_part, GM_GRID, p->gm_dev);
      break;
    case GM_FINISH:  // cycle end: y = R^-1 g, x += M^-1 V y
      hipLaunchKernelGGL(gm_solve_kernel, dim3(1), dim3(64), 0, s, p->gm_dev);
      hipLaunchKernelGGL(gm_combine_kernel<T>, dim3(node_grid(p)), dim3(KB), 0, s, p->n_nodes, basis<T>(p, 0), n,
                         static_cast<T*>(x), work_w<T>(p), work_z<T>(p), M, p->precond, p->gm_dev);
      break;
    case GM_ADD_Z:  // x += z (after the ILU sweeps of the cycle-end combination)
      hipLaunchKernelGGL(gm_add_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, work_z<T>(p), static_cast<T*>(x));
      break;
    case GM_RESIDUAL:  // w = b - w (w = A x), then ||w||
      hipLaunchKernelGGL(gm_residual_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, static_cast<const T*>(b),
                         work_w<T>(p), p->gm_part);
      hipLaunchKernelGGL(gm_beta_kernel, dim3(1), dim3(KB), 0, s, p->gm_part, GM_GRID, p->gm_dev);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// z = M^-1 r with the point diagonal d (not inverted; blk = 0) or the inverted node blocks
// (blk = 1), one node per lane.
template <typename T>
__global__ __launch_bounds__(KB) void pc_apply_kernel(int64_t n_nodes, const T* M, int blk, const T* r, T* z) {
  for (int64_t nd = (int64_t)blockIdx.x * KB + threadIdx.x; nd < n_nodes; nd += (int64_t)gridDim.x * KB) {
    T v[3], w[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = r[3 * nd + c];
    if (blk) {
      precond_node(M, 1, nd, v, w);
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) w[c] = v[c] / M[3 * nd + c];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) z[3 * nd + c] = w[c];
  }
}

template <typename T>
hipError_t pc_apply_t(const fe_problem* p, const void* r, void* z, hipStream_t s) {
  hipLaunchKernelGGL(pc_apply_kernel<T>, dim3(node_grid(p)), dim3(KB), 0, s, p->n_nodes,
                     static_cast<const T*>(pc_buffer(p)), p->precond == FE_PC_BLOCK_JACOBI ? 1 : 0,
                     static_cast<const T*>(r), static_cast<T*>(z));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// CG with a preconditioner applied by separate launches (ILU(0)): Hestenes & Stiefel
// recursion with z = M^-1 r, FP64 dots in fixed order, device-resident scalars.

template <typename T>
__global__ __launch_bounds__(KB) void ipcg_init_kernel(int64_t n, const T* b, T* x, T* r, T* q, double* part,
                                                       IpcgCtrl* c, double rtol, int max_it) {
  __shared__ double sh[KB / 64];
  double v = 0;
  for (int64_t d = (int64_t)blockIdx.x * KB + threadIdx.x; d < n; d += (int64_t)gridDim.x * KB) {
    x[d] = 0;
    q[d] = 0;
    const T t = b[d];
    r[d] = t;
    v += (double)t * (double)t;
  }
  v = wave_sum_last(v);
  if ((threadIdx.x & 63) == WAVE_LAST) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0;
#pragma unroll
    for (int q = 0; q < KB / 64; ++q) t += sh[q];
    part[blockIdx.x] = t;
    if (blockIdx.x == 0) {
      c->rtol = rtol;
      c->max_it = max_it;
      c->iters = 0;
      c->status = CG_RUNNING;
      c->alpha = c->pq = 0;
      c->rzs[0] = c->rzs[1] = 0;
    }
  }
}

// ||r||^2 from the partials; the first call sets ||b|| and the tolerance, later calls
// count the finished iteration and test it.
__global__ __launch_bounds__(KB) void ipcg_check_kernel(const double* part, int np, IpcgCtrl* c, int first) {
  __shared__ double sh[KB / 64];
  if (c->status) return;
  const double rr = group_sum(part, np, sh);
  if (threadIdx.x != 0) return;
  c->rr = rr;
  if (!is_finite(rr)) {
    c->status = FE_ERR_NONFINITE;
    return;
  }
  if (first) {
    c->bb = rr;
    c->tol2 = c->rtol * c->rtol * rr;
    if (rr == 0.0) c->status = CG_CONVERGED;
    else if (c->max_it <= 0) c->status = FE_ERR_NOT_CONVERGED;
    return;
  }
  c->iters += 1;
  if (rr <= c->tol2) c->status = CG_CONVERGED;
  else if (c->iters >= c->max_it) c->status = FE_ERR_NOT_CONVERGED;
}

// p = z + beta p with beta = (r, z)_k / (r, z)_{k-1} (k = 0: p = z); every workgroup sums the
// (r, z) partials itself, workgroup 0 records them in slot k & 1.  q is cleared for the
// next operator application (the matrix-free operator adds into it).
template <typename T>
__global__ __launch_bounds__(KB) void ipcg_direction_kernel(int64_t n, const T* z, T* p, T* q, const double* part,
                                                            int np, IpcgCtrl* c, long k) {
  __shared__ double sh[KB / 64];
  if (c->status) return;
  const double rz = group_sum(part, np, sh);
  const double beta = k == 0 ? 0.0 : rz / c->rzs[(k - 1) & 1];
  if (!is_finite(rz) || !is_finite(beta)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) c->status = FE_ERR_NONFINITE;
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) c->rzs[k & 1] = rz;
  const T bt = T(beta);
  for (int64_t d = (int64_t)blockIdx.x * KB + threadIdx.x; d < n; d += (int64_t)gridDim.x * KB) {
    p[d] = k == 0 ? z[d] : z[d] + bt * p[d];
    q[d] = 0;
  }
}

// alpha = (r, z)_k / (p, A p) (every workgroup sums the partials itself), x += alpha p,
// r -= alpha q, partials of ||r||^2.
template <typename T>
__global__ __launch_bounds__(KB) void ipcg_update_kernel(int64_t n, const T* p, const T* q, T* x, T* r,
                                                         const double* part_pq, int np, IpcgCtrl* c, long k,
                                                         double* part_rr) {
  __shared__ double sh[KB / 64];
  if (c->status) return;
  const double pq = group_sum(part_pq, np, sh);
  if (!(pq > 0.0) || !is_finite(pq)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) c->status = is_finite(pq) ? FE_ERR_BREAKDOWN : FE_ERR_NONFINITE;
    return;
  }
  const double alpha = c->rzs[k & 1] / pq;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    c->alpha = alpha;
    c->pq = pq;
  }
  const T a = T(alpha);
  double v = 0;
  for (int64_t d = (int64_t)blockIdx.x * KB + threadIdx.x; d < n; d += (int64_t)gridDim.x * KB) {
    x[d] += a * p[d];
    const T t = r[d] - a * q[d];
    r[d] = t;
    v += (double)t * (double)t;
  }
  v = wave_sum_last(v);
  if ((threadIdx.x & 63) == WAVE_LAST) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0;
#pragma unroll
    for (int w = 0; w < KB / 64; ++w) t += sh[w];
    part_rr[blockIdx.x] = t;
  }
}

template <typename T> T* ipcg_v(const fe_problem* p, int v) {
  return static_cast<T*>(p->w_ipcg) + (int64_t)v * p->n_dof;
}

template <typename T>
hipError_t ipcg_step_t(const fe_problem* p, int stage, long k, const void* b, void* x, double rtol, int max_it,
                       hipStream_t s) {
  const int64_t n = p->n_dof;
  double* part_pq = p->gm_part;
  double* part_rr = p->gm_part + GM_GRID;
  double* part_rz = p->gm_part + 2 * GM_GRID;
  const int* stop = &p->ipcg->status;
  T* r = ipcg_v<T>(p, 0);
  T* pp = ipcg_v<T>(p, 1);
  T* q = ipcg_v<T>(p, 2);
  T* z = ipcg_v<T>(p, 3);
  switch (stage) {
    case IPCG_INIT:
      hipLaunchKernelGGL(ipcg_init_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, static_cast<const T*>(b),
                         static_cast<T*>(x), r, q, part_rr, p->ipcg, rtol, max_it);
      break;
    case IPCG_CHECK_FIRST:
    case IPCG_CHECK:
      hipLaunchKernelGGL(ipcg_check_kernel, dim3(1), dim3(KB), 0, s, part_rr, GM_GRID, p->ipcg,
                         stage == IPCG_CHECK_FIRST ? 1 : 0);
      break;
    case IPCG_FIRST_DIRECTION:  // (r, z) partials, then p = z
    case IPCG_DIRECTION:
      hipLaunchKernelGGL(gm_dot_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, r, z, part_rz, stop);
      hipLaunchKernelGGL(ipcg_direction_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, z, pp, q, part_rz, GM_GRID,
                         p->ipcg, stage == IPCG_FIRST_DIRECTION ? 0L : k);
      break;
    case IPCG_UPDATE:  // (p, q) partials, then the step
      hipLaunchKernelGGL(gm_dot_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, pp, q, part_pq, stop);
      hipLaunchKernelGGL(ipcg_update_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, n, pp, q, static_cast<T*>(x), r,
                         part_pq, GM_GRID, p->ipcg, k, part_rr);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t gm_setup_t(const fe_problem* p, const void* b, void* x, double rtol, int max_it, int m, hipStream_t s) {
  hipLaunchKernelGGL(gm_setup_kernel<T>, dim3(GM_GRID), dim3(KB), 0, s, p->n_dof, static_cast<const T*>(b),
                     static_cast<T*>(x), work_w<T>(p), static_cast<T*>(pc_buffer(p)), p->precond, p->gm_dev, rtol,
                     max_it, m);
  return hipGetLastError();
}

}  // namespace

hipError_t gm_setup(const fe_problem* p, const void* b, void* x, double rtol, int max_it, int m, hipStream_t s) {
  return p->prec == FE_F64 ? gm_setup_t<double>(p, b, x, rtol, max_it, m, s)
                           : gm_setup_t<float>(p, b, x, rtol, max_it, m, s);
}

hipError_t ipcg_step(const fe_problem* p, int stage, long k, const void* b, void* x, double rtol, int max_it,
                     hipStream_t s) {
  return p->prec == FE_F64 ? ipcg_step_t<double>(p, stage, k, b, x, rtol, max_it, s)
                           : ipcg_step_t<float>(p, stage, k, b, x, rtol, max_it, s);
}

void* ipcg_vec(const fe_problem* p, int v) {
  return static_cast<char*>(p->w_ipcg) + (size_t)v * p->n_dof * (p->prec == FE_F64 ? 8 : 4);
}

hipError_t pc_apply(const fe_problem* p, const void* r, void* z, hipStream_t s) {
  return p->prec == FE_F64 ? pc_apply_t<double>(p, r, z, s) : pc_apply_t<float>(p, r, z, s);
}

hipError_t gm_step(const fe_problem* p, int stage, int j, const void* b, void* x, hipStream_t s, int open_step) {
  return p->prec == FE_F64 ? gm_step_t<double>(p, stage, j, b, x, s, open_step)
                           : gm_step_t<float>(p, stage, j, b, x, s, open_step);
}

void* gm_work_w(const fe_problem* p) {
  return static_cast<char*>(p->w_gm) + (size_t)(p->gm_cap + 1) * p->n_dof * (p->prec == FE_F64 ? 8 : 4);
}

void* gm_work_z(const fe_problem* p) {
  return static_cast<char*>(p->w_gm) + (size_t)(p->gm_cap + 2) * p->n_dof * (p->prec == FE_F64 ? 8 : 4);
}

}  // namespace fe
