// HIP kernels of libfe for general hex8 meshes (fe_problem_create_hex8): any conforming mesh
// of 8-node bricks given by device coordinates [3][n_nodes] (kept as [n_nodes][3]) and
// connectivity [8][n_el].
//
// Element kernels run one lane per (element, Gauss point): a 256-lane workgroup holds 32
// elements x 8 points, the 8 lanes of an element sit side by side in one wave.
//   1. lane (e, p) stages node p of element e (coordinates and the gathered field) in LDS;
//   2. each lane forms the isoparametric Jacobian of its point from the 8 nodal positions,
//      its inverse, the physical basis gradients and the displacement gradient;
//   3. the constitutive law gives the stress, pushed back to the 8 nodes (w detJ B^T sigma);
//   4. the 8 lanes of an element sum their nodal forces by recursive halving (three lane
//      exchanges of 12, 6 and 3 values, no atomics), after which lane p holds node p's total
//      and adds it to the global vector with one hardware FP atomic per component, or, inside
//      the solvers, stores it for a gather by node (gen_gather_kernel, gen_cg_node_kernel).
//
// The sparse Jacobian follows the sort-and-combine assembly of the paper (Sec. III-B):
//   symbolic (once per mesh): every element contributes its 64 node pairs; pairs are
//   bucketed by row node (counting sort) and each row is sorted by (column node, element
//   code), so the whole list is ordered by the int64 key (row, column); runs of equal keys
//   are the duplicates, their first positions give the node-pair pattern, and the sorted
//   element codes of each run say which element blocks sum into that pair;
//   numeric (per tangent): each element's Jacobian K_e = sum_q B_q^T D_q B_q w detJ is symmetric,
//   so its 36 node-pair blocks a <= b are formed, and all 64 written to a per-element buffer; a
//   wave per node then sums every pair's run in sorted order into the CSR values (deterministic:
//   the same bits on every run).
#include "fe_internal.hpp"
#include "fe_device.hpp"

namespace fe {

constexpr int GBLOCK = 256;
constexpr int GEL = GBLOCK / 8;  // elements per element-kernel workgroup
constexpr double GAUSS = 0.57735026918962576451;  // 1/sqrt(3)

// Reference coordinates of local node a: (-1,-1,-1) (1,-1,-1) (1,1,-1) (-1,1,-1), then z = +1.
__device__ __forceinline__ int ref_sx(int a) { return (((a + 1) >> 1) & 1) ? 1 : -1; }
__device__ __forceinline__ int ref_sy(int a) { return (a & 2) ? 1 : -1; }
__device__ __forceinline__ int ref_sz(int a) { return (a & 4) ? 1 : -1; }

// dN_a / dxi_k of the trilinear basis at Gauss point q = qx + 2 qy + 4 qz (xi = +-1/sqrt 3).
template <typename T> __device__ __forceinline__ void node_ref_grad(int a, int q, T dn[3]) {
  const T g = T(GAUSS);
  const T xi = (q & 1) ? g : -g, eta = (q & 2) ? g : -g, zeta = (q & 4) ? g : -g;
  const T sx = T(ref_sx(a)), sy = T(ref_sy(a)), sz = T(ref_sz(a));
  const T fx = 1 + sx * xi, fy = 1 + sy * eta, fz = 1 + sz * zeta;
  dn[0] = T(0.125) * sx * fy * fz;
  dn[1] = T(0.125) * fx * sy * fz;
  dn[2] = T(0.125) * fx * fy * sz;
}
template <typename T> __device__ __forceinline__ void ref_grad(int q, T dn[8][3]) {
#pragma unroll
  for (int a = 0; a < 8; ++a) node_ref_grad<T>(a, q, dn[a]);
}

// Inverse of the isoparametric Jacobian J_ik = dx_i/dxi_k of the element with nodal positions
// xe[a][i] and reference gradients dn; returns det J.
template <typename T> __device__ __forceinline__ T jacobian_inverse(const T (*xe)[3], const T dn[8][3], T Ji[3][3]) {
  T J[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      T s = 0;
#pragma unroll
      for (int a = 0; a < 8; ++a) s += xe[a][i] * dn[a][k];
      J[i][k] = s;
    }
  const T c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1], c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2],
          c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  const T det = J[0][0] * c00 + J[0][1] * c01 + J[0][2] * c02;
  const T id = T(1) / det;
  // (J^-1)_kj = cof(J)_jk / det
  Ji[0][0] = c00 * id;
  Ji[1][0] = c01 * id;
  Ji[2][0] = c02 * id;
  Ji[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * id;
  Ji[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * id;
  Ji[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * id;
  Ji[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * id;
  Ji[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * id;
  Ji[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * id;
  return det;
}

// Physical basis gradients g[a][j] = dN_a/dx_j at Gauss point q; returns det J.
template <typename T> __device__ __forceinline__ T phys_grad(const T (*xe)[3], int q, T g[8][3]) {
  T dn[8][3], Ji[3][3];
  ref_grad<T>(q, dn);
  const T det = jacobian_inverse<T>(xe, dn, Ji);
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int j = 0; j < 3; ++j) g[a][j] = dn[a][0] * Ji[0][j] + dn[a][1] * Ji[1][j] + dn[a][2] * Ji[2][j];
  return det;
}

// Displacement gradient H[c][j] = sum_a u[a][c] g[a][j].
template <typename T> __device__ __forceinline__ void field_grad(const T (*ue)[3], const T g[8][3], T H[3][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      T s = 0;
#pragma unroll
      for (int a = 0; a < 8; ++a) s += ue[a][c] * g[a][j];
      H[c][j] = s;
    }
}

// v of another lane of the aligned group of 8, by DPP (a register move; 32 bits at a time).
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_MIRROR8 = 0x141;  // row_half_mirror: lane q <- 7 - q
constexpr int DPP_XOR2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int DPP_XOR1 = 0xB1;      // quad_perm [1,0,3,2]

// Sum of per-lane values v[8][NV] (node, component) over the 8 lanes of an element (lanes q =
// lane % 8); afterwards lane q holds node q's total in out[NV].  Recursive halving: each step
// sends the half the partner keeps and adds the received half to its own (the first partner is
// 7 - q, whose upper bit differs; the others q ^ 2 and q ^ 1).
template <typename T, int NV> __device__ __forceinline__ void reduce_scatter8(const T v[8][NV], int q, T out[NV]) {
  T h1[4][NV], h2[2][NV];
  const bool b4 = q & 4, b2 = q & 2, b1 = q & 1;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const T send = b4 ? v[a][c] : v[a + 4][c];
      const T keep = b4 ? v[a + 4][c] : v[a][c];
      h1[a][c] = keep + dpp_move<DPP_MIRROR8>(send);
    }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const T send = b2 ? h1[a][c] : h1[a + 2][c];
      const T keep = b2 ? h1[a + 2][c] : h1[a][c];
      h2[a][c] = keep + dpp_move<DPP_XOR2>(send);
    }
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const T send = b1 ? h2[0][c] : h2[1][c];
    const T keep = b1 ? h2[1][c] : h2[0][c];
    out[c] = keep + dpp_move<DPP_XOR1>(send);
  }
}

// Sum of one value over the 8 lanes of an element (every lane gets it).
__device__ __forceinline__ double sum8(double v) {
  v += __shfl_xor(v, 4, 64);
  v += __shfl_xor(v, 2, 64);
  v += __shfl_xor(v, 1, 64);
  return v;
}

struct GenArgs {
  const void* coords;     // real [n_nodes][3]
  const int32_t* conn;    // [8][n_el]
  int64_t n_nodes;
};

static GenArgs gen_args(const fe_problem* p) {
  GenArgs g;
  g.coords = p->coords;
  g.conn = p->conn;
  g.n_nodes = p->n_nodes;
  return g;
}

// ---------------------------------------------------------------------------
// CG scalars on a general mesh (textbook PCG; see gen_cg_node_kernel).  Sums go through GCG_SLOTS
// slots per quantity, two sets in turn: node launch j - 1 adds GCG_Q quantities of iterate j,
// element launch j sums them (every workgroup the same way), and adds (p_j, A p_j) to slots of its
// own that node launch j sums.
constexpr int GCG_SLOTS = 64;
constexpr int GCG_Q = 5;  // (r, M^-1 r), ||r||^2; over constrained dofs (A p = p there) u.u, u.p, p.p with the old p
static_assert(2 * GCG_Q * GCG_SLOTS + 2 * GCG_SLOTS <= 9 * CGS_SLOTS, "slots fit the problem's partial sums");

struct GenCgScalars {
  double v[2], rtol2, tol2, rz_old;
  int max_it;
  // this lane's slots (of 5 x 64, 256 lanes) and the scalars of the iterate before
  __device__ __forceinline__ void request(const ElemArgs& a, int tid) {
    v[0] = a.cg_acc_in[tid];
    v[1] = tid < GCG_Q * GCG_SLOTS - GBLOCK ? a.cg_acc_in[GBLOCK + tid] : 0.0;
    const CgCtrl* c = a.ctrl;
    rtol2 = c->rtol2;
    tol2 = c->tol2;
    rz_old = c->rz[(a.cg_j + 1) & 1];
    max_it = c->max_it;
    if (blockIdx.x == 0)
      for (int i = tid; i < GCG_Q * GCG_SLOTS; i += GBLOCK) a.cg_acc_zero[i] = 0.0;  // slots of iterate j + 1
  }
  // beta_j, or false at a stop; workgroup 0 records the iterate
  __device__ __forceinline__ bool direction(const ElemArgs& a, double* sh, double& beta) {
    static_assert(GCG_SLOTS == 64 && GBLOCK == 256, "one wave per quantity");
    const int wave = threadIdx.x >> 6;
    const double s0 = wave_sum_last(v[0]), s1 = wave_sum_last(v[1]);
    if ((threadIdx.x & 63) == WAVE_LAST) {
      sh[wave] = s0;
      if (wave == 0) sh[4] = s1;
    }
    __syncthreads();
    const double rz = sh[0], rr = sh[1], uu = sh[2], up = sh[3], pp = sh[4];
    __syncthreads();  // sh is reused
    const long j = a.cg_j;
    const double t2 = j == 0 ? rtol2 * rr : tol2;
    int st = CG_RUNNING;
    if (!finite(rr) || !finite(rz)) st = FE_ERR_NONFINITE;
    else if (j == 0 ? rr == 0.0 : rr <= t2) st = CG_CONVERGED;
    else if (j >= max_it) st = FE_ERR_NOT_CONVERGED;
    beta = j == 0 ? 0.0 : rz / rz_old;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      CgCtrl* w = a.ctrl;
      if (j == 0) {
        w->bb = rr;
        w->tol2 = t2;
      }
      w->rr = rr;
      w->iters = (int)j;
      w->beta = beta;
      w->rz[j & 1] = rz;
      w->pq = uu + 2.0 * beta * up + beta * beta * pp;  // constrained share of (p_j, A p_j)
      if (st != CG_RUNNING) w->status = st;
    }
    return st == CG_RUNNING;
  }
};

// ---------------------------------------------------------------------------
// element kernel: OP_RESID, OP_APPLY, OP_VJP (ElemArgs as for the structured kernels; y
// zeroed by the caller; constrained dofs receive nothing, see gen_bc_kernel)

// ELF: the nodal forces go to a.elf ([n_el][8][3], one contiguous run per wave) for
// gen_cg_node_kernel / gen_gather_kernel instead of being added with atomics, which random node
// numbers make the whole cost (33^3 FP32 operator: 53 us with them).  CG: the operator launch of a
// CG iteration, see gen_cg_node_kernel.
template <typename T, int OP, int MS, bool ELF = false, bool CG = false>
__global__ __launch_bounds__(GBLOCK) void gen_elem_kernel(GenArgs g, ElemArgs a, const int* stop) {
  constexpr bool APPLY = OP == OP_APPLY;
  constexpr bool NEED_L = OP == OP_VJP;
  __shared__ alignas(16) T s_c[GEL][8][3];
  __shared__ alignas(16) T s_x[GEL][8][3];
  __shared__ T s_l[NEED_L ? GEL : 1][8][3];
  __shared__ double s_red[6][GBLOCK / 64];
  const int stopped = stop ? *stop : 0;  // (tested once this lane's gathers are on their way)
  GenCgScalars cgs;
  if constexpr (CG) cgs.request(a, threadIdx.x);
  const int tid = threadIdx.x, el = tid >> 3, q = tid & 7;
  const int64_t ne = a.n_el;
  const int64_t e = (int64_t)blockIdx.x * GEL + el;
  const bool valid = e < ne;
  const T* X = static_cast<const T*>(a.x);
  const T* XL = static_cast<const T*>(a.xlin);
  const T* C = static_cast<const T*>(g.coords);
  const bool bc = a.apply_bc && a.mask;
  // stage node q of element e
  int node = 0;
  if (valid) node = g.conn[(int64_t)q * ne + e];
  T uv[3], pv[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int64_t dof = 3 * (int64_t)node + c;
    s_c[el][q][c] = valid ? C[dof] : T(0);
    T v = valid ? X[dof] : T(0);
    if (APPLY && bc && valid && a.mask[dof]) v = T(0);
    if constexpr (CG) {
      uv[c] = v;
      pv[c] = valid ? static_cast<const T*>(a.cg_pvec)[dof] : T(0);
    } else {
      s_x[el][q][c] = v;
    }
    if (NEED_L) s_l[NEED_L ? el : 0][q][c] = valid ? XL[dof] : T(0);
  }
  if (stopped) return;
  if constexpr (CG) {  // p_j = u_j + beta_j p_{j-1}
    double beta;
    if (!cgs.direction(a, &s_red[0][0], beta)) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) s_x[el][q][c] = uv[c] + T(beta) * pv[c];
  }
  __syncthreads();

  T f[8][3];
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int c = 0; c < 3; ++c) f[b][c] = 0;
  double ssum[6] = {0, 0, 0, 0, 0, 0};
  if (valid) {
    T gr[8][3];
    const T wdet = phys_grad<T>(s_c[el], q, gr);  // Gauss weight 1
    T H[3][3], S[3][3];
    field_grad<T>(s_x[el], gr, H);
    const PhaseConst pc = a.mat.ph[a.phase[e]];
    const T sc = (a.scale && OP != OP_VJP) ? static_cast<const T*>(a.scale)[e] : T(1);
    const T lam = T(pc.lam) * sc, mu = T(pc.mu) * sc;
    const T Kb = T(pc.K) * sc, Gs = T(pc.G) * sc, sy = T(pc.sy), Hh = T(pc.H);
    const int64_t pidx = (int64_t)q * ne + e;  // Gauss-point index in [8][n_el] arrays
    const T* st_in = static_cast<const T*>(a.state_in);
    T* st_out = static_cast<T*>(a.state_out);
    T* tang = static_cast<T*>(a.tangent);
    bool done = false;
    if (MS == MS_J2 && pc.model == FE_J2) {
      if (OP == OP_RESID) {
        T epn[6], an = 0, ep[6], al, tn[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) epn[k] = st_in ? st_in[(int64_t)k * 8 * ne + pidx] : T(0);
        if (st_in) an = st_in[(int64_t)6 * 8 * ne + pidx];
        j2_update(H, epn, an, Kb, Gs, sy, Hh, S, ep, al, tn);
        if (st_out) {
#pragma unroll
          for (int k = 0; k < 6; ++k) st_out[(int64_t)k * 8 * ne + pidx] = ep[k];
          st_out[(int64_t)6 * 8 * ne + pidx] = al;
        }
        if (a.store_tangent) {
#pragma unroll
          for (int k = 0; k < 6; ++k) tang[(int64_t)k * 8 * ne + pidx] = tn[k];
        }
        done = true;
      } else if (APPLY) {
        T tn[6], lp, mp, beta, N[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) tn[k] = tang[(int64_t)k * 8 * ne + pidx];
        j2_tangent_coeffs(tn, Kb, Gs, Hh, lp, mp, beta, N);
        j2_apply(H, lp, mp, beta, N, S);
        done = true;
      }
    }
    if (MS == MS_NH && pc.model == FE_NEOHOOKE) {
      if (APPLY) {  // F^-T and ln J of the linearisation, as the residual stored them
        T FiT[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) FiT[i][j] = tang[(int64_t)(3 * i + j) * 8 * ne + pidx];
        nh_apply(H, FiT, tang[(int64_t)9 * 8 * ne + pidx], lam, mu, S);
      } else {
        T FiT[3][3], lnJ;
        if (!nh_kin(H, FiT, lnJ) && a.flags) atomicOr(a.flags, 1);
        nh_stress(H, FiT, lnJ, lam, mu, S);
        if (OP == OP_RESID && a.store_tangent) {
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) tang[(int64_t)(3 * i + j) * 8 * ne + pidx] = FiT[i][j];
          tang[(int64_t)9 * 8 * ne + pidx] = lnJ;
        }
      }
      done = true;
    }
    if (!done) {
      hooke(H, lam, mu, S);
      if (MS == MS_J2 && OP == OP_RESID && st_out) {  // non-J2 phase: state passes through
#pragma unroll
        for (int k = 0; k < 7; ++k) st_out[(int64_t)k * 8 * ne + pidx] = st_in ? st_in[(int64_t)k * 8 * ne + pidx] : T(0);
      }
    }
    // nodal forces of this point: w detJ S g_b
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) f[b][c] = wdet * (S[c][0] * gr[b][0] + S[c][1] * gr[b][1] + S[c][2] * gr[b][2]);
    if (OP == OP_RESID && a.stress_sum) {
      const double w = (double)wdet;
      ssum[0] = w * S[0][0];
      ssum[1] = w * S[1][1];
      ssum[2] = w * S[2][2];
      ssum[3] = w * S[1][2];
      ssum[4] = w * S[0][2];
      ssum[5] = w * S[0][1];
    }
  }
  T fn[3];
  reduce_scatter8<T, 3>(f, q, fn);  // all lanes take part (invalid ones with zeros)

  if (OP == OP_VJP) {
    // out_e = sum_b f_b . (lambda_b - mean lambda): exact (the element's nodal forces sum to
    // zero) and free of the cancellation of a large rigid part of lambda
    double lm[3] = {0, 0, 0};
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) lm[c] += (double)s_l[NEED_L ? el : 0][b][c];
    double d = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) d += (double)fn[c] * ((double)s_l[NEED_L ? el : 0][q][c] - 0.125 * lm[c]);
    d = sum8(d);
    if (valid && q == 0) static_cast<T*>(a.out_el)[e] = T(d);
    return;
  }

  if (OP == OP_RESID && a.stress_sum) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      double v = ssum[k];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
      if ((tid & 63) == 0) s_red[k][tid >> 6] = v;
    }
    __syncthreads();
    if (tid < 6) {
      double v = 0;
      for (int w = 0; w < GBLOCK / 64; ++w) v += s_red[tid][w];
      atomic_add(a.stress_sum + 8 * (blockIdx.x % STRESS_SLOTS) + tid, v);
    }
  }

  if constexpr (ELF) {
    if (valid) {
      T* E = static_cast<T*>(a.elf) + 3 * (8 * e + q);
#pragma unroll
      for (int c = 0; c < 3; ++c) E[c] = fn[c];
    }
    if constexpr (CG) {  // this element's share of (p, A p)
      double d = 0;
#pragma unroll
      for (int c = 0; c < 3; ++c) d += (double)fn[c] * (double)s_x[el][q][c];
      d = wave_sum_last(d);
      if ((tid & 63) == WAVE_LAST) s_red[0][tid >> 6] = d;
      __syncthreads();
      if (tid == 0) {
        double t = 0;
        for (int w = 0; w < GBLOCK / 64; ++w) t += s_red[0][w];
        atomic_add(a.cg_acc_out + (int)(blockIdx.x % GCG_SLOTS), t);
      }
    }
    return;
  }
  T* Y = static_cast<T*>(a.y);
  if (!Y || !valid) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int64_t dof = 3 * (int64_t)node + c;
    if (a.apply_bc && a.mask && a.mask[dof]) continue;
    atomic_add(Y + dof, fn[c]);
  }
}

// Constrained dofs of a masked operator: y = x there (A = P_f K P_f + P_b).  With pa, also the
// per-workgroup partials of x.y over all dofs (CG: p.Ap); x, y complete (kernel boundary).
template <typename T>
__global__ __launch_bounds__(VBLOCK) void gen_bc_kernel(int64_t n, const uint8_t* mask, const T* x, T* y,
                                                        const int* stop, double* pa) {
  __shared__ double sh[VBLOCK / 64];
  if (stop && *stop) return;
  double v = 0;
  for (int64_t i = (int64_t)blockIdx.x * VBLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * VBLOCK) {
    T yi;
    if (mask && mask[i]) {
      yi = x[i];
      y[i] = yi;
    } else {
      yi = y[i];
    }
    if (pa) v += (double)x[i] * (double)yi;
  }
  if (pa) {
    v = block_sum(v, sh);
    if (threadIdx.x == 0) pa[blockIdx.x] = v;
  }
}

// Sum of the element forces at dof 3 node + c over the node's incidences, in element order.
template <typename T>
__device__ __forceinline__ T gather_node(const T* __restrict__ elf, const int32_t* __restrict__ inc, int i0, int i1,
                                         int c) {
  T v = 0;
  int k = i0;
  for (; k + 4 <= i1; k += 4) {  // (four index loads, then four gathers in flight)
    const int n0 = inc[k], n1 = inc[k + 1], n2 = inc[k + 2], n3 = inc[k + 3];
    const T v0 = elf[3 * (int64_t)n0 + c], v1 = elf[3 * (int64_t)n1 + c], v2 = elf[3 * (int64_t)n2 + c],
            v3 = elf[3 * (int64_t)n3 + c];
    v += v0;
    v += v1;
    v += v2;
    v += v3;
  }
  for (; k < i1; ++k) v += elf[3 * (int64_t)inc[k] + c];
  return v;
}

// y = K x from the element forces, y = x on constrained dofs (solver operators other than CG's).
template <typename T>
__global__ __launch_bounds__(VBLOCK) void gen_gather_kernel(int64_t n, const int32_t* inc_ptr, const int32_t* inc,
                                                            const T* elf, const uint8_t* mask, const T* x, T* y,
                                                            const int* stop) {
  if (stop && *stop) return;
  for (int64_t d = (int64_t)blockIdx.x * VBLOCK + threadIdx.x; d < n; d += (int64_t)gridDim.x * VBLOCK) {
    const int64_t nd = d / 3;
    const T v = gather_node(elf, inc, inc_ptr[nd], inc_ptr[nd + 1], (int)(d - 3 * nd));
    y[d] = mask && mask[d] ? x[d] : v;
  }
}

// PCG on a general mesh, two launches an iteration and no floating-point atomics but the slot sums:
//   element launch j: beta_j (or a stop) from the slots of iterate j; p_j = u_j + beta_j p_{j-1} at
//     the gathered nodes; element forces of A p_j; share of (p_j, A p_j);
//   node launch j (below): alpha_j; p_j again, as owner; q = A p_j gathered;
//     x += alpha p, r -= alpha q, u = M^-1 r, and the sums of iterate j + 1.
// Node launch -1 (FIRST) starts from r = b.  Against four launches (direction, operator with
// atomics, constrained rows, update) an iteration at 33^3 FP32 takes 27 instead of 64 us (60^3 FP64 168 instead of 292).  The
// recurrence for A p of the structured launch would save the second reduction, but in FP32 it
// leaves twice the error (9.6e-7 against 4.9e-7 in x at rtol 1e-6).
// u and p are stored with their constrained entries 0, as the element kernel wants them (u is
// re-formed from r here, the constrained p lives in pf).  21 nodes per wave, lane = 3 node + component.
struct GenCgArgs {
  int64_t n_nodes;
  long j;
  const int32_t* inc_ptr;
  const int32_t* inc;
  const void* elf;
  const uint8_t* mask;
  const void* b;        // right-hand side (FIRST)
  void *r, *p, *pf, *x, *u;
  void* dinv;           // inverse diagonal [n_dof] (FIRST: the diagonal, inverted here) or node blocks [n_nodes][6]
  CgCtrl* ctrl;
  const double* pq_in;  // slots of (p_j, A p_j)
  double *pq_zero, *acc_out;
};

constexpr int CGN_NODES = 21;

template <typename T, bool BLK, bool FIRST>
__global__ __launch_bounds__(VBLOCK) void gen_cg_node_kernel(GenCgArgs a) {
  constexpr int W = VBLOCK / 64;
  __shared__ double sh[GCG_Q * W];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double pq = 0, rz = 0, pqc = 0, beta_d = 0;
  int status = 0;
  if (!FIRST) {
    pq = a.pq_in[lane];  // (every wave sums the 64 slots)
    rz = a.ctrl->rz[a.j & 1];
    pqc = a.ctrl->pq;
    beta_d = a.ctrl->beta;
    status = a.ctrl->status;
  }
  if (blockIdx.x == 0 && tid < GCG_SLOTS) a.pq_zero[tid] = 0.0;  // slots of element launch j + 1
  const int64_t nd0 = ((int64_t)blockIdx.x * W + wave) * CGN_NODES + lane / 3;
  const bool ok = lane < 3 * CGN_NODES && nd0 < a.n_nodes;
  const int64_t nd = ok ? nd0 : 0;
  const int c = lane % 3;
  const int64_t dof = 3 * nd + c;
  T* R = static_cast<T*>(a.r);
  T* P = static_cast<T*>(a.p);
  T* PF = static_cast<T*>(a.pf);
  T* X = static_cast<T*>(a.x);
  T* M = static_cast<T*>(a.dinv);
  const bool fixed = a.mask && a.mask[dof];
  T m0, m1 = 0, m2 = 0;
  if (BLK) {  // xx yy zz yz xz xy
    const T* m = M + 6 * nd;
    m0 = m[c == 0 ? 0 : (c == 1 ? 5 : 4)];
    m1 = m[c == 0 ? 5 : (c == 1 ? 1 : 3)];
    m2 = m[c == 0 ? 4 : (c == 1 ? 3 : 2)];
  } else {
    m0 = M[dof];
    if (FIRST) m0 = T(1) / m0;
  }
  const int l0 = lane - c;
  auto precond = [&](T r) {
    if (!BLK) return m0 * r;
    return m0 * __shfl(r, l0, 64) + m1 * __shfl(r, l0 + 1, 64) + m2 * __shfl(r, l0 + 2, 64);
  };
  T r, p = 0, x = 0;
  if (FIRST) {
    r = static_cast<const T*>(a.b)[dof];
  } else {
    r = R[dof];
    p = fixed ? PF[dof] : P[dof];
    x = X[dof];
    const T q0 = gather_node(static_cast<const T*>(a.elf), a.inc, a.inc_ptr[nd], a.inc_ptr[nd + 1], c);
    if (status) return;
    pq = wave_sum_last(pq);
    pq = __shfl(pq, WAVE_LAST, 64) + pqc;
    const int st = !finite(pq) ? FE_ERR_NONFINITE : (pq <= 0.0 ? FE_ERR_BREAKDOWN : CG_RUNNING);
    const double alpha = rz / pq;
    if (blockIdx.x == 0 && tid == 0) {
      a.ctrl->alpha = alpha;
      if (st != CG_RUNNING) a.ctrl->status = st;
    }
    if (st != CG_RUNNING) return;
    const T ta = T(alpha);
    p = precond(r) + T(beta_d) * p;
    x += ta * p;
    r -= ta * (fixed ? p : q0);
  }
  const T u = precond(r);
  double q5[GCG_Q] = {};
  if (ok) {
    if (FIRST && !BLK) M[dof] = m0;
    R[dof] = r;
    X[dof] = x;
    P[dof] = fixed ? T(0) : p;
    static_cast<T*>(a.u)[dof] = fixed ? T(0) : u;
    q5[0] = (double)r * (double)u;
    q5[1] = (double)r * (double)r;
    if (fixed) {
      PF[dof] = p;
      q5[2] = (double)u * (double)u;
      q5[3] = (double)u * (double)p;
      q5[4] = (double)p * (double)p;
    }
  }
#pragma unroll
  for (int k = 0; k < GCG_Q; ++k) {
    const double t = wave_sum_last(q5[k]);
    if (lane == WAVE_LAST) sh[W * k + wave] = t;
  }
  __syncthreads();
  if (tid < GCG_Q) {
    double t = 0;
    for (int w = 0; w < W; ++w) t += sh[W * tid + w];
    atomic_add(a.acc_out + tid * GCG_SLOTS + (int)(blockIdx.x % GCG_SLOTS), t);
  }
}

// Start of a solve: controls, and the slot sets cleared.
__global__ void gen_cg_start_kernel(CgCtrl* ctrl, double rtol, int max_it, double* acc) {
  for (int i = threadIdx.x; i < 2 * (GCG_Q + 1) * GCG_SLOTS; i += blockDim.x) acc[i] = 0.0;
  if (threadIdx.x == 0) {
    ctrl->rtol2 = rtol * rtol;
    ctrl->iters = 0;
    ctrl->max_it = max_it;
    ctrl->alpha = ctrl->beta = ctrl->pq = 0;
    ctrl->rz[0] = ctrl->rz[1] = 0;
    ctrl->status = CG_RUNNING;
  }
}

// ---------------------------------------------------------------------------
// diagonal (NB = 3) or symmetric 3x3 node blocks (NB = 6: xx yy zz yz xz xy) of K at the
// stored linearisation, summed over elements (d zeroed before; constrained dofs skipped)

template <typename T, int MS, int NB>
__global__ __launch_bounds__(GBLOCK) void gen_diag_kernel(GenArgs g, TanArgs ta, T* d, int skip_bc) {
  __shared__ T s_c[GEL][8][3];
  const int tid = threadIdx.x, el = tid >> 3, q = tid & 7;
  const int64_t ne = ta.n_el;
  const int64_t e = (int64_t)blockIdx.x * GEL + el;
  const bool valid = e < ne;
  const T* C = static_cast<const T*>(g.coords);
  int node = 0;
  if (valid) node = g.conn[(int64_t)q * ne + e];
#pragma unroll
  for (int c = 0; c < 3; ++c) s_c[el][q][c] = valid ? C[3 * (int64_t)node + c] : T(0);
  __syncthreads();
  T v[8][NB];
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int k = 0; k < NB; ++k) v[b][k] = 0;
  if (valid) {
    T gr[8][3];
    const T wdet = phys_grad<T>(s_c[el], q, gr);
    QpTangent<T> t;
    load_qp_tangent<T, MS>(ta, e, q, t);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      T B[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
      block_add(t, gr[b], gr[b], wdet, B);
      v[b][0] = B[0][0];
      v[b][1] = B[1][1];
      v[b][2] = B[2][2];
      if (NB == 6) {
        v[b][NB == 6 ? 3 : 0] = B[1][2];
        v[b][NB == 6 ? 4 : 0] = B[0][2];
        v[b][NB == 6 ? 5 : 0] = B[0][1];
      }
    }
  }
  T out[NB];
  reduce_scatter8<T, NB>(v, q, out);
  if (!valid) return;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    if (NB == 3 && skip_bc && ta.mask && ta.mask[3 * (int64_t)node + k]) continue;
    atomic_add(d + (int64_t)NB * node + k, out[k]);
  }
}

template <typename T> __global__ void gen_mask_one_kernel(int64_t n, const uint8_t* mask, T* d) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    if (mask[i]) d[i] = T(1);
}

// ---------------------------------------------------------------------------
// element Jacobians
//
// The 3 x 3 block of nodes a, b is, summed over the Gauss points with their weights w detJ,
//   small strain  lp g_a g_b^T + mp g_b g_a^T + mp (g_a . g_b) I - beta (N g_a)(N g_b)^T
//   Neo-Hookean   lam h_a h_b^T + (mu - lam ln J) h_b h_a^T + mu (g_a . g_b) I,  h = F^-T g
// with the physical basis gradients g: 33 multiply-adds per point and pair, which needs neither
// the 6 x 6 (9 x 9) moduli nor the padding of a 24 x 24 matrix to matrix-core tiles.  K_e is
// symmetric, so only the 36 pairs a <= b are formed; their transposes are written with them.
// A workgroup takes TEL elements: one lane per (element, point) forms the gradients into LDS, then
// one lane per (element, 2 x 2 tile of nodes) sums its four blocks, and the blocks leave through LDS
// in whole lines.  Output: ke[e][a][b][i][k] = K_e[(a, i), (b, k)] (576 reals).

constexpr int TEL = 16;                // elements per workgroup
constexpr int TPAIR = 36;              // node pairs a <= b of an element
constexpr int TBLOCK = 10 * TEL;       // tiles (0,0) (0,1) .. (3,3) of node pairs 2A, 2A + 1
constexpr int TGS = 25;                // reals per (point, element) row of 8 gradients (odd: no bank conflicts)
constexpr int TOS = 9 * TPAIR + 1;     // reals per element of the blocks on their way out

// Pair of local nodes a <= b.
__device__ __forceinline__ int pair_index(int a, int b) { return a * (15 - a) / 2 + b; }

// Bound by the 576 reals per element written (233 MB at 37^3 FP64, 49 us at the copy rate) and its own
// three phases, which four workgroups per CU overlap: 73 us there against 197 us for one wave per
// element on matrix cores (padded tiles, 36 or 81 LDS words of moduli per point).  A lane per pair read
// twice the LDS words (102 us while writing half as much); 32 elements per workgroup left two of
// them per CU (119 us).
template <typename T, int MS>
__global__ __launch_bounds__(TBLOCK) __attribute__((amdgpu_waves_per_eu(3))) void gen_tangent_kernel(GenArgs g, TanArgs ta,
                                                                                                     T* __restrict__ ke) {
  constexpr int NG = 8 * TEL * TGS;
  // per point: c1, c2 [, -beta, N] or [, mu, F^-T]
  constexpr int NCF = MS == MS_LINEAR ? 2 : (MS == MS_J2 ? 9 : 12);
  __shared__ T s_g[NG];                            // gradients, later the blocks
  __shared__ T s_cf[NCF][8 * TEL];
  __shared__ T s_xe[TEL][8][3];
  static_assert(NG >= TEL / 2 * TOS, "the blocks of half the elements fit");
  const int tid = threadIdx.x, el = tid % TEL;
  const int64_t ne = ta.n_el, e0 = (int64_t)blockIdx.x * TEL;
  const int64_t e = e0 + el < ne ? e0 + el : ne - 1;
  if (tid < 8 * TEL) {
    const int q = tid / TEL;
    const int node = g.conn[(int64_t)q * ne + e];
    const T* C = static_cast<const T*>(g.coords) + 3 * (int64_t)node;
#pragma unroll
    for (int c = 0; c < 3; ++c) s_xe[el][q][c] = C[c];
  }
  __syncthreads();
  if (tid < 8 * TEL) {
    const int q = tid / TEL;
    QpTangent<T> t;
    load_qp_tangent<T, MS>(ta, e, q, t);
    T gr[8][3];
    const T w = phys_grad<T>(s_xe[el], q, gr);
    if (MS == MS_NH && t.kind == 1) {
      s_cf[0][tid] = w * t.lam;
      s_cf[1][tid] = w * (t.mu - t.lam * t.lnJ);
      s_cf[2 % NCF][tid] = w * t.mu;
    } else {
      s_cf[0][tid] = w * t.lp;
      s_cf[1][tid] = w * t.mp;
      if (MS != MS_LINEAR) s_cf[2 % NCF][tid] = MS == MS_NH ? w * t.mp : -w * t.beta;
    }
    if (MS == MS_J2)
#pragma unroll
      for (int k = 0; k < 6; ++k) s_cf[(3 + k) % NCF][tid] = t.N[k];
    if (MS == MS_NH)
#pragma unroll
      for (int k = 0; k < 9; ++k)
        s_cf[(3 + k) % NCF][tid] = t.kind == 1 ? t.FiT[k / 3][k % 3] : T(k % 4 == 0 ? 1 : 0);
    T* sg = s_g + tid * TGS;
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int i = 0; i < 3; ++i) sg[3 * a + i] = gr[a][i];
  }
  __syncthreads();
  const int tile = tid / TEL;
  const int ta0 = (tile >= 4) + (tile >= 7) + (tile >= 9), tb0 = tile - ta0 * (7 - ta0) / 2;  // tile (A, B)
  T K[2][2][3][3];
#pragma unroll
  for (int m = 0; m < 36; ++m) K[m / 18][m / 9 % 2][m / 3 % 3][m % 3] = 0;
#pragma unroll 1
  for (int q = 0; q < 8; ++q) {
    const int pt = q * TEL + el;
    const T* ga = s_g + pt * TGS + 6 * ta0;
    const T* gb = s_g + pt * TGS + 6 * tb0;
    T va[2][3], vb[2][3], wa[2][3], wb[2][3];  // w: N g (J2) or h = F^-T g (Neo-Hookean)
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      va[m / 3][m % 3] = ga[m];
      vb[m / 3][m % 3] = gb[m];
    }
    const T c1 = s_cf[0][pt], c2 = s_cf[1][pt], c3 = s_cf[2 % NCF][pt];
    if (MS != MS_LINEAR) {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        T M[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          // Voigt [xx yy zz yz xz xy] of N, or row i of F^-T
          const int at = MS == MS_NH ? 3 * i + k : (i == k ? i : 6 - i - k);
          M[k] = s_cf[(3 + at) % NCF][pt];
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          wa[n][i] = M[0] * va[n][0] + M[1] * va[n][1] + M[2] * va[n][2];
          wb[n][i] = M[0] * vb[n][0] + M[1] * vb[n][1] + M[2] * vb[n][2];
        }
      }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      T x1[3], x2[3], x3[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const T p = MS == MS_NH ? wa[n][i] : va[n][i];
        x1[i] = c1 * p;
        x2[i] = c2 * p;
        if (MS == MS_J2) x3[i] = c3 * wa[n][i];
        if (MS == MS_NH) x3[i] = c3 * va[n][i];
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const T* pb = MS == MS_NH ? wb[m] : vb[m];
        const T dot = MS == MS_NH ? x3[0] * vb[m][0] + x3[1] * vb[m][1] + x3[2] * vb[m][2]
                                  : x2[0] * vb[m][0] + x2[1] * vb[m][1] + x2[2] * vb[m][2];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            T v = K[n][m][i][k] + x1[i] * pb[k];
            v += x2[k] * pb[i];
            if (MS == MS_J2) v += x3[i] * wb[m][k];
            if (i == k) v += dot;
            K[n][m][i][k] = v;
          }
      }
    }
  }
  // half the elements at a time; TOUT lanes then hold 576 / TOUT entries of every K_e
  constexpr int TOUT = 9 * TEL, TENT = 576 / TOUT;
  int from[TENT];
#pragma unroll
  for (int u = 0; u < TENT; ++u) {
    const int entry = tid + TOUT * u, a = entry / 72, b = entry / 9 % 8, m = entry % 9;
    from[u] = 9 * (a <= b ? pair_index(a, b) : pair_index(b, a)) + (a <= b ? m : 3 * (m % 3) + m / 3);
  }
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    __syncthreads();  // s_g is read no more
    if (el / (TEL / 2) == half) {
      T* so = s_g + (el % (TEL / 2)) * TOS;
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          if (n > m && ta0 == tb0) continue;  // (1, 0) of a diagonal tile
          T* sb = so + 9 * pair_index(2 * ta0 + n, 2 * tb0 + m);
#pragma unroll
          for (int k = 0; k < 9; ++k) sb[k] = K[n][m][k / 3][k % 3];
        }
    }
    __syncthreads();
    if (tid < TOUT) {
      const int64_t eh = e0 + half * (TEL / 2);
      T* out = ke + eh * 576 + tid;
#pragma unroll 4
      for (int k = 0; k < TEL / 2; ++k)
        if (eh + k < ne)
#pragma unroll
          for (int u = 0; u < TENT; ++u) out[576 * k + TOUT * u] = s_g[k * TOS + from[u]];
    }
  }
}

// CSR values: one wave per row node.  The rows of the element Jacobians around the node (72 reals
// each, contiguous) are staged in LDS, then every lane sums the run of its entry in sorted order:
// entries of the row are numbered as they lie in vals (3 x 3 deg(a), then k, c), so both the reads and
// the stores are whole lines.  A node of more than ASM_INC elements reads its runs from memory.
// Bound by the Jacobians read and the values written (233 + 107 MB at 37^3 FP64, 72 us at the copy rate):
// 110 us against 158 us with a lane per node pair, whose nine loads and stores each touched 64 lines.
constexpr int ASM_INC = 8;           // elements around a node of a regular mesh
constexpr int ASM_WAVES = VBLOCK / 64;
template <typename T>
__global__ __launch_bounds__(VBLOCK) void gen_assemble_kernel(int64_t n_nodes, const int32_t* __restrict__ adj_ptr,
                                                              const int32_t* __restrict__ adj,
                                                              const int32_t* __restrict__ src_ptr,
                                                              const int32_t* __restrict__ src,
                                                              const int32_t* __restrict__ inc_ptr,
                                                              const int32_t* __restrict__ inc,
                                                              const T* __restrict__ ke, const uint8_t* mask,
                                                              int apply_bc, T* __restrict__ vals) {
  __shared__ T s_row[ASM_WAVES][72 * ASM_INC];
  __shared__ int s_src[ASM_WAVES][8 * ASM_INC];
  __shared__ int s_ptr[ASM_WAVES][8 * ASM_INC + 1];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t a = (int64_t)blockIdx.x * ASM_WAVES + wave;
  int i0 = 0, ni = 0, base = 0, deg = 0;
  if (a < n_nodes) {
    i0 = inc_ptr[a];
    ni = inc_ptr[a + 1] - i0;
    base = adj_ptr[a];
    deg = adj_ptr[a + 1] - base;
  }
  const bool staged = ni <= ASM_INC;
  if (staged) {
    const int row = lane < ni ? inc[i0 + lane] : 0;  // 8 element + local node: 72 reals from row * 72
    if (lane < 8 * ni) s_src[wave][lane] = src[8 * (int64_t)i0 + lane];
    if (lane < deg) s_ptr[wave][lane] = src_ptr[base + lane] - 8 * i0;
    if (lane == 0) s_ptr[wave][deg] = 8 * ni;
    T v[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int w = lane + 64 * t, k = w / 72;
      const int from = __shfl(row, k, 64);
      v[t] = w < 72 * ni ? ke[(int64_t)from * 72 + (w - 72 * k)] : T(0);
    }
#pragma unroll
    for (int t = 0; t < 9; ++t) s_row[wave][lane + 64 * t] = v[t];
  }
  __syncthreads();
  const bool bc = apply_bc && mask;
  for (int o = lane; o < 9 * deg; o += 64) {
    const int i = (o >= 3 * deg) + (o >= 6 * deg), rem = o - 3 * deg * i, k = rem / 3, c = rem - 3 * k, j = 3 * i + c;
    T acc = 0;
    if (staged) {
      const int s1 = s_ptr[wave][k + 1];
      for (int s = s_ptr[wave][k]; s < s1; ++s) acc += s_row[wave][9 * s_src[wave][s] + j];
    } else {
      const int s1 = src_ptr[base + k + 1];
      for (int s = src_ptr[base + k]; s < s1; ++s) {
        const int code = src[s];  // 8 incidence + local column node
        acc += ke[(int64_t)inc[i0 + (code >> 3)] * 72 + 9 * (code & 7) + j];
      }
    }
    if (bc) {
      const int64_t rdof = 3 * a + i, cdof = 3 * (int64_t)adj[base + k] + c;
      if (mask[rdof] || mask[cdof]) acc = rdof == cdof ? T(1) : T(0);
    }
    vals[9 * (int64_t)base + o] = acc;
  }
}

// ---------------------------------------------------------------------------
// symbolic assembly: node-pair pattern by sorting the element pairs

// COO entries per row node: 8 per element that contains it.
__global__ void sym_count_kernel(int64_t ne, const int32_t* conn, int32_t* cnt) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 8 * ne; i += (int64_t)gridDim.x * blockDim.x)
    atomicAdd(cnt + conn[i], 8);
}

// Exclusive scan of int32 in tiles of 2048 (8 per lane); tile totals to sums.
constexpr int SCAN_TILE = 2048;
__global__ __launch_bounds__(256) void scan_tile_kernel(const int32_t* in, int32_t* out, int64_t n, int32_t* sums) {
  __shared__ int32_t sh[256];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + 8 * threadIdx.x;
  int32_t v[8], run = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    v[j] = base + j < n ? in[base + j] : 0;
    run += v[j];
  }
  sh[threadIdx.x] = run;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {  // inclusive Hillis-Steele scan of the lane totals
    const int32_t t = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  int32_t acc = sh[threadIdx.x] - run;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (base + j < n) out[base + j] = acc;
    acc += v[j];
  }
  if (threadIdx.x == 255) sums[blockIdx.x] = sh[255];
}

__global__ void scan_add_kernel(int32_t* out, int64_t n, const int32_t* offs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += offs[i / SCAN_TILE];
}

__global__ void scan_total_kernel(int32_t* dst, const int32_t* src) { *dst = *src; }

// out[0..n) = exclusive scan of in, out[n] = total; tmp holds at least gen_scan_tmp_words(n) int32.
int64_t gen_scan_tmp_words(int64_t n) {
  int64_t w = 0;
  for (int64_t m = n; m > 1;) {
    m = (m + SCAN_TILE - 1) / SCAN_TILE;
    w += 2 * (m + 1);
  }
  return w + 2;
}

static hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int32_t* tmp, hipStream_t s) {
  const int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
  int32_t* sums = tmp;
  int32_t* offs = tmp + tiles + 1;
  hipLaunchKernelGGL(scan_tile_kernel, dim3((unsigned)std::max<int64_t>(tiles, 1)), dim3(256), 0, s, in, out, n, sums);
  if (tiles > 1) {
    hipError_t e = scan_exclusive(sums, offs, tiles, offs + tiles + 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(scan_add_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, n, offs);
    // total = offs[tiles] (the scan of the tile totals, one past its end)
    hipLaunchKernelGGL(scan_total_kernel, dim3(1), dim3(1), 0, s, out + n, offs + tiles);
  } else {
    hipLaunchKernelGGL(scan_total_kernel, dim3(1), dim3(1), 0, s, out + n, sums);
  }
  return hipGetLastError();
}

// Scatter every element's 64 node pairs into its row node's bucket: column node and the
// element code e * 64 + a * 8 + b (order inside a bucket is arbitrary; the row sort fixes it).
__global__ void sym_fill_kernel(int64_t ne, const int32_t* conn, int32_t* cursor, int32_t* col, int32_t* code) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 8 * ne; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e = i % ne;
    const int a = (int)(i / ne);
    const int pos = atomicAdd(cursor + conn[i], 8);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      col[pos + b] = conn[(int64_t)b * ne + e];
      code[pos + b] = (int32_t)(e * 64 + a * 8 + b);
    }
  }
}

// One wave per row: sort the row's bucket by the key (column, code) (all keys distinct: the
// code names the entry) by ranking, write it back in order and count the distinct columns.
constexpr int SYM_MAXROW = 1024;  // COO entries per row node (128 elements sharing a node)
__global__ __launch_bounds__(64) void sym_row_sort_kernel(int64_t n_nodes, const int32_t* ptr, int32_t* col,
                                                          int32_t* code, int32_t* deg) {
  __shared__ long long key[SYM_MAXROW];
  const int l = threadIdx.x;
  for (int64_t r = blockIdx.x; r < n_nodes; r += gridDim.x) {
    const int b = ptr[r], len = ptr[r + 1] - b;
    for (int j = l; j < len; j += 64) key[j] = ((long long)col[b + j] << 32) | (unsigned)code[b + j];
    __syncthreads();
    for (int j = l; j < len; j += 64) {
      const long long kj = key[j];
      int rank = 0;
      for (int i = 0; i < len; ++i) rank += key[i] < kj;
      col[b + rank] = (int32_t)(kj >> 32);
      code[b + rank] = (int32_t)(kj & 0xffffffffll);
    }
    __syncthreads();
    // distinct columns: count run heads of the sorted keys (sorted order = rank order)
    int heads = 0;
    for (int j = l; j < len; j += 64) {
      const long long kj = key[j];
      // kj is a run head when no key with the same column sorts before it
      bool head = true;
      for (int i = 0; i < len; ++i)
        if ((key[i] >> 32) == (kj >> 32) && key[i] < kj) {
          head = false;
          break;
        }
      heads += head;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) heads += __shfl_down(heads, off, 64);
    if (l == 0) deg[r] = heads;
    __syncthreads();
  }
}

// Pair arrays from the sorted buckets: for each run head at sorted position j of row r, its pair
// index is adj_ptr[r] + (heads before j); it records the column node, the row node and where
// its run starts in the sorted code list.  The codes then become 8 incidence + local column node, the
// incidence counted among those of the row (at most 128).
__global__ __launch_bounds__(64) void sym_pairs_kernel(int64_t n_nodes, const int32_t* ptr, const int32_t* col,
                                                       int32_t* code, const int32_t* adj_ptr, int32_t* adj,
                                                       int32_t* pair_row, int32_t* src_ptr, int32_t* inc_ptr,
                                                       int32_t* inc) {
  __shared__ int s_inc[SYM_MAXROW / 8];
  const int l = threadIdx.x;
  for (int64_t r = blockIdx.x; r < n_nodes; r += gridDim.x) {
    const int b = ptr[r], len = ptr[r + 1] - b;
    int run = adj_ptr[r], ii = b / 8;  // (8 entries per incidence)
    if (l == 0) {
      inc_ptr[r] = b / 8;
      if (r == n_nodes - 1) inc_ptr[n_nodes] = ptr[n_nodes] / 8;
    }
    for (int j0 = 0; j0 < len; j0 += 64) {
      const int j = j0 + l;
      // entries of the row's own column with equal local nodes: the incidences of the node, in
      // element order (an element that repeats a node, a collapsed brick, also pairs its copies)
      const int32_t cd = j < len ? code[b + j] : 0;  // element * 64 + local row node * 8 + local column node
      const bool self = j < len && col[b + j] == (int32_t)r && (cd >> 3 & 7) == (cd & 7);
      const unsigned long long ms = __ballot(self);
      if (self) {
        const int k = ii + __popcll(ms & ((1ull << l) - 1ull));
        inc[k] = s_inc[k - b / 8] = (cd >> 6) * 8 + (cd & 7);
      }
      ii += __popcll(ms);
      const bool head = j < len && (j == 0 || col[b + j] != col[b + j - 1]);
      const unsigned long long m = __ballot(head);
      const int before = __popcll(m & ((1ull << l) - 1ull));
      if (head) {
        const int pidx = run + before;
        adj[pidx] = col[b + j];
        pair_row[pidx] = (int32_t)r;
        src_ptr[pidx] = b + j;
      }
      run += __popcll(m);
    }
    __syncthreads();
    for (int j = l; j < len; j += 64) {
      const int32_t cd = code[b + j], mine = cd >> 3;
      int lo = 0, hi = len / 8 - 1;  // mine is one of s_inc, which ascends
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s_inc[mid] < mine) lo = mid + 1;
        else hi = mid;
      }
      code[b + j] = 8 * lo + (cd & 7);
    }
    __syncthreads();
  }
}

__global__ void sym_last_kernel(int32_t* src_ptr, int64_t n_pairs, int32_t total) { src_ptr[n_pairs] = total; }

// CSR indices of the dof-level matrix: 3 x 3 entries per node pair.
__global__ void gen_csr_pattern_kernel(int64_t n_pairs, int64_t n_nodes, const int32_t* adj_ptr, const int32_t* adj,
                                       const int32_t* pair_row, int32_t* row_ptr, int32_t* col_idx) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_pairs; p += (int64_t)gridDim.x * blockDim.x) {
    const int a = pair_row[p], b = adj[p];
    const int base = adj_ptr[a], deg = adj_ptr[a + 1] - base;
    const int64_t k = p - base;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int64_t pos = 9 * (int64_t)base + 3 * (int64_t)i * deg;
      if (k == 0) row_ptr[3 * (int64_t)a + i] = (int32_t)pos;
#pragma unroll
      for (int c = 0; c < 3; ++c) col_idx[pos + 3 * k + c] = 3 * b + c;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) row_ptr[3 * n_nodes] = (int32_t)(9 * n_pairs);
}

// ---------------------------------------------------------------------------
// geometry check (every Gauss point det J > 0) and the mesh volume sum_q w detJ

template <typename T>
__global__ __launch_bounds__(GBLOCK) void gen_volume_kernel(GenArgs g, int64_t ne, double* vol, int* bad) {
  __shared__ T s_c[GEL][8][3];
  __shared__ double sh[GBLOCK / 64];
  const int tid = threadIdx.x, el = tid >> 3, q = tid & 7;
  const int64_t e = (int64_t)blockIdx.x * GEL + el;
  const bool valid = e < ne;
  int node = 0;
  if (valid) node = g.conn[(int64_t)q * ne + e];
#pragma unroll
  for (int c = 0; c < 3; ++c) s_c[el][q][c] = valid ? static_cast<const T*>(g.coords)[3 * (int64_t)node + c] : T(0);
  __syncthreads();
  double v = 0;
  if (valid) {
    T gr[8][3];
    const T det = phys_grad<T>(s_c[el], q, gr);
    if (!(det > T(0))) atomicOr(bad, 1);
    v = (double)det;
  }
  v = block_sum(v, sh);
  if (threadIdx.x == 0) atomic_add(vol, v);
}

// u[3 node + c] = (eps . x_node)_c on constrained dofs; free dofs kept or zeroed.
template <typename T>
__global__ void gen_lift_kernel(int64_t n_nodes, const T* coords, const uint8_t* mask, T* u, int zero_free, double e00,
                                double e01, double e02, double e10, double e11, double e12, double e20, double e21,
                                double e22) {
  for (int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; d < 3 * n_nodes; d += (int64_t)gridDim.x * blockDim.x) {
    if (mask && mask[d]) {
      const int64_t P = d / 3;
      const int c = (int)(d % 3);
      const double x = coords[3 * P], y = coords[3 * P + 1], z = coords[3 * P + 2];
      const double v = c == 0 ? e00 * x + e01 * y + e02 * z : (c == 1 ? e10 * x + e11 * y + e12 * z : e20 * x + e21 * y + e22 * z);
      u[d] = T(v);
    } else if (zero_free) {
      u[d] = T(0);
    }
  }
}

// int32 node ids in range?  (bad |= 1 otherwise)
__global__ void gen_conn_check_kernel(int64_t n, const int32_t* conn, int64_t n_nodes, int* bad) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    if (conn[i] < 0 || conn[i] >= n_nodes) atomicOr(bad, 1);
}

template <typename T> __global__ void gen_fill_kernel(T* x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x[i] = T(0);
}

// coordinates [3][n] -> [n][3] (an element's gather then touches one place per node, not three)
template <typename D> __global__ void gen_coords_kernel(const double* a, D* b, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    for (int c = 0; c < 3; ++c) b[3 * i + c] = D(a[c * n + i]);
}

template <typename T> __global__ void gen_copy_kernel(const T* a, T* b, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = a[i];
}

// ---------------------------------------------------------------------------
// launchers

static unsigned vblocks(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }
static unsigned eblocks(int64_t ne) { return (unsigned)std::max<int64_t>(1, (ne + GEL - 1) / GEL); }

hipError_t gen_setup(fe_problem* p, const double* coords, const int32_t* conn, hipStream_t s) {
  const int64_t ne = p->n_el, nn = p->n_nodes;
  int* bad = p->flags;
  hipError_t e;
  if ((e = hipMemsetAsync(bad, 0, sizeof(int), s)) != hipSuccess) return e;
  hipLaunchKernelGGL(gen_conn_check_kernel, dim3(vblocks(8 * ne)), dim3(256), 0, s, 8 * ne, conn, nn, bad);
  if (p->prec == FE_F64)
    hipLaunchKernelGGL(gen_coords_kernel<double>, dim3(vblocks(nn)), dim3(256), 0, s, coords, (double*)p->coords, nn);
  else
    hipLaunchKernelGGL(gen_coords_kernel<float>, dim3(vblocks(nn)), dim3(256), 0, s, coords, (float*)p->coords, nn);
  hipLaunchKernelGGL(gen_copy_kernel<int32_t>, dim3(vblocks(8 * ne)), dim3(256), 0, s, conn, p->conn, 8 * ne);
  return hipGetLastError();
}

hipError_t gen_check_geometry(const fe_problem* p, double* vol_dev, int* bad, hipStream_t s) {
  const GenArgs g = gen_args(p);
  if (p->prec == FE_F64)
    hipLaunchKernelGGL(gen_volume_kernel<double>, dim3(eblocks(p->n_el)), dim3(GBLOCK), 0, s, g, p->n_el, vol_dev, bad);
  else
    hipLaunchKernelGGL(gen_volume_kernel<float>, dim3(eblocks(p->n_el)), dim3(GBLOCK), 0, s, g, p->n_el, vol_dev, bad);
  return hipGetLastError();
}

// Node-pair pattern: counts, bucket offsets, buckets, row sorts, degrees, pair arrays.
// Returns the number of pairs in *n_pairs (synchronises).  tmp: gen_scan_tmp_words(n_nodes) words.
hipError_t gen_symbolic(fe_problem* p, int32_t* cnt, int32_t* coo_ptr, int32_t* cursor, int32_t* tmp, hipStream_t s,
                        int64_t* n_pairs, int* max_row) {
  const int64_t ne = p->n_el, nn = p->n_nodes;
  hipError_t e;
  if ((e = hipMemsetAsync(cnt, 0, sizeof(int32_t) * nn, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(sym_count_kernel, dim3(vblocks(8 * ne)), dim3(256), 0, s, ne, p->conn, cnt);
  if ((e = scan_exclusive(cnt, coo_ptr, nn, tmp, s)) != hipSuccess) return e;
  // longest bucket (host check against the row-sort capacity)
  std::vector<int32_t> h(nn + 1);
  if ((e = hipMemcpyAsync(h.data(), coo_ptr, sizeof(int32_t) * (nn + 1), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  int mx = 0;
  for (int64_t i = 0; i < nn; ++i) mx = std::max(mx, h[i + 1] - h[i]);
  *max_row = mx;
  if (mx > SYM_MAXROW) return hipSuccess;  // caller reports
  if ((e = hipMemcpyAsync(cursor, coo_ptr, sizeof(int32_t) * nn, hipMemcpyDeviceToDevice, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(sym_fill_kernel, dim3(vblocks(8 * ne)), dim3(256), 0, s, ne, p->conn, cursor, p->gen_col,
                     p->pair_src);
  const unsigned rows_grid = (unsigned)std::min<int64_t>(nn, 65536);
  hipLaunchKernelGGL(sym_row_sort_kernel, dim3(rows_grid), dim3(64), 0, s, nn, coo_ptr, p->gen_col, p->pair_src, cnt);
  if ((e = scan_exclusive(cnt, p->adj_ptr, nn, tmp, s)) != hipSuccess) return e;
  int32_t np = 0;
  if ((e = hipMemcpyAsync(&np, p->adj_ptr + nn, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  *n_pairs = np;
  return hipSuccess;
}

hipError_t gen_pairs(fe_problem* p, const int32_t* coo_ptr, hipStream_t s) {
  const int64_t nn = p->n_nodes;
  const unsigned rows_grid = (unsigned)std::min<int64_t>(nn, 65536);
  hipLaunchKernelGGL(sym_pairs_kernel, dim3(rows_grid), dim3(64), 0, s, nn, coo_ptr, p->gen_col, p->pair_src,
                     p->adj_ptr, p->adj, p->pair_row, p->pair_src_ptr, p->inc_ptr, p->inc);
  hipLaunchKernelGGL(sym_last_kernel, dim3(1), dim3(1), 0, s, p->pair_src_ptr, p->n_pairs, (int32_t)(64 * p->n_el));
  return hipGetLastError();
}

hipError_t gen_csr_pattern(const fe_problem* p, int32_t* row_ptr, int32_t* col_idx, hipStream_t s) {
  hipLaunchKernelGGL(gen_csr_pattern_kernel, dim3(vblocks(p->n_pairs)), dim3(256), 0, s, p->n_pairs, p->n_nodes,
                     p->adj_ptr, p->adj, p->pair_row, row_ptr, col_idx);
  return hipGetLastError();
}

// Element kernel with the nodal forces to p->gen_elf.
template <typename T, bool CG>
static hipError_t gen_elf_t(const fe_problem* p, const ElemArgs& a, const int* stop, hipStream_t s) {
  const GenArgs g = gen_args(p);
  const dim3 grid(eblocks(p->n_el)), block(GBLOCK);
  ElemArgs b = a;
  b.elf = p->gen_elf;
  switch (p->model_set) {
    case MS_J2: timed_launch((gen_elem_kernel<T, OP_APPLY, MS_J2, true, CG>), grid, block, 0, s, g, b, stop); break;
    case MS_NH: timed_launch((gen_elem_kernel<T, OP_APPLY, MS_NH, true, CG>), grid, block, 0, s, g, b, stop); break;
    default: timed_launch((gen_elem_kernel<T, OP_APPLY, MS_LINEAR, true, CG>), grid, block, 0, s, g, b, stop);
  }
  return hipGetLastError();
}

// Solver operator y = A x through the element forces (the caller owns the problem's workspaces).
template <typename T>
static hipError_t gen_solver_operator_t(const fe_problem* p, const ElemArgs& a, const int* stop, hipStream_t s) {
  hipError_t e = gen_elf_t<T, false>(p, a, stop, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gen_gather_kernel<T>, dim3(vblocks(p->n_dof)), dim3(VBLOCK), 0, s, p->n_dof, p->inc_ptr, p->inc,
                     (const T*)p->gen_elf, a.apply_bc ? p->mask : nullptr, (const T*)a.x, (T*)a.y, stop);
  return hipGetLastError();
}

// slots of the general CG in the problem's partial sums: GCG_Q quantities of iterate j, (p_j, A p_j)
static double* gcg_acc(const fe_problem* p, long j) { return p->partials + (j & 1) * GCG_Q * GCG_SLOTS; }
static double* gcg_pq(const fe_problem* p, long j) { return p->partials + (2 * GCG_Q + (j & 1)) * GCG_SLOTS; }

template <typename T>
static hipError_t gen_cg_node_t(const fe_problem* p, const void* b, void* x, long j, hipStream_t s) {
  GenCgArgs a{};
  a.n_nodes = p->n_nodes;
  a.j = j;
  a.inc_ptr = p->inc_ptr;
  a.inc = p->inc;
  a.elf = p->gen_elf;
  a.mask = p->mask;
  a.b = b;
  a.r = p->w_r;
  a.p = p->w_p;
  a.pf = static_cast<T*>(p->gen_elf) + 24 * p->n_el;
  a.x = x;
  a.u = p->w_q;
  a.dinv = pc_buffer(p);
  a.ctrl = p->ctrl;
  a.pq_in = gcg_pq(p, j);
  a.pq_zero = gcg_pq(p, j + 1);
  a.acc_out = gcg_acc(p, j + 1);
  const int64_t waves = (p->n_nodes + CGN_NODES - 1) / CGN_NODES;
  const dim3 grid((unsigned)((waves + VBLOCK / 64 - 1) / (VBLOCK / 64))), block(VBLOCK);
  const bool blk = p->precond == FE_PC_BLOCK_JACOBI;
  if (j < 0) {
    if (blk) hipLaunchKernelGGL((gen_cg_node_kernel<T, true, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((gen_cg_node_kernel<T, false, true>), grid, block, 0, s, a);
  } else {
    if (blk) hipLaunchKernelGGL((gen_cg_node_kernel<T, true, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((gen_cg_node_kernel<T, false, false>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t gen_cgs_init(const fe_problem* p, const void* b, void* x, double rtol, int max_it, hipStream_t s) {
  hipLaunchKernelGGL(gen_cg_start_kernel, dim3(1), dim3(256), 0, s, p->ctrl, rtol, max_it, p->partials);
  return p->prec == FE_F64 ? gen_cg_node_t<double>(p, b, x, -1, s) : gen_cg_node_t<float>(p, b, x, -1, s);
}

hipError_t gen_cgs_operator(const fe_problem* p, long j, hipStream_t s) {
  ElemArgs a{};
  a.n_el = p->n_el;
  a.phase = p->phase;
  a.scale = p->scale;
  a.tangent = p->tangent;
  a.mat = p->mat;
  a.x = p->w_q;
  a.cg_j = j;
  a.cg_pvec = p->w_p;
  a.ctrl = p->ctrl;
  a.cg_acc_in = gcg_acc(p, j);
  a.cg_acc_zero = gcg_acc(p, j + 1);
  a.cg_acc_out = gcg_pq(p, j);
  const int* stop = &p->ctrl->status;
  return p->prec == FE_F64 ? gen_elf_t<double, true>(p, a, stop, s) : gen_elf_t<float, true>(p, a, stop, s);
}

hipError_t gen_cgs_update(const fe_problem* p, void* x, long j, hipStream_t s) {
  return p->prec == FE_F64 ? gen_cg_node_t<double>(p, nullptr, x, j, s) : gen_cg_node_t<float>(p, nullptr, x, j, s);
}

template <typename T, int OP>
static hipError_t gen_elem_t(const fe_problem* p, const ElemArgs& a, const int* stop, hipStream_t s) {
  // operators of a running solver (they pass its status word) own the problem's workspaces; a
  // plain K x may run beside others of the same problem on other streams and keeps to atomics
  if constexpr (OP == OP_APPLY)
    if (stop && p->gen_elf) return gen_solver_operator_t<T>(p, a, stop, s);
  const GenArgs g = gen_args(p);
  const dim3 grid(eblocks(p->n_el)), block(GBLOCK);
  switch (p->model_set) {
    case MS_J2: timed_launch((gen_elem_kernel<T, OP, MS_J2>), grid, block, 0, s, g, a, stop); break;
    case MS_NH: timed_launch((gen_elem_kernel<T, OP, MS_NH>), grid, block, 0, s, g, a, stop); break;
    default: timed_launch((gen_elem_kernel<T, OP, MS_LINEAR>), grid, block, 0, s, g, a, stop);
  }
  if (OP == OP_APPLY && a.apply_bc && p->mask && a.y)
    hipLaunchKernelGGL(gen_bc_kernel<T>, dim3(vblocks(p->n_dof)), dim3(VBLOCK), 0, s, p->n_dof, p->mask,
                       (const T*)a.x, (T*)a.y, stop, (double*)nullptr);
  return hipGetLastError();
}

hipError_t gen_launch_elem(const fe_problem* p, int op, const ElemArgs& a, const int* stop, hipStream_t s) {
  if (op == OP_CG_APPLY) return hipErrorInvalidValue;  // (CG has launches of its own: gen_cgs_operator, gen_cgs_update)
  if (p->prec == FE_F64) {
    if (op == OP_RESID) return gen_elem_t<double, OP_RESID>(p, a, stop, s);
    if (op == OP_APPLY) return gen_elem_t<double, OP_APPLY>(p, a, stop, s);
    return gen_elem_t<double, OP_VJP>(p, a, stop, s);
  }
  if (op == OP_RESID) return gen_elem_t<float, OP_RESID>(p, a, stop, s);
  if (op == OP_APPLY) return gen_elem_t<float, OP_APPLY>(p, a, stop, s);
  return gen_elem_t<float, OP_VJP>(p, a, stop, s);
}

// CG operator on a general mesh: q = A p (q zeroed by the previous update), then the
// constrained rows and the per-workgroup partials of p.q.
hipError_t gen_cg_operator(const fe_problem* p, hipStream_t s) {
  ElemArgs a{};
  a.n_el = p->n_el;
  a.phase = p->phase;
  a.scale = p->scale;
  a.mask = p->mask;
  a.tangent = p->tangent;
  a.flags = p->flags;
  a.mat = p->mat;
  a.x = p->w_p;
  a.y = p->w_q;
  a.apply_bc = 1;
  const int* stop = &p->ctrl->status;
  const GenArgs g = gen_args(p);
  const dim3 grid(eblocks(p->n_el)), block(GBLOCK);
  if (p->prec == FE_F64) {
    switch (p->model_set) {
      case MS_J2: timed_launch((gen_elem_kernel<double, OP_APPLY, MS_J2>), grid, block, 0, s, g, a, stop); break;
      case MS_NH: timed_launch((gen_elem_kernel<double, OP_APPLY, MS_NH>), grid, block, 0, s, g, a, stop); break;
      default: timed_launch((gen_elem_kernel<double, OP_APPLY, MS_LINEAR>), grid, block, 0, s, g, a, stop);
    }
    hipLaunchKernelGGL(gen_bc_kernel<double>, dim3(GEN_CG_GRID), dim3(VBLOCK), 0, s, p->n_dof, p->mask,
                       (const double*)p->w_p, (double*)p->w_q, stop, p->partials);
  } else {
    switch (p->model_set) {
      case MS_J2: timed_launch((gen_elem_kernel<float, OP_APPLY, MS_J2>), grid, block, 0, s, g, a, stop); break;
      case MS_NH: timed_launch((gen_elem_kernel<float, OP_APPLY, MS_NH>), grid, block, 0, s, g, a, stop); break;
      default: timed_launch((gen_elem_kernel<float, OP_APPLY, MS_LINEAR>), grid, block, 0, s, g, a, stop);
    }
    hipLaunchKernelGGL(gen_bc_kernel<float>, dim3(GEN_CG_GRID), dim3(VBLOCK), 0, s, p->n_dof, p->mask,
                       (const float*)p->w_p, (float*)p->w_q, stop, p->partials);
  }
  return hipGetLastError();
}

template <typename T>
static hipError_t gen_diag_t(const fe_problem* p, T* d, int nb, int apply_bc, const TanArgs& ta, hipStream_t s) {
  const GenArgs g = gen_args(p);
  const int64_t n = nb == 3 ? p->n_dof : 6 * p->n_nodes;
  hipLaunchKernelGGL(gen_fill_kernel<T>, dim3(vblocks(n)), dim3(256), 0, s, d, n);
  const dim3 grid(eblocks(p->n_el)), block(GBLOCK);
  const int skip = apply_bc && p->mask ? 1 : 0;
  if (nb == 3) {
    switch (p->model_set) {
      case MS_J2: hipLaunchKernelGGL((gen_diag_kernel<T, MS_J2, 3>), grid, block, 0, s, g, ta, d, skip); break;
      case MS_NH: hipLaunchKernelGGL((gen_diag_kernel<T, MS_NH, 3>), grid, block, 0, s, g, ta, d, skip); break;
      default: hipLaunchKernelGGL((gen_diag_kernel<T, MS_LINEAR, 3>), grid, block, 0, s, g, ta, d, skip);
    }
    if (skip) hipLaunchKernelGGL(gen_mask_one_kernel<T>, dim3(vblocks(p->n_dof)), dim3(256), 0, s, p->n_dof, p->mask, d);
  } else {
    switch (p->model_set) {
      case MS_J2: hipLaunchKernelGGL((gen_diag_kernel<T, MS_J2, 6>), grid, block, 0, s, g, ta, d, 0); break;
      case MS_NH: hipLaunchKernelGGL((gen_diag_kernel<T, MS_NH, 6>), grid, block, 0, s, g, ta, d, 0); break;
      default: hipLaunchKernelGGL((gen_diag_kernel<T, MS_LINEAR, 6>), grid, block, 0, s, g, ta, d, 0);
    }
  }
  return hipGetLastError();
}

hipError_t gen_diag(const fe_problem* p, void* d, int nb, int apply_bc, const TanArgs& ta, hipStream_t s) {
  return p->prec == FE_F64 ? gen_diag_t(p, (double*)d, nb, apply_bc, ta, s) : gen_diag_t(p, (float*)d, nb, apply_bc, ta, s);
}

template <typename T>
static hipError_t gen_tangent_t(const fe_problem* p, T* vals, int apply_bc, const TanArgs& ta, hipStream_t s) {
  const GenArgs g = gen_args(p);
  T* ke = static_cast<T*>(p->ke);
  const dim3 grid((unsigned)((p->n_el + TEL - 1) / TEL)), block(TBLOCK);
  switch (p->model_set) {
    case MS_J2: timed_launch((gen_tangent_kernel<T, MS_J2>), grid, block, 0, s, g, ta, ke); break;
    case MS_NH: timed_launch((gen_tangent_kernel<T, MS_NH>), grid, block, 0, s, g, ta, ke); break;
    default: timed_launch((gen_tangent_kernel<T, MS_LINEAR>), grid, block, 0, s, g, ta, ke);
  }
  const unsigned ablocks = (unsigned)((p->n_nodes + ASM_WAVES - 1) / ASM_WAVES);
  hipLaunchKernelGGL(gen_assemble_kernel<T>, dim3(ablocks), dim3(VBLOCK), 0, s, p->n_nodes, p->adj_ptr, p->adj,
                     p->pair_src_ptr, p->pair_src, p->inc_ptr, p->inc, (const T*)ke, p->mask, apply_bc, vals);
  return hipGetLastError();
}

hipError_t gen_tangent(const fe_problem* p, void* vals, int apply_bc, const TanArgs& ta, hipStream_t s) {
  return p->prec == FE_F64 ? gen_tangent_t(p, (double*)vals, apply_bc, ta, s)
                           : gen_tangent_t(p, (float*)vals, apply_bc, ta, s);
}

hipError_t gen_lift(const fe_problem* p, const double* E, void* u, int zero_free, hipStream_t s) {
  const dim3 gr(vblocks(p->n_dof)), b(256);
  if (p->prec == FE_F64)
    hipLaunchKernelGGL(gen_lift_kernel<double>, gr, b, 0, s, p->n_nodes, (const double*)p->coords, p->mask, (double*)u,
                       zero_free, E[0], E[1], E[2], E[3], E[4], E[5], E[6], E[7], E[8]);
  else
    hipLaunchKernelGGL(gen_lift_kernel<float>, gr, b, 0, s, p->n_nodes, (const float*)p->coords, p->mask, (float*)u,
                       zero_free, E[0], E[1], E[2], E[3], E[4], E[5], E[6], E[7], E[8]);
  return hipGetLastError();
}

hipError_t gen_copy_state(const fe_problem* p, const void* src, void* dst, int64_t n, hipStream_t s) {
  if (p->prec == FE_F64)
    hipLaunchKernelGGL(gen_copy_kernel<double>, dim3(vblocks(n)), dim3(256), 0, s, (const double*)src, (double*)dst, n);
  else
    hipLaunchKernelGGL(gen_copy_kernel<float>, dim3(vblocks(n)), dim3(256), 0, s, (const float*)src, (float*)dst, n);
  return hipGetLastError();
}

}  // namespace fe
