// Node-block ILU(0) preconditioner in an 8-colour node order (needs the assembled CSR).
//
// Sec. V-B (Fig. 7) compares Jacobi with ILU preconditioning of the assembled matrix.
// A natural-order ILU(0) on this mesh has ~7n dependency levels per triangular solve,
// one launch (or grid barrier) each; colouring the nodes by the parities of their grid
// indices leaves 8 levels: no two nodes of one colour share an element, so every colour
// is factored and solved data-parallel.  Blocks are the 3x3 couplings of node pairs; no fill
// outside the block pattern (node pairs sharing an element).
//
// Two colours that differ in the x parity alone only couple along the x-rows of the grid, so a
// sweep takes one launch per class of rows (parities of j and k: colour = (i & 1) + 2 class) with
// one workgroup per row, the two colours in turn behind a workgroup barrier; the last class is
// swept forward and back in one launch: 7 launches an application in place of 16 (colour by
// colour, one lane per node: 36 workgroups at 32^3, 190 us an application; so 48 us; 64^3 316 -> 220 us).
//
// Factor storage: one record of 243 reals per node, nodes by class, then row, then i.  A record
// holds the blocks of the neighbour rows of lower class [9][nL], of the two neighbours in the own
// row [9][2], the inverse of the pivot block [9], and the blocks of the rows of higher class
// [9][nU]; nL = 0, 6, 18, 24 neighbours for class 0 .. 3, nU = 24 - nL.  A sweep reads exactly one
// contiguous part of each record, eight lanes per node, three neighbours per lane.  Slots of the
// factorisation: s = (di+1) + 3 (dj+1) + 9 (dk+1); the colour of i + (di, dj, dk) is colour(i) XOR
// m with m = [di != 0] + 2 [dj != 0] + 4 [dk != 0].

#include <cmath>

#include "fe_internal.hpp"

namespace fe {

namespace {

constexpr int REC = 243;       // reals per node
constexpr int FACTOR_B = 128;  // lanes per workgroup of the factorisation (4 nodes)

// Neighbour rows (dj+1) + 3 (dk+1) of a class in record order: lower classes first.
__device__ __constant__ const int8_t ROW_AT[4][8] = {
    {0, 1, 2, 3, 5, 6, 7, 8}, {3, 5, 0, 1, 2, 6, 7, 8}, {0, 1, 2, 6, 7, 8, 3, 5}, {0, 1, 2, 3, 5, 6, 7, 8}};
__device__ __constant__ const int8_t POS_OF[4][9] = {
    {0, 1, 2, 3, -1, 4, 5, 6, 7}, {2, 3, 4, 0, -1, 1, 5, 6, 7}, {0, 1, 2, 6, -1, 7, 3, 4, 5}, {0, 1, 2, 3, -1, 4, 5, 6, 7}};
__host__ __device__ constexpr int n_lower(int q) { return q == 0 ? 0 : (q == 1 ? 6 : (q == 2 ? 18 : 24)); }

struct Rows {
  int n;
  int cnt[2];      // grid indices in [0, n] of parity 0 and 1
  int64_t off[5];  // first node (in record order) of each class
};

Rows row_classes(int n) {
  Rows c{};
  c.n = n;
  c.cnt[0] = (n + 2) / 2;
  c.cnt[1] = (n + 1) / 2;
  c.off[0] = 0;
  for (int q = 0; q < 4; ++q) c.off[q + 1] = c.off[q] + (int64_t)c.cnt[q & 1] * c.cnt[q >> 1] * (n + 1);
  return c;
}

// record of node (i, j, k)
__device__ __forceinline__ int64_t record(const Rows& c, int i, int j, int k) {
  const int q = (j & 1) + 2 * (k & 1);
  return REC * (c.off[q] + i + (int64_t)(c.n + 1) * ((j >> 1) + (int64_t)c.cnt[q & 1] * (k >> 1)));
}

// where entry e of slot s sits in a record of class q: at + e * step
__device__ __forceinline__ void slot_place(int q, int s, int& at, int& step) {
  const int nl = n_lower(q), r9 = s / 3, di = s % 3;
  if (r9 == 4) {
    at = di == 1 ? 9 * nl + 18 : 9 * nl + (di >> 1);
    step = di == 1 ? 1 : 2;
    return;
  }
  const int pos = POS_OF[q][r9], nlr = nl / 3;
  if (pos < nlr) {
    at = 3 * pos + di;
    step = nl;
  } else {
    at = 9 * nl + 27 + 3 * (pos - nlr) + di;
    step = 24 - nl;
  }
}

__device__ __forceinline__ int slot_mask(int s) {
  return (s % 3 != 1 ? 1 : 0) | ((s / 3) % 3 != 1 ? 2 : 0) | (s / 9 != 1 ? 4 : 0);
}

// 3x3 inverse by the adjugate; false when singular or not finite
__device__ __forceinline__ bool inverse3(const double a[9], double r[9]) {
  const double c00 = a[4] * a[8] - a[5] * a[7], c01 = a[5] * a[6] - a[3] * a[8], c02 = a[3] * a[7] - a[4] * a[6];
  const double det = a[0] * c00 + a[1] * c01 + a[2] * c02;
  if (!(det != 0.0) || !(det - det == 0.0)) return false;
  const double id = 1.0 / det;
  r[0] = c00 * id;
  r[1] = (a[2] * a[7] - a[1] * a[8]) * id;
  r[2] = (a[1] * a[5] - a[2] * a[4]) * id;
  r[3] = c01 * id;
  r[4] = (a[0] * a[8] - a[2] * a[6]) * id;
  r[5] = (a[2] * a[3] - a[0] * a[5]) * id;
  r[6] = c02 * id;
  r[7] = (a[1] * a[6] - a[0] * a[7]) * id;
  r[8] = (a[0] * a[4] - a[1] * a[3]) * id;
  return true;
}

// Row ri of the block of column node nb in CSR row 3 node + ri (columns sorted; entries that are
// not stored are 0).  guess: where the three columns start in the node-structured pattern, tested
// first; any other pattern is searched.
template <typename T>
__device__ __forceinline__ void csr_block_row(const int32_t* rp, const int32_t* ci, const T* v, int64_t row,
                                              int64_t nb, int guess, double out[3]) {
  const int b = rp[row], e = rp[row + 1];
  const int32_t want = (int32_t)(3 * nb);
  int lo = b + guess;
  if (!(lo + 2 < e && ci[lo] == want && ci[lo + 1] == want + 1 && ci[lo + 2] == want + 2 &&
        (lo == b || ci[lo - 1] < want))) {
    lo = b;
    int hi = e - 1;
    while (lo < hi) {  // first column >= 3 nb (sorted row)
      const int mid = (lo + hi) >> 1;
      if (ci[mid] < want) lo = mid + 1;
      else hi = mid;
    }
  }
  out[0] = out[1] = out[2] = 0;
  for (int q = lo; q < e && ci[q] < want + 3; ++q)
    if (ci[q] >= want) {
      const int k = ci[q] - want;
      const double x = (double)v[q];
      out[0] = k == 0 ? x : out[0];
      out[1] = k == 1 ? x : out[1];
      out[2] = k == 2 ? x : out[2];
    }
}

// Factor the rows of colour col (all lower colours are final), 32 lanes per node, lane = slot,
// the row's blocks in registers: for each lower neighbour k in colour order, L_ik = A_ik U_kk^-1
// (formed by its lane, broadcast) and A_ij -= L_ik U_kj for the later j of both patterns; then
// slot 13 <- U_ii^-1.
template <typename T>
__global__ __launch_bounds__(FACTOR_B) void ilu_factor_kernel(Rows c, int col, const int32_t* rp, const int32_t* ci,
                                                              const T* v, T* F, unsigned int* flags) {
  const int n = c.n, q = col >> 1;
  const int s = threadIdx.x & 31, base_lane = threadIdx.x & 32;
  const int cx = c.cnt[col & 1], cy = c.cnt[q & 1], cz = c.cnt[q >> 1];
  const int64_t count = (int64_t)cx * cy * cz;
  const int64_t t0 = (int64_t)blockIdx.x * (FACTOR_B / 32) + (threadIdx.x >> 5);
  const bool live = t0 < count;  // (idle groups keep their lanes for the exchanges of the wave)
  const int64_t t = live ? t0 : 0;
  const int i = 2 * (int)(t % cx) + (col & 1), j = 2 * (int)((t / cx) % cy) + (q & 1), k = 2 * (int)(t / ((int64_t)cx * cy)) + (q >> 1);
  const int di = s % 3 - 1, dj = (s / 3) % 3 - 1, dk = s / 9 - 1;
  const int a = i + di, b = j + dj, d = k + dk;
  const bool in = s < 27 && a >= 0 && a <= n && b >= 0 && b <= n && d >= 0 && d <= n;
  const int mine = col ^ slot_mask(s);  // colour of this lane's column node
  double B[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (live && in) {
    const int64_t node = i + (int64_t)(n + 1) * (j + (int64_t)(n + 1) * k);
    const int64_t nb = a + (int64_t)(n + 1) * (b + (int64_t)(n + 1) * d);
    // rank of the neighbour among the (2 or 3 per axis) neighbours of the node
    const int wx = (i > 0) + (i < n) + 1, wy = (j > 0) + (j < n) + 1;
    const int rank = ((dk + (k > 0)) * wy + (dj + (j > 0))) * wx + (di + (i > 0));
#pragma unroll
    for (int r = 0; r < 3; ++r) csr_block_row(rp, ci, v, 3 * node + r, nb, 3 * rank, B + 3 * r);
  }
  for (int kc = 0; kc < col; ++kc) {
    const int m = col ^ kc;
    for (int sk = 0; sk < 27; ++sk) {
      if (slot_mask(sk) != m) continue;
      const int ox = sk % 3 - 1, oy = (sk / 3) % 3 - 1, oz = sk / 9 - 1;
      const int ka = i + ox, kb = j + oy, kd = k + oz;
      const bool kin = live && ka >= 0 && ka <= n && kb >= 0 && kb <= n && kd >= 0 && kd <= n;
      // U_kj of this lane's column node j, when j comes after k and is adjacent to it
      const int dx = di - ox, dy = dj - oy, dz = dk - oz;
      const bool upd = kin && in && mine > kc && dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1;
      const T* K = F + (kin ? record(c, ka, kb, kd) : 0);
      const int qk = (kb & 1) + 2 * (kd & 1);
      int at, step;
      slot_place(qk, upd ? (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1) : 13, at, step);  // (its own lane: U_kk^-1)
      double u[9], L[9];
      const bool own = kin && s == sk;
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = upd || own ? (double)K[at + e * step] : 0.0;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) L[3 * r + cc] = B[3 * r] * u[cc] + B[3 * r + 1] * u[3 + cc] + B[3 * r + 2] * u[6 + cc];
      if (own) {
#pragma unroll
        for (int e = 0; e < 9; ++e) B[e] = L[e];
      }
#pragma unroll
      for (int e = 0; e < 9; ++e) L[e] = __shfl(L[e], base_lane + sk, 64);
      if (upd) {
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int cc = 0; cc < 3; ++cc)
            B[3 * r + cc] -= L[3 * r] * u[cc] + L[3 * r + 1] * u[3 + cc] + L[3 * r + 2] * u[6 + cc];
      }
    }
  }
  if (!live || s >= 27) return;
  if (s == 13) {
    double di9[9];
    if (!inverse3(B, di9)) {
      atomicOr(flags, 4u);
#pragma unroll
      for (int e = 0; e < 9; ++e) di9[e] = NAN;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) B[e] = di9[e];
  }
  T* R = F + record(c, i, j, k);
  int at, step;
  slot_place(q, s, at, step);
#pragma unroll
  for (int e = 0; e < 9; ++e) R[at + e * step] = T(B[e]);
}

// v + the values of the other lanes of the aligned group of 8 (every lane gets the sum)
template <int CTRL> __device__ __forceinline__ double lane_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double sum8(double v) {
  v = lane_add<0x141>(v);   // row_half_mirror: q <- 7 - q
  v = lane_add<0x4E>(v);    // quad_perm: q ^ 2
  return lane_add<0xB1>(v); // q ^ 1
}

// One x-row of class Q per workgroup, eight lanes per node.  FORWARD:
//   z_i = r_i - sum over lower rows, then (odd i) over the two neighbours in the row, of L_ij z_j;
// class 3, which no other row waits for, is swept back at once.  Otherwise back:
//   z_i = U_ii^-1 (z_i - sum over higher rows, then (even i) over the row, of U_ij z_j), odd i first.
// The row's values live in LDS ([3 (n + 1)] doubles); reads of other rows are of finished classes.
template <typename T, int Q, bool FORWARD>
__global__ __launch_bounds__(1024) void ilu_sweep_kernel(Rows c, const T* __restrict__ F, const T* r, T* z, const int* stop) {
  extern __shared__ double s_y[];
  if (stop && *stop) return;
  constexpr int NL = n_lower(Q), NU = 24 - NL;
  constexpr int CNT = FORWARD ? NL : NU;                   // neighbours in other rows
  constexpr int SEC = FORWARD ? 0 : 9 * NL + 27;           // their blocks' place in the record
  constexpr int ROW0 = FORWARD ? 0 : NL / 3;
  const int n = c.n, np1 = n + 1;
  const int cy = c.cnt[Q & 1];
  const int j = 2 * ((int)blockIdx.x % cy) + (Q & 1), k = 2 * ((int)blockIdx.x / cy) + (Q >> 1);
  const int t = threadIdx.x & 7, groups = blockDim.x >> 3;
  const int64_t row_node = (int64_t)np1 * (j + (int64_t)np1 * k);
  const T* RF = F + record(c, 0, j, k);
  const T* src = FORWARD ? r : z;
  // the blocks that couple the row (lanes 0-2: row t of the block of i - 1, lanes 3-5: of i + 1) and
  // the pivot's inverse (lanes 0-2), requested at once with the rest for the first pass over the row
  // (a group's only one while 8 (n + 1) <= 1024), since each use is behind a barrier
  const int e3 = t % 3, side = t / 3;
  auto row_words = [&](int i, double w[3]) {
    const T* B = RF + (int64_t)REC * i + 9 * NL + side + 6 * e3;
    const int a = i + 2 * side - 1;
    const bool ok = t < 6 && i < np1 && a >= 0 && a <= n;
#pragma unroll
    for (int q = 0; q < 3; ++q) w[q] = ok ? (double)B[2 * q] : 0.0;
  };
  auto pivot_words = [&](int i, double w[3]) {
    const T* D = RF + (int64_t)REC * i + 9 * NL + 18 + 3 * e3;
#pragma unroll
    for (int q = 0; q < 3; ++q) w[q] = t < 3 && i < np1 ? (double)D[q] : 0.0;
  };
  constexpr bool BACK = !FORWARD || Q == 3;
  double rw0[3], pw0[3] = {0, 0, 0};
  row_words(threadIdx.x >> 3, rw0);
  if (BACK) pivot_words(threadIdx.x >> 3, pw0);
  for (int i0 = 0; i0 < np1; i0 += groups) {
    const int i = i0 + (threadIdx.x >> 3);
    const bool live = i < np1;
    double acc[3] = {0, 0, 0};
    if (live && CNT > 0) {
      const T* B = RF + (int64_t)REC * i + SEC;
#pragma unroll
      for (int u = 0; u < (CNT + 7) / 8; ++u) {
        const int nb = t + 8 * u;
        const int row = ROW_AT[Q][ROW0 + (nb < CNT ? nb / 3 : 0)];
        const int a = i + nb % 3 - 1, b = j + row % 3 - 1, d = k + row / 3 - 1;
        if (nb < CNT && a >= 0 && a <= n && b >= 0 && b <= n && d >= 0 && d <= n) {
          const T* x = z + 3 * (a + (int64_t)np1 * (b + (int64_t)np1 * d));
          const double x0 = (double)x[0], x1 = (double)x[1], x2 = (double)x[2];
#pragma unroll
          for (int e = 0; e < 3; ++e)
            acc[e] += (double)B[(3 * e) * CNT + nb] * x0 + (double)B[(3 * e + 1) * CNT + nb] * x1 +
                      (double)B[(3 * e + 2) * CNT + nb] * x2;
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) acc[e] = CNT > 0 ? sum8(acc[e]) : 0.0;
    if (live && t < 3)
      s_y[3 * i + t] = (double)src[3 * (row_node + i) + t] - (t == 0 ? acc[0] : (t == 1 ? acc[1] : acc[2]));
  }
  __syncthreads();
  // coupling inside the row: the nodes of one parity take off their neighbours' finished values
  // and / or are multiplied by U_ii^-1
  auto couple = [&](int par, bool neighbours, bool scale) {
    for (int i0 = 0; i0 < np1; i0 += groups) {
      const int i = i0 + (threadIdx.x >> 3);
      const bool live = i < np1 && (i & 1) == par;
      double y = live && t < 3 ? s_y[3 * i + t] : 0.0;
      if (neighbours) {
        double rw[3] = {rw0[0], rw0[1], rw0[2]}, w = 0;
        if (i0 > 0) row_words(i, rw);
        const int a = i + 2 * side - 1;
        if (live && t < 6 && a >= 0 && a <= n) w = rw[0] * s_y[3 * a] + rw[1] * s_y[3 * a + 1] + rw[2] * s_y[3 * a + 2];
        y -= w + __shfl_down(w, 3, 8);
      }
      if (scale) {
        double pw[3] = {pw0[0], pw0[1], pw0[2]};
        if (i0 > 0) pivot_words(i, pw);
        const double y0 = __shfl(y, 0, 8), y1 = __shfl(y, 1, 8), y2 = __shfl(y, 2, 8);
        y = pw[0] * y0 + pw[1] * y1 + pw[2] * y2;
      }
      if (live && t < 3) s_y[3 * i + t] = y;
    }
    __syncthreads();
  };
  if (FORWARD) couple(1, true, false);
  if (BACK) {
    couple(1, false, true);
    couple(0, true, true);
  }
  for (int w = threadIdx.x; w < 3 * np1; w += blockDim.x) z[3 * row_node + w] = T(s_y[w]);
}

template <typename T>
hipError_t ilu_setup_t(const fe_problem* p, const int32_t* rp, const int32_t* ci, const T* v, hipStream_t s) {
  const Rows c = row_classes(p->n);
  T* F = static_cast<T*>(p->w_ilu);
  for (int col = 0; col < 8; ++col) {
    const int64_t count = (int64_t)c.cnt[col & 1] * c.cnt[(col >> 1) & 1] * c.cnt[col >> 2];
    const int64_t blocks = std::max<int64_t>(1, (count + FACTOR_B / 32 - 1) / (FACTOR_B / 32));
    hipLaunchKernelGGL(ilu_factor_kernel<T>, dim3((unsigned)blocks), dim3(FACTOR_B), 0, s, c, col, rp, ci, v, F,
                       reinterpret_cast<unsigned int*>(p->flags));
  }
  return hipGetLastError();
}

template <typename T, int Q, bool FORWARD>
void sweep(const Rows& c, const T* F, const T* r, T* z, const int* stop, hipStream_t s) {
  const int np1 = c.n + 1;
  const int lanes = std::min(1024, (8 * np1 + 63) / 64 * 64);
  const unsigned rows = (unsigned)(c.cnt[Q & 1] * c.cnt[Q >> 1]);
  if (rows == 0) return;
  hipLaunchKernelGGL((ilu_sweep_kernel<T, Q, FORWARD>), dim3(rows), dim3(lanes), sizeof(double) * 3 * np1, s, c, F, r,
                     z, stop);
}

template <typename T>
hipError_t ilu_apply_t(const fe_problem* p, const T* r, T* z, const int* stop, hipStream_t s) {
  const Rows c = row_classes(p->n);
  const T* F = static_cast<const T*>(p->w_ilu);
  sweep<T, 0, true>(c, F, r, z, stop, s);
  sweep<T, 1, true>(c, F, r, z, stop, s);
  sweep<T, 2, true>(c, F, r, z, stop, s);
  sweep<T, 3, true>(c, F, r, z, stop, s);  // and back
  sweep<T, 2, false>(c, F, r, z, stop, s);
  sweep<T, 1, false>(c, F, r, z, stop, s);
  sweep<T, 0, false>(c, F, r, z, stop, s);
  return hipGetLastError();
}

}  // namespace

size_t ilu_words(const fe_problem* p) { return (size_t)REC * (size_t)p->n_nodes; }

hipError_t ilu_setup(const fe_problem* p, const int32_t* rp, const int32_t* ci, const void* v, hipStream_t s) {
  return p->prec == FE_F64 ? ilu_setup_t(p, rp, ci, static_cast<const double*>(v), s)
                           : ilu_setup_t(p, rp, ci, static_cast<const float*>(v), s);
}

hipError_t ilu_apply(const fe_problem* p, const void* r, void* z, const int* stop, hipStream_t s) {
  return p->prec == FE_F64 ? ilu_apply_t(p, static_cast<const double*>(r), static_cast<double*>(z), stop, s)
                           : ilu_apply_t(p, static_cast<const float*>(r), static_cast<float*>(z), stop, s);
}

}  // namespace fe
