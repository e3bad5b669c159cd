// Assembly of K and f (Eq. eq-1) for 20-node serendipity hexahedra with full 3x3x3 Gauss
// integration (section 2.1), and the 3x3-block CSR product y = K x.
//
// Pipeline (all on the device):
//   1. node -> element incidence (counting sort, each list sorted by element number);
//   2. block-CSR pattern: per node, the sorted union of the nodes of its elements;
//   3. material stiffness of each layer from engineering constants (C = S^-1, Table 1);
//   4. element matrices K_e = sum_q B^T C_q B det J w, one wavefront per element: C_q is the
//      layer's stiffness turned into global axes at the Gauss point (from the geometric frame
//      there and the ply angle), and sums are scalar, in the order of the definition;
//   5. deterministic gather: every block row sums its elements' blocks in element order
//      (no floating-point atomics), then clamped DOFs become identity rows / columns;
//   6. consistent face loads from a 3x3 Gauss rule on each loaded face.
#include <algorithm>
#include <cmath>

#include "element.h"
#include "gx_internal.h"

namespace gx {

constexpr int MAX_ADJ = 32;        // elements sharing one node
constexpr int MAX_ROW = 128;       // blocks in one block row of K

// Faults of an assembly, found on the device and read back together (a wait of the host for
// each took a third of a small assembly)
enum {
  ERR_CONN = 1, ERR_LAYER = 2, ERR_CLAMP = 4, ERR_FACE = 8,      // before anything uses them
  ERR_SHARED = 16, ERR_LONELY = 32, ERR_ROW = 64,                // before the matrix is laid out
  ERR_MATERIAL = 128, ERR_JACOBIAN = 256
};
__global__ void k_check_range(int64_t n, const int32_t* v, int64_t lim, int bit, int* err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && (v[i] < 0 || v[i] >= lim)) atomicOr(err, bit);
}

// ---------------------------------------------------------------------------------------
// 1. node -> element incidence
__global__ void k_ne_count(const int32_t* conn, int64_t n_elems, int32_t* cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_elems * 20) return;
  atomicAdd(&cnt[conn[i]], 1);
}
__global__ void k_ne_fill(const int32_t* conn, int64_t n_elems, const int32_t* ptr,
                          int32_t* cursor, int32_t* idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_elems * 20) return;
  const int n = conn[i];
  const int pos = atomicAdd(&cursor[n], 1);
  idx[ptr[n] + pos] = (int32_t)(i / 20);
}
__global__ void k_ne_sort(int64_t n_nodes, const int32_t* ptr, int32_t* idx, int* err) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= n_nodes) return;
  const int b = ptr[n], e = ptr[n + 1];
  if (e - b > MAX_ADJ) { atomicOr(err, ERR_SHARED); return; }
  if (e == b) atomicOr(err, ERR_LONELY);
  for (int i = b + 1; i < e; ++i) {              // insertion sort (short lists)
    const int v = idx[i];
    int j = i - 1;
    while (j >= b && idx[j] > v) { idx[j + 1] = idx[j]; --j; }
    idx[j + 1] = v;
  }
}

static void build_node_elem(gx_ctx* c, int* err) {
  const int64_t N = c->n_nodes, E = c->n_elems;
  c->ne_ptr.alloc(N + 1);
  DevBuf<int32_t> cur(N);
  DevBuf<int64_t> tmp(scan_tmp_size(N + 1));
  zero(c->ne_ptr, c->stream);
  zero(cur, c->stream);
  hipLaunchKernelGGL(k_ne_count, dim3(nblocks(E * 20, 256)), dim3(256), 0, c->stream,
                     c->conn.p, E, c->ne_ptr.p);
  exclusive_scan32_async(c->ne_ptr.p, N + 1, tmp.p, c->stream);
  c->ne_idx.alloc(E * 20);
  hipLaunchKernelGGL(k_ne_fill, dim3(nblocks(E * 20, 256)), dim3(256), 0, c->stream,
                     c->conn.p, E, c->ne_ptr.p, cur.p, c->ne_idx.p);
  hipLaunchKernelGGL(k_ne_sort, dim3(nblocks(N, 256)), dim3(256), 0, c->stream, N,
                     c->ne_ptr.p, c->ne_idx.p, err);
  GX_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------------------
// 2. block-CSR pattern, one 64-lane work-group per node
__device__ inline void bitonic_sort(int32_t* s, int n) {
  for (int k = 2; k <= n; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int l = i ^ j;
        if (l > i) {
          const bool up = (i & k) == 0;
          const int32_t a = s[i], b = s[l];
          if ((a > b) == up) { s[i] = b; s[l] = a; }
        }
      }
      __syncthreads();
    }
  }
}

// The sorted union of a node's elements' nodes into its row of `rows` (MAX_ROW entries per
// node), its length into row_len; k_pattern_pack then copies the rows to their places.  (The
// sort is the cost: sorting once more to fill took as long as to count.)
__global__ void __launch_bounds__(64) k_pattern(const int32_t* conn, const int32_t* ne_ptr,
                                                const int32_t* ne_idx, int32_t* row_len,
                                                int32_t* rows, int* err) {
  __shared__ int32_t s[MAX_ADJ * 32];
  const int64_t n = blockIdx.x;
  const int b = ne_ptr[n], e = min(ne_ptr[n + 1], b + MAX_ADJ);
  const int cnt = (e - b) * 20;
  int sz = 1;
  while (sz < cnt) sz <<= 1;
  for (int i = threadIdx.x; i < sz; i += 64)
    s[i] = i < cnt ? conn[(int64_t)ne_idx[b + i / 20] * 20 + i % 20] : 0x7fffffff;
  __syncthreads();
  bitonic_sort(s, sz);
  // first occurrences, 64 entries at a time, ranked by ballot
  int len = 0;
  for (int i0 = 0; i0 < cnt; i0 += 64) {
    const int i = i0 + threadIdx.x;
    const bool first = i < cnt && (i == 0 || s[i] != s[i - 1]);
    const uint64_t m = __ballot(first);
    const int at = len + __popcll(m & ((1ull << threadIdx.x) - 1));
    if (first && at < MAX_ROW) rows[n * MAX_ROW + at] = s[i];
    len += __popcll(m);
  }
  if (threadIdx.x == 0) {
    if (len > MAX_ROW) atomicOr(err, ERR_ROW);
    row_len[n] = len;
  }
}

__global__ void __launch_bounds__(256) k_pattern_pack(int64_t n_nodes, const int32_t* rows,
                                                      const int32_t* ptr, int32_t* col) {
  const int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= n_nodes) return;
  const int b = ptr[n], len = ptr[n + 1] - b;
  for (int i = threadIdx.x & 63; i < len; i += 64) col[b + i] = rows[n * MAX_ROW + i];
}

// ---------------------------------------------------------------------------------------
// 3. layer stiffness C = S^-1 from engineering constants (Voigt 11,22,33,23,13,12 with
//    engineering shear strains).  The orthotropic compliance is block diagonal: the normal
//    3x3 block is inverted by cofactors, the shear block is diag(1/G23, 1/G13, 1/G12).
__global__ void k_layer_stiffness(int n_layers, const double* eng, double* C, int* err) {
  const int L = blockIdx.x * blockDim.x + threadIdx.x;
  if (L >= n_layers) return;
  const double* p = eng + 9 * L;
  double E1 = p[0], E2 = p[1], E3 = p[2], G12 = p[3], G13 = p[4], G23 = p[5];
  double n12 = p[6], n13 = p[7], n23 = p[8];
  if (!(G12 > 0)) {                              // isotropic layer given as (E, nu)
    E2 = E3 = E1;
    n13 = n23 = n12;
    G12 = G13 = G23 = E1 / (2.0 * (1.0 + n12));
  }
  const double s11 = 1 / E1, s22 = 1 / E2, s33 = 1 / E3;
  const double s12 = -n12 / E1, s13 = -n13 / E1, s23 = -n23 / E2;
  const double c11 = s22 * s33 - s23 * s23, c22 = s11 * s33 - s13 * s13,
               c33 = s11 * s22 - s12 * s12;
  const double c12 = s13 * s23 - s12 * s33, c13 = s12 * s23 - s13 * s22,
               c23 = s12 * s13 - s11 * s23;
  const double det = s11 * c11 + s12 * c12 + s13 * c13;
  if (!(det > 0) || !(G12 > 0) || !(G13 > 0) || !(G23 > 0) || !(E1 > 0) || !(E2 > 0) ||
      !(E3 > 0)) {
    atomicOr(err, ERR_MATERIAL);
    return;
  }
  double* o = C + 36 * L;
  for (int i = 0; i < 36; ++i) o[i] = 0.0;
  o[0] = c11 / det; o[7] = c22 / det; o[14] = c33 / det;
  o[1] = o[6] = c12 / det;
  o[2] = o[12] = c13 / det;
  o[8] = o[13] = c23 / det;
  o[21] = G23; o[28] = G13; o[35] = G12;
}

// ---------------------------------------------------------------------------------------
// 4. element stiffness, one wavefront per element (four per work-group, grid-stride).
//
// K_e = sum_q w_q B_q^T (C_q B_q), B_q the strain-displacement matrix of the 20 nodes at Gauss point
// q and C_q the layer's stiffness in global axes.  A point is a step: 60 lanes form the
// gradient of a node and a column of C B each and pass them on through the wavefront's own part
// of LDS; then lane (A, B), A <= B, of 55 adds the point to the 3 x 3 blocks of the two nodes of A
// and the two of B.  Products and sums are in the order of the definition (nodes, Gauss
// points and strain rows ascending, one fused multiply-add each): the matrices of these
// thin plies are ill-conditioned (1e8), and another order moves the solution by 1e-8.
//
// Bound by FP64 issue (about 5,000 products per lane and element) and LDS (42 doubles read per
// 144 products): 33,600 elements 4.37 -> 1.00 ms, against one work-group per element with its
// point set-up on 27 of 256 threads and a product of one pair of nodes per thread.  (On the
// matrix instruction, which sums in another order, 0.68 ms.)
struct ElemWave {
  double X[20][3];
  double J[27][9];           // Jacobians, then their inverses (Ji[3 j + i] = dxi_j / dx_i)
  double Cg[27][36];         // stiffness in global axes
  double dv[27];             // det J * weight
  double G[20][3];           // physical gradients at the current point
  double CB[20][18];         // C_q B_b, entry 3 I + k, at the current point
};
constexpr int EW = 4;        // wavefronts per work-group
struct ElemSmem {
  double dNr[27][20][3];     // reference gradients at the Gauss points
  ElemWave wave[EW];
};

// Inverse Jacobian, weight and stiffness of Gauss point q from its Jacobian
// J[3 i + j] = dx_i / dxi_j, in the geometric frame: e1 along dx/dxi, e2 from dx/deta
// (Gram-Schmidt), e3 = e1 x e2; the fibre rotated by the ply angle about e3.
__device__ inline void gauss_point_setup(int q, ElemWave& sm, const double* Cl, double ca,
                                         double sa, int* err) {
  double J[3][3];
#pragma unroll
  for (int i = 0; i < 9; ++i) J[i / 3][i % 3] = sm.J[q][i];
  const double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
                     J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                     J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
  if (!(det > 0)) atomicOr(err, ERR_JACOBIAN);
  const double id = 1.0 / det;
  sm.J[q][0] = (J[1][1] * J[2][2] - J[1][2] * J[2][1]) * id;
  sm.J[q][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * id;
  sm.J[q][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * id;
  sm.J[q][3] = (J[1][2] * J[2][0] - J[1][0] * J[2][2]) * id;
  sm.J[q][4] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * id;
  sm.J[q][5] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * id;
  sm.J[q][6] = (J[1][0] * J[2][1] - J[1][1] * J[2][0]) * id;
  sm.J[q][7] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * id;
  sm.J[q][8] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * id;
  double e1[3] = {J[0][0], J[1][0], J[2][0]}, t2[3] = {J[0][1], J[1][1], J[2][1]};
  const double n1 = sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) e1[i] /= n1;
  const double pr = t2[0] * e1[0] + t2[1] * e1[1] + t2[2] * e1[2];
  double e2[3] = {t2[0] - pr * e1[0], t2[1] - pr * e1[1], t2[2] - pr * e1[2]};
  const double n2 = sqrt(e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) e2[i] /= n2;
  const double e3[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                        e1[0] * e2[1] - e1[1] * e2[0]};
  // material axes (rows of Q, global components)
  double Q[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    Q[0][i] = ca * e1[i] + sa * e2[i];
    Q[1][i] = -sa * e1[i] + ca * e2[i];
    Q[2][i] = e3[i];
  }
  // Bond matrix: local engineering strain = T * global engineering strain
  constexpr int vi[6] = {0, 1, 2, 1, 0, 0}, vj[6] = {0, 1, 2, 2, 2, 1};
  double T[6][6], CT[6][6];
#pragma unroll
  for (int I = 0; I < 6; ++I) {
    const int i = vi[I], j = vj[I];
#pragma unroll
    for (int K = 0; K < 6; ++K) {
      const int k = vi[K], l = vj[K];
      if (I < 3)
        T[I][K] = (K < 3) ? Q[i][k] * Q[i][k] : Q[i][k] * Q[i][l];
      else
        T[I][K] = (K < 3) ? 2.0 * Q[i][k] * Q[j][k] : Q[i][k] * Q[j][l] + Q[i][l] * Q[j][k];
    }
  }
  // C_g = T^T C T; C is a full 3 x 3 normal block and three shear moduli
#pragma unroll
  for (int K = 0; K < 6; ++K) {
#pragma unroll
    for (int I = 0; I < 3; ++I)
      CT[I][K] = __builtin_fma(Cl[6 * I + 2], T[2][K],
                               __builtin_fma(Cl[6 * I + 1], T[1][K], Cl[6 * I] * T[0][K]));
#pragma unroll
    for (int I = 3; I < 6; ++I) CT[I][K] = Cl[7 * I] * T[I][K];
  }
#pragma unroll
  for (int I = 0; I < 6; ++I)
#pragma unroll
    for (int K = I; K < 6; ++K) {
      double s = T[0][I] * CT[0][K];
#pragma unroll
      for (int L = 1; L < 6; ++L) s = __builtin_fma(T[L][I], CT[L][K], s);
      sm.Cg[q][6 * I + K] = s;
      sm.Cg[q][6 * K + I] = s;
    }
  double xq, wq, wy, wz;
  gauss3(q % 3, &xq, &wq);
  gauss3((q / 3) % 3, &xq, &wy);
  gauss3(q / 9, &xq, &wz);
  sm.dv[q] = det * wq * wy * wz;
}

__global__ void __launch_bounds__(64 * EW, 2) k_element(Periodic P, int64_t n_elems,
                                                        const double* xyz, const int32_t* conn,
                                                        const int32_t* elayer,
                                                        const double* Clayer,
                                                        const double* angle, double* Ke,
                                                        int* err) {
  extern __shared__ double smem_raw[];
  ElemSmem& sm = *reinterpret_cast<ElemSmem*>(smem_raw);
  // reference gradients at the 27 Gauss points (q = i + 3 j + 9 k)
  for (int idx = threadIdx.x; idx < 27 * 20; idx += blockDim.x) {
    const int q = idx / 20, a = idx % 20;
    double x0, x1, x2, w, N, d[3];
    gauss3(q % 3, &x0, &w);
    gauss3((q / 3) % 3, &x1, &w);
    gauss3(q / 9, &x2, &w);
    shape_one(a, x0, x1, x2, &N, d);
    for (int j = 0; j < 3; ++j) sm.dNr[q][a][j] = d[j];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ElemWave& W = sm.wave[wv];
  // (the lanes of a wavefront exchange through their own part of LDS: its accesses are
  // performed in order, so only the compiler has to keep them)
  auto fence = [] {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
  };
  const int nb = min(lane / 3, 19), nk = lane % 3;  // this lane's node and column of C B
  // the strain rows that displacement component k enters, ascending, and with which gradient
  // component: k = 0: 11, 13, 12; 1: 22, 23, 12; 2: 33, 23, 13
  const int j1 = nk == 0 ? 4 : 3, j2 = nk == 2 ? 4 : 5;
  int A = 0, Bn = lane;                            // this lane's pairs of nodes
  while (A < 9 && Bn >= 10 - A) { Bn -= 10 - A; ++A; }
  Bn = min(Bn + A, 9);
  for (int64_t e = (int64_t)blockIdx.x * EW + wv; e < n_elems; e += (int64_t)gridDim.x * EW) {
    if (lane < 60)
      W.X[lane / 3][lane % 3] = node_coord(xyz, conn[20 * e + lane / 3], lane % 3, P, e, lane / 3);
    const int L = __builtin_amdgcn_readfirstlane(elayer[e]);
    fence();
    for (int t = lane; t < 27 * 9; t += 64) {      // Jacobians: entry (q, i, j) per lane
      const int q = t / 9, i = (t % 9) / 3, j = t % 3;
      double s = 0.0;
#pragma unroll
      for (int a = 0; a < 20; ++a) s += W.X[a][i] * sm.dNr[q][a][j];
      W.J[q][t % 9] = s;
    }
    fence();
    if (lane < 27) {
      const double an = angle[L] * (M_PI / 180.0);
      gauss_point_setup(lane, W, Clayer + 36 * L, cos(an), sin(an), err);
    }
    fence();
    double acc[2][2][9];
#pragma unroll
    for (int i = 0; i < 36; ++i) acc[i / 18][i / 9 % 2][i % 9] = 0.0;
#pragma unroll 1
    for (int q = 0; q < 27; ++q) {
      {
        const double d0 = sm.dNr[q][nb][0], d1 = sm.dNr[q][nb][1], d2 = sm.dNr[q][nb][2];
        double g[3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
          g[i] = d0 * W.J[q][i] + d1 * W.J[q][3 + i] + d2 * W.J[q][6 + i];
        const double g0 = nk == 0 ? g[0] : nk == 1 ? g[1] : g[2];
        const double g1 = nk == 2 ? g[1] : g[2], g2 = nk == 0 ? g[1] : g[0];
        if (lane < 60) {
          W.G[nb][nk] = g0;
#pragma unroll
          for (int I = 0; I < 6; ++I) {
            const double* c = &W.Cg[q][6 * I];
            W.CB[nb][3 * I + nk] = __builtin_fma(c[j2], g2, __builtin_fma(c[j1], g1, c[nk] * g0));
          }
        }
      }
      fence();
      const double dv = W.dv[q];
      double ga[2][3];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int i = 0; i < 3; ++i) ga[x][i] = W.G[2 * A + x][i];
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        double cb[18];
#pragma unroll
        for (int i = 0; i < 18; ++i) cb[i] = W.CB[2 * Bn + y][i];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const double* g = ga[x];
            const double s0 = __builtin_fma(g[1], cb[15 + k], __builtin_fma(g[2], cb[12 + k], g[0] * cb[k]));
            const double s1 = __builtin_fma(g[0], cb[15 + k], __builtin_fma(g[2], cb[9 + k], g[1] * cb[3 + k]));
            const double s2 = __builtin_fma(g[0], cb[12 + k], __builtin_fma(g[1], cb[9 + k], g[2] * cb[6 + k]));
            acc[x][y][k] = __builtin_fma(dv, s0, acc[x][y][k]);
            acc[x][y][3 + k] = __builtin_fma(dv, s1, acc[x][y][3 + k]);
            acc[x][y][6 + k] = __builtin_fma(dv, s2, acc[x][y][6 + k]);
          }
      }
      fence();
    }
    double* out = Ke + e * 3600;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const int a = 2 * A + x, b = 2 * Bn + y;
        if (lane >= 55 || a > b) continue;
#pragma unroll
        for (int i = 0; i < 9; ++i) out[(a * 20 + b) * 9 + i] = acc[x][y][i];
        if (a != b)
#pragma unroll
          for (int i = 0; i < 9; ++i) out[(b * 20 + a) * 9 + i % 3 * 3 + i / 3] = acc[x][y][i];
      }
    fence();
  }
}

// ---------------------------------------------------------------------------------------
// 5. deterministic gather of element blocks into block rows (element order); clamped DOFs ->
//    identity.  Where each element's 20 blocks go in the row, and which of its nodes this
//    one is, are looked up for all of the node's elements at once; then the values of eight
//    elements are loaded together and added in LDS one element after another.  Bound by
//    memory: 0.97 GB of blocks read and 0.73 GB of rows written for 33,600 elements, 1.14 ->
//    0.62 ms against looking up and adding element by element.
__global__ void __launch_bounds__(64) k_gather(const int32_t* conn, const int32_t* ne_ptr,
                                               const int32_t* ne_idx, const int32_t* row_ptr,
                                               const int32_t* col, const double* Ke,
                                               const uint8_t* fixed, double* val) {
  __shared__ double rv[MAX_ROW * 9];
  __shared__ int32_t rc[MAX_ROW];
  __shared__ uint8_t pos[MAX_ADJ][20];
  __shared__ int32_t self[MAX_ADJ], el[MAX_ADJ];
  const int64_t n = blockIdx.x;
  const int lane = threadIdx.x;
  const int rb = row_ptr[n], len = row_ptr[n + 1] - rb;
  const int eb = ne_ptr[n], ne = ne_ptr[n + 1] - eb;
  for (int i = lane; i < len; i += 64) rc[i] = col[rb + i];
  if (lane < ne) {
    self[lane] = 19;
    el[lane] = ne_idx[eb + lane];
  }
  for (int i = lane; i < len * 9; i += 64) rv[i] = 0.0;
  __syncthreads();
  for (int i = lane; i < ne * 20; i += 64) {
    const int k = i / 20, b = i - 20 * k;
    const int m = conn[20 * (int64_t)el[k] + b];
    int lo = 0, hi = len - 1;                      // binary search of m in the row
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (rc[mid] < m) lo = mid + 1; else hi = mid;
    }
    pos[k][b] = (uint8_t)lo;
    if (m == n) atomicMin(&self[k], b);
  }
  __syncthreads();
  for (int k0 = 0; k0 < ne; k0 += 8) {
    double v[8][3];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int kk = min(k0 + k, ne - 1);
      const double* src = Ke + ((int64_t)el[kk] * 20 + self[kk]) * 180;
#pragma unroll
      for (int u = 0; u < 3; ++u) v[k][u] = src[min(lane + 64 * u, 179)];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k0 + k < ne) {                           // (one wavefront: its LDS accesses are in
#pragma unroll                                     // order, so no barrier between elements)
        for (int u = 0; u < 3; ++u) {
          const int i = lane + 64 * u;
          if (i < 180) rv[9 * pos[k0 + k][i / 9] + i % 9] += v[k][u];
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
      }
  }
  for (int i = lane; i < len * 9; i += 64) {
    const int blk = i / 9, comp = i - 9 * (i / 9);
    const int ri = comp / 3, ci = comp - 3 * (comp / 3);
    const int64_t rd = 3 * n + ri, cd = 3 * (int64_t)rc[blk] + ci;
    double x = rv[i];
    if (fixed[rd] || fixed[cd]) x = (rd == cd) ? 1.0 : 0.0;
    val[(int64_t)rb * 9 + i] = x;
  }
}

// ---------------------------------------------------------------------------------------
// 6. consistent face loads; t = t0 + k ((x - c) . d) n_out, 3x3 Gauss rule on the face;
//    one thread per (face, element node) writes its three components to fl; k_face_gather
//    then sums each node's entries in a fixed order (face, then local node), so f is the
//    same bit for bit on every run
__global__ void k_face_loads(Periodic P, int64_t n_faces, const int32_t* fe, const int32_t* fid,
                             const double* xyz, const int32_t* conn, gx_traction tr,
                             double* fl) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_faces * 20) return;
  const int64_t e = fe[idx / 20];
  const int na = (int)(idx % 20);
  const int face = fid[idx / 20];
  const int ax = face / 2;
  const double sgn = (face & 1) ? 1.0 : -1.0;
  double fl0 = 0, fl1 = 0, fl2 = 0;
  for (int qb = 0; qb < 3; ++qb)
    for (int qc = 0; qc < 3; ++qc) {
      double pb, wb, pc, wc;
      gauss3(qb, &pb, &wb);
      gauss3(qc, &pc, &wc);
      // reference point on the face: fixed axis ax, in-face axes (ax+1)%3, (ax+2)%3
      const double p0 = ax == 0 ? sgn : (ax == 1 ? pc : pb);
      const double p1 = ax == 1 ? sgn : (ax == 2 ? pc : pb);
      const double p2 = ax == 2 ? sgn : (ax == 0 ? pc : pb);
      double x0 = 0, x1 = 0, x2 = 0, tb0 = 0, tb1 = 0, tb2 = 0, tc0 = 0, tc1 = 0, tc2 = 0,
             Na = 0;
      for (int a = 0; a < 20; ++a) {
        double N, d[3];
        shape_one(a, p0, p1, p2, &N, d);
        const double db = ax == 0 ? d[1] : (ax == 1 ? d[2] : d[0]);
        const double dc = ax == 0 ? d[2] : (ax == 1 ? d[0] : d[1]);
        const int64_t nd = conn[20 * e + a];
        const double X0 = node_coord(xyz, nd, 0, P, e, a), X1 = node_coord(xyz, nd, 1, P, e, a),
                     X2 = node_coord(xyz, nd, 2, P, e, a);
        x0 += N * X0; x1 += N * X1; x2 += N * X2;
        tb0 += db * X0; tb1 += db * X1; tb2 += db * X2;
        tc0 += dc * X0; tc1 += dc * X1; tc2 += dc * X2;
        if (a == na) Na = N;
      }
      const double nv0 = tb1 * tc2 - tb2 * tc1, nv1 = tb2 * tc0 - tb0 * tc2,
                   nv2 = tb0 * tc1 - tb1 * tc0;
      const double dA = sqrt(nv0 * nv0 + nv1 * nv1 + nv2 * nv2);
      const double lin = tr.k * ((x0 - tr.c[0]) * tr.d[0] + (x1 - tr.c[1]) * tr.d[1] +
                                 (x2 - tr.c[2]) * tr.d[2]);
      const double w = wb * wc * dA * Na;
      fl0 += (tr.t0[0] + lin * sgn * nv0 / dA) * w;
      fl1 += (tr.t0[1] + lin * sgn * nv1 / dA) * w;
      fl2 += (tr.t0[2] + lin * sgn * nv2 / dA) * w;
    }
  fl[3 * idx] = fl0;
  fl[3 * idx + 1] = fl1;
  fl[3 * idx + 2] = fl2;
}

// f at the loaded nodes: node unode[i] sums the entries uidx[uptr[i] .. uptr[i + 1]) of fl
// (ascending (face, local node) order); clamped components stay zero
__global__ void k_face_gather(int64_t n_unique, const int32_t* uptr, const int32_t* uidx,
                              const int32_t* unode, const double* fl, const uint8_t* fixed,
                              double* f) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_unique) return;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (int32_t k = uptr[i]; k < uptr[i + 1]; ++k) {
    const int64_t j = uidx[k];
    a0 += fl[3 * j];
    a1 += fl[3 * j + 1];
    a2 += fl[3 * j + 2];
  }
  const int64_t d = 3 * (int64_t)unode[i];
  f[d] = fixed[d] ? 0.0 : a0;
  f[d + 1] = fixed[d + 1] ? 0.0 : a1;
  f[d + 2] = fixed[d + 2] ? 0.0 : a2;
}

// the nodes of the loaded faces' elements, 20 per face
__global__ void k_face_nodes(int64_t n_faces, const int32_t* fe, const int32_t* conn,
                             int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 20 * n_faces) out[i] = conn[20 * (int64_t)fe[i / 20] + i % 20];
}

__global__ void k_fixed(int64_t n, const int32_t* nodes, uint8_t* fixed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t d = 3 * (int64_t)nodes[i];
  fixed[d] = fixed[d + 1] = fixed[d + 2] = 1;
}

// ---------------------------------------------------------------------------------------
// y = K x, one 64-lane wavefront per block row.  The values of a row are contiguous, 9 per
// 3x3 block.  Pass u takes the row's blocks 7 u .. 7 u + 6: lane l < 63 reads value
// 63 u + l, i.e. entry l % 9 of block 7 u + l / 9, so every lane multiplies the same
// entry position on every pass and keeps a single sum (the block-row component
// (l % 9) / 3, the x component l % 3), and each pass is one coalesced 504-byte load of
// values.  A row takes ceil(blocks / 7) passes (rounds of 12 past 84 blocks).  All value
// loads of a round are issued; its column indices are loaded once, one block per lane, and
// passed between lanes; then all gathers of x are issued, before the products.  The three
// components are then summed through LDS (lanes 0-2, the 21 sums of their component in a
// fixed order).
constexpr int SPMV_PASSES = 12;                   // 84 blocks per round (rows of the
                                                  // 20-node meshes have at most 81)
__global__ void __launch_bounds__(256) k_spmv(int64_t n_rows, const int32_t* __restrict__ rp,
                                              const int32_t* __restrict__ col,
                                              const double* __restrict__ val,
                                              const double* __restrict__ x,
                                              double* __restrict__ y) {
  __shared__ double red[4][64];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // work-groups are dealt to the eight XCDs in turn; each XCD takes a contiguous eighth of
  // the rows, so the part of x its rows gather stays in its L2
  const int64_t xcd = blockIdx.x & 7, nq = gridDim.x >> 3, nrem = gridDim.x & 7;
  const int64_t lb = xcd * nq + min(xcd, nrem) + (blockIdx.x >> 3);
  const int64_t row = lb * 4 + w;                 // uniform: the row bounds are scalar
  if (row >= n_rows) return;                       // whole wavefronts
  const int q = lane / 9, e = lane - 9 * q, c = e % 3;
  const int b0 = rp[row], nb = rp[row + 1] - b0;
  const double* vrow = val + (int64_t)b0 * 9 + e;
  const int32_t* crow = col + b0;
  double acc = 0.0;
  // one round of P passes over blocks k0 ..; lanes past the row's last block repeat it
  // and are masked
  auto round = [&](int k0, auto np) {
    constexpr int P = decltype(np)::value;
    double pv[P], xv[P];
    // the round's column indices, one block per lane (blocks k0 + 64 .. in a second
    // register past 64 blocks); pass u takes block 7 u + q's from its lane
    const int cl0 = crow[min(k0 + lane, nb - 1)];
    const int cl1 = 7 * P > 64 ? crow[min(k0 + 64 + lane, nb - 1)] : 0;
#pragma unroll
    for (int u = 0; u < P; ++u)                   // read once: kept out of the caches' way
      pv[u] = __builtin_nontemporal_load(&vrow[9 * min(k0 + 7 * u + q, nb - 1)]);
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const int b = 7 * u + q;                     // block within the round (< 84)
      // (a permute reads 0 from an inactive lane, so both run with the whole wavefront
      // active and the block's register is selected afterwards)
      int xi;
      if (7 * u + 6 < 64) {
        xi = __builtin_amdgcn_ds_bpermute(4 * b, cl0);
      } else if (7 * u >= 64) {
        xi = __builtin_amdgcn_ds_bpermute(4 * (b - 64), cl1);
      } else {
        const int i0 = __builtin_amdgcn_ds_bpermute(4 * (b & 63), cl0);
        const int i1 = __builtin_amdgcn_ds_bpermute(4 * (b & 63), cl1);
        xi = b < 64 ? i0 : i1;
      }
      xv[u] = x[3 * (int64_t)xi + c];
    }
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const bool ok = lane < 63 && k0 + 7 * u + q < nb;  // masked, not branched
      acc += ok ? pv[u] * xv[u] : 0.0;
    }
  };
  // exactly the passes the row needs (rounds of SPMV_PASSES past 7 SPMV_PASSES blocks)
  using std::integral_constant;
  switch ((nb + 6) / 7) {
    case 0: break;
    case 1: round(0, integral_constant<int, 1>{}); break;
    case 2: round(0, integral_constant<int, 2>{}); break;
    case 3: round(0, integral_constant<int, 3>{}); break;
    case 4: round(0, integral_constant<int, 4>{}); break;
    case 5: round(0, integral_constant<int, 5>{}); break;
    case 6: round(0, integral_constant<int, 6>{}); break;
    case 7: round(0, integral_constant<int, 7>{}); break;
    case 8: round(0, integral_constant<int, 8>{}); break;
    case 9: round(0, integral_constant<int, 9>{}); break;
    case 10: round(0, integral_constant<int, 10>{}); break;
    case 11: round(0, integral_constant<int, 11>{}); break;
    default:
      for (int k0 = 0; k0 < nb; k0 += 7 * SPMV_PASSES)
        round(k0, integral_constant<int, SPMV_PASSES>{});
  }
  // lanes of one wavefront exchange through LDS without a barrier: its LDS accesses are
  // performed in order
  red[w][lane] = acc;
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_wave_barrier();
  if (lane < 3) {
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < 7; ++t)
#pragma unroll
      for (int j = 0; j < 3; ++j) s += red[w][9 * t + 3 * lane + j];
    y[3 * row + lane] = s;
  }
}

void spmv(gx_ctx* c, const double* x, double* y) {
  hipLaunchKernelGGL(k_spmv, dim3(nblocks(c->n_nodes, 4)), dim3(256), 0, c->stream,
                     c->n_nodes, c->row_ptr.p, c->col.p, c->val.p, x, y);
}

}  // namespace gx

using namespace gx;

extern "C" {

gx_status gx_assemble(gx_ctx* c, const gx_mesh* m, const gx_plystack* ps, const gx_loads* ld,
                      double* f_out) {
  GX_API_BEGIN(c)
  GX_REQUIRE(m && ps && ld && f_out, "null argument");
  GX_REQUIRE(m->n_nodes > 0 && m->n_elems > 0 && m->xyz && m->conn && m->elem_layer,
             "bad mesh");
  GX_REQUIRE(m->n_nodes < ((int64_t)1 << 31) / 3, "too many nodes");
  // the incidence lists and the load lists are 20 entries per element or face, 32-bit offsets
  GX_REQUIRE(m->n_elems <= INT32_MAX / 20, "too many elements");
  GX_REQUIRE(ld->n_faces <= INT32_MAX / 20, "too many load faces");
  GX_REQUIRE(ps->n_layers >= 1 && ps->eng && ps->angle_deg, "bad ply stack");
  Timer tm(c->stream);
  hipStream_t s = c->stream;
  c->assembled = false;
  c->matrix_only = false;
  c->setup_done = false;
  c->sw = Schwarz();
  c->n_nodes = m->n_nodes;
  c->n_elems = m->n_elems;
  const int64_t N = c->n_nodes, E = c->n_elems;
  c->xyz.alloc(3 * N);
  c->conn.alloc(20 * E);
  c->elayer.alloc(E);
  GX_HIP(hipMemcpyAsync(c->xyz.p, m->xyz, 3 * N * sizeof(double), hipMemcpyDefault, s));
  GX_HIP(hipMemcpyAsync(c->conn.p, m->conn, 20 * E * sizeof(int32_t), hipMemcpyDefault, s));
  GX_HIP(hipMemcpyAsync(c->elayer.p, m->elem_layer, E * sizeof(int32_t), hipMemcpyDefault, s));
  c->wrap.release();
  for (int i = 0; i < 3; ++i) c->period[i] = m->elem_wrap ? m->period[i] : 0.0;
  if (m->elem_wrap) {
    c->wrap.alloc(E);
    GX_HIP(hipMemcpyAsync(c->wrap.p, m->elem_wrap, E * sizeof(uint32_t), hipMemcpyDefault, s));
  }
  const int64_t nc = std::max<int64_t>(ld->n_clamped, 0), nf = std::max<int64_t>(ld->n_faces, 0);
  GX_REQUIRE(nc == 0 || ld->clamped, "null clamped list");
  GX_REQUIRE(nf == 0 || (ld->face_elem && ld->face_id), "null face list");
  DevBuf<int32_t> d_clamped(nc);
  c->n_faces = 0;
  c->face_e.alloc(nf);
  c->face_id.alloc(nf);
  if (nc)
    GX_HIP(hipMemcpyAsync(d_clamped.p, ld->clamped, nc * sizeof(int32_t), hipMemcpyDefault, s));
  if (nf) {
    GX_HIP(hipMemcpyAsync(c->face_e.p, ld->face_elem, nf * sizeof(int32_t), hipMemcpyDefault, s));
    GX_HIP(hipMemcpyAsync(c->face_id.p, ld->face_id, nf * sizeof(int32_t), hipMemcpyDefault, s));
  }
  // every index checked before anything uses it
  DevBuf<int> err(1);
  zero(err, s);
  auto check = [&](int64_t n, const int32_t* v, int64_t lim, int bit) {
    if (n)
      hipLaunchKernelGGL(k_check_range, dim3(nblocks(n, 256)), dim3(256), 0, s, n, v, lim, bit,
                         err.p);
  };
  check(20 * E, c->conn.p, N, ERR_CONN);
  check(E, c->elayer.p, ps->n_layers, ERR_LAYER);
  check(nc, d_clamped.p, N, ERR_CLAMP);
  check(nf, c->face_e.p, E, ERR_FACE);
  check(nf, c->face_id.p, 6, ERR_FACE);
  GX_HIP(hipGetLastError());
  int herr = 0;
  to_host(&herr, err.p, 1, s);
  GX_REQUIRE(!(herr & ERR_CONN), "connectivity index out of range");
  GX_REQUIRE(!(herr & ERR_LAYER), "layer index out of range");
  GX_REQUIRE(!(herr & ERR_CLAMP), "clamped node out of range");
  GX_REQUIRE(!(herr & ERR_FACE), "bad load face");
  // clamped DOFs
  c->fixed.alloc(3 * N);
  zero(c->fixed, s);
  if (nc)
    hipLaunchKernelGGL(k_fixed, dim3(nblocks(nc, 256)), dim3(256), 0, s, nc, d_clamped.p,
                       c->fixed.p);
  build_node_elem(c, err.p);
  // pattern
  DevBuf<int32_t> rows((size_t)N * MAX_ROW);
  c->row_ptr.alloc(N + 1);
  zero(c->row_ptr, s);
  hipLaunchKernelGGL(k_pattern, dim3((unsigned)N), dim3(64), 0, s, c->conn.p, c->ne_ptr.p,
                     c->ne_idx.p, c->row_ptr.p, rows.p, err.p);
  DevBuf<int64_t> tmp(scan_tmp_size(N + 1));
  exclusive_scan32_async(c->row_ptr.p, N + 1, tmp.p, s);
  // materials (ps's tables are read by the copies, which the next wait completes)
  DevBuf<double> eng(9 * ps->n_layers);
  c->ang.alloc(ps->n_layers);
  c->Cl.alloc(36 * ps->n_layers);
  c->n_layers = ps->n_layers;
  c->eng.assign(ps->eng, ps->eng + 9 * ps->n_layers);
  to_dev(eng.p, ps->eng, 9 * ps->n_layers, s);
  to_dev(c->ang.p, ps->angle_deg, ps->n_layers, s);
  hipLaunchKernelGGL(k_layer_stiffness, dim3(nblocks(ps->n_layers, 64)), dim3(64), 0, s,
                     ps->n_layers, eng.p, c->Cl.p, err.p);
  DevBuf<int32_t> d_fn(20 * nf);
  std::vector<int32_t> fn(20 * nf);
  if (nf) {
    hipLaunchKernelGGL(k_face_nodes, dim3(nblocks(20 * nf, 256)), dim3(256), 0, s, nf,
                       c->face_e.p, c->conn.p, d_fn.p);
    GX_HIP(hipMemcpyAsync(fn.data(), d_fn.p, fn.size() * sizeof(int32_t), hipMemcpyDeviceToHost,
                          s));
  }
  GX_HIP(hipGetLastError());
  int32_t nnz32 = 0;
  GX_HIP(hipMemcpyAsync(&herr, err.p, sizeof(int), hipMemcpyDeviceToHost, s));
  to_host(&nnz32, c->row_ptr.p + N, 1, s);
  GX_REQUIRE(!(herr & ERR_SHARED), "a node is shared by more than 32 elements");
  GX_REQUIRE(!(herr & ERR_LONELY), "a node belongs to no element");
  GX_REQUIRE(!(herr & ERR_ROW), "a block row has more than 128 blocks");
  GX_REQUIRE(!(herr & ERR_MATERIAL), "singular material compliance");
  // rows of at most MAX_ROW blocks: only with so many can the 32-bit offsets have wrapped
  const int64_t nnzb =
      N > INT32_MAX / MAX_ROW ? scanned32_exact(nnz32, N + 1, tmp.p, s) : (int64_t)nnz32;
  GX_REQUIRE(nnzb <= INT32_MAX, "matrix too large");
  c->nnzb = nnzb;
  c->col.alloc(nnzb);
  hipLaunchKernelGGL(k_pattern_pack, dim3(nblocks(N, 4)), dim3(256), 0, s, N, rows.p,
                     c->row_ptr.p, c->col.p);
  rows.release();
  // element matrices
  c->Ke.alloc((size_t)E * 3600);
  const unsigned eg = (unsigned)std::min<int64_t>((E + EW - 1) / EW, 256 * 8);
  hipLaunchKernelGGL(k_element, dim3(eg), dim3(64 * EW), sizeof(ElemSmem), s, periodic_of(c), E,
                     c->xyz.p, c->conn.p, c->elayer.p, c->Cl.p, c->ang.p, c->Ke.p, err.p);
  // global matrix
  c->val.alloc((size_t)nnzb * 9);
  hipLaunchKernelGGL(k_gather, dim3((unsigned)N), dim3(64), 0, s, c->conn.p, c->ne_ptr.p,
                     c->ne_idx.p, c->row_ptr.p, c->col.p, c->Ke.p, c->fixed.p, c->val.p);
  GX_HIP(hipGetLastError());
  // loads
  GX_HIP(hipMemsetAsync(f_out, 0, 3 * N * sizeof(double), s));
  std::vector<int32_t> order(20 * nf), uptr{0}, unode;
  DevBuf<double> fl(60 * nf);
  DevBuf<int32_t> d_uptr, d_uidx, d_unode;
  if (nf) {
    const int64_t nent = 20 * nf;
    c->n_faces = nf;
    c->traction = ld->traction;
    hipLaunchKernelGGL(k_face_loads, dim3(nblocks(nent, 64)), dim3(64), 0, s, periodic_of(c), nf,
                       c->face_e.p, c->face_id.p, c->xyz.p, c->conn.p, ld->traction, fl.p);
    // per node, its (face, local node) entries in ascending order
    for (int64_t k = 0; k < nent; ++k) order[k] = (int32_t)k;
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return fn[a] < fn[b]; });
    for (int64_t k = 0; k < nent; ++k) {
      if (k > 0 && fn[order[k]] != fn[order[k - 1]]) uptr.push_back((int32_t)k);
      if (k == 0 || fn[order[k]] != fn[order[k - 1]]) unode.push_back(fn[order[k]]);
    }
    uptr.push_back((int32_t)nent);
    d_uptr.alloc(uptr.size());
    d_uidx.alloc(nent);
    d_unode.alloc(unode.size());
    to_dev(d_uptr.p, uptr.data(), uptr.size(), s);
    to_dev(d_uidx.p, order.data(), order.size(), s);
    to_dev(d_unode.p, unode.data(), unode.size(), s);
    hipLaunchKernelGGL(k_face_gather, dim3(nblocks((int64_t)unode.size(), 256)), dim3(256), 0, s,
                       (int64_t)unode.size(), d_uptr.p, d_uidx.p, d_unode.p, fl.p, c->fixed.p,
                       f_out);
  }
  GX_HIP(hipGetLastError());
  to_host(&herr, err.p, 1, s);
  GX_REQUIRE(!(herr & ERR_JACOBIAN), "non-positive Jacobian determinant in an element");
  GX_HIP(hipStreamSynchronize(s));
  c->assembled = true;
  c->phase_ms[0] = tm.ms();
  GX_API_END(c)
}

gx_status gx_matrix_info(gx_ctx* c, int64_t* nr, int64_t* nb) {
  GX_API_BEGIN(c)
  if (!c->assembled) throw Error(GX_ESTATE, "matrix not assembled");
  if (nr) *nr = c->n_nodes;
  if (nb) *nb = c->nnzb;
  GX_API_END(c)
}

gx_status gx_matrix_copy(gx_ctx* c, int32_t* rp, int32_t* col, double* val) {
  GX_API_BEGIN(c)
  if (!c->assembled) throw Error(GX_ESTATE, "matrix not assembled");
  hipStream_t s = c->stream;
  if (rp)
    GX_HIP(hipMemcpyAsync(rp, c->row_ptr.p, (c->n_nodes + 1) * 4, hipMemcpyDefault, s));
  if (col) GX_HIP(hipMemcpyAsync(col, c->col.p, c->nnzb * 4, hipMemcpyDefault, s));
  if (val) GX_HIP(hipMemcpyAsync(val, c->val.p, c->nnzb * 72, hipMemcpyDefault, s));
  GX_HIP(hipStreamSynchronize(s));
  GX_API_END(c)
}

gx_status gx_matrix_load(gx_ctx* c, int64_t n_block_rows, int64_t n_blocks,
                         const int32_t* row_ptr, const int32_t* col, const double* val) {
  GX_API_BEGIN(c)
  GX_REQUIRE(n_block_rows >= 1 && n_blocks >= 0 && row_ptr && (col && val || n_blocks == 0),
             "bad block matrix");
  GX_REQUIRE(n_block_rows < ((int64_t)1 << 31) / 3 && n_blocks < ((int64_t)1 << 31),
             "block matrix too large for 32-bit indices");
  hipStream_t s = c->stream;
  std::vector<int32_t> hp(n_block_rows + 1), hc(n_blocks);
  GX_HIP(hipMemcpyAsync(hp.data(), row_ptr, hp.size() * 4, hipMemcpyDefault, s));
  if (n_blocks) GX_HIP(hipMemcpyAsync(hc.data(), col, hc.size() * 4, hipMemcpyDefault, s));
  GX_HIP(hipStreamSynchronize(s));
  GX_REQUIRE(hp[0] == 0 && hp[n_block_rows] == n_blocks, "row pointers do not span the blocks");
  for (int64_t r = 0; r < n_block_rows; ++r) GX_REQUIRE(hp[r] <= hp[r + 1], "row pointers decrease");
  for (int32_t v : hc) GX_REQUIRE(v >= 0 && v < n_block_rows, "column index out of range");
  c->assembled = false;
  c->setup_done = false;
  c->sw = Schwarz();
  c->n_nodes = n_block_rows;
  c->n_elems = 0;
  c->nnzb = n_blocks;
  c->row_ptr.alloc(n_block_rows + 1);
  c->col.alloc(std::max<int64_t>(n_blocks, 1));
  c->val.alloc(std::max<int64_t>(9 * n_blocks, 1));
  to_dev(c->row_ptr.p, hp.data(), hp.size(), s);
  if (n_blocks) {
    to_dev(c->col.p, hc.data(), hc.size(), s);
    GX_HIP(hipMemcpyAsync(c->val.p, val, 9 * n_blocks * sizeof(double), hipMemcpyDefault, s));
  }
  GX_HIP(hipStreamSynchronize(s));
  c->assembled = true;
  c->matrix_only = true;
  GX_API_END(c)
}

gx_status gx_spmv(gx_ctx* c, const double* x, double* y) {
  GX_API_BEGIN(c)
  if (!c->assembled) throw Error(GX_ESTATE, "matrix not assembled");
  GX_REQUIRE(x && y, "null vector");
  spmv(c, x, y);
  GX_HIP(hipGetLastError());
  GX_HIP(hipStreamSynchronize(c->stream));
  GX_API_END(c)
}

}  // extern "C"
