// 20-node serendipity hexahedron: reference nodes, shape functions and the 3-point Gauss
// rule (section 2.1: quadratic serendipity elements with full integration).  Shared by the
// assembly and the sensitivity kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace gx {

// ---------------------------------------------------------------------------------------
// Serendipity shape functions on the reference cube [-1, 1]^3.
static __device__ __constant__ int8_t c_ref[20][3] = {
    {-1, -1, -1}, {1, -1, -1}, {-1, 1, -1}, {1, 1, -1},
    {-1, -1, 1},  {1, -1, 1},  {-1, 1, 1},  {1, 1, 1},
    {0, -1, -1},  {0, 1, -1},  {0, -1, 1},  {0, 1, 1},
    {-1, 0, -1},  {1, 0, -1},  {-1, 0, 1},  {1, 0, 1},
    {-1, -1, 0},  {1, -1, 0},  {-1, 1, 0},  {1, 1, 0}};

// value and reference gradient of shape function a at (p0, p1, p2)
static __device__ inline void shape_one(int a, double p0, double p1, double p2, double* N,
                                        double* d) {
  const double r0 = c_ref[a][0], r1 = c_ref[a][1], r2 = c_ref[a][2];
  const double f0 = 1 + p0 * r0, f1 = 1 + p1 * r1, f2 = 1 + p2 * r2;
  if (r0 != 0 && r1 != 0 && r2 != 0) {
    const double g = p0 * r0 + p1 * r1 + p2 * r2 - 2;
    *N = 0.125 * f0 * f1 * f2 * g;
    d[0] = 0.125 * r0 * f1 * f2 * (g + f0);
    d[1] = 0.125 * r1 * f0 * f2 * (g + f1);
    d[2] = 0.125 * r2 * f0 * f1 * (g + f2);
  } else if (r0 == 0) {                          // edge along xi: bubble (1 - xi^2)
    const double b = 1 - p0 * p0;
    *N = 0.25 * b * f1 * f2;
    d[0] = -0.5 * p0 * f1 * f2;
    d[1] = 0.25 * b * r1 * f2;
    d[2] = 0.25 * b * f1 * r2;
  } else if (r1 == 0) {                          // edge along eta
    const double b = 1 - p1 * p1;
    *N = 0.25 * b * f0 * f2;
    d[0] = 0.25 * b * r0 * f2;
    d[1] = -0.5 * p1 * f0 * f2;
    d[2] = 0.25 * b * f0 * r2;
  } else {                                       // edge along zeta
    const double b = 1 - p2 * p2;
    *N = 0.25 * b * f0 * f1;
    d[0] = 0.25 * b * r0 * f1;
    d[1] = 0.25 * b * f0 * r1;
    d[2] = -0.5 * p2 * f0 * f1;
  }
}

// Coordinates of element nodes of a periodic mesh: node a of element e is seen at its
// stored coordinates plus the period when bit a of wrap[e] is set (wrap null: never).
struct Periodic {
  const uint32_t* wrap;
  double p[3];
};

static __device__ inline double node_coord(const double* xyz, int64_t nd, int i,
                                           const Periodic& P, int64_t e, int a) {
  double x = xyz[3 * nd + i];
  if (P.wrap && ((P.wrap[e] >> a) & 1u)) x += P.p[i];
  return x;
}

static __device__ inline void gauss3(int i, double* x, double* w) {
  const double s = 0.7745966692414833770358531;  // sqrt(3/5)
  *x = (i == 0) ? -s : ((i == 1) ? 0.0 : s);
  *w = (i == 1) ? 8.0 / 9.0 : 5.0 / 9.0;
}

// Reference gradients of the 20 nodes at the 27 Gauss points (q = i + 3 j + 9 k), by all
// threads of a work-group
static __device__ inline void ref_gradients(double (*dNr)[20][3]) {
  for (int idx = threadIdx.x; idx < 27 * 20; idx += blockDim.x) {
    const int q = idx / 20, a = idx % 20;
    double x0, x1, x2, w, N, d[3];
    gauss3(q % 3, &x0, &w);
    gauss3((q / 3) % 3, &x1, &w);
    gauss3(q / 9, &x2, &w);
    shape_one(a, x0, x1, x2, &N, d);
    for (int j = 0; j < 3; ++j) dNr[q][a][j] = d[j];
  }
}

// What the stress kernels need of one Gauss point of one element: the Jacobian (J[i][j] =
// dx_i / dxi_j), its determinant, the displacement gradient H[i][j] = du_i / dx_j and the
// geometric frame (rows of E: e1 along dx/dxi, e2 from dx/deta, e3 = e1 x e2).
static __device__ inline void point_state(const double (*X)[3], const double (*U)[3],
                                          const double (*dN)[3], double* det, double (&H)[3][3],
                                          double (&E)[3][3]) {
  double J[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, G[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll 4
  for (int a = 0; a < 20; ++a)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        J[i][j] += X[a][i] * dN[a][j];
        G[i][j] += U[a][i] * dN[a][j];             // du_i / dxi_j
      }
  *det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
         J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
         J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
  const double id = 1.0 / *det;
  double Ji[3][3];                               // Ji[j][i] = dxi_j / dx_i
  Ji[0][0] = (J[1][1] * J[2][2] - J[1][2] * J[2][1]) * id;
  Ji[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * id;
  Ji[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * id;
  Ji[1][0] = (J[1][2] * J[2][0] - J[1][0] * J[2][2]) * id;
  Ji[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * id;
  Ji[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * id;
  Ji[2][0] = (J[1][0] * J[2][1] - J[1][1] * J[2][0]) * id;
  Ji[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * id;
  Ji[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * id;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      H[i][j] = G[i][0] * Ji[0][j] + G[i][1] * Ji[1][j] + G[i][2] * Ji[2][j];
  const double n1 = sqrt(J[0][0] * J[0][0] + J[1][0] * J[1][0] + J[2][0] * J[2][0]);
#pragma unroll
  for (int i = 0; i < 3; ++i) E[0][i] = J[i][0] / n1;
  const double pr = J[0][1] * E[0][0] + J[1][1] * E[0][1] + J[2][1] * E[0][2];
#pragma unroll
  for (int i = 0; i < 3; ++i) E[1][i] = J[i][1] - pr * E[0][i];
  const double n2 = sqrt(E[1][0] * E[1][0] + E[1][1] * E[1][1] + E[1][2] * E[1][2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) E[1][i] /= n2;
  E[2][0] = E[0][1] * E[1][2] - E[0][2] * E[1][1];
  E[2][1] = E[0][2] * E[1][0] - E[0][0] * E[1][2];
  E[2][2] = E[0][0] * E[1][1] - E[0][1] * E[1][0];
}

// the context's description (defined where gx_ctx is complete)
template <class Ctx>
inline Periodic periodic_of(const Ctx* c) {
  Periodic P;
  P.wrap = c->wrap.p;
  for (int i = 0; i < 3; ++i) P.p[i] = c->period[i];
  return P;
}

}  // namespace gx
