// Through-thickness stresses and the delamination-onset criterion (section 3.3).
//
// The paper assesses the strength of the curved laminate with the quadratic criterion of
// Camanho et al. (Eq. eq-Camanho),
//
//   F = sqrt( (sigma_r^+ / s33)^2 + (tau_rs / s13)^2 + (tau_rl / s13)^2 ),
//
// sigma_r^+ = max(sigma_r, 0), evaluated in the resin interface layers only; failure
// initiates at F = 1, and since the problem is linear the moment at initiation is M / max F.
//
// Stresses are recovered at the 27 Gauss points of every selected element from the
// displacement: the strain of u_e, rotated into the material axes (the geometric frame
// e1 = unit dx/dxi, e2 = dx/deta made orthogonal, e3 = e1 x e2, turned by the ply angle
// about e3, as in the assembly), times the layer stiffness, then turned back by the ply
// angle into the frame (s, l, r) = (e1, e2, e3).  Two elements per wavefront, lane q of a half
// at Gauss point q; the element's maximum goes to a per-element slot, and those are reduced
// in a fixed order (ties go to the lower element, then the lower point), so the result is
// the same on every run.
#include <cmath>

#include "element.h"
#include "gx_internal.h"

namespace gx {

constexpr int FW = 4;                              // wavefronts per work-group
// The reference gradients sit in LDS (forming them anew at every point was most of the work:
// 92 -> 30 us for 33,600 elements, 11 of 35 element layers selected); what is left is the
// F values written and the layers' elements read.
__global__ void __launch_bounds__(64 * FW) k_failure(Periodic P, int64_t n_elems,
                                                     const double* xyz, const int32_t* conn,
                                                     const int32_t* elayer, const double* Cl,
                                                     const double* ang, const uint8_t* sel,
                                                     const double* u, double s33, double s13,
                                                     double* Fq, double* Fe, int32_t* qe,
                                                     double* Se) {
  __shared__ double dNr[27][20][3], X[2 * FW][20][3], U[2 * FW][20][3];
  ref_gradients(dNr);
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, hl = lane & 31;
  const int s = 2 * w + (lane >> 5);               // this half-wave's element slot
  for (int64_t e0 = (int64_t)blockIdx.x * 2 * FW; e0 < n_elems;
       e0 += (int64_t)gridDim.x * 2 * FW) {
    const int64_t e = e0 + s;
    const int layer = e < n_elems ? elayer[e] : 0;
    const bool in = e < n_elems && sel[layer];
    if (e < n_elems && !in) {
      if (hl < 27 && Fq) Fq[27 * e + hl] = 0.0;
      if (hl == 0) {
        Fe[e] = 0.0;
        qe[e] = 0;
      }
      if (hl < 6) Se[6 * e + hl] = 0.0;
    }
    if (!__any(in)) continue;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);       // (one wavefront: LDS accesses in order)
    __builtin_amdgcn_wave_barrier();
    if (in)
      for (int t = hl; t < 60; t += 32) {
        const int a = t / 3, i = t % 3;
        const int64_t nd = conn[20 * e + a];
        X[s][a][i] = node_coord(xyz, nd, i, P, e, a);
        U[s][a][i] = u[3 * nd + i];
      }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    double F = -1.0, loc[6] = {0, 0, 0, 0, 0, 0};
    if (in && hl < 27) {
      double det, H[3][3], E[3][3];
      point_state(X[s], U[s], dNr[hl], &det, H, E);
      const double an = ang[layer] * (M_PI / 180.0), ca = cos(an), sa = sin(an);
      double Q[3][3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        Q[0][i] = ca * E[0][i] + sa * E[1][i];
        Q[1][i] = -sa * E[0][i] + ca * E[1][i];
        Q[2][i] = E[2][i];
      }
      // strain in the material axes, eps' = Q sym(H) Q^T, engineering Voigt vector
      double T[3][3], em[3][3];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int b = 0; b < 3; ++b)
          T[i][b] = 0.5 * ((H[i][0] + H[0][i]) * Q[b][0] + (H[i][1] + H[1][i]) * Q[b][1] +
                           (H[i][2] + H[2][i]) * Q[b][2]);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
          em[a][b] = Q[a][0] * T[0][b] + Q[a][1] * T[1][b] + Q[a][2] * T[2][b];
      const double ev[6] = {em[0][0], em[1][1], em[2][2], 2.0 * em[1][2], 2.0 * em[0][2],
                            2.0 * em[0][1]};
      const double* C = Cl + 36 * layer;
      double sv[6];
#pragma unroll
      for (int I = 0; I < 6; ++I) {
        double acc = 0.0;
#pragma unroll
        for (int K = 0; K < 6; ++K) acc += C[6 * I + K] * ev[K];
        sv[I] = acc;
      }
      // back to the frame (s, l, r): sigma_geo = Rp sigma' Rp^T, Rp the rotation by the ply
      // angle about e3 (Rp[a][m] = e_a . q_m)
      const double Sm[3][3] = {{sv[0], sv[5], sv[4]}, {sv[5], sv[1], sv[3]}, {sv[4], sv[3], sv[2]}};
      const double Rp[3][3] = {{ca, -sa, 0.0}, {sa, ca, 0.0}, {0.0, 0.0, 1.0}};
      double R1[3][3], Sg[3][3];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int k = 0; k < 3; ++k)
          R1[a][k] = Rp[a][0] * Sm[0][k] + Rp[a][1] * Sm[1][k] + Rp[a][2] * Sm[2][k];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
          Sg[a][b] = R1[a][0] * Rp[b][0] + R1[a][1] * Rp[b][1] + R1[a][2] * Rp[b][2];
      loc[0] = Sg[0][0];
      loc[1] = Sg[1][1];
      loc[2] = Sg[2][2];
      loc[3] = Sg[1][2];
      loc[4] = Sg[0][2];
      loc[5] = Sg[0][1];
      const double sr = loc[2] > 0.0 ? loc[2] / s33 : 0.0;
      const double trs = loc[4] / s13, trl = loc[3] / s13;
      F = sqrt(sr * sr + trs * trs + trl * trl);
      if (Fq) Fq[27 * e + hl] = F;
    }
    // the half-wave's largest F (the lower point on a tie) and who holds it, as a scan from
    // the first point on finds it: a NaN there stays, one further on is passed over
    double best = hl > 0 && F != F ? -1.0 : F;
    int at = hl;
    for (int o = 1; o < 32; o <<= 1) {
      const double ob = __shfl_down(best, o, 32);
      const int oa = __shfl_down(at, o, 32);
      if (hl + o < 27 && ob > best) {
        best = ob;
        at = oa;
      }
    }
    at = __shfl(at, 0, 32);
    if (in && hl == at) {
      Fe[e] = F;
      qe[e] = at;
#pragma unroll
      for (int k = 0; k < 6; ++k) Se[6 * e + k] = loc[k];
    }
  }
}

// The largest F over all elements (ties: the lower element index): every work-group takes a
// slice, then one takes the slices' results in order and packs what the host reads.
struct FailPick {
  double F, stress[6];
  int64_t elem;
  int32_t gauss, layer;
};
constexpr int FSLICE = 64;
__device__ inline void fail_reduce(double& bv, int64_t& bi, double* v, int64_t* ix) {
  const int t = threadIdx.x;
  v[t] = bv;
  ix[t] = bi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
      const double ov = v[t + w];
      const int64_t oi = ix[t + w];
      if (ov > v[t] || (ov == v[t] && oi >= 0 && (ix[t] < 0 || oi < ix[t]))) {
        v[t] = ov;
        ix[t] = oi;
      }
    }
    __syncthreads();
  }
  bv = v[0];
  bi = ix[0];
}
__global__ void __launch_bounds__(256) k_failure_max(int64_t n_elems, const double* Fe,
                                                     double* pv, int64_t* pi) {
  __shared__ double v[256];
  __shared__ int64_t ix[256];
  const int64_t len = (n_elems + FSLICE - 1) / FSLICE, end = min(n_elems, (blockIdx.x + 1) * len);
  double bv = -1.0;
  int64_t bi = -1;
  for (int64_t e = blockIdx.x * len + threadIdx.x; e < end; e += 256)
    if (Fe[e] > bv) {
      bv = Fe[e];
      bi = e;
    }
  fail_reduce(bv, bi, v, ix);
  if (threadIdx.x == 0) {
    pv[blockIdx.x] = bv;
    pi[blockIdx.x] = bi;
  }
}
__global__ void __launch_bounds__(256) k_failure_pick(const double* pv, const int64_t* pi,
                                                      const int32_t* elayer, const int32_t* qe,
                                                      const double* Se, FailPick* out) {
  __shared__ double v[256];
  __shared__ int64_t ix[256];
  const int t = threadIdx.x;
  double bv = t < FSLICE ? pv[t] : -1.0;
  int64_t bi = t < FSLICE ? pi[t] : -1;
  fail_reduce(bv, bi, v, ix);
  if (t != 0) return;
  out->F = bv;
  out->elem = bi;
  if (bi < 0) return;
  out->gauss = qe[bi];
  out->layer = elayer[bi];
  for (int k = 0; k < 6; ++k) out->stress[k] = Se[6 * bi + k];
}

}  // namespace gx

using namespace gx;

extern "C" gx_status gx_failure(gx_ctx* c, const double* u, const int32_t* layer_mask,
                                double s33, double s13, double* F_gauss, double* F_elem,
                                gx_failure_result* out) {
  GX_API_BEGIN(c)
  if (!c->assembled) throw Error(GX_ESTATE, "matrix not assembled");
  if (c->matrix_only) throw Error(GX_ESTATE, "needs an assembled mesh, not a loaded matrix");
  GX_REQUIRE(u && out && s33 > 0 && s13 > 0, "bad failure-criterion arguments");
  hipStream_t st = c->stream;
  const int64_t E = c->n_elems;
  const int nl = c->n_layers;
  std::vector<uint8_t> hs(nl);
  int nsel = 0;
  for (int k = 0; k < nl; ++k) {
    // default: the isotropic layers (G12 <= 0 marks an isotropic entry of the ply stack)
    hs[k] = layer_mask ? (layer_mask[k] != 0) : !(c->eng[9 * k + 3] > 0);
    nsel += hs[k];
  }
  GX_REQUIRE(nsel > 0, "no layer selected for the failure criterion");
  DevBuf<uint8_t> sel(nl);
  to_dev(sel.p, hs.data(), nl, st);
  DevBuf<double> fe, se;
  DevBuf<int32_t> qe(E);
  DevBuf<int64_t> pi(FSLICE);
  DevBuf<double> pv(FSLICE);
  DevBuf<FailPick> pick(1);
  double* Fe = F_elem;
  if (!Fe) {
    fe.alloc(E);
    Fe = fe.p;
  }
  se.alloc(6 * E);
  hipLaunchKernelGGL(k_failure, dim3((unsigned)std::min<int64_t>(nblocks(E, 2 * FW), 2048)),
                     dim3(64 * FW), 0, st, periodic_of(c), E, c->xyz.p, c->conn.p, c->elayer.p,
                     c->Cl.p, c->ang.p, sel.p, u, s33, s13, F_gauss, Fe, qe.p, se.p);
  hipLaunchKernelGGL(k_failure_max, dim3(FSLICE), dim3(256), 0, st, E, Fe, pv.p, pi.p);
  hipLaunchKernelGGL(k_failure_pick, dim3(1), dim3(256), 0, st, pv.p, pi.p, c->elayer.p, qe.p,
                     se.p, pick.p);
  GX_HIP(hipGetLastError());
  FailPick h{};
  to_host(&h, pick.p, 1, st);
  GX_REQUIRE(h.elem >= 0 && h.elem < E, "no element of the selected layers");
  out->F_max = h.F;
  out->elem = h.elem;
  out->gauss = h.gauss;
  out->layer = h.layer;
  for (int k = 0; k < 6; ++k) out->stress[k] = h.stress[k];
  GX_API_END(c)
}
