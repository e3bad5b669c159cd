// Batched banded Cholesky factorisation and triangular solves.
//
// The local problems of the overlapping Schwarz method are solved exactly by a direct
// method (section 2.4: sparse direct subdomain and coarse solves).  In the laminate DOF
// order (through-thickness planes outermost) every subdomain matrix is banded with a
// half bandwidth of about two lattice planes, so its Cholesky factor fits in band storage
// with no fill outside the band.
//
// Storage of a part: entry (r, c), r - B <= c <= r, at off + r * ld + (c - r + B).
//
// Both the factorisation and the solves are chains of dependent 64-row steps, and with few
// matrices a chain's latency, not bandwidth or arithmetic, sets the time.  A matrix whose
// order is several times its bandwidth is therefore eliminated from both ends at once, in
// two parts that meet in a separator of one bandwidth (BandPart, split_rows): half the
// chain, the same entries and the same flops.
//
// Factorisation: right-looking, block columns of NB taken GP at a time; one launch per
// group factors its panels (diagonal blocks, their inverses, kept for the solves, and the
// panel rows), and the trailing window is updated with 128x128 tiles.  Matrices of
// different size and bandwidth run in the same launches.
//
// Solves: see the comment above the solve kernels.
#include <algorithm>

#include "gx_internal.h"

namespace gx {

constexpr int NB = 64;          // factorisation block
constexpr int TS = 64;          // trailing-update tile
constexpr int SB = 64;          // solve block (one wavefront)
static_assert(SB == NB, "solve blocks are the factorisation's");
constexpr int SOLVE_THREADS = 512;

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// The 16x16x4 matrix instruction in the precision of a factor: FP64 factors multiply in FP64,
// FP32 factors (the mixed path) in FP32.  Both take A[l % 16][l / 16] and B[l / 16][l % 16]
// from lane l; the output row of accumulator register q differs: 4 q + l / 16 in FP64,
// 4 (l / 16) + q in FP32.  S is the type staged in LDS and multiplied.
template <class T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef double S;
  typedef v4d V;
  static __device__ inline V mma(S a, S b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ inline int row(int q, int lk) { return 4 * q + lk; }
};
template <>
struct Mfma<float> {
  typedef float S;
  typedef v4f V;
  static __device__ inline V mma(S a, S b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ inline int row(int q, int lk) { return 4 * lk + q; }
};

struct BandArgs {
  const BandPart* part;
  const int64_t* fcb;                             // envelope tables by 64-row blocks
  const int64_t* lrb;
  int phase;                                      // factorisation: before, at the separators
};

// ---- Factorisation: right-looking blocked Cholesky in groups of GP panels of NB columns.
// The columns of a group [k0, k0 + GP NB) are factored by two launches: k_chain for the
// group's own rows, k_far for the rows below them.  The update of the trailing window by
// the group's panels is split in two k_syrk_wide launches: the next group's columns (then
// that group's k_chain, on the same stream), and all further columns on a second stream,
// at the same time.  The separators of split matrices follow in a second phase of the same
// launches, after k_merge.  k0 counts from the first column of the part's phase.
constexpr int GP = 4;                             // panels per group
constexpr int CT = 256;                           // threads of a panel work-group
constexpr int64_t SPIN_LIMIT = (int64_t)1 << 22;  // polls before a wait gives up

// Counters, flags and error words that the next launch takes its numbers from or polls are
// cleared by a kernel, ordered on the stream like the launches themselves.
__global__ void k_clear(int* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}
static void clear(DevBuf<int>& b, hipStream_t st) {
  hipLaunchKernelGGL(k_clear, dim3(nblocks((int64_t)b.n, 256)), dim3(256), 0, st, b.p,
                     (int64_t)b.n);
}

// Loads and stores of data handed between the work-groups of one launch: agent-scope
// relaxed atomics, which bypass the per-XCD caches, so a reader sees the writer's values
// without a cache flush or invalidate on either side.
template <class T>
__device__ inline T co_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ inline void co_store(T* p, T x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Raises a block's flag to this launch's epoch once every thread's hand-over stores have
// completed (waited for per thread, then a barrier).
__device__ inline void chain_signal(int* f, int epoch) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(f, epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Bounded poll of a flag (thread 0); a poll that gives up raises bit 2 of the error word,
// and polls stop early once that bit is up, so every wave still reaches the end of the
// kernel.
__device__ inline void chain_wait(const int* f, int epoch, int* err) {
  for (int64_t k = 0; k < SPIN_LIMIT; ++k) {
    if (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= epoch) return;
    if ((k & 255) == 255 && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 2))
      return;
    __builtin_amdgcn_s_sleep(1);
  }
  atomicOr(err, 2);
}

// One launch per group for the group's own rows: the GP x GP triangle of 64-row blocks from
// the diagonal block of the first panel down.  Work-group (t, j) owns row block t of matrix
// j, the 64 rows [k0 + 64 t, + 64), and keeps its t + 1 blocks in registers from the start:
//   1. Panel by panel, q < t: L(t, q) = A(t, q) Li(q)^T once the inverse Li(q) of that panel's
//      diagonal block is handed over (FP64 instruction); the block is stored.
//   2. Its products are taken off the row's other blocks at once, with the matrix instruction
//      in the factor's precision: A(t, t) -= L(t, q) L(t, q)^T, and for q < m < t
//      A(t, m) -= L(t, q) L(m, q)^T with row block m's result.
//   3. Cholesky of A(t, t) and the inverse of its factor; the inverse is handed to the
//      work-groups of the later row blocks and kept for the triangular solves.
// The launch is a chain of GP diagonal blocks, on one work-group at a time.  What lies
// between two of them is one hand-over (the inverse; a row block's own products never leave
// its work-group), two 64^3 products and the factorisation itself; everything else runs
// beside it.  With a work-group per block a step was two hand-overs and the reload of all
// earlier panels, and one wave factored and inverted the diagonal block: 33 us a step, now 17,
// of which 4 x 2.7 us are the four block columns of step 3.  Per launch: 131 -> 77 us (8 parts, B =
// 370, FP64), 160 -> 94 (FP32, B = 540), 218 -> 151 (32 parts, B = 1,630, beside the update).
// Work-groups are numbered by row block, then matrix, and take their number from a counter
// of the launch when they start, not from their position in the grid; a work-group waits for
// lower row blocks of its matrix only, so every wait is for a work-group that is already
// running: the launch cannot deadlock, whatever order the hardware dispatches its
// work-groups in and whatever else occupies the device.
// A non-positive pivot raises bit 1 of the error word (and may leave NaNs behind it).
template <class T>
__global__ void __launch_bounds__(CT, 2) k_chain(BandArgs a, T* v, int64_t kg, int n_mat,
                                              int* flags, int* ticket, int epoch, double* inv,
                                              T* dinv, int* err) {
  typedef Mfma<T> MT;
  typedef typename MT::S S;
  constexpr int XS = sizeof(S) == 8 ? NB + 1 : NB + 4;   // LDS stride of a finished block
  __shared__ double D[NB][NB + 1];               // a block of A; the diagonal block's factor
  __shared__ double Li[NB][NB + 1];              // the inverse of a diagonal block
  __shared__ double Wd[NB / 16][16][17];         // inverses of the 16x16 diagonal blocks
  __shared__ double rd[NB];                      // reciprocals of the pivots
  __shared__ int tk;
  static_assert(NB * XS * sizeof(S) <= sizeof(D), "finished blocks fit in the block buffers");
  S* X = reinterpret_cast<S*>(&D[0][0]);         // L(t, q) (aliases D)
  S* Y = reinterpret_cast<S*>(&Li[0][0]);        // L(m, q) (aliases Li)
  if (threadIdx.x == 0) tk = atomicAdd(ticket, 1);
  __syncthreads();
  const int b = __builtin_amdgcn_readfirstlane(tk), t = b / n_mat, j = b - t * n_mat;
  const BandPart& P = a.part[j];
  const int64_t k0l = P.fb[a.phase] + kg;
  if (k0l >= P.fe[a.phase] || k0l + NB * t >= P.rows) return;
  const int n = (int)P.rows, B = (int)P.B, rs = (int)P.ld - 1;
  const int k0 = (int)k0l, ce = (int)P.fe[a.phase], r0 = k0 + NB * t;
  const int np = min(t, (ce - k0 + NB - 1) / NB);  // panels left of the row's diagonal block
  const bool diag = r0 < ce;                       // the row block has a panel
  auto reach = [&](int rb, int q) { return NB * (rb - q) <= NB - 1 + B; };  // block not empty
  T* base = v + P.off;
  auto at = [&](int r, int c) { return (uint32_t)(r * rs + B + c); };     // entry (r, c)
  int* fj = flags + (int64_t)j * GP * GP;          // flag of block (m, q): fj[GP m + q]
  int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int li = lane & 15, lk = lane >> 4;
  // Behind this the compiler takes the lane's place for new: the conditions and addresses
  // of one step, kept for the next, would not fit in the registers.
  auto forget = [&]() { asm volatile("" : "+v"(lane), "+v"(li), "+v"(lk)); };
  const int wr = 32 * (w & 1), wc = 32 * (w >> 1);
  // The row's blocks, in the matrix instruction's result layout (entries outside the matrix
  // or the band are 0; the diagonal block keeps its lower triangle): av[d] is A(t, q + d).
  double av[GP - 1][2][4][2], ad[2][4][2];
  auto inside = [&](int q, bool low, int rl, int cl) {
    const int r = r0 + rl, c = k0 + NB * q + cl;
    return r < n && c < ce && c >= r - B && (!low || cl <= rl);
  };
  // The loads of all blocks are issued before the first is used; outside entries load
  // entry (0, 0) and are zeroed by a second look at the conditions.
  auto load = [&](double (&x)[2][4][2], int q, bool low) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int rl = wr + 16 * i + MT::row(e, lk), cl = wc + 16 * jj + li;
          x[i][e][jj] = base[inside(q, low, rl, cl) ? at(r0 + rl, k0 + NB * q + cl) : (uint32_t)B];
        }
  };
  auto clip = [&](double (&x)[2][4][2], int q, bool low) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
          if (!inside(q, low, wr + 16 * i + MT::row(e, lk), wc + 16 * jj + li)) x[i][e][jj] = 0.0;
  };
#pragma unroll
  for (int q = 0; q < GP - 1; ++q)
    if (q < np) load(av[q], q, false);
  if (diag) load(ad, t, true);
  forget();
#pragma unroll
  for (int q = 0; q < GP - 1; ++q)
    if (q < np) clip(av[q], q, false);
  if (diag) clip(ad, t, true);
  // x -= U V^T with finished blocks in LDS
  auto update = [&](double (&x)[2][4][2], const S* U, const S* V) {
    typename MT::V acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) acc[i][jj] = typename MT::V{0, 0, 0, 0};
#pragma unroll 4
    for (int k = 0; k < NB; k += 4) {
      S fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[i] = U[(wr + 16 * i + li) * XS + k + lk];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) fb[jj] = V[(wc + 16 * jj + li) * XS + k + lk];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) acc[i][jj] = MT::mma(fa[i], fb[jj], acc[i][jj]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) x[i][e][jj] -= (double)acc[i][jj][e];
  };
  auto to_D = [&](const double (&x)[2][4][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
          D[wr + 16 * i + MT::row(e, lk)][wc + 16 * jj + li] = x[i][e][jj];
  };
#pragma unroll 1
  for (int q = 0; q < np; ++q) {
    if (reach(t, q)) {
      forget();
      // 1.
      const int c0 = k0 + NB * q;
      to_D(av[0]);
      if (threadIdx.x == 0) chain_wait(fj + GP * q + q, epoch, err);
      __syncthreads();
      const double* iq = inv + ((int64_t)j * GP + q) * NB * NB;
      double lv[NB * NB / CT];                     // all loads issued before any is used
#pragma unroll
      for (int u = 0; u < NB * NB / CT; ++u) lv[u] = co_load(iq + threadIdx.x + CT * u);
#pragma unroll
      for (int u = 0; u < NB * NB / CT; ++u)
        Li[w + CT / NB * u][lane] = lv[u];
      __syncthreads();
      v4d x[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) x[i][jj] = v4d{0, 0, 0, 0};
#pragma unroll 4
      for (int k = 0; k < NB; k += 4) {
        double fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[i] = D[wr + 16 * i + li][k + lk];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) fb[jj] = Li[wc + 16 * jj + li][k + lk];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) x[i][jj] = Mfma<double>::mma(fa[i], fb[jj], x[i][jj]);
      }
      __syncthreads();                             // D and Li are read
      forget();
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const int rl = wr + 16 * i + Mfma<double>::row(e, lk), cl = wc + 16 * jj + li;
            const int r = r0 + rl, c = c0 + cl;
            const bool ok = r < n && c < ce && c >= r - B;
            if (ok) co_store(base + at(r, c), (T)x[i][jj][e]);
            X[rl * XS + cl] = ok ? (S)(T)x[i][jj][e] : (S)0;
          }
      __syncthreads();
      // 2.
      if (diag) update(ad, X, X);
      chain_signal(fj + GP * t + q, epoch);        // (the stores drained beside the product)
#pragma unroll
      for (int d = 1; d < GP - 1; ++d) {
        const int m = q + d;
        if (m >= np || !reach(m, q)) continue;
        if (threadIdx.x == 0) chain_wait(fj + GP * m + q, epoch, err);
        __syncthreads();
        // (the rows are inside the matrix; outside the band they read entry (0, 0))
        T yv[NB * NB / CT];
        const int lo = NB * d + w - B;             // first column of the block's row w
#pragma unroll
        for (int u = 0; u < NB * NB / CT; ++u)
          yv[u] = co_load(base + (lane >= lo + CT / NB * u
                                      ? at(k0 + NB * m + w + CT / NB * u, c0 + lane)
                                      : (uint32_t)B));
        forget();
#pragma unroll
        for (int u = 0; u < NB * NB / CT; ++u)
          Y[(w + CT / NB * u) * XS + lane] = lane >= lo + CT / NB * u ? (S)yv[u] : (S)0;
        __syncthreads();
        update(av[d], X, Y);
        __syncthreads();                           // Y is read
      }
    }
#pragma unroll
    for (int d = 0; d + 1 < GP - 1; ++d)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) av[d][i][e][jj] = av[d + 1][i][e][jj];
    __syncthreads();                               // X is read
  }
  if (!diag) return;
  forget();
  const int nb = min(NB, ce - r0);                 // columns of the panel inside the matrix
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int rl = wr + 16 * i + MT::row(e, lk), cl = wc + 16 * jj + li;
        if (rl == cl && rl >= nb) ad[i][e][jj] = 1.0;   // padding of a short last panel
      }
  to_D(ad);
  __syncthreads();
  // 3. Cholesky of the diagonal block and its inverse, in 16-column blocks.  Stage kb: wave 0
  // factors block column kb for all the rows below it in registers (lane r holds row r;
  // pivots and column entries come from other lanes by reads of their registers), wave 1
  // extends the inverse by block row kb - 1, waves 2 and 3 take column kb - 1's products off
  // the tiles right of column kb; then column kb's products are taken off column kb + 1, a
  // tile to a wave.  With L the factor and W_i the inverses of its diagonal tiles, block row
  // i of the inverse is W_i and -W_i S(i, j), S(i, j) = sum_{j <= k < i} L(i, k) Li(k, j):
  // after the last stage only W_3 and one product are left.
  typedef Mfma<double> M64;
  // scratch tile of wave-local products and of S(3, j): above D's diagonal, read by nothing
  auto tmp = [&](int i, int j2, int l) -> double& { return D[i][16 * (j2 + 1) + l]; };
  auto invert_tile = [&](int i) {                  // W_i, lane c: column c
    const int b0 = 16 * i, c16 = lane & 15;
    double x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = k == c16 ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      x[k] *= rd[b0 + k];
#pragma unroll
      for (int l = k + 1; l < 16; ++l) x[l] -= D[b0 + l][b0 + k] * x[k];
    }
    if (lane < 16)
#pragma unroll
      for (int k = 0; k < 16; ++k) Wd[i][k][c16] = x[k];
  };
  auto row_sum = [&](int i, int j2) {              // S(i, j2) into the scratch tile j2
    v4d acc = v4d{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)                 // k = j2: Li(j2, j2) = W_j2
      acc = M64::mma(D[16 * i + li][16 * j2 + 4 * ks + lk], Wd[j2][4 * ks + lk][li], acc);
#pragma unroll 1
    for (int k = j2 + 1; k < i; ++k)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        acc = M64::mma(D[16 * i + li][16 * k + 4 * ks + lk],
                       Li[16 * k + 4 * ks + lk][16 * j2 + li], acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) tmp(M64::row(e, lk), j2, li) = acc[e];
  };
  auto row_inverse = [&](int i, int j2) {          // Li(i, j2) = -W_i S(i, j2)
    v4d acc = v4d{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      acc = M64::mma(Wd[i][li][4 * ks + lk], tmp(4 * ks + lk, j2, li), acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) Li[16 * i + M64::row(e, lk)][16 * j2 + li] = -acc[e];
  };
  auto tile_update = [&](int ti, int tj, int kb) {  // A(ti, tj) -= L(ti, kb) L(tj, kb)^T
    v4d acc = v4d{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      acc = M64::mma(D[16 * ti + li][16 * kb + 4 * ks + lk], D[16 * tj + li][16 * kb + 4 * ks + lk],
                     acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) D[16 * ti + M64::row(e, lk)][16 * tj + li] -= acc[e];
  };
#pragma unroll 1
  for (int kb = 0; kb < 4; ++kb) {
    const int b0 = 16 * kb;
    if (w == 0) {
      double f[16], u[16], piv = 1.0, g = 0.0;     // piv: pivot i in lane b0 + i
#pragma unroll
      for (int c = 0; c < 16; ++c) f[c] = lane >= b0 + c ? D[lane][b0 + c] : 0.0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        // column i is left unscaled and enters the later ones as (f_i / d) f_i^T: the chain
        // from pivot to pivot is one reciprocal (the hardware's estimate r, then
        // r (1 + e + e^2), e = 1 - d r: full FP64 precision), a product and a
        // subtraction; the square roots follow for all 16 at once.  Column i - 1's
        // products for the columns after i are taken off meanwhile.
        const double d = lane_value(f[i], b0 + i);
        piv = lane == b0 + i ? d : piv;
        double r = __builtin_amdgcn_rcp(d);
        const double e = 1.0 - d * r;
        r += r * (e + e * e);
#pragma unroll
        for (int c = i + 1; c < 16; ++c) {
          if (i > 0) f[c] -= g * u[c];
          u[c] = lane_value(f[i], b0 + c);
        }
        g = f[i] * r;
        if (i < 15) f[i + 1] -= g * u[i + 1];
        __builtin_amdgcn_sched_barrier(0);
      }
      // 1 / sqrt: the hardware's estimate, then two Newton steps q <- q (3 - d q^2) / 2
      const bool bad = !(piv > 0.0);
      if (__any(bad) && lane == 0) atomicOr(err, 1);
      if (bad) piv = 1.0;
      double q = __builtin_amdgcn_rsq(piv);
      q = q * (1.5 - 0.5 * piv * q * q);
      q = q * (1.5 - 0.5 * piv * q * q);
      const double dl = bad ? 1.0 : piv * q;
      if (lane >= b0 && lane < b0 + 16) rd[lane] = q;
#pragma unroll
      for (int c = 0; c < 16; ++c) f[c] *= lane_value(q, b0 + c);
      if (lane >= b0)
#pragma unroll
        for (int c = 0; c < 16; ++c)
          D[lane][b0 + c] = lane > b0 + c ? f[c] : lane == b0 + c ? dl : 0.0;
    } else if (w == 1) {
      if (kb > 0) {
        invert_tile(kb - 1);
#pragma unroll 1
        for (int j2 = 0; j2 < kb - 1; ++j2) {
          row_sum(kb - 1, j2);
          __builtin_amdgcn_wave_barrier();
          row_inverse(kb - 1, j2);
          __builtin_amdgcn_wave_barrier();
        }
        if (kb == 3)
#pragma unroll 1
          for (int j2 = 0; j2 < 3; ++j2) row_sum(3, j2);
      }
    } else if (kb > 0 && kb < 3) {
      int id = w;                                  // dealt to waves 2 and 3 in turn
      for (int tj = kb + 1; tj < 4; ++tj)
        for (int ti = tj; ti < 4; ++ti, ++id)
          if ((id & 1) == 0) tile_update(ti, tj, kb - 1);
    }
    if (kb == 3) break;
    __syncthreads();
    if (kb + 1 + w < 4) tile_update(kb + 1 + w, kb + 1, kb);
    __syncthreads();
  }
  if (w == 0) invert_tile(3);
  __syncthreads();
  if (w < 3) row_inverse(3, w);
  __syncthreads();
  // the inverse first, then what nothing waits for in this launch
  auto inverse = [&](int i, int l) {
    return l > i ? 0.0 : (i >> 4) == (l >> 4) ? Wd[i >> 4][i & 15][l & 15] : Li[i][l];
  };
  double* it = inv + ((int64_t)j * GP + t) * NB * NB;
#pragma unroll 4
  for (int idx = threadIdx.x; idx < NB * NB; idx += CT)
    co_store(it + idx, inverse(idx / NB, idx % NB));
  chain_signal(fj + GP * t + t, epoch);
  T* dj = dinv + P.boff + (int64_t)(r0 / NB) * NB * NB;
#pragma unroll 4
  for (int idx = threadIdx.x; idx < NB * NB; idx += CT) {
    const int i = idx / NB, l = idx % NB;
    dj[idx] = (T)inverse(i, l);
    if (i < nb && l <= i && i - l <= B) base[at(r0 + i, r0 + l)] = (T)D[i][l];
  }
}

template <class S>
struct Chunk;                                     // reduction chunk: KC columns, LDS stride KS
template <>
struct Chunk<double> {
  static constexpr int KC = 32, KS = 34;
};
template <>
struct Chunk<float> {
  static constexpr int KC = 64, KS = 68;
};

// The rows below a group (row blocks GP, GP + 1, .. counted from k0) for all of the
// group's panels, once k_chain has factored the group's own rows: work-group (j, f) owns
// the 64 rows [k0 + 64 (GP + f), + 64) of matrix j and takes the panels in turn: the update
// by the group's earlier panels (from its own results and the group's rows), then the product
// with the inverse of the panel's diagonal block.  Everything it reads was written by earlier
// launches or by itself, so nothing is waited for and plain loads suffice.
template <class T>
__global__ void __launch_bounds__(CT, 2) k_far(BandArgs a, T* v, int64_t kg, int NF, int n_mat,
                                               const double* inv) {
  typedef Mfma<T> MT;
  typedef typename MT::S S;
  constexpr int KC = Chunk<S>::KC, KS = Chunk<S>::KS;
  constexpr int VW = 16 / sizeof(S);             // entries per 16-byte load
  typedef S SV __attribute__((ext_vector_type(VW)));
  constexpr int RP = CT / (KC / VW);             // rows staged per pass
  constexpr int PER = NB / RP;                   // 16-byte loads per thread and operand
  __shared__ __attribute__((aligned(16))) double D[NB][NB + 1];    // the block
  __shared__ __attribute__((aligned(16))) double Li[NB][NB + 1];   // the inverse of the
                                                                   // panel's diagonal block
  static_assert(NB * KS * sizeof(S) <= sizeof(D), "staging fits in the block buffers");
  static_assert(KS * sizeof(S) % 16 == 0, "staged rows start on 16 bytes");
  S* Pr = reinterpret_cast<S*>(&D[0][0]);        // staging of the update (aliases D and Li)
  S* Ps = reinterpret_cast<S*>(&Li[0][0]);
  const int j = blockIdx.x / NF, f = blockIdx.x % NF;
  if (j >= n_mat) return;
  const BandPart& P = a.part[j];
  const int64_t n = P.rows, B = P.B, ld = P.ld;
  const int64_t k0 = P.fb[a.phase] + kg, ce = P.fe[a.phase];
  const int64_t r0 = k0 + (int64_t)NB * (GP + f);
  if (k0 >= ce || r0 >= n) return;
  T* base = v + P.off;
  const int64_t rs = ld - 1;                     // entry (r, c) at r * rs + B + c
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wr = 32 * (w & 1), wc = 32 * (w >> 1);
  const int kc_t = threadIdx.x % (KC / VW) * VW, i0 = threadIdx.x / (KC / VW);
#pragma unroll 1
  for (int p = 0; p < GP; ++p) {
    const int64_t c0 = k0 + (int64_t)NB * p;
    if (c0 >= ce || r0 > c0 + NB - 1 + B) continue;  // no entries in this panel
    const int nb = (int)min<int64_t>(NB, ce - c0);
    // the block's entries and the inverse of the panel's diagonal block are loaded first, so
    // that they arrive during the update
    T av[2][4][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int rl = wr + 16 * i + MT::row(q, lk), cl = wc + 16 * jj + li;
          const int64_t r = r0 + rl, c = c0 + cl;
          av[i][q][jj] = (r < n && cl < nb && c >= r - B) ? base[r * rs + B + c] : (T)0;
        }
    const double* invj = inv + ((int64_t)j * GP + p) * NB * NB;
    double lv[NB * NB / CT];
#pragma unroll
    for (int u = 0; u < NB * NB / CT; ++u) lv[u] = invj[threadIdx.x + CT * u];
    typename MT::V acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) acc[i][jj] = typename MT::V{0, 0, 0, 0};
    if (p > 0) {
      const int64_t lo = max(r0 - B, a.fcb[P.eoff + r0 / NB]);
      const int64_t kstart = lo > k0 ? k0 + (lo - k0) / KC * KC : k0;
      // Each thread loads VW consecutive entries of a row at once (16 bytes: rows start on
      // 128-byte lines and k0 + (kc - k0) + kc_t is a multiple of VW, so the loads are
      // aligned).  The loads are unconditional: rows past the end of the matrix read at
      // most NB rows further, which the band allocation's padding covers, and entries
      // outside the band or the window are masked when they are staged.
      SV xr[PER], xs[PER];
      const int lim_r = (int)min<int64_t>(n - r0, NB), lim_s = (int)min<int64_t>(n - c0, NB);
      const int lo_r = (int)(r0 - B - k0), lo_s = (int)(c0 - B - k0), qend = (int)(c0 - k0);
      const uint32_t or0 = (uint32_t)((r0 + i0) * rs + B + k0 + kc_t);
      const uint32_t os0 = (uint32_t)((c0 + i0) * rs + B + k0 + kc_t);
      const uint32_t ostep = (uint32_t)(RP * rs);
      auto fetch = [&](int64_t kc) {
        const uint32_t kd = (uint32_t)(kc - k0);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          xr[u] = *reinterpret_cast<const SV*>(base + (or0 + u * ostep + kd));
          xs[u] = *reinterpret_cast<const SV*>(base + (os0 + u * ostep + kd));
        }
      };
      if (kstart < c0) fetch(kstart);
      for (int64_t kc = kstart; kc < c0; kc += KC) {
        const int qq = (int)(kc - k0) + kc_t;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int i = i0 + RP * u;
          SV wr_, ws_;
#pragma unroll
          for (int e = 0; e < VW; ++e) {
            const int q = qq + e;
            wr_[e] = (q < qend && i < lim_r && q - i >= lo_r) ? xr[u][e] : (S)0;
            ws_[e] = (q < qend && i < lim_s && q - i >= lo_s) ? xs[u][e] : (S)0;
          }
          *reinterpret_cast<SV*>(&Pr[i * KS + kc_t]) = wr_;
          *reinterpret_cast<SV*>(&Ps[i * KS + kc_t]) = ws_;
        }
        __syncthreads();
        if (kc + KC < c0) fetch(kc + KC);
#pragma unroll 4
        for (int k = 0; k < KC; k += 4) {
          S fa[2], fb[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) fa[i] = Pr[(wr + 16 * i + li) * KS + k + lk];
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) fb[jj] = Ps[(wc + 16 * jj + li) * KS + k + lk];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) acc[i][jj] = MT::mma(fa[i], fb[jj], acc[i][jj]);
        }
        __syncthreads();
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int rl = wr + 16 * i + MT::row(q, lk), cl = wc + 16 * jj + li;
          D[rl][cl] = (double)av[i][q][jj] - (double)acc[i][jj][q];
        }
#pragma unroll
    for (int u = 0; u < NB * NB / CT; ++u) {
      const int idx = threadIdx.x + CT * u;
      Li[idx / NB][idx % NB] = lv[u];
    }
    __syncthreads();
    v4d x[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) x[i][jj] = v4d{0, 0, 0, 0};
#pragma unroll 4
    for (int k = 0; k < NB; k += 4) {
      double fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[i] = D[wr + 16 * i + li][k + lk];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) fb[jj] = Li[wc + 16 * jj + li][k + lk];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) x[i][jj] = Mfma<double>::mma(fa[i], fb[jj], x[i][jj]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int rl = wr + 16 * i + Mfma<double>::row(q, lk), cl = wc + 16 * jj + li;
          const int64_t r = r0 + rl, c = c0 + cl;
          if (r < n && cl < nb && c >= r - B) base[r * rs + B + c] = (T)x[i][jj][q];
        }
    // this panel's rows are read back by the next panel's update (other threads), and the
    // LDS buffers are restaged
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
}

// The update of the trailing window by a group's panels, past the next group's columns,
// in 128 x 128 tiles of its lower triangle.  Eight waves each
// form a 64 x 32 eighth as 4 x 2 matrix-instruction tiles of 16 x 16, so six fragment reads
// from LDS feed eight instructions; two work-groups fit a compute unit.  The panels stream through LDS in chunks
// of KW columns (128 bytes of a row in FP64, 256 in FP32); the next chunk is loaded into registers while the
// current one is multiplied.  Chunks that lie left of the band for every row of the tile
// are skipped.  The LDS row stride (KW plus 2 doubles or 4 floats) spreads the 16 rows x 4
// reduction indices of one fragment read over distinct banks.
// The grid is one-dimensional over (matrix, tile) and consecutive tiles of a matrix go to
// the same XCD (work-groups are dealt round-robin to the eight XCDs), so a matrix's panels
// stay in that XCD's L2 while its tiles run.
constexpr int T2 = 128;                           // tile edge
constexpr int U2 = 512;                           // threads
template <class S>
struct Wide;
template <>
struct Wide<double> {
  static constexpr int KW = 16, KS = 18;
};
template <>
struct Wide<float> {
  static constexpr int KW = 64, KS = 68;
};

template <class T>
__device__ inline void wide_tile(BandArgs a, T* v, int64_t kg, int64_t kk, int64_t ts_lo,
                                 int64_t ts_hi, int64_t per_mat, int64_t lin) {
  typedef Mfma<T> MT;
  typedef typename MT::S S;
  constexpr int KW = Wide<S>::KW, KS = Wide<S>::KS;
  constexpr int VW = 16 / sizeof(S);             // entries per 16-byte load
  typedef S SV __attribute__((ext_vector_type(VW)));
  constexpr int RP = U2 / (KW / VW);             // rows staged per pass
  constexpr int PER = T2 / RP;                   // 16-byte loads per thread and operand
  __shared__ __attribute__((aligned(16))) S Pr[T2][KS];
  __shared__ __attribute__((aligned(16))) S Ps[T2][KS];
  const int j = (int)(lin / per_mat);
  const int64_t tile = lin - (int64_t)j * per_mat;
  const BandPart& P = a.part[j];
  const int64_t n = P.rows, B = P.B, ld = P.ld;
  const int64_t k0 = P.fb[a.phase] + kg, ce = P.fe[a.phase];
  if (k0 >= ce) return;
  const int64_t kj = min<int64_t>(kk, ce - k0);
  const int64_t t0 = k0 + kj;
  const int64_t W = min<int64_t>(B, n - t0);
  if (W <= 0) return;
  const int64_t nt = (W + T2 - 1) / T2;
  const int64_t te = min(ts_hi, nt);
  int64_t ts, rem = tile;
  for (ts = ts_lo; ts < te && rem >= nt - ts; ++ts) rem -= nt - ts;
  if (ts >= te) return;
  const int64_t tr = ts + rem;
  T* base = v + P.off;
  const int64_t r0 = t0 + tr * T2, s0 = t0 + ts * T2, wend = t0 + W;
  const int64_t rs = ld - 1;                     // entry (r, c) at r * rs + B + c
  const int kc_t = threadIdx.x % (KW / VW) * VW, i0 = threadIdx.x / (KW / VW);
  // first chunk with an entry inside the envelope of the tile's rows (its two 64-row blocks)
  const int64_t* fcj = a.fcb + P.eoff;
  const int64_t b0 = r0 / NB;
  const int64_t fmin = b0 + 1 < (n + NB - 1) / NB ? min(fcj[b0], fcj[b0 + 1]) : fcj[b0];
  const int64_t lo = max(r0 - B, fmin) - k0;
  const int64_t kc_first = lo > 0 ? lo / KW * KW : 0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wr = 64 * (w & 1), wc = 32 * (w >> 1);
  const bool idle = ts == tr && wc >= wr + 64;   // above the diagonal of a diagonal tile
  typename MT::V acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) acc[i][jj] = typename MT::V{0, 0, 0, 0};
  SV vr[PER], vs[PER];
  // 32-bit offsets from the matrix start (the host checks that they fit).  Rows past the
  // end of the matrix are not clamped: they read at most T2 rows further, which the band
  // allocation's padding covers, and are masked.  Each thread loads VW consecutive entries
  // of a row at once: rows start on 128-byte lines and k0 + kc + kc_t is a multiple of VW,
  // so every load is 16-byte aligned.
  const uint32_t ostep = (uint32_t)(RP * rs);
  const uint32_t or0 = (uint32_t)((r0 + i0) * rs + B + k0 + kc_t);
  const uint32_t os0 = (uint32_t)((s0 + i0) * rs + B + k0 + kc_t);
  auto load = [&](int64_t kc) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      vr[u] = *reinterpret_cast<const SV*>(base + (or0 + u * ostep + (uint32_t)kc));
      vs[u] = *reinterpret_cast<const SV*>(base + (os0 + u * ostep + (uint32_t)kc));
    }
  };

  // masks in 32-bit tile-relative terms: row i of a block is inside the window if
  // i < lim, and panel column q (0-based in the group) is inside the band of that row if
  // q - i >= lo (the block's first row starts the band at panel column lo)
  const int lim_r = (int)min<int64_t>(wend - r0, T2), lim_s = (int)min<int64_t>(wend - s0, T2);
  const int lo_r = (int)(r0 - B - k0), lo_s = (int)(s0 - B - k0);
  const int kjn = (int)kj;
  auto stage = [&](int64_t kc) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = i0 + RP * u;
      SV wr_, ws_;
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        const int q = (int)kc + kc_t + e;
        wr_[e] = (q < kjn && i < lim_r && q - i >= lo_r) ? vr[u][e] : (S)0;
        ws_[e] = (q < kjn && i < lim_s && q - i >= lo_s) ? vs[u][e] : (S)0;
      }
      *reinterpret_cast<SV*>(&Pr[i][kc_t]) = wr_;
      *reinterpret_cast<SV*>(&Ps[i][kc_t]) = ws_;
    }
  };
  if (kc_first < kj) load(kc_first);
  for (int64_t kc = kc_first; kc < kj; kc += KW) {
    stage(kc);
    __syncthreads();
    if (kc + KW < kj) load(kc + KW);              // in flight during the products below
    if (!idle) {
#pragma unroll 1
      for (int k = 0; k < KW; k += 4) {
        S fa[4], fb[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[i] = Pr[wr + 16 * i + li][k + lk];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) fb[jj] = Ps[wc + 16 * jj + li][k + lk];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) acc[i][jj] = MT::mma(fa[i], fb[jj], acc[i][jj]);
      }
    }
    __syncthreads();
  }
  if (idle) return;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t r = r0 + wr + 16 * i + MT::row(q, lk);
      if (r >= wend) continue;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int64_t s = s0 + wc + 16 * jj + li;
        if (s <= r) {
          T* e = base + r * ld + (s - r + B);
          *e = (T)((S)*e - acc[i][jj][q]);
        }
      }
    }
}

// One tile per work-group: work-group b runs on XCD x = b mod 8 and takes the (b / 8)-th
// tile of that XCD's consecutive share.
template <class T>
__global__ void __launch_bounds__(U2, 4) k_syrk_wide(BandArgs a, T* v, int64_t k0, int64_t kk,
                                                  int64_t ts_lo, int64_t ts_hi,
                                                  int64_t per_mat, int64_t total) {
  const int64_t x = blockIdx.x & 7, q = total >> 3, rem = total & 7;
  wide_tile<T>(a, v, k0, kk, ts_lo, ts_hi, per_mat, x * q + min(x, rem) + (blockIdx.x >> 3));
}

// Number of tiles k_syrk_wide enumerates per matrix for 128-column tile columns [lo, hi).
static int64_t wide_tiles(int64_t max_B, int64_t lo, int64_t hi) {
  const int64_t nt = (max_B + T2 - 1) / T2;
  int64_t c = 0;
  for (int64_t ts = lo; ts < std::min(hi, nt); ++ts) c += nt - ts;
  return c;
}


// The separators between the phases: what the lower part's elimination left in its
// separator window is added to the upper part's window, entry (s, t) of the separator there
// and (ns - 1 - t, ns - 1 - s) in the reversed part.  One 32 x 32 tile per work-group,
// turned in LDS so that both sides run along rows; the window is read and written once.
constexpr int MG = 32;
template <class T>
__global__ void __launch_bounds__(256) k_merge(const BandPart* part, const int32_t* part_of,
                                               T* v) {
  __shared__ T tile[MG][MG + 1];
  const int j = blockIdx.z;
  if (part_of[2 * j + 1] < 0) return;
  const BandPart& u = part[part_of[2 * j]];
  const BandPart& l = part[part_of[2 * j + 1]];
  const int64_t ns = u.rows - u.sep;
  const int64_t s0 = (int64_t)blockIdx.y * MG, t0 = (int64_t)blockIdx.x * MG;
  if (s0 >= ns || t0 > s0 || s0 - (t0 + MG - 1) > u.B) return;
  const int x = threadIdx.x % MG, y = threadIdx.x / MG;
  for (int q = y; q < MG; q += 256 / MG) {          // lower part's row of t0 + q, s along it
    const int64_t s = s0 + x, t = t0 + q;
    if (s < ns && t <= s && s - t <= u.B)
      tile[q][x] = v[l.off + (l.cols + ns - 1 - t) * l.ld + (t - s + l.B)];
  }
  __syncthreads();
  for (int q = y; q < MG; q += 256 / MG) {
    const int64_t s = s0 + q, t = t0 + x;
    if (s < ns && t <= s && s - t <= u.B)
      v[u.off + (u.sep + s) * u.ld + (t - s + u.B)] += tile[x][q];
  }
}

template <class T>
void band_factor_t(BandSet& bs, T* v, T* dinv, hipStream_t st, FactorJob& job, bool threaded) {
  static_assert(GP * NB % T2 == 0, "a group spans whole wide tile columns");
  constexpr int64_t NEXT_TS = GP * NB / T2;              // tile columns of the next group
  for (const BandPart& p : bs.part)
    GX_REQUIRE((p.rows + T2) * p.ld + 64 < ((int64_t)1 << 31),
               "a band matrix of 2^31 entries or more exceeds the update's 32-bit offsets");
  const int NR = (int)((bs.max_B + NB - 1) / NB) + 1;   // row blocks of a panel
  const int NF = NR - 1;                          // row blocks below a group: k_far's
  const int n_part = bs.n_part, n_mat = bs.n_mat;
  job.inv.alloc((size_t)n_part * GP * NB * NB);
  // columns of the longest part in each phase, and the largest separator
  int64_t span[2] = {0, 0}, max_sep = 0;
  for (const BandPart& p : bs.part) {
    for (int h = 0; h < 2; ++h) span[h] = std::max(span[h], p.fe[h] - p.fb[h]);
    max_sep = std::max(max_sep, p.rows - p.sep);
  }
  int64_t n_groups = 0;
  for (int h = 0; h < 2; ++h) n_groups += (span[h] + GP * NB - 1) / (GP * NB);
  job.flags.alloc((size_t)n_part * GP * GP + n_groups);   // then one ticket counter per launch
  clear(job.flags, st);
  int* tickets = job.flags.p + (int64_t)n_part * GP * GP;
  const int64_t nt2 = (bs.max_B + T2 - 1) / T2;
  const int64_t per_rest = wide_tiles(bs.max_B, NEXT_TS, nt2), tot_rest = per_rest * n_part;
  const int64_t per_next = wide_tiles(bs.max_B, 0, NEXT_TS), tot_next = per_next * n_part;
  const unsigned chain_blocks = (unsigned)((int64_t)GP * n_part);
  const unsigned far_blocks = (unsigned)((int64_t)n_part * NF);
  // group g on st: the update of its columns by group g - 1 (after the update of the same
  // columns by group g - 2, which ran on the second stream), then its k_chain and k_far;
  // then the update of the columns from group g + 2 on by its panels on the second stream,
  // at the same time as group g + 1's work on st.  Where a separator follows, the last
  // group's updates of it complete the first phase.
  GX_HIP(hipEventCreateWithFlags(&job.chain, hipEventDisableTiming));
  GX_HIP(hipEventCreateWithFlags(&job.rest[0], hipEventDisableTiming));
  GX_HIP(hipEventCreateWithFlags(&job.rest[1], hipEventDisableTiming));
  const int64_t max_B = bs.max_B, span0 = span[0], span1 = span[1];
  const bool split = bs.split;
  const BandPart* part = bs.d_part.p;
  const int32_t* part_of = bs.d_part_of.p;
  const int64_t *fcb = bs.d_fcb.p, *lrb = bs.d_lrb.p;
  int* flags = job.flags.p;
  double* inv = job.inv.p;
  int* err = job.err.p;
  hipStream_t la = job.la;
  hipEvent_t ev_chain = job.chain, ev_rest[2] = {job.rest[0], job.rest[1]};
  auto launches = [=]() {
    int g = 0;                                      // groups launched in both phases
    for (int phase = 0; phase < (split ? 2 : 1); ++phase) {
      const BandArgs a{part, fcb, lrb, phase};
      const int64_t cols = phase ? span1 : span0;
      const bool tail = split && phase == 0;        // rows remain after the last group
      bool recorded[2] = {false, false};
      int64_t k0 = 0;
      for (;; k0 += GP * NB, ++g) {
        const bool last = k0 >= cols;
        if (last && !tail) break;
        if (recorded[g % 2]) GX_HIP(hipStreamWaitEvent(st, ev_rest[g % 2], 0));
        if (k0 > 0 && max_B > 0)
          hipLaunchKernelGGL(k_syrk_wide<T>, dim3((unsigned)tot_next), dim3(U2), 0, st, a, v,
                             k0 - GP * NB, (int64_t)GP * NB, (int64_t)0, NEXT_TS, per_next,
                             tot_next);
        if (last) break;
        hipLaunchKernelGGL(k_chain<T>, dim3(chain_blocks), dim3(CT), 0, st, a, v, k0,
                           n_part, flags, tickets + g, g + 1, inv, dinv, err);
        if (far_blocks)
          hipLaunchKernelGGL(k_far<T>, dim3(far_blocks), dim3(CT), 0, st, a, v, k0, NF, n_part,
                             (const double*)inv);
        if (tot_rest && (tail || k0 + GP * NB < cols)) {
          GX_HIP(hipEventRecord(ev_chain, st));
          GX_HIP(hipStreamWaitEvent(la, ev_chain, 0));
          hipLaunchKernelGGL(k_syrk_wide<T>, dim3((unsigned)tot_rest), dim3(U2), 0, la, a, v,
                             k0, (int64_t)GP * NB, NEXT_TS, nt2, per_rest, tot_rest);
          GX_HIP(hipEventRecord(ev_rest[g % 2], la));
          recorded[g % 2] = true;
        }
      }
      for (int q = 0; q < 2; ++q)
        if (recorded[q]) GX_HIP(hipStreamWaitEvent(st, ev_rest[q], 0));
      if (tail) {
        const unsigned nt = (unsigned)((max_sep + MG - 1) / MG);
        hipLaunchKernelGGL(k_merge<T>, dim3(nt, nt, n_mat), dim3(256), 0, st, part, part_of, v);
      }
    }
    GX_HIP(hipGetLastError());
  };
  if (!threaded) {
    launches();
    return;
  }
  // The launches only enqueue work (no host wait, no allocation), so a thread of the job
  // may make them while the caller goes on; band_factor_finish and the job's destructor
  // join it, and an error it met is raised by band_factor_finish.
  int dev = 0;
  GX_HIP(hipGetDevice(&dev));
  job.launcher = std::thread([launches, dev, &job]() {
    try {
      GX_HIP(hipSetDevice(dev));
      launches();
    } catch (...) {
      job.launch_error = std::current_exception();
    }
  });
}

FactorJob::~FactorJob() {
  if (launcher.joinable()) launcher.join();
  if (st) (void)hipStreamSynchronize(st);         // nothing of the job may still run when
  if (la) (void)hipStreamSynchronize(la);         // its buffers are released
  if (chain) (void)hipEventDestroy(chain);
  for (hipEvent_t e : rest)
    if (e) (void)hipEventDestroy(e);
}

void band_factor_start(BandSet& bs, hipStream_t st, hipStream_t la, FactorJob& job,
                       const char* what, bool threaded) {
  GX_REQUIRE(!job.st, "factorisation job already started");
  job.st = st;
  job.la = la;
  job.what = what;
  job.err.alloc(1);
  clear(job.err, st);
  if (bs.fp32)
    band_factor_t<float>(bs, bs.v32.p, bs.dinv32.p, st, job, threaded);
  else
    band_factor_t<double>(bs, bs.v64.p, bs.dinv64.p, st, job, threaded);
}

void band_factor_finish(FactorJob& job) {
  GX_REQUIRE(job.st, "factorisation job not started");
  if (job.launcher.joinable()) job.launcher.join();
  if (job.launch_error) std::rethrow_exception(job.launch_error);
  int h = 0;
  to_host(&h, job.err.p, 1, job.st);               // waits for all of the job
  if (h & 2)
    throw Error(GX_EHIP, "banded Cholesky factorisation of " + job.what +
                             ": a work-group timed out waiting for a panel block");
  if (h)
    throw Error(GX_ENOTSPD,
                "non-positive pivot in the banded Cholesky factorisation of " + job.what);
}

// The links of every block: D_b L(b, b - 1) and D_b^T L(b + 1, b)^T, 64 x 64 products on the
// FP64 matrix instruction.  A solve's step from block to block then takes one product on the
// path from one hand-over to the next: D_b (rhs - older blocks) is formed while the
// neighbour's solution is awaited, and only its link follows (in place of the neighbour's
// own block, so the solve reads no more).  Work-group (block, part); each wave forms two of
// the 16 tiles of either product, its operands straight from LDS.
template <class T>
__global__ void __launch_bounds__(512) k_link(const BandPart* part, const T* v, const T* dinv,
                                              double* link) {
  __shared__ double D[SB][SB + 1], L[2][SB][SB + 1];
  const BandPart& P = part[blockIdx.y];
  const int64_t n = P.rows, ncb = (P.cols + SB - 1) / SB, b = blockIdx.x;
  if (b >= ncb) return;
  const int64_t i0 = b * SB, rs = P.ld - 1;
  const T* cb = v + P.off + P.B;
  const T* d = dinv + P.boff + b * SB * SB;
  for (int e = threadIdx.x; e < SB * SB; e += 512) {
    const int i = e / SB, c = e % SB;
    D[i][c] = (double)d[e];
    const int64_t r0 = i0 + i, c0 = i0 - SB + c, r1 = i0 + SB + i, c1 = i0 + c;
    L[0][i][c] = b > 0 && r0 < n && r0 - c0 <= P.B ? (double)cb[r0 * rs + c0] : 0.0;
    L[1][i][c] = r1 < n && c1 < n && r1 - c1 <= P.B ? (double)cb[r1 * rs + c1] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  double* out = link + 2 * P.boff + 2 * b * SB * SB;
  for (int q = 0; q < 4; ++q) {
    const int which = q >> 1, tile = w + 8 * (q & 1), rt = tile >> 2, ct = tile & 3;
    v4d acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < SB; k += 4) {
      const double fa = which ? D[k + lk][16 * rt + li] : D[16 * rt + li][k + lk];
      const double fb = which ? L[1][16 * ct + li][k + lk] : L[0][k + lk][16 * ct + li];
      acc = Mfma<double>::mma(fa, fb, acc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      out[(int64_t)which * SB * SB + (16 * rt + 4 * e + lk) * SB + 16 * ct + li] = acc[e];
  }
}

void band_factor(gx_ctx* c, BandSet& bs, hipStream_t st, const char* what) {
  FactorJob job;
  band_factor_start(bs, st, aux_stream(c->look[0]), job, what);
  band_factor_finish(job);
}

// ---------------------------------------------------------------------------------------
// Solves: forward L y = b, then backward L^T x = y, in place on FP64 right-hand sides.
// A matrix is swept in blocks of 64 rows.  The coupling between consecutive blocks runs
// through the explicit inverse of each 64x64 diagonal block (kept by the factorisation),
// so the serial part of a block is one small product, not a 64-step substitution.
//
// G work-groups share a part: block k belongs to work-group k mod G in the forward sweep and
// likewise from the end in the backward sweep.  A work-group first adds the contributions of
// the blocks that are complete by construction (its own previous block and everything
// before it), then takes the at most G - 1 blocks still in flight from the other
// work-groups (bounded polls of their solutions, below), applies the inverse diagonal block
// and hands its block on.  A timed-out poll raises the launch's error word and proceeds, so
// every wave always reaches the end of the kernel.
//
// What bounds the one-right-hand-side solve: a work-group streams about 22 GB/s however idle
// the device is, so few matrices need many groups; then the chain of (n + B) / 128 hand-overs
// per sweep, which the links (k_link) and lane sums in registers shorten.  Per solve, one
// chain per matrix and four groups -> now (FP64 but where noted): 4 matrices of n = 3,500, B =
// 370: 0.29 -> 0.13 ms; 6 of 16,000, 1,020: 1.77 -> 0.60 ms; 16 of 37,000, 1,220 (9.5 GB): 4.85
// -> 2.05 ms; 5 of 45,000, 2,080, FP32: 6.12 -> 1.40 ms; 16 of 91,000, 1,630 (26 GB): 15.1 ->
// 5.80 ms.  64 of those fill the device with one group per compute unit; they are kept whole
// (split_pays) and stay where they were: 118 GB in 21.9 ms, FP32 59 GB in 12.4 ms.
constexpr int SW = SOLVE_THREADS / 64;           // waves per work-group (8)
constexpr int CL = 32;                            // words from one place counter to the next
                                                  // (and to the error word): a line of its
                                                  // own for each XCD
constexpr int RPW = SB / SW;                      // forward rows per wave (8)
constexpr int GMAX = 16;                          // work-groups per part, 1-RHS solve
constexpr int FL = 3;                             // blocks in flight taken at a time
constexpr int DL = SB * SB / SOLVE_THREADS;       // inverse-block entries per thread (8)
static_assert(DL == RPW, "the inverse-block products reuse the 8-row lane reduction");
constexpr int64_t BAND_PAD = 1024;               // trailing entries of a band allocation

// zero entries after the last matrix: the solves read up to BAND_PAD past its end, the
// trailing update up to T2 rows
static int64_t band_pad(int64_t max_B) { return BAND_PAD + T2 * (max_B + 1); }

// Band entry (r, c) loaded from a clamped, always valid address; the caller masks entries
// outside the band.  The loads are unconditional so that a wave issues all of them before
// it waits for any.
template <class T>
__device__ inline T band_raw(const T* base, int64_t n, int64_t B, int64_t ld, int64_t r,
                             int64_t c) {
  const int64_t rc = min(r, n - 1);
  const int64_t o = min(max(c - rc + B, (int64_t)0), B);
  return base[rc * ld + o];
}

// The 32-bit halves of a double through a lane operation
template <class F>
__device__ inline double by_halves(double v, F f) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  return __longlong_as_double(
      (long long)((uint64_t)f((uint32_t)(u >> 32)) << 32 | f((uint32_t)u)));
}
// lane i's value of a DPP move within its row of 16 lanes (CTRL 0x100 + k: from lane i + k,
// 0x120 + 8: from lane i xor 8)
template <int CTRL>
__device__ inline double row_move(double v) {
  return by_halves(v, [](uint32_t w) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, CTRL, 0xf, 0xf, true);
  });
}
// a + b after the odd 32-lane halves (16-lane rows) of a and the even ones of b have changed
// places: a summed over the pairs of halves (rows) in the even ones, b in the odd ones
template <int LANES>
__device__ inline double swap_add(double a, double b) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
  auto swap = [](uint32_t x, uint32_t y) {
    if constexpr (LANES == 32) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
    else return __builtin_amdgcn_permlane16_swap(x, y, false, false);
  };
  const auto lo = swap((uint32_t)ua, (uint32_t)ub), hi = swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32));
  return __longlong_as_double((long long)((uint64_t)hi[0] << 32 | lo[0])) +
         __longlong_as_double((long long)((uint64_t)hi[1] << 32 | lo[1]));
}

// s[r] summed over the 64 lanes; lane l (a multiple of 8) receives the total of row l >> 3.
// In registers throughout (lane swaps and DPP moves, no LDS): the sum is on the path from one
// hand-over to the next.
__device__ inline double reduce_rows8(const double (&s)[RPW], int lane) {
  double t4[4], t2[2];
#pragma unroll
  for (int r = 0; r < 4; ++r) t4[r] = swap_add<32>(s[r], s[r + 4]);
#pragma unroll
  for (int r = 0; r < 2; ++r) t2[r] = swap_add<16>(t4[r], t4[r + 2]);
  const bool b3 = lane & 8;
  double t = (b3 ? t2[1] : t2[0]) + row_move<0x128>(b3 ? t2[0] : t2[1]);
  t += row_move<0x104>(t);
  t += row_move<0x102>(t);
  t += row_move<0x101>(t);
  return t;
}

// ---- one right-hand side per matrix
// Loads are unconditional: rows past the end of the matrix are clamped to its last row, a
// lane whose column lies outside the band reads a neighbouring entry (the band storage
// carries BAND_PAD zero entries after the last row), and masks are applied by multiplying
// with 0 or 1, so that a wave issues all loads of a step before it waits for any.
//
// Hand-over between the work-groups of a matrix goes through the data itself, not flags:
// the forward sweep writes block k's solution into the scratch vector y and the backward
// sweep its final solution into the scratch vector z, both filled with the marker YMARK
// before the launch; a reader of a block that may still be in flight polls its entries
// until none is YMARK, and the values it polled are the ones it uses.  z is copied into x
// after the launch.  Every access to y and z is an agent-scope relaxed atomic (8 bytes,
// single-copy atomic, past the non-coherent caches), so no fence is needed anywhere: a
// hand-over costs the reader one memory round trip and the writer none.  A marker is a NaN
// payload that arithmetic never produces (a NaN result carries the default payload), so a
// diverged solve still propagates NaN.
// COARSE only names the instance used for the coarse matrix apart in profiles.
constexpr uint64_t YMARK = 0x7FF4D1E5E7C0DE00ull;

__device__ inline bool is_mark(double v) { return __double_as_longlong(v) == (long long)YMARK; }

__device__ inline double poll_load(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void hand_over(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the same in FP32 (the hand-over scratch of the FP32 many-right-hand-side solve): the
// marker is a signalling-NaN payload, which arithmetic never produces either
constexpr uint32_t YMARK32 = 0x7FA5C0DEu;
__device__ inline bool is_mark(float v) { return __float_as_uint(v) == YMARK32; }
__device__ inline float poll_load(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void hand_over(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Spin-limit bookkeeping of a polling loop: true when the wait must give up (time-out, or
// another wait of the launch already timed out).
__device__ inline bool poll_give_up(int64_t& spins, int* err) {
  if ((++spins & 255) == 0 &&
      (spins > SPIN_LIMIT || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
    atomicOr(err, 2);
    return true;
  }
  __builtin_amdgcn_s_sleep(1);
  return false;
}

// One part in the single-right-hand-side solve: factor entries from base, inverse diagonal
// blocks from dv, envelope tables fcb / lrb (by 64-row blocks), the matrix's right-hand side
// x, scratch y, z, and the mate's (BandPtrs) scratch.
template <class T>
struct Solve1 {
  int64_t n, cols, sep, N, B, ld;
  int kind;
  const T* base;
  const T* dv;
  const double* link;
  const int64_t* fcb;
  const int64_t* lrb;
  const double* x;
  double* y;
  double* z;
  const double* mate;
};

// Work-group g of the P that solve part `own` (load(i): the Solve1 of part i; `upper`: the
// upper part of a split matrix).  P is the G of the plan unless groups came too late (gather);
// which blocks of a sum count as complete and which as in flight follows G, whoever is there,
// so the order of summation, and with it every bit of the result, is the plan's.  A split matrix is swept in two segments: the parts' own
// columns, each by its work-groups, and the separator, held by the upper part, by the
// work-groups of both (as many as the in-flight registers allow), so that none is idle
// meanwhile.  The lower part's rows past its own columns (the separator) only sum its
// contributions to them, which the separator's blocks take from its y; its backward sweep
// takes the separator's solution from the upper part's z.  A segment begins with a wait
// for the one before it, which the count of complete blocks rests on.
template <class T, class Load>
__device__ __forceinline__ void band_solve_1_mat(Load load, int own, int upper, int g, int G,
                                                 int P, int* err) {
  int n, cols, sep, B, rs, N;                       // (a part has less than 2^31 entries)
  const T *base, *dv;
  const double* link;
  const int64_t *fcb, *lrb;
  const double *x, *mate;                           // row r at x[dx r], mate[-r]
  double *y, *z;
  int dx;
  bool lower;
  auto use = [&](int part) {
    const Solve1<T> S = load(part);
    n = (int)S.n, cols = (int)S.cols, sep = (int)S.sep, B = (int)S.B, rs = (int)S.ld - 1;
    N = (int)S.N;
    base = S.base, dv = S.dv, link = S.link, fcb = S.fcb, lrb = S.lrb;
    lower = S.kind == PART_LOWER;
    x = lower ? S.x + N - 1 : S.x;
    dx = lower ? -1 : 1;
    y = S.y, z = S.z;
    mate = S.mate + N - 1;
  };
  use(own);
  const bool split = upper >= 0, own_lower = lower;
  // separator groups
  const bool both = 2 * G <= GMAX;
  const int GS = both ? 2 * G : G, PS = both ? 2 * P : P;
  const int gs = both ? 2 * g + own_lower : own_lower ? -1 : g;
  __shared__ double acc[SB];
  __shared__ double part[SW][SB];
  __shared__ double xs[FL][SB];               // polled solutions of blocks in flight
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int UB = 32;                           // band rows in flight per wave (backward)
  // ---- forward: wave w owns rows 8w..8w+7 of the block, lanes run along the columns
#pragma unroll 1
  for (int seg = 0; seg < (split ? 2 : 1); ++seg) {
  int kfirst = 0, span = G, step = P, mine = g;   // first block of the segment, of this group
  if (seg) {
    if (gs < 0) break;
    use(upper);
    kfirst = sep / SB;
    span = GS;
    step = PS;
    mine = kfirst + gs;
    if (threadIdx.x < SB) {
      int64_t spins = 0;
      while (is_mark(poll_load(y + sep - SB + threadIdx.x)) && !poll_give_up(spins, err)) {}
    }
    __syncthreads();
  }
  const int ncb = (cols + SB - 1) / SB;         // blocks with columns of their own
  const int nblk = seg || !split || lower ? (n + SB - 1) / SB : sep / SB;
  for (int k = mine; k < nblk; k += step) {
    const int i0 = k * SB;
    const int nb = (int)min<int>(SB, n - i0);
    const int kc = min(k, ncb);                // column blocks left of the block
    const int kdone = min(max(k - span + 1, kfirst), kc);   // those < kdone are complete
    const int done_end = kdone * SB;
    const int ifirst = i0 + RPW * wave;
    // the right-hand side of the row this lane reduces
    const int ii = RPW * wave + (lane >> 3);
    const bool own = (lane & 7) == 0 && ii < nb;
    double bval = own && k < ncb ? x[dx * (i0 + ii)] : 0.0;
    const T* rp[RPW];                              // rp[r][c] = entry (row, c); scalar, the
                                                   // lanes' offsets from it are 32-bit
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int rc = min<int>(ifirst + r, n - 1);
      rp[r] = base + ((int64_t)rc * rs + B);
    }
    double s[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) s[r] = 0.0;
    // envelope start, rounded down to a 128-byte line (rows start on one: see band_layout)
    constexpr int LA = 128 / (int)sizeof(T);
    const int cstart = max(max<int>(ifirst - B, 0), (int)fcb[k]) / LA * LA;
    {
      // a lane loads V adjacent columns of a row at once (16 bytes: two FP64 or four FP32
      // entries; columns from a line start are multiples of V, so every load is aligned),
      // 64 V columns per step, 512 columns per pass
      constexpr int V = 16 / (int)sizeof(T);
      constexpr int US = 512 / (64 * V);            // steps per pass
      typedef T TV __attribute__((ext_vector_type(V)));
      const int done = (int)(done_end - cstart);    // columns counted from cstart
      const int lo = (int)(ifirst - B - cstart);    // row r's band starts at lo + r
      const double* yc = y + cstart;
      for (int c0 = V * lane; c0 < done + V * lane; c0 += 64 * V * US) {
        TV l[US][RPW];
        double xv[US][V];
#pragma unroll
        for (int u = 0; u < US; ++u) {
          const uint32_t cc = c0 + 64 * V * u;
#pragma unroll
          for (int e = 0; e < V; ++e) xv[u][e] = poll_load(yc + min<uint32_t>(cc + e, (uint32_t)done - 1));
#pragma unroll
          for (int r = 0; r < RPW; ++r)
            l[u][r] = *reinterpret_cast<const TV*>(rp[r] + cstart + cc);
        }
#pragma unroll
        for (int u = 0; u < US; ++u) {
          const int cc = c0 + 64 * V * u;
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const double xe = cc + e < done ? xv[u][e] : 0.0;
#pragma unroll
            for (int r = 0; r < RPW; ++r)
              s[r] += (double)l[u][r][e] * (cc + e >= lo + r ? xe : 0.0);
          }
        }
      }
    }
    // blocks in flight, kdone .. kc - 1 (at most span - 1), the nearest of them left to the
    // link below; up to FL at a time, the last ones together: their factor entries (and,
    // before the last, this block's inverse diagonal block and link) are loaded first; then
    // wave 0 polls their solutions (one round trip when they are done) and passes them on
    // through LDS
    const bool linked = link && k < ncb && kdone < k;
    const int kin = linked ? kc - 1 : kc;
    T dd[DL];
    double lm[DL];
    int kf = kdone;
#pragma unroll 1
    for (;;) {
      const int rest = kin - kf;
      const int nfl = (int)(rest > FL ? (rest - 1) % FL + 1 : rest);
      T pf[FL][RPW];
#pragma unroll
      for (int o = 0; o < FL; ++o) {
        const int cc = min<int>(kf + o, max<int>(kc - 1, 0)) * SB;
#pragma unroll
        for (int r = 0; r < RPW; ++r) pf[o][r] = (rp[r] + cc)[(uint32_t)lane];
      }
      if (rest <= FL) {
        const int64_t kd = min(k, ncb - 1);
#pragma unroll
        for (int u = 0; u < DL; ++u) {
          dd[u] = (dv + kd * SB * SB)[threadIdx.x + SOLVE_THREADS * u];
          if (linked) lm[u] = (link + 2 * kd * SB * SB)[threadIdx.x + SOLVE_THREADS * u];
        }
      }
      if (nfl > 0) {
        if (wave == 0) {
          double xo[FL];
          int64_t spins = 0;
          for (;;) {
            bool ok = true;
#pragma unroll
            for (int o = 0; o < FL; ++o) {
              xo[o] = poll_load((y + min(kf + o, kf + nfl - 1) * SB) + (uint32_t)lane);
              ok = ok && !is_mark(xo[o]);
            }
            if (__all(ok) || poll_give_up(spins, err)) break;
          }
#pragma unroll
          for (int o = 0; o < FL; ++o) xs[o][lane] = xo[o];
        }
        __syncthreads();
        double xo[FL];
#pragma unroll
        for (int o = 0; o < FL; ++o) xo[o] = xs[o][lane];
#pragma unroll
        for (int o = 0; o < FL; ++o) {
          if (o >= nfl) break;
          const int cc = (kf + o) * SB + lane;
#pragma unroll
          for (int r = 0; r < RPW; ++r)
            s[r] += (double)pf[o][r] * (cc >= ifirst + r - B ? xo[o] : 0.0);
        }
      }
      if (rest <= FL) break;
      kf += nfl;
      __syncthreads();                             // xs is taken again
    }
    const double tot = reduce_rows8(s, lane);
    if (k >= ncb) {                                // separator rows of a lower part
      if (own) hand_over(y + i0 + ii, tot);
      __syncthreads();
      continue;
    }
    if (i0 >= sep && own) {                       // the lower part's share of these rows
      int64_t spins = 0;
      double t = poll_load(mate - (i0 + ii));
      while (is_mark(t) && !poll_give_up(spins, err)) t = poll_load(mate - (i0 + ii));
      bval -= t;
    }
    if ((lane & 7) == 0) acc[ii] = own ? bval - tot : 0.0;
    __syncthreads();
    // y = Di acc: thread (wave, lane) holds Di[wave + 8 u][lane] (u < 8) from the prefetch,
    // so each wave forms rows wave + 8 u with one lane-wide reduction
    {
      const double av = acc[lane];
      double pr[RPW];
#pragma unroll
      for (int u = 0; u < DL; ++u) pr[u] = (double)dd[u] * av;
      double yr = reduce_rows8(pr, lane);
      if (linked) {                                // - D L(k, k - 1) y(k - 1): every wave polls
        const double* yp = y + i0 - SB;            // for itself, no barrier on this path
        int64_t spins = 0;
        double yv;
        for (;;) {
          yv = poll_load(yp + (uint32_t)lane);
          if (!__any(is_mark(yv)) || poll_give_up(spins, err)) break;
        }
#pragma unroll
        for (int u = 0; u < DL; ++u) pr[u] = lm[u] * yv;
        yr -= reduce_rows8(pr, lane);
      }
      const int row = wave + SW * (lane >> 3);
      if ((lane & 7) == 0 && row < nb) hand_over(y + i0 + row, yr);
    }
    __syncthreads();
  }
  }
  // ---- backward: lanes own the block's 64 columns, waves split the band rows below it;
  // entry (r, c) = cb[r * rs + c]
#pragma unroll 1
  for (int seg = split ? 1 : 0; seg >= 0; --seg) {
  if (seg && gs < 0) continue;
  if (!seg && split) {                             // the separator's solution
    use(own);
    const int r0 = lower ? cols : sep;
    for (int r = r0 + threadIdx.x; r < n; r += SOLVE_THREADS) {
      int64_t spins = 0;
      while (is_mark(poll_load(lower ? mate - r : z + r)) && !poll_give_up(spins, err)) {}
    }
    __syncthreads();
  }
  // blocks of the segment: all from kbeg to kend
  const int kbeg = seg ? sep / SB : 0;
  const int kend = seg || !split || lower ? (cols + SB - 1) / SB : sep / SB;
  const int span = seg ? GS : G, step = seg ? PS : P;
  const T* cb = base + B;
  for (int kb = kend - 1 - (seg ? gs : g); kb >= kbeg; kb -= step) {
    const int i0 = kb * SB;
    const int nb = (int)min<int>(SB, cols - i0);
    const int rend = min(min<int>(n, i0 + nb + B), (int)lrb[kb]);   // envelope end
    const int kdone = min(kb + span, kend);    // row blocks >= kdone complete
    const int done_beg = min<int>(rend, kdone * SB);
    const int cidx = i0 + lane;
    double sacc = 0.0;
    {
      // lane l loads the V adjacent columns from V (l mod 64 / V) of the rows
      // r0 + 8 (V v + l / (64 / V)) (16 bytes, aligned as above), so one load covers V
      // rows; the row groups' sums are then added and handed to the lanes of their columns
      constexpr int V = 16 / (int)sizeof(T);
      constexpr int LPR = 64 / V;                   // lanes per row
      typedef T TV __attribute__((ext_vector_type(V)));
      const int pr = lane % LPR, hf = lane / LPR;
      double sv[V];
#pragma unroll
      for (int e = 0; e < V; ++e) sv[e] = 0.0;
      const uint32_t rs32 = (uint32_t)rs, cv = V * pr;
      const int lo = (int)(B + i0) + V * pr;         // row r reaches the columns from r - lo on
      for (int r0 = done_beg + wave; r0 < rend; r0 += SW * UB) {
        TV l[UB / V];
        const int left = (int)(rend - 1 - r0);       // rows below r0 inside the envelope
        const int rz = r0 + min<int>(SW * (lane % UB), left);
        const double xz = poll_load(rz < cols ? z + rz : mate - rz);
        const T* cr = cb + r0 * rs + i0;             // (scalar; the lanes' offsets are 32-bit)
#pragma unroll
        for (int v = 0; v < UB / V; ++v)
          l[v] = *reinterpret_cast<const TV*>(
              cr + ((uint32_t)min<int>(SW * (V * v + hf), left) * rs32 + cv));
#pragma unroll
        for (int v = 0; v < UB / V; ++v) {
          const int rr = SW * (V * v + hf);
          const double xu = __shfl(xz, V * v + hf);
#pragma unroll
          for (int e = 0; e < V; ++e)
            sv[e] += (double)l[v][e] * ((rr <= left && (int)r0 + rr <= lo + e) ? xu : 0.0);
        }
      }
#pragma unroll
      for (int m = LPR; m < 64; m *= 2)
#pragma unroll
        for (int e = 0; e < V; ++e) sv[e] += __shfl_xor(sv[e], m);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const double t = __shfl(sv[e], lane / V);
        if (lane % V == e) sacc = t;
      }
    }
    // row blocks in flight, kb + 1 .. kin (at most span - 1), the nearest of them left to
    // the link below; up to FL at a time from the far end, the nearest together: factor
    // entries and, before the last, the inverse diagonal block first, then the polls of their
    // final solutions (rows inside the band only), the last together with this block's
    // forward solution
    const int kin = min<int>(kdone - 1, (rend - 1) / SB);   // last row block in flight
    const bool linked = link && kb + 1 < kdone && rend > (kb + 1) * SB;
    const int kn = linked ? kb + 1 : kb;
    T dd[DL];
    double lm[DL];
    double yown = 0.0;
    int kl = max(kin, kn);                         // the farthest one not yet taken
#pragma unroll 1
    for (;;) {
      const int rest = kl - kn;
      const int nfl = (int)(rest > FL ? (rest - 1) % FL + 1 : rest);
      const int kf = kl - nfl + 1;             // blocks kf .. kl
      const bool lastc = rest <= FL;
      T pf[FL][RPW];
#pragma unroll
      for (int o = 0; o < FL; ++o)
#pragma unroll
        for (int r = 0; r < RPW; ++r)
          pf[o][r] = cb[min<int>((kf + o) * SB + wave + SW * r, n - 1) * rs + cidx];
      if (lastc)
#pragma unroll
        for (int u = 0; u < DL; ++u) {
          dd[u] = (dv + (int64_t)kb * SB * SB)[threadIdx.x + SOLVE_THREADS * u];
          if (linked)
            lm[u] = (link + (2 * (int64_t)kb + 1) * SB * SB)[threadIdx.x + SOLVE_THREADS * u];
        }
      // wave 0 polls (lane l: row l of each block) and passes the values on through LDS
      if (wave == 0) {
        double xo[FL];
        int64_t spins = 0;
        for (;;) {
          bool ok = true;
          if (lastc && lane < nb) {
            yown = poll_load(y + cidx);
            ok = !is_mark(yown);
          }
#pragma unroll
          for (int o = 0; o < FL; ++o) {
            const int rr = (kf + o) * SB + lane;
            const bool need = o < nfl && rr < rend;
            xo[o] = poll_load(z + min<int>(rr, rend - 1));
            ok = ok && (!need || !is_mark(xo[o]));
          }
          if (__all(ok) || poll_give_up(spins, err)) break;
        }
#pragma unroll
        for (int o = 0; o < FL; ++o) xs[o][lane] = xo[o];
      }
      __syncthreads();
      double xr[FL][RPW];
#pragma unroll
      for (int o = 0; o < FL; ++o)
#pragma unroll
        for (int r = 0; r < RPW; ++r) xr[o][r] = xs[o][wave + SW * r];
#pragma unroll
      for (int o = 0; o < FL; ++o) {
        if (o >= nfl) break;
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
          const int rr = (kf + o) * SB + wave + SW * r;
          sacc += (double)pf[o][r] * ((rr < rend && rr - B <= cidx) ? xr[o][r] : 0.0);
        }
      }
      if (lastc) break;
      kl -= nfl;
      __syncthreads();                             // xs is taken again
    }
    part[wave][lane] = sacc;
    if (wave == 0) acc[lane] = lane < nb ? yown : 0.0;
    __syncthreads();
    // z = Di^T (yown - sums): thread (wave, lane) holds Di[wave + 8 u][lane]; each wave
    // forms its rows' right-hand sides (broadcast reads), then its share of every column
    {
      double pc = 0.0;
#pragma unroll
      for (int u = 0; u < DL; ++u) {
        const int r = wave + SW * u;
        double t = acc[r];
#pragma unroll
        for (int w = 0; w < SW; ++w) t -= part[w][r];
        pc += (double)dd[u] * (r < nb ? t : 0.0);
      }
      __syncthreads();
      part[wave][lane] = pc;
    }
    __syncthreads();
    if (!linked) {
      if (wave == 0) {
        double zs = 0.0;
#pragma unroll
        for (int w = 0; w < SW; ++w) zs += part[w][lane];
        if (lane < nb) hand_over(z + cidx, zs);
      }
    } else {                                       // - D^T L(kb + 1, kb)^T z(kb + 1), as above
      const int row = wave + SW * (lane >> 3);
      double zr = 0.0;
#pragma unroll
      for (int w = 0; w < SW; ++w) zr += part[w][row];
      const double* zp = z + i0 + SB;
      const bool in = i0 + SB + lane < n;
      int64_t spins = 0;
      double zv;
      for (;;) {
        zv = poll_load(zp + (uint32_t)lane);
        if (!__any(in && is_mark(zv)) || poll_give_up(spins, err)) break;
      }
      if (!in) zv = 0.0;
      double pr2[DL];
#pragma unroll
      for (int u = 0; u < DL; ++u) pr2[u] = lm[u] * zv;
      zr -= reduce_rows8(pr2, lane);
      if ((lane & 7) == 0 && row < nb) hand_over(z + i0 + row, zr);
    }
    __syncthreads();
  }
  }
}

// Work-groups of one class (blockIdx mod 8, hence of one XCD) take their places in a list of
// (matrix, group, part) in the order they start, from a counter that the marker fill resets.
// The two parts of a matrix wait for each other, and so do the groups of a part: a matrix's
// work-groups are neighbours in the list, so those running are a prefix of it, every
// complete matrix of the prefix finishes, and its slots go to the next ones.  Launches of
// several contexts could each hold a part of the slots and wait for the rest: see gather.
__device__ inline int take_place(int* counter) {
  __shared__ int q;
  if (threadIdx.x == 0) q = atomicAdd(counter, 1);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(q);
}

// A work-group-uniform table entry, into scalar registers (read after an atomic, the
// compiler would otherwise keep its fields, and all that follows from them, per lane).
template <class V>
__device__ inline V uniform_load(const V* p) {
  static_assert(sizeof(V) % 4 == 0, "whole words");
  V out;
  int w[sizeof(V) / 4];
#pragma unroll
  for (size_t i = 0; i < sizeof(V) / 4; ++i)
    w[i] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(p)[i]);
  __builtin_memcpy(&out, w, sizeof(V));
  return out;
}

// The groups of a matrix (G to each of its np parts) begin together.  Launches of other
// contexts may hold some of the slots and wait for theirs in the same way, so the wait is
// bounded: after GATHER (20 ms, a thousand times what a lone launch takes) those who are there
// share the matrix, and whoever comes later leaves; none but the time it takes depends on it.
// w: two words of the matrix, cleared by the marker fill: arrivals, which number the groups, and
// how many of them take part, `most` to a part.  Returns this work-group's number (-1: leave)
// and the groups per part, the same in every lane.
constexpr int64_t GATHER = 2000000;              // ticks of the 100 MHz clock
__device__ inline int2 gather(int* w, int np, int G, int most, int* err) {
  __shared__ int2 mine;
  if (threadIdx.x == 0) {
    int* e = w + 1;
    auto settle = [&](int n) {                   // once: the first to settle it counts
      int none = 0;
      __hip_atomic_compare_exchange_strong(e, &none, n, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    };
    int2 r = {atomicAdd(w, 1), G};
    if (r.x == np * G - 1) settle(np * min(G, most));
    const int64_t t0 = wall_clock64();
    int64_t spins = 0;
    int c;
    while (!(c = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
      if ((++spins & 255) == 0) {
        if (wall_clock64() - t0 > GATHER) {
          const int n = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (n >= np) settle(min(n, np * min(G, most)));
        }
        if (spins > SPIN_LIMIT) {
          atomicOr(err, 2);
          break;
        }
      }
      __builtin_amdgcn_s_sleep(1);
    }
    r.y = c / np;
    if (r.x >= r.y * np) r.x = -1;
    mine = r;
  }
  __syncthreads();
  return {__builtin_amdgcn_readfirstlane(mine.x), __builtin_amdgcn_readfirstlane(mine.y)};
}

// This work-group's part and group in a launch over one band set of n_mat matrices, up to G
// groups per part, both parts of a matrix (PP = 2 if the set has split matrices) in turn;
// part -1: none.  The words of the matrices' gathers follow the place counters.
struct Place {
  int part, g, P;                                // group g of the P that are there
};
__device__ inline Place set_place(const int32_t* part_of, int n_mat, int G, int PP, int most,
                                  int* err) {
  int* counters = err + CL;
  const int x = blockIdx.x & 7, q = take_place(counters + CL * x);
  const int j = q / (G * PP) * 8 + x, m = q % (G * PP);
  if (j >= n_mat) return {-1, 0, G};
  const int np = PP == 2 && uniform_load(part_of + 2 * j + 1) >= 0 ? 2 : 1;
  if (m % PP >= np) return {-1, 0, G};           // no second part
  if (G == 1) return {uniform_load(part_of + 2 * j + m % PP), 0, 1};
  const int2 k = gather(counters + CL * 8 + 2 * j, np, G, most, err);
  if (k.x < 0) return {-1, 0, k.y};
  return {uniform_load(part_of + 2 * j + k.x % np), k.x / np, k.y};
}

// The parts of one band set (set_place)
template <class T, bool COARSE>
__global__ void __launch_bounds__(SOLVE_THREADS) k_band_solve_1(
    BandArgs a, const int32_t* part_of, const T* v, const T* dinv, const double* link,
    const int64_t* xoff, const double* xall, double* yall, double* zall, int G, int PP, int n_mat,
    int most, int* err) {
  const Place pl = set_place(part_of, n_mat, G, PP, most, err);
  if (pl.part < 0) return;
  auto load = [&](int i) -> Solve1<T> {
    const BandPart P = uniform_load(a.part + i);
    const int mp = P.kind == PART_WHOLE ? i
                                        : uniform_load(part_of + 2 * P.mat + (P.kind == PART_UPPER));
    const int64_t mo = uniform_load(&a.part[mp].yoff);
    return {P.rows, P.cols, P.kind == PART_UPPER ? P.sep : P.rows, P.N, P.B, P.ld, P.kind,
            v + P.off, dinv + P.boff, link ? link + 2 * P.boff : nullptr,
            a.fcb + P.eoff, a.lrb + P.eoff,
            xall + uniform_load(xoff + P.mat), yall + P.yoff, zall + P.yoff,
            (P.kind == PART_LOWER ? zall : yall) + mo};
  };
  const BandPart P = uniform_load(a.part + pl.part);
  if (P.rows == 0) return;
  band_solve_1_mat<T>(load, pl.part,
                      P.kind == PART_WHOLE ? -1 : uniform_load(part_of + 2 * P.mat), pl.g, G,
                      pl.P, err);
}

// The parts of several band sets in one launch (all of one precision): the q-th work-group
// of class x to start takes group work[2 i + 1] of part work[2 i], i = q n_class + x (none
// if negative).  Where a part has more than one group the matrix's groups gather first, as in
// set_place: the table counts on all slots of the device, and the joint solves of another
// thread's batch may hold some of them.
template <class T>
__global__ void __launch_bounds__(SOLVE_THREADS) k_band_solve_1_multi(const BandPtrs* __restrict__ tab,
                                                                       const int32_t* __restrict__ work,
                                                                       int n_class, int most,
                                                                       int* err) {
  const int x = blockIdx.x % n_class;
  const int i = take_place(err + CL * (1 + x)) * n_class + x;
  int j = uniform_load(work + 2 * i), g = uniform_load(work + 2 * i + 1);
  if (j < 0) return;
  auto load = [&](int p) -> Solve1<T> {
    const BandPtrs t = uniform_load(tab + p);
    return {t.n, t.cols, t.sep, t.N, t.B, t.B + 1, (int)t.kind, static_cast<const T*>(t.v),
            static_cast<const T*>(t.dinv), t.link, t.fcb, t.lrb, t.x, t.y, t.z, t.mate};
  };
  const int64_t rows = uniform_load(&tab[j].n);
  const int kind = (int)uniform_load(&tab[j].kind);
  const int G = (int)uniform_load(&tab[j].G);
  int P = G;
  if (rows == 0) return;
  // (an upper part stands right before its lower part in the table)
  const int first = kind == PART_LOWER ? j - 1 : j;
  if (G > 1) {
    const int np = kind == PART_WHOLE ? 1 : 2;
    const int2 k = gather(err + CL * (1 + 8) + 2 * first, np, G, most, err);
    if (k.x < 0) return;
    j = first + k.x % np;
    g = k.x / np;
    P = k.y;
  }
  band_solve_1_mat<T>(load, j, kind == PART_WHOLE ? -1 : first, g, G, P, err);
}

// y and z scratch of every part of a multi-set solve back to the marker, its counters to 0
// (65,535 matrices may have twice as many parts as a grid has rows: a row takes several)
__global__ void k_fill_mark_multi(const BandPtrs* tab, int n_part, int* counters) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (blockIdx.y == 0 && i < 8) counters[CL * i] = 0;
  for (int q = blockIdx.y; q < n_part; q += gridDim.y) {
    const BandPtrs t = tab[q];
    if (i < 2) counters[CL * 8 + 2 * q + i] = 0;   // the part's words of gather
    if (i < (t.n + SB - 1) / SB * SB) {
      t.y[i] = __longlong_as_double((long long)YMARK);
      t.z[i] = __longlong_as_double((long long)YMARK);
    }
  }
}

// x <- z for every part of a multi-set solve
__global__ void k_copy_out_multi(const BandPtrs* tab, int n_part) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int q = blockIdx.y; q < n_part; q += gridDim.y) {
    const BandPtrs t = tab[q];
    if (i < t.cols) t.x[t.kind == PART_LOWER ? t.N - 1 - i : i] = t.z[i];
  }
}

// ---- M right-hand sides per matrix (M a multiple of 8, at most MC; row-major, row
// stride M)
// The block products - a 64-row block of the band against 64 solution rows, and the
// inverse diagonal block against the block's right-hand side - are 64 x 64 x M and run on
// FP64 matrix cores: v_mfma_f64_16x16x4, lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and holds D[4 r + l / 16][l % 16] in accumulator register r; wave w
// of the 8 owns row tile w mod 4 and column tile w / 4.  Chunks (64 x 64 of the band plus
// the matching solution rows) are staged through two LDS buffers in turn; the loads of the
// next two chunks are in flight in two register sets while the current one is multiplied
// (the chunk loop is unrolled by two so that each set and buffer has a name of its own).
// Hand-over between work-groups
// goes through marker-filled scratch solutions as in the single-right-hand-side solve
// (forward into y, backward into z, z copied into x afterwards), kept in the factor's
// precision (FP32 factors: FP32 scratch, half the bytes of the solution rows that every
// chunk reads): solution entries are loaded with agent-scope relaxed atomics, and a chunk
// is staged only once none of the entries it needs is a marker (a chunk still in flight
// is polled again until then).
// What bounds it: the latency of a chunk's stages (2.9 us with one work-group per compute
// unit; leaving out the solution rows, the band or the products takes about a quarter off
// each), and for narrow bands the hand-overs.  So what a block needs besides its chunks, its
// right-hand side and its inverse block, is loaded before the sweep and waits in registers
// and in LDS buffers of its own: per solve of 32 columns, 4 matrices of n = 3,500, B = 370
// 0.51 -> 0.46 ms, 6 of 16,000, 1,020 1.92 -> 1.66, 16 of 91,000, 1,630 18.7 -> 17.4 and, FP32, 5 of
// 45,000, 2,080 3.92 -> 3.25 ms.  (Half the waves with the band straight in registers, no LDS
// for it: 2.11 and 21.1 ms in the second and third.)
constexpr int MC = 32;                            // right-hand sides per launch, at most
constexpr int MT = 512;                           // threads per work-group
constexpr int AL = SB * SB / MT;                  // band-chunk entries per thread (8)

template <class T, int M>
__global__ void __launch_bounds__(MT) k_band_solve_m(
    BandArgs a, const int32_t* part_of, const T* v, const T* dinv, const int64_t* xoff,
    const double* xall, T* yall, T* zall, int groups, int PP, int n_mat, int most,
    const int32_t* active, int* err) {
  typedef Mfma<T> MF;
  typedef typename MF::S S;
  typedef T Y;                                    // hand-over scratch: the factor's precision
  constexpr int NCT = (M + 15) / 16;              // column tiles (1 or 2)
  constexpr int MP = 16 * NCT;                    // LDS row stride (zero columns past M)
  constexpr int YL = SB * M / MT;                 // solution-chunk entries per thread
  __shared__ S Ab[3][SB][SB + 1];                 // band chunks (double buffer), and the
  __shared__ S Yc[3][SB * MP];                    // inverse block and its right-hand side
  const Place pl = set_place(part_of, n_mat, groups, PP, most, err);
  const int g = pl.g, G = pl.P;                   // (no sum here depends on their number)
  if (pl.part < 0) return;
  int n, B, rs, n1, ncb, sep;                     // n1: last row of the matrix; ncb: blocks
  const T *cb, *dv;                               // with columns of their own
  const int64_t *fcb, *lrb;
  const double* x;
  Y *y, *z;
  const Y* mate;                                  // the other part's scratch, row r at n1 - r
  bool lower;
  const int mat = uniform_load(&a.part[pl.part].mat);
  if (active && !uniform_load(active + mat)) return;
  auto use = [&](int part) {
    const BandPart P = uniform_load(a.part + part);
    n = (int)P.rows, B = (int)P.B, rs = (int)P.ld - 1, n1 = (int)P.N - 1;
    ncb = (int)(P.cols + SB - 1) / SB;            // (a part has less than 2^31 entries)
    sep = (int)(P.kind == PART_UPPER ? P.sep : P.rows);
    lower = P.kind == PART_LOWER;
    cb = v + P.off + B;                           // entry (r, c) = cb[r * rs + c]
    dv = dinv + P.boff;
    fcb = a.fcb + P.eoff;
    lrb = a.lrb + P.eoff;
    x = xall + uniform_load(xoff + mat);
    y = yall + P.yoff * M;
    z = zall + P.yoff * M;
    const int mp = P.kind == PART_WHOLE ? part : uniform_load(part_of + 2 * mat + !lower);
    mate = (lower ? zall : yall) + uniform_load(&a.part[mp].yoff) * M;
  };
  use(pl.part);
  if (n == 0) return;
  // the separator of a split matrix is swept by the work-groups of both parts (see
  // band_solve_1_mat); the polls of every chunk are all the waiting it needs
  const bool own_lower = lower, split = lower || sep < n;
  const int upper = uniform_load(part_of + 2 * mat);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rt = wave & 3, ct = wave >> 2;        // this wave's row and column tile
  const bool tile = ct < NCT;                      // waves past the column tiles only stage
  const int li = lane & 15, lk = lane >> 4;
  if constexpr (MP > M)
    for (int idx = threadIdx.x; idx < 3 * SB * (MP - M); idx += MT) {
      const int e = idx % (SB * (MP - M));
      Yc[idx / (SB * (MP - M))][(e / (MP - M)) * MP + M + e % (MP - M)] = (S)0;
    }
  // forward chunk kk of block i0: band rows i0.., columns 64 kk..; backward chunk kk:
  // band rows 64 kk.., columns i0..; both with solution rows 64 kk..  Thread t stages band
  // rows t / 64 + 8 u at column t % 64.
  // entry idx of the solution rows of chunk kk: the part's own, or the separator's from the
  // upper part's backward solutions
  auto sol = [&](bool bwd, int kk, int idx) -> const Y* {
    if (bwd && kk >= ncb) return mate + ((int64_t)(n1 - kk * SB - idx / M) * M + idx % M);
    return (bwd ? z : y) + (int64_t)(kk * SB) * M + (uint32_t)idx;
  };
  auto fetch = [&](bool bwd, int i0, int kk, T (&fa)[AL], Y (&fy)[YL]) {
    const int r0 = (bwd ? kk * SB : i0) + wave;
    const int c = (bwd ? i0 : kk * SB) + lane;
#pragma unroll
    for (int u = 0; u < AL; ++u) fa[u] = cb[min(r0 + 8 * u, n - 1) * rs + c];
    const int yend = min(SB, n - kk * SB) * M;   // rows < n
#pragma unroll
    for (int u = 0; u < YL; ++u)
      fy[u] = poll_load(sol(bwd, kk, min((int)threadIdx.x + MT * u, yend - 1)));
  };
  auto stage = [&](int buf, bool bwd, int i0, int nb, int kk, const T (&fa)[AL],
                   Y (&fy)[YL]) {
    {                                              // until every needed entry is handed over
      const int yend = min(SB, n - kk * SB) * M;
      // the first test on the values already loaded is straight-line code, so the wait
      // before it covers only this chunk's loads, not the prefetch of the next one; the
      // polling loop is the slow path of a chunk still in flight
      bool ok = true;
#pragma unroll
      for (int u = 0; u < YL; ++u) ok = ok && ((int)threadIdx.x + MT * u >= yend || !is_mark(fy[u]));
      if (!__all(ok)) {
        int64_t spins = 0;
        for (;;) {
          if (poll_give_up(spins, err)) break;
#pragma unroll
          for (int u = 0; u < YL; ++u)
            fy[u] = poll_load(sol(bwd, kk, min((int)threadIdx.x + MT * u, yend - 1)));
          bool again = false;
#pragma unroll
          for (int u = 0; u < YL; ++u)
            again = again || ((int)threadIdx.x + MT * u < yend && is_mark(fy[u]));
          if (!__any(again)) break;
        }
      }
    }
    const int r0 = (bwd ? kk * SB : i0) + wave;
    const int c = (bwd ? i0 : kk * SB) + lane;
#pragma unroll
    for (int u = 0; u < AL; ++u) {
      const int r = r0 + 8 * u;
      const bool in = r < n && c <= r && c >= r - B && (!bwd || lane < nb);
      Ab[buf][wave + 8 * u][lane] = in ? (S)fa[u] : (S)0;
    }
    const int yend = min(SB, n - kk * SB) * M;   // rows < n
#pragma unroll
    for (int u = 0; u < YL; ++u) {
      const int idx = threadIdx.x + MT * u;
      Yc[buf][(idx / M) * MP + idx % M] = idx < yend ? (S)fy[u] : (S)0;
    }
  };
  // acc += A Yc over the 64-deep chunk for this wave's tile; A = Ab or Ab^T.  Even and odd
  // 4-deep steps go to two accumulators, so consecutive matrix instructions do not wait
  // for each other's result.
  auto mma = [&](int buf, bool trans, typename MF::V& acc) {
    if (!tile) return;
    typename MF::V acc1 = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < SB / 4; ks += 2) {
      const int kq0 = 4 * ks + lk, kq1 = kq0 + 4;
      const S a0 = trans ? Ab[buf][kq0][16 * rt + li] : Ab[buf][16 * rt + li][kq0];
      const S a1 = trans ? Ab[buf][kq1][16 * rt + li] : Ab[buf][16 * rt + li][kq1];
      const S b0 = Yc[buf][kq0 * MP + 16 * ct + li];
      const S b1 = Yc[buf][kq1 * MP + 16 * ct + li];
      acc = MF::mma(a0, b0, acc);
      acc1 = MF::mma(a1, b1, acc1);
    }
    acc += acc1;
  };
  // the chunks kk = first, first + step, .., last (step +1 or -1): chunk q is multiplied
  // from LDS buffer q % 2 while its loads were issued two chunks earlier; each wave stages
  // chunk q + 1 into the other buffer right after its product of chunk q, so one barrier
  // per chunk separates the staging of a buffer from its readers (the product two chunks
  // back, and the next product)
  // (dd, the block's inverse diagonal block, arrives meanwhile and goes to LDS after the first
  // product)
  auto keep = [&](const T (&dd)[AL]) {
#pragma unroll
    for (int u = 0; u < AL; ++u) {
      const int idx = threadIdx.x + MT * u;
      Ab[2][idx >> 6][idx & 63] = (S)dd[u];
    }
  };
  auto sweep = [&](bool bwd, int i0, int nb, int first, int count, int step, const T (&dd)[AL],
                   typename MF::V& acc) {
    if (count <= 0) {
      __syncthreads();                             // finish of the last block read buffer 2
      keep(dd);
      return;
    }
    T fa0[AL], fa1[AL];
    Y fy0[YL], fy1[YL];
    // chunk q, clamped to the last one: every prefetch is issued unconditionally (a chunk
    // past the end repeats the last, never used), which keeps the loads in flight the same
    // on every path and lets each wait count only the chunk it needs
    const int qmax = count - 1;
    auto kk_of = [&](int q) { return first + step * min(q, qmax); };
    fetch(bwd, i0, kk_of(0), fa0, fy0);
    fetch(bwd, i0, kk_of(1), fa1, fy1);
    __syncthreads();                               // the last block's readers are done
    stage(0, bwd, i0, nb, kk_of(0), fa0, fy0);
    for (int q = 0; q < count; q += 2) {
      __syncthreads();
      fetch(bwd, i0, kk_of(q + 2), fa0, fy0);
      mma(0, bwd, acc);
      if (q == 0) keep(dd);
      if (q + 1 >= count) break;
      stage(1, bwd, i0, nb, kk_of(q + 1), fa1, fy1);
      __syncthreads();
      fetch(bwd, i0, kk_of(q + 3), fa1, fy1);
      mma(1, bwd, acc);
      stage(0, bwd, i0, nb, kk_of(q + 2), fa0, fy0);
    }
  };
  // The right-hand side of a block, x forward and the block's forward solution backward, in
  // the layout of the sums; true if some of it is still to come.
  auto rhs = [&](bool bwd, int i0, int nb, double (&bb)[4]) -> bool {
    const int cc = min(16 * ct + li, M - 1);
    bool missing = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = i0 + min(16 * rt + MF::row(r, lk), nb - 1);
      if (!bwd) {
        bb[r] = x[(int64_t)(lower ? n1 - row : row) * M + cc];
      } else {
        const Y yb = poll_load(y + ((int64_t)row * M + cc));
        bb[r] = (double)yb;
        missing = missing || (tile && is_mark(yb));
      }
    }
    return missing;
  };
  // Yc <- rhs - accumulated sums (rows >= nb zero); the product of the inverse block with it
  // is the block's solution, handed over.
  // (bb, the block's right-hand side, and its inverse block are loaded before the sweep so
  // that their latency stays off the chain of hand-overs)
  auto finish = [&](bool bwd, int i0, int nb, double (&bb)[4], bool missing,
                    const typename MF::V& acc) {
    if (__any(missing)) {
      int64_t spins = 0;
      while (__any(rhs(bwd, i0, nb, bb)) && !poll_give_up(spins, err)) {}
    }
    if (!bwd && i0 >= sep) {                       // the lower part's share of these rows
      const int cc = min(16 * ct + li, M - 1);
      int64_t spins = 0;
      Y tb[4];
      for (;;) {
        bool ok = true;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ii = 16 * rt + MF::row(r, lk);
          tb[r] = poll_load(mate + ((int64_t)(n1 - i0 - min(ii, nb - 1)) * M + cc));
          ok = ok && (!tile || ii >= nb || !is_mark(tb[r]));
        }
        if (__all(ok) || poll_give_up(spins, err)) break;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) bb[r] -= (double)tb[r];
    }
    if (tile)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ii = 16 * rt + MF::row(r, lk), col = 16 * ct + li;
        if (col < M) Yc[2][ii * MP + col] = ii < nb ? (S)(bb[r] - (double)acc[r]) : (S)0;
      }
    __syncthreads();
    typename MF::V yv = {0, 0, 0, 0};
    mma(2, bwd, yv);
    Y* dst = bwd ? z : y;
    if (tile)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ii = 16 * rt + MF::row(r, lk), col = 16 * ct + li;
        if (ii < nb && col < M) hand_over(dst + ((int64_t)(i0 + ii) * M + col), (Y)yv[r]);
      }
  };
  // ---- forward: chunks in increasing order; those from kdone on are still in flight
#pragma unroll 1
  for (int seg = 0; seg < (split ? 2 : 1); ++seg) {
    if (seg) use(upper);
    const int kend = seg || !split || lower ? (n + SB - 1) / SB : sep / SB;
    for (int k = seg ? sep / SB + 2 * g + own_lower : g; k < kend; k += seg ? 2 * G : G) {
      const int i0 = k * SB;
      const int nb = (int)min(SB, n - i0);
      const int kfirst = max(max(i0 - B, 0), (int)fcb[k]) / SB;   // envelope start
      T dd[AL];
#pragma unroll
      for (int u = 0; u < AL; ++u) dd[u] = dv[(int64_t)min(k, ncb - 1) * SB * SB + threadIdx.x + MT * u];
      typename MF::V acc = {0, 0, 0, 0};
      double bb[4];
      if (k < ncb) rhs(false, i0, nb, bb);
      sweep(false, i0, nb, kfirst, min(k, ncb) - kfirst, 1, dd, acc);
      if (k < ncb) {
        finish(false, i0, nb, bb, false, acc);
      } else {                                     // separator rows of a lower part
        if (tile)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int ii = 16 * rt + MF::row(r, lk), col = 16 * ct + li;
            if (ii < nb && col < M) hand_over(y + ((int64_t)(i0 + ii) * M + col), (Y)acc[r]);
          }
        __syncthreads();
      }
    }
  }
  // ---- backward: chunks from the far end of the band inwards
#pragma unroll 1
  for (int seg = split ? 1 : 0; seg >= 0; --seg) {
    if (!seg && split) use(pl.part);
    const int kbeg = seg ? sep / SB : 0;
    const int kend = seg || !split || lower ? ncb : sep / SB;
    for (int kb = kend - 1 - (seg ? 2 * g + own_lower : g); kb >= kbeg;
         kb -= seg ? 2 * G : G) {
      const int i0 = kb * SB;
      const int nb = (int)min(SB, n - i0);
      const int klast = (min(min(n, i0 + nb + B), (int)lrb[kb]) - 1) / SB;   // last row block
      T dd[AL];
#pragma unroll
      for (int u = 0; u < AL; ++u) dd[u] = dv[(int64_t)kb * SB * SB + threadIdx.x + MT * u];
      typename MF::V acc = {0, 0, 0, 0};
      double bb[4];
      const bool missing = rhs(true, i0, nb, bb);
      sweep(true, i0, nb, klast, klast - kb, -1, dd, acc);
      finish(true, i0, nb, bb, missing, acc);
    }
  }
}

// Work-groups per part: as many as keep every work-group of the launch resident at once (a
// part waits at the pace of its slowest group); at most GMAX for one right-hand side.  For
// several a group has B / 64 chunks per block, 2 to 3 us each, and the chain passes a block in
// about 7 us, so B / 128 groups (8 at least) keep up with it and more only poll: with 16 in place of
// 8 groups 5 matrices of n = 45,000, B = 2,080 (FP32) 5.60 -> 3.92 ms, but 6 of 16,000, 1,020
// 1.92 -> 1.98 and 4 of 3,500, 370 0.51 -> 0.53 ms.  A matrix's work-groups run on one XCD
// (set_place), so it is the parts on the fullest XCD that are counted, against its eighth of
// the machine: counted together, 14 matrices of 24 parts would put 40 work-groups on an XCD's
// 32 slots.  The solves of one context are stream-ordered, so a launch may count on the whole
// machine; the eigensolver's run beside the interior factorisation, whose updates may hold slots
// for some milliseconds, in which the groups gather.  When several contexts solve concurrently (share > 1) an XCD may hold the fullest
// part of each: which XCD a launch begins with differs from launch to launch, and groups that
// wait for others must all have a slot (four contexts of two matrices with 16 work-groups a
// matrix ran into the poll limit in 7 of 100 set-ups; with 8 in none of 300).
static int solve_groups(BandSet& bs, const void* kernel, int which) {
  if (bs.solve_groups[which] > 0) return bs.solve_groups[which];
  int dev = 0, cus = 0, per_cu = 0;
  GX_HIP(hipGetDevice(&dev));
  GX_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  GX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel,
                                                      which == 0 ? SOLVE_THREADS : MT, 0));
  const int64_t capacity = (int64_t)cus * std::max(per_cu, 0) / 8;   // of an XCD
  std::vector<int64_t> parts(8, 0);
  for (const BandPart& p : bs.part) ++parts[p.mat & 7];
  const int64_t most = *std::max_element(parts.begin(), parts.end()) * std::max(bs.share, 1);
  const int cap = which == 0 ? GMAX
                             : (int)std::min<int64_t>(GMAX, std::max<int64_t>(8, bs.max_B / 128));
  int G = 1;
  const int top = bs.force_groups[which] > 0 ? std::min(bs.force_groups[which], cap) : cap;
  for (int c = top; c >= 2; --c)
    if (most * c <= capacity && bs.max_cols >= (int64_t)2 * SB * c) {
      G = c;
      break;
    }
  bs.solve_groups[which] = G;
  return G;
}

// Whether the links pay in a solve with G groups per part: they shorten the step from one
// hand-over to the next (2.7 -> 1.8 us) but give every work-group a second wait, product and
// reduction per block, so they pay where a step is bound by the hand-over and not by a
// group's share of the stream (64 B w / G bytes at about 22 GB/s).  Measured with eight
// groups, unlinked -> linked, at B w / G bytes: 370: 182 -> 141 us, 1,020: 727 -> 652 us,
// 1,040 (FP32): 2,079 -> 1,885 us, 1,220: 2,032 -> 2,072 us, 1,630: 5,767 -> 5,907 us; with
// sixteen, at 510: 731 -> 555 us, 520 (FP32): 1,940 -> 1,372 us.  (The joint solve of a batch
// asks with its own counts, for the links that a set's own solves were given.)
static bool link_pays(int64_t B, bool fp32, int G) {
  return G > 1 && B * (fp32 ? 4 : 8) <= 1100 * (int64_t)G;
}

static const void* solve1_kernel(const BandSet& bs) {
  return bs.fp32     ? reinterpret_cast<const void*>(&k_band_solve_1<float, false>)
         : bs.coarse ? reinterpret_cast<const void*>(&k_band_solve_1<double, true>)
                     : reinterpret_cast<const void*>(&k_band_solve_1<double, false>);
}

// The links of a factored set whose one-right-hand-side solves will use them.
void band_link(BandSet& bs, hipStream_t st) {
  if (!link_pays(bs.max_B, bs.fp32, solve_groups(bs, solve1_kernel(bs), 0))) return;
  const dim3 grid(nblocks(bs.max_cols, SB), bs.n_part);
  try {
    bs.link.alloc(2 * bs.n_inv);
  } catch (const Error& e) {
    if (e.code != GX_ENOMEM) throw;
    return;                                        // the solves go without
  }
  if (bs.fp32) {
    hipLaunchKernelGGL(k_link<float>, grid, dim3(512), 0, st, bs.d_part.p, bs.v32.p, bs.dinv32.p,
                       bs.link.p);
  } else {
    hipLaunchKernelGGL(k_link<double>, grid, dim3(512), 0, st, bs.d_part.p, bs.v64.p,
                       bs.dinv64.p, bs.link.p);
  }
  GX_HIP(hipGetLastError());
}

// The launch's error word (raised by a poll that timed out), zero until a check clears it;
// the counters of take_place follow it
static int* solve_err(BandSet& bs, hipStream_t st) {
  const size_t words = CL * (1 + 8) + 2 * (size_t)bs.n_mat;
  if (bs.err.n < words) {
    bs.err.alloc(words);
    clear(bs.err, st);
  }
  return bs.err.p;
}
static int solve_parts(const BandSet& bs) { return bs.split ? 2 : 1; }
// Groups of a part that take part in a solve, at most
static int most_groups(int most) { return most > 0 ? most : GMAX; }
static unsigned solve_grid(const BandSet& bs, int G) {
  return (unsigned)((bs.n_mat + 7) / 8 * 8 * G * solve_parts(bs));
}

// the place counters and the matrices' words of set_place
__device__ inline void clear_places(int* counters, int n_mat, int64_t i) {
  if (i < 8) counters[CL * i] = 0;
  for (int64_t j = i; j < 2 * n_mat; j += (int64_t)gridDim.x * blockDim.x)
    counters[CL * 8 + j] = 0;
}

__global__ void k_fill_mark(double* p, int64_t n, int* counters, int n_mat) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  clear_places(counters, n_mat, i);
  if (i < n) p[i] = __longlong_as_double((long long)YMARK);
}

// The forward and backward solution scratch of the single-right-hand-side solve (y, then
// z, 64-aligned segments per matrix), reset to the marker by a fill kernel on the stream
// (so the launch can be captured in a graph).
static void alloc_solve1_scratch(BandSet& bs) {
  if (!bs.ybuf.n) bs.ybuf.alloc(2 * std::max<int64_t>(bs.rows, 8));
}

static double* solve1_scratch(BandSet& bs, hipStream_t st) {
  alloc_solve1_scratch(bs);
  hipLaunchKernelGGL(k_fill_mark, dim3(nblocks((int64_t)bs.ybuf.n, 256)), dim3(256), 0, st,
                     bs.ybuf.p, (int64_t)bs.ybuf.n, solve_err(bs, st) + CL, bs.n_mat);
  return bs.ybuf.p;
}

// The solutions out of the scratch: rows of each part's own columns, w right-hand sides, of
// the active matrices
template <class Y>
__global__ void k_copy_out(const BandPart* part, const int64_t* xoff, int w, const Y* z,
                           double* x, const int32_t* active) {
  const BandPart& P = part[blockIdx.y];
  if (active && !active[P.mat]) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.cols * w) return;
  const int64_t r = i / w, o = P.kind == PART_LOWER ? (P.N - 1 - r) * w + (i - r * w) : i;
  x[xoff[P.mat] + o] = (double)z[P.yoff * w + i];
}

__global__ void k_fill_mark32(float* p, int64_t n, int* counters, int n_mat) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  clear_places(counters, n_mat, i);
  if (i < n) p[i] = __uint_as_float(YMARK32);
}

static void alloc_solvem_scratch(BandSet& bs) {
  const int64_t rows = std::max<int64_t>(bs.rows, 8);
  if (bs.mbuf.n < (size_t)(2 * rows * MC)) bs.mbuf.alloc(2 * rows * MC);
}

static void alloc_panel(BandSet& bs, hipStream_t st) {
  if (bs.d_poff.n) return;
  std::vector<int64_t> po(bs.n_mat + 1, 0);
  for (int j = 0; j < bs.n_mat; ++j) po[j + 1] = po[j] + bs.n[j] * MC;
  bs.panel.alloc(po[bs.n_mat]);
  bs.d_poff.alloc(bs.n_mat + 1);
  to_dev(bs.d_poff.p, po.data(), bs.n_mat + 1, st);
}

// The scratch of solves with ncol right-hand sides, so that it is missed, if there is no room,
// while the set can still be laid out again
void band_reserve(BandSet& bs, hipStream_t st, int ncol) {
  (void)solve_err(bs, st);
  if (ncol == 1) alloc_solve1_scratch(bs);
  else alloc_solvem_scratch(bs);
  if (ncol > MC) alloc_panel(bs, st);
}

template <int M>
static void launch_m(BandSet& bs, const BandArgs& a, const int64_t* d_xoff, double* x,
                     hipStream_t st, const int32_t* active) {
  const int G = bs.fp32 ? solve_groups(bs, reinterpret_cast<const void*>(&k_band_solve_m<float, M>), 1)
                        : solve_groups(bs, reinterpret_cast<const void*>(&k_band_solve_m<double, M>), 1);
  const int PP = solve_parts(bs);
  int* err = solve_err(bs, st);
  // y and z scratch of M columns: segments at yoff * M (64-aligned row offsets)
  alloc_solvem_scratch(bs);
  const int64_t rows = std::max<int64_t>(bs.rows, 8);
  const dim3 cgrid(nblocks(bs.max_cols * M, 256), bs.n_part);
  if (bs.fp32) {                                   // FP32 scratch in the same buffer
    float* y = reinterpret_cast<float*>(bs.mbuf.p);
    float* z = y + rows * M;
    hipLaunchKernelGGL(k_fill_mark32, dim3(nblocks(2 * rows * M, 256)), dim3(256), 0, st, y,
                       2 * rows * M, err + CL, bs.n_mat);
    hipLaunchKernelGGL((k_band_solve_m<float, M>), dim3(solve_grid(bs, G)), dim3(MT), 0, st, a,
                       bs.d_part_of.p, bs.v32.p, bs.dinv32.p, d_xoff, x, y, z, G, PP, bs.n_mat,
                       most_groups(bs.most), active, err);
    hipLaunchKernelGGL(k_copy_out<float>, cgrid, dim3(256), 0, st, bs.d_part.p, d_xoff, M, z, x,
                       active);
  } else {
    double* y = bs.mbuf.p;
    double* z = bs.mbuf.p + rows * M;
    hipLaunchKernelGGL(k_fill_mark, dim3(nblocks(2 * rows * M, 256)), dim3(256), 0, st, y,
                       2 * rows * M, err + CL, bs.n_mat);
    hipLaunchKernelGGL((k_band_solve_m<double, M>), dim3(solve_grid(bs, G)), dim3(MT), 0, st, a,
                       bs.d_part_of.p, bs.v64.p, bs.dinv64.p, d_xoff, x, y, z, G, PP, bs.n_mat,
                       most_groups(bs.most), active, err);
    hipLaunchKernelGGL(k_copy_out<double>, cgrid, dim3(256), 0, st, bs.d_part.p, d_xoff, M, z, x,
                       active);
  }
}

// Columns c0 .. c0 + w of a row-major block of ncol columns to or from a contiguous panel
// of w columns (panel of matrix j at poff[j]).
__global__ void k_panel_copy(const int64_t* nrows, const int64_t* xoff, double* x, int ncol,
                             int c0, int w, const int64_t* poff, double* panel,
                             const int32_t* active, int to_panel) {
  const int j = blockIdx.y;
  if (active && !active[j]) return;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nrows[j] * w) return;
  const int64_t r = e / w, c = e - r * w;
  double* xe = x + xoff[j] + r * ncol + c0 + c;
  double* pe = panel + poff[j] + e;
  if (to_panel)
    *pe = *xe;
  else
    *xe = *pe;
}

void band_solve(BandSet& bs, const int64_t* d_xoff, double* x, hipStream_t st, int ncol,
                const int32_t* active) {
  GX_REQUIRE(ncol == 1 || (ncol % 8 == 0 && ncol <= 2 * MC),
             "banded solve: right-hand sides must be 1 or a multiple of 8 up to 64");
  if (ncol > MC) {
    // panels of at most MC columns through a scratch block; the factor is read once per panel
    alloc_panel(bs, st);
    for (int c0 = 0; c0 < ncol; c0 += MC) {
      const int w = std::min(MC, ncol - c0);
      const dim3 grid(nblocks((int64_t)bs.max_n * w, 256), bs.n_mat);
      hipLaunchKernelGGL(k_panel_copy, grid, dim3(256), 0, st, bs.d_n.p, d_xoff, x, ncol, c0,
                         w, bs.d_poff.p, bs.panel.p, active, 1);
      band_solve(bs, bs.d_poff.p, bs.panel.p, st, w, active);
      hipLaunchKernelGGL(k_panel_copy, grid, dim3(256), 0, st, bs.d_n.p, d_xoff, x, ncol, c0,
                         w, bs.d_poff.p, bs.panel.p, active, 0);
    }
    GX_HIP(hipGetLastError());
    return;
  }
  const BandArgs a{bs.d_part.p, bs.d_fcb.p, bs.d_lrb.p, 0};
  if (ncol == 1 && !active) {
    const int G = solve_groups(bs, solve1_kernel(bs), 0), PP = solve_parts(bs);
    const bool linked = link_pays(bs.max_B, bs.fp32, G);
    const double* link = linked ? bs.link.p : nullptr;
    const dim3 grid(solve_grid(bs, G));
    int* err = solve_err(bs, st);
    double* y = solve1_scratch(bs, st);
    double* z = y + bs.ybuf.n / 2;
    if (bs.fp32)
      hipLaunchKernelGGL((k_band_solve_1<float, false>), grid, dim3(SOLVE_THREADS), 0, st, a,
                         bs.d_part_of.p, bs.v32.p, bs.dinv32.p, link, d_xoff, x, y, z, G, PP,
                         bs.n_mat, most_groups(bs.most), err);
    else if (bs.coarse)
      hipLaunchKernelGGL((k_band_solve_1<double, true>), grid, dim3(SOLVE_THREADS), 0, st, a,
                         bs.d_part_of.p, bs.v64.p, bs.dinv64.p, link, d_xoff, x, y, z, G, PP,
                         bs.n_mat, most_groups(bs.most), err);
    else
      hipLaunchKernelGGL((k_band_solve_1<double, false>), grid, dim3(SOLVE_THREADS), 0, st, a,
                         bs.d_part_of.p, bs.v64.p, bs.dinv64.p, link, d_xoff, x, y, z, G, PP,
                         bs.n_mat, most_groups(bs.most), err);
    hipLaunchKernelGGL(k_copy_out<double>, dim3(nblocks(bs.max_cols, 256), bs.n_part), dim3(256),
                       0, st, bs.d_part.p, d_xoff, 1, z, x, (const int32_t*)nullptr);
  } else {
    switch (ncol) {
      case 8: launch_m<8>(bs, a, d_xoff, x, st, active); break;
      case 16: launch_m<16>(bs, a, d_xoff, x, st, active); break;
      case 24: launch_m<24>(bs, a, d_xoff, x, st, active); break;
      default: launch_m<32>(bs, a, d_xoff, x, st, active); break;
    }
  }
  GX_HIP(hipGetLastError());
}

// Algorithmic bytes of one solve: the factor and the inverse diagonal blocks read once per
// sweep, the FP64 right-hand sides read and written once per sweep.
double band_solve_bytes(const BandSet& bs, int ncol, const int32_t* active_host, bool band) {
  const double w = bs.fp32 ? 4.0 : 8.0;
  double b = 0.0;
  for (int j = 0; j < bs.n_mat; ++j) {
    if (active_host && !active_host[j]) continue;
    const double nblk = (double)((bs.n[j] + SB - 1) / SB);
    const double factor = band ? (double)bs.n[j] * (double)(bs.B[j] + 1) + nblk * SB * SB
                               : (double)bs.env[j];
    b += 2.0 * w * factor + 4.0 * 8.0 * (double)bs.n[j] * ncol;
  }
  return b;
}

// The table of a multi-set solve: matrix j of set k solves in place on x[k] + xoff[k][j]
// (xoff[k]: host offsets of set k's right-hand-side segments).  Synchronises st.
void multi_solve_plan(MultiSolve& m, const std::vector<BandSet*>& sets,
                      const std::vector<double*>& x, const std::vector<const int64_t*>& xoff,
                      hipStream_t st) {
  GX_REQUIRE(!sets.empty() && x.size() == sets.size() && xoff.size() == sets.size(),
             "multi-set solve: one right-hand side and offset list per band set");
  GX_HIP(hipStreamSynchronize(st));                // earlier launches may still read the table
  m.sets = sets;
  m.fp32 = sets[0]->fp32;
  m.host.clear();
  m.max_n = 0;
  m.most = 0;
  std::vector<int> mats;                           // first part of each matrix in the table
  for (size_t k = 0; k < sets.size(); ++k) {
    BandSet& bs = *sets[k];
    GX_REQUIRE(bs.fp32 == m.fp32 && !bs.coarse && x[k] && xoff[k],
               "multi-set solve: band sets of one precision with right-hand sides");
    if (bs.most > 0) m.most = m.most ? std::min(m.most, bs.most) : bs.most;
    alloc_solve1_scratch(bs);
    double *y = bs.ybuf.p, *z = y + bs.ybuf.n / 2;
    for (int j = 0; j < bs.n_mat; ++j) {
      mats.push_back((int)m.host.size());
      for (int h = 0; h < 2; ++h) {
        const int ip = bs.part_of[2 * j + h];
        if (ip < 0) continue;
        const BandPart& p = bs.part[ip];
        const BandPart& o = bs.part[bs.part_of[2 * j + 1 - h] < 0 ? ip : bs.part_of[2 * j + 1 - h]];
        BandPtrs t;
        t.v = m.fp32 ? static_cast<const void*>(bs.v32.p + p.off)
                     : static_cast<const void*>(bs.v64.p + p.off);
        t.dinv = m.fp32 ? static_cast<const void*>(bs.dinv32.p + p.boff)
                        : static_cast<const void*>(bs.dinv64.p + p.boff);
        t.link = bs.link.n ? bs.link.p + 2 * p.boff : nullptr;
        t.x = x[k] + xoff[k][j];
        t.y = y + p.yoff;
        t.z = z + p.yoff;
        t.mate = (p.kind == PART_LOWER ? z : y) + o.yoff;
        t.n = p.rows;
        t.cols = p.cols;
        t.sep = p.kind == PART_UPPER ? p.sep : p.rows;
        t.N = p.N;
        t.B = p.B;
        t.fcb = bs.d_fcb.p + p.eoff;
        t.lrb = bs.d_lrb.p + p.eoff;
        t.G = 1;
        t.kind = p.kind;
        m.max_n = std::max(m.max_n, p.rows);
        m.host.push_back(t);
      }
    }
  }
  const int nm = (int)mats.size();
  m.n_part = (int)m.host.size();
  mats.push_back(m.n_part);
  GX_REQUIRE(nm > 0 && nm <= 65535, "multi-set solve: 1 to 65535 matrices");
  // Work-groups per part.  A matrix waits at the pace of its slowest group, so all of them
  // are to be resident, and work-group i runs on XCD i mod NX (each with its share of the
  // resident capacity).  Matrices go to XCDs largest first, each to the least loaded one
  // with free slots; the spare slots of an XCD then go to its matrices with the most factor
  // entries per group (one more group for each part, at most GMAX, at least two blocks of
  // rows per group).  If there are more parts than slots every part gets one group.
  int dev = 0, cus = 0, per_cu = 0;
  GX_HIP(hipGetDevice(&dev));
  GX_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const void* kf = m.fp32 ? reinterpret_cast<const void*>(&k_band_solve_1_multi<float>)
                          : reinterpret_cast<const void*>(&k_band_solve_1_multi<double>);
  GX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kf, SOLVE_THREADS, 0));
  const int NX = cus % 8 == 0 ? 8 : 1;             // XCDs (MI355X: 8 of 32 CUs)
  const int64_t per_x = (int64_t)cus / NX * std::max(per_cu, 1);
  std::vector<int> xcd(nm, 0);
  std::vector<double> wk(nm);
  auto parts = [&](int j) { return mats[j + 1] - mats[j]; };
  auto first = [&](int j) -> BandPtrs& { return m.host[mats[j]]; };
  for (int j = 0; j < nm; ++j) wk[j] = (double)first(j).N * (double)(first(j).B + 1) / parts(j);
  std::vector<int> order(nm);
  for (int j = 0; j < nm; ++j) order[j] = j;
  std::sort(order.begin(), order.end(),
            [&](int a, int b) { return wk[a] * parts(a) > wk[b] * parts(b); });
  std::vector<double> load(NX, 0.0);
  std::vector<int64_t> used(NX, 0);
  bool fits = true;
  for (int r = 0; r < nm; ++r) {
    const int j = order[r];
    int best = -1;
    for (int pass = 0; pass < 2 && best < 0; ++pass)
      for (int x = 0; x < NX; ++x)
        if ((pass || used[x] + parts(j) <= per_x) && (best < 0 || load[x] < load[best])) best = x;
    xcd[j] = best;
    load[best] += wk[j] * parts(j);
    used[best] += parts(j);
    fits = fits && used[best] <= per_x;
  }
  if (fits)
    for (int x = 0; x < NX; ++x)
      for (;;) {
        int pick = -1;
        for (int j = 0; j < nm; ++j) {
          const BandPtrs& t = first(j);
          if (xcd[j] != x || t.G >= GMAX || t.cols < (int64_t)2 * SB * (t.G + 1) ||
              used[x] + parts(j) > per_x)
            continue;
          if (pick < 0 || wk[j] / (double)t.G > wk[pick] / (double)first(pick).G) pick = j;
        }
        if (pick < 0) break;
        used[x] += parts(pick);
        for (int q = mats[pick]; q < mats[pick + 1]; ++q) ++m.host[q].G;
      }
  for (BandPtrs& t : m.host)
    if (!link_pays(t.B, m.fp32, (int)t.G)) t.link = nullptr;
  // a matrix's work-groups are neighbours in its XCD's list (take_place), the largest
  // matrices first: where there are more parts than slots, the last ones to start are short
  std::vector<std::vector<int32_t>> lists(NX);
  for (int j : order)
    for (int g = 0; g < (int)first(j).G; ++g)
      for (int q = mats[j]; q < mats[j + 1]; ++q) {
        lists[xcd[j]].push_back(q);
        lists[xcd[j]].push_back(g);
      }
  size_t slots = 0;
  for (auto& l : lists) slots = std::max(slots, l.size() / 2);
  std::vector<int32_t> wl(2 * slots * NX, -1);
  for (int x = 0; x < NX; ++x)
    for (size_t q = 0; q < lists[x].size() / 2; ++q) {
      wl[2 * (q * NX + x)] = lists[x][2 * q];
      wl[2 * (q * NX + x) + 1] = lists[x][2 * q + 1];
    }
  m.n_wg = (int)(slots * NX);
  m.n_class = NX;
  if (m.tab.n < m.host.size()) m.tab.alloc(m.host.size());
  to_dev(m.tab.p, m.host.data(), m.host.size(), st);
  if (m.work.n < wl.size()) m.work.alloc(wl.size());
  to_dev(m.work.p, wl.data(), wl.size(), st);
  const size_t words = CL * (1 + 8) + 2 * m.host.size();   // (of a matrix's parts, the first's)
  if (m.err.n < words) {
    multi_solve_check(m, st);                      // a time-out not yet reported
    m.err.alloc(words);
    clear(m.err, st);
  }
  GX_HIP(hipStreamSynchronize(st));                // wl and host are read by the copies
}

// Solves every matrix of the table in place (marker fill, solve, copy-out on st).
void multi_solve(MultiSolve& m, hipStream_t st) {
  GX_REQUIRE(m.n_part > 0, "multi-set solve: no table");
  const unsigned nr = (unsigned)std::min(m.n_part, 65535);
  hipLaunchKernelGGL(k_fill_mark_multi, dim3(nblocks((m.max_n + SB - 1) / SB * SB, 256), nr),
                     dim3(256), 0, st, m.tab.p, m.n_part, m.err.p + CL);
  if (m.fp32)
    hipLaunchKernelGGL(k_band_solve_1_multi<float>, dim3((unsigned)m.n_wg), dim3(SOLVE_THREADS),
                       0, st, m.tab.p, m.work.p, m.n_class, most_groups(m.most), m.err.p);
  else
    hipLaunchKernelGGL(k_band_solve_1_multi<double>, dim3((unsigned)m.n_wg), dim3(SOLVE_THREADS),
                       0, st, m.tab.p, m.work.p, m.n_class, most_groups(m.most), m.err.p);
  hipLaunchKernelGGL(k_copy_out_multi, dim3(nblocks(m.max_n, 256), nr), dim3(256), 0, st,
                     m.tab.p, m.n_part);
  GX_HIP(hipGetLastError());
}

// Raises if a multi-set solve since the last check timed out waiting for a block.
void multi_solve_check(MultiSolve& m, hipStream_t st) {
  if (!m.err.n) return;
  int h = 0;
  to_host(&h, m.err.p, 1, st);
  if (h) {
    clear(m.err, st);
    throw Error(GX_EHIP, "banded solve: a work-group timed out waiting for a block");
  }
}

// Raises if a multi-work-group solve since the last check timed out waiting for a block.
void band_solve_check(BandSet& bs, hipStream_t st) {
  if (!bs.err.n) return;
  int h = 0;
  to_host(&h, bs.err.p, 1, st);
  if (h) {
    clear(bs.err, st);
    throw Error(GX_EHIP, "banded solve: a work-group timed out waiting for a block");
  }
}

// Rows n1 of the upper part's own and n2 of the lower part's own columns of a matrix of
// order n and half bandwidth B eliminated from both ends (n1 = n2 = 0: not split).  Both are
// multiples of the 64-row block and leave a separator of at least B rows between them.  The
// chain of a split matrix has (n + B) / 2 rows instead of n, so there is little to gain
// below three bandwidths, and nothing below a few blocks; thousands of matrices fill the
// device as they are.
static void split_rows(int64_t n, int64_t B, size_t n_mat, int64_t* n1, int64_t* n2) {
  *n1 = *n2 = 0;
  if (n < 3 * B || n < 6 * SB || n_mat > 4096) return;
  const int64_t b = (n - std::max<int64_t>(B, 1)) / SB;    // blocks outside the separator
  *n1 = b / 2 * SB;
  *n2 = (b - b / 2) * SB;
}

// Whether a set's matrices gain by two parts (split_rows).  Where whole matrices leave no
// work-group idle (G each, fewer than GMAX) and a group's share of a block, 64 B w / G bytes,
// takes longer than a hand-over, the chain costs nothing, and two parts add the separator's
// fill and groups that do not divide by two.  Decided by the widest matrix for the whole set:
// the groups of a launch follow its fullest XCD, so a few split matrices would halve those of
// all.  Split against whole, a one-right-hand-side solve (us) and a factorisation with one
// solve (ms), at B w / G bytes (FP64 but where noted):
//     736:  64 of n =  6,000, B =   368          570 /   608     9.7 /  11.1
//     832:  24 of     20,000,     2,080, FP32  1,148 / 1,160    48.8 /  48.3
//   1,024:  32 of     16,000,     1,024        1,545 / 1,717    29.6 /  33.6
//   1,305:  24 of     20,000,     1,632        2,172 / 2,110    47.6 /  51.3
//   1,638:  48 of     16,000,     1,024        2,560 / 2,230    44.6 /  47.3
//   1,664:  48 of     20,000,     2,080, FP32  3,370 / 2,980   103.4 / 102.9
//   3,264:  64 of     20,000,     1,632        5,630 / 5,412   136.2 / 134.7
// (and a factor is solved with tens of times).
constexpr int64_t SPLIT_BYTES = 1500;
static bool split_pays(const std::vector<int64_t>& B, bool fp32) {
  int dev = 0, cus = 0;
  GX_HIP(hipGetDevice(&dev));
  GX_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int64_t G = std::max<int64_t>(cus / (int64_t)B.size(), 1);
  return G >= GMAX || *std::max_element(B.begin(), B.end()) * (fp32 ? 4 : 8) <= SPLIT_BYTES * G;
}

void band_layout(BandSet& bs, const std::vector<int64_t>& n, const std::vector<int64_t>& B,
                 bool fp32, hipStream_t st, const std::vector<int32_t>* first_node,
                 bool may_split) {
  may_split = may_split && split_pays(B, fp32);
  bs.n_mat = (int)n.size();
  bs.n = n;
  bs.B = B;
  bs.fp32 = fp32;
  bs.panel.release();
  bs.d_poff.release();
  bs.ybuf.release();
  bs.mbuf.release();
  bs.link.release();
  bs.max_n = bs.max_B = 0;
  bs.max_cols = 0;
  bs.total = bs.stored = bs.rows = bs.n_inv = 0;
  bs.split = false;
  bs.part.clear();
  bs.part_of.assign(2 * n.size(), -1);
  int64_t nblk = 0;                                // 64-row blocks of all parts
  // the stored half-bandwidth is B rounded up to a multiple of A, the entries of a 128-byte
  // line, and every part starts on a multiple of A: entry (r, c) then sits at an offset
  // congruent to c modulo A, so a row's entries from any multiple of A on fill whole
  // lines.  The extra band entries left of the band are zeros (outside the envelope).
  const int64_t A = fp32 ? 32 : 16;
  for (size_t j = 0; j < n.size(); ++j) {
    bs.B[j] = (B[j] + A - 1) / A * A;
    bs.total = (bs.total + A - 1) / A * A + n[j] * (bs.B[j] + 1);
    bs.max_n = std::max<int64_t>(bs.max_n, n[j]);
    bs.max_B = std::max<int64_t>(bs.max_B, bs.B[j]);
    int64_t n1 = 0, n2 = 0;
    if (may_split) split_rows(n[j], B[j], n.size(), &n1, &n2);
    for (int h = 0; h < (n2 ? 2 : 1); ++h) {
      BandPart p{};
      p.mat = (int)j;
      p.kind = n2 == 0 ? PART_WHOLE : h == 0 ? PART_UPPER : PART_LOWER;
      p.N = n[j];
      p.rows = h == 0 ? n[j] - n2 : n[j] - n1;
      p.cols = h == 0 ? p.rows : n2;
      p.sep = n2 == 0 ? p.rows : h == 0 ? n1 : n2;
      p.B = bs.B[j];
      p.ld = p.B + 1;
      p.fe[0] = p.sep;
      p.fb[1] = p.sep;
      p.fe[1] = p.cols;
      bs.stored = (bs.stored + A - 1) / A * A;
      p.off = bs.stored;
      bs.stored += p.rows * p.ld;
      p.yoff = bs.rows;
      bs.rows += (p.rows + SB - 1) / SB * SB;
      p.boff = bs.n_inv;
      bs.n_inv += (p.cols + SB - 1) / SB * SB * SB;
      p.eoff = nblk;
      nblk += (p.rows + SB - 1) / SB;
      bs.max_cols = std::max(bs.max_cols, p.cols);
      bs.part_of[2 * j + h] = (int32_t)bs.part.size();
      bs.part.push_back(p);
    }
    bs.split = bs.split || n2 > 0;
  }
  bs.n_part = (int)bs.part.size();
  // the envelope: row r from its first column f(r) (3 x its node's first coupled node, or
  // r - B) to the diagonal; env counts its entries, env_flops the Cholesky flops over it
  // (column c: h^2 + 2 h + 1 with h the rows below c that reach it)
  bs.env.assign(n.size(), 0);
  bs.env_flops = 0.0;
  std::vector<int64_t> node0(n.size() + 1, 0);     // first node of each matrix in first_node
  for (size_t j = 0; j < n.size(); ++j) {
    const int64_t nj = n[j];
    node0[j + 1] = node0[j] + nj / 3;
    GX_REQUIRE(!first_node || (nj % 3 == 0 && 2 * node0[j + 1] <= (int64_t)first_node->size()),
               "band layout: a first and a last node for every node of every matrix");
  }
  const int32_t* fn = first_node ? first_node->data() : nullptr;
  const int32_t* ln = first_node ? fn + node0[n.size()] : nullptr;
  for (size_t j = 0; j < n.size(); ++j) {
    const int64_t nj = n[j], Bj = B[j];
    std::vector<int64_t> diff(nj + 1, 0);
    for (int64_t r = 0; r < nj; ++r) {
      int64_t f = fn ? 3 * (int64_t)fn[node0[j] + r / 3] : r - Bj;
      f = std::min(std::max(f, std::max<int64_t>(r - Bj, 0)), r);
      bs.env[j] += r - f + 1;
      ++diff[f];
      --diff[r];
    }
    int64_t h = 0;
    for (int64_t c = 0; c < nj; ++c) {
      h += diff[c];
      bs.env_flops += (double)h * h + 2.0 * h + 1.0;
    }
  }
  // its tables by 64-row blocks, per part.  Rows of a lower part start at the last node that
  // their node couples to, and the separator's window in an upper part is filled by both
  // parts: its rows start at the window's start, or at their band's.
  std::vector<int64_t> fcb(std::max<int64_t>(nblk, 1)), lrb(fcb.size());
  for (const BandPart& p : bs.part) {
    const int64_t nbk = (p.rows + SB - 1) / SB, Bj = B[p.mat], nd = node0[p.mat];
    int64_t* fj = fcb.data() + p.eoff;
    int64_t* lj = lrb.data() + p.eoff;
    std::vector<int64_t> reach(nbk, 0);
    for (int64_t b = 0; b < nbk; ++b) fj[b] = p.rows;
    for (int64_t r = 0; r < p.rows; ++r) {
      int64_t f = r - Bj;
      if (fn && p.kind == PART_LOWER)
        f = p.N - 3 - 3 * (int64_t)ln[nd + (p.N - 1 - r) / 3];
      else if (fn)
        f = 3 * (int64_t)fn[nd + r / 3];
      f = std::min(std::max(f, std::max<int64_t>(r - Bj, 0)), r);
      if (p.kind == PART_UPPER && r >= p.sep) f = std::min(f, std::max(p.sep, r - Bj));
      fj[r / SB] = std::min(fj[r / SB], f);
      reach[f / SB] = std::max(reach[f / SB], r + 1);
    }
    int64_t run = 0;
    for (int64_t b = 0; b < nbk; ++b) {
      run = std::max(run, reach[b]);
      lj[b] = std::max(run, std::min(p.rows, (b + 1) * SB));
    }
  }
  bs.d_fcb.alloc(fcb.size());
  bs.d_lrb.alloc(lrb.size());
  to_dev(bs.d_fcb.p, fcb.data(), fcb.size(), st);
  to_dev(bs.d_lrb.p, lrb.data(), lrb.size(), st);
  bs.d_n.alloc(n.size());
  to_dev(bs.d_n.p, bs.n.data(), n.size(), st);
  bs.d_part.alloc(bs.part.size());
  to_dev(bs.d_part.p, bs.part.data(), bs.part.size(), st);
  bs.d_part_of.alloc(bs.part_of.size());
  to_dev(bs.d_part_of.p, bs.part_of.data(), bs.part_of.size(), st);
  if (fp32) {
    bs.v64.release();
    bs.dinv64.release();
    bs.v32.alloc(bs.stored + band_pad(bs.max_B));
    bs.dinv32.alloc(bs.n_inv);
  } else {
    bs.v32.release();
    bs.dinv32.release();
    bs.v64.alloc(bs.stored + band_pad(bs.max_B));
    bs.dinv64.alloc(bs.n_inv);
  }
  bs.solve_groups[0] = bs.solve_groups[1] = 0;
  GX_HIP(hipStreamSynchronize(st));
}

// All of the set's storage, with the gaps between the parts and the padding: a load outside
// a row's band, masked by a factor 0, must not meet a NaN there.
void band_zero(BandSet& bs, hipStream_t st) {
  if (bs.fp32)
    zero(bs.v32, st);
  else
    zero(bs.v64, st);
}

// ---------------------------------------------------------------------------------------
// Stand-alone factor-and-solve of caller-supplied band matrices (exposed for testing the
// subdomain solver in isolation).
// caller band entry e (bandwidth bw[j], rows of bw[j] + 1 entries) into the set's storage,
// which is zero beforehand
__global__ void k_band_import(int64_t total, const double* src, const double* dscale,
                              const int64_t* off, const int64_t* bw, const int64_t* doff,
                              int n_mat, BandView bv, float* d32, double* d64) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  int j = 0;
  while (j + 1 < n_mat && off[j + 1] <= e) ++j;
  const int64_t B = bw[j], r = (e - off[j]) / (B + 1), c = r + (e - off[j]) % (B + 1) - B;
  if (c < 0) return;                               // left of the first column: none
  double v = src[e];
  if (dscale) v *= dscale[doff[j] + r] * dscale[doff[j] + c];
  const int64_t d = band_pos(bv.part[bv.part_of[2 * j]],
                             bv.part[max(bv.part_of[2 * j + 1], 0)], r, c);
  if (d32) d32[d] = (float)v;
  else d64[d] = v;
}

__global__ void k_band_diag(int64_t rows, const double* src, const int64_t* off,
                            const int64_t* bw, const int64_t* doff, int n_mat,
                            double* dscale) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= rows) return;
  int j = 0;
  while (j + 1 < n_mat && doff[j + 1] <= q) ++j;
  const int64_t r = q - doff[j];
  const double d = src[off[j] + r * (bw[j] + 1) + bw[j]];
  dscale[q] = d > 0.0 ? 1.0 / sqrt(d) : 1.0;
}

__global__ void k_scale_rhs(int64_t rows, int nrhs, const double* dscale, double* x) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows * nrhs) return;
  x[e] *= dscale[e / nrhs];
}

}  // namespace gx

extern "C" gx_status gx_band_factor_solve(gx_ctx* c, int32_t n_mat, const int64_t* n,
                                          const int64_t* bw, const double* band,
                                          int32_t precision, int32_t nrhs, int32_t groups,
                                          double* x) {
  using namespace gx;
  GX_API_BEGIN(c)
  GX_REQUIRE(n_mat >= 1 && n && bw && band && x, "bad band matrices");
  GX_REQUIRE(precision == GX_FP64 || precision == GX_MIXED, "bad precision");
  GX_REQUIRE(nrhs == 1 || (nrhs % 8 == 0 && nrhs <= 2 * MC),
             "nrhs must be 1 or a multiple of 8 up to 64");
  std::vector<int64_t> nv(n, n + n_mat), bv(bw, bw + n_mat), off(n_mat + 1, 0),
      doff(n_mat + 1, 0), xoff(n_mat);
  for (int j = 0; j < n_mat; ++j) {
    GX_REQUIRE(nv[j] >= 1 && bv[j] >= 0 && bv[j] < nv[j], "bad order or bandwidth");
    off[j + 1] = off[j] + nv[j] * (bv[j] + 1);
    doff[j + 1] = doff[j] + nv[j];
    xoff[j] = doff[j] * nrhs;
  }
  hipStream_t s = c->stream;
  const bool fp32 = precision == GX_MIXED;
  BandSet bs;
  DevBuf<int64_t> d_off(n_mat + 1), d_doff(n_mat + 1), d_xoff(n_mat), d_bw(n_mat);
  to_dev(d_off.p, off.data(), n_mat + 1, s);
  to_dev(d_bw.p, bv.data(), n_mat, s);
  to_dev(d_doff.p, doff.data(), n_mat + 1, s);
  to_dev(d_xoff.p, xoff.data(), n_mat, s);
  DevBuf<double> dsc;
  if (fp32) {
    dsc.alloc(doff[n_mat]);
    hipLaunchKernelGGL(k_band_diag, dim3(nblocks(doff[n_mat], 256)), dim3(256), 0, s,
                       doff[n_mat], band, d_off.p, d_bw.p, d_doff.p, n_mat, dsc.p);
  }
  auto factor = [&](bool may_split) {
    band_layout(bs, nv, bv, fp32, s, nullptr, may_split);
    bs.force_groups[0] = bs.force_groups[1] = groups;
    bs.most = c->tune[2];
    band_zero(bs, s);
    hipLaunchKernelGGL(k_band_import, dim3(nblocks(off[n_mat], 256)), dim3(256), 0, s,
                       off[n_mat], band, fp32 ? dsc.p : nullptr, d_off.p, d_bw.p, d_doff.p, n_mat,
                       band_view(bs), fp32 ? bs.v32.p : nullptr, fp32 ? nullptr : bs.v64.p);
    GX_HIP(hipGetLastError());
    band_factor(c, bs, s, "the given band matrices");
    band_reserve(bs, s, nrhs);
  };
  try {
    factor(true);
  } catch (const Error& e) {
    if (e.code != GX_ENOMEM || !bs.split) throw;
    factor(false);                                 // no room for the rows stored twice
  }
  if (nrhs == 1) band_link(bs, s);
  if (fp32)
    hipLaunchKernelGGL(k_scale_rhs, dim3(nblocks(doff[n_mat] * nrhs, 256)), dim3(256), 0, s,
                       doff[n_mat], nrhs, dsc.p, x);
  band_solve(bs, d_xoff.p, x, s, nrhs);
  if (fp32)
    hipLaunchKernelGGL(k_scale_rhs, dim3(nblocks(doff[n_mat] * nrhs, 256)), dim3(256), 0, s,
                       doff[n_mat], nrhs, dsc.p, x);
  GX_HIP(hipGetLastError());
  band_solve_check(bs, s);
  GX_HIP(hipStreamSynchronize(s));
  GX_API_END(c)
}
