// Solve phase: preconditioned CG with one smoothed-aggregation V-cycle per
// iteration, all on the GPU.  Every sweep over a CSR matrix is HBM-bound and
// uses one of two kernel templates around a small operator (per-entry
// product, per-row epilogue):
//   - k_stream (rows of moderate length): a workgroup stages the row
//     pointers of a block of rows in LDS, loads all of the block's nonzeros
//     at once (up to kStreamCap/kBlock independent loads per thread, coalesced
//     column/value streams), stores the products in LDS and sums each row
//     there; with one lane per row the sum is the sequential fold in stored
//     order;
//   - k_vec (fallback for rows too long to stage): a group of G lanes per
//     row (G = 64 is a wavefront per row).
// Workgroups are renumbered so that each XCD (round-robin dispatch over the
// 8 XCDs) owns one contiguous range of rows, which keeps neighbour gathers
// in that XCD's L2.  Dot products are fused into the producing sweep as one
// partial per workgroup (plain stores); the kernels that need them fold them in
// a fixed order, or read the totals of one k_sum launch where they are many, and
// form the CG scalars on the device, so there are no float atomics and no
// device-wide fences.
// Method: PCG from x0 = 0 with recursive-residual stopping, true-residual
// verification and restart; damped-Jacobi/L1 V(nu_pre, nu_post) cycle with
// R = P^T and an exact coarsest solve.  The FP32 cycle keeps CG vectors, dot
// products and updates in FP64 and runs the cycle on FP32 copies (bf16-stored
// P and R optional); the flexible (Polak-Ribiere) beta keeps CG consistent
// with that inexact preconditioner.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <functional>
#include <initializer_list>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <type_traits>

#include "amg_internal.hpp"

namespace amg {
namespace {

// ------------------------------------------------------------ geometry

// Workgroup index remapped so that XCD k (round-robin dispatch) owns the
// contiguous logical range [k*G/8, (k+1)*G/8) when G is a multiple of 8.
__device__ inline int logical_block() {
  const int g = gridDim.x;
  if ((g & 7) == 0) return (blockIdx.x & 7) * (g >> 3) + (blockIdx.x >> 3);
  return blockIdx.x;
}

// Grid of `blocks` workgroups rounded up to a multiple of 8 (surplus
// workgroups find no rows and exit), so the XCD remap applies.
inline int round8(int64_t g) {
  if (g >= 64) g = (g + 7) / 8 * 8;
  return (int)std::max<int64_t>(g, 1);
}

// ----------------------------------------------------------- operators
// An operator supplies
//   PT prod(k, j)                 product for stored entry k (column j)
//   Row row_in(row)               the row's own operands (loaded by the sweep
//                                 kernels before the row sum is formed, so that
//                                 their latency overlaps the matrix stream)
//   void epi(row, s, in, d[])     consumes the row sum s; d[] collects dot partials
//   static constexpr int NRED     number of dot products reduced
// and, with kFold, folds the partial sums of earlier kernels itself (see Fold).

// CG and BiCGSTAB scalars from partial sums, without finalize kernels.  On
// systems of a few 100,000 rows a single-workgroup finalize kernel costs 2.7 us
// (launch and load latency), three or four times per iteration of about ten
// kernels.  In solves whose reductions have at most kFoldMax partials every
// workgroup of the consuming kernel sums them itself: at most 16 KB per sum from
// L2, the loads issued before the kernel's own (fold_load) and the wave sums
// combined after its gathers (fold_total), in one fixed order, so that every
// workgroup holds the same bits.  In larger solves the workgroups that would do
// so are too many (128^3: 8192 of 16 KB and two barriers each, 7.3 against 6.9
// ms): launches of k_sum form the totals first, and the consumers read one value
// per sum (tot): two per CG iteration.  In still larger ones (kEarlyStop) a third
// sums the update (BiCGSTAB: the half step) at once and makes its stop test, so
// that the cycle that follows is not run for nothing.
// (Fewer and longer workgroups, several row blocks each, keep the partials few
// but overlap less: 192^3 mixed 25.8 against 23.6 ms.)

// Rows from which the stop test has a launch of its own ahead of the cycle: 2.7
// us an iteration against a cycle a solve.  Solves to 1e-1 (2 iterations) and 1e-8
// (33 to 48), ms without and with it: 192^3 FP32 cycle 1.94 1.52, 22.5 22.2; 128^3
// 0.87 0.71, 8.60 8.52; 96^3 FP32 cycle 0.39 0.35, 2.97 3.05; 900^2 0.60 0.61 (5
// iterations), 4.39 4.52.
constexpr int kEarlyStop = 3 << 19;

struct NoFold {};

// Sum over the workgroup's threads of np partials: per-thread sum.
__device__ inline double fold_load(const double* __restrict__ p, int np, bool tot) {
  if (tot) return p[0];
  if (np <= kBlock) {
    const double a = p[min((int)threadIdx.x, np - 1)];
    return (int)threadIdx.x < np ? a : 0.0;
  }
  double a[kFoldMax / kBlock];
#pragma unroll
  for (int u = 0; u < kFoldMax / kBlock; ++u) a[u] = p[min((int)threadIdx.x + u * kBlock, np - 1)];
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < kFoldMax / kBlock; ++u) s = (int)threadIdx.x + u * kBlock < np ? s + a[u] : s;
  return s;
}

// Combines NV per-thread sums; every thread gets the totals.  Two barriers, none
// where the sums are totals already (tot).
template <int NV>
__device__ inline void fold_total(double (&v)[NV], bool tot) {
  if (tot) return;
  __shared__ double fold_red[NV][kBlock / 64];
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    const double t = group_sum<64>(v[m]);
    if ((threadIdx.x & 63) == 63) fold_red[m][threadIdx.x >> 6] = t;
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    double s = fold_red[m][0];
#pragma unroll
    for (int k = 1; k < kBlock / 64; ++k) s += fold_red[m][k];
    v[m] = s;
  }
  __syncthreads();
}

// Direction update fused with the product: p' = z + beta p (p' = z on the
// first iteration of a (re)start) and q' = A p', <p', q'>.  q' is formed as
// A z + beta q (the same vector in exact arithmetic, since q = A p), so the
// sweep gathers z only; p and q are read at the row itself (q is updated in
// place by the row's own thread).  p' goes to the second direction buffer.
// beta, the convergence test of the last update and the <r, z> test come from
// the partials of that update (pu) and of the V-cycle (pz).  Workgroup 0
// records the outcome.
//
// No kernel writes a field of the control block that it reads.  This holds for
// the stop flag too: the waves of a workgroup read it one by one, and one that
// left on a flag set meanwhile would leave the others waiting for LDS contents
// it never wrote (row pointers, partial sums).  So a kernel that ends the solve
// tests one flag and writes the next, and passes on what it found set:
//   CG        product  done -> gate[0],  update  gate[0] -> done
//   BiCGSTAB  direction  done -> gate[0],  half step  gate[0] -> gate[1],
//             full step  gate[1] -> done
// and the kernels in between test the flag that was written last.
struct OpSpmvXpay {
  using PT = double;
  static constexpr int NRED = 1;
  const double* v;
  const double* z;
  const double* p;
  double* pn;
  double* q;
  Ctl* ctl;
  const double* pz;
  const double* pu;
  int npz, npu, nz, tot, first, par;
  struct Fold {
    double s[3], rz, pq, thresh;
    int it, maxiter, flexible;
  };
  struct Row {
    double z, p, q;
  };
  __device__ PT prod_v(double a, int j) const { return a * z[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {z[row], first ? 0.0 : p[row], first ? 0.0 : q[row]}; }
  __device__ Fold fold_in() const {
    Fold f;
    f.s[0] = fold_load(pz, npz, tot);
    f.s[1] = nz > 1 ? fold_load(pz + npz, npz, tot) : 0.0;
    f.s[2] = first ? 0.0 : fold_load(pu, npu, tot);
    f.rz = ctl->rz2[par];
    f.pq = ctl->pq;
    f.thresh = ctl->thresh;
    f.it = ctl->it2[par];
    f.maxiter = ctl->maxiter;
    f.flexible = ctl->flexible;
    return f;
  }
  // beta of this iteration; false when the solve ends here
  __device__ bool fold_out(Fold& f, double& beta) const {
    fold_total<3>(f.s, tot);
    const double rzn = f.s[0], rr = f.s[2];
    int st = 0, it = f.it;
    if (!first) {
      ++it;
      if (rr <= f.thresh) st = 1;
      else if (!(rr == rr)) st = -1;
      else if (it >= f.maxiter) st = 2;
    }
    if (st == 0 && !(rzn > 0.0)) st = -1;
    beta = first ? 0.0 : f.flexible ? -f.s[1] / f.pq : rzn / f.rz;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ctl->rz2[par ^ 1] = rzn;
      ctl->it2[par ^ 1] = it;
      if (!first) ctl->rr = rr;
      if (st) {
        ctl->iters = it;
        ctl->state = st;
      }
      ctl->gate[0] = st != 0;
    }
    return st == 0;
  }
  // the sweep found the solve ended
  __device__ void ended() const {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl->gate[0] = 1;
  }
  __device__ void epi_fold(int row, PT s, const Row& a, double beta, double* d) const {
    const double pr = first ? a.z : a.z + beta * a.p;
    const double qn = first ? s : s + beta * a.q;
    pn[row] = pr;
    q[row] = qn;
    d[0] += pr * qn;
  }
};

template <class Op, class = void>
struct HasFold : std::false_type {};
template <class Op>
struct HasFold<Op, std::void_t<typename Op::Fold>> : std::true_type {};

// The folding hooks of a sweep: fold_in before its own loads, fold_out and the
// row epilogue after its row sums (nothing for operators that do not fold),
// and sweep_ended, the test of its stop flag.
template <class Op>
__device__ inline auto fold_in(const Op& op) {
  if constexpr (HasFold<Op>::value) return op.fold_in();
  else return NoFold{};
}
template <class Op, class F>
__device__ inline bool fold_out(const Op& op, F& f, double& beta) {
  if constexpr (HasFold<Op>::value) return op.fold_out(f, beta);
  else return true;
}
template <class Op>
__device__ inline bool sweep_ended(const Op& op, const int* __restrict__ stop) {
  if (!stop || !*stop) return false;
  if constexpr (HasFold<Op>::value) op.ended();
  return true;
}
template <class Op>
__device__ inline void row_epi(const Op& op, int row, typename Op::PT s, const typename Op::Row& in, double beta,
                               double* d) {
  if constexpr (HasFold<Op>::value) op.epi_fold(row, s, in, beta, d);
  else op.epi(row, s, in, d);
}

// r = b - A x, ||r||^2
struct OpTrueResid {
  using PT = double;
  static constexpr int NRED = 1;
  const double* v;
  const double* x;
  const double* b;
  double* r;
  struct Row {
    double b;
  };
  __device__ PT prod_v(PT a, int j) const { return a * x[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {b[row]}; }
  __device__ void epi(int row, PT s, const Row& a, double* d) const {
    const double ri = a.b - s;
    r[row] = ri;
    d[0] += ri * ri;
  }
};

// BiCGSTAB product with its reductions: out = A in, <w, out> and, with
// NRED = 2, <out, out> (v = A y with <r^, v>; t = A z with <s, t>, <t, t>).
template <int N>
struct OpSpmvDots {
  using PT = double;
  static constexpr int NRED = N;
  const double* v;
  const double* in;
  double* out;
  const double* w;
  struct Row {
    double w;
  };
  __device__ PT prod_v(double a, int j) const { return a * in[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {w[row]}; }
  __device__ void epi(int row, PT s, const Row& a, double* d) const {
    out[row] = s;
    d[0] += a.w * s;
    if constexpr (N == 2) d[1] += s * s;
  }
};

// Pre-smoothing from zero fused with the residual:
//   x_i = sw_i b_i ;  r_i = b_i - sum_j a_ij (sw_j b_j).
template <class T, class BT>
struct OpPre {
  using PT = T;
  static constexpr int NRED = 0;
  const T* v;
  const T* sw;
  const BT* b;
  T* x;
  T* r;
  struct Row {
    T b, w;
  };
  __device__ PT prod_v(PT a, int j) const { return a * (sw[j] * (T)b[j]); }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {(T)b[row], sw[row]}; }
  __device__ void epi(int row, PT s, const Row& a, double*) const {
    x[row] = a.w * a.b;
    r[row] = a.b - s;
  }
};

// Residual of the pre-smoothed iterate when x = sw o b was already written
// by the producer of b:  r_i = b_i - sum_j a_ij x_j.
template <class T, class BT>
struct OpResid {
  using PT = T;
  static constexpr int NRED = 0;
  const T* v;
  const BT* b;
  const T* x;
  T* r;
  struct Row {
    T b;
  };
  __device__ PT prod_v(PT a, int j) const { return a * x[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {(T)b[row]}; }
  __device__ void epi(int row, PT s, const Row& a, double*) const { r[row] = a.b - s; }
};

// Further Jacobi sweep in residual form, fused with the new residual:
//   x'_i = x_i + sw_i r_i ;  r'_i = b_i - sum_j a_ij (x_j + sw_j r_j).
template <class T, class BT>
struct OpSweep {
  using PT = T;
  static constexpr int NRED = 0;
  const T* v;
  const T* sw;
  const BT* b;
  const T* x;
  const T* r;
  T* x2;
  T* r2;
  struct Row {
    T x, w, r, b;
  };
  __device__ PT prod_v(PT a, int j) const { return a * (x[j] + sw[j] * r[j]); }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {x[row], sw[row], r[row], (T)b[row]}; }
  __device__ void epi(int row, PT s, const Row& a, double*) const {
    x2[row] = a.x + a.w * a.r;
    r2[row] = a.b - s;
  }
};

// Post-smoothing out_i = x_i + sw_i (b_i - sum_j a_ij x_j); RED >= 1 also
// <b, out>, RED == 2 also <out, q> (level 0 of CG: b = r, out = z).
template <class T, class BT, class OT, int RED>
struct OpPost {
  using PT = T;
  static constexpr int NRED = RED;
  const T* v;
  const T* sw;
  const BT* b;
  const T* x;
  OT* out;
  const double* q;
  struct Row {
    BT b;
    T x, w;
    double q;
  };
  __device__ PT prod_v(PT a, int j) const { return a * x[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const {
    Row a{b[row], x[row], sw[row], 0.0};
    if constexpr (RED >= 2) a.q = q[row];
    return a;
  }
  __device__ void epi(int row, PT s, const Row& a, double* d) const {
    const T o = a.x + a.w * ((T)a.b - s);
    const OT oo = (OT)o;
    out[row] = oo;
    if constexpr (RED >= 1) d[0] += (double)a.b * (double)oo;
    if constexpr (RED >= 2) d[1] += (double)oo * a.q;
  }
};

// y = R x (restriction); R values of type RT (double, float or bf16 bits).
// Also writes the coarse level's pre-smoothed iterate xc = swc o y.
template <class RT, class T>
struct OpRestrict {
  using PT = T;
  static constexpr int NRED = 0;
  const RT* v;
  const T* x;
  T* y;
  const T* swc;
  T* xc;
  struct Row {
    T w;
  };
  __device__ PT prod_v(RT a, int j) const { return (T)ValCvt<RT>::f(a) * x[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {xc ? swc[row] : (T)0}; }
  __device__ void epi(int row, PT s, const Row& a, double*) const {
    y[row] = s;
    if (xc) xc[row] = a.w * s;
  }
};

// x += P xc (prolongation and coarse-grid correction).
template <class RT, class T>
struct OpProlong {
  using PT = T;
  static constexpr int NRED = 0;
  const RT* v;
  const T* xc;
  T* x;
  struct Row {
    T x;
  };
  __device__ PT prod_v(RT a, int j) const { return (T)ValCvt<RT>::f(a) * xc[j]; }
  __device__ PT prod(int k, int j) const { return prod_v(v[k], j); }
  __device__ Row row_in(int row) const { return {x[row]}; }
  __device__ void epi(int row, PT s, const Row& a, double*) const { x[row] = a.x + s; }
};

template <int NRED>
__device__ inline void publish_partials(double (&d)[NRED > 0 ? NRED : 1], double* partials) {
  if constexpr (NRED > 0) {
    block_sum<NRED>(d);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int m = 0; m < NRED; ++m) partials[m * gridDim.x + blockIdx.x] = d[m];
    }
  }
}

// ------------------------------------------------------------ CSR sweeps

// U: staged entries per thread (the block's staging buffer holds kBlock*U
// entries; the shape sizes it to the matrix's largest row block, so that few
// of the unconditional loads are clamped duplicates).
template <int G3, int U, bool NT, class Op>
__global__ void __launch_bounds__(kBlock) k_stream(int n, const int* __restrict__ rp,
                                                   const int* __restrict__ ci, Op op, const int* __restrict__ stop,
                                                   double* __restrict__ partials) {
  if (n <= 0 || sweep_ended(op, stop)) return;
  constexpr int RB = kBlock / G3;
  using PT = typename Op::PT;
  __shared__ int s_rp[RB + 1];
  __shared__ PT s_p[kBlock * U];
  auto fold = fold_in(op);
  double d[Op::NRED > 0 ? Op::NRED : 1] = {}, beta = 0.0;
  const int lr = threadIdx.x / G3, lane = threadIdx.x & (G3 - 1);
  const int r0 = logical_block() * RB;
  for (int t = threadIdx.x; t <= RB; t += kBlock) s_rp[t] = rp[min(r0 + t, n)];
  const int row = r0 + lr;
  const typename Op::Row in = op.row_in(min(row, n - 1));
  __syncthreads();
  const int k0 = s_rp[0];
  const int nk = s_rp[RB] - k0;
  if (nk > 0) {
    // Loads are unconditional (indices clamped to the block's last entry) so
    // that all of them are in flight at once; only the LDS stores are masked.
    int col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) col[u] = stream_load<NT>(ci + k0 + min((int)threadIdx.x + u * kBlock, nk - 1));
    PT pv[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      pv[u] = op.prod_v(stream_load<NT>(op.v + k0 + min((int)threadIdx.x + u * kBlock, nk - 1)), col[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = threadIdx.x + u * kBlock;
      if (j < nk) s_p[j] = pv[u];
    }
  }
  __syncthreads();
  PT s = 0;
  if (row < n) {
    const int e = s_rp[lr + 1] - k0;
    for (int k = s_rp[lr] - k0 + lane; k < e; k += G3) s += s_p[k];
  }
  s = group_sum<G3>(s);
  if (!fold_out(op, fold, beta)) return;
  if (row < n && group_leader<G3>()) row_epi(op, row, s, in, beta, d);
  publish_partials<Op::NRED>(d, partials);
}

template <int G, class Op>
__global__ void __launch_bounds__(kBlock) k_vec(int n, const int* __restrict__ rp, const int* __restrict__ ci, Op op,
                                                const int* __restrict__ stop, double* __restrict__ partials) {
  if (n <= 0 || sweep_ended(op, stop)) return;
  using PT = typename Op::PT;
  constexpr int RB = kBlock / G;
  const int lr = threadIdx.x / G, lane = threadIdx.x & (G - 1);
  double d[Op::NRED > 0 ? Op::NRED : 1] = {}, beta = 0.0;
  auto fold = fold_in(op);
  if (!fold_out(op, fold, beta)) return;
  constexpr int U = 4;
  for (int r0 = logical_block() * RB; r0 < n; r0 += gridDim.x * RB) {
    const int row = r0 + lr;
    const typename Op::Row in = op.row_in(min(row, n - 1));
    PT s = 0;
    if (row < n) {
      const int kb = rp[row], ke = rp[row + 1];
      // U entries per lane in flight (clamped indices, unconditional loads);
      // each lane still adds its entries k, k+G, k+2G, ... in that order
      for (int k = kb + lane; k < ke; k += U * G) {
        int cc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cc[u] = ci[min(k + u * G, ke - 1)];
        PT pv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) pv[u] = op.prod(min(k + u * G, ke - 1), cc[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) s = k + u * G < ke ? s + pv[u] : s;
      }
    }
    s = group_sum<G>(s);
    if (row < n && group_leader<G>()) row_epi(op, row, s, in, beta, d);
  }
  publish_partials<Op::NRED>(d, partials);
}

// Sliced sweep: thread per row, the wave's 64 rows form one slice whose
// entries are stored column-major, so entry j of all 64 rows is one
// coalesced load.  The slice width is uniform across the wave; padding
// entries (column -1) are masked out of the sum.  Each row sums its entries
// in stored order (the same fold as a one-lane CSR sweep).
template <bool NT, class Op>
__global__ void __launch_bounds__(kBlock) k_sell(int n, const int* __restrict__ soff,
                                                 const int* __restrict__ sci, Op op, const int* __restrict__ stop,
                                                 double* __restrict__ partials) {
  if (n <= 0) return;
  using PT = typename Op::PT;
  double d[Op::NRED > 0 ? Op::NRED : 1] = {}, beta = 0.0;
  const int row = logical_block() * kBlock + threadIdx.x;
  const int rc = min(row, n - 1);
  // the wave's 64 rows are one slice: its offsets are scalar loads, which
  // leave the vector loads of the row operands in flight; the done flag is
  // loaded beside them
  const int sl = __builtin_amdgcn_readfirstlane(rc >> 6), lane = rc & 63;
  const int off = soff[sl];
  const int w = (soff[sl + 1] - off) >> 6;
  if (sweep_ended(op, stop)) return;
  auto fold = fold_in(op);
  const typename Op::Row in = op.row_in(rc);
  int col[kSellMaxW];
  typename std::remove_const<typename std::remove_pointer<decltype(op.v)>::type>::type val[kSellMaxW];
#pragma unroll
  for (int j = 0; j < kSellMaxW; ++j) {
    const int p = off + min(j, w - 1) * 64 + lane;
    col[j] = stream_load<NT>(sci + p);
    val[j] = stream_load<NT>(op.v + p);
  }
  PT pv[kSellMaxW];
#pragma unroll
  for (int j = 0; j < kSellMaxW; ++j) pv[j] = op.prod_v(val[j], col[j] < 0 ? rc : col[j]);
  PT s = 0;
#pragma unroll
  for (int j = 0; j < kSellMaxW; ++j) s = j < w && col[j] >= 0 ? s + pv[j] : s;
  if (!fold_out(op, fold, beta)) return;
  if (row < n) row_epi(op, row, s, in, beta, d);
  publish_partials<Op::NRED>(d, partials);
}

// Sliced sweep, offset form: slot j of the wave's slice holds offset
// slots[j].x for every row whose mask bit is set; the slot records are
// wave-uniform (scalar loads), so the only per-entry stream is the values.
// Each row adds its present entries in ascending offset (= column) order.
// UNI: every slot holds one value (op.v by slot): the sweep reads no value per
// entry.  Constant-coefficient operators then cost their vectors: 128^3
// Poisson, FP64: residual 24 -> 14 us, product 31 -> 23, post-smoother 36 -> 19.
// W: slots loaded per slice (the matrix's most, 3, 5, 7 or 8).  Loading a slot
// that no row has costs as much as one that it has: with 8 always, the product
// sweep of 10^7 tridiagonal unknowns (3 slots) took 110 us, now 85, that of 512^2
// (5 slots) 8.9, now 8.2; 7-point operators gain 1 %.  (Bytes are not what
// bounds the 7-point sweeps: storing only the upper triangle of a symmetric
// operator and reading the mirror values from cache took 169 of 691 MB from the
// 192^3 product and left it at 107 us.)
template <bool NT, bool UNI, int W, class Op>
__global__ void __launch_bounds__(kBlock) k_sello(int n, const int* __restrict__ soff,
                                                  const int4* __restrict__ slots, Op op, const int* __restrict__ stop,
                                                  double* __restrict__ partials) {
  if (n <= 0) return;
  using PT = typename Op::PT;
  double d[Op::NRED > 0 ? Op::NRED : 1] = {}, beta = 0.0;
  const int row = logical_block() * kBlock + threadIdx.x;
  const int rc = min(row, n - 1);
  const int sl = __builtin_amdgcn_readfirstlane(rc >> 6), lane = rc & 63;
  const int off = soff[sl];
  const int w = (soff[sl + 1] - off) >> 6;
  const int sb = off >> 6;
  if (sweep_ended(op, stop)) return;
  auto fold = fold_in(op);
  const typename Op::Row in = op.row_in(rc);
  typename std::remove_const<typename std::remove_pointer<decltype(op.v)>::type>::type val[W];
#pragma unroll
  for (int j = 0; j < W; ++j)
    val[j] = UNI ? op.v[sb + j] : stream_load<NT>(op.v + off + min(j, w - 1) * 64 + lane);
  // the slice's W records as one block (the array is padded so the
  // last slice's block stays in bounds)
  int4 rec[W];
#pragma unroll
  for (int j = 0; j < W; ++j) rec[j] = slots[sb + j];
  int col[W];
  bool has[W];
#pragma unroll
  for (int j = 0; j < W; ++j) {
    const unsigned bits = lane < 32 ? (unsigned)rec[j].z : (unsigned)rec[j].w;
    has[j] = j < w && ((bits >> (lane & 31)) & 1u);
    col[j] = has[j] ? rc + rec[j].x : rc;
  }
  PT pv[W];
#pragma unroll
  for (int j = 0; j < W; ++j) pv[j] = op.prod_v(val[j], col[j]);
  PT s = 0;
#pragma unroll
  for (int j = 0; j < W; ++j) s = has[j] ? s + pv[j] : s;
  if (!fold_out(op, fold, beta)) return;
  if (row < n) row_epi(op, row, s, in, beta, d);
  publish_partials<Op::NRED>(d, partials);
}

#define AMG_DISPATCH_G(g, ...)                             \
  switch (g) {                                             \
    case 1: { constexpr int G = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int G = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int G = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int G = 8; __VA_ARGS__; } break;   \
    case 16: { constexpr int G = 16; __VA_ARGS__; } break; \
    case 32: { constexpr int G = 32; __VA_ARGS__; } break; \
    default: { constexpr int G = 64; __VA_ARGS__; } break; \
  }

template <bool NT, class Op>
void sweep_form(const Shape& sh, int n, const int* rp, const int* ci, const Op& op, const int* stop,
                double* partials, hipStream_t s) {
  if (sh.stream >= 3) {
    const int4* slots = reinterpret_cast<const int4*>(ci);
#define AMG_SELLO(W)                                                                                              \
  if (sh.stream == 4)                                                                                             \
    hipLaunchKernelGGL((k_sello<false, true, W, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n, rp, slots, op, stop,   \
                       partials);                                                                                 \
  else                                                                                                            \
    hipLaunchKernelGGL((k_sello<NT, false, W, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n, rp, slots, op, stop,     \
                       partials);
    if (sh.w <= 3) {
      AMG_SELLO(3)
    } else if (sh.w <= 5) {
      AMG_SELLO(5)
    } else if (sh.w <= 7) {
      AMG_SELLO(7)
    } else {
      AMG_SELLO(8)
    }
#undef AMG_SELLO
  } else if (sh.stream == 2) {
    hipLaunchKernelGGL((k_sell<NT, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n, rp, ci, op, stop, partials);
  } else if (sh.stream) {
    switch (sh.u) {
      case 4:
        AMG_DISPATCH_G(sh.g, hipLaunchKernelGGL((k_stream<G, 4, NT, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n,
                                                rp, ci, op, stop, partials));
        break;
      case 8:
        AMG_DISPATCH_G(sh.g, hipLaunchKernelGGL((k_stream<G, 8, NT, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n,
                                                rp, ci, op, stop, partials));
        break;
      default:
        AMG_DISPATCH_G(sh.g, hipLaunchKernelGGL((k_stream<G, 12, NT, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n,
                                                rp, ci, op, stop, partials));
        break;
    }
  } else {
    AMG_DISPATCH_G(sh.g, hipLaunchKernelGGL((k_vec<G, Op>), dim3(sh.grid), dim3(kBlock), 0, s, n, rp, ci, op, stop,
                                            partials));
  }
}

// One sweep over a CSR matrix with operator `op`; returns the grid size
// (= number of partials written per reduced value).
template <class Op>
int sweep(const Shape& sh, int n, const int* rp, const int* ci, const Op& op, const int* stop, double* partials,
          hipStream_t s) {
  if (sh.nt) sweep_form<true>(sh, n, rp, ci, op, stop, partials, s);
  else sweep_form<false>(sh, n, rp, ci, op, stop, partials, s);
  return sh.grid;
}

// ------------------------------------------------------- dense coarse solve

// x = A_L^-1 b with the explicit (symmetric) inverse: thread i reads
// column i = row i, coalesced across threads.
template <class T, class BT, class OT>
__global__ void __launch_bounds__(kBlock) k_coarse(int n, int m, const T* __restrict__ inv, const BT* __restrict__ b,
                                                   OT* __restrict__ x, const int* __restrict__ stop) {
  if (stop && *stop) return;
  __shared__ T sb[kBlock];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  T s = 0;
  for (int j0 = 0; j0 < n; j0 += kBlock) {
    const int jj = j0 + threadIdx.x;
    sb[threadIdx.x] = jj < n ? (T)b[jj] : (T)0;
    __syncthreads();
    const int jn = min(kBlock, n - j0);
    if (i < n)
      for (int t = 0; t < jn; ++t) s += inv[(int64_t)(j0 + t) * m + i] * sb[t];
    __syncthreads();
  }
  if (i < n) x[i] = (OT)s;
}

// ------------------------------------------------------- BLAS1 (FP64)

inline int vec_grid(int n) { return round8(((int64_t)n + kBlock * kVecPer - 1) / (kBlock * kVecPer)); }

// Element range of this workgroup: kBlock*kVecPer consecutive entries.
__device__ inline int vec_base() { return logical_block() * (kBlock * kVecPer); }

// r = b, x = 0, partial <b, b>.
__global__ void __launch_bounds__(kBlock) k_cg_init(int n, const double* __restrict__ b,
                                                    double* __restrict__ r, double* __restrict__ x,
                                                    double* __restrict__ partials) {
  double d[1] = {0.0};
  const int base = vec_base();
  double bv[kVecPer];
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    bv[u] = i < n ? b[i] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      r[i] = bv[u];
      x[i] = 0.0;
      d[0] += bv[u] * bv[u];
    }
  }
  publish_partials<1>(d, partials);
}

// What the vector kernels write for the V-cycle that follows them: its
// level-0 pre-smoothed iterate x0 = sw o r, the right-hand side rounded to the
// cycle precision (two-sweep level 0), or nothing (the cycle reads r itself).
enum X0Mode { X0_NONE = 0, X0_SMOOTHED = 1, X0_COPY = 2 };

X0Mode x0_mode(const Hierarchy& H) {
  if (!H.prm.precondition || H.lv.size() < 2) return X0_NONE;
  if (H.lf > 0) return X0_SMOOTHED;
  return H.fp32() ? X0_COPY : X0_NONE;
}

// x += alpha p ; r -= alpha q ; partials <r, r> (pu); and x0 (see X0Mode).
// alpha from the product sweep's partials (pa) and the <r, z> of parity
// par ^ 1 that it recorded.  Workgroup 0 records <p, q> and the end of the
// solve (found by the product, or a breakdown here).
template <int MODE, class T>
__global__ void __launch_bounds__(kBlock) k_cg_update(int n, double* __restrict__ r,
                                                      const double* __restrict__ p, const double* __restrict__ q,
                                                      const T* __restrict__ sw, T* __restrict__ x0, Ctl* ctl,
                                                      const double* __restrict__ pa, int npa, int tot,
                                                      double* __restrict__ pu, int par) {
  const int ended = ctl->gate[0];
  const double rz = ctl->rz2[par ^ 1];
  const int iters = ctl->it2[par ^ 1];
  double* __restrict__ x = ctl->x;
  if (ended) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl->done = 1;
    return;
  }
  double f[1] = {fold_load(pa, npa, tot)};
  double alpha = 0.0, d[1] = {0.0};
  const int base = vec_base();
  double xv[kVecPer], rv[kVecPer], pv[kVecPer], qv[kVecPer];
  T wv[kVecPer];
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = min(base + (int)threadIdx.x + u * kBlock, n - 1);
    rv[u] = r[i];
    pv[u] = p[i];
    qv[u] = q[i];
    xv[u] = x[i];
    if constexpr (MODE == X0_SMOOTHED) wv[u] = sw[i];
  }
  fold_total<1>(f, tot);
  const double pq = f[0];
  const bool ok = pq > 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->pq = pq;
    if (!ok) {
      ctl->iters = iters;
      ctl->state = -1;
      ctl->done = 1;
    }
  }
  if (!ok) return;
  alpha = rz / pq;
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      x[i] = xv[u] + alpha * pv[u];
      const double ri = rv[u] - alpha * qv[u];
      r[i] = ri;
      if constexpr (MODE == X0_SMOOTHED) x0[i] = wv[u] * (T)ri;
      if constexpr (MODE == X0_COPY) x0[i] = (T)ri;
      d[0] += ri * ri;
    }
  }
  publish_partials<1>(d, pu);
}

// z = r (the identity preconditioner of plain CG).
__global__ void __launch_bounds__(kBlock) k_copy_z(int n, const double* __restrict__ r, double* __restrict__ z,
                                                   const int* __restrict__ stop) {
  if (stop && *stop) return;
  const int base = vec_base();
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) z[i] = r[i];
  }
}

// x0 = sw o r, or r rounded to T when there is no sw (first V-cycle of a
// solve or restart).
template <class T>
__global__ void __launch_bounds__(kBlock) k_sw_mul(int n, const T* __restrict__ sw, const double* __restrict__ r,
                                                   T* __restrict__ x0, const int* __restrict__ stop) {
  if (stop && *stop) return;
  const int base = vec_base();
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) x0[i] = sw ? sw[i] * (T)r[i] : (T)r[i];
  }
}

// <r, z> and <z, q> partials after a single-level (direct) preconditioner.
__global__ void __launch_bounds__(kBlock) k_dots_rz(int n, const double* __restrict__ r,
                                                    const double* __restrict__ z, const double* __restrict__ q,
                                                    const int* __restrict__ stop, double* __restrict__ partials) {
  if (stop && *stop) return;
  double d[2] = {0.0, 0.0};
  const int base = vec_base();
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      d[0] += r[i] * z[i];
      d[1] += z[i] * q[i];
    }
  }
  publish_partials<2>(d, partials);
}

// grad_val[k] = -(lambda[row k] * x[col k]): a group of 8 lanes per row.
__global__ void __launch_bounds__(kBlock) k_pattern_grad(int n, const int* __restrict__ rp,
                                                         const int* __restrict__ ci, const double* __restrict__ lam,
                                                         const double* __restrict__ x, double* __restrict__ g) {
  constexpr int G = 8;
  const int row = blockIdx.x * (kBlock / G) + threadIdx.x / G;
  const int lane = threadIdx.x & (G - 1);
  if (row >= n) return;
  const double li = lam[row];
  for (int k = rp[row] + lane; k < rp[row + 1]; k += G) g[k] = -(li * x[ci[k]]);
}

// ------------------------------------------------------- BiCGSTAB vectors

// r = b, r^ = b, x = 0, partial <b, b>.
__global__ void __launch_bounds__(kBlock) k_bi_init(int n, const double* __restrict__ b, double* __restrict__ r,
                                                    double* __restrict__ rh, double* __restrict__ x,
                                                    double* __restrict__ partials) {
  const int base = vec_base();
  double d[1] = {0.0};
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      const double bi = b[i];
      r[i] = bi;
      rh[i] = bi;
      x[i] = 0.0;
      d[0] += bi * bi;
    }
  }
  publish_partials<1>(d, partials);
}

// p = r on the first iteration of a (re)start, else p = r + beta (p - omega v);
// with x0, also the next V-cycle's level-0 pre-smoothed iterate x0 = sw o p
// (cycle precision T), so that its first sweep only forms the residual, or,
// without sw, p rounded to T.  ||r||^2 and <r^, r> of the last full step come
// from its partials (pf): the stop test, rho and beta = (rho / rho_old)
// (alpha / omega).  rho goes to ctl->rz (rho, alpha and omega are read here and
// written by later kernels only).
template <class T>
__global__ void __launch_bounds__(kBlock) k_bi_dir(int n, const double* __restrict__ r,
                                                   const double* __restrict__ v, double* __restrict__ p,
                                                   const T* __restrict__ sw, T* __restrict__ x0, Ctl* ctl, int first,
                                                   const double* __restrict__ pf, int npf, int tot) {
  const int done = ctl->done, iters = ctl->iters, maxiter = ctl->maxiter;
  const double rho0 = ctl->rho, alpha = ctl->alpha, omega = ctl->omega, thresh = ctl->thresh;
  if (done) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl->gate[0] = 1;
    return;
  }
  double f[2] = {first ? 0.0 : fold_load(pf, npf, tot), first ? 0.0 : fold_load(pf + npf, npf, tot)};
  double beta = 0.0;
  const int base = vec_base();
  double rv[kVecPer], vv[kVecPer], pv[kVecPer];
  T wv[kVecPer];
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = min(base + (int)threadIdx.x + u * kBlock, n - 1);
    rv[u] = r[i];
    vv[u] = v[i];
    pv[u] = p[i];
    wv[u] = x0 && sw ? sw[i] : (T)1;
  }
  fold_total<2>(f, tot);
  const double rr = f[0], rho = first ? rho0 : f[1];
  int st = 0;
  if (!first) {
    if (rr <= thresh) st = 1;
    else if (!(rr == rr)) st = -1;
    else if (iters >= maxiter) st = 2;
    else if (!(rho != 0.0) || !(rho == rho)) st = -1;
  }
  beta = first ? 0.0 : (rho / rho0) * (alpha / omega);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->rz = rho;
    if (!first) ctl->rr = rr;
    if (st) ctl->state = st;
    ctl->gate[0] = st != 0;
  }
  if (st) return;
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      const double pi = first ? rv[u] : rv[u] + beta * (pv[u] - omega * vv[u]);
      p[i] = pi;
      if (x0) x0[i] = wv[u] * (T)pi;
    }
  }
}

// alpha = rho / <r^, v> (partials pa); x += alpha y ; s = r - alpha v ; partials
// <s, s> (ps); with x0 also x0 = sw o s.
template <class T>
__global__ void __launch_bounds__(kBlock) k_bi_half(int n, const double* __restrict__ y,
                                                    const double* __restrict__ r, const double* __restrict__ v,
                                                    double* __restrict__ sv, const T* __restrict__ sw,
                                                    T* __restrict__ x0, Ctl* ctl, const double* __restrict__ pa,
                                                    int npa, int tot, double* __restrict__ ps) {
  const int ended = ctl->gate[0];
  const double rho = ctl->rz;
  double* __restrict__ x = ctl->x;
  if (ended) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl->gate[1] = 1;
    return;
  }
  double f[1] = {fold_load(pa, npa, tot)};
  double alpha = 0.0, d[1] = {0.0};
  const int base = vec_base();
  double xv[kVecPer], yv[kVecPer], rv[kVecPer], vv[kVecPer];
  T wv[kVecPer];
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = min(base + (int)threadIdx.x + u * kBlock, n - 1);
    yv[u] = y[i];
    rv[u] = r[i];
    vv[u] = v[i];
    xv[u] = x[i];
    wv[u] = x0 && sw ? sw[i] : (T)1;
  }
  fold_total<1>(f, tot);
  const bool ok = f[0] != 0.0 && f[0] == f[0];
  alpha = rho / f[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->rho = rho;
    if (ok) ctl->alpha = alpha;
    else ctl->state = -1;
    ctl->gate[1] = !ok;
  }
  if (!ok) return;
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      x[i] = xv[u] + alpha * yv[u];
      const double si = rv[u] - alpha * vv[u];
      sv[i] = si;
      if (x0) x0[i] = wv[u] * (T)si;
      d[0] += si * si;
    }
  }
  publish_partials<1>(d, ps);
}

// ||s||^2 (ps) ends the solve with x = x + alpha y, which is written already;
// else omega = <t, s> / <t, t> (pt), x += omega z ; r = s - omega t ; partials
// <r, r>, <r^, r> (pf).  The iteration is counted here.
__global__ void __launch_bounds__(kBlock) k_bi_full(int n, const double* __restrict__ z,
                                                    const double* __restrict__ sv, const double* __restrict__ t,
                                                    const double* __restrict__ rh, double* __restrict__ r, Ctl* ctl,
                                                    const double* __restrict__ ps, int nps,
                                                    const double* __restrict__ pt, int npt, int tot, double* __restrict__ pf) {
  const int ended = ctl->gate[1];
  const double thresh = ctl->thresh;
  double* __restrict__ x = ctl->x;
  if (ended) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl->done = 1;
    return;
  }
  double f[3] = {fold_load(ps, nps, tot), fold_load(pt, npt, tot), fold_load(pt + npt, npt, tot)};
  double omega = 0.0, d[2] = {0.0, 0.0};
  const int base = vec_base();
  double xv[kVecPer], zv[kVecPer], sl[kVecPer], tv[kVecPer], hv[kVecPer];
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = min(base + (int)threadIdx.x + u * kBlock, n - 1);
    zv[u] = z[i];
    sl[u] = sv[i];
    tv[u] = t[i];
    hv[u] = rh[i];
    xv[u] = x[i];
  }
  fold_total<3>(f, tot);
  const double ss = f[0], ts = f[1], tt = f[2];
  omega = ts / tt;
  int st = 0;
  if (ss <= thresh) st = 1;
  else if (!(ss == ss)) st = -1;
  else if (!(tt > 0.0) || !(omega != 0.0) || !(omega == omega)) st = -1;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->rr = ss;
    ctl->iters += 1;
    ctl->omega = omega;
    if (st) {
      ctl->state = st;
      ctl->done = 1;
    }
  }
  if (st) return;
#pragma unroll
  for (int u = 0; u < kVecPer; ++u) {
    const int i = base + threadIdx.x + u * kBlock;
    if (i < n) {
      x[i] = xv[u] + omega * zv[u];
      const double ri = sl[u] - omega * tv[u];
      r[i] = ri;
      d[0] += ri * ri;
      d[1] += hv[u] * ri;
    }
  }
  publish_partials<2>(d, pf);
}

// ------------------------------------------------------- finalize kernels

// Fixed-order fold of gridDim-sized partial arrays by one workgroup; the
// totals are valid in thread 0.
template <int NV>
__device__ inline void fold_partials(const double* __restrict__ partials, int np, double (&tot)[NV]) {
  __shared__ double red[NV][kFinBlock / 64];
  constexpr int UF = 8;
  double acc[NV];
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    double s = 0.0;
    for (int b0 = 0; b0 < np; b0 += kFinBlock * UF) {
      double t[UF];
#pragma unroll
      for (int u = 0; u < UF; ++u) {
        const int b = b0 + threadIdx.x + u * kFinBlock;
        t[u] = b < np ? partials[m * np + b] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < UF; ++u) s += t[u];
    }
    acc[m] = wave_sum(s);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int m = 0; m < NV; ++m) red[m][w] = acc[m];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      double s = red[m][0];
      for (int k = 1; k < kFinBlock / 64; ++k) s += red[m][k];
      tot[m] = s;
    }
  }
}

// Sums of long partial arrays: value blockIdx.x of the launch sums the np
// entries of its array into out[blockIdx.x].
struct SumArgs {
  const double* src[4];
  int np[4];
};
__global__ void __launch_bounds__(kFinBlock) k_sum(SumArgs a, double* __restrict__ out, const int* __restrict__ stop) {
  if (*stop) return;
  double t[1];
  fold_partials<1>(a.src[blockIdx.x], a.np[blockIdx.x], t);
  if (threadIdx.x == 0) out[blockIdx.x] = t[0];
}

// The same for ||r||^2 of CG's update (of parity par), with its stop test: the
// outcome the next product would find.  One workgroup: the flag is written
// after all its waves have read it.
__global__ void __launch_bounds__(kFinBlock) k_sum_update(const double* __restrict__ pu, int np,
                                                          double* __restrict__ out, Ctl* ctl, int par) {
  if (ctl->done) return;
  double t[1];
  fold_partials<1>(pu, np, t);
  if (threadIdx.x != 0) return;
  const double rr = t[0];
  out[0] = rr;
  const int it = ctl->it2[par ^ 1] + 1;
  const int st = rr <= ctl->thresh ? 1 : !(rr == rr) ? -1 : it >= ctl->maxiter ? 2 : 0;
  if (st) {
    ctl->rr = rr;
    ctl->iters = it;
    ctl->state = st;
    ctl->done = 1;
  }
}

// The same for ||s||^2 of BiCGSTAB's half step: the outcome k_bi_full would
// find (which counts the step otherwise).
__global__ void __launch_bounds__(kFinBlock) k_sum_half(const double* __restrict__ ps, int np,
                                                        double* __restrict__ out, Ctl* ctl) {
  if (ctl->gate[1]) return;
  double t[1];
  fold_partials<1>(ps, np, t);
  if (threadIdx.x != 0) return;
  const double ss = t[0];
  out[0] = ss;
  const int st = ss <= ctl->thresh ? 1 : !(ss == ss) ? -1 : 0;
  if (st) {
    ctl->rr = ss;
    ctl->iters += 1;
    ctl->state = st;
    ctl->gate[1] = 1;
  }
}

__global__ void __launch_bounds__(kFinBlock) k_fin_init(Ctl* ctl, const double* __restrict__ partials, int np,
                                                        double tol, int maxiter, int flexible, double* x) {
  double t[1];
  fold_partials<1>(partials, np, t);
  if (threadIdx.x != 0) return;
  const double bb = t[0];
  ctl->bb = bb;
  ctl->thresh = (tol * tol) * bb;
  ctl->iters = 0;
  ctl->it2[0] = ctl->it2[1] = 0;
  ctl->maxiter = maxiter;
  ctl->flexible = flexible;
  ctl->x = x;
  ctl->state = 0;
  ctl->done = 0;
  ctl->trr = 0.0;
  ctl->rr = bb;
  if (bb == 0.0) {
    ctl->state = 3;  // zero right-hand side: x = 0
    ctl->done = 1;
  } else if (!(bb == bb)) {
    ctl->state = -1;
    ctl->done = 1;
  } else if (maxiter <= 0) {
    ctl->state = 2;
    ctl->done = 1;
  }
}

// End of a chunk of iterations: the outcome of its last update
// (of parity par) for the host; the next product sweep would find the same.
__global__ void __launch_bounds__(kFinBlock) k_fin_chunk(Ctl* ctl, const double* __restrict__ pu, int np, int par) {
  if (ctl->done) return;
  double t[1];
  fold_partials<1>(pu, np, t);
  if (threadIdx.x != 0) return;
  const double rr = t[0];
  const int it = ctl->it2[par ^ 1] + 1;
  ctl->rr = rr;
  ctl->iters = it;
  const int st = rr <= ctl->thresh ? 1 : !(rr == rr) ? -1 : it >= ctl->maxiter ? 2 : 0;
  if (st) {
    ctl->state = st;
    ctl->done = 1;
  }
}

__global__ void __launch_bounds__(kFinBlock) k_fin_trr(Ctl* ctl, const double* __restrict__ partials, int np) {
  double t[1];
  fold_partials<1>(partials, np, t);
  if (threadIdx.x == 0) ctl->trr = t[0];
}

// BiCGSTAB scalars.  rho = <r^, r> (= ||b||^2 at the start, r^ = r = b).
__global__ void __launch_bounds__(kFinBlock) k_bfin_init(Ctl* ctl, const double* __restrict__ partials, int np,
                                                         double tol, int maxiter, double* x) {
  double t[1];
  fold_partials<1>(partials, np, t);
  if (threadIdx.x != 0) return;
  const double bb = t[0];
  ctl->bb = bb;
  ctl->thresh = (tol * tol) * bb;
  ctl->iters = 0;
  ctl->maxiter = maxiter;
  ctl->flexible = 0;
  ctl->x = x;
  ctl->state = 0;
  ctl->done = 0;
  ctl->trr = 0.0;
  ctl->rr = bb;
  ctl->rho = bb;
  ctl->alpha = 1.0;
  ctl->omega = 1.0;
  ctl->beta = 0.0;
  if (bb == 0.0) {
    ctl->state = 3;
    ctl->done = 1;
  } else if (!(bb == bb)) {
    ctl->state = -1;
    ctl->done = 1;
  } else if (maxiter <= 0) {
    ctl->state = 2;
    ctl->done = 1;
  }
}

// End of a chunk of BiCGSTAB iterations: the outcome of its last full step for
// the host; the next direction update would find the same.
__global__ void __launch_bounds__(kFinBlock) k_bfin_chunk(Ctl* ctl, const double* __restrict__ pf, int np) {
  if (ctl->done) return;
  double t[1];
  fold_partials<1>(pf, np, t);
  if (threadIdx.x != 0) return;
  const double rr = t[0];
  ctl->rr = rr;
  const int st = rr <= ctl->thresh ? 1 : !(rr == rr) ? -1 : ctl->iters >= ctl->maxiter ? 2 : 0;
  if (st) {
    ctl->state = st;
    ctl->done = 1;
  }
}

// Restart from the true residual r = b - A x (||r||^2 in trr): r^ = r is
// copied separately; rho = ||r||^2.
__global__ void k_bi_restart(Ctl* ctl) {
  ctl->done = 0;
  ctl->state = 0;
  ctl->rho = ctl->trr;
}

__global__ void k_ctl_restart(Ctl* ctl) {
  ctl->done = 0;
  ctl->state = 0;
  ctl->it2[0] = ctl->it2[1] = ctl->iters;
}

// ------------------------------------------------------------ V-cycle

// Copies the stop flag (0 when there is none) into the instrument record.
__global__ void k_snap_done(const int* stop, int* dst) {
  if (threadIdx.x == 0) dst[0] = stop ? *stop : 0;
}

struct CycleArgs {
  const double* r0;   // level-0 right-hand side (CG residual), FP64
  double* z0;         // level-0 result, FP64
  const double* q;    // CG q (flexible reduction), may be null
  const int* stop;    // flag to return on (null: none, and no reductions)
  double* partials;
  int red;            // 0 none, 1 <r,z>, 2 <r,z> and <z,q>
  int x0_ready;       // what the cycle starts from (X0Mode) already written
};

template <class T>
struct Bufs;

template <>
struct Bufs<double> {
  static double* x(Level& L) { return L.x64.p; }
  static double* b(Level& L) { return L.b64.p; }
  static double* r(Level& L) { return L.r64.p; }
  static double* xs(Level& L) { return L.xs64.p; }
  static double* rs(Level& L) { return L.rs64.p; }
  static const double* v(Level& L) { return L.av(); }
  static const double* sw(Level& L) { return L.sw.p; }
  static const double* inv(Coarse& C) { return C.inv.p; }
};
template <>
struct Bufs<float> {
  static float* x(Level& L) { return L.x32.p; }
  static float* b(Level& L) { return L.b32.p; }
  static float* r(Level& L) { return L.r32.p; }
  static float* xs(Level& L) { return L.xs32.p; }
  static float* rs(Level& L) { return L.rs32.p; }
  static const float* v(Level& L) { return L.av32(); }
  static const float* sw(Level& L) { return L.sw32.p; }
  static const float* inv(Coarse& C) { return C.inv32.p; }
};

template <class T>
void launch_restrict(Hierarchy& H, Level& L, const T* r, T* bc, const T* swc, T* xc, const int* stop, hipStream_t s) {
  if constexpr (std::is_same<T, double>::value) {
    sweep(L.shR, L.nagg, L.rrp.p, L.rci.p, OpRestrict<double, T>{L.rv.p, r, bc, swc, xc}, stop, nullptr, s);
  } else if (H.bf16()) {
    sweep(L.shR, L.nagg, L.rrp.p, L.rci.p, OpRestrict<uint16_t, T>{L.rbf.p, r, bc, swc, xc}, stop, nullptr, s);
  } else {
    sweep(L.shR, L.nagg, L.rrp.p, L.rci.p, OpRestrict<float, T>{L.rv32.p, r, bc, swc, xc}, stop, nullptr, s);
  }
}

template <class T>
void launch_prolong(Hierarchy& H, Level& L, const T* xc, T* x, const int* stop, hipStream_t s) {
  if constexpr (std::is_same<T, double>::value) {
    sweep(L.shP, L.n, L.prp.p, L.pci.p, OpProlong<double, T>{L.pv.p, xc, x}, stop, nullptr, s);
  } else if (H.bf16()) {
    sweep(L.shP, L.n, L.prp.p, L.pci.p, OpProlong<uint16_t, T>{L.pbf.p, xc, x}, stop, nullptr, s);
  } else {
    sweep(L.shP, L.n, L.prp.p, L.pci.p, OpProlong<float, T>{L.pv32.p, xc, x}, stop, nullptr, s);
  }
}

// One V-cycle on level-0 rhs a.r0 -> a.z0 (FP64 at the boundary, T inside).
// With a.red, the level-0 post-smoother emits the <r,z> (and <z,q>) partials.  Extra smoothing sweeps (nu > 1)
// ping-pong through the level's spare buffers.
// Returns the number of partials per reduced value.
template <class T>
int vcycle_impl(Hierarchy& H, const CycleArgs& a, hipStream_t s) {
  const int nl = (int)H.lv.size();
  Coarse& C = H.co;
  const int* stop = a.stop;
  if (!H.prm.precondition) {
    // plain CG: z = r
    const int n = H.n;
    hipLaunchKernelGGL(k_copy_z, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, a.r0, a.z0, stop);
    if (a.red) {
      const int g = vec_grid(n);
      hipLaunchKernelGGL(k_dots_rz, dim3(g), dim3(kBlock), 0, s, n, a.r0, a.z0, a.q ? a.q : a.z0, stop,
                         a.partials);
      return g;
    }
    return 0;
  }
  if (nl == 1) {
    {
      InstScope is(H, KID_COARSE, 0, s, stop);
      hipLaunchKernelGGL((k_coarse<double, double, double>), dim3((C.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                         C.n, C.m, C.inv.p, a.r0, a.z0, stop);
    }
    if (a.red) {
      const int g = vec_grid(C.n);
      hipLaunchKernelGGL(k_dots_rz, dim3(g), dim3(kBlock), 0, s, C.n, a.r0, a.z0, a.q ? a.q : a.z0, stop,
                         a.partials);
      return g;
    }
    return 0;
  }
  const int lf = H.lf;  // levels from here on run the two-sweep cycle
  if (lf == 0) {
    const T* b0;
    if constexpr (std::is_same<T, double>::value) {
      b0 = a.r0;
    } else {
      T* c = Bufs<T>::x(H.lv[0]);
      if (!a.x0_ready)
        hipLaunchKernelGGL((k_sw_mul<T>), dim3(vec_grid(H.n)), dim3(kBlock), 0, s, H.n, (const T*)nullptr, a.r0, c, stop);
      b0 = c;
    }
    return fused_cycle<T>(H, b0, a.r0, a.z0, a.q, a.red, stop, a.partials, s);
  }
  T* cx[AMG_MAX_LEVELS];
  T* cr[AMG_MAX_LEVELS];
  T* sx[AMG_MAX_LEVELS];
  T* sr[AMG_MAX_LEVELS];
  const int npre = H.prm.nu_pre, npost = H.prm.nu_post;
  for (int l = 0; l < lf; ++l) {
    Level& L = H.lv[l];
    cx[l] = Bufs<T>::x(L);
    cr[l] = Bufs<T>::r(L);
    sx[l] = Bufs<T>::xs(L);
    sr[l] = Bufs<T>::rs(L);
    {
      // pre-smoothing from zero: x = sw o b was written by the producer of b
      // (CG update on level 0, restriction below), so only r = b - A x remains
      InstScope is(H, KID_PRE, l, s, stop);
      if (l == 0 && !a.x0_ready)
        sweep(L.shA, L.n, L.arp(), L.aci(), OpPre<T, double>{Bufs<T>::v(L), Bufs<T>::sw(L), a.r0, cx[l], cr[l]}, stop,
              nullptr, s);
      else if (l == 0)
        sweep(L.shA, L.n, L.arp(), L.aci(), OpResid<T, double>{Bufs<T>::v(L), a.r0, cx[l], cr[l]}, stop, nullptr, s);
      else
        sweep(L.shA, L.n, L.arp(), L.aci(), OpResid<T, T>{Bufs<T>::v(L), Bufs<T>::b(L), cx[l], cr[l]}, stop, nullptr,
              s);
    }
    for (int k = 1; k < npre; ++k) {
      if (l == 0)
        sweep(L.shA, L.n, L.arp(), L.aci(),
              OpSweep<T, double>{Bufs<T>::v(L), Bufs<T>::sw(L), a.r0, cx[l], cr[l], sx[l], sr[l]}, stop, nullptr, s);
      else
        sweep(L.shA, L.n, L.arp(), L.aci(),
              OpSweep<T, T>{Bufs<T>::v(L), Bufs<T>::sw(L), Bufs<T>::b(L), cx[l], cr[l], sx[l], sr[l]}, stop, nullptr,
              s);
      std::swap(cx[l], sx[l]);
      std::swap(cr[l], sr[l]);
    }
    {
      InstScope is(H, KID_RESTRICT, l, s, stop);
      Level& Ln = H.lv[l + 1];
      const bool last = (l + 1 == lf);  // the two-sweep levels start from b
      launch_restrict<T>(H, L, cr[l], Bufs<T>::b(Ln), last ? nullptr : Bufs<T>::sw(Ln),
                         last ? nullptr : Bufs<T>::x(Ln), stop, s);
    }
  }
  T* res = Bufs<T>::x(H.lv[lf]);
  int np0 = 0;
  if (H.S == 1) {
    fused_cycle<T>(H, nullptr, nullptr, nullptr, nullptr, 0, stop, nullptr, s);
  } else {  // several systems: no dense tail (lf is the coarsest level)
    hipLaunchKernelGGL((k_coarse<T, T, T>), dim3((C.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, C.n, C.m,
                       Bufs<T>::inv(C), Bufs<T>::b(H.lv[lf]), res, stop);
  }
  for (int l = lf - 1; l >= 0; --l) {
    Level& L = H.lv[l];
    {
      InstScope is(H, KID_PROLONG, l, s, stop);
      launch_prolong<T>(H, L, res, cx[l], stop, s);
    }
    // free T buffers of this level after restriction: cr[l] and sx[l]
    T* cur = cx[l];
    T* spare[2] = {cr[l], sx[l]};
    for (int k = 0; k < npost; ++k) {
      const bool last = (k == npost - 1);
      const T* vv = Bufs<T>::v(L);
      const T* sw = Bufs<T>::sw(L);
      if (l == 0 && last) {
        int np = 0;
        {
          InstScope is(H, KID_POST, l, s, stop);
          if (a.red == 2)
            np = sweep(L.shA, L.n, L.arp(), L.aci(), OpPost<T, double, double, 2>{vv, sw, a.r0, cur, a.z0, a.q}, stop,
                       a.partials, s);
          else if (a.red == 1)
            np = sweep(L.shA, L.n, L.arp(), L.aci(), OpPost<T, double, double, 1>{vv, sw, a.r0, cur, a.z0, a.q}, stop,
                       a.partials, s);
          else
            sweep(L.shA, L.n, L.arp(), L.aci(), OpPost<T, double, double, 0>{vv, sw, a.r0, cur, a.z0, nullptr}, stop,
                  nullptr, s);
        }
        np0 = np;
      } else {
        T* dst = spare[k & 1];
        InstScope is(H, KID_POST, l, s, stop);
        if (l == 0)
          sweep(L.shA, L.n, L.arp(), L.aci(), OpPost<T, double, T, 0>{vv, sw, a.r0, cur, dst, nullptr}, stop, nullptr,
                s);
        else
          sweep(L.shA, L.n, L.arp(), L.aci(), OpPost<T, T, T, 0>{vv, sw, Bufs<T>::b(L), cur, dst, nullptr}, stop,
                nullptr, s);
        spare[k & 1] = cur;
        cur = dst;
      }
    }
    res = cur;
  }
  AMG_HIP(hipGetLastError());
  return np0;
}

int vcycle(Hierarchy& H, const CycleArgs& a, hipStream_t s) {
  if (H.fp32()) return vcycle_impl<float>(H, a, s);
  return vcycle_impl<double>(H, a, s);
}

void read_ctl(Hierarchy& H, hipStream_t s) {
  AMG_HIP(hipMemcpyAsync(H.h_ctl, H.ctl.p, sizeof(Ctl), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
}

// Launch shape of a sweep over a CSR matrix with `n` rows (host row
// pointers): the most rows per workgroup whose nonzeros fit the staging
// buffer, with enough lanes per row for the in-LDS sums of long rows.
// Staged entries per thread of a CSR-stream launch whose largest row block
// holds mx entries.
int stream_u(int mx) {
  for (int u : {4, 8}) if (mx <= u * kBlock) return u;
  return 12;
}

Shape make_shape(const std::vector<int>& rp, int n) {
  Shape sh;
  const double avg = n > 0 ? (double)(rp[n] - rp[0]) / n : 1.0;
  for (int rb = kBlock; rb >= kBlock / 64; rb >>= 1) {
    const int lanes = kBlock / rb;
    if (lanes < avg / 16.0 && rb > kBlock / 64) continue;
    int mx = 0;
    for (int r0 = 0; r0 < n; r0 += rb) mx = std::max(mx, rp[std::min(r0 + rb, n)] - rp[r0]);
    if (mx <= kStreamCap) {
      sh.stream = 1;
      sh.g = lanes;
      sh.u = stream_u(mx);
      sh.rows_per_block = rb;
      sh.max_block_nnz = mx;
      sh.grid = round8(((int64_t)n + rb - 1) / rb);
      return sh;
    }
  }
  sh.stream = 0;
  sh.g = 64;
  sh.rows_per_block = kBlock / 64;
  sh.grid = round8(std::min<int64_t>(((int64_t)n + sh.rows_per_block - 1) / sh.rows_per_block, kMaxGrid));
  return sh;
}

std::vector<int> host_copy(const DBuf<int>& d, int64_t count) {
  std::vector<int> h((size_t)count);
  if (count) AMG_HIP(hipMemcpy(h.data(), d.p, sizeof(int) * count, hipMemcpyDeviceToHost));
  return h;
}

}  // namespace

// ================================================================ public

InstScope::InstScope(Hierarchy& h, int kid, int level, hipStream_t st, const int* stop) : H(h), s(st) {
  on = H.inst.kernel == kid && (H.inst.level == level || H.inst.level < 0) &&
       2 * (H.inst.used + 1) <= (int)H.inst.ev.size();
  if (on) {
    hipLaunchKernelGGL(k_snap_done, dim3(1), dim3(64), 0, s, stop, H.inst.was_done.p + H.inst.used);
    AMG_HIP(hipEventRecord(H.inst.ev[2 * H.inst.used], s));
  }
}

InstScope::~InstScope() {
  if (on) {
    (void)hipEventRecord(H.inst.ev[2 * H.inst.used + 1], s);
    ++H.inst.used;
  }
}

namespace {

// ------------------------------------------------------------- autotuner
//
// Candidate launch shapes of one matrix: every stream shape whose row blocks
// fit the staging buffer (1..64 lanes per row in the in-LDS sums) and the
// direct lanes-per-row form with 1..64 lanes.  Each is timed with HIP events on
// the operator that runs on that matrix in the cycle; the fastest wins.
// Choices are cached in memory and, when AMG_TUNE_CACHE names a file, in a
// text file of "key stream lanes rows_per_block" lines, so that later runs
// (and therefore their rounding) repeat the same choice.

std::vector<Shape> candidate_shapes(const std::vector<int>& rp, int n) {
  std::vector<Shape> out;
  for (int rb = kBlock; rb >= kBlock / 64; rb >>= 1) {
    int mx = 0;
    for (int r0 = 0; r0 < n; r0 += rb) mx = std::max(mx, rp[std::min(r0 + rb, n)] - rp[r0]);
    if (mx > kStreamCap) continue;
    Shape sh;
    sh.stream = 1;
    sh.g = kBlock / rb;
    sh.u = stream_u(mx);
    sh.rows_per_block = rb;
    sh.max_block_nnz = mx;
    sh.grid = round8(((int64_t)n + rb - 1) / rb);
    out.push_back(sh);
  }
  for (int g = 1; g <= 64; g <<= 1) {
    Shape sh;
    sh.stream = 0;
    sh.g = g;
    sh.rows_per_block = kBlock / g;
    sh.grid = round8(std::min<int64_t>(((int64_t)n + sh.rows_per_block - 1) / sh.rows_per_block, kMaxGrid));
    out.push_back(sh);
  }
  return out;
}

std::mutex g_tune_mu;
std::map<std::string, Shape> g_tune;
bool g_tune_loaded = false;

void tune_load() {
  if (g_tune_loaded) return;
  g_tune_loaded = true;
  const char* path = std::getenv("AMG_TUNE_CACHE");
  if (!path) return;
  std::ifstream f(path);
  std::string key;
  Shape sh;
  while (f >> key >> sh.stream >> sh.g >> sh.rows_per_block) g_tune[key] = sh;
}

void tune_store(const std::string& key, const Shape& sh) {
  g_tune[key] = sh;
  const char* path = std::getenv("AMG_TUNE_CACHE");
  if (!path) return;
  std::ofstream f(path, std::ios::app);
  if (f) f << key << ' ' << sh.stream << ' ' << sh.g << ' ' << sh.rows_per_block << '\n';
}

template <class Op>
double time_shape(const Shape& sh, int n, const int* rp, const int* ci, const Op& op, hipStream_t s,
                  hipEvent_t e0, hipEvent_t e1) {
  for (int w = 0; w < 2; ++w) sweep(sh, n, rp, ci, op, nullptr, nullptr, s);
  AMG_HIP(hipEventRecord(e0, s));
  constexpr int reps = 5;
  for (int w = 0; w < reps; ++w) sweep(sh, n, rp, ci, op, nullptr, nullptr, s);
  AMG_HIP(hipEventRecord(e1, s));
  AMG_HIP(hipEventSynchronize(e1));
  float ms = 0.f;
  AMG_HIP(hipEventElapsedTime(&ms, e0, e1));
  return ms / reps;
}

// Shape for one matrix: the tuned one when enabled, else the row-length rule.
template <class MakeOp>
Shape pick_shape(Hierarchy& H, const char* kind, int level, const DBuf<int>& rpd, const DBuf<int>& cid, int n,
                 int ncols, MakeOp make_op, hipStream_t s) {
  const std::vector<int> rp = host_copy(rpd, n + 1);
  Shape rule = make_shape(rp, n);
  if (!H.prm.autotune || n == 0) return rule;
  int maxrow = 0;
  for (int i = 0; i < n; ++i) maxrow = std::max(maxrow, rp[i + 1] - rp[i]);
  char key[256];
  std::snprintf(key, sizeof key, "%s:n%d:nnz%d:max%d:c%d:p%d:t%d:w%d", kind, n, rp[n], maxrow, ncols,
                H.prm.vcycle_prec, H.fp32() && H.prm.transfer_bf16, H.S);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  tune_load();
  auto it = g_tune.find(key);
  if (it != g_tune.end()) {
    Shape sh = it->second;
    // recompute the grid for this matrix
    for (const Shape& c : candidate_shapes(rp, n))
      if (c.stream == sh.stream && c.g == sh.g) return c;
  }
  // representative operands: unit vectors of the cycle precision
  const int64_t len = std::max<int64_t>(n, ncols) + 1;
  hipEvent_t e0, e1;
  AMG_HIP(hipEventCreate(&e0));
  AMG_HIP(hipEventCreate(&e1));
  Shape best = rule;
  double tbest = 1e300;
  {
    auto op = make_op(len);
    for (const Shape& c : candidate_shapes(rp, n)) {
      const double t = time_shape(c, n, rpd.p, cid.p, op.op, s, e0, e1);
      if (t < tbest) {
        tbest = t;
        best = c;
      }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)level;
  tune_store(key, best);
  return best;
}

// Owns the scratch vectors of a timing operator.
template <class Op, class T>
struct TuneOp {
  TBuf<T> a, b, c;
  Op op;
};

}  // namespace

bool tune_lookup(const std::string& key, Shape* out) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  tune_load();
  auto it = g_tune.find(key);
  if (it == g_tune.end()) return false;
  *out = it->second;
  return true;
}

void tune_record(const std::string& key, const Shape& sh) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  tune_load();
  tune_store(key, sh);
}

void choose_shapes(Hierarchy& H, hipStream_t s) {
  const bool f32 = H.fp32();
  for (size_t l = 0; l < H.lv.size(); ++l) {
    Level& L = H.lv[l];
    const int nc = l + 1 < H.lv.size() ? L.nagg : 0;
    if (L.sell) {
      L.shA = Shape{};
      L.shA.stream = L.sell_uniform ? 4 : L.sell_form == 2 ? 3 : 2;
      L.shA.w = L.sell_w;
      L.shA.grid = round8(((int64_t)L.n + kBlock - 1) / kBlock);
    } else if (f32) {
      L.shA = pick_shape(H, "A", (int)l, L.rp, L.ci, L.n, nc, [&](int64_t len) {
        auto t = std::make_unique<TuneOp<OpResid<float, float>, float>>();
        t->a.alloc(len); t->b.alloc(len); t->c.alloc(len);
        AMG_HIP(hipMemsetAsync(t->a.p, 0, t->a.bytes(), s));
        AMG_HIP(hipMemsetAsync(t->b.p, 0, t->b.bytes(), s));
        t->op = OpResid<float, float>{L.v32.p, t->a.p, t->b.p, t->c.p};
        return std::move(*t);
      }, s);
    } else {
      L.shA = pick_shape(H, "A", (int)l, L.rp, L.ci, L.n, nc, [&](int64_t len) {
        TuneOp<OpResid<double, double>, double> t;
        t.a.alloc(len); t.b.alloc(len); t.c.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        AMG_HIP(hipMemsetAsync(t.b.p, 0, t.b.bytes(), s));
        t.op = OpResid<double, double>{L.v.p, t.a.p, t.b.p, t.c.p};
        return t;
      }, s);
    }
    // nontemporal entry streams for operators larger than the last-level cache
    const double abytes = L.sell ? (double)L.sell_len * (L.sell_form == 2 ? 8.0 : 12.0) : 12.0 * (double)L.nnz;
    L.shA.nt = abytes > kLlcBytes ? 1 : 0;
    if (l + 1 == H.lv.size()) continue;
    if (f32 && H.bf16()) {
      L.shP = pick_shape(H, "P", (int)l, L.prp, L.pci, L.n, nc, [&](int64_t len) {
        TuneOp<OpProlong<uint16_t, float>, float> t;
        t.a.alloc(len); t.b.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        AMG_HIP(hipMemsetAsync(t.b.p, 0, t.b.bytes(), s));
        t.op = OpProlong<uint16_t, float>{L.pbf.p, t.a.p, t.b.p};
        return t;
      }, s);
      L.shR = pick_shape(H, "R", (int)l, L.rrp, L.rci, L.nagg, L.n, [&](int64_t len) {
        TuneOp<OpRestrict<uint16_t, float>, float> t;
        t.a.alloc(len); t.b.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        t.op = OpRestrict<uint16_t, float>{L.rbf.p, t.a.p, t.b.p, nullptr, nullptr};
        return t;
      }, s);
    } else if (f32) {
      L.shP = pick_shape(H, "P", (int)l, L.prp, L.pci, L.n, nc, [&](int64_t len) {
        TuneOp<OpProlong<float, float>, float> t;
        t.a.alloc(len); t.b.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        AMG_HIP(hipMemsetAsync(t.b.p, 0, t.b.bytes(), s));
        t.op = OpProlong<float, float>{L.pv32.p, t.a.p, t.b.p};
        return t;
      }, s);
      L.shR = pick_shape(H, "R", (int)l, L.rrp, L.rci, L.nagg, L.n, [&](int64_t len) {
        TuneOp<OpRestrict<float, float>, float> t;
        t.a.alloc(len); t.b.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        t.op = OpRestrict<float, float>{L.rv32.p, t.a.p, t.b.p, nullptr, nullptr};
        return t;
      }, s);
    } else {
      L.shP = pick_shape(H, "P", (int)l, L.prp, L.pci, L.n, nc, [&](int64_t len) {
        TuneOp<OpProlong<double, double>, double> t;
        t.a.alloc(len); t.b.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        AMG_HIP(hipMemsetAsync(t.b.p, 0, t.b.bytes(), s));
        t.op = OpProlong<double, double>{L.pv.p, t.a.p, t.b.p};
        return t;
      }, s);
      L.shR = pick_shape(H, "R", (int)l, L.rrp, L.rci, L.nagg, L.n, [&](int64_t len) {
        TuneOp<OpRestrict<double, double>, double> t;
        t.a.alloc(len); t.b.alloc(len);
        AMG_HIP(hipMemsetAsync(t.a.p, 0, t.a.bytes(), s));
        t.op = OpRestrict<double, double>{L.rv.p, t.a.p, t.b.p, nullptr, nullptr};
        return t;
      }, s);
    }
    // the restriction gathers the fine vector, which a cached stream would
    // evict; the prolongation gathers only the (small) coarse vector, and
    // nontemporal loads measured slower there (192^3: 93.8 vs 89.7 us)
    const double pwb = f32 ? (H.bf16() ? 2.0 : 4.0) : 8.0;
    L.shR.nt = (pwb + 4.0) * (double)L.pnnz > kLlcBytes ? 1 : 0;
    L.shP.nt = 0;
  }
  AMG_HIP(hipStreamSynchronize(s));
}

// Partials per reduced value of the largest reducing grid of a solve on H.
int64_t partials_region(const Hierarchy& H) {
  int64_t np = std::max<int64_t>(vec_grid(H.n), H.lv[0].shA.grid);
  if (H.lf == 0) np = std::max<int64_t>(np, H.lv[0].up.grid);
  return std::max<int64_t>(np, vec_grid(std::max(H.co.n, 1)));
}

// Product, update and V-cycle of CG (1, 1, 2 values); products, half and full
// step of BiCGSTAB (1, 2, 1, 2); the totals behind them.  (The allocation-free
// CG solve admits a system by this count.)
int64_t solve_partials_count(const Hierarchy& H) {
  return partials_region(H) * (H.prm.solver == AMG_SOLVER_PCG ? 4 : 6) + 64;
}

SolveWork solve_work(Hierarchy& H) {
  return SolveWork{H.r.p, H.z.p, H.p.p, H.z2.p, H.q.p, H.partials.p, H.ctl.p, H.h_ctl, true};
}

void alloc_solve_workspace(Hierarchy& H) {
  const int n = H.n;
  H.r.alloc(n);
  H.z.alloc(n);
  H.p.alloc(n);
  H.z2.alloc(n);
  H.q.alloc(n);
  H.partials.alloc(solve_partials_count(H));
  if (!H.ctl.p) {
    H.ctl.alloc(1);
    AMG_HIP(hipMemset(H.ctl.p, 0, sizeof(Ctl)));
  }
  if (!H.h_ctl) AMG_HIP(hipHostMalloc((void**)&H.h_ctl, sizeof(Ctl), hipHostMallocDefault));
  // spare vectors for extra smoothing sweeps
  if (H.prm.nu_pre > 1 || H.prm.nu_post > 1) {
    for (Level& L : H.lv) {
      if (H.fp32()) { L.xs32.alloc(L.n); L.rs32.alloc(L.n); }
      else { L.xs64.alloc(L.n); L.rs64.alloc(L.n); }
    }
  }
}

// Algorithmic bytes of one launch: each matrix array streamed once, each
// distinct vector operand read once (neighbour gathers counted once), each
// output written once.
double kernel_bytes(const Hierarchy& H, int kid, int level, int flexible) {
  const int nl = (int)H.lv.size();
  if (level < 0 || level >= nl) return 0.0;
  const Level& L = H.lv[level];
  const double v = H.fp32() ? 4.0 : 8.0;                        // cycle vector/value bytes
  const double pw = H.fp32() ? (H.bf16() ? 2.0 : 4.0) : 8.0;   // transfer value bytes
  const double n = L.n, nnz = (double)L.nnz;
  auto M = [](double nz, double rows, double w) { return nz * (w + 4.0) + 4.0 * (rows + 1.0); };
  // operator matrix: the sliced copy when present (its padded values, and
  // columns or slot records, and slice offsets), else the CSR arrays
  auto MA = [&](double w) {
    if (!L.sell) return M(nnz, n, w);
    const double slices = 4.0 * ((L.n + 63) / 64 + 1.0);
    if (L.sell_uniform) return (16.0 + w) * (double)(L.sell_len / 64) + slices;
    if (L.sell_form == 2) return (double)L.sell_len * w + 16.0 * (double)(L.sell_len / 64) + slices;
    return (double)L.sell_len * (w + 4.0) + slices;
  };
  const double bw = level == 0 ? 8.0 : v;                       // rhs of the level
  const bool has_next = level + 1 < nl;
  if (nl > 1 && level >= H.lf && H.S == 1 && kid != KID_SPMV_DOT && kid != KID_CG_UPDATE) return fused_bytes(H, kid, level);
  const bool next_coarsest = level + 2 == nl;
  switch (kid) {
    // direction update fused with the product: gathers z, reads old p and q,
    // writes new p and q
    case KID_SPMV_DOT: return MA(8.0) + 40.0 * n;
    // residual of the pre-smoothed iterate: reads b, gathers x, writes r
    case KID_PRE: return MA(v) + (bw + 2.0 * v) * n;
    case KID_POST: {
      const double ow = level == 0 ? 8.0 : v;
      return MA(v) + (bw + 2.0 * v + ow) * n + (level == 0 && flexible ? 8.0 * n : 0.0);
    }
    case KID_RESTRICT: {
      if (!has_next) return 0.0;
      const double nc = (double)L.nagg;
      return M((double)L.pnnz, nc, pw) + v * n + v * nc + (next_coarsest ? 0.0 : 2.0 * v * nc);
    }
    case KID_PROLONG:
      if (!has_next) return 0.0;
      return M((double)L.pnnz, n, pw) + v * (double)L.nagg + 2.0 * v * n;
    // x, r, p, q read; x, r written; sw read and x0 = sw o r written in cycle precision
    case KID_CG_UPDATE: {
      const X0Mode m = x0_mode(H);
      return 48.0 * n + (m == X0_SMOOTHED ? 2.0 : m == X0_COPY ? 1.0 : 0.0) * v * n;
    }
    case KID_XPAY: return 0.0;  // fused into KID_SPMV_DOT
    case KID_COARSE: {
      const double nc = H.co.n;
      return nc * nc * (nl == 1 ? 8.0 : v) + 2.0 * nc * (nl == 1 ? 8.0 : v);
    }
  }
  return 0.0;
}

// Bytes of one PCG iteration (SpMV+dot, update, V-cycle, direction update).
double iteration_bytes(const Hierarchy& H, int flexible) {
  const int nl = (int)H.lv.size();
  if (!H.prm.precondition)  // plain CG; with the flexible beta also z = r (16n), <r,z> and <z,q> partials (24n)
    return kernel_bytes(H, KID_SPMV_DOT, 0, flexible) + kernel_bytes(H, KID_CG_UPDATE, 0, flexible) +
           (flexible ? 40.0 * H.n : 0.0);
  double b = kernel_bytes(H, KID_SPMV_DOT, 0, flexible) + kernel_bytes(H, KID_CG_UPDATE, 0, flexible) +
             kernel_bytes(H, KID_XPAY, 0, flexible) + kernel_bytes(H, KID_COARSE, nl - 1, flexible);
  for (int l = 0; l < nl - 1; ++l) {
    const double n = H.lv[l].n;
    const double v = H.fp32() ? 4.0 : 8.0;
    b += kernel_bytes(H, KID_PRE, l, flexible) + kernel_bytes(H, KID_RESTRICT, l, flexible) +
         kernel_bytes(H, KID_PROLONG, l, flexible) + H.prm.nu_post * kernel_bytes(H, KID_POST, l, flexible);
    b += (H.prm.nu_pre - 1) * (kernel_bytes(H, KID_PRE, l, flexible) + 2.0 * v * n);
  }
  return b;
}

void set_instrument(Hierarchy& H, int kid, int level) {
  if (H.inst.ev.empty()) {
    H.inst.ev.resize(2 * 8192);
    for (auto& e : H.inst.ev) AMG_HIP(hipEventCreate(&e));
    H.inst.was_done.alloc(8192);
  }
  H.inst.kernel = kid;
  H.inst.level = level;
  H.inst.used = 0;
}

void read_instrument(Hierarchy& H, int* launches, double* total_ms, double* min_ms, double* max_ms) {
  double tot = 0.0, mn = 1e300, mx = 0.0;
  std::vector<int> done(H.inst.used);
  if (H.inst.used) {
    AMG_HIP(hipEventSynchronize(H.inst.ev[2 * H.inst.used - 1]));
    AMG_HIP(hipMemcpy(done.data(), H.inst.was_done.p, sizeof(int) * H.inst.used, hipMemcpyDeviceToHost));
  }
  int working = 0;
  for (int i = 0; i < H.inst.used; ++i) {
    if (done[i]) continue;
    float ms = 0.f;
    AMG_HIP(hipEventElapsedTime(&ms, H.inst.ev[2 * i], H.inst.ev[2 * i + 1]));
    tot += ms;
    mn = std::min(mn, (double)ms);
    mx = std::max(mx, (double)ms);
    ++working;
  }
  *launches = working;
  *total_ms = tot;
  *min_ms = working ? mn : 0.0;
  *max_ms = mx;
}

void apply_vcycle(Hierarchy& H, const double* d_r, double* d_z, hipStream_t s) {
  // In place: the two-sweep level 0 of the FP64 cycle and the dense product of a
  // single level gather r while other workgroups write z, so they read a copy
  // (the four-sweep level 0 reads r only at the row it writes; the FP32 cycle
  // rounds r into a buffer of its own).
  if (d_z == d_r && H.prm.precondition && (H.lv.size() == 1 || (H.lf == 0 && !H.fp32()))) {
    hipLaunchKernelGGL(k_copy_z, dim3(vec_grid(H.n)), dim3(kBlock), 0, s, H.n, d_r, H.z.p, (const int*)nullptr);
    d_r = H.z.p;
  }
  CycleArgs a{d_r, d_z, nullptr, nullptr, nullptr, 0, 0};
  vcycle(H, a, s);
  AMG_HIP(hipGetLastError());
}

void pattern_grad(Hierarchy& H, const double* d_lam, const double* d_x, double* d_g, hipStream_t s) {
  Level& L = H.lv[0];
  const int grid = (int)(((int64_t)L.n + kBlock / 8 - 1) / (kBlock / 8));
  hipLaunchKernelGGL(k_pattern_grad, dim3(grid), dim3(kBlock), 0, s, L.n, L.rp.p, L.ci.p, d_lam, d_x, d_g);
  AMG_HIP(hipGetLastError());
}

template <class T>
void launch_cg_update(Hierarchy& H, const SolveWork& w, int n, const double* p, const double* pa, int npa, int tot,
                      double* pu, int par, hipStream_t s) {
  Level& L0 = H.lv[0];
  const dim3 g(vec_grid(n)), b(kBlock);
  switch (x0_mode(H)) {
    case X0_SMOOTHED:
      hipLaunchKernelGGL((k_cg_update<X0_SMOOTHED, T>), g, b, 0, s, n, w.r, p, w.q, Bufs<T>::sw(L0),
                         Bufs<T>::x(L0), w.ctl, pa, npa, tot, pu, par);
      break;
    case X0_COPY:
      hipLaunchKernelGGL((k_cg_update<X0_COPY, T>), g, b, 0, s, n, w.r, p, w.q, (const T*)nullptr,
                         Bufs<T>::x(L0), w.ctl, pa, npa, tot, pu, par);
      break;
    default:
      hipLaunchKernelGGL((k_cg_update<X0_NONE, T>), g, b, 0, s, n, w.r, p, w.q, (const T*)nullptr, (T*)nullptr,
                         w.ctl, pa, npa, tot, pu, par);
  }
}

template <class T>
void launch_sw_mul(Hierarchy& H, const SolveWork& w, int n, hipStream_t s) {
  Level& L0 = H.lv[0];
  const X0Mode m = x0_mode(H);
  if (m == X0_NONE) return;
  hipLaunchKernelGGL((k_sw_mul<T>), dim3(vec_grid(n)), dim3(kBlock), 0, s, n,
                     m == X0_COPY ? (const T*)nullptr : Bufs<T>::sw(L0), w.r, Bufs<T>::x(L0), &w.ctl->done);
}

void read_ctl(const SolveWork& w, hipStream_t s) {
  AMG_HIP(hipMemcpyAsync(w.h_ctl, w.ctl, sizeof(Ctl), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
}

// Captures the launches made by `body` on stream s into an executable graph;
// a failure ends the capture before the error propagates.
template <class F>
void capture_graph_impl(hipStream_t s, hipGraphExec_t& ex, F&& body) {
  hipGraph_t g = nullptr;
  AMG_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed));
  try {
    body();
  } catch (...) {
    (void)hipStreamEndCapture(s, &g);
    if (g) (void)hipGraphDestroy(g);
    throw;
  }
  AMG_HIP(hipStreamEndCapture(s, &g));
  const hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) {
    ex = nullptr;
    throw Error(AMG_ERR_HIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
  }
}

void capture_graph(hipStream_t s, hipGraphExec_t& ex, const std::function<void()>& body) {
  capture_graph_impl(s, ex, body);
}

// Library stream and join events for graph solves.
void graph_stream(Hierarchy& H) {
  if (!H.gr.gs) {
    AMG_HIP(hipStreamCreateWithFlags(&H.gr.gs, hipStreamNonBlocking));
    AMG_HIP(hipEventCreateWithFlags(&H.gr.ev_in, hipEventDisableTiming));
    AMG_HIP(hipEventCreateWithFlags(&H.gr.ev_out, hipEventDisableTiming));
  }
}

// A reduction as its consumer reads it: nv arrays of np partials from p on.
struct Sums {
  double* p;
  int np, nv;
};

// Where the consumers find the sums of a solve: the partials (folded solves),
// or their totals at `out`, in the order given (at most four).
void totals_at(bool tot, std::initializer_list<Sums*> sums, double* out) {
  if (!tot) return;
  for (Sums* s : sums) {
    *s = Sums{out, 1, s->nv};
    out += s->nv;
  }
}

// Launches k_sum for the sums where the solve takes totals, then totals_at.
void total(bool tot, std::initializer_list<Sums*> sums, double* out, const int* stop, hipStream_t st) {
  if (!tot) return;
  SumArgs a{};
  int m = 0;
  for (Sums* s : sums)
    for (int v = 0; v < s->nv; ++v, ++m) {
      a.src[m] = s->p + (int64_t)v * s->np;
      a.np[m] = s->np;
    }
  hipLaunchKernelGGL(k_sum, dim3(m), dim3(kFinBlock), 0, st, a, out, stop);
  totals_at(tot, sums, out);
}

amg_status pcg_solve(Hierarchy& H, const SolveOpts& o, const SolveWork& w, const double* d_b, double* d_x,
                     double tol, amg_info* info, hipStream_t caller) {
  // hierarchies that fit one compute unit: the whole solve in one launch
  if (o.fused_small && H.inst.kernel < 0 && small_solve_ok(H))
    return pcg_solve_small(H, o, w, d_b, d_x, tol, info, caller);
  auto t0 = std::chrono::steady_clock::now();
  Level& L0 = H.lv[0];
  const int n = H.n;
  const bool multi = H.lv.size() > 1;
  // automatic: flexible whenever the preconditioner is not a fixed symmetric
  // operator (FP32 cycle, or unequal pre/post sweep counts)
  const int flexible = o.flexible < 0 ? ((H.fp32() || H.prm.nu_pre != H.prm.nu_post) ? 1 : 0) : o.flexible;
  const bool graphs = w.graphs && o.use_graphs && H.inst.kernel < 0;
  hipStream_t s = caller;
  if (graphs) {
    graph_stream(H);
    AMG_HIP(hipEventRecord(H.gr.ev_in, caller));
    AMG_HIP(hipStreamWaitEvent(H.gr.gs, H.gr.ev_in, 0));
    s = H.gr.gs;
    if (H.gr.key_flex != flexible || H.gr.key_w != 1) {
      H.gr.reset();
      H.gr.key_flex = flexible;
      H.gr.key_w = 1;
    }
  }
  Ctl* ctl = w.ctl;
  const int* done = &ctl->done;      // (device addresses)
  const int* gate = &ctl->gate[0];
  double* part = w.partials;
  const int gv = vec_grid(n);
  const int gu = vec_grid(n);
  // the partials of the product (part), the update (pu) and the V-cycle (pz)
  // are summed by the kernels that need them (fold_load)
  const int64_t region = partials_region(H);
  double* pu = part + region;
  double* pz = part + 2 * region;
  const bool tot = region > kFoldMax, early = tot && n >= kEarlyStop;
  double* pt = part + 4 * region;   // totals: product; update and V-cycle
  Sums start{pz, 0, 1};             // <r, z> as the first product after a (re)start reads it
  int npz = 0;
  // plain CG with the standard beta: z = r needs no copy and <r, z> = ||r||^2
  // no sum of its own (10^7 unknowns: the copy and the dots were 63 of 320 us
  // per iteration, the unused x0 = sw o r another 34)
  const bool plain = !H.prm.precondition && !flexible;
  double* zv = plain ? w.r : w.z;
  hipLaunchKernelGGL(k_cg_init, dim3(gu), dim3(kBlock), 0, s, n, d_b, w.r, d_x, pz);
  hipLaunchKernelGGL(k_fin_init, dim3(1), dim3(kFinBlock), 0, s, ctl, pz, gu, tol, o.maxiter, flexible, d_x);
  AMG_HIP(hipGetLastError());
  // search directions alternate between two buffers (the fused direction
  // update writes the new p while neighbours still gather the old one)
  double* pb[2] = {w.p, w.z2};
  int cur = 0;
  // one PCG iteration: p = z + beta p and q = A p; alpha; x, r update; z = M^-1 r, beta
  auto iteration = [&](int first, int c, hipStream_t st) {
    const int nv = flexible ? 2 : 1;
    // what the product reads: the last update's and V-cycle's sums
    Sums u{pu, gu, 1}, z{pz, npz, nv};
    if (plain) {
      totals_at(tot, {&u}, pt + 1);
      z = u;
    } else {
      totals_at(tot, {&u, &z}, pt + 1);
    }
    if (first) z = start;
    int np;
    {
      InstScope is(H, KID_SPMV_DOT, 0, st, done);
      np = sweep(L0.shA, n, L0.arp(), L0.aci(),
                 OpSpmvXpay{L0.av(), zv, pb[c], pb[c ^ 1], w.q, ctl, z.p, u.p, z.np, u.np, z.nv, tot, first, c}, done, part,
                 st);
    }
    Sums a{part, np, 1};
    total(tot, {&a}, pt, gate, st);
    {
      InstScope is(H, KID_CG_UPDATE, 0, st, gate);
      if (H.fp32()) launch_cg_update<float>(H, w, n, pb[c ^ 1], a.p, a.np, tot, pu, c, st);
      else launch_cg_update<double>(H, w, n, pb[c ^ 1], a.p, a.np, tot, pu, c, st);
    }
    u = Sums{pu, gu, 1};
    if (early) hipLaunchKernelGGL(k_sum_update, dim3(1), dim3(kFinBlock), 0, st, pu, gu, pt + 1, ctl, c);
    if (!plain) {
      vcycle(H, CycleArgs{w.r, w.z, w.q, done, pz, nv, multi ? 1 : 0}, st);
      z = Sums{pz, npz, nv};
      if (early) total(tot, {&z}, pt + 2, done, st);
      else total(tot, {&u, &z}, pt + 1, done, st);
    } else if (!early) {
      total(tot, {&u}, pt + 1, done, st);
    }
  };
  // two iterations captured once per direction-buffer parity and replayed
  auto pair = [&](int c) {
    hipGraphExec_t& ex = H.gr.exec[c];
    if (!ex) capture_graph(s, ex, [&] {
        iteration(0, c, s);
        iteration(0, c ^ 1, s);
      });
    AMG_HIP(hipGraphLaunch(ex, s));
  };
  int restarts = 0;
  amg_status st = AMG_OK;
  for (;;) {
    // (re)start: z = M^-1 r, rz = <r, z>; the first direction is p = z
    if (multi) {
      if (H.fp32()) launch_sw_mul<float>(H, w, n, s);
      else launch_sw_mul<double>(H, w, n, s);
    }
    // (plain CG starts from the partials of ||r||^2 that the start or the true
    // residual left in pz)
    npz = plain ? (restarts ? L0.shA.grid : gu) : vcycle(H, CycleArgs{w.r, w.z, w.q, done, pz, 1, multi ? 1 : 0}, s);
    start = Sums{pz, npz, 1};
    total(tot, {&start}, pt + 1, done, s);
    int first = 1;
    // Iterations are queued in chunks; between chunks the host reads the
    // control block and sizes the next chunk from the observed decay of
    // ||r||^2 so that few iterations are queued past convergence (those
    // return at once on the done flag).
    int chunk = o.check_every > 0 ? o.check_every : 4;
    int it_prev = -1;
    double rr_prev = 0.0;
    for (;;) {
      int left = chunk;
      if (first) {
        iteration(1, cur, s);
        cur ^= 1;
        first = 0;
        --left;
      }
      if (graphs)
        for (; left >= 2; left -= 2) pair(cur);
      for (; left > 0; --left) {
        iteration(0, cur, s);
        cur ^= 1;
      }
      hipLaunchKernelGGL(k_fin_chunk, dim3(1), dim3(kFinBlock), 0, s, ctl, pu, gu, cur ^ 1);
      AMG_HIP(hipGetLastError());
      read_ctl(w, s);
      if (w.h_ctl->done) break;
      if (o.check_every <= 0) {
        const Ctl& c = *w.h_ctl;
        if (it_prev < 0) {  // decay measured from ||r_0||^2 = ||b||^2
          it_prev = 0;
          rr_prev = c.bb;
        }
        int next = 4;
        if (c.thresh <= 0.0) {
          next = 32;
        } else if (c.iters > it_prev && rr_prev > 0.0 && c.rr > 0.0) {
          const double rate = std::log(c.rr / rr_prev) / (double)(c.iters - it_prev);
          if (rate < -1e-3) next = (int)std::min(64.0, std::ceil(std::log(c.thresh / c.rr) / rate));
        }
        it_prev = c.iters;
        rr_prev = c.rr;
        next = std::min(next, std::max(1, c.maxiter - c.iters));
        chunk = std::max(1, std::min(next, 32));
      }
    }
    const int state = w.h_ctl->state;
    if (state == 3) break;  // b = 0
    if (state < 0) {
      st = AMG_ERR_BREAKDOWN;
      break;
    }
    // true residual r = b - A x
    const int np = sweep(L0.shA, n, L0.arp(), L0.aci(), OpTrueResid{L0.av(), d_x, d_b, w.r}, nullptr, pz, s);
    hipLaunchKernelGGL(k_fin_trr, dim3(1), dim3(kFinBlock), 0, s, ctl, pz, np);
    read_ctl(w, s);
    const Ctl& c = *w.h_ctl;
    if (c.trr <= c.thresh) {
      st = AMG_OK;
      break;
    }
    if (state == 1 && restarts < 5 && c.iters < c.maxiter) {
      ++restarts;
      hipLaunchKernelGGL(k_ctl_restart, dim3(1), dim3(1), 0, s, ctl);
      continue;
    }
    st = AMG_NOT_CONVERGED;
    break;
  }
  if (graphs) {
    AMG_HIP(hipEventRecord(H.gr.ev_out, s));
    AMG_HIP(hipStreamWaitEvent(caller, H.gr.ev_out, 0));
  }
  const Ctl& c = *w.h_ctl;
  if (info) {
    info->iters = c.iters;
    info->status = st;
    info->restarts = restarts;
    info->rel_resid = c.state == 3 ? 0.0 : (c.bb > 0 ? std::sqrt(c.trr / c.bb) : 0.0);
    if (st == AMG_ERR_BREAKDOWN) info->rel_resid = NAN;
    info->cache_event = H.cache_event;
    info->setup_ms = H.setup_ms;
    info->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  return st;
}

// Right-preconditioned BiCGSTAB (van der Vorst, 1992), the paper's default
// Krylov method (Section 2.1), from x0 = 0 with shadow residual r^ = b.
// One iteration, every scalar formed on the device:
//   p = r + beta (p - omega v)        k_bi_dir   (p = r after a (re)start)
//   y = M^-1 p                        V-cycle
//   v = A y, <r^, v>                  sweep      -> alpha = rho / <r^, v>
//   x += alpha y, s = r - alpha v     k_bi_half  -> ||s|| test, iteration count
//   z = M^-1 s                        V-cycle
//   t = A z, <s, t>, <t, t>           sweep      -> omega
//   x += omega z, r = s - omega t     k_bi_full  -> ||r|| test, rho, beta
// Stopping, verification and restarts follow pcg_solve.
amg_status bicgstab_solve(Hierarchy& H, const SolveOpts& o, const double* d_b, double* d_x, double tol,
                          amg_info* info, hipStream_t caller) {
  auto t0 = std::chrono::steady_clock::now();
  Level& L0 = H.lv[0];
  const int n = H.n;
  const bool graphs = o.use_graphs && H.inst.kernel < 0;
  if (!H.rh.p) {
    H.rh.alloc(n);
    H.bv.alloc(n);
    H.by.alloc(n);
    H.bs.alloc(n);
    H.bt2.alloc(n);
    AMG_HIP(hipMemsetAsync(H.bv.p, 0, H.bv.bytes(), caller));
  }
  hipStream_t s = caller;
  if (graphs) {
    graph_stream(H);
    AMG_HIP(hipEventRecord(H.gr.ev_in, caller));
    AMG_HIP(hipStreamWaitEvent(H.gr.gs, H.gr.ev_in, 0));
    s = H.gr.gs;
  }
  Ctl* ctl = H.ctl.p;
  const int* done = &ctl->done;      // (device addresses)
  const int* gate = &ctl->gate[0];
  double* part = H.partials.p;
  double* r = H.r.p;
  double* p = H.p.p;
  double* z = H.z.p;
  double* rh = H.rh.p;
  double* v = H.bv.p;
  double* y = H.by.p;
  double* sv = H.bs.p;
  double* t = H.bt2.p;
  // no preconditioner: y = p and z = s are the same vectors (no copies)
  const bool prec = H.prm.precondition != 0;
  if (!prec) {
    y = p;
    z = sv;
  }
  const int gv = vec_grid(n), gu = vec_grid(n);
  const int64_t region = partials_region(H);
  double* ps = part + region;       // <s, s>
  double* pt = part + 2 * region;   // <s, t>, <t, t>
  double* pf = part + 4 * region;   // <r, r>, <r^, r>
  const bool tot = region > kFoldMax, early = tot && n >= kEarlyStop;
  double* ptot = part + 6 * region;  // totals
  Sums full{pf, gu, 2};             // as the direction update reads them
  totals_at(tot, {&full}, ptot + 4);
  hipLaunchKernelGGL(k_bi_init, dim3(gv), dim3(kBlock), 0, s, n, d_b, r, rh, d_x, part);
  hipLaunchKernelGGL(k_bfin_init, dim3(1), dim3(kFinBlock), 0, s, ctl, part, gv, tol, o.maxiter, d_x);
  AMG_HIP(hipGetLastError());
  // with a multilevel cycle the vector kernels also write what the V-cycle
  // that follows them starts from
  const X0Mode x0m = x0_mode(H);
  const bool x0w = x0m != X0_NONE, smoothed = x0m == X0_SMOOTHED;
  auto launch_dir = [&](int first, hipStream_t st) {
    Level& L0c = H.lv[0];
    if (H.fp32())
      hipLaunchKernelGGL(k_bi_dir<float>, dim3(gu), dim3(kBlock), 0, st, n, r, v, p,
                         smoothed ? Bufs<float>::sw(L0c) : nullptr,
                         x0w ? Bufs<float>::x(L0c) : nullptr, ctl, first, full.p, full.np, tot);
    else
      hipLaunchKernelGGL(k_bi_dir<double>, dim3(gu), dim3(kBlock), 0, st, n, r, v, p,
                         smoothed ? Bufs<double>::sw(L0c) : nullptr,
                         x0w ? Bufs<double>::x(L0c) : nullptr, ctl, first, full.p, full.np, tot);
  };
  auto launch_half = [&](const Sums& a, hipStream_t st) {
    Level& L0c = H.lv[0];
    if (H.fp32())
      hipLaunchKernelGGL(k_bi_half<float>, dim3(gu), dim3(kBlock), 0, st, n, y, r, v, sv,
                         smoothed ? Bufs<float>::sw(L0c) : nullptr,
                         x0w ? Bufs<float>::x(L0c) : nullptr, ctl, a.p, a.np, tot, ps);
    else
      hipLaunchKernelGGL(k_bi_half<double>, dim3(gu), dim3(kBlock), 0, st, n, y, r, v, sv,
                         smoothed ? Bufs<double>::sw(L0c) : nullptr, x0w ? Bufs<double>::x(L0c) : nullptr, ctl, a.p,
                         a.np, tot, ps);
  };
  auto iteration = [&](int first, hipStream_t st) {
    launch_dir(first, st);
    if (prec) vcycle(H, CycleArgs{p, y, nullptr, gate, part, 0, x0w ? 1 : 0}, st);
    int np;
    {
      InstScope is(H, KID_SPMV_DOT, 0, st, gate);
      np = sweep(L0.shA, n, L0.arp(), L0.aci(), OpSpmvDots<1>{L0.av(), y, v, rh}, gate, part, st);
    }
    Sums a{part, np, 1};
    total(tot, {&a}, ptot, gate, st);
    launch_half(a, st);
    if (early) hipLaunchKernelGGL(k_sum_half, dim3(1), dim3(kFinBlock), 0, st, ps, gu, ptot + 1, ctl);
    if (prec) vcycle(H, CycleArgs{sv, z, nullptr, gate + 1, part, 0, x0w ? 1 : 0}, st);
    {
      InstScope is(H, KID_SPMV_DOT, 0, st, gate + 1);
      np = sweep(L0.shA, n, L0.arp(), L0.aci(), OpSpmvDots<2>{L0.av(), z, t, sv}, gate + 1, pt, st);
    }
    Sums h{ps, gu, 1}, tt{pt, np, 2}, f{pf, gu, 2};
    if (early) {
      totals_at(tot, {&h}, ptot + 1);
      total(tot, {&tt}, ptot + 2, gate + 1, st);
    } else {
      total(tot, {&h, &tt}, ptot + 1, gate + 1, st);
    }
    hipLaunchKernelGGL(k_bi_full, dim3(gu), dim3(kBlock), 0, st, n, z, sv, t, rh, r, ctl, h.p, h.np, tt.p, tt.np, tot, pf);
    total(tot, {&f}, ptot + 4, done, st);
  };
  int restarts = 0;
  amg_status st = AMG_OK;
  for (;;) {
    int first = 1;
    int chunk = o.check_every > 0 ? o.check_every : 2;
    int it_prev = -1;
    double rr_prev = 0.0;
    for (;;) {
      int left = chunk;
      if (first) {
        iteration(1, s);
        first = 0;
        --left;
      }
      if (graphs && left > 0) {
        if (!H.gr.bexec) capture_graph(s, H.gr.bexec, [&] { iteration(0, s); });
        for (; left > 0; --left) AMG_HIP(hipGraphLaunch(H.gr.bexec, s));
      }
      for (; left > 0; --left) iteration(0, s);
      hipLaunchKernelGGL(k_bfin_chunk, dim3(1), dim3(kFinBlock), 0, s, ctl, pf, gu);
      AMG_HIP(hipGetLastError());
      read_ctl(H, s);
      if (H.h_ctl->done) break;
      if (o.check_every <= 0) {
        // chunk sized from the observed decay of the residual norm, as in PCG
        const Ctl& c = *H.h_ctl;
        if (it_prev < 0) {
          it_prev = 0;
          rr_prev = c.bb;
        }
        int next = 2;
        if (c.thresh <= 0.0) {
          next = 16;
        } else if (c.iters > it_prev && rr_prev > 0.0 && c.rr > 0.0) {
          const double rate = std::log(c.rr / rr_prev) / (double)(c.iters - it_prev);
          if (rate < -1e-3) next = (int)std::min(32.0, std::ceil(std::log(c.thresh / c.rr) / rate));
        }
        it_prev = c.iters;
        rr_prev = c.rr;
        next = std::min(next, std::max(1, c.maxiter - c.iters));
        chunk = std::max(1, std::min(next, 16));
      }
    }
    const int state = H.h_ctl->state;
    if (state == 3) break;  // b = 0
    if (state < 0) {
      st = AMG_ERR_BREAKDOWN;
      break;
    }
    const int np = sweep(L0.shA, n, L0.arp(), L0.aci(), OpTrueResid{L0.av(), d_x, d_b, r}, nullptr, part, s);
    hipLaunchKernelGGL(k_fin_trr, dim3(1), dim3(kFinBlock), 0, s, ctl, part, np);
    read_ctl(H, s);
    const Ctl& c = *H.h_ctl;
    if (c.trr <= c.thresh) {
      st = AMG_OK;
      break;
    }
    if (state == 1 && restarts < 5 && c.iters < c.maxiter) {
      ++restarts;
      hipLaunchKernelGGL(k_bi_restart, dim3(1), dim3(1), 0, s, ctl);
      hipLaunchKernelGGL(k_copy_z, dim3(gv), dim3(kBlock), 0, s, n, r, rh, (const int*)nullptr);
      continue;
    }
    st = AMG_NOT_CONVERGED;
    break;
  }
  if (graphs) {
    AMG_HIP(hipEventRecord(H.gr.ev_out, s));
    AMG_HIP(hipStreamWaitEvent(caller, H.gr.ev_out, 0));
  }
  const Ctl& c = *H.h_ctl;
  if (info) {
    info->iters = c.iters;
    info->status = st;
    info->restarts = restarts;
    info->rel_resid = c.state == 3 ? 0.0 : (c.bb > 0 ? std::sqrt(c.trr / c.bb) : 0.0);
    if (st == AMG_ERR_BREAKDOWN) info->rel_resid = NAN;
    info->cache_event = H.cache_event;
    info->setup_ms = H.setup_ms;
    info->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  return st;
}

}  // namespace amg
