// Whole-solve PCG in one workgroup, for hierarchies small enough to live in
// one compute unit: two levels (the fine level and a dense coarsest level),
// at most 1024 fine rows.  The per-kernel path launches about twenty kernels
// per iteration, so a 1024-unknown solve is bound by launch and
// synchronisation latency, not by bytes.  Here one workgroup of 512 threads
// (thread i owns fine rows i and i + 512) runs every iteration, restart and the final
// true-residual check in a single launch:
//   - the CG vectors and the cycle vectors live in LDS, so every gather of
//     a sweep is an LDS read;
//   - each thread keeps its rows of A_0 in registers for the whole solve
//     (A_0 is applied three times per iteration);
//   - P_0 and R_0 are staged in LDS once per solve; R_0 is applied with a
//     group of lanes per coarse row;
//   - the explicit coarse inverse lives in registers for the whole solve: a
//     thread owns two adjacent rows of a block of columns (28 of them in 112
//     registers, which holds all of an inverse of up to about 165 unknowns;
//     a larger one's other columns are read from L2 in every cycle), and the
//     block sums are added per row in block order.  Reading all of it from L2
//     bounded the solve by the latency of its load rounds (68 of the kernel's
//     160 us for 18 iterations with a 150 x 150 inverse): 32^2 Poisson to
//     1e-10 187 us then, 150 so and 145 with the pre-smoothing done where r
//     is written and the last two steps of a wave's sum in registers.  A_0's columns are kept two to a register
//     and b is read again where it is needed, which leaves room for 28
//     columns without a spill.  16 waves of half as many columns each were
//     slower (222 us, with the inverse in L2): every barrier costs more;
//   - dot products are fixed-order block reductions (wave butterfly, then the
//     8 wave sums in order), so a solve is bitwise reproducible.
// The method is the one of pcg_solve: PCG from x0 = 0, damped-Jacobi (or L1)
// V(1,1) cycle with R = P^T and the exact coarse solve, recursive-residual
// stopping, true-residual verification with at most 5 restarts, flexible
// beta = -<z, q>/<p, q> when requested.  Rows are summed in stored order and
// q = A p is formed directly.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <vector>

#include "amg_internal.hpp"

namespace amg {
namespace {

constexpr int kST = 512;         // threads of the workgroup
constexpr int kSR = 2;           // fine rows per thread (rows t and t + kST)
constexpr int kSN = kST * kSR;   // largest fine level
constexpr int kSRow = 8;         // entries per row of A_0
constexpr int kSCoarse = 256;    // largest padded coarsest level
constexpr int kSPCap = 3200;     // entries of P_0 (and of R_0 = P_0^T) staged in LDS
constexpr int kSBlocks = 8;      // most column blocks of the inverse
constexpr int kSHold = 28;       // inverse columns a thread holds in registers (a multiple of 4)
constexpr int kSCols = 4;        // inverse columns per step beyond those (loads in flight)

struct SmallArgs {
  int n, nc, m, lgR, maxiter, flexible;
  double tol;
  const int* arp;
  const int* aci;
  const double* av;
  const double* sw;
  const int* prp;
  const int* pci;
  const double* pv;
  const int* rrp;
  const int* rci;
  const double* rv;
  const double* inv;
  const double* b;
  double* x;
  Ctl* ctl;
};

// Keeps the compiler from moving memory operations across this point: the
// matrix loads of a phase are loop-invariant, and hoisting all of them out
// of the iteration loop would keep every phase's operands live in registers
// at once.
__device__ inline void phase_fence() { asm volatile("" ::: "memory"); }

// Returns v through an empty asm statement: the compiler cannot treat values
// derived from it as loop-invariant, so the loads they address stay in their
// phase instead of being hoisted out of the iteration loop.
__device__ inline int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// DPP move of a double within rows of 16 lanes (pattern `ctrl`).
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// v of this lane plus v of lane ^ STEP (16 or 32): swapping the odd rows
// (the upper half) of one copy with the even rows (the lower half) of another
// leaves both partners' values side by side in every lane.
template <int STEP>
__device__ inline double swap_sum(double v) {
  const unsigned lo = __double2loint(v), hi = __double2hiint(v);
  if constexpr (STEP == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
  }
}

// Sum over the wavefront, every lane gets the same bits: partner sums within
// quads (lane ^ 1, lane ^ 2), then the mirrored half row and row (lane i with
// 7 - i and 15 - i of its group), then across rows (lane ^ 16, lane ^ 32, by
// register swaps: an LDS permutation costs a round trip each).
// Each step adds two equal-rank partial sums, so all lanes agree.
__device__ inline double wave_sum_fast(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  v = swap_sum<16>(v);
  return swap_sum<32>(v);
}

// Sum of v over the workgroup in a fixed order; every thread gets the total.
// `red` must not be reused before the next barrier.
__device__ inline double wg_sum(double v, double* red) {
  v = wave_sum_fast(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = red[0];
#pragma unroll
  for (int k = 1; k < kST / 64; ++k) s += red[k];
  return s;
}

__global__ void __launch_bounds__(kST) k_pcg_small(SmallArgs a) {
  __shared__ double s_r[kSN], s_z[kSN], s_p[kSN], s_q[kSN], s_xc[kSN], s_rc[kSN];
  __shared__ double s_x1[kSCoarse];
  __shared__ __align__(16) double s_b1[kSCoarse + 4 * kSBlocks];  // zeros past n_c
  __shared__ double s_gp[2 * kST + kSBlocks];  // at most kST / pairs blocks of 2 pairs rows
  __shared__ double s_red[4][kST / 64];
  __shared__ int s_prp[kSN + 1], s_rrp[kSCoarse + 1];
  __shared__ int s_pci[kSPCap], s_rci[kSPCap];
  __shared__ double s_pv[kSPCap], s_rv[kSPCap];
  const int t = threadIdx.x;
  // P_0 and R_0 into LDS (their entry counts are at most kSPCap)
  const int pnz = a.prp[a.n];
  for (int i = t; i <= a.n; i += kST) s_prp[i] = a.prp[i];
  for (int i = t; i <= a.nc; i += kST) s_rrp[i] = a.rrp[i];
  for (int k = t; k < pnz; k += kST) {
    s_pci[k] = a.pci[k];
    s_pv[k] = a.pv[k];
    s_rci[k] = a.rci[k];
    s_rv[k] = a.rv[k];
  }
  // this thread's rows t + q kST: their rows of A_0 in registers (indices
  // clamped into the row; entries past the row's length are masked out of
  // every sum), their smoother weights and iterate
  int row[kSR], na[kSR], acol[kSR][kSRow / 2];   // two 16-bit columns per word
  bool own[kSR];
  double aval[kSR][kSRow], swi[kSR], xi[kSR];
#pragma unroll
  for (int q = 0; q < kSR; ++q) {
    own[q] = t + q * kST < a.n;
    row[q] = own[q] ? t + q * kST : a.n - 1;
    const int ka = a.arp[row[q]];
    na[q] = own[q] ? a.arp[row[q] + 1] - ka : 0;
#pragma unroll
    for (int j = 0; j < kSRow; ++j) {
      const int k = ka + min(j, max(na[q] - 1, 0));
      if (j & 1) acol[q][j / 2] |= a.aci[k] << 16;
      else acol[q][j / 2] = a.aci[k];
      aval[q][j] = a.av[k];
    }
    swi[q] = a.sw[row[q]];
    xi[q] = 0.0;
  }
  __syncthreads();
  // row q of A_0 applied to an LDS vector, summed in stored order
  auto arow = [&](int q, const double* v) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kSRow; ++j) {
      const int cw = opaque(acol[q][j / 2]);       // unpacked here, not kept unpacked
      const double pr = aval[q][j] * v[j & 1 ? cw >> 16 : cw & 0xffff];
      s = j < na[q] ? s + pr : s;
    }
    return s;
  };
  const int gR = 1 << a.lgR;
  const int rrow = t >> a.lgR, rl = t & (gR - 1);
  // coarse product: thread t takes rows 2 gp, 2 gp + 1 of the columns
  // [gc, gc + Lc) (one 16-byte load per column, coalesced over gp).  Lc is a
  // multiple of 4, the same for every block; columns past n_c count as zeros
  // (s_b1 is zero there), and the padded order m covers an odd n_c's last pair.
  const int pairs = (a.nc + 1) >> 1;
  const int nblk = min(kST / pairs, kSBlocks);
  const int Lc = ((a.nc + 4 * nblk - 1) / (4 * nblk)) * 4;
  const int gb = min(t / pairs, nblk - 1), gp = t % pairs, gc = gb * Lc;
  const bool gown = t < nblk * pairs;
  const double* ginv = a.inv + 2 * gp;
  double2 hv[kSHold];
#pragma unroll
  for (int j = 0; j < kSHold; ++j) {
    hv[j] = *reinterpret_cast<const double2*>(ginv + (int64_t)min(gc + j, a.nc - 1) * a.m);
    if (gc + j >= a.nc) hv[j] = double2{0.0, 0.0};
  }
  for (int i = a.nc + t; i < kSCoarse + 4 * kSBlocks; i += kST) s_b1[i] = 0.0;

  // z = M^-1 r (s_r, and s_xc = sw o r by its writer, -> s_z); returns <r, z>, and <z, q> in zq when flexible
  auto vcycle = [&](double& zq) -> double {
#pragma unroll
    for (int q = 0; q < kSR; ++q)                  // residual of the pre-smoothed zero
      if (own[q]) s_rc[row[q]] = s_r[row[q]] - arow(q, s_xc);
    __syncthreads();
    {                                              // b_1 = R r_c, gR lanes per coarse row
      double s = 0.0;
      if (rrow < a.nc) {
        const int k1 = s_rrp[rrow + 1];
        int k = s_rrp[rrow] + rl;
        for (; k + 3 * gR < k1; k += 4 * gR) {     // four entries per step, summed in order
          const double p0 = s_rv[k] * s_rc[s_rci[k]];
          const double p1 = s_rv[k + gR] * s_rc[s_rci[k + gR]];
          const double p2 = s_rv[k + 2 * gR] * s_rc[s_rci[k + 2 * gR]];
          const double p3 = s_rv[k + 3 * gR] * s_rc[s_rci[k + 3 * gR]];
          s = s + p0;
          s = s + p1;
          s = s + p2;
          s = s + p3;
        }
        for (; k < k1; k += gR) s = s + s_rv[k] * s_rc[s_rci[k]];
      }
      for (int o = 1; o < gR; o <<= 1) s += __shfl_xor(s, o, 64);
      if (rrow < a.nc && rl == 0) s_b1[rrow] = s;
    }
    __syncthreads();
    {                                              // x_1 = A_c^-1 b_1
      phase_fence();
      double acc0 = 0.0, acc1 = 0.0;
      auto add = [&](const double2& v, double bj) {
        const double p0 = v.x * bj, p1 = v.y * bj;
        acc0 = acc0 + p0;
        acc1 = acc1 + p1;
      };
#pragma unroll
      for (int j = 0; j < kSHold; j += 4) {
        if (j < Lc) {                              // the same for every thread
#pragma unroll
          for (int u = 0; u < 4; ++u) add(hv[j + u], s_b1[gc + j + u]);
        }
      }
      const int jend = opaque(Lc);
      for (int j0 = kSHold; j0 < jend; j0 += kSCols) {
        double2 v[kSCols];                         // columns past the matrix: its last one, times zero
#pragma unroll
        for (int u = 0; u < kSCols; ++u)
          v[u] = *reinterpret_cast<const double2*>(ginv + (int64_t)min(gc + j0 + u, a.nc - 1) * a.m);
#pragma unroll
        for (int u = 0; u < kSCols; ++u)
          if (j0 + (u & ~3) < jend) add(v[u], s_b1[gc + j0 + u]);
      }
      if (gown) {
        s_gp[gb * a.nc + 2 * gp] = acc0;
        if (2 * gp + 1 < a.nc) s_gp[gb * a.nc + 2 * gp + 1] = acc1;
      }
      __syncthreads();
      if (t < a.nc) {                              // the column blocks' sums in block order
        double s = s_gp[t];
        for (int q = 1; q < nblk; ++q) s += s_gp[q * a.nc + t];
        s_x1[t] = s;
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSR; ++q) {                // x_c += P x_1
      if (!own[q]) continue;
      const int k1 = s_prp[row[q] + 1];
      double s = 0.0;
      for (int k = s_prp[row[q]]; k < k1; ++k) s = s + s_pv[k] * s_x1[s_pci[k]];
      s_xc[row[q]] = s_xc[row[q]] + s;
    }
    __syncthreads();
    double rz = 0.0, zqp = 0.0;                    // post-smoothing
#pragma unroll
    for (int q = 0; q < kSR; ++q) {
      if (!own[q]) continue;
      const int i = row[q];
      const double z = s_xc[i] + swi[q] * (s_r[i] - arow(q, s_xc));
      s_z[i] = z;
      rz += s_r[i] * z;
      zqp += z * s_q[i];
    }
    const double rzt = wg_sum(rz, s_red[0]);
    zq = a.flexible ? wg_sum(zqp, s_red[1]) : 0.0;
    return rzt;
  };

  // r = b, x = 0, ||b||^2
  double bbp = 0.0;
#pragma unroll
  for (int q = 0; q < kSR; ++q) {
    const double bi = own[q] ? a.b[row[q]] : 0.0;
    if (own[q]) {
      s_r[row[q]] = bi;
      s_xc[row[q]] = swi[q] * bi;                  // pre-smoothing from zero
    }
    s_q[t + q * kST] = 0.0;
    bbp += bi * bi;
  }
  const double bb = wg_sum(bbp, s_red[2]);
  const double thresh = (a.tol * a.tol) * bb;
  int iters = 0, restarts = 0, state = 0;
  double rz = 0.0, pq = 0.0, rr = bb, trr = bb;
  if (bb == 0.0) {
    state = 3;
    trr = 0.0;
  } else if (!(bb == bb)) {
    state = -1;
  } else {
    for (;;) {
      // (re)start: z = M^-1 r, p = z
      double zq;
      rz = vcycle(zq);
      if (!(rz > 0.0)) {
        state = -1;
        break;
      }
#pragma unroll
      for (int q = 0; q < kSR; ++q)
        if (own[q]) s_p[row[q]] = s_z[row[q]];
      state = 2;
      while (iters < a.maxiter) {
        __syncthreads();                           // p complete
        double qi[kSR], pqp = 0.0;
#pragma unroll
        for (int q = 0; q < kSR; ++q) {
          qi[q] = own[q] ? arow(q, s_p) : 0.0;
          if (own[q]) {
            s_q[row[q]] = qi[q];
            pqp += s_p[row[q]] * qi[q];
          }
        }
        pq = wg_sum(pqp, s_red[3]);
        if (!(pq > 0.0)) {
          state = -1;
          break;
        }
        const double alpha = rz / pq;
        double rrp = 0.0;
#pragma unroll
        for (int q = 0; q < kSR; ++q) {
          if (!own[q]) continue;
          const int i = row[q];
          xi[q] = xi[q] + alpha * s_p[i];
          const double ri = s_r[i] - alpha * qi[q];
          s_r[i] = ri;
          s_xc[i] = swi[q] * ri;                   // pre-smoothing from zero
          rrp += ri * ri;
        }
        ++iters;
        rr = wg_sum(rrp, s_red[2]);
        if (rr <= thresh) {
          state = 1;
          break;
        }
        if (!(rr == rr)) {
          state = -1;
          break;
        }
        const double rzn = vcycle(zq);
        if (!(rzn > 0.0)) {
          state = -1;
          break;
        }
        const double beta = a.flexible ? -zq / pq : rzn / rz;
        rz = rzn;
#pragma unroll
        for (int q = 0; q < kSR; ++q)
          if (own[q]) s_p[row[q]] = s_z[row[q]] + beta * s_p[row[q]];
      }
      if (state < 0) break;
      // true residual r = b - A x
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kSR; ++q)
        if (own[q]) s_xc[row[q]] = xi[q];
      __syncthreads();
      double tp = 0.0;
#pragma unroll
      for (int q = 0; q < kSR; ++q) {
        if (!own[q]) continue;
        const double ti = a.b[opaque(row[q])] - arow(q, s_xc);
        s_r[row[q]] = ti;
        tp += ti * ti;
      }
      trr = wg_sum(tp, s_red[3]);
      if (trr <= thresh) break;
      if (state == 1 && restarts < 5 && iters < a.maxiter) {
        ++restarts;
#pragma unroll
        for (int q = 0; q < kSR; ++q)              // every read of s_xc lies before wg_sum's barrier
          if (own[q]) s_xc[row[q]] = swi[q] * s_r[row[q]];
        __syncthreads();
        continue;
      }
      break;
    }
  }
#pragma unroll
  for (int q = 0; q < kSR; ++q)
    if (own[q]) a.x[row[q]] = state == 3 ? 0.0 : xi[q];
  if (t == 0) {
    Ctl& c = *a.ctl;
    c.bb = bb;
    c.thresh = thresh;
    c.rz = rz;
    c.pq = pq;
    c.rr = rr;
    c.trr = trr;
    c.iters = iters;
    c.maxiter = a.maxiter;
    c.state = state;
    c.done = 1;
    c.flexible = a.flexible;
    c.restarts = restarts;
  }
}

}  // namespace

// Whether H's solves can run as one workgroup: two levels, at most 1024 fine
// rows with at most 8 entries per row of A_0, at most kSPCap entries of P_0,
// a dense coarsest level of at most 256 (padded) rows; FP64 V(1,1) cycle of
// one system, PCG.  Decided once per hierarchy (host copies of the row
// pointers).  R_0 is applied with the most lanes per coarse row (a power of
// two up to 64) that keeps every coarse row's group within the workgroup.
bool small_solve_ok(Hierarchy& H) {
  if (H.small_checked) return H.small_lgR >= 0;
  H.small_checked = true;
  H.small_lgR = -1;
  if (H.lv.size() != 2 || H.S != 1 || H.fp32() || !H.prm.precondition || H.prm.nu_pre != 1 ||
      H.prm.nu_post != 1 || H.prm.solver != AMG_SOLVER_PCG || !H.prm.symmetric)
    return false;
  const Level& L = H.lv[0];
  if (L.n > kSN || L.n < 1 || H.co.m > kSCoarse || H.co.n != L.nagg || L.nagg < 1 || L.pnnz > kSPCap) return false;
  std::vector<int> h(L.n + 1);
  AMG_HIP(hipMemcpy(h.data(), L.rp.p, sizeof(int) * (L.n + 1), hipMemcpyDeviceToHost));
  for (int r = 0; r < L.n; ++r)
    if (h[r + 1] - h[r] > kSRow) return false;
  int lg = 0;
  while (lg < 6 && (int64_t)L.nagg * (2 << lg) <= kST) ++lg;
  H.small_lgR = lg;
  return true;
}

amg_status pcg_solve_small(Hierarchy& H, const SolveOpts& o, const SolveWork& w, const double* d_b, double* d_x,
                           double tol, amg_info* info, hipStream_t s) {
  auto t0 = std::chrono::steady_clock::now();
  const Level& L = H.lv[0];
  SmallArgs a{};
  a.n = L.n;
  a.nc = H.co.n;
  a.m = H.co.m;
  a.lgR = H.small_lgR;
  a.maxiter = o.maxiter;
  a.flexible = o.flexible < 0 ? 0 : o.flexible;
  a.tol = tol;
  a.arp = L.rp.p;
  a.aci = L.ci.p;
  a.av = L.v.p;
  a.sw = L.sw.p;
  a.prp = L.prp.p;
  a.pci = L.pci.p;
  a.pv = L.pv.p;
  a.rrp = L.rrp.p;
  a.rci = L.rci.p;
  a.rv = L.rv.p;
  a.inv = H.co.inv.p;
  a.b = d_b;
  a.x = d_x;
  a.ctl = w.ctl;
  hipLaunchKernelGGL(k_pcg_small, dim3(1), dim3(kST), 0, s, a);
  AMG_HIP(hipGetLastError());
  AMG_HIP(hipMemcpyAsync(w.h_ctl, w.ctl, sizeof(Ctl), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  const Ctl& c = *w.h_ctl;
  amg_status st;
  if (c.state == 3 || c.trr <= c.thresh) st = AMG_OK;
  else if (c.state < 0) st = AMG_ERR_BREAKDOWN;
  else st = AMG_NOT_CONVERGED;
  if (info) {
    info->iters = c.iters;
    info->status = st;
    info->restarts = c.restarts;
    info->rel_resid = c.state == 3 ? 0.0 : (c.bb > 0 ? std::sqrt(c.trr / c.bb) : 0.0);
    if (st == AMG_ERR_BREAKDOWN) info->rel_resid = NAN;
    info->cache_event = H.cache_event;
    info->setup_ms = H.setup_ms;
    info->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  return st;
}

}  // namespace amg
