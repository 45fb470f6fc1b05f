// Two-sweep V-cycle levels.  With R = P^T, a pre-smoothing step from zero
// (x0 = S b) and one post-smoothing step, the V(1,1) cycle of a level,
//   x0 = S b, r = b - A x0, b' = R r, x1 = x0 + P e, x = x1 + S (b - A x1),
// is linear in (b, e = x'), and its four sweeps collapse into two:
//   down   b' = D b,          D = R (I - A S)
//   up     x  = B b + Q e,    B = 2 S - S A S,  Q = (I - S A) P
// Q lives on the pattern of A P, which the Galerkin product forms anyway, D on
// its transpose, B on the pattern of A.  The dense coarsest inverse is
// multiplied into the smallest levels the same way (X = B + Q X' D, or
// E = X' D), so that the cycle's end is one dense product.
//
// What bounds it: on levels of at most a few 100,000 rows every sweep is a
// chain of dependent memory latencies (row pointers, columns, gathers, the
// reduction) of 2-5 us whatever its bytes, so halving the sweeps halves the
// time; on the coarse levels of large systems D and Q hold 0.4 entries per
// entry of A, so the two sweeps also move fewer bytes than the four (128^3
// Poisson, level 1: 161 against 172 MB, of which 28 are padding of the rows of
// `up` and `dn`).  On a large level 0 the A P rows (8 entries against 7 of A)
// make both forms move the same bytes, and the four-sweep form keeps its
// offset-form matrix: see kFuse0.
//
// The sweep kernel reads rows in the sliced form of struct Ell: the only
// loads ahead of the entries are the slice's offset and the done flag
// (scalar, issued together), then all of a row's entries are in flight, then
// all of its gathers.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <type_traits>

#include "amg_internal.hpp"
#include "sizes.hpp"

namespace amg {
namespace {

constexpr int kEllU = 8;              // entries per lane in flight
constexpr int kDenseRows = 512;       // largest level whose whole cycle becomes one dense matrix
constexpr int64_t kDenseE = 1 << 19;  // most entries of the dense product E = X' D
// Level 0 takes the two-sweep form up to this many entries in its two sweeps
// (time per CG iteration, two-sweep against four-sweep level 0, FP64: 2D 181^2
// (0.4 M entries) 36 against 42 us, 2D 700^2 (6.6 M) 69 against 78, 2D 900^2
// (11 M) 101 against 97; 3D 40^3 (1.5 M) 45 against 49, 64^3 (6.0 M) 62 against
// 61, 80^3 (12 M) 98 against 85).  The line is where 3D systems break even; by
// entries alone 2D systems from there to about 9 M keep the slower four sweeps
// (700^2: a tenth).
constexpr int64_t kFuse0 = 6000000;

__device__ inline int block_of_xcd() {
  const int g = gridDim.x;
  if ((g & 7) == 0) return (blockIdx.x & 7) * (g >> 3) + (blockIdx.x >> 3);
  return blockIdx.x;
}

inline int blocks(int64_t items, int per = kBlock) { return (int)std::max<int64_t>(1, (items + per - 1) / per); }

// ------------------------------------------------------------- operators

template <class T>
struct OpDown {
  static constexpr int NRED = 0;
  using PT = T;
  const T* v;
  const T* b;
  T* y;
  struct Row {};
  __device__ T gather(int c) const { return b[c]; }
  __device__ Row row_in(int) const { return {}; }
  __device__ void epi(int row, T s, const Row&, double*) const { y[row] = s; }
};

// x = [B | Q] (b, e); RED >= 1: <r, x>, RED == 2: <x, q>.
template <class T, class OT, int RED>
struct OpUp {
  static constexpr int NRED = RED;
  using PT = T;
  const T* v;
  const T* b;
  const T* e;
  OT* out;
  int n;
  const double* r;
  const double* q;
  struct Row {
    double r, q;
  };
  __device__ T gather(int c) const { return *(c < n ? b + c : e + (c - n)); }
  __device__ Row row_in(int row) const {
    Row a{0.0, 0.0};
    if constexpr (RED >= 1) a.r = r[row];
    if constexpr (RED >= 2) a.q = q[row];
    return a;
  }
  __device__ void epi(int row, T s, const Row& a, double* d) const {
    const OT o = (OT)s;
    out[row] = o;
    if constexpr (RED >= 1) d[0] += a.r * (double)o;
    if constexpr (RED >= 2) d[1] += (double)o * a.q;
  }
};

template <int G, class Op>
__global__ void __launch_bounds__(kBlock) k_ell(int n, int slices, const int* __restrict__ off,
                                                const int* __restrict__ col, Op op, const int* __restrict__ stop,
                                                double* __restrict__ partials) {
  using T = typename Op::PT;
  const int lane = threadIdx.x & 63;
  const int sl = __builtin_amdgcn_readfirstlane(block_of_xcd() * (kBlock / 64) + (int)(threadIdx.x >> 6));
  const int sc = min(sl, slices - 1);
  const int o0 = off[sc], o1 = off[sc + 1];
  const int done = stop ? *stop : 0;
  if (done) return;
  const int w = sl < slices ? o1 - o0 : 0;
  const int row = sl * (64 / G) + lane / G;
  const typename Op::Row in = op.row_in(min(row, n - 1));
  T s = 0;
  for (int t0 = 0; t0 < w; t0 += kEllU) {
    int c[kEllU];
    T a[kEllU], x[kEllU];
#pragma unroll
    for (int u = 0; u < kEllU; ++u) {
      const int p = (o0 + min(t0 + u, w - 1)) * 64 + lane;
      c[u] = col[p];
      a[u] = op.v[p];
    }
#pragma unroll
    for (int u = 0; u < kEllU; ++u) x[u] = op.gather(max(c[u], 0));
#pragma unroll
    for (int u = 0; u < kEllU; ++u) {
      const T p = a[u] * x[u];
      s = t0 + u < w && c[u] >= 0 ? s + p : s;
    }
  }
  s = group_sum<G>(s);
  double d[Op::NRED > 0 ? Op::NRED : 1] = {};
  if (sl < slices && row < n && group_leader<G>()) op.epi(row, s, in, d);
  if constexpr (Op::NRED > 0) {
    block_sum<Op::NRED>(d);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int m = 0; m < Op::NRED; ++m) partials[m * gridDim.x + blockIdx.x] = d[m];
    }
  }
}

template <class Op>
int ell_sweep(const Ell& E, const Op& op, const int* stop, double* partials, hipStream_t s) {
#define AMG_ELL_G(GG) \
  case GG: hipLaunchKernelGGL((k_ell<GG, Op>), dim3(E.grid), dim3(kBlock), 0, s, E.n, E.slices, E.off.p, E.col.p, op, \
                              stop, partials); break;
  switch (E.g) {
    AMG_ELL_G(1) AMG_ELL_G(2) AMG_ELL_G(4) AMG_ELL_G(8) AMG_ELL_G(16) AMG_ELL_G(32)
    default: hipLaunchKernelGGL((k_ell<64, Op>), dim3(E.grid), dim3(kBlock), 0, s, E.n, E.slices, E.off.p, E.col.p, op,
                                stop, partials);
  }
#undef AMG_ELL_G
  return E.grid;
}

// x = X b, one wavefront (WPR = 1) or one workgroup (WPR = 4) per row; the
// matrix and the vector are loaded independently of each other.
template <int WPR, class T>
__global__ void __launch_bounds__(kBlock) k_dense(int rows, int cols, int ld, const T* __restrict__ X,
                                                  const T* __restrict__ b, T* __restrict__ x,
                                                  const int* __restrict__ stop) {
  __shared__ T s_w[kBlock / 64];
  constexpr int L = 64 * WPR, U = 8;
  const int done = stop ? *stop : 0;
  const int wave = threadIdx.x >> 6;
  const int row = WPR == 1 ? blockIdx.x * (kBlock / 64) + wave : blockIdx.x;
  const int t = WPR == 1 ? threadIdx.x & 63 : threadIdx.x;
  const T* Xr = X + (int64_t)min(row, rows - 1) * ld;
  T s = 0;
  for (int c0 = 0; c0 < cols; c0 += L * U) {
    T a[U], v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = min(c0 + t + u * L, cols - 1);
      a[u] = Xr[c];
      v[u] = b[c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T p = a[u] * v[u];
      s = c0 + t + u * L < cols ? s + p : s;
    }
  }
  if (done) return;
  s = group_sum<64>(s);
  if constexpr (WPR == 1) {
    if ((threadIdx.x & 63) == 63 && row < rows) x[row] = s;
  } else {
    if ((threadIdx.x & 63) == 63) s_w[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) x[row] = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
  }
}

// --------------------------------------------------------------- patterns

__global__ void k_pos_iota(int64_t m, int* __restrict__ a) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < m) a[t] = (int)t;
}

__global__ void k_rows_of(int n, const int* __restrict__ rp, int* __restrict__ rowid) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int k = rp[i]; k < rp[i + 1]; ++k) rowid[k] = i;
}

// Row pointers of m sorted keys in [0, nc) (m >= 1).
__global__ void k_rows_of_keys(int64_t m, int nc, const int* __restrict__ keys, int* __restrict__ rp) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= m) return;
  const int k = keys[t], prev = t > 0 ? keys[t - 1] : -1;
  for (int j = prev + 1; j <= k; ++j) rp[j] = (int)t;
  if (t == m - 1)
    for (int j = k + 1; j <= nc; ++j) rp[j] = (int)m;
}

__global__ void k_gather_i32(int64_t m, const int* __restrict__ perm, const int* __restrict__ a,
                             int* __restrict__ out) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < m) out[t] = a[perm[t]];
}

__global__ void k_fill_int(int64_t m, int v, int* __restrict__ a) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < m) a[t] = v;
}

// Position of (j, i) for every stored (i, j); flags[0] |= 1 when one is absent.
__global__ void k_tpos(int n, const int* __restrict__ rp, const int* __restrict__ ci, int* __restrict__ tpos,
                       int* flags) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int k = rp[i]; k < rp[i + 1]; ++k) {
    const int j = ci[k];
    int lo = rp[j], hi = rp[j + 1];
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (ci[mid] < i) lo = mid + 1; else hi = mid;
    }
    const bool ok = lo < rp[j + 1] && ci[lo] == i;
    tpos[k] = ok ? lo : -1;
    if (!ok) atomicOr(flags, 1);
  }
}

// Slice widths: the steps of the slice's longest row (in all at most the number
// of entries, so their sum fits 32 bits where 64 times it need not).  A row's
// entries are those of row i of the first pattern, then of the second (when
// given).
__global__ void k_ell_width(int n, int slices, int g, const int* __restrict__ rp1, const int* __restrict__ rp2,
                            int* __restrict__ cnt) {
  const int sl = blockIdx.x * blockDim.x + threadIdx.x;
  if (sl > slices) return;
  if (sl == slices) {
    cnt[slices] = 0;
    return;
  }
  const int rows = 64 / g, r1 = min(n, (sl + 1) * rows);
  int w = 0;
  for (int i = sl * rows; i < r1; ++i) w = max(w, rp1[i + 1] - rp1[i] + (rp2 ? rp2[i + 1] - rp2[i] : 0));
  cnt[sl] = (w + g - 1) / g;
}

// Columns and sources: an entry of the first pattern has source k >= 0 and
// column ci1[k], one of the second source -2 - e and column n + ci2[e];
// padding -1.  One wavefront per slice.
__global__ void __launch_bounds__(kBlock) k_ell_fill(int n, int slices, int g, const int* __restrict__ off,
                                                     const int* __restrict__ rp1, const int* __restrict__ ci1,
                                                     const int* __restrict__ rp2, const int* __restrict__ ci2,
                                                     int* __restrict__ col, int* __restrict__ src) {
  const int sl = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (sl >= slices) return;
  const int row = sl * (64 / g) + lane / g;
  const int o = off[sl] * 64, w = off[sl + 1] - off[sl];
  const int k1 = row < n ? rp1[row] : 0, n1 = row < n ? rp1[row + 1] - k1 : 0;
  const int k2 = row < n && rp2 ? rp2[row] : 0, n2 = row < n && rp2 ? rp2[row + 1] - k2 : 0;
  for (int t = 0; t < w; ++t) {
    const int j = t * g + (lane & (g - 1));
    int c = -1, sr = -1;
    if (j < n1) {
      c = ci1[k1 + j];
      sr = k1 + j;
    } else if (j - n1 < n2) {
      c = n + ci2[k2 + j - n1];
      sr = -2 - (k2 + j - n1);
    }
    col[o + t * 64 + lane] = c;
    src[o + t * 64 + lane] = sr;
  }
}

// ----------------------------------------------------------------- values

template <class RT>
__device__ inline double pval(RT v) { return (double)ValCvt<RT>::f(v); }

// (A P) entries from the FP32 cycle's own operands (FP32 A, FP32 or bf16 P),
// accumulated in FP64: through the product map, or by search (thread per row).
// The map's pairs are read four ahead (level 1 of a 128^3 system: one at a time
// 0.93 ms, so 0.45).
// With tpos (the entry a_ji of entry a_ij) the map gives A^T P instead: the
// patterns and the order of the terms are those of A P.
template <class RT, class T>
__global__ void k_ap_map(int64_t m, const int64_t* __restrict__ off, const int2* __restrict__ pairs,
                         const T* __restrict__ av, const int* __restrict__ tpos, const RT* __restrict__ pv,
                         double* __restrict__ ap) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= m) return;
  double acc = 0.0;
  const int64_t p1 = off[e + 1];
  for (int64_t p = off[e]; p < p1; p += 4) {       // four terms' loads in flight, added in order
    int2 pr[4];
    int k[4];
    double a[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) pr[u] = pairs[p + u < p1 ? p + u : p1 - 1];
#pragma unroll
    for (int u = 0; u < 4; ++u) k[u] = tpos ? tpos[pr[u].x] : pr[u].x;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = (double)av[k[u]];
      q[u] = pval(pv[pr[u].y]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = p + u < p1 ? acc + a[u] * q[u] : acc;
  }
  ap[e] = acc;
}

template <class RT>
__global__ void k_ap_search(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                            const float* __restrict__ av, const int* __restrict__ prp, const int* __restrict__ pci,
                            const RT* __restrict__ pv, const int* __restrict__ aprp, const int* __restrict__ apci,
                            double* __restrict__ ap) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int e = aprp[i]; e < aprp[i + 1]; ++e) {
    const int J = apci[e];
    double acc = 0.0;
    for (int k = rp[i]; k < rp[i + 1]; ++k) {
      const int j = ci[k];
      for (int t = prp[j]; t < prp[j + 1]; ++t)
        if (pci[t] == J) acc += (double)av[k] * pval(pv[t]);
    }
    ap[e] = acc;
  }
}

// Q = P - S (A P) (thread per row; P's sorted row is a subset of A P's); q may
// be ap.
template <class RT, class T>
__global__ void k_q_values(int n, const int* __restrict__ prp, const int* __restrict__ pci,
                           const RT* __restrict__ pv, const int* __restrict__ aprp, const int* __restrict__ apci,
                           const double* ap, const T* __restrict__ sw, double* q) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double w = (double)sw[i];
  int t = prp[i];
  const int t1 = prp[i + 1];
  for (int e = aprp[i]; e < aprp[i + 1]; ++e) {
    const int J = apci[e];
    while (t < t1 && pci[t] < J) ++t;
    const double p = t < t1 && pci[t] == J ? pval(pv[t]) : 0.0;
    q[e] = p - w * ap[e];
  }
}

// D^T = P - S (A^T P) on the pattern of A P, for a structurally symmetric A
// with nonsymmetric values: (A^T P)_jK = sum over i in row j of a_ij P_iK.  Where there is no
// product map: kDtLanes lanes per row, one entry each at a time, walk the same
// rows of P together, so every load serves all of them (level 1 of a 128^3
// convection-diffusion system: a thread per row 4.4 ms, so 1.4 ms, the map's
// two kernels 0.54 ms).
constexpr int kDtLanes = 16;
template <class RT, class T>
__global__ void k_dt_values(int n, const int* __restrict__ rp, const int* __restrict__ ci, const T* __restrict__ av,
                            const int* __restrict__ tpos, const int* __restrict__ prp, const int* __restrict__ pci,
                            const RT* __restrict__ pv, const int* __restrict__ aprp, const int* __restrict__ apci,
                            const T* __restrict__ sw, double* __restrict__ dt) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t0 < (int64_t)n * kDtLanes; t0 += stride) {
    const int j = (int)(t0 / kDtLanes), l = (int)(t0 % kDtLanes);
    const double w = (double)sw[j];
    for (int e = aprp[j] + l; e < aprp[j + 1]; e += kDtLanes) {
      const int K = apci[e];
      double acc = 0.0, own = 0.0;
      for (int k = rp[j]; k < rp[j + 1]; ++k) {
        const int i = ci[k];
        for (int t = prp[i]; t < prp[i + 1]; ++t)
          if (pci[t] == K) {
            const double p = pval(pv[t]);
            acc += (double)av[tpos[k]] * p;
            if (i == j) own = p;
          }
      }
      dt[e] = own - w * acc;
    }
  }
}

// Values of the sliced rows.  A: source k >= 0 of `up` is an entry of A and
// becomes that entry of B = 2 S - S A S; every other source indexes the
// entries ap (sources are plain positions when A is false).
template <bool A, class T>
__global__ void __launch_bounds__(kBlock) k_ell_values(int n, int slices, int g, const int* __restrict__ off,
                                                       const int* __restrict__ col, const int* __restrict__ src,
                                                       const T* __restrict__ av, const T* __restrict__ sw,
                                                       const double* __restrict__ ap, T* __restrict__ v) {
  const int sl = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (sl >= slices) return;
  const int row = sl * (64 / g) + lane / g;
  const int o = off[sl] * 64, w = off[sl + 1] - off[sl];
  const double si = A && row < n ? (double)sw[row] : 0.0;
  for (int t = 0; t < w; ++t) {
    const int p = o + t * 64 + lane;
    const int k = src[p];
    double x = 0.0;
    if constexpr (A) {
      if (k >= 0) {
        const int c = col[p];
        x = -(si * (double)av[k] * (double)sw[c]);
        if (c == row) x += 2.0 * si;
      } else if (k <= -2) {
        x = ap[-2 - k];
      }
    } else if (k >= 0) {
      x = ap[k];
    }
    v[p] = (T)x;
  }
}

// --------------------------------------------------------------- dense tail

// T = Q X': row i of T (thread per entry).
__global__ void k_qx(int n, int m, int ld, const int* __restrict__ aprp, const int* __restrict__ apci,
                     const double* __restrict__ q, const double* __restrict__ X, double* __restrict__ T) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)n * m) return;
  const int i = (int)(t / m), K = (int)(t - (int64_t)i * m);
  double s = 0.0;
  for (int e = aprp[i]; e < aprp[i + 1]; ++e) s += q[e] * X[(int64_t)apci[e] * ld + K];
  T[t] = s;
}

// Y[r][j] = sum_K T[r][K] D[K][j] (D^T by rows: entry e of row j is D[apci[e]][j]).
__global__ void k_xd(int rows, int n, int ldt, const int* __restrict__ aprp, const int* __restrict__ apci,
                     const double* __restrict__ dt, const double* __restrict__ T, double* __restrict__ Y) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)rows * n) return;
  const int r = (int)(t / n), j = (int)(t - (int64_t)r * n);
  double s = 0.0;
  for (int e = aprp[j]; e < aprp[j + 1]; ++e) s += T[(int64_t)r * ldt + apci[e]] * dt[e];
  Y[t] = s;
}

// X += B on A's pattern (thread per row).
template <class T>
__global__ void k_add_b(int n, const int* __restrict__ rp, const int* __restrict__ ci, const T* __restrict__ av,
                        const T* __restrict__ sw, double* __restrict__ X) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double si = (double)sw[i];
  for (int k = rp[i]; k < rp[i + 1]; ++k) {
    const int c = ci[k];
    double x = -(si * (double)av[k] * (double)sw[c]);
    if (c == i) x += 2.0 * si;
    X[(int64_t)i * n + c] += x;
  }
}

__global__ void k_f64_to_f32(int64_t m, const double* __restrict__ a, float* __restrict__ b) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < m) b[t] = (float)a[t];
}

// dn sources k (entry of dn's rows) -> entry of A P.
__global__ void k_src_perm(int64_t m, const int* __restrict__ perm, int* __restrict__ src) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < m && src[t] >= 0) src[t] = perm[src[t]];
}

// ------------------------------------------------------------------- host

template <class F>
void cub_run(F&& f, hipStream_t s) {
  size_t tmp = 0;
  AMG_HIP(f(nullptr, tmp));
  TBuf<unsigned char> buf;
  buf.alloc((int64_t)std::max<size_t>(tmp, 1));
  AMG_HIP(f(buf.p, tmp));
}

// Sliced form of the rows of one pattern, or of two side by side; false when
// padding would more than double its `nnz` entries.
bool build_ell(Ell& E, int n, int64_t nnz, const int* rp1, const int* ci1, const int* rp2, const int* ci2,
               hipStream_t s) {
  const double avg = (double)nnz / std::max(n, 1);
  E.n = n;
  E.g = 1;
  while (E.g < 64 && avg > 6.0 * E.g) E.g <<= 1;
  const int rows = 64 / E.g;
  E.slices = (n + rows - 1) / rows;
  TBuf<int> cnt;
  cnt.alloc(E.slices + 1);
  E.off.alloc(E.slices + 1);
  hipLaunchKernelGGL(k_ell_width, dim3(blocks(E.slices + 1)), dim3(kBlock), 0, s, n, E.slices, E.g, rp1, rp2, cnt.p);
  cub_run([&](void* t, size_t& b) {
    return hipcub::DeviceScan::ExclusiveSum(t, b, cnt.p, E.off.p, E.slices + 1, s);
  }, s);
  int steps = 0;
  AMG_HIP(hipMemcpyAsync(&steps, E.off.p + E.slices, sizeof(int), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  if (!ell_fits(steps, nnz, E.slices)) return false;
  E.len = 64 * (int64_t)steps;
  int g = blocks(E.slices, kBlock / 64);
  if (g >= 64) g = (g + 7) / 8 * 8;
  E.grid = g;
  E.col.alloc(std::max<int64_t>(E.len, 1));
  E.src.alloc(std::max<int64_t>(E.len, 1));
  hipLaunchKernelGGL(k_ell_fill, dim3(blocks(E.slices, kBlock / 64)), dim3(kBlock), 0, s, n, E.slices, E.g, E.off.p,
                     rp1, ci1, rp2, ci2, E.col.p, E.src.p);
  AMG_HIP(hipGetLastError());
  return true;
}

// D's values need the transposed entries of A unless the values are
// symmetric: BiCGSTAB may be given any A, and a CG handle's values (also the
// preconditioner of another solver) are looked at.
bool nonsym_values(const Hierarchy& H) {
  return !H.prm.symmetric || H.prm.solver != AMG_SOLVER_PCG || !H.values_sym;
}

// Position of every entry's transpose; false when one is absent.
bool build_tpos(Hierarchy& H, Level& L, hipStream_t s) {
  L.tpos.alloc(L.nnz);
  hipLaunchKernelGGL(k_fill_int, dim3(1), dim3(64), 0, s, (int64_t)1, 0, H.flags.p);
  hipLaunchKernelGGL(k_tpos, dim3(blocks(L.n)), dim3(kBlock), 0, s, L.n, L.rp.p, L.ci.p, L.tpos.p, H.flags.p);
  AMG_HIP(hipGetLastError());
  AMG_HIP(hipMemcpyAsync(H.h_flags, H.flags.p, sizeof(int), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  return H.h_flags[0] == 0;
}

bool build_level_pattern(Hierarchy& H, int l, hipStream_t s) {
  Level& L = H.lv[l];
  const int nc = L.nagg;
  if (L.nnz + L.apnnz >= (int64_t)1 << 30) return false;
  if (nonsym_values(H) && !build_tpos(H, L, s)) return false;  // structurally nonsymmetric
  if (!build_ell(L.up, L.n, L.nnz + L.apnnz, L.rp.p, L.ci.p, L.aprp.p, L.apci.p, s)) return false;
  {
    // transpose of the pattern of A P: a stable sort of its entries by column
    const int64_t m = L.apnnz;
    TBuf<int> rowid, iota, keys, dperm, dci, drp;
    rowid.alloc(m);
    iota.alloc(m);
    keys.alloc(m);
    dperm.alloc(m);   // entry of dn's rows -> entry of A P
    dci.alloc(m);
    drp.alloc(nc + 1);
    hipLaunchKernelGGL(k_rows_of, dim3(blocks(L.n)), dim3(kBlock), 0, s, L.n, L.aprp.p, rowid.p);
    hipLaunchKernelGGL(k_pos_iota, dim3(blocks(m)), dim3(kBlock), 0, s, m, iota.p);
    int bits = 1;
    while ((1ll << bits) < (long long)nc) ++bits;
    cub_run([&](void* t, size_t& b) {
      return hipcub::DeviceRadixSort::SortPairs(t, b, L.apci.p, keys.p, iota.p, dperm.p, (int)m, 0, bits, s);
    }, s);
    hipLaunchKernelGGL(k_rows_of_keys, dim3(blocks(m)), dim3(kBlock), 0, s, m, nc, keys.p, drp.p);
    hipLaunchKernelGGL(k_gather_i32, dim3(blocks(m)), dim3(kBlock), 0, s, m, dperm.p, rowid.p, dci.p);
    if (!build_ell(L.dn, nc, m, drp.p, dci.p, nullptr, nullptr, s)) return false;
    // sources as entries of A P instead of entries of dn's rows
    hipLaunchKernelGGL(k_src_perm, dim3(blocks(L.dn.len)), dim3(kBlock), 0, s, L.dn.len, dperm.p, L.dn.src.p);
  }
  return true;
}

// The level's two-sweep form; false (and nothing kept) where it is not taken.
bool build_level(Hierarchy& H, int l, hipStream_t s) {
  Level& L = H.lv[l];
  if (!build_level_pattern(H, l, s)) {
    L.up.release();
    L.dn.release();
    L.tpos.release();
    return false;
  }
  L.qv.alloc(L.apnnz);
  if (nonsym_values(H)) L.dtv.alloc(L.apnnz);
  if (H.fp32()) {
    L.apt.alloc(L.apnnz);
    L.up.v32.alloc(std::max<int64_t>(L.up.len, 1));
    L.dn.v32.alloc(std::max<int64_t>(L.dn.len, 1));
  } else {
    L.up.v.alloc(std::max<int64_t>(L.up.len, 1));
    L.dn.v.alloc(std::max<int64_t>(L.dn.len, 1));
  }
  return true;
}

template <class T>
T* ell_v(Ell& E) {
  if constexpr (std::is_same<T, double>::value) return E.v.p;
  else return E.v32.p;
}
template <class T>
const T* level_a(const Level& L) {
  if constexpr (std::is_same<T, double>::value) return L.v.p;
  else return L.v32.p;
}
template <class T>
const T* level_sw(const Level& L) {
  if constexpr (std::is_same<T, double>::value) return L.sw.p;
  else return L.sw32.p;
}
template <class T>
T* level_x(Level& L) {
  if constexpr (std::is_same<T, double>::value) return L.x64.p;
  else return L.x32.p;
}
template <class T>
T* level_b(Level& L) {
  if constexpr (std::is_same<T, double>::value) return L.b64.p;
  else return L.b32.p;
}

template <class T, class RT>
void level_values(Hierarchy& H, Level& L, const RT* pv, hipStream_t s) {
  const double* ap = L.apv.p;
  const dim3 b(kBlock);
  const bool ns = nonsym_values(H);
  if constexpr (std::is_same<T, float>::value) {
    if (L.pmaps)
      hipLaunchKernelGGL((k_ap_map<RT, T>), dim3(blocks(L.apnnz)), b, 0, s, L.apnnz, L.apmo.p, L.apm.p, L.v32.p,
                         (const int*)nullptr, pv, L.apt.p);
    else
      hipLaunchKernelGGL(k_ap_search<RT>, dim3(blocks(L.n)), b, 0, s, L.n, L.rp.p, L.ci.p, L.v32.p, L.prp.p, L.pci.p,
                         pv, L.aprp.p, L.apci.p, L.apt.p);
    ap = L.apt.p;
  }
  hipLaunchKernelGGL((k_q_values<RT, T>), dim3(blocks(L.n)), b, 0, s, L.n, L.prp.p, L.pci.p, pv, L.aprp.p, L.apci.p,
                     ap, level_sw<T>(L), L.qv.p);
  if (ns && L.pmaps) {
    hipLaunchKernelGGL((k_ap_map<RT, T>), dim3(blocks(L.apnnz)), b, 0, s, L.apnnz, L.apmo.p, L.apm.p, level_a<T>(L),
                       L.tpos.p, pv, L.dtv.p);
    hipLaunchKernelGGL((k_q_values<RT, T>), dim3(blocks(L.n)), b, 0, s, L.n, L.prp.p, L.pci.p, pv, L.aprp.p,
                       L.apci.p, L.dtv.p, level_sw<T>(L), L.dtv.p);
  } else if (ns)
    hipLaunchKernelGGL((k_dt_values<RT, T>), dim3(stride_grid((int64_t)L.n * kDtLanes, kBlock)), b, 0, s, L.n,
                       L.rp.p, L.ci.p, level_a<T>(L), L.tpos.p, L.prp.p, L.pci.p, pv, L.aprp.p, L.apci.p,
                       level_sw<T>(L), L.dtv.p);
  hipLaunchKernelGGL((k_ell_values<true, T>), dim3(blocks(L.up.slices, kBlock / 64)), b, 0, s, L.n, L.up.slices,
                     L.up.g, L.up.off.p, L.up.col.p, L.up.src.p, level_a<T>(L), level_sw<T>(L), L.qv.p,
                     ell_v<T>(L.up));
  hipLaunchKernelGGL((k_ell_values<false, T>), dim3(blocks(L.dn.slices, kBlock / 64)), b, 0, s, L.nagg, L.dn.slices,
                     L.dn.g, L.dn.off.p, L.dn.col.p, L.dn.src.p, (const T*)nullptr, (const T*)nullptr,
                     ns ? L.dtv.p : L.qv.p, ell_v<T>(L.dn));
  AMG_HIP(hipGetLastError());
}

// Row-major copy of the transposed coarsest inverse (nonsymmetric hierarchies).
__global__ void k_untranspose(int n, int m, const double* __restrict__ a, double* __restrict__ b) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)n * n) return;
  const int i = (int)(t / n), j = (int)(t - (int64_t)i * n);
  b[t] = a[(int64_t)j * m + i];
}

// The dense end.  From the coarsest inverse upwards, a level of at most
// kDenseRows rows is folded in whole (X = B + Q X' D: its two sweeps and the
// product below become one product of n^2 entries, 2 MB at 512 rows); then,
// where the result stays small, the down sweep of the level above (E = X' D).
template <class T>
void tail_values(Hierarchy& H, hipStream_t s) {
  Tail& t = H.tail;
  const dim3 b(kBlock);
  const int nl = (int)H.lv.size();
  const int top = std::max(H.lf, 1);
  int lx = nl - 1, n = H.co.n, ld = H.co.m;
  // the products written below, by the buffer they go to (none of a hierarchy
  // whose end is the coarsest inverse itself)
  int64_t need[3] = {};
  {
    int at = 0, l = lx;
    int64_t m = n;
    auto writes = [&](int w, int64_t count) { need[w] = std::max(need[w], count); };
    if (!H.prm.symmetric) {
      writes(at, m * m);
      at ^= 1;
    }
    for (; l - 1 >= top && H.lv[l - 1].n <= kDenseRows; --l) {
      const int64_t k = H.lv[l - 1].n;
      writes(2, k * m);
      writes(at, k * k);
      at ^= 1;
      m = k;
    }
    if (l - 1 >= H.lf && m * H.lv[l - 1].n <= kDenseE) writes(at, m * H.lv[l - 1].n);
  }
  for (int w = 0; w < 3; ++w) t.w[w].alloc(need[w]);
  const double* X = H.co.inv.p;
  int at = 0;
  if (!H.prm.symmetric) {
    hipLaunchKernelGGL(k_untranspose, dim3(blocks((int64_t)n * n)), b, 0, s, n, ld, X, t.w[at].p);
    X = t.w[at].p;
    ld = n;
    at ^= 1;
  }
  int lb = lx, cols = n;
  const bool ns = nonsym_values(H);
  auto dt = [ns](const Level& L) { return ns ? L.dtv.p : L.qv.p; };
  while (lx - 1 >= top && H.lv[lx - 1].n <= kDenseRows) {
    Level& L = H.lv[lx - 1];
    double* Y = t.w[at].p;
    hipLaunchKernelGGL(k_qx, dim3(blocks((int64_t)L.n * n)), b, 0, s, L.n, n, ld, L.aprp.p, L.apci.p, L.qv.p, X,
                       t.w[2].p);
    hipLaunchKernelGGL(k_xd, dim3(blocks((int64_t)L.n * L.n)), b, 0, s, L.n, L.n, n, L.aprp.p, L.apci.p, dt(L),
                       t.w[2].p, Y);
    hipLaunchKernelGGL(k_add_b<T>, dim3(blocks(L.n)), b, 0, s, L.n, L.rp.p, L.ci.p, level_a<T>(L), level_sw<T>(L), Y);
    X = Y;
    at ^= 1;
    --lx;
    n = ld = cols = L.n;
    lb = lx;
  }
  if (lx - 1 >= H.lf && (int64_t)n * H.lv[lx - 1].n <= kDenseE) {
    Level& L = H.lv[lx - 1];
    hipLaunchKernelGGL(k_xd, dim3(blocks((int64_t)n * L.n)), b, 0, s, n, L.n, ld, L.aprp.p, L.apci.p, dt(L), X,
                       t.w[at].p);
    X = t.w[at].p;
    ld = cols = L.n;
    lb = lx - 1;
  }
  t.lb = lb;
  t.lx = lx;
  t.rows = n;
  t.cols = cols;
  t.ld = ld;
  t.X = X;
  if constexpr (std::is_same<T, float>::value) {
    const int64_t m = (int64_t)n * ld;
    t.X32.alloc(m);
    hipLaunchKernelGGL(k_f64_to_f32, dim3(blocks(m)), b, 0, s, m, X, t.X32.p);
  }
  AMG_HIP(hipGetLastError());
}

template <class T>
const T* tail_x(const Tail& t) {
  if constexpr (std::is_same<T, double>::value) return t.X;
  else return t.X32.p;
}

template <class T>
void all_values(Hierarchy& H, hipStream_t s) {
  const int nl = (int)H.lv.size();
  for (int l = H.lf; l < nl - 1; ++l) {
    Level& L = H.lv[l];
    if constexpr (std::is_same<T, double>::value) level_values<T, double>(H, L, L.pv.p, s);
    else if (H.bf16()) level_values<T, uint16_t>(H, L, L.pbf.p, s);
    else level_values<T, float>(H, L, L.pv32.p, s);
  }
  tail_values<T>(H, s);
}

}  // namespace

// Two-sweep levels reach from the coarsest level up to the first one that is
// left out: single systems with the V(1,1) cycle, level 0 only up to kFuse0
// entries, rows whose padding stays below their entries.
void fused_levels(Hierarchy& H, bool build, hipStream_t s) {
  const int nl = (int)H.lv.size();
  if (build) H.lf = nl - 1;
  if (H.S != 1 || !H.prm.precondition || nl < 2) return;
  if (build) {
    if (H.prm.nu_pre == 1 && H.prm.nu_post == 1) {
      for (int l = nl - 2; l >= 0; --l) {
        if (l == 0 && H.nnz + 2 * H.lv[0].apnnz > kFuse0) break;
        if (!build_level(H, l, s)) break;
        H.lf = l;
      }
    }
  }
  // values that were symmetric when the levels were built and are not any more
  // (the pattern is symmetric then, on every level)
  if (!build && nonsym_values(H))
    for (int l = H.lf; l < nl - 1; ++l) {
      Level& L = H.lv[l];
      if (L.tpos.p) continue;
      if (!build_tpos(H, L, s)) throw Error(AMG_ERR_HIP, "coarse pattern is not symmetric");
      L.dtv.alloc(L.apnnz);
    }
  if (H.fp32()) all_values<float>(H, s);
  else all_values<double>(H, s);
}

template <class T>
int fused_cycle(Hierarchy& H, const T* b0, const double* r, double* z, const double* q, int red, const int* stop,
                double* partials, hipStream_t s) {
  const Tail& t = H.tail;
  const int lf = H.lf, nl = (int)H.lv.size();
  auto rhs = [&](int l) { return l == lf && b0 ? b0 : (const T*)level_b<T>(H.lv[l]); };
  for (int l = lf; l < t.lb; ++l) {
    Level& L = H.lv[l];
    InstScope is(H, KID_RESTRICT, l, s, stop);
    ell_sweep(L.dn, OpDown<T>{ell_v<T>(L.dn), rhs(l), level_b<T>(H.lv[l + 1])}, stop, nullptr, s);
  }
  {
    InstScope is(H, KID_COARSE, nl - 1, s, stop);
    T* x = level_x<T>(H.lv[t.lx]);
    // long rows take a workgroup each
    if (t.cols > 1024)
      hipLaunchKernelGGL((k_dense<4, T>), dim3(t.rows), dim3(kBlock), 0, s, t.rows, t.cols, t.ld, tail_x<T>(t),
                         rhs(t.lb), x, stop);
    else
      hipLaunchKernelGGL((k_dense<1, T>), dim3(blocks(t.rows, kBlock / 64)), dim3(kBlock), 0, s, t.rows, t.cols, t.ld,
                         tail_x<T>(t), rhs(t.lb), x, stop);
  }
  int np = 0;
  for (int l = t.lx - 1; l >= lf; --l) {
    Level& L = H.lv[l];
    InstScope is(H, KID_POST, l, s, stop);
    const T* v = ell_v<T>(L.up);
    const T* b = rhs(l);
    const T* e = level_x<T>(H.lv[l + 1]);
    if (l > 0)
      ell_sweep(L.up, OpUp<T, T, 0>{v, b, e, level_x<T>(L), L.n, nullptr, nullptr}, stop, nullptr, s);
    else if (red == 2)
      np = ell_sweep(L.up, OpUp<T, double, 2>{v, b, e, z, L.n, r, q}, stop, partials, s);
    else if (red == 1)
      np = ell_sweep(L.up, OpUp<T, double, 1>{v, b, e, z, L.n, r, q}, stop, partials, s);
    else
      ell_sweep(L.up, OpUp<T, double, 0>{v, b, e, z, L.n, r, q}, stop, nullptr, s);
  }
  AMG_HIP(hipGetLastError());
  return np;
}

template int fused_cycle<double>(Hierarchy&, const double*, const double*, double*, const double*, int, const int*,
                                 double*, hipStream_t);
template int fused_cycle<float>(Hierarchy&, const float*, const double*, double*, const double*, int, const int*,
                                double*, hipStream_t);

// Algorithmic bytes of a launch on a two-sweep level (stored entries and
// columns, every vector operand once).
double fused_bytes(const Hierarchy& H, int kid, int level) {
  const Level& L = H.lv[level];
  const double v = H.fp32() ? 4.0 : 8.0;
  const double n = L.n, nc = L.nagg;
  const bool down = level < H.tail.lb, up = level < H.tail.lx;
  switch (kid) {
    case KID_RESTRICT: return down ? (v + 4.0) * (double)L.dn.len + 4.0 * (L.dn.slices + 1) + v * (n + nc) : 0.0;
    case KID_POST:
      return up ? (v + 4.0) * (double)L.up.len + 4.0 * (L.up.slices + 1) + v * (n + nc) + (level ? v : 16.0) * n : 0.0;
    case KID_COARSE: return v * ((double)H.tail.rows * H.tail.cols + H.tail.rows + H.tail.cols);
  }
  return 0.0;
}

}  // namespace amg
