// Multi-shift COCG engine (FP64) for the shifted systems of one filter
// application.  In the residual-correction form (and in the literal form) all
// N_c shifted systems of column i share the right-hand side b_i, so one Krylov
// space serves them: K(z_j I - A, b) = K(A, b) for every z_j.  The engine runs
// CG on a real symmetric positive definite seed M = A - s I (s below the
// spectrum) and obtains every shifted system's iterate from the seed's scalars.
//
// Seed CG (x0 = 0):  r_0 = b, p_k = r_k + beta_{k-1} p_{k-1},
//   alpha_k = r_k^T r_k / p_k^T M p_k,  r_{k+1} = r_k - alpha_k M p_k,
//   beta_k = r_{k+1}^T r_{k+1} / r_k^T r_k.
// With R_k the residual polynomial (r_k = R_k(M) b, R_k(0) = 1) and the
// system (M + sigma I) x = b, the shifted residual is collinear with the
// seed's: r^sigma_k = r_k / pi_k with pi_k = R_k(-sigma).  The three-term
// recurrence of R_k gives
//   pi_{k+1} = (1 + c_k + alpha_k sigma) pi_k - c_k pi_{k-1},
//   c_k = beta_{k-1} alpha_k / alpha_{k-1}  (pi_{-1} = pi_0 = 1, beta_{-1} = 0),
// and the shifted iterate follows
//   p^s_k = r_k / pi_k + beta^s_{k-1} p^s_{k-1},  x^s_{k+1} = x^s_k + alpha^s_k p^s_k,
//   alpha^s_k = alpha_k pi_k / pi_{k+1},  beta^s_k = beta_k (pi_k / pi_{k+1})^2.
// (z_j I - A) d = b is (M + sigma_j I) x = b with sigma_j = s - z_j and
// d = -x.  The seed's R_k has real roots (Ritz values of M) and sigma_j is
// off the real axis, so pi_k never vanishes: no breakdown.  A shifted
// system stops (its x and p are frozen) when its residual |r_k| / |pi_k|
// drops below tol |b|; the seed runs until every shift of its column has
// stopped.  The seed's r, p and the pi's are rescaled together when |r_k|
// falls below 1e-100 |b| (the shifted quantities depend on their ratios).
//
// Combining mode (the filter step of FEAST): only the weighted sum
// sum_j Re(g_j d_j) of the solutions is needed, so the engine accumulates it
// into one real block as the iterates advance and never stores them: a shift
// then moves its direction only (32 B per row and column instead of 64).
//
// The seed needs nothing of the shifted systems, so their directions and
// iterates follow it kMsDefer iterations at a time: the seed residuals and the
// scalars of those iterations are kept, and one pass over the directions
// applies them all, in the same order and with the same results as a pass per
// iteration at a quarter of its traffic.  Where there is no memory for so many
// residuals, a pass per iteration it is.
//
// Layout: engine rows in the streaming engine's reverse Cuthill-McKee order,
// blocks n x kp row-major (kp = 64 CPL, column c of lane c / CPL); the seed
// r, p, w are real, the shifted p^s and x^s complex, one n x kp block per
// shift.  Row kernels: 256 threads, a wave per row, the rows cut into eight
// contiguous stripes (one per XCD) swept by that XCD's waves side by side,
// so the SpMV's neighbour rows were read recently into the same L2.
// Reductions: per-workgroup partials summed in a fixed order per column.
#include "device.h"
#include "kernels.h"

namespace rafeast {

namespace {

constexpr int kMT = 256;          // threads of a row kernel
constexpr int kMW = kMT / 64;     // its waves

struct Rows {
  int first, stride, count;
};

// Rows of this wave: workgroup b runs on XCD b mod 8 and takes a share of
// that XCD's contiguous eighth of the rows.
__device__ __forceinline__ Rows my_rows(int n) {
  const int nb = gridDim.x;
  int x = 0, i = (int)blockIdx.x, per_x = nb, lo = 0, hi = n;
  if (nb % 8 == 0) {
    x = (int)(blockIdx.x % 8);
    i = (int)(blockIdx.x / 8);
    per_x = nb / 8;
    const int stripe = (n + 7) / 8;
    lo = min(n, x * stripe);
    hi = min(n, lo + stripe);
  }
  const int stride = per_x * kMW;
  const int first = lo + i * kMW + wave_id();
  return {first, stride, first < hi ? (hi - first + stride - 1) / stride : 0};
}

// Sum the four waves' per-lane values and store the workgroup's partial of
// each column at part[c * gridDim.x + blockIdx.x] (a column's partials together).
template <int CPL>
__device__ __forceinline__ void put_partial(const double (&acc)[CPL], double* __restrict__ part,
                                            int kp) {
  __shared__ double sh[kMW * 64 * CPL];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < CPL; ++q) sh[wv * 64 * CPL + lane * CPL + q] = acc[q];
  __syncthreads();
  for (int e = threadIdx.x; e < kp; e += kMT) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kMW; ++w) s += sh[w * 64 * CPL + e];
    part[(size_t)e * gridDim.x + blockIdx.x] = s;
  }
}

constexpr int kFT = 256;  // threads of a finaliser workgroup (one per column)

// Fixed-order sum of column c's partials over nb workgroups by the kFT
// threads of the calling workgroup; every thread must call it and receives the
// total.
__device__ __forceinline__ double col_total(const double* __restrict__ part, int nb, int c) {
  __shared__ double sh[kFT / 64];
  const int t = threadIdx.x;
  double s = 0.0;
  for (int b = t; b < nb; b += kFT) s += part[(size_t)c * nb + b];
  s = wave_sum_f64(s);
  if ((t & 63) == 0) sh[t >> 6] = s;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

__device__ __forceinline__ zd zinv(zd a) { return zdiv(zd{1.0, 0.0}, a); }

}  // namespace

// r = b (rows gathered through perm), p = 0, every shift's p^s = x^s = 0;
// partials of b^T b.
template <int CPL>
__global__ __launch_bounds__(kMT) void k_ms_init(int n, int k, int kp, int nz,
                                                 const int* __restrict__ perm,
                                                 const double* __restrict__ B, int ldb,
                                                 double* __restrict__ r, double* __restrict__ p,
                                                 cpx<double>* __restrict__ X,
                                                 cpx<double>* __restrict__ Ps,
                                                 double* __restrict__ y,
                                                 double* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  double acc[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q] = 0.0;
  const Rows rw = my_rows(n);
  const size_t blk = (size_t)n * kp;
  for (int t = 0; t < rw.count; ++t) {
    const int row = rw.first + rw.stride * t;
    const int src = perm[row];
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int c = lane * CPL + q;
      const double v = c < k ? B[(size_t)src * ldb + c] : 0.0;
      const size_t o = (size_t)row * kp + c;
      r[o] = v;
      p[o] = 0.0;
      if (y) y[o] = 0.0;
      for (int j = 0; j < nz; ++j) {
        if (!y) X[j * blk + o] = cpx<double>{0.0, 0.0};
        Ps[j * blk + o] = cpx<double>{0.0, 0.0};
      }
      acc[q] += v * v;
    }
  }
  put_partial<CPL>(acc, part, kp);
}

// Column state after the start: |b|, r^T r, the seed scalars and every
// shift's pi; a system with b = 0 is done at once (x = 0).
__global__ __launch_bounds__(kFT) void k_ms_fin0(int k, int nz, int nb, int kp,
                                                 const double* __restrict__ part, MsCols cols) {
  const int c = blockIdx.x;
  const double tot = col_total(part, nb, c);
  const double rr = c < k ? tot : 0.0;
  const int lv = rr > 0.0 ? 1 : 0;
  for (int j = threadIdx.x; j < nz; j += kFT) {
    const int e = j * kp + c;
    cols.pi[e] = cpx<double>{1.0, 0.0};
    cols.pi_prev[e] = cpx<double>{1.0, 0.0};
    cols.bs[e] = cpx<double>{0.0, 0.0};
    cols.live[e] = lv;
    cols.its[e] = 0;
    cols.est[e] = 0.0;
  }
  if (threadIdx.x != 0) return;
  cols.rr[c] = rr;
  cols.bn[c] = sqrt(rr);
  cols.alpha[c] = 0.0;
  cols.alpha_prev[c] = 1.0;
  cols.beta_prev[c] = 0.0;
  cols.scale[c] = 1.0;
  cols.colive[c] = lv;
}

// Seed search direction p = s (r + beta p) for the live columns; with a
// rescale s != 1 the residual is scaled too.
template <int CPL>
__global__ __launch_bounds__(kMT) void k_ms_pupd(int n, int kp, MsCols cols,
                                                 double* __restrict__ r, double* __restrict__ p) {
  const int lane = threadIdx.x & 63;
  double beta[CPL], sc[CPL];
  bool on[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int c = lane * CPL + q;
    on[q] = cols.colive[c] != 0;
    beta[q] = cols.beta_prev[c];
    sc[q] = cols.scale[c];
  }
  const Rows rw = my_rows(n);
  for (int t = 0; t < rw.count; ++t) {
    const size_t o = (size_t)(rw.first + rw.stride * t) * kp + lane * CPL;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!on[q]) continue;
      const double rv = r[o + q];
      p[o + q] = sc[q] * (rv + beta[q] * p[o + q]);
      if (sc[q] != 1.0) r[o + q] = sc[q] * rv;
    }
  }
}

// w = M p = A p - s p on the live columns (a wave per row, the row's entries
// broadcast from the lanes that loaded them, neighbour rows of p gathered
// eight at a time); partials of p^T w.
template <int CPL>
__global__ __launch_bounds__(kMT) void k_ms_spmv(int n, int kp, const int* __restrict__ rowptr,
                                                 const int* __restrict__ col,
                                                 const double* __restrict__ val, double shift,
                                                 const int* __restrict__ colive,
                                                 const double* __restrict__ p,
                                                 double* __restrict__ w,
                                                 double* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int cl = lane * CPL;
  bool on[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) on[q] = colive[cl + q] != 0;
  double acc[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q] = 0.0;
  const Rows rw = my_rows(n);
  for (int t = 0; t < rw.count; ++t) {
    const int row = rw.first + rw.stride * t;
    const int s = rowptr[row], e = rowptr[row + 1];
    const size_t ro = (size_t)row * kp + cl;
    double a[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) a[q] = 0.0;
    for (int base = s; base < e; base += 64) {
      const int m = min(64, e - base);
      // lane l holds entry base + l (own row with value 0 past the end)
      int mc = row;
      double mv = 0.0;
      if (lane < m) {
        mc = col[base + lane];
        mv = val[base + lane];
      }
      for (int t0 = 0; t0 < m; t0 += 8) {
        int jj[8];
        double av[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          jj[u] = __builtin_amdgcn_readlane(mc, t0 + u);
          av[u] = readlane_f64(mv, t0 + u);
        }
        double pv[8][CPL];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) pv[u][q] = p[(size_t)jj[u] * kp + cl + q];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) a[q] = fma(av[u], pv[u][q], a[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!on[q]) continue;
      const double pr = p[ro + q];
      const double wv = a[q] - shift * pr;
      w[ro + q] = wv;
      acc[q] += pr * wv;
    }
  }
  put_partial<CPL>(acc, part, kp);
}

// What a shift's thread of a finaliser reads (nothing past the last shift).
struct ShiftState {
  cpx<double> pi{}, pi_prev{}, bs{};
  int live = 0;
};
__device__ __forceinline__ ShiftState load_shift(const MsCols& cols, int j, int nz, int kp,
                                                 int c) {
  ShiftState v;
  if (j < nz) {
    const int e = j * kp + c;
    v.pi = cols.pi[e];
    v.pi_prev = cols.pi_prev[e];
    v.bs = cols.bs[e];
    v.live = cols.live[e];
  }
  return v;
}

// alpha_k of every live column, then for each shift (a thread each) pi_{k+1}
// and the scalars of iteration k's shifted update, kept in their slot:
// 1 / pi_k, beta^s_{k-1} and alpha^s_k = alpha_k pi_k / pi_{k+1}.
__global__ __launch_bounds__(kFT) void k_ms_fin_alpha(int kp, int k, int nz, int nb, int slot,
                                                      const double* __restrict__ part,
                                                      const cpx<double>* __restrict__ sig,
                                                      const double* __restrict__ g,
                                                      MsCols cols) {
  const int c = blockIdx.x;
  // everything that does not wait for the sum is loaded with its terms: a chain
  // of dependent loads is what such a small kernel spends its time on
  const int alive = cols.colive[c];
  const double rr = cols.rr[c], beta_prev = cols.beta_prev[c], alpha_prev = cols.alpha_prev[c];
  ShiftState v = load_shift(cols, threadIdx.x, nz, kp, c);
  const double pw = col_total(part, nb, c);
  const double alpha = pw != 0.0 ? rr / pw : 0.0;
  const double cc = beta_prev * alpha / alpha_prev;
  for (int j = threadIdx.x; j < nz; j += kFT) {
    if (j >= kFT) v = load_shift(cols, j, nz, kp, c);
    const int e = j * kp + c;
    const bool lv = alive && v.live;
    cpx<double>* sc = cols.sc + (size_t)((slot * nz + j) * 3) * kp + c;
    cols.on[(slot * nz + j) * kp + c] = lv ? 1 : 0;
    if (!lv) continue;
    const zd pk{v.pi.re, v.pi.im}, pm{v.pi_prev.re, v.pi_prev.im};
    const zd f{1.0 + cc + alpha * sig[j].re, alpha * sig[j].im};
    const zd fp = zmul(f, pk);
    const zd pn{fp.re - cc * pm.re, fp.im - cc * pm.im};
    cols.pi_next[e] = cpx<double>{pn.re, pn.im};
    const zd q = zdiv(pk, pn);
    const zd ip = zinv(pk);
    zd as{alpha * q.re, alpha * q.im};
    // combining mode: the weight of this step's update of x^s
    if (g) as = zmul(zd{g[2 * (j * k + c)], g[2 * (j * k + c) + 1]}, as);
    sc[0] = cpx<double>{ip.re, ip.im};
    sc[kp] = v.bs;
    sc[2 * kp] = cpx<double>{as.re, as.im};
  }
  if (threadIdx.x == 0) {
    cols.scale[c] = 1.0;  // a rescale has been applied by the direction update
    if (alive) cols.alpha[c] = alpha;
  }
}

// r_{k+1} = r_k - alpha w into the next slot, or over r_k (INPLACE: there is one
// slot, and rnext is it), partials of its r^T r.
template <int CPL, bool INPLACE>
__global__ __launch_bounds__(kMT) void k_ms_rupd(int n, int kp, MsCols cols,
                                                 const double* __restrict__ r,
                                                 double* __restrict__ rnext,
                                                 const double* __restrict__ w,
                                                 double* __restrict__ part) {
  const int cl = (threadIdx.x & 63) * CPL;
  double alpha[CPL], acc[CPL];
  bool on[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    on[q] = cols.colive[cl + q] != 0;
    alpha[q] = cols.alpha[cl + q];
    acc[q] = 0.0;
  }
  const Rows rw = my_rows(n);
  for (int t = 0; t < rw.count; ++t) {
    const size_t o = (size_t)(rw.first + rw.stride * t) * kp + cl;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!on[q]) continue;
      const double rn = (INPLACE ? rnext : r)[o + q] - alpha[q] * w[o + q];
      rnext[o + q] = rn;
      acc[q] += rn * rn;
    }
  }
  put_partial<CPL>(acc, part, kp);
}

// The shifted updates of ns deferred iterations, in order, for shifts j0 ..
// j0 + NZ - 1 (those below nz): with r_s the residual in slot s,
//   p = r_s / pi + beta^s p,  then y += Re(g alpha^s p) (COMB) or x += alpha^s p.
// A wave takes kSR rows of 64 columns at a time, all their loads together; the
// scalars come from LDS once for the kSR rows.  What bounds it is memory (the
// directions, 32 bytes a row, column and shift for ns iterations); one pass
// per iteration took 27 us on 30,000 rows, 64 columns and 4 shifts, this
// 50 us for four (6.6 TB/s).
constexpr int kSW = 8;   // waves
constexpr int kSR = 4;   // rows of a wave's step
template <int NZ, bool COMB>
__global__ __launch_bounds__(64 * kSW) void k_ms_shift(int n, int kp, int nz, int j0, int ns,
                                                       MsCols cols, const double* __restrict__ r,
                                                       double* __restrict__ y,
                                                       cpx<double>* __restrict__ X,
                                                       cpx<double>* __restrict__ P) {
  extern __shared__ cpx<double> sc[];  // [slot][shift][3][64]
  const int lane = threadIdx.x & 63, c = blockIdx.y * 64 + lane;
  const int wave = wave_id();
  for (int e = threadIdx.x; e < ns * NZ * 3 * 64; e += 64 * kSW) {
    const int l = e & 63, q = (e >> 6) % 3, j = (e >> 6) / 3 % NZ, s = (e >> 6) / (3 * NZ);
    cpx<double> v{0.0, 0.0};
    if (j0 + j < nz)
      v = cols.sc[(size_t)((s * nz + j0 + j) * 3 + q) * kp + blockIdx.y * 64 + l];
    sc[e] = v;
  }
  // bit j of live[s]: shift j0 + j iterated in slot s (it never starts again)
  int live[kMsDefer];
#pragma unroll
  for (int s = 0; s < kMsDefer; ++s) {
    live[s] = 0;
    for (int j = 0; j < NZ && s < ns && j0 + j < nz; ++j)
      live[s] |= (cols.on[(s * nz + j0 + j) * kp + c] != 0) << j;
  }
  const bool any = live[0] != 0;
  __syncthreads();
  if (__ballot(any) == 0) return;  // the same columns in every wave
  const size_t blk = (size_t)n * kp;
  // rows: contiguous stripes, one per XCD, swept by its workgroups side by side
  const int x = blockIdx.x & 7, per_x = gridDim.x >> 3, stripe = (n + 7) / 8;
  const int hi = min(n, (x + 1) * stripe);
  for (int row0 = x * stripe + ((blockIdx.x >> 3) * kSW + wave) * kSR; row0 < hi;
       row0 += per_x * kSW * kSR) {
    double rv[kMsDefer][kSR], yv[kSR];
    cpx<double> p[NZ][kSR], xv[COMB ? 1 : NZ][kSR];
    size_t o[kSR];
#pragma unroll
    for (int i = 0; i < kSR; ++i) o[i] = (size_t)min(row0 + i, hi - 1) * kp + c;
#pragma unroll
    for (int i = 0; i < kSR; ++i) {
#pragma unroll
      for (int s = 0; s < kMsDefer; ++s) rv[s][i] = live[s] ? r[s * blk + o[i]] : 0.0;
      yv[i] = COMB && any ? y[o[i]] : 0.0;
#pragma unroll
      for (int j = 0; j < NZ; ++j) {
        p[j][i] = cpx<double>{0.0, 0.0};
        if (!COMB) xv[COMB ? 0 : j][i] = cpx<double>{0.0, 0.0};
        if (live[0] >> j & 1) {
          p[j][i] = P[(j0 + j) * blk + o[i]];
          if (!COMB) xv[COMB ? 0 : j][i] = X[(j0 + j) * blk + o[i]];
        }
      }
    }
#pragma unroll
    for (int s = 0; s < kMsDefer; ++s) {
      if (s >= ns) break;
#pragma unroll
      for (int j = 0; j < NZ; ++j) {
        if (!(live[s] >> j & 1)) continue;
        const cpx<double>* q = sc + ((s * NZ + j) * 3) * 64 + lane;
        const cpx<double> ip = q[0], b = q[64], a = q[128];
#pragma unroll
        for (int i = 0; i < kSR; ++i) {
          const cpx<double> po = p[j][i];
          const double pr = rv[s][i] * ip.re + (b.re * po.re - b.im * po.im);
          const double pi = rv[s][i] * ip.im + (b.re * po.im + b.im * po.re);
          p[j][i] = cpx<double>{pr, pi};
          if (COMB) {
            yv[i] += a.re * pr - a.im * pi;
          } else {
            xv[COMB ? 0 : j][i].re += a.re * pr - a.im * pi;
            xv[COMB ? 0 : j][i].im += a.re * pi + a.im * pr;
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kSR; ++i) {
      if (row0 + i >= hi) break;
      if (COMB && any) y[o[i]] = yv[i];
#pragma unroll
      for (int j = 0; j < NZ; ++j) {
        if (!(live[0] >> j & 1)) continue;
        P[(j0 + j) * blk + o[i]] = p[j][i];
        if (!COMB) X[(j0 + j) * blk + o[i]] = xv[COMB ? 0 : j][i];
      }
    }
  }
}

// beta_k, beta^s_k = beta_k (pi_k / pi_{k+1})^2, the pi shift, the
// convergence test |r_{k+1}| / |pi_{k+1}| <= tol |b| (or the iteration cap), a
// shift to a thread, and the rescale of a column whose seed residual has
// fallen below 1e-100 |b|.
__global__ __launch_bounds__(kFT) void k_ms_fin_beta(int kp, int nz, int nb,
                                                     const double* __restrict__ part, double tol,
                                                     int maxit, MsCols cols) {
  __shared__ int left;
  const int c = blockIdx.x;
  const int alive = cols.colive[c];
  const double rr = cols.rr[c], bn = cols.bn[c], alpha = cols.alpha[c];
  const int j0 = threadIdx.x, e0 = j0 * kp + c;
  cpx<double> pi0{}, pn0{};
  int live0 = 0, its0 = 0;
  if (j0 < nz) {
    pi0 = cols.pi[e0];
    pn0 = cols.pi_next[e0];
    live0 = cols.live[e0];
    its0 = cols.its[e0];
  }
  if (threadIdx.x == 0) left = 0;
  const double rn = col_total(part, nb, c);  // a barrier inside
  if (!alive) return;  // uniform over the workgroup
  const double beta = rr > 0.0 ? rn / rr : 0.0;
  const double rnorm = sqrt(rn);
  for (int j = threadIdx.x; j < nz; j += kFT) {
    const int e = j * kp + c;
    if (j >= kFT) {
      pi0 = cols.pi[e];
      pn0 = cols.pi_next[e];
      live0 = cols.live[e];
      its0 = cols.its[e];
    }
    if (!live0) continue;
    const zd pk{pi0.re, pi0.im}, pn{pn0.re, pn0.im};
    const zd q = zdiv(pk, pn);
    const zd q2 = zmul(q, q);
    cols.bs[e] = cpx<double>{beta * q2.re, beta * q2.im};
    cols.pi_prev[e] = pi0;
    cols.pi[e] = pn0;
    cols.its[e] = its0 + 1;
    const double est = rnorm / sqrt(pn.re * pn.re + pn.im * pn.im);
    cols.est[e] = bn > 0.0 ? est / bn : 0.0;
    if (est <= tol * bn || its0 + 1 >= maxit)
      cols.live[e] = 0;
    else
      left = 1;
  }
  __syncthreads();
  const bool go = left != 0;
  const bool rescale = go && rn > 0.0 && rn < 1e-200 * bn * bn;
  const double s = 1e100;
  if (rescale)
    for (int j = threadIdx.x; j < nz; j += kFT) {
      const int e = j * kp + c;
      cols.pi[e] = cpx<double>{cols.pi[e].re * s, cols.pi[e].im * s};
      cols.pi_prev[e] = cpx<double>{cols.pi_prev[e].re * s, cols.pi_prev[e].im * s};
    }
  if (threadIdx.x != 0) return;
  cols.alpha_prev[c] = alpha;
  cols.beta_prev[c] = beta;
  cols.rr[c] = rescale ? rn * s * s : rn;
  if (rescale) cols.scale[c] = s;
  cols.colive[c] = go ? 1 : 0;
}

// True residual of shift j: partials of |b - (z_j I - A) d|^2 with d = -x^s_j,
// i.e. of |b + z_j x - A x|^2 (a complex SpMV over x^s_j).
template <int CPL>
__global__ __launch_bounds__(kMT) void k_ms_true(int n, int k, int kp,
                                                 const int* __restrict__ rowptr,
                                                 const int* __restrict__ col,
                                                 const double* __restrict__ val,
                                                 const int* __restrict__ perm,
                                                 const double* __restrict__ B, int ldb,
                                                 double zre, double zim,
                                                 const cpx<double>* __restrict__ x,
                                                 double* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int cl = lane * CPL;
  double acc[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q] = 0.0;
  const Rows rw = my_rows(n);
  for (int t = 0; t < rw.count; ++t) {
    const int row = rw.first + rw.stride * t;
    const int s = rowptr[row], e = rowptr[row + 1];
    double ar[CPL], ai[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) ar[q] = ai[q] = 0.0;
    for (int base = s; base < e; base += 64) {
      const int m = min(64, e - base);
      int mc = row;
      double mv = 0.0;
      if (lane < m) {
        mc = col[base + lane];
        mv = val[base + lane];
      }
      for (int u = 0; u < m; ++u) {
        const int j = __builtin_amdgcn_readlane(mc, u);
        const double a = readlane_f64(mv, u);
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          const cpx<double> v = x[(size_t)j * kp + cl + q];
          ar[q] = fma(a, v.re, ar[q]);
          ai[q] = fma(a, v.im, ai[q]);
        }
      }
    }
    const size_t src = (size_t)perm[row] * ldb;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int c = cl + q;
      if (c >= k) continue;
      const cpx<double> v = x[(size_t)row * kp + c];
      const double sr = B[src + c] + (zre * v.re - zim * v.im) - ar[q];
      const double si = (zre * v.im + zim * v.re) - ai[q];
      acc[q] += sr * sr + si * si;
    }
  }
  put_partial<CPL>(acc, part, kp);
}

// resid[j k + c] = sqrt(sum of the partials) / |b_c| (0 for b_c = 0).
__global__ __launch_bounds__(kFT) void k_ms_fin_true(int k, int kp, int j, int nb,
                                                     const double* __restrict__ part,
                                                     const double* __restrict__ bn,
                                                     double* __restrict__ resid) {
  const int c = blockIdx.x;
  const double s2 = col_total(part, nb, c);
  if (threadIdx.x != 0 || c >= k) return;
  resid[(size_t)j * k + c] = bn[c] > 0.0 ? sqrt(s2) / bn[c] : 0.0;
}

// D[perm[row]][j k + c] = -x^s_j (the solution of (z_j I - A) d = b).
template <int CPL>
__global__ __launch_bounds__(kMT) void k_ms_out(int n, int k, int kp, int nz,
                                                const int* __restrict__ perm,
                                                const cpx<double>* __restrict__ X,
                                                cpx<double>* __restrict__ D, int ldd) {
  const int lane = threadIdx.x & 63;
  const Rows rw = my_rows(n);
  const size_t blk = (size_t)n * kp;
  for (int t = 0; t < rw.count; ++t) {
    const int row = rw.first + rw.stride * t;
    const size_t dst = (size_t)perm[row] * ldd;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int c = lane * CPL + q;
      if (c >= k) continue;
      for (int j = 0; j < nz; ++j) {
        const cpx<double> x = X[j * blk + (size_t)row * kp + c];
        D[dst + (size_t)j * k + c] = cpx<double>{-x.re, -x.im};
      }
    }
  }
}

// Combining mode output: Qt[perm[row]][c] = gq_c Qin[perm[row]][c] - y[row][c]
// (d = -x, so the weighted sum of the solutions is -y) with
// gq_c = sum_j Re(g_{j,c}) (the residual form's q term; Qin null: 0).
template <int CPL>
__global__ __launch_bounds__(kMT) void k_ms_out_y(int n, int k, int kp, int nz,
                                                  const int* __restrict__ perm,
                                                  const double* __restrict__ y,
                                                  const double* __restrict__ g,
                                                  const double* __restrict__ Qin, int ldqin,
                                                  double* __restrict__ Qt, int ldq) {
  const int lane = threadIdx.x & 63;
  double gq[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int c = lane * CPL + q;
    double s = 0.0;
    if (c < k && Qin)
      for (int j = 0; j < nz; ++j) s += g[2 * (j * k + c)];
    gq[q] = s;
  }
  const Rows rw = my_rows(n);
  for (int t = 0; t < rw.count; ++t) {
    const int row = rw.first + rw.stride * t;
    const size_t dst = (size_t)perm[row];
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int c = lane * CPL + q;
      if (c >= k) continue;
      const double qv = Qin ? gq[q] * Qin[dst * ldqin + c] : 0.0;
      Qt[dst * ldq + c] = qv - y[(size_t)row * kp + c];
    }
  }
}

// iters[j k + c] and resid[j k + c] (estimated relative residual) per system.
__global__ void k_ms_report(int k, int kp, int nz, MsCols cols, int* __restrict__ iters,
                            double* __restrict__ resid) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nz * k) return;
  const int j = e / k, c = e % k;
  if (iters) iters[e] = cols.its[j * kp + c];
  if (resid) resid[e] = cols.est[j * kp + c];
}

int ms_cpl(int k) { return (k + 63) / 64; }
int ms_padded(int k) { return 64 * ms_cpl(k); }
int ms_blocks(int n, int num_cu) {
  int nb = num_cu * 4;
  const int need = (n + kMW - 1) / kMW;
  if (nb > need) nb = (need + 7) / 8 * 8;
  return nb < 8 ? 8 : nb;
}
// k_ms_shift's row blocks: as many workgroups as are resident at once, always a
// multiple of the eight stripes that its rows are cut into.
int ms_shift_blocks(int n, int num_cu, int shifts) {
  const int most = num_cu * (shifts <= 4 ? 2 : 1) / 8 * 8;
  const int need = (n + kSR * kSW - 1) / (kSR * kSW);
  const int nb = need < most ? (need + 7) / 8 * 8 : most;
  return nb < 8 ? 8 : nb;
}

namespace {

// The deferred iterations (ns of them) applied to all shifts, a launch for each
// few (what a lane's registers and the scalars' LDS hold).
template <int NZ, bool COMB>
hipError_t launch_shift(hipStream_t st, int n, int ns, const MsWork& W, int nz, int j0) {
  const size_t lds = (size_t)kMsDefer * NZ * 3 * 64 * sizeof(cpx<double>);
  auto fn = k_ms_shift<NZ, COMB>;
  hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  const int nb = ms_shift_blocks(n, W.num_cu, NZ);
  hipLaunchKernelGGL(fn, dim3(nb, W.kp / 64), dim3(64 * kSW), lds, st, n, W.kp, nz, j0, ns, W.cols,
                     W.r, W.y, W.X, W.P);
  return hipGetLastError();
}

hipError_t shift_pass(hipStream_t st, int n, int ns, const MsWork& W, int nz, bool comb) {
  for (int j0 = 0; j0 < nz;) {
    const int left = nz - j0;
    hipError_t e;
    if (comb) {
      if (left > 4) {
        e = launch_shift<8, true>(st, n, ns, W, nz, j0);
        j0 += 8;
      } else if (left > 2) {
        e = launch_shift<4, true>(st, n, ns, W, nz, j0);
        j0 += 4;
      } else {
        e = launch_shift<2, true>(st, n, ns, W, nz, j0);
        j0 += 2;
      }
    } else if (left > 2) {
      e = launch_shift<4, false>(st, n, ns, W, nz, j0);
      j0 += 4;
    } else {
      e = launch_shift<2, false>(st, n, ns, W, nz, j0);
      j0 += 2;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int CPL>
hipError_t run_ms_t(hipStream_t st, const StreamMatrix& A, const MsWork& W, const MsLaunch& L) {
  const int n = A.n, k = L.k, kp = W.kp, nz = L.nz;
  const int nb = W.nb;
  const dim3 grid(nb), blk(kMT), fg(kp), fb(kFT);
  const size_t rblk = (size_t)n * kp;
#define MCHK(expr)                   \
  do {                               \
    hipError_t _e = (expr);          \
    if (_e != hipSuccess) return _e; \
  } while (0)
#define MLAUNCH(...)                 \
  do {                               \
    hipLaunchKernelGGL(__VA_ARGS__); \
    MCHK(hipGetLastError());         \
  } while (0)
  // shifts of the seed form: sigma_j = s - z_j
  std::vector<cpx<double>> sg(nz);
  for (int j = 0; j < nz; ++j) sg[j] = cpx<double>{L.seed - L.z[2 * j], -L.z[2 * j + 1]};
  MCHK(hipMemcpyAsync(W.sig, sg.data(), nz * sizeof(cpx<double>), hipMemcpyHostToDevice, st));
  const bool comb = L.g != nullptr;
  double* yb = comb ? W.y : nullptr;
  MLAUNCH((k_ms_init<CPL>), grid, blk, 0, st, n, k, kp, nz, A.perm, L.B, L.ldb, W.r, W.p, W.X,
          W.P, yb, W.part);
  MLAUNCH(k_ms_fin0, fg, fb, 0, st, k, nz, nb, kp, W.part, W.cols);
  std::vector<int> colive(kp);
  auto census = [&](int& live) -> hipError_t {
    MCHK(hipMemcpyAsync(colive.data(), W.cols.colive, kp * sizeof(int), hipMemcpyDeviceToHost,
                        st));
    MCHK(hipStreamSynchronize(st));
    live = 0;
    for (int c = 0; c < kp; ++c) live += colive[c];
    return hipSuccess;
  };
  int live = 0, it = 0;
  MCHK(census(live));
  // seed residual r_k in slot k mod W.defer of W.r
  for (; it < L.maxit && live > 0; ++it) {
    const int slot = it % W.defer;
    double* r = W.r + slot * rblk;
    MLAUNCH((k_ms_pupd<CPL>), grid, blk, 0, st, n, kp, W.cols, r, W.p);
    MLAUNCH((k_ms_spmv<CPL>), grid, blk, 0, st, n, kp, A.rowptr, A.col, A.val64, L.seed,
            W.cols.colive, W.p, W.w, W.part);
    MLAUNCH(k_ms_fin_alpha, fg, fb, 0, st, kp, k, nz, nb, slot, W.part, W.sig, L.g, W.cols);
    if (slot == W.defer - 1) MCHK(shift_pass(st, n, W.defer, W, nz, comb));
    if (W.defer > 1)
      MLAUNCH((k_ms_rupd<CPL, false>), grid, blk, 0, st, n, kp, W.cols, r,
              W.r + (it + 1) % W.defer * rblk, W.w, W.part);
    else
      MLAUNCH((k_ms_rupd<CPL, true>), grid, blk, 0, st, n, kp, W.cols, (const double*)nullptr, r,
              W.w, W.part);
    MLAUNCH(k_ms_fin_beta, fg, fb, 0, st, kp, nz, nb, W.part, L.tol, L.maxit, W.cols);
    if ((it + 1) % L.chunk == 0 || it + 1 == L.maxit) MCHK(census(live));
  }
  // iterations since the last pass: their residuals are still in slots 0, 1, ...
  if (it % W.defer) MCHK(shift_pass(st, n, it % W.defer, W, nz, comb));
  if (comb) {
    MLAUNCH((k_ms_out_y<CPL>), grid, blk, 0, st, n, k, kp, nz, A.perm, yb, L.g, L.Qin, L.ldqin,
            L.Qt, L.ldq);
    if (L.iters)
      MLAUNCH(k_ms_report, dim3((nz * k + 255) / 256), dim3(256), 0, st, k, kp, nz, W.cols,
              L.iters, (double*)nullptr);
    return hipSuccess;
  }
  MLAUNCH((k_ms_out<CPL>), grid, blk, 0, st, n, k, kp, nz, A.perm, W.X,
          static_cast<cpx<double>*>(L.D), L.ldd);
  if (L.iters)
    MLAUNCH(k_ms_report, dim3((nz * k + 255) / 256), dim3(256), 0, st, k, kp, nz, W.cols, L.iters,
            (double*)nullptr);
  if (L.resid) {
    const size_t bsz = (size_t)n * kp;
    for (int j = 0; j < nz; ++j) {
      MLAUNCH((k_ms_true<CPL>), grid, blk, 0, st, n, k, kp, A.rowptr, A.col, A.val64, A.perm,
              L.B, L.ldb, L.z[2 * j], L.z[2 * j + 1], W.X + j * bsz, W.part);
      MLAUNCH(k_ms_fin_true, fg, fb, 0, st, k, kp, j, nb, W.part, W.cols.bn, L.resid);
    }
  }
  return hipSuccess;
#undef MLAUNCH
#undef MCHK
}

}  // namespace

hipError_t run_mshift(hipStream_t st, const StreamMatrix& A, const MsWork& W, const MsLaunch& L) {
  if (L.k < 1 || L.nz < 1 || L.k > W.kp || W.kp != ms_padded(L.k) || L.nz > W.nz || !A.val64 ||
      W.defer < 1 || W.defer > kMsDefer ||
      W.nb != ms_blocks(A.n, W.num_cu) || L.chunk < 1)
    return hipErrorInvalidValue;
  if (L.g ? (!W.y || !L.Qt || L.ldq < L.k || (L.Qin && L.ldqin < L.k))
          : (!W.X || !L.D || L.ldd < L.nz * L.k))
    return hipErrorInvalidValue;
  switch (ms_cpl(L.k)) {
    case 1: return run_ms_t<1>(st, A, W, L);
    case 2: return run_ms_t<2>(st, A, W, L);
    case 3: return run_ms_t<3>(st, A, W, L);
  }
  return hipErrorInvalidValue;
}

}  // namespace rafeast
