// Streaming COCG engine for systems too large to keep in one workgroup's LDS.
// All shifted systems (z_c I - A) d_c = b_c advance in lock step, one kernel
// sequence per iteration, and every vector is an n x Bp complex block in HBM,
// row-major: row r of a block holds the Bp columns' values contiguously, so
// the gather of a neighbour row is one coalesced read of 64 * CPL columns.
//
// Method: COCG on the unconjugated bilinear form, in the engine precision,
// with reliable updates in FP64: whenever a column's recursive residual has
// dropped by the factor delta since its last check (or below the tolerance,
// or the column hit its iteration cap), the engine folds x into the FP64
// solution x_hi, recomputes the true residual s = b - (zI - A) x_hi in FP64,
// and continues the same Krylov recurrence from r = s (the search direction
// is kept; beta is recomputed from s).  This removes the drift between the
// recursive and the true residual that FP32 storage causes, without the
// restarts that would throw away the recurrence.  The iteration restarts from
// p = s only after a breakdown (p^T (zI - A) p = 0) or a stall: a column
// whose recursive residual has not dropped by delta within 4x the length of
// its previous check interval (and 2x the first interval after its last
// start, the initial plateau a restart has to cross again) is checked early,
// and if its true residual has not at least halved since the last check, the
// recurrence starts afresh.
// Each column has its own scalars and a state on the device:
//   1  iterating
//   0  waiting for the FP64 residual check (reliable update)
//   3  waiting for the FP64 residual check after a breakdown (restart)
//   2  solved (true residual <= tol) or given up (iteration or update
//      budget spent, repeated breakdown); frozen
// Columns that are not in state 1 keep their vectors unchanged while the
// others iterate.  Checks run between chunks of iterations.
//
// Slots: x, r, p and w hold the columns that are not done side by side, in
// slots (slot u holds column slots.col[u]); x_hi keeps all columns in their
// order.  When so many columns are done that a unit of slots (the columns of
// kSL lanes) is left over, the others move together (k_s_move), with a row
// stride of what is left: shifts that converge early stop costing anything,
// and the slowest shift's few columns stay dense in memory.
//
// An iteration: K1 x += alpha p (the last iteration's) and p = r + beta p, K2
// the SpMV w = (zI - A) p gathering only p (a fused form that gathered r and
// the old p and formed p on the fly read twice the neighbour bytes, 20%
// slower), the finalisers turn partials into alpha and beta, K3 updates r.
// Row kernels: 256 threads (4 waves).  Each XCD sweeps one contiguous eighth
// of the rows with all its waves side by side (see row_steps), keeping the
// neighbour gathers in that XCD's L2.  A wave takes eight rows at a time, 8
// lanes each; a lane holds 16 bytes of a row: two FP32 complex columns or one
// FP64 complex column (the per-CU rate from L2 is set by load instructions).
// Reductions are per-workgroup partials, summed in a fixed order by a wave per
// column, so results are deterministic.
//
// What bounds it (random geometric graph of 16,000 points, 67 entries a row, 40
// right-hand sides, 4 shifts of 102 to 530 iterations, FP32): the SpMM 64 us
// with all 160 columns, 24 us with the last shift's 40, from the bytes its
// gathers move from L2 to the CUs (10 TB/s; more waves or rows in flight change
// nothing); the updates 17 and 6 us, memory; the finalisers 5 us each.  The
// whole solve 73.7 ms with groups of 128 columns skipped only when all of them
// were done, 42.1 ms with slots.  Units of 16 lanes (32 FP32 columns) are as
// fast on full blocks and 0-5% slower on the others.
#include <utility>

#include "device.h"
#include "kernels.h"

namespace rafeast {

namespace {

constexpr int kST = 256;             // threads of a row kernel
constexpr int kSW = kST / 64;        // waves of a row kernel
constexpr int kSL = 8;               // lanes of a row
constexpr int kSR = 64 / kSL;        // rows of a wave's step
constexpr int kFinCols = kST / 64;   // slots of a finaliser workgroup, a wave each

// Columns of a lane: 16 bytes.
template <typename T>
constexpr int lane_cols() { return 16 / (int)sizeof(cpx<T>); }
template <typename T>
constexpr int unit_cols() { return kSL * lane_cols<T>(); }

// Rows of a wave.  The rows are cut into 8 contiguous stripes, one per XCD
// (dispatch round-robins workgroup ids over the 8 XCDs, so workgroup b runs
// on XCD b mod 8); inside a stripe the XCD's waves take consecutive rows and
// sweep the stripe together, so the rows in flight on an XCD form a window of
// about (8 waves per XCD) rows and the neighbour rows a gather needs were
// loaded recently into the same L2.  Step k of this wave takes the rows
// first + k * stride .. + kSR - 1 below hi, k < count.
struct RowSteps {
  int first, stride, count, hi;
};

__device__ __forceinline__ RowSteps row_steps(int n) {
  const int nb = gridDim.x;  // a multiple of 8
  const int x = (int)(blockIdx.x % 8), i = (int)(blockIdx.x / 8), per_x = nb / 8;
  const int stripe = (n + 7) / 8;
  const int lo = min(n, x * stripe), hi = min(n, lo + stripe);
  const int stride = per_x * kSW * kSR;
  const int first = lo + (i * kSW + wave_id()) * kSR;
  return {first, stride, first < hi ? (hi - first + stride - 1) / stride : 0, hi};
}

__device__ __forceinline__ bool waiting(int st) { return st == 0 || st == 3; }

// Value of lane U of this lane's group of kSL (all lanes active): the LDS
// crossbar (no memory), since the vector unit is nearly as busy as the gathers.
template <int U>
__device__ __forceinline__ int row_bcast(int v) {
  static_assert(kSL == 8);
  return __builtin_amdgcn_ds_swizzle(v, (U << 5) | 0x18);
}
template <int U>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(row_bcast<U>(__float_as_int(v)));
}
template <int U>
__device__ __forceinline__ double row_bcast(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = row_bcast<U>((int)(b & 0xffffffffLL)), hi = row_bcast<U>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The kSL entries that each row's lanes hold: indices and values.
template <typename T, int... U>
__device__ __forceinline__ void entries_of(int mc, T mv, int (&j)[kSL], T (&a)[kSL],
                                           std::integer_sequence<int, U...>) {
  ((j[U] = row_bcast<U>(mc), a[U] = row_bcast<U>(mv)), ...);
}

template <typename T, int CPL>
struct Chunk {
  cpx<T> v[CPL];
};

template <typename T, int CPL>
__device__ __forceinline__ Chunk<T, CPL> ld(const cpx<T>* __restrict__ p) {
  Chunk<T, CPL> c;
#pragma unroll
  for (int q = 0; q < CPL; ++q) c.v[q] = p[q];
  return c;
}

template <typename T, int CPL>
__device__ __forceinline__ void st(cpx<T>* __restrict__ p, const Chunk<T, CPL>& c) {
#pragma unroll
  for (int q = 0; q < CPL; ++q) p[q] = c.v[q];
}

// The same as a non-temporal store: the value streams past L2 (written once,
// read by a later kernel), which keeps L2 for the rows a gather reuses.
template <typename T, int CPL>
__device__ __forceinline__ void st_nt(cpx<T>* __restrict__ p, const Chunk<T, CPL>& c) {
  T* f = reinterpret_cast<T*>(p);
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    __builtin_nontemporal_store(c.v[q].re, f + 2 * q);
    __builtin_nontemporal_store(c.v[q].im, f + 2 * q + 1);
  }
}

// Sum the workgroup's per-lane values (4 waves of kSR rows) and store its
// partials at part[((slot) * NQ + u) * gridDim.x + blockIdx.x], the unit's
// first slot being blockIdx.y * kSL * CPL.
template <int CPL, int NQ>
__device__ __forceinline__ void put_partials(const double (&acc)[CPL][NQ],
                                             double* __restrict__ part) {
  constexpr int kRow = kSL * CPL * NQ;  // values of a row's lanes
  __shared__ double sh[kSW * kSR * kRow];
  const int g = threadIdx.x / kSL, l = threadIdx.x % kSL;
#pragma unroll
  for (int q = 0; q < CPL; ++q)
#pragma unroll
    for (int u = 0; u < NQ; ++u) sh[g * kRow + (l * CPL + q) * NQ + u] = acc[q][u];
  __syncthreads();
  for (int e = threadIdx.x; e < kRow; e += kST) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kSW * kSR; ++w) s += sh[w * kRow + e];
    part[((size_t)blockIdx.y * kRow + e) * gridDim.x + blockIdx.x] = s;
  }
}

// Slot of a finaliser's wave.
__device__ __forceinline__ int fin_slot() { return blockIdx.x * kFinCols + wave_id(); }

// Fixed-order sums of slot s's partials over nb workgroups, in every lane.
template <int NQ>
__device__ __forceinline__ void slot_sums(const double* __restrict__ part, int nb, int s,
                                          double (&out)[NQ]) {
#pragma unroll
  for (int u = 0; u < NQ; ++u) out[u] = 0.0;
  for (int b = threadIdx.x & 63; b < nb; b += 64)
#pragma unroll
    for (int u = 0; u < NQ; ++u) out[u] += part[((size_t)s * NQ + u) * nb + b];
#pragma unroll
  for (int u = 0; u < NQ; ++u) out[u] = wave_sum_f64(out[u]);
}

// This lane's place: its row of the step and its first slot.
__device__ __forceinline__ int lane_row() { return (threadIdx.x & 63) / kSL; }
template <int CPL>
__device__ __forceinline__ int lane_slot() {
  return ((int)blockIdx.y * kSL + (int)(threadIdx.x % kSL)) * CPL;
}

}  // namespace

// K1: for the iterating columns x += alpha p with the last iteration's alpha
// (whose p is read here anyway), then the new direction p = r + beta p.
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_pupd(int n, int S, StreamSlots sl,
                                                const cpx<T>* __restrict__ r,
                                                cpx<T>* __restrict__ x, cpx<T>* __restrict__ p) {
  const int s0 = lane_slot<CPL>();
  T are[CPL], aim[CPL], bre[CPL], bim[CPL];
  bool live[CPL], any = false;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    are[q] = T(sl.alpha[2 * (s0 + q)]);
    aim[q] = T(sl.alpha[2 * (s0 + q) + 1]);
    bre[q] = T(sl.beta[2 * (s0 + q)]);
    bim[q] = T(sl.beta[2 * (s0 + q) + 1]);
    live[q] = sl.state[s0 + q] == 1;
    any = any || live[q];
  }
  if (!any) return;
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * S + s0;
    const Chunk<T, CPL> r0 = ld<T, CPL>(r + ro);
    Chunk<T, CPL> p0 = ld<T, CPL>(p + ro), x0 = ld<T, CPL>(x + ro);
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!live[q]) continue;
      const cpx<T> po = p0.v[q];
      x0.v[q].re += are[q] * po.re - aim[q] * po.im;
      x0.v[q].im += are[q] * po.im + aim[q] * po.re;
      p0.v[q].re = r0.v[q].re + bre[q] * po.re - bim[q] * po.im;
      p0.v[q].im = r0.v[q].im + bre[q] * po.im + bim[q] * po.re;
    }
    st<T, CPL>(x + ro, x0);
    st<T, CPL>(p + ro, p0);
  }
}

// kSL entries of each of the wave's rows: their rows of p gathered together,
// then added in order.
template <typename T, int CPL>
__device__ __forceinline__ void gather(int mc, T mv, const cpx<T>* __restrict__ p, int S,
                                       T (&ar)[CPL], T (&ai)[CPL]) {
  int j[kSL];
  T a[kSL];
  entries_of(mc, mv, j, a, std::make_integer_sequence<int, kSL>{});
  Chunk<T, CPL> pj[kSL];
#pragma unroll
  for (int u = 0; u < kSL; ++u) pj[u] = ld<T, CPL>(p + (size_t)j[u] * S);
#pragma unroll
  for (int u = 0; u < kSL; ++u)
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      ar[q] += a[u] * pj[u].v[q].re;
      ai[q] += a[u] * pj[u].v[q].im;
    }
}

// Walks the entries of the wave's rows, kSR rows side by side: a row's entries
// are held kSL at a time by its lanes (its own index with value 0 past its
// end), the next ones or the next step's first in flight while these are used.
template <typename V, class Begin, class Use, class End>
__device__ __forceinline__ void walk_rows(int n, const int* __restrict__ rowptr,
                                          const int* __restrict__ col,
                                          const V* __restrict__ val, Begin begin, Use use,
                                          End end) {
  const RowSteps rs = row_steps(n);
  const int l = threadIdx.x % kSL;
  auto bounds = [&](int k, int& row, bool& valid, int& s, int& len) {
    row = rs.first + rs.stride * k + lane_row();
    valid = k < rs.count && row < rs.hi;
    if (!valid) row = 0;
    s = rowptr[row];
    len = valid ? rowptr[row + 1] - s : 0;
  };
  auto entries = [&](int row, int s, int len, int base, int& mc, V& mv) {
    mc = row;
    mv = V(0);
    if (base + l < len) {
      mc = col[s + base + l];
      mv = val[s + base + l];
    }
  };
  if (rs.count == 0) return;
  int row, s, len, mc;
  bool valid;
  V mv;
  bounds(0, row, valid, s, len);
  entries(row, s, len, 0, mc, mv);
  for (int k = 0; k < rs.count; ++k) {
    int lm = 0;
#pragma unroll
    for (int g = 0; g < kSR; ++g) lm = max(lm, __builtin_amdgcn_readlane(len, g * kSL));
    int row_n, s_n, len_n;
    bool valid_n;
    bounds(k + 1, row_n, valid_n, s_n, len_n);
    begin(row, valid);
    for (int base = 0;; base += kSL) {
      const bool last = base + kSL >= lm;
      int mc_n;
      V mv_n;
      if (last)
        entries(row_n, s_n, len_n, 0, mc_n, mv_n);
      else
        entries(row, s, len, base + kSL, mc_n, mv_n);
      if (lm > base) use(mc, mv);
      mc = mc_n;
      mv = mv_n;
      if (last) break;
    }
    end(row, valid);
    row = row_n;
    s = s_n;
    len = len_n;
    valid = valid_n;
  }
}

// K2: w = (z I - A) p over the iterating columns (frozen ones give w = 0) and
// the partials of mu = p^T w.  Lanes of frozen columns gather a live column's
// bytes of the same row, which costs nothing, so that no lane is switched off
// while entries are broadcast.
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_spmm(int n, int S, const int* __restrict__ rowptr,
                                                const int* __restrict__ col,
                                                const T* __restrict__ val, StreamSlots sl,
                                                const cpx<T>* __restrict__ p,
                                                cpx<T>* __restrict__ w,
                                                double* __restrict__ part) {
  const int s0 = lane_slot<CPL>();
  T zre[CPL], zim[CPL];
  bool live[CPL], any = false;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    zre[q] = T(sl.zc[2 * (s0 + q)]);
    zim[q] = T(sl.zc[2 * (s0 + q) + 1]);
    live[q] = sl.state[s0 + q] == 1;
    any = any || live[q];
  }
  const unsigned long long who = __ballot(any);  // the unit's lanes, once per row
  if (who == 0) return;
  const int some = ((int)blockIdx.y * kSL + __builtin_ctzll(who) % kSL) * CPL;
  const cpx<T>* __restrict__ pg = p + (any ? s0 : some);
  double acc[CPL][2];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = acc[q][1] = 0.0;
  Chunk<T, CPL> p0;
  T ar[CPL], ai[CPL];
  walk_rows<T>(
      n, rowptr, col, val,
      [&](int row, bool) {
        p0 = ld<T, CPL>(pg + (size_t)row * S);
#pragma unroll
        for (int q = 0; q < CPL; ++q) ar[q] = ai[q] = T(0);
      },
      [&](int mc, T mv) { gather<T, CPL>(mc, mv, pg, S, ar, ai); },
      [&](int row, bool valid) {
        if (!valid || !any) return;
        Chunk<T, CPL> ww;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          if (live[q]) {
            ww.v[q].re = zre[q] * p0.v[q].re - zim[q] * p0.v[q].im - ar[q];
            ww.v[q].im = zre[q] * p0.v[q].im + zim[q] * p0.v[q].re - ai[q];
          } else {
            ww.v[q] = cpx<T>{T(0), T(0)};
          }
          const double pr = p0.v[q].re, pi = p0.v[q].im, wr_ = ww.v[q].re, wi = ww.v[q].im;
          acc[q][0] += pr * wr_ - pi * wi;
          acc[q][1] += pr * wi + pi * wr_;
        }
        // read by the update kernel, not by this sweep
        st_nt<T, CPL>(w + (size_t)row * S + s0, ww);
      });
  put_partials<CPL, 2>(acc, part);
}

// K3: r -= alpha w; partials of r^T r (complex) and ||r||^2.  With a dense
// operator w holds A p, and w = z p - A p is formed here.
template <typename T, int CPL, bool DENSE>
__global__ __launch_bounds__(kST) void k_s_update(int n, int S, StreamSlots sl,
                                                  cpx<T>* __restrict__ r,
                                                  const cpx<T>* __restrict__ p,
                                                  const cpx<T>* __restrict__ w,
                                                  double* __restrict__ part) {
  const int s0 = lane_slot<CPL>();
  T are[CPL], aim[CPL], zre[CPL], zim[CPL];
  bool live[CPL], any = false;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    are[q] = T(sl.alpha[2 * (s0 + q)]);
    aim[q] = T(sl.alpha[2 * (s0 + q) + 1]);
    zre[q] = DENSE ? T(sl.zc[2 * (s0 + q)]) : T(0);
    zim[q] = DENSE ? T(sl.zc[2 * (s0 + q) + 1]) : T(0);
    live[q] = sl.state[s0 + q] == 1;
    any = any || live[q];
  }
  if (__ballot(any) == 0) return;
  double acc[CPL][3];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0.0;
  const RowSteps rs = row_steps(n);
  for (int k = 0; any && k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * S + s0;
    Chunk<T, CPL> rr = ld<T, CPL>(r + ro), ww = ld<T, CPL>(w + ro), pp{};
    if (DENSE) pp = ld<T, CPL>(p + ro);
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!live[q]) continue;
      if (DENSE) {
        ww.v[q].re = zre[q] * pp.v[q].re - zim[q] * pp.v[q].im - ww.v[q].re;
        ww.v[q].im = zre[q] * pp.v[q].im + zim[q] * pp.v[q].re - ww.v[q].im;
      }
      rr.v[q].re -= are[q] * ww.v[q].re - aim[q] * ww.v[q].im;
      rr.v[q].im -= are[q] * ww.v[q].im + aim[q] * ww.v[q].re;
      const double a = rr.v[q].re, b = rr.v[q].im;
      acc[q][0] += a * a - b * b;
      acc[q][1] += 2.0 * a * b;
      acc[q][2] += a * a + b * b;
    }
    st<T, CPL>(r + ro, rr);
  }
  put_partials<CPL, 3>(acc, part);
}

// alpha = rho / mu for iterating columns; a breakdown (mu = 0 or alpha not
// finite) sends the column to a restart check.  The other columns keep theirs:
// a check still has to add alpha p to x.
__global__ __launch_bounds__(kST) void k_s_fin_mu(int ns, int nb, const double* __restrict__ part,
                                                  StreamSlots sl, StreamCols cols) {
  const int s = fin_slot();
  if (s >= ns || sl.state[s] != 1) return;
  const int c = sl.col[s];
  const zd rho{cols.rho[2 * c], cols.rho[2 * c + 1]};
  double m[2];
  slot_sums<2>(part, nb, s, m);
  if ((threadIdx.x & 63) != 0) return;
  zd a = zdiv(rho, zd{m[0], m[1]});
  if ((m[0] == 0.0 && m[1] == 0.0) || !isfinite(a.re) || !isfinite(a.im)) {
    cols.state[c] = 3;
    sl.state[s] = 3;
    cols.nbd[c] += 1;
    a = zd{0.0, 0.0};
  }
  sl.alpha[2 * s] = cols.alpha[2 * c] = a.re;
  sl.alpha[2 * s + 1] = cols.alpha[2 * c + 1] = a.im;
}

// beta = rho_new / rho; a column whose recursive residual reached its check
// threshold, or whose iteration count reached the cap, waits for a check
// (rho keeps the previous value, which the check's beta needs).
__global__ __launch_bounds__(kST) void k_s_fin_rho(int ns, int nb, const double* __restrict__ part,
                                                   StreamSlots sl, StreamCols cols, int maxit) {
  const int sidx = fin_slot();
  if (sidx >= ns || sl.state[sidx] != 1) return;
  const int c = sl.col[sidx];
  const zd rho{cols.rho[2 * c], cols.rho[2 * c + 1]};
  const int it = cols.it[c] + 1, sp = cols.span[c], lastit = cols.lastit[c];
  const int span0 = cols.span0[c];
  const double ctol2 = cols.ctol2[c];
  double s[3];
  slot_sums<3>(part, nb, sidx, s);
  if ((threadIdx.x & 63) != 0) return;
  double br = 0.0, bi = 0.0;
  cols.it[c] = it;
  const bool stall = sp > 0 && it - lastit > max(max(4 * sp, 2 * span0), 256);
  if (s[2] <= ctol2 || it >= maxit || !isfinite(s[2]) || stall) {
    cols.state[c] = 0;
    sl.state[sidx] = 0;
  } else {
    const zd bt = zdiv(zd{s[0], s[1]}, rho);
    br = bt.re;
    bi = bt.im;
    cols.rho[2 * c] = s[0];
    cols.rho[2 * c + 1] = s[1];
  }
  sl.beta[2 * sidx] = cols.beta[2 * c] = br;
  sl.beta[2 * sidx + 1] = cols.beta[2 * c + 1] = bi;
}

// The scalars of the columns in slots 0 .. ns - 1 (col[u] < 0: none).
__global__ __launch_bounds__(kST) void k_s_slots(int ns, const double* __restrict__ zc,
                                                 StreamCols cols, StreamSlots sl) {
  const int u = blockIdx.x * kST + threadIdx.x;
  if (u >= ns) return;
  const int c = sl.col[u];
  sl.state[u] = c >= 0 ? cols.state[c] : 2;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    sl.zc[2 * u + h] = c >= 0 ? zc[2 * c + h] : 0.0;
    sl.alpha[2 * u + h] = c >= 0 ? cols.alpha[2 * c + h] : 0.0;
    sl.beta[2 * u + h] = c >= 0 ? cols.beta[2 * c + h] : 0.0;
  }
}

// Slots move together: new slot u of a block with row stride S_new takes old
// slot from[u] (-1: zero) of one with stride S.
template <typename T>
__global__ __launch_bounds__(kST) void k_s_move(int n, int S, int S_new,
                                                const int* __restrict__ from,
                                                const cpx<T>* __restrict__ src,
                                                cpx<T>* __restrict__ dst) {
  const int u = blockIdx.y * kSL + (int)(threadIdx.x % kSL);
  const int f = from[u];
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    dst[(size_t)row * S_new + u] = f >= 0 ? src[(size_t)row * S + f] : cpx<T>{T(0), T(0)};
  }
}

// Check, step 1: x_hi += x + alpha p (FP64; x as it stands after the last
// iteration), x = 0 for waiting columns.
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_xhi(int n, int S, int Bp, StreamSlots sl,
                                               const cpx<T>* __restrict__ p,
                                               cpx<T>* __restrict__ x,
                                               cpx<double>* __restrict__ xh) {
  const int s0 = lane_slot<CPL>();
  bool on[CPL], any = false;
  int c[CPL];
  T are[CPL], aim[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    on[q] = waiting(sl.state[s0 + q]);
    c[q] = sl.col[s0 + q];
    are[q] = T(sl.alpha[2 * (s0 + q)]);
    aim[q] = T(sl.alpha[2 * (s0 + q) + 1]);
    any = any || on[q];
  }
  if (!any) return;
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * S + s0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!on[q]) continue;
      cpx<T> xv = x[ro + q];
      const cpx<T> po = p[ro + q];
      xv.re += are[q] * po.re - aim[q] * po.im;
      xv.im += are[q] * po.im + aim[q] * po.re;
      cpx<double>* hp = xh + (size_t)row * Bp + c[q];
      hp->re += (double)xv.re;
      hp->im += (double)xv.im;
      x[ro + q] = cpx<T>{T(0), T(0)};
    }
  }
}

// What a lane of a check's step 2 needs of its columns.
template <int CPL>
struct CheckCols {
  double zre[CPL], zim[CPL], scl[CPL];
  bool on[CPL], rst[CPL], any = false;
  int c[CPL], ci[CPL];
  __device__ __forceinline__ CheckCols(const StreamSlots& sl, int s0,
                                       const double* __restrict__ scale, int kcols) {
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      zre[q] = sl.zc[2 * (s0 + q)];
      zim[q] = sl.zc[2 * (s0 + q) + 1];
      on[q] = waiting(sl.state[s0 + q]);
      rst[q] = sl.state[s0 + q] == 3;
      c[q] = sl.col[s0 + q];
      ci[q] = on[q] ? c[q] % kcols : 0;
      scl[q] = on[q] ? scale[c[q]] : 0.0;
      any = any || on[q];
    }
  }
  // s = b / ||b|| - (z x - A x) of column q at a row, r = s (p = s after a
  // breakdown), its products to acc
  template <typename T>
  __device__ __forceinline__ void put(int q, double bv, cpx<double> x, double axr, double axi,
                                      cpx<T>* __restrict__ r, cpx<T>* __restrict__ p,
                                      double (&acc)[3]) const {
    const double b = scl[q] != 0.0 ? bv * scl[q] : 0.0;
    const double sr = b - (zre[q] * x.re - zim[q] * x.im - axr);
    const double si = -(zre[q] * x.im + zim[q] * x.re - axi);
    *r = cpx<T>{T(sr), T(si)};
    if (rst[q]) *p = cpx<T>{T(sr), T(si)};
    acc[0] += sr * sr - si * si;
    acc[1] += 2.0 * sr * si;
    acc[2] += sr * sr + si * si;
  }
};

// Check, step 2: s = b/||b|| - (z x_hi - A x_hi) in FP64 with the FP64
// values of A; r = s (and p = s after a breakdown); partials of s^T s and
// ||s||^2.  Gathers as k_s_spmm, of the waiting columns (few: 16 bytes each).
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_resid64(
    int n, int S, const int* __restrict__ rowptr, const int* __restrict__ col,
    const double* __restrict__ val, int Bp, StreamSlots sl, const double* __restrict__ B, int ldb,
    int kcols, const double* __restrict__ scale, const int* __restrict__ perm,
    const cpx<double>* __restrict__ xh, cpx<T>* __restrict__ r, cpx<T>* __restrict__ p,
    double* __restrict__ part) {
  const int s0 = lane_slot<CPL>();
  const CheckCols<CPL> cc(sl, s0, scale, kcols);
  const unsigned long long who = __ballot(cc.any);
  if (who == 0) return;
  int mine = 0;
#pragma unroll
  for (int q = CPL - 1; q >= 0; --q)
    if (cc.on[q]) mine = cc.c[q];
  const int some = __builtin_amdgcn_readlane(mine, __builtin_ctzll(who));
  const cpx<double>* __restrict__ xg[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) xg[q] = xh + (cc.on[q] ? cc.c[q] : cc.any ? mine : some);
  double acc[CPL][3];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0.0;
  double ar[CPL], ai[CPL];
  walk_rows<double>(
      n, rowptr, col, val,
      [&](int, bool) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) ar[q] = ai[q] = 0.0;
      },
      [&](int mc, double mv) {
        int j[kSL];
        double a[kSL];
        entries_of(mc, mv, j, a, std::make_integer_sequence<int, kSL>{});
        cpx<double> xj[kSL][CPL];
#pragma unroll
        for (int u = 0; u < kSL; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) xj[u][q] = xg[q][(size_t)j[u] * Bp];
#pragma unroll
        for (int u = 0; u < kSL; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) {
            ar[q] += a[u] * xj[u][q].re;
            ai[q] += a[u] * xj[u][q].im;
          }
      },
      [&](int row, bool valid) {
        if (!valid) return;
        const size_t orow = (size_t)perm[row], ro = (size_t)row * S + s0;
#pragma unroll
        for (int q = 0; q < CPL; ++q)
          if (cc.on[q])
            cc.template put<T>(q, B[orow * ldb + cc.ci[q]], xg[q][(size_t)row * Bp], ar[q], ai[q],
                               r + ro + q, p + ro + q, acc[q]);
      });
  put_partials<CPL, 3>(acc, part);
}

// Dense operator: waiting columns (packed column u: column cidx[u]) of x_hi side by
// side, so that the check's product multiplies them alone.
__global__ __launch_bounds__(kST) void k_s_pack(int n, int Bp, int nw, int ld,
                                                const int* __restrict__ cidx,
                                                const cpx<double>* __restrict__ xh,
                                                cpx<double>* __restrict__ out) {
  const int u = blockIdx.y * kSL + (int)(threadIdx.x % kSL);
  if (u >= nw) return;
  const int c = cidx[u];
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    out[(size_t)row * ld + u] = xh[(size_t)row * Bp + c];
  }
}

// Dense operator, K2 after the product (w holds A p): the partials of
// mu = p^T (z p - A p).
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_mu(int n, int S, StreamSlots sl,
                                              const cpx<T>* __restrict__ p,
                                              const cpx<T>* __restrict__ w,
                                              double* __restrict__ part) {
  const int s0 = lane_slot<CPL>();
  T zre[CPL], zim[CPL];
  bool any = false;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    zre[q] = T(sl.zc[2 * (s0 + q)]);
    zim[q] = T(sl.zc[2 * (s0 + q) + 1]);
    any = any || sl.state[s0 + q] == 1;
  }
  if (__ballot(any) == 0) return;
  double acc[CPL][2];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = acc[q][1] = 0.0;
  const RowSteps rs = row_steps(n);
  for (int k = 0; any && k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * S + s0;
    const Chunk<T, CPL> p0 = ld<T, CPL>(p + ro), a = ld<T, CPL>(w + ro);
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const T wre = zre[q] * p0.v[q].re - zim[q] * p0.v[q].im - a.v[q].re;
      const T wim = zre[q] * p0.v[q].im + zim[q] * p0.v[q].re - a.v[q].im;
      const double pr = p0.v[q].re, pi = p0.v[q].im, wr_ = wre, wi = wim;
      acc[q][0] += pr * wr_ - pi * wi;
      acc[q][1] += pr * wi + pi * wr_;
    }
  }
  put_partials<CPL, 2>(acc, part);
}

// Dense operator, check step 2 after the product: column c's A x_hi (FP64) in
// packed column from[slot] of ax; the rest as k_s_resid64.
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_resid64d(
    int n, int S, int Bp, StreamSlots sl, const double* __restrict__ B, int ldb, int kcols,
    const double* __restrict__ scale, const cpx<double>* __restrict__ xh,
    const cpx<double>* __restrict__ ax, cpx<T>* __restrict__ r, cpx<T>* __restrict__ p,
    double* __restrict__ part) {
  const int s0 = lane_slot<CPL>();
  const CheckCols<CPL> cc(sl, s0, scale, kcols);
  if (__ballot(cc.any) == 0) return;
  int u[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) u[q] = sl.from[s0 + q];
  double acc[CPL][3];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0.0;
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * S + s0, rb = (size_t)row * Bp;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!cc.on[q]) continue;
      const cpx<double> a = ax[rb + u[q]];
      cc.template put<T>(q, B[(size_t)row * ldb + cc.ci[q]], xh[rb + cc.c[q]], a.re, a.im,
                         r + ro + q, p + ro + q, acc[q]);
    }
  }
  put_partials<CPL, 3>(acc, part);
}

// Check, step 3: accept (true residual <= tol), give up (update, iteration
// or breakdown budget spent), or continue: a reliable update keeps p and
// takes beta = s^T s / rho_prev; a restart takes beta = 0, so the next p is
// r = s (after a breakdown, or when ||s|| is not at most half the previous
// check's).  The next check comes when the recursive residual has dropped by
// delta from ||s|| (or reaches tol), or at a stall.
__global__ __launch_bounds__(kST) void k_s_fin_verify(int ns, int nb,
                                                      const double* __restrict__ part,
                                                      StreamSlots sl, StreamCols cols, double tol,
                                                      double delta, int maxit, int max_updates) {
  const int sidx = fin_slot();
  if (sidx >= ns) return;
  const int st0 = sl.state[sidx];
  if (!waiting(st0)) return;
  const int c = sl.col[sidx];
  double s[3];
  slot_sums<3>(part, nb, sidx, s);
  if ((threadIdx.x & 63) != 0) return;
  cols.res[c] = sqrt(s[2]);
  // the check has added alpha p to x
  sl.alpha[2 * sidx] = sl.alpha[2 * sidx + 1] = cols.alpha[2 * c] = cols.alpha[2 * c + 1] = 0.0;
  if (s[2] <= tol * tol || !isfinite(s[2]) || cols.nref[c] >= max_updates ||
      cols.it[c] >= maxit || cols.nbd[c] > 3) {
    cols.state[c] = 2;
    sl.state[sidx] = 2;
    return;
  }
  cols.nref[c] += 1;
  double br = 0.0, bi = 0.0;  // beta = 0 restarts: the next p is r = s
  if (st0 == 0 && s[2] <= 0.25 * cols.sprev[c]) {
    const zd bt = zdiv(zd{s[0], s[1]}, zd{cols.rho[2 * c], cols.rho[2 * c + 1]});
    if (isfinite(bt.re) && isfinite(bt.im)) {
      br = bt.re;
      bi = bt.im;
    }
  }
  const int it = cols.it[c];
  cols.span[c] = it - cols.lastit[c];
  if (cols.lastit[c] == cols.rstart[c]) cols.span0[c] = max(cols.span0[c], it - cols.lastit[c]);
  cols.lastit[c] = it;
  if (br == 0.0 && bi == 0.0) cols.rstart[c] = it;
  cols.sprev[c] = s[2];
  cols.rho[2 * c] = s[0];
  cols.rho[2 * c + 1] = s[1];
  sl.beta[2 * sidx] = cols.beta[2 * c] = br;
  sl.beta[2 * sidx + 1] = cols.beta[2 * c + 1] = bi;
  cols.ctol2[c] = fmax(tol * tol, delta * delta * s[2]);
  cols.state[c] = 1;
  sl.state[sidx] = 1;
}

// Start, step 1: partials of ||b_c||^2 (column c, in slot c, takes RHS column
// c % kcols).
template <int CPL>
__global__ __launch_bounds__(kST) void k_s_bnorm(int n, const double* __restrict__ B, int ldb,
                                                 int kcols, int ncols,
                                                 double* __restrict__ part) {
  const int cl = lane_slot<CPL>();
  double acc[CPL][1];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = 0.0;
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (cl + q >= ncols) continue;
      const double b = B[(size_t)row * ldb + (cl + q) % kcols];
      acc[q][0] += b * b;
    }
  }
  put_partials<CPL, 1>(acc, part);
}

// Start, step 2: per-column set-up; zero columns are solved at once.  Column c
// starts in slot c (S slots).
__global__ __launch_bounds__(kST) void k_s_fin_bnorm(int S, int nb,
                                                     const double* __restrict__ part, int ncols,
                                                     double* __restrict__ scale, StreamCols cols,
                                                     StreamSlots sl, double tol, double delta) {
  const int c = fin_slot();
  if (c >= S) return;
  double s[1] = {0.0};
  if (c < ncols) slot_sums<1>(part, nb, c, s);
  if ((threadIdx.x & 63) != 0) return;
  sl.col[c] = c < ncols ? c : -1;
  cols.it[c] = 0;
  cols.nref[c] = 0;
  cols.nbd[c] = 0;
  cols.alpha[2 * c] = cols.alpha[2 * c + 1] = 0.0;
  cols.beta[2 * c] = cols.beta[2 * c + 1] = 0.0;
  cols.res[c] = 0.0;
  cols.rho[2 * c] = cols.rho[2 * c + 1] = 0.0;
  cols.lastit[c] = 0;
  cols.span[c] = 0;
  cols.span0[c] = 0;
  cols.rstart[c] = 0;
  cols.sprev[c] = 1.0;  // the start residual b / ||b||
  const double nrm = c < ncols ? sqrt(s[0]) : 0.0;
  cols.bn[c] = nrm;
  if (!(nrm > 0.0) || !isfinite(nrm)) {
    scale[c] = 0.0;
    cols.state[c] = 2;
    return;
  }
  scale[c] = 1.0 / nrm;
  cols.ctol2[c] = fmax(tol * tol, delta * delta);
  cols.state[c] = 1;
}

// Start, step 3: r = p = b / ||b|| (engine row order), x = x_hi = 0; partials of r^T r.
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_start(int n, int S, int Bp,
                                                 const double* __restrict__ B, int ldb, int kcols,
                                                 const double* __restrict__ scale,
                                                 const int* __restrict__ perm,
                                                 cpx<T>* __restrict__ x, cpx<T>* __restrict__ r,
                                                 cpx<T>* __restrict__ p,
                                                 cpx<double>* __restrict__ xh,
                                                 double* __restrict__ part) {
  const int cl = lane_slot<CPL>();
  double scl[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) scl[q] = scale[cl + q];
  double acc[CPL][1];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q][0] = 0.0;
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * S + cl, rh = (size_t)row * Bp + cl;
    const size_t orow = (size_t)perm[row];
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const double b = scl[q] != 0.0 ? B[orow * ldb + (cl + q) % kcols] * scl[q] : 0.0;
      const cpx<T> v{T(b), T(0)};
      r[ro + q] = v;
      p[ro + q] = v;
      x[ro + q] = cpx<T>{T(0), T(0)};
      xh[rh + q] = cpx<double>{0.0, 0.0};
      acc[q][0] += (double)v.re * (double)v.re;
    }
  }
  put_partials<CPL, 1>(acc, part);
}

__global__ __launch_bounds__(kST) void k_s_fin_start(int S, int nb,
                                                     const double* __restrict__ part,
                                                     StreamCols cols) {
  const int c = fin_slot();  // column c is in slot c
  if (c >= S || cols.state[c] != 1) return;
  double s[1];
  slot_sums<1>(part, nb, c, s);
  if ((threadIdx.x & 63) != 0) return;
  cols.rho[2 * c] = s[0];
  cols.rho[2 * c + 1] = 0.0;
}

// Output: D[perm[row]][c] = ||b_c|| x_hi[row][c] for c < ncols.
template <typename T, int CPL>
__global__ __launch_bounds__(kST) void k_s_out(int n, int Bp, int ncols,
                                               const double* __restrict__ bn,
                                               const int* __restrict__ perm,
                                               const cpx<double>* __restrict__ xh,
                                               cpx<T>* __restrict__ D, int ldd) {
  const int cl = lane_slot<CPL>();
  const RowSteps rs = row_steps(n);
  for (int k = 0; k < rs.count; ++k) {
    const int row = rs.first + rs.stride * k + lane_row();
    if (row >= rs.hi) break;
    const size_t ro = (size_t)row * Bp + cl;
    const size_t orow = (size_t)perm[row];
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (cl + q >= ncols) continue;
      const cpx<double> h = xh[ro + q];
      const double s = bn[cl + q];
      D[orow * ldd + cl + q] = cpx<T>{T(h.re * s), T(h.im * s)};
    }
  }
}

// Per-column report: iterations, final relative true residual; stats[0] +=
// FP64 residual checks that continued the iteration, stats[1] += columns
// given up after repeated breakdowns.
__global__ void k_s_report(int ncols, StreamCols cols, int* __restrict__ iters,
                           double* __restrict__ resid, int* __restrict__ stats) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncols) return;
  if (iters) iters[c] = cols.it[c];
  if (resid) resid[c] = cols.res[c];
  if (stats) {
    if (cols.nref[c]) atomicAdd(&stats[0], cols.nref[c]);
    if (cols.nbd[c] > 3) atomicAdd(&stats[1], 1);
  }
}

// ---------------------------------------------------------------------------
// host side
int stream_cpl(int k, int ncols, bool fp32) {
  // columns are padded to 128 (FP32 blocks of at least that many) or 64
  (void)k;
  return (fp32 && ncols >= 128) ? 2 : 1;
}

int stream_padded_columns(int k, int ncols, bool fp32) {
  const int gw = 64 * stream_cpl(k, ncols, fp32);
  return (ncols + gw - 1) / gw * gw;
}

int stream_blocks(int n, int num_cu) {
  // row blocks of a unit of slots, the grid's second dimension running over
  // the units: two per CU up to 2^17 rows, where the finalisers' partial sums
  // (one per row block and column) cost more than the extra occupancy gives,
  // four above
  int nb = num_cu * (n <= (1 << 17) ? 2 : 4) / 8 * 8;
  const int need = (n + kSW * kSR - 1) / (kSW * kSR);
  if (nb > need) nb = (need + 7) / 8 * 8;
  return nb < 8 ? 8 : nb;
}

size_t stream_partial_doubles(int n, int Bp, int num_cu) {
  return (size_t)stream_blocks(n, num_cu) * Bp * 3;
}

template <typename T>
static hipError_t run_stream_t(hipStream_t stm, const StreamMatrix& A, const StreamWork& W,
                               const StreamLaunch& L) {
  constexpr int CPL = lane_cols<T>(), UC = unit_cols<T>();
  const int n = A.n, Bp = W.Bp;
  const int nb = stream_blocks(n, W.num_cu);
  const dim3 blk(kST);
  // check spacing: FP32 storage drifts by about kappa * 6e-8 of the residual
  // per check interval, so checks come every decade; FP64 rarely needs one
  const double delta = sizeof(T) == 4 ? 0.1 : 1e-4;
  const T* val = sizeof(T) == 4 ? (const T*)(const void*)A.val32 : (const T*)(const void*)A.val64;
  cpx<T>* X = (cpx<T>*)W.x;
  cpx<T>* R = (cpx<T>*)W.r;
  cpx<T>* P = (cpx<T>*)W.p0;
  cpx<T>* spare = (cpx<T>*)W.p1;
  cpx<T>* Wv = (cpx<T>*)W.w;
  cpx<double>* XH = (cpx<double>*)W.xh;
  const StreamSlots& sl = W.slots;
  hipError_t e = hipSuccess;
#define SLAUNCH(...)                      \
  do {                                    \
    hipLaunchKernelGGL(__VA_ARGS__);      \
    e = hipGetLastError();                \
    if (e != hipSuccess) return e;        \
  } while (0)
  auto padded = [&](int cols) { return (cols + UC - 1) / UC * UC; };
  // slot u < ns holds column hcol[u] (-1: none); row stride S of the slot blocks
  int ns = L.ncols, S = padded(L.ncols);
  std::vector<int> hcol(S, -1), hstate(Bp), hidx(Bp), hfrom(Bp);
  for (int c = 0; c < ns; ++c) hcol[c] = c;
  auto units = [&](int nrb) { return dim3(nrb, S / UC); };
  auto fins = [&] { return dim3((S + kFinCols - 1) / kFinCols); };
  SLAUNCH(k_s_bnorm<CPL>, units(nb), blk, 0, stm, n, L.B, L.ldb, L.k, L.ncols, W.part);
  SLAUNCH(k_s_fin_bnorm, fins(), blk, 0, stm, S, nb, W.part, L.ncols, W.scale, W.cols, sl, L.tol,
          delta);
  SLAUNCH((k_s_start<T, CPL>), units(nb), blk, 0, stm, n, S, Bp, L.B, L.ldb, L.k, W.scale, A.perm,
          X, R, P, XH, W.part);
  SLAUNCH(k_s_fin_start, fins(), blk, 0, stm, S, nb, W.part, W.cols);
  SLAUNCH(k_s_slots, dim3((S + kST - 1) / kST), blk, 0, stm, S, W.zc, W.cols, sl);
  int live = 0, wait = 0;
  auto census = [&]() -> hipError_t {
    hipError_t e2 = hipMemcpyAsync(hstate.data(), W.cols.state, L.ncols * sizeof(int),
                                   hipMemcpyDeviceToHost, stm);
    if (e2 == hipSuccess) e2 = hipStreamSynchronize(stm);
    live = wait = 0;
    for (int c = 0; c < L.ncols; ++c) {
      live += hstate[c] == 1;
      wait += hstate[c] == 0 || hstate[c] == 3;
    }
    return e2;
  };
  // Columns that are done leave their slots when that frees a unit (a dense
  // operator's product, which multiplies slots 0 .. ns - 1, from eight columns
  // on: 4 us of product each per pass on n = 4096 against 15 us for the move).
  auto compact = [&]() -> hipError_t {
    const int left = live + wait;
    if (left == 0 || !(padded(left) < S || (A.dense && ns - left >= 8))) return hipSuccess;
    const int Sn = padded(left);
    int m = 0;
    for (int u = 0; u < ns; ++u)
      if (hcol[u] >= 0 && hstate[hcol[u]] != 2) {
        hidx[m] = hcol[u];
        hfrom[m++] = u;
      }
    for (int u = m; u < Sn; ++u) hidx[u] = hfrom[u] = -1;
    hcol.assign(hidx.begin(), hidx.begin() + Sn);
    hipError_t e2 =
        hipMemcpyAsync(sl.col, hidx.data(), Sn * sizeof(int), hipMemcpyHostToDevice, stm);
    if (e2 == hipSuccess)
      e2 = hipMemcpyAsync(sl.from, hfrom.data(), Sn * sizeof(int), hipMemcpyHostToDevice, stm);
    if (e2 != hipSuccess) return e2;
    // X -> spare, R -> the old X, P -> the old R; the old P is the next spare
    cpx<T>* const old[3] = {X, R, P};
    cpx<T>* const to[3] = {spare, X, R};
    for (int i = 0; i < 3; ++i) {
      hipLaunchKernelGGL((k_s_move<T>), dim3(nb, Sn / kSL), blk, 0, stm, n, S, Sn, sl.from, old[i],
                         to[i]);
      e2 = hipGetLastError();
      if (e2 != hipSuccess) return e2;
    }
    X = to[0];
    R = to[1];
    P = to[2];
    spare = old[2];
    S = Sn;
    ns = m;
    hipLaunchKernelGGL(k_s_slots, dim3((S + kST - 1) / kST), blk, 0, stm, S, W.zc, W.cols, sl);
    return hipGetLastError();
  };
  // Dense operator: A x_hi of the waiting columns, packed (the update's w is
  // free here and holds the packed x_hi, as many columns of it as fit).
  auto dense_check_product = [&]() -> hipError_t {
    int nw = 0;
    for (int u = 0; u < S; ++u) {
      const bool on = hcol[u] >= 0 && (hstate[hcol[u]] == 0 || hstate[hcol[u]] == 3);
      hfrom[u] = on ? nw : -1;
      if (on) hidx[nw++] = hcol[u];
    }
    hipError_t e2 =
        hipMemcpyAsync(sl.from, hfrom.data(), S * sizeof(int), hipMemcpyHostToDevice, stm);
    if (e2 != hipSuccess) return e2;
    cpx<double>* pk = (cpx<double>*)W.w;
    const int room = (int)((size_t)Bp * sizeof(cpx<T>) / sizeof(cpx<double>));
    for (int u0 = 0; u0 < nw; u0 += room) {
      const int m = nw - u0 < room ? nw - u0 : room;
      e2 = hipMemcpyAsync(sl.list, hidx.data() + u0, m * sizeof(int), hipMemcpyHostToDevice, stm);
      if (e2 != hipSuccess) return e2;
      hipLaunchKernelGGL(k_s_pack, dim3(nb, (m + kSL - 1) / kSL), blk, 0, stm, n, Bp, m, room,
                         sl.list, XH, pk);
      e2 = hipGetLastError();
      if (e2 == hipSuccess)
        e2 = dense_apply_f64(*A.dense, stm, 2 * m, (const double*)pk, 2 * room,
                             (double*)((cpx<double>*)W.axh + u0), 2 * Bp, 1.0, 0.0);
      if (e2 != hipSuccess) return e2;
    }
    return hipSuccess;
  };
  auto check = [&]() -> hipError_t {
    const dim3 g = units(nb);
    SLAUNCH((k_s_xhi<T, CPL>), g, blk, 0, stm, n, S, Bp, sl, P, X, XH);
    if (A.dense) {
      e = dense_check_product();
      if (e != hipSuccess) return e;
      SLAUNCH((k_s_resid64d<T, CPL>), g, blk, 0, stm, n, S, Bp, sl, L.B, L.ldb, L.k, W.scale, XH,
              (const cpx<double>*)W.axh, R, P, W.part);
    } else {
      SLAUNCH((k_s_resid64<T, CPL>), g, blk, 0, stm, n, S, A.rowptr, A.col, A.val64, Bp, sl, L.B,
              L.ldb, L.k, W.scale, A.perm, XH, R, P, W.part);
    }
    SLAUNCH(k_s_fin_verify, fins(), blk, 0, stm, S, nb, W.part, sl, W.cols, L.tol, delta, L.maxit,
            L.max_updates);
    return hipSuccess;
  };
  e = census();
  if (e != hipSuccess) return e;
  const int chunk = L.chunk > 0 ? L.chunk : 8;
  // FP32 columns are checked in nearly every pass, so the check follows a
  // pass's iterations at once, without asking whether a column waits (it ends
  // early where none does), and the host reads the states once per pass.  A
  // dense operator's product needs the list of them, and FP64 columns wait
  // once in several passes: there the host looks first.
  const bool always = sizeof(T) == 4 && !A.dense;
  // Every column stays live or waiting from the start until it is done, and
  // each pass gives each live column at least one iteration and checks each
  // waiting one, so no column outlasts maxit + 2 * max_updates + 2 passes.
  const long guard = (long)L.maxit + 2L * L.max_updates + 8;
  for (long pass = 0; pass < guard && live + wait > 0; ++pass) {
    if (live > 0) {
      e = compact();
      if (e != hipSuccess) return e;
      const dim3 g = units(nb);
      for (int k = 0; k < chunk; ++k) {
        SLAUNCH((k_s_pupd<T, CPL>), g, blk, 0, stm, n, S, sl, R, X, P);
        if (A.dense) {
          if constexpr (sizeof(T) == 4)
            e = dense_apply_f32(*A.dense, stm, 2 * ns, (const float*)P, 2 * S, (float*)Wv, 2 * S);
          else
            e = dense_apply_f64(*A.dense, stm, 2 * ns, (const double*)P, 2 * S, (double*)Wv,
                                2 * S, 1.0, 0.0);
          if (e != hipSuccess) return e;
          SLAUNCH((k_s_mu<T, CPL>), g, blk, 0, stm, n, S, sl, P, Wv, W.part);
        } else {
          SLAUNCH((k_s_spmm<T, CPL>), g, blk, 0, stm, n, S, A.rowptr, A.col, val, sl, P, Wv,
                  W.part);
        }
        SLAUNCH(k_s_fin_mu, fins(), blk, 0, stm, S, nb, W.part, sl, W.cols);
        if (A.dense)
          SLAUNCH((k_s_update<T, CPL, true>), g, blk, 0, stm, n, S, sl, R, P, Wv, W.part);
        else
          SLAUNCH((k_s_update<T, CPL, false>), g, blk, 0, stm, n, S, sl, R, P, Wv, W.part);
        SLAUNCH(k_s_fin_rho, fins(), blk, 0, stm, S, nb, W.part, sl, W.cols, L.maxit);
      }
      if (!always) {
        e = census();
        if (e != hipSuccess) return e;
      }
    }
    if (always || wait > 0) {
      e = check();
      if (e == hipSuccess) e = census();
      if (e != hipSuccess) return e;
    }
  }
  S = padded(L.ncols);
  SLAUNCH((k_s_out<T, CPL>), units(nb), blk, 0, stm, n, Bp, L.ncols, W.cols.bn, A.perm, XH,
          (cpx<T>*)L.D, L.ldd);
  SLAUNCH(k_s_report, dim3((L.ncols + 255) / 256), dim3(256), 0, stm, L.ncols, W.cols, L.iters,
          L.resid, L.stats);
#undef SLAUNCH
  return hipSuccess;
}

hipError_t run_stream_cocg(hipStream_t st, const StreamMatrix& A, const StreamWork& W,
                           const StreamLaunch& L, bool fp32) {
  const int gw = 64 * stream_cpl(L.k, L.ncols, fp32);
  if (W.Bp % gw != 0 || W.Bp < L.ncols || W.Bp / gw > kStreamMaxGroups)
    return hipErrorInvalidValue;
  return fp32 ? run_stream_t<float>(st, A, W, L) : run_stream_t<double>(st, A, W, L);
}

}  // namespace rafeast
