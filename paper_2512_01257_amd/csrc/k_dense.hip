// Dense and sparse x dense kernels of the RA-FEAST path on gfx950:
//  - CSR SpMM with FP64 real blocks (Rayleigh-Ritz W = A Q, Phase-1 operator
//    applications, eq. rand-range and eq. B-def),
//  - tall-skinny Gram X^T Y and X S products on FP64 MFMA (Rayleigh-Ritz
//    projection Q^T A Q and CholQR),
//  - Ritz residuals, filter combination (eq. projector-quad), the Philox
//    Gaussian sketch (Algorithm 2, Phase 1) and layout helpers.
#include "device.h"
#include "kernels.h"

namespace rafeast {

// ============================================================================
// SpMM, FP64 real: Y = alpha*A*X + beta*X + gamma*X2.  This form serves a
// single column, some odd widths (launch_spmm_f64) and matrices without nonzeros:
// one wave per row, the row's nonzeros wave-uniform (scalar loads), lanes over
// the columns.
// ============================================================================
__global__ __launch_bounds__(256) void k_spmm_f64(int n, int k, const int* __restrict__ rowptr,
                                                  const int* __restrict__ col,
                                                  const double* __restrict__ val,
                                                  const double* __restrict__ X, int ldx,
                                                  double* __restrict__ Y, int ldy, double alpha,
                                                  double beta, const double* __restrict__ X2,
                                                  int ldx2, double gamma) {
  const int row = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (row >= n) return;
  const int lane = threadIdx.x & 63;
  const int s = rowptr[row], e = rowptr[row + 1];
  for (int c0 = 0; c0 < k; c0 += 64) {
    const int c = c0 + lane;
    const bool ok = c < k;
    // four gathered rows in flight per wave; even and odd nonzeros go to two
    // partial sums in row order
    double acc0 = 0.0, acc1 = 0.0;
    int t = s;
    for (; t + 3 < e; t += 4) {
      const int j0 = col[t], j1 = col[t + 1], j2 = col[t + 2], j3 = col[t + 3];
      const double a0 = val[t], a1 = val[t + 1], a2 = val[t + 2], a3 = val[t + 3];
      if (ok) {
        const double x0 = X[(size_t)j0 * ldx + c], x1 = X[(size_t)j1 * ldx + c];
        const double x2 = X[(size_t)j2 * ldx + c], x3 = X[(size_t)j3 * ldx + c];
        acc0 += a0 * x0;
        acc1 += a1 * x1;
        acc0 += a2 * x2;
        acc1 += a3 * x3;
      }
    }
    for (; t + 1 < e; t += 2) {
      const int j0 = col[t], j1 = col[t + 1];
      const double a0 = val[t], a1 = val[t + 1];
      if (ok) {
        acc0 += a0 * X[(size_t)j0 * ldx + c];
        acc1 += a1 * X[(size_t)j1 * ldx + c];
      }
    }
    if (t < e && ok) acc0 += val[t] * X[(size_t)col[t] * ldx + c];
    if (ok) {
      double y = alpha * (acc0 + acc1);
      if (beta != 0.0) y += beta * X[(size_t)row * ldx + c];
      if (X2 != nullptr) y += gamma * X2[(size_t)row * ldx2 + c];
      Y[(size_t)row * ldy + c] = y;
    }
  }
}

// Entry U of a round, loaded by lane U of each group of L lanes, handed to
// every lane of its group (a row's lanes): a lane swizzle within 32 lanes,
// or a read of lane U when the row has the whole wave.
template <int L, int U>
__device__ __forceinline__ int group_bcast(int v) {
  if constexpr (L == 64)
    return __builtin_amdgcn_readlane(v, U);
  else
    return __builtin_amdgcn_ds_swizzle(v, (0x1f & ~(L - 1)) | (U << 5));
}

template <int L, int U, int C>
struct RoundBcast {
  __device__ __forceinline__ static void run(int jv, double av, int* j, double* a) {
    j[U] = group_bcast<L, U>(jv);
    const long long ab = __double_as_longlong(av);
    const int lo = group_bcast<L, U>((int)(ab & 0xffffffffLL));
    const int hi = group_bcast<L, U>((int)(ab >> 32));
    a[U] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    RoundBcast<L, U + 1, C>::run(jv, av, j, a);
  }
};
template <int L, int C>
struct RoundBcast<L, C, C> {
  __device__ __forceinline__ static void run(int, double, int*, double*) {}
};

// A row's extent and the first round of its entries (lane u < C of the
// row's lanes holds entry u), loaded ahead of the row's gathers.
struct RowHead {
  int s, e, jv;
  double av;
};

// Every load of the SpMM below runs on every lane, at an index that is in
// range whether or not its value is used (an unused row reads row 0, an
// unused entry reads entry 0, an unused gather reads row j of entry 0 or
// column 0), and unused values are dropped where they are consumed:
// with no lane-masked branch around the loads and no select right after
// them, the compiler counts the loads in flight and waits only for the ones
// a step needs.  The matrix has at least one nonzero (checked at launch).
__device__ __forceinline__ void head_bounds(RowHead& h, int row, bool live,
                                            const int* __restrict__ rowptr) {
  const int r = live ? row : 0;
  h.s = __builtin_nontemporal_load(rowptr + r);
  h.e = __builtin_nontemporal_load(rowptr + r + 1);
}

template <int C>
__device__ __forceinline__ void head_entries(RowHead& h, int sub, int t0,
                                             const int* __restrict__ col,
                                             const double* __restrict__ val) {
  // the matrix streams past L2 (it is read once), which keeps L2 for the
  // gathered rows of X
  const int t = sub < C && t0 + sub < h.e ? t0 + sub : 0;
  h.jv = __builtin_nontemporal_load(col + t);
  h.av = __builtin_nontemporal_load(val + t);
}

// One row of Y for the lanes of sub-index sub.
// h holds the row's extent and its first round of entries; later rounds and
// later column passes load their own.
template <int L>
__device__ __forceinline__ void spmm_x2_row(int row, int sub, int k, const RowHead& h,
                                            const int* __restrict__ col,
                                            const double* __restrict__ val,
                                            const double* __restrict__ X, int ldx,
                                            double* __restrict__ Y, int ldy, double alpha,
                                            double beta, const double* __restrict__ X2, int ldx2,
                                            double gamma) {
  constexpr int C = L < 8 ? L : 8;  // nonzeros per round
  // two consecutive columns; rows start at any multiple of 8 bytes
  typedef double Pair __attribute__((ext_vector_type(2), aligned(8)));
  const int s = h.s, e = h.e;
  // round 0 (positions s .. s + C - 1): lane u < C of the row's lanes holds
  // entry u; handed round the row's lanes once, kept for every column pass
  int j0[C];
  double a0[C];
  RoundBcast<L, 0, C>::run(h.jv, h.av, j0, a0);
  for (int c0 = 0; c0 < k; c0 += 2 * L) {
    // with k odd the last lane takes the last two columns, of which its
    // neighbour writes the first as well (the same value); idle lanes read
    // the last two columns with them
    const bool ok = c0 + 2 * sub < k;
    const int c = min(c0 + 2 * sub, k - 2);
    Pair acc0{0.0, 0.0}, acc1{0.0, 0.0};
    // the gathered rows of a round are loaded together; even and odd
    // positions of the row go to two partial sums, in order (a round of one
    // entry alternates between them)
    {
      Pair x[C];
#pragma unroll
      for (int u = 0; u < C; ++u)
        x[u] = *reinterpret_cast<const Pair*>(X + (size_t)j0[u] * ldx + c);
#pragma unroll
      for (int u = 0; u < C; ++u) {
        if (s + u < e) {
          if (u & 1) {
            acc1.x += a0[u] * x[u].x;
            acc1.y += a0[u] * x[u].y;
          } else {
            acc0.x += a0[u] * x[u].x;
            acc0.y += a0[u] * x[u].y;
          }
        }
      }
    }
    // later rounds (rows longer than C): their entries are loaded here
    for (int t0 = s + C; t0 < e; t0 += C) {
      RowHead r = h;
      head_entries<C>(r, sub, t0, col, val);
      int j[C];
      double a[C];
      RoundBcast<L, 0, C>::run(r.jv, r.av, j, a);
      Pair x[C];
#pragma unroll
      for (int u = 0; u < C; ++u)
        x[u] = *reinterpret_cast<const Pair*>(X + (size_t)j[u] * ldx + c);
#pragma unroll
      for (int u = 0; u < C; ++u) {
        if (t0 + u < e) {
          const bool odd = C == 1 ? ((t0 - s) & 1) != 0 : (u & 1) != 0;
          if (odd) {
            acc1.x += a[u] * x[u].x;
            acc1.y += a[u] * x[u].y;
          } else {
            acc0.x += a[u] * x[u].x;
            acc0.y += a[u] * x[u].y;
          }
        }
      }
    }
    if (ok) {
      Pair y{alpha * (acc0.x + acc1.x), alpha * (acc0.y + acc1.y)};
      if (beta != 0.0) {
        const Pair xr = *reinterpret_cast<const Pair*>(X + (size_t)row * ldx + c);
        y.x += beta * xr.x;
        y.y += beta * xr.y;
      }
      if (X2 != nullptr) {
        const Pair x2r = *reinterpret_cast<const Pair*>(X2 + (size_t)row * ldx2 + c);
        y.x += gamma * x2r.x;
        y.y += gamma * x2r.y;
      }
      // Y is not read again here: streamed past L2, which keeps the gathered rows
      __builtin_nontemporal_store(y, reinterpret_cast<Pair*>(Y + (size_t)row * ldy + c));
    }
  }
}

// Two columns per lane (16-byte loads) and 64 / L rows per wave, L the
// power of two of lanes that covers the k >= 2 columns' pairs: each load instruction moves twice the bytes of the
// one-column form, and a wave serves several short rows at once.  Nonzeros
// go to two partial sums (even and odd positions) in row order.
//
// Placement: workgroup b runs on XCD b mod 8 (dispatch deals workgroup ids
// to the eight XCDs in turn).  XCD x owns the x-th contiguous eighth of the
// row blocks (rbx of them) and sweeps it in row order, all columns of a row at
// once, so a gathered row X[j] is fetched into that XCD's L2 once for the rows
// around j that need it.  Rows farther apart than L2 holds come again from the
// infinity cache; sweeping the columns in groups whose rows fit L2 saves those
// reads but reads the matrix once per group and cuts rows that are not whole
// 128-byte lines into partial ones, read and written twice: 100^3 grid, k = 30,
// 64, 84, 148: 307, 397, 988, 1504 us in groups, 194, 393, 620, 1176 us without
// (3D neighbour graph of 30,000 points, k = 84: 129 and 75 us).  A workgroup
// takes rpb consecutive row blocks of 4 * 64 / L rows, one after the other, as
// a pipeline: while a block's gathers are in flight, the next block's first
// entries and the extents of the block after it are loaded.
template <int L>
__global__ __launch_bounds__(256) void k_spmm_f64_x2(int n, int k, int rbx, int rpb,
                                                     const int* __restrict__ rowptr,
                                                     const int* __restrict__ col,
                                                     const double* __restrict__ val,
                                                     const double* __restrict__ X, int ldx,
                                                     double* __restrict__ Y, int ldy, double alpha,
                                                     double beta, const double* __restrict__ X2,
                                                     int ldx2, double gamma) {
  constexpr int RW = 64 / L;  // rows per wave
  constexpr int C = L < 8 ? L : 8;
  const int b = (int)blockIdx.x;
  const int rb0 = (b >> 3) * rpb;
  const int rb1 = min(rbx, rb0 + rpb);
  const int lane = threadIdx.x & 63;
  const int sub = lane % L;
  auto row_of = [&](int rbl) {
    return (((b & 7) * rbx + rbl) * 4 + (int)(threadIdx.x >> 6)) * RW + lane / L;
  };
  auto live = [&](int rbl, int r) { return rbl < rb1 && r < n; };
  int row = row_of(rb0), nrow = row_of(rb0 + 1);
  RowHead h, nh;
  head_bounds(h, row, live(rb0, row), rowptr);
  head_bounds(nh, nrow, live(rb0 + 1, nrow), rowptr);
  head_entries<C>(h, sub, h.s, col, val);
  for (int rbl = rb0; rbl < rb1; ++rbl) {
    if (row >= n) break;
    const int nnrow = row_of(rbl + 2);
    RowHead nnh;
    head_bounds(nnh, nnrow, live(rbl + 2, nnrow), rowptr);
    head_entries<C>(nh, sub, nh.s, col, val);
    spmm_x2_row<L>(row, sub, k, h, col, val, X, ldx, Y, ldy, alpha, beta, X2, ldx2,
                   gamma);
    h = nh;
    nh = nnh;
    row = nrow;
    nrow = nnrow;
  }
}

hipError_t launch_spmm_f64(hipStream_t st, int n, int k, const int* rowptr, const int* col,
                           const double* val, int64_t nnz, const double* X, int ldx, double* Y,
                           int ldy, double alpha, double beta, const double* X2, int ldx2,
                           double gamma, int64_t span) {
  if (n <= 0 || k <= 0) return hipSuccess;
  // Column pairs, or one column a lane.  With odd k the rows of pairs start
  // between 16-byte boundaries and a pass may have half its lanes idle, and one
  // column a lane is as fast or faster (us, pairs and single columns)
  // - for widths of 33 to 63: 3D neighbour graph of 50,000 points, k = 33: 60.8,
  //   56.3; 2D of 30,000, k = 63: 44.3, 43.0; 40^3 grid, k = 33: 37.5, 39.1;
  // - above 64 and 128 on rows of a few entries: tridiagonal n = 64,000, k = 65:
  //   50, 45; k = 119: 54, 52; k = 129: 68, 58; k = 161: 71, 64 (seven entries:
  //   55, 59; 62, 72; 79, 83; 83, 92); n = 250,000, k = 73: 135, 133; k = 81:
  //   138, 146;
  // - above 128 on fewer than 16,384 rows (3D neighbour graph of 9,402 points,
  //   k = 147: 47.3, 45.3), and on long rows whose gathers stay in an XCD's L2,
  //   the longer the rows the wider: n = 64,000, k = 137: 13 entries within 40 of
  //   the diagonal 119, 108; 40 within 120 266, 236; in random order 451, 477;
  //   k = 191: 20 entries 178, 191; 70 470, 427.
  const int64_t len = nnz / n;  // entries a row
  const bool near = (2 * span + 1) * k * 8 <= (3 << 20);  // of 4 MiB
  const bool single =
      k % 2 == 1 &&
      ((k > 32 && k < 64) || (k > 64 && k < (n <= 1 << 17 ? 120 : 80) && len < 4) ||
       (k > 128 && n < 16384) || (k > 128 && k < 192 && len < 4) ||
       (k > 128 && k < 160 + (len < 32 ? len : 32) && len > 10 && near));
  if (nnz > 0 && k >= 2 && !single) {
    // lanes per row: the power of two covering the column pairs (<= 64); on few
    // rows eight at least, which take eight entries a round (us with as few as
    // cover the pairs and with eight, k = 3: 4,000 rows of 70 entries 43, 29;
    // 16,000 rows of 7 23, 22)
    int L = n <= 16384 ? 8 : 1;
    while (L < 64 && 2 * L < k) L *= 2;
    const int rw = 64 / L;
    const int rblocks = (n + 4 * rw - 1) / (4 * rw);
    const int rbx = (rblocks + 7) / 8;
    // Few row blocks: one to a workgroup, so that the chip is full; more: the
    // pipeline over several saves the start of each, the sooner the shorter the
    // rows.  us with 1, 2 and 4 row blocks: rows of 3 entries, 125 blocks
    // (4,000 rows, k = 16) 21, 22, 23; 8,000 blocks (64,000 rows, k = 48) 41, 37,
    // 36; 31,250 (250,000 rows, k = 34) 100, 86, 83; of 13 entries, 8,000 blocks
    // 53, 51, 50; of 70, 2,000 blocks (8,000 rows, k = 148) 86, 96, 117; 3D
    // neighbour graph of 2,000 points, k = 64 (250 blocks): 19.4, 20.9, 24.5;
    // 40^3 grid, k = 147 (16,000 blocks): 78, 76, 79.
    const int rpb = rblocks >= (1 << (len < 10 ? 15 : 16))   ? 4
                    : rblocks >= (1 << (len < 32 ? 10 : 12)) ? 2
                                                             : 1;
    const dim3 grid((unsigned)(8 * ((rbx + rpb - 1) / rpb)));
#define RAFEAST_SPMM_X2(LL)                                                                     \
  hipLaunchKernelGGL(k_spmm_f64_x2<LL>, grid, dim3(256), 0, st, n, k, rbx, rpb, rowptr, col,     \
                     val, X, ldx, Y, ldy, alpha, beta, X2, ldx2, gamma)
    switch (L) {
      case 1: RAFEAST_SPMM_X2(1); break;
      case 2: RAFEAST_SPMM_X2(2); break;
      case 4: RAFEAST_SPMM_X2(4); break;
      case 8: RAFEAST_SPMM_X2(8); break;
      case 16: RAFEAST_SPMM_X2(16); break;
      case 32: RAFEAST_SPMM_X2(32); break;
      default: RAFEAST_SPMM_X2(64); break;
    }
#undef RAFEAST_SPMM_X2
    return hipGetLastError();
  }
  dim3 grid((n + 3) / 4);
  hipLaunchKernelGGL(k_spmm_f64, grid, dim3(256), 0, st, n, k, rowptr, col, val, X, ldx, Y, ldy,
                     alpha, beta, X2, ldx2, gamma);
  return hipGetLastError();
}

// ============================================================================
// Gram G = X^T Y on v_mfma_f64_16x16x4f64.
// Operand layout of the 16x16x4 FP64 MFMA (per lane l of the wave):
//   A (16 x 4):  A[l % 16][l / 16]        B (4 x 16):  B[l / 16][l % 16]
//   D (16 x 16): D[l / 16 + 4 v][l % 16], v = 0..3
// For G = X^T Y the A operand is a 4-row slab of X transposed and B the same
// rows of Y, so lane l reads X[r + l/16][a0 + l%16] and Y[r + l/16][b0 + l%16]:
// 16 consecutive doubles of a row per quarter-wave.
// Rows are split into chunks (grid.x); each wave owns one 16-row tile strip of
// G and four 16-column tiles; partial Grams are summed in chunk order.
// ============================================================================
// Word 3 of a raw buffer descriptor on gfx9-family GPUs (no format, no
// swizzle, stride 0): reads past num_records bytes return zero.
constexpr int kBufferWord3 = 0x00020000;

int gram_chunks(int64_t n) {
  int64_t c = (n + 127) / 128;
  if (c > 256) c = 256;
  if (c < 1) c = 1;
  return (int)c;
}

// Largest k of the symmetric kernel (its tiles: 12 x 13 / 2).
constexpr int kSymMaxK = 192;

// Whether the Gram of one block (same: X is Y) takes the symmetric kernel.  It
// reads X once and computes half the tiles, but has one workgroup a row chunk: up
// to two tiles a row its waves have too little to do on many rows, and from five
// on a chunk's tiles one after the other take longer than the general kernel's
// side by side while those leave CUs idle.  us, general and symmetric, at
// k = 1: n = 16,000 28, 28; 64,000 32, 36; 1e6 73, 139
// k = 16: n = 128,000 44, 42; 250,000 55, 56; 1e6 93, 134
// k = 64: n = 3,000 27, 28; 32,000 51, 37; 1e6 259, 148
// k = 84: n = 1,000 26, 28; 4,000 29, 30; 8,000 34, 32; 1e6 585, 247
// k = 128: n = 1,000 26, 33; 8,000 36, 38; 16,000 50, 39; 1e6 1126, 460
// k = 192: n = 500 29, 41; 8,000 48, 50; 16,000 70, 58; 500,000 951, 484
static bool gram_symmetric(int64_t n, int k1, int k2, bool same) {
  if (!same || k1 != k2 || k1 > kSymMaxK) return false;
  if (k1 <= 32) return n <= (k1 <= 3 ? 1 << 14 : 1 << 17);
  return k1 <= 64 || n > (k1 <= 96 ? 4096 : 8192);
}

// Partial doubles of one row chunk: the symmetric kernel's tiles, or the product.
size_t gram_chunk_doubles(int64_t n, int k1, int k2, bool same) {
  const size_t nt = (k1 + 15) / 16;
  return gram_symmetric(n, k1, k2, same) ? nt * (nt + 1) / 2 * 256 : (size_t)k1 * (size_t)k2;
}

// Row chunks: of the symmetric kernel, whose workgroups hold all tiles of a
// chunk, two per CU, from chunks of 64 rows on.
int gram_chunks_of(int64_t n, int k1, int k2, bool same) {
  if (!gram_symmetric(n, k1, k2, same)) return gram_chunks(n);
  const int64_t c = (n + 63) / 64;
  return (int)(c > 512 ? 512 : c < 1 ? 1 : c);
}

// Enough for X^T Y and for X^T X.
size_t gram_partial_doubles(int64_t n, int k1, int k2) {
  const size_t two = gram_chunks_of(n, k1, k2, false) * gram_chunk_doubles(n, k1, k2, false);
  const size_t one = gram_chunks_of(n, k1, k2, true) * gram_chunk_doubles(n, k1, k2, true);
  return two > one ? two : one;
}

// A workgroup owns a TA x TB block of 16 x 16 output tiles of one row chunk;
// its 4 waves split the chunk's rows (wave w takes batches w, w + 4, ...)
// and add their partial blocks through LDS in a fixed order.  Per 4-row step a
// wave loads TA + TB operand fragments and issues TA * TB MFMAs on them.
// Rows go in batches of U steps (4 U rows) whose loads are issued together,
// unconditionally (a column past k reads column k - 1, which only feeds rows
// or columns of G that are not stored; a row past the chunk reads zero), and
// every tile's MFMA is issued, so no branch separates the loads from the
// MFMAs.
template <int TA, int TB, int U>
__global__ __launch_bounds__(256) void k_gram_partial(int64_t n, int k1, int k2,
                                                      const double* __restrict__ X, int ldx,
                                                      const double* __restrict__ Y, int ldy,
                                                      double* __restrict__ part,
                                                      int64_t rows_per_chunk) {
  constexpr int kBlockVals = TA * TB * 256;  // one wave's partial block
  __shared__ double sh[2 * kBlockVals];
  const int chunk = blockIdx.x;
  const int64_t r_begin = (int64_t)chunk * rows_per_chunk;
  int64_t r_end = r_begin + rows_per_chunk;
  if (r_end > n) r_end = n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tb_n = (k2 + 15) >> 4;
  const int bb_n = (tb_n + TB - 1) / TB;  // tile blocks per block row
  const int blk = blockIdx.y;
  const int ta0 = (blk / bb_n) * TA, tb0 = (blk % bb_n) * TB;
  const int li = lane & 15, lk = lane >> 4;
  int a_col[TA], b_col[TB];
#pragma unroll
  for (int i = 0; i < TA; ++i) a_col[i] = (ta0 + i) * 16 + li;
#pragma unroll
  for (int j = 0; j < TB; ++j) b_col[j] = (tb0 + j) * 16 + li;
  v4d acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};

  // Loads go through buffer descriptors covering exactly the chunk's rows of
  // X and Y: an address is a per-lane 32-bit byte offset (lane row lk, tile
  // column) plus a wave-uniform row offset, and a read past the chunk's last
  // row returns zero, so the last partial batch needs no guard.
  constexpr int BR = 4 * U;  // rows per batch
  const int64_t nrows = r_end > r_begin ? r_end - r_begin : 0;
  const int64_t nbatch = (nrows + BR - 1) / BR;
  const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(X + r_begin * ldx), (short)0, (int)(nrows * ldx * 8), kBufferWord3);
  const __amdgpu_buffer_rsrc_t ys = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(Y + r_begin * ldy), (short)0, (int)(nrows * ldy * 8), kBufferWord3);
  int xo[TA], yo[TB];
#pragma unroll
  for (int i = 0; i < TA; ++i) xo[i] = (lk * ldx + min(a_col[i], k1 - 1)) * 8;
#pragma unroll
  for (int j = 0; j < TB; ++j) yo[j] = (lk * ldy + min(b_col[j], k2 - 1)) * 8;
  for (int64_t bt = wave; bt < nbatch; bt += 4) {
    const int r = (int)(bt * BR);  // row within the chunk
    double a[U][TA], b[U][TB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int xrow = (r + 4 * u) * ldx * 8, yrow = (r + 4 * u) * ldy * 8;
#pragma unroll
      for (int i = 0; i < TA; ++i)
        a[u][i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(xs, xo[i], xrow, 0));
#pragma unroll
      for (int j = 0; j < TB; ++j)
        b[u][j] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(ys, yo[j], yrow, 0));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
  }
  // the 4 waves' blocks summed in a fixed order, (w0 + w2) + (w1 + w3), in
  // two rounds through half the LDS; element (i, j, v, l) of a block is
  // D[l / 16 + 4 v][l % 16] of tile (i, j)
  auto idx = [&](int i, int j, int v) { return ((i * TB + j) * 4 + v) * 64 + lane; };
  if (wave >= 2) {
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) sh[(wave - 2) * kBlockVals + idx(i, j, v)] = acc[i][j][v];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][v] += sh[wave * kBlockVals + idx(i, j, v)];
  }
  __syncthreads();
  if (wave == 1) {
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) sh[idx(i, j, v)] = acc[i][j][v];
  }
  __syncthreads();
  if (wave == 0) {
    double* P = part + (size_t)chunk * k1 * k2;
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int gi = (ta0 + i) * 16 + lk + 4 * v;
          const int gj = (tb0 + j) * 16 + li;
          if (gi < k1 && gj < k2) P[(size_t)gi * k2 + gj] = acc[i][j][v] + sh[idx(i, j, v)];
        }
  }
}

__global__ __launch_bounds__(256) void k_gram_reduce(int chunks, int k1, int k2,
                                                     const double* __restrict__ part,
                                                     double* __restrict__ G, int ldg) {
  __shared__ double sh[4][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = blockIdx.x * 64 + lane;
  const int total = k1 * k2;
  const size_t stride = (size_t)total;
  const int q = (chunks + 3) / 4;
  const int c0 = wave * q, c1 = min(chunks, c0 + q);
  double s = 0.0;
  if (e < total)
    for (int c = c0; c < c1; ++c) s += part[(size_t)c * stride + e];
  sh[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && e < total)
    G[(size_t)(e / k2) * ldg + (e % k2)] = ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
}

// ============================================================================
// Symmetric Gram G = X^T X (CholQR): only the upper 16 x 16 tiles, each
// workgroup all of them for its chunk of rows, so X is read once.  RS rows are
// staged in LDS through registers (two buffers, the loads of the next two
// stages in flight during this stage's MFMAs); the NW waves own TPW consecutive tiles
// each.  A row of LDS is PK doubles, PK = 16 mod 32, so that a fragment (4 rows
// of 16 doubles) covers the banks evenly.  The general kernel above computed all
// tiles from global memory, reading each row for every block row of tiles
// (n = 1e6, k = 84: 575 us; this 230 us, X alone being 139 us at the
// copy rate, and the tiles 137 us of matrix core time).
// ============================================================================
// Two consecutive columns of a row through a descriptor (byte offset off; in:
// whether the first is wanted, in2: the second): one 16-byte load where rows
// and base are 16-byte aligned and k is even (wide), else two.
constexpr int kOutside = 0x7ffffff0;  // past every descriptor
__device__ __forceinline__ double2 load_pair(__amdgpu_buffer_rsrc_t rs, int off, bool in, bool in2,
                                             bool wide) {
  if (wide)
    return __builtin_bit_cast(double2,
                              __builtin_amdgcn_raw_buffer_load_b128(rs, in ? off : kOutside, 0, 0));
  double2 v;
  v.x = __builtin_bit_cast(double,
                           __builtin_amdgcn_raw_buffer_load_b64(rs, in ? off : kOutside, 0, 0));
  v.y = __builtin_bit_cast(
      double, __builtin_amdgcn_raw_buffer_load_b64(rs, in2 ? off + 8 : kOutside, 0, 0));
  return v;
}
static bool wide_rows(const double* X, int ldx, int k) {
  return k % 2 == 0 && ldx % 2 == 0 && ((uintptr_t)X & 15) == 0;
}

template <int NW, int TPW, int RS, int MT>
__global__ __launch_bounds__(64 * NW) void k_gram_sym(int64_t n, int k, int wide,
                                                      const double* __restrict__ X, int ldx,
                                                      double* __restrict__ part,
                                                      int64_t rows_per_chunk) {
  extern __shared__ double sx[];
  constexpr int T = 64 * NW, LPR = T / RS;       // lanes per staged row
  constexpr int NL = (8 * MT + LPR - 1) / LPR;   // column pairs per lane (MT >= tiles per row)
  const int nt = (k + 15) >> 4, ntiles = nt * (nt + 1) / 2;
  const int PK = 16 * (nt | 1);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_chunk;
  const int rows = (int)max<int64_t>(0, min<int64_t>(rows_per_chunk, n - r_begin));
  // a column past k or a row past the chunk lies past the descriptor: zero
  const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(X + r_begin * ldx), (short)0, rows > 0 ? ((rows - 1) * ldx + k) * 8 : 0,
      kBufferWord3);
  const int sr = tid / LPR, sl = tid % LPR;  // staged row, first column pair
  double2 ld[2][NL];  // two stages ahead
  auto load = [&](double2 (&d)[NL], int r0) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int c = 2 * (sl + LPR * u);
      const bool in = r0 + sr < rows;
      d[u] = load_pair(xs, ((r0 + sr) * ldx + c) * 8, in && c < k, in && c + 1 < k, wide != 0);
    }
  };
  auto stage = [&](double* dst, const double2 (&d)[NL]) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int c = 2 * (sl + LPR * u);
      if (c < 16 * nt) *reinterpret_cast<double2*>(dst + sr * PK + c) = d[u];
    }
  };
  // this wave's tiles
  int ti[TPW], tj[TPW];
  bool on[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    int t = wave * TPW + u, I = 0;
    on[u] = t < ntiles;
    t = min(t, ntiles - 1);
    while (t >= nt - I) t -= nt - I++;
    ti[u] = 16 * I + (lane >> 4) * PK + (lane & 15);
    tj[u] = 16 * (I + t) + (lane >> 4) * PK + (lane & 15);
  }
  v4d acc[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u) acc[u] = v4d{0.0, 0.0, 0.0, 0.0};
  const int buf = RS * PK;
  // stage s at rows RS s: its MFMAs, while stage s + 1 waits in registers to be
  // stored at their end and stage s + 2 is being loaded
  auto step = [&](int r0, const double* b, double* next, const double2 (&d)[NL],
                  double2 (&dl)[NL]) {
    if (r0 + 2 * RS < rows) load(dl, r0 + 2 * RS);
#pragma unroll
    for (int q = 0; q < RS / 4; ++q) {
      double fa[TPW], fb[TPW];
#pragma unroll
      for (int u = 0; u < TPW; ++u) {
        fa[u] = b[ti[u] + 4 * q * PK];
        fb[u] = b[tj[u] + 4 * q * PK];
      }
#pragma unroll
      for (int u = 0; u < TPW; ++u)
        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u], fb[u], acc[u], 0, 0, 0);
    }
    if (r0 + RS < rows) stage(next, d);
    __syncthreads();
  };
  load(ld[0], 0);
  load(ld[1], RS);
  stage(sx, ld[0]);
  __syncthreads();
  for (int r0 = 0; r0 < rows; r0 += 2 * RS) {
    step(r0, sx, sx + buf, ld[1], ld[0]);
    if (r0 + RS < rows) step(r0 + RS, sx + buf, sx, ld[0], ld[1]);
  }
  // partial tiles in tile order, accumulator v of lane l at 64 v + l
#pragma unroll
  for (int u = 0; u < TPW; ++u)
    if (on[u])
#pragma unroll
      for (int v = 0; v < 4; ++v)
        part[((size_t)blockIdx.x * ntiles + wave * TPW + u) * 256 + 64 * v + lane] = acc[u][v];
}

// Sum of the chunks' tiles in order (eight groups of chunks, then the groups),
// written to both triangles.
__global__ __launch_bounds__(512) void k_gram_sym_reduce(int chunks, int k,
                                                         const double* __restrict__ part,
                                                         double* __restrict__ G, int ldg) {
  __shared__ double sh[8][64];
  const int nt = (k + 15) >> 4, ntiles = nt * (nt + 1) / 2;
  const int g = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = blockIdx.x * 64 + lane;  // four blocks a tile
  const int per = (chunks + 7) / 8, c0 = g * per, c1 = min(chunks, c0 + per);
  double s = 0.0;
#pragma unroll 8
  for (int c = c0; c < c1; ++c) s += part[(size_t)c * ntiles * 256 + e];
  sh[g][lane] = s;
  __syncthreads();
  if (g != 0) return;
  s = 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q) s += sh[q][lane];
  int t = e >> 8, I = 0;
  while (t >= nt - I) t -= nt - I++;
  const int i = 16 * I + 4 * ((e >> 6) & 3) + (lane >> 4), j = 16 * (I + t) + (lane & 15);
  if (i < k && j < k) {
    G[(size_t)i * ldg + j] = s;
    if (t > 0) G[(size_t)j * ldg + i] = s;
  }
}

template <int NW, int TPW, int RS, int MT>
static hipError_t launch_sym(hipStream_t st, int64_t n, int k, const double* X, int ldx,
                             double* part, int chunks, int64_t rpc) {
  const int nt = (k + 15) / 16;
  const size_t lds = (size_t)2 * RS * 16 * (nt | 1) * sizeof(double);
  auto fn = k_gram_sym<NW, TPW, RS, MT>;
  hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fn, dim3(chunks), dim3(64 * NW), lds, st, n, k,
                     wide_rows(X, ldx, k) ? 1 : 0, X, ldx, part, rpc);
  return hipGetLastError();
}

hipError_t launch_gram(hipStream_t st, int64_t n, int k1, int k2, const double* X, int ldx,
                       const double* Y, int ldy, double* G, int ldg, double* part) {
  return launch_gram_chunks(st, n, k1, k2, X, ldx, Y, ldy, G, ldg, part,
                            gram_chunks_of(n, k1, k2, X == Y && ldx == ldy));
}

hipError_t launch_gram_chunks(hipStream_t st, int64_t n, int k1, int k2, const double* X,
                              int ldx, const double* Y, int ldy, double* G, int ldg, double* part,
                              int chunks) {
  if (k1 <= 0 || k2 <= 0) return hipSuccess;
  if (chunks < 1) chunks = 1;
  const bool same = X == Y && ldx == ldy;
  const int most = gram_chunks_of(n, k1, k2, same);
  if (chunks > most) chunks = most;
  int64_t rpc = (n + chunks - 1) / chunks;
  rpc = (rpc + 3) & ~int64_t(3);
  // a chunk's rows are addressed through 32-bit buffer offsets
  if (rpc * (int64_t)(ldx > ldy ? ldx : ldy) * 8 > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  const int ta_n = (k1 + 15) / 16, tb_n = (k2 + 15) / 16;
  if (gram_symmetric(n, k1, k2, same)) {
    // waves and tiles per wave by the tile count: 10, 21, 45, 78 at k = 64, 96,
    // 144, 192; shorter stages where a row is long, so that two workgroups fit
    hipError_t e;
    if (ta_n <= 4)
      e = launch_sym<4, 3, 32, 4>(st, n, k1, X, ldx, part, chunks, rpc);
    else if (ta_n <= 6)
      e = launch_sym<8, 3, 32, 6>(st, n, k1, X, ldx, part, chunks, rpc);
    else if (ta_n <= 9)
      e = launch_sym<8, 6, 16, 9>(st, n, k1, X, ldx, part, chunks, rpc);
    else
      e = launch_sym<8, 10, 16, 12>(st, n, k1, X, ldx, part, chunks, rpc);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_sym_reduce, dim3(4 * (ta_n * (ta_n + 1) / 2)), dim3(512), 0, st,
                       chunks, k1, part, G, ldg);
    return hipGetLastError();
  }
  // one workgroup per tile block and chunk: 3 x 3 blocks when that still
  // gives twelve or more per chunk, else 2 x 2
  auto nblk = [&](int ta, int tb) { return ((ta_n + ta - 1) / ta) * ((tb_n + tb - 1) / tb); };
  const bool big = nblk(3, 3) >= 12;
  const int blocks = big ? nblk(3, 3) : nblk(2, 2);
  dim3 grid(chunks, blocks);
  if (big)
    hipLaunchKernelGGL((k_gram_partial<3, 3, 2>), grid, dim3(256), 0, st, n, k1, k2, X, ldx, Y,
                       ldy, part, rpc);
  else
    hipLaunchKernelGGL((k_gram_partial<2, 2, 4>), grid, dim3(256), 0, st, n, k1, k2, X, ldx, Y,
                       ldy, part, rpc);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gram_reduce, dim3((k1 * k2 + 63) / 64), dim3(256), 0, st, chunks, k1,
                     k2, part, G, ldg);
  return hipGetLastError();
}

// ============================================================================
// TSMM Y = X S on v_mfma_f64_16x16x4f64: each wave computes a 16-row strip of
// Y for TB 16-column tiles; A operand lane l reads X[r0 + l%16][a0 + l/16],
// B operand reads S[a0 + l/16][b0 + l%16].
// ============================================================================
template <int TB>
__global__ __launch_bounds__(256) void k_tsmm(int64_t n, int k, int k2,
                                              const double* __restrict__ X, int ldx,
                                              const double* __restrict__ S, int lds,
                                              double* __restrict__ Y, int ldy) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * 16;
  if (r0 >= n) return;
  const int tb_n = (k2 + 15) >> 4;
  const int tb0 = blockIdx.y * TB;
  const int nb = min(TB, tb_n - tb0);  // wave-uniform
  const int li = lane & 15, lk = lane >> 4;
  v4d acc[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
  const int64_t arow = r0 + li;
  const bool r_ok = arow < n;
  int bcol[TB];
  bool bok[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    bcol[t] = (tb0 + t) * 16 + li;
    bok[t] = t < nb && bcol[t] < k2;
  }
  for (int a0 = 0; a0 < k; a0 += 4) {
    const int acol = a0 + lk;
    const bool aok = acol < k;
    const double a = (aok && r_ok) ? X[arow * ldx + acol] : 0.0;
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      if (t >= nb) continue;
      const double bv = (aok && bok[t]) ? S[(size_t)acol * lds + bcol[t]] : 0.0;
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv, acc[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    if (!bok[t]) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t r = r0 + lk + 4 * v;
      if (r < n) Y[r * ldy + bcol[t]] = acc[t][v];
    }
  }
}

// The same product with the workgroup's TB * 16 columns of S staged in LDS
// (zero past k and k2) and read from there by every wave, where k_tsmm
// re-reads them from L2 for each 16-row strip.  A workgroup of 8 waves
// takes RW blocks of 128 rows (16 per wave) in turn; a wave loads its A
// fragments 8 k-steps at a time, all issued together through a buffer
// descriptor over its 16 rows (a row past n reads zero; a column past k
// reads column k - 1, which meets a zero row of S), then issues the MFMAs.
constexpr int kTsmmThreads = 512;
constexpr int kTsmmRW = 4;
constexpr int kTsmmMaxLds = 128 * 1024;

template <int TB>
__global__ __launch_bounds__(kTsmmThreads) void k_tsmm_lds(int64_t n, int k, int k2,
                                                           const double* __restrict__ X, int ldx,
                                                           const double* __restrict__ S, int lds,
                                                           double* __restrict__ Y, int ldy) {
  extern __shared__ double sl[];  // kp x (16 TB), row-major
  constexpr int SC = 16 * TB;
  const int kp = (k + 3) & ~3;
  const int tb0 = blockIdx.y * TB;
  for (int e = threadIdx.x; e < kp * SC; e += kTsmmThreads) {
    const int a = e / SC, gc = tb0 * 16 + e % SC;
    sl[e] = (a < k && gc < k2) ? S[(size_t)a * lds + gc] : 0.0;
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int nsteps = kp >> 2;
  constexpr int KB = 8;  // k-steps per batch of A loads
  for (int rb = 0; rb < kTsmmRW; ++rb) {
    const int64_t r0 = (((int64_t)blockIdx.x * kTsmmRW + rb) * (kTsmmThreads / 64) + wave) * 16;
    if (r0 >= n) break;  // wave-uniform
    const int rows = (int)min<int64_t>(16, n - r0);
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(X + r0 * ldx), (short)0, rows * ldx * 8, kBufferWord3);
    v4d acc[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
    for (int s0 = 0; s0 < nsteps; s0 += KB) {
      double a[KB];
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int col = min(4 * (s0 + u) + lk, k - 1);
        a[u] = __builtin_bit_cast(double,
                                  __builtin_amdgcn_raw_buffer_load_b64(xs, (li * ldx + col) * 8, 0, 0));
      }
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        // steps past kp meet rows of sl that do not exist: skip them (uniform)
        if (s0 + u >= nsteps) break;
        const double* srow = sl + (4 * (s0 + u) + lk) * SC + li;
#pragma unroll
        for (int t = 0; t < TB; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], srow[16 * t], acc[t], 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const int c = (tb0 + t) * 16 + li;
      if (c >= k2) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + lk + 4 * v;
        if (r < n) Y[r * ldy + c] = acc[t][v];
      }
    }
  }
}

hipError_t launch_tsmm(hipStream_t st, int64_t n, int k, int k2, const double* X, int ldx,
                       const double* S, int lds, double* Y, int ldy) {
  if (n <= 0 || k2 <= 0) return hipSuccess;
  const int tb_n = (k2 + 15) / 16;
  // one wave covers up to six column tiles, so X is read once for k2 <= 96
  constexpr int TB = 6;
  const size_t lds_bytes = (size_t)((k + 3) & ~3) * 16 * TB * sizeof(double);
  // staging S pays once there are enough rows to give every CU a workgroup
  // of 512 rows; below that the per-strip kernel spreads wider
  if (k >= 1 && lds_bytes <= (size_t)kTsmmMaxLds && n >= (int64_t)1 << 17) {
    hipError_t e = hipFuncSetAttribute((const void*)k_tsmm_lds<TB>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    const int64_t rows_per_wg = (int64_t)kTsmmRW * (kTsmmThreads / 64) * 16;
    dim3 grid((unsigned)((n + rows_per_wg - 1) / rows_per_wg), (tb_n + TB - 1) / TB);
    hipLaunchKernelGGL(k_tsmm_lds<TB>, grid, dim3(kTsmmThreads), lds_bytes, st, n, k, k2, X, ldx,
                       S, lds, Y, ldy);
    return hipGetLastError();
  }
  dim3 grid((unsigned)((n + 63) / 64), (tb_n + TB - 1) / TB);
  hipLaunchKernelGGL(k_tsmm<TB>, grid, dim3(256), 0, st, n, k, k2, X, ldx, S, lds, Y, ldy);
  return hipGetLastError();
}

// ============================================================================
// Y <- Y M in place for an upper triangular M (CholQR's R^{-1}), unless the
// factorization failed (*status == 2).  The upper tiles of M are staged in LDS;
// a wave takes 16 rows at a time, loads all their columns into registers (pairs
// of columns, 16 bytes a lane: lane l holds row l % 16, columns 8 s + 2 (l / 16)
// and the next, which are k-steps 2 s and 2 s + 1; M's rows are staged in that
// order) and writes column tile t from the tiles s <= t, so a row is read once
// and written once.  Measured at n = 1e6, k = 84: 280 us; a product with
// the square M into another block and a copy back were 522 + 251 us.
// ============================================================================
template <int NT, int NW>
__global__ __launch_bounds__(64 * NW) void k_tri_apply(int64_t n, int k, int wide, double* Y,
                                                       int ldy,
                                                       const double* __restrict__ M, int ldm,
                                                       const int* __restrict__ status) {
  extern __shared__ double sm[];  // tiles (s, t), s <= t, by column t
  if (*status == 2) return;
  constexpr int kTiles = NT * (NT + 1) / 2;
  for (int e = threadIdx.x; e < kTiles * 256; e += 64 * NW) {
    int s = e >> 8, t = 0;
    while (s > t) s -= ++t;
    const int r = (e >> 4) & 15, c = e & 15;
    // position r holds row 8 (r / 8) + 2 (r % 4) + (r / 4) % 2 of the tile
    const int i = 16 * s + 8 * (r >> 3) + 2 * (r & 3) + ((r >> 2) & 1), j = 16 * t + c;
    sm[e] = i < k && j < k ? M[(size_t)i * ldm + j] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t step = (int64_t)gridDim.x * NW * 16;
  for (int64_t r0 = ((int64_t)blockIdx.x * NW + wave) * 16; r0 < n; r0 += step) {
    const int rows = (int)min<int64_t>(16, n - r0);
    const __amdgpu_buffer_rsrc_t ys = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Y + r0 * ldy), (short)0, ((rows - 1) * ldy + k) * 8, kBufferWord3);
    double a[4 * NT];
#pragma unroll
    for (int s = 0; s < 2 * NT; ++s) {
      const int c = 8 * s + 2 * lk;
      const bool in = li < rows;
      const double2 v = load_pair(ys, (li * ldy + c) * 8, in && c < k, in && c + 1 < k, wide != 0);
      a[2 * s] = v.x;
      a[2 * s + 1] = v.y;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      v4d acc{0.0, 0.0, 0.0, 0.0};
      const double* col = sm + (t * (t + 1) / 2) * 256 + lane;
#pragma unroll
      for (int q = 0; q < 4 * (t + 1); ++q)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], col[64 * q], acc, 0, 0, 0);
      const int c = 16 * t + li;
      if (c < k) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (lk + 4 * v < rows) Y[(r0 + lk + 4 * v) * ldy + c] = acc[v];
      }
      // M's fragments of later tiles are not read ahead of this tile's: all of
      // them at once spilled registers (888 to 2024 bytes a lane from k = 97 on)
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int NT, int NW>
static hipError_t launch_tri(hipStream_t st, int64_t n, int k, double* Y, int ldy,
                             const double* M, int ldm, const int* status) {
  auto fn = k_tri_apply<NT, NW>;
  const size_t lds = (size_t)NT * (NT + 1) / 2 * 256 * sizeof(double);
  hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  const int64_t want = (n + 16 * NW - 1) / (16 * NW);
  hipLaunchKernelGGL(fn, dim3((unsigned)(want < 1024 ? want : 1024)), dim3(64 * NW), lds, st, n,
                     k, wide_rows(Y, ldy, k) ? 1 : 0, Y, ldy, M, ldm, status);
  return hipGetLastError();
}

hipError_t launch_tri_apply(hipStream_t st, int64_t n, int k, double* Y, int ldy, const double* M,
                            int ldm, const int* status) {
  if (n <= 0 || k <= 0) return hipSuccess;
  if (k > kSymMaxK || ldy > (1 << 22)) return hipErrorInvalidValue;
  const int nt = (k + 15) / 16;
  if (nt <= 2) return launch_tri<2, 4>(st, n, k, Y, ldy, M, ldm, status);
  if (nt <= 4) return launch_tri<4, 4>(st, n, k, Y, ldy, M, ldm, status);
  if (nt <= 6) return launch_tri<6, 4>(st, n, k, Y, ldy, M, ldm, status);
  if (nt <= 9) return launch_tri<9, 8>(st, n, k, Y, ldy, M, ldm, status);
  return launch_tri<12, 8>(st, n, k, Y, ldy, M, ldm, status);
}

// ============================================================================
// Ritz residuals R = W - Q diag(theta) and column norms.  Threads are laid out
// 4 rows x 64 columns; per-thread sums are combined in a fixed order.
// ============================================================================
__global__ __launch_bounds__(256) void k_resid_partial(int64_t n, int k,
                                                       const double* __restrict__ W,
                                                       const double* __restrict__ Q, int ld,
                                                       const double* __restrict__ theta,
                                                       double* __restrict__ R,
                                                       double* __restrict__ part,
                                                       int64_t rows_per_chunk) {
  __shared__ double sh[2][4][64];
  const int chunk = blockIdx.x;
  const int64_t rb = (int64_t)chunk * rows_per_chunk;
  int64_t re = rb + rows_per_chunk;
  if (re > n) re = n;
  const int ty = threadIdx.x >> 6, tx = threadIdx.x & 63;
  for (int c0 = 0; c0 < k; c0 += 64) {
    const int c = c0 + tx;
    double s1 = 0.0, s2 = 0.0;
    if (c < k) {
      const double th = theta[c];
      for (int64_t r = rb + ty; r < re; r += 4) {
        const double q = Q[r * ld + c];
        const double v = W[r * ld + c] - th * q;
        R[r * ld + c] = v;
        s1 += v * v;
        s2 += q * q;
      }
    }
    sh[0][ty][tx] = s1;
    sh[1][ty][tx] = s2;
    __syncthreads();
    if (ty == 0 && c < k) {
      const double a = ((sh[0][0][tx] + sh[0][1][tx]) + sh[0][2][tx]) + sh[0][3][tx];
      const double b = ((sh[1][0][tx] + sh[1][1][tx]) + sh[1][2][tx]) + sh[1][3][tx];
      part[(size_t)chunk * 2 * k + c] = a;
      part[(size_t)chunk * 2 * k + k + c] = b;
    }
    __syncthreads();
  }
}

__global__ void k_resid_final(int chunks, int k, const double* __restrict__ part, double s_win,
                              double* __restrict__ res, double* __restrict__ qn) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= k) return;
  double a = 0.0, b = 0.0;
  for (int ch = 0; ch < chunks; ++ch) {
    a += part[(size_t)ch * 2 * k + c];
    b += part[(size_t)ch * 2 * k + k + c];
  }
  const double q = sqrt(b);
  res[c] = sqrt(a) / (s_win * q);
  qn[c] = q;
}

hipError_t launch_residual(hipStream_t st, int64_t n, int k, const double* W, const double* Q,
                           int ld, const double* theta, double s_win, double* R, double* res,
                           double* qn, double* part) {
  const int chunks = gram_chunks(n);
  const int64_t rpc = (n + chunks - 1) / chunks;
  hipLaunchKernelGGL(k_resid_partial, dim3(chunks), dim3(256), 0, st, n, k, W, Q, ld, theta, R,
                     part, rpc);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_resid_final, dim3((k + 63) / 64), dim3(64), 0, st, chunks, k, part, s_win,
                     res, qn);
  return hipGetLastError();
}

// ============================================================================
// Filter combination (eq. projector-quad, upper-half nodes, real part).
// ============================================================================
__global__ void k_gamma(int nc, int k, const double* __restrict__ zw,
                        const double* __restrict__ theta, double* __restrict__ gamma) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nc * k) return;
  const int j = e / k, i = e % k;
  const zd z{zw[2 * j], zw[2 * j + 1]};
  const zd w{zw[2 * nc + 2 * j], zw[2 * nc + 2 * j + 1]};
  const zd g = zdiv(w, zd{z.re - theta[i], z.im});
  gamma[2 * e] = g.re;
  gamma[2 * e + 1] = g.im;
}

hipError_t launch_gamma(hipStream_t st, int nc, int k, const double* zw, const double* theta,
                        double* gamma) {
  const int tot = nc * k;
  hipLaunchKernelGGL(k_gamma, dim3((tot + 255) / 256), dim3(256), 0, st, nc, k, zw, theta, gamma);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void k_combine(int64_t n, int nc, int k,
                                                 const double* __restrict__ gamma,
                                                 const double* __restrict__ zw, int residual,
                                                 const double* __restrict__ Q, int ldq,
                                                 const cpx<T>* __restrict__ D, int ldd,
                                                 double* __restrict__ Qt, int ldt) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * k) return;
  const int64_t r = e / k;
  const int i = (int)(e % k);
  double acc = 0.0;
  if (residual) {
    const double q = Q[r * ldq + i];
    for (int j = 0; j < nc; ++j) {
      const cpx<T> d = D[r * ldd + (size_t)j * k + i];
      const double gr = gamma[2 * (j * k + i)], gi = gamma[2 * (j * k + i) + 1];
      acc += gr * (q + (double)d.re) - gi * (double)d.im;
    }
  } else {
    for (int j = 0; j < nc; ++j) {
      const cpx<T> d = D[r * ldd + (size_t)j * k + i];
      const double wr = zw[2 * nc + 2 * j], wi = zw[2 * nc + 2 * j + 1];
      acc += wr * (double)d.re - wi * (double)d.im;
    }
  }
  Qt[r * ldt + i] = acc;
}

hipError_t launch_combine(hipStream_t st, int64_t n, int nc, int k, const double* gamma,
                          const double* zw, bool residual_form, const double* Q, int ldq,
                          const void* D, int ldd, bool d32, double* Qt, int ldt) {
  const int64_t tot = n * k;
  dim3 grid((unsigned)((tot + 255) / 256));
  if (d32)
    hipLaunchKernelGGL(k_combine<float>, grid, dim3(256), 0, st, n, nc, k, gamma, zw,
                       residual_form ? 1 : 0, Q, ldq, (const cpx<float>*)D, ldd, Qt, ldt);
  else
    hipLaunchKernelGGL(k_combine<double>, grid, dim3(256), 0, st, n, nc, k, gamma, zw,
                       residual_form ? 1 : 0, Q, ldq, (const cpx<double>*)D, ldd, Qt, ldt);
  return hipGetLastError();
}

// ============================================================================
// Gaussian sketch: Philox4x32-10 (Salmon et al., SC'11) + Box-Muller.
// ============================================================================
__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
  for (int rnd = 0; rnd < 10; ++rnd) {
    const uint32_t lo0 = M0 * c[0], hi0 = __umulhi(M0, c[0]);
    const uint32_t lo1 = M1 * c[2], hi1 = __umulhi(M1, c[2]);
    const uint32_t n0 = hi1 ^ c[1] ^ k0;
    const uint32_t n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

__global__ void k_gaussian(int64_t n, int w, uint32_t s0, uint32_t s1, double* __restrict__ O,
                           int ld) {
  const int pairs = (w + 1) >> 1;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * pairs) return;
  const int64_t i = e / pairs;
  const int kp = (int)(e % pairs);
  uint32_t c[4] = {(uint32_t)(i & 0xFFFFFFFF), (uint32_t)((uint64_t)i >> 32), (uint32_t)kp, 0u};
  philox10(c, s0, s1);
  const uint64_t x1 = ((uint64_t)c[0] << 32) | c[1];
  const uint64_t x2 = ((uint64_t)c[2] << 32) | c[3];
  const double u1 = (double)(x1 >> 11) * 0x1.0p-53 + 0x1.0p-54;
  const double u2 = (double)(x2 >> 11) * 0x1.0p-53 + 0x1.0p-54;
  const double rad = sqrt(-2.0 * log(u1));
  const double ang = 6.283185307179586476925287 * u2;
  O[i * ld + 2 * kp] = rad * cos(ang);
  if (2 * kp + 1 < w) O[i * ld + 2 * kp + 1] = rad * sin(ang);
}

hipError_t launch_gaussian(hipStream_t st, int64_t n, int w, uint64_t seed, double* O, int ld) {
  const int64_t tot = n * ((w + 1) / 2);
  hipLaunchKernelGGL(k_gaussian, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, w,
                     (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), O, ld);
  return hipGetLastError();
}

// ============================================================================
// Layout helpers.
// ============================================================================
__global__ void k_col2row(int64_t n, int k, const double* __restrict__ src,
                          double* __restrict__ dst, int ldd) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * k) return;
  const int64_t r = e / k;
  const int c = (int)(e % k);
  dst[r * ldd + c] = src[(int64_t)c * n + r];
}

hipError_t launch_colmajor_to_rowmajor(hipStream_t st, int64_t n, int k, const double* src,
                                       double* dst, int ldd) {
  const int64_t tot = n * k;
  hipLaunchKernelGGL(k_col2row, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, k, src,
                     dst, ldd);
  return hipGetLastError();
}

__global__ void k_copy_cols(int64_t n, int k, const double* __restrict__ src, int lds,
                            double* __restrict__ dst, int ldd) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * k) return;
  const int64_t r = e / k;
  const int c = (int)(e % k);
  dst[r * ldd + c] = src[r * lds + c];
}

hipError_t launch_copy_cols(hipStream_t st, int64_t n, int k, const double* src, int lds,
                            double* dst, int ldd) {
  const int64_t tot = n * k;
  hipLaunchKernelGGL(k_copy_cols, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, k,
                     src, lds, dst, ldd);
  return hipGetLastError();
}

// p[0..n) = v.  A kernel, not a memset node, so it can sit in a captured graph.
__global__ void k_fill_int(int* __restrict__ p, int v, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_int(hipStream_t st, int* p, int v, int n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_int, dim3((n + 255) / 256), dim3(256), 0, st, p, v, n);
  return hipGetLastError();
}

__global__ void k_row2col(int64_t n, int k, const double* __restrict__ src, int lds,
                          double* __restrict__ dst) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * k) return;
  const int c = (int)(e / n);
  const int64_t r = e % n;
  dst[e] = src[r * lds + c];
}

hipError_t launch_rowmajor_to_colmajor(hipStream_t st, int64_t n, int k, const double* src,
                                       int lds, double* dst) {
  const int64_t tot = n * k;
  if (tot <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_row2col, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, k, src,
                     lds, dst);
  return hipGetLastError();
}

// One block per exported column: norm, first index of the largest |entry|,
// then the scaled column into column-major dst.
__global__ __launch_bounds__(256) void k_export(int64_t n, const int* __restrict__ sel,
                                                const double* __restrict__ src, int lds,
                                                double* __restrict__ dst) {
  __shared__ double s_sq[4], s_mx[4];
  __shared__ int64_t s_ix[4];
  const int c = blockIdx.x;
  const int col = sel[c];
  double sq = 0.0, mx = -1.0;
  int64_t ix = n;
  for (int64_t r = threadIdx.x; r < n; r += 256) {
    const double v = src[r * lds + col];
    sq += v * v;
    const double a = fabs(v);
    if (a > mx) {  // rows visited in increasing order: keeps the first maximum
      mx = a;
      ix = r;
    }
  }
  // wave reduction: (max, lowest index) and sum
  for (int off = 32; off > 0; off >>= 1) {
    const double omx = __shfl_xor(mx, off, 64);
    const int64_t oix = __shfl_xor(ix, off, 64);
    if (omx > mx || (omx == mx && oix < ix)) {
      mx = omx;
      ix = oix;
    }
    sq += __shfl_xor(sq, off, 64);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_sq[wv] = sq;
    s_mx[wv] = mx;
    s_ix[wv] = ix;
  }
  __syncthreads();
  double tsq = 0.0, tmx = -1.0;
  int64_t tix = n;
  for (int w = 0; w < 4; ++w) {
    tsq += s_sq[w];
    if (s_mx[w] > tmx || (s_mx[w] == tmx && s_ix[w] < tix)) {
      tmx = s_mx[w];
      tix = s_ix[w];
    }
  }
  const double sgn = (tix < n && src[tix * lds + col] < 0.0) ? -1.0 : 1.0;
  const double sc = sgn / sqrt(tsq);
  for (int64_t r = threadIdx.x; r < n; r += 256) dst[(int64_t)c * n + r] = src[r * lds + col] * sc;
}

hipError_t launch_export_vectors(hipStream_t st, int64_t n, int cnt, const int* sel,
                                 const double* src, int lds, double* dst, double* part) {
  (void)part;
  if (cnt <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_export, dim3(cnt), dim3(256), 0, st, n, sel, src, lds, dst);
  return hipGetLastError();
}

}  // namespace rafeast
