// Exact shifted solves for standard FEAST, the baseline of Section 5.1 (FEAST
// with sparse direct factorizations of the shifted matrices).  Each shifted
// matrix M_j = z_j I - A is factorized once as M_j = L_j D_j L_j^T (complex
// symmetric: the transpose, not the conjugate transpose; L unit lower
// triangular, D diagonal) and every filter application solves by substitution.
//
// Order: A in reverse Cuthill-McKee order (the streaming engine's), whose lower
// bandwidth b bounds the factors: LDL^T without pivoting creates no fill
// outside the band.  No pivoting is needed: the leading principal submatrices
// of z I - A are z I - A_k with A_k real symmetric, whose eigenvalues z - mu
// are nonzero for Im z != 0, so every pivot exists; and the imaginary part of
// M is Im z I, definite, for which elimination without pivoting has bounded
// element growth (N. J. Higham, Factorizing complex symmetric matrices with
// positive definite real and imaginary parts, Math. Comp. 1998).
//
// Storage: per shift an n x (b + 1) complex array W, row r holding M(r, r - d)
// in W[r][d], d = 0..b (d = 0 the diagonal).  Bands below 31 are kept at b = 31,
// which the blocks below need, as long as that takes no more than 32 GiB and
// fits, and at their own width, with the scalar factors, above.
//
// Factorization: block L D L^T in block columns (panels) of 32.  With the
// window's rows below panel c, M21 (b x 32) and the panel's own block M11 (both
// as updated by the earlier panels), one step is
//   W22 -= M21 M11^{-1} M21^T,
// so a panel needs only the inverse of its 32 x 32 block: the factors kept in W
// are M21 itself and the lower triangle of the symmetric M11^{-1}, over M11.
// The pivots met while inverting are those of the scalar L D L^T.  One launch
// per panel, all shifts together: workgroups own 32 x 32 tiles of the window,
// form -M21 M11^{-1} for their rows and update their tile on the FP64 matrix
// cores; the workgroup of the tile that holds the next panel's block inverts
// it at once (in registers), so no launch is serial.
// Solves: one workgroup per (shift, two right-hand sides), blocks of 32 rows:
//   forward  y_J = b_J - sum_{I < J} M_JI v_I, v_I = M_II^{-1} y_I,
//   backward x_J = M_JJ^{-1} (y_J - sum_{I > J} M_IJ^T x_I),
// with no substitution inside a block: each is products with entries of W, in
// which the rows solved more than one block ago go first, while the block
// before finishes.
#include "device.h"
#include "kernels.h"

#include <algorithm>

namespace rafeast {

namespace {

typedef cpx<double> zc;

__device__ __forceinline__ zc csub(zc a, zc b) { return zc{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ void cfma(zc& s, zc a, zc x) {
  s.re += a.re * x.re - a.im * x.im;
  s.im += a.re * x.im + a.im * x.re;
}

__device__ __forceinline__ bool cfinite(zc a) { return isfinite(a.re) && isfinite(a.im); }

constexpr int kBB = 32;                // panel width, tile and solve block
constexpr size_t kBandSolveRingBytes = 128 * 1024;  // LDS ring of the solve
constexpr int kSolveThreads = 512;
constexpr int kSolveCols = 2;          // right-hand sides per workgroup
constexpr int kSolveSlices = kSolveThreads / kBB;  // threads per block row

// W_j: every entry zero, then z_j on the diagonal and -A(r, c) at (r, r - c)
// for the lower entries c <= r of the reordered CSR.  Thread per row.
__global__ __launch_bounds__(256) void k_band_assemble(int n, int b, const int* __restrict__ rowptr,
                                                       const int* __restrict__ col,
                                                       const double* __restrict__ val,
                                                       const double* __restrict__ z,
                                                       zc* __restrict__ W, size_t stride) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n) return;
  const int j = blockIdx.y;
  zc* __restrict__ row = W + (size_t)j * stride + (size_t)r * (b + 1);
  for (int d = 0; d <= b; ++d) row[d] = zc{0.0, 0.0};
  row[0] = zc{z[2 * j], z[2 * j + 1]};
  for (int t = rowptr[r]; t < rowptr[r + 1]; ++t) {
    const int c = col[t];
    if (c > r || r - c > b) continue;
    row[r - c].re -= val[t];
  }
}

// The panel step.  LDS planes of kBB rows kPitch doubles apart: a fragment read
// (16 rows x 4 columns over the wave) meets each bank pair twice, the least
// 64 eight-byte lanes can.
constexpr int kStepThreads = 256;
constexpr int kPitch = 36;

// Entries of W through raw buffer descriptors over the rows a workgroup's step
// can touch: an entry outside the band is asked for at an offset past the
// descriptor and a row past n lies past it, and both read zero, so no branch
// stands between the loads.
constexpr int kNoEntry = 0x7ffffff0;
typedef unsigned v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const zc* __restrict__ W, int first,
                                                          int end, int ldw) {
  const int rows = max(0, end - first);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)max(0, first) * ldw), (short)0,
                                           rows * ldw * (int)sizeof(zc), 0x00020000);
}
__device__ __forceinline__ zc entry(__amdgpu_buffer_rsrc_t rs, int off) {
  return __builtin_bit_cast(zc, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
}
struct Plane {
  double re[kBB][kPitch], im[kBB][kPitch];
};

// acc += A B over kBB inner indices for this wave's 16 x 16 tile: A's rows
// r0.., B's columns c0.. (BT: B(q, c) = Bm[c][q]).  Lane l holds A(l % 16,
// l / 16) and B(l / 16, l % 16) of a step, D(l / 16 + 4 v, l % 16).
template <bool BT>
__device__ __forceinline__ void tile_product(const Plane& A, const Plane& Bm, int r0, int c0,
                                             v4d& cr, v4d& ci) {
  const int li = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int q = 0; q < kBB; q += 4) {
    const double ar = A.re[r0 + li][q + lk], ai = A.im[r0 + li][q + lk];
    const double br = BT ? Bm.re[c0 + li][q + lk] : Bm.re[q + lk][c0 + li];
    const double bi = BT ? Bm.im[c0 + li][q + lk] : Bm.im[q + lk][c0 + li];
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, ci, 0, 0, 0);
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, bi, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, ci, 0, 0, 0);
  }
}

// The inverse (i11, i12, i22) of two pivots (p11, p12, p22).  From the
// determinant (one reciprocal in the chain) where its square is far from the
// ends of the range, else by the scalar pivots p11 and p22 - p12^2 / p11, whose
// products stay in range whatever the scale of the matrix.  Returns 0, or 1 or 2
// for a vanishing or non-finite first or second pivot.  The branch is uniform;
// the second form is out of the chain.
__device__ __forceinline__ int inverse2(zc p11, zc p12, zc p22, zc& i11, zc& i12, zc& i22) {
  zc det{0.0, 0.0};
  cfma(det, p11, p22);
  cfma(det, zc{-p12.re, -p12.im}, p12);
  const double m = det.re * det.re + det.im * det.im;
  i11 = i12 = i22 = zc{0.0, 0.0};
  if (m > 0x1.0p-900 && m < 0x1.0p+900) {
    const double x = rcp_nr(m);
    const zc q{det.re * x, -det.im * x};
    cfma(i11, p22, q);
    cfma(i12, zc{-p12.re, -p12.im}, q);
    cfma(i22, p11, q);
    return p11.re != 0.0 || p11.im != 0.0 ? 0 : 1;
  }
  if (!(cfinite(p11) && (p11.re != 0.0 || p11.im != 0.0))) return 1;
  const zd one{1.0, 0.0}, l = zdiv_fast(zd{p12.re, p12.im}, zd{p11.re, p11.im});
  zc d2 = p22;
  cfma(d2, zc{-l.re, -l.im}, p12);
  if (!(cfinite(d2) && (d2.re != 0.0 || d2.im != 0.0))) return 2;
  const zd r1 = zdiv_fast(one, zd{p11.re, p11.im}), r2 = zdiv_fast(one, zd{d2.re, d2.im});
  const zd lr = zmul(l, r2);
  i22 = zc{r2.re, r2.im};
  i12 = zc{-lr.re, -lr.im};
  i11 = zc{r1.re, r1.im};
  cfma(i11, zc{lr.re, lr.im}, zc{l.re, l.im});
  return 0;
}

// The 32 x 32 symmetric block held in the waves' tiles (wave w: rows 16 (w /
// 2).., columns 16 (w % 2)..) becomes minus its inverse: the sweep operator on
// two pivots K = (k, k + 1) at a time, with P = A_KK,
//   A_KK = -P^{-1}, A_iK = A_iK P^{-1}, A_ij -= A_iK P^{-1} A_Kj,
// rows k and k + 1 going round through LDS, one barrier a step.  The chain
// write - barrier - read - 1/det - update is all the time there is; one pivot a
// step, with two dependent reciprocals, made the launch 4.4 us longer.
// Returns 0, or 1 + the index of a vanishing or non-finite pivot (the same in
// every thread).
__device__ __forceinline__ int sweep_block(v4d& cr, v4d& ci, zc (*rowbuf)[2][kBB]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = 16 * (wave >> 1), c0 = 16 * (wave & 1);
  const int li = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
  const int col = c0 + li;
  int fail = 0;
#pragma unroll 1
  for (int h = 0; h < kBB && !fail; h += 16) {
#pragma unroll
    for (int kk = 0; kk < 16; kk += 2) {
      const int k = h + kk, vk = kk >> 2;
      zc(*rows)[kBB] = rowbuf[(kk >> 1) & 1];
      // rows k, k + 1: element kk / 4 of two of the four lane groups of the
      // waves with r0 == h
      const bool mine = r0 == h && (lk >> 1) == ((kk & 3) >> 1);
      if (mine) rows[lk & 1][col] = zc{cr[vk], ci[vk]};
      __syncthreads();
      const zc p11 = rows[0][k], p12 = rows[0][k + 1], p22 = rows[1][k + 1];
      const zc a0 = rows[0][col], a1 = rows[1][col];
      zc b0[4], b1[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        b0[v] = rows[0][r0 + lk + 4 * v];
        b1[v] = rows[1][r0 + lk + 4 * v];
      }
      zc i11, i12, i22;
      const int vanished = inverse2(p11, p12, p22, i11, i12, i22);
      if (!fail && vanished) fail = k + vanished;
      // t = P^{-1} A_Kj; in a column of K, -P^{-1}'s own and a = 0, so that the
      // one update below gives A_iK P^{-1}
      const bool ck0 = col == k, ck1 = col == k + 1;
      zc t0{0.0, 0.0}, t1{0.0, 0.0};
      cfma(t0, i11, a0);
      cfma(t0, i12, a1);
      cfma(t1, i12, a0);
      cfma(t1, i22, a1);
      if (ck0) {
        t0 = zc{-i11.re, -i11.im};
        t1 = zc{-i12.re, -i12.im};
      }
      if (ck1) {
        t0 = zc{-i12.re, -i12.im};
        t1 = zc{-i22.re, -i22.im};
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        zc u{0.0, 0.0};
        cfma(u, b0[v], t0);
        cfma(u, b1[v], t1);
        zc a{ck0 || ck1 ? 0.0 : cr[v], ck0 || ck1 ? 0.0 : ci[v]};
        a = csub(a, u);
        if (v == vk && mine) a = (lk & 1) ? t1 : t0;
        cr[v] = a.re;
        ci[v] = a.im;
      }
    }
  }
  return fail;
}

// Writes the lower triangle of the inverse (minus the swept block) over rows
// e.. of W, or the failure.
__device__ __forceinline__ void store_inverse(int n, int e, int ldw, zc* __restrict__ W,
                                              const v4d& cr, const v4d& ci, int fail, int* info) {
  const int wave = threadIdx.x >> 6;
  const int li = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
  const int j = e + 16 * (wave & 1) + li;
  if (fail) {
    if (threadIdx.x == 0) *info = e + fail;
    return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = e + 16 * (wave >> 1) + lk + 4 * v;
    if (i < n && j <= i) W[(size_t)i * ldw + (i - j)] = zc{-cr[v], -ci[v]};
  }
}

// The first panel's block inverted (workgroup j: shift j).
__global__ __launch_bounds__(kStepThreads) void k_band_first(int n, int b, zc* __restrict__ Wall,
                                                             size_t stride,
                                                             int* __restrict__ info) {
  __shared__ zc rowbuf[2][2][kBB];
  zc* __restrict__ W = Wall + (size_t)blockIdx.x * stride;
  const int ldw = b + 1, wave = threadIdx.x >> 6;
  const int li = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
  const int j = 16 * (wave & 1) + li;
  v4d cr, ci;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = 16 * (wave >> 1) + lk + 4 * v, hi = max(i, j), lo = min(i, j);
    zc w{i == j ? 1.0 : 0.0, 0.0};  // rows past n: the identity
    if (hi < n) w = W[(size_t)hi * ldw + (hi - lo)];
    cr[v] = w.re;
    ci[v] = w.im;
  }
  const int fail = sweep_block(cr, ci, rowbuf);
  store_inverse(n, 0, ldw, W, cr, ci, fail, info + blockIdx.x);
}

// Panel c (rows and columns c .. c + 31, its block already inverted) applied
// to one 32 x 32 tile of the window's lower triangle, and the next panel's
// block inverted by the workgroup of tile (0, 0).
// What bounds it: the chain load - product - product - 32 pivots of that
// workgroup, once per panel.  A scalar L D L^T needed two launches a panel, one
// workgroup a shift for the block, its inverse triangle and all multipliers
// (90 us) and the window after it (22 us); this launch takes 16.4 us
// (knn n = 8000, band 258, 8 shifts).  Two workgroups a CU are asked for: the
// pivots' second form otherwise takes the registers of one of them (band 3000,
// 4 shifts: 50 -> 63 ms).
__global__ __launch_bounds__(kStepThreads, 2) void k_band_step(int n, int b, int c, int nz,
                                                            zc* __restrict__ Wall, size_t stride,
                                                            int* __restrict__ info) {
  __shared__ Plane Pi, Ri, Ci;  // Pi: the inverse, then -(rows' M21) M11^{-1}
  __shared__ zc rowbuf[2][2][kBB];
  const int j = (int)blockIdx.x % nz, t = (int)blockIdx.x / nz;
  if (info[j] != 0) return;
  zc* __restrict__ W = Wall + (size_t)j * stride;
  const int ldw = b + 1, e = c + kBB, rend = min(n, e + b);
  int bi = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
  while (bi * (bi + 1) / 2 > t) --bi;
  const int bj = t - bi * (bi + 1) / 2;
  const int i0 = e + bi * kBB, j0 = e + bj * kBB;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = tid & 15, lk = (tid & 63) >> 4;
  const int r0 = 16 * (wave >> 1), c0 = 16 * (wave & 1);
  // the panel's inverse (mirrored) and the rows' and columns' M21
  const int lim = max(rend, min(n, e + kBB));
  const __amdgpu_buffer_rsrc_t rs = rows_of(W, c, lim, ldw);
  auto at = [&](int r, int q) {  // offset of M(c + r, c + q), q <= r
    return r - q <= b ? (r * ldw + (r - q)) * (int)sizeof(zc) : kNoEntry;
  };
  zc p[4], mr[4], mc[4], w[4];
  const int jc = j0 + c0 + li;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int idx = tid + kStepThreads * u, r = idx / kBB, q = idx % kBB;
    p[u] = entry(rs, at(max(r, q), min(r, q)));
    mr[u] = entry(rs, at(i0 - c + r, q));
    mc[u] = entry(rs, at(j0 - c + r, q));
  }
  // this lane's entries of the tile (mirrored in the diagonal tiles)
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + r0 + lk + 4 * v;
    w[v] = entry(rs, at(max(i, jc) - c, min(i, jc) - c));
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int idx = tid + kStepThreads * u, r = idx / kBB, q = idx % kBB;
    Pi.re[r][q] = p[u].re;
    Pi.im[r][q] = p[u].im;
    Ri.re[r][q] = mr[u].re;
    Ri.im[r][q] = mr[u].im;
    Ci.re[r][q] = mc[u].re;
    Ci.im[r][q] = mc[u].im;
  }
  v4d cr, ci;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + r0 + lk + 4 * v;
    // past n the next block is the identity
    cr[v] = w[v].re + (t == 0 && i == jc && i >= n ? 1.0 : 0.0);
    ci[v] = w[v].im;
  }
  __syncthreads();
  v4d tr{0.0, 0.0, 0.0, 0.0}, ti{0.0, 0.0, 0.0, 0.0};
  tile_product<false>(Ri, Pi, r0, c0, tr, ti);
  __syncthreads();  // the inverse has been read
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    Pi.re[r0 + lk + 4 * v][c0 + li] = -tr[v];
    Pi.im[r0 + lk + 4 * v][c0 + li] = -ti[v];
  }
  __syncthreads();
  // summed apart and added once: 64 terms added to the window's entries one by one
  // round at their size each time (errors of the solutions half as large again)
  v4d ur{0.0, 0.0, 0.0, 0.0}, ui{0.0, 0.0, 0.0, 0.0};
  tile_product<true>(Pi, Ci, r0, c0, ur, ui);
  cr += ur;
  ci += ui;
  if (t == 0) {
    const int fail = sweep_block(cr, ci, rowbuf);
    store_inverse(n, e, ldw, W, cr, ci, fail, info + j);
    return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + r0 + lk + 4 * v;
    if (i < rend && jc <= i) W[(size_t)i * ldw + (i - jc)] = zc{cr[v], ci[v]};
  }
}

// X[:, j k + c] = M_j^{-1} B[:, c] for the columns of group g and shift j
// (workgroup g nz + j), with the factors of W_j.  Rows of A in the engine
// order r map to caller rows perm[r]; B (n x k, ldb) and X (n x (nz k)
// complex, ldx) are in caller order.  The solve runs in place in X.
// LDS: a ring of the last ring_rows solved rows of the group's columns
// (ring_rows a power of two >= b + 32).
// Forward: sixteen threads a block row, over consecutive entries of its band
// row (one DPP sum); backward: the block's 32 rows on consecutive threads,
// contiguous in each row of W below, sixteen slices of rows summed through LDS.
// The band's reads (132 KB a block at b = 258) pace it, so they are issued a
// block ahead: entries of rows solved more than one block ago (far) are held
// in registers, multiplied and re-issued for the next block before the chain
// near entries - block sum - inverse runs.  Bands past 32 + 16 kFar entries
// read the rest as they go.  A substitution inside the block with a barrier
// per row took 11.9 us a block and direction (knn n = 8000, 8 shifts, 64
// columns), this 3.4 us.
constexpr int kFar = 15;
__global__ __launch_bounds__(kSolveThreads) void k_band_solve(int n, int b, int nz,
                                                              const zc* __restrict__ Wall,
                                                              size_t stride,
                                                              const int* __restrict__ perm,
                                                              const double* __restrict__ B, int ldb,
                                                              int k, zc* __restrict__ X,
                                                              int64_t ldx, int ring_rows) {
  extern __shared__ zc ring[];  // [ring_rows][kSolveCols]
  __shared__ zc yb[kBB][kSolveCols];
  __shared__ zc part[kSolveThreads / 64][kBB][kSolveCols];
  const int j = (int)blockIdx.x % nz, g = (int)blockIdx.x / nz;
  const zc* __restrict__ W = Wall + (size_t)j * stride;
  const int ldw = b + 1, mask = ring_rows - 1;
  const int c0g = g * kSolveCols, ncol = min(kSolveCols, k - c0g);
  const int tid = threadIdx.x;
  const int fr = tid / kSolveSlices, fs = tid % kSolveSlices;  // row, slice (forward, inverse)
  auto zero = [](zc (&s)[kSolveCols]) {
#pragma unroll
    for (int cc = 0; cc < kSolveCols; ++cc) s[cc] = zc{0.0, 0.0};
  };
  auto addr = [&](zc (&s)[kSolveCols], zc w, int q) {
#pragma unroll
    for (int cc = 0; cc < kSolveCols; ++cc) cfma(s[cc], w, ring[(q & mask) * kSolveCols + cc]);
  };
  // sums over the sixteen lanes of a row, in every lane
  auto sum16 = [](zc (&s)[kSolveCols]) {
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) {
        s[cc].re += dpp_f64(s[cc].re, st);
        s[cc].im += dpp_f64(s[cc].im, st);
      }
  };
  // the inverse's entries (fr, fs), (fr, fs + 16) of the block at r0 (identity past n)
  zc iv[2];
  auto load_inv = [&](int r0) {
    const __amdgpu_buffer_rsrc_t rs = rows_of(W, r0, r0 < 0 ? r0 : min(n, r0 + kBB), ldw);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int q = fs + 16 * u, hi = max(fr, q), lo = min(fr, q);
      iv[u] = entry(rs, (hi * ldw + (hi - lo)) * (int)sizeof(zc));
    }
  };
  zc far[kFar], near[2];

  // ---- forward ----
  // entry t of this thread in block r0: column q = r0 - 1 - fs - 16 t
  auto fwd_rows = [&](int r0) { return rows_of(W, r0, min(n, r0 + kBB), ldw); };
  auto fwd_entry = [&](__amdgpu_buffer_rsrc_t rs, int r0, int t) {
    const int back = 1 + fs + 16 * t, d = fr + back;
    return entry(rs, d <= b && back <= r0 ? (fr * ldw + d) * (int)sizeof(zc) : kNoEntry);
  };
  double bv[kSolveCols];
  size_t xo = 0;
  // the caller's row of a block's rows, read a block before it is used (as an
  // address: waiting for it at once would wait for every load before it)
  int pn = perm[min(fr, n - 1)];
  auto load_rhs = [&](int r0) {
    const int r = r0 + fr, pr = pn;
    pn = perm[min(r + kBB, n - 1)];
#pragma unroll
    for (int cc = 0; cc < kSolveCols; ++cc) bv[cc] = 0.0;
    if (fs == 0 && r < n) {
      xo = (size_t)pr * ldx + (size_t)j * k + c0g;
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc)
        if (cc < ncol) bv[cc] = B[(size_t)pr * ldb + c0g + cc];
    }
  };
  // rows before the first (and, backward, after the last) are zeros
  for (int t = tid; t < ring_rows * kSolveCols; t += kSolveThreads) ring[t] = zc{0.0, 0.0};
#pragma unroll
  for (int t = 0; t < kFar; ++t) far[t] = zc{0.0, 0.0};
  near[0] = near[1] = zc{0.0, 0.0};
  load_inv(0);
  load_rhs(0);
  __syncthreads();
  for (int r0 = 0; r0 < n; r0 += kBB) {
    zc s[kSolveCols];
    zero(s);
#pragma unroll
    for (int t = 0; t < kFar; ++t) addr(s, far[t], r0 - 1 - fs - 16 * (t + 2));
    const __amdgpu_buffer_rsrc_t rc = fwd_rows(r0);
    for (int t = kFar + 2; 16 * t < b; t += 4) {
      zc w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = fwd_entry(rc, r0, t + u);
#pragma unroll
      for (int u = 0; u < 4; ++u) addr(s, w[u], r0 - 1 - fs - 16 * (t + u));
    }
    const int rn = r0 + kBB;
    const __amdgpu_buffer_rsrc_t rx = fwd_rows(rn);
#pragma unroll
    for (int t = 0; t < kFar; ++t) far[t] = fwd_entry(rx, rn, t + 2);
    __syncthreads();  // the block before is solved
#pragma unroll
    for (int t = 0; t < 2; ++t) addr(s, near[t], r0 - 1 - fs - 16 * t);
#pragma unroll
    for (int t = 0; t < 2; ++t) near[t] = fwd_entry(rx, rn, t);
    sum16(s);
    const bool row = fs == 0 && r0 + fr < n;
    zc y[kSolveCols];
#pragma unroll
    for (int cc = 0; cc < kSolveCols; ++cc) y[cc] = zc{bv[cc] - s[cc].re, -s[cc].im};
    if (fs == 0) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) yb[fr][cc] = y[cc];
    }
    const size_t xw = xo;
    load_rhs(rn);
    __syncthreads();
    zc v[kSolveCols];
    zero(v);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) cfma(v[cc], iv[u], yb[fs + 16 * u][cc]);
    load_inv(rn);
    sum16(v);
    if (fs == 0) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) ring[((r0 + fr) & mask) * kSolveCols + cc] = v[cc];
    }
    if (row) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc)
        if (cc < ncol) X[xw + cc] = y[cc];
    }
  }

  // ---- backward, blocks from the last; the ring takes the solved x ----
  const int br = tid % kBB, bs = tid / kBB;  // row, slice
  auto bwd_rows = [&](int r0) {  // none before the first block
    return rows_of(W, r0 + kBB, r0 < 0 ? r0 : min(n, r0 + kBB + b), ldw);
  };
  auto bwd_entry = [&](__amdgpu_buffer_rsrc_t rs, int t) {
    const int i = bs + kSolveSlices * t, d = kBB + i - br;  // row r0 + 32 + i
    return entry(rs, d <= b ? (i * ldw + d) * (int)sizeof(zc) : kNoEntry);
  };
  zc yv[kSolveCols];
  const int last = (n - 1) / kBB * kBB;
  pn = perm[min(last + fr, n - 1)];
  auto load_y = [&](int r0) {
    const int r = r0 + fr, pr = pn;
    pn = perm[max(0, r - kBB)];
#pragma unroll
    for (int cc = 0; cc < kSolveCols; ++cc) yv[cc] = zc{0.0, 0.0};
    if (fs == 0 && r0 >= 0 && r < n) {
      xo = (size_t)pr * ldx + (size_t)j * k + c0g;
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc)
        if (cc < ncol) yv[cc] = X[xo + cc];
    }
  };
  __syncthreads();
  for (int t = tid; t < ring_rows * kSolveCols; t += kSolveThreads) ring[t] = zc{0.0, 0.0};
#pragma unroll
  for (int t = 0; t < kFar; ++t) far[t] = zc{0.0, 0.0};
  near[0] = near[1] = zc{0.0, 0.0};
  load_inv(last);
  load_y(last);
  __syncthreads();
  for (int r0 = last; r0 >= 0; r0 -= kBB) {
    zc s[kSolveCols];
    zero(s);
    const int ib = r0 + kBB + bs;
#pragma unroll
    for (int t = 0; t < kFar; ++t) addr(s, far[t], ib + kSolveSlices * (t + 2));
    const __amdgpu_buffer_rsrc_t rc = bwd_rows(r0);
    for (int t = kFar + 2; kSolveSlices * t < b; t += 4) {
      zc w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = bwd_entry(rc, t + u);
#pragma unroll
      for (int u = 0; u < 4; ++u) addr(s, w[u], ib + kSolveSlices * (t + u));
    }
    const int rn = r0 - kBB;
    const __amdgpu_buffer_rsrc_t rx = bwd_rows(rn);
#pragma unroll
    for (int t = 0; t < kFar; ++t) far[t] = bwd_entry(rx, t + 2);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t) addr(s, near[t], ib + kSolveSlices * t);
#pragma unroll
    for (int t = 0; t < 2; ++t) near[t] = bwd_entry(rx, t);
    // the wave's two slices of a row are 32 lanes apart
#pragma unroll
    for (int cc = 0; cc < kSolveCols; ++cc) {
      s[cc].re += __shfl_xor(s[cc].re, 32, 64);
      s[cc].im += __shfl_xor(s[cc].im, 32, 64);
    }
    if ((tid & 32) == 0) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) part[tid >> 6][br][cc] = s[cc];
    }
    __syncthreads();
    if (fs == 0) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) {
        zc y = yv[cc];
#pragma unroll
        for (int w = 0; w < kSolveThreads / 64; ++w) y = csub(y, part[w][fr][cc]);
        yb[fr][cc] = y;
      }
    }
    const bool row = fs == 0 && r0 + fr < n;
    const size_t xw = xo;
    load_y(rn);
    __syncthreads();
    zc v[kSolveCols];
    zero(v);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) cfma(v[cc], iv[u], yb[fs + 16 * u][cc]);
    load_inv(rn);
    sum16(v);
    if (fs == 0) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc) ring[((r0 + fr) & mask) * kSolveCols + cc] = v[cc];
    }
    if (row) {
#pragma unroll
      for (int cc = 0; cc < kSolveCols; ++cc)
        if (cc < ncol) X[xw + cc] = v[cc];
    }
  }
}

// Partials of |b - (z_j I - A) x|^2 and |b|^2, in FP64 with A in caller order:
// a lane per system, so a row of X is read by consecutive lanes (a workgroup
// per system read it one column at a time: 993 us at n = 8000, 512 systems;
// now 112 us).
__global__ __launch_bounds__(256) void k_band_resid(int n, const int* __restrict__ rowptr,
                                                    const int* __restrict__ col,
                                                    const double* __restrict__ val,
                                                    const double* __restrict__ z,
                                                    const double* __restrict__ B, int ldb, int k,
                                                    int nsys, const zc* __restrict__ X,
                                                    int64_t ldx, double* __restrict__ part) {
  __shared__ double red[2][256];
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int sys = blockIdx.y * 64 + lane, sc = min(sys, nsys - 1), j = sc / k, c = sc % k;
  const double zr = z[2 * j], zi = z[2 * j + 1];
  double rr = 0.0, bb = 0.0;
  for (int i = blockIdx.x * 4 + wv; i < n; i += gridDim.x * 4) {
    const int s = rowptr[i], e = rowptr[i + 1];
    double ar = 0.0, ai = 0.0;
    for (int t = s; t < e; t += 4) {
      zc x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = X[(size_t)col[min(t + u, e - 1)] * ldx + sc];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double a = t + u < e ? val[t + u] : 0.0;
        ar += a * x[u].re;
        ai += a * x[u].im;
      }
    }
    const zc x = X[(size_t)i * ldx + sc];
    const double bi = B[(size_t)i * ldb + c];
    const double sr = bi - (zr * x.re - zi * x.im - ar);
    const double si = -(zr * x.im + zi * x.re - ai);
    rr += sr * sr + si * si;
    bb += bi * bi;
  }
  red[0][threadIdx.x] = rr;
  red[1][threadIdx.x] = bb;
  __syncthreads();
  if (wv == 0 && sys < nsys) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      part[((size_t)blockIdx.x * nsys + sys) * 2 + q] =
          (red[q][lane] + red[q][64 + lane]) + (red[q][128 + lane] + red[q][192 + lane]);
  }
}

// resid[j k + c] = ||B_c - (z_j I - A) X_{j,c}|| / ||B_c|| (0 for B_c = 0): a
// workgroup sums sixteen systems' partials, sixteen threads a system.
__global__ __launch_bounds__(256) void k_band_resid_fin(int nsys, int nb,
                                                        const double* __restrict__ part,
                                                        double* __restrict__ resid) {
  __shared__ double red[2][256];
  const int t = threadIdx.x, sys = blockIdx.x * 16 + t % 16;
  double s[2] = {0.0, 0.0};
  if (sys < nsys)
    for (int b = t / 16; b < nb; b += 16)
#pragma unroll
      for (int q = 0; q < 2; ++q) s[q] += part[((size_t)b * nsys + sys) * 2 + q];
  red[0][t] = s[0];
  red[1][t] = s[1];
  __syncthreads();
  if (t >= 16 || sys >= nsys) return;
  s[0] = s[1] = 0.0;
  for (int g = 0; g < 16; ++g) {
    s[0] += red[0][16 * g + t];
    s[1] += red[1][16 * g + t];
  }
  resid[sys] = s[1] > 0.0 ? sqrt(s[0] / s[1]) : 0.0;
}

// ---------------------------------------------------------------------------
// Bands below 31 kept at their own width (large n: at b = 31 a tridiagonal
// matrix takes 16 times the memory): the scalar L D L^T, W[r][0] = D(r) and
// W[r][d] = L(r, r - d), one wave a shift, and solves by substitution, a lane a
// right-hand side.  Both are serial in the rows, so the wider form is the faster
// one (n = 262,145, 64 shifts, 2 columns, factors and solves: 189, 196 and 234 ms
// at b = 1, 8 and 29, this 320, 436 and 998) and is left for memory only.
// ---------------------------------------------------------------------------
constexpr int kRing = 32;  // rows of a ring, more than b + 1

// One column a step: the window's rows c .. c + b in LDS, the update of its
// b (b + 1) / 2 entries over the lanes, rows read eight steps ahead.
__global__ __launch_bounds__(64) void k_narrow_factor(int n, int b, zc* __restrict__ Wall,
                                                      size_t stride, int* __restrict__ info) {
  __shared__ zc win[kRing][kRing + 1];  // row r in r % 32
  __shared__ zc ms[kRing], ls[kRing];   // column c: M(c + i, c) and L(c + i, c)
  constexpr int kAhead = 8, kPairs = 8;  // 30 * 31 / 2 entries of 64 lanes
  const int lane = threadIdx.x, ldw = b + 1;
  zc* __restrict__ W = Wall + (size_t)blockIdx.x * stride;
  // this lane's entries (c + pi, c + pk), 1 <= pk <= pi <= b (pi = 0: none)
  int pi[kPairs], pk[kPairs];
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    int e = lane + 64 * u, i = 1;
    while (i <= b && e >= i) e -= i++;
    pi[u] = i <= b ? i : 0;
    pk[u] = e + 1;
  }
  for (int e = lane; e < kRing * (kRing + 1); e += 64) (&win[0][0])[e] = zc{0.0, 0.0};
  __syncthreads();
  const int first = min(n, b + 1);
  for (int e = lane; e < first * ldw; e += 64) win[e / ldw][e % ldw] = W[e];
  zc next[kAhead], cur[kAhead];
  auto load = [&](int r0) {  // rows past the matrix are zeros
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      next[u] = zc{0.0, 0.0};
      if (lane <= b && r0 + u < n) next[u] = W[(size_t)(r0 + u) * ldw + lane];
    }
  };
  load(b + 1);
  __syncthreads();
  for (int c0 = 0; c0 < n; c0 += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) cur[u] = next[u];
    load(c0 + kAhead + b + 1);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int c = c0 + u;
      if (c >= n) break;
      const zc d = win[c % kRing][0];
      if (!(cfinite(d) && (d.re != 0.0 || d.im != 0.0))) {
        if (lane == 0) info[blockIdx.x] = 1 + c;
        return;  // the same pivot in every lane
      }
      const zd inv = zdiv(zd{1.0, 0.0}, zd{d.re, d.im});
      if (lane <= b) W[(size_t)c * ldw + lane] = win[c % kRing][lane];
      if (lane >= 1 && lane <= b) {
        zc& w = win[(c + lane) % kRing][lane];
        const zc m = w;
        zc l{0.0, 0.0};
        cfma(l, m, zc{inv.re, inv.im});
        ms[lane] = m;
        ls[lane] = l;
        w = l;
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPairs; ++q)
        if (pi[q]) {
          const zc l = ls[pi[q]];
          cfma(win[(c + pi[q]) % kRing][pi[q] - pk[q]], zc{-l.re, -l.im}, ms[pk[q]]);
        }
      if (lane <= b) win[(c + b + 1) % kRing][lane] = cur[u];
      __syncthreads();
    }
  }
}

// L y = b in dot products with the ring of the last rows' y, then, from the last
// row on, x = y / D - s with s the sums L^T x that the later rows have left in
// the ring.  Band rows go through LDS sixteen at a time, read a block ahead.
__global__ __launch_bounds__(64) void k_narrow_solve(int n, int b, int nz,
                                                     const zc* __restrict__ Wall, size_t stride,
                                                     const int* __restrict__ perm,
                                                     const double* __restrict__ B, int ldb, int k,
                                                     zc* __restrict__ X, int64_t ldx) {
  constexpr int kRows = 16, kPer = kRows * kRing / 64;
  __shared__ zc ring[kRing][64];
  __shared__ zc band[kRows][kRing];
  const int lane = threadIdx.x, ldw = b + 1;
  const int j = (int)blockIdx.x % nz, c = (int)blockIdx.x / nz * 64 + lane;
  const bool on = c < k;
  const int cc = min(c, k - 1);
  const zc* __restrict__ W = Wall + (size_t)j * stride;
  zc* __restrict__ Xc = X + (size_t)j * k + cc;
  zc st[kPer];
  int pr[kRows], pn[kRows];
  auto load_band = [&](int r0) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = lane + 64 * u, r = r0 + e / kRing, d = e % kRing;
      st[u] = zc{0.0, 0.0};
      if (d <= b && r >= 0 && r < n) st[u] = W[(size_t)r * ldw + d];
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i) pn[i] = perm[min(max(r0 + i, 0), n - 1)];
  };
  auto put_band = [&](bool inverse) {
    __syncthreads();  // the block before has been read
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = lane + 64 * u;
      zc v = st[u];
      if (inverse && e % kRing == 0) {
        const zd i = zdiv(zd{1.0, 0.0}, zd{v.re, v.im});  // rows past n: not used
        v = zc{i.re, i.im};
      }
      band[e / kRing][e % kRing] = v;
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i) pr[i] = pn[i];
    __syncthreads();
  };
  auto clear = [&] {
    for (int r = 0; r < kRing; ++r) ring[r][lane] = zc{0.0, 0.0};
  };
  clear();
  double bn[kRows], bv[kRows];
  auto load_rhs = [&] {
#pragma unroll
    for (int i = 0; i < kRows; ++i) bn[i] = B[(size_t)pn[i] * ldb + cc];
  };
  load_band(0);
  load_rhs();
  for (int r0 = 0; r0 < n; r0 += kRows) {
    put_band(false);
#pragma unroll
    for (int i = 0; i < kRows; ++i) bv[i] = bn[i];
    load_band(r0 + kRows);
    load_rhs();
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const int r = r0 + i;
      if (r >= n) break;
      zc s[2] = {zc{0.0, 0.0}, zc{0.0, 0.0}};
      for (int d = 1; d <= b; d += 2) {  // past b the band row is zero
        cfma(s[0], band[i][d], ring[(r - d) & (kRing - 1)][lane]);
        cfma(s[1], band[i][d + 1], ring[(r - d - 1) & (kRing - 1)][lane]);
      }
      const zc y{bv[i] - (s[0].re + s[1].re), -(s[0].im + s[1].im)};
      ring[r & (kRing - 1)][lane] = y;
      if (on) Xc[(size_t)pr[i] * ldx] = y;
    }
  }
  clear();
  zc yn[kRows], yv[kRows];
  auto load_y = [&] {
#pragma unroll
    for (int i = 0; i < kRows; ++i) yn[i] = on ? Xc[(size_t)pn[i] * ldx] : zc{0.0, 0.0};
  };
  const int last = (n - 1) / kRows * kRows;
  load_band(last);
  load_y();
  for (int r0 = last; r0 >= 0; r0 -= kRows) {
    put_band(true);
#pragma unroll
    for (int i = 0; i < kRows; ++i) yv[i] = yn[i];
    load_band(r0 - kRows);
    load_y();
#pragma unroll
    for (int i = kRows - 1; i >= 0; --i) {
      const int r = r0 + i;
      if (r >= n) continue;
      const zc s = ring[r & (kRing - 1)][lane];
      zc x{-s.re, -s.im};
      cfma(x, yv[i], band[i][0]);
      ring[r & (kRing - 1)][lane] = zc{0.0, 0.0};
      if (on) Xc[(size_t)pr[i] * ldx] = x;
      for (int d = 1; d <= b; ++d) cfma(ring[(r - d) & (kRing - 1)][lane], band[i][d], x);
    }
  }
}

}  // namespace

int band_solve_ring_rows(int b) {
  int rows = kBB;
  while (rows < b + kBB) rows *= 2;
  return rows;
}

int band_width(int64_t n, int nz, int b) {
  const int64_t padded = (int64_t)nz * n * kBB * (int64_t)sizeof(zc);
  return b < kBB - 1 && padded <= (int64_t(32) << 30) ? kBB - 1 : b;
}

bool band_supported(int b) {
  return (size_t)band_solve_ring_rows(b) * kSolveCols * sizeof(zc) <= kBandSolveRingBytes;
}

hipError_t band_assemble(hipStream_t st, int n, int b, const int* rowptr, const int* col,
                         const double* val, int nz, const double* z, cpx<double>* W) {
  if (n <= 0 || nz <= 0) return hipSuccess;
  dim3 grid((n + 255) / 256, nz);
  hipLaunchKernelGGL(k_band_assemble, grid, dim3(256), 0, st, n, b, rowptr, col, val, z, W,
                     (size_t)n * (b + 1));
  return hipGetLastError();
}

hipError_t band_factor(hipStream_t st, int n, int b, int nz, cpx<double>* W, int* info) {
  if (n <= 0 || nz <= 0) return hipSuccess;
  if (b < 0) return hipErrorInvalidValue;
  hipError_t e = hipMemsetAsync(info, 0, nz * sizeof(int), st);
  if (e != hipSuccess) return e;
  const size_t stride = (size_t)n * (b + 1);
  if (b < kBB - 1) {
    hipLaunchKernelGGL(k_narrow_factor, dim3(nz), dim3(64), 0, st, n, b, W, stride, info);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_band_first, dim3(nz), dim3(kStepThreads), 0, st, n, b, W, stride, info);
  // shift j of workgroup id % nz: with eight shifts a window stays in one XCD's L2
  for (int c = 0; c + kBB < n; c += kBB) {
    const int m = std::min(n, c + kBB + b) - (c + kBB), mb = (m + kBB - 1) / kBB;
    hipLaunchKernelGGL(k_band_step, dim3(nz * (mb * (mb + 1) / 2)), dim3(kStepThreads), 0, st, n,
                       b, c, nz, W, stride, info);
  }
  return hipGetLastError();
}

hipError_t band_solve(hipStream_t st, int n, int b, int nz, const cpx<double>* W, const int* perm,
                      const double* B, int ldb, int k, cpx<double>* X, int64_t ldx) {
  if (n <= 0 || nz <= 0 || k <= 0) return hipSuccess;
  if (b < kBB - 1) {
    hipLaunchKernelGGL(k_narrow_solve, dim3((k + 63) / 64 * nz), dim3(64), 0, st, n, b, nz, W,
                       (size_t)n * (b + 1), perm, B, ldb, k, X, ldx);
    return hipGetLastError();
  }
  const int ring = band_solve_ring_rows(b);
  const size_t lds = (size_t)ring * kSolveCols * sizeof(zc);
  if (lds > kBandSolveRingBytes) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute((const void*)k_band_solve,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_band_solve, dim3((k + kSolveCols - 1) / kSolveCols * nz),
                     dim3(kSolveThreads), lds, st, n, b, nz, W, (size_t)n * (b + 1), perm, B, ldb,
                     k, X, ldx, ring);
  return hipGetLastError();
}

namespace {
int resid_blocks(int n) { return std::min(256, (n + 3) / 4); }
}  // namespace

size_t band_resid_doubles(int n, int nsys) { return (size_t)resid_blocks(n) * nsys * 2; }

hipError_t band_resid(hipStream_t st, int n, const int* rowptr, const int* col, const double* val,
                      int nz, const double* z, const double* B, int ldb, int k,
                      const cpx<double>* X, int64_t ldx, double* part, double* resid) {
  if (n <= 0 || nz <= 0 || k <= 0) return hipSuccess;
  const int nsys = nz * k, nb = resid_blocks(n);
  hipLaunchKernelGGL(k_band_resid, dim3(nb, (nsys + 63) / 64), dim3(256), 0, st, n, rowptr, col,
                     val, z, B, ldb, k, nsys, X, ldx, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_band_resid_fin, dim3((nsys + 15) / 16), dim3(256), 0, st, nsys, nb, part,
                     resid);
  return hipGetLastError();
}

}  // namespace rafeast
