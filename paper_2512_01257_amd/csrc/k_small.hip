// Small dense kernels of the RA-FEAST path, one workgroup each (k <= 192):
//  - CholQR factor: column scaling, Cholesky G = R^T R (shifted when it
//    fails), R^{-1};  Y <- Y diag(1/sqrt(g_ii)) R^{-1} orthonormalises Y
//    (the QR step of Algorithms 1 and 2);
//  - parallel cyclic Jacobi for the reduced eigenproblem of Rayleigh-Ritz;
//  - Phase-1 truncation: keep the m0 Ritz vectors with largest |op| value.
#include "device.h"
#include "kernels.h"

namespace rafeast {

constexpr int kSmallThreads = 1024;
constexpr int kSmallMaxK = 192;

// ============================================================================
// CholQR factor: M = diag(s) R^{-1}, s_i = 1 / sqrt(g_ii), R^T R = S G S
// (scaled, symmetric part), in 16 x 16 tiles on the FP64 matrix cores, one
// workgroup, the upper tiles in LDS.  Step J:
//   T_J = R_JJ^{-1} by one wave (elimination of [A_JJ | I], below);
//   U_JK = T_J^T A_JK for K > J, and the inverse's column J,
//   X_IJ = -(sum_{I <= t < J} X_It U_tJ) T_J for I < J (X_JJ = T_J);
//   A_KL -= U_JK^T U_JL for J < K <= L, the next diagonal tile first, whose
//   elimination then runs beside the other tiles' updates.
// Every operand is a tile read along its rows: U as U(q, i), X kept transposed,
// so that lane l reads element (l / 16, l % 16) of four rows in 512 consecutive
// bytes; and a product's accumulator v (row l / 16 + 4 v) is fragment v of the
// next product's right operand, so Y = sum U^T X^T feeds T^T Y in registers.
// X_IJ overwrites U_IJ (last read for column J of the inverse), a barrier
// after every wave has read the column.
// A column at a time (a barrier and a pass over the trailing block for each of
// k columns, then for each of k columns of the inverse) took 94 us at k = 64
// and 115 us at k = 84; this CHOL64_US and CHOL84_US us.
// ============================================================================
constexpr int kTile = 256;  // doubles of a 16 x 16 tile

__device__ __forceinline__ int tile_at(int nb, int I, int J) {  // I <= J
  return (I * nb - I * (I - 1) / 2 + (J - I)) * kTile;
}

__device__ __forceinline__ void mm4(const double (&a)[4], const double (&b)[4], v4d& c) {
#pragma unroll
  for (int v = 0; v < 4; ++v) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[v], b[v], c, 0, 0, 0);
}
// element (l / 16 + 4 v, l % 16), v = 0..3, of a tile
__device__ __forceinline__ void frag4(const double* t, double (&f)[4]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) f[v] = t[64 * v + (threadIdx.x & 63)];
}
__device__ __forceinline__ void put4(double* t, const v4d& d) {
#pragma unroll
  for (int v = 0; v < 4; ++v) t[64 * v + (threadIdx.x & 63)] = d[v];
}

// One wave: elimination of [A | I] for the symmetric tile A (fragments a), row
// j of both going round through LDS (row, 32 doubles; a wave's LDS operations
// are in order, so no barrier), leaves L^{-1} where I was and the pivots d;
// T = L^{-T} D^{-1/2}.  Writes T^T (the inverse's own tile) over tile and T to
// ts.  Returns false at a pivot that is not positive and finite.
__device__ __forceinline__ bool tile_inverse(double (&a)[4], double* row, double* tile,
                                             double* ts) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  double e[4], sc[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    e[v] = li == lk + 4 * v ? 1.0 : 0.0;
    sc[v] = 0.0;
  }
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if (lk == (j & 3)) {
      row[li] = a[j >> 2];
      row[16 + li] = e[j >> 2];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const double d = row[j], aj = row[li], ej = row[16 + li];
    double m[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) m[v] = row[lk + 4 * v];
    ok = ok && d > 0.0 && isfinite(d);
    const double inv = rcp_nr(d);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = lk + 4 * v;
      if (i == j) sc[v] = rsq_nr(d);
      const double f = i > j ? m[v] * inv : 0.0;
      a[v] -= f * aj;
      e[v] -= f * ej;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double t = e[v] * sc[v];
    tile[64 * v + lane] = t;
    ts[16 * li + lk + 4 * v] = t;
  }
  return ok;
}

__global__ __launch_bounds__(kSmallThreads) void k_chol_inv(int k, double shift_unit,
                                                            const double* __restrict__ G, int ldg,
                                                            double* __restrict__ M, int ldm,
                                                            int* __restrict__ flag) {
  extern __shared__ double sm[];
  const int nb = (k + 15) >> 4, nt = nb * (nb + 1) / 2;
  double* A = sm;                      // upper tiles
  double* ts = A + (size_t)nt * kTile; // T_J
  double* row = ts + kTile;            // tile_inverse's rows
  double* dsc = row + 32;              // column scales
  int* bad = reinterpret_cast<int*>(dsc + k);  // [0] a scale, [1] a pivot
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NW = kSmallThreads / 64;
  if (tid < 2) bad[tid] = 0;
  __syncthreads();
  for (int i = tid; i < k; i += kSmallThreads) {
    const double d = G[(size_t)i * ldg + i];
    if (d > 0.0 && isfinite(d)) {
      dsc[i] = 1.0 / sqrt(d);
    } else {
      dsc[i] = 0.0;
      bad[0] = 1;
    }
  }
  __syncthreads();
  int status = bad[0] ? 2 : 0;
  for (int attempt = 0; attempt < 2 && status != 2; ++attempt) {
    // tile entries (I, J), J >= I, in tile order; past k the identity
    for (int e = tid; e < nt * kTile; e += kSmallThreads) {
      int t = e / kTile, I = 0;
      while (t >= nb - I) t -= nb - I++;
      const int i = 16 * I + (e % kTile) / 16, j = 16 * (I + t) + e % 16;
      double g = i == j ? 1.0 : 0.0;
      if (i < k && j < k && i != j)
        g = 0.5 * (G[(size_t)i * ldg + j] + G[(size_t)j * ldg + i]) * dsc[i] * dsc[j];
      if (i == j && i < k) g = 1.0 + (attempt == 0 ? 0.0 : shift_unit);
      A[e] = g;
    }
    __syncthreads();
    if (wave == 0) {
      double a[4];
      frag4(A, a);
      if (!tile_inverse(a, row, A, ts) && tid == 0) bad[1] = 1;
    }
    __syncthreads();
    for (int J = 0; J < nb; ++J) {
      if (bad[1]) break;  // uniform
      // U_JK (waves 0 .. nb - 2 - J), then the inverse's X_IJ (the next J
      // waves): at most nb - 1 <= 11 of them, one each
      const int nu = nb - 1 - J;
      const int K = J + 1 + wave, I = wave - nu;
      v4d x{0.0, 0.0, 0.0, 0.0};
      if (wave < nb - 1) {
        double t[4], b[4];
        frag4(ts, t);
        if (wave < nu) {
          double* u = A + tile_at(nb, J, K);
          frag4(u, b);
          mm4(t, b, x);
          put4(u, x);
        } else {
          v4d y{0.0, 0.0, 0.0, 0.0};
          for (int q = I; q < J; ++q) {
            double u[4];
            frag4(A + tile_at(nb, q, J), u);
            frag4(A + tile_at(nb, I, q), b);
            mm4(u, b, y);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) b[v] = -y[v];
          mm4(t, b, x);
        }
      }
      __syncthreads();
      if (wave >= nu && wave < nb - 1) put4(A + tile_at(nb, I, J), x);
      // trailing tiles: wave 0 the next diagonal one and its inverse, the
      // other waves the rest in turn
      if (nu > 0) {
        int t = wave;
        const int left = nu * (nu + 1) / 2;
        while (t < left) {
          int r = 0, c = t;
          while (c >= nu - r) c -= nu - r++;
          const int Kt = J + 1 + r, Lt = Kt + c;
          double ua[4], ub[4], a[4];
          double* dst = A + tile_at(nb, Kt, Lt);
          frag4(A + tile_at(nb, J, Kt), ua);
          frag4(A + tile_at(nb, J, Lt), ub);
          frag4(dst, a);
          v4d d{a[0], a[1], a[2], a[3]};
#pragma unroll
          for (int v = 0; v < 4; ++v) ua[v] = -ua[v];
          mm4(ua, ub, d);
          if (t == 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) a[v] = d[v];
            if (!tile_inverse(a, row, dst, ts) && tid == 0) bad[1] = 1;
            break;
          }
          put4(dst, d);
          t += NW - 1;
        }
      }
      __syncthreads();
    }
    if (!bad[1]) {
      status = attempt;
      break;
    }
    status = attempt == 0 ? 1 : 2;
    __syncthreads();
    if (tid == 0) bad[1] = 0;
    __syncthreads();
  }
  if (status == 2) {
    for (int e = tid; e < k * k; e += kSmallThreads) {
      const int i = e / k, j = e % k;
      M[(size_t)i * ldm + j] = (i == j) ? dsc[i] : 0.0;
    }
    if (tid == 0) *flag = 2;
    return;
  }
  for (int e = tid; e < k * k; e += kSmallThreads) {
    const int r = e / k, c = e % k;
    double x = 0.0;
    if (c >= r) x = A[tile_at(nb, r >> 4, c >> 4) + (c & 15) * 16 + (r & 15)] * dsc[r];
    M[(size_t)r * ldm + c] = x;
  }
  if (tid == 0) *flag = status;
}

// Dynamic LDS budget of the one-workgroup kernels (the static arrays of
// k_jacobi take under 8 KB of the 160 KB).
constexpr size_t kSmallLdsMax = 160 * 1024 - 8192;

hipError_t launch_chol_inv(hipStream_t st, int k, int64_t nrows, const double* G, int ldg,
                           double* M, int ldm, int* flag) {
  if (k < 1 || k > kSmallMaxK) return hipErrorInvalidValue;
  // Shifted CholQR (Fukaya, Kannan, Nakatsukasa, Yamamoto, Yanagisawa 2020):
  // s = 11 (m n + n (n+1)) u ||X||_2^2 with ||X||_2^2 <= trace(G) = k after scaling.
  const double u = 0x1.0p-53;
  const double shift = 11.0 * ((double)nrows * k + (double)k * (k + 1)) * u * (double)k;
  const int nb = (k + 15) / 16;
  const size_t lds = sizeof(double) * ((size_t)kTile * (nb * (nb + 1) / 2 + 1) + 32 + k) + 16;
  hipError_t e = hipFuncSetAttribute((const void*)k_chol_inv,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_chol_inv, dim3(1), dim3(kSmallThreads), lds, st, k, shift, G, ldg, M, ldm,
                     flag);
  return hipGetLastError();
}

// ============================================================================
// Parallel cyclic Jacobi (round-robin pairing).  Each round rotates k/2
// disjoint pairs (p, q) at once: the rotation J (J_pp = J_qq = c, J_pq = s,
// J_qp = -s) zeroing H_pq follows Golub & Van Loan, Alg. 8.5.1.  H <- J^T H J
// is applied per (row pair, column pair) 2x2 block, each block by one thread,
// and V <- V J per (row, pair).  H lives in LDS for k <= 128, else in global
// workspace; V lives in LDS too when both fit, else in global workspace.
// ============================================================================
template <bool kHInLds, bool kVInLds>
__global__ __launch_bounds__(kSmallThreads) void k_jacobi(int k, const double* __restrict__ Hin,
                                                          int ldh, double* __restrict__ theta,
                                                          double* __restrict__ S, int lds,
                                                          double* __restrict__ work) {
  extern __shared__ double sh_h[];
  __shared__ int rp[kSmallMaxK / 2 + 1], rq[kSmallMaxK / 2 + 1], perm[kSmallMaxK];
  __shared__ double rc[kSmallMaxK / 2 + 1], rs[kSmallMaxK / 2 + 1], dg[kSmallMaxK];
  __shared__ double red[2][kSmallThreads / 64];
  // In LDS, H and V rows are k | 1 doubles apart (an odd stride): the rows a
  // wave touches in one access then start in different banks.
  const int hs = kHInLds ? (k | 1) : k, vs = kVInLds ? (k | 1) : k;
  double* H = kHInLds ? sh_h : work;
  double* V = kVInLds ? sh_h + (size_t)k * hs : work + (size_t)k * k;
  const int tid = threadIdx.x;
  for (int e = tid; e < k * k; e += kSmallThreads) {
    const int i = e / k, j = e % k;
    H[i * hs + j] = 0.5 * (Hin[(size_t)i * ldh + j] + Hin[(size_t)j * ldh + i]);
    V[i * vs + j] = (i == j) ? 1.0 : 0.0;
  }
  __syncthreads();
  const int kk = k + (k & 1);
  const int np = kk / 2;
  const int players = kk - 1;  // the last player stays fixed
  const float inv_np = 1.0f / (float)np;
  for (int sweep = 0; sweep < 40; ++sweep) {
    // convergence test on the off-diagonal mass
    double off = 0.0, tot = 0.0;
    for (int i = tid >> 5; i < k; i += kSmallThreads / 32)
      for (int j = tid & 31; j < k; j += 32) {
        const double h = H[i * hs + j];
        tot += h * h;
        if (i != j) off += h * h;
      }
    off = wave_sum(off);
    tot = wave_sum(tot);
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = off;
      red[1][tid >> 6] = tot;
    }
    __syncthreads();
    off = 0.0;
    tot = 0.0;
    for (int w = 0; w < kSmallThreads / 64; ++w) {
      off += red[0][w];
      tot += red[1][w];
    }
    __syncthreads();
    // converged once the off-diagonal mass is at the rounding floor: each
    // of the k (k - 1) off-diagonal entries is then a few units of roundoff
    // of the diagonal, so off / tot ~ k u^2; 64 k u^2 leaves a margin of 8 u
    // per entry (u = 2^-53)
    if (k == 1 || off <= 64.0 * k * 0x1.0p-106 * tot) break;
    for (int r = 0; r < players; ++r) {
      for (int t = tid; t < np; t += kSmallThreads) {
        int p, q;
        if (t == 0) {
          p = r;
          q = kk - 1;
        } else {
          p = (r + t) % players;
          q = (r - t + players) % players;
        }
        double c = 1.0, s = 0.0;
        if (p < k && q < k) {
          const double apq = H[p * hs + q];
          if (fabs(apq) >= 0x1.0p-1000) {
            // this phase is one wave's latency per round: reciprocals and
            // square roots from Newton-refined hardware estimates (a few ulp;
            // the rotation stays orthogonal to working precision)
            const double tau = (H[q * hs + q] - H[p * hs + p]) * rcp_nr(2.0 * apq);
            double tt;
            if (fabs(tau) > 1e150) {
              tt = 0.5 / tau;
            } else {
              const double w = fma(tau, tau, 1.0);
              tt = (tau >= 0.0 ? 1.0 : -1.0) * rcp_nr(fabs(tau) + w * rsq_nr(w));
            }
            c = rsq_nr(fma(tt, tt, 1.0));
            s = tt * c;
          } else if (apq != 0.0) {
            const double tau = (H[q * hs + q] - H[p * hs + p]) / (2.0 * apq);
            const double tt = fabs(tau) > 1e150 ? 0.5 / tau
                              : (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + tt * tt);
            s = tt * c;
          }
        }
        rp[t] = p;
        rq[t] = q;
        rc[t] = c;
        rs[t] = s;
      }
      __syncthreads();
      for (int b = tid; b < np * np; b += kSmallThreads) {
        // b / np in float: exact for b, e < 2^15 and np <= 96
        const int t1 = (int)(((float)b + 0.5f) * inv_np), t2 = b - t1 * np;
        const int p1 = rp[t1], q1 = rq[t1], p2 = rp[t2], q2 = rq[t2];
        const double c1 = rc[t1], s1 = rs[t1], c2 = rc[t2], s2 = rs[t2];
        const bool v_p1 = p1 < k, v_q1 = q1 < k, v_p2 = p2 < k, v_q2 = q2 < k;
        const double h00 = (v_p1 && v_p2) ? H[p1 * hs + p2] : 0.0;
        const double h01 = (v_p1 && v_q2) ? H[p1 * hs + q2] : 0.0;
        const double h10 = (v_q1 && v_p2) ? H[q1 * hs + p2] : 0.0;
        const double h11 = (v_q1 && v_q2) ? H[q1 * hs + q2] : 0.0;
        // rows: J^T
        const double g00 = c1 * h00 - s1 * h10, g01 = c1 * h01 - s1 * h11;
        const double g10 = s1 * h00 + c1 * h10, g11 = s1 * h01 + c1 * h11;
        // columns: J
        const double f00 = c2 * g00 - s2 * g01, f01 = s2 * g00 + c2 * g01;
        const double f10 = c2 * g10 - s2 * g11, f11 = s2 * g10 + c2 * g11;
        if (v_p1 && v_p2) H[p1 * hs + p2] = f00;
        if (v_p1 && v_q2) H[p1 * hs + q2] = f01;
        if (v_q1 && v_p2) H[q1 * hs + p2] = f10;
        if (v_q1 && v_q2) H[q1 * hs + q2] = f11;
      }
      for (int e = tid; e < k * np; e += kSmallThreads) {
        const int row = (int)(((float)e + 0.5f) * inv_np), t = e - row * np;
        const int p = rp[t], q = rq[t];
        if (p < k && q < k) {
          const double c = rc[t], s = rs[t];
          const double vp = V[row * vs + p], vq = V[row * vs + q];
          V[row * vs + p] = c * vp - s * vq;
          V[row * vs + q] = s * vp + c * vq;
        }
      }
      __syncthreads();
    }
  }
  for (int i = tid; i < k; i += kSmallThreads) dg[i] = H[i * hs + i];
  __syncthreads();
  for (int i = tid; i < k; i += kSmallThreads) {
    const double d = dg[i];
    int rank = 0;
    for (int j = 0; j < k; ++j) rank += (dg[j] < d) || (dg[j] == d && j < i);
    theta[rank] = d;
    perm[rank] = i;
  }
  __syncthreads();
  for (int e = tid; e < k * k; e += kSmallThreads) {
    const int row = e / k, c = e % k;
    S[(size_t)row * lds + c] = V[row * vs + perm[c]];
  }
}

hipError_t launch_jacobi(hipStream_t st, int k, const double* H, int ldh, double* theta,
                         double* S, int lds, double* work) {
  if (k < 1 || k > kSmallMaxK) return hipErrorInvalidValue;
  // H (and V) in LDS with rows k | 1 doubles apart
  const size_t hb = sizeof(double) * (size_t)k * (size_t)(k | 1);
  if (2 * hb <= kSmallLdsMax) {
    hipError_t e = hipFuncSetAttribute((const void*)k_jacobi<true, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)(2 * hb));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_jacobi<true, true>), dim3(1), dim3(kSmallThreads), 2 * hb, st, k, H,
                       ldh, theta, S, lds, work);
  } else if (k <= 128) {
    hipError_t e = hipFuncSetAttribute((const void*)k_jacobi<true, false>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)hb);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_jacobi<true, false>), dim3(1), dim3(kSmallThreads), hb, st, k, H, ldh,
                       theta, S, lds, work);
  } else {
    hipLaunchKernelGGL((k_jacobi<false, false>), dim3(1), dim3(kSmallThreads), 0, st, k, H, ldh,
                       theta, S, lds, work);
  }
  return hipGetLastError();
}

// ============================================================================
// Phase-1 truncation: f_i = |a + b theta_i + c theta_i^2| is the op-value of
// Ritz value theta_i; keep the m0 largest (ties to the lower index), in
// ascending-theta order.
// ============================================================================
__global__ __launch_bounds__(256) void k_select(int k, int m0, const double* __restrict__ theta,
                                                const double* __restrict__ S, int lds, double a,
                                                double b, double c, double* __restrict__ Ssel,
                                                double* __restrict__ info) {
  __shared__ double f[kSmallMaxK];
  __shared__ int rank[kSmallMaxK], pos[kSmallMaxK];
  const int tid = threadIdx.x;
  for (int i = tid; i < k; i += 256) {
    const double t = theta[i];
    f[i] = fabs(a + b * t + c * t * t);
  }
  __syncthreads();
  for (int i = tid; i < k; i += 256) {
    int r = 0;
    for (int j = 0; j < k; ++j) r += (f[j] > f[i]) || (f[j] == f[i] && j < i);
    rank[i] = r;
  }
  __syncthreads();
  for (int i = tid; i < k; i += 256) {
    int ps = 0;
    for (int j = 0; j < i; ++j) ps += rank[j] < m0;
    pos[i] = rank[i] < m0 ? ps : -1;
    if (rank[i] == m0 - 1) info[0] = f[i];
    if (rank[i] == m0) info[1] = f[i];
  }
  if (tid == 0 && k <= m0) info[1] = __builtin_nan("");
  __syncthreads();
  for (int e = tid; e < k * k; e += 256) {
    const int row = e / k, i = e % k;
    if (pos[i] >= 0) Ssel[(size_t)row * m0 + pos[i]] = S[(size_t)row * lds + i];
  }
}

hipError_t launch_select(hipStream_t st, int k, int m0, const double* theta, const double* S,
                         int lds, double a, double b, double c, double* Ssel, double* info) {
  if (k < 1 || k > kSmallMaxK || m0 > k) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_select, dim3(1), dim3(256), 0, st, k, m0, theta, S, lds, a, b, c, Ssel,
                     info);
  return hipGetLastError();
}

}  // namespace rafeast
