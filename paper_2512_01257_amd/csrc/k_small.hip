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
// and 115 us at k = 84; this 23 and 36 us.
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
// J_qp = -s) zeroing H_pq follows Golub & Van Loan, Alg. 8.5.1.
//
// Two kernels.  k_jacobi, one workgroup, iterates H alone: the upper triangle
// in LDS (an entry (i, j) is kept at (min, max); packed when the square does not
// fit), H <- J^T H J per 2 x 2 block of pairs t1 <= t2, a block per thread.  A
// round is a chain - rotation parameters by one wave, barrier, update, barrier -
// and the update is LDS traffic, so it touches each block once: with both
// triangles and V in the same rounds a k = 84 matrix took 2.6 us a round,
// now 0.69 us.  The rotations go to a list in memory, and k_jacobi_vec applies
// them to V: the rows of V are independent, so a wave per row runs them on as
// many CUs as there are rows.
// ============================================================================
constexpr int kMaxSweeps = 40;
constexpr int kJacobiPairs = kSmallMaxK / 2;

// A square of kk (k rounded up to even) rows, or its packed upper triangle.
template <bool kPacked>
__device__ __forceinline__ int sym_at(int i, int j, int kk) {
  const int lo = min(i, j), hi = max(i, j);
  return kPacked ? lo * (2 * kk - lo - 1) / 2 + hi : lo * (kk | 1) + hi;
}

// (c, s) = f (e, a) with f within an ulp or two of 1 / sqrt(e^2 + a^2).  f errs the
// same way for all the rotations of a small angle, which would scale V and H
// by as much each round: one step back to c^2 + s^2 = 1.  1 - c is exact, of the
// rounded c: contracted into the product before it, it would miss the rounding.
__device__ __forceinline__ void unit_pair(double e, double a, double f, double& c, double& s) {
#pragma clang fp contract(off)
  c = e * f;
  s = a * f;
  const double g = 0.5 * fma(-s, s, (1.0 - c) * (1.0 + c));
  c = fma(c, g, c);
  s = fma(s, g, s);
}

// NB: blocks per thread.  With k odd the last player is a dummy: its row and
// column are zero and its rotations the identity.
template <int NB, bool kPacked>
__global__ __launch_bounds__(kSmallThreads) void k_jacobi(int k, const double* __restrict__ Hin,
                                                          int ldh, double* __restrict__ theta,
                                                          double2* __restrict__ rot,
                                                          int* __restrict__ out) {
  extern __shared__ double H[];
  __shared__ double2 cs[kJacobiPairs];
  __shared__ double dg[kSmallMaxK];
  __shared__ double red[2][kSmallThreads / 64];
  const int tid = threadIdx.x;
  const int kk = k + (k & 1), np = kk / 2;
  const int players = kk - 1;  // the last player stays fixed
  for (int e = tid; e < kk * kk; e += kSmallThreads) {
    const int i = e / kk, j = e % kk;
    if (j < i) continue;
    double h = 0.0;
    if (j < k) h = 0.5 * (Hin[(size_t)i * ldh + j] + Hin[(size_t)j * ldh + i]);
    H[sym_at<kPacked>(i, j, kk)] = h;
  }
  // The last wave (two with more than 64 pairs) forms the rotations and holds
  // no blocks; the other threads hold NB blocks (t1 <= t2), as packed row by row.
  const int nbt = kSmallThreads - (np <= 64 ? 64 : 128), pt = tid - nbt;
  int t1[NB], t2[NB];
  bool on[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int b = tid + nbt * u;
    on[u] = pt < 0 && b < np * (np + 1) / 2;
    int r = 0, c = on[u] ? b : 0;
    while (c >= np - r) c -= np - r++;
    t1[u] = r;
    t2[u] = r + c;
  }
  // players of slot t in round r
  auto first = [&](int r, int t) {
    const int p = r + t;
    return p >= players ? p - players : p;
  };
  auto second = [&](int r, int t) {
    const int q = r - t;
    return t == 0 ? kk - 1 : q < 0 ? q + players : q;
  };
  __syncthreads();
  int rounds = 0;
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    // convergence test on the off-diagonal mass
    double off = 0.0, tot = 0.0;
    for (int i = tid >> 5; i < k; i += kSmallThreads / 32)
      for (int j = i + (tid & 31); j < k; j += 32) {
        const double h = H[sym_at<kPacked>(i, j, kk)];
        if (i != j) off += 2.0 * h * h;
        else tot += h * h;
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
    tot += off;
    __syncthreads();
    // converged once the off-diagonal mass is at the rounding floor: each
    // of the k (k - 1) off-diagonal entries is then a few units of roundoff
    // of the diagonal, so off / tot ~ k u^2; 64 k u^2 leaves a margin of 8 u
    // per entry (u = 2^-53)
    if (k == 1 || off <= 64.0 * k * 0x1.0p-106 * tot) break;
    for (int r = 0; r < players; ++r) {
      // the blocks' entries are read while the rotations are formed: H changes
      // only past the barrier
      int at[NB][4];
      double h[NB][4];
      if (pt >= 0) {
        __builtin_amdgcn_s_setprio(3);  // the other waves wait for this one
        const int pi = min(pt, np - 1);
        const int p = first(r, pi), q = second(r, pi);
        const double hpp = H[sym_at<kPacked>(p, p, kk)], hqq = H[sym_at<kPacked>(q, q, kk)];
        const double apq = H[sym_at<kPacked>(p, q, kk)];
        double c = 1.0, s = 0.0;
        // t = s / c is the smaller root of t^2 + 2 tau t = 1, tau = d / (2 a),
        // d = h_qq - h_pp, a = h_pq:  with e = |d| + sqrt(d^2 + 4 a^2),
        // t = 2 a sgn(d) / e, c = e / sqrt(e^2 + 4 a^2), s = t c.  This phase
        // is one wave's latency per round, so the two square roots are
        // Newton-refined hardware estimates (a few ulp; the rotation stays
        // orthogonal to working precision) and nothing is divided: a third
        // fewer steps in the chain than from tau.
        const double d = hqq - hpp, a2 = 2.0 * apq, w = fma(d, d, a2 * a2);
        if (apq != 0.0 && w > 0x1.0p-900 && w < 0x1.0p+900) {
          const double e = fabs(d) + w * rsq_nr(w);
          unit_pair(e, d >= 0.0 ? a2 : -a2, rsq_nr(fma(e, e, a2 * a2)), c, s);
        } else if (apq != 0.0) {
          const double tau = (hqq - hpp) / (2.0 * apq);
          const double tt = fabs(tau) > 1e150 ? 0.5 / tau
                            : (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
          c = 1.0 / sqrt(1.0 + tt * tt);
          s = tt * c;
        }
        __builtin_amdgcn_s_setprio(0);
        if (pt < np) {
          cs[pt] = make_double2(c, s);
          rot[(size_t)rounds * np + pt] = make_double2(c, s);
        }
      } else {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          const int p1 = first(r, t1[u]), q1 = second(r, t1[u]);
          const int p2 = first(r, t2[u]), q2 = second(r, t2[u]);
          at[u][0] = sym_at<kPacked>(p1, p2, kk);
          at[u][1] = sym_at<kPacked>(p1, q2, kk);
          at[u][2] = sym_at<kPacked>(q1, p2, kk);
          at[u][3] = sym_at<kPacked>(q1, q2, kk);
#pragma unroll
          for (int e = 0; e < 4; ++e) h[u][e] = H[at[u][e]];
        }
      }
      ++rounds;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        if (!on[u]) continue;
        const double2 j1 = cs[t1[u]], j2 = cs[t2[u]];
        // rows: J^T
        const double g00 = j1.x * h[u][0] - j1.y * h[u][2], g01 = j1.x * h[u][1] - j1.y * h[u][3];
        const double g10 = j1.y * h[u][0] + j1.x * h[u][2], g11 = j1.y * h[u][1] + j1.x * h[u][3];
        // columns: J
        H[at[u][0]] = j2.x * g00 - j2.y * g01;
        H[at[u][1]] = j2.y * g00 + j2.x * g01;
        if (t1[u] != t2[u]) H[at[u][2]] = j2.x * g10 - j2.y * g11;
        H[at[u][3]] = j2.y * g10 + j2.x * g11;
      }
      __syncthreads();
    }
  }
  for (int i = tid; i < k; i += kSmallThreads) dg[i] = H[sym_at<kPacked>(i, i, kk)];
  __syncthreads();
  for (int i = tid; i < k; i += kSmallThreads) {
    const double d = dg[i];
    int rank = 0;
    for (int j = 0; j < k; ++j) rank += (dg[j] < d) || (dg[j] == d && j < i);
    theta[rank] = d;
    out[1 + i] = rank;
  }
  if (tid == 0) out[0] = rounds;
}

// Row blockIdx.x of V = J_1 J_2 ... J_rounds, its columns in the order of the
// eigenvalues.  Lane l holds the row's entries of slots l + 64 w (first and
// second player); after a round the first players move one slot down and the
// second ones one slot up (slot 0's second player stays, its first becomes
// slot 1's second, and the last slot's second player becomes its first), which
// is the next round's pairing, and after a sweep every player is back.
template <int NP>
__device__ __forceinline__ void shift_slots(double (&a)[NP], double (&b)[NP], int np) {
  const int lane = threadIdx.x;
  double na[NP], nb[NP], x[NP];
#pragma unroll
  for (int w = 0; w < NP; ++w) x[w] = w == 0 && lane == 0 ? a[0] : b[w];
  auto down = [](double v) {  // lane l <- lane l + 1
    const long long t = __double_as_longlong(v);
    const int lo = (int)(t & 0xffffffffLL), hi = (int)(t >> 32);
    const int l2 = __builtin_amdgcn_update_dpp(0, lo, 0x130, 0xF, 0xF, false);
    const int h2 = __builtin_amdgcn_update_dpp(0, hi, 0x130, 0xF, 0xF, false);
    return __longlong_as_double(((long long)h2 << 32) | (unsigned)l2);
  };
  auto up = [](double v) {  // lane l <- lane l - 1
    const long long t = __double_as_longlong(v);
    const int lo = (int)(t & 0xffffffffLL), hi = (int)(t >> 32);
    const int l2 = __builtin_amdgcn_update_dpp(0, lo, 0x138, 0xF, 0xF, false);
    const int h2 = __builtin_amdgcn_update_dpp(0, hi, 0x138, 0xF, 0xF, false);
    return __longlong_as_double(((long long)h2 << 32) | (unsigned)l2);
  };
#pragma unroll
  for (int w = 0; w < NP; ++w) {
    na[w] = down(a[w]);
    nb[w] = up(x[w]);
    // the reads of another lane stand outside the lane's own condition: inside
    // it the compiler would put this lane's value of a select for every lane's
    if (w + 1 < NP) {
      const double v = readlane_f64(a[w + 1 < NP ? w + 1 : w], 0);
      na[w] = lane == 63 ? v : na[w];
    }
    if (w > 0) {
      const double v = readlane_f64(x[w > 0 ? w - 1 : 0], 63);
      nb[w] = lane == 0 ? v : nb[w];
    }
    if (lane + 64 * w == np - 1) na[w] = b[w];
  }
  if (lane == 0) nb[0] = b[0];
#pragma unroll
  for (int w = 0; w < NP; ++w) {
    a[w] = na[w];
    b[w] = nb[w];
  }
}

template <int NP>
__global__ __launch_bounds__(64) void k_jacobi_vec(int k, const double2* __restrict__ rot,
                                                   const int* __restrict__ out,
                                                   double* __restrict__ S, int lds) {
  const int row = blockIdx.x, lane = threadIdx.x;
  const int kk = k + (k & 1), np = kk / 2, players = kk - 1;
  const int rounds = out[0];
  double a[NP], b[NP];
  int pa[NP], pb[NP];
#pragma unroll
  for (int w = 0; w < NP; ++w) {
    const int t = lane + 64 * w;
    pa[w] = t;
    pb[w] = t == 0 ? kk - 1 : players - t;
    a[w] = t < np && pa[w] == row ? 1.0 : 0.0;
    b[w] = t < np && pb[w] == row ? 1.0 : 0.0;
  }
  // the list is read kAhead rounds ahead
  constexpr int kAhead = 8;
  double2 c[kAhead][NP];
  auto load = [&](double2 (&d)[NP], int r) {
#pragma unroll
    for (int w = 0; w < NP; ++w) {
      const int t = min(lane + 64 * w, np - 1);
      d[w] = rot[(size_t)min(r, max(rounds - 1, 0)) * np + t];
    }
  };
#pragma unroll
  for (int u = 0; u < kAhead; ++u) load(c[u], u);
  for (int r = 0; r < rounds; r += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (r + u < rounds) {
#pragma unroll
        for (int w = 0; w < NP; ++w) {
          const double va = a[w], vb = b[w];
          a[w] = c[u][w].x * va - c[u][w].y * vb;
          b[w] = c[u][w].y * va + c[u][w].x * vb;
        }
        if (np > 1) shift_slots<NP>(a, b, np);
      }
      load(c[u], r + u + kAhead);
    }
  }
#pragma unroll
  for (int w = 0; w < NP; ++w) {
    if (lane + 64 * w >= np) continue;
    if (pa[w] < k) S[(size_t)row * lds + out[1 + pa[w]]] = a[w];
    if (pb[w] < k && pb[w] != pa[w]) S[(size_t)row * lds + out[1 + pb[w]]] = b[w];
  }
}

// One or two columns: at most one rotation, in one launch (k = 2, the call: 24.8 us
// with the two kernels above, 17.5 with this one).
__global__ __launch_bounds__(64) void k_jacobi_two(int k, const double* __restrict__ H, int ldh,
                                                   double* __restrict__ theta,
                                                   double* __restrict__ S, int lds) {
  if (threadIdx.x != 0) return;
  const double a = H[0];
  if (k == 1) {
    theta[0] = a;
    S[0] = 1.0;
    return;
  }
  const double b = 0.5 * (H[1] + H[ldh]), d = H[ldh + 1];
  // a' = a - t b, d' = d + t b with the smaller root of t^2 + 2 tau t = 1
  double t = 0.0;
  if (b != 0.0) {
    const double tau = (d - a) / (2.0 * b);
    t = fabs(tau) > 1e150 ? 0.5 / tau
                          : (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
  }
  const double c = 1.0 / sqrt(1.0 + t * t), s = t * c;
  const double lo = a - t * b, hi = d + t * b;
  const int p = hi < lo ? 1 : 0;  // column of (c, -s)
  theta[p] = lo;
  theta[1 - p] = hi;
  S[p] = c;
  S[lds + p] = -s;
  S[1 - p] = s;
  S[lds + 1 - p] = c;
}

size_t jacobi_work_doubles(int k) {
  const size_t kk = k + (k & 1);
  return (size_t)kMaxSweeps * (kk - 1) * kk + kk;  // the rotations; rounds and ranks
}

hipError_t launch_jacobi(hipStream_t st, int k, const double* H, int ldh, double* theta,
                         double* S, int lds, double* work) {
  if (k < 1 || k > kSmallMaxK) return hipErrorInvalidValue;
  if (k <= 2) {
    hipLaunchKernelGGL(k_jacobi_two, dim3(1), dim3(64), 0, st, k, H, ldh, theta, S, lds);
    return hipGetLastError();
  }
  const int kk = k + (k & 1), np = kk / 2, blocks = np * (np + 1) / 2;
  double2* rot = reinterpret_cast<double2*>(work);
  int* out = reinterpret_cast<int*>(rot + (size_t)kMaxSweeps * (kk - 1) * np);
  // the square while two blocks a thread suffice (k <= 122: 118 KB of LDS),
  // else the packed triangle
  const size_t square = sizeof(double) * (size_t)kk * (kk | 1);
  const int holders = kSmallThreads - 64;
  const bool packed = blocks > 2 * holders;
  const size_t bytes = packed ? sizeof(double) * (size_t)kk * (kk + 1) / 2 : square;
  const void* fn = packed ? (const void*)k_jacobi<6, true>
                   : blocks > holders ? (const void*)k_jacobi<2, false>
                                            : (const void*)k_jacobi<1, false>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  if (packed)
    hipLaunchKernelGGL((k_jacobi<6, true>), dim3(1), dim3(kSmallThreads), bytes, st, k, H, ldh,
                       theta, rot, out);
  else if (blocks > holders)
    hipLaunchKernelGGL((k_jacobi<2, false>), dim3(1), dim3(kSmallThreads), bytes, st, k, H, ldh,
                       theta, rot, out);
  else
    hipLaunchKernelGGL((k_jacobi<1, false>), dim3(1), dim3(kSmallThreads), bytes, st, k, H, ldh,
                       theta, rot, out);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (np <= 64)
    hipLaunchKernelGGL(k_jacobi_vec<1>, dim3(k), dim3(64), 0, st, k, rot, out, S, lds);
  else
    hipLaunchKernelGGL(k_jacobi_vec<2>, dim3(k), dim3(64), 0, st, k, rot, out, S, lds);
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
