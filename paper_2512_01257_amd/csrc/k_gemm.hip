// Products with the dense operators of the statistical workloads (Section 4):
// kernel PCA, A = K (symmetric n x n); sample covariance, A = scale Xd^T Xd
// with the centred data Xd (rows x n).  Every product is one GEMM form,
//   C (M x N, row-major) = alpha op(A) B + beta C,
// run on the matrix cores: v_mfma_f64_16x16x4f64 in FP64 and
// v_mfma_f32_16x16x4f32 in FP32.
//
// Tiling: a 256-thread workgroup owns a 128 x 32 TN tile of C; its four
// waves own 64 x 16 TN quarters, 4 x TN MFMA tiles of 16 x 16 each, so every
// operand fragment read from LDS feeds several MFMAs (TN = 4 in FP32, 2 in
// FP64).  The inner dimension advances in
// steps of BK, 32 in FP32 and 16 in FP64: the step's A (128 x BK) and B (BK x
// 32 TN) panels are staged in LDS (two buffers; the next step's global loads are
// issued before the current step's MFMAs and stored before or after the last of
// them, one barrier per step).  A may
// be stored by rows or by columns (op(A)(i, k) at A[i lda + k] or
// A[k lda + i]); B and C by rows.  Products with a long inner dimension and
// few output tiles are split into chunks of the inner dimension (grid.z), each
// chunk's product written to a slab of a workspace, and the slabs summed in
// chunk order by a second kernel: no atomics, the same sums every run.
#include "device.h"
#include "kernels.h"

namespace rafeast {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kBM = 128, kGT = 256;
#ifndef RAFEAST_GEMM_BK32
#define RAFEAST_GEMM_BK32 32
#endif
#ifndef RAFEAST_GEMM_BK64
#define RAFEAST_GEMM_BK64 16
#endif
#ifndef RAFEAST_GEMM_TN64
#define RAFEAST_GEMM_TN64 2
#endif
#ifndef RAFEAST_GEMM_TN32
#define RAFEAST_GEMM_TN32 4
#endif
#ifndef RAFEAST_GEMM_XCD
#define RAFEAST_GEMM_XCD 1
#endif
#ifndef RAFEAST_GEMM_VEC_BYTES
#define RAFEAST_GEMM_VEC_BYTES 16
#endif
constexpr int kGemmVecBytes = RAFEAST_GEMM_VEC_BYTES;  // bytes per vector load

// MFMA operand layout (lane l of the wave):
//   A (16 x 4): A[l % 16][l / 16]     B (4 x 16): B[l / 16][l % 16]
//   D (16 x 16): register v of lane l holds D[row(l, v)][l % 16]
template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef v4d Acc;
  static __device__ __forceinline__ Acc step(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int l, int v) { return (l >> 4) + 4 * v; }
};
template <>
struct Mfma<float> {
  typedef v4f Acc;
  static __device__ __forceinline__ Acc step(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int l, int v) { return 4 * (l >> 4) + v; }
};

// ACOL: op(A)(i, k) = A[k lda + i] (else A[i lda + k]).  BK: inner indices
// per LDS step.  VEC: elements per global load along each operand's
// contiguous dimension (VEC > 1 asks for no alignment of the operands; the host
// takes it unless C is smaller than a tile and cuts vectors).  part != nullptr:
// chunk z covers inner indices [z kc, min(K, (z + 1) kc)) and its
// raw product goes to part + z M N (row-major, ld N); otherwise C is written.
// Two waves a SIMD are asked for (LDS allows two or three): told so, the compiler
// keeps the accumulators in the VGPRs that the MFMAs write; else it splits them
// over AGPRs, with copies in every step, and the element form of A by rows took
// more than half of a SIMD's registers, one wave (us before and with it: FP64
// 8192 x 480 x 8192 A by rows 1301 and 1157, by columns 1207 and 1140, 5003 x 334
// x 4002 374 and 313; FP32 65536 x 117 x 1024 187 and 167).  The widest vector
// form of A by rows in FP32 is faster as the compiler lays it out (8192 x 1024 x
// 8192 1070 and 1103).
template <typename T, bool ACOL, int BK, int VEC, int TN>
constexpr int kGemmWaves = sizeof(T) == 4 && !ACOL && VEC > 1 && TN == 4 ? 1 : 2;

template <typename T, bool ACOL, int BK, int VEC, int TN>
__global__ __launch_bounds__(kGT, (kGemmWaves<T, ACOL, BK, VEC, TN>)) void k_gemm(
    int M, int N, int K, int kc, const T* __restrict__ A, int64_t lda, const T* __restrict__ B,
    int64_t ldb, T* __restrict__ C, int64_t ldc, T alpha, T beta, T* __restrict__ part) {
  // Rows are padded so that the four rows a fragment read touches start 16
  // elements apart modulo the banks (every bank pair once), and by a whole
  // number of 16-byte words, so that a panel stored along its rows is stored
  // in vectors; a transposed A is padded by four more, which spreads its stores
  // (eight rows of a vector's column over four banks) at two passes a read.
  // A pad of one element cost four passes a read (FP32, 8192 x 480 x 8192, A by
  // columns: 654 -> 640 us; FP64 the same).  FP32 blocks of 64 columns with A by
  // rows are padded less, so that three workgroups share a CU's LDS (65536 x 64 x
  // 1024 84 -> 79 us, 8192 x 64 x 8192 90 -> 85; by columns the same).
  constexpr int BN = 32 * TN;                   // block tile width
  constexpr bool kLess = sizeof(T) == 4 && !ACOL && TN == 2;
  constexpr int PA = kBM + (kLess ? 10 : ACOL ? 16 : sizeof(T) == 4 ? 20 : 18);
  constexpr int PB = BN + (kLess ? 8 : 16);
  __shared__ __align__(16) T As[2][BK][PA];
  __shared__ __align__(16) T Bs[2][BK][PB];
  typedef typename Mfma<T>::Acc Acc;
  constexpr int NVA = kBM * BK / (kGT * VEC);  // vectors per thread: A panel
  constexpr int NVB = BN * BK / (kGT * VEC);   // and B panel
  constexpr int CA = ACOL ? kBM : BK;          // A panel: contiguous length
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  // Workgroups go to the eight XCDs in turn (linear id b to XCD b mod 8).
  // With a grid of a multiple of eight workgroups, XCD x takes the x-th
  // contiguous eighth of the tiles in (chunk, row tile, column tile) order,
  // so the workgroups that share an A row panel or a chunk share one L2.
  const int gx = gridDim.x, gy = gridDim.y;
  const int G = gx * gy * (int)gridDim.z;
  const int b = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int l = (RAFEAST_GEMM_XCD && G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
  const int tn = l % gx, tm = (l / gx) % gy, tz = l / (gx * gy);
  // the tile's first row and column, and the first ones it stores
  const int is = tm * kBM, js = tn * BN;
  const int i0 = M >= kBM ? min(is, M - kBM) : is, j0 = N >= BN ? min(js, N - BN) : js;
  const int kbeg = tz * kc;
  const int kend = min(K, kbeg + kc);
  const int nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;

  T ra[NVA][VEC], rb[NVB][VEC];
  Acc acc[4][TN];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < TN; ++nt) acc[mt][nt] = Acc{T(0), T(0), T(0), T(0)};

  typedef T LV __attribute__((ext_vector_type(VEC)));
  auto store_row = [&](T* dst, const T (&src)[VEC]) {
    LV v;
#pragma unroll
    for (int u = 0; u < VEC; ++u) v[u] = src[u];
    *reinterpret_cast<LV*>(dst) = v;
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NVA; ++q) {
      const int e = (tid + q * kGT) * VEC;
      const int ca = e % CA, oa = e / CA;
      if (ACOL) {
        store_row(&As[buf][oa][ca], ra[q]);
      } else {
#pragma unroll
        for (int u = 0; u < VEC; ++u) As[buf][ca + u][oa] = ra[q][u];
      }
    }
#pragma unroll
    for (int q = 0; q < NVB; ++q) {
      const int e = (tid + q * kGT) * VEC;
      store_row(&Bs[buf][e / BN][e % BN], rb[q]);
    }
  };
  const int fr = lane >> 4, fc = lane & 15;
  // The fragments of sub-step ks + 4 are read from LDS while the MFMAs of
  // sub-step ks issue (two register sets), so LDS latency overlaps the
  // matrix work.
  // The next step's panels are stored before the last sub-step's MFMAs, which
  // cover them (8192 x 480 x 8192, us after and before: FP64 A by columns 1143
  // and 1105, by rows 1159 and 1109; FP32 by rows 602 and 600), but after them in
  // FP32 with A by columns (580 and 594).
  constexpr bool kStoreInStep = sizeof(T) == 8 || !ACOL;
  auto mfma_step = [&](int cur, bool next) {
    T a[2][4], b[2][TN];
    auto frag = [&](int set, int ks) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) a[set][mt] = As[cur][ks + fr][wm * 64 + mt * 16 + fc];
#pragma unroll
      for (int nt = 0; nt < TN; ++nt) b[set][nt] = Bs[cur][ks + fr][wn * 16 * TN + nt * 16 + fc];
    };
    frag(0, 0);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      const int set = (ks / 4) & 1;
      if (ks + 4 < BK) frag(set ^ 1, ks + 4);
      else if (kStoreInStep && next) store(cur ^ 1);
      // keep the look-ahead reads ahead of this sub-step's MFMAs
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < TN; ++nt)
          acc[mt][nt] = Mfma<T>::step(a[set][mt], b[set][nt], acc[mt][nt]);
    }
  };

  // Element loads from addresses clamped into the matrix, the elements outside
  // it zeroed: tiles that are cut inside a vector, and a last step of the inner
  // dimension that is not whole.
  auto load_any = [&](int k0) {
#pragma unroll
    for (int q = 0; q < NVA; ++q) {
      const int e = (tid + q * kGT) * VEC;
      const int ca = e % CA, oa = e / CA;
#pragma unroll
      for (int u = 0; u < VEC; ++u) {
        const int gi = i0 + (ACOL ? ca + u : oa), gk = k0 + (ACOL ? oa : ca + u);
        const int ci = min(gi, M - 1), ck = min(gk, kend - 1);
        const T va = A[ACOL ? (int64_t)ck * lda + ci : (int64_t)ci * lda + ck];
        ra[q][u] = (gi < M && gk < kend) ? va : T(0);
      }
    }
#pragma unroll
    for (int q = 0; q < NVB; ++q) {
      const int e = (tid + q * kGT) * VEC;
#pragma unroll
      for (int u = 0; u < VEC; ++u) {
        const int gj = j0 + e % BN + u, gb = k0 + e / BN;
        const int cj = min(gj, N - 1), cb = min(gb, kend - 1);
        const T vb = B[(int64_t)cb * ldb + cj];
        rb[q][u] = (gj < N && gb < kend) ? vb : T(0);
      }
    }
  };

  // The fast path takes the whole steps of the inner dimension.  A tile cut by
  // the edge of C is moved back to end there (its first rows or columns are the
  // tile's before it, and only that one stores them), so its loads stay inside
  // the matrix.  Where C is smaller than a tile, rows and columns past it feed
  // only outputs that are never stored: a vector that starts there is read from
  // the tile's first row or column instead, but none may straddle the edge (M, N
  // a multiple of VEC).  Vectors need not start on a 16-byte boundary.
  const bool a_fast = !ACOL || M >= kBM || M % VEC == 0;
  const bool b_fast = N >= BN || N % VEC == 0;
  const int nf = a_fast && b_fast ? (kend - kbeg) / BK : 0;  // whole steps
  if (nf > 0) {
    // Per-thread operand pointers advanced by one step each time,
    // whole-vector loads, no bounds tests in the loop.
    typedef T VT __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
    const T* pa[NVA];
    const T* pb[NVB];
#pragma unroll
    for (int q = 0; q < NVA; ++q) {
      const int e = (tid + q * kGT) * VEC;
      const int ca = e % CA, oa = e / CA;
      int gi = i0 + (ACOL ? ca : oa);
      if (gi >= M) gi = i0;
      pa[q] = ACOL ? A + (int64_t)(kbeg + oa) * lda + gi : A + (int64_t)gi * lda + (kbeg + ca);
    }
#pragma unroll
    for (int q = 0; q < NVB; ++q) {
      const int e = (tid + q * kGT) * VEC;
      int gj = j0 + e % BN;
      if (gj >= N) gj = j0;
      pb[q] = B + (int64_t)(kbeg + e / BN) * ldb + gj;
    }
    const int64_t da = ACOL ? (int64_t)BK * lda : BK, db = (int64_t)BK * ldb;
    auto load = [&]() {
#pragma unroll
      for (int q = 0; q < NVA; ++q) {
        const VT va = *reinterpret_cast<const VT*>(pa[q]);
#pragma unroll
        for (int u = 0; u < VEC; ++u) ra[q][u] = va[u];
        pa[q] += da;
      }
#pragma unroll
      for (int q = 0; q < NVB; ++q) {
        const VT vb = *reinterpret_cast<const VT*>(pb[q]);
#pragma unroll
        for (int u = 0; u < VEC; ++u) rb[q][u] = vb[u];
        pb[q] += db;
      }
    };
    load();
    store(0);
    __syncthreads();
    for (int t = 0; t < nf; ++t) {
      const int cur = t & 1;
      if (t + 1 < nf) load();
      mfma_step(cur, t + 1 < nf);
      if (!kStoreInStep && t + 1 < nf) store(cur ^ 1);
      __syncthreads();
    }
  }
  if (nf < nk) {
    load_any(kbeg + nf * BK);
    store(0);
    __syncthreads();
    for (int t = nf; t < nk; ++t) {
      const int cur = (t - nf) & 1;
      if (t + 1 < nk) load_any(kbeg + (t + 1) * BK);
      mfma_step(cur, t + 1 < nk);
      if (!kStoreInStep && t + 1 < nk) store(cur ^ 1);
      __syncthreads();
    }
  }

  T* __restrict__ slab = part ? part + (size_t)tz * (size_t)M * N : nullptr;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < TN; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int gi = i0 + wm * 64 + mt * 16 + Mfma<T>::row(lane, v);
        const int gj = j0 + wn * 16 * TN + nt * 16 + fc;
        if (gi < is || gi >= M || gj < js || gj >= N) continue;
        if (slab) {
          slab[(size_t)gi * N + gj] = acc[mt][nt][v];
        } else {
          T c = alpha * acc[mt][nt][v];
          if (beta != T(0)) c += beta * C[(int64_t)gi * ldc + gj];
          C[(int64_t)gi * ldc + gj] = c;
        }
      }
}

// C = alpha sum_z slab_z + beta C, slabs in chunk order.
template <typename T>
__global__ __launch_bounds__(256) void k_gemm_reduce(int M, int N, int S,
                                                     const T* __restrict__ part,
                                                     T* __restrict__ C, int64_t ldc, T alpha,
                                                     T beta) {
  const int64_t MN = (int64_t)M * N;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= MN) return;
  T s = T(0);
  for (int z = 0; z < S; ++z) s += part[(size_t)z * MN + e];
  const int64_t i = e / N, j = e % N;
  T c = alpha * s;
  if (beta != T(0)) c += beta * C[i * ldc + j];
  C[i * ldc + j] = c;
}

__global__ __launch_bounds__(256) void k_axpy(int64_t count, double a, const double* __restrict__ x,
                                              double* __restrict__ y) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < count) y[e] += a * x[e];
}

template <typename T, int BK, int TN>
hipError_t launch_tiles(hipStream_t st, bool acol, bool vec, dim3 grid, int M, int N, int K,
                        int kc, const T* A, int64_t lda, const T* B, int64_t ldb, T* C,
                        int64_t ldc, T alpha, T beta, T* part) {
  constexpr int V = kGemmVecBytes / (int)sizeof(T) > 0 ? kGemmVecBytes / (int)sizeof(T) : 1;
  if (acol && vec)
    hipLaunchKernelGGL((k_gemm<T, true, BK, V, TN>), grid, dim3(kGT), 0, st, M, N, K, kc, A, lda,
                       B, ldb, C, ldc, alpha, beta, part);
  else if (acol)
    hipLaunchKernelGGL((k_gemm<T, true, BK, 1, TN>), grid, dim3(kGT), 0, st, M, N, K, kc, A, lda,
                       B, ldb, C, ldc, alpha, beta, part);
  else if (vec)
    hipLaunchKernelGGL((k_gemm<T, false, BK, V, TN>), grid, dim3(kGT), 0, st, M, N, K, kc, A,
                       lda, B, ldb, C, ldc, alpha, beta, part);
  else
    hipLaunchKernelGGL((k_gemm<T, false, BK, 1, TN>), grid, dim3(kGT), 0, st, M, N, K, kc, A,
                       lda, B, ldb, C, ldc, alpha, beta, part);
  return hipGetLastError();
}

// MFMA column tiles per wave: up to four in FP32 (128-wide blocks), up to
// two in FP64 (64-wide blocks: half the accumulators, so two waves fit a
// SIMD); narrow products (the few live columns at the end of a solve) take
// one or two, so a block does not compute many columns it throws away
int gemm_tn(bool f64, int N) {
  const int most = f64 ? RAFEAST_GEMM_TN64 : RAFEAST_GEMM_TN32;
  return N <= 32 ? 1 : (N <= 64 || most == 2) ? 2 : 4;
}

// Chunks of the inner dimension, given room for most of them: two workgroups
// per CU.  Chunks are at least 512 long, and at least 128 below 2,560: a short
// product on few tiles otherwise leaves most CUs idle (us with 512 and 128:
// FP64 602 x 350 x 1391 246 and 68, FP32 2000 x 480 x 2000 165 and 93), while
// for long ones more chunks only add partial sums (3000 x 300 x 3000 167 and
// 168, FP64 600 x 300 x 8000 110 and 121, FP32 4096 x 60 x 4096 48 and 50).
int gemm_chunks(bool f64, int M, int N, int K, size_t most) {
  const int BN = 32 * gemm_tn(f64, N);
  const int tiles = ((M + kBM - 1) / kBM) * ((N + BN - 1) / BN);
  const int want = (512 + tiles - 1) / tiles;
  const int fit = K / (K < 2560 ? 128 : 512);
  return std::max(1, std::min(want, std::min(fit, (int)std::min<size_t>(most, 64))));
}

// C = alpha op(A) B + beta C.  work (nullable, work_elems elements) holds the
// chunk slabs: the inner dimension is split when the output has fewer tiles
// than two per CU and the chunks stay long enough.
template <typename T>
hipError_t gemm(hipStream_t st, bool acol, int M, int N, int K, const T* A, int64_t lda,
                const T* B, int64_t ldb, T* C, int64_t ldc, T alpha, T beta, T* work,
                size_t work_elems) {
  if (M <= 0 || N <= 0) return hipSuccess;
  constexpr bool f64 = sizeof(T) == 8;
  constexpr int TNmax = f64 ? RAFEAST_GEMM_TN64 : RAFEAST_GEMM_TN32;
  const int TN = gemm_tn(f64, N);
  const int BN = 32 * TN;
  // inner indices per LDS step (FP64: 16, so that the staging buffers leave
  // room for two workgroups per CU)
  constexpr int BK = sizeof(T) == 8 ? RAFEAST_GEMM_BK64 : RAFEAST_GEMM_BK32;
  int S = work ? gemm_chunks(f64, M, N, K, work_elems / ((size_t)M * N)) : 1;
  int kc = (K + S - 1) / S;
  kc = (kc + BK - 1) / BK * BK;
  if (K <= 0) kc = BK;
  S = K > 0 ? (K + kc - 1) / kc : 1;
  T* part = S > 1 ? work : nullptr;
  dim3 grid((N + BN - 1) / BN, (M + kBM - 1) / kBM, S);
  // Vector loads, also of rows that start between 16-byte boundaries (us with
  // element and vector loads: FP32 8191 x 480 x 8191 678 and 600; FP64 5003 x
  // 334 x 4002 358 and 312), unless C is smaller than a tile and cuts vectors:
  // no step of the vector form is whole then (us with vector and element form,
  // aligned operands: FP32 4096 x 30 x 4096 60 and 24, 4096 x 126 x 4096 110 and
  // 54; FP64 3000 x 17 x 1500 35 and 23).
  constexpr int V = kGemmVecBytes / (int)sizeof(T) > 0 ? kGemmVecBytes / (int)sizeof(T) : 1;
  const bool vec = V > 1 && (N >= BN || N % V == 0) && (!acol || M >= kBM || M % V == 0);
  hipError_t e;
  if (TN == 1)
    e = launch_tiles<T, BK, 1>(st, acol, vec, grid, M, N, K, kc, A, lda, B, ldb, C, ldc, alpha,
                               beta, part);
  else if (TN == 2)
    e = launch_tiles<T, BK, 2>(st, acol, vec, grid, M, N, K, kc, A, lda, B, ldb, C, ldc, alpha,
                               beta, part);
  else
    e = launch_tiles<T, BK, TNmax>(st, acol, vec, grid, M, N, K, kc, A, lda, B, ldb, C, ldc,
                                   alpha, beta, part);
  if (e != hipSuccess || S == 1) return e;
  const int64_t MN = (int64_t)M * N;
  hipLaunchKernelGGL(k_gemm_reduce<T>, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, st, M,
                     N, S, part, C, ldc, alpha, beta);
  return hipGetLastError();
}

bool fits_int(int64_t v) { return v >= 0 && v < ((int64_t)1 << 31); }

// Y = alpha A X + beta Y for one dense operator, in T.
template <typename T>
hipError_t dense_apply(const DenseOp& A, hipStream_t st, int k, const T* X, int ldx, T* Y,
                       int ldy, T alpha, T beta, const T* a, T* t) {
  if (k == 0) return hipSuccess;
  if (k < 0 || !a || !fits_int(A.n) || !fits_int(A.rows) || ldx < k || ldy < k)
    return hipErrorInvalidValue;
  const int n = (int)A.n, rows = (int)A.rows;
  if (A.kind == 1) {
    // K is symmetric: K(i, kk) = K[kk lda + i], the column-major reading; the
    // workspace serves products up to tcols wide
    const size_t room = t && k <= A.tcols ? (size_t)A.wslabs * n * A.tcols : 0;
    return gemm<T>(st, true, n, k, n, a, A.lda, X, ldx, Y, ldy, alpha, beta, t, room);
  }
  if (A.kind != 2 || !t || k > A.tcols) return hipErrorInvalidValue;
  // T (rows x k, ld kt) = Xd X: Xd(r, j) = a[j lda + r]; the chunk slabs
  // follow T in the workspace.  kt rounds k up to a multiple of 4, so that
  // the second product reads T in whole vectors.
  const int kt = (k + 3) / 4 * 4 <= A.tcols ? (k + 3) / 4 * 4 : k;
  const size_t room = (size_t)(A.wslabs - 1) * rows * A.tcols;
  hipError_t e = gemm<T>(st, true, rows, k, n, a, A.lda, X, ldx, t, kt, T(1), T(0),
                         t + (size_t)rows * A.tcols, room);
  if (e != hipSuccess) return e;
  // Y = alpha scale Xd^T T + beta Y: Xd^T(i, r) = a[i lda + r]
  return gemm<T>(st, false, n, k, rows, a, A.lda, t, kt, Y, ldy, alpha * T(A.scale), beta,
                 nullptr, 0);
}

}  // namespace

hipError_t dense_apply_f64(const DenseOp& A, hipStream_t st, int k, const double* X, int ldx,
                           double* Y, int ldy, double alpha, double beta) {
  return dense_apply<double>(A, st, k, X, ldx, Y, ldy, alpha, beta, A.a64, A.t64);
}

hipError_t dense_apply_f32(const DenseOp& A, hipStream_t st, int k, const float* X, int ldx,
                           float* Y, int ldy) {
  return dense_apply<float>(A, st, k, X, ldx, Y, ldy, 1.0f, 0.0f, A.a32, A.t32);
}

hipError_t dense_axpy(hipStream_t st, int64_t count, double a, const double* x, double* y) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_axpy, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, count, a,
                     x, y);
  return hipGetLastError();
}

size_t gemm_work_elems(bool f64, int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return 0;
  const int S = gemm_chunks(f64, M, N, K, 64);
  return S > 1 ? (size_t)S * M * N : 0;
}

hipError_t launch_gemm_f64(hipStream_t st, bool acol, int M, int N, int K, const double* A,
                           int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc,
                           double alpha, double beta, double* work, size_t work_elems) {
  return gemm<double>(st, acol, M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, work, work_elems);
}

hipError_t launch_gemm_f32(hipStream_t st, bool acol, int M, int N, int K, const float* A,
                           int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc,
                           float alpha, float beta, float* work, size_t work_elems) {
  return gemm<float>(st, acol, M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, work, work_elems);
}

}  // namespace rafeast
