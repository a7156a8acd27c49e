// Dense FP64 pieces of the extraction (paper Sec. 3.1, Algorithm 1):
//  * block inner products C = A^H B of tall vector blocks (moments mu_k = V^H S_k,
//    Gram matrices of the Rayleigh-Ritz basis) on FP64 MFMA, split over the long axis;
//  * tall-skinny products out = A W (Ritz vectors, basis changes);
//  * single-workgroup complex dense kernels for the small matrices (n <= 512):
//    one-sided Jacobi SVD, Hessenberg reduction + shifted QR (Schur form) with
//    eigenvectors, LU with partial pivoting, Cholesky.
// Small matrices are column-major: element (i, j) at a[i + j*lda].
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "cbs_internal.hpp"
#include "dense.hpp"
#include "ranking.hpp"

namespace cbs {

using c64 = double2;

__device__ __forceinline__ c64 zmul(c64 a, c64 b) { return cmul<double>(a, b); }
__device__ __forceinline__ c64 zmulc(c64 a, c64 b) { return cmulc<double>(a, b); }   // conj(a) b
__device__ __forceinline__ c64 zadd(c64 a, c64 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ c64 zsub(c64 a, c64 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ c64 zconj(c64 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ c64 zscale(c64 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ __forceinline__ double zabs(c64 a) { return hypot(a.x, a.y); }
__device__ __forceinline__ c64 zdiv(c64 a, c64 b) { return cdiv<double>(a, b); }
__device__ __forceinline__ c64 zsqrt(c64 a) {
  const double r = zabs(a);
  if (r == 0.0) return make_double2(0, 0);
  double re = sqrt(0.5 * (r + fabs(a.x)));
  double im = a.y / (2.0 * re);
  if (a.x < 0) {
    const double t = fabs(im);
    im = (a.y >= 0) ? re : -re;
    re = t;
  }
  return make_double2(re, im);
}

// ------------------------------------------------------------------ block inner products
typedef double f64x4 __attribute__((ext_vector_type(4)));

// One 16x16 complex tile of C = A^H B per workgroup (4 waves), over a slice of the long
// axis.  MFMA f64 16x16x4: lane l feeds A[l%16][k=l/16] and B[k=l/16][l%16] and holds
// D[4*v + l/16][l%16], v = 0..3.  The k slot of a lane walks 4 consecutive points of its
// vector over 4 instructions, so each lane streams 64 contiguous bytes per step.
// C_re = Ar^T Br + Ai^T Bi, C_im = Ar^T Bi - Ai^T Br.
__global__ void __launch_bounds__(256) k_gram_mfma(int64_t N, int32_t na, int32_t nb, const c64* A,
                                                   int64_t lda, const c64* B, int64_t ldb, int32_t tiles_b,
                                                   int32_t nsplit, int64_t span, double* part) {
  __shared__ double red[4][2][64][4];
  const int tile = blockIdx.x / nsplit, sp = blockIdx.x - tile * nsplit;
  const int ta = tile / tiles_b, tb = tile - ta * tiles_b;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row = ta * 16 + (lane & 15);
  const int col = tb * 16 + (lane & 15);
  const int kk = lane >> 4;
  const bool ra = row < na, cb = col < nb;
  const c64* pa = A + (int64_t)(ra ? row : 0) * lda;
  const c64* pb = B + (int64_t)(cb ? col : 0) * ldb;
  const int64_t lo = sp * span, hi = std::min<int64_t>(lo + span, N);
  f64x4 cre = {0, 0, 0, 0}, cim = {0, 0, 0, 0};
  // each wave takes every 4th block of 16 points
  for (int64_t n0 = lo + wv * 16; n0 < hi; n0 += 64) {
    c64 av[4], bv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t n = n0 + 4 * kk + s;
      const bool ok = n < hi;
      av[s] = (ok && ra) ? pa[n] : make_double2(0, 0);
      bv[s] = (ok && cb) ? pb[n] : make_double2(0, 0);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      cre = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].x, bv[s].x, cre, 0, 0, 0);
      cre = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].y, bv[s].y, cre, 0, 0, 0);
      cim = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].x, bv[s].y, cim, 0, 0, 0);
      cim = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[s].y, bv[s].x, cim, 0, 0, 0);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    red[wv][0][lane][v] = cre[v];
    red[wv][1][lane][v] = cim[v];
  }
  __syncthreads();
  if (tid < 64) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double re = red[0][0][tid][v] + red[1][0][tid][v] + red[2][0][tid][v] + red[3][0][tid][v];
      const double im = red[0][1][tid][v] + red[1][1][tid][v] + red[2][1][tid][v] + red[3][1][tid][v];
      const int i = ta * 16 + mfma16_row<double>(tid, v);
      const int j = tb * 16 + (tid & 15);
      if (i < na && j < nb) {
        double* o = part + (((int64_t)sp * na + i) * nb + j) * 2;
        o[0] = re;
        o[1] = im;
      }
    }
  }
}

// Plain reference version of the same tile (no MFMA), selected with CBS_NO_MFMA=1.
__global__ void __launch_bounds__(256) k_gram_plain(int64_t N, int32_t na, int32_t nb, const c64* A,
                                                    int64_t lda, const c64* B, int64_t ldb, int32_t tiles_b,
                                                    int32_t nsplit, int64_t span, double* part) {
  const int tile = blockIdx.x / nsplit, sp = blockIdx.x - tile * nsplit;
  const int ta = tile / tiles_b, tb = tile - ta * tiles_b;
  const int i = ta * 16 + (threadIdx.x >> 4), j = tb * 16 + (threadIdx.x & 15);
  const int64_t lo = sp * span, hi = std::min<int64_t>(lo + span, N);
  if (i >= na || j >= nb) return;
  c64 acc = make_double2(0, 0);
  for (int64_t n = lo; n < hi; ++n) acc = zadd(acc, zmulc(A[(int64_t)i * lda + n], B[(int64_t)j * ldb + n]));
  double* o = part + (((int64_t)sp * na + i) * nb + j) * 2;
  o[0] = acc.x;
  o[1] = acc.y;
}

// The slices' sums in slice order; eight slices are requested at a time (36 slices, 16 x 16: 3.7 us,
// 9.4 one after the other).
__global__ void __launch_bounds__(64) k_gram_reduce(int32_t na, int32_t nb, int32_t nsplit, const double* part,
                                                    c64* C, int64_t ldc) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= na * nb) return;
  const int i = t / nb, j = t - i * nb;
  const c64* p = reinterpret_cast<const c64*>(part) + t;
  const int64_t stride = (int64_t)na * nb;
  double re = 0, im = 0;
  int s = 0;
  for (; s + 8 <= nsplit; s += 8) {
    c64 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[(s + k) * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      re += v[k].x;
      im += v[k].y;
    }
  }
  for (; s < nsplit; ++s) {
    const c64 v = p[s * stride];
    re += v.x;
    im += v.y;
  }
  C[i + (int64_t)j * ldc] = make_double2(re, im);
}

static bool no_mfma() {
  const char* e = getenv("CBS_NO_MFMA");
  return e && e[0] == '1';
}

int32_t gram(cbs_system* s, int64_t N, int32_t na, const c64* A, int64_t lda, int32_t nb, const c64* B,
             int64_t ldb, c64* C, int64_t ldc, hipStream_t st) {
  if (na <= 0 || nb <= 0) return CBS_OK;
  const int tiles_a = (na + 15) / 16, tiles_b = (nb + 15) / 16;
  const int tiles = tiles_a * tiles_b;
  int nsplit = (int)std::max<int64_t>(1, std::min<int64_t>((2048 + tiles - 1) / tiles, (N + 255) / 256));
  const int64_t span = ((N + nsplit - 1) / nsplit + 63) / 64 * 64;
  nsplit = (int)((N + span - 1) / span);
  double* part = nullptr;
  CBS_TRY(ws_get(s->ws, "gram.part", (size_t)nsplit * na * nb * 2, &part));
  if (no_mfma())
    hipLaunchKernelGGL(k_gram_plain, dim3(tiles * nsplit), dim3(256), 0, st, N, na, nb, A, lda, B, ldb, tiles_b,
                       nsplit, span, part);
  else
    hipLaunchKernelGGL(k_gram_mfma, dim3(tiles * nsplit), dim3(256), 0, st, N, na, nb, A, lda, B, ldb, tiles_b,
                       nsplit, span, part);
  CBS_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_gram_reduce, dim3((na * nb + 63) / 64), dim3(64), 0, st, na, nb, nsplit,
                     (const double*)part, C, ldc);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

// ------------------------------------------------------------------ tall-skinny product
// out[c][n] = sum_k A[k][n] W[k + c*ldw] for c < nc; W staged in LDS per tile of TC columns.
// KU rows of A are requested at a time.  A product of many outputs takes 16 columns a thread, so that
// A is read seldom; one of few, whose workgroups would not fill the chip and whose time is the chain
// of loads over k, 4 columns a thread in workgroups of one wave.  K = 32, us with 16 and with 4:
// N nc = 147 000 (9216 x 16) 22.1 and 7.6, 768 000 (24000 x 32) 24.9 and 20.4, 1 180 000 (73728 x 16)
// 27.4 and 15.4, 2 360 000 (73728 x 32) 31.3 and 26.6, but 103.7 and 139.4 at K = 128, and
// 4 700 000 (294912 x 16) 52 and 101.
template <int TC, int KU>
__global__ void __launch_bounds__(TC == 16 ? 256 : 64) k_tall_gemm(int64_t N, int32_t K, int32_t nc, const c64* A,
                                                                   int64_t lda, const c64* W, int32_t ldw, c64* out,
                                                                   int64_t ldo) {
  extern __shared__ c64 w_s[];   // [K][TC]
  const int c0 = blockIdx.y * TC;
  const int ncl = std::min(TC, nc - c0);
  for (int t = threadIdx.x; t < K * TC; t += blockDim.x) {
    const int k = t / TC, c = t - k * TC;
    w_s[t] = (c < ncl) ? W[k + (int64_t)(c0 + c) * ldw] : make_double2(0, 0);
  }
  __syncthreads();
  for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < N; n += (int64_t)gridDim.x * blockDim.x) {
    c64 acc[TC];
#pragma unroll
    for (int c = 0; c < TC; ++c) acc[c] = make_double2(0, 0);
    int k = 0;
    for (; k + KU <= K; k += KU) {
      c64 a[KU];
#pragma unroll
      for (int u = 0; u < KU; ++u) a[u] = A[(int64_t)(k + u) * lda + n];
#pragma unroll
      for (int u = 0; u < KU; ++u)
#pragma unroll
        for (int c = 0; c < TC; ++c) acc[c] = zadd(acc[c], zmul(a[u], w_s[(k + u) * TC + c]));
    }
    for (; k < K; ++k) {
      const c64 a = A[(int64_t)k * lda + n];
#pragma unroll
      for (int c = 0; c < TC; ++c) acc[c] = zadd(acc[c], zmul(a, w_s[k * TC + c]));
    }
#pragma unroll
    for (int c = 0; c < TC; ++c)
      if (c < ncl) out[(int64_t)(c0 + c) * ldo + n] = acc[c];
  }
}

int32_t tall_gemm(int64_t N, int32_t K, int32_t nc, const c64* A, int64_t lda, const c64* W, int32_t ldw, c64* out,
                  int64_t ldo, hipStream_t st) {
  if (nc <= 0 || N <= 0) return CBS_OK;
  if ((size_t)K * 16 * sizeof(c64) > 64 * 1024) {
    set_error("tall_gemm: inner dimension %d too large", K);
    return CBS_EINVAL;
  }
  if (N * nc <= 1250000) {
    const int gx = (int)((N + 63) / 64);
    hipLaunchKernelGGL((k_tall_gemm<4, 8>), dim3(gx, (nc + 3) / 4), dim3(64), (size_t)K * 4 * sizeof(c64), st, N, K,
                       nc, A, lda, W, ldw, out, ldo);
  } else {
    const int gx = (int)std::min<int64_t>((N + 255) / 256, 2048);
    hipLaunchKernelGGL((k_tall_gemm<16, 2>), dim3(gx, (nc + 15) / 16), dim3(256), (size_t)K * 16 * sizeof(c64), st,
                       N, K, nc, A, lda, W, ldw, out, ldo);
  }
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

// ------------------------------------------------------------------ single-workgroup helpers
constexpr int SWG = 256;   // threads of the single-workgroup kernels

template <int WG>
__device__ double block_max_wg(double v, double* sh) {
  v = fmax(v, __shfl_xor(v, 1, 64));
  for (int o = 2; o < 64; o <<= 1) v = fmax(v, __shfl_xor(v, o, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
  for (int w = 1; w < WG / 64; ++w) r = fmax(r, sh[w]);
  __syncthreads();
  return r;
}

__device__ double block_max(double v, double* sh) { return block_max_wg<SWG>(v, sh); }

__device__ double block_sum(double v, double* sh) {
  for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0;
  for (int w = 0; w < SWG / 64; ++w) r += sh[w];
  __syncthreads();
  return r;
}

// ------------------------------------------------------------------ one-sided Jacobi SVD
// A (n x n, lda) is overwritten by U*Sigma, V starts as the identity and becomes W with
// A_in W = U Sigma.  Columns are paired round-robin (slot 0 fixed, the others rotating by
// one per round, so the slot of every column follows from the round number); each round's
// n/2 disjoint pairs are handled by groups of JWG/(n/2) threads.  Output: sigma sorted
// descending (perm gives the source column of each sorted position), U columns normalised
// in place.
constexpr int JWG = 1024;
__global__ void __launch_bounds__(JWG) k_jacobi_svd(int32_t n, c64* A, int32_t lda, c64* V, int32_t ldv,
                                                     double* sigma, int32_t* perm, int32_t max_sweeps) {
  __shared__ double sh[JWG / 64];
  __shared__ double sflag;
  const int tid = threadIdx.x;
  for (int t = tid; t < n * n; t += JWG) {
    const int i = t % n, j = t / n;
    V[i + (int64_t)j * ldv] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  const int m = (n + 1) / 2 * 2;   // even number of slots (a dummy column when n is odd)
  __syncthreads();
  const int npairs = m / 2;
  int gsize = 1;   // threads per pair: a power of two, so xor shuffles stay inside the group
  while (gsize * 2 * npairs <= JWG && gsize < 64) gsize *= 2;
  // column in slot k after r rotations: slot 0 holds column 0, slot k >= 1 holds
  // column 1 + ((k - 1 - r) mod (m - 1))
  auto slot_col = [&](int k, int r) {
    if (k == 0) return 0;
    int c = (k - 1 - r) % (m - 1);
    if (c < 0) c += m - 1;
    return 1 + c;
  };
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    double offmax = 0;
    for (int round = 0; round < m - 1; ++round) {
      // pairs of this round: (slot k, slot m-1-k)
      for (int pidx = tid / gsize; pidx < npairs; pidx += JWG / gsize) {
        const int sub = tid % gsize;
        int p = slot_col(pidx, round), q = slot_col(m - 1 - pidx, round);
        if (p > q) {
          const int t = p;
          p = q;
          q = t;
        }
        double al = 0, be = 0;
        c64 ga = make_double2(0, 0);
        if (q < n) {
#pragma unroll 4
          for (int i = sub; i < n; i += gsize) {
            const c64 ap = A[i + (int64_t)p * lda], aq = A[i + (int64_t)q * lda];
            al += cabs2<double>(ap);
            be += cabs2<double>(aq);
            ga = zadd(ga, zmulc(ap, aq));
          }
        }
        // reduce inside the group (groups are contiguous lanes; gsize divides 64 or is a multiple)
        for (int o = 1; o < gsize; o <<= 1) {
          al += __shfl_xor(al, o, 64);
          be += __shfl_xor(be, o, 64);
          ga.x += __shfl_xor(ga.x, o, 64);
          ga.y += __shfl_xor(ga.y, o, 64);
        }
        if (q >= n) continue;
        const double g = zabs(ga);
        if (!(g > 1e-15 * sqrt(al * be)) || g == 0.0) continue;
        offmax = fmax(offmax, g / sqrt(al * be));
        const double zeta = (be - al) / (2.0 * g);
        const double t = ((zeta >= 0) ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        const double c = 1.0 / sqrt(1.0 + t * t), sn = c * t;
        const c64 e = make_double2(ga.x / g, -ga.y / g);   // e^{-i phi}
        // two rows at a time: all their loads are issued before the first store (the
        // compiler cannot tell that the stores do not alias the next rows' loads)
        for (int i0 = sub; i0 < n; i0 += 2 * gsize) {
          c64 ap[2], aq[2], vp[2], vq[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int i = min(i0 + u * gsize, n - 1);
            ap[u] = A[i + (int64_t)p * lda];
            aq[u] = A[i + (int64_t)q * lda];
            vp[u] = V[i + (int64_t)p * ldv];
            vq[u] = V[i + (int64_t)q * ldv];
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int i = i0 + u * gsize;
            if (i >= n) break;
            const c64 aqe = zmul(e, aq[u]), vqe = zmul(e, vq[u]);
            A[i + (int64_t)p * lda] = zsub(zscale(ap[u], c), zscale(aqe, sn));
            A[i + (int64_t)q * lda] = zadd(zscale(ap[u], sn), zscale(aqe, c));
            V[i + (int64_t)p * ldv] = zsub(zscale(vp[u], c), zscale(vqe, sn));
            V[i + (int64_t)q * ldv] = zadd(zscale(vp[u], sn), zscale(vqe, c));
          }
        }
      }
      __syncthreads();
    }
    const double om = block_max_wg<JWG>(offmax, sh);
    if (tid == 0) sflag = om;
    __syncthreads();
    if (sflag < 1e-13) break;
  }
  // column norms, sort descending (simple selection by rank)
  for (int j = tid; j < n; j += JWG) {
    double s2 = 0;
    for (int i = 0; i < n; ++i) s2 += cabs2<double>(A[i + (int64_t)j * lda]);
    sigma[512 + j] = sqrt(s2);   // scratch area after the output
  }
  __syncthreads();
  // ranks under a strict total order (ranking.hpp), so perm is a permutation of 0..n-1
  // whatever the values are
  for (int j = tid; j < n; j += JWG) perm[desc_rank(n, sigma + 512, j)] = j;
  __syncthreads();
  for (int r = tid; r < n; r += JWG) sigma[r] = sigma[512 + perm[r]];
  __syncthreads();
  // normalise U columns
  for (int j = tid; j < n; j += JWG) {
    const double sj = sigma[512 + j];
    if (sj > 0)
      for (int i = 0; i < n; ++i) A[i + (int64_t)j * lda] = zscale(A[i + (int64_t)j * lda], 1.0 / sj);
  }
}

// ------------------------------------------------------------------ block one-sided Jacobi SVD
// The same factorisation A W = U Sigma, with the columns in nb blocks of bs: blocks are
// paired round-robin (as the columns above), one workgroup per block pair copies the pair's
// 2 bs columns of A and of W into LDS, runs one full one-sided Jacobi sweep over them (every
// column pair, round-robin inside the pair) and writes them back.  nb - 1 launches make an
// outer sweep; the largest |a_p^H a_q| / (|a_p| |a_q|) of the sweep decides convergence.  The
// single-workgroup kernel above moves both matrices through one CU's caches every round;
// here the rotations run in LDS on nb / 2 CUs.
__global__ void k_svd_init(int32_t n, c64* V, int32_t ldv, unsigned long long* flag) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n * n; t += gridDim.x * blockDim.x) {
    const int i = t % n, j = t / n;
    V[i + (int64_t)j * ldv] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *flag = 0ull;
}

// slot k of nslots after r rotations holds: slot 0 item 0, slot k >= 1 item
// 1 + ((k - 1 - r) mod (nslots - 1))
__device__ __forceinline__ int rr_slot(int k, int r, int nslots) {
  if (k == 0) return 0;
  int c = (k - 1 - r) % (nslots - 1);
  if (c < 0) c += nslots - 1;
  return 1 + c;
}

constexpr int BJ_THREADS = 1024;
constexpr size_t BJ_LDS = 128 * 1024;   // the block pair's columns of A and W

__global__ void __launch_bounds__(BJ_THREADS) k_svd_block(int32_t n, int32_t bs, int32_t nb, int32_t round, c64* A,
                                                          int32_t lda, c64* V, int32_t ldv,
                                                          unsigned long long* flag) {
  __shared__ c64 bj_lds[BJ_LDS / sizeof(c64)];
  __shared__ double sh[BJ_THREADS / 64];
  c64* la = bj_lds;                       // [2 bs][n]
  c64* lv = la + (size_t)2 * bs * n;      // [2 bs][n]
  int bp = rr_slot(blockIdx.x, round, nb), bq = rr_slot(nb - 1 - blockIdx.x, round, nb);
  const int tid = threadIdx.x;
  const int cols = 2 * bs;
  // local column c: block bp's columns first, then bq's; columns at or past n are padding
  auto gcol = [&](int c) { return (c < bs) ? bp * bs + c : bq * bs + (c - bs); };
  for (int t = tid; t < cols * n; t += BJ_THREADS) {
    const int c = t / n, i = t - c * n;
    const int g = gcol(c);
    la[t] = (g < n) ? A[i + (int64_t)g * lda] : make_double2(0, 0);
    lv[t] = (g < n) ? V[i + (int64_t)g * ldv] : make_double2(0, 0);
  }
  __syncthreads();
  // threads per column pair: a power of two up to 64 (one wave), bs pairs per inner round
  int gsize = 64;
  while (gsize * bs > BJ_THREADS) gsize >>= 1;
  const int pidx = tid / gsize, sub = tid % gsize;
  double offmax = 0;
  for (int ir = 0; ir < cols - 1; ++ir) {
    if (pidx < bs) {
      int p = rr_slot(pidx, ir, cols), q = rr_slot(cols - 1 - pidx, ir, cols);
      if (p > q) {
        const int t = p;
        p = q;
        q = t;
      }
      const bool valid = gcol(p) < n && gcol(q) < n;
      c64* ap = la + (size_t)p * n;
      c64* aq = la + (size_t)q * n;
      double al = 0, be = 0;
      c64 ga = make_double2(0, 0);
      if (valid) {
        for (int i = sub; i < n; i += gsize) {
          const c64 x = ap[i], y = aq[i];
          al += cabs2<double>(x);
          be += cabs2<double>(y);
          ga = zadd(ga, zmulc(x, y));
        }
      }
      for (int o = 1; o < gsize; o <<= 1) {
        al += __shfl_xor(al, o, 64);
        be += __shfl_xor(be, o, 64);
        ga.x += __shfl_xor(ga.x, o, 64);
        ga.y += __shfl_xor(ga.y, o, 64);
      }
      const double g = zabs(ga);
      if (valid && g > 1e-15 * sqrt(al * be) && g != 0.0) {
        offmax = fmax(offmax, g / sqrt(al * be));
        const double zeta = (be - al) / (2.0 * g);
        const double t = ((zeta >= 0) ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        const double c = 1.0 / sqrt(1.0 + t * t), sn = c * t;
        const c64 e = make_double2(ga.x / g, -ga.y / g);   // e^{-i phi}
        c64* vp = lv + (size_t)p * n;
        c64* vq = lv + (size_t)q * n;
        for (int i = sub; i < n; i += gsize) {
          const c64 x = ap[i], y = zmul(e, aq[i]);
          ap[i] = zsub(zscale(x, c), zscale(y, sn));
          aq[i] = zadd(zscale(x, sn), zscale(y, c));
          const c64 u = vp[i], w = zmul(e, vq[i]);
          vp[i] = zsub(zscale(u, c), zscale(w, sn));
          vq[i] = zadd(zscale(u, sn), zscale(w, c));
        }
      }
    }
    __syncthreads();
  }
  for (int t = tid; t < cols * n; t += BJ_THREADS) {
    const int c = t / n, i = t - c * n;
    const int g = gcol(c);
    if (g < n) {
      A[i + (int64_t)g * lda] = la[t];
      V[i + (int64_t)g * ldv] = lv[t];
    }
  }
  const double om = block_max_wg<BJ_THREADS>(offmax, sh);
  // values are non-negative, so their bit patterns order like the values
  if (tid == 0 && om > 0) atomicMax(flag, (unsigned long long)__double_as_longlong(om));
}

// column norms, sigma sorted descending with its permutation, U columns normalised (the
// tail of the single-workgroup kernel)
__global__ void __launch_bounds__(JWG) k_svd_finish(int32_t n, c64* A, int32_t lda, double* sigma, int32_t* perm) {
  const int tid = threadIdx.x;
  for (int j = tid; j < n; j += JWG) {
    double s2 = 0;
    for (int i = 0; i < n; ++i) s2 += cabs2<double>(A[i + (int64_t)j * lda]);
    sigma[512 + j] = sqrt(s2);
  }
  __syncthreads();
  for (int j = tid; j < n; j += JWG) perm[desc_rank(n, sigma + 512, j)] = j;
  __syncthreads();
  for (int r = tid; r < n; r += JWG) sigma[r] = sigma[512 + perm[r]];
  __syncthreads();
  for (int j = tid; j < n; j += JWG) {
    const double sj = sigma[512 + j];
    if (sj > 0)
      for (int i = 0; i < n; ++i) A[i + (int64_t)j * lda] = zscale(A[i + (int64_t)j * lda], 1.0 / sj);
  }
}

// ------------------------------------------------------------------ right singular vectors
// Where only sigma and the right singular vectors are wanted (the Rayleigh-Ritz extraction, the
// bands), one-sided Jacobi starts from the pivoted QR A P = Q R and works on the columns of R^H:
// R^H V = U Sigma gives A = (Q V) Sigma (P U)^H, so the right vectors are the rotated columns
// themselves, normalised, in the rows that P names, and no second matrix is rotated.  The columns of
// R^H are already close to orthogonal (Drmac and Veselic, SIAM J. Matrix Anal. Appl. 29, 2008):
// 9-10 sweeps instead of 20-24 on Hankel matrices of a few eigenvalues above noise.
//
// A column pair belongs to a group of 8 to 64 lanes; its three inner products are summed by DPP with
// the four values split over the lanes of each quad.  Order 64 stays in one workgroup's LDS for all
// sweeps, larger orders take their blocks in turn as k_svd_block does.  Latency bound (one workgroup,
// 63 rounds a sweep).  Hankel SVD of order 64: QR 0.17 + sweeps 0.64 ms, where rotating A and W from the
// start took 4.8 ms (21 sweeps of 0.23); order 16 of the bands 0.03 ms (was 0.11).

template <int CTRL>
__device__ __forceinline__ double dppd(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_of(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// the sum and the maximum over the wave, in every lane: 16 lanes by DPP, the four rows by readlane
__device__ __forceinline__ double wave_sum_dpp(double t) {
  t += dppd<0xB1>(t);    // lane ^ 1
  t += dppd<0x4E>(t);    // lane ^ 2
  t += dppd<0x141>(t);   // mirrored in 8 lanes
  t += dppd<0x140>(t);   // mirrored in 16 lanes
  return (lane_of(t, 0) + lane_of(t, 16)) + (lane_of(t, 32) + lane_of(t, 48));
}
__device__ __forceinline__ double wave_max_dpp(double t) {
  t = fmax(t, dppd<0xB1>(t));
  t = fmax(t, dppd<0x4E>(t));
  t = fmax(t, dppd<0x141>(t));
  t = fmax(t, dppd<0x140>(t));
  return fmax(fmax(lane_of(t, 0), lane_of(t, 16)), fmax(lane_of(t, 32), lane_of(t, 48)));
}

// 1 / sqrt(x) for normal x > 0: the hardware's approximation and one step of third order (two
// units in the last place), a fifth of the latency of a square root and a division.
__device__ __forceinline__ double rsqrt1(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// The power of two that a matrix whose largest column has the norm nx is divided by, 0 if there is none:
// the sweeps multiply squares of norms with each other, which overflows past 1e77 otherwise.
__device__ __forceinline__ int sv_exponent(double nx) {
  return nx > 0 && nx <= 1.79769313486231571e308 ? ilogb(nx) : 0;
}

constexpr int SV_T = 1024;
constexpr size_t SV_LDS = 150 * 1024;   // columns of a block pair (or the whole matrix in the QR)

// Pivoted Householder QR of A (n x n): X = R^H (lower triangular) divided by 2^piv[n], piv[k]: the
// column of A taken k-th.  One workgroup; a lane owns CPL columns, a wave 16 rows of them, all in registers, so that the
// inner products with the reflector are sums over a lane's own rows and then over the waves; the
// reflector's rows are read from the pivot's lane.  A wave instruction takes four cycles whatever it
// is for, so the parts that every wave repeats (pivot, reflector) want few waves: with a column per
// wave and 16 waves in LDS a step of order 64 took 4.8 us.
template <int CPL>
__global__ void __launch_bounds__(256 * CPL) k_svd_qr(int32_t n, const c64* A, int32_t lda, c64* X, int32_t* piv) {
  A += blockIdx.y * (int64_t)lda * n;
  X += blockIdx.y * (int64_t)n * n;
  piv += blockIdx.y * (n + 1);
  constexpr int NW = 4 * CPL, RW = 16;
  __shared__ double pn[NW][64 * CPL];   // per wave: squared norms of the columns' remaining rows
  __shared__ c64 pd[NW][64 * CPL];      // per wave: products with the reflector
  __shared__ c64 rowk[64 * CPL];        // row k
  double nmax = 0;   // norm of the largest column, the first pivot's
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i0 = wv * RW;
  c64 m[CPL][RW];
  int pos[CPL];   // step at which the column was taken, n: not yet
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int j = lane + 64 * c;
    double t = 0;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      m[c][r] = (j < n && i0 + r < n) ? A[i0 + r + (int64_t)j * lda] : make_double2(0, 0);
      t += cabs2<double>(m[c][r]);
    }
    pn[wv][j] = t;
    if (wv == 0) rowk[j] = m[c][0];
    pos[c] = j < n ? n : -1;
  }
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    // the remaining column of the largest norm (a NaN counts as the largest)
    double nrm[CPL], best = -1;
    int bc = 0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      nrm[c] = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) nrm[c] += pn[w][lane + 64 * c];
      const double v = pos[c] != n ? -1.0 : nrm[c] == nrm[c] ? nrm[c] : __builtin_inf();
      if (v > best) {
        best = v;
        bc = c;
      }
    }
    const int pl = __ffsll((unsigned long long)__ballot(best == wave_max_dpp(best))) - 1;
    const int pc = CPL == 1 ? 0 : __builtin_amdgcn_readlane(bc, pl), p = pl + 64 * pc;
    // reflector I - b v v^H, v = x - alpha e_k of the pivot's rows k..n-1: |v|^2 = 2 (|x|^2 + |x| |x_k|)
    const double nx2 = lane_of(CPL == 1 ? nrm[0] : (pc ? nrm[CPL - 1] : nrm[0]), pl);
    const c64 xk = rowk[p];
    const double nx = sqrt(nx2), ak = sqrt(cabs2<double>(xk));
    nmax = fmax(nmax, nx);
    const c64 ph = ak > 0 ? make_double2(xk.x / ak, xk.y / ak) : make_double2(1, 0);
    const c64 alpha = zscale(ph, -nx);
    const double vv = nx2 + nx * ak, b = vv > 0 ? 1.0 / vv : 0.0;
    c64 v[RW], d[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) d[c] = make_double2(0, 0);
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      v[r] = make_double2(0, 0);
      if (i0 + r < k) continue;   // wave-uniform
      const c64 src = CPL == 1 || pc == 0 ? m[0][r] : m[CPL - 1][r];
      v[r] = make_double2(lane_of(src.x, pl), lane_of(src.y, pl));
      if (i0 + r == k) v[r] = zsub(v[r], alpha);
#pragma unroll
      for (int c = 0; c < CPL; ++c) d[c] = zadd(d[c], zmulc(v[r], m[c][r]));
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) pd[wv][lane + 64 * c] = d[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int j = lane + 64 * c;
      d[c] = make_double2(0, 0);
#pragma unroll
      for (int w = 0; w < NW; ++w) d[c] = zadd(d[c], pd[w][j]);
      d[c] = zscale(d[c], b);
      const bool on = pos[c] == n && j != p;
      double t = 0;
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        if (i0 + r < k) continue;
        const c64 u = zsub(m[c][r], zmul(v[r], d[c]));
        if (on) m[c][r] = u;
        if (i0 + r == k && j == p) m[c][r] = alpha;
        if (i0 + r > k) t += cabs2<double>(u);
        if (i0 + r == k + 1) rowk[j] = m[c][r];
      }
      pn[wv][j] = t;
      if (j == p) {
        pos[c] = k;
        if (wv == 0) piv[k] = p;
      }
    }
    __syncthreads();
  }
  // R[i][column] is the conjugate of X[position of the column][i]
  const int ex = sv_exponent(nmax);
  if (threadIdx.x == 0) piv[n] = ex;
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    if (lane + 64 * c >= n) continue;
#pragma unroll
    for (int r = 0; r < RW; ++r)
      if (i0 + r < n)
        X[pos[c] + (int64_t)(i0 + r) * n] = pos[c] >= i0 + r ? make_double2(ldexp(m[c][r].x, -ex), -ldexp(m[c][r].y, -ex))
                                                            : make_double2(0, 0);
  }
}

// The same for orders beyond 128, whose columns do not fit the registers: M is a copy of A in global
// memory, a wave owns every NW-th column, four at a time, RP rows a lane.  Every wave finds the pivot
// and forms the reflector by itself, so a step has one barrier.
template <int RP>
__global__ void __launch_bounds__(SV_T) k_svd_qr_big(int32_t n, const c64* A, int32_t lda, c64* M, c64* X,
                                                     int32_t* piv) {
  A += blockIdx.y * (int64_t)lda * n;
  M += blockIdx.y * (int64_t)n * n;
  X += blockIdx.y * (int64_t)n * n;
  piv += blockIdx.y * (n + 1);
  __shared__ double cnb[2][64 * RP];   // squared norms of the remaining parts, -1: taken (this step's, the next's)
  __shared__ int32_t order[64 * RP];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int CB = 4;
  const int NW = blockDim.x >> 6;
  double nmax = 0;   // norm of the largest column, the first pivot's
  for (int j = wv; j < n; j += NW) {
    double t = 0;
    for (int i = lane; i < n; i += 64) {
      const c64 v = A[i + (int64_t)j * lda];
      M[i + j * n] = v;
      t += cabs2<double>(v);
    }
    t = wave_sum_dpp(t);
    if (lane == 0) cnb[0][j] = t;
  }
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    const double* cn = cnb[k & 1];
    double* cnext = cnb[(k + 1) & 1];
    // the remaining column of the largest norm (a NaN counts as the largest)
    double best = -1;
    int p = n;
    for (int j = lane; j < n; j += 64) {
      double v = cn[j];
      if (v != v) v = __builtin_inf();
      if (v > best) {
        best = v;
        p = j;
      }
    }
    const unsigned long long top = __ballot(best == wave_max_dpp(best));
    p = __builtin_amdgcn_readlane(p, __ffsll(top) - 1);
    // reflector I - b v v^H with v = x - alpha e_k of its rows k..n-1
    c64 v[RP];
    double nx2 = 0;
#pragma unroll
    for (int r = 0; r < RP; ++r) {
      const int i = lane + 64 * r;
      v[r] = (i >= k && i < n) ? M[i + p * n] : make_double2(0, 0);
      nx2 += cabs2<double>(v[r]);
    }
    nx2 = wave_sum_dpp(nx2);
    const c64 xk = M[k + p * n];
    const double nx = sqrt(nx2), ak = sqrt(cabs2<double>(xk));
    nmax = fmax(nmax, nx);
    const c64 ph = ak > 0 ? make_double2(xk.x / ak, xk.y / ak) : make_double2(1, 0);
    const c64 alpha = zscale(ph, -nx);
    // |v|^2 = 2 (nx^2 + nx |x_k|)
    const double vv = 2.0 * (nx2 + nx * ak), b = vv > 0 ? 2.0 / vv : 0.0;
#pragma unroll
    for (int r = 0; r < RP; ++r)
      if (lane + 64 * r == k) v[r] = zsub(v[r], alpha);
    for (int j0 = wv; j0 < n; j0 += NW * CB) {
      c64 m[CB][RP];
      c64 d[CB];
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const int j = min(j0 + c * NW, n - 1);
        d[c] = make_double2(0, 0);
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          const int i = lane + 64 * r;
          m[c][r] = (i >= k && i < n) ? M[i + j * n] : make_double2(0, 0);
          d[c] = zadd(d[c], zmulc(v[r], m[c][r]));
        }
      }
#pragma unroll
      for (int c = 0; c < CB; ++c) d[c] = make_double2(wave_sum_dpp(d[c].x) * b, wave_sum_dpp(d[c].y) * b);
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const int j = j0 + c * NW;
        const bool on = j < n && j != p && !(cn[min(j, n - 1)] < 0);   // wave-uniform
        double t = 0;
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          const int i = lane + 64 * r;
          const c64 u = zsub(m[c][r], zmul(v[r], d[c]));
          if (on && i >= k && i < n) M[i + j * n] = u;
          t += i > k && i < n ? cabs2<double>(u) : 0.0;
        }
        t = wave_sum_dpp(t);
        if (j < n && lane == 0) cnext[j] = on ? t : -1.0;
      }
    }
    __syncthreads();
    if (tid == 0) {   // column p is not read again before the end
      order[k] = p;
      piv[k] = p;
      M[k + p * n] = alpha;
    }
  }
  __syncthreads();
  // X[j][k] = conj(R[k][j]), R[k][j] = M[k][order[j]] for j >= k
  const int ex = sv_exponent(nmax);
  if (tid == 0) piv[n] = ex;
  for (int t = tid; t < n * n; t += blockDim.x) {
    const int j = t % n, k = t / n;
    c64 v = make_double2(0, 0);
    if (j >= k) v = zconj(M[k + order[j] * n]);
    X[j + k * n] = make_double2(ldexp(v.x, -ex), ldexp(v.y, -ex));
  }
}

__device__ double block_max_any(double v, double* sh) {
  v = wave_max_dpp(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, sh[w]);
  __syncthreads();
  return r;
}
// LDS column stride: 128 bytes off a multiple of the 64 banks, so that the groups of a wave read
// neighbouring columns from different banks.
__host__ __device__ inline int sv_ldc(int n) { return (n + 7) / 16 * 16 + 8; }
constexpr double SV_TOL2 = 1e-26;
constexpr int SV_SWEEPS = 60;   // at most; also the flags of a matrix
// One sweep over the columns of a block pair in LDS (nb = 2: all columns, `sweeps` times or until
// converged).  flags[s]: the largest (|a_p^H a_q| / |a_p| |a_q|)^2 of sweep s, as bits; a launch of a
// sweep whose predecessor was converged returns at once, so the host may queue several.
// RPL: rows of a column per lane, kept in registers from the inner products to the rotation.
template <int RPL>
__global__ void __launch_bounds__(1024) k_svd_cols(int32_t n, int32_t bs, int32_t nb, int32_t round, int32_t sweep,
                                                   int32_t sweeps, int32_t gsize, c64* X, unsigned long long* flags) {
  extern __shared__ __align__(16) unsigned char sv_smem[];
  __shared__ double sh[16];
  X += blockIdx.y * (int64_t)n * n;
  flags += blockIdx.y * SV_SWEEPS;
  if (sweep > 0 && __longlong_as_double((long long)flags[sweep - 1]) < SV_TOL2) return;
  c64* la = reinterpret_cast<c64*>(sv_smem);   // [2 bs][ldc]
  const int ldc = sv_ldc(n);
  const int bp = rr_slot(blockIdx.x, round, nb), bq = rr_slot(nb - 1 - blockIdx.x, round, nb);
  const int tid = threadIdx.x, cols = 2 * bs;
  auto gcol = [&](int c) { return (c < bs) ? bp * bs + c : bq * bs + (c - bs); };
  for (int t = tid; t < cols * n; t += blockDim.x) {
    const int c = t / n, i = t - c * n, g = gcol(c);
    la[i + c * ldc] = (g < n) ? X[i + g * n] : make_double2(0, 0);
  }
  __syncthreads();
  const int pidx = tid / gsize, sub = tid % gsize;
  double off2 = 0;
  for (int sw = 0; sw < sweeps; ++sw) {
    off2 = 0;
    for (int ir = 0; ir < cols - 1; ++ir) {
      if (pidx < bs) {
        int p = rr_slot(pidx, ir, cols), q = rr_slot(cols - 1 - pidx, ir, cols);
        if (p > q) {
          const int t = p;
          p = q;
          q = t;
        }
        c64* ap = la + p * ldc;
        c64* aq = la + q * ldc;
        double al = 0, be = 0, gx = 0, gy = 0;
        c64 xs[RPL], ys[RPL];
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
          const int i = sub + r * gsize;
          xs[r] = i < n ? ap[i] : make_double2(0, 0);
          ys[r] = i < n ? aq[i] : make_double2(0, 0);
          const c64 x = xs[r], y = ys[r];
          al += cabs2<double>(x);
          be += cabs2<double>(y);
          gx += x.x * y.x + x.y * y.y;
          gy += x.x * y.y - x.y * y.x;
        }
        // lane bits (1, 0) of a quad keep (0,0) al, (1,0) be, (0,1) gx, (1,1) gy
        const bool odd = (sub & 1) != 0, up = (sub & 2) != 0;
        const double k0 = (odd ? gx : al) + dppd<0xB1>(odd ? al : gx);
        const double k1 = (odd ? gy : be) + dppd<0xB1>(odd ? be : gy);
        double t = (up ? k1 : k0) + dppd<0x4E>(up ? k0 : k1);
        if (gsize == 8) {
          t += dppd<0x1B>(dppd<0x141>(t));   // lane ^ 4: mirrored in 8 lanes, then in 4
        } else {
          t += dppd<0x124>(t);   // rotated by 4 in 16 lanes
          t += dppd<0x128>(t);   // rotated by 8
        }
        if (gsize > 16) t += __shfl_xor(t, 16, 64);
        if (gsize > 32) t += __shfl_xor(t, 32, 64);
        al = dppd<0x00>(t);
        gx = dppd<0x55>(t);
        be = dppd<0xAA>(t);
        gy = dppd<0xFF>(t);
        const double g2 = gx * gx + gy * gy, ab = al * be;
        if (g2 > 1e-30 * ab && g2 > 0.0) {   // padding columns are zero
          off2 = fmax(off2, g2 / ab);
          // rotation by c and s e^{-i phi}: with d = be - al and h = sqrt(d^2 + 4 |g|^2),
          // c^2 = (|d| + h) / 2h and s c = sign(d) |g| / h
          const double d = be - al, ih = rsqrt1(d * d + 4.0 * g2);
          const double c2 = 0.5 + 0.5 * fabs(d) * ih, ic = rsqrt1(c2), c = c2 * ic;
          const double f = (d >= 0 ? ih : -ih) * ic;
          const c64 se = make_double2(gx * f, -gy * f);   // s e^{-i phi}
#pragma unroll
          for (int r = 0; r < RPL; ++r) {
            const int i = sub + r * gsize;
            if (i < n) {
              ap[i] = zsub(zscale(xs[r], c), zmul(se, ys[r]));
              aq[i] = zadd(zscale(ys[r], c), zmul(zconj(se), xs[r]));
            }
          }
        }
      }
      __syncthreads();
    }
    if (sweeps > 1) {
      off2 = block_max_any(off2, sh);
      if (!(off2 >= SV_TOL2)) break;
    }
  }
  for (int t = tid; t < cols * n; t += blockDim.x) {
    const int c = t / n, i = t - c * n, g = gcol(c);
    if (g < n) X[i + g * n] = la[i + c * ldc];
  }
  off2 = block_max_any(off2, sh);
  if (tid == 0 && off2 > 0) atomicMax(flags + sweep, (unsigned long long)__double_as_longlong(off2));
}

// a Hermitian positive definite A: U = W, so its own columns are rotated
__global__ void k_svd_copy(int32_t n, const c64* A, int32_t lda, c64* X, int32_t* piv) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n * n) X[t] = A[t % n + (int64_t)(t / n) * lda];
  if (t < n) piv[t] = t;
  if (t == 0) piv[n] = 0;
}

__global__ void k_svd_clear(int32_t n, unsigned long long* flags) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) flags[i] = 0ull;
}

// sigma (descending, with its permutation) and W = P U: column j of W has the normalised column j
// of X in the rows piv; sigma is multiplied by 2^piv[n].  sigma[SV_STATE]: 0, or 1 if the sweep `last`
// was run and still rotated (a sweep after the converged one leaves its flag at zero).
__global__ void __launch_bounds__(SV_T) k_svd_right(int32_t n, const c64* X, const int32_t* piv, c64* W, int32_t ldw,
                                                    double* sigma, int32_t* perm, const unsigned long long* flags,
                                                    int32_t last) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  X += blockIdx.y * (int64_t)n * n;
  piv += blockIdx.y * (n + 1);
  W += blockIdx.y * (int64_t)ldw * n;
  sigma += blockIdx.y * 1024;
  perm += blockIdx.y * 512;
  if (tid == 0)
    sigma[SV_STATE] = __longlong_as_double((long long)flags[blockIdx.y * SV_SWEEPS + last]) >= SV_TOL2 ? 1.0 : 0.0;
  for (int j = wv; j < n; j += SV_T / 64) {
    double t = 0;
    for (int i = lane; i < n; i += 64) t += cabs2<double>(X[i + j * n]);
    t = sqrt(wave_sum_dpp(t));
    if (lane == 0) sigma[512 + j] = ldexp(t, piv[n]);
    const double inv = t > 0 ? 1.0 / t : 0.0;
    for (int i = lane; i < n; i += 64) W[piv[i] + (int64_t)j * ldw] = zscale(X[i + j * n], inv);
  }
  __syncthreads();
  for (int j = tid; j < n; j += SV_T) perm[desc_rank(n, sigma + 512, j)] = j;
  __syncthreads();
  for (int r = tid; r < n; r += SV_T) sigma[r] = sigma[512 + perm[r]];
}

// ------------------------------------------------------------------ small GEMM (one workgroup)
// C = op(A) * B (+ scale of columns), op = identity or conjugate transpose.
__global__ void __launch_bounds__(SWG) k_small_gemm(int32_t m, int32_t n, int32_t k, const c64* A, int32_t lda,
                                                     int32_t transA, const c64* B, int32_t ldb, c64* C,
                                                     int32_t ldc, const double* colscale, const int32_t* bperm) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < m * n; t += gridDim.x * blockDim.x) {
    const int i = t % m, j = t / m;
    const int jb = bperm ? bperm[j] : j;
    c64 acc = make_double2(0, 0);
    for (int l = 0; l < k; ++l) {
      const c64 a = transA ? zconj(A[l + (int64_t)i * lda]) : A[i + (int64_t)l * lda];
      acc = zadd(acc, zmul(a, B[l + (int64_t)jb * ldb]));
    }
    if (colscale) acc = zscale(acc, colscale[j]);
    C[i + (int64_t)j * ldc] = acc;
  }
}

int32_t small_gemm(int32_t m, int32_t n, int32_t k, const c64* A, int32_t lda, bool transA, const c64* B,
                   int32_t ldb, c64* C, int32_t ldc, const double* colscale, const int32_t* bperm, hipStream_t st) {
  if (m <= 0 || n <= 0) return CBS_OK;
  const int g = std::min(1024, (m * n + 255) / 256);
  hipLaunchKernelGGL(k_small_gemm, dim3(g), dim3(256), 0, st, m, n, k, A, lda, (int32_t)transA, B, ldb, C, ldc,
                     colscale, bperm);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

// ------------------------------------------------------------------ eigen-decomposition
// Complex Schur form by Householder reduction to Hessenberg form and single-shift QR
// with Wilkinson shifts and deflation; eigenvectors by back substitution on the
// triangular factor and the accumulated unitary Z.  A (n x n) is destroyed; w receives
// the eigenvalues, Vout the unit-norm eigenvectors.  work: n*n (Z) + n*n (Y).
__global__ void __launch_bounds__(SWG) k_eig(int32_t n, c64* H, int32_t ldh, c64* w, c64* Vout, int32_t ldv,
                                              c64* Z, c64* Y, int32_t* info) {
  __shared__ double sh[SWG / 64];
  __shared__ c64 sv[512];
  __shared__ c64 sg[1];
  __shared__ c64 sxy[2];   // (x, y) of the next Givens rotation of the sweep
  __shared__ int s_lo, s_hi, s_iter, s_done;
  const int tid = threadIdx.x;
  for (int t = tid; t < n * n; t += SWG) {
    const int i = t % n, j = t / n;
    Z[i + (int64_t)j * n] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  // --- Householder reduction to upper Hessenberg form
  for (int k = 0; k + 2 < n; ++k) {
    double nx2 = 0;
    for (int i = k + 1 + tid; i < n; i += SWG) nx2 += cabs2<double>(H[i + (int64_t)k * ldh]);
    nx2 = block_sum(nx2, sh);
    const c64 x0 = H[k + 1 + (int64_t)k * ldh];
    const double nx = sqrt(nx2);
    if (nx == 0.0) continue;
    const double a0 = zabs(x0);
    const c64 ph = (a0 > 0) ? make_double2(x0.x / a0, x0.y / a0) : make_double2(1, 0);
    const c64 alpha = zscale(ph, -nx);   // new subdiagonal value
    // v = x - alpha e1, normalised
    for (int i = k + 1 + tid; i < n; i += SWG) {
      c64 v = H[i + (int64_t)k * ldh];
      if (i == k + 1) v = zsub(v, alpha);
      sv[i] = v;
    }
    __syncthreads();
    double vn2 = 0;
    for (int i = k + 1 + tid; i < n; i += SWG) vn2 += cabs2<double>(sv[i]);
    vn2 = block_sum(vn2, sh);
    if (vn2 == 0.0) continue;
    const double inv = 1.0 / sqrt(vn2);
    for (int i = k + 1 + tid; i < n; i += SWG) sv[i] = zscale(sv[i], inv);
    __syncthreads();
    // left: H[k+1:, j] -= 2 v (v^H H[k+1:, j]) for j >= k
    for (int j = k + tid; j < n; j += SWG) {
      c64 d = make_double2(0, 0);
      for (int i = k + 1; i < n; ++i) d = zadd(d, zmulc(sv[i], H[i + (int64_t)j * ldh]));
      d = zscale(d, 2.0);
      for (int i = k + 1; i < n; ++i) H[i + (int64_t)j * ldh] = zsub(H[i + (int64_t)j * ldh], zmul(sv[i], d));
    }
    __syncthreads();
    // right: H[i, k+1:] -= 2 (H[i, k+1:] v) v^H for all i; same for Z
    for (int i = tid; i < 2 * n; i += SWG) {
      c64* M = (i < n) ? H : Z;
      const int r = (i < n) ? i : i - n;
      const int ld = (i < n) ? ldh : n;
      c64 d = make_double2(0, 0);
      for (int j = k + 1; j < n; ++j) d = zadd(d, zmul(M[r + (int64_t)j * ld], sv[j]));
      d = zscale(d, 2.0);
      for (int j = k + 1; j < n; ++j) M[r + (int64_t)j * ld] = zsub(M[r + (int64_t)j * ld], zmul(d, zconj(sv[j])));
    }
    __syncthreads();
    for (int i = k + 2 + tid; i < n; i += SWG) H[i + (int64_t)k * ldh] = make_double2(0, 0);
    __syncthreads();
  }
  // --- shifted QR on the Hessenberg matrix (full Schur form)
  if (tid == 0) {
    s_hi = n - 1;
    s_iter = 0;
    s_done = 0;
  }
  __syncthreads();
  const double eps = 2.220446049250313e-16;
  int total_iter = 0;
  while (true) {
    if (tid == 0) {
      int hi = s_hi;
      while (hi >= 0) {
        if (hi == 0) {
          w[0] = H[0];
          hi = -1;
          break;
        }
        int l = hi;
        while (l > 0) {
          const double sd = zabs(H[l + (int64_t)(l - 1) * ldh]);
          const double dd = zabs(H[l + (int64_t)l * ldh]) + zabs(H[l - 1 + (int64_t)(l - 1) * ldh]);
          if (sd <= eps * dd || sd < 1e-300) break;
          --l;
        }
        if (l > 0) H[l + (int64_t)(l - 1) * ldh] = make_double2(0, 0);
        if (l == hi) {
          w[hi] = H[hi + (int64_t)hi * ldh];
          --hi;
          s_iter = 0;
          continue;
        }
        // shift from the trailing 2x2 block of the active window [l, hi]
        const c64 a = H[hi - 1 + (int64_t)(hi - 1) * ldh], b = H[hi - 1 + (int64_t)hi * ldh];
        const c64 c = H[hi + (int64_t)(hi - 1) * ldh], d = H[hi + (int64_t)hi * ldh];
        c64 mu;
        if (s_iter > 0 && s_iter % 11 == 0) {
          mu = zadd(d, make_double2(0.75 * zabs(c), 0.0));   // exceptional shift
        } else {
          const c64 hd = zscale(zsub(a, d), 0.5);
          const c64 disc = zsqrt(zadd(zmul(hd, hd), zmul(b, c)));
          const c64 m1 = zadd(zscale(zadd(a, d), 0.5), disc), m2 = zsub(zscale(zadd(a, d), 0.5), disc);
          mu = (zabs(zsub(m1, d)) < zabs(zsub(m2, d))) ? m1 : m2;
        }
        sg[0] = mu;
        s_lo = l;
        sxy[0] = zsub(H[l + (int64_t)l * ldh], mu);
        sxy[1] = H[l + 1 + (int64_t)l * ldh];
        break;
      }
      s_hi = hi;
      if (hi < 0) s_done = 1;
    }
    __syncthreads();
    if (s_done) break;
    if (++total_iter > 60 * n) {
      if (tid == 0) info[0] = 1;   // QR failed to converge
      break;
    }
    const int lo = s_lo, hi = s_hi;
    const c64 mu = sg[0];
    if (tid == 0) s_iter = s_iter + 1;
    // implicit single-shift sweep: Givens rotations chase the bulge from lo to hi.  The
    // pair (x, y) that defines rotation k comes from the column update of rotation k-1
    // (rows k and k+1 of column k-1, through LDS), so every thread forms (c, s) itself.
    for (int k = lo; k < hi; ++k) {
      const c64 x = sxy[0], y = sxy[1];
      const double nx = zabs(x), ny = zabs(y);
      const double r = hypot(nx, ny);
      double c;   // G = [[c, s], [-conj(s), c]] with c real: G [x; y] = [r'; 0]
      c64 s;
      if (r == 0.0) {
        c = 1.0;
        s = make_double2(0, 0);
      } else if (nx == 0.0) {
        c = 0.0;
        s = zscale(zconj(y), 1.0 / ny);
      } else {
        c = nx / r;
        const c64 ux = make_double2(x.x / nx, x.y / nx);   // phase of x
        s = zscale(zmul(ux, zconj(y)), 1.0 / r);
      }
      // rows k, k+1: [hk; hk1] <- [c hk + s hk1; -conj(s) hk + c hk1], columns max(k-1,0)..n-1
      const int j0 = (k > lo) ? k - 1 : lo;
      for (int j = j0 + tid; j < n; j += SWG) {
        const c64 hk = H[k + (int64_t)j * ldh], hk1 = H[k + 1 + (int64_t)j * ldh];
        H[k + (int64_t)j * ldh] = zadd(zscale(hk, c), zmul(s, hk1));
        H[k + 1 + (int64_t)j * ldh] = zsub(zscale(hk1, c), zmul(zconj(s), hk));
      }
      __syncthreads();
      // columns k, k+1 of H (rows 0..min(k+2, hi)) and of Z: M G^H
      const int rmax = std::min(k + 2, hi);
      for (int i = tid; i <= rmax + n; i += SWG) {
        c64* M;
        int r2, ld;
        if (i <= rmax) {
          M = H;
          r2 = i;
          ld = ldh;
        } else {
          M = Z;
          r2 = i - rmax - 1;
          ld = n;
          if (r2 >= n) continue;
        }
        const c64 mk = M[r2 + (int64_t)k * ld], mk1 = M[r2 + (int64_t)(k + 1) * ld];
        const c64 nk = zadd(zscale(mk, c), zmul(zconj(s), mk1));
        M[r2 + (int64_t)k * ld] = nk;
        M[r2 + (int64_t)(k + 1) * ld] = zsub(zscale(mk1, c), zmul(s, mk));
        if (i <= rmax && r2 == k + 1) sxy[0] = nk;   // x of rotation k+1
        if (i <= rmax && r2 == k + 2) sxy[1] = nk;   // y of rotation k+1 (the bulge)
      }
      __syncthreads();
    }
  }
  __syncthreads();
  // --- eigenvectors of the triangular T = H: T y = w_k y, y_k = 1, y_i = 0 for i > k
  double tnorm = 0;
  for (int t = tid; t < n * n; t += SWG) {
    const int i = t % n, j = t / n;
    if (i <= j) tnorm = fmax(tnorm, zabs(H[i + (int64_t)j * ldh]));
  }
  tnorm = block_max(tnorm, sh);
  const double smin = fmax(eps * tnorm, 1e-300);
  for (int k = tid; k < n; k += SWG) {
    const c64 lam = H[k + (int64_t)k * ldh];
    for (int i = n - 1; i > k; --i) Y[i + (int64_t)k * n] = make_double2(0, 0);
    Y[k + (int64_t)k * n] = make_double2(1, 0);
    for (int i = k - 1; i >= 0; --i) {
      c64 acc = H[i + (int64_t)k * ldh];
      for (int j = i + 1; j < k; ++j) acc = zadd(acc, zmul(H[i + (int64_t)j * ldh], Y[j + (int64_t)k * n]));
      c64 d = zsub(H[i + (int64_t)i * ldh], lam);
      if (zabs(d) < smin) d = make_double2(smin, 0);
      Y[i + (int64_t)k * n] = zscale(zdiv(acc, d), -1.0);
    }
  }
  __syncthreads();
  // V = Z Y, columns normalised
  for (int t = tid; t < n * n; t += SWG) {
    const int i = t % n, k = t / n;
    c64 acc = make_double2(0, 0);
    for (int j = 0; j <= k; ++j) acc = zadd(acc, zmul(Z[i + (int64_t)j * n], Y[j + (int64_t)k * n]));
    Vout[i + (int64_t)k * ldv] = acc;
  }
  __syncthreads();
  for (int k = tid; k < n; k += SWG) {
    double s2 = 0;
    for (int i = 0; i < n; ++i) s2 += cabs2<double>(Vout[i + (int64_t)k * ldv]);
    const double inv = (s2 > 0) ? 1.0 / sqrt(s2) : 0.0;
    for (int i = 0; i < n; ++i) Vout[i + (int64_t)k * ldv] = zscale(Vout[i + (int64_t)k * ldv], inv);
  }
}

// The same decomposition for n <= 64 by one wavefront, H and Z in LDS: a rotation of the QR sweep
// needs no barrier (the next one's pair comes from two lanes' registers), and the subdiagonal is
// scanned for small entries by all lanes at once instead of by one.  The eigenvectors of the
// triangular factor take its free lower triangle.  Bound by the chain of a rotation.  Order 20: 0.37 ms;
// 0.86 in the kernel above, mostly one thread's scan and two workgroup barriers per rotation.
__global__ void __launch_bounds__(64) k_eig_wave(int32_t n, const c64* Hin, int32_t ldh, c64* w, c64* Vout,
                                                 int32_t ldv, int32_t* info) {
  extern __shared__ __align__(16) unsigned char ew_smem[];
  const int ld = n | 1, lane = threadIdx.x;   // odd: rows and columns are read without bank conflicts
  c64* H = reinterpret_cast<c64*>(ew_smem);
  c64* Z = H + ld * n;
  c64* sv = Z + ld * n;
  const bool row = lane < n;
  for (int j = 0; j < n; ++j)
    if (row) {
      H[lane + j * ld] = Hin[lane + (int64_t)j * ldh];
      Z[lane + j * ld] = make_double2(lane == j ? 1.0 : 0.0, 0.0);
    }
  __syncthreads();   // one wave: orders the LDS accesses
  // --- Householder reduction to upper Hessenberg form
  for (int k = 0; k + 2 < n; ++k) {
    const bool in = row && lane > k;
    c64 v = in ? H[lane + k * ld] : make_double2(0, 0);
    const double nx2 = wave_sum_dpp(cabs2<double>(v));
    const double nx = sqrt(nx2);
    if (nx == 0.0) continue;
    const c64 x0 = make_double2(lane_of(v.x, k + 1), lane_of(v.y, k + 1));
    const double a0 = sqrt(cabs2<double>(x0));
    const c64 ph = a0 > 0 ? make_double2(x0.x / a0, x0.y / a0) : make_double2(1, 0);
    const double inv = 1.0 / sqrt(2.0 * (nx2 + nx * a0));   // 1 / |x - alpha e1|, alpha = -ph nx
    if (lane == k + 1) v = zadd(v, zscale(ph, nx));
    v = zscale(v, inv);
    sv[lane] = v;
    __syncthreads();
    if (row && lane >= k) {   // left, lane = column
      c64 d = make_double2(0, 0);
      for (int i = k + 1; i < n; ++i) d = zadd(d, zmulc(sv[i], H[i + lane * ld]));
      d = zscale(d, 2.0);
      for (int i = k + 1; i < n; ++i) H[i + lane * ld] = zsub(H[i + lane * ld], zmul(sv[i], d));
    }
    __syncthreads();
    if (row) {   // right, lane = row of H and of Z
      c64 d = make_double2(0, 0), e = d;
      for (int j = k + 1; j < n; ++j) {
        d = zadd(d, zmul(H[lane + j * ld], sv[j]));
        e = zadd(e, zmul(Z[lane + j * ld], sv[j]));
      }
      d = zscale(d, 2.0);
      e = zscale(e, 2.0);
      for (int j = k + 1; j < n; ++j) {
        H[lane + j * ld] = zsub(H[lane + j * ld], zmul(d, zconj(sv[j])));
        Z[lane + j * ld] = zsub(Z[lane + j * ld], zmul(e, zconj(sv[j])));
      }
    }
    __syncthreads();
    if (row && lane > k + 1) H[lane + k * ld] = make_double2(0, 0);
    __syncthreads();
  }
  // --- shifted QR (full Schur form)
  const double eps = 2.220446049250313e-16;
  int hi = n - 1, iter = 0, total = 0;
  while (hi >= 0) {
    // the last small subdiagonal entry at or above row hi opens the active window [lo, hi]
    bool small = false;
    if (lane >= 1 && lane <= hi) {
      const double sd = sqrt(cabs2<double>(H[lane + (lane - 1) * ld]));
      const double dd = sqrt(cabs2<double>(H[lane + lane * ld])) + sqrt(cabs2<double>(H[lane - 1 + (lane - 1) * ld]));
      small = sd <= eps * dd || sd < 1e-300;
    }
    const unsigned long long m = __ballot(small);
    const int lo = m ? 63 - __clzll(m) : 0;
    if (lo > 0 && lane == 0) H[lo + (lo - 1) * ld] = make_double2(0, 0);
    __syncthreads();
    if (lo == hi) {
      --hi;
      iter = 0;
      continue;
    }
    if (++total > 60 * n) {
      if (lane == 0) info[0] = 1;   // QR failed to converge
      break;
    }
    c64 mu;
    {
      const c64 a = H[hi - 1 + (hi - 1) * ld], b = H[hi - 1 + hi * ld], c = H[hi + (hi - 1) * ld], d = H[hi + hi * ld];
      if (iter > 0 && iter % 11 == 0) {
        mu = zadd(d, make_double2(0.75 * zabs(c), 0.0));   // exceptional shift
      } else {
        const c64 hd = zscale(zsub(a, d), 0.5);
        const c64 disc = zsqrt(zadd(zmul(hd, hd), zmul(b, c)));
        const c64 m1 = zadd(zscale(zadd(a, d), 0.5), disc), m2 = zsub(zscale(zadd(a, d), 0.5), disc);
        const bool first = cabs2<double>(zsub(m1, d)) < cabs2<double>(zsub(m2, d));
        mu = make_double2(first ? m1.x : m2.x, first ? m1.y : m2.y);
      }
    }
    ++iter;
    c64 x = zsub(H[lo + lo * ld], mu), y = H[lo + 1 + lo * ld];
    for (int k = lo; k < hi; ++k) {
      // G = [[c, s], [-conj(s), c]], c real, G [x; y] = [r; 0]
      const double nx2 = cabs2<double>(x), ny2 = cabs2<double>(y);
      double c;
      c64 s;
      if (ny2 == 0.0) {
        c = 1.0;
        s = make_double2(0, 0);
      } else if (nx2 == 0.0) {
        c = 0.0;
        s = zscale(zconj(y), 1.0 / sqrt(ny2));
      } else {
        const double inv = rsqrt1(nx2) * rsqrt1(nx2 + ny2);
        c = nx2 * inv;
        s = zscale(zmul(x, zconj(y)), inv);
      }
      const int j0 = (k > lo) ? k - 1 : lo;
      if (row && lane >= j0) {   // rows k, k + 1, lane = column
        const c64 hk = H[k + lane * ld], hk1 = H[k + 1 + lane * ld];
        H[k + lane * ld] = zadd(zscale(hk, c), zmul(s, hk1));
        H[k + 1 + lane * ld] = zsub(zscale(hk1, c), zmul(zconj(s), hk));
      }
      __syncthreads();
      const int rmax = min(k + 2, hi);
      c64 nk = make_double2(0, 0);
      if (lane <= rmax) {   // columns k, k + 1 of H, lane = row
        const c64 mk = H[lane + k * ld], mk1 = H[lane + (k + 1) * ld];
        nk = zadd(zscale(mk, c), zmul(zconj(s), mk1));
        H[lane + k * ld] = nk;
        H[lane + (k + 1) * ld] = zsub(zscale(mk1, c), zmul(s, mk));
      }
      if (row) {
        const c64 mk = Z[lane + k * ld], mk1 = Z[lane + (k + 1) * ld];
        Z[lane + k * ld] = zadd(zscale(mk, c), zmul(zconj(s), mk1));
        Z[lane + (k + 1) * ld] = zsub(zscale(mk1, c), zmul(s, mk));
      }
      // the next rotation's pair: rows k + 1 and k + 2 of column k
      x = make_double2(lane_of(nk.x, k + 1), lane_of(nk.y, k + 1));
      const int l2 = min(k + 2, 63);
      y = make_double2(lane_of(nk.x, l2), lane_of(nk.y, l2));
      __syncthreads();
    }
  }
  __syncthreads();
  const c64 lam = row ? H[lane + lane * ld] : make_double2(0, 0);
  if (row) w[lane] = lam;
  // --- eigenvectors of the triangular T = H: T y = lam_k y, y_k = 1, lane = k; Y[j][k] in H[k + j ld]
  double tnorm = 0;
  for (int j = 0; j < n; ++j) {
    if (row && lane <= j) tnorm = fmax(tnorm, cabs2<double>(H[lane + j * ld]));
  }
  tnorm = sqrt(wave_max_dpp(tnorm));
  const double smin = fmax(eps * tnorm, 1e-300);
  for (int i = n - 2; i >= 0; --i) {
    if (row && lane > i) {
      c64 acc = H[i + lane * ld];
      for (int j = i + 1; j < lane; ++j) acc = zadd(acc, zmul(H[i + j * ld], H[lane + j * ld]));
      c64 d = zsub(H[i + i * ld], lam);
      if (sqrt(cabs2<double>(d)) < smin) d = make_double2(smin, 0);
      H[lane + i * ld] = zscale(zdiv(acc, d), -1.0);
    }
    __syncthreads();
  }
  // V = Z Y, columns normalised, lane = row
  for (int k = 0; k < n; ++k) {
    c64 acc = make_double2(0, 0);
    if (row) {
      acc = Z[lane + k * ld];
      for (int j = 0; j < k; ++j) acc = zadd(acc, zmul(Z[lane + j * ld], H[k + j * ld]));
    }
    const double s2 = wave_sum_dpp(cabs2<double>(acc));
    const double inv = s2 > 0 ? 1.0 / sqrt(s2) : 0.0;
    if (row) Vout[lane + (int64_t)k * ldv] = zscale(acc, inv);
  }
}

int32_t eig(cbs_system* s, int32_t n, c64* H, int32_t ldh, c64* w, c64* V, int32_t ldv, int32_t* info_dev,
            hipStream_t st) {
  if (n <= 0) return CBS_OK;
  if (n > 512) {
    set_error("eig: order %d above 512", n);
    return CBS_EINVAL;
  }
  if (n <= 64) {
    CBS_HIP(hipFuncSetAttribute((const void*)k_eig_wave, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SV_LDS));
    const size_t smem = ((size_t)2 * (n | 1) * n + 64) * sizeof(c64);
    hipLaunchKernelGGL(k_eig_wave, dim3(1), dim3(64), smem, st, n, (const c64*)H, ldh, w, V, ldv, info_dev);
    CBS_HIP(hipGetLastError());
    return CBS_OK;
  }
  c64* Z = nullptr;
  c64* Y = nullptr;
  CBS_TRY(ws_get(s->ws, "eig.Z", (size_t)n * n, &Z));
  CBS_TRY(ws_get(s->ws, "eig.Y", (size_t)n * n, &Y));
  hipLaunchKernelGGL(k_eig, dim3(1), dim3(SWG), 0, st, n, H, ldh, w, V, ldv, Z, Y, info_dev);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

// sigma (descending), perm and the right singular vectors W of A (kept): column perm[r] of W
// belongs to sigma[r].  hermitian: A is Hermitian positive definite.  nbatch matrices lda n apart (W:
// ldw n, sigma: 1024, perm: 512) take the time of one: a matrix is a workgroup or a few (order 64,
// six matrices: 0.85 ms, one after the other 5.0).
int32_t svd_right(cbs_system* s, int32_t n, const c64* A, int32_t lda, c64* W, int32_t ldw, double* sigma,
                  int32_t* perm, bool hermitian, int32_t nbatch, hipStream_t st) {
  if (n <= 0 || nbatch <= 0) return CBS_OK;
  if (n > 256) {
    set_error("svd: order %d above 256", n);
    return CBS_EINVAL;
  }
  constexpr int MAXS = SV_SWEEPS, BATCH = 6;
  int limit = MAXS;   // CBS_SVD_SWEEPS=<n>: at most n sweeps (a test of what a factorisation that needs more reports)
  if (const char* e = getenv("CBS_SVD_SWEEPS")) limit = std::max(1, std::min(atoi(e), MAXS));
  c64* X = nullptr;
  int32_t* piv = nullptr;
  unsigned long long* flags = nullptr;
  CBS_TRY(ws_get(s->ws, "svd.X", (size_t)nbatch * n * n, &X));
  CBS_TRY(ws_get(s->ws, "svd.piv", (size_t)nbatch * (n + 1), &piv));
  CBS_TRY(ws_get(s->ws, "svd.flag", (size_t)nbatch * MAXS, &flags));
  if (hermitian) {
    if (nbatch != 1) {
      set_error("svd_right: Hermitian matrices come one at a time");
      return CBS_EINVAL;
    }
    hipLaunchKernelGGL(k_svd_copy, dim3((n * n + 255) / 256), dim3(256), 0, st, n, A, lda, X, piv);
    CBS_HIP(hipGetLastError());
  } else {
    if (n <= 64)
      hipLaunchKernelGGL(k_svd_qr<1>, dim3(1, nbatch), dim3(256), 0, st, n, A, lda, X, piv);
    else if (n <= 128)
      hipLaunchKernelGGL(k_svd_qr<2>, dim3(1, nbatch), dim3(512), 0, st, n, A, lda, X, piv);
    else {
      c64* M = nullptr;
      CBS_TRY(ws_get(s->ws, "svd.M", (size_t)nbatch * n * n, &M));
      hipLaunchKernelGGL(k_svd_qr_big<4>, dim3(1, nbatch), dim3(SV_T), 0, st, n, A, lda, M, X, piv);
    }
    CBS_HIP(hipGetLastError());
  }
  // column blocks of bs, a pair of them in LDS: two (all columns) up to order 64; 32 columns up to
  // order 128, 16 beyond
  const int bs = n <= 64 ? (n + 1) / 2 : n <= 128 ? 32 : 16;
  int nb = (n + bs - 1) / bs;
  nb += nb & 1;
  // lanes of a column pair: four rows a lane; fewer lanes make long chains, more lanes repeat the
  // rotation angles in more waves (order 64, ten sweeps: two rows 0.75 ms, four 0.64, eight 0.76)
  int gsize = 8;
  while (gsize * 4 < n) gsize <<= 1;
  const int threads = (bs * gsize + 63) / 64 * 64;
  const size_t smem = (size_t)2 * bs * sv_ldc(n) * sizeof(c64);
  const int rpl = (n + gsize - 1) / gsize;
  const void* cols = rpl == 1 ? (const void*)k_svd_cols<1> : rpl == 2 ? (const void*)k_svd_cols<2> : (const void*)k_svd_cols<4>;
  CBS_HIP(hipFuncSetAttribute(cols, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SV_LDS));
  auto sweep_launch = [&](int32_t round, int32_t sweep, int32_t sweeps) -> int32_t {
    int32_t bs_ = bs, nb_ = nb, gs_ = gsize;
    void* args[] = {&n, &bs_, &nb_, &round, &sweep, &sweeps, &gs_, &X, &flags};
    CBS_HIP(hipLaunchKernel(cols, dim3(nb / 2, nbatch), dim3(threads), args, smem, st));
    return CBS_OK;
  };
  hipLaunchKernelGGL(k_svd_clear, dim3(1), dim3(64), 0, st, nbatch * MAXS, flags);
  CBS_HIP(hipGetLastError());
  int sweeps = 0;
  if (nb == 2) {
    CBS_TRY(sweep_launch(0, 0, limit));
  } else {
    for (int s0 = 0; s0 < limit; s0 += BATCH) {
      const int s1 = std::min(s0 + BATCH, limit);
      for (int sw = s0; sw < s1; ++sw)
        for (int r = 0; r < nb - 1; ++r) CBS_TRY(sweep_launch(r, sw, 1));
      std::vector<unsigned long long> h((size_t)nbatch * MAXS);
      CBS_HIP(hipMemcpyAsync(h.data(), flags, h.size() * sizeof(h[0]), hipMemcpyDeviceToHost, st));
      CBS_HIP(hipStreamSynchronize(st));
      bool done = true;
      for (int b = 0; b < nbatch; ++b) {
        bool one = false;
        for (int k = s0; k < s1 && !one; ++k) {
          double om = 0;
          std::memcpy(&om, &h[(size_t)b * MAXS + k], sizeof(om));
          sweeps = std::max(sweeps, k + 1);
          one = !(om >= SV_TOL2);
        }
        done = done && one;
      }
      if (done) break;
    }
  }
  if (const char* v = getenv("CBS_VERBOSE"))
    if (v[0] == '3') fprintf(stderr, "[cbs] svd: order %d, %d blocks of %d, %d sweeps\n", n, nb, bs, sweeps);
  hipLaunchKernelGGL(k_svd_right, dim3(1, nbatch), dim3(SV_T), 0, st, n, (const c64*)X, (const int32_t*)piv, W, ldw, sigma,
                     perm, (const unsigned long long*)flags, nb == 2 ? 0 : limit - 1);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

int32_t svd(int32_t n, c64* A, int32_t lda, c64* V, int32_t ldv, double* sigma, int32_t* perm, hipStream_t st) {
  if (n <= 0) return CBS_OK;
  if (n > 512) {
    set_error("svd: order %d above 512", n);
    return CBS_EINVAL;
  }
  if (n < 4 || getenv("CBS_SVD_SINGLE")) {
    hipLaunchKernelGGL(k_jacobi_svd, dim3(1), dim3(JWG), 0, st, n, A, lda, V, ldv, sigma, perm, 60);
    CBS_HIP(hipGetLastError());
    return CBS_OK;
  }
  // block size: the pair's 2 bs columns of A and W in at most 128 KB of LDS, at least 2
  // blocks; an odd block count gets a padding block
  int bs = 1;
  while (bs * 2 * (int64_t)n * 2 * 2 * sizeof(c64) <= BJ_LDS && bs * 2 * 2 <= n) bs *= 2;
  int nb = (n + bs - 1) / bs;
  nb += nb & 1;
  unsigned long long* flag = nullptr;
  CBS_HIP(hipMalloc(&flag, sizeof(unsigned long long)));
  struct Free {
    unsigned long long* p;
    ~Free() { (void)hipFree(p); }
  } fr{flag};
  hipLaunchKernelGGL(k_svd_init, dim3(std::min(1024, (n * n + 255) / 256)), dim3(256), 0, st, n, V, ldv, flag);
  CBS_HIP(hipGetLastError());
  int sweeps = 0;
  for (int sweep = 0; sweep < 60; ++sweep) {
    for (int r = 0; r < nb - 1; ++r) {
      hipLaunchKernelGGL(k_svd_block, dim3(nb / 2), dim3(BJ_THREADS), 0, st, n, bs, nb, r, A, lda, V, ldv, flag);
      CBS_HIP(hipGetLastError());
    }
    unsigned long long h = 0;
    CBS_HIP(hipMemcpyAsync(&h, flag, sizeof(h), hipMemcpyDeviceToHost, st));
    CBS_HIP(hipStreamSynchronize(st));
    double om = 0;
    std::memcpy(&om, &h, sizeof(om));
    sweeps = sweep + 1;
    if (!(om >= 1e-13)) break;   // converged (or nothing rotated)
    CBS_HIP(hipMemsetAsync(flag, 0, sizeof(unsigned long long), st));
  }
  if (const char* v = getenv("CBS_VERBOSE"))
    if (v[0] == '3') fprintf(stderr, "[cbs] svd: order %d, %d blocks of %d, %d sweeps\n", n, nb, bs, sweeps);
  hipLaunchKernelGGL(k_svd_finish, dim3(1), dim3(JWG), 0, st, n, A, lda, sigma, perm);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

// ------------------------------------------------------------------ LU solve
// B := A^{-1} B for n x n A (destroyed) and nrhs columns, partial pivoting.
__global__ void __launch_bounds__(SWG) k_lu_solve(int32_t n, c64* A, int32_t lda, c64* B, int32_t ldb,
                                                   int32_t nrhs, int32_t* info) {
  __shared__ double sh[SWG / 64];
  __shared__ int sidx[SWG / 64];
  __shared__ int piv;
  const int tid = threadIdx.x;
  for (int k = 0; k < n; ++k) {
    // pivot search
    double best = -1;
    int bi = k;
    for (int i = k + tid; i < n; i += SWG) {
      const double v = zabs(A[i + (int64_t)k * lda]);
      if (v > best) {
        best = v;
        bi = i;
      }
    }
    for (int o = 1; o < 64; o <<= 1) {
      const double ob = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ob > best || (ob == best && oi < bi)) {
        best = ob;
        bi = oi;
      }
    }
    if ((tid & 63) == 0) {
      sh[tid >> 6] = best;
      sidx[tid >> 6] = bi;
    }
    __syncthreads();
    if (tid == 0) {
      double b = sh[0];
      int ii = sidx[0];
      for (int w = 1; w < SWG / 64; ++w)
        if (sh[w] > b || (sh[w] == b && sidx[w] < ii)) {
          b = sh[w];
          ii = sidx[w];
        }
      piv = ii;
      if (b == 0.0) info[0] = 2;   // singular
    }
    __syncthreads();
    const int p = piv;
    if (p != k) {
      for (int j = tid; j < n + nrhs; j += SWG) {
        c64* M = (j < n) ? A : B;
        const int col = (j < n) ? j : j - n;
        const int ld = (j < n) ? lda : ldb;
        const c64 t = M[k + (int64_t)col * ld];
        M[k + (int64_t)col * ld] = M[p + (int64_t)col * ld];
        M[p + (int64_t)col * ld] = t;
      }
    }
    __syncthreads();
    const c64 d = A[k + (int64_t)k * lda];
    const bool ok = zabs(d) > 0;
    for (int i = k + 1 + tid; i < n; i += SWG)
      A[i + (int64_t)k * lda] = ok ? zdiv(A[i + (int64_t)k * lda], d) : make_double2(0, 0);
    __syncthreads();
    // trailing update of A and B
    const int cols = (n - k - 1) + nrhs;
    const int rows = n - k - 1;
    for (int t = tid; t < rows * cols; t += SWG) {
      const int i = k + 1 + t % rows;
      const int cj = t / rows;
      c64* M;
      int col, ld;
      if (cj < n - k - 1) {
        M = A;
        col = k + 1 + cj;
        ld = lda;
      } else {
        M = B;
        col = cj - (n - k - 1);
        ld = ldb;
      }
      M[i + (int64_t)col * ld] = zsub(M[i + (int64_t)col * ld], zmul(A[i + (int64_t)k * lda], M[k + (int64_t)col * ld]));
    }
    __syncthreads();
  }
  // back substitution U x = y, one right-hand side per thread
  for (int c = tid; c < nrhs; c += SWG) {
    for (int i = n - 1; i >= 0; --i) {
      c64 acc = B[i + (int64_t)c * ldb];
      for (int j = i + 1; j < n; ++j) acc = zsub(acc, zmul(A[i + (int64_t)j * lda], B[j + (int64_t)c * ldb]));
      const c64 d = A[i + (int64_t)i * lda];
      B[i + (int64_t)c * ldb] = (zabs(d) > 0) ? zdiv(acc, d) : make_double2(0, 0);
    }
  }
}

int32_t lu_solve(int32_t n, c64* A, int32_t lda, c64* B, int32_t ldb, int32_t nrhs, int32_t* info_dev,
                 hipStream_t st) {
  if (n <= 0) return CBS_OK;
  hipLaunchKernelGGL(k_lu_solve, dim3(1), dim3(SWG), 0, st, n, A, lda, B, ldb, nrhs, info_dev);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

// ------------------------------------------------------------------ Cholesky + inverse
// G = R^H R (upper R), Rinv = R^{-1} (upper); G destroyed.  shift times the trace is added to
// the diagonal first (shifted Cholesky QR).
__global__ void __launch_bounds__(SWG) k_chol_inv(int32_t n, c64* G, int32_t ldg, double shift, c64* Rinv,
                                                   int32_t* info) {
  const int tid = threadIdx.x;
  double tr = 0;
  for (int i = 0; i < n && shift != 0; ++i) tr += G[i + (int64_t)i * ldg].x;
  shift *= tr;
  __syncthreads();
  for (int i = tid; i < n; i += SWG) G[i + (int64_t)i * ldg].x += shift;
  __syncthreads();
  // right-looking: for k, R[k][k] = sqrt(G[k][k]); R[k][j] = G[k][j]/R[k][k]; G[i][j] -= conj(R[k][i]) R[k][j]
  for (int k = 0; k < n; ++k) {
    const double d = G[k + (int64_t)k * ldg].x;
    const double r = (d > 0) ? sqrt(d) : 0.0;
    if (tid == 0 && !(d > 0)) info[0] = 3;
    __syncthreads();
    for (int j = k + 1 + tid; j < n; j += SWG)
      G[k + (int64_t)j * ldg] = (r > 0) ? zscale(G[k + (int64_t)j * ldg], 1.0 / r) : make_double2(0, 0);
    __syncthreads();
    if (tid == 0) G[k + (int64_t)k * ldg] = make_double2(r, 0);
    const int m = n - k - 1;
    for (int t = tid; t < m * m; t += SWG) {
      const int i = k + 1 + t % m, j = k + 1 + t / m;
      if (i <= j)
        G[i + (int64_t)j * ldg] = zsub(G[i + (int64_t)j * ldg], zmulc(G[k + (int64_t)i * ldg], G[k + (int64_t)j * ldg]));
    }
    __syncthreads();
  }
  // inverse of the upper triangle, one column per thread
  for (int c = tid; c < n; c += SWG) {
    for (int i = n - 1; i >= 0; --i) {
      c64 acc = make_double2(i == c ? 1.0 : 0.0, 0.0);
      for (int j = i + 1; j <= c; ++j) acc = zsub(acc, zmul(G[i + (int64_t)j * ldg], Rinv[j + (int64_t)c * n]));
      const double d = G[i + (int64_t)i * ldg].x;
      Rinv[i + (int64_t)c * n] = (i > c) ? make_double2(0, 0) : ((d > 0) ? zscale(acc, 1.0 / d) : make_double2(0, 0));
    }
  }
}

// The same for n up to CI_NMAX by one elimination in LDS, one barrier a row: G = L D L^H with unit
// lower L; the row operations that clear G below the diagonal turn the identity into L^-1, and
// R^-1 = (D^{-1/2} L^-1)^H.  The upper triangle of M holds what is left of G, the strict lower one
// L^-1.  A row's chain (pivot, reciprocal, one update, a barrier) bounds it: 9.7 us for n = 16 (the
// kernel above takes 29), 24 for 32, 57 for 64, 157 for 96 (97 above: 936).
constexpr int CI_NMAX = 96;
template <int TX>
__global__ void __launch_bounds__(TX == 32 ? 256 : 1024) k_chol_inv_lds(int32_t n, const c64* G, int32_t ldg,
                                                                        double shift, c64* Rinv, int32_t* info) {
  extern __shared__ __align__(16) unsigned char ci_smem[];
  c64* M = reinterpret_cast<c64*>(ci_smem);   // [n][n]
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX, TY = blockDim.x / TX;
  for (int t = threadIdx.x; t < n * n; t += blockDim.x) {
    const int j = t / n, i = t - j * n;
    const c64 v = G[i + (int64_t)j * ldg];
    M[i * n + j] = (i <= j) ? v : make_double2(0, 0);
  }
  __syncthreads();
  if (shift != 0) {
    double tr = 0;
    for (int i = 0; i < n; ++i) tr += M[i * n + i].x;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) M[i * n + i].x += shift * tr;
    __syncthreads();
  }
  for (int k = 0; k < n; ++k) {
    const c64* row = M + k * n;
    const double d = row[k].x;
    const double inv = (d > 0) ? 1.0 / d : 0.0;
    if (threadIdx.x == 0 && !(d > 0)) info[0] = 3;
    for (int i = k + 1 + ty; i < n; i += TY) {
      const c64 l = make_double2(row[i].x * inv, -row[i].y * inv);
      for (int j = tx; j < n; j += TX) {
        if (j > k && j < i) continue;
        c64* m = M + i * n + j;
        *m = (j == k) ? make_double2(-l.x, -l.y) : zsub(*m, zmul(l, row[j]));
      }
    }
    __syncthreads();
  }
  for (int t = threadIdx.x; t < n * n; t += blockDim.x) {
    const int c = t / n, i = t - c * n;   // R^-1[i][c], i <= c
    const double d = M[c * n + c].x;
    const double f = (d > 0) ? 1.0 / sqrt(d) : 0.0;
    c64 v = make_double2(0, 0);
    if (i < c) v = make_double2(M[c * n + i].x * f, -M[c * n + i].y * f);
    if (i == c) v = make_double2(f, 0);
    Rinv[t] = v;
  }
}

int32_t chol_inv(int32_t n, c64* G, int32_t ldg, double shift, c64* Rinv, int32_t* info_dev, hipStream_t st) {
  if (n <= 0) return CBS_OK;
  const size_t smem = (size_t)n * n * sizeof(c64);
  if (n <= 32) {
    hipLaunchKernelGGL((k_chol_inv_lds<32>), dim3(1), dim3(256), smem, st, n, (const c64*)G, ldg, shift, Rinv,
                       info_dev);
  } else if (n <= CI_NMAX) {
    CBS_HIP(hipFuncSetAttribute((const void*)k_chol_inv_lds<64>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                CI_NMAX * CI_NMAX * (int)sizeof(c64)));
    hipLaunchKernelGGL((k_chol_inv_lds<64>), dim3(1), dim3(1024), smem, st, n, (const c64*)G, ldg, shift, Rinv,
                       info_dev);
  } else {
    hipLaunchKernelGGL(k_chol_inv, dim3(1), dim3(SWG), 0, st, n, G, ldg, shift, Rinv, info_dev);
  }
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

}  // namespace cbs
