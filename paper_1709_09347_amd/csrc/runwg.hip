// BiCG on small cells: one workgroup carries one run (a system and its dual) through all of its
// iterations.
//
// The launch-per-step iteration of bicg.hip costs its launches: on an 8x8x12 cell a stencil pass of
// 256 runs takes a few microseconds and the fifteen launches of an iteration take fifty.  A run's
// recurrences need nothing from other runs, so where its search direction fits the LDS of one CU
// a workgroup keeps p there and r (and x) in registers; the operator, the projectors and the inner
// products are barriers apart instead of launches apart.  The recurrences, the tests on the
// residuals, the residual replacement and the restart are those of k_s1, k_s2 and k_s3 in the
// complex128 phase; the sums are added in another order.  A launch takes at most `cap` iterations
// of every run and leaves what is unfinished in global memory for the next.
#include <algorithm>
#include <cstdlib>

#include "bicg.hpp"
#include "cbs_internal.hpp"

namespace cbs {

struct WgArgs {
  int32_t nx, ny, nz, N, nruns, L, n_atoms, nnz, start, cap, max_iter, max_ru, hstride, hrows;
  double kin, tol, div_factor;
  double c[5];
  const double* vloc;
  const double2* V;
  const double2* Vd;
  const RunCoef* coef;
  const double* vref;
  BicgScal sc;
  Pair<double>* R;
  Pair<double>* Pg;   // direction between launches, and during a replacement
  Pair<double>* X;
  Pair<double>* Y;
  double* hist;
  const int32_t* seg;
  const int32_t* idx;
  const double* u;
  const double* coeff;
  const int32_t* pt_off;
  const int32_t* pt_key;
  const double* pt_u;
};

// LDS of a run: the direction (primal and dual planes apart, so that a wave's reads are
// conflict-free), per atom the bra sums and the ket coefficients, the partial sums of the waves.
constexpr int WG_RED = 2 * 16 * 4;   // [buffer][wave][value]
static size_t wg_lds_bytes(int64_t N, int32_t n_atoms) {
  return (size_t)N * 32 + (size_t)n_atoms * (48 + 48) * sizeof(double) + WG_RED * sizeof(double);
}
// and, where they fit as well, the potential and the projectors' tables, which every iteration reads
// again: from LDS a bra or ket step is not a trip to L2
static size_t wg_table_bytes(int64_t N, int64_t nnz) {
  return (size_t)N * 8 + (size_t)nnz * 2 * (32 + 4) + (size_t)(N + 1) * 4;
}

// A value that is the same in every lane, in scalar registers (lane 0's).
__device__ __forceinline__ double uni(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ double2 uni(double2 v) { return make_double2(uni(v.x), uni(v.y)); }

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The sums of NV values over the workgroup, the same in every thread: 16 lanes by DPP (a shuffle
// through LDS takes ten times as long, and an iteration waits for two of these chains), then the
// four rows of a wave, then the waves in order.
template <int NV>
__device__ __forceinline__ void wg_sum(double (&v)[NV], double* red, int lane, int wv, int nw) {
  auto row16 = [](double t) {
    t += dpp<0xB1>(t);    // lane ^ 1
    t += dpp<0x4E>(t);    // lane ^ 2
    t += dpp<0x141>(t);   // mirrored in 8 lanes
    t += dpp<0x140>(t);   // mirrored in 16 lanes
    return t;
  };
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double t = row16(v[k]);
    v[k] = (lane_value(t, 0) + lane_value(t, 16)) + (lane_value(t, 32) + lane_value(t, 48));
  }
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wv * 4 + k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = lane_value(row16(lane < nw ? red[lane * 4 + k] : 0.0), 0);
}

// A thread owns NPT points, T apart.  What it needs of a point every iteration (its neighbours'
// places in LDS, its addresses) is worked out anew each time: kept, it would take 30 registers a
// point and spill.  r, q (and x of a single point) fit 128 registers at 1024 threads for one or two
// points, 256 at 512 threads for eight.
template <int P, int NPT, bool HP, bool TAB>
__global__ void __launch_bounds__(NPT <= 2 ? 1024 : 512) k_run_wg(WgArgs a) {
  extern __shared__ __align__(16) unsigned char wg_smem[];
  constexpr bool XREG = NPT == 1;   // x in registers, else in global memory
  const int run = blockIdx.x;
  if (!a.start && a.sc.status[run] != ST_ACT_HI) return;
  const int N = a.N, nx = a.nx, ny = a.ny, nz = a.nz, plane = nx * ny;
  double2* pa = reinterpret_cast<double2*>(wg_smem);
  double2* pb = pa + N;
  double* G = reinterpret_cast<double*>(pb + N);                            // [atom][shift][16]
  Pair<double>* kt = reinterpret_cast<Pair<double>*>(G + 48 * a.n_atoms);   // [atom][shift][4]
  double* red = reinterpret_cast<double*>(kt + 12 * a.n_atoms);
  // TAB: the tables in LDS (ball_u, pt_u, vloc, ball_idx, pt_key, pt_off)
  double4* t_u = reinterpret_cast<double4*>(red + WG_RED);
  double4* t_pu = t_u + a.nnz;
  double* t_v = reinterpret_cast<double*>(t_pu + a.nnz);
  int32_t* t_idx = reinterpret_cast<int32_t*>(t_v + N);
  int32_t* t_key = t_idx + a.nnz;
  int32_t* t_off = t_key + a.nnz;
  int tid = threadIdx.x;
  const int T = blockDim.x, lane = tid & 63, nw = T >> 6;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const RunCoef& cf = a.coef[run];
  const double2 cpa = cf.c[1], cma = cf.c[2], cpb = cf.c[4], cmb = cf.c[5];   // P(z): c0 = 1
  const double2* V = a.V + (int64_t)(run % a.L) * N;
  const double2* Vd = a.Vd + (int64_t)(run % a.L) * N;
  const int64_t base = (int64_t)run * N;
  double2 ra[NPT], rb[NPT], xa[NPT], xb[NPT];
  uint32_t pos[NPT];   // ix | iy << 8 | iz << 20
#pragma unroll
  for (int k = 0; k < NPT; ++k) {
    const int n = min(tid + k * T, N - 1), z = n / plane, t = n - z * plane, y = t / nx;
    pos[k] = (uint32_t)(t - y * nx) | (uint32_t)y << 8 | (uint32_t)z << 20;
    xa[k] = xb[k] = make_double2(0, 0);
  }
  auto valid = [&](int k) { return tid + k * T < N; };
  // --- state
  double2 rho, rho_prev, beta = make_double2(0, 0);
  double vn2, rr = 0, rrt = 0, rmin;
  int it = 0, nru = 0, brk = 0, ru_it = 0, nrestart = 0, status = ST_ACT_HI;
  if (a.start) {
    double s[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const int n = tid + k * T;
      ra[k] = rb[k] = make_double2(0, 0);
      if (!valid(k)) continue;
      ra[k] = V[n];
      rb[k] = Vd[n];
      pa[n] = pb[n] = make_double2(0, 0);
      if (!XREG) a.X[base + n] = Pair<double>{make_double2(0, 0), make_double2(0, 0)};
      const double2 t = cmulc<double>(rb[k], ra[k]);
      s[0] += t.x;
      s[1] += t.y;
      s[2] += cabs2<double>(ra[k]);
      s[3] += cabs2<double>(rb[k]);
    }
    wg_sum<4>(s, red + 64, lane, wv, nw);
    rho = rho_prev = make_double2(s[0], s[1]);
    vn2 = (a.vref != nullptr && a.vref[run] > 0) ? a.vref[run] : s[2];
    // a zero right-hand side is solved by zero; a non-finite one is not "zero" and ends in a
    // breakdown at the first scalar test
    const bool zero = s[2] == 0.0 && s[3] == 0.0;
    rr = zero ? 0.0 : (vn2 > 0 ? sqrt(s[2] / vn2) : 1.0);
    rrt = zero ? 0.0 : (vn2 > 0 ? sqrt(s[3] / vn2) : 1.0);
    rmin = uni(fmax(rr, rrt));
    if (zero) {
      status = ST_DONE;
#pragma unroll
      for (int k = 0; k < NPT; ++k)
        if (valid(k)) a.Y[base + tid + k * T] = Pair<double>{make_double2(0, 0), make_double2(0, 0)};
    }
  } else {
    rho = a.sc.rho[run];
    rho_prev = a.sc.rho_prev[run];
    beta = a.sc.beta[run];
    vn2 = a.sc.vn2[run];
    rmin = a.sc.rmin[run];
    rr = a.sc.relres[2 * run];
    rrt = a.sc.relres[2 * run + 1];
    it = a.sc.iters[run];
    nru = a.sc.nru[run];
    ru_it = a.sc.ru_it[run];
    nrestart = a.sc.nrestart[run];
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const int n = min(tid + k * T, N - 1);
      const Pair<double> r = a.R[base + n], p = a.Pg[base + n];
      ra[k] = r.a;
      rb[k] = r.b;
      if (XREG) {
        const Pair<double> x = a.X[base + n];
        xa[k] = x.a;
        xb[k] = x.b;
      }
      if (valid(k)) {
        pa[n] = p.a;
        pb[n] = p.b;
      }
    }
  }
  if (TAB && status == ST_ACT_HI) {   // the first barrier of an iteration comes before their use
    for (int e = tid; e < a.nnz; e += T) {
      t_u[e] = reinterpret_cast<const double4*>(a.u)[e];
      t_pu[e] = reinterpret_cast<const double4*>(a.pt_u)[e];
      t_idx[e] = a.idx[e];
      t_key[e] = a.pt_key[e];
    }
    for (int n = tid; n < N; n += T) t_v[n] = a.vloc[n];
    for (int n = tid; n <= N; n += T) t_off[n] = a.pt_off[n];
  }
  // --- iterations (repl = false) and residual replacements (repl = true)
  bool repl = false;
  int steps = 0;
  while (status == ST_ACT_HI) {
    asm volatile("" : "+v"(tid));   // what follows from them is not kept across iterations
#pragma unroll
    for (int k = 0; k < NPT; ++k) asm volatile("" : "+v"(pos[k]));
    if (!repl) {
      if (steps == a.cap) break;
      ++steps;
#pragma unroll
      for (int k = 0; k < NPT; ++k) {
        const int n = tid + k * T;
        if (!valid(k)) continue;
        const double2 oa = pa[n], ob = pb[n];
        pa[n] = make_double2(fma(-beta.y, oa.y, fma(beta.x, oa.x, ra[k].x)), fma(beta.y, oa.x, fma(beta.x, oa.y, ra[k].y)));
        pb[n] = make_double2(fma(beta.y, ob.y, fma(beta.x, ob.x, rb[k].x)), fma(-beta.y, ob.x, fma(beta.x, ob.y, rb[k].y)));
      }
    } else {
      // y += x, x = 0; the operator is applied to y, the direction waits in global memory
#pragma unroll
      for (int k = 0; k < NPT; ++k) {
        const int n = tid + k * T;
        if (!valid(k)) continue;
        Pair<double> x;
        if (XREG) x = Pair<double>{xa[k], xb[k]};
        else x = a.X[base + n];
        if (nru > 0) {
          const Pair<double> y = a.Y[base + n];
          x.a = cadd<double>(y.a, x.a);
          x.b = cadd<double>(y.b, x.b);
        }
        a.Y[base + n] = x;
        a.Pg[base + n] = Pair<double>{pa[n], pb[n]};
        pa[n] = x.a;
        pb[n] = x.b;
        xa[k] = xb[k] = make_double2(0, 0);
        if (!XREG) a.X[base + n] = Pair<double>{make_double2(0, 0), make_double2(0, 0)};
      }
    }
    __syncthreads();
    if (HP && a.n_atoms > 0) {
      // bra: a wave per (atom, cell shift), lanes over the ball's entries
      for (int un = wv; un < 3 * a.n_atoms; un += nw) {
        const int atom = un / 3, sg = un - 3 * atom;
        const int lo = a.seg[4 * atom + sg], hi = a.seg[4 * atom + sg + 1];
        double acc[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = 0;
        // two entries a step, their table reads in flight together; past the end weighted by zero
        for (int e0 = lo + lane; e0 < hi; e0 += 128) {
          double4 uu[2];
          int n[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int e = min(e0 + 64 * q, hi - 1);
            uu[q] = TAB ? t_u[e] : reinterpret_cast<const double4*>(a.u)[e];
            n[q] = TAB ? t_idx[e] : a.idx[e];
          }
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const double on = e0 + 64 * q < hi ? 1.0 : 0.0;
            const double2 va = pa[n[q]], vb = pb[n[q]];
            const double us[4] = {on * uu[q].x, on * uu[q].y, on * uu[q].z, on * uu[q].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              acc[4 * i] += us[i] * va.x;
              acc[4 * i + 1] += us[i] * va.y;
              acc[4 * i + 2] += us[i] * vb.x;
              acc[4 * i + 3] += us[i] * vb.y;
            }
          }
        }
        double t = 0;
        if (lo < hi) t = wave_sums<16, double>(acc, lane);
        if ((lane & 3) == 0) G[16 * un + (lane >> 2)] = t;
      }
      __syncthreads();
      // K[w][i] = h_ai z^-w sum_w' z^w' G[w'][i] (dual: 1/conj z)
      for (int t = tid; t < 24 * a.n_atoms; t += T) {
        const int half = t & 1, i = (t >> 1) & 3, w = (t >> 3) % 3, atom = t / 24;
        const double* g = G + 48 * atom + 4 * i + 2 * half;
        const double2 zp = make_double2(half ? cpb.x : cpa.x, half ? cpb.y : cpa.y);
        const double2 zm = make_double2(half ? cmb.x : cma.x, half ? cmb.y : cma.y);
        double2 s = cmul<double>(zm, make_double2(g[0], g[1]));
        s = cadd<double>(s, make_double2(g[16], g[17]));
        s = cadd<double>(s, cmul<double>(zp, make_double2(g[32], g[33])));
        if (w == 0) s = cmul<double>(zp, s);
        if (w == 2) s = cmul<double>(zm, s);
        reinterpret_cast<double2*>(kt + 12 * atom + 4 * w + i)[half] = cscale<double>(s, a.coeff[4 * atom + i]);
      }
      __syncthreads();
    }
    double2 qa[NPT], qb[NPT];
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const int n = min(tid + k * T, N - 1);
      const int ix = pos[k] & 255, iy = (pos[k] >> 8) & 4095, iz = pos[k] >> 20;
      const double vd = (TAB ? t_v[n] : a.vloc[n]) - cf.E;
      const double2 va = pa[n], vb = pb[n];
      double2 sa = cscale<double>(va, 3.0 * a.c[0]), sb = cscale<double>(vb, 3.0 * a.c[0]);
      double2 ua = make_double2(0, 0), ub = ua, da = ua, db = ua;   // from the cells above and below
#pragma unroll
      for (int j = 1; j <= P; ++j) {
        const double cj = a.c[j];
        const int l = n - j + (ix < j ? nx : 0), r = n + j - (ix + j >= nx ? nx : 0);
        const int d = n - j * nx + (iy < j ? plane : 0), u = n + j * nx - (iy + j >= ny ? plane : 0);
        sa = cfma_r<double>(sa, cj, cadd<double>(cadd<double>(pa[l], pa[r]), cadd<double>(pa[d], pa[u])));
        sb = cfma_r<double>(sb, cj, cadd<double>(cadd<double>(pb[l], pb[r]), cadd<double>(pb[d], pb[u])));
        const bool lo = iz < j, hi = iz + j >= nz;
        const int zd = n - j * plane + (lo ? N : 0), zu = n + j * plane - (hi ? N : 0);
        if (lo) {
          da = cfma_r<double>(da, cj, pa[zd]);
          db = cfma_r<double>(db, cj, pb[zd]);
        } else {
          sa = cfma_r<double>(sa, cj, pa[zd]);
          sb = cfma_r<double>(sb, cj, pb[zd]);
        }
        if (hi) {
          ua = cfma_r<double>(ua, cj, pa[zu]);
          ub = cfma_r<double>(ub, cj, pb[zu]);
        } else {
          sa = cfma_r<double>(sa, cj, pa[zu]);
          sb = cfma_r<double>(sb, cj, pb[zu]);
        }
      }
      sa = cfma<double>(cfma<double>(sa, cpa, ua), cma, da);
      sb = cfma<double>(cfma<double>(sb, cpb, ub), cmb, db);
      sa = cfma_r<double>(cscale<double>(sa, a.kin), vd, va);
      sb = cfma_r<double>(cscale<double>(sb, a.kin), vd, vb);
      if (HP && a.n_atoms > 0) {
        const int e1 = TAB ? t_off[n + 1] : a.pt_off[n + 1];
        for (int e = TAB ? t_off[n] : a.pt_off[n]; e < e1; e += 2) {
          // two entries a step, their table reads in flight together
          const int f = min(e + 1, e1 - 1);
          const int32_t* keys = TAB ? t_key : a.pt_key;
          const double4* ptu = TAB ? t_pu : reinterpret_cast<const double4*>(a.pt_u);
          const int key[2] = {keys[e], keys[f]};
          const double4 uu[2] = {ptu[e], ptu[f]};
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            if (e + q >= e1) break;
            const Pair<double>* kk = kt + 12 * (key[q] >> 2) + 4 * (key[q] & 3);
            const double us[4] = {uu[q].x, uu[q].y, uu[q].z, uu[q].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              sa = cfma_r<double>(sa, us[i], kk[i].a);
              sb = cfma_r<double>(sb, us[i], kk[i].b);
            }
          }
        }
      }
      qa[k] = sa;
      qb[k] = sb;
    }
    if (!repl) {
      double sg[2] = {0, 0};
#pragma unroll
      for (int k = 0; k < NPT; ++k)
        if (valid(k)) {
          const double2 t = cmulc<double>(pb[tid + k * T], qa[k]);
          sg[0] += t.x;
          sg[1] += t.y;
        }
      wg_sum<2>(sg, red, lane, wv, nw);
      if (!(sg[0] != 0.0 || sg[1] != 0.0) || !isfinite(sg[0]) || !isfinite(sg[1])) {
        brk = 1;
        repl = true;
        continue;
      }
      const double2 al = uni(cdiv<double>(rho, make_double2(sg[0], sg[1]))), alc = cconj<double>(al);
      double s[4] = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < NPT; ++k) {
        const int n = tid + k * T;
        if (!valid(k)) continue;
        if (XREG) {
          xa[k] = cfma<double>(xa[k], al, pa[n]);
          xb[k] = cfma<double>(xb[k], alc, pb[n]);
        } else {
          Pair<double> x = a.X[base + n];
          x.a = cfma<double>(x.a, al, pa[n]);
          x.b = cfma<double>(x.b, alc, pb[n]);
          a.X[base + n] = x;
        }
        ra[k] = csub<double>(ra[k], cmul<double>(al, qa[k]));
        rb[k] = csub<double>(rb[k], cmul<double>(alc, qb[k]));
        const double2 t = cmulc<double>(rb[k], ra[k]);
        s[0] += t.x;
        s[1] += t.y;
        s[2] += cabs2<double>(ra[k]);
        s[3] += cabs2<double>(rb[k]);
      }
      wg_sum<4>(s, red + 64, lane, wv, nw);
      ++it;
      rr = uni(sqrt(s[2] / vn2));
      rrt = uni(sqrt(s[3] / vn2));
      if (a.hist != nullptr && tid == 0 && it % a.hstride == 0 && it / a.hstride <= a.hrows) {
        const int64_t at = ((int64_t)(it / a.hstride - 1) * a.nruns + run) * 2;
        a.hist[at] = rr;
        a.hist[at + 1] = rrt;
      }
      const double2 rn = make_double2(s[0], s[1]);
      const bool conv = rr < a.tol && rrt < a.tol;
      const bool bad = !(rn.x != 0.0 || rn.y != 0.0) || !isfinite(rn.x) || !isfinite(rn.y) || !isfinite(rr) || !isfinite(rrt);
      if (bad && !conv) brk = 1;
      beta = bad ? make_double2(0, 0) : uni(cdiv<double>(rn, rho));
      rho_prev = rho;
      rho = rn;
      const double cur = fmax(rr, rrt);
      rmin = uni(fmin(rmin, cur));
      repl = conv || bad || it >= a.max_iter || (it - ru_it >= 20 && cur > a.div_factor * rmin);
    } else {
      double s[4] = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < NPT; ++k) {
        const int n = tid + k * T;
        if (!valid(k)) continue;
        ra[k] = csub<double>(V[n], qa[k]);
        rb[k] = csub<double>(Vd[n], qb[k]);
        const double2 t = cmulc<double>(rb[k], ra[k]);
        s[0] += t.x;
        s[1] += t.y;
        s[2] += cabs2<double>(ra[k]);
        s[3] += cabs2<double>(rb[k]);
      }
      wg_sum<4>(s, red + 64, lane, wv, nw);
      rr = uni(sqrt(s[2] / vn2));
      rrt = uni(sqrt(s[3] / vn2));
      ++nru;
      ru_it = it;
      rmin = uni(fmax(rr, rrt));
      repl = false;
      const double2 rn = make_double2(s[0], s[1]);
      if (rr < a.tol && rrt < a.tol) {
        status = ST_DONE;
      } else if (brk || !isfinite(rn.x) || !isfinite(rn.y) || !(rn.x != 0.0 || rn.y != 0.0)) {
        status = ST_BREAKDOWN;
      } else if (it >= a.max_iter || nru >= a.max_ru) {
        status = ST_NOCONV;
      } else {
        beta = uni(cdiv<double>(rn, rho_prev));
        rho = rn;
        const bool restart = rmin > 100.0 * a.tol;   // see k_s3
        if (restart) {
          beta = make_double2(0, 0);
          ++nrestart;
        }
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
          const int n = tid + k * T;
          if (!valid(k)) continue;
          const Pair<double> p = a.Pg[base + n];
          pa[n] = restart ? make_double2(0, 0) : p.a;
          pb[n] = restart ? make_double2(0, 0) : p.b;
        }
      }
    }
  }
  if (status == ST_ACT_HI) {
    // out of iterations in this launch: the next one goes on from here
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const int n = tid + k * T;
      if (!valid(k)) continue;
      a.R[base + n] = Pair<double>{ra[k], rb[k]};
      a.Pg[base + n] = Pair<double>{pa[n], pb[n]};
      if (XREG) a.X[base + n] = Pair<double>{xa[k], xb[k]};
    }
  }
  if (tid == 0) {
    a.sc.rho[run] = rho;
    a.sc.rho_prev[run] = rho_prev;
    a.sc.beta[run] = beta;
    a.sc.vn2[run] = vn2;
    a.sc.rmin[run] = rmin;
    a.sc.relres[2 * run] = rr;
    a.sc.relres[2 * run + 1] = rrt;
    a.sc.iters[run] = it;
    a.sc.nru[run] = nru;
    a.sc.ru_it[run] = ru_it;
    a.sc.nrestart[run] = nrestart;
    a.sc.status[run] = status;
  }
}

// Unfinished runs: n_active[0] = 0, n_active[1] = their number (what the host's poll reads).
__global__ void __launch_bounds__(256) k_wg_count(BicgScal sc, int32_t nruns) {
  __shared__ int cnt[4];
  int c = 0;
  for (int r = threadIdx.x; r < nruns; r += 256) c += sc.status[r] == ST_ACT_HI ? 1 : 0;
  c = wsum<int>(c);
  if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    sc.n_active[0] = 0;
    sc.n_active[1] = cnt[0] + cnt[1] + cnt[2] + cnt[3];
  }
}

// Points a thread, and whether the tables go to LDS (*tab).  A run at a time is quickest with a point
// a thread; past a run per CU two points a thread let a second run share the CU (8x8x12, 672 ball
// entries, microseconds per iteration of 512 runs: 15.8, one point 17.9; 256 runs 11.3 and 9.8), if
// need be with the tables left in L2 (8x8x16, 512 runs: 16.1, one point 20.3, two with the tables in
// LDS and so one run per CU 20.0).  One run or 256: 9.4 and 9.8 with the tables in LDS, 10.4 and 10.8
// from L2.
static int wg_points(const cbs_system* s, int32_t nruns, bool* tab) {
  const size_t own = wg_lds_bytes(s->N, s->proj.n_atoms), tables = wg_table_bytes(s->N, s->proj.nnz);
  *tab = s->proj.n_atoms > 0 && own + tables <= 160 * 1024;
  if (s->N > 1024) return s->N <= 2048 ? 2 : 8;
  const int64_t waves1 = (s->N + 63) / 64, waves2 = (s->N + 127) / 128;
  if (nruns > 256 && 2 * waves1 > 16 && 2 * waves2 <= 16 && 2 * own <= 160 * 1024) {
    *tab = *tab && 2 * (own + tables) <= 160 * 1024;
    return 2;
  }
  return 1;
}

// The cells of this path: p must fit the LDS beside the projectors' sums (4096 points at most), a
// neighbour is one wrap away, and the balls must be few enough that a workgroup walks them faster
// than the other path shares them between runs.  Microseconds per iteration (launch per step /
// workgroup per run): 8x8x12, 256 runs 44 / 7; with 672 ball entries 62 / 10; 16x16x16, 256 runs
// 84 / 27, 512 runs 140 / 55; with 15,704 entries (3.8 a point) 116 / 73 and 203 / 147, one run
// 83 / 60, so that the lines meet near 8 entries a point.
bool run_wg_fits(const cbs_system* s) {
  for (const char* e : {"CBS_BRA_TILE", "CBS_BRA_NW", "CBS_BRA_SPREAD", "CBS_NO_MFMA", "CBS_NO_GRAPH"})
    if (getenv(e) != nullptr) return false;   // these choose among the kernels of the other path
  const char* e = getenv("CBS_RUN_WG");
  if (e && e[0] == '0') return false;
  return s->nx >= s->p && s->ny >= s->p && s->ny < 4096 && s->nz < 4096 && s->N <= 4096 &&
         s->proj.nnz <= 8 * s->N && wg_lds_bytes(s->N, s->proj.n_atoms) <= 160 * 1024;
}

template <int P, bool HP, bool TAB>
static const void* wg_kernel(int npt) {
  return npt == 1 ? (const void*)k_run_wg<P, 1, HP, TAB> : npt == 2 ? (const void*)k_run_wg<P, 2, HP, TAB> : (const void*)k_run_wg<P, 8, true, TAB>;
}
// (Eight points always take the kernel with projectors: without the ket's loop between them the
// scheduler interleaves the points' LDS reads, and 290 registers spill: 45 us an iteration for 24.)
template <int P>
static const void* wg_kernel(int npt, bool hp, bool tab) {
  return !hp ? wg_kernel<P, false, false>(npt) : tab ? wg_kernel<P, true, true>(npt) : wg_kernel<P, true, false>(npt);
}

int32_t launch_run_wg(BicgSolve& b, bool start, int32_t cap, hipStream_t st) {
  const cbs_system* s = b.sys;
  WgArgs a;
  a.nx = s->nx;
  a.ny = s->ny;
  a.nz = s->nz;
  a.N = (int32_t)s->N;
  a.nruns = b.nruns;
  a.L = b.L;
  a.n_atoms = s->proj.n_atoms;
  a.nnz = (int32_t)s->proj.nnz;
  a.start = start;
  a.cap = cap;
  a.max_iter = b.max_iter;
  a.max_ru = b.max_ru;
  a.hstride = b.hist_stride;
  a.hrows = b.hist_rows;
  a.kin = -0.5 / (s->h * s->h);
  a.tol = b.tol;
  a.div_factor = b.div_factor;
  for (int i = 0; i < 5; ++i) a.c[i] = s->fd[i];
  a.vloc = s->vloc64;
  a.V = b.V;
  a.Vd = b.Vd ? b.Vd : b.V;
  a.coef = b.coef;
  a.vref = b.vn2_ref;
  a.sc = b.sc;
  a.R = b.hi.R;
  a.Pg = b.hi.Pb[0];
  a.X = b.hi.X;
  a.Y = b.Y;
  a.hist = b.hist;
  a.seg = s->proj.seg;
  a.idx = s->proj.ball_idx;
  a.u = s->proj.ball_u64;
  a.coeff = s->proj.coeff64;
  a.pt_off = s->proj.pt_off;
  a.pt_key = s->proj.pt_key;
  a.pt_u = s->proj.pt_u64;
  bool tab = false;
  const int npt = wg_points(s, b.nruns, &tab);
  const int nthr = (int)(((s->N + npt - 1) / npt + 63) / 64 * 64);
  size_t smem = wg_lds_bytes(s->N, s->proj.n_atoms);
  const bool hp = a.n_atoms > 0;
  if (tab) smem += wg_table_bytes(s->N, s->proj.nnz);
  const void* f = s->p == 1 ? wg_kernel<1>(npt, hp, tab) : s->p == 2 ? wg_kernel<2>(npt, hp, tab) : s->p == 3 ? wg_kernel<3>(npt, hp, tab) : wg_kernel<4>(npt, hp, tab);
  // always the most a cell can ask for: the attribute is the kernel's, not the launch's, and another
  // thread may be launching it for another cell
  CBS_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
  void* args[] = {&a};
  CBS_HIP(hipLaunchKernel(f, dim3(b.nruns), dim3(nthr), args, smem, st));
  hipLaunchKernelGGL(k_wg_count, dim3(1), dim3(256), 0, st, b.sc, b.nruns);
  CBS_HIP(hipGetLastError());
  return CBS_OK;
}

}  // namespace cbs
