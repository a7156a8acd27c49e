// The operator on vector-major blocks: y_v = c0_v (H0 - E) x_v + cp_v H+ x_v + cm_v H- x_v
// (P(z): 1, z, 1/z) for cbs_apply, cbs_apply_noalloc, cbs_apply_parts, the bands' filter, the
// Rayleigh-Ritz projections and the adjoint.
//
// Three parts read the caller's x and write its y, with no staging copy of either; the
// coefficients travel as kernel arguments (64 vectors a call), so nothing is copied from the
// host and nothing has to outlive the launch:
//   ap_bra      K[atom][w][i] = h_ai sum_w' coef(w' - w) sum_e u_{e,i} x(idx_e)
//   k_ap_local  y = finite differences, potential and cell phases of x (+ beta prev)
//   k_ap_ket    y += sum_i u_{e,i} K[a_e][w_e][i], on the matrix cores, over the 64-point
//               groups that lie in a ball
// The bra is a launch of its own or the first workgroups of the local part's (bra_shape); the
// smallest cells take all three in one (k_ap_cell).
// The BiCG kernels (stencil.hip, nonlocal.hip) keep a run's primal and dual side by side; here
// a vector stands alone, which halves the registers of the z queue and lets a cell be cut into
// z segments until the chip is full.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "apply_shape.hpp"
#include "cbs_internal.hpp"

namespace cbs {

constexpr int AP_VMAX = 64;   // vectors per launch (their coefficients: 3 KB of kernel arguments)
constexpr int AP_VG = 8;      // vectors per ket group: 16 MFMA columns (re, im)

struct ApCoef {
  double2 c0[AP_VMAX], cp[AP_VMAX], cm[AP_VMAX];
};

template <typename R> struct apmf4;
template <> struct apmf4<double> { typedef double T __attribute__((ext_vector_type(4))); };
template <> struct apmf4<float> { typedef float T __attribute__((ext_vector_type(4))); };
__device__ __forceinline__ apmf4<double>::T ap_mfma(double a, double b, apmf4<double>::T c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ apmf4<float>::T ap_mfma(float a, float b, apmf4<float>::T c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------ bra
template <typename R>
struct ApBra {
  int32_t n_atoms, nv, nvb, nlogical;
  int32_t nsub;   // items (an atom and its vectors) per workgroup, four waves each; further waves leave
  int32_t grid;   // with the local part: the launch's first workgroups
  int64_t N;
  const int32_t* seg;
  const int32_t* idx;
  const R* u;       // [nnz][4]
  const R* coeff;   // [n_atoms][4]
  const cplx<R>* x;
  R* kt;            // per group of AP_VG vectors: [atom * 3 + w][i][2 * vectors of the group]
};

// Four waves an item, an atom and VB vectors; a thread takes every 256th ball entry (one table read
// for VB coalesced gathers) and the sums of each cell shift are added over the lanes and waves.  The
// 4 projectors would fill a quarter of an MFMA tile, and the vector units have the same FP64 rate.
// Bound by the gathers that miss L2 (overlapping balls; consecutive workgroups of an XCD share
// the vectors): 48x48x32, 96 atoms, 32 vectors: 38 us in complex128, 24 in complex64, where one
// MFMA workgroup per (atom, 16 pairs) took 145 and 194; with 512 threads 45 us, with the atoms'
// vectors side by side on an XCD 46 us.
template <typename R, typename C, int VB>
__device__ __forceinline__ void ap_bra(const ApBra<R>& a, const ApCoef& cf, unsigned char* smem) {
  const int nsub = a.nsub;
  const int sub = threadIdx.x >> 8, tid = threadIdx.x & 255, lane = tid & 63, wv = tid >> 6;
  const int lb = remap_active(blockIdx.x, a.nlogical);
  if (lb < 0 || sub >= nsub) return;
  C(*red)[3][8 * VB] = reinterpret_cast<C(*)[3][8 * VB]>(smem) + 4 * sub;   // [wave][shift][(vector, i, re/im)]
  const int item = min(lb * nsub + sub, a.n_atoms * a.nvb - 1);   // the last workgroup may repeat the last one
  const int vb = item / a.n_atoms, atom = item - vb * a.n_atoms;
  const int v0 = vb * VB;
  using U4 = typename vec4<R>::T;
  const U4* ut = reinterpret_cast<const U4*>(a.u);
  const cplx<R>* xv[VB];
#pragma unroll
  for (int k = 0; k < VB; ++k) xv[k] = a.x + (int64_t)min(v0 + k, a.nv - 1) * a.N;
  for (int sg = 0; sg < 3; ++sg) {
    const int lo = a.seg[4 * atom + sg], hi = a.seg[4 * atom + sg + 1];
    C acc[8 * VB];
#pragma unroll
    for (int k = 0; k < 8 * VB; ++k) acc[k] = 0;
    // two entries a step; their gathers go out together with the next step's indices; loads past
    // the segment are clamped into it and weighted by zero
    const int last = max(hi - 1, lo);
    int n0 = 0, n1 = 0;
    if (lo < hi) {
      n0 = a.idx[min(lo + tid, last)];
      n1 = a.idx[min(lo + 256 + tid, last)];
    }
    for (int e0 = lo; e0 < hi; e0 += 512) {
      const int ea = e0 + tid, eb = ea + 256;
      const U4 ua = ut[min(ea, last)], ub = ut[min(eb, last)];
      cplx<R> ta[VB], tb[VB];
#pragma unroll
      for (int k = 0; k < VB; ++k) ta[k] = xv[k][n0];
#pragma unroll
      for (int k = 0; k < VB; ++k) tb[k] = xv[k][n1];
      n0 = a.idx[min(ea + 512, last)];
      n1 = a.idx[min(eb + 512, last)];
      const C oa = ea < hi ? (C)1 : (C)0, ob = eb < hi ? (C)1 : (C)0;
      const C wa[4] = {oa * (C)ua.x, oa * (C)ua.y, oa * (C)ua.z, oa * (C)ua.w};
      const C wb[4] = {ob * (C)ub.x, ob * (C)ub.y, ob * (C)ub.z, ob * (C)ub.w};
#pragma unroll
      for (int k = 0; k < VB; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[8 * k + 2 * i] += wa[i] * (C)ta[k].x;
          acc[8 * k + 2 * i + 1] += wa[i] * (C)ta[k].y;
        }
#pragma unroll
      for (int k = 0; k < VB; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[8 * k + 2 * i] += wb[i] * (C)tb[k].x;
          acc[8 * k + 2 * i + 1] += wb[i] * (C)tb[k].y;
        }
    }
    C t = 0;
    if (lo < hi) t = wave_sums<8 * VB, C>(acc, lane);   // uniform over the workgroup
    if ((lane & (64 / (8 * VB) - 1)) == 0) red[wv][sg][lane / (64 / (8 * VB))] = t;
  }
  __syncthreads();
  // wave k: the 12 coefficients of vector v0 + k
  const int k = __builtin_amdgcn_readfirstlane(wv), v = v0 + k;
  if (k >= VB || v >= a.nv || lane >= 12) return;
  const int w = lane >> 2, i = lane & 3, q = 8 * k + 2 * i;
  const double2 d0 = cf.c0[v], dp = cf.cp[v], dm = cf.cm[v];
  cplx<C> s = mkc<C>(0, 0);
#pragma unroll
  for (int w2 = 0; w2 < 3; ++w2) {
    const int d = w2 - w;   // cell shift of the source relative to the entry
    if (d > 1 || d < -1) continue;
    const cplx<C> cd = mkc<C>((C)(d == 0 ? d0.x : d == 1 ? dp.x : dm.x), (C)(d == 0 ? d0.y : d == 1 ? dp.y : dm.y));
    const cplx<C> g = mkc<C>(red[0][w2][q] + red[1][w2][q] + red[2][w2][q] + red[3][w2][q],
                             red[0][w2][q + 1] + red[1][w2][q + 1] + red[2][w2][q + 1] + red[3][w2][q + 1]);
    s = cfma<C>(s, cd, g);
  }
  s = cscale<C>(s, (C)a.coeff[4 * atom + i]);
  const int vg = v / AP_VG, ncol = 2 * min(AP_VG, a.nv - vg * AP_VG);
  R* dst = a.kt + (int64_t)vg * a.n_atoms * 12 * 2 * AP_VG + ((int64_t)(atom * 3 + w) * 4 + i) * ncol +
           2 * (v - vg * AP_VG);
  dst[0] = (R)s.x;
  dst[1] = (R)s.y;
}

template <typename R, typename C, int VB>
__global__ void __launch_bounds__(256) k_ap_bra(ApBra<R> a, ApCoef cf) {
  __shared__ __align__(16) unsigned char smem[4 * 3 * 8 * VB * sizeof(C)];
  ap_bra<R, C, VB>(a, cf, smem);
}

// ------------------------------------------------------------------ local part
template <typename R>
struct ApLocal {
  int32_t nx, ny, nz, ty, ntiles, nseg, zlen, nlogical, nbuf;
  int64_t N;
  double kin, E, beta;
  double c[5], zc[5];   // second-derivative weights, and the same times kin
  const R* vloc;
  const double* vloc64;
  const cplx<R>* x;
  const cplx<R>* prev;   // or NULL
  cplx<R>* y;
};

// One workgroup: one vector, TY full x rows, z planes [z0, z1).  The owned planes are staged in
// LDS for the x and y neighbours (next plane's loads in flight while this one is computed); the
// p planes on either side are read for the owned column only, all at once.  Every thread keeps
// the 2p+1 partial outputs of its column in registers, so a plane is read once for the z
// direction.  R: storage, C: arithmetic precision.  Bound by HBM on large cells: 96x96x32, 24
// complex128 vectors without projectors, 66 us for 226 MB (3.4 TB/s); the pair kernel with its two
// layout passes took 200 us.  48x48x32, 32 vectors: 24 us (was 111 + 37 us of layout passes).
// PIPE: every thread stages at most two elements of a plane; ADD: beta prev is added.
template <typename R, typename C, int P, bool PIPE, bool ADD, int VB>
__global__ void __launch_bounds__(1024) k_ap_local(ApLocal<R> a, ApBra<R> b, ApCoef cf) {
  extern __shared__ __align__(16) unsigned char ap_smem[];
  if constexpr (VB > 0) {
    if ((int)blockIdx.x < b.grid) {
      ap_bra<R, C, VB>(b, cf, ap_smem);
      return;
    }
  }
  cplx<R>* lds = reinterpret_cast<cplx<R>*>(ap_smem);
  const int lb = remap_active(blockIdx.x - (VB > 0 ? b.grid : 0), a.nlogical);
  if (lb < 0) return;
  const int per = a.ntiles * a.nseg;
  const int v = lb / per;
  const int rem = lb - v * per;
  const int seg = rem / a.ntiles;
  const int tile = rem - seg * a.ntiles;
  const int z0 = seg * a.zlen, z1 = min(z0 + a.zlen, a.nz);
  if (z0 >= z1) return;
  const int nx = a.nx, ny = a.ny, nz = a.nz, TY = a.ty;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int tx = tid % nx, ty = tid / nx;
  const int y = tile * TY + ty;
  const bool own = ty < TY && y < ny;
  const int64_t plane = (int64_t)nx * ny;
  const int region = (TY + 2 * P) * nx;
  const int col = own ? tx + nx * y : 0;
  const cplx<R>* xv = a.x + (int64_t)v * a.N;
  cplx<R>* yv = a.y + (int64_t)v * a.N;
  const cplx<R>* pv = ADD ? a.prev + (int64_t)v * a.N : nullptr;
  const cplx<C> c0 = ccast<C, double>(cf.c0[v]), cp = ccast<C, double>(cf.cp[v]), cm = ccast<C, double>(cf.cm[v]);
  const C E = (C)a.E, kin = (C)a.kin, beta = (C)a.beta;
  C cc[P + 1], zc[P + 1];
#pragma unroll
  for (int j = 0; j <= P; ++j) {
    cc[j] = (C)a.c[j];
    zc[j] = (C)a.zc[j];
  }
  // staging: offset within a plane of each element this thread brings in
  constexpr int PF = 2;
  const bool pipe = region <= PF * nthr;
  auto plane_off = [&](int e) {
    const int r = e / nx;
    int gy = (tile * TY - P + r) % ny;
    gy += (gy < 0) ? ny : 0;
    return e - r * nx + nx * gy;
  };
  int soff[PF];
#pragma unroll
  for (int k = 0; k < PF; ++k) soff[k] = (tid + k * nthr < region) ? plane_off(tid + k * nthr) : 0;
  R sre[PF] = {}, sim[PF] = {};
  auto issue = [&](int m) {
#pragma unroll
    for (int k = 0; k < PF; ++k) {   // past the region: element 0, not stored
      const cplx<R> t = xv[plane * m + soff[k]];
      sre[k] = t.x;
      sim[k] = t.y;
    }
  };
  // x neighbours within a row of LDS (nx may be smaller than p: several wraps)
  int xl[P], xr[P];
#pragma unroll
  for (int j = 1; j <= P; ++j) {
    int l = tx - j, r = tx + j;
    while (l < 0) l += nx;
    while (r >= nx) r -= nx;
    xl[j - 1] = l;
    xr[j - 1] = r;
  }
  cplx<R> halo[P];
  auto load_halo = [&](int m0) {   // the owned column of planes m0 .. m0 + P - 1 (wrapped into the cell)
#pragma unroll
    for (int j = 0; j < P; ++j) {
      int iz = m0 + j;
      iz += (iz < 0) ? nz : 0;
      iz -= (iz >= nz) ? nz : 0;
      halo[j] = xv[plane * iz + col];
    }
  };
  cplx<C> acc[2 * P + 1];
#pragma unroll
  for (int d = 0; d <= 2 * P; ++d) acc[d] = mkc<C>(0, 0);
  // plane m contributes s to outputs m - P .. m + P; output m - P is then complete
  auto push = [&](int m, cplx<C> s, cplx<C> in_plane) {
    const int o = m - P;
    const int64_t at = plane * max(o, z0) + col;
    cplx<R> add;
    if constexpr (ADD) add = pv[at];
    acc[P] = cadd<C>(acc[P], in_plane);
#pragma unroll
    for (int d = 0; d <= 2 * P; ++d) acc[d] = cfma_r<C>(acc[d], zc[d > P ? d - P : P - d], s);
    if (own && o >= z0) {
      cplx<C> out = acc[0];
      if constexpr (ADD) out = cfma_r<C>(out, beta, ccast<C, R>(add));
      yv[at] = ccast<R, C>(out);
    }
#pragma unroll
    for (int d = 0; d < 2 * P; ++d) acc[d] = acc[d + 1];
    acc[2 * P] = mkc<C>(0, 0);
  };
  auto phase = [&](int m, cplx<C> s) {
    const C re = m < 0 ? cm.x : m >= nz ? cp.x : c0.x, im = m < 0 ? cm.y : m >= nz ? cp.y : c0.y;
    return cmul<C>(mkc<C>(re, im), s);
  };

  auto pot = [&](int m) { return (sizeof(C) == 8) ? (C)a.vloc64[plane * m + col] : (C)a.vloc[plane * m + col]; };
  load_halo(z0 - P);
  C vl = pot(z0);
  if constexpr (PIPE) issue(z0);
#pragma unroll
  for (int j = 0; j < P; ++j) push(z0 - P + j, phase(z0 - P + j, ccast<C, R>(halo[j])), mkc<C>(0, 0));
  auto owned = [&](int m, bool last) {
    cplx<R>* buf = lds + ((a.nbuf == 2) ? ((m - z0) & 1) * region : 0);
    if (a.nbuf == 1 && m > z0) __syncthreads();   // single buffer: the previous plane is fully read
    const C vd = vl - E;
    if constexpr (PIPE) {
#pragma unroll
      for (int k = 0; k < PF; ++k)
        if (tid + k * nthr < region) buf[tid + k * nthr] = mkc<R>(sre[k], sim[k]);
    } else {
      for (int e = tid; e < region; e += nthr) buf[e] = xv[plane * m + plane_off(e)];
    }
    if (last) {
      load_halo(z1);
    } else {
      vl = pot(m + 1);
      if constexpr (PIPE) issue(m + 1);
    }
    __syncthreads();
    cplx<C> s = mkc<C>(0, 0), in_plane = s;
    if (own) {
      const int row = (ty + P) * nx;
      const cplx<C> c = ccast<C, R>(buf[row + tx]);
      cplx<C> t = cscale<C>(c, (C)2 * cc[0]);
#pragma unroll
      for (int j = 1; j <= P; ++j) {
        const cplx<C> l = ccast<C, R>(buf[row + xl[j - 1]]), r = ccast<C, R>(buf[row + xr[j - 1]]);
        const cplx<C> d = ccast<C, R>(buf[row - j * nx + tx]), u = ccast<C, R>(buf[row + j * nx + tx]);
        t = cfma_r<C>(t, cc[j], cadd<C>(cadd<C>(l, r), cadd<C>(d, u)));
      }
      t = cfma_r<C>(cscale<C>(t, kin), vd, c);
      in_plane = cmul<C>(c0, t);
      s = cmul<C>(c0, c);
    }
    push(m, s, in_plane);
  };
  for (int m = z0; m < z1 - 1; ++m) owned(m, false);
  owned(z1 - 1, true);
#pragma unroll
  for (int j = 0; j < P; ++j) push(z1 + j, phase(z1 + j, ccast<C, R>(halo[j])), mkc<C>(0, 0));
}

// ------------------------------------------------------------------ ket
template <typename R>
struct ApKet {
  int32_t n_atoms, nv, nvg, nlogical;
  int64_t N;
  const int32_t* grp_off;
  const int32_t* grp_key;
  const int32_t* grp_mask;
  const R* grp_u;
  const R* kt;
  cplx<R>* y;
  // the point's own list, for K that is not finite
  const int32_t* pt_off;
  const int32_t* pt_key;
  const R* pt_u;
};

// The ket at point n of one vector (columns col and col + 1 of its group) over the balls that hold the
// point.
template <typename R, typename C>
__device__ void ap_ket_point(const ApKet<R>& a, int64_t n, int vg, int ncol, int col, C& re, C& im) {
  using U4 = typename vec4<R>::T;
  const R* kt = a.kt + (int64_t)vg * a.n_atoms * 12 * 2 * AP_VG + col;
  re = im = 0;
#pragma nounroll
  for (int e = a.pt_off[n]; e < a.pt_off[n + 1]; ++e) {
    const int key = a.pt_key[e];
    const U4 u = reinterpret_cast<const U4*>(a.pt_u)[e];
    const R* k = kt + (int64_t)((key >> 2) * 3 + (key & 3)) * 4 * ncol;
    const C us[4] = {(C)u.x, (C)u.y, (C)u.z, (C)u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      re += us[i] * (C)k[i * ncol];
      im += us[i] * (C)k[i * ncol + 1];
    }
  }
}

// A workgroup adds the ket of one 64-point group to AP_VG vectors: U [64 points x 4] (grouped
// table) times K [4 x 16 columns] summed over the group's keys with MFMA 16x16x4 in four 16-point
// row blocks (those the key's mask names).  A group in the middle of many balls has sixty keys and
// each batch of them is one memory latency, so the four waves take every fourth key; their
// products are added through LDS in wave order and wave w updates vectors 2w and 2w + 1, lane =
// point.  Groups outside every ball touch nothing.  Where a sum is not finite the point's own list gives
// it, so that a NaN in a ball reaches the points of the balls that hold it and no others of their
// groups.  The vector groups vary fastest: they share a
// group's table slice in one XCD's L2.  48x48x32, 96 atoms, 32 vectors: 31 us in complex128 (the
// vectors and 27 MB of table, 3.3 TB/s; 29 with two groups a workgroup), 24 (21) in complex64; one wave per group 31 and 28, one
// thread per point and pair 115 and 61.
// CB: groups of AP_VG vectors a workgroup (their columns share the table's loads).
template <typename R, typename C, int CB>
__global__ void __launch_bounds__(256) k_ap_ket(ApKet<R> a) {
  constexpr int KB = 2;   // keys per batch (4: one wave less per SIMD, 36 us)
  __shared__ C tile[4][KG][17];
  const int lb = remap_active(blockIdx.x, a.nlogical);
  if (lb < 0) return;
  const int nwg = a.nvg / CB;   // workgroups of a point group
  const int g = lb / nwg, vg0 = (lb - g * nwg) * CB;
  const int e0 = a.grp_off[g], e1 = a.grp_off[g + 1];
  if (e0 == e1) return;   // uniform over the workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the vectors' values are requested first: their latency passes under the contraction
  const int64_t n = (int64_t)g * KG + lane, nc = min(n, a.N - 1);
  const int orow = lane & 15, ok4 = lane >> 4;
  int nvec[CB], ncol[CB];
  cplx<R>* yp[CB];
  cplx<R> y0[CB], y1[CB];
  const R* kcol[CB];
  typename apmf4<C>::T acc[CB][4];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const int vg = vg0 + c;
    nvec[c] = min(AP_VG, a.nv - vg * AP_VG);
    ncol[c] = 2 * nvec[c];
    yp[c] = a.y + (int64_t)vg * AP_VG * a.N + nc;
    y0[c] = yp[c][(int64_t)min(2 * wv, nvec[c] - 1) * a.N];
    y1[c] = yp[c][(int64_t)min(2 * wv + 1, nvec[c] - 1) * a.N];
    kcol[c] = a.kt + (int64_t)vg * a.n_atoms * 12 * 2 * AP_VG + (int64_t)ok4 * ncol[c] + min(orow, ncol[c] - 1);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) acc[c][rb] = {0, 0, 0, 0};
  }
  for (int eb = e0; eb < e1; eb += 256) {
    // lane j holds this wave's key number j: entry eb + 4 j + wv of the group
    const int mine = eb + 4 * lane + wv;
    const int nk = min(64, (e1 - eb - wv + 3) >> 2);
    const int keyv = (mine < e1) ? a.grp_key[mine] : 0;
    const int maskv = (mine < e1) ? a.grp_mask[mine] : 0;
    C kbA[KB][CB], ubA[KB][4], kbB[KB][CB], ubB[KB][4];
    int mA[KB], mB[KB];
    auto load = [&](int j0, C (&kb)[KB][CB], C (&ub)[KB][4], int (&m)[KB]) {
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        const bool valid = j0 + j < nk;   // wave-uniform
        const int jj = valid ? j0 + j : 0;
        const int key = __builtin_amdgcn_readlane(keyv, jj);
        m[j] = valid ? __builtin_amdgcn_readlane(maskv, jj) : 0;
#pragma unroll
        for (int c = 0; c < CB; ++c) kb[j][c] = (C)kcol[c][((key >> 2) * 3 + (key & 3)) * 4 * ncol[c]];
        const R* up = a.grp_u + ((int64_t)(eb + 4 * jj + wv) * KG + orow) * 4 + ok4;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) ub[j][rb] = ((m[j] >> rb) & 1) ? (C)up[64 * rb] : (C)0;
      }
    };
    auto mma = [&](const C (&kb)[KB][CB], const C (&ub)[KB][4], const int (&m)[KB]) {
#pragma unroll
      for (int j = 0; j < KB; ++j)
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
          if ((m[j] >> rb) & 1)
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[c][rb] = ap_mfma(ub[j][rb], kb[j][c], acc[c][rb]);
    };
    load(0, kbA, ubA, mA);
    for (int j0 = 0; j0 < nk; j0 += 2 * KB) {
      load(j0 + KB, kbB, ubB, mB);
      mma(kbA, ubA, mA);
      if (j0 + KB >= nk) break;
      load(j0 + 2 * KB, kbA, ubA, mA);
      mma(kbB, ubB, mB);
    }
  }
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    if (c > 0) __syncthreads();   // the tile of the columns before is read
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) tile[wv][16 * rb + mfma16_row<C>(lane, v)][orow] = acc[c][rb][v];
    __syncthreads();
    if (n >= a.N) continue;
    C t[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      t[q] = ((tile[0][lane][4 * wv + q] + tile[1][lane][4 * wv + q]) + tile[2][lane][4 * wv + q]) +
             tile[3][lane][4 * wv + q];
    // zero table entries take part in the products, and zero times an infinite or undefined K is not zero
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (!((t[2 * h] - t[2 * h]) + (t[2 * h + 1] - t[2 * h + 1]) == (C)0))
        ap_ket_point<R, C>(a, n, vg0 + c, ncol[c], min(4 * wv + 2 * h, ncol[c] - 2), t[2 * h], t[2 * h + 1]);
    if (2 * wv < nvec[c]) yp[c][(int64_t)(2 * wv) * a.N] = mkc<R>((R)((C)y0[c].x + t[0]), (R)((C)y0[c].y + t[1]));
    if (2 * wv + 1 < nvec[c])
      yp[c][(int64_t)(2 * wv + 1) * a.N] = mkc<R>((R)((C)y1[c].x + t[2]), (R)((C)y1[c].y + t[3]));
  }
}

// ------------------------------------------------------------------ small cells
// All three parts by one workgroup a vector, a point a thread, with the vector and the projector
// coefficients in LDS (at most 21 KB): on cells this small the time is the launches' and a chain of
// latencies.  Whole calls in complex128: 5x5x8, 3 atoms, one vector 23.8 -> 20.2 us; 8x8x12, 6 atoms,
// 64 vectors 31.7 -> 22.5.
template <typename R>
struct ApPoint {
  const int32_t* off;
  const int32_t* key;
  const R* u;
};

// LDS: the coefficients [atom][w][i], the vector, the segments' sums [atom][w][i][re, im]
static size_t ap_cell_lds(int64_t N, int32_t n_atoms, size_t elem, size_t real) {
  return (size_t)n_atoms * 24 * real + (size_t)N * elem + (size_t)n_atoms * 24 * real;
}

template <typename R, typename C, int P, bool ADD>
__global__ void __launch_bounds__(1024) k_ap_cell(ApLocal<R> a, ApBra<R> b, ApPoint<R> pt, ApCoef cf) {
  extern __shared__ __align__(16) unsigned char ap_smem[];
  const int N = (int)a.N, na = b.n_atoms, nx = a.nx, ny = a.ny, nz = a.nz;
  cplx<C>* kc = reinterpret_cast<cplx<C>*>(ap_smem);
  cplx<R>* xs = reinterpret_cast<cplx<R>*>(kc + 12 * na);
  C* red = reinterpret_cast<C*>(xs + N);
  const int v = blockIdx.x, tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool own = tid < N;
  const int n = own ? tid : 0;
  const int64_t base = (int64_t)v * N + n;
  const cplx<R> x0 = a.x[base];
  const C vl = (sizeof(C) == 8) ? (C)a.vloc64[n] : (C)a.vloc[n];
  const int e0 = pt.off[n], e1 = own ? pt.off[n + 1] : e0;
  cplx<R> add;
  if constexpr (ADD) add = a.prev[base];
  if (own) xs[n] = x0;
  __syncthreads();
  // bra: a wave per atom and cell shift
  using U4 = typename vec4<R>::T;
  const U4* ut = reinterpret_cast<const U4*>(b.u);
  for (int it = wv; it < 3 * na; it += nthr >> 6) {
    const int atom = it / 3, sg = it - 3 * atom;
    const int lo = b.seg[4 * atom + sg], hi = b.seg[4 * atom + sg + 1];
    C acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0;
    const int last = hi - 1;
    for (int eb = lo; eb < hi; eb += 256) {   // four entries a lane; past the segment: weight zero
      int idx[4];
      U4 u[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = min(eb + 64 * k + lane, last);
        idx[k] = b.idx[e];
        u[k] = ut[e];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const C o = eb + 64 * k + lane < hi ? (C)1 : (C)0;
        const C w[4] = {o * (C)u[k].x, o * (C)u[k].y, o * (C)u[k].z, o * (C)u[k].w};
        const cplx<R> t = xs[idx[k]];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[2 * i] += w[i] * (C)t.x;
          acc[2 * i + 1] += w[i] * (C)t.y;
        }
      }
    }
    C t = 0;
    if (lo < hi) t = wave_sums<8, C>(acc, lane);
    if ((lane & 7) == 0) red[8 * it + (lane >> 3)] = t;
  }
  const cplx<C> c0 = ccast<C, double>(cf.c0[v]), cp = ccast<C, double>(cf.cp[v]), cm = ccast<C, double>(cf.cm[v]);
  // local part at the own point
  const int iz = n / (nx * ny), r = n - iz * nx * ny, iy = r / nx, ix = r - iy * nx;
  const cplx<C> c = ccast<C, R>(x0);
  cplx<C> t = cscale<C>(c, (C)2 * (C)a.c[0]), zs = cscale<C>(cmul<C>(c0, c), (C)a.zc[0]);
  int xl = ix, xr = ix, yd = iy, yu = iy;
#pragma unroll
  for (int j = 1; j <= P; ++j) {
    xl = xl == 0 ? nx - 1 : xl - 1;
    xr = xr == nx - 1 ? 0 : xr + 1;
    yd = yd == 0 ? ny - 1 : yd - 1;
    yu = yu == ny - 1 ? 0 : yu + 1;
    const cplx<C> l = ccast<C, R>(xs[n - ix + xl]), q = ccast<C, R>(xs[n - ix + xr]);
    const cplx<C> d = ccast<C, R>(xs[n + (yd - iy) * nx]), u = ccast<C, R>(xs[n + (yu - iy) * nx]);
    t = cfma_r<C>(t, (C)a.c[j], cadd<C>(cadd<C>(l, q), cadd<C>(d, u)));
    const bool below = iz - j < 0, above = iz + j >= nz;
    const cplx<C> sd = ccast<C, R>(xs[n + ((below ? nz : 0) - j) * nx * ny]);
    const cplx<C> su = ccast<C, R>(xs[n + (j - (above ? nz : 0)) * nx * ny]);
    const cplx<C> pd = mkc<C>(below ? cm.x : c0.x, below ? cm.y : c0.y);
    const cplx<C> pu = mkc<C>(above ? cp.x : c0.x, above ? cp.y : c0.y);
    zs = cfma_r<C>(zs, (C)a.zc[j], cadd<C>(cmul<C>(pd, sd), cmul<C>(pu, su)));
  }
  t = cfma_r<C>(cscale<C>(t, (C)a.kin), vl - (C)a.E, c);
  cplx<C> y = cadd<C>(cmul<C>(c0, t), zs);
  if constexpr (ADD) y = cfma_r<C>(y, (C)a.beta, ccast<C, R>(add));
  __syncthreads();
  for (int q = tid; q < 12 * na; q += nthr) {
    const int atom = q / 12, w = (q - 12 * atom) >> 2, i = q & 3;
    cplx<C> s = mkc<C>(0, 0);
#pragma unroll
    for (int w2 = 0; w2 < 3; ++w2) {
      const int d = w2 - w;   // cell shift of the source relative to the entry
      if (d > 1 || d < -1) continue;
      const C* g = red + 8 * (3 * atom + w2) + 2 * i;
      s = cfma<C>(s, mkc<C>(d == 0 ? c0.x : d == 1 ? cp.x : cm.x, d == 0 ? c0.y : d == 1 ? cp.y : cm.y), mkc<C>(g[0], g[1]));
    }
    kc[q] = cscale<C>(s, (C)b.coeff[4 * atom + i]);
  }
  __syncthreads();
  // ket: four entries' loads at a time; past the point's list: weight zero
  const U4* pu = reinterpret_cast<const U4*>(pt.u);
  for (int eb = e0; eb < e1; eb += 4) {
    int key[4];
    U4 u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = min(eb + k, e1 - 1);
      key[k] = pt.key[e];
      u[k] = pu[e];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const C o = eb + k < e1 ? (C)1 : (C)0;
      const cplx<C>* kk = kc + ((key[k] >> 2) * 3 + (key[k] & 3)) * 4;
      const C w[4] = {o * (C)u[k].x, o * (C)u[k].y, o * (C)u[k].z, o * (C)u[k].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) y = cfma_r<C>(y, w[i], kk[i]);
    }
  }
  if (own) a.y[base] = ccast<R, C>(y);
}

// ------------------------------------------------------------------ launches
// Whether k_ap_cell takes the call.  A point has a thread of its own, and one workgroup walks the
// balls of all atoms, which costs more than the launch it saves when they are many or large (whole
// calls in complex128, one vector, apart and in one: 5x5x8, 3 atoms 23.8 and 20.2 us; 8x8x12, 8 atoms
// with 2100 ball entries 25.5 and 24.8; 10x10x10, 12 atoms with 3200 entries 25.6 both; 8x8x12,
// 20 atoms with 1700 entries 25.7 and 26.4, 40 atoms with 10700 entries 27.9 and 39.5).
static bool ap_cell_fits(const cbs_system* s) {
  return s->N <= 1024 && s->proj.n_atoms > 0 && s->proj.n_atoms <= 12 && s->proj.nnz <= 2560;
}

template <typename R, typename C, int P>
static void ap_cell_p(const ApLocal<R>& a, const ApBra<R>& b, const ApPoint<R>& pt, const ApCoef& cf, int32_t nv,
                      size_t smem, hipStream_t st) {
  const int nthr = std::max(((int)a.N + 63) / 64 * 64, 512);   // eight waves for the bra (256 or 1024: + 2 %)
  if constexpr (sizeof(R) == 8) {
    if (a.prev != nullptr) {
      hipLaunchKernelGGL((k_ap_cell<R, C, P, true>), dim3(nv), dim3(nthr), smem, st, a, b, pt, cf);
      return;
    }
  }
  hipLaunchKernelGGL((k_ap_cell<R, C, P, false>), dim3(nv), dim3(nthr), smem, st, a, b, pt, cf);
}

size_t apply_kt_bytes(const cbs_system* s, int32_t n_vec, size_t real_bytes) {
  const int64_t nv = std::min(n_vec, AP_VMAX);
  return (size_t)nv * s->proj.n_atoms * 24 * real_bytes;
}

// Vectors per bra item, and whether the bra shares the local part's launch: neither reads what the
// other writes, so up to 576 items of two vectors the chip has room for both at once and a launch is
// saved (48x48x32, 96 atoms, 8 complex128 vectors, whole call: 57 us, apart 64; 45x37x29, 60 atoms,
// 8: 42, apart 51; 32x32x24, 40 atoms, 24: 46, apart 57).  Past that the table reads of four
// vectors an item count for more: in complex128 in a launch of its own, where the bra keeps L2 for its
// gathers (48x48x32, 32 vectors: 113, together 125), in complex64 together up to 768 items.  That line
// is a middle one, as the cell counts too (together and apart, us): 32x32x24, 40 atoms, 640 items 54 and
// 56; 48x48x32, 96 atoms, 672 items 66 and 73, 768 items 71 and 76, 864 items 86 and 90, 960 items 98 and
// 91, 1056 items 95 and 102; 64x64x40, 170 atoms, 510 items 67 and 70, 680 items 82 and 77, 850 items 105
// and 98, 1020 items 112 and 107.
static int bra_shape(int32_t n_atoms, int32_t nv, bool f32, bool* together) {
  *together = true;
  if ((int64_t)n_atoms * ((nv + 1) / 2) <= 576) return 2;
  *together = f32 && (int64_t)n_atoms * ((nv + 3) / 4) <= 768;
  return 4;
}

template <typename R>
struct ApGrid {
  int32_t grid, nthr, vb;   // vb: vectors per bra item, 0: no bra in this launch
  bool pipe;
  size_t smem;
};

template <typename R, typename C, int P, bool PIPE, int VB>
static void ap_local_pv(const ApLocal<R>& a, const ApBra<R>& b, const ApCoef& cf, const ApGrid<R>& g, hipStream_t st) {
  if constexpr (sizeof(R) == 8) {   // only the bands' filter (complex128) adds a second block
    if (a.prev != nullptr) {
      hipLaunchKernelGGL((k_ap_local<R, C, P, PIPE, true, VB>), dim3(g.grid), dim3(g.nthr), g.smem, st, a, b, cf);
      return;
    }
  }
  hipLaunchKernelGGL((k_ap_local<R, C, P, PIPE, false, VB>), dim3(g.grid), dim3(g.nthr), g.smem, st, a, b, cf);
}

template <typename R, typename C, int P, bool PIPE>
static void ap_local_pp(const ApLocal<R>& a, const ApBra<R>& b, const ApCoef& cf, const ApGrid<R>& g, hipStream_t st) {
  if constexpr (sizeof(R) == 4) {
    if (g.vb == 4) {
      ap_local_pv<R, C, P, PIPE, 4>(a, b, cf, g, st);
      return;
    }
  }
  if (g.vb == 2) ap_local_pv<R, C, P, PIPE, 2>(a, b, cf, g, st);
  else ap_local_pv<R, C, P, PIPE, 0>(a, b, cf, g, st);
}

template <typename R, typename C, int P>
static void ap_local_p(const ApLocal<R>& a, const ApBra<R>& b, const ApCoef& cf, const ApGrid<R>& g, hipStream_t st) {
  if (g.pipe) ap_local_pp<R, C, P, true>(a, b, cf, g, st);
  else ap_local_pp<R, C, P, false>(a, b, cf, g, st);
}

template <typename R, typename C>
static int32_t ap_launch(const cbs_system* s, double E, int32_t nv, const ApCoef& cf, const cplx<R>* x, cplx<R>* y,
                         R* kt, const cplx<R>* prev, double beta, hipStream_t st) {
  const Projector& pr = s->proj;
  const bool f64 = std::is_same<R, double>::value;
  ApLocal<R> a;
  a.nx = s->nx;
  a.ny = s->ny;
  a.nz = s->nz;
  a.N = s->N;
  a.kin = -0.5 / (s->h * s->h);
  a.E = E;
  a.beta = beta;
  for (int i = 0; i < 5; ++i) {
    a.c[i] = s->fd[i];
    a.zc[i] = a.kin * s->fd[i];
  }
  a.vloc = f64 ? (const R*)s->vloc64 : (const R*)s->vloc32;
  a.vloc64 = s->vloc64;
  a.x = x;
  a.prev = prev;
  a.y = y;
  ApBra<R> b{};
  b.n_atoms = pr.n_atoms;
  b.nv = nv;
  b.N = s->N;
  b.seg = pr.seg;
  b.idx = pr.ball_idx;
  b.u = f64 ? (const R*)pr.ball_u64 : (const R*)pr.ball_u32;
  b.coeff = f64 ? (const R*)pr.coeff64 : (const R*)pr.coeff32;
  b.x = x;
  b.kt = kt;
  if (ap_cell_fits(s)) {
    const ApPoint<R> pt{pr.pt_off, pr.pt_key, f64 ? (const R*)pr.pt_u64 : (const R*)pr.pt_u32};
    const size_t smem = ap_cell_lds(s->N, pr.n_atoms, sizeof(cplx<R>), sizeof(C));
    switch (s->p) {
      case 1: ap_cell_p<R, C, 1>(a, b, pt, cf, nv, smem, st); break;
      case 2: ap_cell_p<R, C, 2>(a, b, pt, cf, nv, smem, st); break;
      case 3: ap_cell_p<R, C, 3>(a, b, pt, cf, nv, smem, st); break;
      case 4: ap_cell_p<R, C, 4>(a, b, pt, cf, nv, smem, st); break;
      default: set_error("unsupported finite-difference half-width %d", s->p); return CBS_EINVAL;
    }
    CBS_HIP(hipGetLastError());
    return CBS_OK;
  }
  const ApplyShape shape = apply_shape(s->nx, s->ny, s->nz, s->p, nv, sizeof(cplx<R>));
  const int32_t ty = shape.ty;
  a.ty = ty;
  a.ntiles = (s->ny + ty - 1) / ty;
  a.zlen = (s->nz + shape.nseg - 1) / shape.nseg;
  a.nseg = (s->nz + a.zlen - 1) / a.zlen;
  a.nlogical = nv * a.ntiles * a.nseg;
  const size_t one = (size_t)(ty + 2 * s->p) * s->nx * sizeof(cplx<R>);
  a.nbuf = (2 * one <= 64 * 1024) ? 2 : 1;
  ApGrid<R> g;
  g.nthr = (s->nx * ty + 63) / 64 * 64;
  g.smem = a.nbuf * one;
  g.vb = 0;
  if (pr.n_atoms > 0) {
    bool together = false;
    const int vb = bra_shape(pr.n_atoms, nv, !f64, &together);
    b.nvb = (nv + vb - 1) / vb;
    if (together) {
      g.vb = vb;
      g.nthr = std::max(g.nthr, 256);
    }
    const int items = b.nvb * pr.n_atoms;
    b.nsub = together ? std::max(1, std::min(g.nthr, items) / 256) : 1;   // spread over the CUs first
    const size_t red = (size_t)b.nsub * 4 * 3 * 8 * vb * sizeof(C);
    b.nlogical = (items + b.nsub - 1) / b.nsub;
    b.grid = (b.nlogical + 7) / 8 * 8;
    if (together) {
      g.smem = std::max(g.smem, red);
    } else {
      hipLaunchKernelGGL((k_ap_bra<R, C, 4>), dim3(b.grid), dim3(256), 0, st, b, cf);
      CBS_HIP(hipGetLastError());
    }
  }
  g.grid = (g.vb > 0 ? b.grid : 0) + (a.nlogical + 7) / 8 * 8;
  g.pipe = (ty + 2 * s->p) * s->nx <= 2 * g.nthr;
  switch (s->p) {
    case 1: ap_local_p<R, C, 1>(a, b, cf, g, st); break;
    case 2: ap_local_p<R, C, 2>(a, b, cf, g, st); break;
    case 3: ap_local_p<R, C, 3>(a, b, cf, g, st); break;
    case 4: ap_local_p<R, C, 4>(a, b, cf, g, st); break;
    default: set_error("unsupported finite-difference half-width %d", s->p); return CBS_EINVAL;
  }
  CBS_HIP(hipGetLastError());
  if (pr.n_atoms > 0) {
    ApKet<R> k;
    k.n_atoms = pr.n_atoms;
    k.nv = nv;
    k.nvg = (nv + AP_VG - 1) / AP_VG;
    k.N = s->N;
    // two vector groups a workgroup where they pair up and enough workgroups remain (whole calls:
    // 48x48x32, 32 vectors, 114 -> 112 us in complex128 and 79 -> 75 in complex64; 64x64x40, 64 vectors,
    // 407 -> 378 and 248 -> 233; three groups 99 -> 102; 24x24x16, 24 vectors, 34.6 -> 35.9)
    const int64_t ngroups = (s->N + KG - 1) / KG;
    const int cb = k.nvg % 2 == 0 && ngroups * k.nvg >= 2048 ? 2 : 1;
    k.nlogical = (int32_t)ngroups * (k.nvg / cb);
    k.grp_off = pr.grp_off;
    k.grp_key = pr.grp_key;
    k.grp_mask = pr.grp_mask;
    k.grp_u = f64 ? (const R*)pr.grp_u64 : (const R*)pr.grp_u32;
    k.kt = kt;
    k.y = y;
    k.pt_off = pr.pt_off;
    k.pt_key = pr.pt_key;
    k.pt_u = f64 ? (const R*)pr.pt_u64 : (const R*)pr.pt_u32;
    const dim3 grid((k.nlogical + 7) / 8 * 8);
    if (cb == 2) hipLaunchKernelGGL((k_ap_ket<R, C, 2>), grid, dim3(256), 0, st, k);
    else hipLaunchKernelGGL((k_ap_ket<R, C, 1>), grid, dim3(256), 0, st, k);
    CBS_HIP(hipGetLastError());
  }
  return CBS_OK;
}

template <typename R>
int32_t launch_apply(const cbs_system* s, double E, int32_t n_vec, const double2* c0, const double2* cp,
                     const double2* cm, const void* x, void* y, void* kt, const void* prev, double beta,
                     hipStream_t st) {
  const bool f32 = std::is_same<R, float>::value && lo_arith_fp32();
  for (int32_t v0 = 0; v0 < n_vec; v0 += AP_VMAX) {
    const int32_t nv = std::min(AP_VMAX, n_vec - v0);
    ApCoef cf;
    for (int32_t v = 0; v < AP_VMAX; ++v) {
      const double2 z = make_double2(0, 0);
      cf.c0[v] = v < nv ? c0[v0 + v] : z;
      cf.cp[v] = v < nv ? cp[v0 + v] : z;
      cf.cm[v] = v < nv ? cm[v0 + v] : z;
    }
    const int64_t off = (int64_t)v0 * s->N;
    const cplx<R>* xx = (const cplx<R>*)x + off;
    const cplx<R>* pp = (prev != nullptr) ? (const cplx<R>*)prev + off : nullptr;
    cplx<R>* yy = (cplx<R>*)y + off;
    if constexpr (std::is_same<R, float>::value) {
      if (f32) {
        CBS_TRY((ap_launch<R, float>(s, E, nv, cf, xx, yy, (R*)kt, pp, beta, st)));
        continue;
      }
    }
    CBS_TRY((ap_launch<R, double>(s, E, nv, cf, xx, yy, (R*)kt, pp, beta, st)));
  }
  return CBS_OK;
}

template int32_t launch_apply<double>(const cbs_system*, double, int32_t, const double2*, const double2*,
                                      const double2*, const void*, void*, void*, const void*, double, hipStream_t);
template int32_t launch_apply<float>(const cbs_system*, double, int32_t, const double2*, const double2*,
                                     const double2*, const void*, void*, void*, const void*, double, hipStream_t);

// Coefficients (1, z, 1/z) of P(z) for n vectors.
void apply_coefs(int32_t n, const double* z, std::vector<double2>& c0, std::vector<double2>& cp,
                 std::vector<double2>& cm) {
  c0.assign(n, make_double2(1, 0));
  cp.resize(n);
  cm.resize(n);
  for (int32_t v = 0; v < n; ++v) {
    const double zr = z[2 * v], zi = z[2 * v + 1], d = zr * zr + zi * zi;
    cp[v] = make_double2(zr, zi);
    cm[v] = make_double2(zr / d, -zi / d);
  }
}

}  // namespace cbs
