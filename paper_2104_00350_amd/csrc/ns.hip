// Momentum step of the Navier-Stokes coupling on the staggered grid (sections 2, 3.2, 4.2.3, 4.3 and 4.4):
// explicit Adams-Bashforth prediction (Eq. PredictionExp), volume penalisation with the
// staggered-cell fluid fractions (Eq. Penalization2), the slip / no-penetration velocity ghost
// fill, the variable-density pressure equation (Eq. PressurePoisson, rho0 = min(rho1, rho2),
// p^ = 2p^n - p^(n-1)) solved by the spectral pipeline, and the correction (Eq. correction).
//
// Non-dimensional momentum equation (lengths in domain units, density and viscosity relative to
// the reference fluid of Re):
//   du/dt + div(u u) = (1/rho) [-grad p + (1/Re) div(mu (grad u + grad u^T)) + kappa phi grad C] + g
// with rho = ((C+1) rho2 - (C-1) rho1)/2, mu likewise, phi = C^3 - C - Cn^2 lap C and
// kappa = 3/(2 sqrt2 Re Ca Cn), the factor that gives the planar profile the surface tension of
// the wall condition.
//
// Face field a holds u_a on the face between cell c and c + e_a.  Periodic axes wrap; the bounded
// (last) axis has no-slip box walls: the normal velocity on both walls is zero (the top wall face
// is stored and kept at zero), the tangential velocity has the image -u across a wall, no
// pressure gradient acts through a wall, and cell scalars are reflected.
//
// A thread handles the d faces c + e_a/2 of a cell.  On 3D grids of whole 64 x 8 tiles of columns the kernels
// march in z, a plane's neighbours in LDS and the z neighbours in LDS or registers (k_ns_*_zm); on 2D grids and
// the other 3D ones they take one cell per thread, its neighbours from global memory through the caches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.h"

namespace chib {

namespace {

constexpr int kNsThreads = 256;   // the tiled walk below assumes 2^8 threads

struct NsGrid {
  int n[3];       // cells per axis (1 beyond d); powers of two
  int ln[3];      // log2 of n
  int d;
  int64_t N;
};

template <typename T>
struct NsCoef {
  T inv_h, dt, inv_re, kappa;
  T rho1, rho2, mu1, mu2;
  T g[3];
  T rho0, inv_rho0, rho0_dt;
};

template <typename T>
struct FaceSet {
  T *f[3];
};

template <typename T>
__device__ __forceinline__ T rho_of(const NsCoef<T> &k, T C) {
  return T(0.5) * ((C + T(1)) * k.rho2 - (C - T(1)) * k.rho1);
}

template <typename T>
__device__ __forceinline__ T mu_of(const NsCoef<T> &k, T C) {
  return T(0.5) * ((C + T(1)) * k.mu2 - (C - T(1)) * k.mu1);
}

__device__ __forceinline__ void coords(const NsGrid &g, int64_t c, int *q) {
  q[0] = (int)(c & (g.n[0] - 1));
  q[1] = (int)((c >> g.ln[0]) & (g.n[1] - 1));
  q[2] = (int)(c >> (g.ln[0] + g.ln[1]));
}

// Cells a launch visits: one per thread (flat), or, on 3D grids, a tile of 2^ltx x 2^lty columns
// per workgroup marched through zc consecutive planes, so that the planes above and below a cell
// are still in the caches when its stencil reads them.
struct NsWalk {
  int flat;
  int ltx, lty;         // tile: 2^ltx cells along x by 2^lty along y (ltx + lty = log2 of the workgroup)
  int lbx, lby;         // log2 of the tile counts along x and y
  int zc;               // planes per workgroup
};

template <typename F>
__device__ __forceinline__ void for_each_cell(const NsWalk &wk, const NsGrid &g, F f) {
  if (wk.flat) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < g.N) f(c);
    return;
  }
  const int b = (int)blockIdx.x;
  const int bx = b & ((1 << wk.lbx) - 1);
  const int by = (b >> wk.lbx) & ((1 << wk.lby) - 1);
  const int bz = b >> (wk.lbx + wk.lby);
  const int i = (bx << wk.ltx) + (int)(threadIdx.x & ((1u << wk.ltx) - 1));
  const int j = (by << wk.lty) + (int)(threadIdx.x >> wk.ltx);
  const int64_t row = (int64_t)i + ((int64_t)j << g.ln[0]);
  for (int k = bz * wk.zc; k < (bz + 1) * wk.zc; ++k) f(row + ((int64_t)k << (g.ln[0] + g.ln[1])));
}

// Prediction (Eq. PredictionExp) and penalisation (Eq. Penalization2) on the d faces of each cell:
//   u** = alpha_f (u^n + dt (-(3/2 N^n - 1/2 N^(n-1)) + ((1/Re) V + kappa phi_f dC/dx_a) / rho_f + g_a))
// N: conservative central convective term; V: viscous term with mu from C^(n+1); phi = W.
// Writes N^n over N^(n-1).  first: forward Euler for the convective term.
// Neighbour offsets of a cell: op[b] / om[b] move one cell up / down along axis b (periodic axes
// wrap, the bounded axis steps a plane; validity along it is checked by the caller).
template <int D>
__device__ __forceinline__ void nbr_offsets(const NsGrid &g, const int *q, int *op, int *om) {
#pragma unroll
  for (int b = 0; b < D; ++b) {
    const int sh = b == 0 ? 0 : (b == 1 ? g.ln[0] : g.ln[0] + g.ln[1]);
    if (b < D - 1) {
      op[b] = (((q[b] + 1) & (g.n[b] - 1)) - q[b]) << sh;
      om[b] = (((q[b] - 1) & (g.n[b] - 1)) - q[b]) << sh;
    } else {
      op[b] = 1 << sh;
      om[b] = -(1 << sh);
    }
  }
}

template <typename T, int D>
__device__ __forceinline__ void ns_predict_cell(FaceSet<T> U, const T *__restrict__ C,
                                                const T *__restrict__ phi, FaceSet<T> Nh,
                                                FaceSet<T> Af, FaceSet<T> Us, NsGrid g, NsCoef<T> k,
                                                int first, int64_t c64) {
  constexpr int d = D, bw = D - 1;
  const int c = (int)c64;
  const int nw = g.n[bw];
  int q[3];
  coords(g, c64, q);
  const int w = q[bw];
  int op[3], om[3];
  nbr_offsets<D>(g, q, op, om);
  auto step = [&](int ax, int sgn) { return sgn > 0 ? op[ax] : om[ax]; };
  // face value of component a at index i whose bounded coordinate is wq (zero outside the box and
  // on the top wall face); the load always happens, from the cell itself when i is not valid, so
  // that every load of the stencil can be in flight at once
  auto fv = [&](const T *f, int a, int i, int wq) -> T {
    const bool ok = wq >= 0 && wq < nw && !(a == bw && wq == nw - 1);
    const T v = f[ok ? i : c];
    return ok ? v : T(0);
  };
  auto F1 = [&](const T *f, int a, int ax, int sgn) -> T {
    return fv(f, a, c + step(ax, sgn), w + (ax == bw ? sgn : 0));
  };
  auto F2 = [&](const T *f, int a, int ax1, int s1, int ax2, int s2) -> T {
    return fv(f, a, c + step(ax1, s1) + step(ax2, s2), w + (ax1 == bw ? s1 : 0) + (ax2 == bw ? s2 : 0));
  };
  // cell scalar one cell away (reflected on the bounded axis)
  auto roff = [&](int ax, int sgn) {
    if (ax == bw && (w + sgn < 0 || w + sgn >= nw)) return 0;
    return step(ax, sgn);
  };
#pragma unroll
  for (int a = 0; a < d; ++a) {
    if (a == bw && w == nw - 1) {   // top wall face: no penetration
      Us.f[a][c] = T(0);
      Nh.f[a][c] = T(0);
      continue;
    }
    const T *ua = U.f[a];
    const T u0 = ua[c];
    // convective term
    T N = T(0);
#pragma unroll
    for (int b = 0; b < d; ++b) {
      if (b == a) {
        const T uc0 = T(0.5) * (F1(ua, a, a, -1) + u0);
        const T uc1 = T(0.5) * (u0 + F1(ua, a, a, 1));
        N += (uc1 * uc1 - uc0 * uc0) * k.inv_h;
      } else {
        const T *ub = U.f[b];
        const T e1 = T(0.5) * (u0 + F1(ua, a, b, 1)) * T(0.5) * (fv(ub, b, c, w) + F1(ub, b, a, 1));
        const T e0 = T(0.5) * (F1(ua, a, b, -1) + u0) * T(0.5) * (F1(ub, b, b, -1) + F2(ub, b, b, -1, a, 1));
        const T E1 = (b == bw && w == nw - 1) ? T(0) : e1;
        const T E0 = (b == bw && w == 0) ? T(0) : e0;
        N += (E1 - E0) * k.inv_h;
      }
    }
    // viscous term
    const T mu_c = mu_of(k, C[c]);
    const T mu_a = mu_of(k, C[c + roff(a, 1)]);
    const T tn0 = T(2) * mu_c * (u0 - F1(ua, a, a, -1)) * k.inv_h;
    const T tn1 = T(2) * mu_a * (F1(ua, a, a, 1) - u0) * k.inv_h;
    T V = (tn1 - tn0) * k.inv_h;
#pragma unroll
    for (int b = 0; b < d; ++b) {
      if (b == a) continue;
      const T *ub = U.f[b];
      // edge c + e_a/2 + e_b/2
      const T me1 = T(0.25) * (mu_c + mu_a + mu_of(k, C[c + roff(b, 1)]) + mu_of(k, C[c + roff(a, 1) + roff(b, 1)]));
      const T ub_up = (b == bw && w == nw - 1) ? -u0 : F1(ua, a, b, 1);
      const T tau1 = me1 * ((ub_up - u0) * k.inv_h + (F1(ub, b, a, 1) - fv(ub, b, c, w)) * k.inv_h);
      // edge c + e_a/2 - e_b/2; on the bottom wall the no-slip image and u_b = 0 along the wall
      const T mu_b = mu_of(k, C[c + roff(b, -1)]);
      const T mu_ab = mu_of(k, C[c + roff(b, -1) + roff(a, 1)]);
      const T me0 = T(0.25) * (mu_b + mu_ab + mu_c + mu_a);
      const T ua_m = F1(ua, a, b, -1);
      const T tin = me0 * ((u0 - ua_m) * k.inv_h + (F2(ub, b, b, -1, a, 1) - F1(ub, b, b, -1)) * k.inv_h);
      const T twall = T(0.5) * (mu_c + mu_a) * (u0 - (-u0)) * k.inv_h;
      const T tau0 = (b == bw && w == 0) ? twall : tin;
      V += (tau1 - tau0) * k.inv_h;
    }
    // capillary force and density on the face
    const int ia = c + roff(a, 1);
    const T C0 = C[c], C1 = C[ia];
    const T F = k.kappa * (T(0.5) * (phi[c] + phi[ia])) * (C1 - C0) * k.inv_h;
    const T rf = T(0.5) * (rho_of(k, C0) + rho_of(k, C1));
    const T Np = first ? N : Nh.f[a][c];
    const T us = u0 + k.dt * (-(T(1.5) * N - T(0.5) * Np) + (V * k.inv_re + F) / rf + k.g[a]);
    Us.f[a][c] = Af.f[a][c] * us;
    Nh.f[a][c] = N;
  }
}

template <typename T, int D>
__global__ __launch_bounds__(kNsThreads) void k_ns_predict(FaceSet<T> U, const T *__restrict__ C,
                                                           const T *__restrict__ phi, FaceSet<T> Nh,
                                                           FaceSet<T> Af, FaceSet<T> Us, NsGrid g, NsCoef<T> k,
                                                           int first, NsWalk wk) {
  for_each_cell(wk, g, [&](int64_t c) { ns_predict_cell<T, D>(U, C, phi, Nh, Af, Us, g, k, first, c); });
}

// 3D prediction marching in z over a 64 x 8 tile of columns, every field read once.  The kernel is bound
// by memory (136 bytes per cell at 256^3 FP64), so what counts is that no line is fetched twice: u, C
// and phi of a plane, with a one-cell x/y halo, go to LDS when the plane is first read and every stencil
// value comes from there (neighbours taken through the caches instead re-fetched u and C two to three
// times: 170 bytes read per cell of 88, as other tiles' planes evict a plane before its neighbours ask
// for it).  Three LDS slots hold planes z-1 .. z+1 in turn, so one barrier per plane suffices; plane z+2
// and the own-cell fields of plane z+1 are requested while plane z is computed.
// Each thread forms the xy, xz and yz edges around its three faces: the convective flux
// E_ab = (u_a mean along b)(u_b mean along a) and the shear stress tau_ab = mu_e (du_a/dx_b + du_b/dx_a)
// of an edge are symmetric in a and b; those of the z edges below come from the plane before.  Powers of
// two and of 1/h are taken out of the sums; mu and rho are linear in C, so an edge viscosity or a face
// density is one fused multiply-add on the sum of its cells' distances from the phase with the smaller
// value (from the mean of the phases, FP32 lost 1.7e-5 of the lighter density at a ratio of 1000).  Same
// formulas and wall rules as ns_predict_cell: the planes beyond the box walls hold the images (-u_x, -u_y, u_z = 0, C reflected),
// with which the wall edges take their values without a case of their own.
constexpr int kEx = 64, kEy = 8, kEhx = kEx + 2, kEhy = kEy + 2;
constexpr int kEThreads = kEx * kEy;                        // one thread per column of the tile
constexpr int kEHalo = kEhx * kEhy - kEThreads;              // halo cells of a plane
constexpr int kEFields = 5;                                  // u_x, u_y, u_z, C, phi
template <typename T> constexpr size_t predict_lds() { return (size_t)3 * kEFields * kEhx * kEhy * sizeof(T); }

template <typename T>
struct PredictCoef {
  T mu0, mu1, mus;     // mu of an edge = mu0 + mu1 sum of its cells' (C + mus)
  T rf0, rf1, rfs;     // rho_f = rf0 + rf1 ((C + rfs) + (C' + rfs))
  T n_fac;             // 1/(4h)
  T v_fac;             // 1/(Re h^2)
  T f_fac;             // kappa/(2h)
};

// EQ: equal densities, rho_f the constant rf0 (its reciprocal in inv_rf).
template <typename T, bool EQ>
__global__ __launch_bounds__(kEThreads, 4) void k_ns_predict_zm(FaceSet<T> U, const T *__restrict__ C,
                                                                const T *__restrict__ phi, FaceSet<T> Nh,
                                                                FaceSet<T> Af, FaceSet<T> Us, NsGrid g,
                                                                NsCoef<T> k, PredictCoef<T> q, T inv_rf, int first,
                                                                int zc, int runs) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int PL = kEhx * kEhy;                            // one field of one slot
  T *const s = reinterpret_cast<T *>(smem_raw);              // [slot][field][row][column]
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int tiles_x = nx / kEx, tiles_y = ny / kEy;
  int b = runs ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int bx = b % tiles_x;
  b /= tiles_x;
  const int by = b % tiles_y;
  const int bz = b / tiles_y;
  const int x0 = bx * kEx, y0 = by * kEy, z0 = bz * zc;
  const int tid = (int)threadIdx.x;
  const int tx = tid & (kEx - 1), ty = tid >> 6;
  const int psh = g.ln[0] + g.ln[1];
  const int col = (x0 + tx) + ((y0 + ty) << g.ln[0]);        // own column within a plane
  const int own = (ty + 1) * kEhx + tx + 1;                  // own slot within a field
  // the halo cell this thread also brings (threads below kEHalo): two rows, then two columns
  int hcol = col, hslot = own;
  const bool halo = tid < kEHalo;
  if (halo) {
    int hr, hc;
    if (tid < 2 * kEhx) {
      hr = tid < kEhx ? 0 : kEhy - 1;
      hc = tid < kEhx ? tid : tid - kEhx;
    } else {
      const int e = tid - 2 * kEhx;
      hr = 1 + (e >> 1);
      hc = (e & 1) ? kEhx - 1 : 0;
    }
    hslot = hr * kEhx + hc;
    hcol = ((x0 - 1 + hc) & (nx - 1)) + (((y0 - 1 + hr) & (ny - 1)) << g.ln[0]);
  }
  T v[kEFields], hv[kEFields];                               // the plane in flight: own cell, halo cell
  auto request = [&](int z) {
    const int64_t zb = (int64_t)(z < 0 ? 0 : (z >= nz ? nz - 1 : z)) << psh;
    v[0] = U.f[0][zb + col];
    v[1] = U.f[1][zb + col];
    v[2] = U.f[2][zb + col];
    v[3] = C[zb + col];
    v[4] = phi[zb + col];
    if (halo) {
      hv[0] = U.f[0][zb + hcol];
      hv[1] = U.f[1][zb + hcol];
      hv[2] = U.f[2][zb + hcol];
      hv[3] = C[zb + hcol];
      hv[4] = phi[zb + hcol];
    }
  };
  // the plane in flight into its slot; beyond the walls u_x and u_y change sign, and u_z vanishes there and
  // on the top wall face
  auto store = [&](int z, int slot) {
    const T sg = (z < 0 || z >= nz) ? T(-1) : T(1);
    const bool wz = z < 0 || z >= nz - 1;
    T *p = s + slot * kEFields * PL;
    p[own] = sg * v[0];
    p[PL + own] = sg * v[1];
    p[2 * PL + own] = wz ? T(0) : v[2];
    p[3 * PL + own] = v[3];
    p[4 * PL + own] = v[4];
    if (halo) {
      p[hslot] = sg * hv[0];
      p[PL + hslot] = sg * hv[1];
      p[2 * PL + hslot] = wz ? T(0) : hv[2];
      p[3 * PL + hslot] = hv[3];
      p[4 * PL + hslot] = hv[4];
    }
  };
  auto mu_e = [&](T a, T b, T c, T d) { return q.mu0 + q.mu1 * (((a + q.mus) + (b + q.mus)) + ((c + q.mus) + (d + q.mus))); };
  // 4 E and h tau of the edge between axis a and b with lower cell at slot index i, its neighbour along a at
  // i + oa and along b at j (the same field plane or the one above)
  auto edge_xy = [&](const T *p, int i, T &E, T &t) {
    const T ua = p[i], ub = p[PL + i], uab = p[i + kEhx], uba = p[PL + i + 1];
    const T *c = p + 3 * PL;
    E = (ua + uab) * (ub + uba);
    t = mu_e(c[i], c[i + 1], c[i + kEhx], c[i + kEhx + 1]) * ((uab - ua) + (uba - ub));
  };
  // edge between axis a (field a, in-plane step oa) and z: planes lo and hi
  auto edge_z = [&](const T *lo, const T *hi, int a, int oa, int i, T &E, T &t) {
    const T ua = lo[a * PL + i], uaz = hi[a * PL + i], uz = lo[2 * PL + i], uza = lo[2 * PL + i + oa];
    const T *c0 = lo + 3 * PL, *c1 = hi + 3 * PL;
    E = (ua + uaz) * (uz + uza);
    t = mu_e(c0[i], c0[i + oa], c1[i], c1[i + oa]) * ((uaz - ua) + (uza - uz));
  };
  request(z0 - 1);
  store(z0 - 1, 0);
  request(z0);
  store(z0, 1);
  request(z0 + 1);
  T nh[3], af[3];
  auto request_own = [&](int z) {
    const int64_t c = ((int64_t)z << psh) + col;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      nh[a] = __builtin_nontemporal_load(Nh.f[a] + c);
      af[a] = __builtin_nontemporal_load(Af.f[a] + c);
    }
  };
  __syncthreads();
  T Exm, txm, Eym, tym;                                      // xz and yz edges below the plane
  edge_z(s, s + kEFields * PL, 0, 1, own, Exm, txm);
  edge_z(s, s + kEFields * PL, 1, kEhx, own, Eym, tym);
  int lo_s = 1, hi_s = 2;
  T uzm = s[2 * PL + own];                                   // u_z of the plane below
  for (int z = z0; z < z0 + zc; ++z) {
    store(z + 1, hi_s);
    request_own(z);
    __syncthreads();   // (the slot after this one was last read two planes ago, before the previous barrier)
    if (z + 1 < z0 + zc) request(z + 2);
    const T *p = s + lo_s * kEFields * PL, *pu = s + hi_s * kEFields * PL;
    const T *c = p + 3 * PL, *ph = p + 4 * PL;
    const int i = own;
    // the edges one after another (held apart: with all their LDS reads hoisted together the kernel spills)
    T dE[3], dt[3], E, t, Exz, txz, Eyz, tyz;
    edge_xy(p, i, E, t);
    dE[0] = dE[1] = E;
    dt[0] = dt[1] = t;
    edge_xy(p, i - kEhx, E, t);
    dE[0] -= E;
    dt[0] -= t;
    edge_xy(p, i - 1, E, t);
    dE[1] -= E;
    dt[1] -= t;
    __builtin_amdgcn_sched_barrier(0);
    edge_z(p, pu, 0, 1, i, Exz, txz);
    dE[0] += Exz - Exm;
    dt[0] += txz - txm;
    edge_z(p, pu, 0, 1, i - 1, E, t);
    dE[2] = Exz - E;
    dt[2] = txz - t;
    __builtin_amdgcn_sched_barrier(0);
    edge_z(p, pu, 1, kEhx, i, Eyz, tyz);
    dE[1] += Eyz - Eym;
    dt[1] += tyz - tym;
    edge_z(p, pu, 1, kEhx, i - kEhx, E, t);
    dE[2] += Eyz - E;
    dt[2] += tyz - t;
    __builtin_amdgcn_sched_barrier(0);
    const T C0 = c[i], p0 = ph[i];
    const T m0 = q.mu0 + T(4) * q.mu1 * (C0 + q.mus);
    const int64_t cell = ((int64_t)z << psh) + col;
    auto face = [&](int a, T um, T u0, T up, T Ca, T pa, T dE, T dt_) {
      const T ma = q.mu0 + T(4) * q.mu1 * (Ca + q.mus);
      const T f1 = u0 + up, f0 = um + u0;
      const T N = ((f1 * f1 - f0 * f0) + dE) * q.n_fac;
      const T V = (T(2) * (ma * (up - u0) - m0 * (u0 - um)) + dt_) * q.v_fac;
      const T F = q.f_fac * (p0 + pa) * (Ca - C0);
      // (C + rfs formed anew for each face: held through all three, it spills into the division; 128^3 FP64
      // 60.4 against 57.3 us)
      T Cd = C0;
      asm volatile("" : "+v"(Cd));
      const T VF = EQ ? (V + F) * inv_rf : (V + F) / (q.rf0 + q.rf1 * ((Cd + q.rfs) + (Ca + q.rfs)));
      const T Np = first ? N : nh[a];
      const T us = u0 + k.dt * (-(T(1.5) * N - T(0.5) * Np) + VF + k.g[a]);
      __builtin_nontemporal_store(af[a] * us, Us.f[a] + cell);
      __builtin_nontemporal_store(N, Nh.f[a] + cell);
    };
    face(0, p[i - 1], p[i], p[i + 1], c[i + 1], ph[i + 1], dE[0], dt[0]);
    __builtin_amdgcn_sched_barrier(0);
    face(1, p[PL + i - kEhx], p[PL + i], p[PL + i + kEhx], c[i + kEhx], ph[i + kEhx], dE[1], dt[1]);
    __builtin_amdgcn_sched_barrier(0);
    if (z < nz - 1) {
      face(2, uzm, p[2 * PL + i], pu[2 * PL + i], pu[3 * PL + i], pu[4 * PL + i], dE[2], dt[2]);
    } else {           // top wall face
      Us.f[2][cell] = T(0);
      Nh.f[2][cell] = T(0);
    }
    uzm = p[2 * PL + i];
    Exm = Exz;
    txm = txz;
    Eym = Eyz;
    tym = tyz;
    const int nx_s = 3 - lo_s - hi_s;
    lo_s = hi_s;
    hi_s = nx_s;
  }
}

// Right-hand side of Eq. PressurePoisson at the cell centres:
//   div((1 - rho0/rho_f) grad p^) + (rho0/dt) div u**,  p^ = 2 P0 - P1; no flux through the walls.
template <typename T, int D>
__device__ __forceinline__ void ns_prhs_cell(FaceSet<T> Us, const T *__restrict__ C,
                                             const T *__restrict__ P0, const T *__restrict__ P1,
                                             T *__restrict__ R, NsGrid g, NsCoef<T> k, int64_t c64) {
  constexpr int d = D, bw = D - 1;
  const int c = (int)c64;
  const int nw = g.n[bw];
  int q[3];
  coords(g, c64, q);
  const int w = q[bw];
  int op[3], om[3];
  nbr_offsets<D>(g, q, op, om);
  auto ph = [&](int i) { return T(2) * P0[i] - P1[i]; };
  const T phc = ph(c);
  const T rc = rho_of(k, C[c]);
  T acc1 = T(0), acc2 = T(0);
#pragma unroll
  for (int a = 0; a < d; ++a) {
    // flux (1 - rho0/rho_f) dp^/dx_a through the upper and the lower face of the cell along a
    // (every load happens, from the cell itself where a face lies on a box wall)
    const bool top = a == bw && w == nw - 1, bottom = a == bw && w == 0;
    const int i1 = c + (top ? 0 : op[a]);
    const int i0 = c + (bottom ? 0 : om[a]);
    const T rf1 = T(0.5) * (rc + rho_of(k, C[i1]));
    const T rf0 = T(0.5) * (rho_of(k, C[i0]) + rc);
    const T fu1 = (T(1) - k.rho0 / rf1) * ((ph(i1) - phc) * k.inv_h);
    const T fl0 = (T(1) - k.rho0 / rf0) * ((phc - ph(i0)) * k.inv_h);
    const T uu1 = Us.f[a][c], ul0 = Us.f[a][i0];
    const T fu = top ? T(0) : fu1, uu = top ? T(0) : uu1;
    const T fl = bottom ? T(0) : fl0, ul = bottom ? T(0) : ul0;
    acc1 += fu - fl;
    acc2 += uu - ul;
  }
  R[c] = acc1 * k.inv_h + k.rho0_dt * (acc2 * k.inv_h);
}

template <typename T, int D>
__global__ __launch_bounds__(kNsThreads) void k_ns_pressure_rhs(FaceSet<T> Us, const T *__restrict__ C,
                                                                const T *__restrict__ P0, const T *__restrict__ P1,
                                                                T *__restrict__ R, NsGrid g, NsCoef<T> k, NsWalk wk) {
  for_each_cell(wk, g, [&](int64_t c) { ns_prhs_cell<T, D>(Us, C, P0, P1, R, g, k, c); });
}

// Correction (Eq. correction): u^(n+1) = u** - dt (grad p^(n+1) / rho0 + (1/rho_f - 1/rho0) grad p^)
// on every face but the top wall face; also writes the advecting velocity 2u^(n+1) - u^n of the
// next order-parameter step (Ut, may be absent).
template <typename T, int D>
__device__ __forceinline__ void ns_correct_cell(FaceSet<T> U, FaceSet<T> Ut, FaceSet<T> Us,
                                                const T *__restrict__ C, const T *__restrict__ Pn,
                                                const T *__restrict__ P0, const T *__restrict__ P1,
                                                NsGrid g, NsCoef<T> k, int with_ut, int64_t c64) {
  constexpr int d = D, bw = D - 1;
  const int c = (int)c64;
  const int nw = g.n[bw];
  int q[3];
  coords(g, c64, q);
  const int w = q[bw];
  int op[3], om[3];
  nbr_offsets<D>(g, q, op, om);
  const T phc = T(2) * P0[c] - P1[c];
  const T rc = rho_of(k, C[c]);
  const T pc = Pn[c];
#pragma unroll
  for (int a = 0; a < d; ++a) {
    const bool top = a == bw && w == nw - 1;
    const int ca = c + (top ? 0 : op[a]);
    const T Gn = (Pn[ca] - pc) * k.inv_h;
    const T Gh = ((T(2) * P0[ca] - P1[ca]) - phc) * k.inv_h;
    const T rf = T(0.5) * (rc + rho_of(k, C[ca]));
    const T u1 = Us.f[a][c] - k.dt * (Gn * k.inv_rho0 + (T(1) / rf - k.inv_rho0) * Gh);
    const T un = top ? T(0) : u1;
    const T uo = U.f[a][c];
    U.f[a][c] = un;
    if (with_ut) Ut.f[a][c] = T(2) * un - uo;
  }
}

template <typename T, int D>
__global__ __launch_bounds__(kNsThreads) void k_ns_correct(FaceSet<T> U, FaceSet<T> Ut, FaceSet<T> Us,
                                                           const T *__restrict__ C, const T *__restrict__ Pn,
                                                           const T *__restrict__ P0, const T *__restrict__ P1,
                                                           NsGrid g, NsCoef<T> k, int with_ut, NsWalk wk) {
  for_each_cell(wk, g, [&](int64_t c) { ns_correct_cell<T, D>(U, Ut, Us, C, Pn, P0, P1, g, k, with_ut, c); });
}

// 3D pressure rhs marching in z over a 64 x 8 tile: p^, C, u**_x and u**_y of a plane go to LDS once with
// the halo cells that their differences need (through the caches the neighbours' loads came too late for
// the L2, and a 64^3 grid of 64 workgroups waited for them plane after plane); the z neighbours and the z
// flux below stay in registers.  Same expressions as the per-cell form, with p^ formed once per cell.
constexpr int kPx = 64, kPy = 8, kPThreads = kPx * kPy, kPp = kPx + 2;

template <typename T>
__global__ __launch_bounds__(kPThreads) void k_ns_pressure_rhs_zm(FaceSet<T> Us, const T *__restrict__ C,
                                                                  const T *__restrict__ P0, const T *__restrict__ P1,
                                                                  T *__restrict__ R, NsGrid g, NsCoef<T> k, int zc,
                                                                  int runs) {
  __shared__ T s[2][4][(kPy + 2) * kPp];                     // p^, C, u**_x, u**_y
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int tiles_x = nx / kPx, tiles_y = ny / kPy;
  int b = runs ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int bx = b % tiles_x;
  b /= tiles_x;
  const int by = b % tiles_y;
  const int z0 = (b / tiles_y) * zc;
  const int tid = (int)threadIdx.x, tx = tid & (kPx - 1), ty = tid >> 6;
  const int x0 = bx * kPx, y0 = by * kPy;
  const int psh = g.ln[0] + g.ln[1];
  const int col = x0 + tx + ((y0 + ty) << g.ln[0]);
  const int i = (ty + 1) * kPp + tx + 1;
  // halo cells: the rows below and above (waves 0 and 1), the columns left and right (8 threads each)
  const bool row = tid < 2 * kPx, halo = tid < 2 * kPx + 2 * kPy;
  const int e = tid - 2 * kPx;
  const bool low = row ? tid < kPx : e < kPy;
  const int hr = row ? (low ? 0 : kPy + 1) : 1 + (e & (kPy - 1)), hc = row ? 1 + tx : (low ? 0 : kPx + 1);
  const int hcol = halo ? ((x0 - 1 + hc) & (nx - 1)) + (((y0 - 1 + hr) & (ny - 1)) << g.ln[0]) : col;
  const int hi = hr * kPp + hc;
  const int hf = row ? 1 : 0;                                // the velocity whose difference needs this halo cell
  T v[5], hv[3];
  auto request = [&](int z) {
    const int64_t zb = (int64_t)(z >= nz ? nz - 1 : z) << psh;
    v[0] = T(2) * P0[zb + col] - P1[zb + col];
    v[1] = C[zb + col];
    v[2] = Us.f[0][zb + col];
    v[3] = Us.f[1][zb + col];
    v[4] = Us.f[2][zb + col];
    if (halo) {
      hv[0] = T(2) * P0[zb + hcol] - P1[zb + hcol];
      hv[1] = C[zb + hcol];
      if (low) hv[2] = Us.f[hf][zb + hcol];
    }
  };
  // flux (1 - rho0/rho_f) dp^ through the face between two cells, and u** through the z face below
  auto flux = [&](T r0, T r1, T p0, T p1) { return (T(1) - k.rho0 / (T(0.5) * (r0 + r1))) * ((p1 - p0) * k.inv_h); };
  T fz = T(0), uz = T(0);
  if (z0 > 0) {
    const int64_t m = ((int64_t)(z0 - 1) << psh) + col, c = ((int64_t)z0 << psh) + col;
    fz = flux(rho_of(k, C[m]), rho_of(k, C[c]), T(2) * P0[m] - P1[m], T(2) * P0[c] - P1[c]);
    uz = Us.f[2][m];
  }
  request(z0);
  for (int z = z0; z < z0 + zc; ++z) {
    T (*p)[(kPy + 2) * kPp] = s[z & 1];
    const T ph = v[0], rc = rho_of(k, v[1]), ux = v[2], uy = v[3], uzc = v[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) p[f][i] = v[f];
    if (halo) {
      p[0][hi] = hv[0];
      p[1][hi] = hv[1];
      if (low) p[2 + hf][hi] = hv[2];
    }
    request(z + 1);
    __syncthreads();   // (the slot written next plane was last read a plane ago, before this barrier)
    const bool top = z == nz - 1;
    T acc1 = T(0), acc2 = (ux - p[2][i - 1]) + (uy - p[3][i - kPp]);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int up = a == 0 ? i + 1 : i + kPp, dn = a == 0 ? i - 1 : i - kPp;
      acc1 += flux(rc, rho_of(k, p[1][up]), ph, p[0][up]) - flux(rho_of(k, p[1][dn]), rc, p[0][dn], ph);
    }
    const T fu1 = flux(rc, rho_of(k, v[1]), ph, v[0]);
    const T fu = top ? T(0) : fu1, uu = top ? T(0) : uzc;
    acc1 += fu - fz;
    acc2 += uu - uz;
    R[((int64_t)z << psh) + col] = acc1 * k.inv_h + k.rho0_dt * (acc2 * k.inv_h);
    fz = fu1;
    uz = uzc;
  }
}

// 3D correction marching in z over a 64 x 8 tile.  Bound by memory (128 bytes per cell at 256^3 FP64, 104
// with equal densities): the pressure fields and C of a plane go to LDS once, with the halo column and
// row above, because the neighbours' loads of the same lines came so late that the 4 MB L2 had given
// them up (141 bytes read per cell of 80).  EQ: with equal densities 1/rho_f - 1/rho0 vanishes, and with
// it the term in p^ and the reads of C, p^n and p^(n-1).  u and u** pass through once (streaming).
constexpr int kCx = 64, kCy = 8, kCThreads = kCx * kCy, kCp = kCx + 1;

template <typename T, bool EQ>
__global__ __launch_bounds__(kCThreads) void k_ns_correct_zm(FaceSet<T> U, FaceSet<T> Ut, FaceSet<T> Us,
                                                             const T *__restrict__ C, const T *__restrict__ Pn,
                                                             const T *__restrict__ P0, const T *__restrict__ P1,
                                                             NsGrid g, NsCoef<T> k, int with_ut, int zc, int runs) {
  constexpr int NF = EQ ? 1 : 3;                              // p^(n+1), p^, C
  __shared__ T s[2][NF][(kCy + 1) * kCp];
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int tiles_x = nx / kCx, tiles_y = ny / kCy;
  int b = runs ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int bx = b % tiles_x;
  b /= tiles_x;
  const int by = b % tiles_y;
  const int z0 = (b / tiles_y) * zc;
  const int tid = (int)threadIdx.x, tx = tid & (kCx - 1), ty = tid >> 6;
  const int x0 = bx * kCx, y0 = by * kCy;
  const int psh = g.ln[0] + g.ln[1];
  const int col = x0 + tx + ((y0 + ty) << g.ln[0]);
  const int i = ty * kCp + tx;
  // threads below 64 + 8 also bring a cell of the row above or of the column to the right
  const bool halo = tid < kCx + kCy;
  const int hx = tid < kCx ? x0 + tid : (x0 + kCx) & (nx - 1);
  const int hy = tid < kCx ? (y0 + kCy) & (ny - 1) : y0 + (tid - kCx);
  const int hcol = halo ? hx + (hy << g.ln[0]) : col;
  const int hi = tid < kCx ? kCy * kCp + tid : (tid - kCx) * kCp + kCx;
  T v[NF], hv[NF];
  auto request = [&](int z) {
    const int64_t zb = (int64_t)(z >= nz ? nz - 1 : z) << psh;
    v[0] = Pn[zb + col];
    if (halo) hv[0] = Pn[zb + hcol];
    if constexpr (!EQ) {
      v[1] = T(2) * P0[zb + col] - P1[zb + col];
      v[2] = C[zb + col];
      if (halo) {
        hv[1] = T(2) * P0[zb + hcol] - P1[zb + hcol];
        hv[2] = C[zb + hcol];
      }
    }
  };
  request(z0);
  for (int z = z0; z < z0 + zc; ++z) {
    T (*p)[(kCy + 1) * kCp] = s[z & 1];
    T c[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      c[f] = v[f];
      p[f][i] = v[f];
      if (halo) p[f][hi] = hv[f];
    }
    const int64_t cell = ((int64_t)z << psh) + col;
    request(z + 1);
    T us[3], uo[3] = {T(0), T(0), T(0)};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      us[a] = __builtin_nontemporal_load(Us.f[a] + cell);
      if (with_ut) uo[a] = __builtin_nontemporal_load(U.f[a] + cell);
    }
    __syncthreads();   // (the slot written next plane was last read a plane ago, before this barrier)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int in = a == 0 ? i + 1 : i + kCp;
      auto up = [&](int f) { return a == 2 ? v[f] : p[f][in]; };
      const T Gn = (up(0) - c[0]) * k.inv_h;
      T u1;
      if constexpr (EQ) {
        u1 = us[a] - k.dt * (Gn * k.inv_rho0);
      } else {
        const T Gh = (up(1) - c[1]) * k.inv_h;
        const T rf = T(0.5) * (rho_of(k, c[2]) + rho_of(k, up(2)));
        u1 = us[a] - k.dt * (Gn * k.inv_rho0 + (T(1) / rf - k.inv_rho0) * Gh);
      }
      const T un = (a == 2 && z == nz - 1) ? T(0) : u1;
      __builtin_nontemporal_store(un, U.f[a] + cell);
      if (with_ut) __builtin_nontemporal_store(T(2) * un - uo[a], Ut.f[a] + cell);
    }
  }
}

template <typename T>
NsCoef<T> ns_coef(const Plan &p) {
  NsCoef<T> k;
  k.inv_h = (T)(1.0 / p.h);
  k.dt = (T)p.dt;
  k.inv_re = (T)(1.0 / p.Re);
  k.kappa = (T)(3.0 / (2.0 * 1.4142135623730951 * p.Re * p.Ca * p.Cn));
  k.rho1 = (T)p.rho1;
  k.rho2 = (T)p.rho2;
  k.mu1 = (T)p.mu1;
  k.mu2 = (T)p.mu2;
  for (int a = 0; a < 3; ++a) k.g[a] = (T)p.g[a];
  const double rho0 = p.rho1 < p.rho2 ? p.rho1 : p.rho2;
  k.rho0 = (T)rho0;
  k.inv_rho0 = (T)(1.0 / rho0);
  k.rho0_dt = (T)(rho0 / p.dt);
  return k;
}

template <typename T>
PredictCoef<T> predict_coef(const Plan &p) {
  PredictCoef<T> q;
  // both lines start from the phase with the smaller value (C = -1 or +1)
  q.mu0 = (T)std::min(p.mu1, p.mu2);
  q.mu1 = (T)(0.125 * (p.mu2 - p.mu1));      // a quarter of mu's slope: it meets sums of four cells
  q.mus = p.mu1 <= p.mu2 ? T(1) : T(-1);
  q.rf0 = (T)std::min(p.rho1, p.rho2);
  q.rf1 = (T)(0.25 * (p.rho2 - p.rho1));
  q.rfs = p.rho1 <= p.rho2 ? T(1) : T(-1);
  q.n_fac = (T)(0.25 / p.h);
  q.v_fac = (T)(1.0 / (p.Re * p.h * p.h));
  q.f_fac = (T)(3.0 / (2.0 * 1.4142135623730951 * p.Re * p.Ca * p.Cn) * 0.5 / p.h);
  return q;
}

NsGrid ns_grid(const Plan &p) {
  NsGrid g;
  g.n[0] = p.n[0];
  g.n[1] = p.n[1];
  g.n[2] = p.d == 3 ? p.n[2] : 1;
  g.ln[0] = p.logn[0];
  g.ln[1] = p.logn[1];
  g.ln[2] = p.d == 3 ? p.logn[2] : 0;
  g.d = p.d;
  g.N = p.N;
  return g;
}

// 3D: tiles of 64 x 4 columns (fewer along x on narrower grids) marched through 16 planes; 2D: flat.
NsWalk ns_walk(const Plan &p, unsigned *nb) {
  NsWalk w{};
  w.flat = 1;
  *nb = (unsigned)((p.N + kNsThreads - 1) / kNsThreads);
  if (p.d != 3) return w;
  const int ltx = p.logn[0] < 6 ? p.logn[0] : 6;
  const int lty = 8 - ltx;   // 256 threads
  if (lty > p.logn[1]) return w;
  w.flat = 0;
  w.ltx = ltx;
  w.lty = lty;
  w.lbx = p.logn[0] - ltx;
  w.lby = p.logn[1] - lty;
  w.zc = p.n[2] < 16 ? p.n[2] : 16;
  *nb = (unsigned)((1u << (w.lbx + w.lby)) * (unsigned)(p.n[2] / w.zc));
  return w;
}

// Planes per workgroup of the tiled z-marches: 16 amortise the planes read at the chunk's ends; fewer
// where that leaves the chip short of workgroups (128^3 prediction: 91 us with 32 planes, 63 with 16).
int march_planes(const Plan &p, int tile) {
  int zc = p.n[2] < 16 ? p.n[2] : 16;
  while (zc > 4 && p.N / ((int64_t)tile * zc) < 512) zc >>= 1;
  return zc;
}

template <typename T>
FaceSet<T> faces(void *const *f, int d) {
  FaceSet<T> s;
  for (int a = 0; a < 3; ++a) s.f[a] = (T *)(a < d ? f[a] : f[0]);
  return s;
}

}  // namespace

template <typename T>
hipError_t enqueue_momentum(const Plan &p, int cur, int first, KernelTimer *tm, StepLink *link) {
  hipError_t e = hipSuccess;
  auto mark = [&](const char *name) {
    if (tm && e == hipSuccess) e = tm->mark(name, p.stream);
  };
  if (!p.ns || !p.P[0] || !p.P[1]) return hipErrorInvalidValue;
  const NsGrid g = ns_grid(p);
  const NsCoef<T> k = ns_coef<T>(p);
  unsigned nb = 0;
  const NsWalk wk = ns_walk(p, &nb);
  const T *C = (const T *)p.C[cur];
  const FaceSet<T> U = faces<T>(p.F, p.d), Us = faces<T>(p.Us, p.d), Nh = faces<T>(p.Nh, p.d);
  const FaceSet<T> Af = faces<T>(p.Af, p.d);
  const int runs = tiles_in_runs<T>(p);   // tiles of the marching kernels dealt in runs per die
  const bool with_ut = p.Ut[0] != nullptr;
  const bool eq = p.rho1 == p.rho2;   // equal densities: no term in p^, rho_f a constant
  const FaceSet<T> Ut = with_ut ? faces<T>(p.Ut, p.d) : U;
  mark("ns_phi");
  if (e == hipSuccess) e = enqueue_phi<T>(p, cur, p.W);
  mark("ns_predict");
  if (e == hipSuccess) {
    if (p.d == 2)
      hipLaunchKernelGGL((k_ns_predict<T, 2>), dim3(nb), dim3(kNsThreads), 0, p.stream, U, C, (const T *)p.W, Nh, Af,
                         Us, g, k, first, wk);
    else if (p.n[0] % kEx == 0 && p.n[1] % kEy == 0) {
      const int zc = march_planes(p, kEx * kEy);
      const unsigned nbe = (unsigned)((p.n[0] / kEx) * (p.n[1] / kEy) * (p.n[2] / zc));
      const PredictCoef<T> q = predict_coef<T>(p);
      const T inv_rf = (T)(1.0 / (0.5 * (p.rho1 + p.rho2)));
      if (eq)
        hipLaunchKernelGGL((k_ns_predict_zm<T, true>), dim3(nbe), dim3(kEThreads), predict_lds<T>(), p.stream, U, C,
                           (const T *)p.W, Nh, Af, Us, g, k, q, inv_rf, first, zc, runs);
      else
        hipLaunchKernelGGL((k_ns_predict_zm<T, false>), dim3(nbe), dim3(kEThreads), predict_lds<T>(), p.stream, U, C,
                           (const T *)p.W, Nh, Af, Us, g, k, q, inv_rf, first, zc, runs);
    } else
      hipLaunchKernelGGL((k_ns_predict<T, 3>), dim3(nb), dim3(kNsThreads), 0, p.stream, U, C, (const T *)p.W, Nh, Af,
                         Us, g, k, first, wk);
    e = hipGetLastError();
  }
  mark("ns_vel_fill");
  if (e == hipSuccess && p.G) {
    Plan q = p;
    for (int a = 0; a < 3; ++a) q.F[a] = p.Us[a];
    q.vel_fill = 1;
    // (semi-implicit: the order parameter of the next step's patch is complete already)
    const NextStep nx{p.C[cur], p.C[1 - cur]};
    const bool join = link && link->next && p.NF && p.NP > 0 && p.dg;
    e = enqueue_velocity_fill<T>(q, C, join ? &nx : nullptr);
    if (link) link->dphi_done = join && e == hipSuccess;
  }
  // equal densities: the right-hand side is (rho0/dt) div u** alone, formed inside the forward x transform
  // (as exact as the full expression: 2D FP32 after 20 steps, u off by 2.2e-5 of its norm against 2.3e-5 at
  // 64x32, 5.57e-5 against 5.60e-5 at 1024x512)
  if (eq) {
    mark("ns_div_poisson");
    if (e == hipSuccess) e = enqueue_poisson<T>(p, p.Us, (double)k.rho0_dt * (double)k.inv_h);
  } else {
    mark("ns_pressure_rhs");
    if (e == hipSuccess) {
      if (p.d == 2)
        hipLaunchKernelGGL((k_ns_pressure_rhs<T, 2>), dim3(nb), dim3(kNsThreads), 0, p.stream, Us, C,
                           (const T *)p.P[0], (const T *)p.P[1], (T *)p.W, g, k, wk);
      else if (p.n[0] % kPx == 0 && p.n[1] % kPy == 0) {
        const int zc = march_planes(p, kPx * kPy);
        const unsigned nbp = (unsigned)((p.n[0] / kPx) * (p.n[1] / kPy) * (p.n[2] / zc));
        hipLaunchKernelGGL((k_ns_pressure_rhs_zm<T>), dim3(nbp), dim3(kPThreads), 0, p.stream, Us, C,
                           (const T *)p.P[0], (const T *)p.P[1], (T *)p.W, g, k, zc, runs);
      } else
        hipLaunchKernelGGL((k_ns_pressure_rhs<T, 3>), dim3(nb), dim3(kNsThreads), 0, p.stream, Us, C,
                           (const T *)p.P[0], (const T *)p.P[1], (T *)p.W, g, k, wk);
      e = hipGetLastError();
    }
    mark("ns_poisson");
    if (e == hipSuccess) e = enqueue_poisson<T>(p);
  }
  mark("ns_correct");
  if (e == hipSuccess) {
    if (p.d == 2)
      hipLaunchKernelGGL((k_ns_correct<T, 2>), dim3(nb), dim3(kNsThreads), 0, p.stream, U, Ut, Us, C,
                         (const T *)p.W, (const T *)p.P[0], (const T *)p.P[1], g, k, with_ut ? 1 : 0, wk);
    else if (p.n[0] % kCx == 0 && p.n[1] % kCy == 0) {
      const int zc = march_planes(p, kCx * kCy);
      const unsigned nbc = (unsigned)((p.n[0] / kCx) * (p.n[1] / kCy) * (p.n[2] / zc));
      if (eq)
        hipLaunchKernelGGL((k_ns_correct_zm<T, true>), dim3(nbc), dim3(kCThreads), 0, p.stream, U, Ut, Us, C,
                           (const T *)p.W, (const T *)p.P[0], (const T *)p.P[1], g, k, with_ut ? 1 : 0, zc, runs);
      else
        hipLaunchKernelGGL((k_ns_correct_zm<T, false>), dim3(nbc), dim3(kCThreads), 0, p.stream, U, Ut, Us, C,
                           (const T *)p.W, (const T *)p.P[0], (const T *)p.P[1], g, k, with_ut ? 1 : 0, zc, runs);
    } else
      hipLaunchKernelGGL((k_ns_correct<T, 3>), dim3(nb), dim3(kNsThreads), 0, p.stream, U, Ut, Us, C,
                         (const T *)p.W, (const T *)p.P[0], (const T *)p.P[1], g, k, with_ut ? 1 : 0, wk);
    e = hipGetLastError();
  }
  if (tm && e == hipSuccess) e = tm->end(p.stream);
  return e;
}

template hipError_t enqueue_momentum<double>(const Plan &, int, int, KernelTimer *, StepLink *);
template hipError_t enqueue_momentum<float>(const Plan &, int, int, KernelTimer *, StepLink *);

}  // namespace chib
