// Device kernels of one time step of the hybrid ghost-cell IB / Cahn-Hilliard method
// (Appendix A.1 and sections 4.2.2 and 4.3 of the paper), written for gfx950 (CDNA4):
// 64-wide wavefronts, 256-thread workgroups, 32 KB LDS tiles, XCD-aware tile order.
//
// Step pipeline (C^n in C[cur], C^(n-1) in C[1-cur]; the step overwrites C[1-cur]):
//   K1  rhs + Hartley transform along x     C^n, C^(n-1), faces -> W       (contiguous lines)
//   K2  Hartley transform along y (3D)      W -> W                          (strided columns)
//   K3  cosine transform along the bounded axis, division by (lam-a)(lam+alpha_s),
//       inverse cosine transform            W -> W                          (strided columns)
//   K4  Hartley transform along y (3D)      W -> W
//   K5  Hartley transform along x           W -> C[1-cur]  (= C* on every cell)
//   K6  contact-angle ghost fill of C       C[1-cur] at ghost cells
//   K7  no-penetration / Navier-slip fill of faces touching ghosts
//
// The Hartley transform H[k] = sum x[n] cas(2 pi k n / N) diagonalises the periodic second
// difference exactly as the Fourier transform does (modes k and N-k share an eigenvalue) and
// keeps every array real: N values per line, no half-spectrum padding.  Two real lines are
// transformed at once as the real and imaginary parts of one complex FFT.  The cosine
// transform (type II) diagonalises the second difference with reflecting box walls; it is
// computed from one complex FFT of the even/odd reordered sequence, again two lines at once.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <type_traits>

#include "kernels.h"

namespace chib {

namespace {

constexpr int kThreads = 256;

struct Dims {
  int nx, ny, nz;
  int lnx, lny, lnz;
  int64_t plane;
};

template <typename T>
struct RhsCoef {
  T pe_cn2;   // Pe / Cn^2
  T inv_dt;
  T S;
  T inv_cn2;  // 1 / Cn^2
  T inv_h;
  T inv_h2;
};

// The wall condition dphi/dn = 0 in the rhs (end of section 4.2.2, Eq. WallBCS): g at every ghost
// G becomes g_G + dg_G, dg_G = (phi~_M - phi~_G)/Cn^2 with phi~ = C~^3 - C~ - Cn^2 lap_h C~ the
// explicit chemical potential of the step (k_ghost_dphi).  Through lap_h(g) that changes Q by
// -2d dg_G/h^2 at the ghost and by +dg_G/h^2 at each face neighbour: a sparse patch over the
// ghosts and their neighbours, listed sorted by cell with the first entry of every x-row.  The rhs
// kernels add it in LDS before their x transform: the z-march reads its value dq per entry
// (k_patch_dq), the line-tiled and y-marching kernels form it from dg themselves.
// row == nullptr: no patch.
template <typename T>
struct RhsPatch {
  const int *row;    // [rows + 1]
  const int *cell;   // [np]
  const int *ref;    // [2d+1][np]: own ghost index, then the ghosts at +e_a and -e_a per axis, or -1
  const T *dg;       // [ghosts]
  const T *dq;       // [np] (z-march only)
  int np;
  T inv_h2;
};

// One entry's dq: the neighbouring ghosts' dg in a fixed order (+e_a, -e_a per axis), then the own one.
template <typename T, int D>
__device__ __forceinline__ T patch_dq(const int (&id)[2 * D + 1], const T *__restrict__ dg, T inv_h2) {
  T acc = T(0);
#pragma unroll
  for (int j = 1; j < 2 * D + 1; ++j) {
    const T v = dg[id[j] < 0 ? 0 : id[j]];
    acc += id[j] < 0 ? T(0) : v;
  }
  const T own = dg[id[0] < 0 ? 0 : id[0]];
  if (id[0] >= 0) acc -= T(2 * D) * own;
  return acc * inv_h2;
}

// The patch entries of the x-rows line0 .. line0 + L - 1 of a line tile in LDS (row l at l * pitch,
// element i at i + i/16); one entry per thread, no two entries share a cell.  The list range and the
// thread's first entry are requested by the constructor, before the tile's stencil loads, so that only
// the gather of dg is left when the tile is complete: forming dq here costs the small grids less than
// the launch of k_patch_dq did (2D 128 x 64: 2.1 us of a 37 us step).
template <typename T, int D>
struct TilePatch {
  int e0 = 0, e1 = 0, c = 0;
  int id[2 * D + 1];
  __device__ __forceinline__ void take(const RhsPatch<T> &rp, int e) {
    c = rp.cell[e];
#pragma unroll
    for (int j = 0; j < 2 * D + 1; ++j) id[j] = rp.ref[(int64_t)j * rp.np + e];
  }
  __device__ __forceinline__ TilePatch(const RhsPatch<T> &rp, int64_t line0, int L) {
    if (!rp.row) return;
    e0 = rp.row[line0];
    e1 = rp.row[line0 + L];
    if (e0 + (int)threadIdx.x < e1) take(rp, e0 + (int)threadIdx.x);
  }
  // (the caller has written the tile and holds it behind a barrier)
  __device__ __forceinline__ void add(T *__restrict__ s, const RhsPatch<T> &rp, int64_t line0, int lnx, int pitch) {
    for (int e = e0 + (int)threadIdx.x; e < e1; e += blockDim.x) {
      if (e >= e0 + (int)blockDim.x) take(rp, e);
      const int l = (int)((c >> lnx) - line0);
      const int i = c & ((1 << lnx) - 1);
      const T dq = patch_dq<T, D>(id, rp.dg, rp.inv_h2);
      {
#pragma clang fp contract(off)   // dq is rounded first, as the stored list's entries are
        s[l * pitch + i + (i >> 4)] += dq;
      }
    }
  }
};

// The same from dq per entry (z-march).
template <typename T>
__device__ __forceinline__ void patch_tile(T *__restrict__ s, const RhsPatch<T> &rp, int64_t line0, int lnx,
                                           int pitch, int e0, int e1) {
  for (int e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int c = rp.cell[e];
    const int l = (int)((c >> lnx) - line0);
    const int i = c & ((1 << lnx) - 1);
    s[l * pitch + i + (i >> 4)] += rp.dq[e];
  }
}

// ---------------------------------------------------------------------------------------
// Register DFTs of length R in {2, 4, 8, 16}, natural order in and out.  Forward uses
// exp(-2 pi i / R); INV the conjugate.  Twiddles are powers of w16 = exp(-2 pi i / 16).
constexpr double kC16[16] = {1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
                             0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
                             -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173,
                             0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613};
constexpr double kS16[16] = {0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613,
                             1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
                             0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
                             -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173};

// x <- x * w16^e (forward) or x * conj(w16^e) (INV); e is a compile-time constant after unrolling.
template <typename T, bool INV>
__device__ __forceinline__ void rot16(T &re, T &im, int e) {
  e &= 15;
  if (e == 0) return;
  if (e == 8) {
    re = -re;
    im = -im;
    return;
  }
  if (e == 4 || e == 12) {  // -i (forward, e=4) / +i
    const bool minus_i = (e == 4) != INV;
    const T r = re;
    if (minus_i) {
      re = im;
      im = -r;
    } else {
      re = -im;
      im = r;
    }
    return;
  }
  const T c = (T)kC16[e];
  const T sn = INV ? (T)kS16[e] : -(T)kS16[e];
  const T r = re;
  re = r * c - im * sn;
  im = r * sn + im * c;
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_reg(T *xr, T *xi);

template <typename T, int R1, int R2, bool INV>
__device__ __forceinline__ void dft_split(T *xr, T *xi) {
  constexpr int R = R1 * R2;
  T yr[R], yi[R];
#pragma unroll
  for (int n1 = 0; n1 < R1; ++n1) {
    T ar[R2], ai[R2];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) {
      ar[n2] = xr[n1 + R1 * n2];
      ai[n2] = xi[n1 + R1 * n2];
    }
    dft_reg<T, R2, INV>(ar, ai);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
      rot16<T, INV>(ar[k2], ai[k2], n1 * k2 * (16 / R));
      yr[n1 * R2 + k2] = ar[k2];
      yi[n1 * R2 + k2] = ai[k2];
    }
  }
#pragma unroll
  for (int k2 = 0; k2 < R2; ++k2) {
    T ar[R1], ai[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) {
      ar[n1] = yr[n1 * R2 + k2];
      ai[n1] = yi[n1 * R2 + k2];
    }
    dft_reg<T, R1, INV>(ar, ai);
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
      xr[k2 + R2 * k1] = ar[k1];
      xi[k2 + R2 * k1] = ai[k1];
    }
  }
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_reg(T *xr, T *xi) {
  if constexpr (R == 2) {
    const T ar = xr[0], ai = xi[0];
    xr[0] = ar + xr[1];
    xi[0] = ai + xi[1];
    xr[1] = ar - xr[1];
    xi[1] = ai - xi[1];
  } else if constexpr (R == 4) {
    const T ar = xr[0] + xr[2], ai = xi[0] + xi[2];
    const T br = xr[0] - xr[2], bi = xi[0] - xi[2];
    const T cr = xr[1] + xr[3], ci = xi[1] + xi[3];
    const T dr = xr[1] - xr[3], di = xi[1] - xi[3];
    xr[0] = ar + cr;
    xi[0] = ai + ci;
    xr[2] = ar - cr;
    xi[2] = ai - ci;
    if (!INV) {  // y1 = b - i d, y3 = b + i d
      xr[1] = br + di;
      xi[1] = bi - dr;
      xr[3] = br - di;
      xi[3] = bi + dr;
    } else {
      xr[1] = br - di;
      xi[1] = bi + dr;
      xr[3] = br + di;
      xi[3] = bi - dr;
    }
  } else if constexpr (R == 8) {
    dft_split<T, 2, 4, INV>(xr, xi);
  } else {
    static_assert(R == 16, "radix");
    dft_split<T, 4, 4, INV>(xr, xi);
  }
}

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v >> 1); }

// LDS address of element n of sequence b: b*ps + n*ns, plus padw extra elements after every
// 16 positions (keeps the stride-16 accesses of the radix-16 stages off a single bank).
__device__ __forceinline__ int lds_at(int b, int n, int ps, int ns, int padw) {
  return b * ps + n * ns + (n >> 4) * padw;
}

// Stages `tot` elements from global memory into LDS, element e read from src(e) and written to
// LDS slot dst(e): every thread issues kBatch independent loads before its LDS stores, so a tile
// costs one memory round trip per batch rather than one per element.
constexpr int kBatch = 8;
template <typename T, int NB = kBatch, typename Src, typename Dst>
__device__ __forceinline__ void stage_tile(T *__restrict__ s, int tot, Src src, Dst dst) {
  for (int e0 = threadIdx.x; e0 < tot; e0 += NB * blockDim.x) {
    T v[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int e = e0 + k * blockDim.x;
      v[k] = e < tot ? src(e) : T(0);
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int e = e0 + k * blockDim.x;
      if (e < tot) s[dst(e)] = v[k];
    }
  }
}

// w^r for r = 1..R-1 from w = w^1 by products of at most four factors.
template <typename T, int R>
__device__ __forceinline__ void twiddle_powers(T w1r, T w1i, T *wr, T *wi) {
  wr[1] = w1r;
  wi[1] = w1i;
#pragma unroll
  for (int r = 2; r < R; ++r) {
    const int a = (r & 1) ? r - 1 : r / 2;   // r = a + (r - a)
    const int c = r - a;
    wr[r] = wr[a] * wr[c] - wi[a] * wi[c];
    wi[r] = wr[a] * wi[c] + wi[a] * wr[c];
  }
}

// One Stockham stage of radix R over `np` sequences of length N in LDS.  p = 2^lp is the
// product of the radices of the previous stages.  Inputs are staged in registers.
template <typename T> struct Pair2;
template <> struct Pair2<double> { using type = double2; };
template <> struct Pair2<float> { using type = float2; };

// 16 bytes of a padded LDS tile at an element offset that is only a multiple of 2: the tiles put a
// 2-element gap after every 16 positions, so a 4-float group need not be 16-byte aligned.  One
// 16-byte access for double2, two 8-byte ones for float4.
template <typename T, typename V>
__device__ __forceinline__ void lds_put16(T *a, const V &v) {
  if constexpr (sizeof(T) == 8) {
    *reinterpret_cast<V *>(a) = v;
  } else {
    using H = typename Pair2<T>::type;
    const H *h = reinterpret_cast<const H *>(&v);
    *reinterpret_cast<H *>(a) = h[0];
    *reinterpret_cast<H *>(a + 2) = h[1];
  }
}
template <typename V, typename T>
__device__ __forceinline__ V lds_get16(const T *a) {
  if constexpr (sizeof(T) == 8) {
    return *reinterpret_cast<const V *>(a);
  } else {
    using H = typename Pair2<T>::type;
    V v;
    H *h = reinterpret_cast<H *>(&v);
    h[0] = *reinterpret_cast<const H *>(a);
    h[1] = *reinterpret_cast<const H *>(a + 2);
    return v;
  }
}

// PAIRED: the imaginary part sits right after the real part (io == 1), and both move as one
// 2-element LDS access; with the sequence index fastest across lanes (bfast) the lanes served
// together then touch distinct bank groups, where two separate accesses would collide.
template <typename T, int R, int IT, bool INV, bool PAIRED = false>
__device__ __forceinline__ void fft_stage(T *__restrict__ s, int logN, int lognp, int ps, int ns, int io, int padw,
                                          bool bfast, int lp, const T *__restrict__ twr, const T *__restrict__ twi) {
  using P2 = typename Pair2<T>::type;
  constexpr int LR = ilog2c(R);
  const int nt = blockDim.x;
  const int tid = threadIdx.x;
  const int lq = logN - LR;
  const int total = 1 << (lognp + lq);
  const int p = 1 << lp;
  const int sh = logN - LR - lp;
  const int npm = (1 << lognp) - 1;
  // lds_at(b, n + r d) = lds_at(b, n) + r (d ns + (d / 16) padw) when d is a multiple of 16, and
  // lds_at(b, n) + r d ns when n + (R - 1) d stays in n's group of 16 (d = 1, n a multiple of R)
  // (radix 16 keeps the general form: the linear one would cost it 25 VGPRs and a wave per SIMD)
  const bool rlin = R <= 8 && lq >= 4, wlin = R <= 8 && (lp >= 4 || lp == 0);
  const int rst = rlin ? (ns << lq) + (padw << (lq - 4)) : 0;
  const int wst = lp >= 4 ? (ns << lp) + (padw << (lp - 4)) : ns;
  T xr[IT][R], xi[IT][R];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int item = tid + it * nt;
    if (item < total) {
      int b, i;
      if (bfast) {
        b = item & npm;
        i = item >> lognp;
      } else {
        i = item & ((1 << lq) - 1);
        b = item >> lq;
      }
      auto rd = [&](int r, int a) {
        if constexpr (PAIRED) {
          const P2 v = *reinterpret_cast<const P2 *>(s + a);
          xr[it][r] = v.x;
          xi[it][r] = v.y;
        } else {
          xr[it][r] = s[a];
          xi[it][r] = s[a + io];
        }
      };
      if (rlin) {   // inputs 2^lq >= 16 apart: the padded address is linear in r
        const int a0 = lds_at(b, i, ps, ns, padw);
#pragma unroll
        for (int r = 0; r < R; ++r) rd(r, a0 + r * rst);
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) rd(r, lds_at(b, i + (r << lq), ps, ns, padw));
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int item = tid + it * nt;
    if (item < total) {
      int b, i;
      if (bfast) {
        b = item & npm;
        i = item >> lognp;
      } else {
        i = item & ((1 << lq) - 1);
        b = item >> lq;
      }
      const int k = i & (p - 1);
      if (lp > 0) {
        const int m = k << sh;
        T wr[R], wi[R];
        twiddle_powers<T, R>(twr[m], INV ? -twi[m] : twi[m], wr, wi);
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const T ur = xr[it][r];
          xr[it][r] = ur * wr[r] - xi[it][r] * wi[r];
          xi[it][r] = ur * wi[r] + xi[it][r] * wr[r];
        }
      }
      dft_reg<T, R, INV>(xr[it], xi[it]);
      const int j = ((i - k) << LR) + k;
      auto wr_ = [&](int r, int a) {
        if constexpr (PAIRED) {
          P2 v;
          v.x = xr[it][r];
          v.y = xi[it][r];
          *reinterpret_cast<P2 *>(s + a) = v;
        } else {
          s[a] = xr[it][r];
          s[a + io] = xi[it][r];
        }
      };
      if (wlin) {   // outputs p apart with p >= 16, or p = 1 (then all R in one padding group)
        const int a0 = lds_at(b, j, ps, ns, padw);
#pragma unroll
        for (int r = 0; r < R; ++r) wr_(r, a0 + r * wst);
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) wr_(r, lds_at(b, j + r * p, ps, ns, padw));
      }
    }
  }
  __syncthreads();
}

// Complex FFT of 2^lognp independent length-2^logN sequences held in LDS: mixed-radix
// Stockham autosort with register-resident radix-16 butterflies (then 8, 4 or 2 for the
// remaining factor).  E bounds the tile (elements of T) so that every thread holds at most
// 16 complex values per stage.  No 1/N scaling.
template <typename T, int E, bool INV, int MAXR = 16, int NT = 256, bool PAIRED = false>
__device__ __forceinline__ void lds_fft(T *__restrict__ s, int logN, int lognp, int ps, int ns, int io, int padw,
                                        bool bfast, const T *__restrict__ twr, const T *__restrict__ twi) {
  constexpr int IT16 = (E / 2 / 16 + NT - 1) / NT;
  constexpr int IT8 = (E / 2 / 8 + NT - 1) / NT;
  constexpr int IT4 = (E / 2 / 4 + NT - 1) / NT;
  constexpr int IT2 = (E / 2 / 2 + NT - 1) / NT;
  int lp = 0;
  int rem = logN;
  if constexpr (MAXR >= 16) {
    while (rem >= 4) {
      fft_stage<T, 16, IT16, INV, PAIRED>(s, logN, lognp, ps, ns, io, padw, bfast, lp, twr, twi);
      lp += 4;
      rem -= 4;
    }
  } else if constexpr (MAXR == 4) {
    while (rem >= 2) {
      fft_stage<T, 4, IT4, INV, PAIRED>(s, logN, lognp, ps, ns, io, padw, bfast, lp, twr, twi);
      lp += 2;
      rem -= 2;
    }
  } else {
    while (rem >= 3) {
      fft_stage<T, 8, IT8, INV, PAIRED>(s, logN, lognp, ps, ns, io, padw, bfast, lp, twr, twi);
      lp += 3;
      rem -= 3;
    }
  }
  if (rem == 3) fft_stage<T, 8, IT8, INV, PAIRED>(s, logN, lognp, ps, ns, io, padw, bfast, lp, twr, twi);
  else if (rem == 2) fft_stage<T, 4, IT4, INV, PAIRED>(s, logN, lognp, ps, ns, io, padw, bfast, lp, twr, twi);
  else if (rem == 1) fft_stage<T, 2, IT2, INV, PAIRED>(s, logN, lognp, ps, ns, io, padw, bfast, lp, twr, twi);
}

// Padded LDS pitch of a contiguous line of n elements (one pad element per 16).
__host__ __device__ __forceinline__ int line_pitch(int n) { return n + (n >> 4); }
// Padded LDS size (elements) of a tile of B interleaved columns by N positions.
__host__ __device__ __forceinline__ int col_tile(int N, int B) { return N * B + (N >> 4) * 2; }

// ---------------------------------------------------------------------------------------
// Right-hand side Q of the first Helmholtz equation at one cell:
//   Q = (Pe/Cn^2)(C^/dt - div_h(u C~)) + lap_h((C~^3 - C~ - S C~)/Cn^2)
// with C~ = 2C^n - C^(n-1), C^ = 2C^n - C^(n-1)/2; periodic axes wrap, the bounded (last)
// axis reflects for the Laplacian and has zero normal velocity on its box walls.
// The 2D expression on the values of C~ around the cell (v0, x+-1, y+-1, the latter already v0 beyond a
// wall) and its faces: shared by the line-tiled and the y-marching kernel.  Which products join which sums is
// written out and nothing else is contracted: left to the compiler, the two kernels differed in the last bits,
// and with them a state stepped alone and in a batch too wide for the march.
template <typename T>
__device__ __forceinline__ T rhs_2d(T v0, T cxp, T cxm, T cyp, T cym, T f0, T f0m, T f1, T f1m, bool top, bool bot,
                                    T cn, T cp, const RhsCoef<T> &cf) {
#pragma clang fp contract(off)
  auto bulk = [&](T v) {   // v^3 - v - S v
#pragma clang fp contract(off)
    return fma(-cf.S, v, fma(v * v, v, -v));
  };
  T flux = fma(f0, v0 + cxp, -(f0m * (cxm + v0)));
  const T ft = f1 * (v0 + cyp), fb = f1m * (cym + v0);
  flux += (top ? T(0) : ft) - (bot ? T(0) : fb);
  const T gx = fma(bulk(cxp), cf.inv_cn2, bulk(cxm) * cf.inv_cn2);
  const T gy = fma(bulk(cyp), cf.inv_cn2, bulk(cym) * cf.inv_cn2);
  const T g0 = bulk(v0) * cf.inv_cn2;
  const T A = flux * T(0.5) * cf.inv_h;
  const T cc = fma(T(2), cn, T(-0.5) * cp);
  return fma(fma(T(-4), g0, gx + gy), cf.inv_h2, cf.pe_cn2 * fma(cc, cf.inv_dt, -A));
}

// The same in 3D, for the line-tiled kernels (beyond a wall the caller passes the cell's own C~ and any face).
template <typename T>
__device__ __forceinline__ T rhs_3d(T v0, T cxp, T cxm, T cyp, T cym, T czp, T czm, T f0, T f0m, T f1, T f1m, T f2,
                                    T f2m, bool top, bool bot, T cn, T cp, const RhsCoef<T> &cf) {
  auto gf = [&](T v) { return (v * v * v - v - cf.S * v) * cf.inv_cn2; };
  T flux = f0 * (v0 + cxp) - f0m * (cxm + v0);
  T gsum = gf(cxp) + gf(cxm);
  flux += f1 * (v0 + cyp) - f1m * (cym + v0);
  gsum += gf(cyp) + gf(cym);
  flux += (top ? T(0) : f2 * (v0 + czp)) - (bot ? T(0) : f2m * (czm + v0));
  gsum += gf(czp) + gf(czm);
  const T A = flux * T(0.5) * cf.inv_h;
  const T lap = (gsum - T(6) * gf(v0)) * cf.inv_h2;
  const T cc = T(2) * cn - T(0.5) * cp;
  return cf.pe_cn2 * (cc * cf.inv_dt - A) + lap;
}

template <typename T, int D>
__device__ __forceinline__ T rhs_at(const T *__restrict__ Cn, const T *__restrict__ Cp, const T *__restrict__ F0,
                                    const T *__restrict__ F1, const T *__restrict__ F2, int i, int j, int k,
                                    const Dims &dm, const RhsCoef<T> &cf) {
  const int nx = dm.nx;
  const int64_t c = (int64_t)i + (int64_t)nx * ((int64_t)j + (int64_t)dm.ny * k);
  auto ct = [&](int64_t q) { return T(2) * Cn[q] - Cp[q]; };
  const int64_t rowb = c - i;
  const int ip = (i + 1) & (nx - 1), im = (i - 1) & (nx - 1);
  const T c0 = ct(c);
  const T cxp = ct(rowb + ip), cxm = ct(rowb + im);
  if constexpr (D == 2) {   // (every load happens, from the cell itself beyond a wall)
    const bool top = (j == dm.ny - 1), bot = (j == 0);
    const int64_t cu = top ? c : c + nx, cd = bot ? c : c - nx;
    const T cyp = ct(cu), cym = ct(cd);
    return rhs_2d(c0, cxp, cxm, cyp, cym, F0[c], F0[rowb + im], F1[c], F1[cd], top, bot, Cn[c], Cp[c], cf);
  }
  const int jp = (j + 1) & (dm.ny - 1), jm = (j - 1) & (dm.ny - 1);
  const int64_t cyp_i = c + (int64_t)(jp - j) * nx, cym_i = c + (int64_t)(jm - j) * nx;
  const bool top = (k == dm.nz - 1), bot = (k == 0);
  const int64_t czp_i = top ? c : c + dm.plane, czm_i = bot ? c : c - dm.plane;
  return rhs_3d(c0, cxp, cxm, ct(cyp_i), ct(cym_i), ct(czp_i), ct(czm_i), F0[c], F0[rowb + im], F1[c], F1[cym_i],
                F2[c], F2[czm_i], top, bot, Cn[c], Cp[c], cf);
}

// Untangles the complex FFT of the pair (a + i b) into the Hartley transforms of a and b:
// with Z[k] = p + iq and Z[N-k] = r + is, H_a[k] = (p - q + r + s)/2, H_b[k] = (p + q - r + s)/2.
template <typename T>
__device__ __forceinline__ T hartley_of_pair(T p, T q, T r, T s, int par) {
  return par ? (p + q - r + s) * T(0.5) : (p - q + r + s) * T(0.5);
}

// ---------------------------------------------------------------------------------------
// K1: rhs of L consecutive x-lines into LDS, Hartley transform along x, store to W.
// CLN (3D) fixes the line length: a thread then forms 16 bytes of adjacent cells of every RS-th line from
// 16-byte loads, with the x neighbours from the lanes beside it: 15 requests a thread where the general form
// makes 20 a cell.  The general form was bound by its requests, this one by the memory round trip: 128^3 FP64
// 38 -> 28 us (3.6 TB/s over 48 bytes a cell), FP32 26 -> 17; 64^3 10.5 -> 9.1; 128x256x256 155 -> 104.
template <typename T, int D, int E, int U = 1, int MAXR = 16, int CLN = 0>
__device__ __forceinline__ void rhs_xdht_body(unsigned char *smem_raw, const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                       const T *__restrict__ F0, const T *__restrict__ F1,
                                                       const T *__restrict__ F2, T *__restrict__ W, Dims dm,
                                                       RhsCoef<T> cf, int logL, const T *__restrict__ twr,
                                                       const T *__restrict__ twi, int tile, const RhsPatch<T> &rp) {
  T *s = reinterpret_cast<T *>(smem_raw);
  const int L = 1 << logL;
  const int nx = dm.nx;
  const int line0 = tile * L;
  const int tot = L << dm.lnx;
  const int pitch = line_pitch(nx);
  TilePatch<T, D> patch(rp, line0, L);
  if constexpr (CLN != 0) {
    constexpr int CP = 16 / (int)sizeof(T), NX = 1 << CLN, RS = CP * kThreads / NX;
    typedef T FV __attribute__((ext_vector_type(CP)));
    static_assert(D == 3 && RS >= 1, "fixed-size line");
    const int i = (threadIdx.x & (NX / CP - 1)) * CP, im = (i - 1) & (NX - 1), ip = (i + CP) & (NX - 1);
    const int lane = threadIdx.x & 63;
    const bool first = lane == 0 || i == 0, last = lane == 63 || i + CP == NX;   // no lane of the line beside
    auto ld = [](const T *a) { return *reinterpret_cast<const FV *>(a); };
    for (int l = threadIdx.x / (NX / CP); l < L; l += RS) {
      const int line = line0 + l, j = line & (dm.ny - 1), k = line >> dm.lny;
      const bool top = k == dm.nz - 1, bot = k == 0;
      const int64_t row = (int64_t)line << CLN, c = row + i;
      const int64_t yp = c + ((int64_t)(((j + 1) & (dm.ny - 1)) - j) << CLN);
      const int64_t ym = c + ((int64_t)(((j - 1) & (dm.ny - 1)) - j) << CLN);
      const int64_t zp = top ? c : c + dm.plane, zm = bot ? c : c - dm.plane;
      const FV a0 = ld(Cn + c), b0 = ld(Cp + c), ayp = ld(Cn + yp), byp = ld(Cp + yp), aym = ld(Cn + ym), bym = ld(Cp + ym);
      const FV azp = ld(Cn + zp), bzp = ld(Cp + zp), azm = ld(Cn + zm), bzm = ld(Cp + zm);
      const FV f0 = ld(F0 + c), f1 = ld(F1 + c), f1m = ld(F1 + ym), f2 = ld(F2 + c), f2m = ld(F2 + zm);
      T cl = T(0), fl = T(0), cr = T(0);
      if (first) {
        cl = T(2) * Cn[row + im] - Cp[row + im];
        fl = F0[row + im];
      }
      if (last) cr = T(2) * Cn[row + ip] - Cp[row + ip];
      const FV v = T(2) * a0 - b0, vyp = T(2) * ayp - byp, vym = T(2) * aym - bym;
      const FV vzp = T(2) * azp - bzp, vzm = T(2) * azm - bzm;
      const T below = __shfl_up(v[CP - 1], 1), fbelow = __shfl_up(f0[CP - 1], 1), above = __shfl_down(v[0], 1);
      T *d = s + l * pitch + i + (i >> 4);
#pragma unroll
      for (int m = 0; m < CP; ++m) {
        const T cxm = m ? v[m ? m - 1 : 0] : (first ? cl : below), fm = m ? f0[m ? m - 1 : 0] : (first ? fl : fbelow);
        const T cxp = m < CP - 1 ? v[m < CP - 1 ? m + 1 : 0] : (last ? cr : above);
        d[m] = rhs_3d(v[m], cxp, cxm, vyp[m], vym[m], vzp[m], vzm[m], f0[m], fm, f1[m], f1m[m], f2[m], f2m[m], top, bot,
                      a0[m], b0[m], cf);
      }
    }
  } else {
    // U cells per iteration so that their loads are in flight together
    for (int e0 = threadIdx.x; e0 < tot; e0 += U * blockDim.x) {
      T q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * blockDim.x;
        if (e < tot) {
          const int l = e >> dm.lnx;
          const int i = e & (nx - 1);
          const int line = line0 + l;
          int j, k;
          if (D == 2) {
            j = line;
            k = 0;
          } else {
            j = line & (dm.ny - 1);
            k = line >> dm.lny;
          }
          q[u] = rhs_at<T, D>(Cn, Cp, F0, F1, F2, i, j, k, dm, cf);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * blockDim.x;
        if (e < tot) {
          const int l = e >> dm.lnx;
          const int i = e & (nx - 1);
          s[l * pitch + i + (i >> 4)] = q[u];
        }
      }
    }
  }
  if (patch.e1 > patch.e0) {   // the ghost patch of the tile's lines
    __syncthreads();
    patch.add(s, rp, line0, dm.lnx, pitch);
  }
  __syncthreads();
  lds_fft<T, E, false, MAXR>(s, dm.lnx, logL - 1, 2 * pitch, 1, pitch, 1, false, twr, twi);
  const int half = tot >> 1;
  for (int e = threadIdx.x; e < half; e += blockDim.x) {
    const int b = e >> dm.lnx;
    const int kx = e & (nx - 1);
    const int kk = (nx - kx) & (nx - 1);
    const T *pb = s + b * 2 * pitch;
    const int ak = kx + (kx >> 4), an = kk + (kk >> 4);
    const T p = pb[ak], q = pb[pitch + ak], r = pb[an], sv = pb[pitch + an];
    T *o = W + (int64_t)(line0 + 2 * b) * nx + kx;
    o[0] = (p - q + r + sv) * T(0.5);
    o[nx] = (p + q - r + sv) * T(0.5);
  }
}

template <typename T, int D, int E, int U = 1, int MAXR = 16, int CLN = 0>
__global__ __launch_bounds__(kThreads) void k_rhs_xdht(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                       const T *__restrict__ F0, const T *__restrict__ F1,
                                                       const T *__restrict__ F2, T *__restrict__ W, Dims dm,
                                                       RhsCoef<T> cf, int logL, const T *__restrict__ twr,
                                                       const T *__restrict__ twi, RhsPatch<T> rp) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if constexpr (CLN != 0) {
    dm.lnx = CLN;
    dm.nx = 1 << CLN;
  }
  rhs_xdht_body<T, D, E, U, MAXR, CLN>(smem_raw, Cn, Cp, F0, F1, F2, W, dm, cf, logL, twr, twi, xcd_tile(blockIdx.x, gridDim.x),
                                  rp);
}

// Extra LDS of the y-marching K1 (two rows of C~ for the x neighbours) over the line tile.
__host__ __device__ __forceinline__ int ym_extra(int nx) { return 2 * nx; }

// K1 for 2D grids, marching in y: the workgroup owns the L rows of its tile across the whole x
// range, thread t the columns x = t + 256 m (m < XM, nx <= 256 XM).  C~ = 2C^n - C^(n-1) of row
// y-1 and the raw C^n, C^(n-1) of rows y and y+1 stay in registers, so every value is loaded
// once and y neighbours never leave the thread; the raw values and the faces of row y+2 are requested
// once row y is computed (a row's arithmetic is far shorter than a memory round trip; with the faces requested
// at the head of their own row, 72 instead of 63 us per step of 32 cases, 5.8 million cells, FP64, at three
// waves per SIMD, which is what the tile and ring leave in LDS anyway).  x neighbours come from a two-row
// ring of C~ in LDS (one barrier per row); each Q row goes straight into the line tile, which
// then goes through the same x transform as the line-tiled K1.
template <typename T, int XM, int R>
__device__ __forceinline__ void rhs_ym_body(unsigned char *smem_raw, const T *__restrict__ Cn,
                                            const T *__restrict__ Cp, const T *__restrict__ F0,
                                            const T *__restrict__ F1, T *__restrict__ W, Dims dm, RhsCoef<T> cf,
                                            int logL, const T *__restrict__ twr, const T *__restrict__ twi,
                                            int tile, const RhsPatch<T> &rp) {
  const int nx = dm.nx, ny = dm.ny;
  const int L = 1 << logL;
  const int pitch = line_pitch(nx);
  T *fb = reinterpret_cast<T *>(smem_raw);           // L rows x pitch: Q, then its transform
  T *xr = fb + L * pitch;                             // 2 rows x nx: C~ of the current row
  const int y0 = tile * L;
  const int tid = threadIdx.x;
  TilePatch<T, 2> patch(rp, y0, L);
  auto rowp = [&](const T *__restrict__ a, int y) { return a + (int64_t)(y < 0 ? 0 : (y >= ny ? ny - 1 : y)) * nx; };
  // per column: C~ of row y-1, the raw C^n, C^(n-1) of rows y, y+1 and y+2 (in flight), F1 of row y-1
  T cm[XM], a0[XM], b0[XM], a1[XM], b1[XM], an[XM], bn[XM], f1m[XM];
#pragma unroll
  for (int m = 0; m < XM; ++m) {
    const int i = tid + 256 * m;
    if (i < nx) {
      const T a_m = rowp(Cn, y0 - 1)[i], b_m = rowp(Cp, y0 - 1)[i];
      a0[m] = rowp(Cn, y0)[i];
      b0[m] = rowp(Cp, y0)[i];
      a1[m] = rowp(Cn, y0 + 1)[i];
      b1[m] = rowp(Cp, y0 + 1)[i];
      f1m[m] = rowp(F1, y0 - 1)[i];
      an[m] = rowp(Cn, y0 + 2)[i];
      bn[m] = rowp(Cp, y0 + 2)[i];
      cm[m] = T(2) * a_m - b_m;
    }
  }
  // faces of the row and of the next one (in flight)
  T f0[XM], f0m[XM], f1[XM], g0[XM], g0m[XM], g1[XM];
  auto faces = [&](int m, int y, T *u0, T *u0m, T *u1) {
    const int i = tid + 256 * m;
    const T *r0 = rowp(F0, y), *r1 = rowp(F1, y);
    u0[m] = r0[i];
    u0m[m] = r0[(i - 1) & (nx - 1)];
    u1[m] = r1[i];
  };
#pragma unroll
  for (int m = 0; m < XM; ++m)
    if (tid + 256 * m < nx) {
      faces(m, y0, f0, f0m, f1);
      faces(m, y0 + 1, g0, g0m, g1);
    }
  for (int r = 0; r < L; ++r) {
    const int y = y0 + r;
    const bool top = y == ny - 1, bot = y == 0;
    T *xb = xr + (r & 1) * nx;
#pragma unroll
    for (int m = 0; m < XM; ++m) {
      const int i = tid + 256 * m;
      if (i < nx) xb[i] = T(2) * a0[m] - b0[m];
    }
    __syncthreads();   // the row is in LDS; the ring slot written next row was last read two rows ago
#pragma unroll
    for (int m = 0; m < XM; ++m) {
      const int i = tid + 256 * m;
      if (i < nx) {
        const T v0 = T(2) * a0[m] - b0[m];
        const T cxp = xb[(i + 1) & (nx - 1)], cxm = xb[(i - 1) & (nx - 1)];
        const T cyp = top ? v0 : T(2) * a1[m] - b1[m], cym = bot ? v0 : cm[m];
        fb[r * pitch + i + (i >> 4)] =
            rhs_2d(v0, cxp, cxm, cyp, cym, f0[m], f0m[m], f1[m], f1m[m], top, bot, a0[m], b0[m], cf);
        // slide the window down one row and request the row after next
        cm[m] = v0;
        a0[m] = a1[m];
        b0[m] = b1[m];
        a1[m] = an[m];
        b1[m] = bn[m];
        f1m[m] = f1[m];
        f0[m] = g0[m];
        f0m[m] = g0m[m];
        f1[m] = g1[m];
        if (r + 2 < L) {
          an[m] = rowp(Cn, y + 3)[i];
          bn[m] = rowp(Cp, y + 3)[i];
          faces(m, y + 2, g0, g0m, g1);
        }
      }
    }
  }
  if (patch.e1 > patch.e0) {   // the ghost patch of the tile's rows
    __syncthreads();
    patch.add(fb, rp, y0, dm.lnx, pitch);
  }
  __syncthreads();
  lds_fft<T, tile_elems<T>(), false, R>(fb, dm.lnx, logL - 1, 2 * pitch, 1, pitch, 1, false, twr, twi);
  const int half = (L * nx) >> 1;
  for (int e = tid; e < half; e += blockDim.x) {
    const int b = e >> dm.lnx;
    const int kx = e & (nx - 1);
    const int kk = (nx - kx) & (nx - 1);
    const T *pb = fb + b * 2 * pitch;
    const int ak = kx + (kx >> 4), a2 = kk + (kk >> 4);
    const T p = pb[ak], q = pb[pitch + ak], rr = pb[a2], sv = pb[pitch + a2];
    T *o = W + (int64_t)(y0 + 2 * b) * nx + kx;
    o[0] = (p - q + rr + sv) * T(0.5);
    o[nx] = (p + q - rr + sv) * T(0.5);
  }
}

template <typename T, int XM, int R>
__global__ __launch_bounds__(kThreads, R == 8 && XM < 4 ? 4 : 3) void k_rhs_xdht_ym(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                          const T *__restrict__ F0, const T *__restrict__ F1,
                                                          T *__restrict__ W, Dims dm, RhsCoef<T> cf, int logL,
                                                          const T *__restrict__ twr, const T *__restrict__ twi,
                                                          RhsPatch<T> rp) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  rhs_ym_body<T, XM, R>(smem_raw, Cn, Cp, F0, F1, W, dm, cf, logL, twr, twi, xcd_tile(blockIdx.x, gridDim.x), rp);
}

// K1 for 3D grids, marching in z (2.5D blocking): a workgroup owns L consecutive y rows and
// a chunk of ZC planes.  Thread t owns the x positions x = t + 256 m (m < nx/256, nx >= 256)
// of rows -1..L of the tile, i.e. whole column segments including the two halo rows, and
// keeps C~ of planes z-1, z, z+1 in registers, so y and z neighbours never leave the thread;
// x neighbours (of C~ and of the x faces) come from LDS.  Each plane's L rows of Q go through
// the same Hartley transform as K1 and are stored to W.  Requires nx a multiple of 256.
// Software pipeline: while plane z is transformed and stored, the loads of C^n, C^(n-1) for
// plane z+2 and of the faces and patch entries for plane z+1 are in flight, so a plane only
// ever waits for data requested one plane earlier.  The FFT twiddles are read from LDS: vector
// memory counters retire in order, so a global twiddle load inside the FFT would also wait for
// every request in flight.
template <typename T, int L, int XM, int R, bool SPLIT = false>
__global__ __launch_bounds__(kThreads, (L == 2 && XM == 1 && R == 4) ? 3 : 1) void k_rhs_xdht_zm(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                          const T *__restrict__ F0, const T *__restrict__ F1,
                                                          const T *__restrict__ F2, T *__restrict__ W, Dims dm,
                                                          RhsCoef<T> cf, int zc_log, const T *__restrict__ twr,
                                                          const T *__restrict__ twi, RhsPatch<T> rp) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int nx = 256 * XM, lnx = ilog2c(nx);   // the launcher takes this kernel only for nx = 256 XM
  T *plane = reinterpret_cast<T *>(smem_raw);        // L rows x nx: C~ of plane z
  T *fxp = plane + L * nx;                             // L rows x nx: x faces of plane z
  const int pitch = line_pitch(nx);
  T *fb = fxp + L * nx;                                // L rows x pitch: FFT tile
  T *tw = fb + L * pitch;                              // 2 x nx: the x twiddles (read from LDS, so that
                                                       // the FFT never waits on the global requests in flight)
  const int nyt = dm.ny / L;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int yt = t % nyt;
  const int zc = t / nyt;
  const int y0 = yt * L;
  const int ZC = 1 << zc_log;
  const int z0 = zc * ZC;
  const int tid = threadIdx.x;
  auto gf = [&](T v) { return (v * v * v - v - cf.S * v) * cf.inv_cn2; };
  auto row_of = [&](int r) { return (y0 + r + dm.ny) & (dm.ny - 1); };  // r in -1..L
  auto zbase = [&](int z) { return (int64_t)(z < 0 ? 0 : (z >= dm.nz ? dm.nz - 1 : z)) * dm.plane; };
  // C~ at rows -1..L of planes z-1 (rows 0..L-1 kept), z, z+1; C^ = 2C^n - C^(n-1)/2 of the own
  // rows of planes z, z+1; raw C^n, C^(n-1) of plane z+2 in flight
  T cm[XM][L], c0[XM][L + 2], cp[XM][L + 2], h0[XM][L], hp[XM][L], na[XM][L + 2], nb[XM][L + 2];
  // faces of plane z (F1 at rows -1..L-1, z faces of plane z-1 below) and of plane z+1 in flight
  T f0[XM][L], f1[XM][L + 1], f2[XM][L], uzm[XM][L], nf0[XM][L], nf1[XM][L + 1], nf2[XM][L];
  // Cache policy: C^n, C^(n-1) and the x and z faces are read here for the last time in the step and
  // W is read next by another pass over the whole grid, so all of them go as non-temporal (streaming)
  // accesses that leave the L2 and the Infinity Cache to the y faces (rows shared by neighbouring
  // tiles) and to the next passes; measured 181 -> 168 us together with the x pass out's streaming reads
  auto load_c = [&](int z) {   // planes beyond the box reflect onto the boundary plane
    const int64_t zb = zbase(z);
#pragma unroll
    for (int m = 0; m < XM; ++m)
#pragma unroll
      for (int r = 0; r < L + 2; ++r) {
        const int64_t q = zb + (int64_t)row_of(r - 1) * nx + tid + 256 * m;
        na[m][r] = __builtin_nontemporal_load(Cn + q);
        nb[m][r] = __builtin_nontemporal_load(Cp + q);
      }
  };
  auto load_f = [&](int z) {
    const int64_t zb = zbase(z);
#pragma unroll
    for (int m = 0; m < XM; ++m) {
#pragma unroll
      for (int r = 0; r < L; ++r) {
        const int64_t q = zb + (int64_t)row_of(r) * nx + tid + 256 * m;
        nf0[m][r] = __builtin_nontemporal_load(F0 + q);
        nf2[m][r] = __builtin_nontemporal_load(F2 + q);
      }
#pragma unroll
      for (int r = 0; r < L + 1; ++r) nf1[m][r] = F1[zb + (int64_t)row_of(r - 1) * nx + tid + 256 * m];
    }
  };
  auto take_c = [&](T (&dst)[XM][L + 2], T (&hat)[XM][L]) {
#pragma unroll
    for (int m = 0; m < XM; ++m)
#pragma unroll
      for (int r = 0; r < L + 2; ++r) {
        dst[m][r] = T(2) * na[m][r] - nb[m][r];
        if (r >= 1 && r <= L) hat[m][r - 1] = T(2) * na[m][r] - T(0.5) * nb[m][r];
      }
  };
  auto take_f = [&]() {
#pragma unroll
    for (int m = 0; m < XM; ++m) {
#pragma unroll
      for (int r = 0; r < L; ++r) {
        uzm[m][r] = f2[m][r];
        f0[m][r] = nf0[m][r];
        f2[m][r] = nf2[m][r];
      }
#pragma unroll
      for (int r = 0; r < L + 1; ++r) f1[m][r] = nf1[m][r];
    }
  };
  if constexpr (!SPLIT)
    for (int e = tid; e < nx; e += blockDim.x) {   // ordered before the first FFT by the plane barrier
      tw[e] = twr[e];
      tw[nx + e] = twi[e];
    }
  // prologue: C~ of planes z0-1, z0, z0+1 and the faces of plane z0 (and the z faces below it)
  {
    T th[XM][L];
    load_c(z0 - 1);   // the reflecting wall below plane 0 is plane 0 itself
    take_c(cp, th);
#pragma unroll
    for (int m = 0; m < XM; ++m)
#pragma unroll
      for (int r = 0; r < L; ++r) {
        cm[m][r] = cp[m][r + 1];
        f2[m][r] = z0 > 0 ? F2[zbase(z0 - 1) + (int64_t)row_of(r) * nx + tid + 256 * m] : T(0);
      }
  }
  load_c(z0);
  take_c(c0, h0);
  load_c(z0 + 1);
  take_c(cp, hp);
  load_f(z0);
  take_f();
  // ghost patch (SPLIT: added by the caller afterwards): the entries of the tile's rows of a plane
  // are requested one plane ahead and added to its Q tile after the stencil
  constexpr int PF = 2;
  const bool patch = !SPLIT && rp.row != nullptr;
  int e_lo = 0, e_hi = 0, n_lo = 0, n_hi = 0, pc[PF], npc[PF];
  T pd[PF], npd[PF];
  auto range_of = [&](int z, int &lo, int &hi) {
    const int64_t R0 = (int64_t)z * dm.ny + y0;
    lo = rp.row[R0];
    hi = rp.row[R0 + L];
  };
  // every request is unconditional (indices clamped into the list, which is not empty when the
  // patch is on): a register with a default on one path would have to wait for the load in flight
  auto load_p = [&](int lo, int hi) {
    const int last = hi > 0 ? hi - 1 : 0;
#pragma unroll
    for (int k = 0; k < PF; ++k) {
      const int e = min(lo + tid + 256 * k, last);
      npc[k] = rp.cell[e];
      npd[k] = rp.dq[e];
    }
  };
  const int zlast = z0 + ZC - 1;
  if (patch) {
    range_of(z0, e_lo, e_hi);
    load_p(e_lo, e_hi);
#pragma unroll
    for (int k = 0; k < PF; ++k) {
      pc[k] = npc[k];
      pd[k] = npd[k];
    }
    range_of(min(z0 + 1, zlast), n_lo, n_hi);
  }
  // plane z+1 becomes current: the first use of the requests made at the top of plane z, placed
  // before the stores of W so that the wait does not include their completion
  int nn_lo = 0, nn_hi = 0;
  auto rotate = [&]() {
#pragma unroll
    for (int m = 0; m < XM; ++m) {
#pragma unroll
      for (int r = 0; r < L; ++r) cm[m][r] = c0[m][r + 1];
#pragma unroll
      for (int r = 0; r < L + 2; ++r) c0[m][r] = cp[m][r];
#pragma unroll
      for (int r = 0; r < L; ++r) h0[m][r] = hp[m][r];
    }
    take_c(cp, hp);
    take_f();
    if (patch) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        pc[k] = npc[k];
        pd[k] = npd[k];
      }
      e_lo = n_lo;
      e_hi = n_hi;
      n_lo = nn_lo;
      n_hi = nn_hi;
    }
  };
  for (int zi = 0; zi < ZC; ++zi) {
    const int z = z0 + zi;
    const int64_t zb = (int64_t)z * dm.plane;
    const bool more = zi + 1 < ZC;
    const bool top = z == dm.nz - 1, bot = z == 0;
#pragma unroll
    for (int m = 0; m < XM; ++m)
#pragma unroll
      for (int r = 0; r < L; ++r) {
        plane[r * nx + tid + 256 * m] = c0[m][r + 1];
        fxp[r * nx + tid + 256 * m] = f0[m][r];
      }
    __syncthreads();
    T q[XM][L];
#pragma unroll
    for (int m = 0; m < XM; ++m) {
      const int i = tid + 256 * m;
      const int ip = (i + 1) & (nx - 1), im = (i - 1) & (nx - 1);
#pragma unroll
      for (int r = 0; r < L; ++r) {
        const T v0 = c0[m][r + 1];
        const T cxp = plane[r * nx + ip], cxm = plane[r * nx + im];
        const T cyp = c0[m][r + 2], cym = c0[m][r];
        const T czp = top ? v0 : cp[m][r + 1];
        const T czm = bot ? v0 : cm[m][r];
        T flux = f0[m][r] * (v0 + cxp) - fxp[r * nx + im] * (cxm + v0);
        flux += f1[m][r + 1] * (v0 + cyp) - f1[m][r] * (cym + v0);
        flux += (top ? T(0) : f2[m][r] * (v0 + czp)) - (bot ? T(0) : uzm[m][r] * (czm + v0));
        const T gsum = gf(cxp) + gf(cxm) + gf(cyp) + gf(cym) + gf(czp) + gf(czm);
        const T A = flux * T(0.5) * cf.inv_h;
        const T lap = (gsum - T(6) * gf(v0)) * cf.inv_h2;
        q[m][r] = cf.pe_cn2 * (h0[m][r] * cf.inv_dt - A) + lap;
        if constexpr (SPLIT) W[zb + (int64_t)row_of(r) * nx + i] = q[m][r];
      }
    }
    // plane z+1 follows in this chunk: request what it needs beyond what is held, after the stencil
    // (measured: 6 % faster than before it, with the same registers)
    if (more) {
      load_c(z + 2);
      load_f(z + 1);
      if (patch) {
        load_p(n_lo, n_hi);
        range_of(min(z + 2, zlast), nn_lo, nn_hi);   // (not used past the chunk's last plane)
      }
    }
    if constexpr (SPLIT) {
      __syncthreads();   // every x-neighbour read of this plane is done before the next write
      if (more) rotate();
    } else {
#pragma unroll
    for (int m = 0; m < XM; ++m)
#pragma unroll
      for (int r = 0; r < L; ++r) {
        const int i = tid + 256 * m;
        fb[r * pitch + i + (i >> 4)] = q[m][r];
      }
    __syncthreads();
    const int64_t line0 = (int64_t)z * dm.ny + y0;
    if (patch && e_hi > e_lo) {
#pragma unroll
      for (int k = 0; k < PF; ++k)
        if (e_lo + tid + 256 * k < e_hi) {
          const int l = (int)((pc[k] >> lnx) - line0);
          const int i = pc[k] & (nx - 1);
          fb[l * pitch + i + (i >> 4)] += pd[k];
        }
      if (e_hi - e_lo > PF * 256) patch_tile(fb, rp, line0, lnx, pitch, e_lo + PF * 256, e_hi);
      __syncthreads();
    }
    lds_fft<T, L * 256 * XM, false, R>(fb, lnx, ilog2c(L) - 1, 2 * pitch, 1, pitch, 1, false, tw, tw + nx);
    // (the FFT's final barrier also protects the LDS plane buffers for the next plane's writes)
    if (more) rotate();
    const int half = (L * nx) >> 1;
    for (int e = tid; e < half; e += blockDim.x) {
      const int b = e >> lnx;
      const int kx = e & (nx - 1);
      const int kk = (nx - kx) & (nx - 1);
      const T *pb = fb + b * 2 * pitch;
      const int ak = kx + (kx >> 4), an = kk + (kk >> 4);
      const T p = pb[ak], qq = pb[pitch + ak], rr = pb[an], sv = pb[pitch + an];
      T *o = W + (line0 + 2 * b) * nx + kx;
      __builtin_nontemporal_store((p - qq + rr + sv) * T(0.5), o);
      __builtin_nontemporal_store((p + qq - rr + sv) * T(0.5), o + nx);
    }
    }
  }
}

// Hartley transform of a tile of L = 2^logL lines of length 2^lnx in LDS (behind a barrier), stored to out.
template <typename T, int E, int MAXR>
__device__ __forceinline__ void xdht_tile(T *__restrict__ s, T *__restrict__ out, int line0, int lnx, int logL,
                                          const T *__restrict__ twr, const T *__restrict__ twi) {
  const int nx = 1 << lnx, pitch = line_pitch(nx);
  lds_fft<T, E, false, MAXR>(s, lnx, logL - 1, 2 * pitch, 1, pitch, 1, false, twr, twi);
  T *dst = out + (int64_t)line0 * nx;
  const int half = 1 << (logL + lnx - 1);
  for (int e = threadIdx.x; e < half; e += blockDim.x) {
    const int b = e >> lnx;
    const int kx = e & (nx - 1);
    const int kk = (nx - kx) & (nx - 1);
    const T *pb = s + b * 2 * pitch;
    const int ak = kx + (kx >> 4), an = kk + (kk >> 4);
    const T p = pb[ak], q = pb[pitch + ak], r = pb[an], sv = pb[pitch + an];
    T *o = dst + (int64_t)(2 * b) * nx + kx;
    o[0] = (p - q + r + sv) * T(0.5);
    o[nx] = (p + q - r + sv) * T(0.5);
  }
}

// K5 (and the forward x pass of the SOLVE stage): Hartley transform of L consecutive
// contiguous lines of length nx from `in` to `out`.
template <typename T, int E, int MAXR = 16, int CLN = 0, int CLB = 0>
__device__ __forceinline__ void xdht_body(unsigned char *smem_raw, const T *__restrict__ in, T *__restrict__ out, int lnx,
                                                   int logL, const T *__restrict__ twr, const T *__restrict__ twi, int tile) {
  if constexpr (CLN != 0) lnx = CLN;   // compile-time line length and tile height (see neumann_body)
  if constexpr (CLB != 0) logL = CLB;
  T *s = reinterpret_cast<T *>(smem_raw);
  const int L = 1 << logL;
  const int nx = 1 << lnx;
  const int line0 = tile * L;
  const int tot = L << lnx;
  const int pitch = line_pitch(nx);
  const T *src = in + (int64_t)line0 * nx;
  // (streaming reads: the input is not read again by this pass or the next one)
  constexpr int CP = 16 / (int)sizeof(T);
  typedef T FV __attribute__((ext_vector_type(CP)));
  if constexpr (CLN != 0 && CLB != 0) {
    // fixed size: 16 bytes per thread and every RS-th line, so that offsets step by constants
    constexpr int RS = (CP * kThreads) >> CLN, KR = (1 << CLB) / RS;
    static_assert(RS >= 1 && KR * RS == (1 << CLB), "fixed-size tile");
    const int i = (threadIdx.x & ((1 << CLN) / CP - 1)) * CP, l0 = threadIdx.x / ((1 << CLN) / CP);
    FV v[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k)
      v[k] = __builtin_nontemporal_load(reinterpret_cast<const FV *>(src + (l0 + k * RS) * (1 << CLN) + i));
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      T *d = s + (l0 + k * RS) * pitch + i + (i >> 4);   // CP elements of one padding group
      const T *e = reinterpret_cast<const T *>(&v[k]);
#pragma unroll
      for (int c = 0; c < CP; ++c) d[c] = e[c];
    }
  } else {
    stage_tile(s, tot, [&](int e) { return __builtin_nontemporal_load(src + e); }, [&](int e) {
      const int l = e >> lnx, i = e & (nx - 1);
      return l * pitch + i + (i >> 4);
    });
  }
  __syncthreads();
  xdht_tile<T, E, MAXR>(s, out, line0, lnx, logL, twr, twi);
}

template <typename T, int E, int MAXR = 16, int CLN = 0, int CLB = 0>
__global__ __launch_bounds__(kThreads) void k_xdht(const T *__restrict__ in, T *__restrict__ out, int lnx,
                                                   int logL, const T *__restrict__ twr, const T *__restrict__ twi) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  xdht_body<T, E, MAXR, CLN, CLB>(smem_raw, in, out, lnx, logL, twr, twi, xcd_tile(blockIdx.x, gridDim.x));
}

// The forward x pass of the pressure solve on the divergence of a face field, fac (u_a[c] - u_a[c - e_a])
// summed over the axes (no normal velocity on the box walls): the right-hand side of equal densities
// never goes to memory (256^3 FP64: rhs pass 279 us and transform 43 us before, together 110).
template <typename T, int D, int E, int MAXR, int CLN = 0, int CLB = 0>
__global__ __launch_bounds__(kThreads) void k_div_xdht(const T *__restrict__ U0, const T *__restrict__ U1,
                                                       const T *__restrict__ U2, T *__restrict__ out, Dims dm, T fac,
                                                       int logL, const T *__restrict__ twr, const T *__restrict__ twi) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lnx = CLN ? CLN : dm.lnx;
  if constexpr (CLB != 0) logL = CLB;
  T *s = reinterpret_cast<T *>(smem_raw);
  const int nx = 1 << lnx, pitch = line_pitch(nx);
  const int line0 = xcd_tile(blockIdx.x, gridDim.x) << logL;
  if constexpr (D == 3 && CLN != 0 && CLB != 0) {
    // fixed size: 16 bytes of every field per thread; the x neighbour of a thread's first value is the last
    // one of the lane below (the first lane of a wave or a line asks for it)
    constexpr int CP = 16 / (int)sizeof(T);
    typedef T FV __attribute__((ext_vector_type(CP)));
    constexpr int RS = (CP * kThreads) >> CLN, KR = (1 << CLB) / RS, KB = KR < 4 ? KR : 4;
    static_assert(RS >= 1 && KR % KB == 0, "fixed-size tile");
    const int i = (threadIdx.x & ((1 << CLN) / CP - 1)) * CP, l0 = threadIdx.x / ((1 << CLN) / CP);
    const int im = (i - 1) & ((1 << CLN) - 1);
    const bool first = (threadIdx.x & 63) == 0 || i == 0;
    auto ld = [](const T *p) { return *reinterpret_cast<const FV *>(p); };
#pragma unroll
    for (int k0 = 0; k0 < KR; k0 += KB) {
      FV u0[KB], u1[KB], u1m[KB], u2[KB], u2m[KB];
      T um[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int line = line0 + l0 + (k0 + k) * RS;
        const int j = line & (dm.ny - 1), w = line >> dm.lny;
        const int64_t row = (int64_t)line << CLN;
        u0[k] = ld(U0 + row + i);
        u1[k] = ld(U1 + row + i);
        u1m[k] = ld(U1 + row + i + (((int64_t)((j - 1) & (dm.ny - 1)) - j) << CLN));
        u2[k] = ld(U2 + row + i);
        u2m[k] = ld(U2 + row + i - (w > 0 ? dm.plane : 0));
        if (first) um[k] = U0[row + im];
      }
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int l = l0 + (k0 + k) * RS, w = (line0 + l) >> dm.lny;
        const T below = __shfl_up(u0[k][CP - 1], 1);
        T left = first ? um[k] : below;
        T *d = s + l * pitch + i + (i >> 4);
#pragma unroll
        for (int c = 0; c < CP; ++c) {
          T acc = u0[k][c] - left;
          left = u0[k][c];
          acc += u1[k][c] - u1m[k][c];
          acc += (w < dm.nz - 1 ? u2[k][c] : T(0)) - (w > 0 ? u2m[k][c] : T(0));
          d[c] = fac * acc;
        }
      }
    }
  } else {
    stage_tile<T, 4>(s, nx << logL, [&](int e) {
      const int line = line0 + (e >> lnx), i = e & (nx - 1);
      const int64_t row = (int64_t)line << lnx, c = row + i;
      T acc = U0[c] - U0[row + ((i - 1) & (nx - 1))];
      const int j = D == 2 ? line : line & (dm.ny - 1);
      if constexpr (D == 3) acc += U1[c] - U1[c + (((int64_t)((j - 1) & (dm.ny - 1)) - j) << lnx)];
      const int w = D == 2 ? line : line >> dm.lny, nw = D == 2 ? dm.ny : dm.nz;   // bounded axis
      const int64_t step = D == 2 ? (int64_t)nx : dm.plane;
      const T *Uw = D == 2 ? U1 : U2;
      const T hi = Uw[c], lo = Uw[w > 0 ? c - step : c];
      acc += (w < nw - 1 ? hi : T(0)) - (w > 0 ? lo : T(0));
      return fac * acc;
    }, [&](int e) {
      const int l = e >> lnx, i = e & (nx - 1);
      return l * pitch + i + (i >> 4);
    });
  }
  __syncthreads();
  xdht_tile<T, E, MAXR>(s, out, line0, lnx, logL, twr, twi);
}

template <typename T> struct Vec2;
template <> struct Vec2<double> { using type = double2; };
template <> struct Vec2<float> { using type = float2; };

// K2/K4: in-place Hartley transform along a strided axis of length N = 2^logN.  A tile is
// B = 2^logB adjacent x-columns (contiguous in memory) times N positions; tile t covers
// base = (t >> lognxb) * outer + (t & (nxb-1)) * B, element n at base + n*stride.  Columns
// 2b and 2b+1 form the pair b (real and imaginary parts of one complex line).
template <typename T, int E, int MAXR = 16, int CLN = 0, int CLB = 0>
__global__ __launch_bounds__(kThreads) void k_strided_dht(T *__restrict__ W, int logN, int64_t stride, int logB,
                                                          int lognxb, int64_t outer, const T *__restrict__ twr,
                                                          const T *__restrict__ twi) {
  if constexpr (CLN != 0) logN = CLN;   // compile-time line length and tile width (see neumann_body)
  if constexpr (CLB != 0) logB = CLB;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *s = reinterpret_cast<T *>(smem_raw);
  using V2 = typename Vec2<T>::type;
  const int N = 1 << logN, B = 1 << logB;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t base = (int64_t)(t >> lognxb) * outer + (int64_t)(t & ((1 << lognxb) - 1)) * B;
  const int tot = N << logB;
  // fixed size (as in neumann_body): 16 bytes of adjacent columns per thread, every RS-th position,
  // unsigned 32-bit byte offsets from a uniform base (the caller bounds N * stride * sizeof(T))
  using FV = std::conditional_t<sizeof(T) == 8, double2, float4>;
  constexpr int CP = 16 / (int)sizeof(T);
  constexpr int RS = CLB ? (CP * kThreads) >> CLB : 16, KR = CLN ? (1 << CLN) / RS : 1;
  char *const gb = reinterpret_cast<char *>(W + base);
  if constexpr (CLN != 0 && CLB != 0) {
    static_assert(RS % 16 == 0 && KR * RS == (1 << CLN), "fixed-size tile");
    const int fcol = (threadIdx.x & ((B / CP) - 1)) * CP, fn0 = threadIdx.x / (B / CP);
    const unsigned foff = ((unsigned)fn0 * (unsigned)stride + (unsigned)fcol) * (unsigned)sizeof(T);
    const unsigned fstep = (unsigned)RS * (unsigned)stride * (unsigned)sizeof(T);
    const int fa0 = fn0 * B + (fn0 >> 4) * 2 + fcol, fda = RS * B + (RS >> 4) * 2;
    FV v[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) v[k] = *reinterpret_cast<const FV *>(gb + (foff + k * fstep));
#pragma unroll
    for (int k = 0; k < KR; ++k) lds_put16(s + fa0 + k * fda, v[k]);
  } else {
    stage_tile(s, tot, [&](int e) { return W[base + (e >> logB) * stride + (e & (B - 1))]; }, [&](int e) {
      const int n = e >> logB, col = e & (B - 1);
      return n * B + (n >> 4) * 2 + col;
    });
  }
  __syncthreads();
  lds_fft<T, E, false, MAXR, 256, true>(s, logN, logB - 1, 2, B, 1, 2, true, twr, twi);
  const int lp = logB - 1;
  const int half = tot >> 1;
  if constexpr (CLN != 0 && CLB != 0) {
    // one column pair per thread, every RO-th position; the offset is made opaque so that the
    // compiler forms these addresses here rather than holding them from the staging loads
    constexpr int RO = (2 * kThreads) >> CLB, KO = (1 << CLN) / RO;
    const int b = threadIdx.x & ((B >> 1) - 1), n0 = threadIdx.x >> (logB - 1);
    unsigned ooff = ((unsigned)n0 * (unsigned)stride + 2u * b) * (unsigned)sizeof(T);
    const unsigned ostep = (unsigned)RO * (unsigned)stride * (unsigned)sizeof(T);
    asm volatile("" : "+v"(ooff));
#pragma unroll
    for (int j = 0; j < KO; ++j) {
      const int n = n0 + j * RO;
      const int nn = (N - n) & (N - 1);
      const V2 u0 = *reinterpret_cast<const V2 *>(s + n * B + (n >> 4) * 2 + 2 * b);
      const V2 u1 = *reinterpret_cast<const V2 *>(s + nn * B + (nn >> 4) * 2 + 2 * b);
      V2 v;
      v.x = (u0.x - u0.y + u1.x + u1.y) * T(0.5);
      v.y = (u0.x + u0.y - u1.x + u1.y) * T(0.5);
      *reinterpret_cast<V2 *>(gb + (ooff + j * ostep)) = v;
    }
    return;
  }
  for (int e = threadIdx.x; e < half; e += blockDim.x) {
    const int b = e & ((1 << lp) - 1), n = e >> lp;
    const int nn = (N - n) & (N - 1);
    const int a0 = n * B + (n >> 4) * 2 + 2 * b, a1 = nn * B + (nn >> 4) * 2 + 2 * b;
    const V2 u0 = *reinterpret_cast<const V2 *>(s + a0), u1 = *reinterpret_cast<const V2 *>(s + a1);
    const T p = u0.x, q = u0.y;
    const T r = u1.x, sv = u1.y;
    V2 v;
    v.x = (p - q + r + sv) * T(0.5);
    v.y = (p + q - r + sv) * T(0.5);
    *reinterpret_cast<V2 *>(W + base + n * stride + 2 * b) = v;
  }
}

// K3: along the bounded axis, per column: DCT-II (even/odd reorder + FFT + post-twiddle),
// division by (lam - a)(lam + alpha_s) times the inverse normalisation, inverse DCT-II
// (pre-twiddle + inverse FFT + reorder).  lam = lamx[kx] (+ lamy[ky]) + lamz[kz].
template <typename T, int E, int MAXR = 16, int CLN = 0, int CLB = 0>
__device__ __forceinline__ void neumann_body(unsigned char *smem_raw, T *__restrict__ W, int logN, int64_t stride, int logB,
                                                            int lognxb, int64_t outer, const T *__restrict__ lamx,
                                                            const T *__restrict__ lamy, const T *__restrict__ lamz,
                                                            T a, T alpha_s, T inv_norm, const T *__restrict__ twr,
                                                            const T *__restrict__ twi, const T *__restrict__ dctc,
                                                            const T *__restrict__ dcts, int tile, int poisson) {
  // CLN/CLB != 0 fix the line length and the tile width at compile time, so that the FFT's
  // LDS addresses fold into instruction offsets
  if constexpr (CLN != 0) logN = CLN;
  if constexpr (CLB != 0) logB = CLB;
  T *s = reinterpret_cast<T *>(smem_raw);
  const int N = 1 << logN, B = 1 << logB;
  const int t = tile;
  const int xb = t & ((1 << lognxb) - 1);
  const int oy = t >> lognxb;
  const int64_t base = (int64_t)oy * outer + (int64_t)xb * B;
  const int tot = N << logB;
  // fixed size: a thread keeps 16 bytes of adjacent columns and every (CP kThreads / B)-th
  // position, so its global offsets step by a constant (unsigned 32-bit bytes from a uniform base:
  // the caller bounds N * stride * sizeof(T)) and, the step being even, all its positions share one parity and
  // land on reordered slots a constant LDS distance apart (whole padding groups of 16 positions)
  using FV = std::conditional_t<sizeof(T) == 8, double2, float4>;
  constexpr int CP = 16 / (int)sizeof(T);
  constexpr int RS = CLB ? (CP * kThreads) >> CLB : 2, KR = CLN ? (1 << CLN) / RS : 1;
  const int fcol = (threadIdx.x & ((B / CP) - 1)) * CP, fn0 = threadIdx.x / (B / CP);
  const int fp0 = (fn0 & 1) ? N - 1 - (fn0 >> 1) : fn0 >> 1;
  const int fa0 = fp0 * B + (fp0 >> 4) * 2 + fcol;
  const int fda = ((RS / 2) * B + (RS / 32) * 2) * ((fn0 & 1) ? -1 : 1);
  unsigned foff = ((unsigned)fn0 * (unsigned)stride + (unsigned)fcol) * (unsigned)sizeof(T);   // bytes
  const unsigned fstep = (unsigned)RS * (unsigned)stride * (unsigned)sizeof(T);
  char *const gb = reinterpret_cast<char *>(W + base);
  if constexpr (CLN != 0 && CLB != 0) {
    static_assert(RS % 32 == 0 && KR * RS == (1 << CLN), "fixed-size tile");
    FV v[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) v[k] = *reinterpret_cast<const FV *>(gb + (foff + k * fstep));
#pragma unroll
    for (int k = 0; k < KR; ++k) lds_put16(s + fa0 + k * fda, v[k]);
  } else {
    stage_tile(s, tot, [&](int e) { return W[base + (e >> logB) * stride + (e & (B - 1))]; }, [&](int e) {
      const int n = e >> logB, col = e & (B - 1);
      const int pos = (n & 1) ? (N - 1 - (n >> 1)) : (n >> 1);
      return pos * B + (pos >> 4) * 2 + col;
    });
  }
  __syncthreads();
  lds_fft<T, E, false, MAXR, 256, true>(s, logN, logB - 1, 2, B, 1, 2, true, twr, twi);
  const int half = N >> 1;
  const int lpairs = logB - 1;   // B / 2 column pairs per position
  const int items = (half + 1) << lpairs;
  const T lam_y = lamy ? lamy[oy] : T(0);
  const T hnorm = inv_norm * T(0.5);
  // the pressure (POIS) divides by lam itself and drops the mean mode (lam = 0); the order
  // parameter divides by (lam - a)(lam + alpha_s), which is never zero, so the four divisors of
  // an item share divisions: 1/d1 = d2 / (d1 d2) and so on, in FP64 even 1/(d1 d2) = d3 d4 / (d1 d2 d3 d4)
  auto solve = [&](auto pois) {
    constexpr bool POIS = decltype(pois)::value;
    for (int e = threadIdx.x; e < items; e += blockDim.x) {
      const int b = e & ((1 << lpairs) - 1);
      const int k = e >> lpairs;
      const int kk = (N - k) & (N - 1);
      using V2 = typename Pair2<T>::type;
      T *zk = s + k * B + (k >> 4) * 2 + 2 * b;
      T *zn = s + kk * B + (kk >> 4) * 2 + 2 * b;
      const V2 uk = *reinterpret_cast<const V2 *>(zk), un = *reinterpret_cast<const V2 *>(zn);
      const T p = uk.x, q = uk.y, r = un.x, sv = un.y;
      // (the spectra of the two columns are (p + r, q - sv)/2 and (q + sv, r - p)/2; the halves,
      // the doubling below and the final halving are exact powers of two and fold into hnorm)
      const T var = p + r, vai = q - sv;
      const T vbr = q + sv, vbi = r - p;
      const T c = dctc[k], sn = dcts[k];
      const int kxa = xb * B + 2 * b;
      const T la = lamx[kxa] + lam_y, lb = lamx[kxa + 1] + lam_y;
      const T lk = lamz[k];
      const T lnk = k ? lamz[N - k] : T(0);
      // cosine-transform coefficients X[k], X[N-k] of both columns
      T xa1 = c * var + sn * vai, xa2 = sn * var - c * vai;
      T xb1 = c * vbr + sn * vbi, xb2 = sn * vbr - c * vbi;
      if constexpr (POIS) {
        auto fac = [&](T l) { return l != T(0) ? hnorm / l : T(0); };
        xa1 *= fac(la + lk);
        xb1 *= fac(lb + lk);
        xa2 = k ? xa2 * fac(la + lnk) : T(0);
        xb2 = k ? xb2 * fac(lb + lnk) : T(0);
      } else {
        auto den = [&](T l) { return (l - a) * (l + alpha_s); };
        const T d1 = den(la + lk), d2 = den(lb + lk), d3 = den(la + lnk), d4 = den(lb + lnk);
        const T p12 = d1 * d2, p34 = d3 * d4;
        T r12, r34;
        if constexpr (sizeof(T) == 8) {   // one division (the product of four stays far inside FP64)
          const T rr = hnorm / (p12 * p34);
          r12 = rr * p34;
          r34 = rr * p12;
        } else {                          // two (in FP32 the product of four can underflow the quotient)
          r12 = hnorm / p12;
          r34 = hnorm / p34;
        }
        xa1 *= r12 * d2;
        xb1 *= r12 * d1;
        xa2 = k ? xa2 * (r34 * d4) : T(0);
        xb2 = k ? xb2 * (r34 * d3) : T(0);
      }
      // back to the reordered-sequence spectrum: V'[k] = e^{i pi k/2N} (X[k] - i X[N-k]) / 2
      const T a1 = c * xa1 + sn * xa2, a2 = sn * xa1 - c * xa2;
      const T b1 = c * xb1 + sn * xb2, b2 = sn * xb1 - c * xb2;
      V2 ok;
      ok.x = a1 - b2;
      ok.y = a2 + b1;
      *reinterpret_cast<V2 *>(zk) = ok;
      if (k != 0 && k != half) {
        V2 on;
        on.x = a1 + b2;
        on.y = b1 - a2;
        *reinterpret_cast<V2 *>(zn) = on;
      }
    }
  };
  if (poisson) solve(std::true_type{});
  else solve(std::false_type{});
  __syncthreads();
  lds_fft<T, E, true, MAXR, 256, true>(s, logN, logB - 1, 2, B, 1, 2, true, twr, twi);
  if constexpr (CLN != 0 && CLB != 0) {
    // (an empty asm makes the offset opaque here, so the compiler forms these addresses now
    // instead of holding the staging loads' addresses in registers through the whole solve)
    asm volatile("" : "+v"(foff));
#pragma unroll
    for (int k = 0; k < KR; ++k)
      *reinterpret_cast<FV *>(gb + (foff + k * fstep)) = lds_get16<FV>(s + fa0 + k * fda);
  } else {
    for (int e = threadIdx.x; e < tot; e += blockDim.x) {
      const int n = e >> logB, col = e & (B - 1);
      const int pos = (n & 1) ? (N - 1 - (n >> 1)) : (n >> 1);
      W[base + n * stride + col] = s[pos * B + (pos >> 4) * 2 + col];
    }
  }
}

// The fixed-size instance is held to 128 VGPRs (4 waves per SIMD, as the LDS tile allows): the
// constant addresses free the compiler to hoist more, and at 3 waves it runs no faster.
template <typename T, int E, int MAXR = 16, int CLN = 0, int CLB = 0>
__global__ __launch_bounds__(kThreads, CLN ? 4 : 1) void k_neumann_solve(T *__restrict__ W, int logN, int64_t stride, int logB,
                                                            int lognxb, int64_t outer, const T *__restrict__ lamx,
                                                            const T *__restrict__ lamy, const T *__restrict__ lamz,
                                                            T a, T alpha_s, T inv_norm, const T *__restrict__ twr,
                                                            const T *__restrict__ twi, const T *__restrict__ dctc,
                                                            const T *__restrict__ dcts, int poisson) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  neumann_body<T, E, MAXR, CLN, CLB>(smem_raw, W, logN, stride, logB, lognxb, outer, lamx, lamy, lamz, a, alpha_s, inv_norm, twr, twi, dctc, dcts, xcd_tile(blockIdx.x, gridDim.x), poisson);
}

// ---------------------------------------------------------------------------------------
// Ghost-cell helpers.

template <typename T>
__device__ __forceinline__ T mirror_gather(const T *__restrict__ f, const int *__restrict__ ap,
                                           const T *__restrict__ w, int64_t g, int64_t G, int K) {
  T o1 = T(0), o2 = T(0);
  for (int k = 0; k < K; ++k) o1 += w[(int64_t)k * G + g] * f[ap[(int64_t)k * G + g]];
  for (int k = 0; k < K; ++k) o2 += w[(int64_t)(K + k) * G + g] * f[ap[(int64_t)(K + k) * G + g]];
  return T(2) * o1 - o2;
}

// Neighbours of a cell, as offsets: periodic axes wrap, and along the bounded axis both ends are flagged.  D and
// every index into the per-axis arrays below are compile-time constants: with the dimension at run time the
// compiler kept those arrays in LDS.
template <int D>
struct Nbr {
  int up[D], dn[D];
  bool lo, hi;               // on the first / last layer of the bounded axis
  __device__ __forceinline__ Nbr(int c, const Dims &dm) {
    const int i = c & (dm.nx - 1), r = c >> dm.lnx;
    up[0] = ((i + 1) & (dm.nx - 1)) - i;
    dn[0] = ((i - 1) & (dm.nx - 1)) - i;
    int w = r, nw = dm.ny, step = dm.nx;
    if constexpr (D == 3) {
      const int j = r & (dm.ny - 1);
      up[1] = (((j + 1) & (dm.ny - 1)) - j) << dm.lnx;
      dn[1] = (((j - 1) & (dm.ny - 1)) - j) << dm.lnx;
      w = r >> dm.lny;
      nw = dm.nz;
      step = (int)dm.plane;
    }
    lo = w == 0;
    hi = w == nw - 1;
    up[D - 1] = step;
    dn[D - 1] = -step;
  }
};

// Central-difference gradient at a cell (periodic axes wrap, the bounded axis reflects).
template <int D, typename T>
__device__ __forceinline__ void grad_at(const T *__restrict__ f, int c, const Nbr<D> &nb, T inv2h, T (&g)[D]) {
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const bool w = a == D - 1;
    g[a] = (f[c + (w && nb.hi ? 0 : nb.up[a])] - f[c + (w && nb.lo ? 0 : nb.dn[a])]) * inv2h;
  }
}

// Cell-centred velocity component a: mean of the two faces along a (box-wall faces read 0; every load
// happens, from the cell itself at a wall).
template <int D, typename T>
__device__ __forceinline__ T centred_u(const T *__restrict__ Fa, int c, const Nbr<D> &nb, int a) {
  const bool w = a == D - 1;
  const T lo = Fa[c + (w && nb.lo ? 0 : nb.dn[a])], hi = Fa[c];
  return T(0.5) * ((w && nb.lo ? T(0) : lo) + (w && nb.hi ? T(0) : hi));
}

// Sum over the 16 lanes of an aligned lane group (fixed order: deterministic).
template <typename T>
__device__ __forceinline__ T group16_sum(T v) {
  v += __shfl_xor(v, 8);
  v += __shfl_xor(v, 4);
  v += __shfl_xor(v, 2);
  v += __shfl_xor(v, 1);
  return v;
}

// K6 (static condition, no contact-line friction): per ghost, C_M = 2 IDW(IP1) - IDW(IP2),
// then the wall relation of Eq. WallBCS with mu_f = 0, dC/dn = -cos(theta)(1 - C^2)/(sqrt2 Cn),
// integrated exactly from M back to I: C_I = (C_M + t)/(1 + t C_M), t = tanh(b),
// b = gamma dn cos(theta)/(sqrt2 Cn), C_M taken inside [-1, 1]; C_G = ((gamma+1) C_I - C_M)/gamma
// (Eq. UpdateC).
// Sixteen lanes per ghost: lane s < 2K gathers one weighted averaging point.
template <typename T>
__device__ __forceinline__ void fill_static_body(T *__restrict__ C, const int *__restrict__ gidx,
                                                          const T *__restrict__ dn, const T *__restrict__ gam,
                                                          const int *__restrict__ ap, const T *__restrict__ w,
                                                          T *__restrict__ CGn, T *__restrict__ CGnm1,
                                                          T *__restrict__ CMs, int64_t G, int K, T cb, int init, int64_t tile) {
  const int64_t g = ((int64_t)tile * blockDim.x + threadIdx.x) >> 4;
  const int sl = threadIdx.x & 15;
  // the ghost's own table entries are requested with the gather, not after the lane sum
  const int64_t gs = g < G ? g : G - 1;
  const T ga = gam[gs], dng = dn[gs];
  const int cgi = gidx[gs];
  T v = T(0);
  if (g < G && sl < 2 * K) {
    const int64_t i = g * kGhostSlots + sl;
    v = (sl < K ? T(2) : T(-1)) * w[i] * C[ap[i]];
  }
  const T CM = group16_sum(v);
  if (g >= G || sl != 0) return;
  const T t = tanh(ga * dng * cb);
  const T Mc = CM > T(1) ? T(1) : (CM < T(-1) ? T(-1) : CM);
  const T CI = (Mc + t) / (T(1) + t * Mc);
  const T CG = ((ga + T(1)) * CI - CM) / ga;
  C[cgi] = CG;
  CMs[g] = CM;
  if (init != 2) CGnm1[g] = init ? CG : CGn[g];   // 2: refresh within a step, history kept
  CGn[g] = CG;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_fill_static(T *__restrict__ C, const int *__restrict__ gidx,
                                                          const T *__restrict__ dn, const T *__restrict__ gam,
                                                          const int *__restrict__ ap, const T *__restrict__ w,
                                                          T *__restrict__ CGn, T *__restrict__ CGnm1,
                                                          T *__restrict__ CMs, int64_t G, int K, T cb, int init) {
  fill_static_body<T>(C, gidx, dn, gam, ap, w, CGn, CGnm1, CMs, G, K, cb, init, blockIdx.x);
}

// Dynamic condition, part 1: provisional ghost values C^_G = 2 C^n_G - C^(n-1)_G.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scatter_pg(T *__restrict__ C, const int *__restrict__ gidx,
                                                         const T *__restrict__ CGn, const T *__restrict__ CGnm1,
                                                         int64_t G) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  C[gidx[g]] = T(2) * CGn[g] - CGnm1[g];
}

// Dynamic condition, part 2 (Eqs. interpolationAtWall, ProjectingToNT, WallBCS_recast):
// C_I <- C_I + dt [ -u_I . grad_t C_I + Vs (Cn dC/dn + cos(theta)(1 - C_I*^2)/sqrt2) ],
// C_I* = (gamma C^_G + C_M)/(gamma+1), dC/dn = (C_M - C^_G)/((1+gamma) dn); then
// C_G = ((gamma+1) C_I - C_M)/gamma.  All reads from the provisional field (Jacobi).
// Sixteen lanes per ghost: lane s < 2K one weighted averaging point, lane 2K the ghost itself (one thread
// per ghost walked 2K (1 + 4d) gathers: 23.5 us for 1024 ghosts, 6 us now).  In 2D the lanes' values are added
// in the order of the averaging points, so the sums keep their rounding: C_I integrates it, and the slip
// velocity divides its gradient by Ca, which FP32 runs show in the third digit of single faces.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void k_fill_dynamic(
    const T *__restrict__ C, const T *__restrict__ F0, const T *__restrict__ F1, const T *__restrict__ F2,
    const int *__restrict__ gidx, const T *__restrict__ nrm, const T *__restrict__ dn, const T *__restrict__ gam,
    const int *__restrict__ ap, const T *__restrict__ w, T *__restrict__ CI, T *__restrict__ CGnew,
    T *__restrict__ CMs, int64_t G, int K, Dims dm, T inv2h, T Cn, T Vs, T cos_t, T dt, int init) {
  const int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  const int sl = threadIdx.x & 15;
  const int64_t gs = g < G ? g : G - 1;
  const T ga = gam[gs], dng = dn[gs], ci0 = CI[gs];
  const int cg = gidx[gs];
  T n[D];
#pragma unroll
  for (int a = 0; a < D; ++a) n[a] = nrm[(int64_t)a * G + gs];
  const T *Fs[3] = {F0, F1, F2};
  // per lane: its averaging point's weight, value, gradient and velocity; lane 2K the ghost's own
  const bool own = sl == 2 * K, used = g < G && sl <= 2 * K;
  const int64_t i = (g < G ? g : 0) * kGhostSlots + sl;
  const T wt = used && !own ? w[i] : T(0);
  T f = T(0), gk[D], uk[D];
#pragma unroll
  for (int a = 0; a < D; ++a) gk[a] = uk[a] = T(0);
  if (used) {
    const int c = own ? cg : ap[i];
    f = C[c];
    if (!init) {
      const Nbr<D> nb(c, dm);
      grad_at<D>(C, c, nb, inv2h, gk);
#pragma unroll
      for (int a = 0; a < D; ++a) uk[a] = centred_u<D>(Fs[a], c, nb, a);
    }
  }
  const int base = (threadIdx.x & 63) & ~15;
  auto own_of = [&](T v) { return __shfl(v, base + 2 * K); };
  const T PG = own_of(f);
  T CM, gM[D], uM[D];
  if constexpr (D == 2) {
    T o1 = T(0), o2 = T(0);
    for (int k = 0; k < K; ++k) o1 += __shfl(wt, base + k) * __shfl(f, base + k);
    for (int k = K; k < 2 * K; ++k) o2 += __shfl(wt, base + k) * __shfl(f, base + k);
    CM = T(2) * o1 - o2;
    gM[0] = gM[1] = uM[0] = uM[1] = T(0);
    if (!init)
      for (int k = 0; k < 2 * K; ++k) {
        const T cw = (k < K ? T(2) : T(-1)) * __shfl(wt, base + k);
#pragma unroll
        for (int a = 0; a < D; ++a) {
          gM[a] += cw * __shfl(gk[a], base + k);
          uM[a] += cw * __shfl(uk[a], base + k);
        }
      }
  } else {
    const T cw = (sl < K ? T(2) : T(-1)) * wt;   // (0 on the ghost's own lane)
    CM = group16_sum(cw * f);
#pragma unroll
    for (int a = 0; a < D; ++a) {
      gM[a] = init ? T(0) : group16_sum(cw * gk[a]);
      uM[a] = init ? T(0) : group16_sum(cw * uk[a]);
    }
  }
  const T CIs = (ga * PG + CM) / (ga + T(1));
  if (init) {
    if (g < G && sl == 0) {
      CMs[g] = CM;
      CI[g] = CIs;
      CGnew[g] = PG;
    }
    return;
  }
  T gI[D], uI[D], gn = T(0);
#pragma unroll
  for (int a = 0; a < D; ++a) {
    gI[a] = (ga * own_of(gk[a]) + gM[a]) / (ga + T(1));
    uI[a] = (ga * own_of(uk[a]) + uM[a]) / (ga + T(1));
    gn += gI[a] * n[a];
  }
  if (g >= G || sl != 0) return;
  T adv = T(0);
#pragma unroll
  for (int a = 0; a < D; ++a) adv += uI[a] * (gI[a] - gn * n[a]);
  const T dCdn = (CM - PG) / ((T(1) + ga) * dng);
  const T rhs = -adv + Vs * (Cn * dCdn + cos_t * (T(1) - CIs * CIs) * T(0.70710678118654752440));
  const T ci = ci0 + dt * rhs;
  CMs[g] = CM;
  CI[g] = ci;
  CGnew[g] = ((ga + T(1)) * ci - CM) / ga;
}

// Dynamic condition, part 3: write the new ghost values and rotate the per-ghost history.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_commit_ghosts(T *__restrict__ C, const int *__restrict__ gidx,
                                                            const T *__restrict__ CGnew, T *__restrict__ CGn,
                                                            T *__restrict__ CGnm1, int64_t G, int init) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  const T v = CGnew[g];
  C[gidx[g]] = v;
  CGnm1[g] = init ? v : CGn[g];
  CGn[g] = v;
}

// Explicit chemical potential phi~ = C~^3 - C~ - Cn^2 lap_h C~ of the semi-implicit step at one cell,
// C~ = 2C^n - C^(n-1); periodic axes wrap, the bounded axis reflects (the Laplacian of the solve).
template <typename T>
__device__ __forceinline__ T phit_at(const T *__restrict__ Cn, const T *__restrict__ Cp, int64_t c, const Dims &dm,
                                     int d, T cn2, T inv_h2) {
  auto ct = [&](int64_t q) { return T(2) * Cn[q] - Cp[q]; };
  const int i = (int)(c & (dm.nx - 1));
  const int64_t r = c >> dm.lnx;
  const int j = (int)(r & (dm.ny - 1));
  const int k = (int)(r >> dm.lny);
  const int64_t rowb = c - i;
  const T v = ct(c);
  T acc = ct(rowb + ((i + 1) & (dm.nx - 1))) + ct(rowb + ((i - 1) & (dm.nx - 1)));
  if (d == 2) {
    acc = acc + (j < dm.ny - 1 ? ct(c + dm.nx) : v);
    acc = acc + (j > 0 ? ct(c - dm.nx) : v);
  } else {
    const int jp = (j + 1) & (dm.ny - 1), jm = (j - 1) & (dm.ny - 1);
    acc = acc + ct(c + (int64_t)(jp - j) * dm.nx);
    acc = acc + ct(c + (int64_t)(jm - j) * dm.nx);
    acc = acc + (k < dm.nz - 1 ? ct(c + dm.plane) : v);
    acc = acc + (k > 0 ? ct(c - dm.plane) : v);
  }
  const T lap = (acc - T(2 * d) * v) * inv_h2;
  return v * v * v - v - cn2 * lap;
}

// The wall condition dphi/dn = 0 of the semi-implicit step (end of section 4.2.2, Eq. WallBCS):
// per ghost, dg = (phi~_M - phi~_G)/Cn^2 with phi~_M = 2 IDW(IP1) - IDW(IP2) of phi~ (Eq.
// extrapolation).  Sixteen lanes per ghost: lane s < 2K one weighted averaging point, lane 2K
// the ghost itself; fixed-order lane-group sum.
template <typename T>
__device__ __forceinline__ void ghost_dphi_body(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                const int *__restrict__ gidx, const int *__restrict__ ap,
                                                const T *__restrict__ w, T *__restrict__ dg, int64_t G, int K,
                                                const Dims &dm, int d, T cn2, T inv_h2, T inv_cn2, int64_t tile) {
  const int64_t g = ((int64_t)tile * blockDim.x + threadIdx.x) >> 4;
  const int sl = threadIdx.x & 15;
  T v = T(0);
  if (g < G && sl <= 2 * K) {
    int64_t c;
    T coef;
    if (sl < 2 * K) {
      const int64_t i = g * kGhostSlots + sl;
      c = ap[i];
      coef = (sl < K ? T(2) : T(-1)) * w[i];
    } else {
      c = gidx[g];
      coef = T(-1);
    }
    v = coef * phit_at(Cn, Cp, c, dm, d, cn2, inv_h2);
  }
  const T sum = group16_sum(v);
  if (g < G && sl == 0) dg[g] = sum * inv_cn2;
}

// The same dg from phi~ evaluated once per listed point (many ghosts share averaging points):
// k_point_phit takes one point per thread (the list is sorted by cell, so neighbouring threads read
// neighbouring cells), k_ghost_dg gathers those values per ghost.  Each product and the lane sum are
// those of ghost_dphi_body, in the same order, so both give the same bits.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_point_phit(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                         const int *__restrict__ pt_cell, T *__restrict__ pt_phi,
                                                         int64_t nu, Dims dm, int d, T cn2, T inv_h2) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u < nu) pt_phi[u] = phit_at(Cn, Cp, (int64_t)pt_cell[u], dm, d, cn2, inv_h2);
}

// MIRROR (the explicit step): phi_M alone, the ghost's own value neither read nor needed.
template <typename T, bool MIRROR = false>
__global__ __launch_bounds__(kThreads) void k_ghost_dg(const T *__restrict__ pt_phi, const int *__restrict__ pt_idx,
                                                       const T *__restrict__ w, T *__restrict__ dg, int64_t G, int K,
                                                       T inv_cn2) {
  const int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  const int sl = threadIdx.x & 15;
  T v = T(0);
  if (g < G && (MIRROR ? sl < 2 * K : sl <= 2 * K)) {
    const int64_t i = g * kGhostSlots + sl;
    const T coef = sl < 2 * K ? (sl < K ? T(2) : T(-1)) * w[i] : T(-1);
    v = coef * pt_phi[pt_idx[i]];
  }
  const T sum = group16_sum(v);
  if (g < G && sl == 0) dg[g] = MIRROR ? sum : sum * inv_cn2;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_ghost_dphi(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                         const int *__restrict__ gidx, const int *__restrict__ ap,
                                                         const T *__restrict__ w, T *__restrict__ dg, int64_t G,
                                                         int K, Dims dm, int d, T cn2, T inv_h2, T inv_cn2) {
  ghost_dphi_body<T>(Cn, Cp, gidx, ap, w, dg, G, K, dm, d, cn2, inv_h2, inv_cn2, blockIdx.x);
}

// The rhs patch of every listed cell: dq = (sum of the neighbouring ghosts' dg - 2d dg_own)/h^2,
// the neighbours in a fixed order (+e_a, -e_a per axis).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_patch_dq(const int *__restrict__ ref, const T *__restrict__ dg,
                                                       T *__restrict__ dq, int64_t np, int nref, T twod, T inv_h2) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= np) return;
  T acc = T(0);
  for (int j = 1; j < nref; ++j) {
    const int id = ref[(int64_t)j * np + e];
    if (id >= 0) acc += dg[id];
  }
  const int own = ref[e];
  if (own >= 0) acc -= twod * dg[own];
  dq[e] = acc * inv_h2;
}

// The patch added to a rhs stored cell by cell (stage entry point, stencil-only z-march).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_rhs_patch(T *__restrict__ Q, const int *__restrict__ cell,
                                                        const T *__restrict__ dq, int64_t np) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < np) Q[cell[e]] += dq[e];
}

// K7a: ghost velocities (Eqs. NoPenetration, UpdateVtan, UpdateVandW in vector form) and,
// for the faces touching ghosts, the cell-centred velocity of their non-ghost side, all
// from the faces as they are before this fill.  Blocks [0, nbg) take sixteen lanes per
// ghost (lane s < 2K: one averaging point's gradient and centred velocity, lane 2K: the
// ghost's own gradient); the remaining blocks take one face per thread.  With the static
// condition (capillary = 0) the wall equation makes the bracket Kc of Eq. UpdateVtan zero,
// and no gradient of C is gathered.
// V_tG is rounded before V_nG n joins it, written out so that the fill alone and joined with the one of C gives
// the same bits.
template <typename T, int D, bool CAP>
__device__ __forceinline__ void vel_ghosts_body(
    const T *__restrict__ C, const T *__restrict__ F0, const T *__restrict__ F1, const T *__restrict__ F2,
    const int *__restrict__ gidx, const T *__restrict__ nrm, const T *__restrict__ dn, const T *__restrict__ gam,
    const int *__restrict__ ap, const T *__restrict__ w, const T *__restrict__ CMs, T *__restrict__ UG, int64_t G,
    int K, const int *__restrict__ f_cell, const int *__restrict__ f_axis, const int *__restrict__ f_gL,
    const int *__restrict__ f_gR, T *__restrict__ stashL, T *__restrict__ stashR, int64_t NF, const Dims &dm,
    T inv2h, T Cn, T cos_t, T inv_Ca, T inv_mu, T ls, unsigned nbg, int64_t tile) {
  const T *Fs[3] = {F0, F1, F2};
  if (tile >= nbg) {
    const int64_t f = (int64_t)(tile - nbg) * blockDim.x + threadIdx.x;
    if (f >= NF) return;
    const int ax = f_axis[f], cL = f_cell[f], gL = f_gL[f], gR = f_gR[f];
    const Nbr<D> nl(cL, dm);
    T vL = T(0), vR = T(0);
#pragma unroll
    for (int a = 0; a < D; ++a)
      if (ax == a) {
        // (a list face never lies on a box wall: its right cell is inside)
        const int cR = cL + nl.up[a];
        const Nbr<D> nr(cR, dm);
        if (gL < 0) vL = centred_u<D>(Fs[a], cL, nl, a);
        if (gR < 0) vR = centred_u<D>(Fs[a], cR, nr, a);
      }
    stashL[f] = vL;
    stashR[f] = vR;
    return;
  }
  const int64_t g = ((int64_t)tile * blockDim.x + threadIdx.x) >> 4;
  const int sl = threadIdx.x & 15;
  // the ghost's own table entries are requested with the gathers, not after the lane sums
  const int64_t gs = g < G ? g : G - 1;
  const T ga = gam[gs], dng = dn[gs];
  const int cg = CAP ? gidx[gs] : 0;
  T n[D];
#pragma unroll
  for (int a = 0; a < D; ++a) n[a] = nrm[(int64_t)a * G + gs];
  T gm[D], um[D], gg[D];
#pragma unroll
  for (int a = 0; a < D; ++a) gm[a] = um[a] = gg[a] = T(0);
  if (g < G) {
    if (sl < 2 * K) {
      const int64_t i = g * kGhostSlots + sl;
      const T cw = (sl < K ? T(2) : T(-1)) * w[i];
      const int c = ap[i];
      const Nbr<D> nb(c, dm);
      if constexpr (CAP) {
        T gk[D];
        grad_at<D>(C, c, nb, inv2h, gk);
#pragma unroll
        for (int a = 0; a < D; ++a) gm[a] = cw * gk[a];
      }
#pragma unroll
      for (int a = 0; a < D; ++a) um[a] = cw * centred_u<D>(Fs[a], c, nb, a);
    } else if (CAP && sl == 2 * K) {
      grad_at<D>(C, cg, Nbr<D>(cg, dm), inv2h, gg);
    }
  }
#pragma unroll
  for (int a = 0; a < D; ++a) {
    um[a] = group16_sum(um[a]);
    if constexpr (CAP) {
      gm[a] = group16_sum(gm[a]);
      gg[a] = group16_sum(gg[a]);
    }
  }
  if (g >= G || sl != 0) return;
  T VnM = T(0), gIn = T(0), gI[D];
#pragma unroll
  for (int a = 0; a < D; ++a) {
    VnM += um[a] * n[a];
    gI[a] = CAP ? (ga * gg[a] + gm[a]) / (ga + T(1)) : T(0);
    gIn += gI[a] * n[a];
  }
  const T VnG = -VnM / ga;
  const T den = ls + ga * dng;
  const T fM = (ls - dng) / den;
  T Kc = T(0), fK = T(0);
  if constexpr (CAP) {   // only then are C and C_M read (the static fill may be writing them meanwhile)
    const T CG = C[cg], CM = CMs[g];
    const T CIv = (ga * CG + CM) / (ga + T(1));
    const T dCdn = (CM - CG) / ((T(1) + ga) * dng);
    Kc = (T(1.06066017177982128660) * Cn * dCdn + T(0.75) * cos_t * (T(1) - CIv * CIv)) * inv_Ca;
    fK = ls * (ga + T(1)) * dng * inv_mu / den;
  }
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const T VtM = um[a] - VnM * n[a];
    T VtG = VtM * fM;
    if constexpr (CAP) VtG -= Kc * (gI[a] - gIn * n[a]) * fK;
    UG[(int64_t)a * G + g] = fma(VnG, n[a], VtG);
  }
}

template <typename T, int D, bool CAP>
__global__ __launch_bounds__(kThreads) void k_vel_ghosts(
    const T *__restrict__ C, const T *__restrict__ F0, const T *__restrict__ F1, const T *__restrict__ F2,
    const int *__restrict__ gidx, const T *__restrict__ nrm, const T *__restrict__ dn, const T *__restrict__ gam,
    const int *__restrict__ ap, const T *__restrict__ w, const T *__restrict__ CMs, T *__restrict__ UG, int64_t G,
    int K, const int *__restrict__ f_cell, const int *__restrict__ f_axis, const int *__restrict__ f_gL,
    const int *__restrict__ f_gR, T *__restrict__ stashL, T *__restrict__ stashR, int64_t NF, Dims dm,
    T inv2h, T Cn, T cos_t, T inv_Ca, T inv_mu, T ls, unsigned nbg) {
  vel_ghosts_body<T, D, CAP>(C, F0, F1, F2, gidx, nrm, dn, gam, ap, w, CMs, UG, G, K, f_cell, f_axis, f_gL, f_gR,
                             stashL, stashR, NF, dm, inv2h, Cn, cos_t, inv_Ca, inv_mu, ls, nbg, blockIdx.x);
}

// K6 + K7a in one launch for the static condition, where the velocity fill does not read C:
// blocks [0, nbc) fill the C ghosts, the others compute the ghost velocities and face stashes.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void k_fill_static_vel(
    T *__restrict__ C, const int *__restrict__ gidx, const T *__restrict__ dn, const T *__restrict__ gam,
    const int *__restrict__ ap, const T *__restrict__ w, T *__restrict__ CGn, T *__restrict__ CGnm1,
    T *__restrict__ CMs, int64_t G, int K, T cb, const T *__restrict__ F0, const T *__restrict__ F1,
    const T *__restrict__ F2, const T *__restrict__ nrm, T *__restrict__ UG, const int *__restrict__ f_cell,
    const int *__restrict__ f_axis, const int *__restrict__ f_gL, const int *__restrict__ f_gR, T *__restrict__ stashL,
    T *__restrict__ stashR, int64_t NF, Dims dm, T inv2h, T Cn, T cos_t, T inv_Ca, T inv_mu, T ls,
    unsigned nbc, unsigned nbg) {
  if (blockIdx.x < nbc) {
    fill_static_body<T>(C, gidx, dn, gam, ap, w, CGn, CGnm1, CMs, G, K, cb, 0, blockIdx.x);
    return;
  }
  vel_ghosts_body<T, D, false>(C, F0, F1, F2, gidx, nrm, dn, gam, ap, w, CMs, UG, G, K, f_cell, f_axis, f_gL, f_gR,
                               stashL, stashR, NF, dm, inv2h, Cn, cos_t, inv_Ca, inv_mu, ls, nbg, blockIdx.x - nbc);
}

// K7b: every face touching a ghost becomes the mean of its two cell-centred values.
template <typename T>
__device__ __forceinline__ void vel_faces_body(T *__restrict__ F0, T *__restrict__ F1, T *__restrict__ F2,
                                                        const T *__restrict__ UG, int64_t G,
                                                        const int *__restrict__ f_cell, const int *__restrict__ f_axis,
                                                        const int *__restrict__ f_gL, const int *__restrict__ f_gR,
                                                        const T *__restrict__ stashL, const T *__restrict__ stashR,
                                                        int64_t NF, int64_t tile) {
  const int64_t f = (int64_t)tile * blockDim.x + threadIdx.x;
  if (f >= NF) return;
  const int a = f_axis[f];
  const int gL = f_gL[f], gR = f_gR[f];
  const T vL = gL >= 0 ? UG[(int64_t)a * G + gL] : stashL[f];
  const T vR = gR >= 0 ? UG[(int64_t)a * G + gR] : stashR[f];
  T *Fa = a == 0 ? F0 : (a == 1 ? F1 : F2);
  Fa[f_cell[f]] = T(0.5) * (vL + vR);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_vel_faces(T *__restrict__ F0, T *__restrict__ F1, T *__restrict__ F2,
                                                        const T *__restrict__ UG, int64_t G,
                                                        const int *__restrict__ f_cell, const int *__restrict__ f_axis,
                                                        const int *__restrict__ f_gL, const int *__restrict__ f_gR,
                                                        const T *__restrict__ stashL, const T *__restrict__ stashR,
                                                        int64_t NF) {
  vel_faces_body<T>(F0, F1, F2, UG, G, f_cell, f_axis, f_gL, f_gR, stashL, stashR, NF, blockIdx.x);
}

// K7b together with the first kernel of the next step's ghost patch: the face means read the ghost
// velocities and write faces, the patch reads the filled C, so blocks [0, nbf) take the faces and the
// others phi~ at the listed points (POINTS) or dg.  One launch less per step: 256^3 FP64 6.4 + 9.0 us
// apart, 10 us together; 2D steps are a chain of launches of 2-5 us each.
template <typename T, bool POINTS>
__global__ __launch_bounds__(kThreads) void k_vel_faces_dphi(
    T *__restrict__ F0, T *__restrict__ F1, T *__restrict__ F2, const T *__restrict__ UG, int64_t G,
    const int *__restrict__ f_cell, const int *__restrict__ f_axis, const int *__restrict__ f_gL,
    const int *__restrict__ f_gR, const T *__restrict__ stashL, const T *__restrict__ stashR, int64_t NF, unsigned nbf,
    const T *__restrict__ Cn, const T *__restrict__ Cp, const int *__restrict__ cell, T *__restrict__ out, int64_t nu,
    const int *__restrict__ ap, const T *__restrict__ w, int K, Dims dm, int d, T cn2, T inv_h2, T inv_cn2) {
  if (blockIdx.x < nbf) {
    vel_faces_body<T>(F0, F1, F2, UG, G, f_cell, f_axis, f_gL, f_gR, stashL, stashR, NF, blockIdx.x);
    return;
  }
  const int64_t b = blockIdx.x - nbf;
  if constexpr (POINTS) {
    const int64_t u = b * blockDim.x + threadIdx.x;
    if (u < nu) out[u] = phit_at(Cn, Cp, (int64_t)cell[u], dm, d, cn2, inv_h2);
  } else {
    ghost_dphi_body<T>(Cn, Cp, cell, ap, w, out, G, K, dm, d, cn2, inv_h2, inv_cn2, b);
  }
}

// ---------------------------------------------------------------------------------------
// Chemical potential phi = C^3 - C - Cn^2 lap_h C on every cell, then the mirror value at
// the ghosts (dphi/dn = 0).
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void k_phi(const T *__restrict__ C, T *__restrict__ phi, Dims dm, T cn2,
                                                  T inv_h2, int64_t N) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= N) return;
  const int i = (int)(c & (dm.nx - 1));
  const int64_t r = c >> dm.lnx;
  const int j = (int)(r & (dm.ny - 1));
  const int k = (int)(r >> dm.lny);
  const int64_t rowb = c - i;
  const T c0 = C[c];
  T sum = C[rowb + ((i + 1) & (dm.nx - 1))] + C[rowb + ((i - 1) & (dm.nx - 1))];
  if (D == 2) {
    sum += (j < dm.ny - 1 ? C[c + dm.nx] : c0) + (j > 0 ? C[c - dm.nx] : c0);
  } else {
    const int jp = (j + 1) & (dm.ny - 1), jm = (j - 1) & (dm.ny - 1);
    sum += C[c + (int64_t)(jp - j) * dm.nx] + C[c + (int64_t)(jm - j) * dm.nx];
    sum += (k < dm.nz - 1 ? C[c + dm.plane] : c0) + (k > 0 ? C[c - dm.plane] : c0);
  }
  const T lap = (sum - T(2 * D) * c0) * inv_h2;
  phi[c] = c0 * c0 * c0 - c0 - cn2 * lap;
}

// Mirror value at the ghosts, sixteen lanes per ghost as in the other ghost kernels (one thread per ghost
// walked its 2K gathers one after another: 14.6 -> 7 us at the 256^3 sphere's 42 k ghosts).  ORDERED (2D):
// the lanes' values are added in the order of the averaging points, as in k_fill_dynamic.
template <typename T, bool ORDERED>
__global__ __launch_bounds__(kThreads) void k_phi_ghost(T *__restrict__ phi, const int *__restrict__ gidx,
                                                        const int *__restrict__ ap, const T *__restrict__ w,
                                                        int64_t G, int K) {
  const int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  const int sl = threadIdx.x & 15;
  const int cg = gidx[g < G ? g : G - 1];
  T wt = T(0), f = T(0), m;
  if (g < G && sl < 2 * K) {
    const int64_t i = g * kGhostSlots + sl;
    wt = w[i];
    f = phi[ap[i]];
  }
  if constexpr (ORDERED) {
    const int base = (threadIdx.x & 63) & ~15;
    T o1 = T(0), o2 = T(0);
    for (int k = 0; k < K; ++k) o1 += __shfl(wt, base + k) * __shfl(f, base + k);
    for (int k = K; k < 2 * K; ++k) o2 += __shfl(wt, base + k) * __shfl(f, base + k);
    m = T(2) * o1 - o2;
  } else {
    m = group16_sum((sl < K ? T(2) : T(-1)) * wt * f);
  }
  if (g < G && sl == 0) phi[cg] = m;
}

// Ghost fill of any scalar under the mixed condition a f + b df/dn = g at the wall: the ghost-cell
// procedure of section 4.2.2 with a general boundary condition.  With f_I and (df/dn)_I formed
// from the ghost and the mirror value as for C, f_G = ((gamma+1) g - f_M (a + b/dn)) / (a gamma - b/dn).
// The averaging points are fluid cells, never ghosts, so reads and writes do not overlap.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scalar_fill(T *__restrict__ f, const int *__restrict__ gidx,
                                                          const int *__restrict__ ap, const T *__restrict__ w,
                                                          const T *__restrict__ dn, const T *__restrict__ gam,
                                                          const T *__restrict__ gv, T g0, T a, T b, int64_t G,
                                                          int K) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  const T fM = mirror_gather(f, ap, w, g, G, K);
  const T gg = gv ? gv[g] : g0;
  const T d = dn[g], gm = gam[g];
  f[gidx[g]] = ((gm + T(1)) * gg - fM * (a + b / d)) / (a * gm - b / d);
}

// Explicit step (Eq. ExpCH, non-dimensional) on every cell: the rate
//   R = -div_h(u C^n) + (1/Pe) lap_h phi^n
// (conservative central advection, zero normal velocity on the bounded axis' box walls, where
// the Laplacian reflects), then C^(n+1) = C^n + dt (3/2 R - 1/2 R_prev) with R_prev = R on the
// first step (forward Euler).  R replaces R_prev in place; the ghosts are refilled afterwards.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void k_explicit(const T *__restrict__ C, const T *__restrict__ phi,
                                                       const T *__restrict__ F0, const T *__restrict__ F1,
                                                       const T *__restrict__ F2, T *__restrict__ R,
                                                       T *__restrict__ Cnext, Dims dm, T half_inv_h, T inv_h2,
                                                       T inv_pe, T dt, int first, int64_t N) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= N) return;
  const int nx = dm.nx;
  const int i = (int)(c & (nx - 1));
  const int64_t rowb = c - i;
  const int ip = (i + 1) & (nx - 1), im = (i - 1) & (nx - 1);
  const T c0 = C[c], p0 = phi[c];
  T flux = F0[c] * (c0 + C[rowb + ip]) - F0[rowb + im] * (C[rowb + im] + c0);
  T lsum = phi[rowb + ip] + phi[rowb + im];
  if (D == 2) {
    const int j = (int)(c >> dm.lnx);
    const bool top = j == dm.ny - 1, bot = j == 0;
    flux += (top ? T(0) : F1[c] * (c0 + C[c + nx])) - (bot ? T(0) : F1[c - nx] * (C[c - nx] + c0));
    lsum += (top ? p0 : phi[c + nx]) + (bot ? p0 : phi[c - nx]);
  } else {
    const int j = (int)((c >> dm.lnx) & (dm.ny - 1));
    const int k = (int)(c >> (dm.lnx + dm.lny));
    const int64_t cyp = c + (int64_t)(((j + 1) & (dm.ny - 1)) - j) * nx;
    const int64_t cym = c + (int64_t)(((j - 1) & (dm.ny - 1)) - j) * nx;
    flux += F1[c] * (c0 + C[cyp]) - F1[cym] * (C[cym] + c0);
    lsum += phi[cyp] + phi[cym];
    const bool top = k == dm.nz - 1, bot = k == 0;
    flux += (top ? T(0) : F2[c] * (c0 + C[c + dm.plane])) - (bot ? T(0) : F2[c - dm.plane] * (C[c - dm.plane] + c0));
    lsum += (top ? p0 : phi[c + dm.plane]) + (bot ? p0 : phi[c - dm.plane]);
  }
  const T r = -flux * half_inv_h + inv_pe * (lsum - T(2 * D) * p0) * inv_h2;
  const T rp = first ? r : R[c];
  R[c] = r;
  Cnext[c] = c0 + dt * (T(1.5) * r - T(0.5) * rp);
}

// 3D z-marching forms of k_phi and k_explicit (2.5D blocking): a workgroup owns a 64 x 4 tile of
// (x, y) columns and a chunk of 2^zc_log planes; each thread keeps the values of planes z-1, z,
// z+1 of its own column in registers and the tile's plane z (with its one-cell x/y halo) sits in
// LDS, so every plane is read from memory once instead of three times.  Same sums in the same
// order as the one-cell-per-thread kernels.  Requires nx % 64 == 0 and ny % 4 == 0.
constexpr int kZmTx = 64, kZmTy = 4;

// Halo value of plane base zb that thread (tx, ty) supplies to the tile (x, then y neighbours);
// threads inside the tile supply none (returns their own cell, unused).
template <typename T>
__device__ __forceinline__ T zm_halo(const T *__restrict__ f, int64_t zb, int x, int y, int tx, int ty,
                                     const Dims &dm) {
  const int nx = dm.nx, ny = dm.ny;
  if (tx == 0) return f[zb + ((x - 1) & (nx - 1)) + (int64_t)nx * y];
  if (tx == kZmTx - 1) return f[zb + ((x + 1) & (nx - 1)) + (int64_t)nx * y];
  return T(0);
}
template <typename T>
__device__ __forceinline__ T zm_halo_y(const T *__restrict__ f, int64_t zb, int x, int y, int ty, const Dims &dm) {
  const int nx = dm.nx, ny = dm.ny;
  if (ty == 0) return f[zb + x + (int64_t)nx * ((y - 1) & (ny - 1))];
  if (ty == kZmTy - 1) return f[zb + x + (int64_t)nx * ((y + 1) & (ny - 1))];
  return T(0);
}
template <typename T>
__device__ __forceinline__ void zm_tile_store(T (*s)[kZmTx + 2], int tx, int ty, T own, T hx, T hy) {
  s[ty + 1][tx + 1] = own;
  if (tx == 0) s[ty + 1][0] = hx;
  if (tx == kZmTx - 1) s[ty + 1][kZmTx + 1] = hx;
  if (ty == 0) s[0][tx + 1] = hy;
  if (ty == kZmTy - 1) s[kZmTy + 1][tx + 1] = hy;
}

// Planes are taken kZmU at a time: their loads (own column and halo) are issued together, so a
// thread has kZmU requests in flight per field instead of one.
constexpr int kZmU = 4;

template <typename T>
__global__ __launch_bounds__(kThreads) void k_phi_zm(const T *__restrict__ C, T *__restrict__ phi, Dims dm, T cn2,
                                                     T inv_h2, int zc_log) {
  __shared__ T s[2][kZmTy + 2][kZmTx + 2];
  const int nbx = dm.nx / kZmTx, nby = dm.ny / kZmTy;
  const int t = blockIdx.x;
  const int bx = t % nbx, by = (t / nbx) % nby, bz = t / (nbx * nby);
  const int tx = threadIdx.x & (kZmTx - 1), ty = threadIdx.x / kZmTx;
  const int x = bx * kZmTx + tx, y = by * kZmTy + ty;
  const int z0 = bz << zc_log;
  const int64_t col = x + (int64_t)dm.nx * y;
  auto zb = [&](int z) { return (int64_t)(z < 0 ? 0 : (z >= dm.nz ? dm.nz - 1 : z)) * dm.plane; };
  T cm = C[zb(z0 - 1) + col], c0 = C[zb(z0) + col];
  for (int zg = 0; zg < (1 << zc_log); zg += kZmU) {
    const int zs = z0 + zg;
    T cz[kZmU], hx[kZmU], hy[kZmU];
#pragma unroll
    for (int u = 0; u < kZmU; ++u) {
      cz[u] = C[zb(zs + u + 1) + col];
      hx[u] = zm_halo(C, zb(zs + u), x, y, tx, ty, dm);
      hy[u] = zm_halo_y(C, zb(zs + u), x, y, ty, dm);
    }
#pragma unroll
    for (int u = 0; u < kZmU; ++u) {
      const int z = zs + u;
      const T cp = cz[u];
      T (*sb)[kZmTx + 2] = s[u & 1];
      zm_tile_store(sb, tx, ty, c0, hx[u], hy[u]);
      __syncthreads();   // this slot was last read two planes ago, before the previous barrier
      T sum = sb[ty + 1][tx + 2] + sb[ty + 1][tx];
      sum += sb[ty + 2][tx + 1] + sb[ty][tx + 1];
      sum += (z < dm.nz - 1 ? cp : c0) + (z > 0 ? cm : c0);
      const T lap = (sum - T(6) * c0) * inv_h2;
      phi[zb(z) + col] = c0 * c0 * c0 - c0 - cn2 * lap;
      cm = c0;
      c0 = cp;
    }
  }
}

// The explicit step with phi formed on the way (3D, nx % 64 == 0, ny % 8 == 0), marching in z over a
// 64 x 8 tile: bound by memory, 56 bytes per cell against 80 with phi as a field of its own.  C of a plane
// goes to LDS with a two-cell x/y halo; plane z+1 of phi is formed from it for the tile and its one-cell
// ring (the threads that bring a ring cell keep that column too) and goes to LDS in turn; plane z is
// advanced from phi and C in LDS and the z neighbours in registers.  Four slots of C and three of phi
// leave one barrier per plane: a slot is rewritten two barriers after its last read.  At the ghosts the
// mirror value takes phi's place (a word per 32 cells, a bit each and the index of the first ghost, says
// where), so that C inside the solid, which phi at a ghost would read, reaches no fluid cell and
// the rate is rounded once, as with phi as a field.  256^3 FP64: phi 62, its ghosts 7 and update 217 us before,
// 201 us here (moving 1.34 times its bytes); a step at 256^3 FP32 136.5 us.
constexpr int kXx = 64, kXy = 8, kXThreads = kXx * kXy;        // (explicit_fused asks for whole tiles)
constexpr int kXcp = kXx + 4, kXpp = kXx + 2;                  // row pitch of C and of phi
constexpr int kXcPlane = kXcp * (kXy + 4), kXpPlane = kXpp * (kXy + 2);
constexpr int kXRing1 = kXpPlane - kXThreads;                  // cells around the tile where phi is formed
constexpr int kXHalo = kXcPlane - kXThreads;                   // cells around the tile whose C is held
static_assert(kXHalo <= kXThreads, "one halo cell per thread");

// A uniform address that stays in scalar registers until a lane's 32-bit offset joins it.  (Left to the compiler,
// base + offset of every field is hoisted out of the plane loop, two vector registers each: the FP32 update then
// holds 68 instead of 56 and loses a workgroup per CU.)
template <typename U>
using global_t = __attribute__((address_space(1))) U;
template <typename U>
__device__ __forceinline__ global_t<U> *scalar_base(U *p) {
  global_t<U> *g = (global_t<U> *)p;
  asm("" : "+s"(g));
  return g;
}

template <typename T, bool GHOSTS>
__global__ __launch_bounds__(kXThreads, sizeof(T) == 4 ? 8 : 4) void k_explicit_zm(const T *__restrict__ C, const T *__restrict__ F0,
                                                           const T *__restrict__ F1, const T *__restrict__ F2,
                                                           T *__restrict__ R, T *__restrict__ Cnext, Dims dm, T cn2,
                                                           T half_inv_h, T inv_h2, T inv_pe, T dt, int first, int zc,
                                                           int runs, const GhostWord *__restrict__ g_word,
                                                           const T *__restrict__ g_phi) {
  __shared__ T sc[4][kXcPlane];
  __shared__ T sp[3][kXpPlane];
  const int nx = dm.nx, ny = dm.ny, nz = dm.nz;
  const int lbx = dm.lnx - 6, lby = dm.lny - 3;                // tiles per axis (log2; every n is a power of two)
  const int b = runs ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int x0 = (b & ((1 << lbx) - 1)) * kXx, y0 = ((b >> lbx) & ((1 << lby) - 1)) * kXy, z0 = (b >> (lbx + lby)) * zc;
  const int tid = threadIdx.x, tx = tid & (kXx - 1), ty = tid / kXx;
  const int col = x0 + tx + ((y0 + ty) << dm.lnx);
  const int ic = (ty + 2) * kXcp + tx + 2, ip = (ty + 1) * kXpp + tx + 1;
  // the halo cell of this thread: first the ring of phi (row below, row above, columns), then the outer ring
  int hr, hc;                                                  // row and column within the C plane
  if (tid < kXRing1) {
    const int e = tid - 2 * kXpp;
    hr = tid < kXpp ? 1 : (e < 0 ? kXy + 2 : 2 + (e >> 1));
    hc = e < 0 ? 1 + (tid < kXpp ? tid : tid - kXpp) : ((e & 1) ? kXx + 2 : 1);
  } else {
    const int t = tid - kXRing1, e = t - 2 * kXcp;
    hr = t < kXcp ? 0 : (e < 0 ? kXy + 3 : 1 + (e >> 1));
    hc = e < 0 ? (t < kXcp ? t : t - kXcp) : ((e & 1) ? kXx + 3 : 0);
  }
  const bool halo = tid < kXHalo, ring = tid < kXRing1;
  const int hcol = halo ? ((x0 - 2 + hc) & (nx - 1)) + (((y0 - 2 + hr) & (ny - 1)) << dm.lnx) : col;
  const int hic = hr * kXcp + hc, hip = (hr - 1) * kXpp + hc - 1;
  const int colym = x0 + tx + (((y0 + ty - 1) & (ny - 1)) << dm.lnx);
  const int colxm = ((x0 - 1) & (nx - 1)) + ((y0 + ty) << dm.lnx);   // (the first lane of each row asks for it)
  // planes beyond the walls reflect onto the boundary plane
  auto zb = [&](int z) { return (int64_t)(z < 0 ? 0 : (z >= nz ? nz - 1 : z)) * dm.plane; };
  // a plane's value at a byte offset within it, which all fields share
  const unsigned ob = (unsigned)col * (unsigned)sizeof(T), hb = (unsigned)hcol * (unsigned)sizeof(T);
  const unsigned obx = (unsigned)colxm * (unsigned)sizeof(T), oby = (unsigned)colym * (unsigned)sizeof(T);
  auto in = [](const global_t<T> *p, unsigned off) {
    return *reinterpret_cast<const global_t<T> *>(reinterpret_cast<const global_t<char> *>(p) + off);
  };
  T cn, hn = T(0);                                             // the plane of C in flight, with its ghosts
  GhostWord gw{}, hw{};
  auto word = [](const global_t<GhostWord> *w, unsigned i) { return GhostWord{w[i].bits, w[i].base}; };
  auto request_c = [&](int z) {
    const global_t<T> *p = scalar_base(C + zb(z));
    const global_t<GhostWord> *w = scalar_base(g_word + (zb(z) >> 5));
    if constexpr (GHOSTS) gw = word(w, (unsigned)col >> 5);
    cn = in(p, ob);
    if (halo) {
      if constexpr (GHOSTS) hw = word(w, (unsigned)hcol >> 5);
      hn = in(p, hb);
    }
  };
  // phi's mirror value where the cell at column c is a ghost
  auto mirror = [&](const GhostWord &w, int c, T &v) {
    const uint32_t bit = uint32_t(1) << (c & 31);
    const bool is = w.bits & bit;
    if (is) v = g_phi[w.base + __popc(w.bits & (bit - 1))];
    return is;
  };
  T f0, f0l, f1, f1m, f2, rz;                                  // faces and rate of the plane to advance
  auto request_f = [&](int z) {
    const int64_t c = zb(z);
    const global_t<T> *p0 = scalar_base(F0 + c), *p1 = scalar_base(F1 + c);
    f0 = in(p0, ob);
    if (tx == 0) f0l = in(p0, obx);
    f1 = in(p1, ob);
    f1m = in(p1, oby);
    f2 = in(scalar_base(F2 + c), ob);
    rz = in(scalar_base((const T *)R + c), ob);
  };
  auto phi_of = [&](const T *p, int i, T cm, T c0, T cp) {
    const T sum = ((p[i + 1] + p[i - 1]) + (p[i + kXcp] + p[i - kXcp])) + (cp + cm);
    return c0 * c0 * c0 - c0 - cn2 * ((sum - T(6) * c0) * inv_h2);
  };
  // own column (c*) and ring column (h*): planes z, z+1, z+2
  T c0, c1, h0, h1;
  request_c(z0 - 2);
  c0 = cn;
  h0 = hn;
  request_c(z0 - 1);
  c1 = cn;
  h1 = hn;
  T gv = T(0), ghv = T(0);                                     // phi's mirror value at ghosts of plane z+1
  bool own_g = false, ring_g = false;
  if constexpr (GHOSTS) {
    own_g = mirror(gw, col, gv);
    ring_g = ring && mirror(hw, hcol, ghv);
  }
  sc[(z0 + 3) & 3][ic] = c1;
  if (halo) sc[(z0 + 3) & 3][hic] = h1;
  request_c(z0);
  T pm = T(0), p0 = T(0);
  T f2m = z0 > 0 ? in(scalar_base(F2 + zb(z0 - 1)), ob) : T(0);
  int s1 = 2;                                                  // slot of phi plane z+1
  __syncthreads();
  for (int z = z0 - 2; z < z0 + zc; ++z) {
    // plane z+2 of C arrives, and its ghosts' phi is requested; phi of plane z+1
    const T c2 = cn, h2 = hn;
    const T mo = gv, mh = ghv;
    const bool is_o = own_g, is_h = ring_g;
    if constexpr (GHOSTS) {
      own_g = mirror(gw, col, gv);
      ring_g = ring && mirror(hw, hcol, ghv);
    }
    T *cs = sc[(z + 6) & 3];
    cs[ic] = c2;
    if (halo) cs[hic] = h2;
    const T *cc = sc[(z + 5) & 3];
    T p1 = phi_of(cc, ic, c0, c1, c2);
    if (is_o) p1 = mo;
    sp[s1][ip] = p1;
    if (ring) {
      const T ph = phi_of(cc, hic, h0, h1, h2);
      sp[s1][hip] = is_h ? mh : ph;
    }
    if (z + 1 < z0 + zc) request_c(z + 3);
    if (z == z0 - 1) request_f(z0);
    __syncthreads();
    if (z >= z0) {
      const T *pc = sc[(z + 4) & 3], *pp = sp[s1 >= 1 ? s1 - 1 : 2];
      const bool top = z == nz - 1, bot = z == 0;
      const T up = __shfl_up(f0, 1);
      const T f0m = tx == 0 ? f0l : up;
      T flux = f0 * (c0 + pc[ic + 1]) - f0m * (pc[ic - 1] + c0);
      flux += f1 * (c0 + pc[ic + kXcp]) - f1m * (pc[ic - kXcp] + c0);
      T lsum = (pp[ip + 1] + pp[ip - 1]) + (pp[ip + kXpp] + pp[ip - kXpp]);
      lsum += (top ? p0 : p1) + (bot ? p0 : pm);
      // the face below reads 0 on the bottom wall, the one above on the top wall
      const T fz = top ? T(0) : f2 * (c0 + c1);
      flux += fz - f2m;
      const T r = -flux * half_inv_h + inv_pe * (lsum - T(6) * p0) * inv_h2;
      const T rp = first ? r : rz;
      auto to = [&](T *field) {
        return reinterpret_cast<global_t<T> *>(reinterpret_cast<global_t<char> *>(scalar_base(field + zb(z))) + ob);
      };
      __builtin_nontemporal_store(r, to(R));
      *to(Cnext) = c0 + dt * (T(1.5) * r - T(0.5) * rp);
      f2m = fz;
      if (z + 1 < z0 + zc) request_f(z + 1);
    } else if (z == z0 - 1) {
      f2m = f2m * (c0 + c1);                                   // the z flux below plane z0
    }
    pm = p0;
    p0 = p1;
    c0 = c1;
    c1 = c2;
    h0 = h1;
    h1 = h2;
    s1 = s1 < 2 ? s1 + 1 : 0;
  }
}

// planes per workgroup: 16 (each chunk reads four more of C; 256^3 FP64 206 us, 210 with 32), fewer where
// that leaves under 512 workgroups
inline int explicit_zm_planes(const Plan &p) {
  int zc = p.n[2] < 16 ? p.n[2] : 16;
  while (zc > 4 && p.N / ((int64_t)kXThreads * zc) < 512) zc >>= 1;
  return zc;
}

inline bool stencil_zm_ok(const Plan &p) {
  return p.d == 3 && p.n[0] % kZmTx == 0 && p.n[1] % kZmTy == 0 && p.n[2] >= 16;   // chunks of 16 planes
}
// planes per workgroup: 16, or 8 or 4 (kZmU) on grids that would have fewer than 1024 workgroups
inline int stencil_zm_log(const Plan &p) {
  int l = 4;
  while (l > 2 && (p.N >> (8 + l)) < 1024) --l;
  return l;
}
inline unsigned stencil_zm_blocks(const Plan &p) {
  return (unsigned)((p.n[0] / kZmTx) * (p.n[1] / kZmTy) * (p.n[2] >> stencil_zm_log(p)));
}

template <typename T, int D>
__global__ __launch_bounds__(kThreads) void k_rhs_only(const T *__restrict__ Cn, const T *__restrict__ Cp,
                                                       const T *__restrict__ F0, const T *__restrict__ F1,
                                                       const T *__restrict__ F2, T *__restrict__ Q, Dims dm,
                                                       RhsCoef<T> cf, int64_t N) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= N) return;
  const int i = (int)(c & (dm.nx - 1));
  const int64_t r = c >> dm.lnx;
  const int j = (int)(r & (dm.ny - 1));
  const int k = (int)(r >> dm.lny);
  Q[c] = rhs_at<T, D>(Cn, Cp, F0, F1, F2, i, j, k, dm, cf);
}

// ---------------------------------------------------------------------------------------
// Diagnostics: fixed-order two-pass reductions (deterministic).  Slots: 0 sum C, 1 sum
// alpha C, 2 sum alpha (bulk + gradient energy density), 3 sum |grad alpha| g(C),
// 4 max |C|, 5 count of non-finite C.
// Sum (max for slot 4) of the six slots over a wave by a butterfly of lane exchanges: a fixed
// pairing, so the result does not depend on timing.
__device__ inline void wave_reduce6(double acc[6]) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
#pragma unroll
    for (int s = 0; s < 6; ++s) {
      const double o = __shfl_xor(acc[s], m, 64);
      acc[s] = s == 4 ? fmax(acc[s], o) : acc[s] + o;
    }
  }
}

// Per block: each wave reduces its lanes, then the first lanes combine the waves in index order.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void k_diag_partial(const T *__restrict__ C, const T *__restrict__ alpha,
                                                           double *__restrict__ partial, Dims dm, double Cn,
                                                           double inv_h, double inv4cn, int64_t N) {
  __shared__ double red[kThreads / 64][6];
  double acc[6] = {0, 0, 0, 0, 0, 0};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < N; c += stride) {
    const double v = (double)C[c];
    const double al = alpha ? (double)alpha[c] : 1.0;
    if (!(v == v) || v - v != 0.0) {
      acc[5] += 1.0;
      continue;
    }
    const int i = (int)(c & (dm.nx - 1));
    const int64_t r = c >> dm.lnx;
    const int j = (int)(r & (dm.ny - 1));
    const int k = (int)(r >> dm.lny);
    const int64_t rowb = c - i;
    double g2 = 0.0;
    double ga2 = 0.0;
    {
      const double dx = ((double)C[rowb + ((i + 1) & (dm.nx - 1))] - v) * inv_h;
      g2 += dx * dx;
      if (alpha) {
        const double da = ((double)alpha[rowb + ((i + 1) & (dm.nx - 1))] -
                           (double)alpha[rowb + ((i - 1) & (dm.nx - 1))]) * 0.5 * inv_h;
        ga2 += da * da;
      }
    }
    if (D == 2) {
      const double up = j < dm.ny - 1 ? (double)C[c + dm.nx] : v;
      const double dy = (up - v) * inv_h;
      g2 += dy * dy;
      if (alpha) {
        const double au = j < dm.ny - 1 ? (double)alpha[c + dm.nx] : al;
        const double ad = j > 0 ? (double)alpha[c - dm.nx] : al;
        const double da = (au - ad) * 0.5 * inv_h;
        ga2 += da * da;
      }
    } else {
      const int jp = (j + 1) & (dm.ny - 1), jm = (j - 1) & (dm.ny - 1);
      const double dy = ((double)C[c + (int64_t)(jp - j) * dm.nx] - v) * inv_h;
      g2 += dy * dy;
      const double up = k < dm.nz - 1 ? (double)C[c + dm.plane] : v;
      const double dz = (up - v) * inv_h;
      g2 += dz * dz;
      if (alpha) {
        const double day = ((double)alpha[c + (int64_t)(jp - j) * dm.nx] -
                            (double)alpha[c + (int64_t)(jm - j) * dm.nx]) * 0.5 * inv_h;
        const double au = k < dm.nz - 1 ? (double)alpha[c + dm.plane] : al;
        const double ad = k > 0 ? (double)alpha[c - dm.plane] : al;
        const double daz = (au - ad) * 0.5 * inv_h;
        ga2 += day * day + daz * daz;
      }
    }
    const double bulk = (v * v - 1.0) * (v * v - 1.0) * inv4cn;
    acc[0] += v;
    acc[1] += al * v;
    acc[2] += al * (bulk + 0.5 * Cn * g2);
    acc[3] += sqrt(ga2) * (2.0 + 3.0 * v - v * v * v) * 0.25;
    acc[4] = fmax(acc[4], fabs(v));
  }
  wave_reduce6(acc);
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  if (lane == 0)
    for (int s = 0; s < 6; ++s) red[wv][s] = acc[s];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int s = (int)threadIdx.x;
    double r = red[0][s];
    for (int w = 1; w < kThreads / 64; ++w) r = s == 4 ? fmax(r, red[w][s]) : r + red[w][s];
    partial[(int64_t)blockIdx.x * 8 + s] = r;
  }
}

// 3D diagnostics marching in z: a block owns a 64 x 4 tile of (x, y) columns over zc planes, each
// thread keeps C and alpha of planes z and z+1 (alpha also z-1) of its column in registers, so C and
// alpha come from HBM once; the x and y neighbours are in the same plane as the tile's own loads.
// Tiles go in XCD-aware order, so the neighbouring tiles whose halo rows a tile reads share its L2
// (116 -> 99 us per call at 256^3).  Same per-cell terms as k_diag_partial<T, 3>.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_diag_partial_zm(const T *__restrict__ C, const T *__restrict__ alpha,
                                                              double *__restrict__ partial, Dims dm, double Cn,
                                                              double inv_h, double inv4cn, int zc) {
  __shared__ double red[kThreads / 64][6];
  double acc[6] = {0, 0, 0, 0, 0, 0};
  const int tiles_x = dm.nx >> 6, tiles_y = dm.ny >> 2;
  int b = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = b % tiles_x;
  b /= tiles_x;
  const int by = b % tiles_y;
  const int bz = b / tiles_y;
  const int x = (bx << 6) + ((int)threadIdx.x & 63), y = (by << 2) + ((int)threadIdx.x >> 6);
  const int z0 = bz * zc, z1 = min(z0 + zc, dm.nz);
  const int oxp = ((x + 1) & (dm.nx - 1)) - x, oxm = ((x - 1) & (dm.nx - 1)) - x;
  const int64_t oyp = (int64_t)((((y + 1) & (dm.ny - 1)) - y) << dm.lnx);
  const int64_t oym = (int64_t)((((y - 1) & (dm.ny - 1)) - y) << dm.lnx);
  int64_t c = ((int64_t)y << dm.lnx) + x + (int64_t)z0 * dm.plane;
  double v = (double)C[c];
  double al = alpha ? (double)alpha[c] : 1.0;
  double ad = alpha && z0 > 0 ? (double)alpha[c - dm.plane] : al;
  for (int k = z0; k < z1; ++k, c += dm.plane) {
    double vu = v, au = al;
    if (k < dm.nz - 1) {
      vu = (double)C[c + dm.plane];
      if (alpha) au = (double)alpha[c + dm.plane];
    }
    if (!(v == v) || v - v != 0.0) {
      acc[5] += 1.0;
    } else {
      const double dx = ((double)C[c + oxp] - v) * inv_h;
      const double dy = ((double)C[c + oyp] - v) * inv_h;
      const double dz = (vu - v) * inv_h;
      double g2 = dx * dx;
      g2 += dy * dy;
      g2 += dz * dz;
      double ga2 = 0.0;
      if (alpha) {
        const double da = ((double)alpha[c + oxp] - (double)alpha[c + oxm]) * 0.5 * inv_h;
        const double day = ((double)alpha[c + oyp] - (double)alpha[c + oym]) * 0.5 * inv_h;
        const double daz = (au - ad) * 0.5 * inv_h;
        ga2 += da * da;
        ga2 += day * day + daz * daz;
      }
      const double bulk = (v * v - 1.0) * (v * v - 1.0) * inv4cn;
      acc[0] += v;
      acc[1] += al * v;
      acc[2] += al * (bulk + 0.5 * Cn * g2);
      acc[3] += sqrt(ga2) * (2.0 + 3.0 * v - v * v * v) * 0.25;
      acc[4] = fmax(acc[4], fabs(v));
    }
    ad = al;
    al = au;
    v = vu;
  }
  wave_reduce6(acc);
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  if (lane == 0)
    for (int s = 0; s < 6; ++s) red[wv][s] = acc[s];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int s = (int)threadIdx.x;
    double r = red[0][s];
    for (int w = 1; w < kThreads / 64; ++w) r = s == 4 ? fmax(r, red[w][s]) : r + red[w][s];
    partial[(int64_t)blockIdx.x * 8 + s] = r;
  }
}

__global__ __launch_bounds__(kThreads) void k_diag_final(const double *__restrict__ partial, int nred,
                                                         double *__restrict__ out) {
  __shared__ double red[6][kThreads];
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < nred; b += blockDim.x)
    for (int s = 0; s < 6; ++s) {
      const double v = partial[(int64_t)b * 8 + s];
      if (s == 4) acc[s] = fmax(acc[s], v);
      else acc[s] += v;
    }
  for (int s = 0; s < 6; ++s) red[s][threadIdx.x] = acc[s];
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int s = 0; s < 6; ++s) {
        if (s == 4) red[s][threadIdx.x] = fmax(red[s][threadIdx.x], red[s][threadIdx.x + w]);
        else red[s][threadIdx.x] += red[s][threadIdx.x + w];
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) out[threadIdx.x] = red[threadIdx.x][0];
}

// ---------------------------------------------------------------------------------------
// Host-side launch shapes.

inline int ilog2(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

inline Dims make_dims(const Plan &p) {
  Dims dm;
  dm.nx = p.n[0];
  dm.ny = p.n[1];
  dm.nz = p.d == 3 ? p.n[2] : 1;
  dm.lnx = p.logn[0];
  dm.lny = p.logn[1];
  dm.lnz = p.d == 3 ? p.logn[2] : 0;
  dm.plane = (int64_t)dm.nx * dm.ny;
  return dm;
}

template <typename T>
inline RhsCoef<T> make_coef(const Plan &p) {
  RhsCoef<T> cf;
  cf.pe_cn2 = (T)(p.Pe / (p.Cn * p.Cn));
  cf.inv_dt = (T)(1.0 / p.dt);
  cf.S = (T)p.S;
  cf.inv_cn2 = (T)(1.0 / (p.Cn * p.Cn));
  cf.inv_h = (T)(1.0 / p.h);
  cf.inv_h2 = (T)(1.0 / (p.h * p.h));
  return cf;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

// The rhs' ghost patch (none without ghosts).
template <typename T>
inline RhsPatch<T> make_patch(const Plan &p) {
  RhsPatch<T> rp{};
  if (p.G > 0 && p.NP > 0 && p.pl_dq) {
    rp.row = p.pl_row;
    rp.cell = p.pl_cell;
    rp.ref = p.pl_ref;
    rp.dg = (const T *)p.dg;
    rp.dq = (const T *)p.pl_dq;
    rp.np = (int)p.NP;
    rp.inv_h2 = (T)(1.0 / (p.h * p.h));
  }
  return rp;
}

// phi~ at the listed points first, one evaluation per point (3D, where many ghosts share averaging
// points: 256^3 sphere 29.8 -> 23.5 us with the gather), or inside the gather (2D: one launch less)
inline bool dphi_points(const Plan &p) { return p.d == 3 && p.NU && p.pt_phi; }

inline bool has_patch(const Plan &p) { return p.G > 0 && p.NP > 0 && p.dg; }

// The first kernel of the ghost patch: phi~ at the listed points, or dg itself.
template <typename T>
hipError_t launch_dphi(const Plan &p, const T *Cn, const T *Cp) {
  if (!has_patch(p)) return hipSuccess;
  const Dims dm = make_dims(p);
  if (dphi_points(p))
    hipLaunchKernelGGL((k_point_phit<T>), dim3(blocks_for(p.NU)), dim3(kThreads), 0, p.stream, Cn, Cp, p.pt_cell,
                       (T *)p.pt_phi, p.NU, dm, p.d, (T)(p.Cn * p.Cn), (T)(1.0 / (p.h * p.h)));
  else
    hipLaunchKernelGGL((k_ghost_dphi<T>), dim3(blocks_for(p.G * 16)), dim3(kThreads), 0, p.stream, Cn, Cp, p.gidx,
                       p.apg, (const T *)p.wg, (T *)p.dg, p.G, p.K, dm, p.d, (T)(p.Cn * p.Cn), (T)(1.0 / (p.h * p.h)),
                       (T)(1.0 / (p.Cn * p.Cn)));
  return hipGetLastError();
}

// dg of every ghost from C^n, C^(n-1) (before the rhs pass of a semi-implicit step); need_dq: then dq
// of every patched cell; dphi_done: launch_dphi's kernel ran at the end of the step before.  mirror: 3D
// explicit steps take C^n twice (then C~ = C^n) and phi_M in dg's place.
template <typename T>
hipError_t launch_ghost_patch(const Plan &p, const T *Cn, const T *Cp, bool need_dq, bool dphi_done = false,
                              bool mirror = false) {
  if (!has_patch(p)) return hipSuccess;
  if (!dphi_done) {
    hipError_t e = launch_dphi<T>(p, Cn, Cp);
    if (e != hipSuccess) return e;
  }
  if (dphi_points(p)) {
#define CHIB_GHOST_DG(M)                                                                                       \
  hipLaunchKernelGGL((k_ghost_dg<T, M>), dim3(blocks_for(p.G * 16)), dim3(kThreads), 0, p.stream,              \
                     (const T *)p.pt_phi, p.pt_idx, (const T *)p.wg, (T *)p.dg, p.G, p.K, (T)(1.0 / (p.Cn * p.Cn)))
    if (mirror) CHIB_GHOST_DG(true);
    else CHIB_GHOST_DG(false);
#undef CHIB_GHOST_DG
  }
  if (need_dq)
    hipLaunchKernelGGL((k_patch_dq<T>), dim3(blocks_for(p.NP)), dim3(kThreads), 0, p.stream, p.pl_ref,
                       (const T *)p.dg, (T *)p.pl_dq, p.NP, 2 * p.d + 1, (T)(2 * p.d), (T)(1.0 / (p.h * p.h)));
  return hipGetLastError();
}

// The patch added to a rhs field stored cell by cell.
template <typename T>
hipError_t launch_rhs_patch(const Plan &p, T *Q) {
  const RhsPatch<T> rp = make_patch<T>(p);
  if (!rp.row) return hipSuccess;
  hipLaunchKernelGGL((k_rhs_patch<T>), dim3(blocks_for(p.NP)), dim3(kThreads), 0, p.stream, Q, rp.cell, rp.dq, p.NP);
  return hipGetLastError();
}

// Faces that advect C in the rhs pass: the extrapolated velocity when the momentum equation is
// solved too, else the faces themselves.
inline const void *adv_face(const Plan &p, int a) { return p.Fadv[a] ? p.Fadv[a] : p.F[a]; }

// Launch shapes.  Each pass has a runtime-selected variant (see Plan::Shape): the log2 of
// its lines (x passes) or columns (strided passes) per tile, the largest FFT radix (8 or
// 16: fewer LDS passes against fewer registers) and, for the fused rhs pass, how many cells
// each thread keeps in flight.
inline int max_log_lines(const Plan &p, int E) {
  const int lines = p.d == 3 ? p.n[1] * p.n[2] : p.n[1];
  int L = E / p.n[0];
  if (L > lines) L = lines;
  if (L < 2) L = 2;
  return ilog2(L);
}

inline int max_log_cols(const Plan &p, int N, int E) {
  int B = E / N;
  if (B > p.n[0]) B = p.n[0];
  if (B < 2) B = 2;
  return ilog2(B);
}

inline int clamp_log(int v, int hi) { return v < 1 ? 1 : (v > hi ? hi : v); }

// The fixed-size instances (line length and tile width are template constants, so addresses step by constants
// and loops unroll) serve 64- to 512-point lines at the tile widths and radices below; other shapes take the
// runtime-size kernels, with the same results.  Besides 256 points (one width per radix a tuner may ask for),
// each length has the one shape that the grid's default takes: 16 columns in FP64 and 32 in FP32 (128 bytes a
// row; half as many at 512 points, which fill the 32 KB tile), 16 lines in the x pass (4 at 512).  Per step,
// runtime-size against fixed: 128^3 FP64 105 and 91 us (y 13.7 and 10.9, solve 23.5 and 19.6, inverse y 17.8
// and 15.1, x out 13.9 and 10.1), FP32 78 and 66; 256x64x64 61 and 56; 32x512x512 290 and 273.
template <typename T>
constexpr int fixed_cols(int logn) { return (sizeof(T) == 8 ? 4 : 5) - (logn == 9 ? 1 : 0); }
constexpr int fixed_lines(int logn) { return logn == 9 ? 2 : 4; }
// radix at 64 and 512 points (128 take 16: radix 8 leaves a stage of 2, 97 against 92 us per 128^3 step)
template <typename T> constexpr int fixed_radix() { return sizeof(T) == 8 ? 8 : 16; }

template <typename T>
hipError_t launch_xdht(const Plan &p, const T *in, T *out, const Plan::Shape &sh) {
  constexpr int E = tile_elems<T>();
  const int logL = clamp_log(sh.log_tile, max_log_lines(p, E));
  const int lines = p.d == 3 ? p.n[1] * p.n[2] : p.n[1];
  const unsigned nb = (unsigned)(lines >> logL);
  const size_t lds = (size_t)(1 << logL) * line_pitch(p.n[0]) * sizeof(T);
#define CHIB_XDHT(...)                                                                                         \
  hipLaunchKernelGGL((k_xdht<__VA_ARGS__>), dim3(nb), dim3(kThreads), lds, p.stream, in, out, p.logn[0], logL, \
                     (const T *)p.twr[0], (const T *)p.twi[0])
  // (the fixed-size instances read 16 bytes at a time; a caller's field need only be aligned to its elements)
  const bool wide = ((uintptr_t)in & 15) == 0;
  const bool r8 = sh.radix == 8, fixed = wide && p.logn[0] == 8;
  constexpr int RD = fixed_radix<T>();
  if (wide && p.logn[0] == 6 && logL == 4 && sh.radix == RD) {
    CHIB_XDHT(T, E, RD, 6, 4);
  } else if (wide && p.logn[0] == 7 && logL == 4 && !r8) {
    CHIB_XDHT(T, E, 16, 7, 4);
  } else if (wide && p.logn[0] == 9 && logL == 2 && sh.radix == RD) {
    CHIB_XDHT(T, E, RD, 9, 2);
  } else if (fixed && logL == 3) {
    if (r8) CHIB_XDHT(T, E, 8, 8, 3);
    else CHIB_XDHT(T, E, 16, 8, 3);
  } else if (fixed && logL == 4) {
    if (r8) CHIB_XDHT(T, E, 8, 8, 4);
    else CHIB_XDHT(T, E, 16, 8, 4);
  } else if (r8) {
    CHIB_XDHT(T, E, 8);
  } else {
    CHIB_XDHT(T, E, 16);
  }
#undef CHIB_XDHT
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_div_xdht(const Plan &p, void *const *vel, double fac, const Plan::Shape &sh) {
  constexpr int E = tile_elems<T>();
  const int logL = clamp_log(sh.log_tile, max_log_lines(p, E));
  const int lines = p.d == 3 ? p.n[1] * p.n[2] : p.n[1];
  const unsigned nb = (unsigned)(lines >> logL);
  const size_t lds = (size_t)(1 << logL) * line_pitch(p.n[0]) * sizeof(T);
#define CHIB_DIV(...)                                                                                             \
  hipLaunchKernelGGL((k_div_xdht<T, D, E, __VA_ARGS__>), dim3(nb), dim3(kThreads), lds, p.stream,                 \
                     (const T *)vel[0], (const T *)vel[1], (const T *)vel[D - 1], (T *)p.W, make_dims(p), (T)fac, \
                     logL, (const T *)p.twr[0], (const T *)p.twi[0])
  const bool r8 = sh.radix == 8;
  if constexpr (D == 3) {
    if (p.logn[0] == 8 && (logL == 3 || logL == 4)) {
      if (logL == 3 && r8) CHIB_DIV(8, 8, 3);
      else if (logL == 3) CHIB_DIV(16, 8, 3);
      else if (r8) CHIB_DIV(8, 8, 4);
      else CHIB_DIV(16, 8, 4);
      return hipGetLastError();
    }
    constexpr int RD = fixed_radix<T>();
    const bool rd = sh.radix == RD;
    if (p.logn[0] == 6 && logL == fixed_lines(6) && rd) {
      CHIB_DIV(RD, 6, fixed_lines(6));
      return hipGetLastError();
    }
    if (p.logn[0] == 7 && logL == fixed_lines(7) && !r8) {
      CHIB_DIV(16, 7, fixed_lines(7));
      return hipGetLastError();
    }
    if (p.logn[0] == 9 && logL == fixed_lines(9) && rd) {
      CHIB_DIV(RD, 9, fixed_lines(9));
      return hipGetLastError();
    }
  }
  if (r8) {
    CHIB_DIV(8);
  } else {
    CHIB_DIV(16);
  }
#undef CHIB_DIV
  return hipGetLastError();
}

template <typename T>
hipError_t launch_ydht(const Plan &p, const Plan::Shape &sh) {
  constexpr int E = tile_elems<T>();
  const int nx = p.n[0];
  const int lb = clamp_log(sh.log_tile, max_log_cols(p, p.n[1], E));
  const int lxb = p.logn[0] - lb;
  const unsigned nb = (unsigned)((nx >> lb) * p.n[2]);
  const size_t lds = (size_t)col_tile(p.n[1], 1 << lb) * sizeof(T);
#define CHIB_YDHT(...)                                                                                          \
  hipLaunchKernelGGL((k_strided_dht<__VA_ARGS__>), dim3(nb), dim3(kThreads), lds, p.stream, (T *)p.W, p.logn[1], \
                     (int64_t)nx, lb, lxb, (int64_t)nx * p.n[1], (const T *)p.twr[1], (const T *)p.twi[1])
  const bool r8 = sh.radix == 8;
  const bool fits = (int64_t)nx * p.n[1] * (int64_t)sizeof(T) < (int64_t(1) << 32);
  const bool fixed = fits && p.logn[1] == 8;
  constexpr int WB = fixed_cols<T>(7), RD = fixed_radix<T>();
  if (fits && p.logn[1] == 6 && lb == WB && sh.radix == RD) {
    CHIB_YDHT(T, E, RD, 6, WB);
  } else if (fits && p.logn[1] == 7 && lb == WB && !r8) {
    CHIB_YDHT(T, E, 16, 7, WB);
  } else if (fits && p.logn[1] == 9 && lb == WB - 1 && sh.radix == RD) {
    CHIB_YDHT(T, E, RD, 9, WB - 1);
  } else if (fixed && lb == 3) {
    if (r8) CHIB_YDHT(T, E, 8, 8, 3);
    else CHIB_YDHT(T, E, 16, 8, 3);
  } else if (fixed && lb == 4) {
    if (r8) CHIB_YDHT(T, E, 8, 8, 4);
    else CHIB_YDHT(T, E, 16, 8, 4);
  } else if (r8) {
    CHIB_YDHT(T, E, 8);
  } else {
    CHIB_YDHT(T, E, 16);
  }
#undef CHIB_YDHT
  return hipGetLastError();
}

template <typename T>
hipError_t launch_neumann(const Plan &p, const Plan::Shape &sh) {
  constexpr int E = tile_elems<T>();
  const int nx = p.n[0];
  const int ax = p.d - 1;
  const int Nn = p.n[ax];
  const int lb = clamp_log(sh.log_tile, max_log_cols(p, Nn, E));
  const int lxb = p.logn[0] - lb;
  const int64_t stride = p.d == 3 ? (int64_t)nx * p.n[1] : (int64_t)nx;
  const int64_t outer = p.d == 3 ? (int64_t)nx : 0;
  const unsigned nb = (unsigned)((nx >> lb) * (p.d == 3 ? p.n[1] : 1));
  const size_t lds = (size_t)col_tile(Nn, 1 << lb) * sizeof(T);
  const double norm = (double)p.N;  // 1/(nx [ny] n_last): inverse Hartley scales and the inverse FFT
  const T *lamy = p.d == 3 ? (const T *)p.lam[1] : (const T *)nullptr;
#define CHIB_NEUMANN(...)                                                                                        \
  hipLaunchKernelGGL((k_neumann_solve<__VA_ARGS__>), dim3(nb), dim3(kThreads), lds, p.stream, (T *)p.W,          \
                     p.logn[ax], stride, lb, lxb, outer, (const T *)p.lam[0], lamy, (const T *)p.lam[ax], (T)p.a, \
                     (T)p.alpha_s, (T)(1.0 / norm), (const T *)p.twr[ax], (const T *)p.twi[ax],               \
                     (const T *)p.dctc, (const T *)p.dcts, p.poisson)
  // 256-point lines in a full tile
  constexpr int FB = ilog2c(E / 256);
  const bool fits = stride * Nn * (int64_t)sizeof(T) < (int64_t(1) << 32);
  const bool fixed = fits && p.logn[ax] == 8 && lb == FB;
  constexpr int WB = fixed_cols<T>(7), RD = fixed_radix<T>();
  if (fits && p.logn[ax] == 6 && lb == WB && sh.radix == RD) {
    CHIB_NEUMANN(T, E, RD, 6, WB);
  } else if (fits && p.logn[ax] == 7 && lb == WB && sh.radix == 16) {
    CHIB_NEUMANN(T, E, 16, 7, WB);
  } else if (fits && p.logn[ax] == 9 && lb == WB - 1 && sh.radix == RD) {
    CHIB_NEUMANN(T, E, RD, 9, WB - 1);
  } else if (fixed) {
    if (sh.radix == 8) CHIB_NEUMANN(T, E, 8, 8, FB);
    else CHIB_NEUMANN(T, E, 16, 8, FB);
  } else if (sh.radix == 8) {
    CHIB_NEUMANN(T, E, 8);
  } else {
    CHIB_NEUMANN(T, E, 16);
  }
#undef CHIB_NEUMANN
  return hipGetLastError();
}

template <typename T, int D, int U, int R, int CLN = 0>
void launch_rhs_variant(const Plan &p, const T *Cn, const T *Cp, int logL, unsigned nb, size_t lds) {
  const Dims dm = make_dims(p);
  const RhsCoef<T> cf = make_coef<T>(p);
  hipLaunchKernelGGL((k_rhs_xdht<T, D, tile_elems<T>(), U, R, CLN>), dim3(nb), dim3(kThreads), lds, p.stream, Cn, Cp,
                     (const T *)adv_face(p, 0), (const T *)adv_face(p, 1), (const T *)(D == 3 ? adv_face(p, 2) : adv_face(p, 1)), (T *)p.W, dm, cf,
                     logL, (const T *)p.twr[0], (const T *)p.twi[0], make_patch<T>(p));
}

// y-marching variant (2D, nx up to 1024): unroll = 3.
inline bool ym_ok(const Plan &p) { return p.d == 2 && p.n[0] <= 1024; }

template <typename T, int XM, int R>
void launch_ym_variant(const Plan &p, const T *Cn, const T *Cp, int logL) {
  const Dims dm = make_dims(p);
  const RhsCoef<T> cf = make_coef<T>(p);
  const unsigned nb = (unsigned)(p.n[1] >> logL);
  const size_t lds = ((size_t)(1 << logL) * line_pitch(p.n[0]) + ym_extra(p.n[0])) * sizeof(T);
  hipLaunchKernelGGL((k_rhs_xdht_ym<T, XM, R>), dim3(nb), dim3(kThreads), lds, p.stream, Cn, Cp,
                     (const T *)adv_face(p, 0), (const T *)adv_face(p, 1), (T *)p.W, dm, cf, logL, (const T *)p.twr[0],
                     (const T *)p.twi[0], make_patch<T>(p));
}

template <typename T, int R>
void launch_ym(const Plan &p, const T *Cn, const T *Cp, int logL) {
  if (p.n[0] <= 256) launch_ym_variant<T, 1, R>(p, Cn, Cp, logL);
  else if (p.n[0] <= 512) launch_ym_variant<T, 2, R>(p, Cn, Cp, logL);
  else launch_ym_variant<T, 4, R>(p, Cn, Cp, logL);
}

// z-marching variant (3D, nx a multiple of 256 up to 512): unroll = log2 of the planes per chunk.
inline bool zm_ok(const Plan &p) { return p.d == 3 && (p.n[0] == 256 || p.n[0] == 512) && p.n[1] >= 2; }

template <typename T, int L, int XM, int R, bool SPLIT = false>
void launch_zm_variant(const Plan &p, const T *Cn, const T *Cp, int zc_log) {
  const Dims dm = make_dims(p);
  const RhsCoef<T> cf = make_coef<T>(p);
  const unsigned nb = (unsigned)((p.n[1] / L) * (p.n[2] >> zc_log));
  const size_t lds = ((size_t)2 * L * p.n[0] + (SPLIT ? 0 : (size_t)L * line_pitch(p.n[0]) + 2 * p.n[0])) * sizeof(T);
  hipLaunchKernelGGL((k_rhs_xdht_zm<T, L, XM, R, SPLIT>), dim3(nb), dim3(kThreads), lds, p.stream, Cn, Cp,
                     (const T *)adv_face(p, 0), (const T *)adv_face(p, 1), (const T *)adv_face(p, 2), (T *)p.W, dm, cf, zc_log,
                     (const T *)p.twr[0], (const T *)p.twi[0], make_patch<T>(p));
}

// Whether the line-tiled rhs has a fixed-size form of this grid's lines.
inline bool rhs_wide(const Plan &p) { return p.d == 3 && p.logn[0] >= 6 && p.logn[0] <= 9; }

// Whether pass 0 in this shape takes the z-march, whose patch comes as dq per entry.
inline bool rhs_reads_dq(const Plan &p, const Plan::Shape &sh) { return p.d == 3 && sh.unroll >= 3 && zm_ok(p); }

// Stencil-only z-march (the rhs Q into W, no transform) with L rows per tile.
template <typename T, int XM>
void launch_zm_split(const Plan &p, const T *Cn, const T *Cp, int logL, int zc_log) {
  if (logL <= 1) launch_zm_variant<T, 2, XM, 8, true>(p, Cn, Cp, zc_log);
  else if (logL == 2) launch_zm_variant<T, 4, XM, 8, true>(p, Cn, Cp, zc_log);
  else if constexpr (XM == 1) launch_zm_variant<T, 8, XM, 8, true>(p, Cn, Cp, zc_log);
}

template <typename T, int XM>
void launch_zm_xm(const Plan &p, const T *Cn, const T *Cp, int logL, int radix, int zc_log) {
  if (logL <= 1) {
    if (radix == 4) launch_zm_variant<T, 2, XM, 4>(p, Cn, Cp, zc_log);
    else if (radix == 8) launch_zm_variant<T, 2, XM, 8>(p, Cn, Cp, zc_log);
    else launch_zm_variant<T, 2, XM, 16>(p, Cn, Cp, zc_log);
  } else if (logL == 2) {
    if (radix == 4) launch_zm_variant<T, 4, XM, 4>(p, Cn, Cp, zc_log);
    else if (radix == 8) launch_zm_variant<T, 4, XM, 8>(p, Cn, Cp, zc_log);
    else launch_zm_variant<T, 4, XM, 16>(p, Cn, Cp, zc_log);
  } else if constexpr (XM == 1) {   // (512-wide grids take at most 4 rows per tile)
    if (radix <= 8) launch_zm_variant<T, 8, XM, 8>(p, Cn, Cp, zc_log);
    else launch_zm_variant<T, 8, XM, 16>(p, Cn, Cp, zc_log);
  }
}

// Pass 0.  unroll 1-2: one fused rhs + x-transform kernel per line tile; 2D, 3: the y-marching
// form of it (nx up to 1024); 3D, 3-5: the same fused
// work z-marching over 2^unroll planes (3D, nx 256 or 512); 6-8: a stencil-only z-march over
// 2^(unroll-3) planes writing Q, then the x transform of W in place (with split_only, the
// caller launches that transform itself).
template <typename T, int D>
hipError_t launch_rhs(const Plan &p, const T *Cn, const T *Cp, const Plan::Shape &sh, bool split_only = false) {
  constexpr int E = tile_elems<T>();
  if (D == 3 && rhs_reads_dq(p, sh)) {
    int logL = sh.log_tile < 1 ? 1 : (sh.log_tile > 3 ? 3 : sh.log_tile);
    if (p.n[0] == 512 && logL > 2) logL = 2;   // two 512-wide planes of C~ and x faces plus the tile stay in LDS
    while ((1 << logL) > p.n[1]) --logL;
    const bool split = sh.unroll >= 6;
    int zc_log = split ? sh.unroll - 3 : sh.unroll;
    while ((1 << zc_log) > p.n[2]) --zc_log;
    if (split) {
      if (p.n[0] == 256) launch_zm_split<T, 1>(p, Cn, Cp, logL, zc_log);
      else launch_zm_split<T, 2>(p, Cn, Cp, logL, zc_log);
      hipError_t e = hipGetLastError();
      if (e == hipSuccess) e = launch_rhs_patch<T>(p, (T *)p.W);
      if (e != hipSuccess || split_only) return e;
      return launch_xdht<T>(p, (const T *)p.W, (T *)p.W, p.shape[3]);
    }
    if (p.n[0] == 256) launch_zm_xm<T, 1>(p, Cn, Cp, logL, sh.radix, zc_log);
    else launch_zm_xm<T, 2>(p, Cn, Cp, logL, sh.radix, zc_log);
    return hipGetLastError();
  }
  const int logL = clamp_log(sh.log_tile, max_log_lines(p, E));
  if (D == 2 && sh.unroll == 3 && ym_ok(p)) {
    if (sh.radix <= 8) launch_ym<T, 8>(p, Cn, Cp, logL);
    else launch_ym<T, 16>(p, Cn, Cp, logL);
    return hipGetLastError();
  }
  const int lines = p.d == 3 ? p.n[1] * p.n[2] : p.n[1];
  const unsigned nb = (unsigned)(lines >> logL);
  const size_t lds = (size_t)(1 << logL) * line_pitch(p.n[0]) * sizeof(T);
  const bool r8 = sh.radix <= 8, u2 = sh.unroll >= 2;
  if constexpr (D == 3) {
    if (rhs_wide(p)) {
      switch (p.logn[0] * 2 + r8) {
        case 12: launch_rhs_variant<T, D, 1, 16, 6>(p, Cn, Cp, logL, nb, lds); break;
        case 13: launch_rhs_variant<T, D, 1, 8, 6>(p, Cn, Cp, logL, nb, lds); break;
        case 14: launch_rhs_variant<T, D, 1, 16, 7>(p, Cn, Cp, logL, nb, lds); break;
        case 15: launch_rhs_variant<T, D, 1, 8, 7>(p, Cn, Cp, logL, nb, lds); break;
        case 16: launch_rhs_variant<T, D, 1, 16, 8>(p, Cn, Cp, logL, nb, lds); break;
        case 17: launch_rhs_variant<T, D, 1, 8, 8>(p, Cn, Cp, logL, nb, lds); break;
        case 18: launch_rhs_variant<T, D, 1, 16, 9>(p, Cn, Cp, logL, nb, lds); break;
        default: launch_rhs_variant<T, D, 1, 8, 9>(p, Cn, Cp, logL, nb, lds); break;
      }
      return hipGetLastError();
    }
  }
  if (r8 && u2) launch_rhs_variant<T, D, 2, 8>(p, Cn, Cp, logL, nb, lds);
  else if (r8) launch_rhs_variant<T, D, 1, 8>(p, Cn, Cp, logL, nb, lds);
  else if (u2) launch_rhs_variant<T, D, 2, 16>(p, Cn, Cp, logL, nb, lds);
  else launch_rhs_variant<T, D, 1, 16>(p, Cn, Cp, logL, nb, lds);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_spectral_tail(const Plan &p, KernelTimer *tm = nullptr) {
  hipError_t e = hipSuccess;
  auto mark = [&](const char *name) {
    if (tm && e == hipSuccess) e = tm->mark(name, p.stream);
  };
  if (p.d == 3) {
    mark("ydht_fwd");
    if (e == hipSuccess) e = launch_ydht<T>(p, p.shape[1]);
  }
  mark("neumann_solve");
  if (e == hipSuccess) e = launch_neumann<T>(p, p.shape[2]);
  if (p.d == 3) {
    mark("ydht_inv");
    if (e == hipSuccess) e = launch_ydht<T>(p, p.shape[1]);
  }
  return e;
}

template <typename T>
hipError_t launch_ghost_fill(const Plan &p, T *Cout, int init) {
  if (p.G == 0) return hipSuccess;
  const unsigned nb = blocks_for(p.G);
  const Dims dm = make_dims(p);
  if (!p.dynamic) {
    const T cb = (T)(p.cos_t / (1.4142135623730951 * p.Cn));
    hipLaunchKernelGGL((k_fill_static<T>), dim3(blocks_for(p.G * 16)), dim3(kThreads), 0, p.stream, Cout, p.gidx,
                       (const T *)p.dn,
                       (const T *)p.gamma, p.apg, (const T *)p.wg, (T *)p.CGn, (T *)p.CGnm1, (T *)p.CMs, p.G, p.K, cb,
                       init);
  } else {
    if (!init)
      hipLaunchKernelGGL((k_scatter_pg<T>), dim3(nb), dim3(kThreads), 0, p.stream, Cout, p.gidx,
                         (const T *)p.CGn, (const T *)p.CGnm1, p.G);
#define CHIB_FILL_DYNAMIC(D)                                                                                         \
  hipLaunchKernelGGL((k_fill_dynamic<T, D>), dim3(blocks_for(p.G * 16)), dim3(kThreads), 0, p.stream,                \
                     (const T *)Cout, (const T *)p.F[0], (const T *)p.F[1], (const T *)p.F[D - 1], p.gidx,           \
                     (const T *)p.normal, (const T *)p.dn, (const T *)p.gamma, p.apg, (const T *)p.wg, (T *)p.CI,    \
                     (T *)p.CGnew, (T *)p.CMs, p.G, p.K, dm, (T)(0.5 / p.h), (T)p.Cn, (T)p.Vs, (T)p.cos_t, (T)p.dt,  \
                     init)
    if (p.d == 2) CHIB_FILL_DYNAMIC(2);
    else CHIB_FILL_DYNAMIC(3);
#undef CHIB_FILL_DYNAMIC
    hipLaunchKernelGGL((k_commit_ghosts<T>), dim3(nb), dim3(kThreads), 0, p.stream, Cout, p.gidx,
                       (const T *)p.CGnew, (T *)p.CGn, (T *)p.CGnm1, p.G, init);
  }
  return hipGetLastError();
}

// The face means of the velocity fill; next (the new C and the C before it) adds the first kernel of
// the next step's ghost patch to the launch.
template <typename T>
hipError_t launch_velocity_faces(const Plan &p, const NextStep *next) {
  if (next && p.NF && has_patch(p)) {
    const Dims dm = make_dims(p);
    const unsigned nbf = blocks_for(p.NF);
    const bool pts = dphi_points(p);
#define CHIB_FACES_DPHI(P)                                                                                           \
  hipLaunchKernelGGL((k_vel_faces_dphi<T, P>), dim3(nbf + blocks_for(P ? p.NU : p.G * 16)), dim3(kThreads), 0,       \
                     p.stream, (T *)p.F[0], (T *)p.F[1], (T *)p.F[2], (const T *)p.UG, p.G, p.f_cell, p.f_axis,      \
                     p.f_gL, p.f_gR, (const T *)p.stashL, (const T *)p.stashR, p.NF, nbf, (const T *)next->Cn,       \
                     (const T *)next->Cp, P ? p.pt_cell : p.gidx, (T *)(P ? p.pt_phi : p.dg), p.NU, p.apg,           \
                     (const T *)p.wg, p.K, dm, p.d, (T)(p.Cn * p.Cn), (T)(1.0 / (p.h * p.h)),                        \
                     (T)(1.0 / (p.Cn * p.Cn)))
    if (pts) CHIB_FACES_DPHI(true);
    else CHIB_FACES_DPHI(false);
#undef CHIB_FACES_DPHI
    return hipGetLastError();
  }
  if (p.NF)
    hipLaunchKernelGGL((k_vel_faces<T>), dim3(blocks_for(p.NF)), dim3(kThreads), 0, p.stream, (T *)p.F[0],
                       (T *)p.F[1], (T *)p.F[2], (const T *)p.UG, p.G, p.f_cell, p.f_axis, p.f_gL, p.f_gR,
                       (const T *)p.stashL, (const T *)p.stashR, p.NF);
  return hipGetLastError();
}

// Static condition with the velocity fill: C ghosts and ghost velocities in one launch, then the faces.
template <typename T>
hipError_t launch_static_fills(const Plan &p, T *Cout, const NextStep *next) {
  const Dims dm = make_dims(p);
  const unsigned nbc = blocks_for(p.G * 16), nbg = blocks_for(p.G * 16);
  const T cb = (T)(p.cos_t / (1.4142135623730951 * p.Cn));
#define CHIB_FILL_STATIC_VEL(D)                                                                                     \
  hipLaunchKernelGGL((k_fill_static_vel<T, D>), dim3(nbc + nbg + blocks_for(p.NF)), dim3(kThreads), 0, p.stream,    \
                     Cout, p.gidx, (const T *)p.dn, (const T *)p.gamma, p.apg, (const T *)p.wg, (T *)p.CGn,         \
                     (T *)p.CGnm1, (T *)p.CMs, p.G, p.K, cb, (const T *)p.F[0], (const T *)p.F[1],                  \
                     (const T *)p.F[D - 1], (const T *)p.normal, (T *)p.UG, p.f_cell, p.f_axis, p.f_gL, p.f_gR,     \
                     (T *)p.stashL, (T *)p.stashR, p.NF, dm, (T)(0.5 / p.h), (T)p.Cn, (T)p.cos_t, (T)(1.0 / p.Ca),  \
                     (T)(1.0 / p.mu), (T)p.ls, nbc, nbg)
  if (p.d == 2) CHIB_FILL_STATIC_VEL(2);
  else CHIB_FILL_STATIC_VEL(3);
#undef CHIB_FILL_STATIC_VEL
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? launch_velocity_faces<T>(p, next) : e;
}

template <typename T>
hipError_t launch_velocity_fill(const Plan &p, const T *Cfin, const NextStep *next = nullptr) {
  if (!p.vel_fill || p.G == 0) return hipSuccess;
  const Dims dm = make_dims(p);
  const unsigned nbg = blocks_for(p.G * 16);
#define CHIB_VEL_GHOSTS(D, CAP)                                                                                     \
  hipLaunchKernelGGL((k_vel_ghosts<T, D, CAP>), dim3(nbg + blocks_for(p.NF)), dim3(kThreads), 0, p.stream, Cfin,    \
                     (const T *)p.F[0], (const T *)p.F[1], (const T *)p.F[D - 1], p.gidx, (const T *)p.normal,      \
                     (const T *)p.dn, (const T *)p.gamma, p.apg, (const T *)p.wg, (const T *)p.CMs, (T *)p.UG, p.G, \
                     p.K, p.f_cell, p.f_axis, p.f_gL, p.f_gR, (T *)p.stashL, (T *)p.stashR, p.NF, dm,               \
                     (T)(0.5 / p.h), (T)p.Cn, (T)p.cos_t, (T)(1.0 / p.Ca), (T)(1.0 / p.mu), (T)p.ls, nbg)
  if (p.d == 2 && p.dynamic) CHIB_VEL_GHOSTS(2, true);
  else if (p.d == 2) CHIB_VEL_GHOSTS(2, false);
  else if (p.dynamic) CHIB_VEL_GHOSTS(3, true);
  else CHIB_VEL_GHOSTS(3, false);
#undef CHIB_VEL_GHOSTS
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? launch_velocity_faces<T>(p, next) : e;
}

}  // namespace

// The fills that end a step, on the new field C: ghost values of C, then the velocity fill
// (with the static condition both in one launch plus the face pass).
template <typename T>
hipError_t launch_step_fills(const Plan &p, T *C, KernelTimer *tm, const NextStep *next) {
  hipError_t e = hipSuccess;
  auto mark = [&](const char *name) {
    if (tm && e == hipSuccess) e = tm->mark(name, p.stream);
  };
  if (!p.dynamic && p.vel_fill && p.G) {
    mark("ghost_fills");
    if (e == hipSuccess) e = launch_static_fills<T>(p, C, next);
  } else {
    mark("ghost_fill_C");
    if (e == hipSuccess) e = launch_ghost_fill<T>(p, C, 0);
    if (p.vel_fill && p.G) mark("ghost_fill_u");
    if (e == hipSuccess) e = launch_velocity_fill<T>(p, C, next);
  }
  return e;
}

template <typename T>
hipError_t enqueue_step(const Plan &p, int cur, KernelTimer *tm, StepLink *link) {
  const T *Cn = (const T *)p.C[cur];
  T *Cp = (T *)p.C[1 - cur];
  hipError_t e = hipSuccess;
  auto mark = [&](const char *name) {
    if (tm && e == hipSuccess) e = tm->mark(name, p.stream);
  };
  const bool split = p.d == 3 && p.shape[0].unroll >= 6 && zm_ok(p);
  if (p.G) {
    mark("ghost_dphi");
    if (e == hipSuccess) e = launch_ghost_patch<T>(p, Cn, Cp, rhs_reads_dq(p, p.shape[0]), link && link->dphi_done);
  }
  mark(split ? "rhs_stencil" : "rhs_xdht");
  if (e == hipSuccess)
    e = p.d == 2 ? launch_rhs<T, 2>(p, Cn, Cp, p.shape[0], true) : launch_rhs<T, 3>(p, Cn, Cp, p.shape[0], true);
  if (split) {
    mark("xdht_fwd");
    if (e == hipSuccess) e = launch_xdht<T>(p, (const T *)p.W, (T *)p.W, p.shape[3]);
  }
  if (e == hipSuccess) e = launch_spectral_tail<T>(p, tm);
  mark("xdht_out");
  if (e == hipSuccess) e = launch_xdht<T>(p, (const T *)p.W, Cp, p.shape[3]);
  // another semi-implicit step follows: the first kernel of its ghost patch joins the face pass
  const NextStep nx{Cp, Cn};
  const bool join = link && link->next && p.vel_fill && p.NF && has_patch(p);
  if (e == hipSuccess) e = launch_step_fills<T>(p, Cp, tm, join ? &nx : nullptr);
  if (link) link->dphi_done = join && e == hipSuccess;
  if (tm && e == hipSuccess) e = tm->end(p.stream);
  return e;
}

// Launch shapes before any tuning, from the grid alone.  A pass needs some 1024 workgroups to keep 256
// compute units busy through its memory round trips; past that, larger tiles share a workgroup's fixed
// costs (barriers, twiddles) among more lines.  So every tile takes as many lines as leave that many
// workgroups, within its 32 KB (2D grids: 2 lines or columns, a launch of a few microseconds is all
// latency).  Measured per step against the former fixed shapes {8 lines, 16 columns, line-tiled rhs}:
// 512x256 FP64 40.1 -> 25.5 us, 1024x512 FP32 55.2 -> 33.5 (dynamic angle 64.4 -> 42.8), 64^3 FP64 37.2 -> 32.0.
// Lines of 64 to 512 points take the width of their fixed-size instance from 128 tiles on, which saves more than
// the emptier chip costs (64^3 38 -> 34 us with 256 tiles instead of 1024, 64x64x32 33.9 -> 31.8 with 128).
// rhs, 3D: the z-march reads C once instead of three times and wins from 2^23 cells (256x256x128 FP64 123 us
// line-tiled, 88 marching; 256x128x128 45 and 51 and the march's dq list 5 more, FP32 31 and 37; 512x128x128
// 137 and 105), with the longest march that leaves 512 workgroups (1024 in FP32, whose planes are half as long
// in flight).  Line-tiled, 1024 cells a tile (FP32 2048) beat more and fewer: 128^3 FP64 39, 29.0, 28.1 and
// 29.2 us at 2, 4, 8 and 16 lines, 128x256x256 122, 104 and 108 at 4, 8 and 16, 64^3 12.3 and 9.1 at 2 and 4.  rhs, 2D: the y-march for
// all widths it serves in FP64, at one radix, so that a batch of uneven sizes shares its kernels.
// FP32 keeps the transforms at radix 16 and the rhs at 8: fewer stages round less, and rounding is what limits
// it (64^3 coupled, 10 steps: u off by 2.2e-6 with the solve at radix 8, 1.3e-6 at 16).
template <typename T>
void default_shapes(Plan &p) {
  constexpr int E = tile_elems<T>();
  auto height = [](int64_t items, int hi) {   // log2 of the items per tile
    int l = 1;
    while (l < hi && (items >> (l + 1)) >= 1024) ++l;
    return l;
  };
  if (p.d == 2) {
    const int wide = p.n[0] >= 1024 ? 2 : 1;
    const bool f64 = sizeof(T) == 8;
    // FP32 takes the line-tiled rhs: its requests are half as long and the rows come from L2, so the march gains
    // nothing (1024x512 33.5 and 33.8 us a step, 512x256 26.3 and 26.8, batch of 32 cases 105 and 110)
    p.shape[0] = {1, 8, ym_ok(p) && f64 ? 3 : 1};
    p.shape[1] = {4, 16, 1};
    p.shape[2] = {clamp_log(wide, max_log_cols(p, p.n[1], E)), f64 ? 8 : 16, 1};
    p.shape[3] = {1, f64 ? 8 : 16, 1};
    return;
  }
  const int64_t lines = (int64_t)p.n[1] * p.n[2];
  const int hl = max_log_lines(p, E);
  // radix by line length: 8 where its stages divide the line evenly, else 16 (fewer stages)
  auto radix = [](int logn) { return sizeof(T) == 8 && (logn == 8 || logn % 3 == 0 || logn == 5) ? 8 : 16; };
  if (zm_ok(p) && p.N >= (int64_t(1) << 23)) {
    const int L = sizeof(T) == 8 ? (p.n[0] == 512 ? 1 : 2) : (p.n[0] == 512 ? 2 : 3);
    int zc = 5;
    const int64_t want = sizeof(T) == 8 ? 512 : 1024;
    while (zc > 3 && ((int64_t)(p.n[1] >> L) * (p.n[2] >> zc)) < want) --zc;
    p.shape[0] = {L, sizeof(T) == 4 ? 8 : 4, zc};
  } else {
    // two passes of the block over the tile's cells (see rhs_xdht_body), one on grids of few lines
    const int cap = rhs_wide(p) ? ilog2c(8192 / (int)sizeof(T)) - p.logn[0] : hl;
    int l = rhs_wide(p) && p.n[0] <= 128 ? 2 : 1;
    while (l < cap && (lines >> (l + 1)) >= (rhs_wide(p) ? 512 : 1024)) ++l;
    p.shape[0] = {clamp_log(l, hl), 8, p.n[0] >= 256 ? 2 : 1};
  }
  const int cy = max_log_cols(p, p.n[1], E), cz = max_log_cols(p, p.n[2], E);
  auto width = [&](int64_t items, int logn, int wd, int hi) {
    const bool fixed = logn >= 6 && logn <= 9 && wd <= hi && (logn == 8 || (items >> wd) >= 128);
    return fixed ? wd : height(items, hi);
  };
  p.shape[1] = {width((int64_t)p.n[0] * p.n[2], p.logn[1], p.n[1] == 256 ? 4 : fixed_cols<T>(p.logn[1]), cy),
                p.n[1] == 256 ? 16 : radix(p.logn[1]), 1};
  p.shape[2] = {width((int64_t)p.n[0] * p.n[1], p.logn[2], p.n[2] == 256 ? cz : fixed_cols<T>(p.logn[2]), cz),
                p.n[2] == 256 ? (sizeof(T) == 8 ? 8 : 16) : radix(p.logn[2]), 1};
  p.shape[3] = {width(lines, p.logn[0], p.n[0] == 256 ? (sizeof(T) == 8 ? 3 : 4) : fixed_lines(p.logn[0]), hl),
                p.n[0] == 256 && sizeof(T) == 4 ? 16 : radix(p.logn[0]), 1};
}

// Tile heights of a 2D state inside a batch of `cells` cells: the batch as a whole fills the chip, so each
// tile of the x passes takes the lines that leave it about 1024 workgroups, and past two million cells 2048
// (32 cases of 5.8 million cells: FP64 148 us a step with 1024, 139 with 2048, 144 with 4096; 6 cases of 1.3
// million: 64 with 1024, 69 with 2048).  The bounded axis takes the widths of the fixed-size solves, FP32,
// which has none here, only past two million cells (32 cases 113 -> 108 us; 6 cases 58 -> 61).  Heights
// change no result.
template <typename T>
void batch_heights(Plan &p, int64_t cells) {
  constexpr int E = tile_elems<T>();
  const bool large = cells >= (int64_t(1) << 21);
  const int64_t per = large ? cells / 2048 : cells / 1024;   // elements per workgroup
  auto height = [&](int n, int hi) {
    int l = 1;
    while (l < hi && ((int64_t)n << (l + 1)) <= per) ++l;
    return l;
  };
  const int hl = max_log_lines(p, E);
  p.shape[0].log_tile = height(p.n[0], hl);
  const int hc = max_log_cols(p, p.n[1], E);
  p.shape[2].log_tile =
      sizeof(T) == 8 || large ? clamp_log(fixed_cols<T>(p.logn[1]), hc) : height(p.n[1], hc);
  p.shape[3].log_tile = height(p.n[0], hl);
}

// Times every candidate shape of each pass on the state's buffers (the spectral workspace
// only; the fields are not modified) and keeps the fastest.  `out` receives the chosen
// shapes.  The candidates: lines/columns per tile from 2 to the 32 KB LDS limit, radix 8 or
// 16, and 1 or 2 cells in flight per thread in the fused rhs pass.
template <typename T>
hipError_t tune_shapes(Plan &p, int cur, int reps) {
  constexpr int E = tile_elems<T>();
  hipEvent_t e0, e1;
  hipError_t e = hipEventCreate(&e0);
  if (e != hipSuccess) return e;
  e = hipEventCreate(&e1);
  if (e != hipSuccess) {
    (void)hipEventDestroy(e0);
    return e;
  }
  auto time_it = [&](auto &&launch) -> float {
    float best = 1e30f;
    for (int w = 0; w < 2 && e == hipSuccess; ++w) e = launch();
    for (int r = 0; r < reps && e == hipSuccess; ++r) {
      e = hipEventRecord(e0, p.stream);
      if (e == hipSuccess) e = launch();
      if (e == hipSuccess) e = hipEventRecord(e1, p.stream);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      float ms = 0.f;
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
      if (ms < best) best = ms;
    }
    return best;
  };
  // the transform passes are timed where the step runs them, right after the passes before them
  // (untimed): repeated on their own, W stays in the 256 MB Infinity Cache, which the fused rhs
  // pass's streaming traffic flushes in a real step, and the tuner would favour other shapes
  auto time_after = [&](auto &&pre, auto &&launch) -> float {
    float best = 1e30f;
    for (int w = 0; w < 2 && e == hipSuccess; ++w) {
      e = pre();
      if (e == hipSuccess) e = launch();
    }
    for (int r = 0; r < reps && e == hipSuccess; ++r) {
      e = pre();
      if (e == hipSuccess) e = hipEventRecord(e0, p.stream);
      if (e == hipSuccess) e = launch();
      if (e == hipSuccess) e = hipEventRecord(e1, p.stream);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      float ms = 0.f;
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
      if (ms < best) best = ms;
    }
    return best;
  };
  const T *Cn = (const T *)p.C[cur];
  const T *Cp = (const T *)p.C[1 - cur];
  e = launch_ghost_patch<T>(p, Cn, Cp, true);   // the rhs candidates read the ghost patch
  auto rhs = [&]() { return p.d == 2 ? launch_rhs<T, 2>(p, Cn, Cp, p.shape[0]) : launch_rhs<T, 3>(p, Cn, Cp, p.shape[0]); };
  // pass 0: fused rhs
  if (e == hipSuccess) {
    const int hi = max_log_lines(p, E);
    float best = 1e30f;
    Plan::Shape bs = p.shape[0];
    for (int lt = 1; lt <= hi; ++lt)
      for (int radix : {4, 8, 16})
        for (int un : {1, 2, 3, 4, 5, 6, 7, 8}) {
          const int zl = un >= 6 ? un - 3 : un;
          if (radix == 4 && (p.d != 3 || un < 3 || un > 5 || lt > 2)) continue;   // z-march only
          if (un == 2 && rhs_wide(p)) continue;   // the same kernel as with one cell in flight
          if (un >= 3 && p.d == 2 && (un != 3 || !ym_ok(p))) continue;
          if (un >= 3 && p.d == 3 && (!zm_ok(p) || lt > 3 || (1 << lt) > p.n[1] || (1 << zl) > p.n[2])) continue;
          if (un >= 6 && radix == 16) continue;   // the stencil-only kernel has no transform
          Plan::Shape sh{lt, radix, un};
          const float t = time_it([&]() {
            return p.d == 2 ? launch_rhs<T, 2>(p, Cn, Cp, sh) : launch_rhs<T, 3>(p, Cn, Cp, sh);
          });
          if (e != hipSuccess) break;
          if (t < best) {
            best = t;
            bs = sh;
          }
        }
    p.shape[0] = bs;
  }
  // pass 1: strided Hartley (3D); pass 2: bounded-axis solve (in place on W)
  if (p.d == 3 && e == hipSuccess) {
    const int hi = max_log_cols(p, p.n[1], E);
    float best = 1e30f;
    Plan::Shape bs = p.shape[1];
    for (int lt = 1; lt <= hi; ++lt)
      for (int radix : {8, 16}) {
        Plan::Shape sh{lt, radix, 1};
        // the shape serves the forward pass (after the rhs) and the inverse one (after the solve)
        const float t = time_after(rhs, [&]() { return launch_ydht<T>(p, sh); }) +
                        time_after([&]() {
                          hipError_t r = rhs();
                          if (r == hipSuccess) r = launch_ydht<T>(p, sh);
                          return r == hipSuccess ? launch_neumann<T>(p, p.shape[2]) : r;
                        }, [&]() { return launch_ydht<T>(p, sh); });
        if (e != hipSuccess) break;
        if (t < best) {
          best = t;
          bs = sh;
        }
      }
    p.shape[1] = bs;
  }
  if (e == hipSuccess) {
    const int hi = max_log_cols(p, p.n[p.d - 1], E);
    float best = 1e30f;
    Plan::Shape bs = p.shape[2];
    for (int lt = 1; lt <= hi; ++lt)
      for (int radix : {8, 16}) {
        Plan::Shape sh{lt, radix, 1};
        const float t = time_after([&]() {
          hipError_t r = rhs();
          return (r == hipSuccess && p.d == 3) ? launch_ydht<T>(p, p.shape[1]) : r;
        }, [&]() { return launch_neumann<T>(p, sh); });
        if (e != hipSuccess) break;
        if (t < best) {
          best = t;
          bs = sh;
        }
      }
    p.shape[2] = bs;
  }
  // pass 3: x Hartley, W -> W (in place: each tile is read whole before it is written)
  if (e == hipSuccess) {
    const int hi = max_log_lines(p, E);
    float best = 1e30f;
    Plan::Shape bs = p.shape[3];
    for (int lt = 1; lt <= hi; ++lt)
      for (int radix : {8, 16}) {
        Plan::Shape sh{lt, radix, 1};
        const float t = time_after([&]() {
          hipError_t r = rhs();
          if (r == hipSuccess) r = launch_spectral_tail<T>(p);
          return r;
        }, [&]() { return launch_xdht<T>(p, (const T *)p.W, (T *)p.W, sh); });
        if (e != hipSuccess) break;
        if (t < best) {
          best = t;
          bs = sh;
        }
      }
    p.shape[3] = bs;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return e;
}

template <typename T>
hipError_t enqueue_initial_fill(const Plan &p, int cur) {
  T *C = (T *)p.C[cur];
  hipError_t e = launch_ghost_fill<T>(p, C, 1);
  if (e != hipSuccess) return e;
  e = launch_velocity_fill<T>(p, C);
  if (e != hipSuccess) return e;
  return hipMemcpyAsync(p.C[1 - cur], p.C[cur], (size_t)p.N * sizeof(T), hipMemcpyDeviceToDevice, p.stream);
}

template <typename T>
hipError_t enqueue_ghost_refresh(const Plan &p, int cur) {
  if (p.dynamic) return hipErrorInvalidValue;   // the dynamic fill advances C_I: not repeatable
  return launch_ghost_fill<T>(p, (T *)p.C[cur], 2);
}

template <typename T>
hipError_t enqueue_rhs(const Plan &p, int cur, void *out) {
  const Dims dm = make_dims(p);
  const RhsCoef<T> cf = make_coef<T>(p);
  const T *F2 = (const T *)(p.d == 3 ? adv_face(p, 2) : adv_face(p, 1));
  hipError_t e = launch_ghost_patch<T>(p, (const T *)p.C[cur], (const T *)p.C[1 - cur], true);
  if (e != hipSuccess) return e;
  if (p.d == 2)
    hipLaunchKernelGGL((k_rhs_only<T, 2>), dim3(blocks_for(p.N)), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                       (const T *)p.C[1 - cur], (const T *)adv_face(p, 0), (const T *)adv_face(p, 1), F2, (T *)out, dm, cf, p.N);
  else
    hipLaunchKernelGGL((k_rhs_only<T, 3>), dim3(blocks_for(p.N)), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                       (const T *)p.C[1 - cur], (const T *)adv_face(p, 0), (const T *)adv_face(p, 1), F2, (T *)out, dm, cf, p.N);
  e = hipGetLastError();
  return e == hipSuccess ? launch_rhs_patch<T>(p, (T *)out) : e;
}

template <typename T>
hipError_t enqueue_solve(const Plan &p, const void *in, void *out) {
  hipError_t e = launch_xdht<T>(p, (const T *)in, (T *)p.W, p.shape[3]);
  if (e != hipSuccess) return e;
  if ((e = launch_spectral_tail<T>(p)) != hipSuccess) return e;
  return launch_xdht<T>(p, (const T *)p.W, (T *)out, p.shape[3]);
}

template <typename T>
hipError_t enqueue_poisson(const Plan &p, void *const *vel, double fac) {
  Plan q = p;
  q.poisson = 1;
  hipError_t e = !vel ? launch_xdht<T>(q, (const T *)q.W, (T *)q.W, q.shape[3])
                 : q.d == 2 ? launch_div_xdht<T, 2>(q, vel, fac, q.shape[3])
                            : launch_div_xdht<T, 3>(q, vel, fac, q.shape[3]);
  if (e != hipSuccess) return e;
  if ((e = launch_spectral_tail<T>(q)) != hipSuccess) return e;
  return launch_xdht<T>(q, (const T *)q.W, (T *)q.W, q.shape[3]);
}

template <typename T>
hipError_t enqueue_velocity_fill(const Plan &p, const void *Cfin, const NextStep *next) {
  return launch_velocity_fill<T>(p, (const T *)Cfin, next);
}

template <typename T>
hipError_t enqueue_phi(const Plan &p, int cur, void *out) {
  const Dims dm = make_dims(p);
  const T cn2 = (T)(p.Cn * p.Cn), ih2 = (T)(1.0 / (p.h * p.h));
  if (p.d == 2)
    hipLaunchKernelGGL((k_phi<T, 2>), dim3(blocks_for(p.N)), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                       (T *)out, dm, cn2, ih2, p.N);
  else if (stencil_zm_ok(p))
    hipLaunchKernelGGL((k_phi_zm<T>), dim3(stencil_zm_blocks(p)), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                       (T *)out, dm, cn2, ih2, stencil_zm_log(p));
  else
    hipLaunchKernelGGL((k_phi<T, 3>), dim3(blocks_for(p.N)), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                       (T *)out, dm, cn2, ih2, p.N);
  if (p.G && p.d == 2)
    hipLaunchKernelGGL((k_phi_ghost<T, true>), dim3(blocks_for(p.G * 16)), dim3(kThreads), 0, p.stream, (T *)out,
                       p.gidx, p.apg, (const T *)p.wg, p.G, p.K);
  else if (p.G)
    hipLaunchKernelGGL((k_phi_ghost<T, false>), dim3(blocks_for(p.G * 16)), dim3(kThreads), 0, p.stream, (T *)out,
                       p.gidx, p.apg, (const T *)p.wg, p.G, p.K);
  return hipGetLastError();
}

template <typename T>
hipError_t enqueue_diag(const Plan &p, int cur) {
  const Dims dm = make_dims(p);
  if (p.d == 2)
    hipLaunchKernelGGL((k_diag_partial<T, 2>), dim3(p.nred), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                       (const T *)p.alpha, (double *)p.partial, dm, p.Cn, 1.0 / p.h, 0.25 / p.Cn, p.N);
  int nred = p.nred;
  if (p.d == 3) {
    // z-march when whole 64 x 4 column tiles fit and the block count fits the partial buffer
    // (p.nred blocks); thicker z-chunks until it does
    int64_t blocks = -1;
    int zc = 16;
    if (p.n[0] % 64 == 0 && p.n[1] % 4 == 0) {
      const int64_t cols = (int64_t)(p.n[0] / 64) * (p.n[1] / 4);
      for (;; zc *= 2) {
        blocks = cols * ((p.n[2] + zc - 1) / zc);
        if (blocks <= p.nred || zc >= p.n[2]) break;
      }
    }
    if (blocks > 0 && blocks <= p.nred) {
      nred = (int)blocks;
      hipLaunchKernelGGL((k_diag_partial_zm<T>), dim3((unsigned)blocks), dim3(kThreads), 0, p.stream,
                         (const T *)p.C[cur], (const T *)p.alpha, (double *)p.partial, dm, p.Cn, 1.0 / p.h,
                         0.25 / p.Cn, zc);
    } else {
      hipLaunchKernelGGL((k_diag_partial<T, 3>), dim3(p.nred), dim3(kThreads), 0, p.stream, (const T *)p.C[cur],
                         (const T *)p.alpha, (double *)p.partial, dm, p.Cn, 1.0 / p.h, 0.25 / p.Cn, p.N);
    }
  }
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(kThreads), 0, p.stream, (const double *)p.partial, nred,
                     (double *)p.red_out);
  return hipGetLastError();
}

template <typename T>
int max_log_tile(const Plan &p, int pass) {
  constexpr int E = tile_elems<T>();
  if (pass == 0 || pass == 3) return max_log_lines(p, E);
  return max_log_cols(p, p.n[pass == 1 ? 1 : p.d - 1], E);
}

template void default_shapes<double>(Plan &);
template void default_shapes<float>(Plan &);
template void batch_heights<double>(Plan &, int64_t);
template void batch_heights<float>(Plan &, int64_t);
template int max_log_tile<double>(const Plan &, int);
template int max_log_tile<float>(const Plan &, int);
template hipError_t tune_shapes<double>(Plan &, int, int);
template hipError_t tune_shapes<float>(Plan &, int, int);
template hipError_t enqueue_step<double>(const Plan &, int, KernelTimer *, StepLink *);
template hipError_t enqueue_step<float>(const Plan &, int, KernelTimer *, StepLink *);
template hipError_t enqueue_initial_fill<double>(const Plan &, int);
template hipError_t enqueue_initial_fill<float>(const Plan &, int);
template hipError_t enqueue_ghost_refresh<double>(const Plan &, int);
template hipError_t enqueue_ghost_refresh<float>(const Plan &, int);
template hipError_t enqueue_rhs<double>(const Plan &, int, void *);
template hipError_t enqueue_rhs<float>(const Plan &, int, void *);
template hipError_t enqueue_solve<double>(const Plan &, const void *, void *);
template hipError_t enqueue_solve<float>(const Plan &, const void *, void *);
template hipError_t enqueue_poisson<double>(const Plan &, void *const *, double);
template hipError_t enqueue_poisson<float>(const Plan &, void *const *, double);
template hipError_t enqueue_velocity_fill<double>(const Plan &, const void *, const NextStep *);
template hipError_t enqueue_velocity_fill<float>(const Plan &, const void *, const NextStep *);
template <typename T>
hipError_t enqueue_explicit_step(const Plan &p, int cur, int first, KernelTimer *tm, StepLink *link) {
  if (!p.R) return hipErrorInvalidValue;
  const T *Cn = (const T *)p.C[cur];
  T *Cnext = (T *)p.C[1 - cur];
  hipError_t e = hipSuccess;
  auto mark = [&](const char *name) {
    if (tm && e == hipSuccess) e = tm->mark(name, p.stream);
  };
  const Dims dm = make_dims(p);
  const T hih = (T)(0.5 / p.h), ih2 = (T)(1.0 / (p.h * p.h)), ipe = (T)(1.0 / p.Pe), dt = (T)p.dt;
  const T cn2 = (T)(p.Cn * p.Cn);
  const bool mirror = p.G == 0 || (has_patch(p) && dphi_points(p) && p.gwords);
  if (explicit_fused(p.d, p.n, p.N) && mirror) {
    if (p.G) {
      mark("ghost_dphi");
      if (e == hipSuccess) e = launch_ghost_patch<T>(p, Cn, Cn, false, link && link->dphi_done, true);
    }
    mark("explicit_update");
    if (e == hipSuccess) {
      const int zc = explicit_zm_planes(p);
      // (in runs up to half that size in FP64: in launch order and in runs 50.1 and 42.2 us at 32 MiB a field, 99.5 and
      // 104.9 (256x256x128) or 107.5 and 103.1 (128x256x256) at 64, 200 and 208 at 128; FP32 64.1 and 44.2 at 32, 111.2
      // and 108.7 (256^3) or 108.1 and 112.2 (512x256x128) at 64, 212 and 219 at 128)
      const unsigned nb = (unsigned)((p.n[0] / kXx) * (p.n[1] / kXy) * (p.n[2] / zc));
#define CHIB_EXPLICIT_ZM(GH)                                                                                          \
  hipLaunchKernelGGL((k_explicit_zm<T, GH>), dim3(nb), dim3(kXThreads), 0, p.stream, Cn, (const T *)p.F[0],          \
                     (const T *)p.F[1], (const T *)p.F[2], (T *)p.R, Cnext, dm, cn2, hih, ih2, ipe, dt, first, zc,   \
                     tiles_in_runs<T>(p) && (sizeof(T) == 4 || p.N < (int64_t(1) << 23)), p.gwords,                  \
                     (const T *)p.dg)
      if (p.G) CHIB_EXPLICIT_ZM(true);
      else CHIB_EXPLICIT_ZM(false);
#undef CHIB_EXPLICIT_ZM
      e = hipGetLastError();
    }
    const NextStep nx{Cnext, Cnext};
    const bool join = link && link->next && p.vel_fill && p.NF && p.G;
    if (e == hipSuccess) e = launch_step_fills<T>(p, Cnext, tm, join ? &nx : nullptr);
    if (link) link->dphi_done = join && e == hipSuccess;
    if (tm && e == hipSuccess) e = tm->end(p.stream);
    return e;
  }
  mark("phi");
  if (e == hipSuccess) e = enqueue_phi<T>(p, cur, p.W);
  mark("explicit_update");
  if (e == hipSuccess) {
    const T *F2 = (const T *)(p.d == 3 ? p.F[2] : p.F[1]);
    if (p.d == 2)
      hipLaunchKernelGGL((k_explicit<T, 2>), dim3(blocks_for(p.N)), dim3(kThreads), 0, p.stream, Cn,
                         (const T *)p.W, (const T *)p.F[0], (const T *)p.F[1], F2, (T *)p.R, Cnext, dm, hih, ih2,
                         ipe, dt, first, p.N);
    else
      hipLaunchKernelGGL((k_explicit<T, 3>), dim3(blocks_for(p.N)), dim3(kThreads), 0, p.stream, Cn,
                         (const T *)p.W, (const T *)p.F[0], (const T *)p.F[1], F2, (T *)p.R, Cnext, dm, hih, ih2,
                         ipe, dt, first, p.N);
    e = hipGetLastError();
  }
  if (link) link->dphi_done = false;
  if (e == hipSuccess) e = launch_step_fills<T>(p, Cnext, tm, nullptr);
  if (tm && e == hipSuccess) e = tm->end(p.stream);
  return e;
}

template <typename T>
hipError_t enqueue_scalar_fill(const Plan &p, void *f, double a, double b, double g, const void *g_ghost) {
  if (!p.G) return hipSuccess;
  hipLaunchKernelGGL((k_scalar_fill<T>), dim3(blocks_for(p.G)), dim3(kThreads), 0, p.stream, (T *)f, p.gidx, p.ap,
                     (const T *)p.w, (const T *)p.dn, (const T *)p.gamma, (const T *)g_ghost, (T)g, (T)a, (T)b, p.G,
                     p.K);
  return hipGetLastError();
}

template hipError_t enqueue_scalar_fill<double>(const Plan &, void *, double, double, double, const void *);
template hipError_t enqueue_scalar_fill<float>(const Plan &, void *, double, double, double, const void *);
template hipError_t enqueue_explicit_step<double>(const Plan &, int, int, KernelTimer *, StepLink *);
template hipError_t enqueue_explicit_step<float>(const Plan &, int, int, KernelTimer *, StepLink *);
template hipError_t enqueue_phi<double>(const Plan &, int, void *);
template hipError_t enqueue_phi<float>(const Plan &, int, void *);
template hipError_t enqueue_diag<double>(const Plan &, int);
template hipError_t enqueue_diag<float>(const Plan &, int);

}  // namespace chib

// =======================================================================================
// Batched sweep: many independent 2D cases advanced together.  Each phase of the step is
// one grouped launch over all cases: block b belongs to the case c with
// off[c] <= b < off[c+1] (per-case tile counts, prefix-summed), whose pointers, sizes,
// coefficients and tile shapes are read from a descriptor in device memory.  No block ever
// waits for another; the order between phases is the stream order (or the graph's edges).
namespace chib {

template <typename T>
struct CaseDesc {
  T *C[2];                 // C[p] = C^n and C[1-p] = C^(n-1) (then C^(n+1)) for launch parity p
  T *F0, *F1, *W;
  Dims dm;
  RhsCoef<T> cf;
  const T *twr0, *twi0, *twr1, *twi1, *lamx, *lamy, *dctc, *dcts;
  T a, alpha_s, inv_norm;
  int logL_rhs, logL_out, logB, lognxb;
  const int *gidx, *ap;
  const T *dn, *gam, *normal, *w;
  T *CGn, *CGnm1, *CMs, *UG;
  int64_t G, NF;
  int K, vel_fill;
  T cb, inv2h, Cn, cos_t, inv_Ca, inv_mu, ls;
  const int *f_cell, *f_axis, *f_gL, *f_gR;
  T *stashL, *stashR;
  unsigned nbg;
  RhsPatch<T> rp;          // dphi/dn = 0 at the ghosts: the rhs patch
  T *dg;                   // [G]: written by kb_dphi
  T cn2, inv_h2, inv_cn2;
};

namespace {

__device__ __forceinline__ int find_case(const int *__restrict__ off, int n, int b) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

template <typename T, int E, int U, int R>
__global__ __launch_bounds__(kThreads) void kb_rhs(const CaseDesc<T> *__restrict__ cs, const int *__restrict__ off,
                                                   int n, int parity) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int blk = xcd_tile(blockIdx.x, gridDim.x), c = find_case(off, n, blk);
  const CaseDesc<T> &d = cs[c];
  rhs_xdht_body<T, 2, E, U, R>(smem_raw, d.C[parity], d.C[1 - parity], d.F0, d.F1, d.F1, d.W, d.dm, d.cf,
                               d.logL_rhs, d.twr0, d.twi0, blk - off[c], d.rp);
}

// dg of every ghost of every case, before the rhs pass.
template <typename T>
__global__ __launch_bounds__(kThreads) void kb_dphi(const CaseDesc<T> *__restrict__ cs, const int *__restrict__ off,
                                                    int n, int parity) {
  const int c = find_case(off, n, blockIdx.x);
  const CaseDesc<T> &d = cs[c];
  ghost_dphi_body<T>(d.C[parity], d.C[1 - parity], d.gidx, d.ap, d.w, d.dg, d.G, d.K, d.dm, 2, d.cn2, d.inv_h2,
                     d.inv_cn2, (int64_t)(blockIdx.x - off[c]));
}

template <typename T, int R>
__global__ __launch_bounds__(kThreads, 3) void kb_rhs_ym(const CaseDesc<T> *__restrict__ cs,
                                                      const int *__restrict__ off, int n, int parity) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int blk = xcd_tile(blockIdx.x, gridDim.x), c = find_case(off, n, blk);
  const CaseDesc<T> &d = cs[c];
  const int t = blk - off[c];
  // the same instantiation as the single-state launch for this width, so results match bit for bit
  if (d.dm.nx <= 256)
    rhs_ym_body<T, 1, R>(smem_raw, d.C[parity], d.C[1 - parity], d.F0, d.F1, d.W, d.dm, d.cf, d.logL_rhs, d.twr0, d.twi0, t, d.rp);
  else if (d.dm.nx <= 512)
    rhs_ym_body<T, 2, R>(smem_raw, d.C[parity], d.C[1 - parity], d.F0, d.F1, d.W, d.dm, d.cf, d.logL_rhs, d.twr0, d.twi0, t, d.rp);
  else
    rhs_ym_body<T, 4, R>(smem_raw, d.C[parity], d.C[1 - parity], d.F0, d.F1, d.W, d.dm, d.cf, d.logL_rhs, d.twr0, d.twi0, t, d.rp);
}

template <typename T, int E, int R>
__global__ __launch_bounds__(kThreads) void kb_neumann(const CaseDesc<T> *__restrict__ cs, const int *__restrict__ off,
                                                       int n) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int blk = xcd_tile(blockIdx.x, gridDim.x), c = find_case(off, n, blk);
  const CaseDesc<T> &d = cs[c];
#define CHIB_BODY(...)                                                                                            \
  neumann_body<__VA_ARGS__>(smem_raw, d.W, d.dm.lny, (int64_t)d.dm.nx, d.logB, d.lognxb, (int64_t)0, d.lamx,      \
                            (const T *)nullptr, d.lamy, d.a, d.alpha_s, d.inv_norm, d.twr1, d.twi1, d.dctc, d.dcts, \
                            blk - off[c], 0)
  // fixed sizes in FP64 (32 cases: 42 -> 35 us).  FP32 keeps the one runtime-size body: next to others it
  // contracts into other fused multiply-adds than alone, and a member steps as it does alone, bit for bit.
  if constexpr (sizeof(T) == 8) {
    if (d.dm.lny == 6 && d.logB == fixed_cols<T>(6)) CHIB_BODY(T, E, R, 6, fixed_cols<T>(6));
    else if (d.dm.lny == 7 && d.logB == fixed_cols<T>(7)) CHIB_BODY(T, E, R, 7, fixed_cols<T>(7));
    else if (d.dm.lny == 8 && d.logB == fixed_cols<T>(8)) CHIB_BODY(T, E, R, 8, fixed_cols<T>(8));
    else if (d.dm.lny == 9 && d.logB == fixed_cols<T>(9)) CHIB_BODY(T, E, R, 9, fixed_cols<T>(9));
    else CHIB_BODY(T, E, R);
  } else {
    CHIB_BODY(T, E, R);
  }
#undef CHIB_BODY
}

template <typename T, int E, int R>
__global__ __launch_bounds__(kThreads) void kb_out(const CaseDesc<T> *__restrict__ cs, const int *__restrict__ off,
                                                   int n, int parity) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int blk = xcd_tile(blockIdx.x, gridDim.x), c = find_case(off, n, blk);
  const CaseDesc<T> &d = cs[c];
  xdht_body<T, E, R>(smem_raw, d.W, d.C[1 - parity], d.dm.lnx, d.logL_out, d.twr0, d.twi0,
                     blk - off[c]);
}

// Static C fill and (with the velocity fill) the ghost velocities of every case in one launch:
// per case, the first blocks fill C, the following ones compute ghost velocities and face stashes.
template <typename T>
__global__ __launch_bounds__(kThreads) void kb_fill(const CaseDesc<T> *__restrict__ cs, const int *__restrict__ off,
                                                    int n, int parity) {
  const int c = find_case(off, n, blockIdx.x);
  const CaseDesc<T> &d = cs[c];
  const int64_t t = (int64_t)(blockIdx.x - off[c]);
  const int64_t nbc = (d.G * 16 + kThreads - 1) / kThreads;
  if (t < nbc) {
    fill_static_body<T>(d.C[1 - parity], d.gidx, d.dn, d.gam, d.ap, d.w, d.CGn, d.CGnm1, d.CMs, d.G, d.K, d.cb, 0, t);
    return;
  }
  vel_ghosts_body<T, 2, false>(d.C[1 - parity], d.F0, d.F1, d.F1, d.gidx, d.normal, d.dn, d.gam, d.ap, d.w, d.CMs,
                               d.UG, d.G, d.K, d.f_cell, d.f_axis, d.f_gL, d.f_gR, d.stashL, d.stashR, d.NF, d.dm,
                               d.inv2h, d.Cn, d.cos_t, d.inv_Ca, d.inv_mu, d.ls, d.nbg, t - nbc);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void kb_velf(const CaseDesc<T> *__restrict__ cs, const int *__restrict__ off,
                                                    int n) {
  const int c = find_case(off, n, blockIdx.x);
  const CaseDesc<T> &d = cs[c];
  vel_faces_body<T>(d.F0, d.F1, d.F1, d.UG, d.G, d.f_cell, d.f_axis, d.f_gL, d.f_gR, d.stashL, d.stashR, d.NF,
                    (int64_t)(blockIdx.x - off[c]));
}

}  // namespace

// Host side: descriptors from the member plans, per-phase tile offsets, one batched step.
template <typename T>
void fill_case_desc(const Plan &p, int cur, void *desc_host) {
  CaseDesc<T> d{};
  d.C[0] = (T *)p.C[cur];
  d.C[1] = (T *)p.C[1 - cur];
  d.F0 = (T *)p.F[0];
  d.F1 = (T *)p.F[1];
  d.W = (T *)p.W;
  d.dm = make_dims(p);
  d.cf = make_coef<T>(p);
  d.twr0 = (const T *)p.twr[0];
  d.twi0 = (const T *)p.twi[0];
  d.twr1 = (const T *)p.twr[1];
  d.twi1 = (const T *)p.twi[1];
  d.lamx = (const T *)p.lam[0];
  d.lamy = (const T *)p.lam[1];
  d.dctc = (const T *)p.dctc;
  d.dcts = (const T *)p.dcts;
  d.a = (T)p.a;
  d.alpha_s = (T)p.alpha_s;
  d.inv_norm = (T)(1.0 / (double)p.N);
  constexpr int E = tile_elems<T>();
  d.logL_rhs = clamp_log(p.shape[0].log_tile, max_log_lines(p, E));
  d.logL_out = clamp_log(p.shape[3].log_tile, max_log_lines(p, E));
  d.logB = clamp_log(p.shape[2].log_tile, max_log_cols(p, p.n[1], E));
  d.lognxb = p.logn[0] - d.logB;
  d.gidx = p.gidx;
  d.ap = p.apg;   // the batch's ghost kernels take the ghost-major tables
  d.dn = (const T *)p.dn;
  d.gam = (const T *)p.gamma;
  d.normal = (const T *)p.normal;
  d.w = (const T *)p.wg;
  d.CGn = (T *)p.CGn;
  d.CGnm1 = (T *)p.CGnm1;
  d.CMs = (T *)p.CMs;
  d.UG = (T *)p.UG;
  d.G = p.G;
  d.NF = p.NF;
  d.K = p.K;
  d.vel_fill = p.vel_fill && p.G > 0;
  d.cb = (T)(p.cos_t / (1.4142135623730951 * p.Cn));
  d.inv2h = (T)(0.5 / p.h);
  d.Cn = (T)p.Cn;
  d.cos_t = (T)p.cos_t;
  d.inv_Ca = (T)(1.0 / p.Ca);
  d.inv_mu = (T)(1.0 / p.mu);
  d.ls = (T)p.ls;
  d.f_cell = p.f_cell;
  d.f_axis = p.f_axis;
  d.f_gL = p.f_gL;
  d.f_gR = p.f_gR;
  d.stashL = (T *)p.stashL;
  d.stashR = (T *)p.stashR;
  d.nbg = blocks_for(p.G * 16);
  d.rp = make_patch<T>(p);
  d.dg = (T *)p.dg;
  d.cn2 = (T)(p.Cn * p.Cn);
  d.inv_h2 = (T)(1.0 / (p.h * p.h));
  d.inv_cn2 = (T)(1.0 / (p.Cn * p.Cn));
  std::memcpy(desc_host, &d, sizeof(d));
}

template <typename T>
size_t case_desc_bytes() {
  return sizeof(CaseDesc<T>);
}

// Per-phase tile counts of one case (0 rhs, 1 neumann, 2 out, 3 fill, 4 dphi, 5 velf) and the
// LDS bytes of its tiles (0 rhs, 1 neumann, 2 out).
template <typename T>
void case_tiles(const Plan &p, int *tiles, size_t *lds) {
  constexpr int E = tile_elems<T>();
  const int lr = clamp_log(p.shape[0].log_tile, max_log_lines(p, E));
  const int lo = clamp_log(p.shape[3].log_tile, max_log_lines(p, E));
  const int lb = clamp_log(p.shape[2].log_tile, max_log_cols(p, p.n[1], E));
  tiles[0] = p.n[1] >> lr;
  tiles[1] = p.n[0] >> lb;
  tiles[2] = p.n[1] >> lo;
  const bool vf = p.vel_fill && p.G > 0;
  tiles[3] = (int)blocks_for(p.G * 16) + (vf ? (int)(blocks_for(p.G * 16) + blocks_for(p.NF)) : 0);
  const bool pt = make_patch<T>(p).row != nullptr;
  tiles[4] = pt ? (int)blocks_for(p.G * 16) : 0;   // (the ghost velocities run inside phase 3)
  tiles[5] = vf ? (int)blocks_for(p.NF) : 0;
  lds[0] = (size_t)(1 << lr) * line_pitch(p.n[0]) * sizeof(T);
  lds[1] = (size_t)col_tile(p.n[1], 1 << lb) * sizeof(T);
  lds[2] = (size_t)(1 << lo) * line_pitch(p.n[0]) * sizeof(T);
  lds[3] = ym_ok(p) ? lds[0] + (size_t)ym_extra(p.n[0]) * sizeof(T) : 0;   // 0: no y-march
}

template <typename T>
hipError_t enqueue_batch_step(const BatchLaunch &bl, int parity) {
  constexpr int E = tile_elems<T>();
  const CaseDesc<T> *cs = (const CaseDesc<T> *)bl.descs;
  const int n = bl.n;
  const int *off = bl.off;
  auto O = [&](int ph) { return off + ph * (n + 1); };
  const unsigned nb0 = bl.total[0], nb1 = bl.total[1], nb2 = bl.total[2];
  const unsigned nb3 = bl.total[3], nb4 = bl.total[4], nb5 = bl.total[5];
  const bool r8 = bl.radix_rhs <= 8, u2 = bl.unroll >= 2;
  if (nb4) hipLaunchKernelGGL((kb_dphi<T>), dim3(nb4), dim3(kThreads), 0, bl.stream, cs, O(4), n, parity);
  if (bl.unroll == 3 && bl.lds[3]) {
    if (r8) hipLaunchKernelGGL((kb_rhs_ym<T, 8>), dim3(nb0), dim3(kThreads), bl.lds[3], bl.stream, cs, O(0), n, parity);
    else hipLaunchKernelGGL((kb_rhs_ym<T, 16>), dim3(nb0), dim3(kThreads), bl.lds[3], bl.stream, cs, O(0), n, parity);
  } else if (r8 && u2) hipLaunchKernelGGL((kb_rhs<T, E, 2, 8>), dim3(nb0), dim3(kThreads), bl.lds[0], bl.stream, cs, O(0), n, parity);
  else if (r8) hipLaunchKernelGGL((kb_rhs<T, E, 1, 8>), dim3(nb0), dim3(kThreads), bl.lds[0], bl.stream, cs, O(0), n, parity);
  else if (u2) hipLaunchKernelGGL((kb_rhs<T, E, 2, 16>), dim3(nb0), dim3(kThreads), bl.lds[0], bl.stream, cs, O(0), n, parity);
  else hipLaunchKernelGGL((kb_rhs<T, E, 1, 16>), dim3(nb0), dim3(kThreads), bl.lds[0], bl.stream, cs, O(0), n, parity);
  if (bl.radix_neu == 8) hipLaunchKernelGGL((kb_neumann<T, E, 8>), dim3(nb1), dim3(kThreads), bl.lds[1], bl.stream, cs, O(1), n);
  else hipLaunchKernelGGL((kb_neumann<T, E, 16>), dim3(nb1), dim3(kThreads), bl.lds[1], bl.stream, cs, O(1), n);
  if (bl.radix_out == 8) hipLaunchKernelGGL((kb_out<T, E, 8>), dim3(nb2), dim3(kThreads), bl.lds[2], bl.stream, cs, O(2), n, parity);
  else hipLaunchKernelGGL((kb_out<T, E, 16>), dim3(nb2), dim3(kThreads), bl.lds[2], bl.stream, cs, O(2), n, parity);
  if (nb3) hipLaunchKernelGGL((kb_fill<T>), dim3(nb3), dim3(kThreads), 0, bl.stream, cs, O(3), n, parity);
  if (nb5) hipLaunchKernelGGL((kb_velf<T>), dim3(nb5), dim3(kThreads), 0, bl.stream, cs, O(5), n);
  return hipGetLastError();
}

template void fill_case_desc<double>(const Plan &, int, void *);
template void fill_case_desc<float>(const Plan &, int, void *);
template size_t case_desc_bytes<double>();
template size_t case_desc_bytes<float>();
template void case_tiles<double>(const Plan &, int *, size_t *);
template void case_tiles<float>(const Plan &, int *, size_t *);
template hipError_t enqueue_batch_step<double>(const BatchLaunch &, int);
template hipError_t enqueue_batch_step<float>(const BatchLaunch &, int);

}  // namespace chib
