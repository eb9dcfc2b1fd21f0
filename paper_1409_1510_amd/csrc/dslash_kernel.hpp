// Multi-rhs HISQ half Dslash kernel template for gfx950 (Section 1, Eq. 3 and Eq. 4).
//
// One thread owns one output site and a tile of RT right-hand sides (register blocking over rhs,
// Section 2): each link of the site is loaded once per tile and applied to RT neighbour vectors.
// Several tiles of the same sites are kept close together, either as the 4 waves of one
// workgroup (SPB = 64 sites per workgroup: the waves read the same links through the CU's L1 --
// the 2-d site x rhs blocking of Section 2) or as neighbouring workgroups on one XCD (SPB = 256:
// the links are found in that XCD's L2).  Workgroups are remapped so that each XCD owns a
// contiguous range of site blocks.  Hops are accumulated in a fixed order with explicit FMAs, so
// the result for a rhs does not depend on n, on RT or on the workgroup shape.  Which shape is
// fastest depends on the GPU, the lattice and n; the launcher picks it by timing (Section 2,
// automatic tuning of the launch configuration).
//
// Layouts: links as packed by links.hip (planes of V/2 complex per matrix entry, per output
// parity); vectors [n][3][V/2] complex (colour-planar structure of arrays).
#pragma once

#include "internal.hpp"

#include <type_traits>

namespace dslash {

template <typename Real> struct CT;
template <> struct CT<double> { using T = double2; };
template <> struct CT<float> { using T = float2; };

typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));

template <bool NT> __device__ inline void ld_link(const double2 *p, double &re, double &im) {
  if constexpr (NT) {
    d2v v = __builtin_nontemporal_load(reinterpret_cast<const d2v *>(p));
    re = v.x;
    im = v.y;
  } else {
    double2 v = *p;
    re = v.x;
    im = v.y;
  }
}
template <bool NT> __device__ inline void ld_link(const float2 *p, float &re, float &im) {
  if constexpr (NT) {
    f2v v = __builtin_nontemporal_load(reinterpret_cast<const f2v *>(p));
    re = v.x;
    im = v.y;
  } else {
    float2 v = *p;
    re = v.x;
    im = v.y;
  }
}
template <bool NT> __device__ inline void ld_link(const __half2 *p, float &re, float &im) {
  __half2 h;
  if constexpr (NT) {
    unsigned u = __builtin_nontemporal_load(reinterpret_cast<const unsigned *>(p));
    h = *reinterpret_cast<__half2 *>(&u);
  } else {
    h = *p;
  }
  float2 v = __half22float2(h);
  re = v.x;
  im = v.y;
}

__device__ inline double fmaR(double a, double b, double c) { return fma(a, b, c); }
__device__ inline float fmaR(float a, float b, float c) { return fmaf(a, b, c); }

template <typename Real> struct Lnk {
  Real re[3][3], im[3][3];
};

// Row 2 of a 14-real Naik link from rows 0 and 1 and the stored scale z: z * conj(row0 x row1).
template <typename Real>
__device__ inline void naik_row2(Lnk<Real> &L, Real zr, Real zi) {
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int b1 = (b + 1) % 3, b2 = (b + 2) % 3;
    // cross_b = r0[b1] r1[b2] - r0[b2] r1[b1]
    Real cr = (L.re[0][b1] * L.re[1][b2] - L.im[0][b1] * L.im[1][b2]) -
              (L.re[0][b2] * L.re[1][b1] - L.im[0][b2] * L.im[1][b1]);
    Real ci = (L.re[0][b1] * L.im[1][b2] + L.im[0][b1] * L.re[1][b2]) -
              (L.re[0][b2] * L.im[1][b1] + L.im[0][b2] * L.re[1][b1]);
    // row2_b = z * conj(cross_b)
    L.re[2][b] = zr * cr + zi * ci;
    L.im[2][b] = zi * cr - zr * ci;
  }
}

// Load the link of a hop at site s; a 14-real Naik link gets row 2 = z * conj(row0 x row1).
template <typename Real, typename LT, bool R14, bool NT>
__device__ inline void load_link(const LT *__restrict__ links, int plane, unsigned vh, unsigned s,
                                 Lnk<Real> &L) {
  const LT *p = links + size_t(plane) * vh + s;
  constexpr int rows = R14 ? 2 : 3;
#pragma unroll
  for (int a = 0; a < rows; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) ld_link<NT>(p + (a * 3 + b) * vh, L.re[a][b], L.im[a][b]);
  if constexpr (R14) {
    Real zr, zi;
    ld_link<NT>(p + 6 * vh, zr, zi);
    naik_row2(L, zr, zi);
  }
}

// Row 2 of a 13-real Naik link from rows 0 and 1 and the real scale z: z * conj(row0 x row1).
template <typename Real>
__device__ inline void naik_row2_real(Lnk<Real> &L, Real z) {
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int b1 = (b + 1) % 3, b2 = (b + 2) % 3;
    Real cr = (L.re[0][b1] * L.re[1][b2] - L.im[0][b1] * L.im[1][b2]) -
              (L.re[0][b2] * L.re[1][b1] - L.im[0][b2] * L.im[1][b1]);
    Real ci = (L.re[0][b1] * L.im[1][b2] + L.im[0][b1] * L.re[1][b2]) -
              (L.re[0][b2] * L.im[1][b1] + L.im[0][b2] * L.re[1][b1]);
    L.re[2][b] = z * cr;
    L.im[2][b] = -(z * ci);
  }
}

__device__ inline void sincos_r(float x, float &s, float &c) { sincosf(x, &s, &c); }
__device__ inline void sincos_r(double x, double &s, double &c) { sincos(x, &s, &c); }

// A 9-real Naik link N = c U with U in SU(3), from u01, u02, u10, the phases th0 = arg u00 and
// th2 = arg u20, and c: |u00| and |u20| follow from the unit norms of row 0 and column 0, and the
// four remaining entries from the orthogonality of rows 1 and 2 to row 0 and from
// row2 = conj(row0 x row1), row1 = conj(row2 x row0) (det U = 1); with n = 1 - |u00|^2:
//   u11 = -(conj(u20 u02) + conj(u00) u01 u10) / n    u12 = (conj(u01 u20) - conj(u00) u02 u10) / n
//   u21 = (conj(u10 u02) - conj(u00) u01 u20) / n     u22 = -(conj(u01 u10) + conj(u00) u02 u20) / n
template <typename Real>
__device__ inline void naik_from9(Lnk<Real> &L, Real u01r, Real u01i, Real u02r, Real u02i, Real u10r,
                                  Real u10i, Real th0, Real th2, Real c) {
  const Real nn = (u01r * u01r + u01i * u01i) + (u02r * u02r + u02i * u02i);
  const Real a2 = Real(1) - nn;
  const Real a0 = sqrt(a2 > Real(0) ? a2 : Real(0));
  const Real b2 = nn - (u10r * u10r + u10i * u10i);
  const Real b0 = sqrt(b2 > Real(0) ? b2 : Real(0));
  Real s0, c0, s2, c2;
  sincos_r(th0, s0, c0);
  sincos_r(th2, s2, c2);
  const Real u00r = a0 * c0, u00i = a0 * s0;
  const Real u20r = b0 * c2, u20i = b0 * s2;
  const Real inv = Real(1) / nn;
  const Real pr = u20r * u02r - u20i * u02i, pi = u20r * u02i + u20i * u02r;  // u20 u02
  const Real qr = u01r * u10r - u01i * u10i, qi = u01r * u10i + u01i * u10r;  // u01 u10
  const Real tr = u01r * u20r - u01i * u20i, ti = u01r * u20i + u01i * u20r;  // u01 u20
  const Real vr = u02r * u10r - u02i * u10i, vi = u02r * u10i + u02i * u10r;  // u02 u10
  const Real u11r = -(pr + (u00r * qr + u00i * qi)) * inv, u11i = -(-pi + (u00r * qi - u00i * qr)) * inv;
  const Real u12r = (tr - (u00r * vr + u00i * vi)) * inv, u12i = (-ti - (u00r * vi - u00i * vr)) * inv;
  const Real u21r = (vr - (u00r * tr + u00i * ti)) * inv, u21i = (-vi - (u00r * ti - u00i * tr)) * inv;
  const Real u22r = -(qr + (u00r * pr + u00i * pi)) * inv, u22i = -(-qi + (u00r * pi - u00i * pr)) * inv;
  L.re[0][0] = c * u00r; L.im[0][0] = c * u00i;
  L.re[0][1] = c * u01r; L.im[0][1] = c * u01i;
  L.re[0][2] = c * u02r; L.im[0][2] = c * u02i;
  L.re[1][0] = c * u10r; L.im[1][0] = c * u10i;
  L.re[1][1] = c * u11r; L.im[1][1] = c * u11i;
  L.re[1][2] = c * u12r; L.im[1][2] = c * u12i;
  L.re[2][0] = c * u20r; L.im[2][0] = c * u20i;
  L.re[2][1] = c * u21r; L.im[2][1] = c * u21i;
  L.re[2][2] = c * u22r; L.im[2][2] = c * u22i;
}

// Load Naik hop k (8..15) at site s of a link array with plane stride vh, rebuilding what the
// storage format NR (18, 14, 13 or 9, see link_plane) leaves out.
template <typename Real, typename LT, int NR, bool NT>
__device__ inline void load_naik(const LT *__restrict__ links, int k, unsigned vh, unsigned s, Lnk<Real> &L) {
  if constexpr (NR == 18 || NR == 14) {
    load_link<Real, LT, NR == 14, NT>(links, link_plane(k, NR), vh, s, L);
  } else if constexpr (NR == 13) {
    const LT *p = links + size_t(link_plane(k, NR)) * vh + s;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) ld_link<NT>(p + (a * 3 + b) * vh, L.re[a][b], L.im[a][b]);
    Real zr, zi;
    ld_link<NT>(links + size_t(naik_scale_plane(k, NR)) * vh + s, zr, zi);
    naik_row2_real(L, (k & 1) ? zi : zr);
  } else {
    static_assert(NR == 9, "Naik storage formats: 18, 14, 13, 9");
    const LT *p = links + size_t(link_plane(k, NR)) * vh + s;
    Real a1r, a1i, a2r, a2i, b0r, b0i, t0, t2, cr, ci;
    ld_link<NT>(p, a1r, a1i);
    ld_link<NT>(p + vh, a2r, a2i);
    ld_link<NT>(p + 2 * vh, b0r, b0i);
    ld_link<NT>(p + 3 * vh, t0, t2);
    ld_link<NT>(links + size_t(naik_scale_plane(k, NR)) * vh + s, cr, ci);
    naik_from9(L, a1r, a1i, a2r, a2i, b0r, b0i, t0, t2, (k & 1) ? ci : cr);
  }
}

// acc += sign * L v for the RT right-hand sides of the tile (sign -1 for backward hops).
template <typename Real, int RT, bool NEG>
__device__ inline void apply_hop(const Lnk<Real> &L, const typename CT<Real>::T *__restrict__ in,
                                 unsigned vh, unsigned nbr, const bool *act,
                                 Real (&acc_re)[RT][3], Real (&acc_im)[RT][3]) {
  using C = typename CT<Real>::T;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    if (!act[r]) continue;
    C v[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) v[b] = in[(unsigned)(r * 3 + b) * vh + nbr];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Real lr = NEG ? -L.re[a][b] : L.re[a][b];
        const Real li = NEG ? -L.im[a][b] : L.im[a][b];
        acc_re[r][a] = fmaR(lr, v[b].x, acc_re[r][a]);
        acc_re[r][a] = fmaR(-li, v[b].y, acc_re[r][a]);
        acc_im[r][a] = fmaR(lr, v[b].y, acc_im[r][a]);
        acc_im[r][a] = fmaR(li, v[b].x, acc_im[r][a]);
      }
    }
  }
}

// LDS forms: the same FMA sequence as apply_hop, but every lane computes every rhs of the tile
// (inactive lanes and rhs read clamped, in-range addresses; only active results are stored), so
// the hops are straight-line code the compiler can schedule across.  rr[r]: the rhs of the tile
// to read for r.  Per-lane offsets are 32-bit: a tile spans less than 4 GB (checked at launch).
template <typename Real, int RT, bool NEG>
__device__ inline void apply_hop_all(const Lnk<Real> &L, const typename CT<Real>::T *__restrict__ in,
                                     unsigned vh, unsigned nbr, const int (&rr)[RT],
                                     Real (&acc_re)[RT][3], Real (&acc_im)[RT][3]) {
  using C = typename CT<Real>::T;
  const char *base = reinterpret_cast<const char *>(in);
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    C v[3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
      v[b] = *reinterpret_cast<const C *>(base + (unsigned(rr[r] * 3 + b) * vh + nbr) * unsigned(sizeof(C)));
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Real lr = NEG ? -L.re[a][b] : L.re[a][b];
        const Real li = NEG ? -L.im[a][b] : L.im[a][b];
        acc_re[r][a] = fmaR(lr, v[b].x, acc_re[r][a]);
        acc_re[r][a] = fmaR(-li, v[b].y, acc_re[r][a]);
        acc_im[r][a] = fmaR(lr, v[b].y, acc_im[r][a]);
        acc_im[r][a] = fmaR(li, v[b].x, acc_im[r][a]);
      }
    }
  }
}

// apply_hop_all with the gathers as raw buffer loads: the tile's colour planes are one buffer
// (wave-uniform descriptor), the neighbour is a byte offset within a plane (the lane's only
// address operand) and the plane start a scalar offset, so a gather costs no vector address
// arithmetic.
typedef unsigned v2u_t __attribute__((__vector_size__(8)));
typedef unsigned v4u_t __attribute__((__vector_size__(16)));
__device__ inline void buf_load(__amdgpu_buffer_rsrc_t rs, unsigned off, unsigned soff, float2 &v) {
  const v2u_t u = __builtin_amdgcn_raw_buffer_load_b64(rs, off, soff, 0);
  v.x = __uint_as_float(u[0]);
  v.y = __uint_as_float(u[1]);
}
__device__ inline void buf_load(__amdgpu_buffer_rsrc_t rs, unsigned off, unsigned soff, double2 &v) {
  const v4u_t u = __builtin_amdgcn_raw_buffer_load_b128(rs, off, soff, 0);
  v.x = __hiloint2double(int(u[1]), int(u[0]));
  v.y = __hiloint2double(int(u[3]), int(u[2]));
}
template <typename Real, int RT, bool NEG>
__device__ inline void apply_hop_buf(const Lnk<Real> &L, __amdgpu_buffer_rsrc_t rs, unsigned plane_bytes,
                                     unsigned off, const int (&rr)[RT], Real (&acc_re)[RT][3],
                                     Real (&acc_im)[RT][3]) {
  using C = typename CT<Real>::T;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    C v[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) buf_load(rs, off, unsigned(rr[r] * 3 + b) * plane_bytes, v[b]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Real lr = NEG ? -L.re[a][b] : L.re[a][b];
        const Real li = NEG ? -L.im[a][b] : L.im[a][b];
        acc_re[r][a] = fmaR(lr, v[b].x, acc_re[r][a]);
        acc_re[r][a] = fmaR(-li, v[b].y, acc_re[r][a]);
        acc_im[r][a] = fmaR(lr, v[b].y, acc_im[r][a]);
        acc_im[r][a] = fmaR(li, v[b].x, acc_im[r][a]);
      }
    }
  }
}

// apply_hop_buf for the 32-site form: rhs r of a lane sits in the vector offset (off + r * 3
// planes) and the colour plane in the scalar offset, so that the buffer range check covers the
// rhs (a rhs past n reads 0 instead of memory past the vectors).
template <typename Real, int RT, bool NEG>
__device__ inline void apply_hop_buf32(const Lnk<Real> &L, __amdgpu_buffer_rsrc_t rs, unsigned plane_bytes,
                                       unsigned off, Real (&acc_re)[RT][3], Real (&acc_im)[RT][3]) {
  using C = typename CT<Real>::T;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    C v[3];
    const unsigned vo = off + unsigned(r * 3) * plane_bytes;
#pragma unroll
    for (int b = 0; b < 3; ++b) buf_load(rs, vo, unsigned(b) * plane_bytes, v[b]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Real lr = NEG ? -L.re[a][b] : L.re[a][b];
        const Real li = NEG ? -L.im[a][b] : L.im[a][b];
        acc_re[r][a] = fmaR(lr, v[b].x, acc_re[r][a]);
        acc_re[r][a] = fmaR(-li, v[b].y, acc_re[r][a]);
        acc_im[r][a] = fmaR(lr, v[b].y, acc_im[r][a]);
        acc_im[r][a] = fmaR(li, v[b].x, acc_im[r][a]);
      }
    }
  }
}

// Neighbour indices (within the input parity) of output site s at coordinates (x, y, z, t) for
// the four hops of direction mu: +1, -1, +3, -3.
__device__ inline void hop_sites(const Geometry &g, int mu, unsigned s, unsigned rowbase, int x, int y, int z, int t,
                                 unsigned &f1, unsigned &b1, unsigned &f3, unsigned &b3) {
  if (mu == 0) {
    const int xf1 = x + 1 >= g.lx ? x + 1 - g.lx : x + 1;
    const int xb1 = x - 1 < 0 ? x - 1 + g.lx : x - 1;
    const int xf3 = x + 3 >= g.lx ? x + 3 - g.lx : x + 3;
    const int xb3 = x - 3 < 0 ? x - 3 + g.lx : x - 3;
    f1 = rowbase + (xf1 >> 1);
    b1 = rowbase + (xb1 >> 1);
    f3 = rowbase + (xf3 >> 1);
    b3 = rowbase + (xb3 >> 1);
  } else {
    const int c = mu == 1 ? y : (mu == 2 ? z : t);
    const int L = mu == 1 ? g.ly : (mu == 2 ? g.lz : g.lt);
    const int S = mu == 1 ? g.sy : (mu == 2 ? g.sz : g.st);
    f1 = s + (c + 1 >= L ? 1 - L : 1) * S;
    b1 = s + (c - 1 < 0 ? L - 1 : -1) * S;
    f3 = s + (c + 3 >= L ? 3 - L : 3) * S;
    b3 = s + (c - 3 < 0 ? L - 3 : -3) * S;
  }
}

// Unsigned division by a run-time constant d with a multiply-high, two shifts and two adds
// (Granlund and Montgomery, "Division by invariant integers using multiplication", 1994, the
// unsigned round-up method): l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1, and
// q = (t + ((n - t) >> min(l, 1))) >> max(l - 1, 0) with t = mulhi(m, n), exact for every
// 32-bit n.  The lattice extents are divisors of this kind; the multipliers are set on the host.
struct FastDiv {
  unsigned m;
  int s1, s2;
};
inline FastDiv make_fastdiv(unsigned d) {
  int l = 0;
  while ((1ull << l) < d) ++l;
  const unsigned long long m = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
  return FastDiv{unsigned(m), l < 1 ? l : 1, l > 1 ? l - 1 : 0};
}
__device__ inline unsigned fast_div(unsigned n, const FastDiv &f) {
  const unsigned t = __umulhi(f.m, n);
  return (t + ((n - t) >> f.s1)) >> f.s2;
}

// Neighbour index (within the input parity) of output site s at (x, y, z, t) for the hop of
// direction mu by d = +1, -1, +3 or -3 (one periodic wrap: every extent is at least 4); the same
// values as hop_sites.
__device__ inline unsigned hop_site(const Geometry &g, int mu, int d, unsigned s, unsigned rowbase, int x, int y,
                                    int z, int t) {
  if (mu == 0) {
    const int xn = x + d;
    return rowbase + ((xn < 0 ? xn + g.lx : (xn >= g.lx ? xn - g.lx : xn)) >> 1);
  }
  const int c = mu == 1 ? y : (mu == 2 ? z : t);
  const int L = mu == 1 ? g.ly : (mu == 2 ? g.lz : g.lt);
  const int S = mu == 1 ? g.sy : (mu == 2 ? g.sz : g.st);
  const int cn = c + d;
  return s + (cn < 0 ? d + L : (cn >= L ? d - L : d)) * S;
}

// Rhs of tile r0 a wave computes: rr[r] (clamped to the last rhs), ract[r] (rhs active);
// returns whether any rhs of the tile is active.  All values are uniform across the wave.
struct Args {
  const void *links;
  const void *in;
  void *out;
  Geometry g;
  int out_parity;
  int n;
  int ntiles;   // ceil(n / RT)
  int ngroups;  // tile groups per site block
  int nsblk;    // site blocks
  double mass2;
  const void *pvec;       // epilogue: q = mass2 * pvec - D in
  double *partial;        // epilogue: Re<pvec, q> per rhs per 64-site wave, [n][ceil(V/2 / 64)]
  const int *active;      // per-rhs mask or null
  int xmap;               // LDS form, XCD map: 0 contiguous ranges, 1 z slabs, 2 y slabs
  int zmap_bps;           //   64-site blocks per (z, t) plane
  int zmap_zr;            //   z-slab map: z slices owned by each XCD (Lz / 8)
  FastDiv div_xh, div_y, div_z;  // division by Lx/2, Ly, Lz (site decoding of the LDS form)
};

template <int RT>
__device__ inline bool tile_rhs(const Args &a, int r0, int (&rr)[RT], bool (&ract)[RT]) {
  bool any = false;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int q = r0 + r;
    ract[r] = q < a.n && (!a.active || a.active[q]);
    rr[r] = q < a.n ? r : a.n - 1 - r0;
    any = any || ract[r];
  }
  return any;
}


// SPB: sites per 256-thread workgroup (256: one tile per workgroup; 64: 4 tiles, one per wave).
template <typename Real, typename LT, int RT, int NR, bool EPI, int SPB, bool NT>
__global__ void __launch_bounds__(256) k_dslash(Args a) {
  using C = typename CT<Real>::T;
  constexpr int TPB = 256 / SPB;  // tiles per workgroup
  const Geometry &g = a.g;
  // XCD-aware order: the hardware deals workgroups round-robin to the 8 XCDs; each XCD gets a
  // contiguous range of logical blocks (all rhs tiles of consecutive site blocks).
  const int nb = a.nsblk * a.ngroups;
  const int chunk = gridDim.x >> 3;
  const int lb = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if (lb >= nb) return;  // uniform for the whole workgroup
  const int sblk = lb / a.ngroups;
  const int grp = lb - sblk * a.ngroups;
  const int tile = grp * TPB + (TPB == 1 ? 0 : int(threadIdx.x) / SPB);
  const int r0 = tile * RT;
  const unsigned vh = g.vh;
  const unsigned s = sblk * SPB + (threadIdx.x % SPB);
  const bool valid = s < vh && tile < a.ntiles;
  const size_t tile_off = size_t(r0) * 3 * vh;
  const C *__restrict__ in = static_cast<const C *>(a.in) + tile_off;
  C *__restrict__ out = static_cast<C *>(a.out) + tile_off;
  const LT *__restrict__ links = static_cast<const LT *>(a.links);

  bool act[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) act[r] = valid && (r0 + r < a.n) && (!a.active || a.active[r0 + r]);

  Real acc_re[RT][3], acc_im[RT][3];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc_re[r][c] = acc_im[r][c] = Real(0);

  if (valid) {
    const int xh = s % g.lxh;
    int rest = s / g.lxh;
    const int y = rest % g.ly;
    rest /= g.ly;
    const int z = rest % g.lz;
    const int t = rest / g.lz;
    const int x = 2 * xh + ((y + z + t + a.out_parity) & 1);
    const unsigned rowbase = s - xh;
    constexpr int recon = NR;
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      unsigned f1, b1, f3, b3;
      if (mu == 0) {
        const int xf1 = x + 1 >= g.lx ? x + 1 - g.lx : x + 1;
        const int xb1 = x - 1 < 0 ? x - 1 + g.lx : x - 1;
        const int xf3 = x + 3 >= g.lx ? x + 3 - g.lx : x + 3;
        const int xb3 = x - 3 < 0 ? x - 3 + g.lx : x - 3;
        f1 = rowbase + (xf1 >> 1);
        b1 = rowbase + (xb1 >> 1);
        f3 = rowbase + (xf3 >> 1);
        b3 = rowbase + (xb3 >> 1);
      } else {
        const int c = mu == 1 ? y : (mu == 2 ? z : t);
        const int L = mu == 1 ? g.ly : (mu == 2 ? g.lz : g.lt);
        const int S = mu == 1 ? g.sy : (mu == 2 ? g.sz : g.st);
        f1 = s + (c + 1 >= L ? 1 - L : 1) * S;
        b1 = s + (c - 1 < 0 ? L - 1 : -1) * S;
        f3 = s + (c + 3 >= L ? 3 - L : 3) * S;
        b3 = s + (c - 3 < 0 ? L - 3 : -3) * S;
      }
      Lnk<Real> Lk;
      load_link<Real, LT, false, NT>(links, link_plane(mu, recon), vh, s, Lk);
      apply_hop<Real, RT, false>(Lk, in, vh, f1, act, acc_re, acc_im);
      load_link<Real, LT, false, NT>(links, link_plane(4 + mu, recon), vh, s, Lk);
      apply_hop<Real, RT, true>(Lk, in, vh, b1, act, acc_re, acc_im);
      load_naik<Real, LT, NR, NT>(links, 8 + mu, vh, s, Lk);
      apply_hop<Real, RT, false>(Lk, in, vh, f3, act, acc_re, acc_im);
      load_naik<Real, LT, NR, NT>(links, 12 + mu, vh, s, Lk);
      apply_hop<Real, RT, true>(Lk, in, vh, b3, act, acc_re, acc_im);
    }
  }

  if constexpr (!EPI) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      if (!act[r]) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        C o;
        o.x = acc_re[r][c];
        o.y = acc_im[r][c];
        out[(unsigned)(r * 3 + c) * vh + s] = o;
      }
    }
  } else {
    // q = m^2 p - D_eo t, and per-rhs FP64 partials of Re<p, q> per 64-site wave (the same
    // grouping for every workgroup shape, so the reduction is independent of the launch shape)
    const C *__restrict__ pv = static_cast<const C *>(a.pvec) + tile_off;
    const Real m2 = Real(a.mass2);
    double dot[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      dot[r] = 0.0;
      if (!act[r]) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const C p = pv[(unsigned)(r * 3 + c) * vh + s];
        C o;
        o.x = fmaR(m2, p.x, -acc_re[r][c]);
        o.y = fmaR(m2, p.y, -acc_im[r][c]);
        out[(unsigned)(r * 3 + c) * vh + s] = o;
        dot[r] = fma(double(p.x), double(o.x), dot[r]);
        dot[r] = fma(double(p.y), double(o.y), dot[r]);
      }
    }
    if (a.partial && tile < a.ntiles) {
      const int lane = threadIdx.x & 63;
      const unsigned wave_sites = s - lane;  // first site of this wave (SPB is a multiple of 64)
      const unsigned nw = (vh + 63) / 64;
      if (wave_sites < vh) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          double v = dot[r];
#pragma unroll
          for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
          if (lane == 0 && r0 + r < a.n) a.partial[size_t(r0 + r) * nw + wave_sites / 64] = v;
        }
      }
    }
  }
}

// Row form of the register-tile kernel (one rhs per thread, 18-real links) for launches too small to
// fill the chip: one rhs of 64 sites is a workgroup of three waves, wave w computing row w of every
// hop.  What bounds such a launch is its serial chain, not a rate: k_dslash waits for memory hop by
// hop, and the LDS forms stage all 144 link planes of 64 sites before the few waves that hold a rhs
// tile start.  Here every load of the kernel (16 gathers and 48 link entries a lane) is in flight
// at once, and a third of the link loads and FMAs is left on each wave.  The links, used by one wave
// each, stay in registers; the gathered vectors, used by all three, are loaded once (component w by
// wave w) and exchanged through LDS.  Each row keeps its FMA order, and the fused form sums <p, q> over
// the rows in wave 0 in the order of k_dslash: same bits.
// Half Dslash, microseconds, the fastest other form -> this (MI355X): 8^4, 1 rhs: FP64 5.6 -> 4.3, fused
// M 6.7 -> 4.6, FP32 6.2 -> 4.2, FP16 links 5.4 -> 3.7; 8^4, 8 rhs: 6.6 -> 5.0, 6.8 -> 4.5, 6.8 -> 4.0;
// 16^4, 1 rhs: 14.5 -> 13.4, 10.8 -> 8.0, 7.7 -> 5.9.
template <typename Real, typename LT, bool EPI, bool NT>
__global__ void __launch_bounds__(192) k_dslash_rows(Args a) {
  using C = typename CT<Real>::T;
  __shared__ C vs[48 * 64];
  const Geometry &g = a.g;
  const int chunk = gridDim.x >> 3;
  const int lb = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if (lb >= a.nsblk * a.ntiles) return;  // uniform for the whole workgroup
  const int sblk = lb / a.ntiles;
  const int r = lb - sblk * a.ntiles;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned vh = g.vh;
  const bool valid = sblk * 64u + lane < vh;
  const unsigned s = valid ? sblk * 64u + lane : vh - 1;
  const unsigned nw = (vh + 63) / 64;
  if (a.active && !a.active[r]) {  // uniform
    if constexpr (EPI) {
      if (a.partial && threadIdx.x == 0) a.partial[size_t(r) * nw + sblk] = 0.0;
    }
    return;
  }
  const size_t off = size_t(r) * 3 * vh + size_t(w) * vh;
  const C *__restrict__ in = static_cast<const C *>(a.in) + off;
  const LT *__restrict__ lk = static_cast<const LT *>(a.links) + size_t(w) * 3 * vh + s;

  const unsigned row = fast_div(s, a.div_xh);
  const int xh = int(s - row * g.lxh);
  const unsigned rz = fast_div(row, a.div_y);
  const int y = int(row - rz * g.ly);
  const unsigned t = fast_div(rz, a.div_z);
  const int z = int(rz - t * g.lz);
  const int x = 2 * xh + ((y + z + int(t) + a.out_parity) & 1);
  C v[16];
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    unsigned f1, b1, f3, b3;
    hop_sites(g, mu, s, s - xh, x, y, z, int(t), f1, b1, f3, b3);
    v[mu * 4] = in[f1];
    v[mu * 4 + 1] = in[b1];
    v[mu * 4 + 2] = in[f3];
    v[mu * 4 + 3] = in[b3];
  }
  Real lr[16][3], li[16][3];
#pragma unroll
  for (int h = 0; h < 16; ++h)
#pragma unroll
    for (int b = 0; b < 3; ++b)  // in the order of use: hop h % 4 of direction h / 4
      ld_link<NT>(lk + size_t(link_plane((h & 3) * 4 + (h >> 2), 18) + b) * vh, lr[h][b], li[h][b]);
  C p;
  if constexpr (EPI) p = (static_cast<const C *>(a.pvec) + off)[s];
#pragma unroll
  for (int h = 0; h < 16; ++h) vs[(h * 3 + w) * 64 + lane] = v[h];
  __syncthreads();

  Real re = Real(0), im = Real(0);
#pragma unroll
  for (int h = 0; h < 16; ++h)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const C u = vs[(h * 3 + b) * 64 + lane];
      const Real xr = (h & 1) ? -lr[h][b] : lr[h][b];
      const Real xi = (h & 1) ? -li[h][b] : li[h][b];
      re = fmaR(xr, u.x, re);
      re = fmaR(-xi, u.y, re);
      im = fmaR(xr, u.y, im);
      im = fmaR(xi, u.x, im);
    }
  C o;
  if constexpr (!EPI) {
    o.x = re;
    o.y = im;
    if (valid) (static_cast<C *>(a.out) + off)[s] = o;
  } else {
    const Real m2 = Real(a.mass2);
    o.x = fmaR(m2, p.x, -re);
    o.y = fmaR(m2, p.y, -im);
    if (valid) (static_cast<C *>(a.out) + off)[s] = o;
    if (a.partial) {
      __syncthreads();  // every wave has read its vectors
      vs[w * 64 + lane] = o;
      vs[(3 + w) * 64 + lane] = p;
      __syncthreads();
      if (w == 0) {
        double d = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C oc = vs[c * 64 + lane], pc = vs[(3 + c) * 64 + lane];
          d = fma(double(pc.x), double(oc.x), d);
          d = fma(double(pc.y), double(oc.y), d);
        }
        if (!valid) d = 0.0;
#pragma unroll
        for (int o2 = 32; o2 > 0; o2 >>= 1) d += __shfl_down(d, o2, 64);
        if (lane == 0) a.partial[size_t(r) * nw + sblk] = d;
      }
    }
  }
}

// Word 3 of a raw buffer descriptor on CDNA (32-bit data format, no swizzle, no stride): a
// plain byte-addressed range checked against its size.
constexpr int kBufWord3 = 0x00020000;

// LDS of the whole-site form: the stored link planes of 64 sites, for 14-real Naik links the
// 8 x 3 rebuilt row-2 entries in the arithmetic type, then the neighbour table (16 byte
// offsets per site).
constexpr size_t kNbrTableBytes = size_t(16) * 64 * sizeof(unsigned);
// rebuilt Naik entries kept in LDS per site (arithmetic type): row 2 of the 8 Naik links for
// formats 14 and 13, all 9 entries for format 9
constexpr int lds_rebuilt_entries(int nr) { return (nr == 14 || nr == 13) ? 24 : (nr == 9 ? 72 : 0); }
// stored planes copied into LDS per site: all of them, except for format 9, whose Naik links are
// rebuilt straight from global memory (keeping their 36 stored planes in LDS as well would take
// a workgroup past half of a CU's LDS, one workgroup per CU instead of two)
constexpr int lds_staged_planes(int nr) { return nr == 9 ? 72 : link_planes_total(nr); }
template <typename Real, typename LT, int NR> constexpr size_t lds_nbr_offset() {
  return size_t(lds_staged_planes(NR)) * 64 * sizeof(LT) + size_t(lds_rebuilt_entries(NR)) * 64 * sizeof(typename CT<Real>::T);
}

// LDS of the 32-site form: the same pieces for 32 sites.
template <typename Real, typename LT, bool R14> constexpr size_t lds32_nbr_offset() {
  return size_t(R14 ? 128 : 144) * 32 * sizeof(LT) + (R14 ? size_t(24) * 32 * sizeof(typename CT<Real>::T) : 0);
}
constexpr size_t kNbrTable32Bytes = size_t(16) * 32 * sizeof(unsigned);

// 64-site block of LDS-form workgroup `bid` (of `nbid`, dealt round-robin to the 8 XCDs) under
// the XCD map of the launch (false: none).
__device__ inline bool lds_block_at(const Args &a, int bid, int nbid, int &sblk) {
  const Geometry &g = a.g;
  if (a.xmap == 2 || a.xmap == 3) {
    // XCD k owns the blocks [k, k+1) * bps/8 of every (z, t) plane (with Lx = 32: four y rows).
    // Map 2 walks the planes z-major (t fastest): the sites in flight on an XCD span a few z
    // slices of a thin slab whose t extent is the whole lattice, so the t and z neighbours they
    // gather (the Naik hops reach 3 slices away) are mostly still in that XCD's L2 while Lt is
    // small.  Map 3 walks z tiles of 4 slices, t within a tile and z fastest: a z neighbour is at
    // most 3 planes back in the walk inside a tile and a t neighbour 4 or 12, so on large
    // lattices (64^3 x 16: 4 blocks per plane and XCD, 16 planes in flight) the window that has
    // to stay in L2 no longer grows with Lt; hops that cross a tile boundary re-fetch.
    const int k = bid & 7, j = bid >> 3;
    const int bpx = a.zmap_bps >> 3;
    const int w = j / bpx;  // position of the (z, t) plane in the XCD's walk
    int z, t;
    if (a.xmap == 2) {
      z = w / g.lt;
      t = w - z * g.lt;
    } else {
      const int tile = w / (4 * g.lt), rem = w - tile * 4 * g.lt;
      t = rem >> 2;
      z = tile * 4 + (rem & 3);
    }
    if (z >= g.lz) return false;
    sblk = (t * g.lz + z) * a.zmap_bps + k * bpx + (j - w * bpx);
  } else if (a.xmap == 1) {
    // XCD k owns the z slices [k Lz/8, (k+1) Lz/8) for every t: the z and t neighbours of its
    // sites stay mostly in its own L2 (with contiguous chunks, Lt = 8 would give each XCD a single
    // t slice and send every t hop to another XCD's data)
    const int k = bid & 7, j = bid >> 3;
    const int per_t = a.zmap_zr * a.zmap_bps;
    const int t = j / per_t;
    if (t >= g.lt) return false;
    const int rem = j - t * per_t;
    const int zl = rem / a.zmap_bps;
    sblk = (t * g.lz + k * a.zmap_zr + zl) * a.zmap_bps + (rem - zl * a.zmap_bps);
  } else {
    const int chunk = nbid >> 3;
    sblk = (bid & 7) * chunk + (bid >> 3);
    if (sblk >= a.nsblk) return false;
  }
  return true;
}
__device__ inline bool lds_block(const Args &a, int &sblk) { return lds_block_at(a, blockIdx.x, gridDim.x, sblk); }

// Naik link k (0..7: hops 8 + k) of lane `lane` from the staged LDS copy: rows 0 and 1 from the
// stored planes and, for 14- and 13-real links, row 2 from the entries rebuilt once per site;
// 9-real links entirely from the rebuilt entries.  (SB: sites per LDS plane)
template <typename Real, typename LT, int NR, int SB = 64>
__device__ inline void load_naik_lds(const LT *__restrict__ sl, const typename CT<Real>::T *__restrict__ row2,
                                     int k, int lane, Lnk<Real> &L) {
  if constexpr (NR == 18) {
    load_link<Real, LT, false, false>(sl, link_plane(8 + k, NR), unsigned(SB), unsigned(lane), L);
  } else if constexpr (NR == 9) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const typename CT<Real>::T v = row2[(k * 9 + a * 3 + b) * SB + lane];
        L.re[a][b] = v.x;
        L.im[a][b] = v.y;
      }
  } else {
    const LT *p = sl + link_plane(8 + k, NR) * SB + lane;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) ld_link<false>(p + (a * 3 + b) * SB, L.re[a][b], L.im[a][b]);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const typename CT<Real>::T v = row2[(k * 3 + b) * SB + lane];
      L.re[2][b] = v.x;
      L.im[2][b] = v.y;
    }
  }
}

// Write one rhs tile of an LDS-form workgroup: w = acc, or for the fused M form
// q = m2 p - acc with the per-64-site FP64 partials of Re<p, q> (all 64 lanes of the wave take
// part in the reduction; the partial of block sblk is written by lane 0).
template <typename Real, int RT, bool EPI>
__device__ inline void store_tile(const Args &a, int r0, unsigned s, int lane, int sblk, const bool (&act)[RT],
                                  const Real (&acc_re)[RT][3], const Real (&acc_im)[RT][3]) {
  using C = typename CT<Real>::T;
  const unsigned vh = a.g.vh;
  const size_t tile_off = size_t(r0) * 3 * vh;
  C *__restrict__ out = static_cast<C *>(a.out) + tile_off;
  if constexpr (!EPI) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      if (!act[r]) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        C o;
        o.x = acc_re[r][c];
        o.y = acc_im[r][c];
        out[(unsigned)(r * 3 + c) * vh + s] = o;
      }
    }
  } else {
    const C *__restrict__ pv = static_cast<const C *>(a.pvec) + tile_off;
    const Real m2 = Real(a.mass2);
    double dot[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      dot[r] = 0.0;
      if (!act[r]) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const C p = pv[(unsigned)(r * 3 + c) * vh + s];
        C o;
        o.x = fmaR(m2, p.x, -acc_re[r][c]);
        o.y = fmaR(m2, p.y, -acc_im[r][c]);
        out[(unsigned)(r * 3 + c) * vh + s] = o;
        dot[r] = fma(double(p.x), double(o.x), dot[r]);
        dot[r] = fma(double(p.y), double(o.y), dot[r]);
      }
    }
    if (a.partial) {
      const unsigned nw = (vh + 63) / 64;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        double v = dot[r];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0 && r0 + r < a.n) a.partial[size_t(r0 + r) * nw + sblk] = v;
      }
    }
  }
}

// raw link-entry load (optionally non-temporal) for LDS staging
template <bool NT> __device__ inline float2 ld_raw(const float2 *p) {
  if constexpr (NT) {
    const unsigned long long u = __builtin_nontemporal_load(reinterpret_cast<const unsigned long long *>(p));
    return *reinterpret_cast<const float2 *>(&u);
  } else {
    return *p;
  }
}
template <bool NT> __device__ inline double2 ld_raw(const double2 *p) {
  if constexpr (NT) {
    const d2v v = __builtin_nontemporal_load(reinterpret_cast<const d2v *>(p));
    double2 o;
    o.x = v.x;
    o.y = v.y;
    return o;
  } else {
    return *p;
  }
}
template <bool NT> __device__ inline __half2 ld_raw(const __half2 *p) {
  if constexpr (NT) {
    const unsigned u = __builtin_nontemporal_load(reinterpret_cast<const unsigned *>(p));
    return *reinterpret_cast<const __half2 *>(&u);
  } else {
    return *p;
  }
}

// LDS-staged form: a workgroup of 64 sites x WPB waves first copies the links of its 64 sites
// (all 16 hops) into LDS, then the waves loop over the rhs tiles (wave w takes tiles w, w+WPB,
// ...), reading the links from LDS for every tile.  Only WPB*RT rhs of a site block are in
// flight at a time, so the neighbour vectors other workgroups gather are far more likely to be
// found in L2 than when every thread holds all n rhs; the links still come from HBM once.
// Same site order, hop order and FMA sequence per rhs as k_dslash (bit-identical output), and
// the same per-64-site grouping of the fused <p, Mp> partials.
// (the second launch bound is the waves per SIMD: two workgroups share a CU -- with 16 waves at
// most 64 VGPRs, with 8 at most 128 -- except with FP64 links, whose 147 KB take a CU's LDS alone)
template <typename Real, typename LT, int RT, int NR, bool EPI, int WPB, bool NT>
__global__ void __launch_bounds__(64 * WPB, WPB / 4 * (sizeof(LT) > 8 ? 1 : 2)) k_dslash_lds(Args a) {
  static_assert(WPB == 4 || WPB == 8 || WPB == 16, "4, 8 or 16 waves per workgroup");
  using C = typename CT<Real>::T;
  constexpr int recon = NR;
  constexpr int PL = lds_staged_planes(NR);  // stored planes per site staged in LDS
  extern __shared__ __align__(16) unsigned char smem_raw[];
  LT *sl = reinterpret_cast<LT *>(smem_raw);
  const Geometry &g = a.g;
  int sblk;
  if (!lds_block(a, sblk)) return;  // uniform for the whole workgroup
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned vh = g.vh;
  const unsigned s = sblk * 64 + lane;
  const bool valid = s < vh;
  const LT *__restrict__ links = static_cast<const LT *>(a.links);
  // every lane computes: a lane past the last site works on site 0 (in-range addresses) and
  // stores nothing
  const unsigned sc = valid ? s : 0u;
  // stage the links of the 64 sites: plane-major, lane-minor (conflict-free LDS access); each
  // wave issues a batch of CH plane loads before it writes any of them, so their latencies
  // overlap.  With NT the global loads carry the non-temporal hint, so the streamed links do
  // not push the neighbour vectors out of L2.
  if constexpr (PL % WPB == 0 && (PL / WPB) % (PL / WPB % 9 == 0 ? 9 : 8) == 0) {
    constexpr int PPW = PL / WPB;
    constexpr int CH = PPW % 9 == 0 ? 9 : 8;
#pragma unroll 1
    for (int c0 = 0; c0 < PPW; c0 += CH) {
      LT v[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) v[i] = ld_raw<NT>(links + size_t(wave + (c0 + i) * WPB) * vh + sc);
#pragma unroll
      for (int i = 0; i < CH; ++i) sl[(wave + (c0 + i) * WPB) * 64 + lane] = v[i];
    }
  } else {  // plane counts that do not split into whole batches (Naik formats 13 and 9)
    constexpr int PPW = (PL + WPB - 1) / WPB;
    constexpr int CH = 8;
#pragma unroll 1
    for (int c0 = 0; c0 < PPW; c0 += CH) {
      LT v[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int pl = wave + (c0 + i) * WPB;
        if (pl < PL) v[i] = ld_raw<NT>(links + size_t(pl) * vh + sc);
      }
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int pl = wave + (c0 + i) * WPB;
        if (pl < PL) sl[pl * 64 + lane] = v[i];
      }
    }
  }
  // 14-, 13- and 9-real Naik links: rebuild what the format leaves out once per site (not once
  // per rhs tile) into LDS entries of the arithmetic type after the staged planes, with the same
  // arithmetic as load_naik: the whole link for 9 here, from global memory; row 2 for 14 and 13
  // from the staged planes after the barrier below
  C *row2 = reinterpret_cast<C *>(sl + PL * 64);
  if constexpr (NR == 9) {
    for (int item = threadIdx.x; item < 8 * 64; item += 64 * WPB) {
      const int k = item >> 6, ln = item & 63;
      const unsigned site = sblk * 64 + ln;
      Lnk<Real> Lk;
      load_naik<Real, LT, NR, NT>(links, 8 + k, vh, site < vh ? site : 0u, Lk);
#pragma unroll
      for (int ra = 0; ra < 3; ++ra)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          C v;
          v.x = Lk.re[ra][b];
          v.y = Lk.im[ra][b];
          row2[(k * 9 + ra * 3 + b) * 64 + ln] = v;
        }
    }
  }
  // neighbour table: the byte offsets (within a colour plane) of the 16 neighbours of the 64
  // sites, [mu][site][+1, -1, +3, -3], built once per workgroup (one hop per wave and lane with
  // 16 waves) so the rhs-tile loop does no site arithmetic
  unsigned *nbt = reinterpret_cast<unsigned *>(smem_raw + lds_nbr_offset<Real, LT, NR>());
  {
    const unsigned q1 = fast_div(sc, a.div_xh);
    const unsigned q2 = fast_div(q1, a.div_y);
    const unsigned q3 = fast_div(q2, a.div_z);
    const int xh = int(sc - q1 * unsigned(g.lxh));
    const int y = int(q1 - q2 * unsigned(g.ly));
    const int z = int(q2 - q3 * unsigned(g.lz));
    const int t = int(q3);
    const int x = 2 * xh + ((y + z + t + a.out_parity) & 1);
    const unsigned rowbase = sc - unsigned(xh);
    for (int h = wave; h < 16; h += WPB) {
      const int mu = h >> 2, k = h & 3;
      const int d = k == 0 ? 1 : (k == 1 ? -1 : (k == 2 ? 3 : -3));
      nbt[(mu * 64 + lane) * 4 + k] = hop_site(g, mu, d, sc, rowbase, x, y, z, t) * unsigned(sizeof(C));
    }
  }
  __syncthreads();
  if constexpr (NR == 14 || NR == 13) {
    for (int item = threadIdx.x; item < 8 * 64; item += 64 * WPB) {
      const int k = item >> 6, ln = item & 63;
      Lnk<Real> Lk;
      load_naik<Real, LT, NR, false>(sl, 8 + k, 64u, unsigned(ln), Lk);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        C v;
        v.x = Lk.re[2][b];
        v.y = Lk.im[2][b];
        row2[(k * 3 + b) * 64 + ln] = v;
      }
    }
    __syncthreads();
  }
  // a tile spans RT * 3 colour planes of less than 4 GiB in all (checked at launch)
  const unsigned plane_bytes = vh * unsigned(sizeof(C));
  for (int tile = wave; tile < a.ntiles; tile += WPB) {
    const int r0 = tile * RT;
    int rr[RT];
    bool ract[RT];
    if (!tile_rhs<RT>(a, r0, rr, ract)) {  // the whole tile is inactive (uniform)
      if constexpr (EPI) {
        if (a.partial && lane == 0) {
          const unsigned nw = (vh + 63) / 64;
#pragma unroll
          for (int r = 0; r < RT; ++r)
            if (r0 + r < a.n) a.partial[size_t(r0 + r) * nw + sblk] = 0.0;
        }
      }
      continue;
    }
    const char *in = static_cast<const char *>(a.in) + size_t(r0) * 3 * plane_bytes;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(in), short(0), int(RT * 3 * plane_bytes), kBufWord3);
    Real acc_re[RT][3], acc_im[RT][3];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc_re[r][c] = acc_im[r][c] = Real(0);
    // hop order as in k_dslash: per mu, fat fwd, fat bwd, Naik fwd, Naik bwd
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      const uint4 nb = reinterpret_cast<const uint4 *>(nbt)[mu * 64 + lane];
      Lnk<Real> Lk;
      load_link<Real, LT, false, false>(sl, link_plane(mu, recon), 64u, lane, Lk);
      apply_hop_buf<Real, RT, false>(Lk, rs, plane_bytes, nb.x, rr, acc_re, acc_im);
      load_link<Real, LT, false, false>(sl, link_plane(4 + mu, recon), 64u, lane, Lk);
      apply_hop_buf<Real, RT, true>(Lk, rs, plane_bytes, nb.y, rr, acc_re, acc_im);
      load_naik_lds<Real, LT, NR>(sl, row2, mu, lane, Lk);
      apply_hop_buf<Real, RT, false>(Lk, rs, plane_bytes, nb.z, rr, acc_re, acc_im);
      load_naik_lds<Real, LT, NR>(sl, row2, 4 + mu, lane, Lk);
      apply_hop_buf<Real, RT, true>(Lk, rs, plane_bytes, nb.w, rr, acc_re, acc_im);
    }
    bool act[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) act[r] = valid && ract[r];
    store_tile<Real, RT, EPI>(a, r0, s, lane, sblk, act, acc_re, acc_im);
  }
}

// Window of the buffer loads of the rhs tile `tile` (of `width` rhs, n in all): its first rhs, the bytes
// of the rhs that exist, and the scalar offset from one colour plane to the next.  A wave without a
// tile (tile * width >= n) gets an empty window and must have step 0: a raw buffer load compares its
// vector offset with the window's size minus the scalar offset, and 0 bytes minus a plane wraps
// round to a range that lets the load through, past the caller's vector.
struct TileWindow {
  int rhs;
  unsigned bytes, step;
};
__host__ __device__ constexpr TileWindow tile_window(int tile, int width, int n, unsigned plane_bytes) {
  const int r0 = tile * width < n ? tile * width : n;
  const int live = n - r0 < width ? n - r0 : width;
  return {r0, unsigned(live) * 3u * plane_bytes, live > 0 ? plane_bytes : 0u};
}

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// ---- pair form -------------------------------------------------------------------------------
// 16 bytes at an address that need only be a multiple of 8 (complex64 vectors)
typedef float f4a8_t __attribute__((ext_vector_type(4), aligned(8)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));

// Link entries of the sites of a lane (LDS plane-major, sites adjacent).
template <typename LT> struct LinkPair;
template <> struct LinkPair<double2> {
  __device__ static void load(const double2 *p, double (&re)[1], double (&im)[1]) {
    const double2 v = *p;
    re[0] = v.x;
    im[0] = v.y;
  }
};
template <> struct LinkPair<float2> {
  __device__ static void load(const float2 *p, float (&re)[2], float (&im)[2]) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    re[0] = v.x;
    im[0] = v.y;
    re[1] = v.z;
    im[1] = v.w;
  }
};
template <> struct LinkPair<__half2> {
  __device__ static void load(const __half2 *p, float (&re)[2], float (&im)[2]) {
    const uint2 u = *reinterpret_cast<const uint2 *>(p);
    const float2 a = __half22float2(*reinterpret_cast<const __half2 *>(&u.x));
    const float2 b = __half22float2(*reinterpret_cast<const __half2 *>(&u.y));
    re[0] = a.x;
    im[0] = a.y;
    re[1] = b.x;
    im[1] = b.y;
  }
};

// LDS of the pair form: as the whole-site form, with the neighbour table per pair of sites.
template <typename Real> constexpr size_t nbr_table_pair_bytes() {
  return size_t(4) * (sizeof(Real) == 4 ? 32 : 64) * sizeof(uint4);
}

// Waves per SIMD of the pair form: 128 registers and 16 waves per CU (two workgroups of 8 waves with
// FP32 links, four of 4 with FP16 links), or 256 registers and 8 waves with two FP32 rhs per lane, whose
// gathers do not fit in 128.  FP64 links take a CU's LDS alone: one workgroup.
template <typename LT, int RT> constexpr int pair_waves_per_simd(int wpb) {
  return sizeof(LT) > 8 ? wpb / 4 : (RT == 2 ? (wpb > 8 ? wpb / 4 : 2) : (wpb == 4 && sizeof(LT) > 4 ? 2 : 4));
}
// Hops gathered ahead: as many as fit in the registers
constexpr int kLook64 = 6;  // (3, 6 and 12: within 1 % of each other)
template <typename LT, int RT, bool EPI> constexpr int pair_look(int wpb) {
  if (sizeof(LT) > 8) return wpb == 16 ? (RT == 1 ? 2 : 1) : (RT == 1 ? kLook64 : 2);
  return EPI ? 2 : 3;
}
// the (re, im) of site s of a lane's 16 gathered bytes
__device__ inline void site_value(const v4u_t &x, int s, float &re, float &im) {
  re = __uint_as_float(x[2 * s]);
  im = __uint_as_float(x[2 * s + 1]);
}
__device__ inline void site_value(const v4u_t &x, int, double &re, double &im) {
  re = __hiloint2double(int(x[1]), int(x[0]));
  im = __hiloint2double(int(x[3]), int(x[2]));
}

// Whole-site LDS form with two neighbouring sites (2 i, 2 i + 1) per lane, for complex64 vectors
// on lattices with Lx divisible by 4 (a pair never straddles an x row; V/2 is then a multiple of
// 16).  What bounds the one-site form is the rate at which a CU's vector memory path takes load
// instructions: a wave's 8-byte loads move 32 bytes per clock, its 16-byte loads 62 (measured on
// L1-resident data), so a tile's gathers alone cost ~41 us of the 76 us launch at 32^3 x 8 with
// 16 rhs (FP32).  Here every gather, link staging load and store is 16 bytes wide: 66 us by the tuner's
// clock (58 us of that remain without any arithmetic or link reads), 69 us in a kernel trace, where
// 355 MB, 1.41 times the compulsory bytes, go past L2 at 5.2 TB/s.
//   * y, z and t neighbours of a pair are a pair; the eight x neighbours of a pair are all among
//     the pair itself and the pairs before and after it in its row (three loads, not four), picked
//     by the parity of the row.
//   * the two 32-lane halves of a wave take different rhs: lane (pair i, half h) computes rhs
//     r0 + h RT + r of a tile of 2 RT; the rhs offset is in the buffer loads' vector offset, so a
//     rhs past n reads past the buffer's range (returns 0) and is not stored.
// FP64 runs the same kernel with one site per lane and one rhs group (its gathers are 16 bytes already;
// 32^3 x 8, 8 rhs: 96.4 -> 94.5 us, fused M form 103.7 -> 98.6; 16 rhs: 135 -> 132 and 146 -> 138 us:
// one workgroup fills a CU's LDS, so the link staging is not hidden).
// Same hop order and FMA sequence per site and rhs as k_dslash, and the same tree over the 64
// sites of a block for the fused <p, Mp> partials (bit-identical outputs).
template <typename Real, typename LT, int RT, int NR, bool EPI, int WPB, bool NT>
__global__ void __launch_bounds__(64 * WPB, (pair_waves_per_simd<LT, RT>(WPB))) k_dslash_pair(Args a) {
  using C = typename CT<Real>::T;
  using V16 = std::conditional_t<sizeof(Real) == 4, f4a8_t, d2v>;  // 16 bytes of a vector in memory
  constexpr int S = 16 / int(sizeof(C));     // sites per lane, and rhs groups of a wave
  constexpr int LPH = 64 / S;                // lanes of a group
  constexpr unsigned CB = sizeof(C);
  constexpr int PL = lds_staged_planes(NR);
  constexpr int SPL = 16 / int(sizeof(LT));  // sites per lane, and planes per wave, of a staging load
  extern __shared__ __align__(16) unsigned char smem_raw[];
  LT *sl = reinterpret_cast<LT *>(smem_raw);
  const Geometry &g = a.g;
  int sblk;
  if (!lds_block(a, sblk)) return;  // uniform for the whole workgroup
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pi = lane % LPH, h = S == 1 ? 0 : lane / LPH;
  const unsigned vh = g.vh;
  const unsigned s0 = unsigned(sblk) * 64;
  const LT *__restrict__ links = static_cast<const LT *>(a.links);
  const unsigned plane_bytes = vh * unsigned(sizeof(C));
  // neighbour table of the lanes' sites, byte offsets within a colour plane: [mu] the sites (pairs) at
  // +1, -1, +3, -3; with pairs [0] is the pair before, the pair itself, the pair after in its x row,
  // and the row's parity
  uint4 *nbt = reinterpret_cast<uint4 *>(smem_raw + lds_nbr_offset<Real, LT, NR>());
  // ---- gathers of one tile: LOOK hops ahead of the arithmetic (the compiler alone keeps one hop in
  // flight).  Hop i = 4 (mu - MU0) + k is held in slot i % (LOOK + 1).
  constexpr int LOOK = pair_look<LT, RT, EPI>(WPB);
  constexpr int NH = S == 2 ? 12 : 16;  // hops gathered one by one (with two sites per lane all but x)
  constexpr int MU0 = S == 2 ? 1 : 0;
  v4u_t v[LOOK + 1][RT][3], xm[S == 2 ? RT : 1][3], xc[S == 2 ? RT : 1][3], xp[S == 2 ? RT : 1][3];
  uint4 nb;
  bool odd;
  int pj = pi;
  __amdgpu_buffer_rsrc_t rs;
  const unsigned hoff = unsigned(h * RT * 3) * plane_bytes;
  auto gather = [&](unsigned off, int r, int b, unsigned step) -> v4u_t {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, off + hoff + unsigned(r * 3) * plane_bytes,
                                                 unsigned(b) * step, 0);
  };
  auto issue = [&](auto ic, unsigned step) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i % 4 == 0) nb = nbt[(MU0 + i / 4) * LPH + pj];
    const unsigned off = (i & 3) == 0 ? nb.x : ((i & 3) == 1 ? nb.y : ((i & 3) == 2 ? nb.z : nb.w));
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int b = 0; b < 3; ++b) v[i % (LOOK + 1)][r][b] = gather(off, r, b, step);
  };
  // the x pairs (S = 2) and the first LOOK hops of a tile; its buffer covers the rhs that exist (past the
  // last tile none: the loads read nothing and return 0).  step: the window's, or plane_bytes where the
  // tile is known to exist
  auto start_tile = [&](int tile, unsigned step) {
    const TileWindow w = tile_window(tile, S * RT, a.n, plane_bytes);
    const char *in = static_cast<const char *>(a.in) + size_t(w.rhs) * 3 * plane_bytes;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(in), short(0), int(w.bytes), kBufWord3);
    if constexpr (S == 2) {
      const uint4 nx = nbt[pj];
      odd = nx.w != 0;
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          xm[r][b] = gather(nx.x, r, b, step);
          xc[r][b] = gather(nx.y, r, b, step);
          xp[r][b] = gather(nx.z, r, b, step);
        }
    }
    static_for<LOOK>([&](auto ic) { issue(ic, step); });
  };
  // the active rhs of a tile, one bit each (uniform: scalar loads)
  auto tile_mask = [&](int tile) -> unsigned {
    unsigned m = 0;
#pragma unroll
    for (int k = 0; k < S * RT; ++k) {
      const int q = tile * S * RT + k;
      if (q < a.n && (!a.active || a.active[q])) m |= 1u << k;
    }
    return m;
  };
  // first tile from `tile` on with an active rhs (its rhs in `mask`); the tiles passed over get zero
  // partials
  unsigned mask = 0;
  auto next_tile = [&](int tile) -> int {
    for (; tile < a.ntiles; tile += WPB) {
      mask = tile_mask(tile);
      if (mask) break;
      if constexpr (EPI) {
        if (a.partial && lane < S * RT && tile * S * RT + lane < a.n)
          a.partial[size_t(tile * S * RT + lane) * ((vh + 63) / 64) + sblk] = 0.0;
      }
    }
    return tile;
  };

  // ---- set-up: link loads first, then the neighbour table and the first tile's gathers behind them,
  // so that their latencies overlap; a wave load covers SPL planes, 16 bytes a lane
  int tile;
  {
    constexpr int NI = (PL + SPL - 1) / SPL;   // wave loads
    constexpr int PW = (NI + WPB - 1) / WPB;   // of them per wave
    constexpr int CH = PW <= 9 ? PW : 9;       // in flight before any is written to LDS
    constexpr int LPP = 64 / SPL;              // lanes per plane
    constexpr bool whole = PL % (SPL * WPB * CH) == 0;
    const int pp = lane / LPP, st = (lane % LPP) * SPL;
    const unsigned ls = s0 + st < vh ? s0 + st : 0u;  // a lane past the last site stages site 0's links
    u4_t w[CH];
    auto fetch = [&](int c0) {
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int pl = (wave + (c0 + i) * WPB) * SPL + pp;
        if (whole || (c0 + i < PW && pl < PL)) {
          const u4_t *q = reinterpret_cast<const u4_t *>(links + size_t(pl) * vh + ls);
          if constexpr (NT) w[i] = __builtin_nontemporal_load(q);
          else w[i] = *q;
        }
      }
    };
    auto stash = [&](int c0) {
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int pl = (wave + (c0 + i) * WPB) * SPL + pp;
        if (whole || (c0 + i < PW && pl < PL)) *reinterpret_cast<u4_t *>(sl + pl * 64 + st) = w[i];
      }
    };
    fetch(0);
    if (wave < 4) {  // wave mu: with two rhs groups each half writes two of the four offsets
      const int mu = wave;
      const unsigned sp = s0 + S * pi < vh ? s0 + S * pi : 0u;  // first site of the lane (0 past the end)
      const unsigned q1 = fast_div(sp, a.div_xh);
      const unsigned q2 = fast_div(q1, a.div_y);
      const unsigned q3 = fast_div(q2, a.div_z);
      const int xh = int(sp - q1 * unsigned(g.lxh));
      const int y = int(q1 - q2 * unsigned(g.ly));
      const int z = int(q2 - q3 * unsigned(g.lz));
      const int t = int(q3);
      const unsigned rowbase = sp - unsigned(xh);
      const int par = (y + z + t + a.out_parity) & 1;
      if constexpr (S == 2) {
        uint2 n;
        if (mu == 0) {
          n.x = h ? (rowbase + unsigned(xh + 2 >= g.lxh ? 0 : xh + 2)) * CB
                  : (rowbase + unsigned(xh == 0 ? g.lxh - 2 : xh - 2)) * CB;
          n.y = h ? unsigned(par) : sp * CB;
        } else {
          const int d = h ? 3 : 1;
          n.x = hop_site(g, mu, d, sp, rowbase, 0, y, z, t) * CB;
          n.y = hop_site(g, mu, -d, sp, rowbase, 0, y, z, t) * CB;
        }
        reinterpret_cast<uint2 *>(nbt)[(mu * LPH + pi) * 2 + h] = n;
      } else {
        const int x = 2 * xh + par;
        uint4 n;
        n.x = hop_site(g, mu, 1, sp, rowbase, x, y, z, t) * CB;
        n.y = hop_site(g, mu, -1, sp, rowbase, x, y, z, t) * CB;
        n.z = hop_site(g, mu, 3, sp, rowbase, x, y, z, t) * CB;
        n.w = hop_site(g, mu, -3, sp, rowbase, x, y, z, t) * CB;
        nbt[mu * LPH + pi] = n;
      }
    }
    __syncthreads();
    tile = next_tile(wave);
    if constexpr (PW > CH) {
#pragma unroll 1
      for (int c0 = 0; c0 + CH < PW; c0 += CH) {
        stash(c0);
        fetch(c0 + CH);
      }
    }
    // also without a tile: a branch here would make the waits below cover the gathers
    start_tile(tile, tile_window(tile, S * RT, a.n, plane_bytes).step);
    stash((PW - 1) / CH * CH);
  }
  // compressed Naik links: rebuilt once per site, as in the one-site form
  C *row2 = reinterpret_cast<C *>(sl + PL * 64);
  if constexpr (NR == 9) {
    for (int item = threadIdx.x; item < 8 * 64; item += 64 * WPB) {
      const int k = item >> 6, ln = item & 63;
      const unsigned site = s0 + ln;
      Lnk<Real> Lk;
      load_naik<Real, LT, NR, NT>(links, 8 + k, vh, site < vh ? site : 0u, Lk);
#pragma unroll
      for (int e = 0; e < 9; ++e) row2[(k * 9 + e) * 64 + ln] = C{Lk.re[e / 3][e % 3], Lk.im[e / 3][e % 3]};
    }
  }
  __syncthreads();
  if constexpr (NR == 14 || NR == 13) {
    for (int item = threadIdx.x; item < 8 * 64; item += 64 * WPB) {
      const int k = item >> 6, ln = item & 63;
      Lnk<Real> Lk;
      load_naik<Real, LT, NR, false>(sl, 8 + k, 64u, unsigned(ln), Lk);
#pragma unroll
      for (int b = 0; b < 3; ++b) row2[(k * 3 + b) * 64 + ln] = C{Lk.re[2][b], Lk.im[2][b]};
    }
    __syncthreads();
  }

  // entry (ra, b) of the link of hop k (0..15) for the lane's sites
  auto link_entry = [&](int k, int ra, int b, Real (&re)[S], Real (&im)[S]) {
    if constexpr (NR == 9) {
      if (k >= 8) {
        LinkPair<C>::load(row2 + S * pj + ((k - 8) * 9 + ra * 3 + b) * 64, re, im);
        return;
      }
    } else if constexpr (NR != 18) {
      if (k >= 8 && ra == 2) {
        LinkPair<C>::load(row2 + S * pj + ((k - 8) * 3 + b) * 64, re, im);
        return;
      }
    }
    LinkPair<LT>::load(sl + S * pj + (link_plane(k, NR) + ra * 3 + b) * 64, re, im);
  };
  while (tile < a.ntiles) {
    const int q0 = tile * S * RT + h * RT;  // this lane's first rhs
    Real acc_re[RT][S][3], acc_im[RT][S][3];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) acc_re[r][s][c] = acc_im[r][s][c] = Real(0);
    // The arithmetic of a hop ends here for the scheduler, and the link reads of the next one start
    // (left to itself the compiler issues the LDS reads of all 16 hops at once and spills them).
    auto fence = [&] {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int s = 0; s < S; ++s)
          asm volatile("" : "+v"(acc_re[r][s][0]), "+v"(acc_re[r][s][1]), "+v"(acc_re[r][s][2]), "+v"(acc_im[r][s][0]),
                       "+v"(acc_im[r][s][1]), "+v"(acc_im[r][s][2]), "+v"(pj));
    };
    // acc += sign * L x, x[r][b] = the lane's sites (re, im) (hops +1, -1, +3, -3 are k / 4 = 0 .. 3)
    auto hop = [&](auto kc, const v4u_t (&x)[RT][3]) {
      constexpr int k = decltype(kc)::value;
      constexpr bool neg = (k / 4) & 1;
#pragma unroll
      for (int ra = 0; ra < 3; ++ra) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          Real lre[S], lim[S];
          link_entry(k, ra, b, lre, lim);
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const Real lr = neg ? -lre[s] : lre[s];
            const Real li = neg ? -lim[s] : lim[s];
#pragma unroll
            for (int r = 0; r < RT; ++r) {
              Real vx, vy;
              site_value(x[r][b], s, vx, vy);
              acc_re[r][s][ra] = fmaR(lr, vx, acc_re[r][s][ra]);
              acc_re[r][s][ra] = fmaR(-li, vy, acc_re[r][s][ra]);
              acc_im[r][s][ra] = fmaR(lr, vy, acc_im[r][s][ra]);
              acc_im[r][s][ra] = fmaR(li, vx, acc_im[r][s][ra]);
            }
          }
        }
      }
      fence();
    };
    fence();
    if constexpr (S == 2) {
      static_for<4>([&](auto kc) {  // x direction: +1, -1, +3, -3 from shifts of the row by -2..2 sites
        constexpr int k = decltype(kc)::value;
        v4u_t x[RT][3];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const v4u_t M = xm[r][b], Z = xc[r][b], P = xp[r][b];
            const v4u_t lo = {M[2], M[3], Z[0], Z[1]}, hi = {Z[2], Z[3], P[0], P[1]};  // shifts -1, +1
            const v4u_t u = k == 0 ? hi : (k == 1 ? Z : (k == 2 ? P : lo));  // rows of odd parity
            const v4u_t w = k == 0 ? Z : (k == 1 ? lo : (k == 2 ? hi : M));  // rows of even parity
#pragma unroll
            for (int e = 0; e < 4; ++e) x[r][b][e] = odd ? u[e] : w[e];
          }
        hop(std::integral_constant<int, 4 * k>{}, x);
      });
    }
    const bool valid = s0 + S * pi < vh;
    bool act[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) act[r] = valid && ((mask >> (h * RT + r)) & 1u);
    const size_t tile_off = size_t(q0) * 3 * vh + s0 + S * pi;  // the lane's first output
    V16 pv[RT][3];
    static_for<NH>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      if constexpr (i + LOOK < NH) issue(std::integral_constant<int, i + LOOK>{}, plane_bytes);
      if constexpr (EPI && i + LOOK == NH) {
        const C *p = static_cast<const C *>(a.pvec) + tile_off;
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (act[r]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) pv[r][c] = *reinterpret_cast<const V16 *>(p + size_t(r * 3 + c) * vh);
          }
      }
      hop(std::integral_constant<int, 4 * (i & 3) + MU0 + i / 4>{}, v[i % (LOOK + 1)]);
    });
    const int done = tile;
    tile = next_tile(tile + WPB);
    if (tile < a.ntiles) start_tile(tile, plane_bytes);
    C *out = static_cast<C *>(a.out) + tile_off;
    if constexpr (!EPI) {
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        if (!act[r]) continue;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          V16 o;
#pragma unroll
          for (int s = 0; s < S; ++s) {
            o[2 * s] = acc_re[r][s][c];
            o[2 * s + 1] = acc_im[r][s][c];
          }
          *reinterpret_cast<V16 *>(out + size_t(r * 3 + c) * vh) = o;
        }
      }
    } else {
      const Real m2 = Real(a.mass2);
      const unsigned nw = (vh + 63) / 64;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        double d[S];
#pragma unroll
        for (int s = 0; s < S; ++s) d[s] = 0.0;
        if (act[r]) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const V16 p = pv[r][c];
            V16 o;
#pragma unroll
            for (int s = 0; s < S; ++s) {
              o[2 * s] = fmaR(m2, p[2 * s], -acc_re[r][s][c]);
              o[2 * s + 1] = fmaR(m2, p[2 * s + 1], -acc_im[r][s][c]);
              d[s] = fma(double(p[2 * s]), double(o[2 * s]), d[s]);
              d[s] = fma(double(p[2 * s + 1]), double(o[2 * s + 1]), d[s]);
            }
            *reinterpret_cast<V16 *>(out + size_t(r * 3 + c) * vh) = o;
          }
        }
        if (a.partial) {
          // the tree of k_dslash over the 64 sites: site s + site (s + 32), then + (s + 16), ..., + (s + 1)
#pragma unroll
          for (int off = LPH / 2; off > 0; off >>= 1) {
#pragma unroll
            for (int s = 0; s < S; ++s) d[s] += __shfl_down(d[s], off, 64);
          }
          if (pi == 0 && done * S * RT + h * RT + r < a.n)
            a.partial[size_t(done * S * RT + h * RT + r) * nw + sblk] = S == 2 ? d[0] + d[S - 1] : d[0];
        }
      }
    }
  }
}

// 32-site LDS form (plain half Dslash): a workgroup of 32 sites x WPB waves stages half the links
// of the whole-site form, so that an FP64 workgroup (74 KB) shares a CU with another (and an
// FP32 or FP16 one with three).  The two 32-lane halves of a wave take different rhs: lane
// (site i, half h) computes rhs r0 + h RT + r of a tile of 2 RT rhs.  Workgroups 2j and 2j+1 of
// an XCD take the two halves of the 64-site block the XCD map gives for j.  The rhs offset of a
// lane goes into the buffer loads' vector offset, so a rhs past n reads past the buffer's range
// (returns 0) and is not stored.  Same hop order and FMA sequence per rhs as k_dslash
// (bit-identical output).  The second launch bound: FP64 two workgroups per CU, else four.
template <typename Real, typename LT, int RT, bool R14, int WPB, bool NT>
__global__ void __launch_bounds__(64 * WPB, WPB / 4 * (sizeof(LT) > 8 ? 2 : 4)) k_dslash_lds32(Args a) {
  static_assert(WPB == 4 || WPB == 8, "4 or 8 waves per workgroup");
  using C = typename CT<Real>::T;
  constexpr int recon = R14 ? 14 : 18;
  constexpr int PL = R14 ? 128 : 144;  // stored planes per site
  extern __shared__ __align__(16) unsigned char smem_raw[];
  LT *sl = reinterpret_cast<LT *>(smem_raw);
  const Geometry &g = a.g;
  const int bx = blockIdx.x;
  int sblk;
  if (!lds_block_at(a, ((bx >> 3) >> 1) * 8 + (bx & 7), gridDim.x >> 1, sblk)) return;  // uniform
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int si = lane & 31, h = lane >> 5;
  const unsigned vh = g.vh;
  const unsigned s = sblk * 64 + ((bx >> 3) & 1) * 32 + si;
  const bool valid = s < vh;
  const unsigned sc = valid ? s : 0u;
  const LT *__restrict__ links = static_cast<const LT *>(a.links);
  // stage the links of the 32 sites, [plane][32]: a wave load covers planes 2 pp and 2 pp + 1
  {
    constexpr int PPW = PL / 2 / WPB;  // plane pairs per wave
    constexpr int CH = PPW % 9 == 0 ? 9 : 8;
    static_assert(PPW % CH == 0, "whole batches");
#pragma unroll 1
    for (int c0 = 0; c0 < PPW; c0 += CH) {
      LT v[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) v[i] = ld_raw<NT>(links + size_t(2 * (wave + (c0 + i) * WPB) + h) * vh + sc);
#pragma unroll
      for (int i = 0; i < CH; ++i) sl[(2 * (wave + (c0 + i) * WPB) + h) * 32 + si] = v[i];
    }
  }
  // neighbour table [mu][site][+1, -1, +3, -3] (byte offsets within a colour plane)
  unsigned *nbt = reinterpret_cast<unsigned *>(smem_raw + lds32_nbr_offset<Real, LT, R14>());
  {
    const unsigned q1 = fast_div(sc, a.div_xh);
    const unsigned q2 = fast_div(q1, a.div_y);
    const unsigned q3 = fast_div(q2, a.div_z);
    const int xh = int(sc - q1 * unsigned(g.lxh));
    const int y = int(q1 - q2 * unsigned(g.ly));
    const int z = int(q2 - q3 * unsigned(g.lz));
    const int t = int(q3);
    const int x = 2 * xh + ((y + z + t + a.out_parity) & 1);
    const unsigned rowbase = sc - unsigned(xh);
    for (int hp = 2 * wave + h; hp < 16; hp += 2 * WPB) {
      const int mu = hp >> 2, k = hp & 3;
      const int d = k == 0 ? 1 : (k == 1 ? -1 : (k == 2 ? 3 : -3));
      nbt[(mu * 32 + si) * 4 + k] = hop_site(g, mu, d, sc, rowbase, x, y, z, t) * unsigned(sizeof(C));
    }
  }
  __syncthreads();
  C *row2 = reinterpret_cast<C *>(sl + PL * 32);
  if constexpr (R14) {
    for (int item = threadIdx.x; item < 8 * 32; item += 64 * WPB) {
      const int k = item >> 5, ln = item & 31;
      Lnk<Real> Lk;
      load_link<Real, LT, true, false>(sl, link_plane(8 + k, recon), 32u, ln, Lk);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        C v;
        v.x = Lk.re[2][b];
        v.y = Lk.im[2][b];
        row2[(k * 3 + b) * 32 + ln] = v;
      }
    }
    __syncthreads();
  }

  const unsigned plane_bytes = vh * unsigned(sizeof(C));
  for (int tile = wave; tile < a.ntiles; tile += WPB) {
    const int r0 = tile * 2 * RT;
    const int q0 = r0 + h * RT;  // this lane's first rhs
    bool act[RT];
    bool any = false;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      act[r] = q0 + r < a.n && (!a.active || a.active[q0 + r]);
      any = any || act[r];
    }
    if (!__builtin_amdgcn_ballot_w64(any)) continue;  // the whole tile is inactive (uniform)
    const char *in = static_cast<const char *>(a.in) + size_t(r0) * 3 * plane_bytes;
    // the rhs of the tile that exist: a lane's gathers past them are out of range
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(in), short(0), int(unsigned(min(2 * RT, a.n - r0)) * 3u * plane_bytes), kBufWord3);
    Real acc_re[RT][3], acc_im[RT][3];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc_re[r][c] = acc_im[r][c] = Real(0);
    const unsigned hoff = unsigned(h * RT * 3) * plane_bytes;
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      const uint4 nb = reinterpret_cast<const uint4 *>(nbt)[mu * 32 + si];
      Lnk<Real> Lk;
      load_link<Real, LT, false, false>(sl, link_plane(mu, recon), 32u, unsigned(si), Lk);
      apply_hop_buf32<Real, RT, false>(Lk, rs, plane_bytes, nb.x + hoff, acc_re, acc_im);
      load_link<Real, LT, false, false>(sl, link_plane(4 + mu, recon), 32u, unsigned(si), Lk);
      apply_hop_buf32<Real, RT, true>(Lk, rs, plane_bytes, nb.y + hoff, acc_re, acc_im);
      load_naik_lds<Real, LT, R14 ? 14 : 18, 32>(sl, row2, mu, si, Lk);
      apply_hop_buf32<Real, RT, false>(Lk, rs, plane_bytes, nb.z + hoff, acc_re, acc_im);
      load_naik_lds<Real, LT, R14 ? 14 : 18, 32>(sl, row2, 4 + mu, si, Lk);
      apply_hop_buf32<Real, RT, true>(Lk, rs, plane_bytes, nb.w + hoff, acc_re, acc_im);
    }
    C *__restrict__ out = static_cast<C *>(a.out) + size_t(r0) * 3 * vh;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      if (!(valid && act[r])) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        C o;
        o.x = acc_re[r][c];
        o.y = acc_im[r][c];
        out[(unsigned)((h * RT + r) * 3 + c) * vh + s] = o;
      }
    }
  }
}

// Direction-pipelined LDS form: the workgroup (64 sites x WPB waves) stages the links of one
// direction mu at a time -- X(x,mu), X(x-mu,mu)^dag, N(x,mu), N(x-3mu,mu)^dag -- in one of two
// LDS buffers.  While the waves apply direction mu to their rhs tiles, the links of mu+1 are
// already being loaded into registers, so link streaming overlaps the neighbour gathers and
// the FMAs, and a workgroup needs a quarter of the LDS of the whole-site form.  Each wave keeps
// the accumulators of TPW rhs tiles across the four directions (ntiles <= TPW * WPB).  Same hop
// order and FMA sequence per rhs as k_dslash, same per-64-site partials.
// (16 waves x 1 tile: at most 64 VGPRs, so that two workgroups share a CU)
template <typename Real, typename LT, int RT, bool R14, bool EPI, int WPB, int TPW, bool NT>
__global__ void __launch_bounds__(64 * WPB, (WPB == 16 && TPW == 1) ? 8 : 1) k_dslash_mu(Args a) {
  using C = typename CT<Real>::T;
  constexpr int recon = R14 ? 14 : 18;
  constexpr int NS = R14 ? 7 : 9;            // stored planes of a Naik hop
  constexpr int PM = 18 + 2 * NS;            // stored planes of one direction
  constexpr int NPF = (PM + WPB - 1) / WPB;  // planes each wave stages
  constexpr int BUF = PM * 64;               // link entries per buffer
  extern __shared__ __align__(16) unsigned char smem_raw[];
  LT *sl = reinterpret_cast<LT *>(smem_raw);          // two buffers of BUF entries
  C *row2 = reinterpret_cast<C *>(sl + 2 * BUF);      // 14-real Naik: two buffers of 2 x 3 x 64
  int sblk;
  if (!lds_block(a, sblk)) return;  // uniform for the whole workgroup
  const Geometry &g = a.g;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned vh = g.vh;
  const unsigned s = sblk * 64 + lane;
  const bool valid = s < vh;
  const LT *__restrict__ links = static_cast<const LT *>(a.links);

  LT pre[NPF];
  // issue the loads of direction mu's planes (local plane p -> stored plane)
  auto fetch = [&](int mu) {
#pragma unroll
    for (int i = 0; i < NPF; ++i) {
      const int p = wave + i * WPB;
      if (p < PM && valid) {
        int gp;
        if (p < 9) gp = link_plane(mu, recon) + p;
        else if (p < 18) gp = link_plane(4 + mu, recon) + p - 9;
        else if (p < 18 + NS) gp = link_plane(8 + mu, recon) + p - 18;
        else gp = link_plane(12 + mu, recon) + p - 18 - NS;
        pre[i] = ld_raw<NT>(links + size_t(gp) * vh + s);
      }
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NPF; ++i) {
      const int p = wave + i * WPB;
      if (p < PM && valid) sl[buf * BUF + p * 64 + lane] = pre[i];
    }
  };
  // 14-real Naik: row 2 of the two Naik hops of the buffer, once per site
  auto rebuild = [&](int buf) {
    if constexpr (R14) {
      for (int item = threadIdx.x; item < 2 * 64; item += 64 * WPB) {
        const int k = item >> 6, ln = item & 63;
        Lnk<Real> Lk;
        load_link<Real, LT, true, false>(sl + buf * BUF, 18 + k * NS, 64u, ln, Lk);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          C v;
          v.x = Lk.re[2][b];
          v.y = Lk.im[2][b];
          row2[(buf * 6 + k * 3 + b) * 64 + ln] = v;
        }
      }
      __syncthreads();
    }
  };

  // every lane computes: a lane past the last site works on site 0 and stores nothing
  const unsigned sc = valid ? s : 0u;
  int x, y, z, t;
  {
    const int xh = sc % g.lxh;
    int rest = sc / g.lxh;
    y = rest % g.ly;
    rest /= g.ly;
    z = rest % g.lz;
    t = rest / g.lz;
    x = 2 * xh + ((y + z + t + a.out_parity) & 1);
  }
  const unsigned rowbase = sc - (x >> 1);

  int rr[TPW][RT];
  bool ract[TPW][RT], tact[TPW];
  Real acc_re[TPW][RT][3], acc_im[TPW][RT][3];
#pragma unroll
  for (int tw = 0; tw < TPW; ++tw) {
    const int tile = wave + tw * WPB;
    tact[tw] = tile < a.ntiles && tile_rhs<RT>(a, tile * RT, rr[tw], ract[tw]);
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc_re[tw][r][c] = acc_im[tw][r][c] = Real(0);
  }

  fetch(0);
  stash(0);
  __syncthreads();
  rebuild(0);
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    const int buf = mu & 1;
    if (mu < 3) fetch(mu + 1);
    unsigned f1, b1, f3, b3;
    hop_sites(g, mu, sc, rowbase, x, y, z, t, f1, b1, f3, b3);
    const LT *bl = sl + buf * BUF;
#pragma unroll
    for (int tw = 0; tw < TPW; ++tw) {
      if (!tact[tw]) continue;  // uniform
      const C *__restrict__ in = static_cast<const C *>(a.in) + size_t((wave + tw * WPB) * RT) * 3 * vh;
      Lnk<Real> Lk;
      load_link<Real, LT, false, false>(bl, 0, 64u, lane, Lk);
      apply_hop_all<Real, RT, false>(Lk, in, vh, f1, rr[tw], acc_re[tw], acc_im[tw]);
      load_link<Real, LT, false, false>(bl, 9, 64u, lane, Lk);
      apply_hop_all<Real, RT, true>(Lk, in, vh, b1, rr[tw], acc_re[tw], acc_im[tw]);
      if constexpr (!R14) {
        load_link<Real, LT, false, false>(bl, 18, 64u, lane, Lk);
      } else {
#pragma unroll
        for (int ra = 0; ra < 2; ++ra)
#pragma unroll
          for (int cb = 0; cb < 3; ++cb) ld_link<false>(bl + (18 + ra * 3 + cb) * 64 + lane, Lk.re[ra][cb], Lk.im[ra][cb]);
#pragma unroll
        for (int cb = 0; cb < 3; ++cb) {
          const C v = row2[(buf * 6 + cb) * 64 + lane];
          Lk.re[2][cb] = v.x;
          Lk.im[2][cb] = v.y;
        }
      }
      apply_hop_all<Real, RT, false>(Lk, in, vh, f3, rr[tw], acc_re[tw], acc_im[tw]);
      if constexpr (!R14) {
        load_link<Real, LT, false, false>(bl, 27, 64u, lane, Lk);
      } else {
#pragma unroll
        for (int ra = 0; ra < 2; ++ra)
#pragma unroll
          for (int cb = 0; cb < 3; ++cb)
            ld_link<false>(bl + (18 + NS + ra * 3 + cb) * 64 + lane, Lk.re[ra][cb], Lk.im[ra][cb]);
#pragma unroll
        for (int cb = 0; cb < 3; ++cb) {
          const C v = row2[(buf * 6 + 3 + cb) * 64 + lane];
          Lk.re[2][cb] = v.x;
          Lk.im[2][cb] = v.y;
        }
      }
      apply_hop_all<Real, RT, true>(Lk, in, vh, b3, rr[tw], acc_re[tw], acc_im[tw]);
    }
    if (mu < 3) {
      stash(buf ^ 1);
      __syncthreads();
      rebuild(buf ^ 1);
    }
  }
#pragma unroll
  for (int tw = 0; tw < TPW; ++tw) {
    const int tile = wave + tw * WPB;
    if (tile >= a.ntiles) continue;
    const int r0 = tile * RT;
    if (!tact[tw]) {  // inactive tile: zero partials, nothing stored
      if constexpr (EPI) {
        if (a.partial && lane == 0) {
          const unsigned nw = (vh + 63) / 64;
#pragma unroll
          for (int r = 0; r < RT; ++r)
            if (r0 + r < a.n) a.partial[size_t(r0 + r) * nw + sblk] = 0.0;
        }
      }
      continue;
    }
    bool act[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) act[r] = valid && ract[tw][r];
    store_tile<Real, RT, EPI>(a, r0, s, lane, sblk, act, acc_re[tw], acc_im[tw]);
  }
}

// Row form up to this many workgroups (64-site blocks times rhs), the number that is resident at two
// per CU in FP64, twice that for the smaller links.  FP64: 512 (16^4, 1 rhs) 13.4 us against 14.5 with
// k_dslash, fused 14.2 against 15.2; 1024 (2 rhs) fused slower than its 16.6, and the LDS forms are
// ahead from 648 (12^4, 4 rhs: 9.0 against 9.3).  FP32: 1024 (16^4, 2 rhs) 9.6 against 11.3 of the LDS
// forms, FP16 links 7.6 against 9.1; 1296 (12^4, 8 rhs) 12.3 against 9.4, 9.0 against 8.6.
template <typename Real> constexpr int kRowsMaxBlocks = sizeof(Real) == 8 ? 512 : 1024;

using DslashFn = void (*)(const Args &, dim3, hipStream_t);

template <typename Real, typename LT, int RT, int NR, bool EPI, int SPB, bool NT>
void launch_t(const Args &a, dim3 grid, hipStream_t st) {
  if constexpr (RT == 1 && NR == 18 && SPB == 64) {
    if (a.nsblk * a.ntiles <= kRowsMaxBlocks<Real>) {
      k_dslash_rows<Real, LT, EPI, NT><<<(a.nsblk * a.ntiles + 7) / 8 * 8, 192, 0, st>>>(a);
      return;
    }
  }
  k_dslash<Real, LT, RT, NR, EPI, SPB, NT><<<grid, 256, 0, st>>>(a);
}

// Whether the pair form runs a whole-site LDS launch (elem: bytes of a stored link entry, 16, 8 or 4;
// nr: reals of a Naik link; rt rhs per thread; wpb waves; ntiles rhs tiles; nsblk 64-site blocks), or the
// one-site form.  The pair form looks ahead where the one-site form has more waves in flight, so it
// pays where its waves have work; a configuration that is forced or was stored for the one-site form
// must not lose by it elsewhere.  Measured on 1520 launches (8 lattices of 256 to 10368 blocks, 2 to 32
// rhs, all formats), one-site time over pair time, geometric mean and range, where the rule takes
// the pair form | where it does not:
//   FP64         1.14 (1.01-1.43), 8 waves 1.10 (0.98-1.32) | one rhs in 8 waves on few blocks 0.97 (0.84-1.07)
//   FP32  4 waves 1.16 (0.92-1.55) | 0.95 (0.81-1.02): one tile, or r14 and r13 plain on small lattices
//         8 waves 1.11 (0.78-1.58) | 0.94 (0.70-1.25): idle waves, the 9-real format that reads its
//                                    rebuilt links from LDS in full
//        16 waves 1.08 (0.98-1.22) | 0.86 (0.65-1.09): idle waves
//   FP16  4 waves 1.10 (0.94-1.25) | 1.01 (0.86-1.26): one tile, 9 reals, four rhs on two tiles
//         8 waves 1.10 (0.93-1.55) | 0.92 (0.67-1.26): idle waves, formats that rebuild, four rhs
//        16 waves 1.07 (0.92-1.21) | 0.79 (0.61-0.98): idle waves
// With at most one workgroup per CU the one-site form has no further waves to offer.  (The 0.78 is 16^4
// with 32 rhs in FP32; the fastest launch of each of the 266 cases stays within 2 % of both forms' best.)
constexpr int kCUs = 256;
__host__ __device__ constexpr bool pair_form_pays(int elem, int nr, int rt, int wpb, bool epi, int ntiles, int nsblk) {
  if (elem == 16) return rt <= 2 && !(rt == 1 && wpb == 8 && nsblk < 3 * kCUs);
  if (rt < 2) return false;
  const bool f16 = elem == 4;
  if (wpb == 4) {
    if (rt > 2) return !f16 || ntiles >= 3 || nsblk <= kCUs;
    if (f16 && nr == 9) return false;
    if (!f16 && (nr == 14 || nr == 13) && !epi && nsblk < 6 * kCUs) return false;
    return ntiles >= 2;
  }
  if (wpb == 8) {
    const bool every = nr == 9 || (f16 && (rt > 2 || nr != 18));  // needs a tile for every wave
    return ntiles >= (every ? 8 : (rt > 2 ? 2 : 3)) || (rt > 2 && nsblk <= kCUs);
  }
  return ntiles >= 16 || nsblk <= kCUs;
}

template <typename Real, typename LT, int RT, int NR, bool EPI, int WPB, bool NT>
void launch_lds(const Args &a, dim3 grid, hipStream_t st) {
  constexpr bool f64 = sizeof(Real) == 8;
  if constexpr (f64 ? RT <= 2 : RT >= 2 && !(sizeof(LT) == 4 && NR == 9 && RT == 2 && WPB == 4)) {
    if ((f64 || a.g.lx % 4 == 0) && pair_form_pays(sizeof(LT), NR, RT, WPB, EPI, a.ntiles, a.nsblk)) {
      k_dslash_pair<Real, LT, f64 ? RT : RT / 2, NR, EPI, WPB, NT>
          <<<grid, 64 * WPB, lds_nbr_offset<Real, LT, NR>() + nbr_table_pair_bytes<Real>(), st>>>(a);
      return;
    }
  }
  if constexpr (!f64 || RT > 2 || (RT == 1 && WPB == 8)) {
    constexpr size_t lds = lds_nbr_offset<Real, LT, NR>() + kNbrTableBytes;
    k_dslash_lds<Real, LT, RT, NR, EPI, WPB, NT><<<grid, 64 * WPB, lds, st>>>(a);
  }
}

template <typename Real, typename LT, int RT, bool R14, bool EPI, int WPB, int TPW, bool NT>
void launch_mu(const Args &a, dim3 grid, hipStream_t st) {
  constexpr size_t lds = 2 * size_t(R14 ? 32 : 36) * 64 * sizeof(LT) +
                         (R14 ? size_t(12) * 64 * sizeof(typename CT<Real>::T) : 0);
  k_dslash_mu<Real, LT, RT, R14, EPI, WPB, TPW, NT><<<grid, 64 * WPB, lds, st>>>(a);
}

// direction-pipelined forms: 4 = 16 waves x 1 tile each, 5 = 16 waves x 2 tiles, 6 = 8 waves x 2
template <typename Real, typename LT, bool R14, bool EPI, bool NT>
DslashFn pick_mu(int rt, int lds) {
  if (rt == 1) {
    if (lds == 4) return launch_mu<Real, LT, 1, R14, EPI, 16, 1, NT>;
    if (lds == 5) return launch_mu<Real, LT, 1, R14, EPI, 16, 2, NT>;
    if (lds == 6) return launch_mu<Real, LT, 1, R14, EPI, 8, 2, NT>;
  } else if (rt == 2) {
    if (lds == 4) return launch_mu<Real, LT, 2, R14, EPI, 16, 1, NT>;
    if (lds == 5) return launch_mu<Real, LT, 2, R14, EPI, 16, 2, NT>;
    if (lds == 6) return launch_mu<Real, LT, 2, R14, EPI, 8, 2, NT>;
  }
  return nullptr;
}

template <typename Real, typename LT, int NR, bool EPI, int WPB, bool NT>
DslashFn pick_lds_rt(int rt) {
  switch (rt) {
    case 1: return launch_lds<Real, LT, 1, NR, EPI, WPB, NT>;
    case 2: return launch_lds<Real, LT, 2, NR, EPI, WPB, NT>;
    case 4:
      if constexpr (WPB <= 8) return launch_lds<Real, LT, 4, NR, EPI, WPB, NT>;
      return nullptr;
    default: return nullptr;
  }
}

template <typename Real, typename LT, int RT, bool R14, int WPB, bool NT>
void launch_lds32(const Args &a, dim3 grid, hipStream_t st) {
  constexpr size_t lds = lds32_nbr_offset<Real, LT, R14>() + kNbrTable32Bytes;
  k_dslash_lds32<Real, LT, RT, R14, WPB, NT><<<grid, 64 * WPB, lds, st>>>(a);
}

// 32-site form: lds 1 = 4 waves, 2 = 8 waves; rhs_per_thread 1 or 2; plain half Dslash only
template <typename Real, typename LT, bool R14, bool NT>
DslashFn pick_lds32(int rt, int lds) {
  if (lds == 1) return rt == 1 ? launch_lds32<Real, LT, 1, R14, 4, NT> : (rt == 2 ? launch_lds32<Real, LT, 2, R14, 4, NT> : nullptr);
  if (lds == 2) return rt == 1 ? launch_lds32<Real, LT, 1, R14, 8, NT> : (rt == 2 ? launch_lds32<Real, LT, 2, R14, 8, NT> : nullptr);
  return nullptr;
}

// lds: 1 = 4 waves per 64-site workgroup, 2 = 8 waves, 3 = 16 waves; 4-6 the direction-pipelined
// forms (Naik formats 18 and 14 only)
template <typename Real, typename LT, int NR, bool EPI, bool NT>
DslashFn pick_lds(int rt, int lds) {
  if constexpr (sizeof(LT) > 8) {  // FP64: the whole-site forms only (one workgroup per CU)
    if (lds == 1) return pick_lds_rt<Real, LT, NR, EPI, 4, NT>(rt);
    if (lds == 2) return pick_lds_rt<Real, LT, NR, EPI, 8, NT>(rt);
    if (lds == 3) return pick_lds_rt<Real, LT, NR, EPI, 16, NT>(rt);
    return nullptr;
  } else {
    if (lds >= 4) {
      if constexpr (NR == 18 || NR == 14) return pick_mu<Real, LT, NR == 14, EPI, NT>(rt, lds);
      return nullptr;
    }
    if (lds == 1) return pick_lds_rt<Real, LT, NR, EPI, 4, NT>(rt);
    if (lds == 2) return pick_lds_rt<Real, LT, NR, EPI, 8, NT>(rt);
    if (lds == 3) return pick_lds_rt<Real, LT, NR, EPI, 16, NT>(rt);
    return nullptr;
  }
}

template <typename Real, typename LT, int NR, bool EPI, int SPB, bool NT>
DslashFn pick_rt(int rt) {
  switch (rt) {
    case 1: return launch_t<Real, LT, 1, NR, EPI, SPB, NT>;
    case 2: return launch_t<Real, LT, 2, NR, EPI, SPB, NT>;
    case 4: return launch_t<Real, LT, 4, NR, EPI, SPB, NT>;
    case 8: return launch_t<Real, LT, 8, NR, EPI, SPB, NT>;
    default:
      if constexpr (!EPI && sizeof(Real) == 4) return launch_t<Real, LT, 16, NR, EPI, SPB, NT>;
      return nullptr;
  }
}

// Every form for Naik storage format NR (the 32-site and direction-pipelined forms: 18 and 14).
template <typename Real, typename LT, int NR>
DslashFn pick_all(bool epi, int rt, int spb, bool nt, int lds) {
  if (lds) {
    if (spb == 32) {
      if constexpr (NR == 18 || NR == 14)
        return epi ? nullptr : (nt ? pick_lds32<Real, LT, NR == 14, true>(rt, lds) : pick_lds32<Real, LT, NR == 14, false>(rt, lds));
      return nullptr;
    }
    if (spb != 64) return nullptr;
    if (nt) return epi ? pick_lds<Real, LT, NR, true, true>(rt, lds) : pick_lds<Real, LT, NR, false, true>(rt, lds);
    return epi ? pick_lds<Real, LT, NR, true, false>(rt, lds) : pick_lds<Real, LT, NR, false, false>(rt, lds);
  }
  if (spb != 64 && spb != 256) return nullptr;
  if (epi) {
    if (spb == 64) return nt ? pick_rt<Real, LT, NR, true, 64, true>(rt) : pick_rt<Real, LT, NR, true, 64, false>(rt);
    return nt ? pick_rt<Real, LT, NR, true, 256, true>(rt) : pick_rt<Real, LT, NR, true, 256, false>(rt);
  }
  if (spb == 64) return nt ? pick_rt<Real, LT, NR, false, 64, true>(rt) : pick_rt<Real, LT, NR, false, 64, false>(rt);
  return nt ? pick_rt<Real, LT, NR, false, 256, true>(rt) : pick_rt<Real, LT, NR, false, 256, false>(rt);
}

}  // namespace dslash

// per-precision tables (dslash_f64.hip, dslash_f32.hip, dslash_f16.hip)
dslash::DslashFn dslash_fn_f64(bool epi, int rt, int spb, bool nt, int lds);
dslash::DslashFn dslash_fn_f32(bool epi, int recon, int rt, int spb, bool nt, int lds);
dslash::DslashFn dslash_fn_f16(bool epi, int recon, int rt, int spb, bool nt, int lds);
