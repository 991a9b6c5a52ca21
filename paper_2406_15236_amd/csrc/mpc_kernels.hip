// mpc_kernels.hip -- gfx950 kernels of the MPC-SRD step (arXiv:2406.15236, Sec. II).
//
// Cells are grouped into tiles (runs of at most 32 cells of one row).  A state
// buffer holds the particles of a tile's collision of the previous step next
// to each other, grouped by the tile that they reach in the next step, and
// every tile has a list of those runs (first slot, count).
//
// One step t on the device (steady state):
//   prefix  : position of every tile's output, the prefix of the particles per
//             tile (a launch of its own for more than kTileDirect tiles only)
//   collide : per tile: gather its runs, stream (Eq. 1), order by cell and
//             logical index in LDS, sum the cells, rotate (Eq. 2) + scale with
//             the draws, stream + bin for step t+1, write the state into the
//             other buffer grouped by next-step tile and append one run per
//             such tile to its list; beside that, the random draws, phantom
//             particles and lattice shifts of step t + 1, which depend on the
//             step index only
// and after the last of n steps
//   advance : t += n, and the buffers in turn.
// When the state was set from outside, its tiling changed or its binning was
// exported, a counting sort by tile puts it in this order first.  Every kernel reads the step index and buffer from Ctrl and adds
// the number j of its step in the launch sequence, so that a captured graph of
// steps can be replayed.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "mpc_internal.h"
#include "philox_dev.h"
#include "sample_table.h"

namespace mpc {

// Box parameters and tile/control tables are read-only while a kernel runs.
// Reading them through the constant address space lets the compiler use
// scalar loads that later global stores cannot clobber (otherwise every use
// after a store becomes a per-lane reload from memory).
#define MPC_AS4 __attribute__((address_space(4)))
using BoxRef = const MPC_AS4 BoxDev&;
template <typename T>
__device__ __forceinline__ const MPC_AS4 T* as_const(const T* p) {
  return (const MPC_AS4 T*)p;
}
__device__ __forceinline__ Tile load_tile(const Tile* p, uint32_t i) {
  const MPC_AS4 Tile& r = as_const(p)[i];
  Tile t;
  t.c0 = r.c0;
  t.nc = r.nc;
  t.box = r.box;
  t.tid = r.tid;
  t.x0 = r.x0;
  t.y0 = r.y0;
  t.z0 = r.z0;
  return t;
}
__device__ __forceinline__ PBlock load_pblock(const PBlock* p, uint32_t i) {
  const MPC_AS4 PBlock& r = as_const(p)[i];
  PBlock b;
  b.box = r.box;
  b.p0 = r.p0;
  return b;
}

// ---------------------------------------------------------------------------
// Random draws of the method
// ---------------------------------------------------------------------------
// Angles here are at most 2 pi.  Told so, the compiler drops the reduction of
// huge arguments from sin and cos (the limit is that of their short branch),
// which set the register count of the collide with the thermostat and of the
// draws (109 instead of 81 VGPRs in a kernel of their own).
constexpr double kSmallAngle = 0x1p30;

__device__ __forceinline__ Words4 draw(BoxRef B, uint32_t j, uint32_t id, uint64_t t,
                                       uint32_t tag) {
  return philox10(j, id, (uint32_t)t, tag, B.key_lo, B.key_hi);
}

// Lattice shift of step t: s_k = u24(w_k) - 1/2 (exact 2^-24 grid).
__device__ __forceinline__ void shift_of(BoxRef B, uint64_t t, double s[3]) {
  const Words4 w = draw(B, 0, 0, t, kTagShift);
  s[0] = u24_of(w.w[0]) - 0.5;
  s[1] = u24_of(w.w[1]) - 0.5;
  s[2] = u24_of(w.w[2]) - 0.5;
}

// Uniform random axis on the unit sphere: z = 1 - 2 u1, phi = 2 pi u2.
__device__ __forceinline__ void axis_of(BoxRef B, uint64_t t, uint32_t key, double n[3]) {
  const Words4 w = draw(B, 0, key, t, kTagAxis);
  const double u1 = u53_of(w.w[0], w.w[1]);
  const double u2 = u53_of(w.w[2], w.w[3]);
  const double z = 1.0 - 2.0 * u1;
  const double r = sqrt(1.0 - z * z);
  const double phi = kTwoPi * u2;
  double sp, cp;
  __builtin_assume(__builtin_fabs(phi) < kSmallAngle);
  sincos(phi, &sp, &cp);
  n[0] = r * cp;
  n[1] = r * sp;
  n[2] = z;
}

// Attempt j of the gamma draw: the normal z (Box-Muller cosine branch of
// THERMO draw j, words 0 and 1) and log of the acceptance uniform (words 2
// and 3).  Neither depends on the shape.
__device__ __forceinline__ void gamma_attempt(uint32_t key_lo, uint32_t key_hi, uint64_t t,
                                              uint32_t key, uint32_t j, double& z, double& lu) {
  const Words4 w = philox10(j, key, (uint32_t)t, kTagThermo, key_lo, key_hi);
  const double u1 = u32_open_of(w.w[0]);
  const double u2 = (double)w.w[1] * 0x1p-32;
  const double ph = kTwoPi * u2;
  __builtin_assume(__builtin_fabs(ph) < kSmallAngle);
  z = sqrt(-2.0 * log(u1)) * cos(ph);
  lu = log(u53_open_of(w.w[2], w.w[3]));
}

// Gamma(shape, 1) by Marsaglia-Tsang with shape 3 (n - 1) / 2 for the n
// particles of a cell: d v for an accepted attempt, else -1.
struct GammaDC {
  double d, c;
};
__device__ __forceinline__ GammaDC gamma_dc(uint32_t n) {
  const double d = 1.5 * (double)(n - 1) - 1.0 / 3.0;
  return {d, 1.0 / sqrt(9.0 * d)};
}
__device__ __forceinline__ bool gamma_accepts(uint32_t n, double z, double lu) {
  const GammaDC g = gamma_dc(n);
  double vv = 1.0 + g.c * z;
  if (vv <= 0.0) return false;
  vv = vv * vv * vv;
  const double rhs = 0.5 * z * z + g.d - g.d * vv + g.d * log(vv);
  return lu < rhs;
}
// Smallest n that accepts attempt (z, lu), kNeverAccepted if that is more than
// a cell can hold.  The acceptance bound rises with n: with y = c z it is
// (z^2 / 9) N(y) / y^2, N(y) = 3 (log(1 + y) - y + y^2 / 2 - y^3 / 3) =
// -3 int_0^y s^3 / (1 + s) ds, and N(y) / y^2 rises to 0 as |y| falls.  So an
// attempt accepted for n is accepted for every larger n.  The search starts
// where the leading term of the bound, -z^4 / (108 d), crosses lu.
__device__ __forceinline__ uint32_t gamma_least(double z, double lu) {
  const double ds = z * z * z * z / (-108.0 * lu);
  uint32_t n = (uint32_t)fmin(2.0 + ds * (2.0 / 3.0), (double)kNeverAccepted);
  if (n < kNeverAccepted && gamma_accepts(n, z, lu)) {
#pragma unroll 1
    while (n > 2u && gamma_accepts(n - 1u, z, lu)) --n;
  } else {
#pragma unroll 1
    while (n < kNeverAccepted && !gamma_accepts(n + 1u, z, lu)) ++n;
    n = min(n + 1u, kNeverAccepted);
  }
  return n;
}

// Phantom particles of a wall-cut cell: Poisson(<N_c> f_w) count by inversion
// on draw 0, truncated at 127.
__device__ __forceinline__ int phantom_count(BoxRef B, uint64_t t, uint32_t key, double fw) {
  const double lam = B.density * fw;
  const Words4 w = draw(B, 0, key, t, kTagPhantom);
  const double u = u53_of(w.w[0], w.w[1]);
  int k = 0;
  double pk = exp(-lam);
  double F = pk;
#pragma unroll 1
  while (u >= F && k < 127) {
    k += 1;
    pk = pk * lam / (double)k;
    F = F + pk;
  }
  return k;
}

// Normal number m of a cell's phantom stream (draw 1 + m/4; Box-Muller pair
// (m%4)/2; cosine for even m, sine for odd m).  `cache` keeps the last draw.
struct PhantomCache {
  uint32_t j;
  Words4 w;
};
__device__ __forceinline__ double phantom_normal(BoxRef B, uint64_t t, uint32_t key,
                                                 uint32_t m, PhantomCache& pc) {
  const uint32_t j = 1 + m / 4;
  if (pc.j != j) {
    pc.w = draw(B, j, key, t, kTagPhantom);
    pc.j = j;
  }
  const uint32_t pr = (m % 4) / 2;
  const double r = sqrt(-2.0 * log(u32_open_of(pc.w.w[2 * pr])));
  const double th = kTwoPi * ((double)pc.w.w[2 * pr + 1] * 0x1p-32);
  __builtin_assume(__builtin_fabs(th) < kSmallAngle);
  return (m % 2 == 0) ? r * cos(th) : r * sin(th);
}

// Wall volume fraction of shifted z layer cz (layer spans [cz - sz, cz + 1 - sz)).
__device__ __forceinline__ double wall_fraction(double sz, int cz, int H) {
  if (sz >= 0.0) {
    if (cz == 0) return sz;
    if (cz == H) return 1.0 - sz;
  } else {
    if (cz == -1) return 1.0 + sz;
    if (cz == H - 1) return -sz;
  }
  return 0.0;
}

// ---------------------------------------------------------------------------
// Storage forms
// ---------------------------------------------------------------------------
// Periodic wrap into [0, L): one image shift (selects), then the rare cases
// (rounding onto L, far outside, non-finite) on a cold path.
__device__ __forceinline__ double wrap64_rare(double x, double L) {
  if (x == L) return 0.0;
  if (isfinite(x)) {
    x = x - L * floor(x / L);
    if (x >= L || x < 0.0) x = 0.0;
  }
  return x;
}
__device__ __forceinline__ double wrap64(double x, double L) {
  const double lo = x + L, hi = x - L;
  x = x < 0.0 ? lo : (x >= L ? hi : x);
  if (__builtin_expect(!(x >= 0.0 && x < L), 0)) x = wrap64_rare(x, L);
  return x;
}

__device__ __forceinline__ float wrap32_rare(float x, float L) {
  if (x == L) return 0.0f;
  if (isfinite(x)) {
    x = x - L * floorf(x / L);
    if (x >= L || x < 0.0f) x = 0.0f;
  }
  return x;
}
__device__ __forceinline__ float wrap32(float x, float L) {
  const float lo = x + L, hi = x - L;
  x = x < 0.0f ? lo : (x >= L ? hi : x);
  if (__builtin_expect(!(x >= 0.0f && x < L), 0)) x = wrap32_rare(x, L);
  return x;
}

// Whether x may lie outside [0, L), from the high words: a negative x, a NaN
// and an infinity have larger ones than any L, and so has x >= L (for x < L
// they can be equal only if L > 2^21).  Of a wavefront's particles most stay
// inside, and then one 32-bit comparison per axis stands for the wraps (ten
// instructions each) and for the range checks of the cell coordinates.
__device__ __forceinline__ bool maybe_outside(double x, double L) {
  return (uint32_t)((uint64_t)__double_as_longlong(x) >> 32) >=
         (uint32_t)((uint64_t)__double_as_longlong(L) >> 32);
}
__device__ __forceinline__ bool maybe_outside(float x, float L) {
  return __float_as_uint(x) >= __float_as_uint(L);
}

// Lees-Edwards shear of a periodic box (Sec. II, boundary conditions): at
// time tau = t_end h the image above the box (z + L_z) is displaced by
// d = (U tau) mod L_x along x and moves with U.  A particle through a z face
// re-enters displaced by -/+ d with v_x -/+ U; a collision cell across a z
// face is formed with the image on the other side, in that image's frame.
__device__ __forceinline__ double le_offset(BoxRef B, uint64_t t_end) {
  const double d = B.leu * ((double)t_end * B.h);
  return d - B.Ld[0] * floor(d / B.Ld[0]);
}

// Eq.(1) in FP64 with periodic x, y and (walls) time-reversed bounce-back in z;
// dle: Lees-Edwards offset at the end of this streaming.
template <bool W>
__device__ __forceinline__ void stream_f64(double (&x)[3], double (&v)[3], BoxRef B,
                                           double dle, bool le) {
  double xe = fma(B.h, v[0], x[0]);
  double ye = fma(B.h, v[1], x[1]);
  double ze = fma(B.h, v[2], x[2]);
  if (W) {
    const double H = B.Ld[2];
    const bool lo = ze < 0.0, hi = ze > H;
    if (lo || hi) {
      const double zw = lo ? 0.0 : H;
      const double tr2 = 2.0 * ((ze - zw) / v[2]);
      if (B.slip) {  // specular reflection
        ze = ze - tr2 * v[2];
      } else {       // bounce-back in the frame of the (moving) wall
        const double uw = lo ? -B.uw : B.uw;
        xe = xe - tr2 * (v[0] - uw);
        ye = ye - tr2 * v[1];
        ze = ze - tr2 * v[2];
        v[0] = 2.0 * uw - v[0];
        v[1] = -v[1];
      }
      if (ze < 0.0) ze = 0.0;
      if (ze > H) ze = H;
      v[2] = -v[2];
    }
  } else {
    if (le && (ze >= B.Ld[2] || ze < 0.0)) {
      if (ze >= B.Ld[2]) {
        xe = xe - dle;
        v[0] = v[0] - B.leu;
      } else {
        xe = xe + dle;
        v[0] = v[0] + B.leu;
      }
    }
  }
  if (maybe_outside(xe, B.Ld[0]) || maybe_outside(ye, B.Ld[1]) ||
      (!W && maybe_outside(ze, B.Ld[2]))) {
    xe = wrap64(xe, B.Ld[0]);
    ye = wrap64(ye, B.Ld[1]);
    if (!W) ze = wrap64(ze, B.Ld[2]);
  }
  x[0] = xe;
  x[1] = ye;
  x[2] = ze;
}

template <bool W>
__device__ __forceinline__ void stream_f32(float (&x)[3], float (&v)[3], BoxRef B, double dle,
                                           bool le) {
  float xe = fmaf(B.hf, v[0], x[0]);
  float ye = fmaf(B.hf, v[1], x[1]);
  float ze = fmaf(B.hf, v[2], x[2]);
  if (W) {
    const float H = B.Lf[2];
    const bool lo = ze < 0.0f, hi = ze > H;
    if (lo || hi) {
      const float zw = lo ? 0.0f : H;
      const float tr2 = 2.0f * ((ze - zw) / v[2]);
      if (B.slip) {
        ze = ze - tr2 * v[2];
      } else {
        const float uw = lo ? -B.uwf : B.uwf;
        xe = xe - tr2 * (v[0] - uw);
        ye = ye - tr2 * v[1];
        ze = ze - tr2 * v[2];
        v[0] = 2.0f * uw - v[0];
        v[1] = -v[1];
      }
      if (ze < 0.0f) ze = 0.0f;
      if (ze > H) ze = H;
      v[2] = -v[2];
    }
  } else {
    if (le && (ze >= B.Lf[2] || ze < 0.0f)) {
      if (ze >= B.Lf[2]) {
        xe = xe - (float)dle;
        v[0] = v[0] - B.leuf;
      } else {
        xe = xe + (float)dle;
        v[0] = v[0] + B.leuf;
      }
    }
  }
  if (maybe_outside(xe, B.Lf[0]) || maybe_outside(ye, B.Lf[1]) ||
      (!W && maybe_outside(ze, B.Lf[2]))) {
    xe = wrap32(xe, B.Lf[0]);
    ye = wrap32(ye, B.Lf[1]);
    if (!W) ze = wrap32(ze, B.Lf[2]);
  }
  x[0] = xe;
  x[1] = ye;
  x[2] = ze;
}

// Split form: unshifted cell (packed) + offset in [0, 1) per axis.
__device__ __forceinline__ void split_decode(uint32_t cell, int (&c)[3]) {
  c[0] = (int)(cell & ((1u << kSplitXBits) - 1));
  c[1] = (int)((cell >> kSplitXBits) & ((1u << kSplitYBits) - 1));
  c[2] = (int)(cell >> (kSplitXBits + kSplitYBits));
}
__device__ __forceinline__ uint32_t split_encode(const int (&c)[3]) {
  return (uint32_t)c[0] | ((uint32_t)c[1] << kSplitXBits) |
         ((uint32_t)c[2] << (kSplitXBits + kSplitYBits));
}
__device__ __forceinline__ int wrap_cell_rare(int c, int L) { return ((c % L) + L) % L; }
__device__ __forceinline__ int wrap_cell(int c, int L) {
  c = c < 0 ? c + L : (c >= L ? c - L : c);
  if (__builtin_expect(c < 0 || c >= L, 0)) c = wrap_cell_rare(c, L);
  return c;
}
// FP64 value -> (cell, offset) with the offset rounded to FP32.
__device__ __forceinline__ void split_from_double(double xd, int& c, float& o) {
  const double fl = floor(xd);
  c = (int)fl;
  o = (float)(xd - fl);
  if (o >= 1.0f) {
    o = 0.0f;
    c += 1;
  }
}

template <bool W>
__device__ __forceinline__ void stream_split(uint32_t& cell, float (&o)[3], float (&v)[3],
                                             BoxRef B, double dle, bool le) {
  int c[3];
  split_decode(cell, c);
  int cn[3];
  float on[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float y = fmaf(B.hf, v[k], o[k]);
    float fl = floorf(y);
    y = y - fl;
    if (y == 1.0f) {
      y = 0.0f;
      fl += 1.0f;
    }
    on[k] = y;
    cn[k] = c[k] + (int)fl;
  }
  if (W) {
    const int H = B.L[2];
    const bool out = cn[2] < 0 || cn[2] > H || (cn[2] == H && on[2] > 0.0f) ||
                     !isfinite(on[2]);
    if (out) {
      // crossing particle: the bounce is done in FP64 from the exact position
      double xd[3], vd[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        xd[k] = (double)c[k] + (double)o[k];
        vd[k] = (double)v[k];
      }
      double xe[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) xe[k] = fma(B.h, vd[k], xd[k]);
      const double Hd = B.Ld[2];
      if (xe[2] < 0.0 || xe[2] > Hd) {
        const bool lo = xe[2] < 0.0;
        const double zw = lo ? 0.0 : Hd;
        const double tr2 = 2.0 * ((xe[2] - zw) / vd[2]);
        if (B.slip) {
          xe[2] = xe[2] - tr2 * vd[2];
        } else {
          const double uw = lo ? -B.uw : B.uw;
          xe[0] = xe[0] - tr2 * (vd[0] - uw);
          xe[1] = xe[1] - tr2 * vd[1];
          xe[2] = xe[2] - tr2 * vd[2];
          v[0] = (float)(2.0 * uw - vd[0]);
          v[1] = -v[1];
        }
        if (xe[2] < 0.0) xe[2] = 0.0;
        if (xe[2] > Hd) xe[2] = Hd;
        v[2] = -v[2];
      }
      xe[0] = wrap64(xe[0], B.Ld[0]);
      xe[1] = wrap64(xe[1], B.Ld[1]);
#pragma unroll
      for (int k = 0; k < 3; ++k) split_from_double(xe[k], cn[k], on[k]);
    }
  } else {
    if (le && (cn[2] >= B.L[2] || cn[2] < 0)) {
      // through a sheared face: x -/+ d in FP64, v_x -/+ U
      const bool up = cn[2] >= B.L[2];
      double xd = (double)cn[0] + (double)on[0];
      xd = wrap64(up ? xd - dle : xd + dle, B.Ld[0]);
      split_from_double(xd, cn[0], on[0]);
      v[0] = (float)(up ? (double)v[0] - B.leu : (double)v[0] + B.leu);
    }
  }
  if ((unsigned)cn[0] >= (unsigned)B.L[0] || (unsigned)cn[1] >= (unsigned)B.L[1] ||
      (!W && (unsigned)cn[2] >= (unsigned)B.L[2])) {
    cn[0] = wrap_cell(cn[0], B.L[0]);
    cn[1] = wrap_cell(cn[1], B.L[1]);
    if (!W) cn[2] = wrap_cell(cn[2], B.L[2]);
  }
  o[0] = on[0];
  o[1] = on[1];
  o[2] = on[2];
  cell = split_encode(cn);
}

// c + L if c < 0, c - L if c >= L (c within one period of [0, L)); branch-free.
__device__ __forceinline__ int wrap1(int c, int L) {
  c += L & -(int)(c < 0);
  c -= L & -(int)(c >= L);
  return c;
}

// Shifted cell coordinates c_k = floor(x_k + s_k) of a position given as
// integer part ci_k plus fraction xf_k in double (exact), with periodic wrap
// (walls: z becomes the layer index c_z + 1 in [0, H+1]).  Invalid -> err.
//
// coords_fast: the same for a position whose shifted coordinates all lie in
// [0, L); false if that is not certain.
__device__ __forceinline__ bool coords_fast(const double (&x)[3], const double (&s)[3], BoxRef B,
                                            bool walls, int (&c)[3]) {
  const double y[3] = {x[0] + s[0], x[1] + s[1], x[2] + s[2]};
#pragma unroll
  for (int k = 0; k < 3; ++k) c[k] = (int)floor(y[k]);
  if (walls) c[2] += 1;
  return !(maybe_outside(y[0], B.Ld[0]) || maybe_outside(y[1], B.Ld[1]) ||
           maybe_outside(y[2], B.Ld[2]));
}

template <bool W>
__device__ __forceinline__ bool coords_of(const int (&ci)[3], const double (&xf)[3],
                                          const double (&s)[3], BoxRef B, int (&c)[3],
                                          uint32_t& err, double dle, bool le) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double y = xf[k] + s[k];
    const bool in = y >= -2.0 && y < B.Ld[k] + 2.0;
    ok = ok && in;
    c[k] = ci[k] + (int)floor(in ? y : 0.0);
  }
  if (!W && le && (c[2] < 0 || c[2] >= B.L[2])) {
    // Lees-Edwards: a cell across a z face is formed with the image on the
    // other side (x -/+ d of the collision time)
    const double xi = c[2] >= B.L[2] ? xf[0] - dle : xf[0] + dle;
    c[0] = wrap1(ci[0] + (int)floor(xi + s[0]), B.L[0]);
  }
  c[0] = wrap1(c[0], B.L[0]);
  c[1] = wrap1(c[1], B.L[1]);
  if (W) {
    c[2] += 1;
  } else {
    c[2] = wrap1(c[2], B.L[2]);
  }
  ok = ok && (unsigned)c[0] < (unsigned)B.L[0] && (unsigned)c[1] < (unsigned)B.L[1] &&
       (unsigned)c[2] < (unsigned)B.nlz;
  if (__builtin_expect(!ok, 0)) {
    err |= kErrKey;
    c[0] = c[1] = c[2] = 0;
  }
  return ok;
}

// Split form: c_k = cell_k + floor(o_k + s_k) with the sum in FP32, which
// gives the exact floor: o is an FP32 offset in [0, 1) and s lies on the
// 2^-24 grid in [-1/2, 1/2), so o + s is exact whenever it is below 1 or near
// 0 (Sterbenz), and a sum of at least 1 stays below 2.
template <bool W>
__device__ __forceinline__ bool coords_split(const int (&ci)[3], const float (&o)[3],
                                             const double (&s)[3], BoxRef B, int (&c)[3],
                                             uint32_t& err) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float y = o[k] + (float)s[k];
    const bool in = y >= -2.0f && y < 2.0f;
    ok = ok && in;
    c[k] = ci[k] + (int)floorf(in ? y : 0.0f);
  }
  c[0] = wrap1(c[0], B.L[0]);
  c[1] = wrap1(c[1], B.L[1]);
  if (W) {
    c[2] += 1;
  } else {
    c[2] = wrap1(c[2], B.L[2]);
  }
  ok = ok && (unsigned)c[0] < (unsigned)B.L[0] && (unsigned)c[1] < (unsigned)B.L[1] &&
       (unsigned)c[2] < (unsigned)B.nlz;
  if (__builtin_expect(!ok, 0)) {
    err |= kErrKey;
    c[0] = c[1] = c[2] = 0;
  }
  return ok;
}

__device__ __forceinline__ uint32_t linear_key(const int (&c)[3], BoxRef B) {
  return (uint32_t)((c[2] * B.L[1] + c[1]) * B.L[0] + c[0]);
}

template <bool W>
__device__ __forceinline__ uint32_t key_of(const int (&ci)[3], const double (&xf)[3],
                                           const double (&s)[3], BoxRef B, uint32_t& err,
                                           double dle, bool le) {
  int c[3];
  coords_of<W>(ci, xf, s, B, c, err, dle, le);
  return linear_key(c, B);
}

// Per-form particle access.  P = position type, V = velocity type,
// Vs = LDS velocity type, R = rotation arithmetic type.
template <int F>
struct Form;

template <>
struct Form<kFormF64> {
  struct P {
    double x[3];
  };
  struct Vv {
    double v[3];
  };
  using Vs = double;
  using Xs = double;
  __device__ static Xs pos(const P& p, int k) { return p.x[k]; }
  // record: three 16-byte words (x0 x1 | x2 v0 | v1 v2)
  __device__ static void load(const StatePtrs& S, uint32_t i, P& p, Vv& v) {
    const double2* r = (const double2*)S.rec + 3 * (size_t)i;
    const double2 a = r[0], b = r[1], c = r[2];
    p.x[0] = a.x;
    p.x[1] = a.y;
    p.x[2] = b.x;
    v.v[0] = b.y;
    v.v[1] = c.x;
    v.v[2] = c.y;
  }
  __device__ static void load_all(const StatePtrs& S, uint32_t i, P& p, Vv& v, uint32_t& id) {
    load(S, i, p, v);
    id = S.id[i];
  }
  __device__ static void store_all(const StatePtrs& S, uint32_t j, const P& p, const Vv& v,
                                   uint32_t id) {
    double2* r = (double2*)S.rec + 3 * (size_t)j;
    r[0] = make_double2(p.x[0], p.x[1]);
    r[1] = make_double2(p.x[2], v.v[0]);
    r[2] = make_double2(v.v[1], v.v[2]);
    S.id[j] = id;
  }
  template <bool W>
  __device__ static void stream(P& p, Vv& v, BoxRef B, double dle, bool le) {
    stream_f64<W>(p.x, v.v, B, dle, le);
  }
  template <bool W>
  __device__ static uint32_t key(const P& p, const double (&s)[3], BoxRef B,
                                 uint32_t& err, double dle, bool le) {
    const int ci[3] = {0, 0, 0};
    const double xf[3] = {p.x[0], p.x[1], p.x[2]};
    return key_of<W>(ci, xf, s, B, err, dle, le);
  }
  template <bool W>
  __device__ static void coords(const P& p, const double (&s)[3], BoxRef B, int (&c)[3],
                                uint32_t& err, double dle, bool le) {
    const double xf[3] = {p.x[0], p.x[1], p.x[2]};
    if (coords_fast(xf, s, B, W, c)) return;
    const int ci[3] = {0, 0, 0};
    coords_of<W>(ci, xf, s, B, c, err, dle, le);
  }
  // x coordinate of the collision cell (as coords)
  __device__ static int cell_x(const P& p, const double (&s)[3], BoxRef B, double dle, bool le) {
    const double y = (double)p.x[0] + s[0];
    if (!le && !maybe_outside(y, B.Ld[0])) return (int)floor(y);
    int c = (int)floor(y >= -2.0 && y < B.Ld[0] + 2.0 ? y : 0.0);
    if (le) {
      const double cz = floor((double)p.x[2] + s[2]);
      if (cz < 0.0 || cz >= B.Ld[2])
        c = wrap1((int)floor((cz < 0.0 ? (double)p.x[0] + dle : (double)p.x[0] - dle) + s[0]),
                  B.L[0]);
    }
    return wrap1(c, B.L[0]);
  }
  // Lees-Edwards side of the collision cell: +1 below the lower z face,
  // -1 above the upper one, else 0
  __device__ static int le_side(const P& p, double sz, BoxRef B) {
    const double cz = floor(p.x[2] + sz);
    return cz < 0.0 ? 1 : (cz >= B.Ld[2] ? -1 : 0);
  }
};

template <>
struct Form<kFormF32> {
  struct P {
    float x[3];
  };
  struct Vv {
    float v[3];
  };
  using Vs = float;
  using Xs = float;
  __device__ static Xs pos(const P& p, int k) { return p.x[k]; }
  // record: three 8-byte words (x0 x1 | x2 v0 | v1 v2)
  __device__ static void load(const StatePtrs& S, uint32_t i, P& p, Vv& v) {
    const float2* r = (const float2*)S.rec + 3 * (size_t)i;
    const float2 a = r[0], b = r[1], c = r[2];
    p.x[0] = a.x;
    p.x[1] = a.y;
    p.x[2] = b.x;
    v.v[0] = b.y;
    v.v[1] = c.x;
    v.v[2] = c.y;
  }
  __device__ static void load_all(const StatePtrs& S, uint32_t i, P& p, Vv& v, uint32_t& id) {
    load(S, i, p, v);
    id = S.id[i];
  }
  __device__ static void store_all(const StatePtrs& S, uint32_t j, const P& p, const Vv& v,
                                   uint32_t id) {
    float2* r = (float2*)S.rec + 3 * (size_t)j;
    r[0] = make_float2(p.x[0], p.x[1]);
    r[1] = make_float2(p.x[2], v.v[0]);
    r[2] = make_float2(v.v[1], v.v[2]);
    S.id[j] = id;
  }
  template <bool W>
  __device__ static void stream(P& p, Vv& v, BoxRef B, double dle, bool le) {
    stream_f32<W>(p.x, v.v, B, dle, le);
  }
  template <bool W>
  __device__ static uint32_t key(const P& p, const double (&s)[3], BoxRef B,
                                 uint32_t& err, double dle, bool le) {
    const int ci[3] = {0, 0, 0};
    const double xf[3] = {(double)p.x[0], (double)p.x[1], (double)p.x[2]};
    return key_of<W>(ci, xf, s, B, err, dle, le);
  }
  template <bool W>
  __device__ static void coords(const P& p, const double (&s)[3], BoxRef B, int (&c)[3],
                                uint32_t& err, double dle, bool le) {
    const double xf[3] = {(double)p.x[0], (double)p.x[1], (double)p.x[2]};
    if (coords_fast(xf, s, B, W, c)) return;
    const int ci[3] = {0, 0, 0};
    coords_of<W>(ci, xf, s, B, c, err, dle, le);
  }
  // x coordinate of the collision cell (as coords)
  __device__ static int cell_x(const P& p, const double (&s)[3], BoxRef B, double dle, bool le) {
    const double y = (double)p.x[0] + s[0];
    if (!le && !maybe_outside(y, B.Ld[0])) return (int)floor(y);
    int c = (int)floor(y >= -2.0 && y < B.Ld[0] + 2.0 ? y : 0.0);
    if (le) {
      const double cz = floor((double)p.x[2] + s[2]);
      if (cz < 0.0 || cz >= B.Ld[2])
        c = wrap1((int)floor((cz < 0.0 ? (double)p.x[0] + dle : (double)p.x[0] - dle) + s[0]),
                  B.L[0]);
    }
    return wrap1(c, B.L[0]);
  }
  __device__ static int le_side(const P& p, double sz, BoxRef B) {
    const double cz = floor((double)p.x[2] + sz);
    return cz < 0.0 ? 1 : (cz >= B.Ld[2] ? -1 : 0);
  }
};

template <>
struct Form<kFormSplit> {
  struct P {
    uint32_t cell;
    float o[3];
  };
  struct Vv {
    float v[3];
  };
  using Vs = float;
  using Xs = float;
  __device__ static Xs pos(const P& p, int k) { return p.o[k]; }
  // record: two 16-byte words (cell o0 o1 o2 | v0 v1 v2 id).  The gather
  // reads the id word with a load of its own after the 28 bytes of state
  // (measured 8 % faster for the collide than one 16-byte load of v and id).
  __device__ static void load(const StatePtrs& S, uint32_t i, P& p, Vv& v) {
    const uint4* r = (const uint4*)S.rec + 2 * (size_t)i;
    const uint4 a = r[0];
    const uint32_t* w = (const uint32_t*)(r + 1);
    p.cell = a.x;
    p.o[0] = __uint_as_float(a.y);
    p.o[1] = __uint_as_float(a.z);
    p.o[2] = __uint_as_float(a.w);
    v.v[0] = __uint_as_float(w[0]);
    v.v[1] = __uint_as_float(w[1]);
    v.v[2] = __uint_as_float(w[2]);
  }
  __device__ static void load_all(const StatePtrs& S, uint32_t i, P& p, Vv& v, uint32_t& id) {
    load(S, i, p, v);
    id = S.id[(size_t)i * (sizeof(RecSplit) / 4)];
  }
  __device__ static void store_all(const StatePtrs& S, uint32_t j, const P& p, const Vv& v,
                                   uint32_t id) {
    uint4* r = (uint4*)S.rec + 2 * (size_t)j;
    r[0] = make_uint4(p.cell, __float_as_uint(p.o[0]), __float_as_uint(p.o[1]),
                      __float_as_uint(p.o[2]));
    r[1] = make_uint4(__float_as_uint(v.v[0]), __float_as_uint(v.v[1]), __float_as_uint(v.v[2]),
                      id);
  }
  template <bool W>
  __device__ static void stream(P& p, Vv& v, BoxRef B, double dle, bool le) {
    stream_split<W>(p.cell, p.o, v.v, B, dle, le);
  }
  template <bool W>
  __device__ static void coords(const P& p, const double (&s)[3], BoxRef B, int (&c)[3],
                                uint32_t& err, double dle, bool le) {
    int ci[3];
    split_decode(p.cell, ci);
    if (!le) {
      // inside without a wrap (|y| < 2 also excludes NaN), else the full rule
      const float y[3] = {p.o[0] + (float)s[0], p.o[1] + (float)s[1], p.o[2] + (float)s[2]};
      bool in = true;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        c[k] = ci[k] + (int)floorf(y[k]);
        in = in && fabsf(y[k]) < 2.0f && (unsigned)c[k] < (unsigned)B.L[k];
      }
      if (W) c[2] += 1;
      if (!in) coords_split<W>(ci, p.o, s, B, c, err);
      return;
    }
    // Lees-Edwards: the image offset is applied in FP64
    const double xf[3] = {(double)p.o[0], (double)p.o[1], (double)p.o[2]};
    coords_of<W>(ci, xf, s, B, c, err, dle, le);
  }
  template <bool W>
  __device__ static uint32_t key(const P& p, const double (&s)[3], BoxRef B,
                                 uint32_t& err, double dle, bool le) {
    int c[3];
    coords<W>(p, s, B, c, err, dle, le);
    return linear_key(c, B);
  }
  // x coordinate of the collision cell (as coords)
  __device__ static int cell_x(const P& p, const double (&s)[3], BoxRef B, double dle, bool le) {
    const int cx = (int)(p.cell & ((1u << kSplitXBits) - 1));
    if (le) {
      int ci[3];
      split_decode(p.cell, ci);
      const int cz = ci[2] + (int)floor((double)p.o[2] + s[2]);
      const double xo = (double)p.o[0];
      if (cz < 0 || cz >= B.L[2])
        return wrap1(wrap1(cx + (int)floor((cz < 0 ? xo + dle : xo - dle) + s[0]), B.L[0]), B.L[0]);
      return wrap1(cx + (int)floor(xo + s[0]), B.L[0]);
    }
    return wrap1(cx + (int)floorf(p.o[0] + (float)s[0]), B.L[0]);
  }
  __device__ static int le_side(const P& p, double sz, BoxRef B) {
    int ci[3];
    split_decode(p.cell, ci);
    const int cz = ci[2] + (int)floor((double)p.o[2] + sz);
    return cz < 0 ? 1 : (cz >= B.L[2] ? -1 : 0);
  }
};

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t value) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    p[i] = value;
}

__global__ void k_set_ctrl(Ctrl* c, uint64_t step, uint32_t cur, int32_t reorder, int clear_err) {
  c->step = step;
  c->cur = cur;
  c->tri = 0u;
  c->reorder = reorder;
  if (clear_err) c->err = 0u;
}

__global__ void k_advance(Ctrl* c, uint32_t n) {
  c->step = c->step + n;
  c->cur = (c->cur + n) & 1u;
  c->tri = (c->tri + n) % 3u;
}

// hist[c] += 1 for every active lane, one atomic per distinct key in the
// wavefront; returns the lane's rank among all particles counted for c (the
// old count of its run's leader plus its place in the run).
__device__ __forceinline__ uint32_t wave_hist_rank(uint32_t* hist, uint32_t c, bool active) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint64_t pending = __ballot(active);
  uint64_t mine = 0;
  while (pending) {
    const int lead = __ffsll((unsigned long long)pending) - 1;
    const uint32_t lc = (uint32_t)__builtin_amdgcn_readlane((int)c, lead);
    const uint64_t same = __ballot(active && c == lc) & pending;
    if (active && c == lc) mine = same;
    pending &= ~same;
  }
  const uint32_t before = (uint32_t)__popcll(mine & lt_mask);
  uint32_t old = 0;
  if (active && before == 0) old = atomicAdd(&hist[c], (uint32_t)__popcll(mine));
  const int lead_lane = active ? (__ffsll((unsigned long long)mine) - 1) : (int)lane;
  old = __shfl(old, lead_lane, 64);
  return old + before;
}

// Binning export: cell key, histogram and in-cell rank of step t for the
// particles of state buffer S (the input of that step).
template <int F, bool W>
__global__ __launch_bounds__(kThreads) void k_key_hist(Dev d, StatePtrs S, uint64_t t) {
  using Fm = Form<F>;
  __shared__ double s_sh[3];
  const PBlock pb = load_pblock(d.pblocks, blockIdx.x);
  BoxRef B = as_const(d.boxes)[pb.box];
  if (threadIdx.x == 0) {
    double s[3];
    shift_of(B, t, s);
    s_sh[0] = s[0];
    s_sh[1] = s[1];
    s_sh[2] = s[2];
  }
  __syncthreads();
  const double s[3] = {s_sh[0], s_sh[1], s_sh[2]};
  const uint32_t pend = B.pbase + B.np;
  uint32_t err = 0;
#pragma unroll
  for (int k = 0; k < kPartBlock / kThreads; ++k) {
    const uint32_t i = pb.p0 + k * kThreads + threadIdx.x;
    uint32_t key = 0;
    if (i < pend) {
      typename Fm::P p;
      typename Fm::Vv v;
      Fm::load(S, i, p, v);
      const double dle = W ? 0.0 : le_offset(B, t + 1);
      Fm::template stream<W>(p, v, B, dle, !W && B.le);
      key = B.cbase + Fm::template key<W>(p, s, B, err, dle, !W && B.le);
      d.key[i] = key;
    }
    const uint32_t rk = wave_hist_rank(d.hist, key, i < pend);
    if (i < pend) d.rank[i] = (uint16_t)min(rk, 0xffffu);
  }
  if (err) atomicOr(&d.ctrl->err, err);
}

// ---------------------------------------------------------------------------
// Device-wide exclusive scan of hist -> offset (reduce, top, down-sweep)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int dlt = 1; dlt < 64; dlt <<= 1) {
    const uint32_t y = __shfl_up(x, dlt, 64);
    if (lane >= dlt) x += y;
  }
  return x;
}

// Exclusive block scan of one value per thread; returns the block total too.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* s_w,
                                                         uint32_t& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  const uint32_t inc = wave_inclusive_scan(x);
  if (lane == 63) s_w[wid] = inc;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const uint32_t sw = s_w[w];
    if (w < wid) pre += sw;
    tot += sw;
  }
  total = tot;
  __syncthreads();
  return pre + inc - x;
}

__global__ __launch_bounds__(kThreads) void k_scan_reduce(const uint32_t* __restrict__ hist,
                                                          uint32_t* __restrict__ blk) {
  __shared__ uint32_t s_w[kThreads / 64];
  const uint4* h4 = (const uint4*)(hist + (uint64_t)blockIdx.x * kScanBlock);
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems / 4; ++k) {
    const uint4 q = h4[k * kThreads + threadIdx.x];
    sum += q.x + q.y + q.z + q.w;
  }
  uint32_t total;
  block_exclusive_scan(sum, s_w, total);
  if (threadIdx.x == 0) blk[blockIdx.x] = total;
}

// One workgroup of 1024 threads scans all block totals in place (exclusive).
__global__ __launch_bounds__(1024) void k_scan_top(uint32_t* __restrict__ blk, uint32_t nblk) {
  __shared__ uint32_t s_w[16];
  __shared__ uint32_t s_carry;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (uint32_t base = 0; base < nblk; base += 1024) {
    const uint32_t i = base + threadIdx.x;
    const uint32_t x = i < nblk ? blk[i] : 0u;
    uint32_t total;
    const uint32_t ex = block_exclusive_scan(x, s_w, total);
    const uint32_t carry = s_carry;
    if (i < nblk) blk[i] = carry + ex;
    __syncthreads();
    if (threadIdx.x == 0) s_carry = carry + total;
    __syncthreads();
  }
}

// Each thread owns kScanItems consecutive cells.
__global__ __launch_bounds__(kThreads) void k_scan_down(Dev d, uint32_t nblk) {
  __shared__ uint32_t s_w[kThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)threadIdx.x * kScanItems;
  const uint4* h4 = (const uint4*)(d.hist + base);
  uint32_t v[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems / 4; ++k) {
    const uint4 q = h4[k];
    v[4 * k] = q.x;
    v[4 * k + 1] = q.y;
    v[4 * k + 2] = q.z;
    v[4 * k + 3] = q.w;
  }
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) sum += v[k];
  uint32_t total;
  uint32_t run = (nblk > 1 ? d.scan_blk[blockIdx.x] : 0u) + block_exclusive_scan(sum, s_w, total);
  uint4* o4 = (uint4*)(d.offset + base);
#pragma unroll
  for (int k = 0; k < kScanItems / 4; ++k) {
    uint4 q;
    q.x = run;
    run += v[4 * k];
    q.y = run;
    run += v[4 * k + 1];
    q.z = run;
    run += v[4 * k + 2];
    q.w = run;
    run += v[4 * k + 3];
    o4[k] = q;
  }
  if (blockIdx.x == nblk - 1 && threadIdx.x == kThreads - 1)
    d.offset[(uint64_t)nblk * kScanBlock] = run;
}

// Binning export: slot of each particle inside its cell segment (the order
// inside a segment is made canonical afterwards).
__global__ __launch_bounds__(kThreads) void k_scatter(const uint32_t* __restrict__ key,
                                                      const uint16_t* __restrict__ rank,
                                                      const uint32_t* __restrict__ offset,
                                                      uint32_t* __restrict__ perm, uint32_t n,
                                                      uint32_t ncell, Ctrl* ctrl) {
  // Every particle already holds its rank among the particles of its cell
  // (taken when the cell's count was accumulated): no atomics here.
  uint32_t bad = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t i = blockIdx.x * (kThreads * 4) + k * kThreads + threadIdx.x;
    if (i >= n) continue;
    const uint32_t c = key[i];
    if (c >= ncell) {
      bad = 1;
      continue;
    }
    const uint32_t slot = offset[c] + rank[i];
    if (slot >= offset[c + 1] || slot >= n) {
      bad = 1;
    } else {
      perm[slot] = i;
    }
  }
  if (bad) atomicOr(&ctrl->err, kErrKey);
}

// The collide workgroup is a single wavefront.  LDS instructions of one wave
// execute in issue order, so lanes see each other's LDS writes without a
// hardware barrier; a wavefront-scope fence keeps the compiler from moving LDS
// accesses across phase boundaries.  (A workgroup barrier would also wait for
// every outstanding global load and store of the wave.)
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// Inclusive sum over the 64 lanes (DPP row shifts and broadcasts, no LDS).
__device__ __forceinline__ uint32_t wave_scan_dpp(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return (uint32_t)x;
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ---------------------------------------------------------------------------
// Tiles
// ---------------------------------------------------------------------------
// Tile (key order) of the cell with coordinates c.
__device__ __forceinline__ uint32_t tile_of(BoxRef B, const int (&c)[3]) {
  return B.tbase + ((uint32_t)c[2] * (uint32_t)B.L[1] + (uint32_t)c[1]) * B.ntx +
         (uint32_t)c[0] / B.T;
}

// Sort by tile of a state set from outside (order arbitrary): particles per
// tile of step t (high word of the tile's counter), and of every particle its
// tile and its rank there (in the arrays of the chains, which no run uses yet)
// ... Neighbouring lanes of one tile share an atomic, so that a state already in
// order (its tiling changed, its binning exported) does not queue at one word
// (256^3 FP64: 4.7 ms, 9.5 with an atomic each).  Of a random state every
// particle takes one, which bounds the kernel: 25 a nanosecond (256^3: 6.6 ms,
// 7.3 on the whole 64-bit counter).
template <int F, bool W>
__global__ __launch_bounds__(kThreads) void k_tile_count(Dev d, uint32_t from) {
  using Fm = Form<F>;
  __shared__ double s_sh[3];
  const PBlock pb = load_pblock(d.pblocks, blockIdx.x);
  BoxRef B = as_const(d.boxes)[pb.box];
  const uint64_t t = d.ctrl->step;
  const StatePtrs S = d.S[from];
  if (threadIdx.x == 0) {
    double s[3];
    shift_of(B, t, s);
    s_sh[0] = s[0];
    s_sh[1] = s[1];
    s_sh[2] = s[2];
  }
  __syncthreads();
  const double s[3] = {s_sh[0], s_sh[1], s_sh[2]};
  const double dle = W ? 0.0 : le_offset(B, t + 1);
  const uint32_t pend = B.pbase + B.np, lane = threadIdx.x & 63;
  uint32_t err = 0;
  constexpr int U = kPartBlock / kThreads;
  uint32_t tl[U], old[U], lead[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const uint32_t i = pb.p0 + k * kThreads + threadIdx.x;
    tl[k] = kNoSlot;
    old[k] = 0u;
    if (i < pend) {
      typename Fm::P p;
      typename Fm::Vv v;
      Fm::load(S, i, p, v);
      Fm::template stream<W>(p, v, B, dle, !W && B.le);
      int c[3];
      Fm::template coords<W>(p, s, B, c, err, dle, !W && B.le);
      tl[k] = tile_of(B, c);
    }
    const uint32_t before = __shfl_up(tl[k], 1, 64);
    const uint64_t heads = __ballot(lane == 0 || before != tl[k]);
    const uint64_t upto = heads & (~0ull >> (63u - lane)), after = heads & ~(~0ull >> (63u - lane));
    lead[k] = 63u - (uint32_t)__clzll((long long)upto);
    const uint32_t end = after ? (uint32_t)__ffsll((unsigned long long)after) - 1u : 64u;
    if (lane == lead[k] && i < pend)
      old[k] = atomicAdd((uint32_t*)&d.tcnt[0][tl[k]] + 1, end - lane);
  }
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const uint32_t i = pb.p0 + k * kThreads + threadIdx.x;
    const uint32_t rank = __shfl(old[k], (int)lead[k], 64) + (lane - lead[k]);
    if (i < pend) {
      d.rnext[0][i] = tl[k];
      d.rnext[1][i] = rank;
    }
  }
  if (err) atomicOr(&d.ctrl->err, err);
}

// ... and, once the prefix of those counts is known, the records into the other
// buffer, tile by tile.  Consecutive lanes move consecutive words of a record,
// so that a record is one access.  Of a random state one side of the move is
// random; single particles of whole sectors are better written (split form, 32
// bytes with the index: 256^3 7.3 ms, a gather 10.8), others better read, after
// their slots' indices were placed in the id array (FP64: 5.5 + 6.9 ms; records
// and ids written at random 14.9, three stores a lane 16.1).
__global__ __launch_bounds__(kThreads) void k_tile_scatter(Dev d, uint32_t from, uint32_t to) {
  __shared__ uint32_t s_j[kPartBlock];
  const uint32_t i0 = blockIdx.x * kPartBlock;
#pragma unroll
  for (int k = 0; k < kPartBlock / kThreads; ++k) {
    const uint32_t q = k * kThreads + threadIdx.x, i = i0 + q;
    s_j[q] = i < d.ntot ? d.toff[d.rnext[0][i]] + d.rnext[1][i] : kNoSlot;
  }
  __syncthreads();
  constexpr uint32_t W = sizeof(RecSplit) / sizeof(uint4);
  const uint4* in = (const uint4*)d.S[from].rec + (size_t)i0 * W;
  uint4* out = (uint4*)d.S[to].rec;
#pragma unroll
  for (uint32_t k = 0; k < W * (kPartBlock / kThreads); ++k) {
    const uint32_t w = k * kThreads + threadIdx.x, j = s_j[w / W];
    if (j < d.ntot) out[(size_t)j * W + w % W] = in[w];
  }
}
__global__ __launch_bounds__(kThreads) void k_tile_place(Dev d, uint32_t to) {
  uint32_t* id = d.S[to].id;
  uint32_t j[kPartBlock / kThreads];
#pragma unroll
  for (int k = 0; k < kPartBlock / kThreads; ++k) {
    const uint32_t i = blockIdx.x * kPartBlock + k * kThreads + threadIdx.x;
    j[k] = i < d.ntot ? d.toff[d.rnext[0][i]] + d.rnext[1][i] : kNoSlot;
  }
#pragma unroll
  for (int k = 0; k < kPartBlock / kThreads; ++k)
    if (j[k] < d.ntot) id[j[k]] = blockIdx.x * kPartBlock + k * kThreads + threadIdx.x;
}
// caller: the slots are in the caller's order, their ids their numbers
template <int F>
__global__ __launch_bounds__(kThreads) void k_tile_gather(Dev d, uint32_t from, uint32_t to,
                                                          int caller) {
  using Word = typename std::conditional<F == kFormF64, double2, float2>::type;
  constexpr uint32_t W = rec_bytes(F) / sizeof(Word);
  static_assert(W * sizeof(Word) == rec_bytes(F), "whole words");
  __shared__ uint32_t s_i[kPartBlock];
  const StatePtrs in = d.S[from], out = d.S[to];
  const uint32_t j0 = blockIdx.x * kPartBlock;
#pragma unroll
  for (int k = 0; k < kPartBlock / kThreads; ++k) {
    const uint32_t q = k * kThreads + threadIdx.x, j = j0 + q;
    uint32_t i = 0;
    if (j < d.ntot) {
      i = min(out.id[j], d.ntot - 1u);
      out.id[j] = caller ? i : in.id[i];
    }
    s_i[q] = i;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < W * (kPartBlock / kThreads); ++k) {
    const uint32_t w = k * kThreads + threadIdx.x, q = w / W;
    if (j0 + q < d.ntot)
      ((Word*)out.rec)[(size_t)j0 * W + w] = ((const Word*)in.rec)[(size_t)s_i[q] * W + w % W];
  }
}

// Before a sort: no particles, no runs, no chains in any set.
__global__ __launch_bounds__(kThreads) void k_tile_clear(Dev d) {
  const uint64_t stride = (uint64_t)gridDim.x * kThreads, i0 = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  for (uint64_t i = i0; i < d.ntile; i += stride) {
#pragma unroll
    for (int k = 0; k < 3; ++k) d.tcnt[k][i] = 0ull;
  }
  const uint64_t heads = (uint64_t)d.ntile * d.maxr;
  for (uint64_t i = i0; i < heads; i += stride) {
#pragma unroll
    for (int k = 0; k < 2; ++k) d.rhead[k][i] = kNoSlot;
  }
}

// ... and one run per occupied tile.
__global__ __launch_bounds__(kThreads) void k_tile_runs(Dev d, uint32_t to) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= d.ntile) return;
  const uint32_t n = (uint32_t)(d.tcnt[0][i] >> 32);
  d.tcnt[0][i] = (unsigned long long)n << 32 | (n ? 1u : 0u);
  d.runs[to][(size_t)i * d.maxr] = Run{d.toff[i], n};
}

// ---------------------------------------------------------------------------
// Output position of every tile
// ---------------------------------------------------------------------------
// Set of tile counters that step j of a launch sequence reads; the next of the
// three is counted up by its collide, the one after that cleared.
__device__ __forceinline__ uint32_t counter_set(const Dev& d, uint32_t j) {
  return (as_const(d.ctrl)->tri + j) % 3u;
}

// Particles per block of kTileBlock tiles (only for more than kTileOne tiles;
// below that every block of the prefix sums the counts before it).
__global__ __launch_bounds__(kThreads) void k_tile_reduce(Dev d, uint32_t j) {
  __shared__ uint32_t s_w[kThreads / 64];
  const unsigned long long* cnt = d.tcnt[counter_set(d, j)];
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kTileBlock / kThreads; ++k) {
    const uint32_t i = blockIdx.x * kTileBlock + k * kThreads + threadIdx.x;
    if (i < d.ntile) sum += (uint32_t)(cnt[i] >> 32);
  }
  uint32_t total;
  block_exclusive_scan(sum, s_w, total);
  if (threadIdx.x == 0) d.tblk[blockIdx.x] = total;
}

// toff: exclusive prefix of the particles per tile.
__global__ __launch_bounds__(kThreads) void k_tile_prefix(Dev d, uint32_t j) {
  __shared__ uint32_t s_w[kThreads / 64];
  const unsigned long long* cnt = d.tcnt[counter_set(d, j)];
  const uint32_t blk = blockIdx.x;
  const uint32_t b0 = blk * kTileBlock;
  // particles of all tiles before this block
  uint32_t before = 0;
  if (d.ntile > kTileOne) {
    for (uint32_t i = threadIdx.x; i < blk; i += kThreads) before += d.tblk[i];
  } else {
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < b0; i += kThreads) before += (uint32_t)(cnt[i] >> 32);
  }
  uint32_t run;
  block_exclusive_scan(before, s_w, run);
  constexpr int K = kTileBlock / kThreads;
  const uint32_t i0 = b0 + threadIdx.x * K;
  uint32_t c[K], sum = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    c[k] = i0 + k < d.ntile ? (uint32_t)(cnt[i0 + k] >> 32) : 0u;
    sum += c[k];
  }
  uint32_t total;
  run += block_exclusive_scan(sum, s_w, total);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (i0 + k < d.ntile) d.toff[i0 + k] = run;
    run += c[k];
  }
}

// ---------------------------------------------------------------------------
// Side work of a collide: what the next step reads besides the particles
// ---------------------------------------------------------------------------
// Box that owns global cell c (boxes are stored in ascending cbase).
__device__ __forceinline__ uint32_t box_of_cell(const BoxDev* boxes, uint32_t nbox, uint32_t c) {
  uint32_t lo = 0, hi = nbox;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (as_const(boxes)[mid].cbase <= c) {
      lo = mid;
    } else {
      hi = mid;
    }
  }
  return lo;
}

// Random draws of the cells of step t into set `buf`: the rotation axis and,
// with the thermostat, the gamma draw.  The number of particles n of a cell,
// which sets the shape, is known to the collide only; so an attempt is kept
// with the smallest n that accepts it.  Attempt 0 stands in the cell's record.
// A cell whose attempt 0 is not accepted for every n (one in 37) gets a chain
// of later attempts up to one that is, in its draw block's segment of `later`
// (entry 0 unused).  Such cells are listed first and worked out many at a
// time: made at once by every wavefront they took the draws from 0.3 to 1.1 ms
// at 256^3.  The collide then needs neither logarithm nor cosine, which had
// cost it a quarter of its wavefronts in registers.
struct DrawList {
  uint16_t* cell;  // LDS, kDrawList entries: cells of the block still to do
  uint32_t* used;  // LDS: entries taken of the block's segment
  uint32_t n;      // entries of `cell` (uniform)
};

// Chains of the listed cells of draw block `blk`.
__device__ __forceinline__ void draw_chains(const Dev& d, uint32_t nbox, uint32_t blk, uint64_t t,
                                            uint32_t buf, DrawList& l) {
  const uint32_t lane = threadIdx.x & 63;
  wave_sync();
  Attempt* seg = d.later[buf] + (size_t)blk * later_seg(d.drawb);
  for (uint32_t q = lane; q < l.n; q += 64) {
    const uint32_t c = blk * d.drawb + l.cell[q];
    BoxRef B = as_const(d.boxes)[box_of_cell(d.boxes, nbox, c)];
    uint32_t word = 0, prev = 0;
#pragma unroll 1
    for (uint32_t j = 0; j < 64; ++j) {
      double z, lu;
      gamma_attempt(B.key_lo, B.key_hi, t, c - B.cbase, j, z, lu);
      const uint32_t least = gamma_least(z, lu);
      if (j == 0) {
        word = least;
        continue;
      }
      const uint32_t m = 1u + atomicAdd(l.used, 1u);
      if (m >= later_seg(d.drawb)) {
        atomicOr(&d.ctrl->err, kErrDraws);
        break;
      }
      seg[m] = Attempt{z, (uint16_t)least, 0, 0};
      if (prev) {
        seg[prev].next = (uint16_t)m;
      } else {
        word |= m << 16;
      }
      prev = m;
      if (least == 2u) break;
    }
    d.least[buf][c] = word;
  }
  l.n = 0u;
  wave_sync();
}

// The draws of up to 64 cells from cell k of draw block `blk` on.
template <bool M>
__device__ __forceinline__ void draw_cells(const Dev& d, uint32_t nbox, uint32_t ctot, uint32_t blk,
                                           uint32_t k, uint64_t t, uint32_t buf, DrawList& l) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t c = blk * d.drawb + k + lane;
  bool later = false;
  if (c < ctot) {
    BoxRef B = as_const(d.boxes)[box_of_cell(d.boxes, nbox, c)];
    double n[3], z = 0.0;
    axis_of(B, t, c - B.cbase, n);
    if (M) {
      double lu;
      gamma_attempt(B.key_lo, B.key_hi, t, c - B.cbase, 0, z, lu);
      later = !gamma_accepts(2u, z, lu);
      if (!later) d.least[buf][c] = 2u;
    }
    double2* o = (double2*)d.draws[buf] + 2 * (size_t)c;
    o[0] = make_double2(n[0], n[1]);
    o[1] = make_double2(n[2], z);
  }
  if (M) {
    if (k == 0u) {
      if (lane == 0) *l.used = 0u;
    }
    const uint64_t m = __ballot(later);
    if (later) l.cell[l.n + lanes_below(m)] = (uint16_t)(k + lane);
    l.n += (uint32_t)__popcll(m);
    if (l.n > (uint32_t)kDrawList - 64u || (k + 64u >= d.drawb && l.n))
      draw_chains(d, nbox, blk, t, buf, l);
  }
}

// Phantom particles of the cells of the two wall-cut layers of every box:
// count, velocity sum and squared-speed sum (velocities N(0, kT/m) per
// component; rounded to FP32 for the split form), read by the cell sums.
__device__ __forceinline__ void phantom_sums(const Dev& d, uint32_t nbox, uint32_t i, uint64_t t,
                                             uint32_t buf, int round32) {
  uint32_t lo = 0, hi = nbox;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (d.boxes[mid].wcbase <= i) {
      lo = mid;
    } else {
      hi = mid;
    }
  }
  BoxRef B = as_const(d.boxes)[lo];
  if (B.slip) return;  // slip walls carry no phantoms
  double sh[3];
  shift_of(B, t, sh);
  const uint32_t plane = (uint32_t)B.L[0] * (uint32_t)B.L[1];
  const uint32_t li = i - B.wcbase;
  const uint32_t top = li / plane;
  const int H = B.L[2];
  // key layer (c_z + 1) of the cut cells: c_z in {0, H} for s_z >= 0, {-1, H-1} else
  const int czk = sh[2] >= 0.0 ? (top ? H + 1 : 1) : (top ? H : 0);
  const uint32_t lkey = (uint32_t)czk * plane + (li - top * plane);
  const double fw = wall_fraction(sh[2], czk - 1, H);
  if (!(fw > 0.0)) return;
  const int nph = phantom_count(B, t, lkey, fw);
  PhantomSums ps;
  ps.v[0] = ps.v[1] = ps.v[2] = 0.0;
  ps.v2 = 0.0;
  PhantomCache pc;
  pc.j = 0xffffffffu;
  // phantoms move with the wall that fills their part of the cell
  const double uw = top ? B.uw : -B.uw;
#pragma unroll 1
  for (int q = 0; q < nph; ++q) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double vp = B.sd * phantom_normal(B, t, lkey, 3 * q + k, pc);
      if (k == 0) vp = vp + uw;
      if (round32) vp = (double)(float)vp;
      ps.v[k] = ps.v[k] + vp;
      ps.v2 = ps.v2 + vp * vp;
    }
  }
  ps.n = (double)nph;
  ps.pad = 0.0;
  d.phs[buf][B.cbase + lkey] = ps;
}

// Shifts and offsets of one box for step t.
__device__ __forceinline__ void box_step(const Dev& d, uint32_t i, uint64_t t, uint32_t buf) {
  BoxRef B = as_const(d.boxes)[i];
  BoxStep st;
  shift_of(B, t, st.s);
  shift_of(B, t + 1, st.sn);
  st.d1 = B.le ? le_offset(B, t + 1) : 0.0;
  st.d2 = B.le ? le_offset(B, t + 2) : 0.0;
  // first row of the window of next-step rows around a row: the lattice moves
  // by sn - s, so particles move to rows between -1 and 1, or for shifts
  // beyond half a cell between 0 and 2 or -2 and 0
  for (int k = 1; k < 3; ++k) {
    const double ds = st.sn[k] - st.s[k];
    const int lk = k == 1 ? B.L[1] : B.nlz;
    st.w[k - 1] = lk < 4 ? -1 : (ds > 0.5 ? 0 : (ds < -0.5 ? -2 : -1));
  }
  d.bstep[buf][i] = st;
}

// One wavefront's part of the side work for step t: 64 boxes' step data, or
// 64 wall-cut cells' phantoms, or the draws of one draw block.
template <bool W, bool M>
__device__ __forceinline__ void side_work(const Dev& d, const Side& w, uint32_t b, uint64_t t,
                                          uint32_t buf, DrawList& l) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t nbs = (w.nbox + 63u) / 64u;
  if (b < nbs) {
    if (b * 64u + lane < w.nbox) box_step(d, b * 64u + lane, t, buf);
    return;
  }
  b -= nbs;
  if (W) {
    const uint32_t nph = (w.wcells + 63u) / 64u;
    if (b < nph) {
      if (b * 64u + lane < w.wcells) phantom_sums(d, w.nbox, b * 64u + lane, t, buf, w.round32);
      return;
    }
    b -= nph;
  }
  if (b >= (w.ctot + d.drawb - 1u) / d.drawb) return;
#pragma unroll 1
  for (uint32_t k = 0; k < d.drawb; k += 64)
    draw_cells<M>(d, w.nbox, w.ctot, b, k, t, buf, l);
}

// The side work of the first step after a sort.
template <bool W, bool M>
__global__ __launch_bounds__(64) void k_side(Dev d, Side w, uint32_t buf) {
  __shared__ uint16_t s_dcell[kDrawList];
  __shared__ uint32_t s_dused;
  DrawList l{s_dcell, &s_dused, 0u};
  side_work<W, M>(d, w, blockIdx.x, as_const(d.ctrl)->step, buf, l);
}

// ---------------------------------------------------------------------------
// Collide (+ stream/bin of the next step)
// ---------------------------------------------------------------------------
// Appends the run [start, start + n) of the output buffer to the list of tile
// `dest`: a slot of its table, or (table full) a chain of single particles
// from one of maxr heads.
__device__ __forceinline__ void push_run(const Dev& d, uint32_t out, uint32_t set, uint32_t dest,
                                         uint32_t start, uint32_t n) {
  if (dest >= d.ntile) return;
  const uint32_t slot =
      (uint32_t)atomicAdd(&d.tcnt[set][dest], (unsigned long long)n << 32 | 1ull);
  if (slot < d.maxr) {
    d.runs[out][(size_t)dest * d.maxr + slot] = Run{start, n};
  } else {
    uint32_t* next = d.rnext[out];
    for (uint32_t q = 0; q + 1 < n; ++q) next[start + q] = start + q + 1;
    next[start + n - 1] = atomicExch(&d.rhead[out][(size_t)dest * d.maxr + slot % d.maxr], start);
  }
}

// Per-cell record of the collision, FP64 forms: the update rotates with the
// vector formula in FP64.
struct CellLds {
  double V[3];   // centre-of-mass velocity
  double n[3];   // rotation axis
  double kappa;  // thermostat scale; 0 = the cell does not collide
};
// Split form: kappa R(alpha, n) built in FP64 and rounded to FP32, so the
// FP32 rotation's rounding differs from cell to cell (FP32 cos and sin of the
// one angle would bias every collision's energy the same way).
struct CellLdsSplit {
  float V[3];
  float R[9];    // kappa * rotation matrix, row major
  float coll;    // 0 = the cell does not collide
};
// SRD+a (Eqs. 3-4) adds the centre of mass in the cell frame and the angular
// velocity of the correction omega x r_ic.
struct CellLdsAmc : CellLds {
  double rc[3];
  double om[3];
};
struct CellLdsSplitAmc : CellLdsSplit {
  double rc[3];  // FP64: the correction is formed in FP64 and rounded once
  double om[3];
};
template <int F, bool A>
struct CellRec {
  using T = CellLds;
};
template <>
struct CellRec<kFormF64, true> {
  using T = CellLdsAmc;
};
template <>
struct CellRec<kFormF32, true> {
  using T = CellLdsAmc;
};
template <>
struct CellRec<kFormSplit, false> {
  using T = CellLdsSplit;
};
template <>
struct CellRec<kFormSplit, true> {
  using T = CellLdsSplitAmc;
};

// Position of a particle in the frame of its (shifted) cell, frac(x + s),
// from the stored coordinate (FP64 and FP32 forms: x; split form: the offset,
// whose cell index is an integer and drops out).  Exact for the FP32 forms.
template <typename X>
__device__ __forceinline__ double frame_pos(X x, double s) {
  const double y = (double)x + s;
  return y - floor(y);
}

// Rotation by alpha about n (Eq. 2): R u = cos(a) u + sin(a) n x u +
// (1 - cos(a)) (n . u) n.
template <typename T>
__device__ __forceinline__ void rotate(T ca, T sa, T omc, const T (&n)[3], const T (&u)[3],
                                       T (&r)[3]) {
  const T nu = n[0] * u[0] + n[1] * u[1] + n[2] * u[2];
  const T cx[3] = {n[1] * u[2] - n[2] * u[1], n[2] * u[0] - n[0] * u[2],
                   n[0] * u[1] - n[1] * u[0]};
#pragma unroll
  for (int a = 0; a < 3; ++a) r[a] = ca * u[a] + sa * cx[a] + omc * nu * n[a];
}

// The cell sums.  Each half of a cell's fluid particles is summed by one lane
// in canonical order, and the pair of lanes (lane bit 0 = half) combines first
// half, then second, so that both hold the same total whatever the tiling.
// A pair sums the three components of the momentum (and of the centre of mass,
// SRD+a) together, or, in passes of at most ten cells, one of them: six lanes
// a cell in place of two (50 particles per cell, four cells a pass: collide
// 1.52 -> 1.44 ms at 96^3; with 20 cells in two rounds it gained nothing in
// FP64 and cost 4 % in FP32).  The terms of the kinetic energy come from the
// lanes that hold the particles, so that its sum is one read and one addition
// per particle.
__device__ __forceinline__ double pair_xor(double x) { return __shfl_xor(x, 1, 64); }
__device__ __forceinline__ float pair_xor(float x) { return __shfl_xor(x, 1, 64); }

// Fixed-point cell sums (Sec. III.C, reproducibility): a term x becomes the
// integer trunc(x 2^80) in 128-bit two's complement; sums are exact, hence
// independent of the order of the terms, and the value is the integer rounded
// once to FP64, times 2^-80.  Terms need |x| < 2^37 (no sum of at most 2^10
// terms can overflow); others (and NaN) set kErrFixRange.  While summing, the
// integer is kept as four signed digits of 32 bits, each an FP64 number: the
// digits of a term come out by truncation, exactly, and the sums of at most
// 2^10 of them stay below 2^53.  Fifteen FP64 operations a term; 128-bit
// shifts, a negation and an addition with carry had taken about forty.
struct FixSum {
  double d[4];  // digits of 2^0, 2^32, 2^64, 2^96
};
struct Fix {
  uint64_t lo, hi;
};
__device__ __forceinline__ void fix_add(FixSum& a, double x, uint32_t& err) {
  if (!(fabs(x) < 0x1p37)) {
    err |= kErrFixRange;
    return;
  }
  double r = x * 0x1p-16;
  double w = __builtin_trunc(r);
  a.d[3] += w;
  r = (r - w) * 0x1p32;
  w = __builtin_trunc(r);
  a.d[2] += w;
  r = (r - w) * 0x1p32;
  w = __builtin_trunc(r);
  a.d[1] += w;
  a.d[0] += __builtin_trunc((r - w) * 0x1p32);
}
// Exact sum over the lane pair (both lanes hold the total), as one integer.
__device__ __forceinline__ Fix fix_pair(const FixSum& a) {
  Fix f = {0ull, 0ull};
#pragma unroll
  for (int k = 3; k >= 0; --k) {
    const long long t = (long long)(a.d[k] + pair_xor(a.d[k]));
    // f = f 2^32 + t
    f.hi = f.hi << 32 | f.lo >> 32;
    f.lo <<= 32;
    const uint64_t nlo = f.lo + (uint64_t)t;
    f.hi += (t < 0 ? ~0ull : 0ull) + (nlo < f.lo ? 1ull : 0ull);
    f.lo = nlo;
  }
  return f;
}
// Nearest FP64 of the integer, times 2^-80.  The 128-bit magnitude is
// normalised so that its top 64 bits carry the rounding position, with the
// bits below OR-ed into bit 0 (sticky); the u64 -> f64 conversion then rounds
// to nearest even once.
__device__ __forceinline__ double fix_value(Fix a) {
  const bool neg = (int64_t)a.hi < 0;
  uint64_t lo = a.lo, hi = a.hi;
  if (neg) {
    lo = ~lo + 1ull;
    hi = ~hi + (lo == 0ull ? 1ull : 0ull);
  }
  double d;
  if (hi == 0) {
    d = (double)lo * 0x1p-80;
  } else {
    const int lz = __clzll((long long)hi);
    const uint64_t top = lz ? (hi << lz) | (lo >> (64 - lz)) : hi;
    const uint64_t rest = lo << lz;
    d = ldexp((double)(top | (rest != 0ull ? 1ull : 0ull)), 64 - lz - 80);
  }
  return neg ? -d : d;
}

template <int N>
struct Width {
  static constexpr int value = N;
};

// Plain or fixed-point FP64 sums of m v[q] (kScale) or of v[q] for N arrays v,
// one half of the cell, [qb, qe), per lane; both lanes of a pair get the totals.
template <bool X, bool kScale, int N, typename T>
__device__ __forceinline__ void half_sums(const T* const (&v)[N], double m, uint32_t qb,
                                          uint32_t qe, uint32_t half, uint32_t& err,
                                          double (&out)[N]) {
  if constexpr (X) {
    FixSum f[N] = {};
    for (uint32_t q = qb; q < qe; ++q) {
#pragma unroll
      for (int k = 0; k < N; ++k)
        fix_add(f[k], kScale ? m * (double)v[k][q] : (double)v[k][q], err);
    }
#pragma unroll
    for (int k = 0; k < N; ++k) out[k] = fix_value(fix_pair(f[k]));
  } else {
    double P[N];
#pragma unroll
    for (int k = 0; k < N; ++k) P[k] = 0.0;
    if (!kScale || m == 1.0) {  // 1 * v is v
#pragma unroll 4
      for (uint32_t q = qb; q < qe; ++q) {
#pragma unroll
        for (int k = 0; k < N; ++k) P[k] = P[k] + (double)v[k][q];
      }
    } else {
#pragma unroll 4
      for (uint32_t q = qb; q < qe; ++q) {
#pragma unroll
        for (int k = 0; k < N; ++k) P[k] = P[k] + m * (double)v[k][q];
      }
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const double o = pair_xor(P[k]);
      out[k] = half ? o + P[k] : P[k] + o;
    }
  }
}

// Mean velocity of a cell along N axes: its momentum, phantoms included (nph
// of them with velocity sums pv), by its mass.
template <int F, bool X, int N>
__device__ __forceinline__ void mean_velocity(const typename Form<F>::Vs* const (&v)[N], double m,
                                              uint32_t qb, uint32_t qe, uint32_t half,
                                              uint32_t ntot, uint32_t nph, const double (&pv)[N],
                                              uint32_t& err, double (&V)[N]) {
  if constexpr (X || F != kFormSplit) {
    // fixed-point or FP64 sums of the FP64 terms m v_i
    half_sums<X, true>(v, m, qb, qe, half, err, V);
    const double Mtot = (double)(ntot ? ntot : 1u) * m;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (nph) V[k] = V[k] + m * pv[k];
      V[k] = V[k] / Mtot;
    }
  } else {
    // compensated FP32 momentum sums (Neumaier)
    const float mf = (float)m;
    float s[N], c[N];
#pragma unroll
    for (int k = 0; k < N; ++k) s[k] = c[k] = 0.f;
    auto add = [&](int k, float x) {
      const float tt = s[k] + x;
      if (fabsf(s[k]) >= fabsf(x)) {
        c[k] += (s[k] - tt) + x;
      } else {
        c[k] += (x - tt) + s[k];
      }
      s[k] = tt;
    };
#pragma unroll 4
    for (uint32_t q = qb; q < qe; ++q) {
#pragma unroll
      for (int k = 0; k < N; ++k) add(k, mf * v[k][q]);
    }
    const float Mf = (float)(ntot ? ntot : 1u) * mf;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const float os = pair_xor(s[k]), oc = pair_xor(c[k]);
      // first half's (s, c), then the second half's s added, then its c
      const float s0 = half ? os : s[k], c0 = half ? oc : c[k];
      const float s1 = half ? s[k] : os, c1 = half ? c[k] : oc;
      s[k] = s0;
      c[k] = c0;
      add(k, s1);
      c[k] += c1;
      if (nph) add(k, (float)(m * pv[k]));
      V[k] = (double)((s[k] + c[k]) / Mf);
    }
  }
}

// The rest of a cell, by its pair of lanes: V and rc are its mean velocity
// and (SRD+a) its centre of mass in the cell frame, sk the kinetic-energy
// terms, sx the cell-frame positions (SRD+a).  Every lane of the wavefront
// calls this; only the first lane of a valid pair writes `out`.
template <int F, bool W, bool M, bool A, bool X>
__device__ __forceinline__ void cell_work(BoxRef B, const double (&axis)[3], double Ek,
                                          const PhantomSums* __restrict__ ph, uint32_t nph,
                                          const typename Form<F>::Vs* __restrict__ sv0,
                                          const typename Form<F>::Vs* __restrict__ sv1,
                                          const typename Form<F>::Vs* __restrict__ sv2,
                                          const double* __restrict__ sx0,
                                          const double* __restrict__ sx1,
                                          const double* __restrict__ sx2,
                                          const double* __restrict__ sk, const double (&V)[3],
                                          const double (&rc)[3], uint32_t b, uint32_t e,
                                          uint32_t half, bool valid,
                                          typename CellRec<F, A>::T* out, uint32_t& err) {
  const uint32_t nf = valid ? e - b : 0u;
  const uint32_t mid = b + (nf + 1) / 2;
  const uint32_t qb = half ? mid : b, qe = valid ? (half ? e : mid) : b;
  const uint32_t ntot = nf + nph;
  const double m = B.mass;
  double kappa = 1.0, K = 0.0;
  // kinetic-energy terms: SRD+a adds them here, next to its moments
  auto term = [&](double u0, double u1, double u2) { return m * (u0 * u0 + u1 * u1 + u2 * u2); };
  if constexpr (M && A && X) {
    FixSum f = {};
    for (uint32_t q = qb; q < qe; ++q)
      fix_add(f, term((double)sv0[q] - V[0], (double)sv1[q] - V[1], (double)sv2[q] - V[2]), err);
    K = fix_value(fix_pair(f));
  }
  if constexpr (M && !A) {
    const double* const ks[1] = {sk};
    double Ks[1];
    half_sums<X, false>(ks, 1.0, qb, qe, half, err, Ks);
    K = Ks[0];
    if (W && nph) {
      const double pv[3] = {ph->v[0], ph->v[1], ph->v[2]}, pv2 = ph->v2;
      // sum over phantoms of m |v - V|^2 from their velocity sums
      const double vV = pv[0] * V[0] + pv[1] * V[1] + pv[2] * V[2];
      const double VV = V[0] * V[0] + V[1] * V[1] + V[2] * V[2];
      K = K + m * (pv2 - 2.0 * vV + (double)nph * VV);
    }
    if (Ek > 0.0 && K > 0.0) kappa = sqrt((2.0 * Ek) / K);
  }
  // SRD+a (Eqs. 3-4, periodic boxes): omega = I^-1 dL with
  // dL = sum r_ic x (u_i - D u_i) and I the inertia tensor, both about the
  // centre of mass of the cell-frame positions (the mass m cancels; the
  // thermostat's energy below restores it).  A pair
  // uses the pseudo-inverse of its singular I (omega = dL / (tr I / 2), since
  // tr I = |r_1 - r_2|^2), three or more Cramer's rule, and det I = 0 gives
  // omega = 0.  Both lanes of the pair build identical totals.
  double om[3] = {0.0, 0.0, 0.0};
  if constexpr (A) {
    // Moments about the centre of mass: M = sum r_ic u_i^T and S = sum r_ic
    // r_ic^T (15 sums, no per-particle rotation).  Then I = tr(S) 1 - S, the
    // angular momentum before the rotation L0 = eps : M, after it
    // L_D = sum r_ic x D u_i = eps : (M D^T), and dL = L0 - L_D.
    double mm[9], ss[6];  // mm[3a+b] = M_ab; ss: xx, yy, zz, xy, xz, yz
#pragma unroll
    for (int k = 0; k < 9; ++k) mm[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) ss[k] = 0.0;
    if constexpr (X) {
      // one pass per row a of M, with S_aa and S_a(a+1 mod 3): five exact
      // sums live at a time
#pragma unroll 1
      for (int a = 0; a < 3; ++a) {
        FixSum f5[5] = {};
        const int a1 = a == 2 ? 0 : a + 1;
        for (uint32_t q = qb; q < qe; ++q) {
          const double r[3] = {sx0[q] - rc[0], sx1[q] - rc[1], sx2[q] - rc[2]};
          const double u[3] = {(double)sv0[q] - V[0], (double)sv1[q] - V[1],
                               (double)sv2[q] - V[2]};
          const double ra = a == 0 ? r[0] : (a == 1 ? r[1] : r[2]);
          const double rb = a1 == 0 ? r[0] : (a1 == 1 ? r[1] : r[2]);
          fix_add(f5[0], ra * u[0], err);
          fix_add(f5[1], ra * u[1], err);
          fix_add(f5[2], ra * u[2], err);
          fix_add(f5[3], ra * ra, err);
          fix_add(f5[4], ra * rb, err);
        }
        double v5[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          v5[k] = fix_value(fix_pair(f5[k]));
        }
        // scatter into mm / ss (ss: xx, yy, zz, xy, xz, yz; a = 2 gives zx = xz)
#pragma unroll
        for (int b2 = 0; b2 < 3; ++b2) {
          if (a == 0) mm[b2] = v5[b2];
          if (a == 1) mm[3 + b2] = v5[b2];
          if (a == 2) mm[6 + b2] = v5[b2];
        }
        if (a == 0) { ss[0] = v5[3]; ss[3] = v5[4]; }
        if (a == 1) { ss[1] = v5[3]; ss[5] = v5[4]; }
        if (a == 2) { ss[2] = v5[3]; ss[4] = v5[4]; }
      }
    } else {
    for (uint32_t q = qb; q < qe; ++q) {
      const double r[3] = {sx0[q] - rc[0], sx1[q] - rc[1], sx2[q] - rc[2]};
      const double u[3] = {(double)sv0[q] - V[0], (double)sv1[q] - V[1], (double)sv2[q] - V[2]};
      if (M) K = K + term(u[0], u[1], u[2]);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b2 = 0; b2 < 3; ++b2) mm[3 * a + b2] = fma(r[a], u[b2], mm[3 * a + b2]);
      ss[0] = fma(r[0], r[0], ss[0]);
      ss[1] = fma(r[1], r[1], ss[1]);
      ss[2] = fma(r[2], r[2], ss[2]);
      ss[3] = fma(r[0], r[1], ss[3]);
      ss[4] = fma(r[0], r[2], ss[4]);
      ss[5] = fma(r[1], r[2], ss[5]);
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double o = pair_xor(mm[k]);
      mm[k] = half ? o + mm[k] : mm[k] + o;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const double o = pair_xor(ss[k]);
      ss[k] = half ? o + ss[k] : ss[k] + o;
    }
    if (M) {
      const double o = pair_xor(K);
      K = half ? o + K : K + o;
    }
    }
    const double xx = ss[1] + ss[2], yy = ss[0] + ss[2], zz = ss[0] + ss[1];
    const double xy = -ss[3], xz = -ss[4], yz = -ss[5];
    // rotation matrix D(alpha, n), row major
    const double n[3] = {axis[0], axis[1], axis[2]};
    const double ca = B.ca, sa = B.sa, omc = B.omc;
    const double D[9] = {ca + omc * n[0] * n[0],        omc * n[0] * n[1] - sa * n[2],
                         omc * n[0] * n[2] + sa * n[1], omc * n[1] * n[0] + sa * n[2],
                         ca + omc * n[1] * n[1],        omc * n[1] * n[2] - sa * n[0],
                         omc * n[2] * n[0] - sa * n[1], omc * n[2] * n[1] + sa * n[0],
                         ca + omc * n[2] * n[2]};
    // (M D^T)_bc = row b of M . row c of D
    auto md = [&](int b2, int c) {
      return mm[3 * b2] * D[3 * c] + mm[3 * b2 + 1] * D[3 * c + 1] + mm[3 * b2 + 2] * D[3 * c + 2];
    };
    const double LD[3] = {md(1, 2) - md(2, 1), md(2, 0) - md(0, 2), md(0, 1) - md(1, 0)};
    double a9[3] = {(mm[5] - mm[7]) - LD[0], (mm[6] - mm[2]) - LD[1], (mm[1] - mm[3]) - LD[2]};
    if (nf == 2) {
      const double hm = 0.5 * (xx + yy + zz);
      if (hm > 0.0) {
        const double ih = 1.0 / hm;
#pragma unroll
        for (int k = 0; k < 3; ++k) om[k] = a9[k] * ih;
      }
    } else if (nf >= 3) {
      // adjugate of the symmetric I
      const double c00 = yy * zz - yz * yz, c01 = xz * yz - xy * zz, c02 = xy * yz - yy * xz;
      const double c11 = xx * zz - xz * xz, c12 = xy * xz - xx * yz, c22 = xx * yy - xy * xy;
      const double det = xx * c00 + xy * c01 + xz * c02;
      if (det != 0.0) {
        const double id = 1.0 / det;
        om[0] = (c00 * a9[0] + c01 * a9[1] + c02 * a9[2]) * id;
        om[1] = (c01 * a9[0] + c11 * a9[1] + c12 * a9[2]) * id;
        om[2] = (c02 * a9[0] + c12 * a9[1] + c22 * a9[2]) * id;
      }
    }
    if constexpr (M) {
      // the thermostat scales the corrected relative velocities D u_i +
      // omega x r_ic to the drawn energy; their kinetic energy is
      // K + m (2 omega . L_D + omega . I omega), K that of the u_i
      if (Ek > 0.0) {
        const double Io[3] = {xx * om[0] + xy * om[1] + xz * om[2],
                              xy * om[0] + yy * om[1] + yz * om[2],
                              xz * om[0] + yz * om[1] + zz * om[2]};
        double cr = 0.0, q = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          cr = cr + om[k] * LD[k];
          q = q + om[k] * Io[k];
        }
        const double K2 = K + m * (2.0 * cr + q);
        if (K2 > 0.0) kappa = sqrt((2.0 * Ek) / K2);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) om[k] = kappa * om[k];
    }
  }
  if (!valid || half) return;
  // cells that do not collide keep v exactly (kappa = 0 / coll = 0 marks them)
  const bool coll = nf > 0 && ntot >= 2;
  if constexpr (A) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      out->om[k] = coll ? om[k] : 0.0;
    }
  }
  if constexpr (F == kFormSplit) {
    const double n[3] = {axis[0], axis[1], axis[2]};
    const double ca = B.ca, sa = B.sa, omc = B.omc;
    const double R[9] = {ca + omc * n[0] * n[0],        omc * n[0] * n[1] - sa * n[2],
                         omc * n[0] * n[2] + sa * n[1], omc * n[1] * n[0] + sa * n[2],
                         ca + omc * n[1] * n[1],        omc * n[1] * n[2] - sa * n[0],
                         omc * n[2] * n[0] - sa * n[1], omc * n[2] * n[1] + sa * n[0],
                         ca + omc * n[2] * n[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) out->V[k] = coll ? (float)V[k] : 0.0f;
#pragma unroll
    for (int k = 0; k < 9; ++k) out->R[k] = coll ? (float)(kappa * R[k]) : 0.0f;
    out->coll = coll ? 1.0f : 0.0f;
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      out->V[k] = coll ? V[k] : 0.0;
      out->n[k] = coll ? axis[k] : 0.0;
    }
    out->kappa = coll ? kappa : 0.0;
  }
}

// Tile index of the it-th work item of this workgroup (XCD-aware order:
// workgroup b runs on XCD b % 8; each XCD takes a contiguous part of the tile
// list, which the host ordered so that neighbouring rows are close in it).
struct TileWalk {
  uint32_t first, stride, per_xcd, xcd, ntiles;
  __device__ uint32_t tile(uint32_t it) const {
    if (per_xcd) {
      if (it >= per_xcd) return 0xffffffffu;
      const uint32_t t = xcd * per_xcd + it;
      return t < ntiles ? t : 0xffffffffu;
    }
    return it < ntiles ? it : 0xffffffffu;
  }
};

// Sources of a tile: its runs, then (more than maxr runs) its chains, one per
// lane.  f(i, active) is called by the whole wavefront for up to 64 slots at
// a time.
template <class Fn>
__device__ __forceinline__ void for_each_source(const Dev& d, uint32_t in, uint32_t tid,
                                                uint32_t nrun, uint32_t lane, Fn f) {
  const uint32_t nt = min(nrun, d.maxr);
  for (uint32_t r = 0; r < nt; ++r) {
    const Run run = d.runs[in][(size_t)tid * d.maxr + r];
    const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)run.count);
    for (uint32_t q0 = 0; q0 < n; q0 += 64) {
      const uint32_t i = run.start + q0 + lane;
      f(i, q0 + lane < n && i < d.ntot);
    }
  }
  if (nrun <= d.maxr) return;
  uint32_t i = lane < d.maxr ? d.rhead[in][(size_t)tid * d.maxr + lane] : kNoSlot;
  while (__ballot(i < d.ntot)) {
    const bool on = i < d.ntot;
    f(i, on);
    i = on ? d.rnext[in][i] : kNoSlot;
  }
}

// One wavefront per tile (persistent grid).  The particles stay in registers,
// four per lane, from the gather to the store; LDS holds what lanes exchange:
// the ids of each cell for the canonical order, the velocities in that order
// for the cell sums, the cells' records.  That is 10 KB in FP64 (it was
// 18.8 KB with the positions and the binning of single cells in LDS), so
// registers decide the waves per SIMD.  What bounds it is the chain of one
// pass (runs, gather, ids, sums, rotation, atomics, stores; the wavefronts wait
// half of the time) against HBM traffic at 0.8 of the copy rate.  At 256^3
// cells of 10 particles a step takes 4.4 ms (FP64), 4.6 (thermostat), 3.4
// (split, thermostat) and 6.2 (SRD+a, thermostat), where a collide of sorted
// slots with a scan and a scatter beside it took 6.9, 7.3, 6.5 and 8.8.
// SRD+a is bound by LDS: what shares its place there (ids and positions, the
// energy terms added along with the moments) took it from 20.4 to 16.3 KB, ten
// wavefronts per CU instead of eight, and from 7.06 to 6.20 ms (split 17.3 to
// 13.2 KB, 6.02 to 5.22).  With fixed-point sums it needs the registers of two
// wavefronts per SIMD (105 spills at three).
template <int F, bool W, bool M, bool A, bool X, bool E>
__global__ __launch_bounds__(kCollideThreads) __attribute__((amdgpu_waves_per_eu(A && X ? 2 : (A || F == kFormF64 ? 3 : 4), F == kFormF64 ? 3 : 8)))
void k_collide(Dev d, Side w, uint32_t j, uint32_t ntiles, int xcd_remap) {
  using Fm = Form<F>;
  using Vs = typename Fm::Vs;
  constexpr int NT = kCollideThreads;
  constexpr int NS = kTileCap / kCollideThreads;
  static_assert(kTileMaxCells < NT, "one lane per cell offset (nc + 1) of a tile");
  static_assert(2 * kTileMaxCells <= NT, "two lanes per cell in the cell sums");
  static_assert(kMaxRuns <= NT, "one lane per run of a tile");
  static_assert(NT == 64, "the workgroup is one wavefront (see wave_sync)");
  // id segments, each padded to a multiple of four (read four at a time);
  // before the ids: run marks and source slots; after them: far tiles
  constexpr int kIds = kTileCap + 4 * kTileMaxCells;
  // (SRD+a: in the place of the positions, which come after the ids and go
  // before the far tiles)
  __shared__ __align__(16) uint32_t s_ids[A ? 4 : kIds];
  __shared__ uint32_t s_cnt[kTileMaxCells];
  __shared__ uint32_t s_off[kTileMaxCells + 1];  // offsets: plain | padded << 16
  __shared__ uint32_t s_delta[kMaxRuns];
  __shared__ uint32_t s_grp[kGroups + 1];
  __shared__ uint32_t s_tot[kTileMaxCells + 1];  // offsets of the whole tile (several passes)
  __shared__ __align__(16) Vs s_v[3][kTileCap];  // streamed velocities, canonical order
  // SRD+a: cell-frame positions, alike
  __shared__ __align__(16) double s_x[A ? 3 : 1][A ? kTileCap : 1];
  static_assert(sizeof(double) * 3 * kTileCap >= sizeof(uint32_t) * kIds, "ids fit");
  uint32_t* const s_id = A ? (uint32_t*)&s_x[0][0] : s_ids;
  // kinetic-energy terms: in the place of the velocities (SRD+a, which reads
  // them after the momentum, adds the terms along with its moments)
  static_assert(sizeof(Vs) * 3 * kTileCap >= sizeof(double) * kTileCap, "terms fit");
  double* const s_k = (double*)&s_v[0][0];
  // mean velocities in FP64 where the cell's record has FP32 but the sums were
  // not FP32 ones
  constexpr bool kWide = F == kFormSplit && X;
  __shared__ double s_mean[kWide ? 3 : 1][kWide ? kTileMaxCells : 1];
  __shared__ typename CellRec<F, A>::T s_cell[kTileMaxCells];

  // side work: the cells still to draw, in the place of the velocities
  static_assert(sizeof(Vs) * 3 * kTileCap >= sizeof(uint16_t) * kDrawList, "list fits");
  __shared__ uint32_t s_dused;

  const uint64_t t = as_const(d.ctrl)->step + j;
  const uint32_t cur = (as_const(d.ctrl)->cur + j) & 1u;
  const uint32_t tcu = counter_set(d, j), tnx = tcu == 2u ? 0u : tcu + 1u,
                 tcl = tnx == 2u ? 0u : tnx + 1u;
  const int32_t R = as_const(d.ctrl)->reorder;
  // side work: every w.period-th group of eight workgroups (one per XCD) until
  // it is done
  const uint32_t group = blockIdx.x / 8u, turn = group / w.period;
  if (turn * 8u < w.blocks && group - turn * w.period == w.period - 1u) {
    DrawList dl{(uint16_t*)&s_v[0][0], &s_dused, 0u};
    side_work<W, M>(d, w, turn * 8u + blockIdx.x % 8u, t + 1, cur ^ 1u, dl);
    return;
  }
  const uint32_t block = blockIdx.x - min(turn * 8u, w.blocks), blocks = gridDim.x - w.blocks;
  // the state is always written into the other buffer; logical indices are
  // renumbered to the canonical (cell, index) order on reorder steps
  const bool renumber = R > 0 && (t + 1) % (uint64_t)R == 0;
  const uint32_t nxt = cur ^ 1u;
  const StatePtrs in = d.S[cur];
  const StatePtrs out = d.S[nxt];
  uint32_t err = 0;
  const uint32_t lane = threadIdx.x;
  const uint32_t maxr = d.maxr;

  TileWalk walk;
  walk.ntiles = ntiles;
  walk.first = block;
  walk.stride = blocks;
  walk.per_xcd = 0;
  walk.xcd = 0;
  if (xcd_remap && blocks % 8 == 0) {  // w.blocks is a multiple of 8
    walk.xcd = block % 8;
    walk.per_xcd = (ntiles + 7) / 8;
    walk.first = block / 8;
    walk.stride = blocks / 8;
  }

  // Software pipeline over tiles: the run list and the output position are
  // fetched one tile ahead.
  struct Ahead {
    uint32_t nrun, np, base;
    Run run;
  };
  auto fetch = [&](const Tile& T, Ahead& a) {
    const unsigned long long c = as_const(d.tcnt[tcu])[T.tid];
    a.nrun = (uint32_t)c;
    a.np = (uint32_t)(c >> 32);
    if (w.direct) {  // few tiles, one a wavefront: its own prefix
      uint32_t sum = 0;
#pragma unroll 4
      for (uint32_t i = lane; i < T.tid; i += 64) sum += (uint32_t)(d.tcnt[tcu][i] >> 32);
      a.base = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_dpp(sum), 63);
      if (lane == 0) d.toff[T.tid] = a.base;
    } else {
      a.base = as_const(d.toff)[T.tid];
    }
    a.run = Run{0u, 0u};
    if (lane < min(a.nrun, maxr)) a.run = d.runs[cur][(size_t)T.tid * maxr + lane];
  };

  uint32_t it = walk.first;
  uint32_t tcur = walk.tile(it);
  Tile T, Tn;
  Ahead cu, ah;
  if (tcur != 0xffffffffu) {
    T = load_tile(d.tiles, tcur);
    fetch(T, cu);
  }

  while (tcur != 0xffffffffu) {
    BoxRef B = as_const(d.boxes)[T.box];
    const MPC_AS4 BoxStep& bs = as_const(d.bstep[cur])[T.box];
    const uint32_t tnext = walk.tile(it + walk.stride);
    // tiles lie inside one row: (x0 .. x0 + nc - 1, y0, z0)
    const int x0 = (int)T.x0, y0 = (int)T.y0, z0 = (int)T.z0, nc = (int)T.nc;
    const int L0 = B.L[0], L1 = B.L[1], L2 = B.L[2];
    // the tiles before and after it in its row
    const int xn = x0 + nc >= L0 ? 0 : x0 + nc, ncn = min((int)B.T, L0 - xn);
    const int xp = x0 == 0 ? (int)((B.ntx - 1) * B.T) : x0 - (int)B.T;
    const int ncp = min((int)B.T, L0 - xp);
    const int wy = bs.w[0], wz = bs.w[1];
    const double snext[3] = {bs.sn[0], bs.sn[1], bs.sn[2]};
    const double st[3] = {bs.s[0], bs.s[1], bs.s[2]};
    const double d1 = E ? bs.d1 : 0.0, d2 = E ? bs.d2 : 0.0;
    bool fetched = tnext == 0xffffffffu;
    if (lane == 0) d.tcnt[tcl][T.tid] = 0ull;  // counted up by the next step

    // local cell of a streamed particle: its row is known (the tile was found
    // from the same numbers); out of range only after an error
    auto local_cell = [&](const typename Fm::P& p) -> uint32_t {
      const uint32_t lc = (uint32_t)(Fm::cell_x(p, st, B, d1, E && B.le) - x0);
      if (lc >= (uint32_t)nc) {
        err |= kErrKey;
        return 0u;
      }
      return lc;
    };

    // a tile of more than one pass: particles per cell first
    const bool slow = cu.np > (uint32_t)kTileCap;
    if (slow) {
      wave_sync();
      if (lane < (uint32_t)kTileMaxCells) s_cnt[lane] = 0u;
      wave_sync();
      for_each_source(d, cur, T.tid, cu.nrun, lane, [&](uint32_t i, bool on) {
        if (on) {
          typename Fm::P p;
          typename Fm::Vv v;
          Fm::load(in, i, p, v);
          Fm::template stream<W>(p, v, B, d1, E && B.le);
          atomicAdd(&s_cnt[local_cell(p)], 1u);
        }
      });
      wave_sync();
      const uint32_t n = lane < (uint32_t)kTileMaxCells ? s_cnt[lane] : 0u;
      const uint32_t inc = wave_scan_dpp(n);
      if (lane <= (uint32_t)kTileMaxCells) s_tot[lane] = inc - n;
      wave_sync();
    }

    uint32_t cs = 0, base = cu.base;
    do {
      uint32_t ii[NS], np, ce = (uint32_t)nc;
      if (slow) {
        const uint32_t b = s_tot[cs];
        // largest ce in (cs, nc] with at most one pass of particles
        if (s_tot[nc] - b > (uint32_t)kTileCap) {
          uint32_t lo = cs + 1, hi = (uint32_t)nc;
          while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) / 2;
            if (s_tot[mid] - b <= (uint32_t)kTileCap) {
              lo = mid;
            } else {
              hi = mid;
            }
          }
          ce = lo;
        }
        np = (uint32_t)__builtin_amdgcn_readfirstlane((int)(s_tot[ce] - b));
        ce = (uint32_t)__builtin_amdgcn_readfirstlane((int)ce);
        if (lane < (uint32_t)kTileMaxCells) s_cnt[lane] = 0u;
        wave_sync();
        if (np > (uint32_t)kTileCap) {
          // one cell beyond capacity: its particles are streamed and binned
          // for the next step, each a run of its own, and do not collide
          err |= kErrCellOverflow;
          for_each_source(d, cur, T.tid, cu.nrun, lane, [&](uint32_t i, bool on) {
            if (on) {
              typename Fm::P p;
              typename Fm::Vv v;
              uint32_t id;
              Fm::load_all(in, i, p, v, id);
              Fm::template stream<W>(p, v, B, d1, E && B.le);
              if (local_cell(p) == cs) {
                const uint32_t j = base + atomicAdd(&s_cnt[0], 1u);
                if (j < d.ntot) {
                  Fm::store_all(out, j, p, v, renumber ? j : id);
                  Fm::template stream<W>(p, v, B, d2, E && B.le);
                  int c[3];
                  Fm::template coords<W>(p, snext, B, c, err, d2, E && B.le);
                  push_run(d, nxt, tnx, tile_of(B, c), j, 1u);
                }
              }
            }
          });
          base += np;
          cs = ce;
          wave_sync();
          continue;
        }
        // source slots of the pass, cell by cell
        for_each_source(d, cur, T.tid, cu.nrun, lane, [&](uint32_t i, bool on) {
          if (on) {
            typename Fm::P p;
            typename Fm::Vv v;
            Fm::load(in, i, p, v);
            Fm::template stream<W>(p, v, B, d1, E && B.le);
            const uint32_t lc = local_cell(p);
            if (lc >= cs && lc < ce) {
              const uint32_t q = s_tot[lc] - b + atomicAdd(&s_cnt[lc], 1u);
              if (q < (uint32_t)kTileCap) s_id[q] = i;
            }
          }
        });
        wave_sync();
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint32_t q = lane + k * NT;
          ii[k] = q < np ? s_id[q] : 0u;
        }
        wave_sync();
      } else if (__builtin_expect(cu.nrun > maxr, 0)) {
        // runs of the table by their lanes, then the chains, a lane each
        const uint32_t inc = wave_scan_dpp(cu.run.count);
        const uint32_t pre = inc - cu.run.count;
        wave_sync();
        for (uint32_t q = 0; q < cu.run.count && pre + q < (uint32_t)kTileCap; ++q)
          s_id[pre + q] = cu.run.start + q;
        uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        uint32_t i = lane < maxr ? d.rhead[cur][(size_t)T.tid * maxr + lane] : kNoSlot;
        while (const uint64_t m = __ballot(i < d.ntot)) {
          const uint32_t q = n + lanes_below(m);
          n += (uint32_t)__popcll(m);
          if (i < d.ntot) {
            if (q < (uint32_t)kTileCap) s_id[q] = i;
            i = d.rnext[cur][i];
          }
        }
        np = min(n, (uint32_t)kTileCap);
        if (np != cu.np) err |= kErrKey;
        wave_sync();
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint32_t q = lane + k * NT;
          ii[k] = q < np ? s_id[q] : 0u;
        }
        wave_sync();
      } else {
        // slots of the runs, one after the other: a mark at the first entry
        // of each run, and per run the distance from entry to slot
        const uint32_t inc = wave_scan_dpp(cu.run.count);
        const uint32_t pre = inc - cu.run.count;
        np = min((uint32_t)__builtin_amdgcn_readlane((int)inc, 63), (uint32_t)kTileCap);
        if (np != cu.np) err |= kErrKey;
        wave_sync();
#pragma unroll
        for (int k = 0; k < NS; ++k) s_id[lane + k * NT] = 0u;
        wave_sync();
        if (cu.run.count && pre < (uint32_t)kTileCap) {
          s_id[pre] = 1u;
          s_delta[lane] = cu.run.start - pre;
        }
        wave_sync();
        uint32_t before = 0;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint32_t q = lane + k * NT;
          const bool mk = s_id[q] != 0u;
          const uint64_t m = __ballot(mk);
          const uint32_t r = before + lanes_below(m) + (mk ? 1u : 0u);
          before += (uint32_t)__popcll(m);
          ii[k] = q < np ? s_delta[r - 1u] + q : 0u;
        }
        wave_sync();
      }

      if (np == 0u) {
        cs = ce;
        continue;
      }

      // gather (one memory round trip), stream, local cells
      typename Fm::P p[NS];
      typename Fm::Vv v[NS];
      uint32_t idk[NS], meta[NS];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * NT;
        idk[k] = 0u;
        if (q < np) Fm::load_all(in, ii[k] < d.ntot ? ii[k] : 0u, p[k], v[k], idk[k]);
      }
      // with the gather: the draws of cell cs + j, by lanes 2j and 2j + 1
      double axis[3], z0g;
      uint32_t least;
      {
        const uint32_t c = T.c0 + min(cs + (lane >> 1), (uint32_t)nc - 1u);
        const double2* r = (const double2*)d.draws[cur] + 2 * (size_t)c;
        const double2 r0 = r[0], r1 = r[1];
        axis[0] = r0.x;
        axis[1] = r0.y;
        axis[2] = r1.x;
        z0g = r1.y;
        least = M ? d.least[cur][c] : 0u;
      }
      if (!fetched) {
        fetched = true;
        Tn = load_tile(d.tiles, tnext);
        fetch(Tn, ah);
      }
      if (lane < (uint32_t)kTileMaxCells) s_cnt[lane] = 0u;
      if (lane < (uint32_t)kGroups + 1u) s_grp[lane] = 0u;
      for (uint32_t q = lane; q < (uint32_t)kIds / 4; q += NT)
        ((uint4*)s_id)[q] = make_uint4(kNoSlot, kNoSlot, kNoSlot, kNoSlot);
      wave_sync();
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * NT;
        meta[k] = 0u;
        if (q < np) {
          Fm::template stream<W>(p[k], v[k], B, d1, E && B.le);
          const uint32_t lc = local_cell(p[k]);
          meta[k] = lc | atomicAdd(&s_cnt[lc], 1u) << 8;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_sync();
      {
        const uint32_t n = lane < (uint32_t)kTileMaxCells ? s_cnt[lane] : 0u;
        const uint32_t w = n | ((n + 3u) & ~3u) << 16;
        const uint32_t inc = wave_scan_dpp(w);
        if (lane <= (uint32_t)kTileMaxCells) s_off[lane] = inc - w;
      }
      wave_sync();
      // canonical position: rank by logical index inside the cell
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * NT;
        if (q < np) s_id[(s_off[meta[k] & 0xffu] >> 16) + (meta[k] >> 8)] = idk[k];
      }
      wave_sync();
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * NT;
        if (q < np) {
          const uint32_t lc = meta[k] & 0xffu;
          const uint32_t o = s_off[lc], o1 = s_off[lc + 1];
          const uint32_t b = o & 0xffffu;
          uint32_t r = 0;
          for (uint32_t a = o >> 16; a < o1 >> 16; a += 4) {
            const uint4 w = *(const uint4*)&s_id[a];
            r += (w.x < idk[k] ? 1u : 0u) + (w.y < idk[k] ? 1u : 0u) + (w.z < idk[k] ? 1u : 0u) +
                 (w.w < idk[k] ? 1u : 0u);
          }
          const uint32_t qc = min(b + r, (uint32_t)kTileCap - 1u);
          if constexpr (E) {
            const int side = B.le ? Fm::le_side(p[k], st[2], B) : 0;
            if ((o1 & 0xffffu) - b >= 2u) {
              // a colliding cell across a z face: its image's velocity frame
              if (side < 0) v[k].v[0] = (Vs)((double)v[k].v[0] - B.leu);
              if (side > 0) v[k].v[0] = (Vs)((double)v[k].v[0] + B.leu);
            }
          }
          s_v[0][qc] = v[k].v[0];
          s_v[1][qc] = v[k].v[1];
          s_v[2][qc] = v[k].v[2];
          meta[k] = lc | qc << 8;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_sync();
      if constexpr (A) {
        // after every lane's last look at the ids
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint32_t qc = meta[k] >> 8;
          if (lane + k * NT < np) {
            // under Lees-Edwards shear a particle taken as its image (side
            // -1 / +1) sits at x - d / x + d
            double xq = (double)Fm::pos(p[k], 0);
            if constexpr (E) {
              const int side = B.le ? Fm::le_side(p[k], st[2], B) : 0;
              if (side < 0) xq = xq - d1;
              if (side > 0) xq = xq + d1;
            }
            s_x[0][qc] = frame_pos(xq, st[0]);
            s_x[1][qc] = frame_pos(Fm::pos(p[k], 1), st[1]);
            s_x[2][qc] = frame_pos(Fm::pos(p[k], 2), st[2]);
          }
        }
        wave_sync();
      }

      // mean velocities (and centres of mass): a lane per cell and half for the
      // three components, or per component too
      const uint32_t ncell = ce - cs;
      const bool phantoms = W && !B.slip && wall_fraction(st[2], z0 - 1, L2) > 0.0;
      auto means = [&](auto width, uint32_t cell, uint32_t k0, bool valid) {
        constexpr int N = decltype(width)::value;
        const uint32_t half = lane & 1u, c = valid ? cell : cs;
        const uint32_t b = s_off[c] & 0xffffu, n = valid ? (s_off[c + 1] & 0xffffu) - b : 0u;
        const uint32_t mid = b + (n + 1) / 2, qb = half ? mid : b, qe = half ? b + n : mid;
        uint32_t nph = 0;
        double pv[N], V[N];
        const Vs* vs[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
          pv[k] = 0.0;
          vs[k] = s_v[k0 + k];
        }
        if (W && phantoms && n) {
          const PhantomSums& ph = d.phs[cur][T.c0 + c];
          nph = (uint32_t)ph.n;
#pragma unroll
          for (int k = 0; k < N; ++k) pv[k] = ph.v[k0 + k];
        }
        mean_velocity<F, X, N>(vs, B.mass, qb, qe, half, n + nph, nph, pv, err, V);
        if (valid && !half) {
#pragma unroll
          for (int k = 0; k < N; ++k) {
            if constexpr (kWide) {
              s_mean[k0 + k][c] = V[k];
            } else {
              s_cell[c].V[k0 + k] = (decltype(s_cell[c].V[0] + 0))V[k];
            }
          }
        }
        if constexpr (A) {
          const double* xs[N];
          double rc[N];
#pragma unroll
          for (int k = 0; k < N; ++k) xs[k] = s_x[k0 + k];
          half_sums<X, false>(xs, 1.0, qb, qe, half, err, rc);
          if (valid && !half) {
#pragma unroll
            for (int k = 0; k < N; ++k) s_cell[c].rc[k0 + k] = rc[k] / (double)(n ? n : 1u);
          }
        }
      };
      if (6u * ncell <= (uint32_t)NT) {
        const uint32_t u = lane >> 1;
        const uint32_t k0 = (u >= ncell ? 1u : 0u) + (u >= 2u * ncell ? 1u : 0u);
        means(Width<1>{}, cs + u - k0 * ncell, k0, u < 3u * ncell);
      } else {
        means(Width<3>{}, cs + (lane >> 1), 0u, (lane >> 1) < ncell);
      }
      wave_sync();
      auto mean_of = [&](uint32_t c, int k) -> double {
        if constexpr (kWide) {
          return s_mean[k][c];
        } else {
          return (double)s_cell[c].V[k];
        }
      };
      if constexpr (M && !A) {
        // kinetic-energy terms by the particles' lanes
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint32_t q = lane + k * NT;
          if (q < np) {
            const uint32_t lc = meta[k] & 0xffu;
            const double dx = (double)v[k].v[0] - mean_of(lc, 0),
                         dy = (double)v[k].v[1] - mean_of(lc, 1),
                         dz = (double)v[k].v[2] - mean_of(lc, 2);
            s_k[meta[k] >> 8] = B.mass * (dx * dx + dy * dy + dz * dz);
          }
        }
        wave_sync();
      }
      // the rest: two lanes per cell (lanes 2j and 2j + 1 for cell cs + j)
      {
        const uint32_t j = lane >> 1;
        const uint32_t c = cs + j;
        const bool valid = c < ce;
        const uint32_t b = valid ? s_off[c] & 0xffffu : 0u, e = valid ? s_off[c + 1] & 0xffffu : 0u;
        // thermostat: target energy E_k = kT * Gamma(3 (n - 1) / 2), n with
        // phantoms; 0 means "no scaling"
        const uint32_t nph = W && phantoms && e > b ? (uint32_t)d.phs[cur][T.c0 + c].n : 0u;
        double Ek = 0.0;
        if constexpr (M) {
          const uint32_t n = e - b + nph;
          const bool draw = e > b && n >= 2u;
          if (draw) {
            double z = z0g;
            bool ok = n >= (least & 0xffffu);
            if (!ok) {  // the first listed attempt that n accepts
              const Attempt* seg =
                  d.later[cur] + (size_t)((T.c0 + c) / d.drawb) * later_seg(d.drawb);
              uint32_t a = least >> 16;
              while (a && !ok) {
                const Attempt at = seg[a];
                z = at.z;
                ok = n >= at.least;
                a = at.next;
              }
            }
            const GammaDC g = gamma_dc(n);
            const double vv = 1.0 + g.c * z;
            if (ok) Ek = B.kT * (g.d * (vv * vv * vv));
          }
        }
        auto* rec = &s_cell[valid ? c : cs];
        const uint32_t cv = valid ? c : cs;
        const double V[3] = {mean_of(cv, 0), mean_of(cv, 1), mean_of(cv, 2)};
        double rc[3] = {0.0, 0.0, 0.0};
        if constexpr (A) {
#pragma unroll
          for (int k = 0; k < 3; ++k) rc[k] = rec->rc[k];
        }
        cell_work<F, W, M, A, X>(B, axis, Ek, W ? d.phs[cur] + T.c0 + (valid ? c : 0u) : nullptr,
                                 nph, s_v[0], s_v[1], s_v[2], s_x[0], s_x[A ? 1 : 0],
                                 s_x[A ? 2 : 0], s_k, V, rc, b, e, lane & 1u, valid, rec, err);
      }
      wave_sync();

      // rotate + scale, gravity; the group of each particle: the next step's
      // tile, one of three in each of nine rows, or "far"; its place there
      uint32_t gk[NS];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * NT;
        gk[k] = 0u;
        __builtin_amdgcn_sched_barrier(0);
        if (q < np) {
          const uint32_t lc = meta[k] & 0xffu;
          const auto& C = s_cell[lc];
          int side = 0;
          if constexpr (E) side = B.le ? Fm::le_side(p[k], st[2], B) : 0;
          auto& vv = v[k].v;
          if constexpr (F == kFormSplit) {
            if (C.coll != 0.0f) {
              const float u[3] = {vv[0] - C.V[0], vv[1] - C.V[1], vv[2] - C.V[2]};
#pragma unroll
              for (int a = 0; a < 3; ++a)
                vv[a] = C.V[a] + fmaf(C.R[3 * a], u[0], fmaf(C.R[3 * a + 1], u[1], C.R[3 * a + 2] * u[2]));
              if constexpr (A) {
                // omega x r_ic in FP64 (|omega| is large in ill-conditioned
                // cells), added to the FP32 rotation result with one rounding
                double xq = (double)Fm::pos(p[k], 0);
                if constexpr (E) {
                  if (side < 0) xq = xq - d1;
                  if (side > 0) xq = xq + d1;
                }
                const double r[3] = {frame_pos(xq, st[0]) - C.rc[0],
                                     frame_pos(Fm::pos(p[k], 1), st[1]) - C.rc[1],
                                     frame_pos(Fm::pos(p[k], 2), st[2]) - C.rc[2]};
                vv[0] = (float)((double)vv[0] + (C.om[1] * r[2] - C.om[2] * r[1]));
                vv[1] = (float)((double)vv[1] + (C.om[2] * r[0] - C.om[0] * r[2]));
                vv[2] = (float)((double)vv[2] + (C.om[0] * r[1] - C.om[1] * r[0]));
              }
              if constexpr (E) {  // leave the Lees-Edwards image frame
                if (side < 0) vv[0] = (float)((double)vv[0] + B.leu);
                if (side > 0) vv[0] = (float)((double)vv[0] - B.leu);
              }
            }
            if (B.grav) {
#pragma unroll
              for (int a = 0; a < 3; ++a) vv[a] = vv[a] + (float)B.gh[a];
            }
          } else {
            double w[3] = {(double)vv[0], (double)vv[1], (double)vv[2]};
            if (C.kappa != 0.0) {
              const double u[3] = {w[0] - C.V[0], w[1] - C.V[1], w[2] - C.V[2]};
              const double nd[3] = {C.n[0], C.n[1], C.n[2]};
              double r[3];
              rotate<double>(B.ca, B.sa, B.omc, nd, u, r);
#pragma unroll
              for (int a = 0; a < 3; ++a) w[a] = C.V[a] + C.kappa * r[a];
              if constexpr (A) {
                double xq = (double)Fm::pos(p[k], 0);
                if constexpr (E) {
                  if (side < 0) xq = xq - d1;
                  if (side > 0) xq = xq + d1;
                }
                const double rr[3] = {frame_pos(xq, st[0]) - C.rc[0],
                                      frame_pos(Fm::pos(p[k], 1), st[1]) - C.rc[1],
                                      frame_pos(Fm::pos(p[k], 2), st[2]) - C.rc[2]};
                w[0] = w[0] + (C.om[1] * rr[2] - C.om[2] * rr[1]);
                w[1] = w[1] + (C.om[2] * rr[0] - C.om[0] * rr[2]);
                w[2] = w[2] + (C.om[0] * rr[1] - C.om[1] * rr[0]);
              }
              if constexpr (E) {  // leave the Lees-Edwards image frame
                if (side < 0) w[0] = w[0] + B.leu;
                if (side > 0) w[0] = w[0] - B.leu;
              }
            }
            if (B.grav) {
#pragma unroll
              for (int a = 0; a < 3; ++a) w[a] = w[a] + B.gh[a];
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) vv[a] = (Vs)w[a];
          }
          typename Fm::P pn = p[k];
          typename Fm::Vv vn = v[k];
          Fm::template stream<W>(pn, vn, B, d2, E && B.le);
          int c[3];
          Fm::template coords<W>(pn, snext, B, c, err, d2, E && B.le);
          const int seg = (unsigned)(c[0] - x0) < (unsigned)nc    ? 1
                          : (unsigned)(c[0] - xp) < (unsigned)ncp ? 0
                          : (unsigned)(c[0] - xn) < (unsigned)ncn ? 2
                                                                  : 3;
          int ry = c[1] - y0 - wy, rz = c[2] - z0 - wz;
          if ((unsigned)ry >= 3u || (!W && (unsigned)rz >= 3u)) {
            ry = wrap1(ry, L1);
            if (!W) rz = wrap1(rz, L2);
          }
          uint32_t g = (uint32_t)((rz * 3 + ry) * 3 + seg);
          if (!((unsigned)ry < 3u && (unsigned)rz < 3u && seg < 3)) {
            g = (uint32_t)kGroups;
            s_id[q] = tile_of(B, c);
          }
          gk[k] = g | atomicAdd(&s_grp[g], 1u) << 8;
        }
      }
      wave_sync();
      // the groups one after the other in the pass's output; a run for each
      uint32_t far0, nfar;
      uint32_t gn = 0, gpre, gdest = kNoSlot;
      {
        gn = lane < (uint32_t)kGroups + 1u ? s_grp[lane] : 0u;
        gpre = wave_scan_dpp(gn) - gn;
        if (lane < (uint32_t)kGroups + 1u) s_grp[lane] = gpre;
        far0 = (uint32_t)__builtin_amdgcn_readlane((int)gpre, kGroups);
        nfar = (uint32_t)__builtin_amdgcn_readlane((int)gn, kGroups);
        if (lane < (uint32_t)kGroups && gn) {
          const int row = (int)lane / 3, seg = (int)lane - 3 * row;
          const int rz = row / 3, ry = row - 3 * rz;
          const int y = wrap1(y0 + wy + ry, L1);
          const int z = W ? z0 + wz + rz : wrap1(z0 + wz + rz, L2);
          const int xs = seg == 0 ? xp : (seg == 1 ? x0 : xn);
          gdest = B.tbase + ((uint32_t)z * (uint32_t)L1 + (uint32_t)y) * B.ntx +
                  (uint32_t)xs / B.T;
        }
      }
      wave_sync();
      if (__builtin_expect(nfar != 0u, 0)) {
        // far particles: ordered by destination, a run for each, by the rank of
        // every one among all (particles of several cells a step, 64^3 FP64: with
        // the destinations found one after the other, and their chains read
        // three times, 823 us a step)
        uint32_t fd[NS];
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const uint32_t q = lane + k * NT;
          fd[k] = q < np && (gk[k] & 0xffu) == (uint32_t)kGroups ? s_id[q] : kNoSlot;
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < NS; ++k)
          if (fd[k] != kNoSlot) s_id[gk[k] >> 8] = fd[k];
        if (lane < 4u) s_id[nfar + lane] = kNoSlot;  // whole groups of four
        wave_sync();
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          if (fd[k] != kNoSlot) {
            const uint32_t me = gk[k] >> 8, f = fd[k];
            uint32_t lt = 0, eq = 0, eb = 0;
            for (uint32_t a = 0; a < nfar; a += 4) {
              const uint4 w = *(const uint4*)&s_id[a];
              const uint32_t e = (w.x == f ? 1u : 0u) | (w.y == f ? 2u : 0u) |
                                 (w.z == f ? 4u : 0u) | (w.w == f ? 8u : 0u);
              lt += (w.x < f ? 1u : 0u) + (w.y < f ? 1u : 0u) + (w.z < f ? 1u : 0u) +
                    (w.w < f ? 1u : 0u);
              eq += (uint32_t)__popc(e);
              if (a + 4 <= me) {
                eb += (uint32_t)__popc(e);
              } else if (a < me) {
                eb += (uint32_t)__popc(e & ((1u << (me - a)) - 1u));
              }
            }
            gk[k] = (uint32_t)kGroups | (lt + eb) << 8;
            if (eb == 0u) push_run(d, nxt, tnx, f, base + far0 + lt, eq);
          }
        }
      }
      if (gdest != kNoSlot) push_run(d, nxt, tnx, gdest, base + gpre, gn);
      // the pass's particles, grouped by next-step tile, into its slots;
      // logical indices: the canonical (cell, index) position on reorder steps
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * NT;
        if (q < np) {
          const uint32_t j = base + s_grp[gk[k] & 0xffu] + (gk[k] >> 8);
          if (j < d.ntot) {
            Fm::store_all(out, j, p[k], v[k], renumber ? base + (meta[k] >> 8) : idk[k]);
          } else {
            err |= kErrKey;
          }
        }
      }
      base += np;
      cs = ce;
      wave_sync();
    } while (cs < (uint32_t)nc);
    if (cu.nrun > maxr && lane < maxr) d.rhead[cur][(size_t)T.tid * maxr + lane] = kNoSlot;
    // advance the pipeline
    it += walk.stride;
    tcur = tnext;
    if (tnext != 0xffffffffu) {
      if (!fetched) {
        Tn = load_tile(d.tiles, tnext);
        fetch(Tn, ah);
      }
      T = Tn;
      cu = ah;
    }
  }
  if (err) atomicOr(&d.ctrl->err, err);
}

// Runtime flags (form, walls, thermostat, SRD+a, fixed-point sums,
// Lees-Edwards) -> the k_collide instantiation.  SRD+a next to walls runs
// with slip walls only (the host refuses it with no-slip walls).
static Side side_of(const Launch& l) {
  Side w{};
  w.nbox = l.nbox;
  w.ctot = (uint32_t)l.ctot;
  w.wcells = l.walls ? l.wcells : 0u;
  w.round32 = l.round_phantoms;
  return w;
}

struct CollideLaunchOp {
  template <int F, bool W, bool M, bool A, bool X, bool E>
  static hipError_t run(const Dev& d, const Launch& l, int*) {
    Side w = side_of(l);
    const uint32_t side = (w.nbox + 63u) / 64u + (w.wcells + 63u) / 64u +
                          (w.ctot + d.drawb - 1u) / d.drawb;
    w.direct = d.ntile <= kTileDirect && l.ntiles <= l.collide_grid;
    w.blocks = (side + 7u) / 8u * 8u;
    // spread over the launch where there are several times as many collide
    // workgroups as fit the chip (its arithmetic runs beside their memory
    // traffic), else first (it takes the longest)
    w.period = l.collide_grid > 4u * l.resident && l.collide_grid % 8u == 0u
                   ? std::max(1u, (w.blocks + l.collide_grid) / w.blocks)
                   : 1u;
    hipLaunchKernelGGL((k_collide<F, W, M, A, X, E>), dim3(w.blocks + l.collide_grid),
                       dim3(kCollideThreads), 0, l.stream, d, w, l.seq, (uint32_t)l.ntiles,
                       l.xcd_remap);
    return hipGetLastError();
  }
};
struct CollideOccOp {
  template <int F, bool W, bool M, bool A, bool X, bool E>
  static hipError_t run(const Dev&, const Launch&, int* n) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, k_collide<F, W, M, A, X, E>,
                                                        kCollideThreads, 0);
  }
};
// Lees-Edwards (E) is built for periodic boxes only.
template <class Op, int F, bool W, bool M, bool A, bool X>
static hipError_t collide_pick_e(const Dev& d, const Launch& l, int* n) {
  if constexpr (W) {
    return l.le ? hipErrorInvalidValue : Op::template run<F, W, M, A, X, false>(d, l, n);
  } else {
    return l.le ? Op::template run<F, W, M, A, X, true>(d, l, n)
                : Op::template run<F, W, M, A, X, false>(d, l, n);
  }
}
template <class Op, int F, bool W, bool M, bool A>
static hipError_t collide_pick_x(const Dev& d, const Launch& l, int* n) {
  return l.fixed ? collide_pick_e<Op, F, W, M, A, true>(d, l, n)
                 : collide_pick_e<Op, F, W, M, A, false>(d, l, n);
}
template <class Op, int F, bool W, bool M>
static hipError_t collide_pick_a(const Dev& d, const Launch& l, int* n) {
  return l.amc ? collide_pick_x<Op, F, W, M, true>(d, l, n)
               : collide_pick_x<Op, F, W, M, false>(d, l, n);
}
template <class Op, int F, bool W>
static hipError_t collide_pick_m(const Dev& d, const Launch& l, int* n) {
  return l.mbs ? collide_pick_a<Op, F, W, true>(d, l, n) : collide_pick_a<Op, F, W, false>(d, l, n);
}
template <class Op, int F>
static hipError_t collide_pick_w(const Dev& d, const Launch& l, int* n) {
  return l.walls ? collide_pick_m<Op, F, true>(d, l, n) : collide_pick_m<Op, F, false>(d, l, n);
}
template <class Op>
static hipError_t collide_dispatch(const Dev& d, const Launch& l, int* n) {
  switch (l.form) {
    case kFormF64: return collide_pick_w<Op, kFormF64>(d, l, n);
    case kFormF32: return collide_pick_w<Op, kFormF32>(d, l, n);
    case kFormSplit: return collide_pick_w<Op, kFormSplit>(d, l, n);
    default: return hipErrorInvalidValue;
  }
}

hipError_t collide_occupancy(const Launch& l, int* blocks_per_cu) {
  return collide_dispatch<CollideOccOp>(Dev{}, l, blocks_per_cu);
}

// ---------------------------------------------------------------------------
// Canonical permutation for export: sort each cell segment by logical index
// (ids[slot * stride], or the slot itself when ids is null).
// ---------------------------------------------------------------------------
__global__ void k_canon_perm(uint32_t* __restrict__ perm, const uint32_t* __restrict__ offset,
                             uint64_t ncell, uint32_t n, const uint32_t* __restrict__ ids,
                             uint32_t stride) {
  const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  const uint32_t b = offset[c], e = offset[c + 1];
  if (e > n || b > e) return;
  auto rk = [&](uint32_t slot) { return ids && slot < n ? ids[(size_t)slot * stride] : slot; };
  for (uint32_t i = b + 1; i < e; ++i) {
    const uint32_t x = perm[i];
    const uint32_t kx = rk(x);
    uint32_t j = i;
    while (j > b && rk(perm[j - 1]) > kx) {
      perm[j] = perm[j - 1];
      --j;
    }
    perm[j] = x;
  }
}

// ---------------------------------------------------------------------------
// Sampled state: the stored slots of selected logical particles, then a gather
// of their records as FP64 in cell units (the split form's cell + offset is
// exact in FP64).  A logical index with no stored slot yields NaN.  A sample
// of at most 1/32 of the box goes into a hash table of 8 to 16 entries per
// particle, and every slot looks its index up there; a larger one uses the
// inverse of the whole index array, four bytes written at random per particle
// of the box (24 ms at 384^3, where the table of 32768 takes 1 ms), because
// the table would take more memory than that.
// ---------------------------------------------------------------------------
// keys: mask + 1 entries, kNoSlot = free
__global__ __launch_bounds__(kThreads) void k_sample_insert(const uint32_t* __restrict__ lidx,
                                                            uint32_t m, uint32_t* keys,
                                                            uint32_t mask) {
  const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
  if (k >= m) return;
  const uint32_t key = lidx[k];
  uint32_t h = sample_hash(key, mask);
  for (;;) {  // at most m of 8 m entries are taken
    const uint32_t old = atomicCAS(&keys[h], kNoSlot, key);
    if (old == kNoSlot || old == key) return;
    h = (h + 1u) & mask;
  }
}
__global__ __launch_bounds__(kThreads) void k_sample_find(const uint32_t* __restrict__ id,
                                                          uint32_t id_stride, uint32_t pbase,
                                                          uint32_t np,
                                                          const uint32_t* __restrict__ keys,
                                                          uint32_t* __restrict__ slots,
                                                          uint32_t mask) {
  const uint32_t stride = gridDim.x * kThreads * 4u;
  for (uint64_t q0 = (uint64_t)blockIdx.x * kThreads * 4u; q0 < np; q0 += stride) {
    uint32_t l[4], h[4], kk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t q = q0 + k * kThreads + threadIdx.x;
      l[k] = q < np ? id[(size_t)(pbase + (uint32_t)q) * id_stride] - pbase : kNoSlot;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      h[k] = sample_hash(l[k], mask);
      kk[k] = keys[h[k]];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      while (kk[k] != kNoSlot && kk[k] != l[k]) {
        h[k] = (h[k] + 1u) & mask;
        kk[k] = keys[h[k]];
      }
      if (kk[k] != kNoSlot && l[k] < np)
        slots[h[k]] = pbase + (uint32_t)(q0 + k * kThreads + threadIdx.x);
    }
  }
}
// slot of each sampled particle (kNoSlot: none)
__global__ __launch_bounds__(kThreads) void k_sample_slots(uint32_t* __restrict__ lidx, uint32_t m,
                                                           const uint32_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ slots,
                                                           uint32_t mask) {
  const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
  if (k >= m) return;
  const uint32_t key = lidx[k];
  uint32_t h = sample_hash(key, mask);
  while (keys[h] != key) h = (h + 1u) & mask;  // every key was inserted
  lidx[k] = slots[h];
}

__global__ void k_invert_ids(const uint32_t* __restrict__ id, uint32_t id_stride, uint32_t pbase,
                             uint32_t np, uint32_t* __restrict__ inv) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < np; q += stride) {
    const uint32_t j = pbase + (uint32_t)q;
    const uint32_t l = id[(size_t)j * id_stride] - pbase;
    if (l < np) inv[l] = j;
  }
}

// slot of particle k: sel[k], or with inv the slot inv[sel[k]]
template <int F>
__global__ __launch_bounds__(kThreads) void k_gather_particles(StatePtrs S,
                                                                const uint32_t* __restrict__ inv,
                                                                uint32_t pbase, uint32_t np,
                                                                const uint32_t* __restrict__ sel,
                                                                uint32_t m, double* __restrict__ out) {
  const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
  if (k >= m) return;
  uint32_t j = sel[k];
  if (inv) j = j < np ? inv[j] : kNoSlot;
  double r[6];
  if (j == kNoSlot || j - pbase >= np) {
#pragma unroll
    for (int c = 0; c < 6; ++c) r[c] = __builtin_nan("");
  } else if constexpr (F == kFormF64) {
    const RecF64 q = ((const RecF64*)S.rec)[j];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[c] = q.x[c];
      r[3 + c] = q.v[c];
    }
  } else if constexpr (F == kFormF32) {
    const RecF32 q = ((const RecF32*)S.rec)[j];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[c] = (double)q.x[c];
      r[3 + c] = (double)q.v[c];
    }
  } else {
    const RecSplit q = ((const RecSplit*)S.rec)[j];
    int ci[3];
    split_decode(q.cell, ci);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[c] = (double)ci[c] + (double)q.o[c];
      r[3 + c] = (double)q.v[c];
    }
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) out[(uint64_t)c * m + k] = r[c];
}

// ---------------------------------------------------------------------------
// State of a box from / to FP64 arrays x[3][m], v[3][m] in physical units
// (staged on the device between the caller's host arrays and the records).
// The conversions are a few operations per value against 48 bytes over PCIe;
// made on the host, one particle after the other, they had taken 37 ms (in)
// and 68 ms (out) for the 2.6 million particles of a 64^3 box.
// ---------------------------------------------------------------------------
// *bad is set if a position is outside the box or a value is not finite.
__global__ __launch_bounds__(kThreads) void k_state_check(const BoxDev* boxes, uint32_t box,
                                                          const double* __restrict__ x,
                                                          const double* __restrict__ v, uint32_t m,
                                                          double a, uint32_t* bad) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= m) return;
  BoxRef B = as_const(boxes)[box];
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double xi = x[(size_t)k * m + i] / a;
    const bool in =
        (B.walls && k == 2) ? (xi >= 0.0 && xi <= B.Ld[k]) : (xi >= 0.0 && xi < B.Ld[k]);
    ok = ok && in && isfinite(v[(size_t)k * m + i]);
  }
  if (!ok) *bad = 1u;
}

// Particles i0 .. i0 + m - 1 of the box into its slots of the same numbers.
template <int F>
__global__ __launch_bounds__(kThreads) void k_state_pack(const BoxDev* boxes, uint32_t box,
                                                         StatePtrs S, uint32_t i0,
                                                         const double* __restrict__ x,
                                                         const double* __restrict__ v, uint32_t m,
                                                         double a) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= m) return;
  BoxRef B = as_const(boxes)[box];
  const uint32_t j = B.pbase + i0 + i;
  double xi[3], vi[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    xi[k] = x[(size_t)k * m + i] / a;
    vi[k] = v[(size_t)k * m + i] / a;
  }
  typename Form<F>::P p;
  typename Form<F>::Vv w;
  if constexpr (F == kFormF64) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      p.x[k] = xi[k];
      w.v[k] = vi[k];
    }
  } else if constexpr (F == kFormF32) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      float f = (float)xi[k];
      if (!(B.walls && k == 2) && f >= B.Lf[k]) f = nextafterf(B.Lf[k], 0.0f);
      p.x[k] = f;
      w.v[k] = (float)vi[k];
    }
  } else {
    int c[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      split_from_double(xi[k], c[k], p.o[k]);
      if (!(B.walls && k == 2) && c[k] >= B.L[k]) c[k] -= B.L[k];
      w.v[k] = (float)vi[k];
    }
    p.cell = split_encode(c);
  }
  Form<F>::store_all(S, j, p, w, j);
}

// Logical particles i0 .. i0 + m - 1 of the box (np particles from slot pbase
// on).  x[0][] holds kUnset before; an index outside the box sets *bad.
template <int F>
__global__ __launch_bounds__(kThreads) void k_state_unpack(StatePtrs S, uint32_t pbase, uint32_t np,
                                                           uint32_t i0, double* __restrict__ x,
                                                           double* __restrict__ v, uint32_t m,
                                                           double a, uint32_t* bad) {
  const uint32_t q = blockIdx.x * kThreads + threadIdx.x;
  if (q >= np) return;
  typename Form<F>::P p;
  typename Form<F>::Vv w;
  uint32_t id;
  Form<F>::load_all(S, pbase + q, p, w, id);
  const uint32_t l = id - pbase;
  if (l >= np) *bad = 1u;
  const uint32_t i = l - i0;
  if (l >= np || l < i0 || i >= m) return;
  double xi[3];
  if constexpr (F == kFormSplit) {
    int c[3];
    split_decode(p.cell, c);
#pragma unroll
    for (int k = 0; k < 3; ++k) xi[k] = (double)c[k] + (double)p.o[k];
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) xi[k] = (double)p.x[k];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    x[(size_t)k * m + i] = xi[k] * a;
    v[(size_t)k * m + i] = (double)w.v[k] * a;
  }
}

// kUnset: a NaN that no position has (unset entries mean that the logical
// indices are not a permutation).
constexpr uint64_t kUnset = 0x7ff8dead7ff8deadull;
__global__ __launch_bounds__(kThreads) void k_state_unset(double* x, uint32_t m, uint32_t* bad,
                                                          int check) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (!check && i == 0) *bad = 0u;
  if (i >= m) return;
  if (!check) {
    x[i] = __longlong_as_double((long long)kUnset);
  } else if ((uint64_t)__double_as_longlong(x[i]) == kUnset) {
    *bad = 1u;
  }
}

// ---------------------------------------------------------------------------
// FP64 state of box 0 from / to caller-owned device arrays x[3][n], v[3][n]
// in physical units (the allocation-free entry point).  Load: cell units
// (x / a, v / a) into state buffer `cur`, logical indices the identity; a
// position outside [0, L) ([0, H] on a walled z) or a non-finite value sets
// kErrKey.  Store: x[id[j]] = a * stored x[j], likewise v.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_load_f64(Dev d, const double* __restrict__ x,
                                                       const double* __restrict__ v, uint32_t n,
                                                       double a, uint32_t cur) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  BoxRef B = as_const(d.boxes)[0];
  const StatePtrs S = d.S[cur];
  bool ok = true;
  RecF64 r;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double xi = x[(uint64_t)k * n + i] / a;
    const double vi = v[(uint64_t)k * n + i] / a;
    const bool in = (B.walls && k == 2) ? (xi >= 0.0 && xi <= B.Ld[k]) : (xi >= 0.0 && xi < B.Ld[k]);
    ok = ok && in && isfinite(vi);
    r.x[k] = in ? xi : 0.0;
    r.v[k] = isfinite(vi) ? vi : 0.0;
  }
  ((RecF64*)S.rec)[i] = r;
  S.id[i] = i;
  if (!ok) atomicOr(&d.ctrl->err, kErrKey);
}

__global__ __launch_bounds__(kThreads) void k_store_f64(Dev d, double* __restrict__ x,
                                                        double* __restrict__ v, uint32_t n,
                                                        double a, uint32_t cur) {
  const uint32_t j = blockIdx.x * kThreads + threadIdx.x;
  if (j >= n) return;
  const StatePtrs S = d.S[cur];
  const uint32_t l = S.id[j];
  if (l >= n) return;
  const RecF64 r = ((const RecF64*)S.rec)[j];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    x[(uint64_t)k * n + l] = r.x[k] * a;
    v[(uint64_t)k * n + l] = r.v[k] * a;
  }
}

// ---------------------------------------------------------------------------
// Device init: positions uniform, velocities normal (INIT streams keyed by
// the init seed; counter {draw, particle, box, tag}).
// ---------------------------------------------------------------------------
template <int F>
__global__ __launch_bounds__(kThreads) void k_init_state(Dev d, uint32_t k0, uint32_t k1) {
  const PBlock pb = load_pblock(d.pblocks, blockIdx.x);
  BoxRef B = as_const(d.boxes)[pb.box];
  const StatePtrs S = d.S[d.ctrl->cur];
  const uint32_t pend = B.pbase + B.np;
  for (int s = 0; s < kPartBlock / kThreads; ++s) {
    const uint32_t i = pb.p0 + s * kThreads + threadIdx.x;
    if (i >= pend) continue;
    const uint32_t li = i - B.pbase;
    const Words4 a = philox10(0, li, pb.box, kTagInitPos, k0, k1);
    const Words4 b = philox10(1, li, pb.box, kTagInitPos, k0, k1);
    double x[3] = {u53_of(a.w[0], a.w[1]) * B.Ld[0], u53_of(a.w[2], a.w[3]) * B.Ld[1],
                   u53_of(b.w[0], b.w[1]) * B.Ld[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (x[k] >= B.Ld[k]) x[k] = nextafter(B.Ld[k], 0.0);
    const Words4 c = philox10(0, li, pb.box, kTagInitVel, k0, k1);
    const double r0 = sqrt(-2.0 * log(u32_open_of(c.w[0])));
    const double r1 = sqrt(-2.0 * log(u32_open_of(c.w[2])));
    const double t0 = kTwoPi * ((double)c.w[1] * 0x1p-32);
    const double t1 = kTwoPi * ((double)c.w[3] * 0x1p-32);
    const double v[3] = {B.sd * r0 * cos(t0), B.sd * r0 * sin(t0), B.sd * r1 * cos(t1)};
    if constexpr (F == kFormF64) {
      RecF64 r;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        r.x[k] = x[k];
        r.v[k] = v[k];
      }
      ((RecF64*)S.rec)[i] = r;
      S.id[i] = i;
    } else if constexpr (F == kFormF32) {
      RecF32 r;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        float xf = (float)x[k];
        if (xf >= B.Lf[k]) xf = nextafterf(B.Lf[k], 0.0f);
        r.x[k] = xf;
        r.v[k] = (float)v[k];
      }
      ((RecF32*)S.rec)[i] = r;
      S.id[i] = i;
    } else {
      RecSplit r;
      int c3[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        float o;
        split_from_double(x[k], c3[k], o);
        if (c3[k] >= B.L[k]) {
          c3[k] = B.L[k] - 1;
          o = nextafterf(1.0f, 0.0f);
        }
        r.o[k] = o;
        r.v[k] = (float)v[k];
      }
      r.cell = split_encode(c3);
      r.id = i;
      ((RecSplit*)S.rec)[i] = r;
    }
  }
}

// ---------------------------------------------------------------------------
// Observables: momentum and energy of slots in a fixed order as per-block
// partial sums (FP64), of many blocks summed further by k_obs_sums, the rest in
// order on the host; else, and for the relative energy, sums that do not depend
// on the order (k_obs_exact).
// ---------------------------------------------------------------------------
template <int F>
__device__ __forceinline__ void load_vel_d(const StatePtrs& S, uint32_t i, double (&v)[3]) {
  if constexpr (F == kFormF64) {
    const RecF64& r = ((const RecF64*)S.rec)[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = r.v[k];
  } else if constexpr (F == kFormF32) {
    const RecF32& r = ((const RecF32*)S.rec)[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = (double)r.v[k];
  } else {
    const RecSplit& r = ((const RecSplit*)S.rec)[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = (double)r.v[k];
  }
}

__device__ __forceinline__ double block_sum_d(double x, double* s_red) {
  // deterministic tree sum over the block (fixed order)
  s_red[threadIdx.x] = x;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) s_red[threadIdx.x] = s_red[threadIdx.x] + s_red[threadIdx.x + w];
    __syncthreads();
  }
  const double r = s_red[0];
  __syncthreads();
  return r;
}

// Order in which the observables of an FP64 box add its particles after a
// step: by obs tile (To cells of a row), in it by pass (as many whole cells as
// kObsPass particles allow), in a pass by the particle's cell of the next step
// (rows y +- 1, z +- 1 around the tile, cells x0 - 1 .. x0 + nc of each row;
// all others last), then by cell and logical index.  The slots themselves
// depend on the order in which runs were appended; a total momentum is a sum
// of rounding errors, and in slot order its digits would change from run to
// run.  One wavefront per obs tile; the particles of its cells lie in the
// output of one to three collide tiles.  Their cells and ids are read once, four slots
// per lane in flight; a crowded neighbourhood (more than kObsList particles)
// is read again for each pass.
template <bool W>
__global__ __launch_bounds__(64) void k_obs_order(Dev d, uint32_t box, uint32_t cur, uint32_t To,
                                                  uint32_t* __restrict__ order) {
  using Fm = Form<kFormF64>;
  constexpr int kWin = 9 * (kTileMaxCells + 2) + 1;
  constexpr int NS = kObsPass / 64;
  static_assert(kWin <= 5 * 64, "five window entries per lane");
  __shared__ uint32_t s_cnt[kTileMaxCells], s_off[kTileMaxCells + 1], s_before;
  __shared__ uint32_t s_id[kObsPass], s_slot[kObsPass], s_can[kObsPass], s_pc[kWin];
  __shared__ uint8_t s_lc[kObsPass];
  __shared__ uint32_t s_lid[kObsList], s_lslot[kObsList], s_n;
  __shared__ uint8_t s_llc[kObsList];
  const uint32_t lane = threadIdx.x;
  BoxRef B = as_const(d.boxes)[box];
  const MPC_AS4 BoxStep& bs = as_const(d.bstep[cur ^ 1u])[box];  // of the last step
  const StatePtrs S = d.S[cur];
  const int L0 = B.L[0], L1 = B.L[1], L2 = B.L[2];
  const uint32_t nx = ((uint32_t)L0 + To - 1) / To;
  const uint32_t row = blockIdx.x / nx;
  const int x0 = (int)((blockIdx.x - row * nx) * To);
  const int y0 = (int)(row % (uint32_t)L1), z0 = (int)(row / (uint32_t)L1);
  const int nc = min((int)To, L0 - x0), WX = nc + 2;
  const uint32_t t0 = B.tbase + row * B.ntx + (uint32_t)x0 / B.T;
  const uint32_t t1 = B.tbase + row * B.ntx + (uint32_t)(x0 + nc - 1) / B.T;
  const uint32_t i0 = d.toff[t0];
  const uint32_t i1 = min(t1 + 1u < d.ntile ? d.toff[t1 + 1] : d.ntot, d.ntot);
  const double st[3] = {bs.s[0], bs.s[1], bs.s[2]};
  const double sn[3] = {bs.sn[0], bs.sn[1], bs.sn[2]};
  const bool le = !W && B.le;
  uint32_t err = 0;
  // cells (stored positions are those of the last step's collision) and ids of
  // slots i0 .. i1: f(cell, id, slot)
  auto sweep = [&](auto f) {
    for (uint32_t q0 = i0; q0 < i1; q0 += 256) {
      typename Fm::P p[4];
      uint32_t id[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = q0 + k * 64 + lane;
        typename Fm::Vv v;
        id[k] = 0u;
        if (i < i1) Fm::load_all(S, i, p[k], v, id[k]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = q0 + k * 64 + lane;
        if (i < i1) f(Fm::cell_x(p[k], st, B, bs.d1, le) - x0, id[k], i);
      }
    }
  };
  if (lane < (uint32_t)kTileMaxCells) s_cnt[lane] = 0u;
  if (lane == 0) s_before = s_n = 0u;
  wave_sync();
  sweep([&](int c, uint32_t id, uint32_t i) {
    if (c < 0) {
      atomicAdd(&s_before, 1u);
    } else if (c < nc) {
      atomicAdd(&s_cnt[c], 1u);
      const uint32_t q = atomicAdd(&s_n, 1u);
      if (q < (uint32_t)kObsList) {
        s_lid[q] = id;
        s_lslot[q] = i;
        s_llc[q] = (uint8_t)c;
      }
    }
  });
  wave_sync();
  {
    const uint32_t n = lane < (uint32_t)kTileMaxCells ? s_cnt[lane] : 0u;
    const uint32_t inc = wave_scan_dpp(n);
    if (lane <= (uint32_t)kTileMaxCells) s_off[lane] = inc - n;
  }
  wave_sync();
  uint32_t base = i0 + s_before;
  for (int cs = 0; cs < nc;) {
    const uint32_t b = s_off[cs];
    int ce = cs + 1;
    while (ce < nc && s_off[ce + 1] - b <= (uint32_t)kObsPass) ++ce;
    const uint32_t np = s_off[ce] - b;
    if (lane < (uint32_t)kTileMaxCells) s_cnt[lane] = 0u;
    for (uint32_t q = lane; q < (uint32_t)kWin; q += 64) s_pc[q] = 0u;
    wave_sync();
    auto place_in_pass = [&](int c, uint32_t id, uint32_t i) {
      if (c < cs || c >= ce) return;
      const uint32_t q = s_off[c] - b + atomicAdd(&s_cnt[c], 1u);
      if (np > (uint32_t)kObsPass) {  // a cell that did not collide
        if (base + q < d.ntot) order[base + q] = i;
      } else if (q < (uint32_t)kObsPass) {
        s_id[q] = id;
        s_slot[q] = i;
        s_lc[q] = (uint8_t)c;
      }
    };
    if (s_n <= (uint32_t)kObsList) {
      for (uint32_t q = lane; q < s_n; q += 64) place_in_pass(s_llc[q], s_lid[q], s_lslot[q]);
    } else {
      sweep(place_in_pass);
    }
    wave_sync();
    if (np <= (uint32_t)kObsPass) {
      for (uint32_t q = lane; q < np; q += 64) {
        const uint32_t c = s_lc[q], e = s_off[c + 1] - b, id = s_id[q];
        uint32_t r = s_off[c] - b;
        for (uint32_t k = r; k < e; ++k) r += s_id[k] < id ? 1u : 0u;
        s_can[min(r, (uint32_t)kObsPass - 1u)] = s_slot[q];
      }
      wave_sync();
      uint32_t place[NS];
      typename Fm::P p[NS];
      typename Fm::Vv v[NS];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * 64;
        if (q < np) Fm::load(S, s_can[q], p[k], v[k]);
      }
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * 64;
        place[k] = 0u;
        __builtin_amdgcn_sched_barrier(0);
        if (q < np) {
          Fm::template stream<W>(p[k], v[k], B, bs.d2, le);
          int c[3];
          Fm::template coords<W>(p[k], sn, B, c, err, bs.d2, le);
          const int dx = wrap1(c[0] - x0 + 1, L0);
          int dy = c[1] - y0, dz = c[2] - z0;
          dy += L1 & -(int)(dy < -1);
          dy -= L1 & -(int)(dy > 1);
          if (!W) {
            dz += L2 & -(int)(dz < -1);
            dz -= L2 & -(int)(dz > 1);
          }
          const bool near = (unsigned)dx < (unsigned)WX && (unsigned)(dy + 1) < 3u &&
                            (unsigned)(dz + 1) < 3u;
          const uint32_t e = near ? (uint32_t)(((dz + 1) * 3 + dy + 1) * WX + dx) : (uint32_t)(9 * WX);
          place[k] = e << 16 | atomicAdd(&s_pc[e], 1u);
        }
      }
      wave_sync();
      uint32_t n5[5], sum = 0;
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        const int i = (int)lane * 5 + m;
        n5[m] = i < kWin ? s_pc[i] : 0u;
        sum += n5[m];
      }
      uint32_t run = wave_scan_dpp(sum) - sum;
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        if ((int)lane * 5 + m < kWin) s_pc[lane * 5 + m] = run;
        run += n5[m];
      }
      wave_sync();
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const uint32_t q = lane + k * 64;
        const uint32_t j = base + s_pc[place[k] >> 16] + (place[k] & 0xffffu);
        if (q < np && j < d.ntot) order[j] = s_can[q];
      }
    }
    base += np;
    cs = ce;
    wave_sync();
  }
}

template <int F>
__global__ __launch_bounds__(kThreads) void k_obs_pass1(Dev d, uint32_t pb0, uint32_t cur,
                                                        const uint32_t* __restrict__ order) {
  __shared__ double s_red[kThreads];
  const uint32_t blk = pb0 + blockIdx.x;
  const PBlock pb = load_pblock(d.pblocks, blk);
  BoxRef B = as_const(d.boxes)[pb.box];
  const StatePtrs S = d.S[cur];
  const uint32_t pend = B.pbase + B.np;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int s = 0; s < kPartBlock / kThreads; ++s) {
    const uint32_t i = pb.p0 + s * kThreads + threadIdx.x;
    if (i >= pend) continue;
    double v[3];
    load_vel_d<F>(S, order ? min(order[i], d.ntot - 1u) : i, v);
    acc[0] += B.mass * v[0];
    acc[1] += B.mass * v[1];
    acc[2] += B.mass * v[2];
    acc[3] += 0.5 * B.mass * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  }
  for (int k = 0; k < 4; ++k) {
    const double r = block_sum_d(acc[k], s_red);
    if (threadIdx.x == 0) d.partials[(uint64_t)blk * 4 + k] = r;
  }
}

// Sums that do not depend on the order of their terms (of the velocities where
// no order of the slots is fixed, and of every form's relative energy).  A term
// x becomes three whole digits of 40 bits on a fixed grid of exponents, with
// the top digit in bin floor(e / 40) of the largest exponent e so far: digits
// below the third are cut off term by term and those that a larger exponent
// pushes out are dropped, so that what is left at the end depends on the terms
// alone.  It is short of the true sum by less than n 2^-80 times the largest
// term.  The digits are FP64 numbers: at most 8192 of 2^40 a thread stay below
// 2^53.  The kernel reads what plain sums read, once, and is bound by that;
// about 11 FP64 operations a term take a tenth of the time.
struct ExactSum {
  double a[3];  // digits, lowest first
  int anchor;   // bin of the top digit; -1: none yet
};
__device__ __forceinline__ void exact_grow(ExactSum& s, uint32_t e) {
  const int b = e == 2047u ? kObsBad : (int)(e / 40u);
  const int by = b - s.anchor;
  s.a[0] = by == 1 ? s.a[1] : (by == 2 ? s.a[2] : 0.0);
  s.a[1] = by == 1 ? s.a[2] : 0.0;
  s.a[2] = 0.0;
  s.anchor = b;
}
__device__ __forceinline__ void exact_add(ExactSum& s, double x) {
  const uint32_t e = (uint32_t)((uint64_t)__double_as_longlong(x) >> 52) & 0x7ffu;
  if (__builtin_expect(e >= 40u * (uint32_t)(s.anchor + 1), 0)) exact_grow(s, e);
  // 2^(1023 - 40 anchor); any finite number once a term was not finite
  const uint32_t se = s.anchor == kObsBad ? 1023u : 2046u - 40u * (uint32_t)s.anchor;
  double r = x * __longlong_as_double((long long)((uint64_t)se << 52));
  double w = __builtin_trunc(r);
  s.a[2] += w;
  r = (r - w) * 0x1p40;
  w = __builtin_trunc(r);
  s.a[1] += w;
  s.a[0] += __builtin_trunc((r - w) * 0x1p40);
}
// Digits of a sum anchored at bin `from`, lowest first, moved to bin `to`.
__device__ __forceinline__ void exact_move(long long (&v)[3], int from, int to) {
  const int by = to - from;
  v[0] = by == 0 ? v[0] : (by == 1 ? v[1] : (by == 2 ? v[2] : 0ll));
  v[1] = by == 0 ? v[1] : (by == 1 ? v[2] : 0ll);
  v[2] = by == 0 ? v[2] : 0ll;
}

// NV = 4: momentum and energy; 1: sum m |v - vmean|^2.  Particles [blockIdx.x
// per, (blockIdx.x + 1) per) of the box into row blockIdx.x.
template <int F, int NV>
__global__ __launch_bounds__(kThreads) void k_obs_exact(Dev d, uint32_t box, uint32_t cur,
                                                        Vec3 vmean, uint32_t per) {
  __shared__ ObsRow<NV> s_row[kThreads / 64];
  BoxRef B = as_const(d.boxes)[box];
  const StatePtrs S = d.S[cur];
  const uint32_t i0 = blockIdx.x * per, i1 = min(i0 + per, B.np);
  const double V[3] = {vmean.v[0], vmean.v[1], vmean.v[2]};
  ExactSum acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = ExactSum{{0.0, 0.0, 0.0}, -1};
  // a pass of four particles a thread, the next one's loads in flight beside it
  constexpr int U = kPartBlock / kThreads;
  double v[U][3], w[U][3];
  auto load = [&](uint32_t q, double (&r)[U][3]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = q + u * kThreads + threadIdx.x;
      if (i < i1) load_vel_d<F>(S, B.pbase + i, r[u]);
    }
  };
  load(i0, v);
  for (uint32_t q = i0; q < i1; q += kPartBlock) {
    load(q + kPartBlock, w);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (q + u * kThreads + threadIdx.x < i1) {
        if constexpr (NV == 4) {
#pragma unroll
          for (int k = 0; k < 3; ++k) exact_add(acc[k], B.mass * v[u][k]);
          exact_add(acc[3], 0.5 * B.mass *
                                (v[u][0] * v[u][0] + v[u][1] * v[u][1] + v[u][2] * v[u][2]));
        } else {
          const double dx = v[u][0] - V[0], dy = v[u][1] - V[1], dz = v[u][2] - V[2];
          exact_add(acc[0], B.mass * (dx * dx + dy * dy + dz * dz));
        }
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) v[u][k] = w[u][k];
    }
  }
  // the wavefront, then the block: all at their largest bin, as integers (at
  // most 2^53 a thread, 2^61 a block)
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    int top = acc[k].anchor;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) top = max(top, __shfl_xor(top, m, 64));
    long long t[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) t[j] = acc[k].anchor == kObsBad ? 0ll : (long long)acc[k].a[j];
    exact_move(t, acc[k].anchor, top);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) t[j] += __shfl_xor(t[j], m, 64);
      if (lane == 0) s_row[wave].d[k][j] = t[j];
    }
    if (lane == 0) s_row[wave].anchor[k] = top;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const int k = (int)threadIdx.x;
    int top = -1;
    for (int w = 0; w < kThreads / 64; ++w) top = max(top, s_row[w].anchor[k]);
    long long sum[3] = {0, 0, 0};
    for (int w = 0; w < kThreads / 64; ++w) {
      long long t[3] = {s_row[w].d[k][0], s_row[w].d[k][1], s_row[w].d[k][2]};
      exact_move(t, s_row[w].anchor[k], top);
#pragma unroll
      for (int j = 0; j < 3; ++j) sum[j] += t[j];
    }
    ObsRow<NV>& o = ((ObsRow<NV>*)((ObsTotal*)d.obs + 4))[blockIdx.x];
#pragma unroll
    for (int j = 0; j < 3; ++j) o.d[k][j] = sum[j];
    o.anchor[k] = top;
  }
}

// All rows of a box to one total: kThreads threads for each value.
template <int NV>
__global__ __launch_bounds__(kThreads * NV) void k_obs_total(Dev d, uint32_t rows) {
  constexpr uint32_t kWaves = kThreads / 64;
  __shared__ ObsTotal s_t[kWaves * NV];
  const ObsRow<NV>* row = (const ObsRow<NV>*)((const ObsTotal*)d.obs + 4);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, k = wave / kWaves;
  __int128 s[3] = {0, 0, 0};
  int top = -1;
  auto move = [&](int to) {  // as exact_move
    const int by = to - top;
    s[0] = by == 0 ? s[0] : (by == 1 ? s[1] : (by == 2 ? s[2] : 0));
    s[1] = by == 0 ? s[1] : (by == 1 ? s[2] : 0);
    s[2] = by == 0 ? s[2] : 0;
    top = to;
  };
#pragma unroll 4
  for (uint32_t q = threadIdx.x % kThreads; q < rows; q += kThreads) {
    long long t[3] = {row[q].d[k][0], row[q].d[k][1], row[q].d[k][2]};
    const int at = row[q].anchor[k];
    if (at > top) move(at);
    exact_move(t, at, top);
#pragma unroll
    for (int j = 0; j < 3; ++j) s[j] += t[j];
  }
  int all = top;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) all = max(all, __shfl_xor(all, m, 64));
  move(all);
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const uint64_t lo = __shfl_xor((unsigned long long)s[j], m, 64);
      const int64_t hi = __shfl_xor((long long)(s[j] >> 64), m, 64);
      s[j] += (__int128)hi << 64 | lo;
    }
  }
  auto put = [&](ObsTotal& o) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      o.lo[j] = (uint64_t)s[j];
      o.hi[j] = (int64_t)(s[j] >> 64);
    }
    o.anchor = top;
  };
  if (lane == 0) put(s_t[wave]);
  __syncthreads();
  if (lane == 0 && wave == k * kWaves) {
    for (uint32_t w = wave; w < wave + kWaves; ++w) all = max(all, s_t[w].anchor);
    move(all);
    __int128 sum[3] = {s[0], s[1], s[2]};
    for (uint32_t w = wave + 1; w < wave + kWaves; ++w) {
#pragma unroll
      for (int j = 0; j < 3; ++j) s[j] = (__int128)s_t[w].hi[j] << 64 | s_t[w].lo[j];
      top = s_t[w].anchor;
      move(all);
#pragma unroll
      for (int j = 0; j < 3; ++j) sum[j] += s[j];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) s[j] = sum[j];
    put(((ObsTotal*)d.obs)[k]);
  }
}

// Sums of many blocks' partials: each thread adds a stride of them and the
// block its threads, as pairs (high, low) with the rounding error of every
// addition kept (Knuth's two-sum), about 106 bits.
struct Pair {
  double hi, lo;
};
__device__ __forceinline__ Pair pair_add(Pair a, double x, double xlo) {
  const double t = a.hi + x, z = t - a.hi;
  const double e = (a.hi - (t - z)) + (x - z);
  const double lo = a.lo + (e + xlo);
  const double hi = t + lo;
  return Pair{hi, lo - (hi - t)};
}
__global__ __launch_bounds__(kThreads) void k_obs_sums(Dev d, uint32_t pb0, uint32_t npb) {
  __shared__ Pair s_p[kThreads];
  const uint32_t per = (npb + kObsSums - 1) / kObsSums;
  const uint32_t q0 = blockIdx.x * per, q1 = min(npb, q0 + per);
  for (int k = 0; k < 4; ++k) {
    Pair a{0.0, 0.0};
    for (uint32_t q = q0 + threadIdx.x; q < q1; q += kThreads)
      a = pair_add(a, d.partials[4 * (size_t)(pb0 + q) + k], 0.0);
    s_p[threadIdx.x] = a;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w)
        s_p[threadIdx.x] =
            pair_add(s_p[threadIdx.x], s_p[threadIdx.x + w].hi, s_p[threadIdx.x + w].lo);
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      d.obs[8 * blockIdx.x + k] = s_p[0].hi;
      d.obs[8 * blockIdx.x + 4 + k] = s_p[0].lo;
    }
    __syncthreads();
  }
}

template <int F>
__global__ __launch_bounds__(kThreads) void k_remove_mean(Dev d, const double* vmean) {
  const PBlock pb = load_pblock(d.pblocks, blockIdx.x);
  BoxRef B = as_const(d.boxes)[pb.box];
  const StatePtrs S = d.S[d.ctrl->cur];
  const uint32_t pend = B.pbase + B.np;
  const double V[3] = {vmean[3 * pb.box], vmean[3 * pb.box + 1], vmean[3 * pb.box + 2]};
  for (int s = 0; s < kPartBlock / kThreads; ++s) {
    const uint32_t i = pb.p0 + s * kThreads + threadIdx.x;
    if (i >= pend) continue;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if constexpr (F == kFormF64) {
        double* p = ((RecF64*)S.rec)[i].v;
        p[k] = p[k] - V[k];
      } else if constexpr (F == kFormF32) {
        float* p = ((RecF32*)S.rec)[i].v;
        p[k] = (float)((double)p[k] - V[k]);
      } else {
        float* p = ((RecSplit*)S.rec)[i].v;
        p[k] = (float)((double)p[k] - V[k]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
#define MPC_FORM_DISPATCH(form, KERNEL, ...)                                  \
  do {                                                                       \
    switch (form) {                                                          \
      case kFormF64: hipLaunchKernelGGL(KERNEL<kFormF64>, __VA_ARGS__); break; \
      case kFormF32: hipLaunchKernelGGL(KERNEL<kFormF32>, __VA_ARGS__); break; \
      default: hipLaunchKernelGGL(KERNEL<kFormSplit>, __VA_ARGS__); break;     \
    }                                                                        \
  } while (0)

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t value, hipStream_t s) {
  uint64_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)blocks), dim3(kThreads), 0, s, p, n, value);
  return hipGetLastError();
}
hipError_t launch_zero_u32(uint32_t* p, uint64_t n, hipStream_t s) {
  return launch_fill_u32(p, n, 0u, s);
}

hipError_t launch_set_ctrl(const Dev& d, const Launch& l, uint64_t step, uint32_t cur,
                           int32_t reorder, int clear_err) {
  hipLaunchKernelGGL(k_set_ctrl, dim3(1), dim3(1), 0, l.stream, d.ctrl, step, cur, reorder,
                     clear_err);
  return hipGetLastError();
}

// Binning export: cell keys, ranks, offsets and slots of step t for buffer S.
hipError_t launch_binning(const Dev& d, const Launch& l, const StatePtrs& S, uint64_t t) {
  hipError_t e = launch_zero_u32(d.hist, (uint64_t)l.nscan * kScanBlock, l.stream);
  if (e != hipSuccess) return e;
  if (l.npblocks == 0) return hipSuccess;
  const dim3 g(l.npblocks), b(kThreads);
  switch (l.form * 2 + (l.walls ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_key_hist<kFormF64, false>), g, b, 0, l.stream, d, S, t); break;
    case 1: hipLaunchKernelGGL((k_key_hist<kFormF64, true>), g, b, 0, l.stream, d, S, t); break;
    case 2: hipLaunchKernelGGL((k_key_hist<kFormF32, false>), g, b, 0, l.stream, d, S, t); break;
    case 3: hipLaunchKernelGGL((k_key_hist<kFormF32, true>), g, b, 0, l.stream, d, S, t); break;
    case 4: hipLaunchKernelGGL((k_key_hist<kFormSplit, false>), g, b, 0, l.stream, d, S, t); break;
    default: hipLaunchKernelGGL((k_key_hist<kFormSplit, true>), g, b, 0, l.stream, d, S, t); break;
  }
  if (l.nscan > 1) {
    hipLaunchKernelGGL(k_scan_reduce, dim3(l.nscan), dim3(kThreads), 0, l.stream, d.hist,
                       d.scan_blk);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, l.stream, d.scan_blk, l.nscan);
  }
  hipLaunchKernelGGL(k_scan_down, dim3(l.nscan), dim3(kThreads), 0, l.stream, d, l.nscan);
  const uint32_t blocks = (uint32_t)((l.ntot + kThreads * 4 - 1) / (kThreads * 4));
  hipLaunchKernelGGL(k_scatter, dim3(blocks), dim3(kThreads), 0, l.stream, d.key, d.rank,
                     d.offset, d.perm, (uint32_t)l.ntot, (uint32_t)l.ctot, d.ctrl);
  return hipGetLastError();
}

// Output positions of the tiles for step l.seq of a launch sequence.
static hipError_t launch_tile_prefix(const Dev& d, const Launch& l) {
  const dim3 g((d.ntile + kTileBlock - 1) / kTileBlock), b(kThreads);
  if (d.ntile > kTileOne) hipLaunchKernelGGL(k_tile_reduce, g, b, 0, l.stream, d, l.seq);
  hipLaunchKernelGGL(k_tile_prefix, g, b, 0, l.stream, d, l.seq);
  return hipGetLastError();
}

// Sort of the state in buffer `from` into buffer `to` by tile of the next
// step, the run lists of `to`, and the side work of that step.
// caller: every box's slots are in the caller's order.
hipError_t launch_sort(const Dev& d, const Launch& l, uint32_t from, uint32_t to, int caller) {
  if (l.npblocks == 0) return hipSuccess;
  hipError_t e;
  const uint64_t clear = (uint64_t)d.ntile * std::max(d.maxr, 2u) / kThreads + 1;
  hipLaunchKernelGGL(k_tile_clear, dim3((uint32_t)std::min<uint64_t>(clear, 65536)), dim3(kThreads),
                     0, l.stream, d);
  const dim3 gc(l.npblocks), b(kThreads);
  switch (l.form * 2 + (l.walls ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_tile_count<kFormF64, false>), gc, b, 0, l.stream, d, from); break;
    case 1: hipLaunchKernelGGL((k_tile_count<kFormF64, true>), gc, b, 0, l.stream, d, from); break;
    case 2: hipLaunchKernelGGL((k_tile_count<kFormF32, false>), gc, b, 0, l.stream, d, from); break;
    case 3: hipLaunchKernelGGL((k_tile_count<kFormF32, true>), gc, b, 0, l.stream, d, from); break;
    case 4: hipLaunchKernelGGL((k_tile_count<kFormSplit, false>), gc, b, 0, l.stream, d, from); break;
    default: hipLaunchKernelGGL((k_tile_count<kFormSplit, true>), gc, b, 0, l.stream, d, from); break;
  }
  if ((e = launch_tile_prefix(d, l)) != hipSuccess) return e;
  const dim3 gp((uint32_t)((l.ntot + kPartBlock - 1) / kPartBlock));
  if (l.form == kFormSplit) {
    hipLaunchKernelGGL(k_tile_scatter, gp, b, 0, l.stream, d, from, to);
  } else {
    hipLaunchKernelGGL(k_tile_place, gp, b, 0, l.stream, d, to);
    if (l.form == kFormF64) {
      hipLaunchKernelGGL(k_tile_gather<kFormF64>, gp, b, 0, l.stream, d, from, to, caller);
    } else {
      hipLaunchKernelGGL(k_tile_gather<kFormF32>, gp, b, 0, l.stream, d, from, to, caller);
    }
  }
  hipLaunchKernelGGL(k_tile_runs, dim3((d.ntile + kThreads - 1) / kThreads), dim3(kThreads), 0,
                     l.stream, d, to);
  const Side w = side_of(l);
  const dim3 g((w.nbox + 63u) / 64u + (w.wcells + 63u) / 64u + (w.ctot + d.drawb - 1u) / d.drawb);
  switch ((l.walls ? 2 : 0) + (l.mbs ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_side<false, false>), g, dim3(64), 0, l.stream, d, w, to); break;
    case 1: hipLaunchKernelGGL((k_side<false, true>), g, dim3(64), 0, l.stream, d, w, to); break;
    case 2: hipLaunchKernelGGL((k_side<true, false>), g, dim3(64), 0, l.stream, d, w, to); break;
    default: hipLaunchKernelGGL((k_side<true, true>), g, dim3(64), 0, l.stream, d, w, to); break;
  }
  return hipGetLastError();
}

hipError_t launch_prefix(const Dev& d, const Launch& l) {
  // a collide with one wavefront per tile and few tiles sums them itself
  if (d.ntile <= kTileDirect && l.ntiles <= l.collide_grid) return hipSuccess;
  return launch_tile_prefix(d, l);
}

hipError_t launch_advance(const Dev& d, const Launch& l, uint32_t n) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(1), 0, l.stream, d.ctrl, n);
  return hipGetLastError();
}

hipError_t launch_collide(const Dev& d, const Launch& l) {
  if (l.ntiles == 0) return hipSuccess;
  return collide_dispatch<CollideLaunchOp>(d, l, nullptr);
}

hipError_t launch_canon_perm(const Dev& d, const Launch& l, const StatePtrs& ids) {
  const uint64_t blocks = (l.ctot + kThreads - 1) / kThreads;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_canon_perm, dim3((uint32_t)blocks), dim3(kThreads), 0, l.stream, d.perm,
                     d.offset, l.ctot, (uint32_t)l.ntot, (const uint32_t*)ids.id, ids.id_stride);
  return hipGetLastError();
}

hipError_t launch_gather_particles(const Dev& d, const Launch& l, const StatePtrs& S,
                                  uint32_t* inv, uint32_t* keys, uint32_t mask, uint32_t pbase,
                                  uint32_t np, uint32_t* sel, uint32_t m, double* out) {
  if (m == 0 || np == 0) return hipSuccess;
  (void)d;
  const dim3 gm((m + kThreads - 1) / kThreads), b(kThreads);
  if (keys) {
    uint32_t* slots = keys + (size_t)mask + 1;
    const hipError_t e = launch_fill_u32(keys, 2ull * ((uint64_t)mask + 1), kNoSlot, l.stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sample_insert, gm, b, 0, l.stream, sel, m, keys, mask);
    const uint32_t blocks =
        (uint32_t)std::min<uint64_t>(8192, ((uint64_t)np + 4 * kThreads - 1) / (4 * kThreads));
    hipLaunchKernelGGL(k_sample_find, dim3(blocks), b, 0, l.stream, (const uint32_t*)S.id,
                       S.id_stride, pbase, np, keys, slots, mask);
    hipLaunchKernelGGL(k_sample_slots, gm, b, 0, l.stream, sel, m, keys, slots, mask);
  } else {
    const hipError_t e = launch_fill_u32(inv, np, kNoSlot, l.stream);
    if (e != hipSuccess) return e;
    uint64_t blocks = ((uint64_t)np + kThreads - 1) / kThreads;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_invert_ids, dim3((uint32_t)blocks), dim3(kThreads), 0, l.stream,
                       (const uint32_t*)S.id, S.id_stride, pbase, np, inv);
  }
  MPC_FORM_DISPATCH(l.form, k_gather_particles, gm, b, 0, l.stream, S, inv, pbase, np, sel, m,
                    out);
  return hipGetLastError();
}

hipError_t launch_state_in(const Dev& d, const Launch& l, const StatePtrs& S, uint32_t box,
                           uint32_t i0, const double* x, const double* v, uint32_t m, double a,
                           uint32_t* bad) {
  const dim3 g((m + kThreads - 1) / kThreads), b(kThreads);
  if (bad) {
    hipLaunchKernelGGL(k_state_check, g, b, 0, l.stream, d.boxes, box, x, v, m, a, bad);
  } else {
    MPC_FORM_DISPATCH(l.form, k_state_pack, g, b, 0, l.stream, d.boxes, box, S, i0, x, v, m, a);
  }
  return hipGetLastError();
}

hipError_t launch_state_out(const Launch& l, const StatePtrs& S, uint32_t pbase, uint32_t np,
                            uint32_t i0, double* x, double* v, uint32_t m, double a,
                            uint32_t* bad) {
  const dim3 gm((m + kThreads - 1) / kThreads), b(kThreads);
  hipLaunchKernelGGL(k_state_unset, gm, b, 0, l.stream, x, m, bad, 0);
  MPC_FORM_DISPATCH(l.form, k_state_unpack, dim3((np + kThreads - 1) / kThreads), b, 0, l.stream, S,
                    pbase, np, i0, x, v, m, a, bad);
  hipLaunchKernelGGL(k_state_unset, gm, b, 0, l.stream, x, m, bad, 1);
  return hipGetLastError();
}

hipError_t launch_load_f64(const Dev& d, const Launch& l, const double* x, const double* v,
                           uint32_t n, double a, uint32_t cur) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_load_f64, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, l.stream,
                     d, x, v, n, a, cur);
  return hipGetLastError();
}

hipError_t launch_store_f64(const Dev& d, const Launch& l, double* x, double* v, uint32_t n,
                            double a, uint32_t cur) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_store_f64, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0,
                     l.stream, d, x, v, n, a, cur);
  return hipGetLastError();
}

hipError_t launch_init_state(const Dev& d, const Launch& l, uint64_t seed) {
  if (l.npblocks == 0) return hipSuccess;
  MPC_FORM_DISPATCH(l.form, k_init_state, dim3(l.npblocks), dim3(kThreads), 0, l.stream, d,
                    (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32));
  return hipGetLastError();
}

hipError_t launch_obs_order(const Dev& d, const Launch& l, uint32_t box, uint32_t nrows,
                            uint32_t l0, uint32_t cur, uint32_t To, uint32_t* order) {
  const uint32_t grid = nrows * ((l0 + To - 1) / To);
  if (l.walls) {
    hipLaunchKernelGGL(k_obs_order<true>, dim3(grid), dim3(64), 0, l.stream, d, box, cur, To, order);
  } else {
    hipLaunchKernelGGL(k_obs_order<false>, dim3(grid), dim3(64), 0, l.stream, d, box, cur, To, order);
  }
  return hipGetLastError();
}

hipError_t launch_obs_pass1(const Dev& d, const Launch& l, uint32_t pb0, uint32_t npb, uint32_t cur,
                            const uint32_t* order) {
  if (npb == 0) return hipSuccess;
  MPC_FORM_DISPATCH(l.form, k_obs_pass1, dim3(npb), dim3(kThreads), 0, l.stream, d, pb0, cur,
                    order);
  return hipGetLastError();
}

// Blocks and particles of each, whole passes: eight blocks per compute unit for
// the loads in flight (256^3 split, two passes of 0.9 ms: 1.9 ms with 1024
// blocks and more, 2.3 with 512); few enough for the host to add their rows where
// that takes at most four passes a block (a launch less: 24x20x18 FP32 85 and 80
// us a call).
static uint32_t obs_exact_blocks(uint32_t np, uint32_t* per) {
  const uint64_t passes = ((uint64_t)np + kPartBlock - 1) / kPartBlock;
  const uint64_t each =
      passes <= 4 * kObsFew
          ? (passes + kObsFew - 1) / kObsFew
          : std::max<uint64_t>((passes + kObsRows - 1) / kObsRows, std::min<uint64_t>(4, (passes + 2047) / 2048));
  // whole numbers below 2^53 in every thread
  static_assert(((1ull << 31) / kPartBlock / kObsRows) * (kPartBlock / kThreads) <= 8192, "terms");
  *per = (uint32_t)(each * kPartBlock);
  return (uint32_t)((passes + each - 1) / each);
}
template <int F, int NV>
static hipError_t obs_exact_form(const Dev& d, const Launch& l, uint32_t box, uint32_t np,
                                 uint32_t cur, const Vec3& vmean, ObsResult<NV>* out) {
  uint32_t per;
  const uint32_t rows = obs_exact_blocks(np, &per);
  hipLaunchKernelGGL((k_obs_exact<F, NV>), dim3(rows), dim3(kThreads), 0, l.stream, d, box, cur,
                     vmean, per);
  out->rows = rows <= kObsFew ? rows : 0u;
  if (!out->rows)
    hipLaunchKernelGGL(k_obs_total<NV>, dim3(1), dim3(kThreads * NV), 0, l.stream, d, rows);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return out->rows ? hipMemcpyAsync(out->row, (ObsTotal*)d.obs + 4, sizeof(ObsRow<NV>) * rows,
                                    hipMemcpyDeviceToHost, l.stream)
                   : hipMemcpyAsync(out->total, d.obs, sizeof(ObsTotal) * NV, hipMemcpyDeviceToHost,
                                    l.stream);
}
template <int NV>
hipError_t launch_obs_exact(const Dev& d, const Launch& l, uint32_t box, uint32_t np, uint32_t cur,
                            const Vec3& vmean, ObsResult<NV>* out) {
  switch (l.form) {
    case kFormF64: return obs_exact_form<kFormF64, NV>(d, l, box, np, cur, vmean, out);
    case kFormF32: return obs_exact_form<kFormF32, NV>(d, l, box, np, cur, vmean, out);
    default: return obs_exact_form<kFormSplit, NV>(d, l, box, np, cur, vmean, out);
  }
}
template hipError_t launch_obs_exact<4>(const Dev&, const Launch&, uint32_t, uint32_t, uint32_t,
                                        const Vec3&, ObsResult<4>*);
template hipError_t launch_obs_exact<1>(const Dev&, const Launch&, uint32_t, uint32_t, uint32_t,
                                        const Vec3&, ObsResult<1>*);

hipError_t launch_obs_sums(const Dev& d, const Launch& l, uint32_t pb0, uint32_t npb) {
  hipLaunchKernelGGL(k_obs_sums, dim3(kObsSums), dim3(kThreads), 0, l.stream, d, pb0, npb);
  return hipGetLastError();
}

hipError_t launch_remove_mean(const Dev& d, const Launch& l, const double* vmean) {
  if (l.npblocks == 0) return hipSuccess;
  MPC_FORM_DISPATCH(l.form, k_remove_mean, dim3(l.npblocks), dim3(kThreads), 0, l.stream, d,
                    vmean);
  return hipGetLastError();
}

}  // namespace mpc
