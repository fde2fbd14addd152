// Per-ray device code: geometry, the descent through the maximum mipmap,
// final samples, clearance angle and disc occlusion.  Used by the forward,
// adjoint and persistent kernels, so every caller makes the same decisions.
//
// Everything is FP32 and relative to the ray origin p (texel centre):
//   * texture-space offsets  d(u) = K u  with  u = t / (1 + c t)  (central
//     projection maps the straight ray to a straight texture line);
//   * tip height above p     dH(t) = t (2 s + x) / (sqrt(1 + x (2 s + x)) + 1),
//     x = t / rho, the cancellation-free form of |p + t L| - |p|;
//   * bilinear heights minus h_p.
// Absolute coordinates would lose the metre-scale detail near the origin
// (an FP32 ulp at the Moon's radius is 0.125 m).
#pragma once

#include "common.h"

#define SS_INF __builtin_inff()

// Kernels that trace rays: 256 threads, held to `waves` wavefronts per SIMD.  The
// descent is bound by instruction issue and gathers together, so wavefronts in flight
// count: the 8 suns of a 4096^2 tile take 7.64 ms at the 6 its free allocation (84
// VGPRs) gives, 6.76 at 7 (72, 24 bytes of them in scratch) and 7.04 at 8, which spills
// in the levels.
//
// Kernels that hold more than a descent lose by the spills what a seventh wavefront
// gives.  us at 7 / 6 wavefronts: the exact mode, 1024^2 tiles at 1.5 deg 213 / 205 and
// at another azimuth 267 / 236, 512^2 151 / 138, 2048^2 1027 / 1033; the adjoint, 1024^2
// replaying 81 / 75, from a record 25.6 / 24.5, 2048^2 in the penumbra 290 / 283 (left
// to itself the allocation takes 97 to 121 VGPRs there, 4 wavefronts, and the 2048^2
// replay takes 365 where it takes 320 at 6).  The points' adjoint at 7 / 6 / 5 / 4: a
// 512 x 384 image 46.3 / 42.4 / 34.4 / 33.3, 1920 x 1080 201 / 203 / 194 / 215.
#define SS_RAY_KERNEL_AT(waves) \
  __global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(waves)))
#define SS_RAY_KERNEL SS_RAY_KERNEL_AT(7)

// Workgroup ids are dealt round-robin over the 8 XCDs.  xcd_remap gives each
// XCD one contiguous run of [0, nb) (the first nb % 8 XCDs one id more);
// xcd_remap_grouped does so inside each group of grp ids (grp a multiple of 8,
// so an id keeps its XCD).  Both are bijections of [0, nb).
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int per = nb >> 3, rem = nb & 7, x = b & 7, k = b >> 3;
  return x * per + min(x, rem) + k;
}

__device__ __forceinline__ int xcd_remap_grouped(int b, int nb, int grp) {
  const int lo = (b / grp) * grp;
  return lo + xcd_remap(b - lo, min(grp, nb - lo));
}

__device__ __forceinline__ float ss_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float ss_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

template <bool SPHERE>
struct Ray {
  int i, j;          // texel holding the origin
  float ox, oy;      // origin minus that texel's centre, in texels (-0 at centres)
  float hp;          // reference height: relative heights are taken from it
  float dz;          // origin height above hp (-0 at centres, whose height is hp)
  float Kx, Ky;      // texture-space velocity per unit u (texels)
  float invKx, invKy;
  float c;           // projective constant: u = t / (1 + c t)
  float sp, cp;      // n.L and |n x L| at the origin (radial normal n)
  float sp2;         // 2 sp
  float invrho;      // 1 / |p|
  float uexit;       // u where the path leaves the tile
  float uhmin;       // u where the tip height is smallest (-inf: rising from the start)
  int sx, sy;        // direction of travel along columns / rows
};

// Ray from the surface point at texel (i, j)'s centre plus (ox, oy) texels,
// at height hp + dz.  Positions are taken relative to the texel centre and
// shifted by (ox, oy); heights relative to hp, a stored height, with the
// origin dz above it.  At centres ox = oy = dz = -0, which every sum below
// drops exactly, so those rays compute as if the terms were absent.
//
// NORMAL: divisions and roots by their short exact forms (rcp_rn), the same bits
// for the origins ray_init lets through; without them the set-up took a tenth of a
// descent ray's instructions.
template <bool SPHERE, bool NORMAL>
__device__ __forceinline__ void ray_init_as(const TileK& T, int i, int j, float hp, Ray<SPHERE>& r,
                                            float ox, float oy, float dz) {
  auto inv = [](float x) { return NORMAL ? rcp_rn(x) : 1.0f / x; };
  auto quot = [](float p, float q, float iq) { return NORMAL ? div_rn(p, q, iq) : p / q; };
  auto root = [](float x) { return NORMAL ? sqrt_rn(x) : sqrtf(x); };
  r.i = i;
  r.j = j;
  r.ox = ox;
  r.oy = oy;
  r.hp = hp;
  r.dz = dz;
  const float X = ((float)i + 0.5f + ox - 0.5f * (float)T.W) * T.texel;
  const float Y = ((float)j + 0.5f + oy - 0.5f * (float)T.H) * T.texel;
  if (SPHERE) {
    // n = (a, b, 1)/g with a = X/R, b = Y/R, g = |(a, b, 1)|; rho = R (1 + h_p/R)
    const float a = X * T.invR, b = Y * T.invR;
    const float g = root(1.0f + a * a + b * b);
    const float ig = inv(g);
    const float r1 = 1.0f + (hp + dz) * T.invR;
    r.sp = (a * T.Lx + b * T.Ly + T.Lz) * ig;
    const float cx = b * T.Lz - T.Ly, cy = T.Lx - a * T.Lz, cz = a * T.Ly - b * T.Lx;
    r.cp = root(cx * cx + cy * cy + cz * cz) * ig;
    const float rt = r1 * T.texel, ir1 = inv(r1);
    const float sc = quot(g, rt, inv(rt));
    r.Kx = (T.Lx - a * T.Lz) * sc;
    r.Ky = (T.Ly - b * T.Lz) * sc;
    r.c = quot(T.Lz * g, r1, ir1) * T.invR;
    r.invrho = quot(T.invR, r1, ir1);
    // |p + t L| is smallest at t = -rho s (ahead of p only when the sun is
    // below the local horizon)
    if (r.sp < 0.0f) {
      const float th = -r.sp / r.invrho;
      r.uhmin = th / (1.0f + r.c * th);
    } else {
      r.uhmin = -SS_INF;
    }
  } else {
    r.sp = T.Lz;
    r.cp = sqrtf(T.Lx * T.Lx + T.Ly * T.Ly);
    r.Kx = T.Lx / T.texel;
    r.Ky = T.Ly / T.texel;
    r.c = 0.0f;
    r.invrho = 0.0f;
    r.uhmin = T.Lz >= 0.0f ? -SS_INF : SS_INF;
  }
  r.sp2 = 2.0f * r.sp;
  r.sx = r.Kx > 0.0f ? 1 : (r.Kx < 0.0f ? -1 : 0);
  r.sy = r.Ky > 0.0f ? 1 : (r.Ky < 0.0f ? -1 : 0);
  // +inf on an axis the path never moves along: every crossing time on it is
  // then +-inf (the numerators are half-integers, never 0)
  r.invKx = r.sx ? inv(r.Kx) : SS_INF;
  r.invKy = r.sy ? inv(r.Ky) : SS_INF;
  // leaving the tile: first boundary in the direction of travel
  const float ex = (float)(r.sx > 0 ? T.W - i : -i) - 0.5f - ox;
  const float ey = (float)(r.sy > 0 ? T.H - j : -j) - 0.5f - oy;
  const float ux = r.sx ? quot(ex, r.Kx, r.invKx) : SS_INF;
  const float uy = r.sy ? quot(ey, r.Ky, r.invKy) : SS_INF;
  r.uexit = fminf(ux, uy);
}

template <bool SPHERE>
__device__ __forceinline__ void ray_init(const TileK& T, int i, int j, float hp, Ray<SPHERE>& r,
                                         float ox = -0.0f, float oy = -0.0f, float dz = -0.0f) {
  ray_init_as<SPHERE, true>(T, i, j, hp, r, ox, oy, dz);
  // every operand and result of the short forms is an ordinary number: an origin
  // near the surface, a sun off its zenith, a path that moves along both axes
  const bool ok = fabsf(r.hp + r.dz) * T.invR < 0.5f && r.cp > 1e-9f && r.cp < 2.0f &&
                  fabsf(r.invKx) < 1e30f && fabsf(r.invKy) < 1e30f;
  if (!ok) ray_init_as<SPHERE, false>(T, i, j, hp, r, ox, oy, dz);
}


template <bool SPHERE>
__device__ __forceinline__ float u_to_t(const Ray<SPHERE>& r, float u) {
  return SPHERE ? u * ss_rcp(1.0f - r.c * u) : u;
}

template <bool SPHERE>
__device__ __forceinline__ float t_to_u(const Ray<SPHERE>& r, float t) {
  return SPHERE ? t * ss_rcp(1.0f + r.c * t) : t;
}

// Tip height above the reference height hp: the rise above the origin,
// |p + t L| - |p| (sphere) or t L_z (plane), plus the origin's dz.
template <bool SPHERE>
__device__ __forceinline__ float tip_rise(const Ray<SPHERE>& r, const TileK& T, float t) {
  if (SPHERE) {
    const float x = t * r.invrho;
    const float q = 2.0f * r.sp + x;
    return t * q * ss_rcp(ss_sqrt(1.0f + x * q) + 1.0f) + r.dz;
  }
  return t * T.Lz + r.dz;
}

// The same tip height at the texture parameter u (t = u / A, A = 1 - c u):
// |p + t L| - |p| = u P / ((S + A) A) with P = 2 s A + u/rho and
// S = sqrt(A^2 + (u/rho) P), still free of cancellation; one reciprocal
// fewer than converting u to t first.
template <bool SPHERE>
__device__ __forceinline__ float tip_rise_u(const Ray<SPHERE>& r, const TileK& T, float u) {
  if (SPHERE) {
    const float A = fmaf(-r.c, u, 1.0f);
    const float v = u * r.invrho;
    const float P = fmaf(r.sp2, A, v);
    const float S = ss_sqrt(fmaf(A, A, v * P));
    return u * P * ss_rcp((S + A) * A) + r.dz;
  }
  return u * T.Lz + r.dz;
}

// Keeps an index inside [0, n): a negative index wraps to a huge unsigned
// value and lands on n - 1.  Only rounding at a tile edge can produce an index
// outside the level, so this is a memory-safety guard, not a behaviour.
__device__ __forceinline__ unsigned inside(int v, int n) { return min((unsigned)v, (unsigned)(n - 1)); }

// Row-major index y w + x.  Rows and widths stay below 2^24, so the full-rate
// 24-bit multiply gives the exact product (the 32-bit one issues at quarter
// rate).
__device__ __forceinline__ unsigned idx2(unsigned y, unsigned w, unsigned x) {
  return __umul24(y, w) + x;
}

__device__ __forceinline__ float mip_at(const TileK& T, int m, int cx, int cy) {
  const LevelK k = T.lev[m];
  return k.p[idx2(inside(cy, k.h), (unsigned)k.w, inside(cx, k.w))];
}

// True when every height of the tile is known to be a finite number (the mipmap's
// build says so, and the host has had the heights looked at again where a call
// relies on it).  A sample that touches a missing or infinite height can count as in
// shadow whatever the maxima say, so only then may samples be passed over that
// stepping through the run would have reached.
__device__ __forceinline__ bool heights_finite(const TileK& T) {
  if (T.L < 2) return false;
  const float* top = T.lev[T.L - 1].p;
  return __builtin_amdgcn_readfirstlane((int)(finite_word(top[0], finite_key(T.W, T.H)) ^
                                              __float_as_uint(top[1]))) == 0;
}

// One mip level as a buffer resource: 32-bit offsets, and an offset past the
// end reads 0 instead of faulting (the hardware range check), so gathers for
// candidates that are then discarded need no clamping.
struct Level {
  __amdgpu_buffer_rsrc_t rs;
  int w, h;
};

__device__ __forceinline__ Level level_from(const LevelK& k) {
  Level L;
  L.rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(k.p), 0, k.w * k.h * 4, 0x00020000);
  L.w = k.w;
  L.h = k.h;
  return L;
}

__device__ __forceinline__ Level level_of(const TileK& T, int m) { return level_from(T.lev[m]); }

// (A texel outside the level may give any offset; the range check makes the
// load return 0 or an in-range value, and such candidates are discarded.)
__device__ __forceinline__ float level_at(const Level& L, int cx, int cy) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                       L.rs, (int)(idx2((unsigned)cy, (unsigned)L.w, (unsigned)cx) * 4u), 0, 0));
}

typedef float f32x2 __attribute__((ext_vector_type(2)));

// The value, and the two neighbours in a row, at a byte offset of a level.
__device__ __forceinline__ float value_at(const Level& L, unsigned a) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(L.rs, (int)a, 0, 0));
}
__device__ __forceinline__ f32x2 pair_at(const Level& L, unsigned a) {
  return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(L.rs, (int)a, 0, 0));
}

// Bilinear sample of the terrain below the ray tip at ray length t (u = u(t)):
// clearance height and the tap layout (for the adjoint).
struct Sample {
  float dh;
  float fx, fy;
  int x0, y0;   // unclamped lower-left tap (texel indices)
};

template <bool SPHERE>
__device__ __forceinline__ Sample sample_at(const Ray<SPHERE>& r, const TileK& T, float t, float u) {
  Sample s;
  const float dx = fmaf(r.Kx, u, r.ox), dy = fmaf(r.Ky, u, r.oy);
  const float flx = floorf(dx), fly = floorf(dy);
  s.fx = dx - flx;
  s.fy = dy - fly;
  s.x0 = r.i + (int)flx;
  s.y0 = r.j + (int)fly;
  // clamp to the edge (the tap index is -1 only left of the first centre)
  const unsigned x0 = (unsigned)min(max(s.x0, 0), T.W - 1), x1 = inside(s.x0 + 1, T.W);
  const unsigned y0 = (unsigned)min(max(s.y0, 0), T.H - 1), y1 = inside(s.y0 + 1, T.H);
  const Level L0 = level_of(T, 0);
  const float h00 = level_at(L0, x0, y0) - r.hp, h10 = level_at(L0, x1, y0) - r.hp;
  const float h01 = level_at(L0, x0, y1) - r.hp, h11 = level_at(L0, x1, y1) - r.hp;
  const float hb = (1.0f - s.fy) * ((1.0f - s.fx) * h00 + s.fx * h10) +
                   s.fy * ((1.0f - s.fx) * h01 + s.fx * h11);
  s.dh = tip_rise(r, T, t) - hb;
  return s;
}

// Height of the bilinear terrain at continuous texel coordinates (qx, qy)
// above the reference height ref (texel i covers [i, i+1); taps clamp to the
// edge, as for the samples).  Differences of nearby heights are exact in
// FP32, so the result carries no rounding of the absolute height.
__device__ __forceinline__ float terrain_above(const TileK& T, float qx, float qy, float ref) {
  const float x = qx - 0.5f, y = qy - 0.5f;
  const float flx = floorf(x), fly = floorf(y);
  const float fx = x - flx, fy = y - fly;
  const int x0 = (int)flx, y0 = (int)fly;
  const unsigned xa = (unsigned)min(max(x0, 0), T.W - 1), xb = (unsigned)min(max(x0 + 1, 0), T.W - 1);
  const unsigned ya = (unsigned)min(max(y0, 0), T.H - 1), yb = (unsigned)min(max(y0 + 1, 0), T.H - 1);
  const unsigned W = (unsigned)T.W;
  const float h00 = T.h[idx2(ya, W, xa)] - ref, h10 = T.h[idx2(ya, W, xb)] - ref;
  const float h01 = T.h[idx2(yb, W, xa)] - ref, h11 = T.h[idx2(yb, W, xb)] - ref;
  return (1.0f - fy) * ((1.0f - fx) * h00 + fx * h10) + fy * ((1.0f - fx) * h01 + fx * h11);
}

// Visible part of the sun disc above a chord at d disc radii below its centre
// (Sec. 3.4, Eq. 6 first term; circular segment).  s is exactly 0 or 1 when
// |d| >= 1 (the disc wholly below or above the clearance, zero derivative) and
// strictly inside (0, 1) otherwise, so the adjoint can tell the rays it may
// skip from the forward's output alone.
__device__ __forceinline__ float disc_fraction(float alpha, const TileK& T) {
  if (!(alpha < SS_INF)) return 1.0f;
  const float dd = alpha * T.inv_rL;
  if (dd <= -1.0f) return 0.0f;
  if (dd >= 1.0f) return 1.0f;
  const float v = (3.14159265358979f - acosf(dd) + dd * sqrtf(fmaxf(0.0f, 1.0f - dd * dd))) *
                  0.318309886183791f;
  return fminf(fmaxf(v, 1.17549435e-38f), 0.99999994f);
}

// Clearance of a sample: the signed angle at p between L and the terrain point
// below the ray tip (positive: below the ray), atan2(num, den) with the terms
// below; to first order (dh / t) |n x L| (Sec. 3.4, Eq. 5).  Runs are compared by the
// tangent key num/den (den > 0; +inf / -inf when the angle is beyond +-pi/2),
// which orders like the angle, so atan runs once per ray.
struct SegOut {
  float key;
  float t;        // ray length of the deciding sample
  float u;
  int n;          // its index on the half-texel grid
  int valid;
};

template <bool SPHERE>
__device__ __forceinline__ void clearance_terms(const Ray<SPHERE>& r, float t, float dh, float& num,
                                                float& den) {
  if (SPHERE) {
    const float x = t * r.invrho;
    const float w = ss_sqrt(1.0f + x * (2.0f * r.sp + x));
    num = dh * r.cp;
    den = t * w - dh * (r.sp + x);
  } else {
    num = dh * r.cp;
    den = t - dh * r.sp;
  }
}

__device__ __forceinline__ float tangent_key(float num, float den) {
  return den > 0.0f ? num * ss_rcp(den) : (num >= 0.0f ? SS_INF : -SS_INF);
}

// True when every sample at ray length >= t clears the angle whose tangent is
// need_tan (an angle in (-pi/2, pi/2)), given that no terrain rises above
// `top` (relative to the reference height hp, and at least the origin's dz,
// i.e. not below the origin): the clearance of the point at that height below
// the tip grows with t on the plane and on the sphere.  Used for the
// result-invariant early exits.
template <bool SPHERE>
__device__ __forceinline__ bool clears(const Ray<SPHERE>& r, const TileK& T, float t, float top,
                                       float need_tan) {
  const float d = tip_rise(r, T, t) - top;
  if (!(d > 0.0f)) return false;
  float num, den;
  clearance_terms(r, t, d, num, den);
  return den <= 0.0f || num >= need_tan * den;  // den <= 0: at least pi/2
}

// tan(min(alpha, r_L) + margin) for the tangent key of alpha (tan addition).
__device__ __forceinline__ float need_tangent(const TileK& T, float key) {
  const float k = fmaxf(fminf(key, T.tan_rL), -1e30f);
  return (k + T.tan_margin) * ss_rcp(1.0f - k * T.tan_margin);
}

// tan(alpha + margin) for the tangent key of alpha: samples that clear it cannot take
// the deciding sample's place, where those that clear need_tangent's may on a lit ray.
__device__ __forceinline__ float keep_tangent(const TileK& T, float key) {
  const float k = fmaxf(key, -1e30f);
  return k * T.tan_margin < 0.5f ? (k + T.tan_margin) * ss_rcp(1.0f - k * T.tan_margin) : SS_INF;
}

// The smallest of a run's final samples by height above the terrain (Alg. 1,
// final level), as `<=` scanning from the near end.
struct Deepest {
  float dh, t, u;
  int n;
  bool found;
};

// The three samples n_c - 1, n_c, n_c + 1 of the half-texel grid
// t_n = (n + 1) delta/2, any taps.
template <bool SPHERE>
__device__ __forceinline__ Deepest samples_any(const TileK& T, const Ray<SPHERE>& r, float ncf,
                                               unsigned& n_smp) {
  Deepest d{SS_INF, 0.0f, 0.0f, -1, false};
  const int nc = (int)ncf;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int n = nc - 1 + k;
    const float t = (float)(n + 1) * T.half_delta;
    const float u = t_to_u(r, t);
    if (n >= 0 && u < r.uexit) {
      const Sample s = sample_at(r, T, t, u);
      n_smp++;
      if (s.dh <= d.dh) d = Deepest{s.dh, t, u, n, true};
    }
  }
  return d;
}

// The same three samples where every tap lies inside the tile: no clamping, a
// row's two taps with one 8-byte load, and all six loads issued before the
// first is waited for (samples that do not count are evaluated and dropped;
// the range check of the buffer keeps even their loads in bounds).
template <bool SPHERE>
__device__ __forceinline__ Deepest samples_inside(const TileK& T, const Ray<SPHERE>& r, float ncf,
                                                  unsigned& n_smp) {
  const Level L0 = level_of(T, 0);
  const int base = __mul24(r.j, L0.w) + r.i;
  float t[3], u[3], fx[3], fy[3];
  f32x2 lo[3], hi[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    t[k] = (ncf + (float)k) * T.half_delta;
    u[k] = t_to_u(r, t[k]);
    const float dx = fmaf(r.Kx, u[k], r.ox), dy = fmaf(r.Ky, u[k], r.oy);
    const float flx = floorf(dx), fly = floorf(dy);
    fx[k] = dx - flx;
    fy[k] = dy - fly;
    const unsigned a = 4u * (unsigned)(__mul24((int)fly, L0.w) + ((int)flx + base));
    lo[k] = pair_at(L0, a);
    hi[k] = pair_at(L0, a + 4u * (unsigned)L0.w);
  }
  Deepest d{SS_INF, 0.0f, 0.0f, -1, false};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    // as sample_at
    const float h00 = lo[k].x - r.hp, h10 = lo[k].y - r.hp;
    const float h01 = hi[k].x - r.hp, h11 = hi[k].y - r.hp;
    const float hb = (1.0f - fy[k]) * ((1.0f - fx[k]) * h00 + fx[k] * h10) +
                     fy[k] * ((1.0f - fx[k]) * h01 + fx[k] * h11);
    const float dh = tip_rise(r, T, t[k]) - hb;
    const bool ok = ncf + (float)k >= 1.0f && u[k] < r.uexit;
    n_smp += ok ? 1u : 0u;
    const bool take = ok && dh <= d.dh;
    d.dh = take ? dh : d.dh;
    d.t = take ? t[k] : d.t;
    d.u = take ? u[k] : d.u;
    d.n = take ? (int)ncf - 1 + k : d.n;
    d.found = d.found || take;
  }
  return d;
}

// Lane masks: a condition over the wavefront as a scalar, combined by scalar
// instructions and turned back where a lane selects by it.
typedef unsigned long long Lanes;
__device__ __forceinline__ Lanes lanes(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool of(Lanes m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// 2 v + the lane's bit of m: one add with carry (two wait states after a mask the
// vector unit may have written).
__device__ __forceinline__ int twice_plus(int v, Lanes m) {
  int out;
  Lanes carry;
  asm("s_nop 1\n\tv_addc_co_u32_e64 %0, %1, %2, %2, %3"
      : "=v"(out), "=s"(carry)
      : "v"(v), "s"(m));
  return out;
}

// A run's state on its way down: the chosen texel, the ray's stretch inside it,
// and the rays that still have a run.
struct Stretch {
  int x, y;
  float u0, u1;
  Lanes have;
};

// What the rays of a wavefront share on their way down: where they head, when
// that is the same way for all of them, and (on the sphere) the quartic of each
// ray's tip height, r(u) = a1 u + a2 u^2 + a3 u^3 + a4 u^4 + ..., the series of
// |p + t L| - |p| with t = u / (1 - c u).
struct Heading {
  int ex, ey;  // 1: forward along the columns / rows, 0: backward
  bool same;
  float a2, a3, a4;
};

template <bool SPHERE>
__device__ __forceinline__ Heading heading_of(const TileK& T, const Ray<SPHERE>& r) {
  Heading d;
  d.ex = __builtin_amdgcn_readfirstlane(r.sx > 0 ? 1 : 0);
  d.ey = __builtin_amdgcn_readfirstlane(r.sy > 0 ? 1 : 0);
  // (the bounds of the tip height's fit hold for origins within 5% of the radius
  // whose path moves at least 0.95 of a texel per nominal texel of travel; how
  // far a final sample lies from its base texel, for at most 1.09)
  const float k2 = (r.Kx * r.Kx + r.Ky * r.Ky) * (4.0f * T.half_delta * T.half_delta);
  d.same = lanes(!(r.sx == 2 * d.ex - 1 && r.sy == 2 * d.ey - 1 && fabsf(r.invKx) < 1e30f &&
                   fabsf(r.invKy) < 1e30f &&
                   (!SPHERE || (fabsf(r.hp + r.dz) * T.invR < 0.05f && k2 > 0.9f && k2 < 1.2f)))) == 0;
  d.a2 = d.a3 = d.a4 = 0.0f;
  if (SPHERE) {
    const float k = r.cp * r.cp * r.invrho;
    const float b2 = 0.5f * k, b3 = -0.5f * r.sp * k * r.invrho;
    const float b4 = k * (5.0f * r.sp * r.sp - 1.0f) * 0.125f * r.invrho * r.invrho;
    d.a2 = fmaf(r.sp, r.c, b2);
    d.a3 = fmaf(r.c, fmaf(r.sp, r.c, 2.0f * b2), b3);
    d.a4 = fmaf(r.c, fmaf(r.c, fmaf(r.sp, r.c, 3.0f * b2), 3.0f * b3), b4);
  }
  return d;
}

// The quartic's second-order expansion at the middle of a stretch, plus the
// reference height: tip height above sea level ~ k0 + u (k1 + u k2).
struct TipFit {
  float k0, k1, k2;
};

template <bool SPHERE>
__device__ __forceinline__ TipFit tip_fit(const Ray<SPHERE>& r, const Heading& d, float u0,
                                          float u1) {
  const float uc = 0.5f * (u0 + u1), w = uc * uc;
  TipFit f;
  f.k2 = fmaf(uc, fmaf(6.0f * d.a4, uc, 3.0f * d.a3), d.a2);
  f.k1 = fmaf(-w, fmaf(8.0f * d.a4, uc, 3.0f * d.a3), r.sp);
  f.k0 = fmaf(w * uc, fmaf(3.0f * d.a4, uc, d.a3), r.hp) + r.dz;
  return f;
}

// One step of a descent for a wavefront whose rays head the same way: the ray
// crosses up to three texels (before both lines, after the first, after both)
// split at c1 <= c2, with maxima M0 .. M2 (-inf: no such texel, its bound is then
// +inf).  Sets t1 (the second texel over the first) and t2 (the third over those)
// and moves the stretch to the choice.
//
// The choice is the smallest of the texels' bounds, tip height less texel
// maximum.  An exact tip height costs 11 operations with a root and a
// reciprocal, and only the order of the bounds matters, so on the sphere they
// are taken from the run's fit (two FMAs) and used when they differ by more than
// the fit and the rounding can: err is twice the fit's bound, and heights carry
// a few ulps of the bound itself.  A wavefront with a closer pair evaluates the
// exact bounds, so the choices are those of the exact bounds in every case.
// RISING: every tip rises along the run, so it is lowest where it enters a piece.
// TOP: a first piece over a texel without a height (NaN) counts as absent, as in
// the walk of descend_apart; further down it ends the run.
template <bool SPHERE, bool RISING, bool TOP>
__device__ __forceinline__ void pick_piece(const TileK& T, const Ray<SPHERE>& r, const TipFit& f,
                                           float err, float M0, float M1, float M2, float c1,
                                           float c2, Stretch& st, Lanes& t1, Lanes& t2,
                                           unsigned& n_lb) {
  // where the tip is lowest on each piece
  const float p0 = RISING ? st.u0 : __builtin_amdgcn_fmed3f(r.uhmin, st.u0, c1);
  const float p1 = RISING ? c1 : __builtin_amdgcn_fmed3f(r.uhmin, c1, c2);
  const float p2 = RISING ? c2 : __builtin_amdgcn_fmed3f(r.uhmin, c2, st.u1);
  const bool ok0 = c1 > st.u0, ok1 = c2 > c1, ok2 = st.u1 > c2;
  float lb0, lb1, lb2, b01, n0, n1;
  Lanes found;
  auto order = [&](float v0, float v1, float v2) {
    // an absent piece has bound +inf
    lb0 = ok0 ? v0 : SS_INF;
    if (TOP) lb0 = v0 == v0 ? lb0 : SS_INF;
    lb1 = ok1 ? v1 : SS_INF;
    lb2 = ok2 ? v2 : SS_INF;
    // strict argmin from the far end == '<=' from the near end
    const bool s1 = lb1 <= lb0;
    b01 = s1 ? lb1 : lb0;
    const bool s2 = lb2 <= b01;
    t1 = lanes(s1);
    t2 = lanes(s2);
    // (below +inf; written so because a ballot of `< inf` comes out as "not equal to
    // inf", which a missing height passes)
    found = lanes((s2 ? lb2 : b01) <= 3.402823466e38f);
    n0 = s2 ? c2 : (s1 ? c1 : st.u0);
    n1 = s2 ? st.u1 : (s1 ? c2 : c1);
  };
  if (SPHERE) {
    order(fmaf(p0, fmaf(p0, f.k2, f.k1), f.k0 - M0), fmaf(p1, fmaf(p1, f.k2, f.k1), f.k0 - M1),
          fmaf(p2, fmaf(p2, f.k2, f.k1), f.k0 - M2));
    const float close = fmaf(fabsf(b01), 1e-6f, err);
    const Lanes unsure = lanes(fabsf(lb1 - lb0) < close) | lanes(fabsf(lb2 - b01) < close);
    if (unsure & st.have)
      order(tip_rise_u(r, T, p0) - (M0 - r.hp), tip_rise_u(r, T, p1) - (M1 - r.hp),
            tip_rise_u(r, T, p2) - (M2 - r.hp));
  } else {
    order(tip_rise_u(r, T, p0) - (M0 - r.hp), tip_rise_u(r, T, p1) - (M1 - r.hp),
          tip_rise_u(r, T, p2) - (M2 - r.hp));
  }
  n_lb += (ok0 && M0 != -SS_INF ? 1u : 0u) + (ok1 && M1 != -SS_INF ? 1u : 0u) +
          (ok2 && M2 != -SS_INF ? 1u : 0u);
  st.have &= found;
  st.u0 = n0;
  st.u1 = n1;
}

// True when no sample a descent can still reach from the level-lv texel of st
// matters: they all clear `need` (clears) over the highest terrain their taps can
// touch.  The samples lie within 0.83 texel of the base texel's stretch and their
// taps within two texels of the base texel, so the two by two texels one level up
// that surround the chosen texel by half its size hold every tap (lv >= 1).
template <bool SPHERE>
__device__ __forceinline__ bool out_of_reach(const TileK& T, const Ray<SPHERE>& r, const Level& up,
                                             const Stretch& st, float need) {
  const int x = min(max((st.x - 1) >> 1, 0), up.w - 2);
  const int y = min(max((st.y - 1) >> 1, 0), up.h - 2);
  const unsigned a = 4u * (unsigned)(__mul24(y, up.w) + x);
  const f32x2 p = pair_at(up, a), q = pair_at(up, a + 4u * (unsigned)up.w);
  const float M = fmaxf(fmaxf(p.x, p.y), fmaxf(q.x, q.y));
  const float t0 = fmaxf(M, r.hp) - r.hp;
  const float tlo = fmaxf(T.half_delta, u_to_t(r, st.u0) - 1.75f * T.half_delta);
  return clears(r, T, tlo, r.dz > t0 ? r.dz : t0, need);
}

// The descent of a run for such a wavefront, from the level-m texel (cx, cy)
// under u = ua whose lines ahead lie at ux, uy; no ray crosses a second line of
// either axis before ub (a run is one level-m texel of travel long, so a second
// crossing is rare; such a wavefront takes descend_apart).  The levels run in step over the wavefront (a ray that
// has lost its run only idles), so the loop and each level's geometry are scalar.
// EX: the columns run forward.
//
// Bound by instruction issue and by gathers (16 address cycles each), so a level
// reads its four children as two pairs and takes about 50 instructions where the
// walk in descend_apart takes 105 and three gathers, and the top texels one step
// where the walk takes up to four.  On the 8 suns of a 4096^2 tile: 10.85 ms with
// that walk, 9.16 with this descent, 6.76 with the early end below.
//
// A run ends early once nothing below the chosen texel can matter
// (out_of_reach), tested three and five levels below the top: most runs of lit
// rays pass far above their terrain.  The four maxima around the texel cost two
// loads and about 35 instructions, a level two and 50, the final samples six and 150.
// Tested earlier the bound is too coarse, and more tests cost more than they end.
template <bool SPHERE, bool RISING, bool EX>
__device__ __forceinline__ void descend_together(const TileK& T, const Ray<SPHERE>& r,
                                                 const Heading& d, unsigned errs, int m, int cx,
                                                 int cy, float ux, float uy, float ua, float ub,
                                                 float need, Stretch& st, unsigned& n_lb) {
  const Level Lt = level_of(T, m);
  LevelK next = T.lev[m - 1];
  const int sx = EX ? 1 : -1, sy = 2 * d.ey - 1;
  const Lanes flipx = EX ? 0 : ~0ull, flipy = d.ey ? 0 : ~0ull;
  TipFit f{0.0f, 0.0f, 0.0f};
  if (SPHERE) f = tip_fit(r, d, ua, ub);
  float err = fit_err_top(errs);
  asm("" : "+v"(err));  // beside a literal, a second scalar operand costs a move
  Lanes t1, t2;
  {
    const Lanes xfirst = lanes(ux <= uy);
    const float c1 = __builtin_amdgcn_fmed3f(of(xfirst) ? ux : uy, ua, ub);
    const float c2 = __builtin_amdgcn_fmed3f(of(xfirst) ? uy : ux, ua, ub);
    const int cx1 = cx + sx, cy1 = cy + sy;
    const Lanes x0 = lanes((unsigned)cx < (unsigned)Lt.w), x1 = lanes((unsigned)cx1 < (unsigned)Lt.w);
    const Lanes y0 = lanes((unsigned)cy < (unsigned)Lt.h), y1 = lanes((unsigned)cy1 < (unsigned)Lt.h);
    st.u0 = ua;
    st.u1 = ub;
    st.have = lanes(true);
    const unsigned a = 4u * (unsigned)(__mul24(cy, Lt.w) + cx), ay = a + (unsigned)(4 * sy * Lt.w);
    float M0 = value_at(Lt, a);
    float M1 = value_at(Lt, of(xfirst) ? a + (unsigned)(4 * sx) : ay);
    float M2 = value_at(Lt, ay + (unsigned)(4 * sx));
    M0 = of(x0 & y0) ? M0 : -SS_INF;
    M1 = of((xfirst & x1 & y0) | (~xfirst & x0 & y1)) ? M1 : -SS_INF;
    M2 = of(x1 & y1) ? M2 : -SS_INF;
    pick_piece<SPHERE, RISING, true>(T, r, f, err, M0, M1, M2, c1, c2, st, t1, t2, n_lb);
    st.x = of(t2 | (t1 & xfirst)) ? cx1 : cx;
    st.y = of(t2 | (t1 & ~xfirst)) ? cy1 : cy;
  }
  // low edge of the chosen texel relative to the origin texel centre, in texels
  float fx = (float)((st.x << m) - r.i) - 0.5f - r.ox;
  float fy = (float)((st.y << m) - r.j) - 0.5f - r.oy;
  int lv = m, stop = max(m - 3, 0);
  for (int part = 0;; ++part) {
#pragma clang loop unroll(disable)
    for (; lv > stop; --lv) {
      const Level L = level_from(next);
      next = T.lev[max(lv - 2, 0)];  // the next level's geometry, ahead of its use
      const float fh = __builtin_bit_cast(float, (126 + lv) << 23);  // 2^(lv - 1)
      const float mxr = fx + fh, myr = fy + fh;  // mid-lines (exact at texel centres)
      const float umx = mxr * r.invKx, umy = myr * r.invKy;
      const Lanes xfirst = lanes(umx <= umy);
      const float c1 = __builtin_amdgcn_fmed3f(of(xfirst) ? umx : umy, st.u0, st.u1);
      const float c2 = __builtin_amdgcn_fmed3f(of(xfirst) ? umy : umx, st.u0, st.u1);
      // the rows of children before and after the mid-line
      const unsigned a = (unsigned)__mul24(st.y, 8 * L.w) + 8u * (unsigned)st.x;
      const unsigned ra = a + (unsigned)(d.ey ? 0 : 4 * L.w), rc = a + (unsigned)(d.ey ? 4 * L.w : 0);
      float M0, Mx, My, M2;
      if (((L.w | L.h) & 1) == 0) {
        const f32x2 p = pair_at(L, ra), q = pair_at(L, rc);
        M0 = EX ? p.x : p.y;
        Mx = EX ? p.y : p.x;
        My = EX ? q.x : q.y;
        M2 = EX ? q.y : q.x;
      } else {
        // children beyond a ragged edge are absent: only the high ones can be.  (A
        // pair could end past the level there: single loads, kept apart.)
        const Lanes hx = lanes(2 * st.x + 1 < L.w) | flipx, hy = lanes(2 * st.y + 1 < L.h) | flipy;
        const Lanes lx = lanes(2 * st.x + 1 < L.w) | ~flipx, ly = lanes(2 * st.y + 1 < L.h) | ~flipy;
        unsigned r1 = ra + 4u, r3 = rc + 4u;
        asm("" : "+v"(r1), "+v"(r3));
        const float p0 = value_at(L, ra), p1 = value_at(L, r1), q0 = value_at(L, rc), q1 = value_at(L, r3);
        M0 = of(lx & ly) ? (EX ? p0 : p1) : -SS_INF;
        Mx = of(hx & ly) ? (EX ? p1 : p0) : -SS_INF;
        My = of(lx & hy) ? (EX ? q0 : q1) : -SS_INF;
        M2 = of(hx & hy) ? (EX ? q1 : q0) : -SS_INF;
      }
      pick_piece<SPHERE, RISING, false>(T, r, f, err, M0, of(xfirst) ? Mx : My, M2, c1, c2, st, t1,
                                        t2, n_lb);
      // child bits: flipped on an axis whose mid-line the chosen piece lies beyond
      const Lanes mx = (t2 | (t1 & xfirst)) ^ flipx, my = (t2 | (t1 & ~xfirst)) ^ flipy;
      st.x = twice_plus(st.x, mx);
      st.y = twice_plus(st.y, my);
      fx = of(mx) ? mxr : fx;
      fy = of(my) ? myr : fy;
    }
    if (lv == 0) return;
    if (lv >= 2 && T.prune) {
      const Level up = level_of(T, lv + 1);
      if (up.w >= 2 && up.h >= 2) {
        st.have &= ~lanes(out_of_reach(T, r, up, st, need));
        if (st.have == 0) return;
      }
    }
    if (SPHERE && part == 0 && m >= SS_REFIT_FROM) {
      f = tip_fit(r, d, st.u0, st.u1);
      err = fit_err_low(errs);
      asm("" : "+v"(err));
    }
    stop = part == 0 ? max(m - 5, 0) : 0;
  }
}

// The descent of a run for any wavefront: a walk over the level-m texels crossed
// for u in [ua, ub] (gx, gy: the grid lines ahead of the first, (cx, cy)), then
// the children of the chosen one.
template <bool SPHERE>
__device__ __forceinline__ void descend_apart(const TileK& T, const Ray<SPHERE>& r, int m, int cx,
                                              int cy, float gx, float gy, float ua, float ub,
                                              bool& found, Stretch& st, unsigned& n_lb) {
  found = false;
  const int S = 1 << m;
  const bool rising = r.uhmin <= ua;  // tip height grows over the whole run
  const int ex = r.Kx >= 0.0f ? 1 : 0, ey = r.Ky >= 0.0f ? 1 : 0;
  const float stx = (float)(r.sx * S), sty = (float)(r.sy * S);
  const Level Ltop = level_of(T, m);
  const unsigned lwm = (unsigned)Ltop.w, lhm = (unsigned)Ltop.h;
  float best = SS_INF, bu0 = ua, bu1 = ua, brise = 0.0f;
  int bx = cx, by = cy, have = 0;
  float u0 = ua;
  for (int it = 0; it < 8; ++it) {
    const float ux = gx * r.invKx;
    const float uy = gy * r.invKy;
    const float u1 = fminf(fminf(ux, uy), ub);
    // a piece in a texel outside the level is a rounding sliver at the tile edge
    const bool ok = u1 > u0 && (unsigned)cx < lwm && (unsigned)cy < lhm;
    // where the tip is lowest on [u0, u1] (a piece that is not ok is discarded)
    const float uc = __builtin_amdgcn_fmed3f(r.uhmin, u0, u1);
    // lower bound of the clearance over the piece: lowest tip height minus
    // the texel's maximum height (Sec. 3.2, Eq. 4 with the maximum mipmap)
    const float rise = tip_rise_u(r, T, uc);
    const float lb = rise - (level_at(Ltop, cx, cy) - r.hp);
    n_lb += ok ? 1u : 0u;
    const bool take = ok && lb <= best;
    best = take ? lb : best;
    bx = take ? cx : bx;
    by = take ? cy : by;
    bu0 = take ? u0 : bu0;
    bu1 = take ? u1 : bu1;
    brise = take ? rise : brise;
    have |= take ? 1 : 0;
    u0 = fmaxf(u0, u1);
    if (!(u1 < ub)) break;
    const bool mx = ux <= uy, my = uy <= ux;
    cx += mx ? r.sx : 0;
    gx += mx ? stx : 0.0f;
    cy += my ? r.sy : 0;
    gy += my ? sty : 0.0f;
  }
  if (!have) return;
  // descend: the children of the chosen texel crossed by the ray.  The
  // parent's two mid-lines split its stretch [bu0, bu1] into at most three
  // pieces, in order: before both crossings, after the first, after both.  The
  // child before a mid-line (in the direction of travel) is the low one when
  // moving forward or not at all; each crossing flips that axis, so the
  // children follow from which mid-line comes first.  A crossing outside the
  // stretch (an infinite one on an axis the path does not move along, too)
  // leaves its piece empty.
  const int bfx = 1 - ex, bfy = 1 - ey;  // child bits before the mid-lines
  // parent's low edge relative to the origin texel centre, in texels
  float fx = (float)((bx << m) - r.i) - 0.5f - r.ox;
  float fy = (float)((by << m) - r.j) - 0.5f - r.oy;
  for (int lv = m; lv > 0; --lv) {
    const int half = 1 << (lv - 1);
    const float fh = (float)half;
    const Level Lc = level_of(T, lv - 1);
    const int px = 2 * bx, py = 2 * by;
    const float mxr = fx + fh, myr = fy + fh;  // mid-lines (exact)
    const float umx = mxr * r.invKx, umy = myr * r.invKy;
    const bool xfirst = umx <= umy;
    const float c1 = __builtin_amdgcn_fmed3f(fminf(umx, umy), bu0, bu1);
    const float c2 = __builtin_amdgcn_fmed3f(fmaxf(umx, umy), bu0, bu1);
    const int xa = px + bfx, ya = py + bfy;  // before both
    const int xc = px + ex, yc = py + ey;    // after both
    const int xb = xfirst ? xc : xa, yb = xfirst ? ya : yc;
    const float M0 = level_at(Lc, xa, ya), M1 = level_at(Lc, xb, yb), M2 = level_at(Lc, xc, yc);
    // tip rise at each piece's entry: the first piece enters where the parent
    // did (already known); identical to evaluating it again
    float r0, r1, r2;
    if (rising) {
      r0 = brise;
      r1 = tip_rise_u(r, T, c1);
      r2 = tip_rise_u(r, T, c2);
    } else {
      r0 = tip_rise_u(r, T, fminf(fmaxf(r.uhmin, bu0), c1));
      r1 = tip_rise_u(r, T, fminf(fmaxf(r.uhmin, c1), c2));
      r2 = tip_rise_u(r, T, fminf(fmaxf(r.uhmin, c2), bu1));
    }
    // children beyond a ragged edge are absent; px and py always exist, so
    // only the high children px + 1, py + 1 can be missing
    const bool hx = px + 1 < Lc.w, hy = py + 1 < Lc.h;
    const bool ina = (ex == 1 || hx) && (ey == 1 || hy);  // before both
    const bool inc = (ex == 0 || hx) && (ey == 0 || hy);  // after both
    const bool inb = xfirst ? ((ex == 0 || hx) && (ey == 1 || hy)) : ((ex == 1 || hx) && (ey == 0 || hy));
    const bool ok0 = c1 > bu0 && ina;
    const bool ok1 = c2 > c1 && inb;
    const bool ok2 = bu1 > c2 && inc;
    // an absent piece has bound +inf; present ones are finite
    const float lb0 = ok0 ? r0 - (M0 - r.hp) : SS_INF;
    const float lb1 = ok1 ? r1 - (M1 - r.hp) : SS_INF;
    const float lb2 = ok2 ? r2 - (M2 - r.hp) : SS_INF;
    n_lb += (ok0 ? 1u : 0u) + (ok1 ? 1u : 0u) + (ok2 ? 1u : 0u);
    // strict argmin from the far end == '<=' from the near end
    const bool t1 = lb1 <= lb0;
    const float b01 = t1 ? lb1 : lb0;
    const bool t2 = lb2 <= b01;
    if (!((t2 ? lb2 : b01) < SS_INF)) return;  // no piece inside the level
    const int nx = t2 ? xc : (t1 ? xb : xa);
    const int ny = t2 ? yc : (t1 ? yb : ya);
    fx = nx != px ? mxr : fx;
    fy = ny != py ? myr : fy;
    bx = nx;
    by = ny;
    brise = t2 ? r2 : (t1 ? r1 : r0);
    const float nu0 = t2 ? c2 : (t1 ? c1 : bu0);
    const float nu1 = t2 ? bu1 : (t1 ? c2 : c1);
    bu0 = nu0;
    bu1 = nu1;
  }
  st = Stretch{bx, by, bu0, bu1, 0};
  found = true;
}

// One concatenated run (Sec. 3.3): descent from level m0 = run_m0(T.run[j]) over the
// texels the ray crosses (Sec. 3.2, Fig. 3b), strict argmin from the far end
// (kept here as '<=' scanning from the near end), then three samples half a
// texel apart around the chosen base texel (Alg. 1, final level).
template <bool SPHERE>
__device__ __forceinline__ void descend_run(const TileK& T, const Ray<SPHERE>& r, const Heading& d,
                                            int jseg, float need, SegOut& out, unsigned& n_lb,
                                            unsigned& n_smp) {
  out.valid = 0;
  const float ta = T.tau[jseg], tb = T.tau[jseg + 1];
  const float ua = t_to_u(r, ta);
  const float ub = fminf(t_to_u(r, tb), r.uexit);
  const int m = run_m0(T.run[jseg]);
  const int S = 1 << m;
  // the next grid line ahead of the current texel on each axis (+1 when the
  // path moves forward or not at all)
  const int ex = r.Kx >= 0.0f ? 1 : 0, ey = r.Ky >= 0.0f ? 1 : 0;
  // top level: the level-m texel under u = ua
  const int cx = (r.i >> m) + (int)floorf(ldexpf((float)(r.i & (S - 1)) + 0.5f + r.ox + r.Kx * ua, -m));
  const int cy = (r.j >> m) + (int)floorf(ldexpf((float)(r.j & (S - 1)) + 0.5f + r.oy + r.Ky * ua, -m));
  // those grid lines relative to the origin texel centre, in texels; they
  // are half-integers, exact in FP32, and move by +-2^m per step
  const float gx = (float)(((cx + ex) << m) - r.i) - 0.5f - r.ox;
  const float gy = (float)(((cy + ey) << m) - r.j) - 0.5f - r.oy;
  const float ux = gx * r.invKx, uy = gy * r.invKy;
  const float ux2 = (gx + (float)(r.sx * S)) * r.invKx, uy2 = (gy + (float)(r.sy * S)) * r.invKy;
  const unsigned errs = jseg < SS_FITRUNS ? T.fit_err[jseg] : SS_FIT_NONE;
  Stretch st;
  if (d.same && m > 0 && errs != SS_FIT_NONE && lanes(fminf(ux2, uy2) < ub) == 0) {
    const bool rising = lanes(!(r.uhmin <= ua)) == 0;
    if (rising && d.ex)
      descend_together<SPHERE, true, true>(T, r, d, errs, m, cx, cy, ux, uy, ua, ub, need, st, n_lb);
    else if (rising)
      descend_together<SPHERE, true, false>(T, r, d, errs, m, cx, cy, ux, uy, ua, ub, need, st, n_lb);
    else if (d.ex)
      descend_together<SPHERE, false, true>(T, r, d, errs, m, cx, cy, ux, uy, ua, ub, need, st, n_lb);
    else
      descend_together<SPHERE, false, false>(T, r, d, errs, m, cx, cy, ux, uy, ua, ub, need, st, n_lb);
  } else {
    bool found;
    descend_apart(T, r, m, cx, cy, gx, gy, ua, ub, found, st, n_lb);
    st.have = lanes(found);
  }
  if (st.have == 0) return;
  // final samples on the half-texel grid t_n = (n + 1) delta/2 around the
  // middle of the base texel's stretch of ray
  const float tin = u_to_t(r, st.u0), tout = u_to_t(r, st.u1);
  const float tmid = 0.5f * (tin + tout);
  const float ncf = floorf((tmid - T.half_delta) * T.two_over_delta + 0.5f);
  // the samples lie within 3/4 texel of that middle, their taps two texels
  // around the base texel
  const bool in = T.W >= 7 && T.H >= 7 && (unsigned)(st.x - 3) <= (unsigned)(T.W - 7) &&
                  (unsigned)(st.y - 3) <= (unsigned)(T.H - 7);
  Deepest s;
  if ((lanes(!in) & st.have) == 0)
    s = samples_inside(T, r, ncf, n_smp);
  else
    s = samples_any(T, r, ncf, n_smp);
  if (!(of(st.have) && s.found)) return;
  float num, den;
  clearance_terms(r, s.t, s.dh, num, den);
  out.key = tangent_key(num, den);
  out.t = s.t;
  out.u = s.u;
  out.n = s.n;
  out.valid = 1;
}

// One run of Alg. 1 read literally: point samples instead of the texels the
// ray crosses.  Positions along run j are indices n on the half-texel grid
// t_n = (n + 1) delta/2 (the algorithm's normalised t in [0, 1] is
// (n - a_j) / 2^(m0+1)).  Level m = m0 .. 1 reads the maximum mipmap at the
// level-m texel under the ray tip at n = a_j + K, a_j + K - 2^m and
// a_j + K - 2^(m+1) (far to near; strict '<' keeps the far one on a tie) and
// continues from the smallest H - max h at K* with K = K* + 2^m; K starts at
// 2^(m0+1).  Level 0 samples the heightfield bilinearly at the three grid
// points and the chosen sample's clearance is the run's.  A level with no
// sample inside the tile ends the run.
template <bool SPHERE>
__device__ __forceinline__ void point_run(const TileK& T, const Ray<SPHERE>& r, int jseg,
                                          SegOut& out, unsigned& n_lb, unsigned& n_smp) {
  out.valid = 0;
  const int m0 = run_m0(T.run[jseg]);
  const int a = run_a0(T.run[jseg]);
  int K = 2 << m0;
  for (int m = m0; m >= 1; --m) {
    const int step = 1 << m;
    const Level Lm = level_of(T, m);
    float best = SS_INF;
    int kstar = -1;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int kk = K - q * step;
      const float t = (float)(a + kk + 1) * T.half_delta;
      const float u = t_to_u(r, t);
      // texel under the tip (positions before the edge are >= 0 by construction)
      const int cx = (int)floorf((float)r.i + 0.5f + r.ox + r.Kx * u) >> m;
      const int cy = (int)floorf((float)r.j + 0.5f + r.oy + r.Ky * u) >> m;
      const bool ok = u < r.uexit && (unsigned)cx < (unsigned)Lm.w && (unsigned)cy < (unsigned)Lm.h;
      const float v = tip_rise(r, T, t) - (level_at(Lm, cx, cy) - r.hp);
      n_lb += ok ? 1u : 0u;
      const bool take = ok && v < best;
      best = take ? v : best;
      kstar = take ? kk : kstar;
    }
    if (kstar < 0) return;
    K = kstar + step;
  }
  float bdh = SS_INF, bt = 0.0f, bu = 0.0f;
  int found = 0, bn = -1;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const float t = (float)(a + K - q + 1) * T.half_delta;
    const float u = t_to_u(r, t);
    if (u < r.uexit) {
      const Sample s = sample_at(r, T, t, u);
      n_smp++;
      if (s.dh < bdh) {
        bdh = s.dh;
        bt = t;
        bu = u;
        bn = a + K - q;
        found = 1;
      }
    }
  }
  if (!found) return;
  float num, den;
  clearance_terms(r, bt, bdh, num, den);
  out.key = tangent_key(num, den);
  out.t = bt;
  out.u = bu;
  out.n = bn;
  out.valid = 1;
}

struct RayResult {
  float alpha;
  float key;      // tangent key of alpha (orders like alpha)
  float t, u;     // deciding sample
  int n;          // its index on the step grid t = delta/2 + n step
  int valid;
};

__device__ __forceinline__ float angle_of(float key) {
  return key == SS_INF ? SS_INF : (key == -SS_INF ? -SS_INF : atanf(key));
}

// Smallest clearance over the concatenated runs (Sec. 3.3), each by the
// texel descent (POINT = false) or Alg. 1's point samples (POINT = true): over runs
// j0, j0 + stride, ...  KEEP: the deciding sample itself counts as a result, not only
// its clearance up to r_L, so a run ends early only where it cannot hold that sample.
template <bool SPHERE, bool POINT = false, bool KEEP = false>
__device__ __forceinline__ RayResult shadow_dp(const TileK& T, const Ray<SPHERE>& r, float top,
                                               unsigned& n_lb, unsigned& n_smp, int j0 = 0,
                                               int stride = 1) {
  RayResult res;
  res.t = 0.0f;
  res.u = 0.0f;
  res.n = -1;
  res.valid = 0;
  float best = SS_INF;                    // tangent key of the smallest clearance so far
  float need = need_tangent(T, SS_INF);   // tan(min(alpha, r_L) + margin)
  Heading way{};
  if (!POINT) way = heading_of(T, r);
  for (int j = j0; j < T.nseg; j += stride) {
    const float ta = T.tau[j];
    if (!(t_to_u(r, ta) < r.uexit)) break;  // the run starts outside the tile
    if (T.prune) {
      // every final sample of run j lies at t >= tau_j - 3 delta/4
      const float tlo = fmaxf(T.half_delta, ta - 1.5f * T.half_delta);
      if (clears(r, T, tlo, top, need)) break;  // nothing ahead is high enough
    }
    SegOut so;
    if (POINT)
      point_run(T, r, j, so, n_lb, n_smp);
    else
      descend_run(T, r, way, j, KEEP ? keep_tangent(T, best) : need, so, n_lb, n_smp);
    if (so.valid && so.key < best) {
      best = so.key;
      res.t = so.t;
      res.u = so.u;
      res.n = so.n;
      res.valid = 1;
      need = need_tangent(T, best);
    }
    if (T.prune && best <= -T.tan_rL) break;  // umbra: nothing can change s = 0
  }
  res.key = best;
  res.alpha = angle_of(best);
  return res;
}

// Ray length of step k: t_k = delta/2 + k step, rounded once, so that the
// exact mode (step delta/2) and uniform stepping at half a texel place their
// samples at bit-identical t.
__device__ __forceinline__ float step_t(const TileK& T, int k, float step) {
  return fmaf((float)k, step, T.half_delta);
}

// True when the steps from ray length t (texture parameter u) to te of every
// ray of the wavefront all clear `need` over the highest terrain their taps can
// touch: the two by two texels of level m that hold the taps between the first
// step's position and the last one's (the path is a line, so the rest lies
// between).
template <bool SPHERE>
__device__ __forceinline__ bool steps_clear(const TileK& T, const Ray<SPHERE>& r, const Level& L,
                                            int m, float t, float u, float te, float need) {
  const float ue = fminf(t_to_u(r, fminf(te, T.ucap)), r.uexit);
  const float xa = floorf(fmaf(r.Kx, u, r.ox)), xb = floorf(fmaf(r.Kx, ue, r.ox));
  const float ya = floorf(fmaf(r.Ky, u, r.oy)), yb = floorf(fmaf(r.Ky, ue, r.oy));
  // taps i + floor and the next, clamped to the tile as the samples clamp theirs
  const int x0 = min(max(r.i + (int)fminf(xa, xb), 0), T.W - 1);
  const int y0 = min(max(r.j + (int)fminf(ya, yb), 0), T.H - 1);
  const int x1 = min(max(r.i + (int)fmaxf(xa, xb) + 1, 0), T.W - 1);
  const int y1 = min(max(r.j + (int)fmaxf(ya, yb) + 1, 0), T.H - 1);
  const int cx = min(x0 >> m, L.w - 2), cy = min(y0 >> m, L.h - 2);
  const unsigned a = 4u * (unsigned)(__mul24(cy, L.w) + cx);
  const f32x2 p = pair_at(L, a), q = pair_at(L, a + 4u * (unsigned)L.w);
  const float M = fmaxf(fmaxf(p.x, p.y), fmaxf(q.x, q.y));
  const float t0 = fmaxf(M, r.hp) - r.hp;
  const bool clear = x1 >> m <= cx + 1 && y1 >> m <= cy + 1 &&
                     clears(r, T, t, r.dz > t0 ? r.dz : t0, need);
  return lanes(!clear) == 0;
}

// True when the taps of steps k .. k + n - 1 of every ray of the wavefront lie off the
// tile's edges and all of those steps count.  u: the texture parameter of step k.
template <bool SPHERE>
__device__ __forceinline__ bool steps_whole(const TileK& T, const Ray<SPHERE>& r, float step, int k,
                                            int n, float u) {
  const float te = step_t(T, k + n - 1, step), ue = t_to_u(r, te);
  const float xa = (float)r.i + fmaf(r.Kx, u, r.ox), xb = (float)r.i + fmaf(r.Kx, ue, r.ox);
  const float ya = (float)r.j + fmaf(r.Ky, u, r.oy), yb = (float)r.j + fmaf(r.Ky, ue, r.oy);
  const bool whole = te <= T.ucap && ue < r.uexit && fminf(xa, xb) >= 1.0f &&
                     fminf(ya, yb) >= 1.0f && fmaxf(xa, xb) < (float)(T.W - 2) &&
                     fmaxf(ya, yb) < (float)(T.H - 2);
  return lanes(!whole) == 0;
}

// Keeps the smaller of `res` and the clearance of step k, whose tip lies dh above the
// terrain; of equal ones the first.
template <bool SPHERE>
__device__ __forceinline__ void take_step(const Ray<SPHERE>& r, int k, float t, float u, float dh,
                                          RayResult& res, unsigned& n_smp) {
  n_smp++;
  float num, den;
  clearance_terms(r, t, dh, num, den);
  const float key = tangent_key(num, den);
  if (key < res.key) {
    res.key = key;
    res.t = t;
    res.u = u;
    res.n = k;
    res.valid = 1;
  }
}

// N steps from step k, for which steps_whole holds: as sample_at without the clamps,
// two 8-byte gathers a step, the N steps' gathers in flight together.
template <bool SPHERE, int N>
__device__ __forceinline__ void steps_inside(const TileK& T, const Ray<SPHERE>& r, const Level& L0,
                                             float step, int k, RayResult& res, unsigned& n_smp) {
  const int base = __mul24(r.j, L0.w) + r.i;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const float t = step_t(T, k + c, step);
    const float u = t_to_u(r, t);
    const float dx = fmaf(r.Kx, u, r.ox), dy = fmaf(r.Ky, u, r.oy);
    const float flx = floorf(dx), fly = floorf(dy);
    const float fx = dx - flx, fy = dy - fly;
    const unsigned a = 4u * (unsigned)(__mul24((int)fly, L0.w) + ((int)flx + base));
    const f32x2 lo = pair_at(L0, a), hi = pair_at(L0, a + 4u * (unsigned)L0.w);
    const float h00 = lo.x - r.hp, h10 = lo.y - r.hp;
    const float h01 = hi.x - r.hp, h11 = hi.y - r.hp;
    const float hb = (1.0f - fy) * ((1.0f - fx) * h00 + fx * h10) +
                     fy * ((1.0f - fx) * h01 + fx * h11);
    take_step(r, k + c, t, u, tip_rise(r, T, t) - hb, res, n_smp);
  }
}

// The smallest clearance over the steps k = 0, 1, ... of a ray up to the cap or the
// tile edge, kept as a tangent key; the first smallest step decides.  res holds what is
// known of the ray already.
//
// The wavefront's rays step together, in chunks of SS_CHUNK steps.  pass: steps that
// cannot matter to any of the rays are passed over (steps_clear), four chunks where
// that can be shown, else a chunk, else half of one.  lev: the mip level for a chunk.
// Steps that all count and lie inside the tile run without clamps.
//
// Bound by instruction issue (53 a step inside, 65 with the clamps and four gathers;
// 50 a look at the terrain's maxima) and by the gathers' latency, so the gathers of
// half a chunk, two a step, are in flight at once.  A 1024^2 tile at 1.5 deg, one-texel
// steps to 30 km: 764 us step by step, 600 without the clamps, 285 passing over 64 and
// 16 steps, 262 with the halves, 245 with the gathers of eight steps at a time for four.
// A fourth size of 256 steps is worth 2% or costs as much, and sizes that double and
// halve as they go cost 10% more.
template <bool SPHERE>
__device__ __forceinline__ void step_through(const TileK& T, const Ray<SPHERE>& r, float top,
                                             float step, int lev, bool pass, RayResult& res,
                                             unsigned& n_smp) {
  constexpr int HALF = SS_CHUNK / 2, MID = 4 * SS_CHUNK;
  const Level L0 = level_of(T, 0);
  const int mh = min(max(lev - 1, 0), T.L - 1), ma = min(lev, T.L - 1);
  const int mb = min(lev + 2, T.L - 1);
  auto fits = [&](int m) { return pass && min(T.lev[m].w, T.lev[m].h) >= 2; };
  const bool small = fits(ma), mid = fits(mb);
  bool done = false;
  for (int k = 0; k < (1 << 22) && !done; k += SS_CHUNK) {
    const float t = step_t(T, k, step);
    if (t > T.ucap) break;
    const float u = t_to_u(r, t);
    if (!(u < r.uexit)) break;
    if (T.prune) {
      if (res.key <= -T.tan_rL) break;
      const float need = need_tangent(T, res.key);
      if (clears(r, T, t, top, need)) break;
      if (mid && (k & (MID - 1)) == 0 &&
          steps_clear(T, r, level_of(T, mb), mb, t, u, step_t(T, k + MID - 1, step), need)) {
        k += MID - SS_CHUNK;
        continue;
      }
      if (small && steps_clear(T, r, level_of(T, ma), ma, t, u, step_t(T, k + SS_CHUNK - 1, step), need)) continue;
    }
    if (steps_whole(T, r, step, k, SS_CHUNK, u)) {
      for (int q = k; q < k + SS_CHUNK; q += HALF) {
        const float tq = step_t(T, q, step);
        if (small && steps_clear(T, r, level_of(T, mh), mh, tq, t_to_u(r, tq), step_t(T, q + HALF - 1, step),
                                 need_tangent(T, res.key)))
          continue;
        steps_inside<SPHERE, HALF>(T, r, L0, step, q, res, n_smp);
      }
    } else {
      for (int c = 0; c < SS_CHUNK; ++c) {
        const float tc = step_t(T, k + c, step);
        const float uc = t_to_u(r, tc);
        if (tc > T.ucap || !(uc < r.uexit)) {
          done = true;
          break;
        }
        take_step(r, k + c, tc, uc, sample_at(r, T, tc, uc).dh, res, n_smp);
      }
    }
  }
  res.alpha = angle_of(res.key);
}

// Uniform stepping (Sec. 2, Fig. 1b): every step.
// KEEP: as in shadow_dp; every step before an exit is taken.
template <bool SPHERE, bool KEEP>
__device__ __forceinline__ RayResult shadow_uniform(const TileK& T, const Ray<SPHERE>& r, float top,
                                                    unsigned& n_smp) {
  RayResult res;
  res.key = SS_INF;
  res.t = 0.0f;
  res.u = 0.0f;
  res.n = -1;
  res.valid = 0;
  step_through(T, r, top, T.ustep, T.ulev, !KEEP && T.prune == 1 && heights_finite(T), res, n_smp);
  return res;
}

// Entry m >= 0 of the tap-bound pyramid: the largest height any bilinear tap
// of a sample inside level-m texel (cx, cy) can read (also for samples up to
// half a texel outside it).
// The exact walk's pyramid level differs between lanes, so reading the level's
// offset from the kernel arguments would put a dependent memory load before
// every bound; kernels that run the walk copy the offsets to LDS first.
__device__ __forceinline__ void bound_tab_fill(const TileK& T, int* tab) {
  if (threadIdx.x >= 1 && threadIdx.x < (unsigned)T.L)
    tab[threadIdx.x] = (int)(T.lev[threadIdx.x].p - T.mm);
}

__device__ __forceinline__ float bound_at(const TileK& T, const int* tab, int m, int cx, int cy) {
  const float* base = m == 0 ? T.bnd : T.bmm + tab[m];
  const int w = (T.W + (1 << m) - 1) >> m;
  return base[idx2((unsigned)cy, (unsigned)w, (unsigned)cx)];
}

// Exact mode: the smallest clearance over every sample of the grid
// t_n = (n + 1) delta/2 up to the cap or the tile edge -- the grid of the
// descent's final samples (Alg. 1), i.e. uniform stepping at half a texel --
// found by branch and bound over the tap-bound pyramid (the global
// minimisation of Sec. 2 made exact).  A per-lane walk front to back over
// the sample index n and a pyramid level m:
//   * the level-m texel holding sample n bounds the terrain under every
//     sample whose position lies in it; if the point at that height below the
//     tip at t_n already clears the angle that could still matter, every
//     sample up to the texel's exit is skipped and the walk climbs a level;
//   * otherwise it descends a level, and at level 0 evaluates sample n.
// Every iteration either advances n or lowers m, so the walk ends.  The skips
// use the same margin as the other result-invariant exits, so the output is
// bit-identical to uniform stepping at half a texel (prune = 0 evaluates
// every sample).
//
// That walk is for tiles with missing or infinite heights, for prune = 0, for the
// forward that records the deciding sample (KEEP), for rays that may start anywhere
// (NEAR false), for steep suns and where the host finds that it costs less (know_heights).
// Otherwise the wavefront's rays step through the grid together (step_through): 64
// lanes at levels and samples of their own run every branch of an iteration, so the
// walk takes as long as its slowest ray at 130 instructions an iteration, mostly
// waiting for one gather.  Same results; us with the walk / stepping, 2048^2 tiles at
// 0.2 deg 6332 / 4385, at 1.5 deg in 4 x 16 ray tiles 902 to 1446 / 704 to 1101 over
// four azimuths, 1024^2 in 8 x 8 ray tiles 218 to 264 / 203 to 286.
//
// Branch and bound prunes best with a good incumbent: the descent (Sec. 3.2)
// runs first and its deciding sample, a sample of the same grid computed by
// the same arithmetic, seeds the minimum when it lies within the cap.  A ray
// the descent already finds in umbra is then done.
template <bool SPHERE, bool KEEP, bool NEAR>
__device__ __forceinline__ RayResult shadow_exact(const TileK& T, const Ray<SPHERE>& r, float top,
                                                  unsigned& n_tst, unsigned& n_smp,
                                                  const int* tab) {
  RayResult res;
  res.t = 0.0f;
  res.u = 0.0f;
  res.n = -1;
  res.valid = 0;
  float best = SS_INF;
  if (T.prune) {
    unsigned n_lb = 0, n_dp = 0;
    const RayResult d = shadow_dp<SPHERE, false, KEEP>(T, r, top, n_lb, n_dp);
    n_tst += n_lb;
    n_smp += n_dp;
    if (d.valid && d.t <= T.ucap) {
      res = d;
      best = d.key;
    }
  }
  if (!KEEP && NEAR && T.prune == 1 && T.Lz <= SS_EXACT_STEEP && heights_finite(T)) {
    res.key = best;
    step_through(T, r, top, T.half_delta, chunk_level(0.5), true, res, n_smp);
    return res;
  }
  float need = need_tangent(T, best);
  const int mtop = T.L - 1;
  const int ex = r.Kx >= 0.0f ? 1 : 0, ey = r.Ky >= 0.0f ? 1 : 0;
  // where the samples end: the cap, or the tile edge
  const float uend = fminf(r.uexit, t_to_u(r, T.ucap));
  int n = 0, m = 0;
  // the level-0 texel whose test last failed: its next sample is evaluated
  // without testing again (a test only ever skips work, so this changes no
  // result; the texel's second sample rarely clears where the first did not)
  int fx0 = -1, fy0 = -1;
  const bool umbra = T.prune && best <= -T.tan_rL;  // settled by the descent
  for (int it = 0; it < (umbra ? 0 : (1 << 24)); ++it) {
    const float t = step_t(T, n, T.half_delta);
    if (t > T.ucap) break;
    const float u = t_to_u(r, t);
    if (!(u < r.uexit)) break;
    // texel under sample n (rounding past the edge is clamped)
    const int ix = min(max((int)floorf((float)r.i + 0.5f + r.ox + r.Kx * u), 0), T.W - 1);
    const int iy = min(max((int)floorf((float)r.j + 0.5f + r.oy + r.Ky * u), 0), T.H - 1);
    const int cx = ix >> m, cy = iy >> m;
    bool skip = false;
    if (T.prune && !(m == 0 && ix == fx0 && iy == fy0)) {
      n_tst++;
      // relative to the origin the bound must be at least 0 (see clears)
      const float b0 = fmaxf(bound_at(T, tab, m, cx, cy) - r.hp, 0.0f);
      const float top = r.dz > b0 ? r.dz : b0;
      skip = clears(r, T, t, top, need);
    }
    if (skip) {
      // first grid sample at or past the texel's exit (a sample a rounding
      // error past the exit is still under the bound's half-texel margin)
      const float ux = ((float)(((cx + ex) << m) - r.i) - 0.5f - r.ox) * r.invKx;
      const float uy = ((float)(((cy + ey) << m) - r.j) - 0.5f - r.oy) * r.invKy;
      const float tb = u_to_t(r, fminf(fminf(ux, uy), uend));
      const float nb = ceilf(tb * T.two_over_delta) - 1.0f;
      n = max(n + 1, (int)fminf(nb, 16777216.0f));
      m = min(m + 1, mtop);
    } else if (m > 0) {
      --m;
    } else {
      fx0 = ix;
      fy0 = iy;
      const Sample s = sample_at(r, T, t, u);
      n_smp++;
      float num, den;
      clearance_terms(r, t, s.dh, num, den);
      const float key = tangent_key(num, den);
      if (key < best) {
        best = key;
        res.t = t;
        res.u = u;
        res.n = n;
        res.valid = 1;
        need = need_tangent(T, best);
        if (T.prune && best <= -T.tan_rL) break;  // umbra: nothing can change s = 0
      }
      ++n;
    }
  }
  res.key = best;
  res.alpha = angle_of(best);
  return res;
}

// No terrain rises above this (relative to h_p, at least 0).
template <bool SPHERE>
__device__ __forceinline__ float terrain_top(const TileK& T, const Ray<SPHERE>& r) {
  const float t0 = T.prune ? fmaxf(mip_at(T, T.L - 1, 0, 0), r.hp) - r.hp : 0.0f;
  return r.dz > t0 ? r.dz : t0;
}

// The shadow clearance of one ray by the chosen method.  KEEP: for a caller that hands
// out the deciding sample.  NEAR: the wavefront's rays start beside each other.
template <bool SPHERE, int MODE, bool KEEP = false, bool NEAR = true>
__device__ __forceinline__ RayResult trace_ray(const TileK& T, const Ray<SPHERE>& r, unsigned& n_lb,
                                               unsigned& n_smp, const int* tab) {
  const float top = terrain_top(T, r);
  if (MODE == SS_MODE_EXACT) return shadow_exact<SPHERE, KEEP, NEAR>(T, r, top, n_lb, n_smp, tab);
  if (MODE == SS_MODE_POINT) return shadow_dp<SPHERE, true>(T, r, top, n_lb, n_smp);
  if (MODE == SS_MODE_UNIFORM) return shadow_uniform<SPHERE, KEEP>(T, r, top, n_smp);
  return shadow_dp<SPHERE, false, KEEP>(T, r, top, n_lb, n_smp);
}
