// Parameter block shared by the host set-up and the gfx950 kernels.
//
// The host forms every per-(tile, sun) quantity in FP64 and rounds it once to
// FP32 here; the kernels work in FP32 relative to each ray's origin.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#define SS_MAXLEV 18   // supports max(width, rows) <= 65536
#define SS_MAXSEG 48   // concatenated runs per ray
#define SS_TILEK_BYTES 928
#define SS_FITRUNS 29          // runs with bounds of the tip height's fit
#define SS_REFIT 3             // the fit is taken again this many levels below a run's top
#define SS_REFIT_FROM 7        // in runs of this level and up
#define SS_FIT_NONE 0xffffffffu  // no fit: the run takes the general descent

// One mip level: its texels [h][w].  The address, the width and the row count
// a gather needs sit side by side, so a kernel reads them with one scalar load.
struct LevelK {
  const float* p;
  int w, h;
};

struct TileK {
  const float* h;            // level 0: the heightfield, [H][W]
  const float* mm;           // levels >= 1, packed (lev[m].p)
  const float* bnd;          // tap-bound pyramid level 0, [H][W] (exact mode only)
  const float* bmm;          // its levels >= 1, packed like mm
  int W, H, L;               // size and number of mip levels (incl. level 0)
  int rx0, ry0, RW, RH;      // ray window: origins (rx0 + x, ry0 + y), x < RW, y < RH
  LevelK lev[SS_MAXLEV];     // level m of the heightfield (m = 0) and its mipmap
  float texel;               // texel spacing on the tangent plane (m)
  float invR;                // 1 / body radius (0 on the plane)
  float Lx, Ly, Lz;          // unit vector toward the sun centre, tile frame
  float half_delta;          // delta/2, delta = texel / cos(elev): first sample and grid step
  float two_over_delta;      // 2 / delta
  float rL, inv_rL;          // sun disc angular radius and its inverse
  float prune_margin;        // safety margin (rad) of the result-invariant exits
  float tan_rL;              // tan(r_L)
  float tan_margin;          // tan(prune_margin)
  float ustep;               // uniform stepping: step in ray length (m)
  float ucap;                // uniform stepping: cap on ray length (m), +inf = tile edge
  int nseg;                  // number of concatenated runs
  float tau[SS_MAXSEG + 1];  // ray length where run j starts (tau[nseg] = end)
  unsigned run[SS_MAXSEG];   // run j: grid index of its start, and its top mip level (run_pack)
  int prune;                 // 1: result-invariant early exits enabled; 2: but stepping passes
                             // over nothing (the heights may not all be finite)
  int wg_group;              // per-tile kernels: workgroup ids are remapped within groups of
                             // this many (8 per CU: twice the SIMDs)
  int ulev;                  // uniform stepping: chunk_level
  unsigned fit_err[SS_FITRUNS];  // run j: error bounds of the tip height's fits (fit_err_pack)
};
// The batched workspace holds one block per (tile, sun) pair, and how many
// pairs the fixed array of the allocation-free call takes follows from this
// size: callers rely on which batches fit.
static_assert(sizeof(TileK) == SS_TILEK_BYTES, "the parameter block's size is part of the interface");

// The word after the mipmap's top texel: finite_word(top, key) when every height of
// the tile is a finite number (any other value: not known to be).  The tile's size
// and top are in it so that a word left by another tile in the same memory hardly
// passes for it.  It says what a build saw, and heights may have gone missing since
// (maxima do not show it), so a call that relies on it has the heights looked at first
// (launch_finite_check).
__host__ __device__ inline unsigned finite_key(int W, int H) {
  return 0x5f3c9a17u ^ ((unsigned)W * 0x9e3779b1u) ^ ((unsigned)H * 0x85ebca6bu);
}
__device__ __forceinline__ unsigned finite_word(float top, unsigned key) {
  return __builtin_bit_cast(unsigned, top) ^ key;
}

// The exact mode steps for suns below 30 degrees (the sine) and walks above, where rays
// climb out of the terrain's reach within a few samples: us stepping / walking, 1024^2
// at 20 deg 190 / 223, at 45 89 / 73, at 75 60 / 50, 512^2 at 20 137 / 140, at 75 29 / 23.
#define SS_EXACT_STEEP 0.5f

// Steps are taken SS_CHUNK at a time.
#define SS_CHUNK 16

// The finest mip level of whose texels two by two hold the taps of a chunk of
// `step` texels per step: one texel there spans the chunk's travel (a tenth to
// spare for tiles whose plane bends away) and the taps around its ends.
constexpr int chunk_level(double step) {
  int m = 0;
  while (m < SS_MAXLEV && (double)(1LL << m) < (SS_CHUNK - 1) * step * 1.1 + 2.0) ++m;
  return m;
}

// Run j starts at half-texel grid index a0 (tau_j = (a0 + 1) delta/2) and
// descends from mip level m0.  a0 stays below 2^27: at most SS_MAXSEG runs of
// 2^(m0 + 1) half texels, m0 < SS_MAXLEV.
__host__ __device__ inline unsigned run_pack(int a0, int m0) {
  return (unsigned)a0 | ((unsigned)m0 << 27);
}
__host__ __device__ inline int run_a0(unsigned run) { return (int)(run & 0x7ffffffu); }
__host__ __device__ inline int run_m0(unsigned run) { return (int)(run >> 27); }

// Twice the bound (metres) of the tip height's second-order fit against the
// kernels' exact FP32 tip height over the rays of a tile: over a whole run of
// level m that starts at ray length t0 and ends at t1, and, once it is taken again
// SS_REFIT levels down, over the stretch left there.  The parts: rounding of
// either form (a few ulps of the terms' size), the third- and fourth-order terms
// of the series over the stretch, and the series' remainder over the ray.
// lz: the sun's z; ext: half the tile's diagonal; rho >= 0.95 R (origins further
// down take the general descent).  Where the series is not small, or the bounds
// are coarse against the terrain under one texel, there is no fit.  The figure
// only decides where exact bounds are evaluated, never a result.
__host__ __device__ inline double fit_err_at(double radius, double lz, double ext, double t1,
                                             double len) {
  const double rho = 0.95 * radius, g = sqrt(1.0 + (ext / radius) * (ext / radius));
  const double s = fmin(1.0, fabs(lz) + ext / radius), c = fabs(lz) * g / rho;
  if (!(c * t1 <= 0.25)) return 1e30;
  const double q = 1.0 / (1.0 - c * t1), U = t1 * q, d = 0.5 * len * q * q, x = U / rho;
  if (!(x <= 0.25)) return 1e30;
  const double a3 = s * c * c + c / rho + 0.5 * s / (rho * rho);
  const double a4 = s * c * c * c + 1.5 * c * c / rho + 1.5 * s * c / (rho * rho) +
                    0.5 / (rho * rho * rho);
  const double x5 = x * x * x * x * x;
  return 2.0 * (1.5e-6 * (s * U + 0.5 * U * x) + (a3 + 4.0 * a4 * U) * d * d * d +
                a4 * d * d * d * d + rho * x5 * (s + c * rho + 0.25 * x));
}

// Both bounds of a run (run_pack), rounded up to 16-bit floats: the upper half
// holds over the whole run, the lower half once the fit is taken again (runs of
// level SS_REFIT_FROM and up; a stretch inside one texel of the level reached is
// at most 1.5 texels of travel long).  From the fields of TileK, so that the
// host and the expand kernel form the same.
__host__ __device__ inline unsigned run_fit_err(int W, int H, float texel, float invR, float Lz,
                                                double half_delta, unsigned run) {
  if (invR == 0.0f) return 0u;  // the plane's tip height is linear as it is
  const double radius = 1.0 / (double)invR, w = W, h = H;
  const double ext = 0.5 * sqrt(w * w + h * h) * (double)texel;
  const int m = run_m0(run);
  const double t1 = (double)(run_a0(run) + (2 << m) + 1) * half_delta;
  const double len = (double)(2 << m) * half_delta;
  const double top = fit_err_at(radius, Lz, ext, t1, len);
  const double low = fit_err_at(radius, Lz, ext, t1, ldexp(1.5 * len, -SS_REFIT));
  if (!((m >= SS_REFIT_FROM ? low : top) < 0.02 * (double)texel)) return SS_FIT_NONE;
  const float f[2] = {(float)fmin(top, 1e30), (float)fmin(low, 1e30)};
  unsigned u[2];
  memcpy(u, f, sizeof u);
  return ((u[0] + 0x10000u) & 0xffff0000u) | ((u[1] + 0x10000u) >> 16);
}
__device__ inline float fit_err_top(unsigned e) { return __builtin_bit_cast(float, e & 0xffff0000u); }
__device__ inline float fit_err_low(unsigned e) { return __builtin_bit_cast(float, e << 16); }

// Ray length where the run starting at half-texel grid index a begins:
// tau = (a + 1) delta/2, one FP64 product rounded once to FP32.  The per-tile
// set-up on the host and the batched call's expand kernel on the device both
// form it this way, so their parameter blocks agree bit for bit.
__host__ __device__ inline float run_start_len(int a, double half_delta) {
  return (float)((double)(a + 1) * half_delta);
}

#ifdef __HIP_DEVICE_COMPILE__
#define SS_RCP_SEED(x) __builtin_amdgcn_rcpf(x)
#define SS_RSQ_SEED(x) __builtin_amdgcn_rsqf(x)
#define SS_RCP64_SEED(x) __builtin_amdgcn_rcp(x)
#else  // the host pass only parses the kernels
#define SS_RCP_SEED(x) (1.0f / (x))
#define SS_RSQ_SEED(x) (1.0f / sqrtf(x))
#define SS_RCP64_SEED(x) (1.0 / (x))
#endif

// The correctly rounded reciprocal, root and quotient, as 1.0f / x, sqrtf(x) and
// a / b give them, where operands and results are normal numbers with exponents
// well inside the range (a numerator below 2^-100 leaves a residual of denormals):
// without the scaling and special cases of the general sequences they take 3, 5 and
// 5 (given y = rcp_rn(b)) instructions in place of 11, 16 and 11.  The hardware's
// reciprocal and reciprocal root are within an ulp; one Newton step rounds correctly
// for every mantissa (no theorem, but there are only 2^24 of two adjacent exponents:
// ss_probe_rounding compares them all with the general forms).  The quotient follows
// from a correctly rounded y by Markstein's theorem: after the first correction q is
// within an ulp, after the second it is rounded correctly.
__device__ inline float rcp_rn(float x) {
  const float y = SS_RCP_SEED(x);
  return fmaf(fmaf(-x, y, 1.0f), y, y);
}
__device__ inline float sqrt_rn(float x) {
  const float y = SS_RSQ_SEED(x), s = x * y;
  return fmaf(fmaf(-s, s, x), 0.5f * y, s);
}
__device__ inline float div_rn(float a, float b, float y) {
  float q = a * y;
  q = fmaf(fmaf(-b, q, a), y, q);
  return fmaf(fmaf(-b, q, a), y, q);
}

// n / d in FP64 rounded correctly for operands and results inside the range: the
// general sequence without its scaling and fix-up, which leave such operands alone.
__device__ inline double quot64_rn(double n, double d) {
  double y = SS_RCP64_SEED(d);
  y = fma(fma(-d, y, 1.0), y, y);
  y = fma(fma(-d, y, 1.0), y, y);
  const double q = n * y;
  return fma(fma(-d, q, n), y, q);
}

// The same for a divisor whose correctly rounded reciprocal y is known: after the
// second correction the quotient is rounded correctly (Markstein).
__device__ inline double quot64_by_rn(double n, double d, double y) {
  double q = n * y;
  q = fma(fma(-d, q, n), y, q);
  return fma(fma(-d, q, n), y, q);
}

// Ray tile shapes: lanes of one wavefront cover TW x TH texels (TW * TH = 64),
// a 256-thread workgroup covers 2 x 2 wavefront tiles.
enum { SS_TILE_8x8 = 1, SS_TILE_16x4 = 2, SS_TILE_4x16 = 3, SS_TILE_32x2 = 4 };
