// Heights moved between gnomonic tile frames (Sec. 3.3: visible tiles stitched
// into one texture; Sec. 4: cube-sphere faces) on gfx950.
//
// A frame is the plane tangent to the sphere at unit vector c with unit axes
// ex (+column) and ey (+row), texel spacing D in the plane and the plane
// coordinates (ox, oy) of its grid centre.  Destination texel (i, j) stands
// for the surface direction of P = R c + X ex + Y ey with
// X = ox + (i + 1/2 - W/2) D (Y likewise); its source texel coordinates come
// from central projection onto the source plane (P scaled so that P . c_s =
// R), and if they fall inside the source tile the texel receives the source's
// bilinear height there (texel centres, taps clamped).  Heights are radial,
// so they carry over unchanged.
//
// Positions and the blend are FP64, evaluated in a fixed order without
// contraction and rounded once to float32: a stitched halo is then the same
// float in every implementation of this definition, so shadows across seams
// do not depend on how the halo was built.
#include "kernels.h"

namespace ss {

namespace {

__device__ __forceinline__ double dot3(const double* a, const double* b) {
#pragma clang fp contract(off)
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// SAFE: divisions inside the range (the launcher looks at the frames).  A lane
// takes SS_RES_ROWS texels of one column, whose column part is then formed once.
// Bound by FP64 instructions, 72 a texel and ten conversions at a quarter of the
// rate, where the general divisions and a texel per lane took 95: 37 us for the
// half of a 4096^2 tile a source covers (2 and 8 rows per lane: 38.5 and 37.4; 72
// us for the whole tile before, of which half found itself outside the source).
#define SS_RES_ROWS 4

template <bool SAFE>
__global__ __launch_bounds__(256) void resample_kernel(ResampleK K) {
#pragma clang fp contract(off)
  const int i = K.i0 + blockIdx.x * 64 + (threadIdx.x & 63);
  const int jt = K.j0 + (blockIdx.y * 4 + (threadIdx.x >> 6)) * SS_RES_ROWS;
  if (i >= K.i1) return;
  const double X = K.oxd + ((double)i + 0.5 - 0.5 * (double)K.Wd) * K.Dd;
  double C[3];
  for (int k = 0; k < 3; ++k) C[k] = K.R * K.cd[k] + X * K.exd[k];
  // positions and taps of every row first, so that their loads overlap; texels
  // outside the source read a tap inside it and are not written
  double fx[SS_RES_ROWS], fy[SS_RES_ROWS];
  float h00[SS_RES_ROWS], h10[SS_RES_ROWS], h01[SS_RES_ROWS], h11[SS_RES_ROWS];
  bool in[SS_RES_ROWS];
#pragma unroll
  for (int row = 0; row < SS_RES_ROWS; ++row) {
    const int j = jt + row;
    const double Y = K.oyd + ((double)j + 0.5 - 0.5 * (double)K.Hd) * K.Dd;
    double P[3];
    for (int k = 0; k < 3; ++k) P[k] = C[k] + Y * K.eyd[k];
    const double z = dot3(P, K.cs);
    const double s = SAFE ? quot64_rn(K.R, z) : K.R / z;
    const double Xs = s * dot3(P, K.exs), Ys = s * dot3(P, K.eys);
    const double ax = Xs - K.oxs, ay = Ys - K.oys;
    const double qx = (SAFE ? quot64_by_rn(ax, K.Ds, K.invDs) : ax / K.Ds) + 0.5 * (double)K.Ws;
    const double qy = (SAFE ? quot64_by_rn(ay, K.Ds, K.invDs) : ay / K.Ds) + 0.5 * (double)K.Hs;
    in[row] = j < K.j1 && z > 0.0 && qx >= 0.0 && qx < (double)K.Ws && qy >= 0.0 && qy < (double)K.Hs;
    const double x = qx - 0.5, y = qy - 0.5;
    const double x0 = floor(x), y0 = floor(y);
    fx[row] = x - x0;
    fy[row] = y - y0;
    // x0 >= -1 and < Ws inside the source, so the clamps keep every tap there
    const int xi = in[row] ? (int)x0 : 0, yi = in[row] ? (int)y0 : 0;
    const int i0 = max(xi, 0), i1 = min(xi + 1, K.Ws - 1);
    // (rows and widths stay within 2^16, products below 2^30)
    const unsigned r0 = __umul24((unsigned)max(yi, 0), (unsigned)K.Ws);
    const unsigned r1 = __umul24((unsigned)min(yi + 1, K.Hs - 1), (unsigned)K.Ws);
    h00[row] = K.src[r0 + i0];
    h10[row] = K.src[r0 + i1];
    h01[row] = K.src[r1 + i0];
    h11[row] = K.src[r1 + i1];
  }
#pragma unroll
  for (int row = 0; row < SS_RES_ROWS; ++row) {
    const double gx = fx[row], gy = fy[row];
    const double v = (1.0 - gy) * ((1.0 - gx) * (double)h00[row] + gx * (double)h10[row]) +
                     gy * ((1.0 - gx) * (double)h01[row] + gx * (double)h11[row]);
    if (in[row]) K.dst[(size_t)(jt + row) * K.Wd + i] = (float)v;
  }
}

// The destination texels [i0, i1) x [j0, j1) that can fall into the source: its
// four corners seen from the destination plane.  When all lie in front of that
// plane the source's image is the quadrilateral they span (a central projection
// maps lines to lines), so its bounding box holds every covered texel; otherwise
// the whole tile stays.  Seen the other way round a position is off by up to
// 5e-9 (R + E)^2 / R, E metres out in the plane, as a frame's axes need only be
// orthogonal and of unit length within 1e-9: both the corners and the box are
// moved out by twice that (0.1 m on the Moon), and the box by two texels.
void covered(const ResampleK& K, int* i0, int* i1, int* j0, int* j1) {
  *i0 = *j0 = 0;
  *i1 = K.Wd;
  *j1 = K.Hd;
  double lo[2] = {1e300, 1e300}, hi[2] = {-1e300, -1e300}, out = 0.0;
  auto slack = [&](double e) { return 1e-8 * (K.R + e) * (1.0 + e / K.R); };
  const double sx = 0.5 * K.Ws * K.Ds, sy = 0.5 * K.Hs * K.Ds;
  const double grow = slack(fmax(fabs(K.oxs) + sx, fabs(K.oys) + sy));
  for (int c = 0; c < 4; ++c) {
    const double X = K.oxs + ((c & 1) ? 1.0 : -1.0) * (sx + grow);
    const double Y = K.oys + ((c & 2) ? 1.0 : -1.0) * (sy + grow);
    double P[3], z = 0.0, x = 0.0, y = 0.0;
    for (int k = 0; k < 3; ++k) {
      P[k] = K.R * K.cs[k] + X * K.exs[k] + Y * K.eys[k];
      z += P[k] * K.cd[k];
      x += P[k] * K.exd[k];
      y += P[k] * K.eyd[k];
    }
    if (!(z > 1e-3 * K.R)) return;
    x *= K.R / z;
    y *= K.R / z;
    out = fmax(out, fmax(fabs(x), fabs(y)));
    const double q[2] = {(x - K.oxd) / K.Dd + 0.5 * K.Wd, (y - K.oyd) / K.Dd + 0.5 * K.Hd};
    if (!isfinite(q[0]) || !isfinite(q[1])) return;
    for (int a = 0; a < 2; ++a) {
      lo[a] = fmin(lo[a], q[a]);
      hi[a] = fmax(hi[a], q[a]);
    }
  }
  if (!(hi[0] - lo[0] < 1e9 && hi[1] - lo[1] < 1e9)) return;
  const double pad = 2.0 + slack(out) / K.Dd;
  *i0 = (int)fmin(fmax(floor(lo[0] - pad), 0.0), (double)K.Wd);
  *i1 = (int)fmin(fmax(ceil(hi[0] + pad), 0.0), (double)K.Wd);
  *j0 = (int)fmin(fmax(floor(lo[1] - pad), 0.0), (double)K.Hd);
  *j1 = (int)fmin(fmax(ceil(hi[1] + pad), 0.0), (double)K.Hd);
}

bool ordinary(double v) { return fabs(v) > 1e-60 && fabs(v) < 1e60; }

}  // namespace

// Launched over the covered texels alone: on a 4096^2 tile across a cube-face
// seam each of the two sources covers half.
hipError_t launch_resample(const ResampleK& frames, hipStream_t stream) {
  ResampleK K = frames;
  covered(K, &K.i0, &K.i1, &K.j0, &K.j1);
  if (K.i0 >= K.i1 || K.j0 >= K.j1) return hipSuccess;
  K.invDs = 1.0 / K.Ds;
  const dim3 grid((unsigned)((K.i1 - K.i0 + 63) / 64),
                  (unsigned)((K.j1 - K.j0 + 4 * SS_RES_ROWS - 1) / (4 * SS_RES_ROWS)));
  if (ordinary(K.R) && ordinary(K.Ds) && ordinary(K.Dd))
    hipLaunchKernelGGL(resample_kernel<true>, grid, dim3(256), 0, stream, K);
  else
    hipLaunchKernelGGL(resample_kernel<false>, grid, dim3(256), 0, stream, K);
  return hipGetLastError();
}

}  // namespace ss
