// Maximum mipmap for gfx950 (Sec. 3.2, "Maximum mipmaps").
//
// A 256-thread workgroup reads one 64 x 64 block of the source level with
// coalesced 16-byte loads (each thread a 4 x 4 patch: four rows of float4) and
// writes up to six levels of that block:
//   +1, +2  in registers (2 x 2 and 1 x 1 per thread),
//   +3, +4  by cross-lane max within the wavefront (no LDS),
//   +5, +6  through a 4 x 4 LDS tile.
// Every texel is read from HBM once per launch; levels are written once.
//
// The build also says whether every height is a finite number, which the levels do
// not show (a maximum passes over a missing height): in the word after the top texel,
// inside the top level's 64-float slot (finite_word).  A launch hands its part of the
// answer to the next as NaN texels in the last level it writes; the workgroup that
// reads such a texel puts its maximum back from the level below.  No other workgroup
// reads it, so this takes no further launch, memory or pass: 16 multiply-adds a thread,
// and a barrier where fewer than five levels are written (a 4096^2 tile's first launch
// 16.5 us before and 17.2 with it; both launches of a 256^2 tile 5.8 and 6.4).  Builds
// that no stepping follows (a batch of descents, the tap-bound pyramid) leave it out and
// say "not known": 40 tiles of 64^2 in a batch 2.5 us each for 2.8.
#include "kernels.h"
#include "ray.h"

namespace ss {

struct MipDst {
  int off[6];
  int w[6];
  int h[6];
  const float* below;  // the level under the source (nullptr: the source is level 0)
  int bw, bh;
  int last;            // the last level written is the top
  unsigned key;        // finite_key of the tile
};

__device__ __forceinline__ float canon(float v) { return v + 0.0f; }  // -0 -> +0

// The value a lane of the same 16 holds (DPP control CTRL); 0 where there is none.
template <int CTRL>
__device__ __forceinline__ float from_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Writes F levels of one 64 x 64 block from its texels v (a 4 x 4 patch a thread,
// -inf where there is none).  CHECK: with the answer on finite heights, where mine says
// that this thread has seen another.  WORD: the top gets its word, "not known" without
// CHECK (the tap-bound pyramid has none).
template <bool CHECK, bool WORD>
__device__ __forceinline__ void block_levels(int F, const float (&v)[4][4], bool mine, float* dst,
                                             const MipDst& d, int bx, int by, float (&lds)[4][4],
                                             int (&lds_bad)[4]) {
  const int t = threadIdx.x;
  const int c4 = t & 15, rg = t >> 4;
  if (CHECK) {
    const bool wave_bad = __any(mine);
    if ((t & 63) == 0) lds_bad[t >> 6] = wave_bad;
  }
  // for the last level written, after a barrier: NaN hands the answer on, and the
  // thread that writes the top's texel leaves it beside it
  float mark = 0.0f;
  bool bad = false;
  auto gather = [&] {
    __syncthreads();
    if (!CHECK) return;
    bad = (lds_bad[0] | lds_bad[1] | lds_bad[2] | lds_bad[3]) != 0;
    mark = bad && !d.last ? __builtin_nanf("") : 0.0f;
  };
  auto verdict = [&](float top) {
    if (WORD && d.last)
      reinterpret_cast<unsigned*>(dst)[d.off[F - 1] + 1] =
          !CHECK || bad ? ~finite_word(top, d.key) : finite_word(top, d.key);
  };
  if (CHECK && F < 5) gather();
  // level +1: 2 x 2 per thread
  float a[2][2];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c)
      a[r][c] = fmaxf(fmaxf(v[2 * r][2 * c], v[2 * r][2 * c + 1]),
                      fmaxf(v[2 * r + 1][2 * c], v[2 * r + 1][2 * c + 1])) +
                (CHECK && F == 1 ? mark : 0.0f);
  {
    const int w1 = d.w[0], h1 = d.h[0];
    float* L1 = dst + d.off[0];
    const int cc = bx * 32 + c4 * 2;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int rr = by * 32 + rg * 2 + r;
      if (rr < h1) {
        if ((w1 & 1) == 0 && cc + 1 < w1) {
          *reinterpret_cast<float2*>(L1 + (size_t)rr * w1 + cc) = make_float2(a[r][0], a[r][1]);
        } else {
          if (cc < w1) L1[(size_t)rr * w1 + cc] = a[r][0];
          if (cc + 1 < w1) L1[(size_t)rr * w1 + cc + 1] = a[r][1];
        }
      }
    }
  }
  if (F == 1) {
    if (t == 0) verdict(a[0][0]);
    return;
  }
  // level +2: one value per thread
  float b2 = fmaxf(fmaxf(a[0][0], a[0][1]), fmaxf(a[1][0], a[1][1]));
  {
    const int rr = by * 16 + rg, cc = bx * 16 + c4;
    if (rr < d.h[1] && cc < d.w[1]) dst[d.off[1] + (size_t)rr * d.w[1] + cc] = b2 + (CHECK && F == 2 ? mark : 0.0f);
  }
  if (F == 2) {
    if (t == 0) verdict(b2);
    return;
  }
  // level +3: lanes (c4, c4^1) x (rg, rg^1) of the same wavefront
  float b3 = fmaxf(b2, __shfl_xor(b2, 1, 64));
  b3 = fmaxf(b3, __shfl_xor(b3, 16, 64));
  if (((c4 | rg) & 1) == 0) {
    const int rr = by * 8 + (rg >> 1), cc = bx * 8 + (c4 >> 1);
    if (rr < d.h[2] && cc < d.w[2]) dst[d.off[2] + (size_t)rr * d.w[2] + cc] = b3 + (CHECK && F == 3 ? mark : 0.0f);
  }
  if (F == 3) {
    if (t == 0) verdict(b3);
    return;
  }
  // level +4: lanes (c4, c4^2) x (rg, rg^2)
  float b4 = fmaxf(b3, __shfl_xor(b3, 2, 64));
  b4 = fmaxf(b4, __shfl_xor(b4, 32, 64));
  if (((c4 | rg) & 3) == 0) {
    const int rr = by * 4 + (rg >> 2), cc = bx * 4 + (c4 >> 2);
    if (rr < d.h[3] && cc < d.w[3]) dst[d.off[3] + (size_t)rr * d.w[3] + cc] = b4 + (CHECK && F == 4 ? mark : 0.0f);
    lds[rg >> 2][c4 >> 2] = b4;
  }
  if (F == 4) {
    if (t == 0) verdict(b4);
    return;
  }
  gather();
  if (t < 4) {
    const int r5 = t >> 1, c5 = t & 1;
    const float m5 = fmaxf(fmaxf(lds[2 * r5][2 * c5], lds[2 * r5][2 * c5 + 1]),
                           fmaxf(lds[2 * r5 + 1][2 * c5], lds[2 * r5 + 1][2 * c5 + 1]));
    const int rr = by * 2 + r5, cc = bx * 2 + c5;
    if (rr < d.h[4] && cc < d.w[4]) dst[d.off[4] + (size_t)rr * d.w[4] + cc] = m5 + (CHECK && F == 5 ? mark : 0.0f);
    if (F == 5 && t == 0) verdict(m5);
  }
  if (F == 5) return;
  if (t == 0) {
    float m6 = lds[0][0];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) m6 = fmaxf(m6, lds[r][c]);
    if (by < d.h[5] && bx < d.w[5]) dst[d.off[5] + (size_t)by * d.w[5] + bx] = m6 + (CHECK ? mark : 0.0f);
    verdict(m6);
  }
}

template <int F, bool CHECK>
__global__ __launch_bounds__(256) void maxmip_kernel(const float* src, int sw, int sh, float* dst,
                                                     MipDst d, int nbx, int vec_ok) {
  __shared__ float lds[4][4];
  __shared__ int lds_bad[4];  // per wavefront
  const int b = blockIdx.x;
  const int bx = b % nbx, by = b / nbx;
  const int t = threadIdx.x;
  const int c4 = t & 15, rg = t >> 4;
  const int col0 = bx * 64 + c4 * 4, row0 = by * 64 + rg * 4;
  const float NEG = -__builtin_inff();
  float v[4][4];
  float zero[4];  // 0 times finite numbers adds up to 0, anything else to NaN
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row0 + r;
    zero[r] = 0.0f;
    if (row < sh && vec_ok && col0 + 3 < sw) {
      const float4 q = *reinterpret_cast<const float4*>(src + (size_t)row * sw + col0);
      v[r][0] = canon(q.x);
      v[r][1] = canon(q.y);
      v[r][2] = canon(q.z);
      v[r][3] = canon(q.w);
#pragma unroll
      for (int c = 0; c < 4; ++c) zero[r] = fmaf(v[r][c], 0.0f, zero[r]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        v[r][c] = NEG;
        if (row < sh && col0 + c < sw) {
          v[r][c] = canon(src[(size_t)row * sw + col0 + c]);
          zero[r] = fmaf(v[r][c], 0.0f, zero[r]);
        }
      }
    }
  }
  const bool mine = CHECK && !((zero[0] + zero[1]) + (zero[2] + zero[3]) == 0.0f);
  if (mine && d.below) {
    for (int k = 0; k < 16; ++k) {
      const int y = row0 + (k >> 2), x = col0 + (k & 3);
      if (y < sh && x < sw && __builtin_isnan(v[k >> 2][k & 3])) {
        const bool hx = 2 * x + 1 < d.bw, hy = 2 * y + 1 < d.bh;  // absent beyond the edge
        const float* p = d.below + (size_t)(2 * y) * d.bw + 2 * x;
        const float m = fmaxf(fmaxf(canon(p[0]), hx ? canon(p[1]) : NEG),
                              fmaxf(hy ? canon(p[d.bw]) : NEG, hx && hy ? canon(p[d.bw + 1]) : NEG));
        const_cast<float*>(src)[(size_t)y * sw + x] = m;
        v[k >> 2][k & 3] = m;
      }
    }
  }
  block_levels<CHECK, true>(F, v, mine, dst, d, bx, by, lds, lds_bad);
}

// Tap-bound level 0: the maximum over the 3 x 3 block around each texel, clipped to
// the tile (repeating the edge row or column gives the same maximum), -0 stored as +0;
// and the first F levels of its maximum mipmap in the same pass.
//
// Bound by memory: the heights are read once and every level is written once, where a
// launch for level 0 and one for the mipmap read level 0 again (a 4096^2 tile: 24.8 and
// 16.4 us; 26.4 now, 38.6 with the patch read float by float).  Each thread takes the
// columns' maxima over three rows of its 4 x 4 patch and the columns beside the patch
// from the lanes next to it (DPP, 16 lanes to a row); the block's outer columns are
// loaded, from the L2 that neighbouring blocks share (xcd_remap: 1.5 us of it).
// VEC: 16-byte rows; a template and not a branch, as a branch's loads were merged into
// single floats.
template <bool VEC>
__global__ __launch_bounds__(256) void bound_kernel(const float* __restrict__ src, int W, int H,
                                                    float* __restrict__ level0, float* dst, MipDst d,
                                                    int F, int nbx) {
  __shared__ float lds[4][4];
  __shared__ int unused[4];
  const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);  // neighbours in one L2
  const int bx = b % nbx, by = b / nbx;
  const int t = threadIdx.x;
  const int c4 = t & 15, rg = t >> 4;
  const int col0 = bx * 64 + c4 * 4, row0 = by * 64 + rg * 4;
  const float NEG = -__builtin_inff();
  // the block's outer column of this lane, where it has one
  const int side = c4 == 0 ? max(col0 - 1, 0) : min(col0 + 4, W - 1);
  const bool outer = c4 == 0 || c4 == 15;
  // six rows: the patch's and one on either side, repeated at the tile's edge
  float q[6][4], o[6];
  auto row_at = [&](int r) { return src + (size_t)min(max(row0 + r - 1, 0), H - 1) * W; };
  if (VEC) {
    // W is a multiple of 4: a patch lies inside or beyond the edge as a whole, and
    // one beyond it repeats the last column for the lane before it
    float4 x[6];
#pragma unroll
    for (int r = 0; r < 6; ++r)
      x[r] = *reinterpret_cast<const float4*>(row_at(r) + min(col0, W - 4));
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      q[r][0] = col0 < W ? x[r].x : x[r].w;
      q[r][1] = x[r].y;
      q[r][2] = x[r].z;
      q[r][3] = x[r].w;
    }
  } else {
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) q[r][c] = row_at(r)[min(col0 + c, W - 1)];
  }
#pragma unroll
  for (int r = 0; r < 6; ++r) o[r] = outer ? row_at(r)[side] : NEG;
  float v[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float m[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = fmaxf(fmaxf(q[r][c], q[r + 1][c]), q[r + 2][c]);
    const float mo = fmaxf(fmaxf(o[r], o[r + 1]), o[r + 2]);
    float left = from_lane<0x111>(m[3]), right = from_lane<0x101>(m[0]);  // row_shr:1, row_shl:1
    if (c4 == 0) left = mo;
    if (c4 == 15) right = mo;
    v[r][0] = canon(fmaxf(fmaxf(left, m[0]), m[1]));
    v[r][1] = canon(fmaxf(fmaxf(m[0], m[1]), m[2]));
    v[r][2] = canon(fmaxf(fmaxf(m[1], m[2]), m[3]));
    v[r][3] = canon(fmaxf(fmaxf(m[2], m[3]), right));
    const int row = row0 + r;
    if (VEC) {
      const bool in = row < H && col0 < W;
      if (in)
        *reinterpret_cast<float4*>(level0 + (size_t)row * W + col0) =
            make_float4(v[r][0], v[r][1], v[r][2], v[r][3]);
#pragma unroll
      for (int c = 0; c < 4; ++c) v[r][c] = in ? v[r][c] : NEG;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (row < H && col0 + c < W)
          level0[(size_t)row * W + col0 + c] = v[r][c];
        else
          v[r][c] = NEG;
      }
    }
  }
  if (F > 0) block_levels<false, false>(F, v, false, dst, d, bx, by, lds, unused);
}

hipError_t launch_bound(const float* src, int W, int H, float* level0, float* dst_base,
                        const int* dst_off, const int* dst_w, const int* dst_h, int F,
                        hipStream_t stream) {
  MipDst d{};
  for (int k = 0; k < F; ++k) {
    d.off[k] = dst_off[k];
    d.w[k] = dst_w[k];
    d.h[k] = dst_h[k];
  }
  const int nbx = (W + 63) / 64, nby = (H + 63) / 64;
  const int vec_ok = W % 4 == 0 && ((reinterpret_cast<uintptr_t>(src) |
                                     reinterpret_cast<uintptr_t>(level0)) & 15) == 0;
  if (vec_ok)
    hipLaunchKernelGGL(bound_kernel<true>, dim3(nbx * nby), dim3(256), 0, stream, src, W, H, level0,
                       dst_base, d, F, nbx);
  else
    hipLaunchKernelGGL(bound_kernel<false>, dim3(nbx * nby), dim3(256), 0, stream, src, W, H, level0,
                       dst_base, d, F, nbx);
  return hipGetLastError();
}

// The heights read once more, before a call that passes over terrain where all of them
// are known to be finite.  A height can go missing after the build without a change to
// any maximum, and a mipmap can be filled in beside a word from an earlier build; the
// check only ever takes the word back, so calls on other streams see the same tile the
// same way.  Bound by memory, four 16-byte loads in flight a thread: 4.0 us up to 2048^2,
// 11.4 at 4096^2 and 48 at 8192^2 (5.6 TB/s), where stepping takes hundreds.
__global__ __launch_bounds__(256) void finite_check_kernel(const float* __restrict__ h, unsigned n,
                                                           float* top, unsigned key) {
  if (finite_word(top[0], key) != __float_as_uint(top[1])) return;  // not said to be finite
  typedef float quad __attribute__((ext_vector_type(4), aligned(4)));
  const unsigned stride = gridDim.x * 256u, quads = n >> 2, at = blockIdx.x * 256u + threadIdx.x;
  float zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // as in maxmip_kernel
  auto add = [&](quad v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) zero[c] = fmaf(v[c], 0.0f, zero[c]);
  };
  const quad* q = reinterpret_cast<const quad*>(h);
  unsigned k = at;
  for (; k < quads && quads - k > 3 * stride; k += 4 * stride) {
    const quad a = q[k], b = q[k + stride], c = q[k + 2 * stride], d = q[k + 3 * stride];
    add(a);
    add(b);
    add(c);
    add(d);
  }
  for (; k < quads; k += stride) add(q[k]);
  if (at < (n & 3)) zero[0] = fmaf(h[(quads << 2) + at], 0.0f, zero[0]);
  if (!((zero[0] + zero[1]) + (zero[2] + zero[3]) == 0.0f))
    reinterpret_cast<unsigned*>(top)[1] = ~finite_word(top[0], key);
}

hipError_t launch_finite_check(const TileK& T, hipStream_t stream) {
  const unsigned n = (unsigned)T.W * (unsigned)T.H;  // below 2^30
  const unsigned blocks = (n / 4 + 1023) / 1024;     // four 16-byte loads a thread
  hipLaunchKernelGGL(finite_check_kernel, dim3(blocks < 1 ? 1 : (blocks < 8192 ? blocks : 8192)),
                     dim3(256), 0, stream, T.h, n, const_cast<float*>(T.lev[T.L - 1].p),
                     finite_key(T.W, T.H));
  return hipGetLastError();
}

hipError_t launch_maxmip(const float* src, int sw, int sh, float* dst_base, const int* dst_off,
                         const int* dst_w, const int* dst_h, int F, const float* below, int bw,
                         int bh, int last, unsigned key, bool check, hipStream_t stream) {
  MipDst d;
  d.below = below;
  d.bw = bw;
  d.bh = bh;
  d.last = last;
  d.key = key;
  for (int k = 0; k < 6; ++k) {
    d.off[k] = k < F ? dst_off[k] : 0;
    d.w[k] = k < F ? dst_w[k] : 0;
    d.h[k] = k < F ? dst_h[k] : 0;
  }
  const int nbx = (sw + 63) / 64, nby = (sh + 63) / 64;
  const int nb = nbx * nby;
  if (nb == 0) return hipSuccess;
  const int vec_ok = ((reinterpret_cast<uintptr_t>(src) & 15) == 0) && (sw % 4 == 0);
  dim3 grid(nb), block(256);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, src, sw, sh, dst_base, d, nbx, vec_ok);
  };
  switch (F) {
    case 1: check ? launch(maxmip_kernel<1, true>) : launch(maxmip_kernel<1, false>); break;
    case 2: check ? launch(maxmip_kernel<2, true>) : launch(maxmip_kernel<2, false>); break;
    case 3: check ? launch(maxmip_kernel<3, true>) : launch(maxmip_kernel<3, false>); break;
    case 4: check ? launch(maxmip_kernel<4, true>) : launch(maxmip_kernel<4, false>); break;
    case 5: check ? launch(maxmip_kernel<5, true>) : launch(maxmip_kernel<5, false>); break;
    default: check ? launch(maxmip_kernel<6, true>) : launch(maxmip_kernel<6, false>); break;
  }
  return hipGetLastError();
}

}  // namespace ss
