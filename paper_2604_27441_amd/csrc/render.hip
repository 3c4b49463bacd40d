// RGB-D unprojection and z-buffered rendering of a new view: the receiver
// step after recovery, which turns each recovered RGB-D pair into 3-D points
// (an RGB-D frame projected into Cartesian space, Sec. 2) and renders them
// for a viewpoint (Sec. 5 microbenchmarks).
//
// Pinhole camera, pixel centres at integer coordinates, depth = z in mm
// (0 = no measurement).  Unprojection writes an organised cloud, one float4
// (X, Y, Z, valid) per pixel.  Rendering moves each point by X' = R X + t,
// projects it to the nearest target pixel centre and keeps, per pixel, the
// point of smallest Z' (ties to the lower index) with a 64-bit atomic min on
// (bits of Z', point index), first among the points of a tile: positive floats
// order like their bit patterns.
// A resolve pass then writes the winner's colour and Z' rounded to mm.
#include <math.h>

#include "kernels.h"

namespace revo {

namespace {

constexpr int RT = 256;

struct Intr {
  float fx, fy, cx, cy;
};
struct Pose {
  float r[9], t[3];
};

// grid (columns / RT, rows, frames)
__global__ __launch_bounds__(RT) void unproject_kernel(const uint16_t* __restrict__ depth, int H, int W, Intr k,
                                                       float4* __restrict__ pts) {
  const int u = blockIdx.x * RT + threadIdx.x;
  if (u >= W) return;
  const int v = blockIdx.y;
  const long long i = ((long long)blockIdx.z * H + v) * W + u;
  const float z = (float)depth[i];
  pts[i] = make_float4(((float)u - k.cx) * z / k.fx, ((float)v - k.cy) * z / k.fy, z, z > 0.0f ? 1.0f : 0.0f);
}

__global__ void zbuf_clear_kernel(unsigned long long* __restrict__ zbuf, long long n) {
  const long long i = (long long)blockIdx.x * RT + threadIdx.x;
  if (i < n) zbuf[i] = ~0ull;
}

// Target pixel and key of point p (index n), false when it is not rendered.
__device__ __forceinline__ bool project_point(const float4& p, unsigned n, const Pose& P, const Intr& k, int Ho, int Wo,
                                              int& iu, int& iv, unsigned long long& key) {
  if (!(p.w > 0.0f)) return false;
  const float x = P.r[0] * p.x + P.r[1] * p.y + P.r[2] * p.z + P.t[0];
  const float y = P.r[3] * p.x + P.r[4] * p.y + P.r[5] * p.z + P.t[1];
  const float z = P.r[6] * p.x + P.r[7] * p.y + P.r[8] * p.z + P.t[2];
  if (!(z > 0.0f)) return false;
  const float fu = k.fx * x / z + k.cx + 0.5f, fv = k.fy * y / z + k.cy + 0.5f;
  if (!(fu >= 0.0f && fu < (float)Wo && fv >= 0.0f && fv < (float)Ho)) return false;
  iu = (int)floorf(fu);
  iv = (int)floorf(fv);
  if (iu >= Wo || iv >= Ho) return false;  // fu just below Wo can round up to it
  key = ((unsigned long long)__float_as_uint(z) << 32) | n;
  return true;
}

// Splat of one tile of 64 x 4 SPT source points, grid (tiles across, tiles down,
// frames), wave w taking rows w, w + 4, ...  What bounds a large launch is the
// rate of atomics on the z-buffer's lines: in a turned view 64 neighbouring
// points land on pieces of some 30 lines, and one atomic per point takes 79 us
// with four 1280x720 frames (clear, splat and resolve).  The tile's target
// pixels mostly fill a small box, so its points first meet in a z-buffer of that
// box in LDS, and the box's winners then go to the z-buffer row by row, whole
// lines per wave: 50 us.  A box that does not fit (a depth edge, noise in the
// depth, a strong rotation) is cut to the columns around its points' mean, and
// the other points, or all of a box too tall for that, go to the z-buffer
// themselves.
// The box costs a wave two more barriers and a pass over its pixels, so a wave
// whose atomics are cheap already sends its points itself: those whose points,
// per lane, continue on their left neighbour's line and rarely on its very
// pixel (atomics on one pixel take turns).  Calls of 400 000 points or fewer
// never fill the chip, so they take one row per wave, count no lines and box
// only points that collide.  us with an atomic per point, with a box for every
// tile of 64 x 16, and as it is (captured launches; the view is 100 mm aside and 5
// degrees off unless said): four 1280x720 frames 79, 51, 50,
// unmoved 44, 48, 43, at half size 83, 28, 29, a tenth of the points valid 34.6,
// 39.5, 33.8, depth all noise 91, 80, 75; one 640x480 frame 11.7, 12.0, 11.6,
// unmoved 8.9, 10.9, 9.0, 6 m back 21.6, 11.8, 15.4; one 256x192 frame 6.1, 8.7,
// 6.2.  Behind the atomic per point by 4 to 12 %: one unmoved 1280x720 frame 14.0,
// 16.3, 14.7, two 640x480 frames of patches of a fifth of the points 11.3, 13.5,
// 12.1, one 1280x720 frame of a few bands of rows 10.3, 13.3, 11.5, four frames of
// much missing depth 400 mm nearer 40.6, 46.2, 42.6.  (12 to 20 for a lone frame's
// MAX_SAME give 11.3 to 13.4 from 6 m back, but 6.4 to 6.6 for the 256x192 frame.)
// The minimum is the same by every way.  16 KB of LDS leave 8 workgroups per CU.
constexpr int SW = 64, SBOX = 2048;
constexpr long long SMALL_SPLAT = 400000;  // points of all frames of a call
template <int SPT>
__global__ __launch_bounds__(RT) void splat_kernel(const float4* __restrict__ pts, int H, int W, Pose P, Intr k,
                                                   int Ho, int Wo, unsigned long long* __restrict__ zbuf) {
  constexpr int SH = 4 * SPT;
  // most new lines and repeated pixels of a wave's points that still go themselves
  constexpr int MAX_LINES = SPT == 1 ? 64 : 28, MAX_SAME = SPT == 1 ? 24 : 8;
  __shared__ unsigned long long box[SBOX];
  __shared__ int ext[4][RT / 64], boxed[RT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int u = blockIdx.x * SW + lane;
  const float4* src = pts + (long long)blockIdx.z * H * W;
  unsigned long long* dst = zbuf + (long long)blockIdx.z * Ho * Wo;
  int iu[SPT], iv[SPT];
  unsigned long long key[SPT];
  bool ok[SPT];
  int u0 = Wo, u1 = -1, v0 = Ho, v1 = -1;
  float4 p[SPT];
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int v = blockIdx.y * SH + wave + 4 * i;
    p[i] = u < W && v < H ? src[(unsigned)(v * W + u)] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int v = blockIdx.y * SH + wave + 4 * i;
    ok[i] = project_point(p[i], (unsigned)(v * W + u), P, k, Ho, Wo, iu[i], iv[i], key[i]);
    if (ok[i]) {
      u0 = min(u0, iu[i]);
      u1 = max(u1, iu[i]);
      v0 = min(v0, iv[i]);
      v1 = max(v1, iv[i]);
    }
  }
  int lines = 0, same = 0;
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    // (in a wave of 64 the lanes without a neighbour in their row of 16 count as
    // a new line; a line is 8 pixels, rows need not start on one)
    const unsigned px = ok[i] ? (unsigned)iv[i] * Wo + iu[i] : ~0u;
    const unsigned left = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)px, 0x111, 0xF, 0xF, false);
    lines += __popcll(__ballot(ok[i] && (px ^ left) >= 8u));
    same += __popcll(__ballot(ok[i] && px == left));
  }
  const bool direct = lines <= MAX_LINES && same <= MAX_SAME;
  if (direct) {
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      if (ok[i]) atomicMin(dst + (long long)iv[i] * Wo + iu[i], key[i]);
      ok[i] = false;
    }
  }
  if (lane == 0) boxed[wave] = !direct;
  __syncthreads();
  if (!(boxed[0] | boxed[1] | boxed[2] | boxed[3])) return;
  if (direct) {
    u0 = Wo; u1 = -1; v0 = Ho; v1 = -1;
  } else {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      u0 = min(u0, __shfl_xor(u0, o));
      u1 = max(u1, __shfl_xor(u1, o));
      v0 = min(v0, __shfl_xor(v0, o));
      v1 = max(v1, __shfl_xor(v1, o));
    }
  }
  if (lane == 0) {
    ext[0][wave] = u0;
    ext[1][wave] = u1;
    ext[2][wave] = v0;
    ext[3][wave] = v1;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < RT / 64; ++w) {
    u0 = min(u0, ext[0][w]);
    u1 = max(u1, ext[1][w]);
    v0 = min(v0, ext[2][w]);
    v1 = max(v1, ext[3][w]);
  }
  if (u1 < u0) return;  // nothing to render
  // rows of the box start at a multiple of 8 pixels, one 64-byte line
  u0 &= ~7;
  int bw = u1 - u0 + 1;
  const int bh = v1 - v0 + 1;
  if ((long long)bw * bh > SBOX) {
    // the columns around the points' mean that fit, the other points by themselves
    const bool some = bh <= SBOX / 64;
    if (some) {
      __syncthreads();  // ext is read
      float su = 0.0f;
      int nu = 0;
#pragma unroll
      for (int i = 0; i < SPT; ++i)
        if (ok[i]) {
          su += (float)(iu[i] - u0);
          ++nu;
        }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        su += __shfl_xor(su, o);
        nu += __shfl_xor(nu, o);
      }
      if (lane == 0) {
        ext[0][wave] = __float_as_int(su);
        ext[1][wave] = nu;
      }
      __syncthreads();
      su = 0.0f;
      nu = 0;
#pragma unroll
      for (int w = 0; w < RT / 64; ++w) {
        su += __int_as_float(ext[0][w]);
        nu += ext[1][w];
      }
      const int width = (SBOX / bh) & ~7;
      u0 += max(0, min((int)(su / (float)nu) - width / 2, bw - width)) & ~7;
      bw = min(width, u1 - u0 + 1);
    }
#pragma unroll
    for (int i = 0; i < SPT; ++i)
      if (ok[i] && (!some || (unsigned)(iu[i] - u0) >= (unsigned)bw)) {
        atomicMin(dst + (long long)iv[i] * Wo + iu[i], key[i]);
        ok[i] = false;
      }
    if (!some) return;
  }
  const int n = bw * bh;
  for (int i = tid; i < n; i += RT) box[i] = ~0ull;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SPT; ++i)
    if (ok[i]) atomicMin(&box[(iv[i] - v0) * bw + iu[i] - u0], key[i]);
  __syncthreads();
  const float inv = 1.0f / (float)bw;
  for (int i = tid; i < n; i += RT) {
    const unsigned long long b = box[i];
    if (b == ~0ull) continue;
    const int r = (int)(((float)i + 0.5f) * inv);  // i / bw: both below 2^13
    atomicMin(dst + (long long)(v0 + r) * Wo + u0 + (i - r * bw), b);
  }
}

// grid (target columns / RT, target rows, frames)
__global__ __launch_bounds__(RT) void resolve_kernel(const unsigned long long* __restrict__ zbuf,
                                                     const uint8_t* __restrict__ rgb, int H, int W, int Ho, int Wo,
                                                     uint8_t* __restrict__ rgb_out, uint16_t* __restrict__ depth_out) {
  const int u = blockIdx.x * RT + threadIdx.x;
  if (u >= Wo) return;
  const long long o = ((long long)blockIdx.z * Ho + blockIdx.y) * Wo + u;
  const unsigned long long key = zbuf[o];
  uint8_t c0 = 0, c1 = 0, c2 = 0;
  uint16_t d = 0;
  if (key != ~0ull) {
    const long long n = (long long)blockIdx.z * H * W + (unsigned)(key & 0xffffffffu);
    c0 = rgb[3 * n]; c1 = rgb[3 * n + 1]; c2 = rgb[3 * n + 2];
    d = (uint16_t)fminf(rintf(__uint_as_float((unsigned)(key >> 32))), 65535.0f);
  }
  rgb_out[3 * o] = c0; rgb_out[3 * o + 1] = c1; rgb_out[3 * o + 2] = c2;
  depth_out[o] = d;
}

}  // namespace

int launch_unproject(const uint16_t* depth, int B, int H, int W, const float* intr, float* pts, hipStream_t s) {
  if (B <= 0 || H <= 0 || W <= 0 || B > 65535 || H > 65535 || !depth || !intr || !pts) return -22;
  if (((uintptr_t)pts & 15) || intr[0] == 0.0f || intr[1] == 0.0f) return -22;
  const Intr k{intr[0], intr[1], intr[2], intr[3]};
  unproject_kernel<<<dim3(cdiv(W, RT), H, B), RT, 0, s>>>(depth, H, W, k, reinterpret_cast<float4*>(pts));
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

int launch_render_view(const float* pts, const uint8_t* rgb, int B, int H, int W, const float* pose,
                       const float* intr, int Ho, int Wo, unsigned long long* zbuf, uint8_t* rgb_out,
                       uint16_t* depth_out, hipStream_t s) {
  if (B <= 0 || H <= 0 || W <= 0 || Ho <= 0 || Wo <= 0 || B > 65535 || H > 65535 || Ho > 65535) return -22;
  if ((long long)H * W > 0xffffffffLL || !pts || !rgb || !pose || !intr || !zbuf || !rgb_out || !depth_out) return -22;
  if (((uintptr_t)pts & 15) || ((uintptr_t)zbuf & 7) || ((uintptr_t)depth_out & 1)) return -22;
  Pose P;
  for (int i = 0; i < 3; ++i) {
    for (int j = 0; j < 3; ++j) P.r[3 * i + j] = pose[4 * i + j];
    P.t[i] = pose[4 * i + 3];
  }
  const Intr k{intr[0], intr[1], intr[2], intr[3]};
  const long long nz = (long long)B * Ho * Wo;
  if (cdivll(nz, RT) > 0x7fffffffLL) return -22;
  zbuf_clear_kernel<<<(unsigned)cdivll(nz, RT), RT, 0, s>>>(zbuf, nz);
  const float4* p4 = reinterpret_cast<const float4*>(pts);
  if ((long long)B * H * W <= SMALL_SPLAT)
    splat_kernel<1><<<dim3(cdiv(W, SW), cdiv(H, 4), B), RT, 0, s>>>(p4, H, W, P, k, Ho, Wo, zbuf);
  else
    splat_kernel<2><<<dim3(cdiv(W, SW), cdiv(H, 8), B), RT, 0, s>>>(p4, H, W, P, k, Ho, Wo, zbuf);
  resolve_kernel<<<dim3(cdiv(Wo, RT), Ho, B), RT, 0, s>>>(zbuf, rgb, H, W, Ho, Wo, rgb_out, depth_out);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

}  // namespace revo
