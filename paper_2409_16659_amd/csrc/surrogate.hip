// surrogate.hip -- C ABI of the learned surrogate (declared in
// include/mlf_surrogate.h): a convolutional neural operator that maps the
// layer heights h(t) of a periodic multilayer film to h(t + K).
//
// Network (all convolutions periodic):
//   x_i  = (h_i - mean(h_i)) / s                            (per sample, layer)
//   r_0  = E * patches_4x4(x) + b_E                         (latent grid ny/4 x nx/4, C channels)
//   r_{l+1} = r_l + W2_l (*) gelu(W1_l (*) r_l + b1_l) + b2_l,   l < L   (3x3 convs)
//   D    = pixel_shuffle(W_D r_L + b_D)                     (N x ny x nx)
//   Delta_i = D_i - mean(D_i)                               (no net mass change)
//   h'   = h + s Delta
// Training minimises mean((Delta - (h(t+K) - h(t)) / s)^2) with Adam.
// The 3x3 convolutions run on BF16 MFMA with FP32 accumulation
// (nop_kernels.hpp); everything else is FP32 on the VALU.  Master weights,
// gradients and Adam moments are FP32.
#include "../../include/mlf_surrogate.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "nop_kernels.hpp"

namespace {

constexpr int kPatch = 4;
constexpr int kRedBlocks = 512;  // partial sums of the pixel reductions
constexpr int kWgSlices = 85;    // slices of the weight gradient (3 x 85 workgroups: one per CU of 256)

// ---- elementwise and reduction kernels (FP32) ------------------------------

// Four consecutive values of a caller's image, which is aligned to its
// elements only: one 16-byte access all the same.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ inline float4 load4(const float* p) {
  const f32x4u v = *reinterpret_cast<const f32x4u*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}

// mean over the grid of each (sample, layer) plane: out[bi] (one block of
// 1024 threads each; 16-byte loads into four independent partial sums, then
// a tree in LDS; a fixed order, so the result is reproducible)
__global__ void __launch_bounds__(1024) plane_mean(const float* __restrict__ a, float* __restrict__ out, long long n) {
  __shared__ float red[1024];
  const float* p = a + (long long)blockIdx.x * n;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  long long done = 0;
  if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
    const long long n4 = n / 4;
    const float4* p4 = reinterpret_cast<const float4*>(p);
    long long t = threadIdx.x;
    for (; t + 7 * 1024 < n4; t += 8 * 1024) {  // eight loads in flight, added in order
      float4 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = p4[t + 1024 * q];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        s0 += v[q].x;
        s1 += v[q].y;
        s2 += v[q].z;
        s3 += v[q].w;
      }
    }
    for (; t < n4; t += 1024) {
      const float4 v = p4[t];
      s0 += v.x;
      s1 += v.y;
      s2 += v.z;
      s3 += v.w;
    }
    done = n4 * 4;
  }
  for (long long t = done + threadIdx.x; t < n; t += 1024) s0 += p[t];
  red[threadIdx.x] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  for (int w = 512; w >= 64; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x >= 64) return;
  float s = red[threadIdx.x];
  for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w, 64);  // the tree's last levels
  if (threadIdx.x == 0) out[blockIdx.x] = s / (float)n;
}

// prediction tail: o = h + s * (d - mean[plane]), the decoder output made
// mass-free and added to the input in one pass
__global__ void sub_mean_axpy(const float* __restrict__ h, const float* __restrict__ d,
                              const float* __restrict__ mean, float* __restrict__ o, float s, long long n_plane) {
  const long long base = (long long)blockIdx.y * n_plane;
  const float mu = mean[blockIdx.y];
  for (long long t = blockIdx.x * 256LL + threadIdx.x; t < n_plane; t += (long long)gridDim.x * 256) {
    const float dv = d[base + t] - mu;
    o[base + t] = h[base + t] + s * dv;
  }
}

// Wave-local LDS hand-off: the lanes of one wave write, then read what
// other lanes of the same wave wrote (no workgroup barrier is needed).
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// patch layer into the latent grid:
//   out[b][py][px][c] = bias[c] + sum_j W[j][c] P[b][i][4py+u][4px+v],  j = (i*4+u)*4+v
// and its BF16 copy: the patch encoder (P = (h - mean) / s, W = E, bias = b_E)
// and the decoder's input gradient (P = dD - mean, W = W_D, no bias, and with
// SUMS its column sums, colp[row of 64 pixels][C]).  A wave takes 64 latent
// pixels of one row (one per lane; coalesced patch loads) and 32 channels, so
// the weights are the same for all its lanes (scalar loads); the 64 x 32
// outputs are transposed through LDS so that each store writes whole 128-byte
// channel runs.  P = (img - pmean[plane]) * pscale is formed on the fly.
// Needs (batch gy gx) % 64 == 0.
template <bool SUMS>
__global__ void __launch_bounds__(256) patch_to_latent(const float* __restrict__ P, const float* __restrict__ W,
                                                       const float* __restrict__ bias, float* __restrict__ out,
                                                       __bf16* __restrict__ outb, float* __restrict__ colp, int nl,
                                                       int ny, int nx, int C, int batch,
                                                       const float* __restrict__ pmean, float pscale) {
  constexpr int RS = 33;  // LDS row stride of a pixel's 32 outputs (odd: no bank conflicts)
  __shared__ float so[4][64 * RS];
  const int gy = ny / kPatch, gx = nx / kPatch;
  const long long npix = (long long)batch * gy * gx;
  const int groups = C / 32;
  const long long waves = npix / 64 * groups;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* s = so[wave];
  for (long long wv = blockIdx.x * 4LL + wave; wv < waves; wv += gridDim.x * 4LL) {
    const int c0 = (int)(wv % groups) * 32;
    const long long pbase = (wv / groups) * 64;
    const long long pix = pbase + lane;
    const int px = (int)(pix % gx), py = (int)((pix / gx) % gy), b = (int)(pix / ((long long)gx * gy));
    float acc[32];
#pragma unroll
    for (int c = 0; c < 32; ++c) acc[c] = bias ? bias[c0 + c] : 0.f;
    for (int i = 0; i < nl; ++i)
      for (int u = 0; u < kPatch; ++u) {
        float4 pv = load4(P + (((long long)b * nl + i) * ny + kPatch * py + u) * nx + kPatch * px);
        const float mu = pmean[b * nl + i];
        pv = make_float4((pv.x - mu) * pscale, (pv.y - mu) * pscale, (pv.z - mu) * pscale, (pv.w - mu) * pscale);
        const float ps[4] = {pv.x, pv.y, pv.z, pv.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float* wr = W + (long long)((i * kPatch + u) * kPatch + v) * C + c0;
#pragma unroll
          for (int c = 0; c < 32; ++c) acc[c] += wr[c] * ps[v];
        }
      }
#pragma unroll
    for (int c = 0; c < 32; ++c) s[lane * RS + c] = acc[c];
    wave_sync();
    float cs = 0.f;
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int p = 2 * k + (lane >> 5), ch = lane & 31;
      const float v = s[p * RS + ch];
      out[(pbase + p) * C + c0 + ch] = v;
      outb[(pbase + p) * C + c0 + ch] = (__bf16)v;
      if constexpr (SUMS) cs += v;
    }
    if constexpr (SUMS) {
      cs += __shfl_xor(cs, 32, 64);
      if (lane < 32) colp[(wv / groups) * C + c0 + lane] = cs;
    }
    wave_sync();  // reads done before the next pass overwrites the rows
  }
}

// decoder + pixel shuffle: D[b][i][4py+u][4px+v] = bd[j] + sum_c Wd[j][c] r[b][py][px][c], j = (i*4+u)*4+v
// A wave takes 64 latent pixels of one row (one per lane) and the 16
// outputs j of one layer i, so the weights are the same for all its lanes
// (scalar loads) and a batch of B films gives B * (gy * gx / 64) * N waves.
// The pixels' channels are staged through LDS 32 at a time with coalesced
// loads (8 lanes per 128-byte run); the channel order of the sums is
// ascending, 4 per step.  Needs (batch gy gx) % 64 == 0.
__global__ void __launch_bounds__(256) dec_fwd(const float* __restrict__ r, const float* __restrict__ Wd,
                                               const float* __restrict__ bd, float* __restrict__ D, int nl, int ny,
                                               int nx, int C, int batch) {
  constexpr int CH = 32, RS = CH + 4;
  __shared__ float sr[4][64 * RS];
  const int gy = ny / kPatch, gx = nx / kPatch;
  const long long npix = (long long)batch * gy * gx;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long wv = (long long)blockIdx.x * 4 + wave;
  if (wv >= npix / 64 * nl) return;
  const int i = (int)(wv % nl);
  const long long pbase = (wv / nl) * 64;
  const long long pix = pbase + lane;
  const int px = (int)(pix % gx), py = (int)((pix / gx) % gy), b = (int)(pix / ((long long)gx * gy));
  const float* W = Wd + (long long)16 * i * C;
  float* s = sr[wave];
  float acc[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = bd[16 * i + j];
  for (int c0 = 0; c0 < C; c0 += CH) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int p = q * 8 + (lane >> 3), cq = lane & 7;
      *reinterpret_cast<float4*>(s + p * RS + 4 * cq) =
          *reinterpret_cast<const float4*>(r + (pbase + p) * C + c0 + 4 * cq);
    }
    wave_sync();
    float4 rv[CH / 4];
#pragma unroll
    for (int t = 0; t < CH / 4; ++t) rv[t] = *reinterpret_cast<const float4*>(s + lane * RS + 4 * t);
#pragma unroll
    for (int t = 0; t < CH / 4; ++t) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float* wp = W + (long long)j * C + c0 + 4 * t;
        acc[j] += wp[0] * rv[t].x + wp[1] * rv[t].y + wp[2] * rv[t].z + wp[3] * rv[t].w;
      }
    }
    wave_sync();  // reads done before the next chunk overwrites the rows
  }
#pragma unroll
  for (int u = 0; u < kPatch; ++u)
    *reinterpret_cast<float4*>(D + (((long long)b * nl + i) * ny + kPatch * py + u) * nx + kPatch * px) =
        make_float4(acc[4 * u], acc[4 * u + 1], acc[4 * u + 2], acc[4 * u + 3]);
}

// The two patch layers for small batches (small_batch): with the weights as scalar operands each wave waits for its scalar
// loads some thirty times, which nothing hides while the device is mostly
// idle (one film: encoder 14 us, decoder 21 us, whatever the split).  Here a
// workgroup first brings everything it needs into LDS or registers with all
// loads in flight at once, and the waves read weights as LDS broadcasts; the
// sums and their order are those of patch_to_latent and dec_fwd.
//
// Encoder side: a workgroup takes 64 pixels and 32 channels, 8 per wave.
template <bool SUMS, int NL>
__global__ void __launch_bounds__(256) patch_to_latent_small(const float* __restrict__ P, const float* __restrict__ W,
                                                             const float* __restrict__ bias, float* __restrict__ out,
                                                             __bf16* __restrict__ outb, float* __restrict__ colp,
                                                             int ny, int nx, int C, const float* __restrict__ pmean,
                                                             float pscale) {
  constexpr int J = 16 * NL, RS = 33;
  __shared__ __attribute__((aligned(16))) float sw[J * 32];
  __shared__ float so[64 * RS];
  const int gy = ny / kPatch, gx = nx / kPatch, groups = C / 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = (int)(blockIdx.x % groups) * 32;
  const long long run = blockIdx.x / groups, pix = run * 64 + lane;
  const int px = (int)(pix % gx), py = (int)((pix / gx) % gy), b = (int)(pix / ((long long)gx * gy));
  float4 pv[NL][kPatch];
#pragma unroll
  for (int i = 0; i < NL; ++i)
#pragma unroll
    for (int u = 0; u < kPatch; ++u)
      pv[i][u] = load4(P + (((long long)b * NL + i) * ny + kPatch * py + u) * nx + kPatch * px);
  for (int t = threadIdx.x; t < J * 8; t += 256)
    *reinterpret_cast<float4*>(sw + 4 * t) = *reinterpret_cast<const float4*>(W + (long long)(t / 8) * C + c0 + 4 * (t % 8));
  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = bias ? bias[c0 + 8 * wave + c] : 0.f;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const float mu = pmean[b * NL + i];
#pragma unroll
    for (int u = 0; u < kPatch; ++u) {
      const float ps[4] = {(pv[i][u].x - mu) * pscale, (pv[i][u].y - mu) * pscale, (pv[i][u].z - mu) * pscale,
                           (pv[i][u].w - mu) * pscale};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float* wr = sw + ((i * kPatch + u) * kPatch + v) * 32 + 8 * wave;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += wr[c] * ps[v];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) so[lane * RS + 8 * wave + c] = acc[c];
  __syncthreads();
  // stores as in patch_to_latent: each wave 16 of the pixels, whole 128-byte
  // channel runs
  const int ch = lane & 31;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int p = 16 * wave + 2 * k + (lane >> 5);
    const float v = so[p * RS + ch];
    out[(run * 64 + p) * C + c0 + ch] = v;
    outb[(run * 64 + p) * C + c0 + ch] = (__bf16)v;
  }
  if constexpr (SUMS) {
    if (threadIdx.x < 32) {
      float cs = 0.f;
#pragma unroll
      for (int p = 0; p < 64; ++p) cs += so[p * RS + threadIdx.x];
      colp[run * C + c0 + threadIdx.x] = cs;
    }
  }
}

// Decoder side: a workgroup takes 64 pixels and one layer, one output row u
// per wave.
template <int C>
__global__ void __launch_bounds__(256) dec_small(const float* __restrict__ r, const float* __restrict__ Wd,
                                                 const float* __restrict__ bd, float* __restrict__ D, int nl, int ny,
                                                 int nx) {
  constexpr int RS = C + 4;
  __shared__ __attribute__((aligned(16))) float sr[64 * RS];
  __shared__ __attribute__((aligned(16))) float sw[16 * C];
  const int gy = ny / kPatch, gx = nx / kPatch;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = (int)(blockIdx.x % nl);
  const long long pbase = (long long)(blockIdx.x / nl) * 64, pix = pbase + lane;
  const int px = (int)(pix % gx), py = (int)((pix / gx) % gy), b = (int)(pix / ((long long)gx * gy));
  const float* W = Wd + (long long)16 * i * C;
  constexpr int PQ = 64 * C / 4 / 256, WQ = 16 * C / 4 / 256;  // 16-byte pieces per thread
  float4 a[PQ], w[WQ];
#pragma unroll
  for (int q = 0; q < PQ; ++q) a[q] = *reinterpret_cast<const float4*>(r + pbase * C + 4 * (threadIdx.x + 256 * q));
#pragma unroll
  for (int q = 0; q < WQ; ++q) w[q] = *reinterpret_cast<const float4*>(W + 4 * (threadIdx.x + 256 * q));
#pragma unroll
  for (int q = 0; q < PQ; ++q) {
    const int e = 4 * (threadIdx.x + 256 * q);
    *reinterpret_cast<float4*>(sr + e / C * RS + e % C) = a[q];
  }
#pragma unroll
  for (int q = 0; q < WQ; ++q) *reinterpret_cast<float4*>(sw + 4 * (threadIdx.x + 256 * q)) = w[q];
  float acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = bd[16 * i + 4 * wave + j];
  __syncthreads();
#pragma unroll 8
  for (int c = 0; c < C; c += 4) {
    const float4 rv = *reinterpret_cast<const float4*>(sr + lane * RS + c);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 wp = *reinterpret_cast<const float4*>(sw + (4 * wave + j) * C + c);
      acc[j] += wp.x * rv.x + wp.y * rv.y + wp.z * rv.z + wp.w * rv.w;
    }
  }
  *reinterpret_cast<float4*>(D + (((long long)b * nl + i) * ny + kPatch * py + wave) * nx + kPatch * px) =
      make_float4(acc[0], acc[1], acc[2], acc[3]);
}

// Weight (and, for the decoder, bias) gradients of the patch layers:
//   part[blk][j][c] = sum_{pix of the block} P[pix][j] Q[pix][c],  and with
//   SUMS part[blk][16 NL C + j] = sum P[pix][j],
// P[pix][j] = (img - pmean[plane]) * pscale the 4x4 patch values of latent
// pixel pix (j = 16 i + 4 u + v) and Q a latent tensor.  A wavefront takes
// runs of 64 pixels of one latent row and accumulates all 16 NL x C products
// on the FP32 matrix cores (v_mfma_f32_16x16x4_f32: FP32 inputs and sums), four
// pixels per instruction, operands straight from global memory: lane l holds
// patch value l % 16 and channels (C / 16)(l % 16) .. of pixel l / 16, so that
// column r of channel tile n is channel (C / 16) r + n and every lane loads
// whole 16-byte pieces.  The block's four wavefronts are summed through LDS.
// Bound by the latent tensor's bytes: 134 MB at batch 64; with LDS-staged
// VALU products 116 us, now 50 us.
typedef float f32x4m __attribute__((ext_vector_type(4)));
template <int NL, int C, bool SUMS>
__global__ void __launch_bounds__(256, 2) patch_outer(const float* __restrict__ img, const float* __restrict__ pmean,
                                                      float pscale, const float* __restrict__ lat,
                                                      float* __restrict__ part, int ny, int nx, long long runs) {
  constexpr int NT = C / 16, JC = 16 * NL * C;
  __shared__ float red[NL * NT * 256 + 16 * NL];
  const int lane = threadIdx.x & 63, r = lane & 15, k = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gx = nx / kPatch, gy = ny / kPatch;
  f32x4m acc[NL][NT];
  float ps[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    ps[i] = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[i][n] = f32x4m{0.f, 0.f, 0.f, 0.f};
  }
  const int xr = gx / 64;
  for (long long run = blockIdx.x * 4LL + wave; run < runs; run += gridDim.x * 4LL) {
    const int px0 = (int)(run % xr) * 64, py = (int)((run / xr) % gy);
    const long long b = run / ((long long)xr * gy);
    const float* ip = img + (b * NL * ny + kPatch * py + (r >> 2)) * (long long)nx + kPatch * (px0 + k) + (r & 3);
    const float* lp = lat + (run * 64 + k) * C + NT * r;
    float mu[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) mu[i] = pmean[b * NL + i];
#pragma unroll 4
    for (int s = 0; s < 16; ++s) {  // pixels px0 + 4 s + k
      float a[NL], q[NT];
#pragma unroll
      for (int i = 0; i < NL; ++i) a[i] = (ip[(long long)i * ny * nx + 16 * s] - mu[i]) * pscale;
#pragma unroll
      for (int n = 0; n < NT; n += 4) {
        const float4 v = *reinterpret_cast<const float4*>(lp + (long long)4 * s * C + n);
        q[n] = v.x, q[n + 1] = v.y, q[n + 2] = v.z, q[n + 3] = v.w;
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        if constexpr (SUMS) ps[i] += a[i];
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], q[n], acc[i][n], 0, 0, 0);
      }
    }
  }
  if constexpr (SUMS) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      ps[i] += __shfl_xor(ps[i], 16, 64);
      ps[i] += __shfl_xor(ps[i], 32, 64);
    }
  }
  for (int w = 3; w >= 1; --w) {  // wavefronts 3, 2, 1 into wavefront 0, in this order
    if (wave == w) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int j = 0; j < 4; ++j) red[((i * NT + n) * 4 + j) * 64 + lane] = acc[i][n][j];
        if (SUMS && k == 0) red[NL * NT * 256 + 16 * i + r] = ps[i];
      }
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][n][j] += red[((i * NT + n) * 4 + j) * 64 + lane];
        if (SUMS) ps[i] += red[NL * NT * 256 + 16 * i + r];
      }
    }
    __syncthreads();
  }
  if (wave != 0) return;
  float* o = part + (long long)blockIdx.x * (JC + (SUMS ? 16 * NL : 0));
  // D: rows (patch values) 4 k + j, column r = channel NT r + n
#pragma unroll
  for (int i = 0; i < NL; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int n = 0; n < NT; n += 4)
        *reinterpret_cast<float4*>(o + (long long)(16 * i + 4 * k + j) * C + NT * r + n) =
            make_float4(acc[i][n][j], acc[i][n + 1][j], acc[i][n + 2][j], acc[i][n + 3][j]);
    if (SUMS && k == 0) o[JC + 16 * i + r] = ps[i];
  }
}

// out[k] = sum_r part[r][k] (fixed order: r ascending), for many columns.
// With few columns per thread in flight the latency of the loads bounds it,
// so 16 rows' are issued together, also in the last group (its absent rows
// repeat the last one's address and count as 0): 36864 columns of 85 rows 4.7
// us, 6.6 with eight and a last group row by row; 147456 columns 9.0 us (5.6
// TB/s), 9.6.
__global__ void sum_rows(const float* __restrict__ part, float* __restrict__ out, int rows, long long K) {
  for (long long k = blockIdx.x * 256LL + threadIdx.x; k < K; k += (long long)gridDim.x * 256) {
    float s = 0.f;
    int r = 0;
    for (; r + 16 <= rows; r += 16) {
      float v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = part[(long long)(r + q) * K + k];
#pragma unroll
      for (int q = 0; q < 16; ++q) s += v[q];
    }
    if (r < rows) {
      float v[15];
#pragma unroll
      for (int q = 0; q < 15; ++q) v[q] = part[(long long)min(r + q, rows - 1) * K + k];
#pragma unroll
      for (int q = 0; q < 15; ++q) s += r + q < rows ? v[q] : 0.f;
    }
    out[k] = s;
  }
}

// The same for few columns and many rows: a workgroup takes 8 columns, 128
// row groups of them (rows g, g + 128, ...) side by side and then a tree in
// LDS, so that the chain of dependent additions is rows / 128 long instead of
// rows (K = 128, 512 rows, one thread per column: 32 us; now 4 us).
constexpr int kFewCols = 8, kFewGroups = 128;
__global__ void __launch_bounds__(kFewCols* kFewGroups) sum_rows_few(const float* __restrict__ part,
                                                                     float* __restrict__ out, int rows, int K) {
  __shared__ float red[kFewGroups][kFewCols];
  const int c = threadIdx.x % kFewCols, g = threadIdx.x / kFewCols;
  const int k = blockIdx.x * kFewCols + c;
  float s = 0.f;
  if (k < K) {
    int r = g;
    for (; r + 3 * kFewGroups < rows; r += 4 * kFewGroups) {
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = part[(long long)(r + q * kFewGroups) * K + k];
#pragma unroll
      for (int q = 0; q < 4; ++q) s += v[q];
    }
    for (; r < rows; r += kFewGroups) s += part[(long long)r * K + k];
  }
  red[g][c] = s;
  __syncthreads();
  for (int w = kFewGroups / 2; w > 0; w >>= 1) {
    if (g < w) red[g][c] += red[g + w][c];
    __syncthreads();
  }
  if (g == 0 && k < K) out[k] = red[0][c];
}

// BF16 conv weights: w[o][co][ci] and the flipped transpose wt[o][ci][co] = w[8-o][co][ci]
__global__ void conv_weights(const float* __restrict__ w, __bf16* __restrict__ wb, __bf16* __restrict__ wt, int C) {
  const long long n = 9LL * C * C;
  for (long long t = blockIdx.x * 256LL + threadIdx.x; t < n; t += (long long)gridDim.x * 256) {
    const int o = (int)(t / ((long long)C * C));
    const int co = (int)((t / C) % C), ci = (int)(t % C);
    wb[t] = (__bf16)w[t];
    wt[((long long)(8 - o) * C + ci) * C + co] = (__bf16)w[t];
  }
}

// Loss and its gradient in one pass over the decoder output d, the plane means
// that make it mass-free, and the heights: e = (d - mean) - (h1 - h0) inv_s,
// grad = k e (where given), part[plane][block] = sum e^2, in FP64 (the pass is
// bound by its bytes).  Grid: (loss_blocks(n_plane), planes).
__global__ void __launch_bounds__(256) loss_grad(const float* __restrict__ d, const float* __restrict__ mean,
                                                 const float* __restrict__ h0, const float* __restrict__ h1,
                                                 float inv_s, float k, float* __restrict__ grad,
                                                 double* __restrict__ part, long long n_plane) {
  __shared__ double red[4];
  const long long base = (long long)blockIdx.y * n_plane;
  const float mu = mean[blockIdx.y];
  double s = 0.0;
  for (long long t = (blockIdx.x * 256LL + threadIdx.x) * 4; t < n_plane; t += (long long)gridDim.x * 1024) {
    const float4 dv = *reinterpret_cast<const float4*>(d + base + t);
    const float4 a = load4(h0 + base + t), b = load4(h1 + base + t);
    float4 g;
    auto one = [&](float dd, float x0, float x1) {
      const float free = dd - mu;
      const float tgt = (x1 - x0) * inv_s;
      const float e = free - tgt;
      s += e * e;
      return k * e;
    };
    g.x = one(dv.x, a.x, b.x);
    g.y = one(dv.y, a.y, b.y);
    g.z = one(dv.z, a.z, b.z);
    g.w = one(dv.w, a.w, b.w);
    if (grad) *reinterpret_cast<float4*>(grad + base + t) = g;
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// out = sum of n partials in FP64, fixed order (one workgroup)
__global__ void __launch_bounds__(256) loss_finish(const double* __restrict__ part, double* __restrict__ out, int n) {
  __shared__ double red[4];
  double s = 0.0;
  for (int t = threadIdx.x; t < n; t += 256) s += part[t];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ void adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                     long long n, float lr, float b1, float b2, float eps, float c1, float c2) {
  for (long long t = blockIdx.x * 256LL + threadIdx.x; t < n; t += (long long)gridDim.x * 256) {
    const float gg = g[t];
    const float mm = b1 * m[t] + (1.f - b1) * gg;
    const float vv = b2 * v[t] + (1.f - b2) * gg * gg;
    m[t] = mm;
    v[t] = vv;
    p[t] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  }
}

// Workgroups of loss_grad per plane: 4096 values each, 16 to 1024 of them.
int loss_blocks(long long n_plane) { return (int)std::max(16LL, std::min(n_plane / 4096, 1024LL)); }

unsigned grid1(long long n) { return (unsigned)std::max(1LL, std::min((n + 255) / 256, 16384LL)); }
// per-plane elementwise kernels: blockIdx.y = plane
dim3 plane_grid(long long n_plane, long long planes) {
  return dim3((unsigned)std::max(1LL, std::min((n_plane + 255) / 256, 1024LL)), (unsigned)planes);
}

}  // namespace

// ---- judge arithmetic ---------------------------------------------------------
// Errors of sample blockIdx.x of a against b (each [S][N][plane] FP32), in
// FP64 with a fixed summation order: out[2s] = |a - b| / |b| and
// out[2s+1] = |a - b| / |b - mean_i b| (L2 norms over all layers and
// nodes; mean_i b the per-layer mean, so the second is relative to the
// perturbation of the reference).  Two passes: per-layer sums of b, then
// the three squared norms.
constexpr int kErrThreads = 1024;
__global__ void __launch_bounds__(kErrThreads) sample_errors(const float* __restrict__ a, const float* __restrict__ b,
                                                             double* __restrict__ out, int nl, long long plane) {
  __shared__ double red[kErrThreads / 64][3];
  __shared__ double means[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = kErrThreads / 64;
  const long long base = (long long)blockIdx.x * nl * plane;
  for (int i = 0; i < nl; ++i) {
    double s = 0.0;
    for (long long e = threadIdx.x; e < plane; e += kErrThreads) s += (double)b[base + i * plane + e];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) red[wv][0] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int j = 0; j < nw; ++j) t += red[j][0];
      means[i] = t / (double)plane;
    }
    __syncthreads();
  }
  double d2 = 0.0, b2 = 0.0, p2 = 0.0;
  for (int i = 0; i < nl; ++i) {
    const double mu = means[i];
    for (long long e = threadIdx.x; e < plane; e += kErrThreads) {
      const double bv = b[base + i * plane + e], av = a[base + i * plane + e];
      d2 += (av - bv) * (av - bv);
      b2 += bv * bv;
      p2 += (bv - mu) * (bv - mu);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    d2 += __shfl_down(d2, off, 64);
    b2 += __shfl_down(b2, off, 64);
    p2 += __shfl_down(p2, off, 64);
  }
  if (lane == 0) red[wv][0] = d2, red[wv][1] = b2, red[wv][2] = p2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double sd = 0.0, sb = 0.0, sp = 0.0;
    for (int j = 0; j < nw; ++j) sd += red[j][0], sb += red[j][1], sp += red[j][2];
    out[2 * blockIdx.x] = sqrt(sd / sb);
    out[2 * blockIdx.x + 1] = sqrt(sd / sp);
  }
}

// Element conversion between the solver's FP64 heights and the network's FP32.
template <typename S, typename D>
__global__ void __launch_bounds__(256) convert(const S* __restrict__ src, D* __restrict__ dst, long long n) {
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
    dst[t] = (D)src[t];
}

// ============================================================= handle ====
struct mlf_nop {
  mlf_nop_params p;
  int C, L, J, gy, gx;
  long long npar;
  // parameter offsets (floats)
  long long oWe, obe, oW1, ob1, oW2, ob2, oWd, obd;  // oW1/ob1/oW2/ob2: block 0, stride per block
  long long blk_stride;
  unsigned char* ws;
  hipStream_t stream;
  // workspace regions
  float *par, *grad, *am, *av;
  __bf16 *w1b, *w1t, *w2b, *w2t;  // [L][9][C][C]
  float *D, *dD, *mean, *mean_h;  // mean: of D, then of dD; mean_h: of the input heights
  double *loss_part, *loss;
  float *r, *a, *dr;              // r: [L+1][lat], a: [L][lat], dr: [lat]
  __bf16 *rb, *gb, *cb, *cb2;     // rb: [L+1][lat], gb: [L][lat], cb, cb2: [lat]
  float *part;
  long long lat, img;            // floats per latent tensor / per image batch tensor (max batch)
  long long part_floats;
  int adam_t;
  std::string err;
};

namespace {

mlf_status nfail(mlf_nop* m, mlf_status st, const std::string& s) {
  if (m) m->err = s;
  return st;
}

mlf_status nhip(mlf_nop* m, hipError_t e, const char* what) {
  if (e == hipSuccess) return MLF_OK;
  return nfail(m, MLF_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define NHIP(call)                                                \
  do {                                                            \
    mlf_status _s = nhip(m, (call), #call);                       \
    if (_s != MLF_OK) return _s;                                  \
  } while (0)

#define NLAUNCH(...)                                              \
  do {                                                            \
    hipLaunchKernelGGL(__VA_ARGS__);                              \
    NHIP(hipGetLastError());                                      \
  } while (0)

mlf_status check_params(const mlf_nop_params* p) {
  if (!p) return MLF_EINVAL;
  if (p->n_layers < 1 || p->n_layers > 4) return MLF_EINVAL;
  if (p->nx < 64 * kPatch || p->nx % (64 * kPatch) || p->ny < 4 * kPatch || p->ny % (4 * kPatch)) return MLF_EINVAL;
  if (p->width != 64 && p->width != 128) return MLF_EUNSUPPORTED;
  // the convolutions index within one latent image in 32-bit arithmetic
  if ((long long)(p->ny / kPatch) * (p->nx / kPatch) * p->width >= (1LL << 31)) return MLF_EINVAL;
  if (p->blocks < 0 || p->blocks > 32 || p->batch < 1 || p->batch > 4096) return MLF_EINVAL;
  if (!(p->scale > 0.0) || !std::isfinite(p->scale)) return MLF_EINVAL;
  return MLF_OK;
}

struct Layout {
  long long npar, oWe, obe, oW1, ob1, oW2, ob2, blk, oWd, obd;
  long long lat, img, part_floats;
  size_t bytes;
  size_t off[32];
};

long long a64(long long v) { return (v + 63) / 64 * 64; }

Layout layout_of(const mlf_nop_params* p) {
  Layout s;
  const long long C = p->width, N = p->n_layers, J = N * kPatch * kPatch, L = p->blocks;
  s.oWe = 0;
  s.obe = s.oWe + C * J;
  s.oW1 = s.obe + C;
  s.ob1 = s.oW1 + 9 * C * C;
  s.oW2 = s.ob1 + C;
  s.ob2 = s.oW2 + 9 * C * C;
  s.blk = 2 * (9 * C * C + C);
  s.oWd = s.oW1 + L * s.blk;
  s.obd = s.oWd + J * C;
  s.npar = s.obd + J;
  const long long gy = p->ny / kPatch, gx = p->nx / kPatch;
  s.lat = (long long)p->batch * gy * gx * C;
  s.img = (long long)p->batch * N * p->ny * p->nx;
  s.part_floats = std::max<long long>({(long long)kWgSlices * 9 * C * C, (long long)kRedBlocks * (J * C + J),
                                       (long long)kRedBlocks * J, s.lat / 64});
  // regions: floats then bf16, 256-byte aligned
  const long long npa = a64(s.npar);
  std::vector<long long> sz = {
      npa * 4, npa * 4, npa * 4, npa * 4,                                   // par grad am av
      a64(L * 9 * C * C) * 2 * 4,                                           // w1b w1t w2b w2t (bf16 each)
      a64(s.img) * 4, a64(s.img) * 4,                                       // D dD
      a64(p->batch * N) * 4, a64(p->batch * N) * 4,                         // mean mean_h
      a64(p->batch * N * loss_blocks((long long)p->ny * p->nx)) * 8, 256,   // loss_part loss
      a64((L + 1) * s.lat) * 4, a64(std::max(1LL, L) * s.lat) * 4,          // r a
      a64(s.lat) * 4,                                                       // dr
      a64((L + 1) * s.lat) * 2, a64(std::max(1LL, L) * s.lat) * 2,          // rb gb
      a64(s.lat) * 2, a64(s.lat) * 2,                                       // cb cb2
      a64(s.part_floats) * 4};
  size_t o = 0;
  for (size_t i = 0; i < sz.size(); ++i) {
    s.off[i] = o;
    o += (size_t)((sz[i] + 255) / 256 * 256);
  }
  s.bytes = o;
  return s;
}

// Launch shape by workload (measured on 64 x 64 latent grids, u = batch rows x
// 64-pixel column tiles): workgroups of 4 waves (4 latent rows), two per CU.
// Large batches (training) give each workgroup all channels, so that each
// staged slab of weights serves more products; small ones (the judged runs'
// windows) split the output channels into groups of 32 to fill the device,
// medium ones at C = 128 into groups of 64 (a prediction of 16 films 290
// us with groups of 64, 317 with 32; of 12 films 245 / 235; of 48 films 788 /
// 930; at C = 64 of 32 films 250 with all channels, 259 with 32).
// Every shape gives the same bits.  The dynamic LDS above 64 KiB of every
// shape is enabled when the handle is created (set_lds_limits, on the
// handle's device).
template <int C, int CO, int EPI>
mlf_status conv_fwd_launch(mlf_nop* m, long long rows, const __bf16* in, const __bf16* w, const float* bias,
                           float* out, const float* res, __bf16* outb, float* colp) {
  const size_t lds = nop::conv3x3_fwd_lds(CO, 4);
  const unsigned xt = (unsigned)(m->gx / 64);
  NLAUNCH((nop::conv3x3_fwd<C, CO, 4, EPI>), dim3((unsigned)(rows / 4) * xt, C / CO), dim3(256), lds, m->stream,
          in, w, bias, out, res, outb, colp, m->gy, m->gx);
  return MLF_OK;
}

template <int C, int EPI>
mlf_status conv_fwd_t(mlf_nop* m, int batch, const __bf16* in, const __bf16* w, const float* bias, float* out,
                      const float* res, __bf16* outb, float* colp) {
  const long long rows = (long long)batch * m->gy, u = rows * (m->gx / 64);
  if (u >= (C == 64 ? 2048 : 4096)) return conv_fwd_launch<C, C, EPI>(m, rows, in, w, bias, out, res, outb, colp);
  if (C == 128 && u >= 1024) return conv_fwd_launch<C, 64, EPI>(m, rows, in, w, bias, out, res, outb, colp);
  return conv_fwd_launch<C, 32, EPI>(m, rows, in, w, bias, out, res, outb, colp);
}

template <int EPI>
mlf_status conv_fwd_e(mlf_nop* m, int batch, const __bf16* in, const __bf16* w, const float* bias, float* out,
                      const float* res, __bf16* outb, float* colp = nullptr) {
  return m->C == 64 ? conv_fwd_t<64, EPI>(m, batch, in, w, bias, out, res, outb, colp)
                    : conv_fwd_t<128, EPI>(m, batch, in, w, bias, out, res, outb, colp);
}

mlf_status conv_fwd(mlf_nop* m, int batch, const __bf16* in, const __bf16* w, const float* bias, float* out) {
  return conv_fwd_e<nop::kEpiPlain>(m, batch, in, w, bias, out, nullptr, nullptr);
}

// weight gradients of nslice slices of the batch's pixels into m->part
// ([nslice][9][C][C]); a workgroup per (slice, row offset) with all channel
// pairs: 16 waves at C = 128 (32 x 32 channel tiles: 4 waves per SIMD hide
// more of the staging and LDS latency than 8 waves with 64 x 32 tiles),
// 4 at C = 64 (32 x 32).  kWgSlices slices (3 kWgSlices workgroups, one per
// CU of a 256-CU device), fewer when the batch has fewer chunks; the grid
// is padded to a multiple of 8 for the kernel's XCD grouping.
template <int C>
constexpr int kWgW = C == 128 ? 4 : 2;  // waves along each of co and ci

int wgrad_slices(const mlf_nop* m, int batch) {
  const long long chunks = (long long)batch * m->gy * (m->gx / nop::kWgChunk);
  return (int)std::max<long long>(1, std::min<long long>(chunks, kWgSlices));
}

template <int C>
mlf_status wgrad_launch(mlf_nop* m, int batch, const __bf16* in, const __bf16* dout) {
  const int ns = wgrad_slices(m, batch);
  const unsigned grid = (unsigned)((3 * ns + 7) / 8 * 8);
  NLAUNCH((nop::conv3x3_wgrad<C, kWgW<C>, kWgW<C>>), dim3(grid), dim3(64 * kWgW<C> * kWgW<C>),
          nop::conv3x3_wgrad_lds(C), m->stream, in, dout, m->part, batch, m->gy, m->gx, ns);
  return MLF_OK;
}

// Dynamic LDS limits of every convolution shape the launchers above can
// pick for width C (hipFuncSetAttribute applies on the current device).
template <typename K>
mlf_status set_lds(mlf_nop* m, K kern, size_t bytes) {
  NHIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                           (int)bytes));
  return MLF_OK;
}

template <int C, int EPI>
mlf_status set_fwd_lds(mlf_nop* m) {
  mlf_status st = set_lds(m, nop::conv3x3_fwd<C, 32, 4, EPI>, nop::conv3x3_fwd_lds(32, 4));
  if (st == MLF_OK) st = set_lds(m, nop::conv3x3_fwd<C, 64, 4, EPI>, nop::conv3x3_fwd_lds(64, 4));
  if (st == MLF_OK) st = set_lds(m, nop::conv3x3_fwd<C, C, 4, EPI>, nop::conv3x3_fwd_lds(C, 4));
  return st;
}

template <int C>
mlf_status set_lds_limits_c(mlf_nop* m) {
  mlf_status st = set_fwd_lds<C, nop::kEpiPlain>(m);
  if (st == MLF_OK) st = set_fwd_lds<C, nop::kEpiGelu>(m);
  if (st == MLF_OK) st = set_fwd_lds<C, nop::kEpiResid>(m);
  if (st == MLF_OK) st = set_fwd_lds<C, nop::kEpiGeluB>(m);
  if (st == MLF_OK) st = set_fwd_lds<C, nop::kEpiGrad>(m);
  if (st == MLF_OK) st = set_fwd_lds<C, nop::kEpiAcc>(m);
  if (st == MLF_OK) st = set_lds(m, nop::conv3x3_wgrad<C, kWgW<C>, kWgW<C>>, nop::conv3x3_wgrad_lds(C));
  return st;
}

mlf_status set_lds_limits(mlf_nop* m) { return m->C == 64 ? set_lds_limits_c<64>(m) : set_lds_limits_c<128>(m); }

// dW (FP32, [9][C][C]) = sum over the batch of the weight gradient
mlf_status conv_wgrad(mlf_nop* m, int batch, const __bf16* in, const __bf16* dout, float* dw) {
  const mlf_status st = m->C == 64 ? wgrad_launch<64>(m, batch, in, dout) : wgrad_launch<128>(m, batch, in, dout);
  if (st != MLF_OK) return st;
  const long long K = 9LL * m->C * m->C;
  NLAUNCH(sum_rows, dim3(grid1(K)), dim3(256), 0, m->stream, m->part, dw, wgrad_slices(m, batch), K);
  return MLF_OK;
}

// out[0..K) = sum of the `rows` rows of m->part (few columns)
mlf_status reduce_part(mlf_nop* m, long long rows, int K, float* out) {
  NLAUNCH(sum_rows_few, dim3((unsigned)((K + kFewCols - 1) / kFewCols)), dim3(kFewCols * kFewGroups), 0, m->stream,
          m->part, out, (int)rows, K);
  return MLF_OK;
}

// Weight gradient of a patch layer (with SUMS also its bias gradient, which
// follows the weights in the parameter vector) into dw.
template <int NL, bool SUMS>
mlf_status patch_grad_nl(mlf_nop* m, int batch, const float* img, const float* mean, float scale, const float* lat,
                         float* dw) {
  const long long runs = (long long)batch * m->gy * (m->gx / 64);
  const unsigned blocks = (unsigned)std::min<long long>(kRedBlocks, (runs + 3) / 4);
  if (m->C == 64)
    NLAUNCH((patch_outer<NL, 64, SUMS>), dim3(blocks), dim3(256), 0, m->stream, img, mean, scale, lat, m->part,
            m->p.ny, m->p.nx, runs);
  else
    NLAUNCH((patch_outer<NL, 128, SUMS>), dim3(blocks), dim3(256), 0, m->stream, img, mean, scale, lat, m->part,
            m->p.ny, m->p.nx, runs);
  return reduce_part(m, blocks, m->J * m->C + (SUMS ? m->J : 0), dw);
}
template <bool SUMS>
mlf_status patch_grad(mlf_nop* m, int batch, const float* img, const float* mean, float scale, const float* lat,
                      float* dw) {
  switch (m->p.n_layers) {
    case 1: return patch_grad_nl<1, SUMS>(m, batch, img, mean, scale, lat, dw);
    case 2: return patch_grad_nl<2, SUMS>(m, batch, img, mean, scale, lat, dw);
    case 3: return patch_grad_nl<3, SUMS>(m, batch, img, mean, scale, lat, dw);
    default: return patch_grad_nl<4, SUMS>(m, batch, img, mean, scale, lat, dw);
  }
}

mlf_status refresh_weights(mlf_nop* m) {
  const long long cc = 9LL * m->C * m->C;
  for (int l = 0; l < m->L; ++l) {
    NLAUNCH(conv_weights, dim3(grid1(cc)), dim3(256), 0, m->stream, m->par + m->oW1 + l * m->blk_stride,
            m->w1b + l * cc, m->w1t + l * cc, m->C);
    NLAUNCH(conv_weights, dim3(grid1(cc)), dim3(256), 0, m->stream, m->par + m->oW2 + l * m->blk_stride,
            m->w2b + l * cc, m->w2t + l * cc, m->C);
  }
  return MLF_OK;
}

// Whether `runs` runs of 64 latent pixels take the patch kernels for small
// batches.  A prediction at C = 128 of 1 / 4 / 12 films takes 94 / 114 / 206 us
// with them, 117 / 128 / 199 with the others; at C = 64 of 8 / 16 films 90 /
// 123 against 98 / 122.
bool small_batch(const mlf_nop* m, long long runs) { return runs * m->C <= 65536; }

// A patch layer into the latent grid (with SUMS its column sums into m->part).
template <bool SUMS>
mlf_status to_latent(mlf_nop* m, int batch, const float* P, const float* W, const float* bias, float* out,
                     __bf16* outb, const float* mean, float scale) {
  const int N = m->p.n_layers;
  const long long runs = (long long)batch * m->gy * m->gx / 64;
  if (!small_batch(m, runs)) {
    NLAUNCH((patch_to_latent<SUMS>), dim3(grid1(runs * 2 * m->C)), dim3(256), 0, m->stream, P, W, bias, out, outb,
            m->part, N, m->p.ny, m->p.nx, m->C, batch, mean, scale);
    return MLF_OK;
  }
  const dim3 grid((unsigned)(runs * (m->C / 32)));
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, m->stream, P, W, bias, out, outb, m->part, m->p.ny, m->p.nx, m->C,
                       mean, scale);
  };
  switch (N) {
    case 1: launch(patch_to_latent_small<SUMS, 1>); break;
    case 2: launch(patch_to_latent_small<SUMS, 2>); break;
    case 3: launch(patch_to_latent_small<SUMS, 3>); break;
    default: launch(patch_to_latent_small<SUMS, 4>); break;
  }
  NHIP(hipGetLastError());
  return MLF_OK;
}

// Forward pass to the decoder output m->D and its plane means m->mean (the
// increment is their difference, formed by the prediction's tail or by the
// loss).  `train` keeps the pre-activations for the backward pass.
mlf_status forward(mlf_nop* m, int batch, const float* h, bool train) {
  const int N = m->p.n_layers;
  const long long plane = (long long)m->p.ny * m->p.nx;
  const long long npix = (long long)batch * m->gy * m->gx;
  NLAUNCH(plane_mean, dim3(batch * N), dim3(1024), 0, m->stream, h, m->mean_h, plane);
  mlf_status st = to_latent<false>(m, batch, h, m->par + m->oWe, m->par + m->obe, m->r, m->rb, m->mean_h,
                                   (float)(1.0 / m->p.scale));
  if (st != MLF_OK) return st;
  const long long cc = 9LL * m->C * m->C;
  for (int l = 0; l < m->L; ++l) {
    float* rl = m->r + l * m->lat;
    __bf16* rlb = m->rb + l * m->lat;
    float* al = m->a + l * m->lat;
    __bf16* glb = m->gb + l * m->lat;
    // a = W1 * r + b1 and its GELU in BF16; r_{l+1} = r + W2 * gelu(a) + b2
    // and its BF16 copy, both in the convolutions' epilogues
    const float* b1 = m->par + m->ob1 + l * m->blk_stride;
    st = train ? conv_fwd_e<nop::kEpiGelu>(m, batch, rlb, m->w1b + l * cc, b1, al, nullptr, glb)
               : conv_fwd_e<nop::kEpiGeluB>(m, batch, rlb, m->w1b + l * cc, b1, nullptr, nullptr, glb);
    if (st != MLF_OK) return st;
    st = conv_fwd_e<nop::kEpiResid>(m, batch, glb, m->w2b + l * cc, m->par + m->ob2 + l * m->blk_stride,
                                    m->r + (l + 1) * m->lat, rl, m->rb + (l + 1) * m->lat);
    if (st != MLF_OK) return st;
  }
  const float* rL = m->r + m->L * m->lat;
  const unsigned runs = (unsigned)(npix / 64);
  if (!small_batch(m, runs))
    NLAUNCH(dec_fwd, dim3((runs * N + 3) / 4), dim3(256), 0, m->stream, rL, m->par + m->oWd, m->par + m->obd, m->D, N,
            m->p.ny, m->p.nx, m->C, batch);
  else if (m->C == 64)
    NLAUNCH(dec_small<64>, dim3(runs * N), dim3(256), 0, m->stream, rL, m->par + m->oWd, m->par + m->obd, m->D, N,
            m->p.ny, m->p.nx);
  else
    NLAUNCH(dec_small<128>, dim3(runs * N), dim3(256), 0, m->stream, rL, m->par + m->oWd, m->par + m->obd, m->D, N,
            m->p.ny, m->p.nx);
  NLAUNCH(plane_mean, dim3(batch * N), dim3(1024), 0, m->stream, m->D, m->mean, plane);
  return MLF_OK;
}

// Loss of the current increment against the target into m->loss (times the
// number of values), with want_grad its gradient into m->dD.
mlf_status loss_and_grad(mlf_nop* m, int batch, const float* h0, const float* h1, bool want_grad) {
  const int planes = batch * m->p.n_layers;
  const long long plane = (long long)m->p.ny * m->p.nx, img = planes * plane;
  NLAUNCH(loss_grad, dim3(loss_blocks(plane), planes), dim3(256), 0, m->stream, m->D, m->mean, h0, h1,
          (float)(1.0 / m->p.scale), 2.f / (float)img, want_grad ? m->dD : nullptr, m->loss_part, plane);
  NLAUNCH(loss_finish, dim3(1), dim3(256), 0, m->stream, m->loss_part, m->loss, planes * loss_blocks(plane));
  return MLF_OK;
}

// Loss of loss_and_grad on the host (synchronises).
mlf_status read_loss(mlf_nop* m, int batch, double* loss) {
  double sum = 0.0;
  NHIP(hipMemcpyAsync(&sum, m->loss, sizeof sum, hipMemcpyDeviceToHost, m->stream));
  NHIP(hipStreamSynchronize(m->stream));
  *loss = sum / ((double)batch * m->p.n_layers * m->p.ny * m->p.nx);
  return MLF_OK;
}

// gradient of the loss w.r.t. all parameters into m->grad (after forward
// from the heights h and loss_and_grad with the gradient)
mlf_status backward(mlf_nop* m, int batch, const float* h) {
  const int N = m->p.n_layers;
  const long long plane = (long long)m->p.ny * m->p.nx;
  const long long rows = (long long)batch * m->gy * m->gx / 64;
  const long long cc = 9LL * m->C * m->C;
  mlf_status st;
  // the projection (no net mass change) is symmetric: the gradient is
  // projected where it is read, from its plane means
  NLAUNCH(plane_mean, dim3(batch * N), dim3(1024), 0, m->stream, m->dD, m->mean, plane);
  // decoder: weights and bias, input gradient
  if ((st = patch_grad<true>(m, batch, m->dD, m->mean, 1.f, m->r + m->L * m->lat, m->grad + m->oWd)) != MLF_OK)
    return st;
  if ((st = to_latent<true>(m, batch, m->dD, m->par + m->oWd, nullptr, m->dr, m->cb, m->mean, 1.f)) != MLF_OK)
    return st;
  // residual blocks, last to first; m->dr (and its BF16 copy m->cb) hold
  // dL/dr_{l+1}, m->part its column sums
  for (int l = m->L - 1; l >= 0; --l) {
    const long long ob = l * m->blk_stride;
    if ((st = reduce_part(m, rows, m->C, m->grad + m->ob2 + ob)) != MLF_OK) return st;
    if ((st = conv_wgrad(m, batch, m->gb + l * m->lat, m->cb, m->grad + m->oW2 + ob)) != MLF_OK) return st;
    if ((st = conv_fwd_e<nop::kEpiGrad>(m, batch, m->cb, m->w2t + l * cc, nullptr, nullptr, m->a + l * m->lat, m->cb2,
                                        m->part)) != MLF_OK)
      return st;
    if ((st = reduce_part(m, rows, m->C, m->grad + m->ob1 + ob)) != MLF_OK) return st;
    if ((st = conv_wgrad(m, batch, m->rb + l * m->lat, m->cb2, m->grad + m->oW1 + ob)) != MLF_OK) return st;
    if ((st = conv_fwd_e<nop::kEpiAcc>(m, batch, m->cb2, m->w1t + l * cc, nullptr, m->dr, m->dr,
                                       l > 0 ? m->cb : nullptr, m->part)) != MLF_OK)
      return st;
  }
  // encoder
  if ((st = reduce_part(m, rows, m->C, m->grad + m->obe)) != MLF_OK) return st;
  return patch_grad<false>(m, batch, h, m->mean_h, (float)(1.0 / m->p.scale), m->dr, m->grad + m->oWe);
}

mlf_status check_batch(mlf_nop* m, int batch) {
  if (batch < 1 || batch > m->p.batch) return nfail(m, MLF_EINVAL, "batch must be 1..the batch it was created for");
  return MLF_OK;
}

}  // namespace

extern "C" {

mlf_status mlf_nop_query_sizes(const mlf_nop_params* p, size_t* param_count, size_t* workspace_bytes) {
  mlf_status st = check_params(p);
  if (st != MLF_OK) return st;
  const Layout s = layout_of(p);
  if (param_count) *param_count = (size_t)s.npar;
  if (workspace_bytes) *workspace_bytes = s.bytes;
  return MLF_OK;
}

mlf_status mlf_nop_create(const mlf_nop_params* p, void* workspace, void* stream, mlf_nop** out) {
  if (!out) return MLF_EINVAL;
  *out = nullptr;
  mlf_status st = check_params(p);
  if (st != MLF_OK) return st;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return MLF_EINVAL;
  mlf_nop* m = new (std::nothrow) mlf_nop();
  if (!m) return MLF_EINVAL;
  const Layout s = layout_of(p);
  m->p = *p;
  m->C = p->width;
  m->L = p->blocks;
  m->J = p->n_layers * kPatch * kPatch;
  m->gy = p->ny / kPatch;
  m->gx = p->nx / kPatch;
  m->npar = s.npar;
  m->oWe = s.oWe, m->obe = s.obe, m->oW1 = s.oW1, m->ob1 = s.ob1, m->oW2 = s.oW2, m->ob2 = s.ob2;
  m->blk_stride = s.blk, m->oWd = s.oWd, m->obd = s.obd;
  m->lat = s.lat, m->img = s.img, m->part_floats = s.part_floats;
  m->ws = static_cast<unsigned char*>(workspace);
  m->stream = static_cast<hipStream_t>(stream);
  unsigned char* w = m->ws;
  const long long cc = 9LL * m->C * m->C * m->L;
  m->par = reinterpret_cast<float*>(w + s.off[0]);
  m->grad = reinterpret_cast<float*>(w + s.off[1]);
  m->am = reinterpret_cast<float*>(w + s.off[2]);
  m->av = reinterpret_cast<float*>(w + s.off[3]);
  __bf16* wb = reinterpret_cast<__bf16*>(w + s.off[4]);
  m->w1b = wb;
  m->w1t = wb + cc;
  m->w2b = wb + 2 * cc;
  m->w2t = wb + 3 * cc;
  m->D = reinterpret_cast<float*>(w + s.off[5]);
  m->dD = reinterpret_cast<float*>(w + s.off[6]);
  m->mean = reinterpret_cast<float*>(w + s.off[7]);
  m->mean_h = reinterpret_cast<float*>(w + s.off[8]);
  m->loss_part = reinterpret_cast<double*>(w + s.off[9]);
  m->loss = reinterpret_cast<double*>(w + s.off[10]);
  m->r = reinterpret_cast<float*>(w + s.off[11]);
  m->a = reinterpret_cast<float*>(w + s.off[12]);
  m->dr = reinterpret_cast<float*>(w + s.off[13]);
  m->rb = reinterpret_cast<__bf16*>(w + s.off[14]);
  m->gb = reinterpret_cast<__bf16*>(w + s.off[15]);
  m->cb = reinterpret_cast<__bf16*>(w + s.off[16]);
  m->cb2 = reinterpret_cast<__bf16*>(w + s.off[17]);
  m->part = reinterpret_cast<float*>(w + s.off[18]);
  m->adam_t = 0;
  if ((st = set_lds_limits(m)) != MLF_OK) {
    delete m;
    return st;
  }
  *out = m;
  return MLF_OK;
}

mlf_status mlf_nop_set_params(mlf_nop* m, const float* host) {
  if (!m || !host) return MLF_EINVAL;
  const size_t bytes = (size_t)m->npar * sizeof(float);
  NHIP(hipMemcpyAsync(m->par, host, bytes, hipMemcpyHostToDevice, m->stream));
  NHIP(hipMemsetAsync(m->am, 0, bytes, m->stream));
  NHIP(hipMemsetAsync(m->av, 0, bytes, m->stream));
  mlf_status st = refresh_weights(m);
  if (st != MLF_OK) return st;
  NHIP(hipStreamSynchronize(m->stream));
  m->adam_t = 0;
  return MLF_OK;
}

mlf_status mlf_nop_get_params(mlf_nop* m, float* host) {
  if (!m || !host) return MLF_EINVAL;
  NHIP(hipMemcpyAsync(host, m->par, (size_t)m->npar * sizeof(float), hipMemcpyDeviceToHost, m->stream));
  NHIP(hipStreamSynchronize(m->stream));
  return MLF_OK;
}

mlf_status mlf_nop_predict(mlf_nop* m, int32_t batch, const float* h, float* out) {
  if (!m || !h || !out) return MLF_EINVAL;
  mlf_status st = check_batch(m, batch);
  if (st != MLF_OK) return st;
  if ((st = forward(m, batch, h, false)) != MLF_OK) return st;
  const long long plane = (long long)m->p.ny * m->p.nx;
  NLAUNCH(sub_mean_axpy, plane_grid(plane, (long long)batch * m->p.n_layers), dim3(256), 0, m->stream, h, m->D,
          m->mean, out, (float)m->p.scale, plane);
  return MLF_OK;
}

mlf_status mlf_nop_loss(mlf_nop* m, int32_t batch, const float* h0, const float* h1, double* loss) {
  if (!m || !h0 || !h1 || !loss) return MLF_EINVAL;
  mlf_status st = check_batch(m, batch);
  if (st != MLF_OK) return st;
  if ((st = forward(m, batch, h0, false)) != MLF_OK) return st;
  if ((st = loss_and_grad(m, batch, h0, h1, false)) != MLF_OK) return st;
  return read_loss(m, batch, loss);
}

mlf_status mlf_nop_gradient(mlf_nop* m, int32_t batch, const float* h0, const float* h1, float* host_grad,
                            double* loss) {
  if (!m || !h0 || !h1 || !loss) return MLF_EINVAL;
  mlf_status st = check_batch(m, batch);
  if (st != MLF_OK) return st;
  if ((st = forward(m, batch, h0, true)) != MLF_OK) return st;
  if ((st = loss_and_grad(m, batch, h0, h1, true)) != MLF_OK) return st;
  if ((st = backward(m, batch, h0)) != MLF_OK) return st;
  if ((st = read_loss(m, batch, loss)) != MLF_OK) return st;  // after everything is enqueued
  if (host_grad) {
    NHIP(hipMemcpyAsync(host_grad, m->grad, (size_t)m->npar * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    NHIP(hipStreamSynchronize(m->stream));
  }
  return MLF_OK;
}

mlf_status mlf_nop_train_step(mlf_nop* m, int32_t batch, const float* h0, const float* h1, float lr, double* loss) {
  if (!(lr > 0.f)) return nfail(m, MLF_EINVAL, "learning rate must be > 0");
  mlf_status st = mlf_nop_gradient(m, batch, h0, h1, nullptr, loss);
  if (st != MLF_OK) return st;
  m->adam_t += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, (float)m->adam_t), c2 = 1.f - std::pow(b2, (float)m->adam_t);
  NLAUNCH(adam, dim3(grid1(m->npar)), dim3(256), 0, m->stream, m->par, m->grad, m->am, m->av, m->npar, lr, b1, b2,
          1e-8f, c1, c2);
  return refresh_weights(m);
}

mlf_status mlf_nop_time_conv(mlf_nop* m, int32_t batch, int32_t reps, float* ms) {
  if (!m || reps < 1 || !ms) return MLF_EINVAL;
  mlf_status st = check_batch(m, batch);
  if (st != MLF_OK) return st;
  if (m->L < 1) return nfail(m, MLF_EINVAL, "no convolution layers");
  hipEvent_t ev[5];
  for (int i = 0; i < 5; ++i) NHIP(hipEventCreate(&ev[i]));
  // operands: the first block's input and weights as they stand; outputs
  // into the first block's activations (residual: r_1 from r_0)
  const float* bias = m->par + m->ob1;
  __bf16* r1b = m->rb + m->lat;
  float* r1 = m->r + m->lat;
  st = conv_fwd(m, batch, m->rb, m->w1b, bias, m->a);
  for (int k = 0; k < 4 && st == MLF_OK; ++k) {
    st = nhip(m, hipEventRecord(ev[k], m->stream), "hipEventRecord");
    for (int i = 0; i < reps && st == MLF_OK; ++i) {
      if (k == 0) st = conv_fwd(m, batch, m->rb, m->w1b, bias, m->a);
      else if (k == 1) st = conv_fwd_e<nop::kEpiGelu>(m, batch, m->rb, m->w1b, bias, m->a, nullptr, m->gb);
      else if (k == 2) st = conv_fwd_e<nop::kEpiResid>(m, batch, m->gb, m->w2b, bias, r1, m->r, r1b);
      else st = m->C == 64 ? wgrad_launch<64>(m, batch, m->rb, m->gb) : wgrad_launch<128>(m, batch, m->rb, m->gb);
    }
  }
  if (st == MLF_OK) st = nhip(m, hipEventRecord(ev[4], m->stream), "hipEventRecord");
  if (st == MLF_OK) st = nhip(m, hipEventSynchronize(ev[4]), "hipEventSynchronize");
  for (int k = 0; k < 4 && st == MLF_OK; ++k) {
    float t = 0.f;
    st = nhip(m, hipEventElapsedTime(&t, ev[k], ev[k + 1]), "hipEventElapsedTime");
    ms[k] = t / reps;
  }
  for (int i = 0; i < 5; ++i) (void)hipEventDestroy(ev[i]);
  return st;
}

mlf_status mlf_nop_errors(mlf_nop* m, int32_t n, const float* a, const float* b, double* out) {
  if (!m || !a || !b || !out || n < 1) return MLF_EINVAL;
  const long long plane = (long long)m->p.ny * m->p.nx;
  NLAUNCH(sample_errors, dim3((unsigned)n), dim3(kErrThreads), 0, m->stream, a, b, out, m->p.n_layers, plane);
  return MLF_OK;
}

mlf_status mlf_convert_heights(const void* src, int32_t to_f32, void* dst, int64_t n, void* stream) {
  if (!src || !dst || n < 1) return MLF_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (to_f32)
    hipLaunchKernelGGL((convert<double, float>), dim3(grid1(n)), dim3(256), 0, s, static_cast<const double*>(src),
                       static_cast<float*>(dst), (long long)n);
  else
    hipLaunchKernelGGL((convert<float, double>), dim3(grid1(n)), dim3(256), 0, s, static_cast<const float*>(src),
                       static_cast<double*>(dst), (long long)n);
  return hipGetLastError() == hipSuccess ? MLF_OK : MLF_EDEVICE;
}

int32_t mlf_nop_steps_done(const mlf_nop* m) { return m ? m->adam_t : -1; }

const char* mlf_nop_last_error(const mlf_nop* m) { return m ? m->err.c_str() : "null surrogate"; }

mlf_status mlf_nop_destroy(mlf_nop* m) {
  if (!m) return MLF_EINVAL;
  delete m;
  return MLF_OK;
}

}  // extern "C"
