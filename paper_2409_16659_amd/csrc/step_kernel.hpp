// step_kernel.hpp -- fused N-layer thin-film lattice Boltzmann step for
// gfx950 (one or two time steps per launch).
//
// What one step computes (Sec. III with the pressure and friction of Sec. II
// of Richter, Malgaretti & Harting, arXiv 2409.16659), per node and layer:
//   moments   h_i = sum_k f_ki, q_i = sum_k c_k f_ki
//   z_i = z_{i-1} + h_i; grad z_i, lap z_i (isotropic 9-point stencils)
//   phi_lk = S_lk phi_k(z_{l+k} - z_l), phi'_lk  (Eq. wetting_potential)
//   Delta_i = -(gamma_i + sum_k phi_ik) lap z_i
//             - sum_k phi'_ik (1 + |grad z_i|^2/2)
//             + sum_{l<i} phi'_{l,i-l} (1 + |grad z_l|^2/2)
//             (Eqs. Laplace_pressure, disjoining_pressure)
//   p_i = sum_{j>=i} Delta_j; F_i = -h_i grad p_i + friction_i (Eq. force)
//   f*_ki = f_ki - (f_ki - f^eq_ki)/tau + 3 w_k c_k.F_i   (Eq. BGK)
//   f_ki(x + c_k, t+1) = f*_ki(x), periodic
//
// Layout and schedule (gfx950, wave64):
//  * Populations are stored per direction k: plane k = ny rows of `pitch`
//    nodes, x fastest, and each node holds the populations of all N layers
//    next to each other.  One 4N- (FP32), 8N- (FP64) or 2N-byte (16-bit)
//    vector access then moves a direction's populations of every layer,
//    N times fewer memory instructions than one access per layer; the step
//    is otherwise bound by the rate of vector-memory instructions.
//  * Streaming is split by axis: the y-shift is applied when a population is
//    written (push) and the x-shift when it is read (pull).  Plane k stores
//    at column x the population that belongs to node x + c_kx:
//      f_k(x, y) = S_k(x - c_kx, y),   S_k(x, y + c_ky) <- f*_k(x, y).
//    Every store of a wavefront is thus a column-aligned run (no partial
//    cache lines written twice); only loads carry the +-1 column offsets,
//    which the caches absorb.
//  * The rest population is stored as its deviation from the per-layer
//    reference height hbar_i (moving populations as they are), so that FP32
//    (and 16-bit) storage keeps the small height perturbations exact to
//    storage precision; heights are hbar_i + dh_i and interface heights are
//    handled as deviations dz_i from the reference stack.
//  * The rest plane may have its own storage type R (FP32 rest with 16-bit
//    moving populations): the rest population carries the height, whose
//    per-step change is far below a 16-bit ulp of its deviation, while the
//    moving ones are rebuilt from the moments every step.  The buffer is the
//    rest plane followed by the eight moving planes, addressed in bytes.
//  * A wavefront owns a strip of columns and marches along a segment of rows
//    in +y, one lane per column (overlapped tiling: two halo columns on each
//    side per step).  Neighbours in x come from the neighbouring lanes (DPP
//    wavefront shifts folded into the subtractions that use them), rows pass
//    through registers, so wavefronts exchange no data.  Those of a workgroup
//    meet every two rows, so that the columns neighbouring strips share are
//    read from L2.  Every row forms its stencil features once (two neighbour
//    differences per value) instead of nine neighbour reads per node.
//  * With tau = 1 a step needs only the moments of the row, so a second step
//    runs on the first one's output without leaving the wavefront: the
//    streamed populations reach the neighbouring lanes by DPP and the
//    neighbouring rows as they are marched.  Populations then move through
//    memory once per two steps, for three more halo columns and rows on each
//    side.  Intermediate values are rounded as their storage would round
//    them: results do not depend on how steps are paired.
//  * What bounds it (two steps per launch; share of the SIMDs' cycles in which a
//    vector instruction issues, SQ_ACTIVE_INST_VALU): FP32, 3 layers, 4096 x
//    4096, memory, 4.7 TB/s of population traffic at 0.90 of the streaming copy
//    with the vector units at 0.67 (386 us per step against 750 us for one step
//    per launch from LDS-tiled workgroups); f16mix, 4 layers, the vector units,
//    0.89 (449 us against 588 us); 1024 x 1024 x 3 FP32, held by the Infinity
//    Cache, 0.65 over the dispatch and 0.81 while its wavefronts run, half of it
//    on the recomputed rows of 10-row segments (29.6 us against 41.1 us).  FP64
//    films of three layers (777 x 515) issue in 0.19 of the cycles: one
//    wavefront per SIMD waits for its own results and loads.
//  * Moments wait two rows for their collision in the wavefront's own LDS, and
//    the next row's populations are prefetched into registers as loaded
//    (unconverted), so that the wait for them falls where they are used.
//  * Friction: the Poiseuille profiles of Sec. II.A.2 are fixed by the
//    interface velocities v_i (v_0 = 0).  Flux, bottom/top velocities and
//    stress continuity give a symmetric diagonally dominant tridiagonal
//    system in v, solved by Thomas elimination without pivoting:
//      g_i v_{i-1} + 2 (g_i + g_{i+1}) v_i + g_{i+1} v_{i+1}
//          = 3 (g_i U_i + g_{i+1} U_{i+1}),   g_i = mu_i / h_i, g_{N+1} = 0,
//    and friction_i = 2 mu_i h_i a_i = 6 g_i (v_{i-1} + v_i - 2 U_i).
//    With slip lengths the profile's bottom velocity w_i replaces v_{i-1}
//    (see the slip branch below); the system stays tridiagonal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace mlf {

constexpr int kMaxLayers = 4;
constexpr int kQ = 9;
constexpr int kXcds = 8;  // MI355X: workgroup b runs on XCD b % 8

// D2Q9 ordering: rest, then counter-clockwise from east.
//   k:  0  1  2  3  4  5  6  7  8
//  cx:  0  1  1  0 -1 -1 -1  0  1
//  cy:  0  0  1  1  1  0 -1 -1 -1

template <typename C>
struct StepConsts {
  int nx, ny, pitch;
  int wout, nstrip, seg_h, nseg;   // strips: columns, count; segments: rows, count
  long long plane;                 // elements per (layer, direction) plane
  C hbar[kMaxLayers];              // reference heights
  C dbar[kMaxLayers][kMaxLayers];  // reference gaps z_{l+k} - z_l, [l][k-1]
  C gamma[kMaxLayers];             // gamma_{i,i+1}
  C mu[kMaxLayers];
  C sa[kMaxLayers][kMaxLayers];   // S_lk a/(a-b), [l][k-1]
  C sb[kMaxLayers][kMaxLayers];   // S_lk b/(a-b)
  C sab[kMaxLayers][kMaxLayers];  // S_lk a b/(a-b)
  C khs[kMaxLayers];              // k h*, [k-1]
  C omega;                           // 1/tau
  C scale[kMaxLayers], iscale[kMaxLayers];  // storage scale per layer (16-bit formats)
  int ea, eb;                        // runtime exponents (generic path)
  unsigned pairs;                    // bit l*4 + k-1 set: S_lk != 0
  int slip_on;                       // any slip length != 0
  C slip[kMaxLayers];                // slip lengths beta_i
  int* flag;                         // guard flag (0 ok, 1 h<=0, 2 non-finite)
  int sr_on;                         // stochastic rounding of a 16-bit rest plane
  unsigned sr_step;                  // step count of this launch (its random draws)
};

// Storage access through raw buffer descriptors: one descriptor per group of
// three direction planes (base address and byte size in scalar registers),
// the plane's offset inside its group as the scalar offset, and per-lane
// 32-bit byte offsets shared by the planes of one type.  Accesses beyond the
// descriptor's size read zero and drop the write instead of faulting.
constexpr int kRsrcWord3 = 0x00020000;  // gfx9-family raw buffer, 32-bit format
// Per-lane offset of a masked access: at least the descriptor size (a group
// of three planes is limited to 2 GiB) and, with any plane offset added,
// still below 2^32, so the access is out of range whether or not the range
// check includes the scalar offset.
constexpr uint32_t kMasked = 0x80000000u;

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kRsrcWord3);
}

// Element formats.  16-bit formats hold the deviations of the populations
// scaled by a per-layer power of two (IEEE half: keeps the small populations
// out of the subnormal range; bfloat16: scale 1) and are converted to and
// from FP32 with round-to-nearest-even.
template <typename T>
struct Elem {
  static constexpr bool kScaled = sizeof(T) == 2;
};

template <int NW>
struct Words {
  uint32_t w[NW];
};
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// NW consecutive 32-bit words at byte offset voff + soff (+ j) through the
// widest raw buffer accesses (16, 12, 8, 4 bytes).
template <int NW>
__device__ inline void load_words(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, uint32_t (&w)[NW]) {
  int j = 0;
#pragma unroll
  for (; j + 4 <= NW; j += 4) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(voff + 4 * j), (int)soff, 0);
    w[j] = v.x, w[j + 1] = v.y, w[j + 2] = v.z, w[j + 3] = v.w;
  }
  if constexpr (NW % 4 == 3) {
    const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, (int)(voff + 4 * (NW - 3)), (int)soff, 0);
    w[NW - 3] = v.x, w[NW - 2] = v.y, w[NW - 1] = v.z;
  } else if constexpr (NW % 4 == 2) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)(voff + 4 * (NW - 2)), (int)soff, 0);
    w[NW - 2] = v.x, w[NW - 1] = v.y;
  } else if constexpr (NW % 4 == 1) {
    w[NW - 1] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(voff + 4 * (NW - 1)), (int)soff, 0);
  }
}
template <int NW>
__device__ inline void store_words(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, const uint32_t (&w)[NW]) {
  int j = 0;
#pragma unroll
  for (; j + 4 <= NW; j += 4)
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[j], w[j + 1], w[j + 2], w[j + 3]}, r, (int)(voff + 4 * j),
                                           (int)soff, 0);
  if constexpr (NW % 4 == 3)
    __builtin_amdgcn_raw_buffer_store_b96(u32x3{w[NW - 3], w[NW - 2], w[NW - 1]}, r,
                                          (int)(voff + 4 * (NW - 3)), (int)soff, 0);
  else if constexpr (NW % 4 == 2)
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[NW - 2], w[NW - 1]}, r, (int)(voff + 4 * (NW - 2)), (int)soff, 0);
  else if constexpr (NW % 4 == 1)
    __builtin_amdgcn_raw_buffer_store_b32(w[NW - 1], r, (int)(voff + 4 * (NW - 1)), (int)soff, 0);
}

__device__ inline float half_bits_to_f32(uint32_t b) {
  return (float)__builtin_bit_cast(_Float16, (unsigned short)(b & 0xffffu));
}
__device__ inline uint32_t f32_to_half_bits(float v) { return __builtin_bit_cast(unsigned short, (_Float16)v); }
__device__ inline float bf16_bits_to_f32(uint32_t b) { return __builtin_bit_cast(float, b << 16); }
__device__ inline uint32_t f32_to_bf16_bits(float v) { return __builtin_bit_cast(unsigned short, (__bf16)v); }

// 32-bit integer mixer (C. Wellons' "lowbias32": xorshift-multiply rounds).
__host__ __device__ inline uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

// Random bits of pair `pair` of layers (2 pair and 2 pair + 1 take the low
// and high 16 bits) of node `node` at the step whose key is `step_key`
// (mix32 of the step count, the same for the whole launch): a counter-based
// hash, so the draws depend on where and when they are taken, not on the
// launch shape.
__device__ inline uint32_t sr_bits(uint32_t node, int pair, uint32_t step_key) {
  return mix32((node * 2u + (uint32_t)pair) ^ step_key);
}

// Stochastic rounding of v to the 16-bit type T with the 16-bit uniform
// k16: the representable value just below or just above v, the upper one
// with probability equal to v's distance from the lower one over their gap
// (to 2^-16), so the rounding error has zero mean.  The gap is a power of
// two, so (k16 2^-16) gap and v - lo are exact in FP32 (away from the
// 16-bit type's smallest subnormals) and the comparison needs no division.
// Values T holds exactly are returned unchanged.
template <typename T>
__device__ inline float sr_round(float v, uint32_t k16) {
  constexpr bool kHalf = std::is_same_v<T, _Float16>;
  const uint32_t b = kHalf ? f32_to_half_bits(v) : f32_to_bf16_bits(v);  // nearest
  const float n = kHalf ? half_bits_to_f32(b) : bf16_bits_to_f32(b);
  if (!(n != v) || !(v - v == 0.f)) return n;  // exact, or not finite
  // the neighbour of n on v's side (sign-magnitude bit patterns)
  const bool neg = (b & 0x8000u) != 0;
  uint32_t o;
  if (n < v)
    o = neg ? (b == 0x8000u ? 0x0001u : b - 1) : b + 1;
  else
    o = neg ? b + 1 : (b == 0u ? 0x8001u : b - 1);
  const float m = kHalf ? half_bits_to_f32(o) : bf16_bits_to_f32(o);
  const float lo = n < m ? n : m, hi = n < m ? m : n;
  return (float)k16 * 0x1p-16f * (hi - lo) < v - lo ? hi : lo;
}

// The NL populations of one direction at one node (layers next to each
// other) as loaded, and their conversion to the arithmetic type C.
template <typename T, int NL>
struct Raw {
  // 16-bit types with an odd layer count take one 2-byte access per layer
  static constexpr int kWords = sizeof(T) == 2 ? (NL % 2 == 0 ? NL / 2 : NL) : NL * (int)sizeof(T) / 4;
  uint32_t w[kWords];
};
template <typename T, int NL>
__device__ inline void load_raw(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, Raw<T, NL>& v) {
  if constexpr (sizeof(T) == 2 && NL % 2 != 0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) v.w[i] = __builtin_amdgcn_raw_buffer_load_b16(r, (int)(voff + 2 * i), (int)soff, 0);
  } else {
    load_words<Raw<T, NL>::kWords>(r, voff, soff, v.w);
  }
}
template <typename T, int NL, typename C>
__device__ inline void unpack(const Raw<T, NL>& r, C (&v)[NL]) {
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if constexpr (sizeof(T) == 4) {
      v[i] = C(__builtin_bit_cast(float, r.w[i]));
    } else if constexpr (sizeof(T) == 8) {
      v[i] = C(__builtin_bit_cast(double, (unsigned long long)r.w[2 * i] | ((unsigned long long)r.w[2 * i + 1] << 32)));
    } else {
      const uint32_t b = NL % 2 != 0 ? r.w[i] : ((i & 1) ? (r.w[i / 2] >> 16) : (r.w[i / 2] & 0xffffu));
      v[i] = C(std::is_same_v<T, _Float16> ? half_bits_to_f32(b) : bf16_bits_to_f32(b));
    }
  }
}
// A value as a plane of type T holds it (scaled, rounded, read back).
template <typename T, typename C>
__device__ inline C as_stored(C v, C scale, C iscale) {
  if constexpr (std::is_same_v<T, _Float16>) return C((float)(_Float16)(float)(v * scale)) * iscale;
  else if constexpr (std::is_same_v<T, __bf16>) return C((float)(__bf16)(float)(v * scale)) * iscale;
  else return v;
}
template <typename T, int NL, typename C>
__device__ inline void store_node(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, const C (&v)[NL]) {
  if constexpr (sizeof(T) == 4) {
    uint32_t w[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) w[i] = __builtin_bit_cast(uint32_t, (float)v[i]);
    store_words<NL>(r, voff, soff, w);
  } else if constexpr (sizeof(T) == 8) {
    uint32_t w[2 * NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const unsigned long long b = __builtin_bit_cast(unsigned long long, (double)v[i]);
      w[2 * i] = (uint32_t)b;
      w[2 * i + 1] = (uint32_t)(b >> 32);
    }
    store_words<2 * NL>(r, voff, soff, w);
  } else {
    uint32_t b[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i)
      b[i] = std::is_same_v<T, _Float16> ? f32_to_half_bits((float)v[i]) : f32_to_bf16_bits((float)v[i]);
    if constexpr (NL % 2 == 0) {
      uint32_t w[NL / 2];
#pragma unroll
      for (int j = 0; j < NL / 2; ++j) w[j] = b[2 * j] | (b[2 * j + 1] << 16);
      store_words<NL / 2>(r, voff, soff, w);
    } else {
#pragma unroll
      for (int i = 0; i < NL; ++i)
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)b[i], r, (int)(voff + 2 * i), (int)soff, 0);
    }
  }
}

// Reciprocal: the hardware approximation (1 ulp) in FP32, a correctly
// rounded division in FP64.
__device__ inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double rcp(double x) { return 1.0 / x; }

template <int E, typename C>
__device__ inline C ipow_c(C r) {
  if constexpr (E == 1) {
    return r;
  } else if constexpr (E % 2 == 0) {
    C h = ipow_c<E / 2>(r);
    return h * h;
  } else {
    return r * ipow_c<E - 1>(r);
  }
}

template <typename C>
__device__ inline C ipow_rt(C r, int e) {
  C v = C(1), b = r;
  while (e > 0) {
    if (e & 1) v *= b;
    b *= b;
    e >>= 1;
  }
  return v;
}

// r^a and r^b; EA == 0 selects the runtime exponents.
template <int EA, int EB, typename C>
__device__ inline void pow_ab(C r, const StepConsts<C>& k, C& ra, C& rb) {
  if constexpr (EA == 9 && EB == 3) {
    C r3 = r * r * r;
    rb = r3;
    ra = r3 * r3 * r3;
  } else if constexpr (EA > 0) {
    ra = ipow_c<EA>(r);
    rb = ipow_c<EB>(r);
  } else {
    ra = ipow_rt(r, k.ea);
    rb = ipow_rt(r, k.eb);
  }
}

// phi = S_lk phi_k(d) = S (a r^b - b r^a)/(a - b) and
// phi' = S a b (r^a - r^b)/((a - b) d) of pair (l, k) from r^a, r^b, 1/d.
// With compile-time exponents only S a/(a - b) is read from the constants
// (b/a and b are literals): fewer live scalar registers in the row loop.
template <int EA, int EB, typename C>
__device__ inline void wetting(const StepConsts<C>& k, int l, int kk, C ra, C rb, C rd, C& phi, C& dphi) {
  const C s = k.sa[l][kk - 1];
  if constexpr (EA > 0) {
    phi = s * (rb - C(double(EB) / double(EA)) * ra);
    dphi = (s * C(EB)) * (ra - rb) * rd;
  } else {
    phi = s * rb - k.sb[l][kk - 1] * ra;
    dphi = k.sab[l][kk - 1] * (ra - rb) * rd;
  }
}

__host__ __device__ inline int wrap(int v, int n) {
  v = v < 0 ? v + n : v;
  v = v >= n ? v - n : v;
  if (v < 0 || v >= n) v = ((v % n) + n) % n;  // only for n < 3
  return v;
}

// Lanes lost on each side of a wavefront (and rows on each side of a
// segment) by `steps` steps: two stencil levels a step, and one column for
// the streaming between two steps (the first step's streaming is in its
// loads).
__host__ __device__ constexpr int march_halo(int steps) { return steps == 2 ? 5 : 2; }

// Strips of equal width (one wavefront each) over nx columns, at most
// 64 - 2 march_halo(steps) wide; recomputing the count from the width
// guarantees no empty strip.
__host__ __device__ inline int strip_width(int nx, int steps) {
  const int m = 64 - 2 * march_halo(steps);
  const int n = (nx + m - 1) / m;
  return (nx + n - 1) / n;
}
__host__ __device__ inline int strip_count(int nx, int steps) {
  const int wo = strip_width(nx, steps);
  return (nx + wo - 1) / wo;
}

// Tile of workgroup b in a grid of gridDim.x (a multiple of kXcds)
// workgroups: consecutive tiles go to the same XCD.
__device__ inline int tile_of_block(int b, int nblocks) {
  const int per = nblocks / kXcds;
  return (b % kXcds) * per + b / kXcds;
}

// ---- isotropic 9-point stencils from row features --------------------------
// A node's row feature pair is d = (e - c) - (w - c) and s = (e - c) + (w - c)
// of its value c and its two neighbours in x; rows A, B, N are y - 1, y and
// y + 1, and v_B = c_B - c_A, v_N = c_N - c_B are the differences between
// rows.  Every stencil is then a combination of per-row values that each row
// forms once (two differences instead of nine neighbour reads per node), and
// of small differences, so that no term cancels against a sum of heights.
//   d/dx = d_B / 3 + (d_N + d_A) / 12
//   d/dy = (v_N + v_B) / 2 + (s_N - s_A) / 12
//   lap  = 2 s_B / 3 + (s_N + s_A) / 6 + (v_N - v_B)
template <typename C>
__device__ inline C stencil_gx(C dA, C dB, C dN) {
  return C(1.0 / 3.0) * dB + C(1.0 / 12.0) * (dN + dA);
}
template <typename C>
__device__ inline C stencil_gy(C sA, C sN, C vB, C vN) {
  return C(0.5) * (vN + vB) + C(1.0 / 12.0) * (sN - sA);
}
template <typename C>
__device__ inline C stencil_lap(C sA, C sB, C sN, C vB, C vN) {
  return C(2.0 / 3.0) * sB + (C(1.0 / 6.0) * (sN + sA) + (vN - vB));
}

// Moments of one layer from its nine streamed populations, gathered by the
// row they come from: (a, d) = (sum, east-going minus west-going) of the
// populations 2, 3, 4 (from row y - 1), 0, 1, 5 (row y) and 6, 7, 8 (row
// y + 1).  A kernel that produces the rows one after the other keeps two
// values per row and layer instead of nine populations.
template <typename C>
struct RowSums {
  C a, d;
};
template <typename C>
__device__ inline RowSums<C> sums_n(C f2, C f3, C f4) {
  return {(f2 + f4) + f3, f2 - f4};
}
template <typename C>
__device__ inline RowSums<C> sums_m(C f0, C f1, C f5) {
  return {f0 + (f1 + f5), f1 - f5};
}
template <typename C>
__device__ inline RowSums<C> sums_s(C f6, C f7, C f8) {
  return {(f8 + f6) + f7, f8 - f6};
}
template <typename C>
__device__ inline void moments(const RowSums<C>& n, const RowSums<C>& m, const RowSums<C>& s, C& dh, C& qx, C& qy) {
  dh = m.a + (n.a + s.a);
  qx = m.d + (n.d + s.d);
  qy = n.a - s.a;
}

// Pressures p_i = sum_{j>=i} Delta_j of one node (Eqs. Laplace_pressure,
// disjoining_pressure, wetting_potential) from its interface deviations dz
// (interface i + 1) and their Laplacians and squared gradients.
template <typename C, int NL, int EA, int EB>
__device__ inline void node_pressure(const StepConsts<C>& kc, const C (&dz)[NL], const C (&lap)[NL], const C (&qq)[NL],
                                     C (&p)[NL]) {
  C dzv[NL + 1], q1[NL + 1];
  dzv[0] = C(0);
  q1[0] = C(1);
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    dzv[i + 1] = dz[i];
    q1[i + 1] = C(1) + C(0.5) * qq[i];
  }
  C sphi[NL + 1], dup[NL + 1], ddn[NL + 1];
#pragma unroll
  for (int i = 0; i <= NL; ++i) sphi[i] = dup[i] = ddn[i] = C(0);
#pragma unroll
  for (int l = 0; l < NL; ++l) {
#pragma unroll
    for (int kk = 1; kk <= NL - l; ++kk) {
      // pairs with S_lk = 0 contribute exactly zero (uniform branch)
      if (!(kc.pairs >> (l * 4 + kk - 1) & 1u)) continue;
      const C d = kc.dbar[l][kk - 1] + (dzv[l + kk] - dzv[l]);
      const C rd = rcp(d);
      const C rr = kc.khs[kk - 1] * rd;
      C ra, rb;
      pow_ab<EA, EB>(rr, kc, ra, rb);
      C phi, dphi;
      wetting<EA, EB>(kc, l, kk, ra, rb, rd, phi, dphi);
      sphi[l] += phi;
      dup[l] += dphi;
      ddn[l + kk] += dphi * q1[l];
    }
  }
  C acc = C(0);
#pragma unroll
  for (int i = NL; i >= 1; --i) {
    const C delta = -(kc.gamma[i - 1] + sphi[i]) * lap[i - 1] - dup[i] * q1[i] + ddn[i];
    acc += delta;
    p[i - 1] = acc;
  }
}

// Force (pressure gradient gpx, gpy, plus friction) and the BGK collision
// with forcing of one node from its moments dh (rest-height deviation), qx,
// qy.  With tau = 1 fo is the post-collision state f^eq + 3 w_k c_k.F;
// otherwise it is omega (f^eq) + forcing and the caller adds (1 - omega) f.
template <typename C, int NL, bool TAU1>
__device__ inline void node_collide(const StepConsts<C>& kc, const C (&dh2)[NL], const C (&qx2)[NL],
                                    const C (&qy2)[NL], const C (&gpx)[NL], const C (&gpy)[NL], C (&fo)[NL][kQ]) {
  C h[NL], ux[NL], uy[NL], g[NL + 1], rh[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    h[i] = kc.hbar[i] + dh2[i];
    rh[i] = rcp(h[i]);
    ux[i] = qx2[i] * rh[i];
    uy[i] = qy2[i] * rh[i];
    g[i] = kc.mu[i] * rh[i];
  }
  g[NL] = C(0);
  // Friction 6 g_i (w_i + v_i - 2 U_i) of every layer: Thomas elimination
  // for the interface velocities v (x and y share pivots), and the bottom
  // velocities w of the layers' profiles
  C cpr[NL], vx[NL], vy[NL], fx[NL], fy[NL];
  if (!kc.slip_on) {
    // no slip: w_i = v_{i-1}; solved for v / 3, which leaves g_i U_i +
    // g_{i+1} U_{i+1} on the right
    C tx[NL + 1], ty[NL + 1];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      tx[i] = g[i] * ux[i];
      ty[i] = g[i] * uy[i];
    }
    tx[NL] = ty[NL] = C(0);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C d = g[i] + g[i + 1];
      if (i == 0) {
        const C im = rcp(C(2) * d);
        cpr[i] = g[i + 1] * im;
        vx[i] = (tx[i] + tx[i + 1]) * im;
        vy[i] = (ty[i] + ty[i + 1]) * im;
      } else {
        const C im = rcp(C(2) * d - g[i] * cpr[i - 1]);
        cpr[i] = g[i + 1] * im;
        const C rx = tx[i] + tx[i + 1], ry = ty[i] + ty[i + 1];
        vx[i] = (rx - g[i] * vx[i - 1]) * im;
        vy[i] = (ry - g[i] * vy[i - 1]) * im;
      }
    }
#pragma unroll
    for (int i = NL - 2; i >= 0; --i) {
      vx[i] -= cpr[i] * vx[i + 1];
      vy[i] -= cpr[i] * vy[i + 1];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C g18 = C(18) * g[i];
      fx[i] = g18 * (i > 0 ? vx[i] + vx[i - 1] : vx[i]) - C(12) * tx[i];
      fy[i] = g18 * (i > 0 ? vy[i] + vy[i - 1] : vy[i]) - C(12) * ty[i];
    }
  } else {
    // slip lengths beta_i, rho = beta_i / h_i:
    //   w_i = A_i v_{i-1} + B_i v_i + E_i U_i,  A = 1 / ((1 + rho)(1 + 3 rho)),
    //   B = -rho (3 rho + 2) A,  E = 6 rho (rho + 1) A;
    // stress continuity g_i (4 v_i + 2 w_i - 6 U_i) + g_{i+1} (4 w_{i+1} + 2 v_{i+1} - 6 U_{i+1}) = 0
    C sa[NL + 1], sb[NL + 1], se[NL + 1];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C r = kc.slip[i] * rh[i];
      sa[i] = rcp((C(1) + r) * (C(1) + C(3) * r));
      sb[i] = -r * (C(3) * r + C(2)) * sa[i];
      se[i] = C(6) * r * (r + C(1)) * sa[i];
    }
    sa[NL] = sb[NL] = se[NL] = C(0);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C sub = C(2) * g[i] * sa[i];
      const C diag = g[i] * (C(4) + C(2) * sb[i]) + C(4) * g[i + 1] * sa[i + 1];
      const C sup = g[i + 1] * (C(4) * sb[i + 1] + C(2));
      const C k0 = g[i] * (C(6) - C(2) * se[i]), k1 = g[i + 1] * (C(6) - C(4) * se[i + 1]);
      const C rx = k0 * ux[i] + (i + 1 < NL ? k1 * ux[i + 1] : C(0));
      const C ry = k0 * uy[i] + (i + 1 < NL ? k1 * uy[i + 1] : C(0));
      if (i == 0) {
        const C im = rcp(diag);
        cpr[i] = sup * im;
        vx[i] = rx * im;
        vy[i] = ry * im;
      } else {
        const C im = rcp(diag - sub * cpr[i - 1]);
        cpr[i] = sup * im;
        vx[i] = (rx - sub * vx[i - 1]) * im;
        vy[i] = (ry - sub * vy[i - 1]) * im;
      }
    }
#pragma unroll
    for (int i = NL - 2; i >= 0; --i) {
      vx[i] -= cpr[i] * vx[i + 1];
      vy[i] -= cpr[i] * vy[i + 1];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C wx = sa[i] * (i > 0 ? vx[i - 1] : C(0)) + sb[i] * vx[i] + se[i] * ux[i];
      const C wy = sa[i] * (i > 0 ? vy[i - 1] : C(0)) + sb[i] * vy[i] + se[i] * uy[i];
      const C g6 = C(6) * g[i];
      fx[i] = g6 * ((wx + vx[i]) - C(2) * ux[i]);
      fy[i] = g6 * ((wy + vy[i]) - C(2) * uy[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const C qx = qx2[i], qy = qy2[i];
    const C Fx = fx[i] - h[i] * gpx[i], Fy = fy[i] - h[i] * gpy[i];
    // Shallow-water equilibrium with the rest population as deviation
    // from hbar, split into its even part (quadratic in U, shared by
    // opposite directions) and odd part c.q/c_s^2 w_k; the forcing
    // 3 w_k c_k.F is odd too.  With q_k = c_k.q and u_k = c_k.U:
    //   f^eq_k = w_k (3 q_k + 4.5 q_k u_k - 1.5 q.U),  k >= 1,
    // whose even parts are, with a = q_x U_x, b = q_y U_y and q_x U_y = q_y U_x,
    //   a/3 - b/6, b/3 - a/6 (axial) and (a + b)/12 +- q_x U_y / 4 (diagonal).
    const C a = qx * ux[i], b = qy * uy[i], m = qx * uy[i];
    const C qu = a + b, t = C(1.0 / 12.0) * qu;
    C gx = C(1.0 / 3.0) * a - C(1.0 / 6.0) * b, gy = C(1.0 / 3.0) * b - C(1.0 / 6.0) * a;  // even, axial
    C gp = t + C(0.25) * m, gm = t - C(0.25) * m;                                      // even, diagonal
    C X = qx, Y = qy;  // odd: a third of X, Y (axial), a twelfth of Y + X, Y - X (diagonal)
    fo[i][0] = dh2[i] - C(2.0 / 3.0) * qu;
    if constexpr (!TAU1) {
      const C w = kc.omega;
      fo[i][0] *= w;
      gx *= w;
      gy *= w;
      gp *= w;
      gm *= w;
      X *= w;
      Y *= w;
    }
    X += Fx;
    Y += Fy;
    const C P = Y + X, M = Y - X;
    fo[i][1] = gx + C(1.0 / 3.0) * X;
    fo[i][5] = gx - C(1.0 / 3.0) * X;
    fo[i][3] = gy + C(1.0 / 3.0) * Y;
    fo[i][7] = gy - C(1.0 / 3.0) * Y;
    fo[i][2] = gp + C(1.0 / 12.0) * P;
    fo[i][6] = gp - C(1.0 / 12.0) * P;
    fo[i][4] = gm + C(1.0 / 12.0) * M;
    fo[i][8] = gm - C(1.0 / 12.0) * M;
  }
}

// ---- the step as a march of independent wavefronts --------------------------

// Value of the next / previous lane of the wavefront (0 past its ends).
__device__ inline float lane_next(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}
__device__ inline float lane_prev(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
template <int CTRL>
__device__ inline double lane_shift(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}
__device__ inline double lane_next(double v) { return lane_shift<0x130>(v); }
__device__ inline double lane_prev(double v) { return lane_shift<0x138>(v); }

// Guard of a row's moments: `low` where a height is not positive, `inf` where
// a moment is not finite.
__device__ inline bool not_finite(float v) { return __builtin_amdgcn_classf(v, 0x207); }
__device__ inline bool not_finite(double v) { return __builtin_amdgcn_class(v, 0x207); }
template <typename C, int NL>
__device__ inline void guard_row(const StepConsts<C>& kc, const C (&dh)[NL], const C (&qx)[NL], const C (&qy)[NL],
                                 bool mine, bool& low, bool& inf) {
  C hmin = C(1);
  bool nf = false;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const C h = kc.hbar[i] + dh[i];
    hmin = h < hmin ? h : hmin;  // NaN: below
    nf = nf || not_finite(h + qx[i] + qy[i]);  // NaN or infinite if any of them is
  }
  low = low || (mine && !(hmin > C(0)));
  inf = inf || (mine && nf);
}

// ---- films one row high ------------------------------------------------------
// On one periodic row the three rows of every stencil are the node's own row:
// the y-components of the fluxes and gradients vanish up to rounding.  Films of
// one row have their own evaluation order (nine-point sums as written), shared
// by the kernels that hold such a film in LDS for many steps
// (d2q9_row_kernel.hpp, FP64 and FP32) and by row_tile below, so that all of
// them give the same bits.

// Moments of one layer from its nine populations.
template <typename C>
__device__ inline void row_moments(const C* f, C& dh, C& qx, C& qy) {
  dh = f[0] + f[1] + f[2] + f[3] + f[4] + f[5] + f[6] + f[7] + f[8];
  qx = (f[1] + f[2] + f[8]) - (f[4] + f[5] + f[6]);
  qy = (f[2] + f[3] + f[4]) - (f[6] + f[7] + f[8]);
}

// Pressures of one node from the interface deviations around it (z(i, r, c):
// interface i + 1, row r, column c of the 3x3 neighbourhood).
template <typename C, int NL, int EA, int EB, typename Z>
__device__ inline void row_pressure(const StepConsts<C>& kc, Z&& z, C (&p)[NL]) {
  C dzv[NL + 1], lap[NL + 1], qq[NL + 1];
  dzv[0] = C(0);
  qq[0] = C(0);
  lap[0] = C(0);
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const C sw = z(i, 0, 0), s = z(i, 0, 1), se = z(i, 0, 2);
    const C wv = z(i, 1, 0), cc = z(i, 1, 1), e = z(i, 1, 2);
    const C nw = z(i, 2, 0), nn = z(i, 2, 1), ne = z(i, 2, 2);
    const C gx = (e - wv) * C(1.0 / 3.0) + ((ne + se) - (nw + sw)) * C(1.0 / 12.0);
    const C gy = (nn - s) * C(1.0 / 3.0) + ((ne + nw) - (se + sw)) * C(1.0 / 12.0);
    lap[i + 1] = (C(4) * ((e + wv) + (nn + s)) + ((ne + nw) + (se + sw)) - C(20) * cc) * C(1.0 / 6.0);
    qq[i + 1] = gx * gx + gy * gy;
    dzv[i + 1] = cc;
  }
  C sphi[NL + 1], dup[NL + 1], ddn[NL + 1];
#pragma unroll
  for (int i = 0; i <= NL; ++i) sphi[i] = dup[i] = ddn[i] = C(0);
#pragma unroll
  for (int l = 0; l < NL; ++l) {
#pragma unroll
    for (int kk = 1; kk <= NL - l; ++kk) {
      if (!(kc.pairs >> (l * 4 + kk - 1) & 1u)) continue;
      const C d = kc.dbar[l][kk - 1] + (dzv[l + kk] - dzv[l]);
      const C rd = rcp(d);
      const C rr = kc.khs[kk - 1] * rd;
      C ra, rb;
      pow_ab<EA, EB>(rr, kc, ra, rb);
      C phi, dphi;
      wetting<EA, EB>(kc, l, kk, ra, rb, rd, phi, dphi);
      sphi[l] += phi;
      dup[l] += dphi;
      ddn[l + kk] += dphi * (C(1) + C(0.5) * qq[l]);
    }
  }
  C acc = C(0);
#pragma unroll
  for (int i = NL; i >= 1; --i) {
    const C delta = -(kc.gamma[i - 1] + sphi[i]) * lap[i] - dup[i] * (C(1) + C(0.5) * qq[i]) + ddn[i];
    acc += delta;
    p[i - 1] = acc;
  }
}

// Force (pressure gradient from the 3x3 pressure neighbourhood pz(i, r, c),
// laid out as z above and read where used, plus friction), and the BGK
// collision with forcing of one node from its moments dh (rest-height
// deviation), qx, qy.  With tau = 1 fo is the post-collision state
// f^eq + 3 w_k c_k.F; otherwise it is omega (f^eq) + forcing and the caller
// adds (1 - omega) f.
template <typename C, int NL, bool TAU1, typename P>
__device__ inline void row_collide(const StepConsts<C>& kc, const C (&dh2)[NL], const C (&qx2)[NL],
                                    const C (&qy2)[NL], P&& pz, C (&fo)[NL][kQ]) {
  C h[NL], ux[NL], uy[NL], g[NL + 1], rh[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    h[i] = kc.hbar[i] + dh2[i];
    rh[i] = rcp(h[i]);
    ux[i] = qx2[i] * rh[i];
    uy[i] = qy2[i] * rh[i];
    g[i] = kc.mu[i] * rh[i];
  }
  g[NL] = C(0);
  // Thomas elimination for the interface velocities v (x and y share
  // pivots) and the bottom velocities w of the layers' profiles
  C cpr[NL], vx[NL], vy[NL], wx[NL], wy[NL];
  if (!kc.slip_on) {
    // no slip: w_i = v_{i-1}
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C diag = C(2) * (g[i] + g[i + 1]);
      const C rx = C(3) * (g[i] * ux[i] + (i + 1 < NL ? g[i + 1] * ux[i + 1] : C(0)));
      const C ry = C(3) * (g[i] * uy[i] + (i + 1 < NL ? g[i + 1] * uy[i + 1] : C(0)));
      if (i == 0) {
        const C im = rcp(diag);
        cpr[i] = g[i + 1] * im;
        vx[i] = rx * im;
        vy[i] = ry * im;
      } else {
        const C im = rcp(diag - g[i] * cpr[i - 1]);
        cpr[i] = g[i + 1] * im;
        vx[i] = (rx - g[i] * vx[i - 1]) * im;
        vy[i] = (ry - g[i] * vy[i - 1]) * im;
      }
    }
#pragma unroll
    for (int i = NL - 2; i >= 0; --i) {
      vx[i] -= cpr[i] * vx[i + 1];
      vy[i] -= cpr[i] * vy[i + 1];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      wx[i] = i > 0 ? vx[i - 1] : C(0);
      wy[i] = i > 0 ? vy[i - 1] : C(0);
    }
  } else {
    // slip lengths beta_i, rho = beta_i / h_i:
    //   w_i = A_i v_{i-1} + B_i v_i + E_i U_i,  A = 1 / ((1 + rho)(1 + 3 rho)),
    //   B = -rho (3 rho + 2) A,  E = 6 rho (rho + 1) A;
    // stress continuity g_i (4 v_i + 2 w_i - 6 U_i) + g_{i+1} (4 w_{i+1} + 2 v_{i+1} - 6 U_{i+1}) = 0
    C sa[NL + 1], sb[NL + 1], se[NL + 1];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C r = kc.slip[i] * rh[i];
      sa[i] = rcp((C(1) + r) * (C(1) + C(3) * r));
      sb[i] = -r * (C(3) * r + C(2)) * sa[i];
      se[i] = C(6) * r * (r + C(1)) * sa[i];
    }
    sa[NL] = sb[NL] = se[NL] = C(0);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C sub = C(2) * g[i] * sa[i];
      const C diag = g[i] * (C(4) + C(2) * sb[i]) + C(4) * g[i + 1] * sa[i + 1];
      const C sup = g[i + 1] * (C(4) * sb[i + 1] + C(2));
      const C k0 = g[i] * (C(6) - C(2) * se[i]), k1 = g[i + 1] * (C(6) - C(4) * se[i + 1]);
      const C rx = k0 * ux[i] + (i + 1 < NL ? k1 * ux[i + 1] : C(0));
      const C ry = k0 * uy[i] + (i + 1 < NL ? k1 * uy[i + 1] : C(0));
      if (i == 0) {
        const C im = rcp(diag);
        cpr[i] = sup * im;
        vx[i] = rx * im;
        vy[i] = ry * im;
      } else {
        const C im = rcp(diag - sub * cpr[i - 1]);
        cpr[i] = sup * im;
        vx[i] = (rx - sub * vx[i - 1]) * im;
        vy[i] = (ry - sub * vy[i - 1]) * im;
      }
    }
#pragma unroll
    for (int i = NL - 2; i >= 0; --i) {
      vx[i] -= cpr[i] * vx[i + 1];
      vy[i] -= cpr[i] * vy[i + 1];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      wx[i] = sa[i] * (i > 0 ? vx[i - 1] : C(0)) + sb[i] * vx[i] + se[i] * ux[i];
      wy[i] = sa[i] * (i > 0 ? vy[i - 1] : C(0)) + sb[i] * vy[i] + se[i] * uy[i];
    }
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const C sw = pz(i, 0, 0), s = pz(i, 0, 1), se = pz(i, 0, 2);
    const C wv = pz(i, 1, 0), e = pz(i, 1, 2);
    const C nw = pz(i, 2, 0), nn = pz(i, 2, 1), ne = pz(i, 2, 2);
    const C gpx = (e - wv) * C(1.0 / 3.0) + ((ne + se) - (nw + sw)) * C(1.0 / 12.0);
    const C gpy = (nn - s) * C(1.0 / 3.0) + ((ne + nw) - (se + sw)) * C(1.0 / 12.0);
    const C frx = C(6) * g[i] * ((wx[i] + vx[i]) - C(2) * ux[i]);
    const C fry = C(6) * g[i] * ((wy[i] + vy[i]) - C(2) * uy[i]);
    const C Fx = -h[i] * gpx + frx;
    const C Fy = -h[i] * gpy + fry;
    const C qx = qx2[i], qy = qy2[i];
    const C qu = qx * ux[i] + qy * uy[i];
    const C t15 = C(1.5) * qu;
    // Shallow-water equilibrium with the rest population as deviation
    // from hbar, split into its even part (quadratic in U, shared by
    // opposite directions) and odd part c.q/c_s^2 w_k; the forcing
    // 3 w_k c_k.F is odd too.  With q_k = c_k.q and u_k = c_k.U:
    //   f^eq_k = w_k (3 q_k + 4.5 q_k u_k - 1.5 q.U),  k >= 1.
    const C ex = C(1.0 / 9.0) * (C(4.5) * qx * ux[i] - t15);  // axial x, even
    const C ey = C(1.0 / 9.0) * (C(4.5) * qy * uy[i] - t15);  // axial y, even
    const C spq = qx + qy, smq = qy - qx, spu = ux[i] + uy[i], smu = uy[i] - ux[i];
    const C ep = C(1.0 / 36.0) * (C(4.5) * spq * spu - t15);  // diagonal (1,1), even
    const C em = C(1.0 / 36.0) * (C(4.5) * smq * smu - t15);  // diagonal (-1,1), even
    C ox, oy;                                                  // axial odd parts
    if constexpr (TAU1) {
      ox = C(1.0 / 3.0) * (qx + Fx);
      oy = C(1.0 / 3.0) * (qy + Fy);
      fo[i][0] = dh2[i] - C(2.0 / 3.0) * qu;
    } else {
      const C w = kc.omega;
      ox = C(1.0 / 3.0) * (w * qx + Fx);
      oy = C(1.0 / 3.0) * (w * qy + Fy);
      fo[i][0] = w * (dh2[i] - C(2.0 / 3.0) * qu);
    }
    const C op = C(0.25) * (ox + oy), om = C(0.25) * (oy - ox);  // diagonal odd parts
    C gx = ex, gy = ey, gp = ep, gm = em;
    if constexpr (!TAU1) {
      gx = kc.omega * ex;
      gy = kc.omega * ey;
      gp = kc.omega * ep;
      gm = kc.omega * em;
    }
    fo[i][1] = gx + ox;
    fo[i][5] = gx - ox;
    fo[i][3] = gy + oy;
    fo[i][7] = gy - oy;
    fo[i][2] = gp + op;
    fo[i][6] = gp - op;
    fo[i][4] = gm + om;
    fo[i][8] = gm - om;
  }
}

// One tile of STEPS steps of a film one row high by one wavefront: lane l
// holds column x0 - HALO + l, neighbours come from the neighbouring lanes.
// Strips and halos as for march_tile, whose row pipeline would spend five rows
// on one (f16, 3 layers, 64 nodes: 6.0 us per step, launch included, 12.0 by
// the march).
template <typename R, typename S, typename C, int NL, bool TAU1, int EA, int EB, int STEPS>
__device__ inline void row_tile(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst,
                                const StepConsts<C>& kc, int tile, uint32_t sr_step) {
  constexpr int HALO = march_halo(STEPS);
  const int lane = threadIdx.x & 63;
  const int x0 = tile * kc.wout;
  const int w = min(kc.wout, kc.nx - x0);
  if (w <= 0) return;
  constexpr int kCxRow[kQ] = {0, 1, 1, 0, -1, -1, -1, 0, 1};
  const int x = wrap(x0 - HALO + lane, kc.nx);
  const long long rest = kc.plane * NL * (long long)sizeof(R);  // bytes before the moving planes
  C f[NL][kQ], fo[NL][kQ];
  // pre-collision f_k(x) = S_k(x - c_kx)
#pragma unroll
  for (int i = 0; i < NL; ++i) f[i][0] = C(reinterpret_cast<const R*>(src)[(long long)x * NL + i]);
#pragma unroll
  for (int k = 1; k < kQ; ++k) {
    const S* s = reinterpret_cast<const S*>(src + rest) + ((k - 1) * kc.plane + wrap(x - kCxRow[k], kc.nx)) * NL;
#pragma unroll
    for (int i = 0; i < NL; ++i) f[i][k] = C(s[i]);
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if constexpr (Elem<R>::kScaled) f[i][0] *= kc.iscale[i];
    if constexpr (Elem<S>::kScaled) {
#pragma unroll
      for (int k = 1; k < kQ; ++k) f[i][k] *= kc.iscale[i];
    }
  }
  bool low = false, inf = false;
#pragma unroll 1
  for (int s = 0; s < STEPS; ++s) {
    const int cut = 3 * s;  // lanes whose populations the wavefront's ends have spoilt
    const bool mine = lane >= cut && lane < 64 - cut;
    C dh[NL], qx[NL], qy[NL], zc[NL], zm[NL], zp[NL], p[NL], pm[NL], pp[NL];
    C acc = C(0);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      row_moments(f[i], dh[i], qx[i], qy[i]);
      acc += dh[i];
      zc[i] = acc;
      zm[i] = lane_prev(acc);
      zp[i] = lane_next(acc);
    }
    guard_row<C, NL>(kc, dh, qx, qy, mine, low, inf);
    row_pressure<C, NL, EA, EB>(kc, [&](int i, int, int c) { return c == 0 ? zm[i] : (c == 1 ? zc[i] : zp[i]); }, p);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      pm[i] = lane_prev(p[i]);
      pp[i] = lane_next(p[i]);
    }
    row_collide<C, NL, TAU1>(
        kc, dh, qx, qy, [&](int i, int, int c) { return c == 0 ? pm[i] : (c == 1 ? p[i] : pp[i]); }, fo);
#pragma unroll
    for (int i = 0; i < NL; ++i)
#pragma unroll
      for (int k = 0; k < kQ; ++k) {
        if constexpr (!TAU1) fo[i][k] += (C(1) - kc.omega) * f[i][k];
        // as stored, streamed to the next step's node (the y-shift stays in the row)
        if constexpr (STEPS == 2) {
          const C v = k == 0 ? as_stored<R>(fo[i][k], kc.scale[i], kc.iscale[i])
                             : as_stored<S>(fo[i][k], kc.scale[i], kc.iscale[i]);
          f[i][k] = kCxRow[k] == 0 ? v : (kCxRow[k] > 0 ? lane_prev(v) : lane_next(v));
        }
      }
  }
  if (lane >= HALO && lane < HALO + w) {
    R* d0 = reinterpret_cast<R*>(dst) + (long long)x * NL;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      C v = Elem<R>::kScaled ? fo[i][0] * kc.scale[i] : fo[i][0];
      if constexpr (Elem<R>::kScaled) {
        if (kc.sr_on)
          v = sr_round<R>(v, (sr_bits((uint32_t)x, i / 2, mix32(sr_step + 0x9e3779b9u)) >> (16 * (i % 2))) & 0xffffu);
      }
      d0[i] = (R)v;
    }
#pragma unroll
    for (int k = 1; k < kQ; ++k) {
      S* d = reinterpret_cast<S*>(dst + rest) + ((k - 1) * kc.plane + x) * NL;
#pragma unroll
      for (int i = 0; i < NL; ++i) d[i] = (S)(Elem<S>::kScaled ? fo[i][k] * kc.scale[i] : fo[i][k]);
    }
  }
  if (inf) kc.flag[0] = 2;
  else if (low) kc.flag[0] = 1;
}

// Whether the row pipelines keep their interface features in LDS, and the LDS
// of one wavefront in bytes.
template <typename C>
__host__ __device__ constexpr bool march_zlds(int nl, int steps) {
  return (nl == 4 && steps == 2) || (sizeof(C) == 8 && nl >= 3);
}
template <typename C>
__host__ __device__ constexpr size_t march_lds(int nl, int steps) {
  return (size_t)steps * 2 * (march_zlds<C>(nl, steps) ? 5 : 3) * nl * 64 * sizeof(C);
}

// Row pipeline of one step in a wavefront marching towards +y: features of
// the interface deviations and of the pressures of the last two rows (row
// r - 2 in slot P, r - 1 in slot P ^ 1, P the parity of row r, so that a
// loop unrolled by two moves no registers), and the moments of the last two
// rows, which only the row after next needs, in the wavefront's own part of
// LDS (`mom`: [2][3 NL][64], one slot per parity): with them in registers the
// two-step kernels spill, and every reload from scratch waits for all loads
// in flight.
// ZL keeps the interface features zs, zd there too (four layers and two
// steps).
template <typename C, int NL, bool ZL>
struct RowPipe {
  C zc[NL], zv[NL], zs[ZL ? 1 : 2][NL], zd[ZL ? 1 : 2][NL];
  C pc[NL], pv[NL], ps[2][NL], pd[2][NL];
  C* mom;  // this lane's column: moments [2][3 NL], with ZL features [2][2 NL]

  static constexpr int kWords = 2 * (ZL ? 5 : 3) * NL * 64;  // values per wavefront

  __device__ void clear(C* wave_mom) {
    mom = wave_mom + (threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < NL; ++i) zc[i] = zv[i] = pc[i] = pv[i] = C(0);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        ps[j][i] = pd[j][i] = C(0);
        if constexpr (!ZL) zs[j][i] = zd[j][i] = C(0);
      }
#pragma unroll
    for (int q = 0; q < kWords / 64; ++q) mom[q * 64] = C(0);
  }

  // Takes the moments of row r, forms the pressures of row r - 1, and with
  // COLLIDE the collision of row r - 2 (into fo); moves on by a row.  Valid
  // in lanes with two valid neighbours on each side; collisions from the
  // fifth row on.
  template <int P, bool TAU1, int EA, int EB>
  __device__ void advance(const StepConsts<C>& kc, const C (&dh0)[NL], const C (&qx0)[NL], const C (&qy0)[NL],
                          bool collide, C (&fo)[NL][kQ]) {
    C lap[NL], qq[NL], p[NL], dz[NL];
    C acc = C(0);
    C* zl = mom + 6 * NL * 64;
    constexpr int A = P, B = P ^ 1;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      C sA, sB, dA, dB;
      if constexpr (ZL) {
        sA = zl[(A * 2 * NL + i) * 64], dA = zl[(A * 2 * NL + NL + i) * 64];
        sB = zl[(B * 2 * NL + i) * 64], dB = zl[(B * 2 * NL + NL + i) * 64];
      } else {
        sA = zs[A][i], sB = zs[B][i], dA = zd[A][i], dB = zd[B][i];
      }
      acc += dh0[i];
      const C c = acc;
      const C e = lane_next(c) - c, w = lane_prev(c) - c;
      const C s = e + w, d = e - w, v = c - zc[i];
      lap[i] = stencil_lap(sA, sB, s, zv[i], v);
      const C gx = stencil_gx(dA, dB, d), gy = stencil_gy(sA, s, zv[i], v);
      qq[i] = gx * gx + gy * gy;
      dz[i] = zc[i];
      if constexpr (ZL) {
        zl[(A * 2 * NL + i) * 64] = s;
        zl[(A * 2 * NL + NL + i) * 64] = d;
      } else {
        zs[A][i] = s;
        zd[A][i] = d;
      }
      zv[i] = v;
      zc[i] = c;
    }
    node_pressure<C, NL, EA, EB>(kc, dz, lap, qq, p);
    __builtin_amdgcn_sched_barrier(0);
    C dh2[NL], qx2[NL], qy2[NL];
    C* m = mom + P * 3 * NL * 64;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      dh2[i] = m[i * 64];
      qx2[i] = m[(NL + i) * 64];
      qy2[i] = m[(2 * NL + i) * 64];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      m[i * 64] = dh0[i];
      m[(NL + i) * 64] = qx0[i];
      m[(2 * NL + i) * 64] = qy0[i];
    }
    C gpx[NL], gpy[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const C c = p[i];
      const C e = lane_next(c) - c, w = lane_prev(c) - c;
      const C s = e + w, d = e - w, v = c - pc[i];
      gpx[i] = stencil_gx(pd[A][i], pd[B][i], d);
      gpy[i] = stencil_gy(ps[A][i], s, pv[i], v);
      ps[A][i] = s;
      pd[A][i] = d;
      pv[i] = v;
      pc[i] = c;
    }
    if (collide) node_collide<C, NL, TAU1>(kc, dh2, qx2, qy2, gpx, gpy, fo);
    __builtin_amdgcn_sched_barrier(0);
  }
};

// One tile (a strip of kc.wout columns x a segment of kc.seg_h rows) of STEPS
// (1 or 2) time steps by one wavefront.  `tile` is uniform: strips first, so
// that a workgroup's wavefronts are neighbours along a row.
// Lane l holds column x0 - HALO + l; x neighbours come from the neighbouring
// lanes, rows are marched in +y, and nothing is shared between wavefronts.
// `sr_step` is the film's step count, the counter of its stochastic-rounding
// draws (read only when kc.sr_on; one step only).  AHEAD loads a row while the
// one before it is processed.
template <typename R, typename S, typename C, int NL, bool TAU1, int EA, int EB, int STEPS, bool AHEAD>
__device__ inline void march_tile(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst,
                                  const StepConsts<C>& kc, int tile, uint32_t sr_step, C* wave_lds) {
  static_assert(STEPS == 1 || (STEPS == 2 && TAU1), "two steps need tau = 1");
  constexpr int HALO = march_halo(STEPS);
  const int lane = threadIdx.x & 63;
  const int seg = tile / kc.nstrip;
  const int x0 = (tile - seg * kc.nstrip) * kc.wout;
  const int w = min(kc.wout, kc.nx - x0);
  const int y0 = seg * kc.seg_h;
  const int rows = min(kc.seg_h, kc.ny - y0);
  const int npass = kc.seg_h + 2 * HALO;  // of every wavefront of the workgroup (barriers)
  constexpr uint32_t nodeb = NL * sizeof(S), nodebr = NL * sizeof(R);  // bytes per node
  const uint32_t rowb = (uint32_t)kc.pitch * nodeb;    // bytes per row, moving planes
  const uint32_t rowbr = (uint32_t)kc.pitch * nodebr;  // bytes per row, rest plane
  const uint32_t planeb = (uint32_t)(kc.plane * (long long)nodeb);
  const uint32_t planebr = (uint32_t)(kc.plane * (long long)nodebr);
  if (rows <= 0) {  // a wavefront past the last tile (uniform): the barriers only
    for (int it = 0; it < npass; it += 2) __builtin_amdgcn_s_barrier();
    return;
  }
  // descriptors of the plane groups {0, 1, 2}, {3, 4, 5}, {6, 7, 8}
  const uint32_t g0b = planebr + 2u * planeb, g1b = 3u * planeb;
  __amdgpu_buffer_rsrc_t rs[3], rd[3];
  rs[0] = make_rsrc(src, g0b);
  rs[1] = make_rsrc(src + g0b, g1b);
  rs[2] = make_rsrc(src + (long long)g0b + g1b, g1b);
  rd[0] = make_rsrc(dst, g0b);
  rd[1] = make_rsrc(dst + g0b, g1b);
  rd[2] = make_rsrc(dst + (long long)g0b + g1b, g1b);

  const int x = wrap(x0 - HALO + lane, kc.nx);
  const uint32_t bx = (uint32_t)x * nodeb;
  const uint32_t bxm = (uint32_t)wrap(x - 1, kc.nx) * nodeb;
  const uint32_t bxp = (uint32_t)wrap(x + 1, kc.nx) * nodeb;
  const uint32_t bxr = (uint32_t)x * nodebr;
  const bool out_lane = lane >= HALO && lane < HALO + w;

  // Populations of one row as loaded (converted where they are used, so that
  // the loads stay in flight until then).  Pre-collision f_k(x, y) =
  // S_k(x - c_kx, y): directions 1, 2, 8 read column x - 1, directions 4, 5,
  // 6 column x + 1.
  Raw<R, NL> w0;
  Raw<S, NL> wk[kQ - 1];
  auto load_row = [&](int y, Raw<R, NL>& r0, Raw<S, NL> (&rk)[kQ - 1]) {
    const uint32_t row = (uint32_t)y * rowb, rowr = (uint32_t)y * rowbr;
    load_raw<R, NL>(rs[0], bxr, rowr, r0);
    load_raw<S, NL>(rs[0], bxm, planebr + row, rk[0]);
    load_raw<S, NL>(rs[0], bxm, planebr + planeb + row, rk[1]);
    load_raw<S, NL>(rs[1], bx, row, rk[2]);
    load_raw<S, NL>(rs[1], bxp, planeb + row, rk[3]);
    load_raw<S, NL>(rs[1], bxp, 2u * planeb + row, rk[4]);
    load_raw<S, NL>(rs[2], bxp, row, rk[5]);
    load_raw<S, NL>(rs[2], bx, planeb + row, rk[6]);
    load_raw<S, NL>(rs[2], bxm, 2u * planeb + row, rk[7]);
  };
  // Post-collision f*_k(x, y) goes to S_k(x, y + c_ky); rows yS, y, yN are
  // y - 1, y, y + 1.  v holds scaled values (as stored).
  auto store_row = [&](bool ok, int yS, int y, int yN, const C (&v)[kQ][NL]) {
    const uint32_t vo = ok ? bx : kMasked, vr = ok ? bxr : kMasked;
    const uint32_t oS = (uint32_t)yS * rowb, oC = (uint32_t)y * rowb, oN = (uint32_t)yN * rowb;
    store_node<R, NL>(rd[0], vr, (uint32_t)y * rowbr, v[0]);
    store_node<S, NL>(rd[0], vo, planebr + oC, v[1]);
    store_node<S, NL>(rd[0], vo, planebr + planeb + oN, v[2]);
    store_node<S, NL>(rd[1], vo, oN, v[3]);
    store_node<S, NL>(rd[1], vo, planeb + oN, v[4]);
    store_node<S, NL>(rd[1], vo, 2u * planeb + oC, v[5]);
    store_node<S, NL>(rd[2], vo, oS, v[6]);
    store_node<S, NL>(rd[2], vo, planeb + oS, v[7]);
    store_node<S, NL>(rd[2], vo, 2u * planeb + oS, v[8]);
  };
  auto scaled = [&](const C (&fo)[NL][kQ], C (&v)[kQ][NL]) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      v[0][i] = Elem<R>::kScaled ? fo[i][0] * kc.scale[i] : fo[i][0];
#pragma unroll
      for (int k = 1; k < kQ; ++k) v[k][i] = Elem<S>::kScaled ? fo[i][k] * kc.scale[i] : fo[i][k];
    }
  };

  typedef RowPipe<C, NL, march_zlds<C>(NL, STEPS)> Pipe;
  Pipe pipe;
  pipe.clear(wave_lds);
  // second step: its pipeline, and the row sums of the first step's output
  // that still wait for a row (N of the last two rows, by parity, M of the
  // last one)
  std::conditional_t<STEPS == 2, Pipe, int> pipe2;
  RowSums<C> ns[2][NL], ms[NL];
  if constexpr (STEPS == 2) {
    pipe2.clear(wave_lds + Pipe::kWords);
#pragma unroll
    for (int i = 0; i < NL; ++i) ns[0][i] = ns[1][i] = ms[i] = RowSums<C>{C(0), C(0)};
  }
  bool low = false, inf = false;
  const int niter = rows + 2 * HALO;
  int yl = wrap(y0 - HALO, kc.ny);       // row being loaded
  int ys = wrap(y0 - 2 * HALO, kc.ny);   // row being stored (valid from iteration 2 HALO on)
  auto next_row = [&](int y) { return y + 1 == kc.ny ? 0 : y + 1; };
  if constexpr (AHEAD) load_row(yl, w0, wk);
  // Every iteration issues the same vector-memory sequence (the next row's
  // loads, then this row's stores; lanes and rows without output store out
  // of range, which the hardware drops): the compiler's wait for a row's
  // loads then never covers the stores issued after them.
  auto body = [&](auto parity, int it) {
    constexpr int P = decltype(parity)::value;
    const bool live = it < niter;  // false in the last pass of an odd count
    C dh[NL], qx[NL], qy[NL];
    if constexpr (!AHEAD) load_row(yl, w0, wk);
    {
      C f0[NL], f[kQ - 1][NL];
      unpack<R, NL>(w0, f0);
#pragma unroll
      for (int k = 0; k < kQ - 1; ++k) unpack<S, NL>(wk[k], f[k]);
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        if constexpr (Elem<R>::kScaled) f0[i] *= kc.iscale[i];
        if constexpr (Elem<S>::kScaled) {
#pragma unroll
          for (int k = 0; k < kQ - 1; ++k) f[k][i] *= kc.iscale[i];
        }
        moments(sums_n(f[1][i], f[2][i], f[3][i]), sums_m(f0[i], f[0][i], f[4][i]), sums_s(f[5][i], f[6][i], f[7][i]),
                dh[i], qx[i], qy[i]);
      }
    }
    guard_row<C, NL>(kc, dh, qx, qy, true, low, inf);
    if (it + 1 < niter) yl = next_row(yl);
    if constexpr (AHEAD) load_row(yl, w0, wk);
    __builtin_amdgcn_sched_barrier(0);
    // collisions of rows that no output needs are skipped (uniform branches
    // without vector-memory instructions): the first four rows of a step
    // only feed its stencils
    C fo[NL][kQ], v[kQ][NL];
#pragma unroll
    for (int i = 0; i < NL; ++i)
#pragma unroll
      for (int k = 0; k < kQ; ++k) fo[i][k] = C(0);
    pipe.template advance<P, TAU1, EA, EB>(kc, dh, qx, qy, it >= 4, fo);
    if constexpr (STEPS == 1) {
      if constexpr (!TAU1) {
        // f* = (1 - omega) f + [omega f^eq + forcing]; the pre-collision
        // populations of the row are re-read (cache hits: loaded two rows ago)
        Raw<R, NL> r0;
        Raw<S, NL> rk[kQ - 1];
        load_row(ys, r0, rk);
        C f[kQ][NL];
        unpack<R, NL>(r0, f[0]);
#pragma unroll
        for (int k = 1; k < kQ; ++k) unpack<S, NL>(rk[k - 1], f[k]);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          if constexpr (Elem<R>::kScaled) f[0][i] *= kc.iscale[i];
#pragma unroll
          for (int k = 0; k < kQ; ++k) {
            if constexpr (Elem<S>::kScaled)
              if (k > 0) f[k][i] *= kc.iscale[i];
            fo[i][k] += (C(1) - kc.omega) * f[k][i];
          }
        }
      }
      scaled(fo, v);
      if constexpr (Elem<R>::kScaled) {
        // stochastic rounding of the stored rest population, in the scaled
        // form the store writes, so that the store's conversion is exact
        if (kc.sr_on) {
          const uint32_t node = (uint32_t)ys * (uint32_t)kc.nx + (uint32_t)x;
          const uint32_t key = mix32(sr_step + 0x9e3779b9u);
          uint32_t bits[(NL + 1) / 2];
#pragma unroll
          for (int j = 0; j < (NL + 1) / 2; ++j) bits[j] = sr_bits(node, j, key);
#pragma unroll
          for (int i = 0; i < NL; ++i)
            v[0][i] = sr_round<R>(v[0][i], (bits[i / 2] >> (16 * (i % 2))) & 0xffffu);
        }
      }
    } else {
      if (it >= 4) {
        // first step's output as its storage would hold it, streamed into
        // the second step's rows without leaving the wavefront
        C mh[NL], mx[NL], my[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          C f[kQ];
          f[0] = as_stored<R>(fo[i][0], kc.scale[i], kc.iscale[i]);
#pragma unroll
          for (int k = 1; k < kQ; ++k) f[k] = as_stored<S>(fo[i][k], kc.scale[i], kc.iscale[i]);
          const RowSums<C> n = sums_n(lane_prev(f[2]), f[3], lane_next(f[4]));
          const RowSums<C> m = sums_m(f[0], lane_prev(f[1]), lane_next(f[5]));
          const RowSums<C> s = sums_s(lane_next(f[6]), f[7], lane_prev(f[8]));
          moments(ns[P][i], ms[i], s, mh[i], mx[i], my[i]);
          ns[P][i] = n;
          ms[i] = m;
        }
        if (it >= 6) {
          guard_row<C, NL>(kc, mh, mx, my, live && lane >= 3 && lane < 61, low, inf);
          pipe2.template advance<P, TAU1, EA, EB>(kc, mh, mx, my, it >= 2 * HALO, fo);
        }
      }
      scaled(fo, v);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int yn = next_row(ys);
    store_row(out_lane && live && it >= 2 * HALO, ys == 0 ? kc.ny - 1 : ys - 1, ys, yn, v);
    ys = yn;
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll 1
  for (int it = 0; it < npass; it += 2) {
    if (it < niter) {
      body(std::integral_constant<int, 0>{}, it);
      body(std::integral_constant<int, 1>{}, it + 1);
    }
    // keeps the workgroup's strips on the same rows, so that the columns
    // neighbouring strips share are read from L2: 4096 x 4096 x 3 FP32 470 ->
    // 416 us per step (a no-op for workgroups of one wavefront)
    __builtin_amdgcn_s_barrier();
  }
  if (inf) kc.flag[0] = 2;
  else if (low) kc.flag[0] = 1;
}

// Lanes of the workgroups that the step kernel is compiled for: 512 (at most
// 256 registers per lane) or, where that is not enough for the working set
// with a row ahead, 256 (512 registers, one wavefront per SIMD).  FP64
// arithmetic on four layers needs the latter everywhere; on three layers
// (274 registers) it serves workgroups of up to 256 lanes, and wider ones
// load each row when they come to it, since the row ahead would spill: 2048 x
// 2048 at 256 x 40 394 us per step against 414 without the row ahead, 1000 x
// 1000 at 256 x 18 103.5 / 112.6, 777 x 515 at 64 x 10 36.0 / 38.1.
template <typename C, int NL>
constexpr int step_lanes(int block_w) {
  return sizeof(C) == 8 && (NL == 4 || (NL == 3 && block_w <= 256)) ? 256 : 512;
}

template <typename R, typename S, typename C, int NL, bool TAU1, int EA, int EB, int STEPS, int LANES>
__global__ void __launch_bounds__(LANES)
step_kernel(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst, const StepConsts<C> kc) {
  constexpr bool kAhead = !(sizeof(C) == 8 && NL == 3 && LANES == 512);
  const int group = tile_of_block(blockIdx.x, gridDim.x);
  const int nw = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (group * nw >= kc.nstrip * kc.nseg) return;  // padding workgroup (uniform)
  extern __shared__ unsigned char smem_raw[];
  C* lds = reinterpret_cast<C*>(smem_raw + wave * march_lds<C>(NL, STEPS));
  march_tile<R, S, C, NL, TAU1, EA, EB, STEPS, kAhead>(src, dst, kc, group * nw + wave, kc.sr_step, lds);
}

// One step of a film one row high.
template <typename R, typename S, typename C, int NL, bool TAU1, int EA, int EB>
__global__ void __launch_bounds__(512)
row_step_kernel(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst, const StepConsts<C> kc) {
  const int tile = blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  row_tile<R, S, C, NL, TAU1, EA, EB, 1>(src, dst, kc, tile, kc.sr_step);
}

// ---- batches of independent films -----------------------------------------
// Per-film entry of the device table: step constants (launch geometry
// included), byte offset of the film's populations in both buffers, and
// its layer count.
template <typename C>
struct BatchFilm {
  StepConsts<C> kc;
  long long offset;
  int nl;
  int pad;
};

template <typename R, typename S, typename C, int NL, bool TAU1, int EA, int EB, int STEPS>
__device__ inline void batch_tile(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst,
                                  const StepConsts<C>& kc, int tile, uint32_t step, C* lds) {
  if (kc.ny == 1) {  // uniform for the workgroup: one film per item
    row_tile<R, S, C, NL, TAU1, EA, EB, STEPS>(src, dst, kc, tile, step);
    return;
  }
  march_tile<R, S, C, NL, TAU1, EA, EB, STEPS, true>(src, dst, kc, tile, step, lds);
}

// One launch advances every film of a batch by STEPS steps.  Work item w
// (film, group of tiles, one per wavefront) is items[w]; items are ordered by the
// cost of a tile, longest first.  With
// gridDim.x < n_items the workgroups are persistent and take items
// w = r * gridDim.x + tile_of_block(blockIdx.x, gridDim.x), r = 0, 1, ...;
// either way consecutive items run on one XCD.  `flip` selects the source
// buffer (0: a -> b, 1: b -> a); `step` is the batch's step count (every
// film's stochastic-rounding counter, so that a film draws as it would
// stepped alone).
template <typename R, typename S, typename C, bool TAU1, int EA, int EB, int STEPS>
__global__ void __launch_bounds__(256, sizeof(C) == 8 ? 1 : 2)
batch_kernel(const BatchFilm<C>* __restrict__ films, const int2* __restrict__ items, int n_items,
             unsigned char* __restrict__ buf_a, unsigned char* __restrict__ buf_b, int flip, uint32_t step) {
  const int slot = tile_of_block(blockIdx.x, gridDim.x);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  extern __shared__ unsigned char smem_raw[];
  C* lds = reinterpret_cast<C*>(smem_raw + wave * march_lds<C>(kMaxLayers, STEPS));
  for (int w = slot; w < n_items; w += gridDim.x) {
    const int2 item = items[w];
    const BatchFilm<C>& bf = films[item.x];
    const unsigned char* src = (flip ? buf_b : buf_a) + bf.offset;
    unsigned char* dst = (flip ? buf_a : buf_b) + bf.offset;
    const int tile = item.y * nw + wave;
    switch (bf.nl) {
      case 1: batch_tile<R, S, C, 1, TAU1, EA, EB, STEPS>(src, dst, bf.kc, tile, step, lds); break;
      case 2: batch_tile<R, S, C, 2, TAU1, EA, EB, STEPS>(src, dst, bf.kc, tile, step, lds); break;
      case 3: batch_tile<R, S, C, 3, TAU1, EA, EB, STEPS>(src, dst, bf.kc, tile, step, lds); break;
      default: batch_tile<R, S, C, 4, TAU1, EA, EB, STEPS>(src, dst, bf.kc, tile, step, lds); break;
    }
  }
}

}  // namespace mlf
