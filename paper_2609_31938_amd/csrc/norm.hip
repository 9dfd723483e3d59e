// The normalised block form's prologue as one pass over the new chunk: each
// pixel (n, t, p) of x [N][Ci][T][H*W] (bf16) is normalised by the root mean
// square of its Ci channel values, then a per-channel gain and bias and SiLU
// apply, and one round-to-nearest-even conversion writes u (same layout):
//   r[n,t,p] = 1 / sqrt( (1/Ci) sum_c x[n,c,t,p]^2 + eps )
//   u[n,c,t,p] = RNE_bf16( SiLU( x[n,c,t,p] * r[n,t,p] * gamma[c] + beta[c] ) )
// (the decoder residual block's normalisation and activation ahead of its
// causal convolution; fp32 arithmetic, hardware reciprocal square root,
// exponential and reciprocal).
//
// A workgroup owns 128 consecutive pixels of one (n, t) frame plane and all
// Ci channels.  Aligned form (AL: H*W a multiple of 8, 16-byte-aligned x and u):
// thread (channel lane cl = tid / 16, pixel group pg = tid % 16) reads 16-byte
// runs of 8 pixels of channels cl, cl + 16, ...; the 16 channel lanes' partial
// sums of squares meet in LDS, and a second sweep over the same runs (L2-hot)
// writes u; with at most 384 channels the tile stays in registers between
// the two sweeps (all loads in flight at once, x read once).  Without AL (a
// plane of any size, any 2-byte alignment) the same 16 bytes are read and
// written unaligned, and a plane's last, partial run element by element (read
// two bytes at a time by two channel lanes a pixel, odd planes spent 32 to 53
// us more in this pass: the block form 208 -> 208 at 135x241, two frames, 268
// us, 236 now; 400 -> 400 at 67x121 316, 263 now).  x is read from HBM once and
// u written once: an HBM-bound pass.
#include "c3c_internal.h"
#include "fuse_dev.h"

namespace c3c {
namespace {

constexpr int NPX = 128;  // pixels per workgroup

// 8 pixels, of which the first m lie in the plane (zeros past them)
template <bool AL>
__device__ inline fuse_u32x4 load8(const uint16_t* p, int64_t m) {
  fuse_u32x4 v = {0u, 0u, 0u, 0u};
  if (AL) {
    v = *reinterpret_cast<const fuse_u32x4*>(p);
  } else if (m >= 8) {
    __builtin_memcpy(&v, p, 16);  // at any 2-byte alignment
  } else {
#pragma unroll
    for (int e = 0; e < 7; ++e)
      if (e < m) v[e >> 1] |= static_cast<uint32_t>(p[e]) << (16 * (e & 1));
  }
  return v;
}

template <bool AL>
__device__ inline void store8(uint16_t* p, fuse_u32x4 v, int64_t m) {
  if (AL) {
    *reinterpret_cast<fuse_u32x4*>(p) = v;
  } else if (m >= 8) {
    __builtin_memcpy(p, &v, 16);
  } else {
#pragma unroll
    for (int e = 0; e < 7; ++e)
      if (e < m) p[e] = static_cast<uint16_t>(v[e >> 1] >> (16 * (e & 1)));
  }
}

// The whole tile in registers (Ci <= 16 * CPL channel rows,
// CPL per lane): every load of x is issued before the first sum is formed, x
// is read once, and the second sweep works on the registers.  The smallest
// of CPL = 6, 12, 24 that holds the call's channels is launched (fewer
// registers, more workgroups per compute unit).
constexpr int kMaxCpl = 24;
template <int CPL, bool AL>
__global__ __launch_bounds__(256) void rms_prologue_regs(const uint16_t* __restrict__ x,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta, float eps,
                                                         uint16_t* __restrict__ u, int64_t Ci,
                                                         int64_t T, int64_t hw, int64_t tiles) {
  __shared__ float part[16][NPX];
  __shared__ float rr[NPX];
  const int tid = threadIdx.x;
  const int cl = tid >> 4, pg = tid & 15;
  const int64_t b = blockIdx.x;
  const int64_t tile = b % tiles, nt = b / tiles;
  const int64_t n = nt / T, t = nt % T;
  const int64_t p0 = tile * NPX + static_cast<int64_t>(pg) * 8;
  const bool in = p0 < hw;
  const uint16_t* xb = x + ((n * Ci) * T + t) * hw + p0;  // channel 0 of this group
  uint16_t* ub = u + ((n * Ci) * T + t) * hw + p0;
  const int64_t cstride = T * hw;  // elements between channel planes
  fuse_u32x4 v[CPL];
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    const int64_t c = cl + 16 * i;
    v[i] = (in && c < Ci) ? load8<AL>(xb + c * cstride, hw - p0) : fuse_u32x4{0u, 0u, 0u, 0u};
  }
  float ss[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) ss[e] = 0.f;
#pragma unroll
  for (int i = 0; i < CPL; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = fuse_widen(v[i][e] & 0xffffu), hi = fuse_widen(v[i][e] >> 16);
      ss[2 * e] = __builtin_fmaf(lo, lo, ss[2 * e]);
      ss[2 * e + 1] = __builtin_fmaf(hi, hi, ss[2 * e + 1]);
    }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[cl][pg * 8 + e] = ss[e];
  __syncthreads();
  if (tid < NPX) {
    float sum = 0.f;
#pragma unroll
    for (int l = 0; l < 16; ++l) sum += part[l][tid];
    rr[tid] = __builtin_amdgcn_rsqf(sum / static_cast<float>(Ci) + eps);
  }
  __syncthreads();
  if (!in) return;
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = rr[pg * 8 + e];
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    const int64_t c = cl + 16 * i;
    if (c >= Ci) break;
    const float g = gamma[c], bb = beta[c];
    fuse_u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = fuse_silu(__builtin_fmaf(fuse_widen(v[i][e] & 0xffffu) * r[2 * e], g, bb));
      const float d = fuse_silu(__builtin_fmaf(fuse_widen(v[i][e] >> 16) * r[2 * e + 1], g, bb));
      o[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((fuse_f32x2{a, d}), fuse_bf16x2));
    }
    store8<AL>(ub + c * cstride, o, hw - p0);
  }
}

// More channels than the registers hold: x is read again for the second sweep.
template <bool AL>
__global__ __launch_bounds__(256) void rms_prologue_pass(const uint16_t* __restrict__ x,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta, float eps,
                                                         uint16_t* __restrict__ u, int64_t Ci,
                                                         int64_t T, int64_t hw, int64_t tiles) {
  constexpr int LANES = 16;  // channel lanes
  constexpr int PPT = 8;     // pixels per thread
  __shared__ float part[LANES][NPX];
  __shared__ float rr[NPX];
  const int tid = threadIdx.x;
  const int cl = tid >> 4, pg = tid & 15;
  const int64_t b = blockIdx.x;
  const int64_t tile = b % tiles, nt = b / tiles;  // nt = n * T + t
  const int64_t n = nt / T, t = nt % T;
  const int64_t p0 = tile * NPX + static_cast<int64_t>(pg) * PPT;  // this thread's first pixel
  const bool in = p0 < hw;
  // element (c, p0) of this (n, t) plane
  auto at = [&](int64_t c) { return ((n * Ci + c) * T + t) * hw + p0; };

  float ss[PPT];
#pragma unroll
  for (int e = 0; e < PPT; ++e) ss[e] = 0.f;
  if (in) {
    for (int64_t c = cl; c < Ci; c += LANES) {
      const fuse_u32x4 v = load8<AL>(x + at(c), hw - p0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = fuse_widen(v[e] & 0xffffu), hi = fuse_widen(v[e] >> 16);
        ss[2 * e] = __builtin_fmaf(lo, lo, ss[2 * e]);
        ss[2 * e + 1] = __builtin_fmaf(hi, hi, ss[2 * e + 1]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < PPT; ++e) part[cl][pg * PPT + e] = ss[e];
  __syncthreads();
  if (tid < NPX) {
    float s = 0.f;
#pragma unroll
    for (int l = 0; l < LANES; ++l) s += part[l][tid];
    rr[tid] = __builtin_amdgcn_rsqf(s / static_cast<float>(Ci) + eps);
  }
  __syncthreads();
  if (!in) return;
  float r[PPT];
#pragma unroll
  for (int e = 0; e < PPT; ++e) r[e] = rr[pg * PPT + e];
  for (int64_t c = cl; c < Ci; c += LANES) {
    const float g = gamma[c], bb = beta[c];
    const fuse_u32x4 v = load8<AL>(x + at(c), hw - p0);
    fuse_u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = fuse_silu(__builtin_fmaf(fuse_widen(v[e] & 0xffffu) * r[2 * e], g, bb));
      const float d = fuse_silu(__builtin_fmaf(fuse_widen(v[e] >> 16) * r[2 * e + 1], g, bb));
      o[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((fuse_f32x2{a, d}), fuse_bf16x2));
    }
    store8<AL>(u + at(c), o, hw - p0);
  }
}

template <bool AL>
auto pick_kernel(int64_t Ci) {
  return Ci <= 16 * 6         ? rms_prologue_regs<6, AL>
         : Ci <= 16 * 12      ? rms_prologue_regs<12, AL>
         : Ci <= 16 * kMaxCpl ? rms_prologue_regs<kMaxCpl, AL>
                              : rms_prologue_pass<AL>;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

hipError_t launch_rms_prologue(const Geo& g, const void* x, const float* gamma, const float* beta,
                               float eps, void* u, hipStream_t s) {
  const c3c_conv_desc& d = g.d;
  const int64_t hw = d.H * d.W;
  if (d.N * d.Ci * d.T * hw == 0) return hipSuccess;
  const int64_t tiles = (hw + NPX - 1) / NPX;
  const int64_t blocks = d.N * d.T * tiles;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  const bool al = hw % 8 == 0 && aligned16(x) && aligned16(u);
  auto k = al ? pick_kernel<true>(d.Ci) : pick_kernel<false>(d.Ci);
  hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(x), gamma, beta, eps, static_cast<uint16_t*>(u),
                     d.Ci, d.T, hw, tiles);
  return hipGetLastError();
}

}  // namespace c3c
