// Fast route, shared parts: the packed-weight layout and its repack / unpack
// kernels, and the dispatch of one fast call to the kernels of conv_bf16.hip,
// conv_head.hip, conv_tap1x1.hip, pointwise.hip and conv_f32.hip.
#include "c3c_internal.h"

namespace c3c {

PackDims pack_dims(const c3c_conv_desc& d) {
  PackDims p;
  const bool f32 = d.dtype == C3C_DTYPE_F32;
  p.rows = f32 ? 32 : 16;
  p.kpl = f32 ? 1 : 8;
  p.kstep = (64 / p.rows) * p.kpl;
  p.taps = d.Kt * d.Kh * d.Kw;
  p.chunks = (d.Ci + p.kstep - 1) / p.kstep;
  p.cofrags = (d.Co + p.rows - 1) / p.rows;
  return p;
}

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- repack
// packed index (tap, chunk, cofrag, lane, e) <-> w[co][ci][tap]
template <typename T>
__global__ __launch_bounds__(256) void repack_kernel(const T* __restrict__ w, T* __restrict__ wp,
                                                     int64_t total, int64_t Ci, int64_t Co,
                                                     int64_t taps, int64_t chunks,
                                                     int64_t cofrags, int rows, int kpl) {
  const int kstep = (64 / rows) * kpl;
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; idx < total;
       idx += static_cast<int64_t>(gridDim.x) * 256) {
    int64_t r = idx;
    const int e = static_cast<int>(r % kpl);
    r /= kpl;
    const int lane = static_cast<int>(r % 64);
    r /= 64;
    const int64_t cf = r % cofrags;
    r /= cofrags;
    const int64_t ch = r % chunks;
    const int64_t tap = r / chunks;
    const int64_t co = cf * rows + lane % rows;
    const int64_t ci = ch * kstep + (lane / rows) * kpl + e;
    T v = T(0);
    if (co < Co && ci < Ci) v = w[(co * Ci + ci) * taps + tap];
    wp[idx] = v;
  }
}

// 16-bit weights, fragment geometry rows = 16, kpl = 8 (32 input channels
// per chunk): one workgroup per (chunk, output fragment) block.  The block's
// 16 output channels x 32 input channels x all taps are contiguous runs of
// w (32 * taps elements per output channel), read coalesced into LDS; each
// thread then writes whole 16-byte lane slots (8 consecutive input channels
// of one output channel at one tap) of the block's fragments, one 1 KiB
// fragment per 64 threads.  Channels past Ci / Co are zeros.  vec: w is
// 16-byte aligned and Ci * taps a multiple of 8, so a full chunk's runs are
// read as 16-byte pieces (the tail chunk, and other calls, element by
// element).
constexpr int kRepackMaxTaps = 48;
__global__ __launch_bounds__(256) void repack_block16(const uint16_t* __restrict__ w,
                                                      u32x4* __restrict__ wp, int64_t Ci,
                                                      int64_t Co, int taps, int64_t chunks,
                                                      int64_t cofrags, int vec) {
  __shared__ __align__(16) uint16_t tile[16 * 32 * kRepackMaxTaps];
  const int64_t cf = blockIdx.x % cofrags, ch = blockIdx.x / cofrags;
  const int row = 32 * taps;  // elements of one output channel's run
  const int64_t ci0 = ch * 32;
  const int64_t ci_n = Ci - ci0 < 32 ? Ci - ci0 : 32;  // real input channels of the chunk
  if (vec && ci_n == 32) {
    const int nv = row / 8;  // 16-byte pieces of a run
    for (int q = threadIdx.x; q < 16 * nv; q += 256) {
      const int r = q / nv, u = q - r * nv;
      const int64_t co = cf * 16 + r;
      *reinterpret_cast<u32x4*>(tile + r * row + 8 * u) =
          co < Co ? *reinterpret_cast<const u32x4*>(w + (co * Ci + ci0) * taps + 8 * u) : u32x4{0u, 0u, 0u, 0u};
    }
  } else {
    for (int q = threadIdx.x; q < 16 * row; q += 256) {
      const int r = q / row, u = q - r * row;
      const int64_t co = cf * 16 + r;
      const bool ok = co < Co && u < ci_n * taps;
      tile[q] = ok ? w[(co * Ci + ci0) * taps + u] : static_cast<uint16_t>(0);
    }
  }
  __syncthreads();
  // thread -> (tap t, lane L): lane L holds output channel L % 16, input
  // channels 8 (L / 16) .. + 7
  for (int q = threadIdx.x; q < taps * 64; q += 256) {
    const int t = q >> 6, L = q & 63;
    const int base = ((L & 15) * 32 + 8 * (L >> 4)) * taps + t;
    uint32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = static_cast<uint32_t>(tile[base + (2 * e) * taps]) |
             (static_cast<uint32_t>(tile[base + (2 * e + 1) * taps]) << 16);
    wp[((t * chunks + ch) * cofrags + cf) * 64 + L] = u32x4{v[0], v[1], v[2], v[3]};
  }
}

template <typename T>
__global__ __launch_bounds__(256) void unpack_kernel(const T* __restrict__ wp, T* __restrict__ w,
                                                     int64_t total, int64_t Ci, int64_t taps,
                                                     int64_t chunks, int64_t cofrags, int rows,
                                                     int kpl) {
  const int64_t kstep = (64 / rows) * kpl;
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; idx < total;
       idx += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t tap = idx % taps;
    const int64_t ci = (idx / taps) % Ci;
    const int64_t co = idx / (taps * Ci);
    const int64_t ch = ci / kstep, rem = ci % kstep;
    const int64_t lane = co % rows + rows * (rem / kpl);
    const int64_t e = rem % kpl;
    const int64_t cf = co / rows;
    w[idx] = wp[((((tap * chunks + ch) * cofrags + cf) * 64 + lane) * kpl) + e];
  }
}

}  // namespace

hipError_t launch_repack(const Geo& g, const void* w, void* wpack, hipStream_t s) {
  const PackDims p = pack_dims(g.d);
  const int64_t total = p.elems();
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (g.d.dtype == C3C_DTYPE_F32)
    hipLaunchKernelGGL(repack_kernel<float>, dim3(blocks), dim3(256), 0, s,
                       static_cast<const float*>(w), static_cast<float*>(wpack), total, g.d.Ci,
                       g.d.Co, p.taps, p.chunks, p.cofrags, p.rows, p.kpl);
  else if (p.rows == 16 && p.kpl == 8 && p.taps <= kRepackMaxTaps &&
           p.chunks * p.cofrags <= 0x7fffffff && (reinterpret_cast<uintptr_t>(wpack) & 15u) == 0)
    hipLaunchKernelGGL(repack_block16, dim3(static_cast<unsigned>(p.chunks * p.cofrags)), dim3(256),
                       0, s, static_cast<const uint16_t*>(w), static_cast<u32x4*>(wpack), g.d.Ci,
                       g.d.Co, static_cast<int>(p.taps), p.chunks, p.cofrags,
                       ((reinterpret_cast<uintptr_t>(w) & 15u) == 0 && (g.d.Ci * p.taps) % 8 == 0) ? 1 : 0);
  else
    hipLaunchKernelGGL(repack_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s,
                       static_cast<const uint16_t*>(w), static_cast<uint16_t*>(wpack), total,
                       g.d.Ci, g.d.Co, p.taps, p.chunks, p.cofrags, p.rows, p.kpl);
  return hipGetLastError();
}

hipError_t launch_unpack(const Geo& g, const void* wpack, void* w, hipStream_t s) {
  const PackDims p = pack_dims(g.d);
  const int64_t total = g.d.Co * g.d.Ci * p.taps;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (g.d.dtype == C3C_DTYPE_F32)
    hipLaunchKernelGGL(unpack_kernel<float>, dim3(blocks), dim3(256), 0, s,
                       static_cast<const float*>(wpack), static_cast<float*>(w), total, g.d.Ci,
                       p.taps, p.chunks, p.cofrags, p.rows, p.kpl);
  else
    hipLaunchKernelGGL(unpack_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s,
                       static_cast<const uint16_t*>(wpack), static_cast<uint16_t*>(w), total,
                       g.d.Ci, p.taps, p.chunks, p.cofrags, p.rows, p.kpl);
  return hipGetLastError();
}

hipError_t launch_fast(const Geo& g, const void* x, const void* cache, const void* wpack,
                       const void* bias, void* y, void* cache_out, void* ws, int64_t ws_bytes,
                       hipStream_t s, const Fuse& fu, LaunchInfo* info) {
  // the fast route's two spatial forms: 3x3 / stride 1 / pad 1, and 1x1
  const bool one = g.d.Kh == 1;
  hipError_t e;
  if (g.d.dtype == C3C_DTYPE_BF16) {
    if (one) {
      // Two kernels: the 4-wave 192 x 128 kernel (1.2-1.5x the pointwise
      // kernel at Co = 768 and 384) unless its padded output
      // channels exceed the 160-channel pointwise tile's by more than 10%
      // (Co = 96, 160, 256, 320 stay on the pointwise kernel) or its tiles
      // leave half the compute units idle.  The fused form (prologue /
      // residual) is in the pointwise kernel only.
      const int64_t pad_tap = (g.d.Co + kTap1x1TileCo - 1) / kTap1x1TileCo * kTap1x1TileCo;
      const int64_t pad_pw = (g.d.Co + kPointwiseTileCo - 1) / kPointwiseTileCo * kPointwiseTileCo;
      if (!fu.any() && 10 * pad_tap <= 11 * pad_pw && tap1x1_eligible(g) &&
          2 * tap1x1_blocks(g) >= device_compute_units()) {
        bool written = false;
        e = launch_tap1x1(g, x, cache, wpack, bias, y, cache_out, &written, s, info);
        if (e != hipSuccess || written || info) return e;
      } else
        e = launch_fast_tap1x1(g, x, cache, wpack, bias, y, s, fu, info);
    } else if (!fu.any() && head_eligible(g, x, cache, y)) {
      // few output channels (a decoder's RGB head): the spatial taps as N
      bool written = false;
      e = launch_head(g, x, cache, wpack, bias, y, cache_out, &written, s, info);
      if (e != hipSuccess || written || info) return e;
    } else {
      bool written = false;
      e = launch_fast_bf16(g, x, cache, wpack, bias, y, cache_out, ws, ws_bytes, &written, s, fu,
                           info);
      if (e != hipSuccess || written || info) return e;
    }
  } else {
    bool written = false;
    e = launch_fast_f32(g, x, cache, wpack, bias, y, cache_out, &written, s, info);
    if (e != hipSuccess || written || info) return e;
  }
  if (e != hipSuccess || info) return e;
  return launch_cache_copy(g, x, cache, cache_out, s, fu);
}

}  // namespace c3c
