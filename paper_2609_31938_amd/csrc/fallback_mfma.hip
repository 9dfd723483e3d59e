// Fallback route, bf16 / fp16: the generic direct Conv3D on matrix cores.
//
// The same sums as the direct kernel in fallback.hip (any kernel size,
// stride, dilation, groups, padding and frame range; fp32 accumulation, the
// bias added once, one rounding), as an implicit GEMM whose K dimension runs
// in the order in which w stores it:
//   K = (input channel of the group, kt, kh, kw),  Ktot = (Ci / groups) Kt Kh Kw,
// so that row co of w is a contiguous row of the B operand and needs neither
// a repack nor scratch memory (a fallback call has neither), and few input
// channels or many groups pad K to a multiple of 32 once, not once per tap.
//   D^T[px][co] = sum_K A[px][K] B[K][co], v_mfma_f32_16x16x32_{bf16,f16}:
// lane l supplies pixel l % 16 (A) or output channel l % 16 (B) at K = 8 (l /
// 16) .. + 7, and holds pixels 4 (l / 16) .. + 3 of output channel l % 16.
//
// Workgroup: 4 waves, BCO output channels of one group x 128 output pixels
// (8 fragments of 16 columns, 1, 2, 4 or 8 fragments side by side) of one
// (n, t) frame.  K is walked in chunks of kc (a multiple of 32).
//   * A chunk's input windows -- every channel it touches, each of the Kt
//     source frames, [rows][8-pixel segments] as NCTHW stores them -- go to
//     LDS once per chunk (zeros outside the image and for frames outside Z,
//     the fused prologue applied to the new chunk's), so an input element is
//     loaded once per tile, not once per tap, and in 16-byte pieces.
//   * The A operand is gathered from the windows: LDS byte offset = koff[K]
//     (channel, frame, kh, kw; a table built per chunk) + the pixel's own
//     offset (stride).  Eight 2-byte reads a lane serve WCO products.
//   * The B operand is read from w (L1 / L2) one 32-K stage ahead.
// What bounds it, measured on 192 -> 192, 1x3x3 at stride 2, 240x416, four
// frames, f16 (66 GFLOP): 0.159 ms (417 TFLOP/s; the direct kernel took
// 2.95 ms).  In the runs that took 0.150, 0.12 without the A gather (8 reads, 8 address adds and 4 packs a
// fragment), 0.13 without the staging, 0.14 without the weight reads.  The
// waves of the 192-channel tile sit side by side along the output channels,
// so no weight byte is read twice: as 2 x 2 waves (half the gather, each
// weight read by two waves) it took 0.181, 0.115 of it without the weight
// reads, whose 16 rows a fragment are 16 half-used lines.  Smaller tiles
// keep 2 x 2 or 1 x 4 waves (128 channels: 0.096 against 0.106 ms).  Two
// workgroups per compute unit (LDS at most 64 KiB) overlap one's staging
// with the other's products.
//
// Loads of 8 pixels whose address is not 16-byte aligned (AL = false: an odd
// width, an unaligned tensor) are dword-aligned 16 + 4 bytes, shifted into
// place (v_alignbit); a straddling dword at a plane's end stays within the
// dword that holds the plane's last element.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "c3c_internal.h"
#include "fuse_dev.h"

namespace c3c {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int FM_FRAGS = 8;         // pixel fragments (of 16 columns) per workgroup
constexpr int FM_ROUNDS = 4;        // 64-lane rounds of one staged plane: at most 256 segments
constexpr int FM_LDS = 64 * 1024;   // two workgroups per compute unit
constexpr int FM_KC_MAX = 1152;     // K per chunk

struct FmArgs {
  const uint16_t* x;
  const uint16_t* cache;
  const uint16_t* w;
  const uint16_t* bias;
  uint16_t* y;
  const float* scale;      // fused prologue (NULL: none)
  const float* shift;
  const uint16_t* residual;
  int64_t hw, hwo;
  int64_t st, dt, p_l, Z;
  int N, Ci, Co, T, Tc, H, W, Kt, Kw, KhKw;
  int sh, sw, dh, dw, ph, pw, To, Ho, Wo;
  int cig, cog, taps, Ktot;
  int kc, kc_aligned;      // K per chunk; 1: a multiple of taps (one table serves every chunk)
  int rows, segs, rowp, planep, rounds;
  int fc;                  // column fragments per tile (rows of pixels: FM_FRAGS / fc)
  int tiles_w, tiles_h, co_tiles, groups, nblocks;
  int has_bias, w_al;      // w_al: 16-byte reads of w are aligned
  uint32_t w_bytes;
};

template <bool F16>
__device__ inline f32x4 fm_mma(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c,
                                                  0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

template <bool F16>
__device__ inline float fm_widen(uint16_t v) {
  if constexpr (F16)
    return __half2float(__ushort_as_half(v));
  else
    return fuse_widen(v);
}

template <bool F16>
__device__ inline uint16_t fm_round(float v) {
  if constexpr (F16)
    return __half_as_ushort(__float2half_rn(v));
  else
    return static_cast<uint16_t>(
        __builtin_bit_cast(uint32_t, __builtin_convertvector((fuse_f32x2{v, 0.f}), fuse_bf16x2)));
}

// dword d of an 8-element run of which the first nv are kept: its bit mask
__device__ inline uint32_t fm_mask(int nv, int d) {
  return (nv > 2 * d ? 0xffffu : 0u) | (nv > 2 * d + 1 ? 0xffff0000u : 0u);
}

template <int WCO, int WPX, int WAVES_CO, int WAVES_PX, bool F16, bool AL>
__global__ __launch_bounds__(256, 2) void fallback_mfma(FmArgs a) {
  static_assert(WAVES_CO * WAVES_PX == 4 && WPX * WAVES_PX == FM_FRAGS, "4 waves tile the 8 pixel fragments");
  constexpr int BCO = 16 * WCO * WAVES_CO;
  // segments a lane loads at a time while staging (4 where 8 would spill)
  constexpr int FLY = WCO * WPX >= 24 && !(F16 && AL) ? 4 : 8;
  constexpr uint32_t OOB = 0x80000000u;  // beyond every resource's size
  extern __shared__ __align__(16) unsigned char fm_lds[];
  int* const koff = reinterpret_cast<int*>(fm_lds);
  unsigned char* const tile = fm_lds + a.kc * 4;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wco = wave % WAVES_CO, wpx = wave / WAVES_CO;
  const int j = lane & 15, g4 = lane >> 4;

  // workgroup -> tile, XCD-contiguous; the output-channel tiles of one pixel
  // tile are neighbours (they stage the same windows)
  int L;
  {
    const int b = blockIdx.x, per = a.nblocks / 8, rem = a.nblocks % 8;
    const int xcd = b % 8, slot = b / 8;
    L = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + slot;
  }
  const int ct = L % a.co_tiles;
  L /= a.co_tiles;
  const int g = L % a.groups;
  L /= a.groups;
  const int tw = L % a.tiles_w;
  L /= a.tiles_w;
  const int th = L % a.tiles_h;
  L /= a.tiles_h;
  const int t = L % a.To, n = L / a.To;
  const int fr = FM_FRAGS / a.fc;
  const int h0 = th * fr, w0 = tw * 16 * a.fc;
  const int co_end = (g + 1) * a.cog;
  const int co_w = g * a.cog + ct * BCO + wco * 16 * WCO;  // this wave's first output channel

  // window origin: the column of the first pixel's first tap, rounded down to
  // a multiple of 8 so that a segment lies wholly left of the image or not
  const int cx = w0 * a.sw - a.pw;
  const int x0 = (cx >> 3) * 8, cadj = cx - x0;
  const int hy = h0 * a.sh - a.ph;

  // this lane's segments of a staged plane
  int le[FM_ROUNDS], lo[FM_ROUNDS], nv[FM_ROUNDS];
#pragma unroll
  for (int r = 0; r < FM_ROUNDS; ++r) {
    const int lt = lane + 64 * r;
    const int row = lt / a.segs, seg = lt - row * a.segs;
    const int gh = hy + row, gw = x0 + 8 * seg;
    const bool in = lt < a.rows * a.segs;
    const bool ok = in && gh >= 0 && gh < a.H && gw >= 0 && gw < a.W;
    le[r] = ok ? gh * a.W + gw : 0;
    nv[r] = ok ? min(a.W - gw, 8) : 0;
    lo[r] = in ? row * a.rowp + seg * 16 : -1;
  }

  // LDS offset of this lane's pixel of each of the wave's fragments
  int poff[WPX];
#pragma unroll
  for (int pf = 0; pf < WPX; ++pf) {
    const int q = wpx * WPX + pf;
    const int row = q / a.fc, cfr = q - row * a.fc;
    poff[pf] = row * a.sh * a.rowp + (cadj + (16 * cfr + j) * a.sw) * 2;
  }

  // weights: row co of w at K = 8 g4 .. + 7 of a stage; output channels past
  // the group's last are clamped (they feed columns that are never stored)
  const uint32_t wpb = static_cast<uint32_t>((reinterpret_cast<uintptr_t>(a.w) >> 1) & 1u);
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(a.w - wpb), 0, static_cast<int>((a.w_bytes + 2 * wpb + 3) & ~3u), 0x00020000);
  uint32_t wrow[WCO];  // element index of this lane's first K in row co
#pragma unroll
  for (int cf = 0; cf < WCO; ++cf)
    wrow[cf] = static_cast<uint32_t>(min(co_w + 16 * cf + j, co_end - 1)) * static_cast<uint32_t>(a.Ktot) +
               static_cast<uint32_t>(8 * g4) + wpb;
  // A load of 8 weights per row at K = k0 + 8 g4 .. ; past the row's end
  // (the stage after the last one) zeros.  WAL: 16-byte aligned rows, else
  // dword-aligned loads shifted into place.
  auto load_w = [&](auto wal, int k0, u32x4 (&dst)[WCO]) __attribute__((always_inline)) {
    const bool live = k0 + 8 * g4 < a.Ktot;
#pragma unroll
    for (int cf = 0; cf < WCO; ++cf) {
      const uint32_t e = wrow[cf] + static_cast<uint32_t>(k0);
      if constexpr (decltype(wal)::value) {
        dst[cf] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrs, live ? 2u * e : OOB, 0, 0));
      } else {
        const uint32_t off = live ? (2u * e) & ~3u : OOB;
        const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrs, off, 0, 0));
        const uint32_t v4 = __builtin_amdgcn_raw_buffer_load_b32(wrs, off, 16, 0);
        const uint32_t s = (e & 1u) * 16u;
        dst[cf] = u32x4{__builtin_amdgcn_alignbit(v[1], v[0], s), __builtin_amdgcn_alignbit(v[2], v[1], s),
                        __builtin_amdgcn_alignbit(v[3], v[2], s), __builtin_amdgcn_alignbit(v4, v[3], s)};
      }
    }
  };

  // stage the windows of channels [c_lo, c_lo + nch) of the group into LDS:
  // a wave takes every fourth (channel, frame) plane, FLY / R at a time (R: the
  // lane rounds of one plane), so FLY loads a lane are in flight
  auto stage = [&](auto rounds, int c_lo, int nch) __attribute__((always_inline)) {
    constexpr int R = decltype(rounds)::value, U = FLY / R;
    const int planes = nch * a.Kt;
    for (int p0 = wave; p0 < planes; p0 += 4 * U) {
      u32x4 v[U][R];
      uint32_t v4[U][R], par[U];
      bool pro[U];
      int64_t nc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + 4 * u;
        const int cl = p / a.Kt, kt = p - cl * a.Kt;
        const int64_t f = t * a.st + kt * a.dt - a.p_l;  // Eq. 1 source frame in Z
        const bool live = p < planes && f >= 0 && f < a.Z;
        const bool in_cache = f < a.Tc;
        pro[u] = a.scale != nullptr && live && !in_cache;
        nc[u] = static_cast<int64_t>(n) * a.Ci + g * a.cig + c_lo + cl;
        const uint16_t* src =
            live ? (in_cache ? a.cache + (nc[u] * a.Tc + f) * a.hw : a.x + (nc[u] * a.T + (f - a.Tc)) * a.hw) : a.w;
        par[u] = AL ? 0u : static_cast<uint32_t>((reinterpret_cast<uintptr_t>(src) >> 1) & 1u);
        const uint32_t bytes = live ? (static_cast<uint32_t>(a.hw) * 2u + 2u * par[u] + 3u) & ~3u : 0u;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(src - par[u]), 0, static_cast<int>(bytes), 0x00020000);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const uint32_t e = static_cast<uint32_t>(le[r]) + par[u];
          const uint32_t off = nv[r] > 0 ? (AL ? 2u * e : (2u * e) & ~3u) : OOB;
          v[u][r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
          if (!AL) v4[u][r] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 16, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + 4 * u;
        if (p >= planes) continue;
        float psc = 0.f, psh = 0.f;
        if (!F16 && pro[u]) {
          psc = a.scale[nc[u]];
          psh = a.shift[nc[u]];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          u32x4 o = v[u][r];
          if (!AL) {
            const uint32_t s = ((static_cast<uint32_t>(le[r]) + par[u]) & 1u) * 16u;
            o = u32x4{__builtin_amdgcn_alignbit(o[1], o[0], s), __builtin_amdgcn_alignbit(o[2], o[1], s),
                      __builtin_amdgcn_alignbit(o[3], o[2], s), __builtin_amdgcn_alignbit(v4[u][r], o[3], s)};
          }
          if (!F16 && pro[u]) o = fuse_seg8(o, psc, psh, true);
          if (!AL || (!F16 && pro[u]))  // positions outside the image stay zero
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] &= fm_mask(nv[r], d);
          if (lo[r] >= 0) *reinterpret_cast<u32x4*>(tile + p * a.planep + lo[r]) = o;
        }
      }
    }
  };

  f32x4 acc[WCO][WPX];
#pragma unroll
  for (int cf = 0; cf < WCO; ++cf)
#pragma unroll
    for (int pf = 0; pf < WPX; ++pf) acc[cf][pf] = f32x4{0.f, 0.f, 0.f, 0.f};

  // One chunk of K: its table and windows, then its 32-K stages.  Fragment pf
  // + 1's eight elements are read from LDS before fragment pf's products, the
  // first fragment of the next stage before the last one's.
  auto gather = [&](const int (&ko)[8], int pf, uint32_t (&h)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = *reinterpret_cast<const uint16_t*>(fm_lds + ko[e] + poff[pf]);
  };
  auto offsets = [&](int kl, int (&ko)[8]) __attribute__((always_inline)) {
    const int4 lo4 = *reinterpret_cast<const int4*>(koff + kl + 8 * g4);
    const int4 hi4 = *reinterpret_cast<const int4*>(koff + kl + 8 * g4 + 4);
    ko[0] = lo4.x; ko[1] = lo4.y; ko[2] = lo4.z; ko[3] = lo4.w;
    ko[4] = hi4.x; ko[5] = hi4.y; ko[6] = hi4.z; ko[7] = hi4.w;
  };
  auto products = [&](const uint32_t (&h)[8], int pf, const u32x4 (&w)[WCO]) __attribute__((always_inline)) {
    u32x4 av;
#pragma unroll
    for (int d = 0; d < 4; ++d) av[d] = h[2 * d] | (h[2 * d + 1] << 16);
#pragma unroll
    for (int cf = 0; cf < WCO; ++cf) acc[cf][pf] = fm_mma<F16>(av, w[cf], acc[cf][pf]);
  };
  auto run = [&](auto wal) __attribute__((always_inline)) {
    u32x4 wr[WCO], wn[WCO];
    load_w(wal, 0, wr);
    for (int kb = 0; kb < a.Ktot; kb += a.kc) {
      const int kend = min(kb + a.kc, a.Ktot);
      const int c_lo = kb / a.taps, nch = (kend - 1) / a.taps - c_lo + 1;
      if (kb > 0) __syncthreads();  // the previous chunk's reads are done
      if (kb == 0 || !a.kc_aligned)
        for (int q = tid; q < a.kc; q += 256) {
          const int k = kb + q;
          int v = a.kc * 4;
          if (k < a.Ktot) {
            const int ci = k / a.taps, tap = k - ci * a.taps;
            const int kt = tap / a.KhKw, rem = tap - kt * a.KhKw;
            const int kh = rem / a.Kw, kw = rem - kh * a.Kw;
            v += ((ci - c_lo) * a.Kt + kt) * a.planep + kh * a.dh * a.rowp + kw * a.dw * 2;
          }
          koff[q] = v;
        }
      if (a.rounds == 1) stage(std::integral_constant<int, 1>{}, c_lo, nch);
      else if (a.rounds == 2) stage(std::integral_constant<int, 2>{}, c_lo, nch);
      else stage(std::integral_constant<int, 4>{}, c_lo, nch);
      __syncthreads();
      const int full = (kend - kb) / 32;  // stages wholly inside the chunk (and Ktot)
      int ko[8];
      uint32_t h[2][8];
      offsets(0, ko);
      gather(ko, 0, h[0]);
      for (int s = 0; s < full; ++s) {
        load_w(wal, kb + 32 * (s + 1), wn);
        int kn[8];
        // the chunk's last stage reads its own offsets again (never past the table)
        offsets(min(32 * (s + 1), a.kc - 32), kn);
#pragma unroll
        for (int pf = 0; pf < WPX; ++pf) {
          if (pf + 1 < WPX) gather(ko, pf + 1, h[(pf + 1) & 1]);
          else gather(kn, 0, h[(pf + 1) & 1]);
          products(h[pf & 1], pf, wr);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) ko[e] = kn[e];
#pragma unroll
        for (int cf = 0; cf < WCO; ++cf) wr[cf] = wn[cf];
      }
      if (kb + 32 * full < kend) {
        // Ktot's last, partial stage: K past Ktot is the next row of w and
        // the table's stand-in offset 0, both masked to zero
        const int left = a.Ktot - (kb + 32 * full) - 8 * g4;
        offsets(32 * full, ko);
#pragma unroll
        for (int cf = 0; cf < WCO; ++cf)
#pragma unroll
          for (int d = 0; d < 4; ++d) wr[cf][d] &= fm_mask(left, d);
#pragma unroll
        for (int pf = 0; pf < WPX; ++pf) {
          gather(ko, pf, h[0]);
#pragma unroll
          for (int e = 0; e < 8; ++e) h[0][e] = e < left ? h[0][e] : 0u;
          products(h[0], pf, wr);
        }
      }
    }
  };
  if (a.w_al) run(std::true_type{});
  else run(std::false_type{});

  // epilogue: bias once, the residual, one rounding, NCTHW store
#pragma unroll
  for (int cf = 0; cf < WCO; ++cf) {
    const int co = co_w + 16 * cf + j;
    if (co >= co_end) continue;
    const float bb = a.has_bias ? fm_widen<F16>(a.bias[co]) : 0.f;
    const int64_t row0 = ((static_cast<int64_t>(n) * a.Co + co) * a.To + t) * a.hwo;
#pragma unroll
    for (int pf = 0; pf < WPX; ++pf) {
      const int q = wpx * WPX + pf;
      const int row = q / a.fc, cfr = q - row * a.fc;
      const int oh = h0 + row, ow = w0 + 16 * cfr + 4 * g4;
      if (oh >= a.Ho || ow >= a.Wo) continue;
      const int64_t at = row0 + static_cast<int64_t>(oh) * a.Wo + ow;
      const int m = min(a.Wo - ow, 4);
      float rr[4] = {0.f, 0.f, 0.f, 0.f};
      if (!F16 && a.residual)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r < m) rr[r] = fuse_widen(a.residual[at + r]);
      uint16_t v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = fm_round<F16>(acc[cf][pf][r] + bb + rr[r]);
      if (m == 4) {
        // one 8-byte store at any 2-byte alignment
        const uint2 o = make_uint2(v[0] | (static_cast<uint32_t>(v[1]) << 16), v[2] | (static_cast<uint32_t>(v[3]) << 16));
        __builtin_memcpy(a.y + at, &o, 8);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r < m) a.y[at + r] = v[r];
      }
    }
  }
}

constexpr int FM_CFGS = 6;
constexpr int FM_BCO[FM_CFGS] = {192, 128, 96, 64, 32, 16};

// Whether the direct kernel takes less time than blocks workgroups of the
// 16-channel tile (the wider ones always win).  With few products an output
// (a depthwise or thinly grouped call) a workgroup here does a 16 x 32 product
// for a few useful ones and its time is its fixed cost, 1.49 us of a compute
// unit for 128 pixels (0.42 more where planes are not aligned, 0.07 a staged
// source plane).  A direct one costs 1.88 us for 512 pixels, 0.18 a product,
// 0.26 a source plane and 0.135 an output channel, and 3.6 + 0.6 us a product
// from start to end, a fifth of which a full device still shows.  Fitted to
// 2489 calls, 591 of which go to the direct kernel; on 35 the faster kernel is
// more than 6% ahead of the one taken (1.25 at most).  Depthwise 1x3x3, 272
// channels at 97x117, two frames: 89 us direct, 187 here; 1x5x5, 280 channels
// at 23x44, four frames: 66 direct, 87 here; 3x3x3 at stride 2, 512 channels at
// 151x328, four frames: 1690 direct, 1270 here.
bool direct_pays(const Geo& g, int64_t Ktot, int64_t blocks, bool al) {
  const c3c_conv_desc& d = g.d;
  const int64_t cig = d.Ci / d.groups, cog = d.Co / d.groups;
  const int64_t gy = d.groups * ((cog + kFallbackDirectCo - 1) / kFallbackDirectCo);
  if (gy > 65535) return false;  // past the direct kernel's grid
  const int64_t nb = gy * ((g.Ho * g.Wo + kFallbackDirectPx - 1) / kFallbackDirectPx) * g.To * d.N;
  const double cus = static_cast<double>(device_compute_units()), k = static_cast<double>(Ktot);
  const double planes = static_cast<double>(cig * d.Kt);
  const double here = static_cast<double>(blocks) / cus * ((al ? 1.49 : 1.91) + 0.07 * planes);
  const double chain = 3.6 + 0.6 * k;
  const double direct = 0.22 * chain + static_cast<double>(nb) / cus *
                        (1.88 + 0.18 * k + 0.26 * planes + 0.135 * static_cast<double>(cog));
  return here > chain && here > direct;
}

// The tile of a call: output-channel configuration (index into the list
// above), columns of pixel fragments, K per chunk.  False: the windows of a
// 128-pixel tile do not fit LDS or the lane rounds (large strides, dilations
// or kernels), a size passes the kernel's 32-bit arithmetic, or the products
// are too few: the direct kernel takes the call.  al: planes aligned for
// 16-byte loads.
bool pick(const Geo& g, bool al, FmArgs* a, int* cfg) {
  const c3c_conv_desc& d = g.d;
  const int64_t lim = int64_t(1) << 29;
  for (int64_t v : {d.N, d.Ci, d.Co, d.T, d.Tc, d.H, d.W, g.To, g.Ho, g.Wo})
    if (v >= lim) return false;
  for (int64_t v : {d.stride_h, d.stride_w, d.dil_h, d.dil_w, d.pad_h, d.pad_w})
    if (v > 1024) return false;
  if (d.N * g.To > 65535) return false;  // the fallback's documented limit (the direct kernel's grid)
  const int64_t taps = d.Kt * d.Kh * d.Kw;
  if (d.Kt > 1024 || d.Kh > 1024 || d.Kw > 1024 || taps > 65536) return false;
  const int64_t cig = d.Ci / d.groups, cog = d.Co / d.groups;
  const int64_t Ktot = cig * taps;
  if (Ktot >= (1 << 28) || d.Co * Ktot * 2 >= 0x7ffffff0 || d.H * d.W * 2 >= 0x7ffffff0) return false;

  // pixel tile: the fewest tiles, then the smallest window
  int64_t best_tiles = -1, best_win = 0;
  for (int fc : {1, 2, 4, 8}) {
    const int64_t fr = FM_FRAGS / fc, bw = 16 * fc;
    const int64_t rows = (fr - 1) * d.stride_h + (d.Kh - 1) * d.dil_h + 1;
    // columns from a segment's start to the first pixel's first tap: the same
    // for every tile, whose origin is a multiple of 16 columns
    const int64_t adj = (8 - d.pad_w % 8) % 8;
    const int64_t segs = (adj + (bw - 1) * d.stride_w + (d.Kw - 1) * d.dil_w + 1 + 7) / 8;
    if (rows * segs > 64 * FM_ROUNDS) continue;
    const int64_t plane = rows * segs * 16;
    const int64_t ch32 = (32 + taps - 2) / taps + 1 < cig ? (32 + taps - 2) / taps + 1 : cig;
    if (32 * 4 + ch32 * d.Kt * plane > FM_LDS) continue;
    const int64_t tiles = ((g.Ho + fr - 1) / fr) * ((g.Wo + bw - 1) / bw);
    if (best_tiles < 0 || tiles < best_tiles || (tiles == best_tiles && rows * segs < best_win)) {
      best_tiles = tiles;
      best_win = rows * segs;
      a->fc = fc;
      a->rows = static_cast<int>(rows);
      a->segs = static_cast<int>(segs);
      a->tiles_h = static_cast<int>((g.Ho + fr - 1) / fr);
      a->tiles_w = static_cast<int>((g.Wo + bw - 1) / bw);
    }
  }
  if (best_tiles < 0) return false;
  a->rowp = a->segs * 16;
  a->planep = a->rows * a->rowp;
  a->rounds = (a->rows * a->segs + 63) / 64;

  // K per chunk: the largest whose windows and table fit, or a multiple of
  // taps at least half as large (its channels do not straddle chunks)
  auto fits = [&](int64_t kc) {
    int64_t nch = kc % taps == 0 ? kc / taps : (kc + taps - 2) / taps + 1;
    if (nch > cig) nch = cig;
    return kc * 4 + nch * d.Kt * a->planep <= FM_LDS;
  };
  const int64_t kmax = (Ktot + 31) / 32 * 32 < FM_KC_MAX ? (Ktot + 31) / 32 * 32 : FM_KC_MAX;
  int64_t any = 0, whole = 0;
  for (int64_t kc = kmax; kc >= 32; kc -= 32) {
    if (!fits(kc)) continue;
    if (any == 0) any = kc;
    if (whole == 0 && kc % taps == 0) whole = kc;
  }
  if (any == 0) return false;
  const int64_t kc = 2 * whole >= any ? whole : any;
  a->kc = static_cast<int>(kc);
  a->kc_aligned = kc % taps == 0 || kc >= Ktot;

  // output channels per workgroup: a workgroup's time goes as its channels
  // plus the gather's and the staging's share, about 160 channels' worth
  // (measured, 3x3 at stride 2: 128 -> 128 from 240x416, 0.096 ms on 128-,
  // 0.115 on 192-, 0.161 on 64-channel tiles; 96 -> 96 from 480x832, 0.19 on
  // 96-, 0.22 on 128-channel tiles); up to two per compute unit run at once
  const double cus = static_cast<double>(device_compute_units());
  double best = -1;
  int64_t blocks = 0;
  for (int i = 0; i < FM_CFGS; ++i) {
    const int64_t ct = (cog + FM_BCO[i] - 1) / FM_BCO[i];
    const int64_t nb = ct * d.groups * best_tiles * g.To * d.N;
    const double rounds = static_cast<double>(nb) / (2.0 * cus);
    const double cost = (rounds > 1.0 ? rounds : 1.0) * (FM_BCO[i] + 160);
    if (best < 0 || cost < best) {
      best = cost;
      *cfg = i;
      a->co_tiles = static_cast<int>(ct);
      blocks = nb;
    }
  }
  if (blocks > 0x7fffffff || (FM_BCO[*cfg] == 16 && direct_pays(g, Ktot, blocks, al))) return false;
  a->nblocks = static_cast<int>(blocks);
  a->groups = static_cast<int>(d.groups);
  a->cig = static_cast<int>(cig);
  a->cog = static_cast<int>(cog);
  a->taps = static_cast<int>(taps);
  a->Ktot = static_cast<int>(Ktot);
  return true;
}

template <bool F16, bool AL>
void launch_cfg(int cfg, const FmArgs& a, size_t lds, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.nblocks)), block(256);
  switch (cfg) {
    case 0: hipLaunchKernelGGL((fallback_mfma<3, 8, 4, 1, F16, AL>), grid, block, lds, s, a); break;
    case 1: hipLaunchKernelGGL((fallback_mfma<4, 4, 2, 2, F16, AL>), grid, block, lds, s, a); break;
    case 2: hipLaunchKernelGGL((fallback_mfma<3, 4, 2, 2, F16, AL>), grid, block, lds, s, a); break;
    case 3: hipLaunchKernelGGL((fallback_mfma<4, 2, 1, 4, F16, AL>), grid, block, lds, s, a); break;
    case 4: hipLaunchKernelGGL((fallback_mfma<2, 2, 1, 4, F16, AL>), grid, block, lds, s, a); break;
    default: hipLaunchKernelGGL((fallback_mfma<1, 2, 1, 4, F16, AL>), grid, block, lds, s, a); break;
  }
}

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

bool launch_fallback_mfma(const Geo& g, const void* x, const void* cache, const void* w, const void* bias,
                          void* y, hipStream_t s, const Fuse& fu, LaunchInfo* info, hipError_t* err) {
  const c3c_conv_desc& d = g.d;
  FmArgs a{};
  int cfg = 0;
  *err = hipSuccess;
  const bool al = d.W % 8 == 0 && al16(x) && (cache == nullptr || al16(cache));
  if (g.To < 1 || !pick(g, al, &a, &cfg)) return false;
  if (info) {
    info->kernel = C3C_KERNEL_FALLBACK_DIRECT;
    info->tile_co = FM_BCO[cfg];
    info->tile_h = FM_FRAGS / a.fc;
    info->tile_w = 16 * a.fc;
    info->workgroups = a.nblocks;
    return true;
  }
  a.x = static_cast<const uint16_t*>(x);
  a.cache = static_cast<const uint16_t*>(cache);
  a.w = static_cast<const uint16_t*>(w);
  a.bias = static_cast<const uint16_t*>(bias);
  a.y = static_cast<uint16_t*>(y);
  a.scale = fu.scale;
  a.shift = fu.shift;
  a.residual = fu.residual;
  a.hw = d.H * d.W;
  a.hwo = g.Ho * g.Wo;
  a.st = d.stride_t; a.dt = d.dil_t; a.p_l = g.p_l; a.Z = g.Z;
  a.N = static_cast<int>(d.N); a.Ci = static_cast<int>(d.Ci); a.Co = static_cast<int>(d.Co);
  a.T = static_cast<int>(d.T); a.Tc = static_cast<int>(d.Tc);
  a.H = static_cast<int>(d.H); a.W = static_cast<int>(d.W);
  a.Kt = static_cast<int>(d.Kt); a.Kw = static_cast<int>(d.Kw); a.KhKw = static_cast<int>(d.Kh * d.Kw);
  a.sh = static_cast<int>(d.stride_h); a.sw = static_cast<int>(d.stride_w);
  a.dh = static_cast<int>(d.dil_h); a.dw = static_cast<int>(d.dil_w);
  a.ph = static_cast<int>(d.pad_h); a.pw = static_cast<int>(d.pad_w);
  a.To = static_cast<int>(g.To); a.Ho = static_cast<int>(g.Ho); a.Wo = static_cast<int>(g.Wo);
  a.has_bias = d.has_bias ? 1 : 0;
  a.w_bytes = static_cast<uint32_t>(d.Co * a.Ktot * 2);
  a.w_al = al16(w) && a.Ktot % 8 == 0;
  int64_t nch = a.kc % a.taps == 0 ? a.kc / a.taps : (a.kc + a.taps - 2) / a.taps + 1;
  if (nch > a.cig) nch = a.cig;
  const size_t lds = static_cast<size_t>(a.kc) * 4 + static_cast<size_t>(nch) * d.Kt * a.planep;
  const bool f16 = d.dtype == C3C_DTYPE_F16;
  if (f16) {
    if (al) launch_cfg<true, true>(cfg, a, lds, s);
    else launch_cfg<true, false>(cfg, a, lds, s);
  } else {
    if (al) launch_cfg<false, true>(cfg, a, lds, s);
    else launch_cfg<false, false>(cfg, a, lds, s);
  }
  *err = hipGetLastError();
  return true;
}

}  // namespace c3c
