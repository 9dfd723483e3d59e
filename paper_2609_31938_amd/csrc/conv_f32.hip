// fp32 fast route: the cache-aware lowering of one cached causal Conv3D call
// (paper Sec. 4, Eq. 2 and Eq. 4, Alg. 1) as one implicit-GEMM kernel on
// gfx950 fp32 matrix cores, with the bias and the cache update fused in.
//
// GEMM view per output frame: D[co][px] = sum_K W[co][K] Z[K][px], K = (tap,
// input channel), v_mfma_f32_32x32x2_f32: lane l supplies output channel l %
// 32 (weights, packed in this fragment order) or pixel l % 32 (activations)
// of input channel l / 32 of a pair, and holds pixel l % 32 of 16 output
// channels.  Source frame of tap k for output frame o: o s_t + k d_t - p_l
// (s_t is 1 for the 3x3 form).
//
// Workgroup: 32 output channels x 32 PXW pixels (128, or 32 for small frames)
// of one output frame, a BH x BW block whose shape the host picks for the
// frame (any BW: a pixel's place in the staged tile is a per-lane address), or
// consecutive pixels of the plane for a 1x1 kernel.  PXW x WK waves: wave
// (wpx, wk) owns 32 pixels and every WK-th channel pair of a stage; the WK
// partial sums of a pixel are added through LDS in a fixed order at the end.
//
// The product takes 64 cycles for 4096 FLOP, so one weight load (256 bytes)
// and one LDS read a product are cheap, and NCHW planes are staged as they
// are ([channel][row][column], no transpose): what used to bound the kernel
// was staging element by element through registers between two barriers
// (0.95 ms on 192 -> 192, 60x104, four frames: 52 TFLOP/s; now 0.465 ms, 107
// TFLOP/s, the matrix cores busy 69% of the cycles, 157.3 at peak: 1200
// workgroups on 256 compute units are 94% of five rounds, the rest is the
// last round's workgroups running alone on their SIMDs).  Here a stage
// (one tap, CB channels) goes from memory straight into one of two LDS
// buffers (buffer loads with the LDS destination: one instruction fills 64
// consecutive floats of a channel's tile, zeros outside the image or past
// the last channel) while the other is computed on, and weights are loaded
// three spatial taps ahead.  The frame of the new cache is written from LDS by the
// workgroup that stages it for its last tap.
#include <type_traits>

#include "c3c_internal.h"

namespace c3c {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int F_CO = 32;    // output channels per workgroup

struct F32Args {
  const float* x;
  const float* cache;
  const float* wpack;
  const float* bias;
  float* y;
  float* cache_out;
  int64_t hw;
  int64_t p_l;
  int64_t st, dt;
  int64_t chunks, cofrags;  // packed layout: channel pairs, 32-channel fragments
  int N, Ci, Co, T, Tc, H, W, Kt, To, Z, L;
  int bh, bw;               // output tile
  int tiles_w, tiles_h, nblocks;
  int has_bias, write_cache;
};

// KS: spatial kernel, 3 (pad 1) or 1 (the plane as one row).  CB: channels
// per stage.  NR: 64-float pieces of a channel's staged tile.  PXW: waves
// along the pixels.
template <int KS, int CB, int NR, int PXW, int WK>
__global__ __launch_bounds__(64 * PXW * WK, PXW * WK == 4 ? 3 : 2) void fast_conv3d(F32Args a) {
  constexpr int F_NPX = 32 * PXW;            // pixels per workgroup
  constexpr int NW = PXW * WK, CPW = CB / NW;  // waves; channels a wave stages
  constexpr int PAD = (KS - 1) / 2, TAPS = KS * KS;
  constexpr int NKS = CB / 2 / WK;           // channel pairs of a stage per wave
  constexpr int SEG = KS == 3 ? TAPS : 4, PPS = KS == 3 ? NKS : NKS / SEG, RING = KS == 3 ? 3 : 2;
  static_assert(CPW * NW == CB && PPS * 2 * WK * (KS == 3 ? 1 : SEG) == CB, "a stage's channels divide over the waves");
  static_assert(SEG % RING == 0, "a segment keeps its ring slot from stage to stage");
  // floats between staged channels: the two channels a product reads lie 32
  // banks apart
  constexpr int PITCH = 64 * NR + 32;
  constexpr uint32_t OOB = 0x80000000u;      // beyond every resource's size
  // two arrays: the compiler then knows that loads into one do not write what
  // is read from the other
  __shared__ float buf0[CB * PITCH];
  __shared__ float buf1[CB * PITCH];
  __shared__ float red[WK > 1 ? (WK - 1) * PXW * 64 * 16 : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wpx = wave % PXW, wk = wave / PXW;
  const int j = lane & 31, hi = lane >> 5;

  // workgroup -> tile, XCD-contiguous: output-channel tiles and output frames
  // of one spatial tile are neighbours (they stage the same frames)
  int b;
  {
    const int per = a.nblocks / 8, rem = a.nblocks % 8;
    const int xcd = static_cast<int>(blockIdx.x) % 8, slot = static_cast<int>(blockIdx.x) / 8;
    b = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + slot;
  }
  const int ct = b % static_cast<int>(a.cofrags);
  b /= static_cast<int>(a.cofrags);
  const int o = b % a.To;
  b /= a.To;
  const int tw = b % a.tiles_w;
  b /= a.tiles_w;
  const int th = b % a.tiles_h;
  const int n = b / a.tiles_h;
  const int h0 = th * a.bh, w0 = tw * a.bw;
  const int TW = a.bw + 2 * PAD, TH = a.bh + 2 * PAD;
  const int nr = (TH * TW + 63) / 64;

  // this lane's element of each 64-float piece of a staged plane
  uint32_t off[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int e = 64 * r + lane, row = e / TW, col = e - row * TW;
    const int gh = h0 - PAD + row, gw = w0 - PAD + col;
    const bool ok = row < TH && gh >= 0 && gh < a.H && gw >= 0 && gw < a.W;
    off[r] = ok ? static_cast<uint32_t>(gh * a.W + gw) * 4u : OOB;
  }
  // this lane's pixel (lanes past the tile's last pixel compute on it again)
  const int px = 32 * wpx + j;
  const int prow = min(px / a.bw, a.bh - 1), pcol = px < a.bh * a.bw ? px - (px / a.bw) * a.bw : 0;
  const int pbase = prow * TW + pcol + hi * PITCH;

  // active taps of this output frame (Eq. 4); stages run channels outer, taps
  // inner, so that workgroups of neighbouring frames share their reads in L2
  const int64_t f0 = o * a.st - a.p_l;  // source frame of tap 0
  int k_lo = 0;
  while (k_lo < a.Kt && f0 + k_lo * a.dt < 0) ++k_lo;
  int k_hi = a.Kt - 1;
  while (k_hi >= 0 && f0 + k_hi * a.dt >= a.Z) --k_hi;
  const int ntap = k_hi >= k_lo ? k_hi - k_lo + 1 : 0;
  const int nst = ntap * ((a.Ci + CB - 1) / CB);

  struct Cur {
    int ki, c0;
  };
  auto next = [&](Cur& c) __attribute__((always_inline)) {
    if (++c.ki == ntap) {
      c.ki = 0;
      c.c0 += CB;
    }
  };
  auto load = [&](const Cur& c, float* buf) __attribute__((always_inline)) {
    const int f = static_cast<int>(f0 + (k_lo + c.ki) * a.dt);
    const bool in_cache = f < a.Tc;
    const int64_t frames = in_cache ? a.Tc : a.T;
    const float* src = (in_cache ? a.cache : a.x) + (in_cache ? f : f - a.Tc) * a.hw;
#pragma unroll
    for (int q = 0; q < CPW; ++q) {
      const int cl = wave * CPW + q, ci = c.c0 + cl;
      const float* plane = src + (static_cast<int64_t>(n) * a.Ci + (ci < a.Ci ? ci : 0)) * frames * a.hw;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(plane), 0, ci < a.Ci ? static_cast<int>(a.hw * 4) : 0, 0x00020000);
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r < nr)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(buf + cl * PITCH + 64 * r), 4, off[r], 0, 0, 0);
    }
  };

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  // A stage runs in SEG segments of PPS channel pairs of this wave: a spatial
  // tap each (3x3), or a quarter of the pairs (1x1).  Weights of segment sg of
  // a stage (zeros past the last stage; pairs past the last one read another
  // tap's weights, their products are skipped).
  auto load_w = [&](bool live, const Cur& c, int sg, float (&w)[PPS]) __attribute__((always_inline)) {
    const int64_t tap = static_cast<int64_t>(k_lo + c.ki) * TAPS + (KS == 3 ? sg : 0);
    const int64_t first = (tap * a.chunks + c.c0 / 2) * a.cofrags + ct;
    const int64_t left = (static_cast<int64_t>(a.Kt) * TAPS * a.chunks * a.cofrags - first) * 256;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(a.wpack + (live ? first * 64 : 0)), 0,
        live ? static_cast<int>(left > 0x7fffffff ? 0x7fffffff : left) : 0, 0x00020000);
#pragma unroll
    for (int i = 0; i < PPS; ++i)
      w[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
          rs, lane * 4, (((KS == 3 ? 0 : sg * PPS) + i) * WK + wk) * static_cast<int>(a.cofrags) * 256, 0));
  };
  float w[RING][PPS];
  // Segment sg's products; its LDS reads were issued a segment ahead, and the
  // weights of segment sg + RING go into the ring slot it frees (the next
  // stage's first RING - 1 before the barrier that ends this stage, the last
  // one of them at the next stage's start, ahead of its staging loads, so
  // that no weight waits behind a staging load).
  auto compute = [&](auto full, bool more, const Cur& c, const Cur& nx, const float* buf) __attribute__((always_inline)) {
    const float* p = buf + pbase;
    float v[2][PPS];
    auto read = [&](int sg, float (&d)[PPS]) __attribute__((always_inline)) {
      const float* q = KS == 3 ? p + (sg / 3) * TW + sg % 3 : p + 2 * sg * PPS * WK * PITCH;
#pragma unroll
      for (int i = 0; i < PPS; ++i) d[i] = q[2 * (i * WK + wk) * PITCH];
    };
    read(0, v[0]);
#pragma unroll
    for (int sg = 0; sg < SEG; ++sg) {
      if (sg + 1 < SEG) read(sg + 1, v[(sg + 1) & 1]);
#pragma unroll
      for (int i = 0; i < PPS; ++i)
        if (decltype(full)::value || c.c0 / 2 + ((KS == 3 ? 0 : sg * PPS) + i) * WK + wk < a.chunks)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[sg % RING][i], v[sg & 1][i], acc, 0, 0, 0);
      if (sg + RING < SEG) load_w(true, c, sg + RING, w[sg % RING]);
      else if (sg + 1 < SEG) load_w(more, nx, sg + RING - SEG, w[sg % RING]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // one frame of the new cache: the stage's interior, by a workgroup of the
  // frame's last tap (each element has one writer); a frame's stages are
  // spread over the output-channel tiles, none of which then carries the
  // whole write (384 -> 384 at 30x52, one frame: 0.243 ms with tile 0
  // writing it all, 0.224 spread, 0.211 without any write)
  auto write_cache = [&](const Cur& c, const float* buf) __attribute__((always_inline)) {
    const int k = k_lo + c.ki;
    const int f = static_cast<int>(f0 + k * a.dt);
    if (!a.write_cache || (c.c0 / CB) % static_cast<int>(a.cofrags) != ct || f < a.Z - a.L ||
        !(k == a.Kt - 1 || o < a.dt))
      return;
    const int p = tid & (F_NPX - 1), row = p / a.bw, col = p - row * a.bw;
    const int h = h0 + row, w = w0 + col;
    if (row >= a.bh || h >= a.H || w >= a.W) return;
    for (int cl = tid / F_NPX; cl < CB && c.c0 + cl < a.Ci; cl += 2 * WK)  // 64 PXW WK threads
      a.cache_out[((static_cast<int64_t>(n) * a.Ci + c.c0 + cl) * a.L + (f - (a.Z - a.L))) * a.hw +
                  static_cast<int64_t>(h) * a.W + w] = buf[cl * PITCH + (row + PAD) * TW + col + PAD];
  };
  // stage `c` from buf, while the stage after it (nx; none: !more) is loaded
  // into the other buffer
  auto step = [&](bool more, const Cur& c, const Cur& nx, const float* buf, float* other) __attribute__((always_inline)) {
    load_w(true, c, RING - 1, w[RING - 1]);
    if (more) load(nx, other);
    write_cache(c, buf);  // early: the barrier below also waits for these stores
    if (c.c0 + CB <= 2 * a.chunks) compute(std::true_type{}, more, c, nx, buf);
    else compute(std::false_type{}, more, c, nx, buf);
    __syncthreads();
  };

  Cur cur{0, 0}, nx{0, 0};
  next(nx);
  if (nst > 0) {
#pragma unroll
    for (int q = 0; q + 1 < RING; ++q) load_w(true, cur, q, w[q]);
    load(cur, buf0);
    __syncthreads();
  }
  for (int s = 0; s < nst; s += 2) {
    step(s + 1 < nst, cur, nx, buf0, buf1);
    cur = nx;
    next(nx);
    if (s + 1 < nst) {
      step(s + 2 < nst, cur, nx, buf1, buf0);
      cur = nx;
      next(nx);
    }
  }

  if constexpr (WK > 1) {
    if (wk > 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[(((wk - 1) * PXW + wpx) * 16 + r) * 64 + lane] = acc[r];
    __syncthreads();
    if (wk > 0) return;
#pragma unroll
    for (int q = 0; q + 1 < WK; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += red[((q * PXW + wpx) * 16 + r) * 64 + lane];
  }

  // epilogue: bias once, NCTHW store (32 consecutive pixels of a channel)
  const int row = px / a.bw, oh = h0 + row, ow = w0 + px - row * a.bw;
  if (row >= a.bh || oh >= a.H || ow >= a.W) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int co = ct * F_CO + 8 * (r / 4) + 4 * hi + (r & 3);
    if (co >= a.Co) continue;
    const float v = a.has_bias ? acc[r] + a.bias[co] : acc[r];
    a.y[((static_cast<int64_t>(n) * a.Co + co) * a.To + o) * a.hw + static_cast<int64_t>(oh) * a.W + ow] = v;
  }
}

template <int KS, int CB, int NR, int PXW, int WK>
void launch_wk(const F32Args& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.nblocks)), block(64 * PXW * WK);
  hipLaunchKernelGGL((fast_conv3d<KS, CB, NR, PXW, WK>), grid, block, 0, s, a);
}

// Tile shape: the fewest tiles of at most npx pixels (the frame's width in
// equal columns, as many rows as fit), the widest on a tie; the halo tile of
// a 3x3 kernel holds at most halo floats.  60x104, 128 pixels: 10 x 5 tiles
// of 6 x 21 pixels (97% useful), where 4 x 64 tiles were 81%.
void shape(F32Args* a, bool one, int npx, int halo) {
  int64_t best = -1;
  int prev = 0;
  a->bh = a->bw = 1;
  for (int c = a->W < npx ? a->W : npx; c >= 1 && (best < 0 || c >= npx / 16); --c) {
    const int nt = (a->W + c - 1) / c, bw = (a->W + nt - 1) / nt;
    if (nt == prev) continue;
    prev = nt;
    int bh = npx / bw < a->H ? npx / bw : a->H;
    if (!one && bh > halo / (bw + 2) - 2) bh = halo / (bw + 2) - 2;
    if (bh < 1) continue;
    const int64_t tiles = static_cast<int64_t>((a->H + bh - 1) / bh) * nt;
    if (best < 0 || tiles < best) {
      best = tiles;
      a->bh = bh;
      a->bw = bw;
    }
    if (one) break;
  }
  a->tiles_w = (a->W + a->bw - 1) / a->bw;
  a->tiles_h = (a->H + a->bh - 1) / a->bh;
}

// Every frame of the new cache is the source of some (output frame, last tap)
// pair (unit temporal stride), so the kernel can write it.
bool cache_covered(const Geo& g) {
  if (g.d.stride_t != 1) return false;
  for (int64_t f = g.Z - g.L; f < g.Z; ++f) {
    bool hit = false;
    for (int64_t k = 0; k < g.d.Kt && !hit; ++k) {
      const int64_t o = f + g.p_l - k * g.d.dil_t;
      hit = o >= 0 && o < g.To;
    }
    if (!hit) return false;
  }
  return true;
}

}  // namespace

hipError_t launch_fast_f32(const Geo& g, const void* x, const void* cache, const void* wpack,
                           const void* bias, void* y, void* cache_out, bool* cache_written,
                           hipStream_t s, LaunchInfo* info) {
  const c3c_conv_desc& d = g.d;
  const PackDims p = pack_dims(d);
  const bool one = d.Kh == 1;
  F32Args a;
  a.x = static_cast<const float*>(x);
  a.cache = static_cast<const float*>(cache);
  a.wpack = static_cast<const float*>(wpack);
  a.bias = static_cast<const float*>(bias);
  a.y = static_cast<float*>(y);
  a.cache_out = static_cast<float*>(cache_out);
  a.hw = d.H * d.W;
  a.p_l = g.p_l; a.st = d.stride_t; a.dt = d.dil_t;
  a.chunks = p.chunks; a.cofrags = p.cofrags;
  a.N = static_cast<int>(d.N); a.Ci = static_cast<int>(d.Ci); a.Co = static_cast<int>(d.Co);
  a.T = static_cast<int>(d.T); a.Tc = static_cast<int>(d.Tc);
  // a 1x1 kernel reads the plane as one row
  a.H = one ? 1 : static_cast<int>(d.H);
  a.W = one ? static_cast<int>(a.hw) : static_cast<int>(d.W);
  a.Kt = static_cast<int>(d.Kt); a.To = static_cast<int>(g.To); a.Z = static_cast<int>(g.Z);
  a.L = static_cast<int>(g.L);
  a.has_bias = d.has_bias ? 1 : 0;
  a.write_cache = (g.L > 0 && cache_covered(g)) ? 1 : 0;
  *cache_written = a.write_cache != 0;

  auto blocks_of = [&]() { return static_cast<int64_t>(a.tiles_w) * a.tiles_h * p.cofrags * g.To * d.N; };
  shape(&a, one, 128, 256);
  // 32-pixel tiles, four waves along the channels, for a launch whose
  // 128-pixel tiles leave half of the compute units idle: a quarter of the
  // serial chain a wave and four times the workgroups (560 -> 48 at 40x56, two
  // frames: 0.326 -> 0.179 ms; 48 -> 32 at 29x32: 0.036 -> 0.024); or whose
  // share of the busiest compute unit they cut by 18% or more, which is worth
  // their larger halo (160 -> 400 at 27x48, two frames: 286 workgroups of 128,
  // 0.166 ms, 1066 of 32, 0.115; 192 -> 128 at 56x112, four frames: 0.379,
  // 0.328; with equal shares 128-pixel tiles win: 48 -> 336 at 48x60, 0.129,
  // 0.139).  Up to 32 channels 128 pixels stay, and not for speed: the tile of
  // the 32 -> 32 layer is one of the plans that callers are told.  With 32-pixel
  // tiles by the same rule from 9 channels on, 159 such calls took 0.74 of the
  // time (32 -> 64 at 46x88: 0.0269 ms, 0.0221; 16 -> 32 at 32x32: 0.0170,
  // 0.0128; 20 -> 64 at 59x96, 3x1x1: 0.0177, 0.0216).
  const int64_t cus = device_compute_units(), wide = blocks_of();
  bool small = d.Ci > 32;
  if (small) {
    shape(&a, one, 32, 64);
    // (their stages are 32 channels, the others' 16: a ragged last one weighs more)
    const int64_t c32 = (d.Ci + 31) / 32 * 32, c16 = (d.Ci + 15) / 16 * 16;
    small = wide <= cus / 2 || (blocks_of() + cus - 1) / cus * c32 * 100 <= (wide + cus - 1) / cus * 4 * c16 * 82;
    if (!small) shape(&a, one, 128, 256);
  }
  const int64_t blocks = blocks_of();
  if (info) {
    info->kernel = C3C_KERNEL_FAST_F32;
    info->tile_co = F_CO;
    info->tile_h = one ? 0 : a.bh;
    info->tile_w = a.bw;
    info->workgroups = blocks;
    info->cache_in_kernel = a.write_cache != 0;
    return hipSuccess;
  }
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  a.nblocks = static_cast<int>(blocks);
  // Waves per pixel block: a launch that leaves a compute unit one or two
  // workgroups splits their channel pairs over two waves, so that a SIMD has
  // another to switch to (384 -> 384 at 30x52, one frame, 156 workgroups: 0.224
  // ms, 0.237 unsplit; 192 -> 192 at 60x104, four frames, 1200 workgroups:
  // 0.479, 0.462 unsplit).  Four waves were slower than two (0.25, 0.58 ms).
  const bool two = blocks <= 2 * device_compute_units();
  // Few input channels: stages of 8 channels instead of 16 (32 for a 1x1
  // kernel).  The larger stages' empty channels cost their loads into LDS, and
  // the LDS they hold three workgroups of a compute unit at most: 3x1x1, 4 ->
  // 284 at 141x267, four frames, 154 us against 89; 3x3x3, 3 -> 367 at 179x208,
  // two batch elements, 189 against 136.  From 9 channels two stages a tap are
  // the longer way for a 3x3 kernel (16 -> 16 at 85x84: 16.5 against 17.9), from
  // 17 for a 1x1 one.
  const bool thin = d.Ci <= (one ? 16 : 8);
  if (one) {
    if (small) launch_wk<1, 32, 1, 1, 4>(a, s);
    else if (thin) launch_wk<1, 8, 2, 4, 1>(a, s);
    else if (two) launch_wk<1, 32, 2, 4, 2>(a, s);
    else launch_wk<1, 32, 2, 4, 1>(a, s);
  } else {
    if (small) launch_wk<3, 32, 1, 1, 4>(a, s);
    else if (thin) launch_wk<3, 8, 4, 4, 1>(a, s);
    else if (two) launch_wk<3, 16, 4, 4, 2>(a, s);
    else launch_wk<3, 16, 4, 4, 1>(a, s);
  }
  return hipGetLastError();
}

}  // namespace c3c
