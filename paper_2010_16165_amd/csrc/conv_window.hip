// Convolutions with the input of a workgroup's pixels in LDS and the weights
// streamed straight from L2 into registers (Sec. III, Sec. IV-B-1: operator
// k x c x r x s with its fused epilogue).
//
// What it takes: windows of at most 25 taps, padded by at most half their shorter side
// (window_patch.h), tensors and weights under 2 GiB, tiles whose input fits LDS with all channels.
// What it is for: layers that a pipeline of LDS stages does not fill - one image or a few, deep
// layers of any batch, strided windows.  There a chain of dependent stages (load, barrier,
// multiply) leaves the matrix pipe idle most of the time (512 -> 359 channels, 3 x 3 on a 7 x 7
// image: 13.9 us, of which 16 dependent stages of 2250 clocks each).  Here a tile has no stages:
//
//   * The tile's whole input, all channels, goes to LDS once.  Input pixels of a window are
//     taken as one row of pixels, first to last, rows and images one behind the other: the patch
//     is one contiguous run of memory and a tap a constant distance in it.  What the run holds
//     beyond the image border is not used: each lane knows which taps of its pixel lie inside
//     (one bit each), and reads zeros (patch pixel 0) for the others.
//   * Weights are not shared between the waves of a workgroup: waves lie side by side along the
//     filters (WF) or take every WK-th step of the reduction, each over all pixels of the tile.
//     So no weight is read twice in a workgroup, none goes through LDS, and no barrier stands in
//     the loop: a wave loads fragments in MFMA layout D steps ahead and multiplies.
//     (Loading the pixels like that as well reads at 9.5 TB/s where a pixel's bytes are a multiple
//     of 512, since neighbouring lanes then hit one bank of the L1, against 27 TB/s for runs of
//     64 bytes or more: that version took 33 us where this one takes 14.3, 256 -> 180 at 14 x 14 x 64.)
//   * The waves' partial sums meet in LDS at the end, in the order of the waves; the tiles are
//     shared out between the waves for the epilogue (shortcut, ReLU, one rounding, 16 bytes per lane).
//   * Workgroups are numbered so that those of one XCD share what is larger, the filters of a
//     group or the pixels of a region, in that XCD's L2.
//
// Measured, before -> now (us per launch in a replayed graph): 3 x 3, 512 -> 359 at 7 x 7, one
// image 13.9 -> 5.2; 64 -> 45 at 56 x 56, one image 6.4 -> 3.9; stride 2, 229 -> 117 at 25 x 25 x 9
// 22.2 -> 5.7; 256 -> 180 at 14 x 14 x 20 12.5 -> 7.8, x 64 19.1 -> 14.3; 163 -> 183 at 14 x 14 x 256
// 41 -> 29; with listed output channels 359 -> 359 of 512 at 7 x 7 x 20 16.4 -> 10.2; fc, 2048 -> 1000 on 64 pixels 12.3 -> 4.6.  A kernel that does nothing takes 1.7.
// Single precision runs through the same code on the 16 x 16 x 4 MFMA: a chunk is then 4 channels
// (16 bytes as well), a step 16 channels in four MFMAs, each of which takes one channel of every
// lane's chunk.  A CIFAR-size network of 21 layers on 32 images: 410 us (one thread per pixel and
// four filters, vector FMAs) -> 111.
// Clocks of a launch of one image (3 x 3, 256 -> 180 at 14 x 14, eight waves, about 10 000 with the 3600 that an empty
// launch takes): arguments 430, first weights asked for 400, pixels 1100, tables and the wait 1400, multiplication 1500,
// exchange 500, sums and store 1100.  Arguments in one go, tables by waves of their own, the shortcut asked for with the
// pixels, partial sums beside the patch and added up without choices: ResNet-18, one image 92.8 -> 88.9 us, ResNet-50, 9 images
// 264 -> 257, ResNet-34, 20 images 353 -> 347.
// What bounds it: below some ten images latency (arguments, patch, first weights, one store);
// then the weights, which every tile reads anew (45 bytes per clock and compute unit), and the
// vector instructions that work out pixel addresses, beside the matrix pipe.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <iterator>

#include "conv16.h"
#include "device_utils.h"
#include "fupr.h"
#include "layout.h"
#include "tuning.h"
#include "window_patch.h"

namespace fupr {
namespace {

constexpr uint32_t kOutside = 0x80000000u;   // beyond every tensor this kernel accepts
constexpr int kMaxTaps = 25;                 // taps whose validity fits one register
constexpr size_t kLdsLimit = 160 * 1024;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef void __attribute__((address_space(3)))* LdsPtr;

enum { kOneTap = 0, kWindow = 1, kCat = 2 };

struct WindowParams {
  const uint16_t* x;
  const uint16_t* x2;    // kCat: the channels from step split_steps on
  const uint16_t* w;
  const float* bias;
  // A block's pruned output filters have no shortcut tensor: filter j adds into channel keep[j]
  // of y (keep_n entries, in 0 .. yC - 1); the workgroup's part of the list lies in LDS at keep_at.
  union { const uint16_t* res; const int32_t* keep; };
  uint16_t* y;
  uint32_t x_bytes, x2_bytes, w_bytes, res_bytes, y_bytes;
  int H, W, pix;         // input extent; bytes per pixel
  int pixels;            // N * H * W
  int P, Q, PQ, M, ycs;
  int R, S, stride, pad;
  int Kp, cpt, nsteps;
  union { int split_steps, keep_at; };   // (kCat, kWindow)
  int H2, W2, pix2, stride2;
  union { int rH, keep_n; };
  union { int rW, yC; };
  int rcs, rss, roff, relu;
  int mgroups, fgroups, total, per_xcd, filter_major;
  int WF, WK;            // waves along the filters, along the reduction (powers of two)
  int log2_WF;
  int slots, slots2;     // 16-byte LDS slots per pixel (kCat: of the first, of the second tensor)
  int live, live2;       // of these, slots that hold channels of the tensor
  int res_linear;        // the shortcut's pixels are the output's
  int table_at, table_bytes, pixels_at, patch2_at;   // LDS byte offsets (the patch starts at 0)
  FastDiv divPQ, divQ, divC, divS, divSlots, divSlots2;
  FastDiv divG;          // by mgroups or fgroups, whichever runs fastest
  int part_at;           // LDS byte offset of the partial sums; 0: over the patch, after a barrier
  int pad_[4];
};
static_assert(sizeof(WindowParams) == 320, "load_arguments");

__device__ __forceinline__ uint32_t clamp_below(uint32_t v, uint32_t floor2) {
  const short2_t a = __builtin_bit_cast(short2_t, v), f = __builtin_bit_cast(short2_t, floor2);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, f));
}

__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, soff, 0));
}

// lane i moves the 16 bytes at offset off of the buffer to the i-th slot after
// lds_base; an offset outside the buffer writes zeros
__device__ __forceinline__ void load_to_lds(const i32x4& rsrc, uint32_t off, uint32_t lds_base) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, 0 offen lds"
      :
      : "s"(lds_base), "v"(off), "s"(rsrc)
      : "memory", "m0");
}

__device__ __forceinline__ i32x4 make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}

// Tiles so small that the wave which finishes one hands its own sum over as well: what it adds up is then read in
// a row without a choice, 60 instructions for eight waves in place of 200 (1200 clocks of a launch of 10 000).
constexpr bool all_partial_sums(int tiles) { return tiles <= 4; }

// Adds the partial sums of WK = 2, 4, 8 (or 16) waves up, in their order, for TILES tiles that follow each other; up to
// eight waves' are asked for before the first is added.  Every read stands here once and the numbers are told apart by what is
// left out: with a variant for each, the last read of all three became one instruction, and structurizecfg (AMD clang 22.0.0git,
// roc-7.2.0) left its address undefined where WK is 2 (right before that pass, poison behind it).
template <int TILES>
__device__ __forceinline__ void add_up(const f32x4* src, int next, int WK, f32x4* sums) {
  f32x4 u[8][TILES];
  auto ask = [&](int from, int to) {
#pragma unroll
    for (int k = from; k < to; ++k)
#pragma unroll
      for (int t = 0; t < TILES; ++t) u[k][t] = src[k * next + t * 64];
  };
  auto add = [&](int from, int to) {
#pragma unroll
    for (int k = from; k < to; ++k)
#pragma unroll
      for (int t = 0; t < TILES; ++t) sums[t] += u[k][t];
  };
  ask(0, 2);
  if (WK > 2) ask(2, 4);
  if (WK > 4) ask(4, 8);
  add(0, 2);
  if (WK > 2) add(2, 4);
  if (WK > 4) add(4, 8);
#pragma unroll 1
  for (int k = 8; k < WK; ++k)
#pragma unroll
    for (int t = 0; t < TILES; ++t) sums[t] += src[k * next + t * 64];
}

// A wave's tile is MT x NT tiles of 16 pixels x 16 filters.  D: steps of weights in flight per
// wave; G: steps whose pixels are read from LDS together.  IX: every filter adds into its listed
// channel of y (p.keep); without it p.keep is not read.  `given`: the kernel's arguments, of several in a row the one
// numbered `which`.
template <int EL, int MODE, int MT, int NT, int D, int G, bool IX>
__device__ __forceinline__ void window_tile(const WindowParams& given, const int which) {
  // Short launches load them all at once.  Longer ones leave it to the compiler, behind one look at every line: 3 x 3 with a
  // shortcut, 77 -> 102 channels at 57 x 38 x 6 6.60 -> 6.54 us, 86 -> 46 at 30 x 50 x 8 2.7 % less; networks are equal.
  constexpr bool kShort = MT <= 2;
  if constexpr (!kShort) touch_arguments<sizeof(WindowParams)>();
  const WindowParams p = kShort ? load_arguments<WindowParams>(which) : given;
  constexpr bool F32 = EL == FUPR_F32, BF = EL == FUPR_BF16;
  constexpr uint32_t ES = F32 ? 4 : 2;       // bytes per element
  extern __shared__ uint4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  const uint32_t lds_base = (uint32_t)(uintptr_t)(LdsPtr)lds;
  constexpr int TT = MT * NT, BM = MT * 16;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int waves = p.WF * p.WK;
  if (wave >= waves) return;                 // (conv_window_two_kernel)
  const int wk = wave >> p.log2_WF, wf = wave & (p.WF - 1);

  const int l = tile_of_workgroup(blockIdx.x, p.per_xcd, p.total);
  if (l < 0) return;
  const int slow = div_by(l, p.divG);
  const int fast = l - slow * (p.filter_major ? p.mgroups : p.fgroups);
  const int mg = p.filter_major ? fast : slow, fg = p.filter_major ? slow : fast;
  const int m0 = mg * BM;
  const int f0 = (fg * p.WF + wf) * (NT * 16);

  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.w), 0, p.w_bytes, 0x00020000);
  uint32_t a_off[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
    a_off[t] = F32 ? (uint32_t)(g * 4 * p.Kp + min(f0 + t * 16 + li, p.Kp - 1)) * 4u
                   : (uint32_t)(g * p.Kp + min(f0 + t * 16, p.Kp - 16) + li) * 16u;
  const uint32_t a_step = (uint32_t)p.Kp * 64u;
  uint4 a[D][NT];
  // of this wave's next step (steps past the end read the last step's weights, and are not multiplied)
  const uint32_t w_last = (uint32_t)(p.nsteps - 1) * a_step, w_step = (uint32_t)p.WK * a_step;
  uint32_t w_at = min((uint32_t)wk * a_step, w_last);
  auto load_weights = [&](uint4* av) {
    const uint32_t so = w_at;
    w_at = min(w_at + w_step, w_last);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if constexpr (F32) {
        // four channels of the lane's chunk and filter; the last step may end inside itself,
        // and what lies beyond the weights reads as zero
        const uint32_t at = a_off[t] + so, row = (uint32_t)p.Kp * 4u;
        av[t].x = __builtin_amdgcn_raw_buffer_load_b32(wr, at, 0, 0);
        av[t].y = __builtin_amdgcn_raw_buffer_load_b32(wr, at + row, 0, 0);
        av[t].z = __builtin_amdgcn_raw_buffer_load_b32(wr, at + 2 * row, 0, 0);
        av[t].w = __builtin_amdgcn_raw_buffer_load_b32(wr, at + 3 * row, 0, 0);
      } else {
        av[t] = load16(wr, a_off[t], so);
      }
    }
  };

  // The first weights and the biases need no index arithmetic beyond these lines and are the last to
  // arrive in a cold L2: they are asked for before anything else (a 16-bit network of 22 short launches 93.9 ->
  // 92.9 us).  Single precision loads them four bytes at a time and asks for its pixels first (101.3 against
  // 103.9 us for 15 launches); so do tiles of more than two, which are long launches and gain nothing.
  auto first_weights = [&] {
#pragma unroll
    for (int d = 0; d < D; ++d) load_weights(a[d]);
  };
  constexpr bool kWeightsFirst = !F32 && MT <= 2;
  if constexpr (kWeightsFirst) first_weights();
  f32x4 bias4[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) bias4[t] = *reinterpret_cast<const f32x4*>(p.bias + min(f0 + t * 16 + g * 4, p.Kp - 4));

  // ---- the pixels' input into LDS ----
  // Patch pixel 0 is zeros.  kWindow: pixel 1 + i is input pixel first + i of the batch taken
  // as one row of pixels, so that a tap is a constant distance; else it is the input pixel of
  // output pixel m0 + i.
  auto split_pixel = [&](int m, int* n, int* pp, int* qq) {
    *n = div_by(m, p.divPQ);
    const int rem = m - *n * p.PQ;
    *pp = div_by(rem, p.divQ);
    *qq = rem - *pp * p.Q;
  };
  int first = m0, patch_pixels = 1 + BM;
  if constexpr (MODE == kWindow) {
    auto origin_of = [&](int m) {
      int n, pp, qq;
      split_pixel(m, &n, &pp, &qq);
      return window_origin(n, pp, qq, p.H, p.W, p.stride, p.pad);
    };
    first = origin_of(m0);
    const int last = origin_of(min(m0 + BM, p.M) - 1) + window_reach(p.R, p.S, p.W);
    patch_pixels = 1 + last - first + 1;
  }
  const int stride64 = waves * 64;
  // pixels that follow each other in memory: slot after slot, stepping
  auto fill_run = [&](const i32x4& rsrc, int slots, const FastDiv& by, int live, int pix, int limit, int at) {
    const int step_pix = div_by(stride64, by), step_c = stride64 - step_pix * slots;   // (scalar)
    int slot = wave * 64 + lane;
    int pixel = div_by(slot, by), c = slot - pixel * slots;
    pixel += first - 1;                       // input pixel
    const int zero = first - 1;
    uint32_t off = (uint32_t)pixel * (uint32_t)pix + (uint32_t)c * 16u;
    const uint32_t step_off = (uint32_t)(step_pix * pix + step_c * 16), wrap_off = (uint32_t)(pix - slots * 16);
    const int count = patch_pixels * slots;
    for (int base = wave * 64; base < count; base += stride64) {
      const bool ok = c < live && pixel != zero && (unsigned)pixel < (unsigned)limit;
      load_to_lds(rsrc, ok ? off : kOutside, lds_base + at + base * 16);
      c += step_c;
      pixel += step_pix;
      off += step_off;
      const bool wrap = c >= slots;
      c -= wrap ? slots : 0;
      pixel += wrap ? 1 : 0;
      off += wrap ? wrap_off : 0u;
    }
  };
  // a pixel of every stride-th column and row
  auto fill_strided = [&](const i32x4& rsrc, int slots, const FastDiv& by, int live, int pix, int stride, int H, int W,
                          int at) {
    const int count = patch_pixels * slots;
    for (int base = wave * 64; base < count; base += stride64) {
      const int slot = base + lane;
      const int pixel = div_by(slot, by), c = slot - pixel * slots, m = m0 + pixel - 1;
      int n, pp, qq;
      split_pixel(m, &n, &pp, &qq);
      const bool ok = c < live && pixel > 0 && m < p.M;
      const uint32_t in = (uint32_t)((n * H + pp * stride) * W + qq * stride);
      load_to_lds(rsrc, ok ? in * (uint32_t)pix + (uint32_t)c * 16u : kOutside, lds_base + at + base * 16);
    }
  };
  const i32x4 xr = make_rsrc(p.x, p.x_bytes);
  if (MODE == kOneTap && p.stride != 1)
    fill_strided(xr, p.slots, p.divSlots, p.live, p.pix, p.stride, p.H, p.W, 0);
  else
    fill_run(xr, p.slots, p.divSlots, p.live, p.pix, p.pixels, 0);
  if constexpr (MODE == kCat) {
    const i32x4 x2r = make_rsrc(p.x2, p.x2_bytes);
    fill_strided(x2r, p.slots2, p.divSlots2, p.live2, p.pix2, p.stride2, p.H2, p.W2, p.patch2_at);
  }
  if constexpr (!kWeightsFirst) first_weights();

  // The two tables of a window, by waves of their own where there are enough.  Per chunk of 8 channels: its LDS
  // distance from the window origin, and its tap.  (What is multiplied here lies inside the patch: 24 bits.)
  u32x2* table = reinterpret_cast<u32x2*>(lds + p.table_at);
  constexpr int kPixelWaves = (BM + 63) / 64;
  const int apart = waves > kPixelWaves ? kPixelWaves : 0;   // waves that leave the taps to the others
  if (MODE == kWindow && wave >= apart) {
    const int entries = p.table_bytes / 8;
    for (int j = tid - apart * 64; j < entries; j += stride64 - apart * 64) {
      const int tap = div_by(j, p.divC), cc = j - __mul24(tap, p.cpt);
      const int r = div_by(tap, p.divS), s = tap - __mul24(r, p.S);
      const bool ok = tap < p.R * p.S;
      u32x2 e;
      e[0] = ok ? (uint32_t)((__mul24(__mul24(r, p.W) + s, p.slots) + cc) * 16) : 0u;
      e[1] = ok ? (uint32_t)tap : 31u;
      table[j] = e;
    }
  }

  // per pixel of the tile: LDS address of the window origin, and which taps lie inside the image
  u32x2* pixel_table = reinterpret_cast<u32x2*>(lds + p.pixels_at);
  if (MODE == kWindow && (apart == 0 || wave < apart)) {
    for (int i = tid; i < BM; i += stride64) {
      const int m = m0 + i;
      int n, pp, qq;
      split_pixel(min(m, p.M - 1), &n, &pp, &qq);
      const int ih = pp * p.stride - p.pad, iw = qq * p.stride - p.pad;
      const int lo = max(0, -iw), hi = min(p.S, p.W - iw);   // columns lo .. hi - 1 of the window
      const uint32_t cols = hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
      uint32_t taps = 0;
      for (int r = 0; r < p.R; ++r)
        taps |= (uint32_t)(ih + r) < (uint32_t)p.H ? cols << (r * p.S) : 0u;
      u32x2 e;
      e[0] = (uint32_t)((1 + (n * p.H + ih) * p.W + iw - first) * p.slots * 16);
      e[1] = m < p.M ? taps : 0u;
      pixel_table[i] = e;
    }
  }

  // per filter of the workgroup: its channel of y, -1 for one that does not exist or points outside
  if constexpr (IX) {
    int* list = reinterpret_cast<int*>(lds + p.keep_at);
    for (int i = tid; i < p.WF * NT * 16; i += stride64) {
      const int k = fg * p.WF * NT * 16 + i, c = p.keep[min(k, p.keep_n - 1)];
      list[i] = k < p.keep_n && (unsigned)c < (unsigned)p.yC ? c : -1;
    }
  }

  // The shortcut, of the pairs of filter tiles that this wave will finish (an odd last tile is alone).  After
  // the exchange between 16-lane rows lane (pixel, g) holds channels (g >> 1) * 8 .. + 7 of tile t + (g & 1): 16-byte
  // accesses; a lone tile keeps 8 bytes.  Small tiles ask for it here, where it arrives with the pixels; the others, whose
  // registers are taken, all at once when they have multiplied (asked for pair by pair in front of each store it
  // cost a memory latency per pair).
  constexpr int NP = (NT + 1) / 2;
  constexpr int NR = IX ? 1 : F32 ? NT : NP;     // (single precision: 16 bytes a tile)
  constexpr bool kShortcutFirst = !IX && MT * NR <= 2, kShortcutLater = !IX && !kShortcutFirst;
  const __amdgpu_buffer_rsrc_t rr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.res), 0, p.res_bytes, 0x00020000);
  auto res_at = [&](int m) {     // byte offset of output pixel m's shortcut pixel
    if (p.res_linear) return (uint32_t)(m * p.rcs) * ES;
    int n, pp, qq;
    split_pixel(m, &n, &pp, &qq);
    return (uint32_t)(((n * p.rH + pp * p.rss) * p.rW + qq * p.rss) * p.rcs) * ES;
  };

  u32x4 shortcut[IX ? 1 : MT][NR];
  auto ask_shortcut = [&] {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = m0 + mt * 16 + li;
      const uint32_t ro = m < p.M ? res_at(m) : 0u;
#pragma unroll
      for (int pr = 0; pr < NP; ++pr) {
        if (((mt * NP + pr) & (p.WK - 1)) != wk) continue;
        if constexpr (F32) {
#pragma unroll
          for (int u = 2 * pr; u < (2 * pr + 2 < NT ? 2 * pr + 2 : NT); ++u) {
            const int kk = f0 + u * 16 + g * 4 - p.roff;
            shortcut[mt][u] = __builtin_amdgcn_raw_buffer_load_b128(
                rr, m < p.M && kk >= 0 && kk < p.rcs ? ro + (uint32_t)kk * 4u : kOutside, 0, 0);
          }
          continue;
        }
        const bool pair = 2 * pr + 1 < NT;
        const int kk = f0 + pr * 32 + (pair ? (g & 1) * 16 + (g >> 1) * 8 : g * 4) - p.roff;
        const uint32_t at = m < p.M && kk >= 0 && kk < p.rcs ? ro + (uint32_t)kk * 2u : kOutside;
        if (pair) {
          shortcut[mt][pr] = __builtin_amdgcn_raw_buffer_load_b128(rr, at, 0, 0);
        } else {
          const u32x2 r2 = __builtin_amdgcn_raw_buffer_load_b64(rr, at, 0, 0);
          shortcut[mt][pr] = u32x4{r2[0], r2[1], 0u, 0u};
        }
      }
    }
  };
  if constexpr (kShortcutFirst) {
    if (p.res) ask_shortcut();
  }

  // the first wave of a column starts from the bias, the others from zero
  f32x4 acc[MT][NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const f32x4 b4 = wk == 0 ? bias4[t] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][t] = b4;
  }

  // (twice: the loads to LDS have landed, and the compiler knows that the weights have, or it waits for them anew in every
  // step of the first round: 3 x 3, 77 -> 102 channels at 57 x 38 x 6 6.71 -> 6.67 us, ResNet-18 of 11 images, half
  // pruned, 148.6 -> 148.1)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();

  uint32_t origin[MT], origin2[MT], inside[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int i = mt * 16 + li;
    origin2[mt] = inside[mt] = 0;
    if constexpr (MODE == kWindow) {
      const u32x2 e = pixel_table[i];
      origin[mt] = e[0];
      inside[mt] = e[1];
    } else {
      origin[mt] = (uint32_t)((1 + i) * p.slots * 16 + g * 16);
      if constexpr (MODE == kCat) origin2[mt] = (uint32_t)(p.patch2_at + (1 + i) * p.slots2 * 16 + g * 16);
    }
  }

  // Steps are taken in groups of G: the pixels of a group, and the table entries of the group
  // after it, are read from LDS while the group before is multiplied.
  uint4 b[2][G][MT];
  u32x2 entry[G];
  auto look_up = [&](int step) {
    if constexpr (MODE == kWindow) {
#pragma unroll
      for (int i = 0; i < G; ++i) entry[i] = table[(step + i * p.WK) * 4 + g];
    }
  };
  auto read_pixels = [&](int step, uint4 (*bv)[MT]) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      if constexpr (MODE == kWindow) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          // a tap outside the image reads patch pixel 0, which lies at LDS address 0
          const uint32_t in = (uint32_t)__builtin_amdgcn_sbfe((int)inside[mt], entry[i][1], 1);
          bv[i][mt] = *reinterpret_cast<const uint4*>(lds + ((origin[mt] + entry[i][0]) & in));
        }
      } else {
        const int st = step + i * p.WK;
        const bool second = MODE == kCat && st >= p.split_steps;
        const uint32_t off = (uint32_t)(second ? st - p.split_steps : st) * 64u;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const uint32_t at = st < p.nsteps ? (second ? origin2[mt] : origin[mt]) + off : 0u;
          bv[i][mt] = *reinterpret_cast<const uint4*>(lds + at);
        }
      }
    }
  };

  int left = (p.nsteps - wk + p.WK - 1) / p.WK;   // this wave's steps
  int step = wk;
  look_up(step);
  read_pixels(step, b[0]);
  look_up(step + G * p.WK);
  static_assert(D % (2 * G) == 0, "the pixel buffers alternate");
  auto group = [&](int gi, bool more) {
    step += G * p.WK;
    read_pixels(step, b[(gi + 1) & 1]);
    look_up(step + G * p.WK);
    // (left alone, the scheduler sinks every read to just before its use)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const int d = gi * G + i;
      // A step past the end is not multiplied: its weights are the last step's, and an infinite one
      // times the zeros of its pixels would be NaN.  Against multiplying it: a bf16 network of 22 short
      // launches 96.8 -> 97.7 us (zeros in place of the weights, by mask or by range check: 97.9 -
      // 98.6), an fp32 one, four MFMAs of 32 clocks less per step, 115.0 -> 111.1.
      if (!more && i > 0 && d >= left) break;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          {
          if constexpr (F32) {
            // MFMA k takes channel k of every lane's chunk of four
            const uint4 &av = a[d][t], &bv = b[gi & 1][i][mt];
            acc[mt][t] = mfma_16x16x4(av.x, bv.x, acc[mt][t]);
            acc[mt][t] = mfma_16x16x4(av.y, bv.y, acc[mt][t]);
            acc[mt][t] = mfma_16x16x4(av.z, bv.z, acc[mt][t]);
            acc[mt][t] = mfma_16x16x4(av.w, bv.w, acc[mt][t]);
          } else {
            acc[mt][t] = mfma_16x16x32<BF>(a[d][t], b[gi & 1][i][mt], acc[mt][t]);
          }
        }
      if (more) load_weights(a[d]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  for (; left > D; left -= D) {
#pragma unroll
    for (int gi = 0; gi < D / G; ++gi) group(gi, true);
  }
  // the last round loads nothing and ends at the last group that holds a step
#pragma unroll
  for (int gi = 0; gi < D / G; ++gi)
    if (gi * G < left) group(gi, false);

  // ---- epilogue: shortcut, ReLU, one rounding ----
  const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, 0x00020000);
  if constexpr (kShortcutLater) {
    if (p.res) ask_shortcut();
  }
  const uint32_t floor2 = p.relu ? 0u : 0x80008000u;
  // The waves of a column share its pairs of filter tiles: wave e % WK finishes pair e, the
  // others hand it their sums through LDS (where that is short over the patch, which nobody reads any more).
  // Listed channels are updated with 2-byte accesses (they have gaps, and the words between two
  // waves' channels are shared).  What a wave will add to is asked for here, before the exchange
  // of the partial sums, so that its latency passes meanwhile.
  i32x4 channel[IX ? NT : 1];
  uint16_t old[IX ? MT : 1][IX ? NT : 1][4];
  auto listed_at = [&](int mt, int t, int i) {
    const int m = m0 + mt * 16 + li, c = channel[t][i];
    return m < p.M && c >= 0 ? (uint32_t)(m * p.ycs + c) * 2u : kOutside;
  };
  if constexpr (IX) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
      channel[t] = *reinterpret_cast<const i32x4*>(lds + p.keep_at + ((wf * NT + t) * 16 + g * 4) * 4);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int pr = 0; pr < NP; ++pr)
        if (((mt * NP + pr) & (p.WK - 1)) == wk)
#pragma unroll
          for (int t = 2 * pr; t < (2 * pr + 2 < NT ? 2 * pr + 2 : NT); ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              old[mt][t][i] = __builtin_amdgcn_raw_buffer_load_b16(yr, listed_at(mt, t, i), 0, 0);
  }
  // [giver][column][tile][lane]; small tiles: [wave along the reduction] and so on
  f32x4* part = reinterpret_cast<f32x4*>(lds + p.part_at);
  constexpr bool kAll = all_partial_sums(TT);
  if (p.WK > 1) {
    if (p.part_at == 0) __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int giver = (wk - (mt * NP + t / 2)) & (p.WK - 1);   // 0: the owner
        if constexpr (kAll) part[((wk * p.WF + wf) * TT + mt * NT + t) * 64 + lane] = acc[mt][t];
        else if (giver > 0) part[(((giver - 1) * p.WF + wf) * TT + mt * NT + t) * 64 + lane] = acc[mt][t];
      }
    __syncthreads();
  }
  if (f0 >= p.Kp) return;
  auto finish = [&](const f32x4& av, uint32_t r0, uint32_t r1) {
    float v[4] = {av[0], av[1], av[2], av[3]};
    if (p.res) {
      v[0] += to_float<BF>((uint16_t)(r0 & 0xffffu));
      v[1] += to_float<BF>((uint16_t)(r0 >> 16));
      v[2] += to_float<BF>((uint16_t)(r1 & 0xffffu));
      v[3] += to_float<BF>((uint16_t)(r1 >> 16));
    }
    u32x2 o;
    o[0] = clamp_below(pack2<BF>(v[0], v[1]), floor2);
    o[1] = clamp_below(pack2<BF>(v[2], v[3]), floor2);
    return o;
  };
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m0 + mt * 16 + li;
    const uint32_t yo = m < p.M ? (uint32_t)(m * p.ycs) * ES : kOutside;
#pragma unroll
    for (int pr = 0; pr < NP; ++pr) {
      if (((mt * NP + pr) & (p.WK - 1)) != wk) continue;
      const int t = 2 * pr;
      if constexpr (F32) {
        // single precision: a lane's four channels of a tile are 16 bytes
#pragma unroll
        for (int u = t; u < (t + 2 < NT ? t + 2 : NT); ++u) {
          const int k0 = f0 + u * 16 + g * 4;
          f32x4 r4 = {0.f, 0.f, 0.f, 0.f};
          if (p.res) r4 = __builtin_bit_cast(f32x4, shortcut[mt][u]);
          f32x4 v = acc[mt][u];
          if (p.WK > 1) {
            v = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (kAll) {
              add_up<1>(part + (wf * TT + mt * NT + u) * 64 + lane, p.WF * TT * 64, p.WK, &v);
            } else
            for (int k = 0; k < p.WK; ++k) {
              const int from = ((k - wk) & (p.WK - 1)) - 1;
              const f32x4 q = part[((max(from, 0) * p.WF + wf) * TT + mt * NT + u) * 64 + lane];
              v += from < 0 ? acc[mt][u] : q;
            }
          }
          v += r4;
          if (p.relu)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), yr,
                                                 k0 < p.ycs ? yo + (uint32_t)k0 * 4u : kOutside, 0, 0);
        }
        continue;
      }
      const bool pair = t + 1 < NT;
      auto totals = [&](f32x4* s0, f32x4* s1) {
        // in the order of the waves, whichever of them adds up: the sum does not depend on the tile
        *s0 = acc[mt][t];
        *s1 = acc[mt][pair ? t + 1 : t];
        if (p.WK > 1) {
          const f32x4 own0 = *s0, own1 = *s1;
          *s0 = *s1 = f32x4{0.f, 0.f, 0.f, 0.f};
          if constexpr (kAll) {
            f32x4 sums[2] = {*s0, *s1};
            const f32x4* src = part + (wf * TT + mt * NT + t) * 64 + lane;
            if (pair) add_up<2>(src, p.WF * TT * 64, p.WK, sums);
            else add_up<1>(src, p.WF * TT * 64, p.WK, sums);
            *s0 = sums[0];
            *s1 = sums[1];
            return;
          }
          for (int k = 0; k < p.WK; ++k) {
            const int from = ((k - wk) & (p.WK - 1)) - 1;          // -1: this wave itself
            const f32x4* src = part + ((max(from, 0) * p.WF + wf) * TT + mt * NT + t) * 64 + lane;
            const f32x4 u0 = src[0], u1 = src[pair ? 64 : 0];
            *s0 += from < 0 ? own0 : u0;
            *s1 += from < 0 ? own1 : u1;
          }
        }
      };
      if constexpr (IX) {
        f32x4 s[2];
        totals(&s[0], &s[1]);
#pragma unroll
        for (int u = 0; u < (pair ? 2 : 1); ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float v = s[u][i] + to_float<BF>(old[mt][t + u][i]);
            if (p.relu) v = fmaxf(v, 0.f);
            __builtin_amdgcn_raw_buffer_store_b16(from_float<BF>(v), yr, listed_at(mt, t + u, i), 0, 0);
          }
        continue;
      }
      const int k0 = f0 + t * 16 + (pair ? (g & 1) * 16 + (g >> 1) * 8 : g * 4);
      u32x4 r4 = {0u, 0u, 0u, 0u};
      if (p.res) r4 = shortcut[mt][pr];
      f32x4 s0, s1;
      totals(&s0, &s1);
      const uint32_t off = k0 < p.ycs ? yo + (uint32_t)k0 * 2u : kOutside;
      if (pair) {
        uint32_t ra0 = 0, ra1 = 0, rb0 = 0, rb1 = 0;
        if (p.res) {
          const auto q0 = __builtin_amdgcn_permlane16_swap(r4[0], r4[2], false, false);
          const auto q1 = __builtin_amdgcn_permlane16_swap(r4[1], r4[3], false, false);
          ra0 = q0[0]; ra1 = q1[0];   // tile t
          rb0 = q0[1]; rb1 = q1[1];   // tile t + 1
        }
        const u32x2 oa = finish(s0, ra0, ra1);
        const u32x2 ob = finish(s1, rb0, rb1);
        const auto w0 = __builtin_amdgcn_permlane16_swap(oa[0], ob[0], false, false);
        const auto w1 = __builtin_amdgcn_permlane16_swap(oa[1], ob[1], false, false);
        const u32x4 o4 = {w0[0], w1[0], w0[1], w1[1]};
        __builtin_amdgcn_raw_buffer_store_b128(o4, yr, off, 0, 0);
      } else {
        __builtin_amdgcn_raw_buffer_store_b64(finish(s0, r4[0], r4[1]), yr, off, 0, 0);
      }
    }
  }
}

template <int EL, int MODE, int MT, int NT, int D, int G, int THREADS, int MINWAVES, bool IX>
__global__ __launch_bounds__(THREADS, MINWAVES) void conv_window_kernel(const WindowParams p) {
  window_tile<EL, MODE, MT, NT, D, G, IX>(p, 0);
}

// D: steps of weights in flight; G: steps per group of pixel reads; vgprs: registers as the estimate below was fitted
// with.  (They were those of the 16-bit window form; 16 x 48, 32 x 16 and 32 x 32, which hold the shortcut while they multiply, take 4
// - 8 more now, one-tap forms up to 18, fp32 up to 18.  With each form's own registers, in steps of 8, 6 % of plans are others
// and no network or operator of 46 is faster or slower by more than its runs differ.)
struct WindowTile {
  int MT, NT, D, G, threads, min_waves, vgprs;
  const char *three, *one_tap, *other, *single;
};
#define FUPR_NAMES(t) "conv3x3p_w" t, "conv1x1p_w" t, "conv16t_w" t, "conv32_w" t
constexpr WindowTile kTiles[] = {
    {1, 1, 8, 4, 1024, 4, 85, FUPR_NAMES("16x16")},  {1, 3, 4, 2, 1024, 4, 92, FUPR_NAMES("16x48")},
    {2, 1, 8, 2, 1024, 4, 87, FUPR_NAMES("32x16")},  {2, 2, 4, 2, 1024, 4, 96, FUPR_NAMES("32x32")},
    {2, 3, 4, 2, 512, 2, 122, FUPR_NAMES("32x48")},  {4, 1, 6, 1, 512, 2, 89, FUPR_NAMES("64x16")},
    {4, 2, 4, 1, 512, 2, 114, FUPR_NAMES("64x32")},  {4, 3, 4, 1, 512, 2, 148, FUPR_NAMES("64x48")},
    {4, 4, 4, 1, 512, 2, 180, FUPR_NAMES("64x64")},  {7, 2, 4, 1, 512, 2, 168, FUPR_NAMES("112x32")},
    {7, 3, 4, 1, 512, 2, 214, FUPR_NAMES("112x48")}, {7, 4, 2, 1, 512, 2, 227, FUPR_NAMES("112x64")},
};
#undef FUPR_NAMES
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
// The tiles compiled for listed channels: what a wave adds to is held in registers.
constexpr bool listed_tile(const WindowTile& T) { return T.MT * T.NT <= 12; }

struct WindowPlan {
  WindowParams p;
  int tile, mode, patch_slots;
  size_t lds;
};

int window_rows(const Conv16Params& c) { return c.nchunk / (c.cpt * c.S); }

// What a call brings and a plan does not depend on: addresses, the output's and the shortcut's layout.
void set_call(const Conv16Params& c, int N, WindowParams* p) {
  const uint32_t es = c.dt == FUPR_F32 ? 4 : 2;
  p->y_bytes = (uint32_t)c.M * (uint32_t)c.ycs * es;
  p->res_bytes = c.res ? (uint32_t)N * (uint32_t)(c.rH * c.rW) * (uint32_t)c.rcs * es : 0;
  p->x = c.x; p->x2 = c.x2; p->w = c.w; p->bias = c.bias; p->res = c.res; p->y = c.y;
  p->ycs = c.ycs; p->relu = c.relu;
  p->rH = c.rH; p->rW = c.rW; p->rcs = c.rcs; p->rss = c.rss; p->roff = c.roff;
  p->res_linear = c.rss == 1 && c.rH == c.P && c.rW == c.Q;
  if (c.keep) {
    p->keep = c.keep; p->keep_n = c.keep_n; p->yC = c.yC;
  }
}

bool plan_window(const Conv16Params& c, int N, int tile, int WF, int WK, WindowPlan* out) {
  const WindowTile& T = kTiles[tile];
  const int waves = WF * WK, R = window_rows(c);
  if (waves * 64 > T.threads) return false;
  WindowParams p{};
  const int mode = c.x2 ? kCat : (R == 1 && c.S == 1 && c.pad == 0 ? kOneTap : kWindow);
  const int es = c.dt == FUPR_F32 ? 4 : 2;
  if (es == 4 && (T.MT * T.NT > 8 || T.NT == 3)) return false;   // (not compiled for single precision)
  if (c.keep && (mode != kWindow || es != 2 || !listed_tile(T))) return false;
  const uint64_t x_bytes = (uint64_t)N * c.H * c.W * c.xcs * es;
  const uint64_t x2_bytes = c.x2 ? (uint64_t)N * c.H2 * c.W2 * c.xcs2 * es : 0;
  p.x_bytes = (uint32_t)x_bytes; p.x2_bytes = (uint32_t)x2_bytes; p.w_bytes = c.w_bytes;
  p.H = c.H; p.W = c.W; p.pix = c.xcs * es; p.pixels = N * c.H * c.W;
  p.P = c.P; p.Q = c.Q; p.PQ = c.PQ; p.M = c.M;
  p.R = R; p.S = c.S; p.stride = c.stride; p.pad = c.pad;
  p.Kp = c.Kp; p.cpt = c.cpt; p.nsteps = c.nsteps;
  p.H2 = c.H2; p.W2 = c.W2; p.pix2 = c.xcs2 * es; p.stride2 = c.stride2;
  p.WF = WF; p.WK = WK;
  while ((1 << p.log2_WF) < WF) ++p.log2_WF;
  if ((WF & (WF - 1)) || (WK & (WK - 1))) return false;
  const int BM = T.MT * 16, NF = WF * T.NT * 16;
  p.mgroups = (c.M + BM - 1) / BM;
  p.fgroups = (c.Kp + NF - 1) / NF;
  const int64_t total = (int64_t)p.mgroups * p.fgroups;
  if (total >= (int64_t(1) << 28)) return false;
  p.total = (int)total;
  p.per_xcd = tiles_per_xcd(p.total);
  p.filter_major = (uint64_t)c.w_bytes > x_bytes + x2_bytes;
  // LDS slots per pixel: 16 lanes read 16 bytes each of neighbouring output pixels, which is
  // free of bank conflicts at odd multiples of 32 bytes
  auto pad_slots = [&](int chunks) {
    int s = chunks;
    if (c.stride == 2 && mode == kWindow) return s | 1;
    while (s % 4 != 2) ++s;
    return s;
  };
  int pixels = 1 + BM;
  if (mode == kWindow) {
    if (!window_runs_are_whole(R, c.S, c.pad)) return false;
    pixels = (int)std::min<int64_t>(most_run_pixels(BM, R, c.S, c.stride, c.H, c.W, c.P, c.Q), 1 << 20);
    p.table_bytes = (int)(p.nsteps + (T.D + 2 * T.G + 2) * WK) * 32;
  }
  p.live = c.x2 ? std::min(c.split, c.xcs / 8) : c.cpt;
  p.slots = pad_slots(c.x2 ? c.split : round_up(c.cpt, mode == kOneTap ? 4 : 1));
  if (c.x2) {
    p.split_steps = c.split / 4;
    p.live2 = c.cpt - c.split;
    p.slots2 = pad_slots(round_up(p.live2, 4));
  }
  size_t end = round_up_sz((size_t)pixels * p.slots * 16, 1024);
  if (c.x2) {
    p.patch2_at = (int)end;
    end += round_up_sz((size_t)pixels * p.slots2 * 16, 1024);
  }
  p.table_at = (int)end;
  p.pixels_at = p.table_at + p.table_bytes;
  if (mode == kWindow) end = (size_t)p.pixels_at + (size_t)BM * 8;
  out->patch_slots = pixels * (p.slots + p.slots2);
  // The partial sums lie beside the patch, which saves a barrier, where no workgroup less fits a compute unit for it.
  const int givers = WK == 1 ? 0 : all_partial_sums(T.MT * T.NT) ? WK : WK - 1;
  const size_t reduce = (size_t)givers * WF * T.MT * T.NT * 1024, beside = round_up_sz(end, 1024) + reduce;
  out->lds = std::max(end, reduce);
  const int by_waves = std::max(1, std::min(32 / waves, 512 / T.vgprs * 4 / waves));
  if (reduce > 0 && beside <= kLdsLimit && std::min((int)(kLdsLimit / out->lds), by_waves) <= (int)(kLdsLimit / beside)) {
    p.part_at = (int)round_up_sz(end, 1024);
    out->lds = beside;
  }
  if (c.keep) {
    p.keep_at = (int)round_up_sz(out->lds, 16);
    out->lds = (size_t)p.keep_at + (size_t)NF * 4;
  }
  if (out->lds > kLdsLimit) return false;
  p.divPQ = fast_div(p.PQ); p.divQ = fast_div(p.Q); p.divC = fast_div(p.cpt); p.divS = fast_div(p.S);
  p.divSlots = fast_div(p.slots); p.divSlots2 = fast_div(std::max(p.slots2, 1));
  p.divG = fast_div(p.filter_major ? p.mgroups : p.fgroups);
  out->p = p;
  out->tile = tile;
  out->mode = mode;
  return true;
}

// Two convolutions of one tensor that do not need each other (a block's first 3 x 3 and its projection shortcut) as
// one launch: blockIdx.y says which.  The window has the plan it has alone, the 1 x 1 convolution the cut of its reduction,
// hence both their bits.  Saves a launch, whose start and end cost 3600 clocks with nothing in between, and the smaller one
// runs where the other leaves compute units free.  The grid and the waves of a workgroup are the larger one's: waves that the
// other does not need end at once, and so do workgroups beyond its tiles (tile_of_workgroup).
struct TwoWindowParams {
  WindowParams p[2];
};

template <int EL, int WINDOW, int TAP>
__global__ __launch_bounds__(kTiles[WINDOW].threads, kTiles[WINDOW].min_waves) void conv_window_two_kernel(const TwoWindowParams two) {
  constexpr WindowTile A = kTiles[WINDOW], B = kTiles[TAP];
  if (blockIdx.y == 0) window_tile<EL, kWindow, A.MT, A.NT, A.D, A.G, false>(two.p[0], 0);
  else window_tile<EL, kOneTap, B.MT, B.NT, B.D, B.G, false>(two.p[1], 1);
}
// The tiles that it is compiled for, of the window and of the 1 x 1 convolution: those that plans reach.  Of 3800 pairs of
// basic-block networks at 96 - 224 pixels 48 % run as 32 x 16 beside 16 x 16, 42 % as 16 x 16 beside 16 x 16, 4 % as 32 x 48 beside
// it, 5 % with 32 x 16 for the 1 x 1 convolution; 64 x 32 and 64 x 48 are 1 % of 14 000 pairs of any sizes.
constexpr int kTwoWindow[] = {0, 2, 4, 6, 7}, kTwoTap[] = {0, 2};

template <int EL, int WINDOW, int TAP>
fupr_status launch_two_as(const WindowPlan& a, const WindowPlan& b, hipStream_t st) {
  auto kernel = conv_window_two_kernel<EL, WINDOW, TAP>;
  const size_t lds = std::max(a.lds, b.lds);
  if (lds > 64 * 1024) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
    if (attr != hipSuccess) return FUPR_ERR_LAUNCH;
  }
  TwoWindowParams two{{a.p, b.p}};
  void* list[] = {&two};
  const unsigned blocks = (unsigned)std::max(a.p.per_xcd, b.p.per_xcd) * kXcds;
  const unsigned threads = (unsigned)std::max(a.p.WF * a.p.WK, b.p.WF * b.p.WK) * 64;
  return launched(hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(blocks, 2), dim3(threads), list, lds, st),
                  "conv_window_two_kernel");
}

template <int EL, int WINDOW>
fupr_status launch_two_of(const WindowPlan& a, const WindowPlan& b, hipStream_t st) {
  switch (b.tile) {
    case 0: return launch_two_as<EL, WINDOW, 0>(a, b, st);
    case 2: return launch_two_as<EL, WINDOW, 2>(a, b, st);
  }
  return FUPR_ERR_LIMIT;
}

template <int EL>
fupr_status launch_two(const WindowPlan& a, const WindowPlan& b, hipStream_t st) {
  switch (a.tile) {
    case 0: return launch_two_of<EL, 0>(a, b, st);
    case 2: return launch_two_of<EL, 2>(a, b, st);
    case 4: return launch_two_of<EL, 4>(a, b, st);
    case 6: return launch_two_of<EL, 6>(a, b, st);
    case 7: return launch_two_of<EL, 7>(a, b, st);
  }
  return FUPR_ERR_LIMIT;
}

template <int EL, int MODE, int TILE, bool IX>
fupr_status launch_as(const WindowPlan& plan, hipStream_t st) {
  constexpr WindowTile T = kTiles[TILE];
  if constexpr ((EL == FUPR_F32 && (T.MT * T.NT > 8 || T.NT == 3)) || (IX && !listed_tile(T))) {
    return FUPR_ERR_LIMIT;
  } else {
  auto kernel = conv_window_kernel<EL, MODE, T.MT, T.NT, T.D, T.G, T.threads, T.min_waves, IX>;
  if (plan.lds > 64 * 1024) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
    if (attr != hipSuccess) return FUPR_ERR_LAUNCH;
  }
  void* list[] = {const_cast<WindowParams*>(&plan.p)};
  return launched(hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)(plan.p.per_xcd * kXcds)),
                                  dim3(plan.p.WF * plan.p.WK * 64), list, plan.lds, st),
                  "conv_window_kernel");
  }
}

template <int EL, int MODE, bool IX = false>
fupr_status dispatch(const WindowPlan& plan, hipStream_t st) {
  switch (plan.tile) {
#define FUPR_TILE(i) case i: return launch_as<EL, MODE, i, IX>(plan, st);
    FUPR_TILE(0) FUPR_TILE(1) FUPR_TILE(2) FUPR_TILE(3) FUPR_TILE(4) FUPR_TILE(5)
    FUPR_TILE(6) FUPR_TILE(7) FUPR_TILE(8) FUPR_TILE(9) FUPR_TILE(10) FUPR_TILE(11)
#undef FUPR_TILE
  }
  return FUPR_ERR_LIMIT;
}

int num_compute_units() {
  static const int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      return 256;
    }
    return n;
  }();
  return cus;
}

// Estimated clocks of a plan.  The constants are a fit over 420 layer shapes (1 - 256 images of the
// ImageNet networks' layers, and arbitrary ones) x every tile and wave arrangement, 12 800 launches:
// the plan with the least estimate is 2.6 % slower than the best one in the mean, 27 % at worst.
double estimate(const Conv16Params& c, const WindowPlan& plan) {
  const WindowParams& p = plan.p;
  const WindowTile& T = kTiles[plan.tile];
  const int waves = p.WF * p.WK, cus = num_compute_units();
  const int per_cu = (p.total + cus - 1) / cus;                    // workgroups of the busiest unit
  const int fit = std::max(1, std::min({(int)(kLdsLimit / plan.lds), 32 / waves, 512 / T.vgprs * 4 / waves}));
  const int rounds = (per_cu + std::min(per_cu, fit) - 1) / std::min(per_cu, fit);
  const double steps = round_up((p.nsteps + p.WK - 1) / p.WK, T.G);
  const double clocks = c.dt == FUPR_F32 ? 128.0 : 16.0;           // of the matrix pipe per tile and step
  const double tiles = T.MT * T.NT, slots = plan.patch_slots, out = tiles * 256.0 * p.WF * (c.res ? 2 : 1);
  // what a workgroup takes of its compute unit: the matrix pipe and the vector instructions beside
  // it, what it reads (45 bytes per clock), LDS
  const double mfma = waves * steps * tiles * clocks / 4.0 + 0.376 * waves * steps * (40.35 * T.MT + 26.78) / 4.0;
  const double reads = (slots * 16.0 * p.live / p.slots + (double)p.nsteps * p.WF * T.NT * 1024.0) / 45.1;
  const double lds = waves * steps * T.MT * 11.55 + slots * 0.25;
  const double work = std::max({mfma, reads, lds}) + out * 0.0185;
  // and how long it takes when it has the unit to itself
  const double alone = 3356.0 + 82.0 * waves + out / waves * 0.67 + slots / (waves * 64.0) * 45.3 +
                       steps * (34.1 / T.G + tiles * clocks) +
                       (p.WK > 1 ? 455.0 + (p.WK - 1) * tiles * 460.0 / p.WK : 0.0) +
                       tiles * (c.res ? 87.0 : 58.0) / p.WK;
  return 2893.0 + std::max(rounds * alone, per_cu * work + 0.62 * alone);
}

// The plan with the least estimate among those that fit; only those that cut the reduction into
// WK parts if WK > 0.
bool pick_window(const Conv16Params& c, int N, int only_WK, WindowPlan* best) {
  // The tuning switch window_tile=<index>x<waves along the filters>x<waves along the reduction>
  // forces a tile.
  char text[32];
  if (tuning_text("window_tile", text, sizeof(text))) {
    int tile = -1, wf = 1, wk = 4;
    if (std::sscanf(text, "%dx%dx%d", &tile, &wf, &wk) != 3 || tile < 0 || tile >= kNumTiles) return false;
    if (wf < 1 || wk < 1 || wf * wk > 16) return false;
    return plan_window(c, N, tile, wf, wk, best);
  }
  // A 1 x 1 reduction of at most four steps is not cut: all of its weights are in flight at once
  // anyway, and its sums are those of a pair of 1 x 1 convolutions in one launch (conv1x1.hip).
  const bool whole = c.dt != FUPR_F32 && c.nchunk == c.cpt && c.nsteps <= 4;
  double least = 0.0;
  bool any = false;
  for (int tile = 0; tile < kNumTiles; ++tile)
    for (int wf = 1; wf <= 8; wf *= 2) {
      if (wf > 1 && (wf / 2) * kTiles[tile].NT * 16 >= c.Kp) break;   // half of the waves would be idle
      for (int waves = whole ? wf : 4; waves <= (whole ? wf : 8); waves *= 2) {
        WindowPlan plan;
        if (waves < wf || (only_WK > 0 && waves / wf != only_WK)) continue;
        if (!plan_window(c, N, tile, wf, waves / wf, &plan)) continue;
        const double cost = estimate(c, plan);
        if (!any || cost < least) {
          *best = plan;
          least = cost;
          any = true;
        }
      }
    }
  return any;
}

// How the reduction is cut decides the order of the sums, so it is chosen for the batch the caller
// runs (plan_N), the tile for the images of this launch: sub-batches of one batch give its bits.
bool pick_for_batch(const Conv16Params& c, int N, WindowPlan* plan) {
  if (c.plan_N <= 0 || c.plan_N == N) return pick_window(c, N, 0, plan);
  Conv16Params whole = c;
  whole.M = (int)((int64_t)c.plan_N * c.PQ);
  return pick_window(whole, c.plan_N, 0, plan) && pick_window(c, N, plan->p.WK, plan);
}

// The choice is a function of sizes alone; each thread remembers its last answer for every one of 128
// hashes of the sizes (about 100 plans are weighed for one, 4 - 7 us of host time; sizes with one hash
// replace each other: 11 of the 52 operators of an irregular ResNet-50 are weighed on every pass).
struct Sizes {
  int dt, N, plan_N, H, W, P, Q, M, R, S, stride, pad, Kp, cpt, xcs, split, xcs2, stride2, res, two, H2, W2, listed;
  bool operator==(const Sizes& o) const { return std::memcmp(this, &o, sizeof(o)) == 0; }
};
struct Remembered {
  Sizes sizes;
  int state;             // 0: empty, 1: a plan, -1: none fits
  WindowPlan plan;
};

bool plan_for(const Conv16Params& c, int N, WindowPlan* plan) {
  if (tuning_any()) return pick_for_batch(c, N, plan);
  const WithoutTuning no_switches;   // (one that another thread sets meanwhile is in no plan that is kept)
  constexpr int kEntries = 128;
  thread_local Remembered table[kEntries];
  const Sizes z = {(int)c.dt, N, c.plan_N, c.H, c.W, c.P, c.Q, c.M, window_rows(c), c.S, c.stride, c.pad, c.Kp,
                   c.cpt, c.xcs, c.split, c.xcs2, c.stride2, c.res ? 1 : 0, c.x2 ? 1 : 0, c.H2, c.W2, c.keep ? 1 : 0};
  uint32_t h = 2166136261u;
  for (size_t i = 0; i < sizeof(z) / sizeof(int); ++i)
    h = (h ^ (uint32_t)reinterpret_cast<const int*>(&z)[i]) * 16777619u;
  Remembered& r = table[(h ^ (h >> 15)) % kEntries];
  if (r.state == 0 || !(r.sizes == z)) {
    r.state = pick_for_batch(c, N, &r.plan) ? 1 : -1;
    r.sizes = z;
  }
  if (r.state > 0) *plan = r.plan;
  return r.state > 0;
}

// Sizes for which this kernel is the faster one.  (The switches that choose among the other
// kernels' tiles ask for those kernels.)
bool wanted(const Conv16Params& c, int N) {
  if (tuning_off("conv_window")) return false;
  const int R = window_rows(c);
  if (c.keep && (c.dt == FUPR_F32 || (R == 1 && c.S == 1))) return false;
  if (R * c.S > kMaxTaps || (c.x2 && c.split % 8 != 0)) return false;
  const uint64_t es = c.dt == FUPR_F32 ? 4 : 2;
  if ((uint64_t)c.nsteps * 64 * (uint64_t)c.Kp >= kOutside) return false;   // bytes of the weights (w_bytes has 32 bits)
  for (uint64_t elements : {(uint64_t)N * c.H * c.W * c.xcs, (uint64_t)c.M * c.ycs,
                            c.x2 ? (uint64_t)N * c.H2 * c.W2 * c.xcs2 : 0,
                            c.res ? (uint64_t)N * c.rH * c.rW * c.rcs : 0})
    if (elements * es >= kOutside) return false;
  if (c.res && c.dt != FUPR_F32 && c.roff % 8 != 0) return false;   // 16-byte shortcut loads
  if (tuning_any()) {
    char text[64];
    for (const char* other : {"patch_tile", "pipe_tile", "pipe_order", "stream_tile", "stream_blocks", "conv_tile"})
      if (tuning_text(other, text, sizeof(text))) return false;
    if (tuning_text("window_tile", text, sizeof(text))) return true;
  }
  if (c.dt == FUPR_F32) return true;
  const double M = (double)(c.plan_N > 0 ? c.plan_N : N) * c.PQ;
  if (R == 1 && c.S == 1) {
    // Layers that are bound by the bytes of their tensors stay with the 1 x 1 kernels that keep
    // loads in flight across tiles (32 -> 256 channels with a shortcut at 56 x 56 x 26, 89 MB: 19.3
    // against 26.7 us; 1024 -> 204 at 14 x 14 x 87, 42 MB: 19.5 against 23.0 us); below they spend
    // most of their time starting up (32 -> 256 at 56 x 56 x 10, 34 MB: 10.6 against 8.6 us).
    const double bytes = 2.0 * M * (c.cpt * 8.0 + c.ycs * (c.res ? 2.0 : 1.0));
    // Reductions so deep that no 64-pixel tile fits LDS read all weights for every 32 pixels: from
    // 3.2 thousand million products on the pipelined kernel's large tiles are faster (two tensors,
    // 1280 -> 2048 channels, on 1568 pixels 25.7 against 20.6 us, on 3136 60.5 against 28.0; on
    // 1176 pixels, 3.1 thousand million, 18.2 against 20.2).
    if (c.cpt > 150 && M * (c.cpt * 8.0) * c.Kp > 3.2e9 && conv1x1_pipe_applies(c)) return false;
    return bytes <= 36e6;
  }
  // Listed channels are updated two bytes at a time here and mostly 16 at a time by the patch
  // kernel, whose start costs more (this kernel against that one: 180 -> 180 of 256
  // at 14 x 14 x 12 8.4 against 12.6 us, 90 -> 90 of 128 at 28 x 28 x 20 11.7 against 15.7; 45 -> 45 of
  // 64 at 56 x 56 x 12, 1.8 million sums, 13.6 against 12.9, x 64 47.8 against 37.7).
  if (c.keep && M * c.Kp > 1.6e6) return false;
  // Thin reductions over very many pixels: the patch kernel keeps its weights in LDS from tile
  // to tile (51 -> 30 channels at 56 x 56 x 149: 32.2 against 35.6 us; x 64: 22.3 against 23.1 the
  // other way).  With 33 to 64 channels that pays from some 140 000 pixels on (51 -> 45 at 56 x 56 x
  // 64 27.7 against 25.5 us, x 48 23.0 against 22.6, x 32 17.7 against 18.6), with at most 32
  // channels and 32 filters from 90 000 on (32 -> 32 x 64 18.9 against 16.5, x 32 13.5 against
  // 12.7, x 24 10.5 against 12.1); measured on images of that width, and padded as that kernel wants it.
  const bool measured = c.Q <= 64 && c.pad == 1 && c.cpt >= 2 && !c.keep;
  const double many = measured && c.cpt > 4 ? 140e3 : measured && c.Kp <= 32 ? 90e3 : 262144;
  return !(R == 3 && c.S == 3 && c.stride == 1 && c.cpt <= 8 && M > many);
}

// What the launch list calls it: the family of kernels the layer belongs to, and the tile.
const char* name_of(const Conv16Params& c, int tile) {
  if (c.dt == FUPR_F32) return kTiles[tile].single;
  const int R = window_rows(c);
  if (R == 1 && c.S == 1) return kTiles[tile].one_tap;
  return R == 3 && c.S == 3 && c.stride == 1 && c.cpt >= 2 ? kTiles[tile].three : kTiles[tile].other;
}

}  // namespace

bool conv_window_applies(const Conv16Params& c, int N) {
  WindowPlan plan;
  return wanted(c, N) && plan_for(c, N, &plan);
}

const char* conv_window_name(const Conv16Params& c, int N) {
  WindowPlan plan;
  return plan_for(c, N, &plan) ? name_of(c, plan.tile) : "conv16t_w";
}

static fupr_status dispatch_window(const WindowPlan& plan, fupr_dtype dt, bool listed, hipStream_t st) {
  const bool bf16 = dt == FUPR_BF16;
  if (dt == FUPR_F32)
    return plan.mode == kOneTap ? dispatch<FUPR_F32, kOneTap>(plan, st) : dispatch<FUPR_F32, kWindow>(plan, st);
  if (plan.mode == kCat)
    return bf16 ? dispatch<FUPR_BF16, kCat>(plan, st) : dispatch<FUPR_F16, kCat>(plan, st);
  if (plan.mode == kOneTap)
    return bf16 ? dispatch<FUPR_BF16, kOneTap>(plan, st) : dispatch<FUPR_F16, kOneTap>(plan, st);
  if (listed)
    return bf16 ? dispatch<FUPR_BF16, kWindow, true>(plan, st) : dispatch<FUPR_F16, kWindow, true>(plan, st);
  return bf16 ? dispatch<FUPR_BF16, kWindow>(plan, st) : dispatch<FUPR_F16, kWindow>(plan, st);
}

// Both convolutions' plans, if they can run as one launch.
static bool plan_two(const Conv16Params& window, const Conv16Params& tap, int N, WindowPlan* a, WindowPlan* b) {
  if (window.dt == FUPR_F32 || window.keep || tap.keep || window.x2 || tap.x2 || tuning_off("conv_two")) return false;
  // Up to some 1800 output pixels two launches in one are the faster ones, although a workgroup of the 1 x 1 convolution
  // (3 - 18 KB of LDS) then takes the room of one of the other's (30 - 152 KB).  Pairs of ResNet-18 and -34 one at a time, 1 - 250
  // images of 128 and 224 pixels, 0 - 50 % pruned, us of the network: up to 1764 pixels -3.3 .. -0.2, but for 64 channels of 128
  // filters pruned by half at 1024 and 1536 pixels (+0.6, +1.2); at 2048 to 5120 -3.6 .. +5.1; above -7 .. +7.2 of 200 - 1160.
  if (window.M > 1800) return false;
  if (!wanted(window, N) || !wanted(tap, N) || !plan_for(window, N, a) || !plan_for(tap, N, b)) return false;
  if (a->mode != kWindow || b->mode != kOneTap) return false;
  if (std::find(std::begin(kTwoWindow), std::end(kTwoWindow), a->tile) == std::end(kTwoWindow)) return false;
  // The 1 x 1 convolution with as many waves as the other has, its reduction cut as when it is alone: with the plan it has alone,
  // often one or two waves of a workgroup of eight, ResNet-34 of 20 images took 346.0 us in place of 344.5, ResNet-18 of 12 138.2
  // in place of 137.1, of one image 76.4 in place of 76.7.
  const int waves = a->p.WF * a->p.WK, WK = b->p.WK;
  const int only = tuning_int("two_tap", -1);
  double least = 0.0;
  bool any = false;
  for (int tile : kTwoTap) {
    WindowPlan plan;
    if (only >= 0 && only != tile) continue;
    const int WF = waves / WK;
    if (WF < 1 || (WF > 1 && (WF / 2) * kTiles[tile].NT * 16 >= tap.Kp) || !plan_window(tap, N, tile, WF, WK, &plan)) continue;
    const double cost = estimate(tap, plan);
    if (any && cost >= least) continue;
    *b = plan;
    least = cost;
    any = true;
  }
  return any;
}

bool conv_window_two_applies(const Conv16Params& window, const Conv16Params& tap, int N) {
  WindowPlan a, b;
  return plan_two(window, tap, N, &a, &b);
}

bool launch_conv_window_two(const Conv16Params& window, const Conv16Params& tap, int N, void* stream, fupr_status* status) {
  WindowPlan a, b;
  if (!plan_two(window, tap, N, &a, &b)) return false;
  set_call(window, N, &a.p);
  set_call(tap, N, &b.p);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  *status = window.dt == FUPR_BF16 ? launch_two<FUPR_BF16>(a, b, st) : launch_two<FUPR_F16>(a, b, st);
  return true;
}

bool launch_conv_window(const Conv16Params& c, int N, void* stream, fupr_status* status) {
  WindowPlan plan;
  if (!wanted(c, N) || !plan_for(c, N, &plan)) return false;
  set_call(c, N, &plan.p);
  *status = dispatch_window(plan, c.dt, c.keep != nullptr, reinterpret_cast<hipStream_t>(stream));
  return true;
}

}  // namespace fupr
