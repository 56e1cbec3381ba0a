// A bottleneck block's 3 x 3 convolution, its last 1 x 1 convolution (with the shortcut, or over two
// concatenated tensors) and the next block's first 1 x 1 convolution in one launch (Table II's
// bottleneck blocks; Sec. III: what an operator boundary costs).
//
// The three operators of one tile of BM output pixels never leave the workgroup: the 3 x 3
// convolution's output stays in LDS, and the block's output, which has to be written anyway, is
// multiplied by the next convolution's filters from LDS instead of being read back.  Per pixel and
// block that removes 2 x (narrow + narrow) + wide channels of traffic and two launches.
//
//   * Phase 1, 3 x 3: the tile's input, one run of pixels (window_patch.h), goes to LDS once; a
//     wave takes a pair of filter tiles and a share of the pixels.
//   * Phase 2, 1 x 1: groups of WAVES x 32 filters; a wave takes 32 of them for all pixels of the
//     tile, adds the shortcut, rounds, and writes the result to memory and to LDS.
//   * Phase 3, 1 x 1: the group's channels times the next convolution's filters, into accumulators
//     that live as long as the tile.  One barrier per group (its buffer in LDS alternates).
//   * Weights never pass through LDS: a wave loads the MFMA fragments that it alone needs from L2 a
//     few steps ahead, across phases and barriers.
//   * The 3 x 3's reduction is cut over waves that have no filters of their own; the partial sums meet in
//     LDS in the order of the waves.
//
// Measured, three launches -> one (us, event-timed; the channels in, 3 x 3, wide, next): 64, 64, 512, 64 at
// 28 x 28 x 64 images 57 -> 39; 128, 128, 1024, 128 at 14 x 14 x 64 46 -> 28, x 9 22.5 -> 19.4 (but longer inside a network: stays apart), one image 19.3
// against 22 here (stays apart); 32, 32, 256, 64 at 56 x 56 x 9 25.7 -> 15.4, one image 19 -> 9.7, x 64 55
// against 59 (stays apart).  ResNet-50: 64 images 772 -> 670, nine irregular ones of 193 x 193 296 -> 269.
// What bounds it: weights, which every tile reads anew through the vector path (with the pixels 21 - 41 bytes per clock
// and compute unit over whole launches, by counters), and the start and the 3 x 3, which wait for memory with one workgroup
// per compute unit; at large batches little is in flight: 1.9 - 3.0 TB/s counted at 256 images where the launches
// apart stream at 4.7 - 4.8.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "bottleneck.h"
#include "device_utils.h"
#include "fupr.h"
#include "layout.h"
#include "recall.h"
#include "tuning.h"
#include "window_patch.h"

namespace fupr {
namespace {

constexpr uint32_t kOutside = 0x80000000u;   // beyond every tensor this kernel accepts
constexpr size_t kLdsLimit = 160 * 1024;
constexpr int kComputeUnits = 256;
constexpr int kSharers = 32;                 // workgroups of an XCD that run at once, at least

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef void __attribute__((address_space(3)))* LdsPtr;

struct BlockParams {
  const uint16_t *x, *x2, *w1, *w2, *w3, *res;
  const float *b1, *b2, *b3;
  uint16_t *y, *h;
  uint32_t x_bytes, x2_bytes, w1_bytes, w2_bytes, w3_bytes, res_bytes, y_bytes, h_bytes;
  int H, W, pix, pixels;            // input of the 3 x 3: extent, bytes per pixel, pixels of the batch
  int Q, PQ, M, stride;
  int Kp1, cpt, steps1;
  int Kp2, steps2, split_steps;     // steps from split_steps on read x2
  int Kp3, steps3;
  int ycs, hcs, relu1, relu2, relu3;
  int H2, W2, pix2, stride2;
  int slots, slots_mid, slots2, live, live2;
  int table_at, pixels_at, mid_at, patch2_at, spare_at;   // LDS byte offsets (the patch starts at 0)
  int WF1;                          // waves along the filters of the 3 x 3 (a power of two)
  int groups, total, per_xcd;
  FastDiv divPQ, divQ, divC, divSlots, divSlots2;
};

__device__ __forceinline__ uint32_t clamp_below(uint32_t v, uint32_t floor2) {
  const short2_t a = __builtin_bit_cast(short2_t, v), f = __builtin_bit_cast(short2_t, floor2);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, f));
}

__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, soff, 0));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
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

// MT tiles of 16 pixels, WAVES waves; D: steps of weights in flight per wave (even); NT3: filter
// tiles per wave of the third convolution, 0: there is none.
template <bool BF, int MT, int WAVES, int D, int NT3>
__global__ __launch_bounds__(WAVES * 64, 2) void bottleneck_kernel(const BlockParams p) {
  touch_arguments<sizeof(BlockParams)>();
  extern __shared__ uint4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  const uint32_t lds_base = (uint32_t)(uintptr_t)(LdsPtr)lds;
  constexpr int BM = MT * 16, THREADS = WAVES * 64, GF = WAVES * 32;
  constexpr int kWidePixel = GF * 2 + 32;             // bytes: an odd multiple of 32
  constexpr int kWideBytes = BM * kWidePixel;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
  if (tile >= p.total) return;
  const int m0 = tile * BM;

  // phase 1: WF waves lie along the filters (pairs of tiles), WK take every WK-th step of the reduction
  const int WF = p.WF1, WK = WAVES / WF;
  const int wf = wave & (WF - 1), wk = wave / WF;

  const __amdgpu_buffer_rsrc_t w1r = buffer_of(p.w1, p.w1_bytes);
  const __amdgpu_buffer_rsrc_t w2r = buffer_of(p.w2, p.w2_bytes);
  const __amdgpu_buffer_rsrc_t w3r = buffer_of(p.w3, p.w3_bytes);
  // byte offset of the lane's fragment of a filter tile (a tile that does not exist reads the last one)
  auto fragment = [&](int f, int Kp) { return (uint32_t)(g * Kp + min(f, Kp - 16) + li) * 16u; };

  uint4 a[D][2];
  uint32_t a_off[2];
  auto load_a = [&](const __amdgpu_buffer_rsrc_t& r, int step, int last, int Kp, uint4* av) {
    const uint32_t so = (uint32_t)min(step, last) * ((uint32_t)Kp * 64u);
    av[0] = load16(r, a_off[0], so);
    av[1] = load16(r, a_off[1], so);
  };

  // ---- the pixels' input into LDS: patch pixel 0 is zeros, pixel 1 + i is input pixel first + i ----
  auto split_pixel = [&](int m, int* n, int* pp, int* qq) {
    *n = div_by(m, p.divPQ);
    const int rem = m - *n * p.PQ;
    *pp = div_by(rem, p.divQ);
    *qq = rem - *pp * p.Q;
  };
  auto origin_of = [&](int m) {
    int n, pp, qq;
    split_pixel(m, &n, &pp, &qq);
    return window_origin(n, pp, qq, p.H, p.W, p.stride, 1);
  };
  const int first = origin_of(m0);
  const int last = origin_of(min(m0 + BM, p.M) - 1) + window_reach(3, 3, p.W);
  {
    const i32x4 xr = make_rsrc(p.x, p.x_bytes);
    const int step_pix = div_by(THREADS, p.divSlots), step_c = THREADS - step_pix * p.slots;   // (scalar)
    int pixel = div_by(tid, p.divSlots), c = tid - pixel * p.slots;
    pixel += first - 1;                       // input pixel
    const int zero = first - 1;
    uint32_t off = (uint32_t)pixel * (uint32_t)p.pix + (uint32_t)c * 16u;
    const uint32_t step_off = (uint32_t)(step_pix * p.pix + step_c * 16), wrap_off = (uint32_t)(p.pix - p.slots * 16);
    const int count = (1 + last - first + 1) * p.slots;
    for (int base = wave * 64; base < count; base += THREADS) {
      const bool ok = c < p.live && pixel != zero && (unsigned)pixel < (unsigned)p.pixels;
      load_to_lds(xr, ok ? off : kOutside, lds_base + base * 16);
      c += step_c;
      pixel += step_pix;
      off += step_off;
      const bool wrap = c >= p.slots;
      c -= wrap ? p.slots : 0;
      pixel += wrap ? 1 : 0;
      off += wrap ? wrap_off : 0u;
    }
  }
  if (p.x2) {   // the second tensor's pixel of every output pixel
    const i32x4 x2r = make_rsrc(p.x2, p.x2_bytes);
    const int count = BM * p.slots2;
    for (int base = wave * 64; base < count; base += THREADS) {
      const int slot = base + lane;
      const int pixel = div_by(slot, p.divSlots2), c = slot - pixel * p.slots2, m = m0 + pixel;
      int n, pp, qq;
      split_pixel(m, &n, &pp, &qq);
      const uint32_t in = (uint32_t)((n * p.H2 + pp * p.stride2) * p.W2 + qq * p.stride2);
      load_to_lds(x2r, c < p.live2 && m < p.M ? in * (uint32_t)p.pix2 + (uint32_t)c * 16u : kOutside,
                  lds_base + p.patch2_at + base * 16);
    }
  }

  // All workgroups of an XCD walk the weights in step, and the XCD's L2 holds none of them yet: left to
  // the loop, every line would be waited for at the latency of memory, a few steps at a time.  So the
  // first workgroups of an XCD ask for all of them at once, a share each, into a spare KB of LDS.
  {
    const int sharers = min(p.per_xcd, kSharers) * WAVES;
    const int me = (int)(blockIdx.x >> 3) * WAVES + wave;
    auto ask = [&](const uint16_t* w, uint32_t bytes) {
      const i32x4 r = make_rsrc(w, bytes);
      for (uint32_t at = (uint32_t)me * 1024u; at < bytes; at += (uint32_t)sharers * 1024u)
        load_to_lds(r, at + (uint32_t)lane * 16u, lds_base + p.spare_at);
    };
    if (me < sharers) {
      ask(p.w1, p.w1_bytes);
      ask(p.w2, p.w2_bytes);
      if constexpr (NT3 > 0) ask(p.w3, p.w3_bytes);
    }
  }

  // the first weights and all biases travel with the pixels
#pragma unroll
  for (int t = 0; t < 2; ++t) a_off[t] = fragment(wf * 32 + t * 16, p.Kp1);
#pragma unroll
  for (int d = 0; d < D; ++d) load_a(w1r, wk + d * WK, p.steps1 - 1, p.Kp1, a[d]);

  const __amdgpu_buffer_rsrc_t rr = buffer_of(p.res, p.res_bytes);
  const __amdgpu_buffer_rsrc_t yr = buffer_of(p.y, p.y_bytes);
  const __amdgpu_buffer_rsrc_t b2r = buffer_of(p.b2, (uint32_t)p.Kp2 * 4u);
  // after the exchange between 16-lane rows lane (pixel, g) holds channels (g >> 1) * 8 .. + 7 of
  // filter tile g & 1 of its wave's two
  const int own = (g & 1) * 16 + (g >> 1) * 8;
  uint32_t row[MT];      // byte offset of the lane's pixel in the block's output, and in the shortcut
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m0 + mt * 16 + li;
    row[mt] = m < p.M ? (uint32_t)(m * p.ycs + own) * 2u : kOutside;
  }
  // (Every load from here on is issued whatever the layer: waits are counted, and a load that may or
  // may not be there makes the compiler wait for more than it needs.  Without a shortcut its extent is
  // 0: zeros.)
  u32x4 r4[MT];
  auto load_res = [&](int f0, int mt) {
    r4[mt] = __builtin_amdgcn_raw_buffer_load_b128(rr, f0 + own < p.ycs ? row[mt] + (uint32_t)f0 * 2u : kOutside, 0, 0);
  };
  f32x4 b2v[2];
  auto load_b2 = [&](int f0, int t) {
    b2v[t] = __builtin_bit_cast(
        f32x4, __builtin_amdgcn_raw_buffer_load_b128(b2r, (uint32_t)(f0 + t * 16 + g * 4) * 4u, 0, 0));
  };
  load_b2(wave * 32, 0);
  load_b2(wave * 32, 1);
  constexpr int N3 = NT3 > 0 ? NT3 : 1;
  // (a multiple of D: loaded in equal parts with the steps of phase 2's last round)
  constexpr int DC = N3 == 1 ? WAVES : N3 == 2 ? 4 : 2;    // steps of phase 3 weights in flight
  const bool third = NT3 > 0 && wave * (N3 * 16) < p.Kp3;   // this wave has filters of the third convolution
  f32x4 acc3[MT][N3];
  f32x4 b1v[2];
  {
    const float* b1 = p.b1;
#pragma unroll
    for (int t = 0; t < 2; ++t)
      b1v[t] = *reinterpret_cast<const f32x4*>(b1 + min(wf * 32 + t * 16, p.Kp1 - 16) + g * 4);
    if constexpr (NT3 > 0) {
      const float* b3 = p.b3;
#pragma unroll
      for (int t = 0; t < N3; ++t) {
        const f32x4 b4 = *reinterpret_cast<const f32x4*>(b3 + min((wave * N3 + t) * 16, p.Kp3 - 16) + g * 4);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc3[mt][t] = b4;
      }
    }
  }

  // per chunk of 8 channels: its LDS distance from the window origin, and its tap
  u32x2* table = reinterpret_cast<u32x2*>(lds + p.table_at);
  for (int j = tid; j < (p.steps1 + 1) * 4; j += THREADS) {
    const int tap = div_by(j, p.divC), cc = j - tap * p.cpt;
    const int r = (tap * 11) >> 5, s = tap - r * 3;   // (tap / 3 for taps below 16)
    const bool ok = tap < 9;
    u32x2 e;
    e[0] = ok ? (uint32_t)(((r * p.W + s) * p.slots + cc) * 16) : 0u;
    e[1] = ok ? (uint32_t)tap : 31u;
    table[j] = e;
  }
  // per pixel of the tile: LDS address of the window origin, and which taps lie inside the image
  u32x2* pixel_table = reinterpret_cast<u32x2*>(lds + p.pixels_at);
  for (int i = tid; i < BM; i += THREADS) {
    const int m = m0 + i;
    int n, pp, qq;
    split_pixel(min(m, p.M - 1), &n, &pp, &qq);
    const int ih = pp * p.stride - 1, iw = qq * p.stride - 1;
    const int lo = max(0, -iw), hi = min(3, p.W - iw);
    const uint32_t cols = hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
    uint32_t taps = 0;
    for (int r = 0; r < 3; ++r) taps |= (uint32_t)(ih + r) < (uint32_t)p.H ? cols << (r * 3) : 0u;
    u32x2 e;
    e[0] = (uint32_t)((1 + (n * p.H + ih) * p.W + iw - first) * p.slots * 16);
    e[1] = m < p.M ? taps : 0u;
    pixel_table[i] = e;
  }
  // the channels between the 3 x 3 convolution's filters and the end of the second one's step are zeros
  {
    const int from = p.Kp1 / 8, per = (p.x2 ? p.split_steps : p.steps2) * 4 - from;
    for (int i = tid; i < BM * per; i += THREADS) {
      const int pixel = i / per, c = from + i - pixel * per;
      *reinterpret_cast<uint4*>(lds + p.mid_at + (pixel * p.slots_mid + c) * 16) = uint4{0u, 0u, 0u, 0u};
    }
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // ---- phase 1: the 3 x 3 convolution ----
  uint32_t a2_off[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) a2_off[t] = fragment(wave * 32 + t * 16, p.Kp2);
  auto load_a2 = [&](int step, int t, uint4* av) {
    av[t] = load16(w2r, a2_off[t], (uint32_t)min(step, p.steps2 - 1) * ((uint32_t)p.Kp2 * 64u));
  };
  {
    uint32_t origin[MT], inside[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const u32x2 e = pixel_table[mt * 16 + li];
      origin[mt] = e[0];
      inside[mt] = e[1];
    }
    f32x4 acc[MT][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt][t] = wk == 0 ? b1v[t] : f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 b[2][MT];
    // (the table's last row is a tap outside every image, whose pixel is the patch's zeros)
    int step = wk;
    u32x2 entry = table[min(step, p.steps1) * 4 + g];
    auto read = [&](uint4* bv) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const uint32_t in = (uint32_t)__builtin_amdgcn_sbfe((int)inside[mt], entry[1], 1);
        bv[mt] = *reinterpret_cast<const uint4*>(lds + ((origin[mt] + entry[0]) & in));
      }
      step += WK;
      entry = table[min(step, p.steps1) * 4 + g];
    };
    read(b[0]);
    // rounds of D steps; the last one loads the second convolution's first weights
    int left = (p.steps1 - wk + WK - 1) / WK;      // (wk may be past the end: none)
    int next = wk + D * WK;
    auto round = [&](auto more) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        read(b[(d + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (more.value || d < left) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[mt][t] = mfma_16x16x32<BF>(a[d][t], b[d & 1][mt], acc[mt][t]);
        }
        if constexpr (more.value) {
          load_a(w1r, next, p.steps1 - 1, p.Kp1, a[d]);
          next += WK;
        } else {
          load_a2(d, 0, a[d]);
          load_a2(d, 1, a[d]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    for (; left > D; left -= D) round(std::true_type{});
    round(std::false_type{});
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) load_res(wave * 32, mt);   // (in the order that the groups load)

    // the WK partial sums of a pair of tiles meet in LDS, in the order of the waves
    f32x4* part = reinterpret_cast<f32x4*>(lds);   // [wave of the reduction][of the filters][tile][lane]
    if (WK > 1) {
      __syncthreads();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          if ((mt & (WK - 1)) != wk) part[((wave * MT + mt) * 2 + t) * 64 + lane] = acc[mt][t];
      __syncthreads();
    }
    const uint32_t floor2 = p.relu1 ? 0u : 0x80008000u;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if ((mt & (WK - 1)) != wk) continue;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (wf * 32 + t * 16 >= p.Kp1) break;
        f32x4 v = acc[mt][t];
        if (WK > 1) {
          v = f32x4{0.f, 0.f, 0.f, 0.f};
          for (int k = 0; k < WK; ++k) {
            const f32x4 q = part[(((k * WF + wf) * MT + mt) * 2 + t) * 64 + lane];
            v += k == wk ? acc[mt][t] : q;
          }
        }
        u32x2 o;
        o[0] = clamp_below(pack2<BF>(v[0], v[1]), floor2);
        o[1] = clamp_below(pack2<BF>(v[2], v[3]), floor2);
        *reinterpret_cast<u32x2*>(lds + p.mid_at + (mt * 16 + li) * p.slots_mid * 16 +
                                  (wf * 32 + t * 16 + g * 4) * 2) = o;
      }
    }
  }
  __syncthreads();   // the 3 x 3 convolution's output is in LDS, its input is not read any more

  // ---- phases 2 and 3, group of filters by group of filters ----
  uint32_t mid_pixel[MT], x2_pixel[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    mid_pixel[mt] = (uint32_t)(p.mid_at + (mt * 16 + li) * p.slots_mid * 16 + g * 16);
    x2_pixel[mt] = (uint32_t)(p.patch2_at + (mt * 16 + li) * p.slots2 * 16 + g * 16);
  }
  uint4 c[DC][N3];
  uint32_t c_off[N3];
#pragma unroll
  for (int t = 0; t < N3; ++t) c_off[t] = third ? fragment((wave * N3 + t) * 16, p.Kp3) : kOutside;
  auto load_c = [&](int step, uint4* cv) {
    const uint32_t so = (uint32_t)min(step, p.steps3 - 1) * ((uint32_t)p.Kp3 * 64u);
#pragma unroll
    for (int t = 0; t < N3; ++t) cv[t] = load16(w3r, c_off[t], so);
  };
  const uint32_t floor2 = p.relu2 ? 0u : 0x80008000u;

  for (int group = 0; group < p.groups; ++group) {
    const int f0 = group * GF + wave * 32;
    // (a wave whose filters do not exist multiplies the last ones again and writes zeros)
    f32x4 acc[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[mt][t] = b2v[t];
    uint4 b[2][MT];
    auto read = [&](int step, uint4* bv) {
      const bool second = step >= p.split_steps;
      const uint32_t off = (uint32_t)(second ? step - p.split_steps : step) * 64u;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        bv[mt] = *reinterpret_cast<const uint4*>(lds + (second ? x2_pixel[mt] : mid_pixel[mt]) + off);
    };
    read(0, b[0]);
    int s0 = 0;
    // the last round loads the group's weights of the third convolution
    auto round = [&](auto more, int left) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        read(min(s0 + d + 1, p.steps2 - 1), b[(d + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (more.value || d < left) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[mt][t] = mfma_16x16x32<BF>(a[d][t], b[d & 1][mt], acc[mt][t]);
        }
        if constexpr (more.value) {
          load_a2(s0 + d + D, 0, a[d]);
          load_a2(s0 + d + D, 1, a[d]);
        } else if constexpr (NT3 > 0) {
#pragma unroll
          for (int k = d * DC / D; k < (d + 1) * DC / D; ++k) load_c(group * WAVES + k, c[k]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (p.steps2 <= D) {   // (apart, so that its waits do not count the loads of a round before it)
      round(std::false_type{}, p.steps2);
    } else {
      for (; s0 + D < p.steps2; s0 += D) round(std::true_type{}, D);
      round(std::false_type{}, p.steps2 - s0);
    }

    char* wide = lds + (group & 1) * kWideBytes;
    auto finish = [&](const f32x4& av, uint32_t r0, uint32_t r1) {
      const float v[4] = {av[0] + to_float<BF>((uint16_t)(r0 & 0xffffu)), av[1] + to_float<BF>((uint16_t)(r0 >> 16)),
                          av[2] + to_float<BF>((uint16_t)(r1 & 0xffffu)), av[3] + to_float<BF>((uint16_t)(r1 >> 16))};
      u32x2 o;
      o[0] = clamp_below(pack2<BF>(v[0], v[1]), floor2);
      o[1] = clamp_below(pack2<BF>(v[2], v[3]), floor2);
      return o;
    };
    const int k0 = f0 + own;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const auto q0 = __builtin_amdgcn_permlane16_swap(r4[mt][0], r4[mt][2], false, false);
      const auto q1 = __builtin_amdgcn_permlane16_swap(r4[mt][1], r4[mt][3], false, false);
      const u32x2 oa = finish(acc[mt][0], q0[0], q1[0]);
      const u32x2 ob = finish(acc[mt][1], q0[1], q1[1]);
      const auto s0 = __builtin_amdgcn_permlane16_swap(oa[0], ob[0], false, false);
      const auto s1 = __builtin_amdgcn_permlane16_swap(oa[1], ob[1], false, false);
      u32x4 o4 = {s0[0], s1[0], s0[1], s1[1]};
      __builtin_amdgcn_raw_buffer_store_b128(o4, yr, k0 < p.ycs ? row[mt] + (uint32_t)f0 * 2u : kOutside, 0, 0);
      if constexpr (NT3 > 0) {
        if (k0 >= p.Kp2) o4 = u32x4{0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(wide + (mt * 16 + li) * kWidePixel + (wave * 32 + own) * 2) = o4;
      }
    }

    // what the next group needs: biases, weights, shortcut values, one load after the other
    // (past the last group: the last filters again, no shortcut)
#pragma unroll
    for (int t = 0; t < 2; ++t) a2_off[t] = fragment(f0 + GF + t * 16, p.Kp2);
    auto load_next = [&](int k) {
      if (k < 2) load_b2(f0 + GF, k);
      else if (k < 2 + 2 * D) load_a2((k - 2) / 2, k & 1, a[(k - 2) / 2]);
      else load_res(f0 + GF, k - 2 - 2 * D);
    };
    constexpr int kNext = 2 + 2 * D + MT;
    if constexpr (NT3 == 0) {
#pragma unroll
      for (int k = 0; k < kNext; ++k) load_next(k);
    } else {
      __syncthreads();   // the group's channels are in LDS
      const int steps = third ? min(WAVES, p.steps3 - group * WAVES) : 0;
      const char* pixel = wide + li * kWidePixel + g * 16;
      auto read3 = [&](int step, uint4* bv) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          bv[mt] = *reinterpret_cast<const uint4*>(pixel + mt * 16 * kWidePixel + step * 64);
      };
      read3(0, b[0]);
#pragma unroll
      for (int s = 0; s < WAVES; ++s) {
        if (s < steps) {
          if (s + 1 < WAVES) read3(s + 1, b[(s + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < N3; ++t)
              acc3[mt][t] = mfma_16x16x32<BF>(c[s % DC][t], b[s & 1][mt], acc3[mt][t]);
        }
        if constexpr (DC < WAVES)
          if (s + DC < WAVES) load_c(group * WAVES + s + DC, c[s % DC]);
#pragma unroll
        for (int k = s * kNext / WAVES; k < (s + 1) * kNext / WAVES; ++k) load_next(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  if constexpr (NT3 > 0) {
    if (!third) return;
    const __amdgpu_buffer_rsrc_t hr = buffer_of(p.h, p.h_bytes);
    const uint32_t floor3 = p.relu3 ? 0u : 0x80008000u;
#pragma unroll
    for (int t = 0; t < N3; ++t) {
      const int k0 = (wave * N3 + t) * 16 + g * 4;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int m = m0 + mt * 16 + li;
        const f32x4& v = acc3[mt][t];
        u32x2 o;
        o[0] = clamp_below(pack2<BF>(v[0], v[1]), floor3);
        o[1] = clamp_below(pack2<BF>(v[2], v[3]), floor3);
        __builtin_amdgcn_raw_buffer_store_b64(o, hr, m < p.M && k0 < p.hcs ? (uint32_t)(m * p.hcs + k0) * 2u : kOutside,
                                              0, 0);
      }
    }
  }
}

struct BlockTile {
  int MT, waves, D;
  const char* name;
};
constexpr BlockTile kTiles[] = {
    {1, 8, 8, "bottleneck_16x256"}, {2, 8, 6, "bottleneck_32x256"}, {4, 8, 4, "bottleneck_64x256"},
    {2, 4, 6, "bottleneck_32x128"}, {4, 4, 4, "bottleneck_64x128"},
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// LDS slots of 16 bytes per pixel: 16 lanes read 16 bytes each of neighbouring pixels, which is free
// of bank conflicts at odd multiples of 32 bytes
int pad_slots(int chunks, bool strided) {
  if (strided) return chunks | 1;
  while (chunks % 4 != 2) ++chunks;
  return chunks;
}

struct BlockPlan {
  BlockParams p;
  int tile, nt3;
  size_t lds;
};

bool plan_block(const BottleneckArgs& a, int N, int tile, BlockPlan* out) {
  const BlockTile& T = kTiles[tile];
  const int BM = T.MT * 16, GF = T.waves * 32;
  BlockParams p{};
  const PackedLayout L1 = packed_layout(a.s1, a.dt), L2 = packed_layout(a.s2, a.dt);
  if (std::max(weight_bytes(L1), weight_bytes(L2)) >= kOutside) return false;   // (32-bit offsets)
  p.H = a.H; p.W = a.W; p.pix = a.xcs * 2; p.pixels = N * a.H * a.W;
  const int P = out_extent(a.H, 3, a.s1.stride, 1);
  p.Q = out_extent(a.W, 3, a.s1.stride, 1);
  p.PQ = P * p.Q;
  p.M = N * p.PQ;
  p.stride = a.s1.stride;
  p.Kp1 = L1.Kp; p.cpt = L1.Cp / 8; p.steps1 = L1.nchunk_pad / 4;
  p.Kp2 = L2.Kp; p.steps2 = L2.nchunk_pad / 4;
  p.x_bytes = (uint32_t)p.pixels * (uint32_t)p.pix;
  p.w1_bytes = (uint32_t)p.steps1 * 64u * (uint32_t)p.Kp1;
  p.w2_bytes = (uint32_t)p.steps2 * 64u * (uint32_t)p.Kp2;
  p.slots = pad_slots(p.cpt, p.stride == 2);
  p.live = p.cpt;
  p.split_steps = p.steps2;
  if (a.two) {
    p.split_steps = round_up(a.s1.K, FUPR_CAT_ALIGN) / 32;
    p.live2 = L2.Cp / 8 - p.split_steps * 4;
    p.slots2 = pad_slots((p.steps2 - p.split_steps) * 4, false);
    p.H2 = a.H2; p.W2 = a.W2; p.pix2 = a.x2cs * 2; p.stride2 = a.stride2;
    p.x2_bytes = (uint32_t)N * (uint32_t)(a.H2 * a.W2) * (uint32_t)p.pix2;
  }
  p.slots_mid = pad_slots(std::max(p.split_steps * 4, p.Kp1 / 8), false);
  p.groups = (p.Kp2 + GF - 1) / GF;
  p.WF1 = 1;
  while (p.WF1 * 32 < p.Kp1) p.WF1 *= 2;
  if (p.WF1 > T.waves) return false;
  out->nt3 = 0;
  if (a.third) {
    const PackedLayout L3 = packed_layout(a.s3, a.dt);
    if (weight_bytes(L3) >= kOutside) return false;
    p.Kp3 = L3.Kp; p.steps3 = L3.nchunk_pad / 4;
    p.w3_bytes = (uint32_t)p.steps3 * 64u * (uint32_t)p.Kp3;
    const int per_wave = (p.Kp3 / 16 + T.waves - 1) / T.waves;
    out->nt3 = per_wave > 2 ? 4 : per_wave;
    if (per_wave > 4 || T.MT * out->nt3 > 8) return false;   // (registers)
  }
  const int run = (int)std::min<int64_t>(most_run_pixels(BM, 3, 3, p.stride, p.H, p.W, P, p.Q), 1 << 20);
  size_t end = round_up_sz((size_t)run * p.slots * 16, 1024);
  p.table_at = (int)end;
  end += (size_t)(p.steps1 + 1) * 32;
  p.pixels_at = (int)end;
  end += (size_t)BM * 8;
  // the third convolution's two input buffers lie where the patch and the tables were
  if (a.third) end = std::max(end, (size_t)2 * BM * (GF * 2 + 32));
  if (p.WF1 < T.waves) end = std::max(end, (size_t)T.waves * T.MT * 2048);   // and the 3 x 3's partial sums
  p.mid_at = (int)round_up_sz(end, 1024);
  end = (size_t)p.mid_at + (size_t)BM * p.slots_mid * 16;
  if (a.two) {
    p.patch2_at = (int)round_up_sz(end, 1024);
    end = (size_t)p.patch2_at + round_up_sz((size_t)BM * p.slots2 * 16, 1024);
  }
  p.spare_at = (int)round_up_sz(end, 1024);
  out->lds = (size_t)p.spare_at + 1024;
  if (out->lds > kLdsLimit) return false;
  p.total = (p.M + BM - 1) / BM;
  p.per_xcd = (p.total + 7) / 8;
  out->p = p;
  out->tile = tile;
  return true;
}

// What only a launch needs: plans that are weighed do without.
void set_divisions(BlockParams& p) {
  p.divPQ = fast_div(p.PQ); p.divQ = fast_div(p.Q); p.divC = fast_div(p.cpt);
  p.divSlots = fast_div(p.slots); p.divSlots2 = fast_div(std::max(p.slots2, 1));
}

template <bool BF, int TILE, int NT3>
fupr_status launch_as(const BlockPlan& plan, hipStream_t st) {
  constexpr BlockTile T = kTiles[TILE];
  if constexpr (T.MT * NT3 > 8) {
    return FUPR_ERR_LIMIT;
  } else {
  auto kernel = bottleneck_kernel<BF, T.MT, T.waves, T.D, NT3>;
  if (plan.lds > 64 * 1024) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
    if (attr != hipSuccess) return FUPR_ERR_LAUNCH;
  }
  void* list[] = {const_cast<BlockParams*>(&plan.p)};
  return launched(hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)(plan.p.per_xcd * 8)),
                                  dim3(T.waves * 64), list, plan.lds, st),
                  "bottleneck_kernel");
  }
}

template <bool BF, int TILE>
fupr_status dispatch_third(const BlockPlan& plan, hipStream_t st) {
  switch (plan.nt3) {
    case 0: return launch_as<BF, TILE, 0>(plan, st);
    case 1: return launch_as<BF, TILE, 1>(plan, st);
    case 2: return launch_as<BF, TILE, 2>(plan, st);
    default: return launch_as<BF, TILE, 4>(plan, st);
  }
}

template <bool BF>
fupr_status dispatch(const BlockPlan& plan, hipStream_t st) {
  switch (plan.tile) {
    case 0: return dispatch_third<BF, 0>(plan, st);
    case 1: return dispatch_third<BF, 1>(plan, st);
    case 2: return dispatch_third<BF, 2>(plan, st);
    case 3: return dispatch_third<BF, 3>(plan, st);
    case 4: return dispatch_third<BF, 4>(plan, st);
  }
  return FUPR_ERR_LIMIT;
}

// Estimated us of a plan: a fit over 480 blocks (ResNet-50's, regular and irregular channel counts, 1 - 128
// images) x five tiles, 1932 launches, to 10 % in the mean square; the tile with the least estimate is
// 0.6 % slower than the best one in the mean, 34 % at worst (one image, deep layers).
double estimate(const BottleneckArgs& a, const BlockPlan& plan) {
  const BlockParams& p = plan.p;
  const BlockTile& T = kTiles[plan.tile];
  const int WK = T.waves / p.WF1, GF = T.waves * 32, BM = T.MT * 16;
  const int resident = std::max(1, std::min(T.waves == 8 ? 1 : 2, (int)(kLdsLimit / plan.lds)));
  const int per_cu = (p.total + kComputeUnits - 1) / kComputeUnits;
  const double wide = a.two ? 32.0 * (p.steps2 - p.split_steps) : a.s2.K;
  const double in = 1.0 * p.stride * p.stride * a.s1.C, out = (double)a.s2.K + (a.third ? a.s3.K : 0);
  // clocks of a workgroup that has the compute unit to itself; of its weights and pixels on the way
  // from L2 to the compute unit (fitted: 36 bytes per clock); all tensors at memory's rate
  const double alone = ((p.steps1 + WK - 1) / WK) * (96.5 + 88.1 * T.MT) +
                       p.groups * (764.0 + p.steps2 * (49.7 + 83.5 * T.MT) +
                                   T.waves * (451.0 + 59.1 * T.MT * plan.nt3)) +
                       (WK > 1 ? 8975.0 : 0.0);
  const double bytes = 64.0 * p.steps1 * p.Kp1 + 64.0 * p.steps2 * p.groups * GF + 64.0 * p.steps3 * p.Kp3 +
                       BM * 2.0 * (1.3 * in + wide + out);
  const double clocks = std::max((per_cu + resident - 1) / resident * alone, per_cu * bytes / 35.7 + 0.364 * alone);
  const double busy = clocks / 2400.0, memory = p.M * 2.0 * (in + wide + out) / 3.24e6;
  return 4.7 + std::max(busy, memory) + 0.02 * std::min(busy, memory);
}

// Estimated us of the same operators as launches of their own, fitted to the same blocks (to 6 %).
double estimate_apart(const BottleneckArgs& a, int64_t M) {
  auto one = [](double bytes, double flops) {
    const double mb = bytes / 1e6;
    return 6.33 + std::pow(std::pow(mb / 20.7, 0.793) + std::pow(flops / 673e6, 0.793), 1.0 / 0.793) + 0.168 * std::sqrt(mb);
  };
  const double m = (double)M, second = a.two ? a.s2.C - round_up(a.s1.K, FUPR_CAT_ALIGN) : 0;
  return one(m * 2 * (a.s1.stride * a.s1.stride * a.s1.C + a.s1.K), m * 18 * a.s1.C * a.s1.K) +
         one(m * 2 * (a.s1.K + second + (a.two ? 0 : a.s2.K) + a.s2.K), m * 2 * (a.s1.K + second) * a.s2.K) +
         (a.third ? one(m * 2 * (a.s2.K + a.s3.K), m * 2 * a.s2.K * a.s3.K) : 0.0);
}

// The tile with the least estimate; only those with that many waves if waves > 0.  (About ten plans, 2 us of host
// time: a model asks once for a batch size and keeps the answer.)
bool pick_block(const BottleneckArgs& a, int N, int waves, BlockPlan* best, double* cost) {
  const int forced = tuning_int("bottleneck_tile", -1);
  if (forced >= 0) {
    *cost = 0.0;
    return forced < kNumTiles && plan_block(a, N, forced, best);
  }
  bool any = false;
  for (int tile = 0; tile < kNumTiles; ++tile) {
    BlockPlan plan;
    if ((waves > 0 && kTiles[tile].waves != waves) || !plan_block(a, N, tile, &plan)) continue;
    const double c = estimate(a, plan);
    if (any && c >= *cost) continue;
    *best = plan;
    *cost = c;
    any = true;
  }
  return any;
}

// The plan with which a batch of N images runs the block as one launch, -1: the operators run apart.
int choose(const BottleneckArgs& a, int N) {
  if (tuning_off("bottleneck_fuse")) return -1;
  const int64_t M = (int64_t)N * out_extent(a.H, 3, a.s1.stride, 1) * out_extent(a.W, 3, a.s1.stride, 1);
  // 32-bit byte offsets into every tensor
  for (int64_t elements : {(int64_t)N * a.H * a.W * a.xcs, M * a.ycs, a.two ? (int64_t)N * a.H2 * a.W2 * a.x2cs : 0,
                           a.third ? M * a.hcs : 0})
    if (elements * 2 >= (int64_t)kOutside) return -1;
  BlockPlan plan;
  double cost;
  if (!pick_block(a, N, 0, &plan, &cost)) return -1;
  // 5 % less than the launches apart, which is what the two estimates are uncertain by; 15 % where the
  // two 1 x 1 convolutions would run as a pair (32 -> 256 -> 32 at 56 x 56 x 24 29 against 33 us, x 64 59
  // against 55).  Both were fitted to launches between events, which takes some 1.5 us more for each than one
  // after the other: that decides where they are short (nine irregular images 269 -> 264 us; a network at 64
  // images, whose sub-batches run side by side, 684 against 670 when it is counted there too).
  if (tuning_int("bottleneck_tile", -1) >= 0) return plan.tile;
  const double gap = M < 8192 ? 1.5 : 0.0, apart = estimate_apart(a, M);
  if (cost - gap >= (a.pair ? 0.85 : 0.95) * (apart - gap * (a.third ? 3 : 2))) return -1;
  // Under 4096 pixels even tiles of 16 leave compute units idle, and the launches apart, which split their filters as
  // well, are shorter inside a network than between events.  Each block by itself as one launch and as several, us
  // of the captured pass, blocks without a pair: of 208 taken without these lines 109 lost; of the 93 taken with them 13 lose,
  // up to 0.7 % of a pass (13.8 of 21.6 us estimated gains 1.0 at 12 x 12 x 16 images, 20.4 of 25.9 loses 1.8
  // at 14 x 14 x 16).  Where two sub-batches overlap (from 64 images on, split_count in model.cpp) 38 of 40 lost, up
  // to 19 us (231 -> 1024 -> 231 channels, 6 x 6 x 192 images, 38 of 46 us estimated).
  const bool halves = N >= 64;
  if (!a.pair && M < (halves ? 8192 : 4096) && (halves || cost + 2.0 > 0.78 * apart)) return -1;
  return plan.tile;
}

}  // namespace

bool bottleneck_applies(const BottleneckArgs& a) {
  if (a.dt == FUPR_F32 || a.s1.R != 3 || a.s1.S != 3 || a.s1.pad != 1 || a.s1.stride < 1 || a.s1.stride > 2) return false;
  if (a.s2.R != 1 || a.s2.S != 1 || a.s2.stride != 1 || a.s2.pad != 0) return false;
  if (a.third && (a.s3.R != 1 || a.s3.S != 1 || a.s3.stride != 1 || a.s3.pad != 0)) return false;
  const WithoutTuning no_switches;   // (they can change between a model's plan and its passes)
  BlockPlan plan;
  for (int tile = 0; tile < kNumTiles; ++tile)
    if (plan_block(a, 1, tile, &plan)) return true;
  return false;
}

int bottleneck_plan(const BottleneckArgs& a, int N) {
  if (tuning_any()) return choose(a, N);
  const WithoutTuning no_switches;   // (one that is set meanwhile is in no answer that is kept)
  return recall<BottleneckArgs, choose>(a, N);
}

// The order of the 3 x 3 convolution's sums depends on the number of waves: a part keeps its batch's.
int bottleneck_plan_part(const BottleneckArgs& a, int plan, int count) {
  BlockPlan part;
  double cost;
  return pick_block(a, count, kTiles[plan].waves, &part, &cost) ? part.tile : plan;
}

const char* bottleneck_name(int plan) { return kTiles[plan].name; }

fupr_status launch_bottleneck(const BottleneckArgs& a, int tile, int count, void* stream) {
  BlockPlan plan;
  if (!plan_block(a, count, tile, &plan)) return FUPR_ERR_LIMIT;
  BlockParams& p = plan.p;
  set_divisions(p);
  const PackedLayout L1 = packed_layout(a.s1, a.dt), L2 = packed_layout(a.s2, a.dt);
  auto weights = [](const void* blob, const PackedLayout& L) {
    return reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(blob) + L.weight_offset);
  };
  p.x = (const uint16_t*)a.x; p.x2 = (const uint16_t*)a.x2; p.res = (const uint16_t*)a.res;
  p.w1 = weights(a.packed1, L1); p.b1 = (const float*)a.packed1;
  p.w2 = weights(a.packed2, L2); p.b2 = (const float*)a.packed2;
  p.y = (uint16_t*)a.y; p.ycs = a.ycs;
  p.y_bytes = (uint32_t)p.M * (uint32_t)a.ycs * 2u;
  p.res_bytes = a.res ? p.y_bytes : 0u;
  p.relu1 = a.relu1; p.relu2 = a.relu2; p.relu3 = a.relu3;
  if (a.third) {
    const PackedLayout L3 = packed_layout(a.s3, a.dt);
    p.w3 = weights(a.packed3, L3); p.b3 = (const float*)a.packed3;
    p.h = (uint16_t*)a.h; p.hcs = a.hcs;
    p.h_bytes = (uint32_t)p.M * (uint32_t)a.hcs * 2u;
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  return a.dt == FUPR_BF16 ? dispatch<true>(plan, st) : dispatch<false>(plan, st);
}

}  // namespace fupr
