// A basic block's two 3 x 3 convolutions (Table II; Sec. IV-B-1) in one launch: a workgroup computes a
// rectangle of TH x TW output pixels of one image, its first convolution on the rectangle and a ring of
// one pixel around it.  The tensor between the two stays in LDS, one launch and two passes over it are
// saved, and the ring is multiplied twice (14 x 14: 1.31 times the first convolution's work).
//
//   * The rectangle's input with its border, all channels, goes to LDS once; what lies outside the image
//     is zeros there, so that a tap is an addition to a pixel's address and nothing else.
//   * WF waves lie along the filters, one tile of 16 each at a time, the others along the pixels; a wave's
//     weights come from L2 straight into registers, D steps ahead.
//   * Outside the image the second convolution reads zeros: the first one's values there are not stored.
//   * Sums run over the reduction in one order whatever the rectangle, except in rectangles of 14 columns and 6 or 14
//     rows at stride 1 in 16 bits.  With the ring their rows are tiles of 16 pixels, and what is read from LDS
//     for one row is multiplied for the three output rows that have a tap there (multiply_rows).
//
// Measured, two launches -> one (us, event-timed): 64 -> 45 -> 64 channels at 56 x 56, one image 13.0 -> 8.8, 8
// images 20.0 -> 13.5, 32 images 35.5 -> 20.8, 64 images 54.7 -> 36.0 (43.2 not by rows), 250 images 137 -> 121 (150);
// 128 -> 90 -> 128 at 28 x 28 x 64 44.9 -> 31.1 (36.9); single precision, 16 -> 12 -> 16 at 32 x 32 x 32 images
// 16.4 -> 11.0, 32 -> 23 -> 32 at 16 x 16 x 32 16.3 -> 12.  Networks: ResNet-18, one image 97.6 -> 92.9, 64 images
// 377 -> 345; ResNet-20 in single precision, 32 images 111 -> 103.
// What bounds it: at a few images the start (index arithmetic, arguments, first weights: 4000 of 11 000
// clocks) and the weights' latency; at many, LDS where a read of 1 KB, 8 clocks, serves one MFMA of 4 clocks
// per compute unit, and by rows the serial chain of a workgroup, load, multiply, multiply, store, of which
// one or two fit into LDS together (ResNet-18's three at 64 images: 45 MB each in 35 us by counters, 1.3 TB/s; the
// matrix pipe busy 42 % of it).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <type_traits>

#include "basic_block.h"
#include "device_utils.h"
#include "fupr.h"
#include "layout.h"
#include "recall.h"
#include "tuning.h"

namespace fupr {
namespace {

constexpr uint32_t kOutside = 0x80000000u;   // beyond every tensor this kernel accepts
constexpr size_t kLdsLimit = 160 * 1024;
constexpr int kComputeUnits = 256;
constexpr int kWaves = 8, kThreads = kWaves * 64;
constexpr int kSharers = 32;                 // workgroups of an XCD that run at once, at least

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef void __attribute__((address_space(3)))* LdsPtr;

struct BasicParams {
  const void *x, *w1, *w2, *res;
  const float *b1, *b2;
  void* y;
  uint32_t x_bytes, w1_bytes, w2_bytes, res_bytes, y_bytes;
  int H, W, pix, stride;            // input: extent, bytes per pixel; of the first convolution
  int P, Q, TH, TW, MW, IW;         // output extent; rectangle; pixels per row of its ring and of its input
  int mids, outs;                   // (TH + 2) * (TW + 2), TH * TW
  int Kp1, cpt1, nchunk1, steps1, Kp2, cpt2, nchunk2, steps2;
  int rH, rW, rcs, rss, roff, ycs, relu1, relu2;
  int rows1, rows2;                 // steps of one row of taps (multiply_rows)
  int slots1, slots2, in_pixels;
  int mid_at, table1_at, table2_at, zero_at;   // LDS byte offsets (the input starts at 0)
  int WF, log2_WF, tiles_w, tiles, total, per_xcd;
  FastDiv divC1, divC2, divMW, divTW, divSlots, divIW, divTiles, divTilesW;
};

__device__ __forceinline__ uint32_t clamp_below(uint32_t v, uint32_t floor2) {
  const short2_t a = __builtin_bit_cast(short2_t, v), f = __builtin_bit_cast(short2_t, floor2);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, f));
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

// M tiles of 16 pixels x one tile of 16 filters over all steps of a reduction, pixels from LDS.  a holds
// the weights of the first D steps.  (Single precision adds each step's 16 products up on their own, then the sum
// to the others': a quarter as many roundings at the size of the whole sum.  Without it the error of a block of 16
// channels against 64 bits was 2.0e-7 of the result, 1.2e-7 with two launches; with it 1.1e-7.)
template <int EL, int M, int D, int NB, class Load>
__device__ __forceinline__ void multiply(const char* lds, const uint32_t (&origin)[M], const uint32_t* table, int g,
                                         uint32_t zero_at, int steps, uint4 (&a)[D], f32x4 (&acc)[M], Load&& load) {
  // Units of U tiles are read from LDS NB - 1 ahead of the one that is multiplied.
  // (Two in single precision, whose sums of a step need registers.)
  constexpr int most = EL == FUPR_F32 ? 2 : 4, U = M < most ? M : most, NU = (M + U - 1) / U;
  static_assert((NB == 2 || NB == 3) && D * NU % NB == 0, "pixel buffers in turn");
  uint4 b[NB][U];
  auto read = [&](uint32_t entry, int u, uint4* bv) {
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (u * U + k < M) {
        // (the chunks that pad the last step point past everything: zeros)
        const uint32_t at = min(origin[u * U + k] + entry, zero_at);
        bv[k] = *reinterpret_cast<const uint4*>(lds + at);
      }
  };
  // e[k]: the table's entry of step s0 + d + k
  uint32_t e[3] = {table[g], table[min(1, steps) * 4 + g], table[min(2, steps) * 4 + g]};
#pragma unroll
  for (int k = 0; k < NB - 1; ++k) read(e[k / NU], k % NU, b[k]);
  int s0 = 0;
  auto round = [&](auto more, int left) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (!more.value && d > 0 && d >= left) break;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int now = (d * NU + u) % NB;
        read(e[(u + NB - 1) / NU], (u + NB - 1) % NU, b[(now + NB - 1) % NB]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < U; ++k)
          if (u * U + k < M) {
            f32x4& c = acc[u * U + k];
            if constexpr (EL == FUPR_F32) {
              f32x4 sum = mfma_16x16x4(a[d].x, b[now][k].x, f32x4{0.f, 0.f, 0.f, 0.f});
              sum = mfma_16x16x4(a[d].y, b[now][k].y, sum);
              sum = mfma_16x16x4(a[d].z, b[now][k].z, sum);
              c += mfma_16x16x4(a[d].w, b[now][k].w, sum);
            } else {
              c = mfma_16x16x32<EL == FUPR_BF16>(a[d], b[now][k], c);
            }
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      e[0] = e[1];
      e[1] = e[2];
      e[2] = table[min(s0 + d + 3, steps) * 4 + g];
      if constexpr (more.value) load(s0 + d + D, a[d]);
    }
  };
  for (; s0 + D < steps; s0 += D) round(std::true_type{}, D);
  round(std::false_type{}, steps - s0);
}

// M tiles of 16 pixels that are M rows of a tensor in LDS, one below the other, x one tile of 16 filters.  The
// reduction goes row of taps by row of taps, each padded to whole steps: a step's pixels at one row of the
// tensor are read once and multiplied for the three output rows that have a tap there, (M + 2) / (3 M) LDS
// reads per MFMA instead of one (64 x 56 x 56 x 64 -> 45 -> 64 43 -> 36 us, 64 x 28 x 28 x 128 -> 90 -> 128
// 36.9 -> 31.1 us).  a holds the three rows' weights of the first DQ steps: more of them spill with eight
// rows in 128 registers and were slower (41 us at four).
template <bool BF, int M, int DQ, class Load>
__device__ __forceinline__ void multiply_rows(const char* lds, uint32_t base, uint32_t row_stride, const uint32_t* table,
                                              int g, uint32_t zero_at, int steps, uint4 (&a)[DQ][3], f32x4 (&acc)[M],
                                              Load&& load) {
  constexpr int ROWS = M + 2, NB = DQ * ROWS % 4 == 0 ? 4 : 3;
  static_assert(DQ * ROWS % NB == 0, "the pixel buffers in turn, over a round");
  uint4 b[NB];
  // (the chunks that pad a row's last step: zeros at every row)
  uint32_t at[2], stride[2];               // this step's and the next one's
  auto start = [&](int step, int k) {
    const uint32_t entry = table[min(step, steps) * 4 + g];
    const bool pad = entry == kOutside;
    at[k] = pad ? zero_at : base + entry;
    stride[k] = pad ? 0u : row_stride;
  };
  auto read = [&](int k, uint4& v) {
    v = *reinterpret_cast<const uint4*>(lds + min(at[k], zero_at));
    at[k] += stride[k];
  };
  start(0, 0);
  start(1, 1);
#pragma unroll
  for (int i = 0; i < NB - 1; ++i) read(0, b[i]);
  int s0 = 0;
  auto round = [&](auto more, int left) {
#pragma unroll
    for (int d = 0; d < DQ; ++d) {
      if (!more.value && d > 0 && d >= left) break;
      if (!more.value && d == left - 1) {
        // the weights beside a padding chunk are another row's
        const bool pad = stride[0] == 0u;
#pragma unroll
        for (int r = 0; r < 3; ++r) a[d][r] = pad ? uint4{0u, 0u, 0u, 0u} : a[d][r];
      }
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const int now = (d * ROWS + i) % NB;
        if (i + NB - 1 < ROWS) read(0, b[(now + NB - 1) % NB]);
        else read(1, b[(now + NB - 1) % NB]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 3; ++r)
          if (i - r >= 0 && i - r < M) acc[i - r] = mfma_16x16x32<BF>(a[d][r], b[now], acc[i - r]);
        __builtin_amdgcn_sched_barrier(0);
      }
      at[0] = at[1];
      stride[0] = stride[1];
      start(s0 + d + 2, 1);
      if constexpr (more.value)
#pragma unroll
        for (int r = 0; r < 3; ++r) load(s0 + d + DQ, r, a[d][r]);
    }
  };
  for (; s0 + DQ < steps; s0 += DQ) round(std::true_type{}, DQ);
  round(std::false_type{}, steps - s0);
}

// MA, MB: tiles of 16 pixels per wave of the first and of the second convolution.  ROWS: the tiles are rows of
// the rectangle, 16 pixels with its ring, and multiply_rows multiplies them (16-bit types, stride 1).
template <int EL, int MA, int MB, int D, int NB, int MINWAVES, bool ROWS>
__global__ __launch_bounds__(kThreads, MINWAVES) void basic_block_kernel(const BasicParams p) {
  touch_arguments<sizeof(BasicParams)>();
  constexpr bool F32 = EL == FUPR_F32, BF = EL == FUPR_BF16;
  constexpr int ES = F32 ? 4 : 2;            // bytes per element
  extern __shared__ uint4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  const uint32_t lds_base = (uint32_t)(uintptr_t)(LdsPtr)lds;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (waves that have no filters, of two workgroups on one compute unit, lie on different SIMDs)
  const int wp = wave >> p.log2_WF, WP = kWaves >> p.log2_WF;
  const int wf = (wave + 2 * wp + (int)(blockIdx.x >> 3)) & (p.WF - 1);

  const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
  if (tile >= p.total) return;
  const int n = div_by(tile, p.divTiles), in_image = tile - n * p.tiles;
  const int th = div_by(in_image, p.divTilesW), tw = in_image - th * p.tiles_w;
  const int oh0 = th * p.TH, ow0 = tw * p.TW;

  const __amdgpu_buffer_rsrc_t w1r = buffer_of(p.w1, p.w1_bytes);
  const __amdgpu_buffer_rsrc_t w2r = buffer_of(p.w2, p.w2_bytes);
  // a wave's fragment of one filter tile (past the last step: the last one again, not multiplied)
  auto load_fragment = [&](const __amdgpu_buffer_rsrc_t& r, int f, int step, int steps, int Kp, uint4& v) {
    if constexpr (F32) {
      // four channels of the lane's chunk and filter; what lies beyond the weights reads as zero
      const uint32_t row = (uint32_t)Kp * 4u;
      const uint32_t at = (uint32_t)(min(step, steps - 1) * 16 + g * 4) * row + (uint32_t)min(f + li, Kp - 1) * 4u;
      v.x = __builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0);
      v.y = __builtin_amdgcn_raw_buffer_load_b32(r, at + row, 0, 0);
      v.z = __builtin_amdgcn_raw_buffer_load_b32(r, at + 2 * row, 0, 0);
      v.w = __builtin_amdgcn_raw_buffer_load_b32(r, at + 3 * row, 0, 0);
    } else {
      const uint32_t at = (uint32_t)(g * Kp + min(f, Kp - 16) + li) * 16u;
      v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                        r, at, (uint32_t)min(step, steps - 1) * ((uint32_t)Kp * 64u), 0));
    }
  };

  // (the first weights are the last to arrive in a cold L2: they are asked for before anything else; single
  // precision, which loads them four bytes at a time, asks for its pixels first)
  uint4 a[D];
  auto load1 = [&](int f) {
    return [&, f](int step, uint4& v) { load_fragment(w1r, f, step, p.steps1, p.Kp1, v); };
  };
  auto load2 = [&](int f) {
    return [&, f](int step, uint4& v) { load_fragment(w2r, f, step, p.steps2, p.Kp2, v); };
  };
  // ROWS: the weights of tap row r, step q of a row
  constexpr int DQ = ROWS ? D : 1;
  uint4 ar[DQ][3];
  auto load_row = [&](const __amdgpu_buffer_rsrc_t& rsrc, int f, int q, int r, int steps, int cpt, int Kp, uint4& v) {
    const uint32_t at = (uint32_t)(g * Kp + min(f, Kp - 16) + li) * 16u;
    const uint32_t so = (uint32_t)(r * 3 * cpt + min(q, steps - 1) * 4) * (uint32_t)(Kp * 16);
    v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, so, 0));
  };
  auto load_rows1 = [&](int f) {
    return [&, f](int q, int r, uint4& v) { load_row(w1r, f, q, r, p.rows1, p.cpt1, p.Kp1, v); };
  };
  auto load_rows2 = [&](int f) {
    return [&, f](int q, int r, uint4& v) { load_row(w2r, f, q, r, p.rows2, p.cpt2, p.Kp2, v); };
  };
  auto first_weights = [&] {
    if constexpr (ROWS) {
#pragma unroll
      for (int d = 0; d < DQ; ++d)
#pragma unroll
        for (int r = 0; r < 3; ++r) load_rows1(wf * 16)(d, r, ar[d][r]);
    } else {
#pragma unroll
      for (int d = 0; d < D; ++d) load1(wf * 16)(d, a[d]);
    }
  };
  if constexpr (!F32) first_weights();
  const f32x4 b1v = *reinterpret_cast<const f32x4*>(p.b1 + min(wf * 16 + g * 4, p.Kp1 - 4));
  const f32x4 b2v = *reinterpret_cast<const f32x4*>(p.b2 + min(wf * 16 + g * 4, p.Kp2 - 4));

  // ---- the rectangle's input into LDS ----
  {
    const i32x4 xr = make_rsrc(p.x, p.x_bytes);
    const int ih0 = (oh0 - 1) * p.stride - 1, iw0 = (ow0 - 1) * p.stride - 1;
    const int step_pix = div_by(kThreads, p.divSlots), step_c = kThreads - step_pix * p.slots1;   // (scalar)
    const int step_row = div_by(step_pix, p.divIW), step_col = step_pix - step_row * p.IW;
    const int first = div_by(tid, p.divSlots);
    int c = tid - first * p.slots1, row = div_by(first, p.divIW), col = first - row * p.IW;
    // (multiplications of 32 bits are quarter rate: everything but the start is stepped)
    uint32_t off = (uint32_t)((n * p.H + ih0 + row) * p.W + iw0 + col) * (uint32_t)p.pix + (uint32_t)c * 16u;
    const uint32_t step_off = (uint32_t)((step_row * p.W + step_col) * p.pix + step_c * 16);
    const uint32_t wrap_off = (uint32_t)(p.pix - p.slots1 * 16), turn_off = (uint32_t)((p.W - p.IW) * p.pix);
    const int live = p.cpt1, count = p.in_pixels * p.slots1;
    for (int base = wave * 64; base < count; base += kThreads) {
      const bool ok = c < live && (unsigned)(ih0 + row) < (unsigned)p.H && (unsigned)(iw0 + col) < (unsigned)p.W &&
                      base + lane < count;
      load_to_lds(xr, ok ? off : kOutside, lds_base + base * 16);
      c += step_c;
      const bool wrap = c >= p.slots1;
      c -= wrap ? p.slots1 : 0;
      col += step_col + (wrap ? 1 : 0);
      row += step_row;
      off += step_off + (wrap ? wrap_off : 0u);
      const bool turn = col >= p.IW;
      col -= turn ? p.IW : 0;
      row += turn ? 1 : 0;
      off += turn ? turn_off : 0u;
    }
  }
  if constexpr (F32) first_weights();
  // All workgroups of an XCD walk the weights in step: its first ones ask for all of them at once, a
  // share each, so that the loop below finds them in L2 (into 1 KB of LDS that nobody reads).
  {
    const int sharers = min(p.per_xcd, kSharers) * kWaves, me = (int)(blockIdx.x >> 3) * kWaves + wave;
    auto ask = [&](const void* w, uint32_t bytes) {
      const i32x4 r = make_rsrc(w, bytes);
      for (uint32_t at = (uint32_t)me * 1024u; at < bytes; at += (uint32_t)sharers * 1024u)
        load_to_lds(r, at + (uint32_t)lane * 16u, lds_base + p.zero_at + 1024);
    };
    if (me < sharers) {
      ask(p.w1, p.w1_bytes);
      ask(p.w2, p.w2_bytes);
    }
  }

  // per chunk of 16 bytes: its LDS distance from the first tap
  uint32_t* table1 = reinterpret_cast<uint32_t*>(lds + p.table1_at);
  uint32_t* table2 = reinterpret_cast<uint32_t*>(lds + p.table2_at);
  auto make_table = [&](uint32_t* table, int steps, int nchunk, int cpt, const FastDiv& by, int width, int slots) {
    for (int j = tid; j < (steps + 1) * 4; j += kThreads) {
      const int tap = div_by(j, by), cc = j - tap * cpt;
      const int r = (tap * 11) >> 5, s = tap - r * 3;   // (tap / 3 for taps below 16)
      table[j] = j < nchunk ? (uint32_t)(((r * width + s) * slots + cc) * 16) : kOutside;
    }
  };
  if constexpr (ROWS) {
    auto make_row_table = [&](uint32_t* table, int steps, int cpt, const FastDiv& by, int slots) {
      for (int j = tid; j < (steps + 1) * 4; j += kThreads) {
        const int s = div_by(j, by), cc = j - s * cpt;
        table[j] = s < 3 ? (uint32_t)((s * slots + cc) * 16) : kOutside;
      }
    };
    make_row_table(table1, p.rows1, p.cpt1, p.divC1, p.slots1);
    make_row_table(table2, p.rows2, p.cpt2, p.divC2, p.slots2);
  } else {
    make_table(table1, p.steps1, p.nchunk1, p.cpt1, p.divC1, p.IW, p.slots1);
    make_table(table2, p.steps2, p.nchunk2, p.cpt2, p.divC2, p.MW, p.slots2);
  }
  if (tid < 64) reinterpret_cast<uint32_t*>(lds + p.zero_at)[tid] = 0u;

  // Pixels of a wave lie WP * 16 apart: the row and column of the first are divided out, the others stepped.
  // (ROWS: a wave's tiles are rows one below the other, 16 pixels apart.)
  const int apart = ROWS ? 16 : WP * 16;
  uint32_t origin_a[MA];
  const int first_a = ROWS ? wp * MA * 16 + li : wp * 16 + li;
  const int dr_a = ROWS ? 1 : div_by(apart, p.divMW), dc_a = ROWS ? 0 : apart - dr_a * p.MW;
  const int r_a = ROWS ? wp * MA : div_by(first_a, p.divMW), c_a = ROWS ? li : first_a - r_a * p.MW;
  if constexpr (!ROWS) {
    const uint32_t unit = (uint32_t)(p.stride * p.slots1 * 16);
    const uint32_t step = (uint32_t)(dr_a * p.IW + dc_a) * unit, turn = (uint32_t)(p.IW - p.MW) * unit;
    uint32_t origin = (uint32_t)(r_a * p.IW + c_a) * unit;
    int c = c_a;
#pragma unroll
    for (int mt = 0; mt < MA; ++mt) {
      origin_a[mt] = first_a + mt * apart < p.mids ? origin : 0u;
      c += dc_a;
      origin += step;
      const bool over = c >= p.MW;
      c -= over ? p.MW : 0;
      origin += over ? turn : 0u;
    }
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // ---- the first convolution, on the rectangle and the ring around it ----
  {
    for (int f = wf * 16; f < p.Kp1; f += p.WF * 16) {
      if (f != wf * 16) {
        if constexpr (ROWS) {
#pragma unroll
          for (int d = 0; d < DQ; ++d)
#pragma unroll
            for (int r = 0; r < 3; ++r) load_rows1(f)(d, r, ar[d][r]);
        } else {
#pragma unroll
          for (int d = 0; d < D; ++d) load1(f)(d, a[d]);
        }
      }
      f32x4 acc[MA];
      f32x4 b4 = b1v;
      if (f != wf * 16) b4 = *reinterpret_cast<const f32x4*>(p.b1 + min(f + g * 4, p.Kp1 - 4));
#pragma unroll
      for (int mt = 0; mt < MA; ++mt) acc[mt] = b4;
      if constexpr (ROWS)
        multiply_rows<BF, MA, DQ>(lds, (uint32_t)((r_a * p.IW + li) * p.slots1 * 16), (uint32_t)(p.IW * p.slots1 * 16),
                                  table1, g, (uint32_t)p.zero_at, p.rows1, ar, acc, load_rows1(f));
      else
        multiply<EL, MA, D, NB>(lds, origin_a, table1, g, (uint32_t)p.zero_at, p.steps1, a, acc, load1(f));
      const uint32_t floor2 = p.relu1 ? 0u : 0x80008000u;
      int r = r_a, c = c_a;
      char* to = lds + p.mid_at + first_a * p.slots2 * 16 + (f + g * 4) * ES;
      const int to_step = apart * p.slots2 * 16;
#pragma unroll
      for (int mt = 0; mt < MA; ++mt, to += to_step) {
        const bool inside = (unsigned)(oh0 - 1 + r) < (unsigned)p.P && (unsigned)(ow0 - 1 + c) < (unsigned)p.Q;
        c += dc_a;
        r += dr_a;
        const bool over = !ROWS && c >= p.MW;
        c -= over ? p.MW : 0;
        r += over ? 1 : 0;
        if (first_a + mt * apart >= p.mids || (F32 && f + g * 4 >= p.Kp1)) continue;
        const f32x4& v = acc[mt];
        if constexpr (F32) {
          f32x4 o;
#pragma unroll
          for (int k = 0; k < 4; ++k) o[k] = inside ? (p.relu1 ? fmaxf(v[k], 0.f) : v[k]) : 0.f;
          *reinterpret_cast<f32x4*>(to) = o;
        } else {
          u32x2 o;
          o[0] = inside ? clamp_below(pack2<BF>(v[0], v[1]), floor2) : 0u;
          o[1] = inside ? clamp_below(pack2<BF>(v[2], v[3]), floor2) : 0u;
          *reinterpret_cast<u32x2*>(to) = o;
        }
      }
    }
  }

  // ---- the second convolution, shortcut, ReLU, one rounding ----
  const __amdgpu_buffer_rsrc_t rr = buffer_of(p.res, p.res_bytes);
  const __amdgpu_buffer_rsrc_t yr = buffer_of(p.y, p.y_bytes);
  if constexpr (ROWS) {
#pragma unroll
    for (int d = 0; d < DQ; ++d)
#pragma unroll
      for (int r = 0; r < 3; ++r) load_rows2(wf * 16)(d, r, ar[d][r]);
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d) load2(wf * 16)(d, a[d]);
  }
  uint32_t origin_b[MB], y_at[MB], r_at[MB];
  {
    // (ROWS: 16 lanes for a row of TW pixels)
    const int first = wp * 16 + li, dr = ROWS ? 1 : div_by(apart, p.divTW), dc = ROWS ? 0 : apart - dr * p.TW;
    int r = ROWS ? wp * MB : div_by(first, p.divTW), c = ROWS ? li : first - r * p.TW;
    const uint32_t unit = (uint32_t)(p.slots2 * 16), yu = (uint32_t)(p.ycs * ES), ru = (uint32_t)(p.rss * p.rcs * ES);
    uint32_t origin = (uint32_t)p.mid_at + (uint32_t)(r * p.MW + c) * unit;
    uint32_t y = (uint32_t)((n * p.P + oh0 + r) * p.Q + ow0 + c) * yu;
    uint32_t res = (uint32_t)((n * p.rH + (oh0 + r) * p.rss) * p.rW + (ow0 + c) * p.rss) * (uint32_t)(p.rcs * ES);
    const uint32_t step = (uint32_t)(dr * p.MW + dc) * unit, turn = (uint32_t)(p.MW - p.TW) * unit;
    const uint32_t y_step = (uint32_t)(dr * p.Q + dc) * yu, y_turn = (uint32_t)(p.Q - p.TW) * yu;
    const uint32_t r_step = (uint32_t)(dr * p.rW + dc) * ru, r_turn = (uint32_t)(p.rW - p.TW) * ru;
#pragma unroll
    for (int mt = 0; mt < MB; ++mt) {
      const bool in = ROWS ? c < p.TW : first + mt * apart < p.outs, ok = in && oh0 + r < p.P && ow0 + c < p.Q;
      origin_b[mt] = in ? origin : (uint32_t)p.mid_at;
      y_at[mt] = ok ? y : kOutside;
      r_at[mt] = ok ? res : kOutside;
      c += dc;
      r += dr;
      origin += step;
      y += y_step;
      res += r_step;
      const bool over = !ROWS && c >= p.TW;
      c -= over ? p.TW : 0;
      r += over ? 1 : 0;
      origin += over ? turn : 0u;
      y += over ? y_turn : 0u;
      res += over ? r_turn : 0u;
    }
  }
  __syncthreads();
  for (int f = wf * 16; f < p.Kp2; f += p.WF * 16) {
    if (f != wf * 16) {
      if constexpr (ROWS) {
#pragma unroll
        for (int d = 0; d < DQ; ++d)
#pragma unroll
          for (int r = 0; r < 3; ++r) load_rows2(f)(d, r, ar[d][r]);
      } else {
#pragma unroll
        for (int d = 0; d < D; ++d) load2(f)(d, a[d]);
      }
    }
    const int k0 = f + g * 4, kk = k0 - p.roff;
    f32x4 acc[MB];
    f32x4 b4 = b2v;
    if (f != wf * 16) b4 = *reinterpret_cast<const f32x4*>(p.b2 + min(k0, p.Kp2 - 4));
#pragma unroll
    for (int mt = 0; mt < MB; ++mt) acc[mt] = b4;
    // (without a shortcut its extent is 0: zeros)
    const bool in_res = kk >= 0 && kk < p.rcs;
    u32x2 early[MB];                       // ROWS: registers to spare for the shortcut while it multiplies
    if constexpr (ROWS)
#pragma unroll
      for (int mt = 0; mt < MB; ++mt)
        early[mt] = __builtin_amdgcn_raw_buffer_load_b64(rr, in_res ? r_at[mt] + (uint32_t)kk * 2u : kOutside, 0, 0);
    if constexpr (ROWS)
      multiply_rows<BF, MB, DQ>(lds, (uint32_t)(p.mid_at + (wp * MB * 16 + li) * p.slots2 * 16),
                                (uint32_t)(16 * p.slots2 * 16), table2, g, (uint32_t)p.zero_at, p.rows2, ar, acc,
                                load_rows2(f));
    else
      multiply<EL, MB, D, NB>(lds, origin_b, table2, g, (uint32_t)p.zero_at, p.steps2, a, acc, load2(f));
    const uint32_t floor2 = p.relu2 ? 0u : 0x80008000u;
    if constexpr (F32) {
      f32x4 r[MB];
#pragma unroll
      for (int mt = 0; mt < MB; ++mt)
        r[mt] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                              rr, in_res ? r_at[mt] + (uint32_t)kk * 4u : kOutside, 0, 0));
#pragma unroll
      for (int mt = 0; mt < MB; ++mt) {
        f32x4 v = acc[mt];
        v += r[mt];
        if (p.relu2)
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], 0.f);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), yr,
                                               k0 < p.ycs ? y_at[mt] + (uint32_t)k0 * 4u : kOutside, 0, 0);
      }
    } else {
      u32x2 r[MB];
#pragma unroll
      for (int mt = 0; mt < MB; ++mt)
        r[mt] = ROWS ? early[mt] : __builtin_amdgcn_raw_buffer_load_b64(
                                       rr, in_res ? r_at[mt] + (uint32_t)kk * 2u : kOutside, 0, 0);
#pragma unroll
      for (int mt = 0; mt < MB; ++mt) {
        const f32x4& v = acc[mt];
        u32x2 o;
        o[0] = clamp_below(pack2<BF>(v[0] + to_float<BF>((uint16_t)(r[mt][0] & 0xffffu)),
                                     v[1] + to_float<BF>((uint16_t)(r[mt][0] >> 16))), floor2);
        o[1] = clamp_below(pack2<BF>(v[2] + to_float<BF>((uint16_t)(r[mt][1] & 0xffffu)),
                                     v[3] + to_float<BF>((uint16_t)(r[mt][1] >> 16))), floor2);
        __builtin_amdgcn_raw_buffer_store_b64(o, yr, k0 < p.ycs ? y_at[mt] + (uint32_t)k0 * 2u : kOutside, 0, 0);
      }
    }
  }
}

// MA, MB: most tiles of 16 pixels per wave; D: steps of weights in flight; NB: pixel buffers; min_waves:
// waves per SIMD the registers allow (a third buffer would spill 91 of 128 with eight tiles).  rows: the
// tiles are rows (MA and MB rows per wave exactly).
struct BasicTile {
  int MA, MB, D, NB, min_waves;
  bool rows;
};
constexpr BasicTile kTiles[] = {{2, 1, 6, 3, 4, false},  {3, 2, 6, 3, 4, false}, {4, 3, 6, 3, 4, false},
                                {6, 4, 6, 2, 4, false},  {8, 7, 6, 2, 4, false}, {16, 13, 6, 3, 2, false},
                                {4, 3, 4, 2, 4, true},   {8, 6, 4, 2, 2, true},
                                {8, 7, 2, 2, 4, true},   {16, 14, 4, 2, 2, true}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
// Rectangles that are weighed, rows x columns, and the name of each.  The last two are multiplied by rows.
struct Rectangle {
  int rows, cols;
  bool by_rows;
  const char* name;
};
constexpr Rectangle kRectangles[] = {
    {2, 8, false, "basic_block_2x8"},     {4, 4, false, "basic_block_4x4"},   {4, 8, false, "basic_block_4x8"},
    {7, 7, false, "basic_block_7x7"},     {8, 8, false, "basic_block_8x8"},   {7, 14, false, "basic_block_7x14"},
    {8, 16, false, "basic_block_8x16"},   {14, 14, false, "basic_block_14x14"},
    {6, 14, true, "basic_block_6x14r"},   {14, 14, true, "basic_block_14x14r"}};
constexpr int kNumRectangles = sizeof(kRectangles) / sizeof(kRectangles[0]);

// LDS slots of 16 bytes per pixel: 16 lanes read 16 bytes each of neighbouring pixels, which is free
// of bank conflicts at odd multiples of 32 bytes
int pad_slots(int chunks, bool strided) {
  if (strided) return chunks | 1;
  while (chunks % 4 != 2) ++chunks;
  return chunks;
}

struct BasicPlan {
  BasicParams p;
  int rectangle, tile;
  size_t lds;
};

bool plan_basic(const BasicBlockArgs& a, int N, int rectangle, int WF, BasicPlan* out) {
  const Rectangle& R = kRectangles[rectangle];
  if (R.by_rows && (a.dt == FUPR_F32 || a.s1.stride != 1)) return false;
  BasicParams& p = out->p;
  p = BasicParams{};
  const int es = (int)elem_size(a.dt), per_chunk = 16 / es;
  const PackedLayout L1 = packed_layout(a.s1, a.dt), L2 = packed_layout(a.s2, a.dt);
  if (std::max(weight_bytes(L1), weight_bytes(L2)) >= kOutside) return false;   // (32-bit offsets)
  p.H = a.H; p.W = a.W; p.stride = a.s1.stride;
  p.P = out_extent(a.H, 3, p.stride, 1);
  p.Q = out_extent(a.W, 3, p.stride, 1);
  p.TH = std::min(R.rows, p.P);
  p.TW = std::min(R.cols, p.Q);
  p.MW = p.TW + 2;
  p.mids = (p.TH + 2) * p.MW;
  p.outs = p.TH * p.TW;
  p.IW = (p.TW + 1) * p.stride + 3;
  p.in_pixels = ((p.TH + 1) * p.stride + 3) * p.IW;
  p.Kp1 = L1.Kp; p.cpt1 = L1.Cp / per_chunk; p.nchunk1 = 9 * p.cpt1; p.steps1 = (p.nchunk1 + 3) / 4;
  p.Kp2 = L2.Kp; p.cpt2 = L2.Cp / per_chunk; p.nchunk2 = 9 * p.cpt2; p.steps2 = (p.nchunk2 + 3) / 4;
  p.w1_bytes = (uint32_t)(L1.nchunk_pad * L1.Kp) * (es == 4 ? 4u : 16u);
  p.w2_bytes = (uint32_t)(L2.nchunk_pad * L2.Kp) * (es == 4 ? 4u : 16u);
  p.WF = WF;
  while ((1 << p.log2_WF) < WF) ++p.log2_WF;
  const int WP = kWaves / WF;
  p.rows1 = (3 * p.cpt1 + 3) / 4;
  p.rows2 = (3 * p.cpt2 + 3) / 4;
  int ma = ((p.mids + 15) / 16 + WP - 1) / WP, mb = ((p.outs + 15) / 16 + WP - 1) / WP;
  if (R.by_rows) {
    if (p.TH != R.rows || p.TW != R.cols || p.MW != 16) return false;
    ma = (p.TH + 2) / WP;
    mb = p.TH / WP;
  }
  out->tile = 0;
  auto fits = [&](const BasicTile& T) {
    return T.rows == R.by_rows && (T.rows ? T.MA == ma && T.MB == mb && ma * WP == p.TH + 2 && mb * WP == p.TH
                                          : T.MA >= ma && T.MB >= mb);
  };
  while (out->tile < kNumTiles && !fits(kTiles[out->tile])) ++out->tile;
  if (out->tile == kNumTiles) return false;
  p.slots1 = pad_slots(p.cpt1, p.stride == 2);
  p.slots2 = pad_slots(std::max(p.cpt2, p.Kp1 / per_chunk), false);
  size_t end = round_up_sz((size_t)p.in_pixels * p.slots1 * 16, 1024);
  p.mid_at = (int)end;
  end += (size_t)p.mids * p.slots2 * 16;
  p.table1_at = (int)end;
  end += (size_t)(p.steps1 + 1) * 16;
  p.table2_at = (int)end;
  end += (size_t)(p.steps2 + 1) * 16;
  p.zero_at = (int)round_up_sz(end, 16);      // 256 bytes of zeros, past everything that is read
  out->lds = (size_t)p.zero_at + 1024 + 1024;
  if (out->lds > kLdsLimit) return false;
  p.tiles_w = (p.Q + p.TW - 1) / p.TW;
  p.tiles = p.tiles_w * ((p.P + p.TH - 1) / p.TH);
  const int64_t total = (int64_t)N * p.tiles;
  if (total >= (int64_t(1) << 28)) return false;
  p.total = (int)total;
  p.per_xcd = (p.total + 7) / 8;
  out->rectangle = rectangle;
  return true;
}

// What only a launch needs: plans that are weighed do without.
void set_divisions(BasicParams& p) {
  p.divC1 = fast_div(p.cpt1); p.divC2 = fast_div(p.cpt2); p.divMW = fast_div(p.MW); p.divTW = fast_div(p.TW);
  p.divSlots = fast_div(p.slots1); p.divIW = fast_div(p.IW); p.divTiles = fast_div(p.tiles);
  p.divTilesW = fast_div(p.tiles_w);
}

template <int EL, int TILE>
fupr_status launch_as(const BasicPlan& plan, hipStream_t st) {
  constexpr BasicTile T = kTiles[TILE];
  if constexpr (T.rows && EL == FUPR_F32) {
    return FUPR_ERR_LIMIT;             // (no such plan)
  } else {
    auto kernel = basic_block_kernel<EL, T.MA, T.MB, T.D, T.NB, T.min_waves, T.rows>;
    if (plan.lds > 64 * 1024) {
      static const hipError_t attr = hipFuncSetAttribute(
          reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
      if (attr != hipSuccess) return FUPR_ERR_LAUNCH;
    }
    void* list[] = {const_cast<BasicParams*>(&plan.p)};
    return launched(hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)(plan.p.per_xcd * 8)),
                                    dim3(kThreads), list, plan.lds, st),
                    "basic_block_kernel");
  }
}

template <int EL>
fupr_status dispatch(const BasicPlan& plan, hipStream_t st) {
  switch (plan.tile) {
    case 0: return launch_as<EL, 0>(plan, st);
    case 1: return launch_as<EL, 1>(plan, st);
    case 2: return launch_as<EL, 2>(plan, st);
    case 3: return launch_as<EL, 3>(plan, st);
    case 4: return launch_as<EL, 4>(plan, st);
    case 5: return launch_as<EL, 5>(plan, st);
    case 6: return launch_as<EL, 6>(plan, st);
    case 7: return launch_as<EL, 7>(plan, st);
    case 8: return launch_as<EL, 8>(plan, st);
    case 9: return launch_as<EL, 9>(plan, st);
  }
  return FUPR_ERR_LIMIT;
}

// Estimated us of a plan: a fit over 228 blocks (ResNet-18's at several image sizes, CIFAR-size ones in single
// precision, 1 - 128 images) x every rectangle and wave arrangement, 6015 launches, to 9 % in the mean
// square; the plan with the least estimate is 1.8 % slower than the best one in the mean, 20 % at worst.  (Single
// precision before its sums of a step were added up apart, which took 2 us of 103 of a network of six blocks:
// the rule that takes a plan asks for a larger gain there.)
double estimate(const BasicBlockArgs& a, const BasicPlan& plan) {
  const BasicParams& p = plan.p;
  const BasicTile& T = kTiles[plan.tile];
  const int WP = kWaves / p.WF, ft1 = (p.Kp1 + 15) / 16, ft2 = (p.Kp2 + 15) / 16;
  const double mfma = a.dt == FUPR_F32 ? 128.0 : 16.0;   // clocks of the matrix pipe per tile and step
  const double es = (double)elem_size(a.dt), slots = (double)p.in_pixels * p.slots1;
  const int per_cu = (p.total + kComputeUnits - 1) / kComputeUnits;
  const int resident = std::max(1, std::min({per_cu, T.min_waves / 2, (int)(kLdsLimit / plan.lds)}));
  const double pixels = (double)p.total / p.tiles * p.P * p.Q;
  const double hbm = pixels * es * (p.stride * p.stride * a.s1.C + 2.0 * a.s2.K) / 4.5e6;
  if (T.rows) {
    // (the same form, fitted to 128 launches of 41 blocks to 7 %; LDS reads are hidden)
    const int st1 = 3 * p.rows1, st2 = 3 * p.rows2;
    const double alone = 8042.0 + 2.75 * slots + (ft1 + p.WF - 1) / p.WF * st1 * T.MA * 16.0 +
                         (ft2 + p.WF - 1) / p.WF * T.MB * (st2 * 16.0 + 328.0);
    const double matrix = 4.92 * WP * (ft1 * T.MA * st1 + ft2 * T.MB * st2);
    const double memory = ((ft1 * st1 + ft2 * st2) * 1024.0 * WP + p.in_pixels * a.s1.C * es + 140.0 * slots +
                           2.0 * p.outs * a.s2.K * es) / 76.8;
    const double clocks = std::max((per_cu + resident - 1) / resident * alone,
                                   per_cu * (std::max(matrix, memory) + 0.40 * (matrix + memory)) + 0.27 * alone);
    return 3.62 + std::max(clocks / 2400.0, hbm);
  }
  // clocks of a workgroup that has the compute unit to itself
  const double alone = 11267.0 + 0.788 * slots + (ft1 + p.WF - 1) / p.WF * p.steps1 * T.MA * (mfma + 12.0) +
                       (ft2 + p.WF - 1) / p.WF * T.MB * (p.steps2 * (mfma + 12.0) + 581.0);
  // and what it takes of the compute unit: LDS, matrix pipe, vector memory
  const double tiles = (double)WP * (ft1 * T.MA * p.steps1 + ft2 * T.MB * p.steps2);
  const double lds = 1.43 * tiles, matrix = 0.0795 * mfma * tiles;
  const double memory = ((ft1 * p.steps1 + ft2 * p.steps2) * 1024.0 * WP + p.in_pixels * a.s1.C * es + 77.6 * slots +
                         2.0 * p.outs * a.s2.K * es) / 216.0;
  const double clocks = std::max((per_cu + resident - 1) / resident * alone,
                                 per_cu * (std::max({lds, matrix, memory}) + 1.867 * (lds + matrix + memory)) + 0.557 * alone);
  return 3.62 + std::max(clocks / 2400.0, hbm);
}

// Estimated us of the two operators as launches of their own, fitted to the same blocks (to 6 %).
double estimate_apart(const BasicBlockArgs& a, double pixels) {
  const double es = (double)elem_size(a.dt), rate = a.dt == FUPR_F32 ? 102e6 : 810e6;
  auto one = [&](double bytes, double flops) {
    const double mb = bytes / 1e6;
    return 6.46 + std::max(mb / 3.5, flops / rate) + 0.339 * std::sqrt(mb);
  };
  return one(pixels * es * (a.s1.stride * a.s1.stride * a.s1.C + a.s1.K), pixels * 18 * a.s1.C * a.s1.K) +
         one(pixels * es * (a.s1.K + 2.0 * a.s2.K), pixels * 18 * a.s1.K * a.s2.K);
}

// The tuning switch basic_tile=<index of the rectangle>x<waves along the filters> forces a plan.
// like >= 0: only rectangles whose sums' order is that one's.  (Some thirty plans, 2 - 20 us of host time: a model
// asks once for a batch size and keeps the answer, a thread remembers it for the next model.)
bool pick_basic(const BasicBlockArgs& a, int N, int like, BasicPlan* best, double* cost) {
  char text[32];
  if (tuning_text("basic_tile", text, sizeof(text))) {
    int rectangle = -1, wf = 8;
    *cost = 0.0;
    if (std::sscanf(text, "%dx%d", &rectangle, &wf) != 2 || rectangle < 0 || rectangle >= kNumRectangles) return false;
    if (wf != 1 && wf != 2 && wf != 4 && wf != 8) return false;
    return plan_basic(a, N, rectangle, wf, best);
  }
  bool any = false;
  const int last = kNumRectangles - 1;
  const bool by_rows = plan_basic(a, N, last, kWaves, best) || plan_basic(a, N, last, 4, best);
  for (int r = 0; r < kNumRectangles; ++r)
    for (int wf = 1; wf <= kWaves; wf *= 2) {
      BasicPlan plan;
      // (14 columns by rows: never slower than other tiles of them, 36.0 against 43.2 us at 64 x 56 x 56 x 64)
      if (!kRectangles[r].by_rows && kRectangles[r].cols == 14 && by_rows) continue;
      if (like >= 0 && kRectangles[r].by_rows != kRectangles[like].by_rows) continue;
      if (!plan_basic(a, N, r, wf, &plan)) continue;
      // (a near tie is better by rows: 17.0 against 21.3 us at 20 x 56 x 56 x 64 -> 32 -> 64)
      const double c = estimate(a, plan) * (by_rows && !kRectangles[r].by_rows ? 1.02 : 1.0);
      if (any && c >= *cost) continue;
      *best = plan;
      *cost = c;
      any = true;
    }
  return any;
}

// A plan's number.
int number_of(const BasicPlan& plan) { return plan.rectangle * (kWaves + 1) + plan.p.WF; }
int rectangle_of(int number) { return number / (kWaves + 1); }
int waves_of(int number) { return number % (kWaves + 1); }

// The plan with which a batch of N images runs the block as one launch, -1: it runs as two.
int choose(const BasicBlockArgs& a, int N) {
  if (tuning_off("basic_fuse")) return -1;
  BasicPlan plan;
  double cost;
  if (!pick_basic(a, N, -1, &plan, &cost)) return -1;
  char text[32];
  if (tuning_text("basic_tile", text, sizeof(text))) return number_of(plan);
  // Short launches: 8 % less than the launches apart, which is what the two estimates are uncertain by;
  // both were fitted to launches between events, which takes some 1.5 us more for each than one after
  // the other.  Long ones: one after the other they take longer than alone by more than the launches apart
  // do, which are better at running side by side, so 22 %, and 25 % where a compute unit holds one workgroup
  // at a time.  Networks at 8 - 20 %: ResNet-34 of 256 images 0.986x, ResNet-18 of 128, unpruned, 0.990x, of 80,
  // unpruned, 0.993x, of 250 0.994x; at 23 - 30 %: of 64 1.12x, of 160 1.07x, of 200 1.02x.
  const double apart =
      estimate_apart(a, (double)N * out_extent(a.H, 3, a.s1.stride, 1) * out_extent(a.W, 3, a.s1.stride, 1));
  const bool one_at_a_time = plan.p.total > kComputeUnits && plan.lds > kLdsLimit / 2;
  if (apart > 30.0 ? cost >= (one_at_a_time ? 0.75 : 0.78) * apart : cost - 1.5 >= 0.92 * (apart - 3.0)) return -1;
  if (a.alone) return number_of(plan);   // (the call's own time, which one launch less shortens: 8.6 -> 7.9 us)
  // Inside a network, each block by itself as one launch and as two, us of the captured pass:
  if (a.dt == FUPR_F32) {
    // The two launches are 3 - 4 us shorter than between events, and shorter still below some 128K
    // elements: blocks of 16 channels at 32 x 32 gain 0.5 us at 8 images and lose 1.3 at one to four, where whole
    // networks took 1.05 times as long (20 layers, 4 images: 83.0 us apart, 88.0 as blocks).
    // Past 12.5 us the launches apart have the faster pixels (64 images, 56 layers: 375 - 410 us apart, 433 as blocks).
    if (cost + 3.4 > apart || cost > 12.5 || (int64_t)N * a.H * a.W * a.s1.C < (1 << 17)) return -1;
  } else {
    // From 192 images on two sub-batches run side by side (split_count in model.cpp), which short launches apart are
    // better at: 3.6 - 4.5 us a block lost at 24 x 24 (ResNet-18 of 192 images of 96 x 96 206.4 us apart, 213.6 as
    // blocks); 5.9 gained at 56 x 56.
    if (N >= 192 && apart < 60.0) return -1;
    // The shortest ones have to be clearly shorter (10.5 of 13.2 us lost 0.7, 9.5 of 13.3 gains 1.0).
    if (apart < 14.5 && cost + 1.5 > 0.88 * apart) return -1;
  }
  return number_of(plan);
}

}  // namespace

bool basic_block_applies(const BasicBlockArgs& a) {
  for (const fupr_conv_shape* s : {&a.s1, &a.s2})
    if (s->R != 3 || s->S != 3 || s->pad != 1) return false;
  if ((a.s1.stride != 1 && a.s1.stride != 2) || a.s2.stride != 1) return false;
  const WithoutTuning no_switches;   // (they can change between a model's plan and its passes)
  BasicPlan plan;
  for (int r = 0; r < kNumRectangles; ++r)
    for (int wf = 1; wf <= kWaves; wf *= 2)
      if (plan_basic(a, 1, r, wf, &plan)) return true;
  return false;
}

int basic_block_plan(const BasicBlockArgs& a, int N) {
  if (tuning_any()) return choose(a, N);
  const WithoutTuning no_switches;   // (one that is set meanwhile is in no answer that is kept)
  return recall<BasicBlockArgs, choose>(a, N);
}

// The sums' order depends on by_rows alone: a part keeps its batch's.
int basic_block_plan_part(const BasicBlockArgs& a, int plan, int count) {
  BasicPlan part;
  double cost;
  return pick_basic(a, count, rectangle_of(plan), &part, &cost) ? number_of(part) : plan;
}

const char* basic_block_name(int plan) { return kRectangles[rectangle_of(plan)].name; }

fupr_status launch_basic_block(const BasicBlockArgs& a, const ConvArgs& first, const ConvArgs& second, int number,
                               int count, void* stream) {
  BasicPlan plan;
  if (!plan_basic(a, count, rectangle_of(number), waves_of(number), &plan)) return FUPR_ERR_LIMIT;
  BasicParams& p = plan.p;
  set_divisions(p);
  const uint32_t es = (uint32_t)elem_size(a.dt);
  p.x = first.x; p.res = second.res; p.y = second.y;
  p.w1 = reinterpret_cast<const char*>(first.packed) + packed_layout(a.s1, a.dt).weight_offset;
  p.w2 = reinterpret_cast<const char*>(second.packed) + packed_layout(a.s2, a.dt).weight_offset;
  p.b1 = reinterpret_cast<const float*>(first.packed);
  p.b2 = reinterpret_cast<const float*>(second.packed);
  p.pix = first.xcs * (int)es;
  p.x_bytes = (uint32_t)count * (uint32_t)(p.H * p.W) * (uint32_t)p.pix;
  p.ycs = second.ycs;
  p.y_bytes = (uint32_t)count * (uint32_t)(p.P * p.Q * p.ycs) * es;
  p.relu1 = first.relu; p.relu2 = second.relu;
  if (second.res) {
    p.rH = second.rH; p.rW = second.rW; p.rcs = second.rcs; p.rss = second.rss; p.roff = second.roff;
    p.res_bytes = (uint32_t)count * (uint32_t)(p.rH * p.rW * p.rcs) * es;
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  return a.dt == FUPR_F32 ? dispatch<FUPR_F32>(plan, st)
                          : a.dt == FUPR_BF16 ? dispatch<FUPR_BF16>(plan, st) : dispatch<FUPR_F16>(plan, st);
}

}  // namespace fupr
