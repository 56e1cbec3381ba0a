// A whole small-image network in ONE kernel: one workgroup per image, every
// activation tensor of that image AND the current layer's parameters resident
// in LDS, layers walked from a table.
//
// At CIFAR sizes (Table II, 32x32 inputs) each per-layer kernel runs for a few
// microseconds and the forward pass is bound by launches and by activations
// bouncing through L2; here an image's activations never leave the compute unit
// between the input read and the logits write.  What the paper removes by
// folding non-parametric operators into convolutions ("Sys.", "BN", "Add"
// columns of Table VI) is removed here one level further: the operator
// boundaries themselves.
//
// Per layer: the next layer's parameter blob and tap table are on their way from
// global memory into LDS WHILE the current layer is computed, so no
// global-memory latency sits on the layer chain; both MFMA operands of the
// current layer (filters = A, pixels = B) come from LDS.
// A work item is MT pixel tiles x NT filter tiles of 16 x 16, so every LDS
// fragment feeds several MFMAs.
//
// The instruction stream around the MFMAs is what bounds a network this small,
// so it is kept short: the accumulator starts from the bias, and the shortcut is
// added by one more MFMA step whose filter operand is a one-hot (identity)
// fragment built in registers — the epilogue is ReLU, one rounding and one LDS
// store.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "device_utils.h"
#include "fupr.h"
#include "layout.h"

namespace fupr {
namespace {

// floor(v / d) for v < 2^16 from the host's reciprocal of d (0 stands for d = 1).
__device__ __forceinline__ int div_magic(int v, uint32_t magic) {
  return magic ? (int)__umulhi((uint32_t)v, magic) : v;
}

// Zeroes the halo ring (hp pixels wide) around a P x Q tensor whose interior
// starts at byte offset org; Wh = Q + 2*hp pixels per row, ps2 bytes per pixel,
// chunks 16-byte units per pixel that hold channels.
template <int THREADS>
__device__ __forceinline__ void zero_halo(char* act, int org, int P, int Q, int Wh, int ps2,
                                          int chunks, int hp, int tid) {
  const int raw = org - hp * (Wh + 1) * ps2;
  const int top_bottom = 2 * hp * Wh;
  const int total = (top_bottom + 2 * hp * P) * chunks;
  for (int i = tid; i < total; i += THREADS) {
    const int px = i / chunks, ch = i - px * chunks;
    int row, col;
    if (px < top_bottom) {
      const int rr = px / Wh;
      col = px - rr * Wh;
      row = rr < hp ? rr : P + rr;
    } else {
      const int q = px - top_bottom;
      const int rr = q / (2 * hp), cc = q - rr * 2 * hp;
      row = hp + rr;
      col = cc < hp ? cc : Q + cc;
    }
    *reinterpret_cast<uint4*>(act + raw + (row * Wh + col) * ps2 + ch * 16) = uint4{0u, 0u, 0u, 0u};
  }
}

// The filter fragment of the shortcut step for filter tile ft: row i (= filter
// ft*16 + i) has a single 1.0 at reduction index i, so the MFMA adds shortcut
// channel ft*16 + i to that filter's accumulator; rows beyond the shortcut's
// channel count stay zero (a shortcut with fewer channels than the block
// output is the zero-padded kind).
template <bool BF>
__device__ __forceinline__ uint4 identity_fragment(int ft, int res_cs, int li, int g) {
  const uint32_t one = BF ? 0x3f80u : 0x3c00u;
  const bool on = g == (li >> 3) && ft * 16 + li < res_cs;
  const uint32_t v = on ? one << ((li & 1) * 16) : 0u;
  const int j = (li & 7) >> 1;
  return uint4{j == 0 ? v : 0u, j == 1 ? v : 0u, j == 2 ? v : 0u, j == 3 ? v : 0u};
}

// Pixel addressing of a wave's first work item, kept from one layer to the next:
// consecutive layers of one resolution give a wave the same pixels at the same
// strides, so the divisions and multiplications behind these offsets are done
// once per resolution rather than once per layer.
struct PixelCache {
  int rin[4];    // byte offset of the pixel's window from the window of pixel 0, per pixel tile
};

typedef short short2_t __attribute__((ext_vector_type(2)));

// max(x, floor) on two packed 16-bit floats, as signed 16-bit integers: with
// floor = 0 this is ReLU (negative floats are negative integers), with floor =
// the most negative integer it is the identity.
__device__ __forceinline__ uint32_t clamp_below(uint32_t v, uint32_t floor2) {
  const short2_t a = __builtin_bit_cast(short2_t, v), f = __builtin_bit_cast(short2_t, floor2);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, f));
}

// All work items of one conv layer that fall to this wave.  LAST: the layer
// writes the network output to global memory instead of LDS.
//
// Every activation tensor in LDS carries a ring of zero pixels as wide as the
// largest padding of any convolution, so a tap never needs a bounds check: the
// K loop is MT + 1 address additions, MT + NT LDS reads and MT * NT MFMAs per
// step, plus one table read per step issued a whole group of steps ahead.  D
// steps of operands are kept in flight (ring of register buffers, loop
// unrolled by D).
template <bool BF, int WAVES, int MT, int NT, bool LAST>
__device__ __forceinline__ void conv_items(const ResLayer& L, const ResParams& p, char* act,
                                           int n, int lane, int wave, PixelCache& pc) {
  constexpr int D = (MT + NT <= 3) ? 4 : (MT + NT == 4 ? 3 : 2);
  const int li = lane & 15, g = lane >> 4;
  const int nsteps = L.nsteps, FT = L.FT, M = L.M, Q = L.Q;
  const bool has_res = L.res_org >= 0;
  const bool full_pixels = (L.flags & kResFullPixels) != 0;     // no pixel tile is ragged
  const bool full_filters = (L.flags & kResFullFilters) != 0;   // no filter tile is missing or partly stored
  const bool reuse = (L.flags & kResReuse) != 0;                // pc holds this layer's first item
  const uint32_t floor2 = (L.flags & kResRelu) ? 0u : 0x80008000u;
  const int ycs = LAST ? p.y_cs : L.cs_out;
  const int wstep = L.wstep;
  const int a_lane = L.wts_off + g * (wstep >> 2) + li * 16;
  const float* bias = reinterpret_cast<const float*>(act + L.w_off);
  const int tab_lane = L.tab_off + g * 4;
  const int n_items = L.n_items, n_fgroups = L.n_fgroups;

  for (int item = wave; item < n_items; item += WAVES) {
    const int pg = div_magic(item, L.magicF);
    const int ft0 = (item - pg * n_fgroups) * NT;
    // filter tiles past the last one repeat it (computed, not stored)
    int ft[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) ft[t] = min(ft0 + t, FT - 1);

    // Table entries of the first two groups of steps and the bias are requested
    // first: their latency passes while the addresses are worked out.  (The
    // table is padded by 2 * D steps, so no index needs clamping.)
    int e0[D], e_cur[D];   // entries of steps 0 .. D-1 and D .. 2D-1
#pragma unroll
    for (int d = 0; d < D; ++d) e0[d] = *reinterpret_cast<const int*>(act + tab_lane + d * 16);
#pragma unroll
    for (int d = 0; d < D; ++d)
      e_cur[d] = *reinterpret_cast<const int*>(act + tab_lane + (D + d) * 16);
    int tptr = tab_lane + 2 * D * 16;
    f32x4 b4[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
      b4[t] = *reinterpret_cast<const f32x4*>(bias + ft[t] * 16 + g * 4);

    int m[MT], rin[MT], rout[MT];
    if (reuse && item == wave) {
      // same pixels, same strides as in the previous layer; output strides = input strides
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        m[mt] = 0;   // not looked at: no pixel tile is ragged
        rin[mt] = pc.rin[mt];
        rout[mt] = rin[mt] + g * 8;
      }
    } else {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        m[mt] = (pg * MT + mt) * 16 + li;
        const int mc = min(m[mt], M - 1);
        const int pp = div_magic(mc, L.magicQ), qq = mc - pp * Q;
        rin[mt] = pp * L.in_row + qq * L.in_col;
        rout[mt] = pp * L.out_row + qq * L.out_col + g * 8;
        pc.rin[mt] = rin[mt];
      }
    }

    // shortcut operands: 16 bytes of the shortcut pixel per lane
    uint4 rb[MT][NT];
    if (has_res) {
      int cres[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
        cres[t] = L.res_org + min(ft[t] * 2 + (g & 1), (L.res_cs >> 3) - 1) * 16;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        int rres;
        if (L.flags & kResLikeOut) {
          rres = rout[mt] - g * 8;
        } else {
          const int mc = min(m[mt], M - 1);
          const int pp = div_magic(mc, L.magicQ), qq = mc - pp * Q;
          rres = pp * L.res_row + qq * L.res_col;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
          rb[mt][t] = *reinterpret_cast<const uint4*>(act + rres + cres[t]);
      }
    }

    int aptr = a_lane + ft0 * 256;
    uint4 a[D][NT], b[D][MT];
    auto operands = [&](const int e, uint4* av, uint4* bv) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        bv[mt] = *reinterpret_cast<const uint4*>(act + rin[mt] + e);   // e includes the origin
#pragma unroll
      for (int t = 0; t < NT; ++t)
        av[t] = *reinterpret_cast<const uint4*>(act + aptr + (ft[t] - ft0) * 256);
      aptr += wstep;
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < nsteps) operands(e0[d], a[d], b[d]);

    // The accumulator starts from the bias.  The shortcut goes in first: one
    // MFMA step whose filter fragment is one-hot.
    f32x4 acc[MT][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (has_res && ft[t] * 16 < L.res_cs) {
        const uint4 ia = identity_fragment<BF>(ft[t], L.res_cs, li, g);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt][t] = mfma_16x16x32<BF>(ia, rb[mt][t], b4[t]);
      } else {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt][t] = b4[t];
      }
    }

    // scheduling hint: one LDS read and one address addition in the shadow of
    // each of the next n MFMAs (a wave alone on its SIMD otherwise issues the
    // MFMAs back to back and only then the reads)
    auto interleave = [](int n) {
#pragma unroll
      for (int i = 0; i < n; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);   // vector ALU
      }
    };
    auto mfmas = [&](const uint4* av, const uint4* bv) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mt][t] = mfma_16x16x32<BF>(av[t], bv[mt], acc[mt][t]);
    };
    // The table entries a step needs are read a whole group of D steps ahead
    // of it.  Main part: groups whose D steps and D refills all exist, no
    // condition inside; then at most 2D - 1 steps with conditions.
    int step0 = 0;
    for (; step0 + 2 * D <= nsteps; step0 += D) {
      int e_nxt[D];
#pragma unroll
      for (int d = 0; d < D; ++d) e_nxt[d] = *reinterpret_cast<const int*>(act + tptr + d * 16);
      tptr += D * 16;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        mfmas(a[d], b[d]);
        operands(e_cur[d], a[d], b[d]);
      }
      interleave(D * MT * NT);
#pragma unroll
      for (int d = 0; d < D; ++d) e_cur[d] = e_nxt[d];
    }
    for (; step0 < nsteps; step0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (step0 + d < nsteps) {
          mfmas(a[d], b[d]);
          if (step0 + d + D < nsteps) operands(e_cur[d], a[d], b[d]);
        }
      }
    }

    // epilogue: one rounding, ReLU on the rounded pair, store
    if (!LAST && MT % 2 == 0 && full_pixels && full_filters) {
      // Two pixel tiles at a time.  A lane holds 4 channels (8 bytes) of one
      // pixel of each tile; lanes 16 apart hold the next 4 channels of the same
      // pixel.  Swapping odd 16-lane rows of the first tile's registers with
      // even rows of the second's gives every lane 8 consecutive channels of
      // ONE pixel (even rows: first tile, odd rows: second tile): half as many
      // LDS stores, each 16 bytes.
#pragma unroll
      for (int mt = 0; mt < MT; mt += 2) {
        const int wsel = ((g & 1) ? rout[mt + 1] : rout[mt]) - g * 8 + (g >> 1) * 16;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const uint32_t p0 = clamp_below(pack2<BF>(acc[mt][t][0], acc[mt][t][1]), floor2);
          const uint32_t p1 = clamp_below(pack2<BF>(acc[mt][t][2], acc[mt][t][3]), floor2);
          const uint32_t q0 = clamp_below(pack2<BF>(acc[mt + 1][t][0], acc[mt + 1][t][1]), floor2);
          const uint32_t q1 = clamp_below(pack2<BF>(acc[mt + 1][t][2], acc[mt + 1][t][3]), floor2);
          const auto r0 = __builtin_amdgcn_permlane16_swap(p0, q0, false, false);
          const auto r1 = __builtin_amdgcn_permlane16_swap(p1, q1, false, false);
          *reinterpret_cast<uint4*>(act + wsel + (L.out_org + (ft0 + t) * 32)) =
              uint4{r0[0], r1[0], r0[1], r1[1]};
        }
      }
      continue;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        uint2 o;
        o.x = clamp_below(pack2<BF>(acc[mt][t][0], acc[mt][t][1]), floor2);
        o.y = clamp_below(pack2<BF>(acc[mt][t][2], acc[mt][t][3]), floor2);
        const int k0 = (ft0 + t) * 16 + g * 4;
        if (!full_pixels && m[mt] >= M) continue;
        if (!full_filters && (ft0 + t >= FT || k0 >= ycs)) continue;
        if constexpr (LAST) {
          uint16_t* yp = reinterpret_cast<uint16_t*>(p.y) +
                         ((size_t)n * p.out_pixels + m[mt]) * p.y_cs;
          *reinterpret_cast<uint2*>(yp + k0) = o;
        } else {
          *reinterpret_cast<uint2*>(act + rout[mt] + (L.out_org + (ft0 + t) * 32)) = o;
        }
      }
    }
  }
}

template <bool BF, int WAVES, int MT, int NT>
__device__ __forceinline__ void conv_layer(const ResLayer& L, const ResParams& p, char* act,
                                           int n, int lane, int wave, PixelCache& pc) {
  if (L.flags & kResLast) conv_items<BF, WAVES, MT, NT, true>(L, p, act, n, lane, wave, pc);
  else conv_items<BF, WAVES, MT, NT, false>(L, p, act, n, lane, wave, pc);
}

// What a computing wave needs of a ResRow.
struct RowWork {
  int32_t kind, wts_off, kp16, in_org, out_org, res_org, tap_row, tap_col, out_row, out_col, res_row, res_col;
  int32_t half_in, half_out, half_res, res_cs;
  int in, out, res;          // the wave's entries of wave_in, wave_out, wave_res
  int swizzle, res_step;
};

// Byte address bits 5 and 6 of a chunk of the pixel in column x are flipped by this (row_swizzle_mask); s: shift | mask << 2.
__device__ __forceinline__ int swizzle_of(int x, int s) { return ((x >> (s & 3)) & ((s >> 2) & 3)) << 5; }

// The layer table is read through the constant address space so that every
// descriptor load is a scalar load (a uniform load from plain global memory
// after the kernel's first store becomes a vector load whose wait would also
// drain the parameter staging in flight).
typedef const uint32_t __attribute__((address_space(4)))* ConstWords;
typedef void __attribute__((address_space(3)))* LdsPtr;

template <class T>
__device__ __forceinline__ T load_words(ConstWords w) {
  constexpr int kWords = sizeof(T) / 4;
  struct Raw { uint32_t u[kWords]; } raw;
#pragma unroll
  for (int i = 0; i < kWords; ++i) raw.u[i] = w[i];
  return __builtin_bit_cast(T, raw);
}

__device__ __forceinline__ RowWork load_work(ConstWords entry, int wave) {
  constexpr int kAt = offsetof(ResRow, kind) / 4, kWaveAt = offsetof(ResRow, wave_in) / 4;
  struct Head { int32_t v[16]; };
  struct Work { Head head; int in, out, res, swizzle, res_step; };
  const ConstWords w = entry + kWaveAt + (wave >> 1);
  const int at = (wave & 1) * 16;
  const Work work = {load_words<Head>(entry + kAt), (int)(w[0] >> at & 0xffffu), (int)(w[kResRowWaves / 2] >> at & 0xffffu),
                     (int)(w[kResRowWaves] >> at & 0xffffu), (int)entry[offsetof(ResRow, swizzle) / 4],
                     (int)entry[offsetof(ResRow, res_step) / 4]};
  return __builtin_bit_cast(RowWork, work);
}

// One work item of a row layer: M vertically neighbouring tiles of 16 pixels x one tile of 16 filters of a 3 x 3
// convolution padded by 1, stride S, CPT 8-channel chunks per tap.
//
// A tile is 16 pixels of one row, or, in images 8 wide, 8 pixels of row t and 8 of row t + P / 2, so that the
// tap one row down of tile t is the centre tap of tile t + 1: what is read from LDS for one row is
// multiplied for all tiles that have a tap there, and at stride 1 an item reads M + 2 rows where tile by tile it
// would read 3 M.  The 3 * CPT chunks of a row of taps are FULL steps of four chunks and REM chunks over;
// those of two or three rows of taps share a step where they fit one (REM 2 and 1).  Lanes with nothing left
// multiply the zero chunks that pad the weights (there is one: 9 * CPT is no multiple of 4 then) with zeros, or with a
// pixel of the same window, so that an infinite pixel stays in the windows that see it: the left halo where REM is 1 or 3; where
// it is 2, the second row of taps, read with the third one (stride 1), or zeros in the place of the row below (stride 2).
// (Zeros everywhere: ResNet-56, 128 images 81.2 -> 81.6 us.)
// The filters of an item stay in registers.
//
// A layer is some 50 MFMAs per wave, so instructions in front of them count: what depends on the wave comes
// from the host, and no division or multiplication of lane numbers is left but the quick 24-bit one.
template <bool BF, int S, int CPT, int M, bool RES>
__device__ __forceinline__ void rows_item(const RowWork& L, char* act, int lane, const uint4& one_hot) {
  constexpr int T = 3 * CPT, FULL = T / 4, REM = T % 4, C0 = 4 * FULL;
  constexpr int EXTRA = REM == 0 ? 0 : REM == 3 ? 3 : REM == 2 ? 2 : 1;
  constexpr int NB = FULL + (REM ? 1 : 0), ROWS = S * (M - 1) + 3;
  constexpr int AHEAD = NB <= 4 ? 2 : 1;   // rows read ahead of the one that is multiplied
  const int li = lane & 15, g = lane >> 4;
  const int ft = L.in >> 14;
  const bool halves = (L.kind & kResRowHalves) != 0;
  const int col = halves ? li & 7 : li;
  const bool second = halves && li >= 8;
  const int row = L.tap_row, ps = L.tap_col;

  // pixels: byte offsets of this lane's chunk of every step, for the first row.  Chunk c of tap s lies at
  // s * ps + (c * 16 ^ flip[s]); a step's four chunks are of one tap, or from lane group `up` on of the next.
  const int first = L.in_org + (L.in & 0x3fff) * 16;
  const int lp = __mul24(col, S * ps) + (second ? L.half_in : 0) + first;
  constexpr bool FLIP = M != 8;   // (items of 8 tiles are for tensors whose chunks lie in order)
  int flip[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) flip[s] = FLIP ? swizzle_of(S * col + s, L.swizzle) : 0;
  int at[NB];
#pragma unroll
  for (int q = 0; q < FULL; ++q) {
    const int tap = 4 * q / CPT, up = (tap + 1) * CPT - 4 * q, c = 4 * q - tap * CPT;
    int chunk = (g + c) * 16, f = flip[tap], to = tap * ps;
    if (up < 4 && g >= up) {
      chunk -= CPT * 16;
      f = flip[tap < 2 ? tap + 1 : 2];
      to += ps;
    }
    at[q] = lp + to + (chunk ^ f);
  }
  int last_at = 0;   // REM 2: the last row's step, whose second half is not needed
  if constexpr (CPT == 1) {
    at[0] = g == 3 ? L.in_org : lp + __mul24(g, ps) + (g == 0 ? flip[0] : g == 1 ? flip[1] : flip[2]);
  } else if constexpr (REM > 0) {
    // (the chunks over are the last ones of the third tap)
    const int chunk = (C0 - 2 * CPT + (REM == 3 ? g : REM == 2 ? (g & 1) : 0)) * 16;
    last_at = lp + 2 * ps + (chunk ^ flip[2]);
    at[FULL] = last_at + (REM == 2 ? (g >= 2 ? row : 0) : REM == 1 ? (g >= 2 ? 2 * row : g == 1 ? row : 0) : 0);
    if (REM != 2 && g == 3) at[FULL] = L.in_org;
  }
  uint4 b[AHEAD + 1][NB];
  auto read_row = [&](int i, uint4* bv) {
#pragma unroll
    for (int q = 0; q < FULL; ++q) bv[q] = *reinterpret_cast<const uint4*>(act + at[q] + i * row);
    if constexpr (REM == 1) {
      if (i % S == 0 && i < S * M) bv[FULL] = *reinterpret_cast<const uint4*>(act + at[FULL] + i * row);
    } else if constexpr (REM == 2) {
      if (S == 1 ? i < ROWS - 1 : i % S == 0) bv[FULL] = *reinterpret_cast<const uint4*>(act + (i == ROWS - 1 ? last_at : at[FULL]) + i * row);
    } else if constexpr (REM == 3) {
      bv[FULL] = *reinterpret_cast<const uint4*>(act + at[FULL] + i * row);
    }
  };

  // filters: chunk j of filter f lies at j * Kp * 16 + f * 16
  const int kp16 = L.kp16;
  const int aft = li * 16 + (L.wts_off + ft * 256);
  uint4 a[3][FULL > 0 ? FULL : 1], ax[EXTRA > 0 ? EXTRA : 1];
  auto chunk = [&](int j) { return *reinterpret_cast<const uint4*>(act + aft + __mul24(j, kp16)); };
  const int ag = aft + __mul24(g, kp16);
  auto filters_of_row = [&](int r) {
#pragma unroll
    for (int q = 0; q < FULL; ++q) a[r][q] = *reinterpret_cast<const uint4*>(act + ag + (r * T + 4 * q) * kp16);
  };

  auto extra_filters = [&](int r) {
    if constexpr (REM == 3) {
      ax[r] = chunk(g < 3 ? r * T + C0 + g : 9 * CPT);
    } else if constexpr (REM == 2) {
      if (r == 0) ax[0] = chunk(g < 2 ? C0 + g : T + C0 + g - 2);
      if (r == 2 && S == 1) ax[1] = chunk(g < 2 ? 9 * CPT + g : 2 * T + C0 + g - 2);
      if (r == 2 && S == 2) ax[1] = chunk(g < 2 ? 2 * T + C0 + g : 9 * CPT + g - 2);
    } else if constexpr (REM == 1) {
      if (r == 0) ax[0] = chunk(g < 3 ? g * T + C0 : 9 * CPT);
    }
  };
  // (channels the shortcut does not have: any of its chunks, times zero)
  uint4 ia;
  int from = 0;
  if constexpr (RES) {
    const int chunk = min(ft * 2 + (g & 1), (L.res_cs >> 3) - 1) * 16;
    from = __mul24(col, L.res_col) + (second ? L.half_res : 0) + (FLIP ? chunk ^ swizzle_of(__mul24(col, L.res_step) + 1, L.swizzle >> 8) : chunk) +
           (L.res_org + L.res * 16);
    ia = one_hot;
    if (ft * 16 + 16 > L.res_cs && ft * 16 + li >= L.res_cs) ia = uint4{0u, 0u, 0u, 0u};
  }
  uint4 rb[RES ? M : 1];

  read_row(0, b[0]);
  filters_of_row(0);
#pragma unroll
  for (int r = 0; r < 3; ++r) extra_filters(r);
  const f32x4 bias = *reinterpret_cast<const f32x4*>(act + g * 16 + (L.wts_off - 256 + ft * 64));
  if constexpr (RES) {
#pragma unroll
    for (int t = 0; t < M; ++t) rb[t] = *reinterpret_cast<const uint4*>(act + from + t * L.res_row);
  }
  filters_of_row(1);
  if constexpr (AHEAD == 2) read_row(1, b[1]);
  filters_of_row(2);
  __builtin_amdgcn_sched_barrier(0);   // (left alone, every read is moved to just before its MFMA)
  f32x4 acc[M];
#pragma unroll
  for (int t = 0; t < M; ++t) {
    if constexpr (RES) acc[t] = mfma_16x16x32<BF>(ia, rb[t], bias);
    else acc[t] = bias;
  }

  uint4 above = {};   // REM 2 at stride 1: what the row before read of the chunks over
  const uint32_t floor2 = (L.kind & kResRowRelu) ? 0u : 0x80008000u;
  const int out = __mul24(col, L.out_col) + (second ? L.half_out : 0) + ((g & 1) ? L.out_row : 0) +
                  ((ft * 32 + (g >> 1) * 16) ^ (FLIP ? swizzle_of(col + 1, L.swizzle >> 4) : 0)) + (L.out_org + L.out * 16);
  // tiles t and t + 1 are complete: rounding, ReLU, and the row exchange of conv_items
  auto store = [&](int t) {
    const uint32_t p0 = clamp_below(pack2<BF>(acc[t][0], acc[t][1]), floor2);
    const uint32_t p1 = clamp_below(pack2<BF>(acc[t][2], acc[t][3]), floor2);
    const uint32_t q0 = clamp_below(pack2<BF>(acc[t + 1][0], acc[t + 1][1]), floor2);
    const uint32_t q1 = clamp_below(pack2<BF>(acc[t + 1][2], acc[t + 1][3]), floor2);
    const auto r0 = __builtin_amdgcn_permlane16_swap(p0, q0, false, false);
    const auto r1 = __builtin_amdgcn_permlane16_swap(p1, q1, false, false);
    *reinterpret_cast<uint4*>(act + out + t * L.out_row) = uint4{r0[0], r1[0], r0[1], r1[1]};
  };
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const uint4* bv = b[i % (AHEAD + 1)];
    // the tile that has its row r of taps here
    auto tile = [&](int r) { return i - r >= 0 && (i - r) % S == 0 && (i - r) / S < M ? (i - r) / S : -1; };
    if (i + AHEAD < ROWS) read_row(i + AHEAD, b[(i + AHEAD) % (AHEAD + 1)]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < FULL; ++q) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
        if (tile(r) >= 0) acc[tile(r)] = mfma_16x16x32<BF>(a[r][q], bv[q], acc[tile(r)]);
    }
    if constexpr (REM == 3) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
        if (tile(r) >= 0) acc[tile(r)] = mfma_16x16x32<BF>(ax[r], bv[FULL], acc[tile(r)]);
    } else if constexpr (REM == 2) {
      if (tile(0) >= 0) acc[tile(0)] = mfma_16x16x32<BF>(ax[0], bv[FULL], acc[tile(0)]);
      if constexpr (S == 1) {
        if (tile(2) >= 0) acc[tile(2)] = mfma_16x16x32<BF>(ax[1], above, acc[tile(2)]);
        above = bv[FULL];
      } else if (tile(2) >= 0) {
        const uint4 &v = bv[FULL], own = {g < 2 ? v.x : 0u, g < 2 ? v.y : 0u, g < 2 ? v.z : 0u, g < 2 ? v.w : 0u};
        acc[tile(2)] = mfma_16x16x32<BF>(ax[1], own, acc[tile(2)]);
      }
    } else if constexpr (REM == 1) {
      if (tile(0) >= 0) acc[tile(0)] = mfma_16x16x32<BF>(ax[0], bv[FULL], acc[tile(0)]);
    }
    // (a row later than they are complete, under this row's MFMAs)
    if (i >= S + 3 && (i - S - 3) % (2 * S) == 0) store((i - S - 3) / S);
    __builtin_amdgcn_sched_barrier(0);
  }
  store(M - 2);
  // (or the last stores of all sizes become one, with an address for each: more instructions, and the compiler has lost
  // such an address elsewhere - add_up in conv_window.hip)
  asm volatile("; rows %0 %1 %2 %3" ::"n"(S), "n"(CPT), "n"(M), "n"(RES));
}

template <bool BF, int S, int CPT, int M>
__device__ __forceinline__ void rows_case(const RowWork& L, char* act, int lane, const uint4& one_hot) {
  if (S == 1 && L.res_org >= 0 && (L.in >> 14) * 16 < L.res_cs) rows_item<BF, S, CPT, M, S == 1>(L, act, lane, one_hot);
  else rows_item<BF, S, CPT, M, false>(L, act, lane, one_hot);
}

template <bool BF>
__device__ __forceinline__ void rows_layer(const RowWork& L, char* act, int lane, const uint4& one_hot) {
#define FUPR_ROWS(S, CPT, M) case row_kind(S, CPT, M): rows_case<BF, S, CPT, M>(L, act, lane, one_hot); break;
  switch (L.kind & 255) {
    FUPR_ROWS(1, 1, 2) FUPR_ROWS(1, 2, 2) FUPR_ROWS(1, 3, 2) FUPR_ROWS(1, 4, 2)
    FUPR_ROWS(1, 5, 2) FUPR_ROWS(1, 6, 2) FUPR_ROWS(1, 7, 2) FUPR_ROWS(1, 8, 2)
    FUPR_ROWS(1, 1, 4) FUPR_ROWS(1, 2, 4) FUPR_ROWS(1, 3, 4) FUPR_ROWS(1, 4, 4) FUPR_ROWS(1, 1, 8) FUPR_ROWS(1, 2, 8)
    FUPR_ROWS(2, 1, 2) FUPR_ROWS(2, 2, 2) FUPR_ROWS(2, 3, 2) FUPR_ROWS(2, 4, 2) FUPR_ROWS(2, 1, 4) FUPR_ROWS(2, 2, 4)
  }
#undef FUPR_ROWS
}

// Global mean over the M interior pixels of the input, per channel, in fp32 (one barrier inside):
// L.MT partial sums over interleaved pixels, then their sum in order.
template <bool BF>
__device__ __forceinline__ void mean_layer(const ResLayer& L, const ResParams& p, char* lds,
                                           char* act, int n, int tid) {
  float* part = reinterpret_cast<float*>(lds);   // parts x cs_out floats of scratch
  const int cs = L.cs_out, M = L.M, Q = L.Q, parts = L.MT;
  if (tid < parts * cs) {
    const int c = tid % cs, k = tid / cs;
    float acc = 0.f;
    for (int i = k; i < M; i += parts) {
      const int pp = div_magic(i, L.magicQ), qq = i - pp * Q;
      acc += to_float<BF>(*reinterpret_cast<const uint16_t*>(act + L.in_org + pp * L.in_row +
                                                             qq * L.in_col + c * 2));
    }
    part[k * cs + c] = acc;
  }
  __syncthreads();
  if (tid < cs) {
    float acc = 0.f;
    for (int k = 0; k < parts; ++k) acc += part[k * cs + tid];
    const uint16_t o = from_float<BF>(acc / (float)M);
    if (L.flags & kResLast) reinterpret_cast<uint16_t*>(p.y)[(size_t)n * p.y_cs + tid] = o;
    else *reinterpret_cast<uint16_t*>(act + L.out_org + tid * 2) = o;
  }
}

// The first eight dwords of a ResLayer: all that staging needs.
struct StageHead {
  const void* packed;
  const void* table;
  int32_t blob_units, tab_units, w_off, tab_off;
};
static_assert(sizeof(StageHead) == 32, "StageHead mirrors the head of ResLayer");

// One wave-wide global -> LDS load: lane i moves 16 bytes from its own global
// address to the i-th 16-byte slot after lds_base (M0 holds the base).  Written
// as inline assembly so that the compiler does not take it for an LDS store
// that later LDS reads might alias (it would wait for the whole transfer before
// the current layer's first LDS access); the kernel orders it by hand: issued
// after the barrier that retires the destination's previous contents, awaited
// (vmcnt) before the barrier that publishes it.
__device__ __forceinline__ void load_to_lds(const void* src_base, uint32_t lane_offset,
                                            uint32_t lds_base) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2"
      :
      : "s"(lds_base), "v"(lane_offset), "s"(src_base)
      : "memory", "m0");
}

__device__ __forceinline__ uint32_t lds_address(const char* p) {
  return (uint32_t)(uintptr_t)(LdsPtr)p;
}

// A layer's parameter blob and tap table go from global memory straight into
// LDS, issued before the current layer is computed and awaited after it: no
// register is held and no global-memory latency sits on the layer chain.  `me` of
// `stagers` waves do it; the last of them takes the table.
__device__ __forceinline__ void stage_params(const StageHead& H, int me, int stagers, char* act, int lane) {
  if (me < 0) return;
  const char* src = reinterpret_cast<const char*>(H.packed);
  const uint32_t dst = lds_address(act + H.w_off);
  const uint32_t lane_offset = lane * 16;
  // (whole loads four at a time and without a look at the lanes; then the rest)
  const int whole = H.blob_units & ~63, step = stagers * 64;
  int u = me * 64;
  for (; u + 3 * step < whole; u += 4 * step)
#pragma unroll
    for (int k = 0; k < 4; ++k) load_to_lds(src + (size_t)(u + k * step) * 16, lane_offset, dst + (u + k * step) * 16);
  for (; u < whole; u += step) load_to_lds(src + (size_t)u * 16, lane_offset, dst + u * 16);
  if (u == whole && u + lane < H.blob_units) load_to_lds(src + (size_t)u * 16, lane_offset, dst + u * 16);
  // the table (at most 64 slots) goes through the last wave, which has the
  // smallest share of the blob
  if (me == stagers - 1 && lane < H.tab_units)
    load_to_lds(H.table, lane_offset, lds_address(act + H.tab_off));
}

__device__ __forceinline__ void staging_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Asks for the layer table's 64-byte lines, so that each layer's descriptor is found in the scalar cache (16 KB,
// cold when a kernel starts: a line from L2 took 700 clocks of every layer).  `me` of `waves` waves, eight
// lines at a time; lines past the end repeat the last one.
__device__ __forceinline__ void touch_table(const void* table, int bytes, int me, int waves) {
  const int last = (min(bytes, 15 * 1024) - 4) >> 6;
  for (int at = me * 8; at <= last; at += waves * 8) {
    const uint64_t base = reinterpret_cast<uint64_t>(table);
    uint64_t line[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) line[i] = base + (uint64_t)(min(at + i, last) * 64);
    int sink;
    // (the loads have landed before the compiler can give the register to anything else)
    asm volatile(
        "s_load_dword %0, %1, 0\n\ts_load_dword %0, %2, 0\n\ts_load_dword %0, %3, 0\n\ts_load_dword %0, %4, 0\n\t"
        "s_load_dword %0, %5, 0\n\ts_load_dword %0, %6, 0\n\ts_load_dword %0, %7, 0\n\ts_load_dword %0, %8, 0\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&s"(sink)
        : "s"(line[0]), "s"(line[1]), "s"(line[2]), "s"(line[3]), "s"(line[4]), "s"(line[5]), "s"(line[6]),
          "s"(line[7]));
  }
}

// Before the first layer: its parameters, the image into the interior of its LDS tensor, zeros around it.
template <int THREADS, bool ROWS>
__device__ __forceinline__ void start(const ResParams& p, ConstWords table, char* act, int n, int tid, int lane, int wave) {
  stage_params(load_words<StageHead>(table), wave, THREADS / 64, act, lane);
  const int cpp = p.in_cs >> 3;
  const uint4* src = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(p.x) +
                                                    (size_t)n * p.in_H * p.in_W * p.in_cs);
  const int total = p.in_H * p.in_W * cpp;
  for (int i = tid; i < total; i += THREADS) {
    const int pix = i / cpp, ch = i - pix * cpp;
    const int row = pix / p.in_W, col = pix - row * p.in_W;
    const int flip = ROWS ? swizzle_of(col + 1, row_swizzle_shift(p.in_ps2) | row_swizzle_mask(p.in_ps2) << 2) : 0;
    *reinterpret_cast<uint4*>(act + p.in_org + (row * p.in_Wh + col) * p.in_ps2 + (ch * 16 ^ flip)) = src[i];
  }
  if (p.hp > 0 && p.in_H * p.in_W > 1)
    zero_halo<THREADS>(act, p.in_org, p.in_H, p.in_W, p.in_Wh, p.in_ps2, ROWS ? p.in_ps2 >> 4 : cpp, p.hp, tid);
}

constexpr int kLayerWords = sizeof(ResLayer) / 4;

template <bool BF>
__global__ __launch_bounds__(kResThreads) void resident_kernel(const ResParams p) {
  extern __shared__ uint4 lds4[];
  char* lds = reinterpret_cast<char*>(lds4);
  char* act = lds + kResScratchBytes;
  constexpr int WAVES = kResThreads / 64;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = blockIdx.x;
  ConstWords table = (ConstWords)(uintptr_t)p.layers;

  start<kResThreads, false>(p, table, act, n, tid, lane, wave);
  ResLayer L = load_words<ResLayer>(table);
  staging_done();
  __syncthreads();

  const int n_layers = p.n_layers;
  PixelCache pc;
  for (int l = 0; l < n_layers; ++l) {
    const bool has_next = l + 1 < n_layers;
    if (has_next) {
      // the waves that have no work item in the current layer (or all, when every one has) stage the next one's parameters
      const StageHead Hn = {L.next_packed, L.next_table, L.next_blob_units,
                            L.next_tab_units, L.next_w_off, L.next_tab_off};
      const int busy = (L.flags & kResMean) || L.n_items >= WAVES ? 0 : L.n_items;
      stage_params(Hn, wave - busy, WAVES - busy, act, lane);
    }

    if (L.flags & kResZeroHalo)
      zero_halo<kResThreads>(act, L.hz_org, L.hz_P, L.hz_Q, L.hz_Wh, L.hz_ps2, L.hz_chunks, L.hz_hp, tid);
    if (L.flags & kResMean) {
      mean_layer<BF>(L, p, lds, act, n, tid);
    } else {
      switch (L.MT * 8 + L.NT) {
        case 1 * 8 + 1: conv_layer<BF, WAVES, 1, 1>(L, p, act, n, lane, wave, pc); break;
        case 1 * 8 + 2: conv_layer<BF, WAVES, 1, 2>(L, p, act, n, lane, wave, pc); break;
        case 2 * 8 + 1: conv_layer<BF, WAVES, 2, 1>(L, p, act, n, lane, wave, pc); break;
        case 2 * 8 + 2: conv_layer<BF, WAVES, 2, 2>(L, p, act, n, lane, wave, pc); break;
        default: conv_layer<BF, WAVES, 4, 1>(L, p, act, n, lane, wave, pc); break;
      }
    }
    if (has_next) L = load_words<ResLayer>(table + (l + 1) * kLayerWords);   // in flight across the barrier
    staging_done();
    __syncthreads();   // this layer's output and the next layer's parameters are visible
  }
}

// The mean behind the row layers (one barrier inside): each wave sums every eighth row of the image, a lane two
// channels; then the first wave adds the waves' sums up in order.  Little code, since all of it is run once and
// comes from a cold instruction cache: unrolled over pixels and channels it took 5500 clocks.
template <bool BF, int WAVES>
__device__ __forceinline__ void mean_rows(const ResLayer& L, char* scratch, char* act, int lane, int wave) {
  float2* part = reinterpret_cast<float2*>(scratch);   // WAVES x cs_out floats
  const int swizzle = row_swizzle_shift(L.in_col) | row_swizzle_mask(L.in_col) << 2, pairs = L.cs_out >> 1;
  if (lane < pairs) {
    float2 sum = {0.f, 0.f};
    for (int row = wave; row * L.Q < L.M; row += WAVES) {
      const char* at = act + L.in_org + row * L.in_row + (lane & 3) * 4;
#pragma unroll 8
      for (int x = 0; x < L.Q; ++x) {
        const uint32_t v = *reinterpret_cast<const uint32_t*>(at + x * L.in_col + ((lane >> 2) * 16 ^ swizzle_of(x + 1, swizzle)));
        sum.x += to_float<BF>((uint16_t)v);
        sum.y += to_float<BF>((uint16_t)(v >> 16));
      }
    }
    part[wave * pairs + lane] = sum;
  }
  __syncthreads();
  if (wave == 0 && lane < pairs) {
    float2 sum = {0.f, 0.f};
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
      const float2 v = part[k * pairs + lane];
      sum.x += v.x;
      sum.y += v.y;
    }
    *reinterpret_cast<uint32_t*>(act + L.out_org + lane * 4) = pack2<BF>(sum.x / (float)L.M, sum.y / (float)L.M);
  }
}

// The parts of a ResRow that the waves which stage and those which compute load ahead of a layer.
struct RowStage {
  const void* next_packed;
  const void* next_table;
  int32_t next_blob_units, next_tab_units, next_w_off, next_tab_off;
  int32_t flags, hz_org, hz_P, hz_Q, hz_Wh, hz_ps2, hz_chunks, hz_hp;
};
static_assert(sizeof(RowStage) == 64 && offsetof(RowStage, hz_hp) == offsetof(ResRow, hz_hp), "the head of ResRow");
constexpr int kRowWords = sizeof(ResRow) / 4;

// Networks of row layers (the CIFAR networks of Table II, and others like them).
//
// Measured against the kernel above, which runs every network: ResNet-20, one image, 53.3 -> 33.2 us; ResNet-56, 128
// images, 128 -> 81 us.  There a layer took 5500 clocks for 1300 of MFMAs: a third in front of the first MFMA (the
// layer's descriptor from a cold scalar cache, address arithmetic, the parameters' issue by waves that also
// compute) and, tile by tile, LDS reads that were waited for one at a time.  Here it takes 3400.
// What bounds it: the chain of a layer on two waves per SIMD - descriptor and addresses 700 clocks, LDS reads and MFMAs
// 2000 (of all clocks LDS is busy in 39 %, the matrix pipe in 32 %), last store, barrier 500.  Without any work in the
// layers ResNet-56 takes 21 us, with the parameters' staging 41 (an L2 latency per layer, hidden here).  Tried and not
// kept: filters read row by row in front of their MFMAs instead of at once, the shortcut added last (2 % slower
// together); the next layer's descriptor asked for ahead of the layer (1 % slower: every LDS wait then waits for it
// too); wave priorities (equal).
//
// Eight waves compute, two per SIMD with the registers for tall items; four stage the
// next layer's parameters and zero halos meanwhile.  Both kinds meet at the same barriers: one before the first layer,
// one after each, one inside the mean.
template <bool BF>
__global__ __launch_bounds__(kResRowThreads) void resident_rows_kernel(const ResParams p) {
  extern __shared__ uint4 lds4[];
  char* act = reinterpret_cast<char*>(lds4) + kResScratchBytes;
  constexpr int WAVES = kResRowWaves, STAGERS = kResRowThreads / 64 - WAVES;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = blockIdx.x;
  ConstWords table = (ConstWords)(uintptr_t)p.rows;
  const int n_layers = p.n_layers;

  start<kResRowThreads, true>(p, (ConstWords)(uintptr_t)p.layers, act, n, tid, lane, wave);
  touch_table(p.rows, n_layers * (int)sizeof(ResRow), wave, kResRowThreads / 64);
  if (n_layers >= 2) touch_table(p.layers + (n_layers - 2), 2 * (int)sizeof(ResLayer), wave, kResRowThreads / 64);
  staging_done();

  if (wave >= WAVES) {
    RowStage S = load_words<RowStage>(table);
    __syncthreads();
    for (int l = 0; l < n_layers; ++l) {
      if (l + 1 < n_layers)
        stage_params(StageHead{S.next_packed, S.next_table, S.next_blob_units, S.next_tab_units, S.next_w_off, S.next_tab_off},
                     wave - WAVES, STAGERS, act, lane);
      if (S.flags & kResZeroHalo)
        zero_halo<STAGERS * 64>(act, S.hz_org, S.hz_P, S.hz_Q, S.hz_Wh, S.hz_ps2, S.hz_chunks, S.hz_hp, tid - WAVES * 64);
      if (S.flags & kResMean) __syncthreads();
      if (l + 1 < n_layers) S = load_words<RowStage>(table + (l + 1) * kRowWords);
      staging_done();
      __syncthreads();
    }
    return;
  }

  const uint4 one_hot = identity_fragment<BF>(0, 16, lane & 15, lane >> 4);
  int l = 0;
  RowWork R = load_work(table, wave);
  __syncthreads();
  for (; l < n_layers && R.kind != kResTail; ++l) {
    int ln = lane;
    asm volatile("" : "+v"(ln));   // (else what depends on the lane is worked out for all sizes in front of the loop, and spilled)
    if (R.in != kResNoItem) rows_layer<BF>(R, act, ln, one_hot);
    // (any earlier, and a wave's first wait for LDS would wait for this too)
    if (l + 1 < n_layers) R = load_work(table + (l + 1) * kRowWords, wave);
    __syncthreads();
  }
  PixelCache pc;
  for (; l < n_layers; ++l) {
    const ResLayer L = load_words<ResLayer>((ConstWords)(uintptr_t)p.layers + l * kLayerWords);
    if (L.flags & kResMean) mean_rows<BF, WAVES>(L, reinterpret_cast<char*>(lds4), act, lane, wave);
    else if (L.MT * 8 + L.NT == 1 * 8 + 2) conv_layer<BF, WAVES, 1, 2>(L, p, act, n, lane, wave, pc);
    else conv_layer<BF, WAVES, 1, 1>(L, p, act, n, lane, wave, pc);
    __syncthreads();
  }
}

std::once_flag g_attr_once;
hipError_t g_attr_status = hipSuccess;

}  // namespace

fupr_status launch_resident(const ResParams& p, int N, fupr_dtype dt, void* stream) {
  std::call_once(g_attr_once, [] {
    for (const void* kernel : {reinterpret_cast<const void*>(&resident_kernel<true>),
                               reinterpret_cast<const void*>(&resident_kernel<false>),
                               reinterpret_cast<const void*>(&resident_rows_kernel<true>),
                               reinterpret_cast<const void*>(&resident_rows_kernel<false>)}) {
      const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLdsLimit);
      if (e != hipSuccess) g_attr_status = e;
    }
  });
  if (g_attr_status != hipSuccess) return FUPR_ERR_LAUNCH;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  const dim3 grid(N), threads(p.rows ? kResRowThreads : kResThreads);
  const bool bf = dt == FUPR_BF16;
  if (p.rows) {
    if (bf) hipLaunchKernelGGL(resident_rows_kernel<true>, grid, threads, p.lds_bytes, hs, p);
    else hipLaunchKernelGGL(resident_rows_kernel<false>, grid, threads, p.lds_bytes, hs, p);
  } else {
    if (bf) hipLaunchKernelGGL(resident_kernel<true>, grid, threads, p.lds_bytes, hs, p);
    else hipLaunchKernelGGL(resident_kernel<false>, grid, threads, p.lds_bytes, hs, p);
  }
  return launch_status("resident_kernel");
}

}  // namespace fupr
