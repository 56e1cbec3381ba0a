// The ImageNet stem of Table II in one kernel: 7 x 7 stride-2 convolution of a
// 3-channel image (bias and ReLU in the epilogue, Sec. VI-B-3) followed by the
// 3 x 3 stride-2 max-pool.  The convolution's output, the largest tensor of
// the network, never leaves the registers.
//
// GEMM view: rows = 64 filters (MFMA operand A), columns = 16 convolution pixels
// of one row (operand B).  The reduction index is (r, column pair j, 2 pixels x 4
// channels): with 4 channels per pixel (the fourth has zero weights) the 8 values
// one lane feeds an MFMA with are two neighbouring input pixels, so the 7 x 7 x 3 =
// 147 products per output take 7 MFMA 16x16x32 steps (7 rows x 4 pairs x 8 = 224,
// tap s = 7 and channel 3 have zero weights) instead of the 13 steps of one
// 8-channel chunk per tap.  The filter fragments are rebuilt from the packed blob
// once per workgroup and stay in registers.
//
// Every wave walks down a strip of 7 pool columns (15 convolution columns) by itself.
// An input row is one fragment, which the 3 - 4 convolution rows that need it share: a
// convolution row loads two rows (straight from memory, two convolution rows ahead) and
// multiplies by seven.  The maximum over three rows is taken in registers as the rows
// come, over three columns between neighbouring lanes.  So no LDS, no barrier and no
// second pass stands between the input and the maxima.  Measured, before (input patch and
// convolution tile in LDS, three phases between barriers) -> now, images of 224 x 224: one
// 6.9 -> 4.7 us, 12 12.6 -> 9.7, 64 40.3 -> 26.1, 256 141 -> 88.  At 256 images the input and
// the result, 308 MB, pass at 3.5 TB/s (a large copy: 4.8), and the matrix pipe is busy for 43 us
// (28 MFMAs of 16 clocks per convolution row of a strip); one image is latency.
//
// Max-pool over ReLU outputs: positions outside the convolution's output count
// as 0, which never wins against the window's centre tap (>= 0, always inside).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device_utils.h"
#include "fupr.h"
#include "layout.h"
#include "stem_pool.h"

namespace fupr {
namespace {

constexpr uint32_t kOutside = 0x80000000u;
constexpr int kCols = 7;     // pool columns of a strip: 15 of a fragment's 16 convolution pixels
constexpr int kRing = 12;    // input rows in registers: 7 of this convolution row, 5 on their way
constexpr int kWaves = 4;

struct StemParams {
  const uint16_t* x;
  const uint16_t* w;     // [49 (+3)][64][8]
  const float* bias;
  uint16_t* y;
  uint32_t x_bytes, w_bytes;
  int H, W, xcs;         // input
  int SH, SW;            // convolution output
  int P, Q, ycs;         // pool output
  int TP;                // pool rows of a strip
  int strips_q;          // strips side by side
  int total, per_xcd;    // strips; workgroups per XCD
  FastDiv div_image, div_q;   // by strips per image, strips_q
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short short2_t __attribute__((ext_vector_type(2)));

// non-negative values of either 16-bit format order like their bit patterns
__device__ __forceinline__ uint32_t max2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(short2_t, a),
                                                                __builtin_bit_cast(short2_t, b)));
}

// the value n lanes to the right (row_shl) or left (row_shr) in the same 16 lanes; 0 past the end
template <int CONTROL>
__device__ __forceinline__ uint32_t neighbour(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CONTROL, 0xf, 0xf, true);
}
constexpr int kRight1 = 0x101, kRight2 = 0x102, kLeft1 = 0x111;

template <bool BF>
__global__ __launch_bounds__(kWaves * 64, 2) void stem_pool_kernel(const StemParams p) {
  __shared__ uint4 staged[28 * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;

  const __amdgpu_buffer_rsrc_t xrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.x), 0, p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.w), 0, p.w_bytes, 0x00020000);

  // Workgroup b runs on XCD b % 8: each XCD takes a contiguous eighth of the strips, so that the
  // input that neighbouring strips share is read into its L2 once.
  const int strip = ((blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3)) * kWaves + wave;
  const bool live = strip < p.total;
  const int n = div_by(live ? strip : 0, p.div_image);
  const int rows_q = (p.P + p.TP - 1) / p.TP;
  const int rem = (live ? strip : 0) - n * rows_q * p.strips_q;
  const int tp = div_by(rem, p.div_q), tq = rem - tp * p.strips_q;
  const int p0 = tp * p.TP, p1 = min(p0 + p.TP, p.P);    // pool rows p0 .. p1 - 1
  const int q0 = tq * kCols;
  const int sw = 2 * q0 - 1 + li;                        // this lane's convolution column
  const int sh0 = 2 * p0 - 1;                            // the strip's first convolution row
  const int last = live ? 2 * (p1 - p0) : -1;            // its last one, counted from sh0

  // a lane's two pixels of an input row
  const int iw = 2 * sw - 3 + 2 * g;
  const bool in0 = (unsigned)iw < (unsigned)p.W, in1 = (unsigned)(iw + 1) < (unsigned)p.W;
  const uint32_t pix = (uint32_t)p.xcs * 2u, col = (uint32_t)iw * pix;
  const int ih0 = 2 * sh0 - 3;
  u32x2 b[kRing][2];
  auto load_row = [&](int r, u32x2* dst) {               // input row ih0 + r
    const int ih = ih0 + r;
    const bool ok = (unsigned)ih < (unsigned)p.H && r <= 2 * last + 6;
    const uint32_t off = (uint32_t)((n * p.H + ih) * p.W) * pix + col;
    dst[0] = __builtin_amdgcn_raw_buffer_load_b64(xrsrc, ok && in0 ? off : kOutside, 0, 0);
    dst[1] = __builtin_amdgcn_raw_buffer_load_b64(xrsrc, ok && in1 ? off + pix : kOutside, 0, 0);
  };
#pragma unroll
  for (int r = 0; r < 10; ++r) load_row(r, b[r]);

  // ---- filters: [r * 4 + j][filter][2 taps x 4 channels] in LDS, then registers -----
#pragma unroll
  for (int i = 0; i < 28 * 64 / (kWaves * 64); ++i) {
    const int e = tid + i * kWaves * 64;
    const int ch = e >> 6, f = e & 63;
    const int r = ch >> 2, j = ch & 3;
    const int tap = r * 7 + 2 * j;
    const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(wrsrc, (uint32_t)(tap * 64 + f) * 16u, 0, 0);
    const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(
        wrsrc, 2 * j + 1 < 7 ? (uint32_t)((tap + 1) * 64 + f) * 16u : kOutside, 0, 0);
    staged[e] = uint4{lo[0], lo[1], hi[0], hi[1]};
  }
  f32x4 bias4[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) bias4[t] = *reinterpret_cast<const f32x4*>(p.bias + t * 16 + g * 4);
  __syncthreads();
  uint4 a[7][4];
#pragma unroll
  for (int k = 0; k < 7; ++k)
#pragma unroll
    for (int t = 0; t < 4; ++t) a[k][t] = staged[((k * 4 + g) * 64) + t * 16 + li];

  // Where a pool row goes: after the exchanges below a lane holds 8 channels of pool column li / 2.
  const int odd = li & 1, gq = q0 + (li >> 1);
  uint16_t* const y_lane = p.y + (int64_t)n * p.P * p.Q * p.ycs + gq * p.ycs + ((g & 1) * 2 + odd) * 16 + (g >> 1) * 8;
  const bool stores = (li >> 1) < kCols && gq < p.Q;
  const uint32_t keep_col = (unsigned)sw < (unsigned)p.SW ? 0xffffffffu : 0u;

  uint32_t run[4][2];   // maxima of this pool row so far: [filter tile][channel pair]
#pragma unroll
  for (int t = 0; t < 4; ++t) run[t][0] = run[t][1] = 0u;
  // six convolution rows at a time, so that every register of the ring has a fixed place
  for (int i0 = 0; i0 <= last; i0 += 6) {
#pragma unroll
    for (int u = 0; u < 6; ++u) {
      const int i = i0 + u;                 // convolution row sh0 + i: input rows 2 i .. 2 i + 6
      if (i > last) break;
      load_row(2 * i + 10, b[(2 * u + 10) % kRing]);
      load_row(2 * i + 11, b[(2 * u + 11) % kRing]);
      f32x4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = bias4[t];
#pragma unroll
      for (int k = 0; k < 7; ++k) {
        const u32x2* bk = b[(2 * u + k) % kRing];
        const uint4 bv = {bk[0][0], bk[0][1], bk[1][0], bk[1][1]};
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma_16x16x32<BF>(a[k][t], bv, acc[t]);
      }
      const uint32_t keep = (unsigned)(sh0 + i) < (unsigned)p.SH ? keep_col : 0u;
      uint32_t v[4][2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        v[t][0] = pack2<BF>(fmaxf(acc[t][0], 0.f), fmaxf(acc[t][1], 0.f)) & keep;
        v[t][1] = pack2<BF>(fmaxf(acc[t][2], 0.f), fmaxf(acc[t][3], 0.f)) & keep;
      }
      // Rows 0, 2, 4, .. end a pool row and begin the next one (row 0 only begins).
      if (u % 2 == 0 && i > 0) {
        // columns 2 q, 2 q + 1, 2 q + 2 of pool column q: tiles 0 and 2 in the even lane of a
        // pair, tiles 1 and 3 in the odd one
        uint32_t o[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const uint32_t e = max2(run[2 * h][c], v[2 * h][c]), f = max2(run[2 * h + 1][c], v[2 * h + 1][c]);
            const uint32_t me = max2(max2(e, neighbour<kRight1>(e)), neighbour<kRight2>(e));
            const uint32_t mf = max2(max2(f, neighbour<kRight1>(f)), neighbour<kLeft1>(f));
            o[h][c] = odd ? mf : me;
          }
        // the exchange between 16-lane rows makes 8 consecutive channels of one tile
        const auto w0 = __builtin_amdgcn_permlane16_swap(o[0][0], o[1][0], false, false);
        const auto w1 = __builtin_amdgcn_permlane16_swap(o[0][1], o[1][1], false, false);
        const int gp = p0 + (i >> 1) - 1;
        if (stores)
          *reinterpret_cast<u32x4*>(y_lane + (int64_t)gp * p.Q * p.ycs) = u32x4{w0[0], w1[0], w0[1], w1[1]};
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) run[t][c] = u % 2 == 0 ? v[t][c] : max2(run[t][c], v[t][c]);
    }
  }
}

int stem_compute_units() {
  static int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0) {
      (void)hipGetLastError();
      return 256;
    }
    return n;
  }();
  return cus;
}

// Pool rows of a strip.  A strip computes one convolution row twice, so long strips are the
// cheapest; a batch that does not fill the GPU with them is cut finer.  The cost counts clocks:
// 448 of the matrix pipe per row, as much again in latency where a SIMD has one wave only, and
// the start of a wave.  The values do not depend on the cut: every convolution output is the same sum.
int stem_rows(int N, int P, int strips_q) {
  const int64_t simds = 4 * (int64_t)stem_compute_units();
  int best = 1;
  int64_t least = 0;
  for (int tp = 1; tp <= std::min(P, 32); ++tp) {
    const int64_t strips = (int64_t)N * ((P + tp - 1) / tp) * strips_q;
    const int64_t waves = (strips + simds - 1) / simds, rows = 2 * tp + 1;
    const int64_t cost = waves * (rows * 448 + 1500) + (waves == 1 ? rows * 448 : 0);
    if (least && cost >= least) continue;
    least = cost;
    best = tp;
  }
  return best;
}

bool plan_stem(const fupr_conv_shape& s, fupr_dtype dt, int N, int H, int W, int xcs, int ycs,
               int pool_k, int pool_stride, int pool_pad, StemParams* out) {
  if (dt != FUPR_BF16 && dt != FUPR_F16) return false;
  if (s.R != 7 || s.S != 7 || s.stride != 2 || s.pad != 3 || s.C > 4 || s.K != 64) return false;
  if (pool_k != 3 || pool_stride != 2 || pool_pad != 1) return false;
  if (xcs % 4 != 0 || ycs != 64) return false;
  StemParams p{};
  p.H = H; p.W = W; p.xcs = xcs;
  p.SH = out_extent(H, 7, 2, 3);
  p.SW = out_extent(W, 7, 2, 3);
  p.P = out_extent(p.SH, 3, 2, 1);
  p.Q = out_extent(p.SW, 3, 2, 1);
  p.ycs = ycs;
  p.strips_q = (p.Q + kCols - 1) / kCols;
  p.TP = stem_rows(N, p.P, p.strips_q);
  const int64_t per_image = (int64_t)((p.P + p.TP - 1) / p.TP) * p.strips_q;
  if ((int64_t)N * H * W * xcs * 2 >= (int64_t)kOutside) return false;
  const int64_t total = (int64_t)N * per_image;
  if (total >= (int64_t(1) << 30)) return false;
  p.total = (int)total;
  p.per_xcd = (int)((total + 8 * kWaves - 1) / (8 * kWaves));
  p.div_image = fast_div((int)per_image);
  p.div_q = fast_div(p.strips_q);
  *out = p;
  return true;
}

}  // namespace

bool stem_pool_applies(const fupr_conv_shape& s, fupr_dtype dt, int N, int H, int W, int xcs,
                       int ycs, int pool_k, int pool_stride, int pool_pad) {
  StemParams p;
  return plan_stem(s, dt, N, H, W, xcs, ycs, pool_k, pool_stride, pool_pad, &p);
}

fupr_status launch_stem_pool(const fupr_conv_shape& s, fupr_dtype dt, int N, int H, int W, int xcs,
                             int ycs, const void* x, const void* packed, void* y, void* stream) {
  StemParams p;
  if (!plan_stem(s, dt, N, H, W, xcs, ycs, 3, 2, 1, &p)) return FUPR_ERR_LIMIT;
  const PackedLayout L = packed_layout(s, dt);
  const char* blob = reinterpret_cast<const char*>(packed);
  p.x = reinterpret_cast<const uint16_t*>(x);
  p.w = reinterpret_cast<const uint16_t*>(blob + L.weight_offset);
  p.bias = reinterpret_cast<const float*>(blob);
  p.y = reinterpret_cast<uint16_t*>(y);
  p.x_bytes = (uint32_t)((int64_t)N * H * W * xcs * 2);
  p.w_bytes = (uint32_t)((size_t)L.nchunk_pad * L.Kp * 16);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const dim3 grid((unsigned)(p.per_xcd * 8)), block(kWaves * 64);
  if (dt == FUPR_BF16) hipLaunchKernelGGL(stem_pool_kernel<true>, grid, block, 0, st, p);
  else hipLaunchKernelGGL(stem_pool_kernel<false>, grid, block, 0, st, p);
  return launch_status("stem_pool_kernel");
}

}  // namespace fupr
