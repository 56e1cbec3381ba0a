// Internal: sizes of the packed parameter blob and small helpers shared by the
// host passes, the kernel launchers and the model executor.
#pragma once
#include <cstddef>
#include <cstdint>

#include "fupr.h"

namespace fupr {

inline int round_up(int a, int b) { return (a + b - 1) / b * b; }
inline size_t round_up_sz(size_t a, size_t b) { return (a + b - 1) / b * b; }
inline size_t elem_size(fupr_dtype dt) { return dt == FUPR_F32 ? 4 : 2; }
inline bool dtype_ok(int dt) { return dt == FUPR_F32 || dt == FUPR_BF16 || dt == FUPR_F16; }
inline int c_align(fupr_dtype dt) { return dt == FUPR_F32 ? 4 : 8; }
inline int min_c_stride(int C, fupr_dtype dt) { return round_up(C, c_align(dt)); }
inline int out_extent(int in, int k, int stride, int pad) { return (in + 2 * pad - k) / stride + 1; }

bool shape_ok(const fupr_conv_shape* s);

struct PackedLayout {
  int Kp;          // filters incl. zero padding
  int Cp;          // channels per tap incl. zero padding
  int nchunk;      // 16-bit: R*S*Cp/8 chunks of 8 channels; fp32: R*S*Cp rows
  int nchunk_pad;  // 16-bit: nchunk rounded up to 4; fp32: = nchunk
  size_t weight_offset, total_bytes;
};

inline PackedLayout packed_layout(const fupr_conv_shape& s, fupr_dtype dt) {
  PackedLayout L;
  if (dt == FUPR_F32) {
    L.Kp = round_up(s.K, 4);
    L.Cp = round_up(s.C, 4);
    L.nchunk = L.nchunk_pad = s.R * s.S * L.Cp;
    L.weight_offset = round_up_sz((size_t)L.Kp * 4, 256);
    L.total_bytes = L.weight_offset + (size_t)L.nchunk * L.Kp * 4;
  } else {
    L.Kp = round_up(s.K, 16);
    L.Cp = round_up(s.C, 8);
    L.nchunk = s.R * s.S * (L.Cp / 8);
    L.nchunk_pad = round_up(L.nchunk, 4);
    L.weight_offset = round_up_sz((size_t)L.Kp * 4, 256);
    L.total_bytes = L.weight_offset + (size_t)L.nchunk_pad * L.Kp * 8 * 2;
  }
  L.total_bytes = round_up_sz(L.total_bytes, 256);
  return L;
}

inline size_t weight_bytes(const PackedLayout& L) { return L.total_bytes - L.weight_offset; }

// FUPR_OK if the HIP runtime has no pending error, else FUPR_ERR_LAUNCH (the
// runtime's message goes to stderr when the environment has FUPR_DEBUG set).
fupr_status launch_status(const char* what);
// The same from what the launch itself returned (an int: hipError_t), without asking the runtime.
fupr_status launched(int error, const char* what);

// Launchers (kernels.hip); all arguments already validated.
struct ConvArgs {
  const void* x;
  const void* packed;
  const void* res;
  void* y;
  int N, H, W, C, xcs;   // input
  int P, Q, K, ycs;      // output
  int R, S, stride, pad;
  int rH, rW, rC, rcs, rss, roff;  // residual tensor geometry
  int relu;
  fupr_dtype dt;
  const int32_t* keep;   // device, K entries: filter j adds into channel keep[j] of y; else nullptr
  int yC;                // with keep: channels of y
  // second input of a convolution over two concatenated tensors; x2 = nullptr otherwise
  const void* x2;
  int H2, W2, xcs2, stride2;
  int plan_N;            // images of the whole batch when the launch is a part of one, else 0
  int split_c;           // input channels taken from x (a multiple of 32); the others come from x2
};
fupr_status launch_conv(const ConvArgs& a, void* stream);
// indexed: the convolution adds into listed channels of a wider tensor (ConvArgs::keep); res_at >= 0:
// it has a shortcut at that channel offset; first_c > 0: it reads two tensors, the first of that
// many channels
const char* conv_kernel_name(const fupr_conv_shape& s, fupr_dtype dt, int N, int H, int W,
                             bool indexed = false, int res_at = -1, int first_c = 0);
// fupr_conv_fused / fupr_conv_cat_fused (x2 != nullptr) on a part of a batch of plan_N images.
fupr_status conv_fused_part(const fupr_conv_shape* shape, const fupr_tensor* x, const fupr_tensor* x2,
                            int32_t x2_stride, const void* packed, const fupr_residual* res,
                            uint32_t flags, const fupr_tensor* y, int plan_N, void* stream);
// What fupr_conv_fused checks, and the launcher's arguments of a call that passes.
fupr_status conv_args(const fupr_conv_shape* shape, const fupr_tensor* x, const void* packed,
                      const fupr_residual* res, uint32_t flags, const fupr_tensor* y, ConvArgs* out);
// fupr_conv_scatter_fused likewise.
fupr_status conv_scatter_part(const fupr_conv_shape* shape, const fupr_tensor* x, const void* packed,
                              const int32_t* keep_idx, uint32_t flags, const fupr_tensor* y, int plan_N,
                              void* stream);
// The convolution is one that conv_window.hip takes at this batch size (arguments as for
// conv_kernel_name).
bool conv_is_small(const fupr_conv_shape& s, fupr_dtype dt, int N, int H, int W, int res_at, int first_c);
// Two convolutions of the same tensor, neither with a shortcut, that can run as one launch: one with a window, the
// other 1 x 1, in either order.  convs_beside_part runs them, as two launches where a tensor overlaps another.
bool convs_beside(const fupr_conv_shape& s1, const fupr_conv_shape& s2, fupr_dtype dt, int N, int H, int W);
fupr_status convs_beside_part(const fupr_conv_shape* shape1, const void* packed1, uint32_t flags1, const fupr_tensor* y1,
                              const fupr_conv_shape* shape2, const void* packed2, uint32_t flags2, const fupr_tensor* y2,
                              const fupr_tensor* x, int plan_N, void* stream);
// A global mean and the 1 x 1 convolution of its 1 x 1 image (fc) as one launch, for few images.  mid: the mean, which
// only a run as two launches writes (where a tensor overlaps another).
bool mean_fc_applies(const fupr_conv_shape& s, fupr_dtype dt, int N, int H, int W);
fupr_status mean_fc_part(const fupr_tensor* x, const fupr_tensor* mid, const fupr_conv_shape* shape, const void* packed,
                         uint32_t flags, const fupr_tensor* y, int plan_N, void* stream);
// fupr_conv_cat_fused followed by a 1 x 1 convolution of its output, in one launch
// (what fupr_conv_conv1x1_fused is to fupr_conv_fused); for the model executor.
fupr_status conv_cat_conv1x1_fused(const fupr_conv_shape* shape1, const fupr_tensor* x1,
                                   const fupr_tensor* x2, int32_t x2_stride, const void* packed1,
                                   uint32_t flags1, const fupr_tensor* y,
                                   const fupr_conv_shape* shape2, const void* packed2,
                                   uint32_t flags2, const fupr_tensor* h, void* stream);
// Shapes only: can convolution s1 on an N x H x W input (res_at as above) and convolution s2 on its
// output run as one launch (fupr_conv_conv1x1_fused)?
bool conv_pair_fusable(const fupr_conv_shape& s1, const fupr_conv_shape& s2, fupr_dtype dt, int N,
                       int H, int W, int res_at);

// ---- whole network in one kernel, activations resident in LDS ----------------
// One workgroup per image walks a table of layers; see resident.hip.

constexpr int kResMaxLayers = 256;
constexpr int kResThreads = 1024;
// the kernel of row layers: waves that compute, and threads with those that stage parameters
constexpr int kResRowWaves = 8, kResRowThreads = 768;
constexpr size_t kResLdsLimit = 160 * 1024;
constexpr int kResScratchBytes = 2048;            // start of LDS: partial sums of the mean layer

// One layer of the table the kernel walks (device memory, read with scalar
// loads).  Everything the kernel would otherwise derive per layer is worked out
// once on the host: LDS byte offsets, byte strides per output row / column,
// reciprocal multipliers for the two divisions, the work-item count.
//
// Tensors in LDS carry a halo of zero pixels.  in_org is the LDS byte offset of
// the pixel that tap (0, 0) of output pixel (0, 0) reads (the tap table's entries
// include it); out_org and res_org
// are the offsets of interior pixel (0, 0).  For the global-mean layer M is the
// INPUT pixel count, Q its width, in_org its interior origin, in_row / in_col
// its byte strides.
struct ResLayer {
  const void* packed;        // conv: blob (bias + weights) in global memory
  const void* table;         // conv: tap table in global memory, (nsteps + kResTablePad) * 4 LDS byte offsets
  int32_t blob_units;        // 16-byte units staged to w_off
  int32_t tab_units;         // 16-byte units staged to tab_off
  int32_t w_off, tab_off;    // LDS byte offsets of the blob and of the table
  int32_t wts_off, wstep;    // LDS byte offset of the weights; bytes per MFMA step (4 chunks)
  int32_t in_org, out_org, res_org;   // res_org < 0: no shortcut
  int32_t in_row, in_col;    // bytes from an output pixel's window to the next row's / column's
  int32_t out_row, out_col, res_row, res_col;
  int32_t M, Q;              // output pixels, output width
  uint32_t magicQ;           // floor(m / Q) = mulhi(m, magicQ) for m < 2^16; 0 when Q = 1
  uint32_t magicF;           // floor(item / n_fgroups), likewise
  int32_t nsteps, FT;        // MFMA steps along (r, s, c); filter tiles of 16
  int32_t MT, NT;            // work item: MT pixel tiles x NT filter tiles
  int32_t n_fgroups, n_items;
  int32_t cs_out, res_cs;    // lanes written per output pixel, lanes held per shortcut pixel
  int32_t flags;
  // halo of the output tensor, zeroed by this layer when kResZeroHalo is set
  int32_t hz_org, hz_P, hz_Q, hz_Wh, hz_ps2, hz_chunks, hz_hp;
  int32_t pad_[1];
  // what staging the NEXT layer's parameters needs (a copy of that layer's first
  // eight dwords), so that no load stands between a layer's start and the staging
  const void* next_packed;
  const void* next_table;
  int32_t next_blob_units, next_tab_units, next_w_off, next_tab_off;
};
static_assert(sizeof(ResLayer) == 192, "ResLayer is read as 48 dwords");
constexpr int kResMean = 1, kResRelu = 2, kResLast = 4, kResZeroHalo = 8;
// kResFullPixels: the pixel count is a multiple of a work item's pixels (no
// clamped pixel).  kResFullFilters: no work item has a missing filter tile and
// all 16 lanes of every filter tile are stored.  kResReuse: a wave's first work
// item covers the same pixels at the same strides as in the previous conv
// layer, no pixel tile is ragged, and the output's strides are the input's.
// kResLikeOut: the shortcut tensor has the output's strides.
constexpr int kResFullPixels = 16, kResReuse = 32, kResLikeOut = 64, kResFullFilters = 128;
// An entry with n_items = 0 and no flag is not a layer of the network: it only
// stages the parameters of the entry after it (no wave has a work item, so all
// stage).  The planner puts one in front of a layer whose parameters find no
// room in LDS during the layer before it.
constexpr int kResTablePad = 8;   // steps of padding after a tap table (2 * deepest prefetch)

// A row layer: a 3 x 3 convolution in tiles that are neighbours along the columns (rows_item in resident.hip), each
// computing wave at most one work item.  A network whose convolutions are row layers all, then a global mean and
// a 1 x 1 convolution of it, runs on a kernel of its own that reads one of these per layer (of the last two the
// staging part only); what a wave needs is worked out on the host.
struct ResRow {
  // staging the NEXT layer's parameters, and the halo this layer zeroes when kResZeroHalo is in flags
  const void* next_packed;
  const void* next_table;
  int32_t next_blob_units, next_tab_units, next_w_off, next_tab_off;
  int32_t flags;             // as in ResLayer
  int32_t hz_org, hz_P, hz_Q, hz_Wh, hz_ps2, hz_chunks, hz_hp;
  // the work: LDS byte offsets and strides
  int32_t kind;              // row_kind(), + kResRowRelu, + kResRowHalves
  int32_t wts_off, kp16;     // weights (the bias lies 256 bytes in front of them); bytes per chunk of all filters
  int32_t in_org, out_org, res_org;   // tap (0, 0) of pixel (0, 0); pixel (0, 0); likewise, < 0: no shortcut
  int32_t tap_row, tap_col;  // from a tap to the next one down / to the right
  int32_t out_row, out_col, res_row, res_col;
  int32_t half_in, half_out, half_res;   // kResRowHalves: from a tile's first eight pixels to the other eight
  int32_t res_cs;            // lanes held per shortcut pixel
  // per computing wave, in 16-byte units from the tensor's first pixel: the item's first pixel in the input
  // (+ filter tile << 14; kResNoItem: nothing to do), the output and the shortcut tensor
  uint16_t wave_in[kResRowWaves], wave_out[kResRowWaves], wave_res[kResRowWaves];
  int32_t swizzle;           // shift | mask << 2, of the input; << 4 of the output; << 8 of the shortcut tensor
  int32_t res_step;          // columns of the shortcut tensor between neighbouring pixels
  int32_t pad_[2];
};
static_assert(sizeof(ResRow) == 192 && offsetof(ResRow, kind) == 64 && offsetof(ResRow, wave_in) == 128, "ResRow is read in parts");
constexpr uint16_t kResNoItem = 0xffff;
constexpr int kResRowRelu = 256, kResRowHalves = 512;
// Pixel strides of row layers are multiples of 32 bytes.  Reads of 16 pixels x 4 chunks run at LDS's full rate at odd
// ones; at 64 and 128 bytes the pairs of chunks of a pixel in column x (halo included) lie in another order:
// 32-byte pair j at j ^ (x >> 2 & 1) or j ^ (x >> 1 & 3).
constexpr int row_swizzle_shift(int ps) { return ps == 64 ? 2 : 1; }
constexpr int row_swizzle_mask(int ps) { return ps == 64 ? 1 : ps == 128 ? 3 : 0; }
constexpr int kResNothing = -1, kResTail = -2;   // kinds: an entry that only stages; the mean and what follows
// The sizes that exist: cpt 8-channel chunks per tap, m tiles per work item; -1: not one of them.
constexpr int row_kind(int stride, int cpt, int m) {
  const int most = stride == 1 ? (m == 8 ? 2 : m == 4 ? 4 : m == 2 ? 8 : 0) : (m == 4 ? 2 : m == 2 ? 4 : 0);
  if (cpt > most) return -1;
  return cpt - 1 + (stride == 1 ? (m == 2 ? 0 : m == 4 ? 8 : 12) : (m == 2 ? 14 : 18));
}

struct ResParams {
  const void* x;             // N images, NHWC
  void* y;                   // N x out_pixels x y_cs
  const ResLayer* layers;    // device memory
  int in_H, in_W, in_Wh;     // image extent and pixels per LDS row (in_W + 2 * hp)
  int in_cs, in_ps2;         // global channel stride (elements), LDS pixel stride (bytes)
  int in_org;                // LDS byte offset of the image's interior pixel (0, 0)
  int hp;                    // halo width of every LDS tensor larger than 1 x 1
  int y_cs, out_pixels;
  int n_layers;
  int lds_bytes;
  const ResRow* rows;        // device memory: the layers for the kernel of row layers; nullptr: the other kernel
};

fupr_status launch_resident(const ResParams& p, int N, fupr_dtype dt, void* stream);

}  // namespace fupr
