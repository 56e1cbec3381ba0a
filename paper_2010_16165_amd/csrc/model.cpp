// Whole-network executor: validates an operator list, plans which intermediate
// tensors share workspace memory, and enqueues one kernel per operator on the
// caller's stream (Table II networks after fusion and filter removal).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "basic_block.h"
#include "bottleneck.h"
#include "fupr.h"
#include "layout.h"
#include "stem_pool.h"
#include "tuning.h"

using namespace fupr;

namespace {

// One kernel launch of the per-operator schedule: `count` consecutive operators.
enum { kBottleneck = 1, kBasic = 2, kBeside = 3, kMeanFc = 4 };   // bottleneck.hip, basic_block.hip, conv_window.hip

struct Launch {
  int first, count;
  int block = 0;        // kBottleneck or kBasic: a block in one launch; kBeside: two convolutions of one tensor;
                        // kMeanFc: a global mean and the layer behind it
  int plan = -1;        // ... and its kernel's plan for the batch
};

struct TensorInfo {
  int C, H, W, cs;   // per image
  int buffer;        // workspace buffer id; -1 = network input, -2 = network output
  int last_use;      // index of the last operator reading it
};

}  // namespace

constexpr int kMaxSplit = 4;

struct fupr_model {
  fupr_dtype dt;
  std::vector<fupr_op_desc> ops;
  std::vector<TensorInfo> tensors;        // n_ops + 1
  std::vector<size_t> buffer_elems;       // per image, per workspace buffer
  std::vector<char> pair_planned;         // per operator: the workspace lets it run together with the next one
  bool blocks = false;                    // fupr_model_fuse_blocks
  // The launches of a batch size, and blocks as one launch: the same workspace buffers, tensors placed in them so that
  // what a block reads outlives the block.  Made at the first pass of that many images and kept.
  struct Placement {
    std::vector<Launch> launches;
    std::vector<int> buffer;              // per tensor, as TensorInfo::buffer; -3: not needed; empty: the model's own
    // per number of images of a sub-batch (up to two for each of at most four splits): the block's plan
    // per operator that starts one
    mutable std::map<int, std::shared_ptr<const std::vector<int>>> parts;
    mutable std::mutex parts_mutex;
  };
  std::map<int, std::shared_ptr<const Placement>> placed;
  std::mutex placed_mutex;
  // shapes of the block that starts with an operator
  struct Block {
    int kind;                             // kBottleneck, kBasic, or 0
    int count;                            // its operators
    BottleneckArgs bottleneck;
    BasicBlockArgs basic;
  };
  std::vector<Block> block_args;
  std::vector<Launch> launches[2];        // per schedule, with no tuning switch set
  int schedule = FUPR_SCHEDULE_AUTO;
  bool resident_ok = false;               // the whole network fits one LDS-resident kernel
  ResParams resident{};                   // x, y, y_cs filled per call
  std::vector<ResLayer> res_layers;       // host copy of the layer table
  std::vector<ResRow> res_rows;           // and of the table of row layers; empty: they are not all row layers
  std::vector<int32_t> res_tables;        // tap tables of all layers, back to back
  std::vector<size_t> res_table_at;       // first entry of each layer's table
  const void* res_dev = nullptr;          // the caller's device copy of the table (fupr_model_set_table)
  // Per-operator schedule: the batch runs as sub-batches on streams the caller
  // lends (fupr_model_set_side_streams) that fork from and join the caller's
  // stream, so that one sub-batch's launch gaps, prologues and tails are filled
  // by the other's work.
  int n_side = 0;
  hipStream_t side_stream[kMaxSplit - 1] = {};
  hipEvent_t fork_event = nullptr, join_event[kMaxSplit - 1] = {};
  std::mutex side_mutex;                  // one forked enqueue at a time: the events are shared
};

struct fupr_graph {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

// Shape of one work item of the LDS-resident kernel for a conv layer: MT pixel
// tiles x NT filter tiles.  Picks the shape with the smallest estimated layer
// time from three measured rates: the compute unit's LDS port (about 5.6 clocks
// per 1 KB fragment read, 16 per 8-byte-per-lane store), MFMA 16x16x32 issue on
// the busiest of the four SIMDs (16 clocks, 24 when a wave has a single
// accumulator and every MFMA waits for the one before), and vector
// instructions beside them (about 2.7 clocks each).  Items go round robin
// over 16 waves, hence over the 4 SIMDs.
// The tuning switch res_item="M/FT/nsteps:MTxNT,..." overrides the choice per
// layer class (an aid for sweeps).
void resident_item_shape(int M, int FT, int nsteps, bool has_res, int* MT_out, int* NT_out) {
  static const int shapes[5][2] = {{4, 1}, {2, 2}, {2, 1}, {1, 2}, {1, 1}};
  char env[128];
  if (tuning_text("res_item", env, sizeof(env))) {
    const char* c = env;
    while (*c) {
      int em = 0, ef = 0, es = 0, mt = 0, nt = 0, used = 0;
      if (std::sscanf(c, "%d/%d/%d:%dx%d%n", &em, &ef, &es, &mt, &nt, &used) == 5) {
        if (em == M && ef == FT && es == nsteps)
          for (const auto& sh : shapes)
            if (sh[0] == mt && sh[1] == nt) { *MT_out = mt; *NT_out = nt; return; }
        c += used;
      }
      while (*c && *c != ',') ++c;
      if (*c == ',') ++c;
    }
  }
  const int waves = kResThreads / 64;
  const int n_ptiles = (M + 15) / 16;
  const int steps = nsteps + (has_res ? 1 : 0);
  double best = 1e30;
  for (const auto& sh : shapes) {
    const int mt = sh[0], nt = sh[1];
    const int items = ((n_ptiles + mt - 1) / mt) * ((FT + nt - 1) / nt);
    const int rounds = (items + waves - 1) / waves;
    const int simd_items = (items + 3) / 4;
    const double lds = (double)items * (nsteps * (mt * 5.6 + nt * 5.0 + 2.0) +
                                        (has_res ? mt * nt * 5.6 : 0.0) + mt * nt * 16.0 + nt * 5.0);
    const double mfma = (double)simd_items * steps * mt * nt * (mt * nt == 1 ? 24.0 : 16.0);
    const double valu = (double)simd_items * (20.0 + 9.0 * mt + nsteps * (mt + 1.0) + 8.0 * mt * nt) * 2.7;
    const double t = std::max(lds, mfma + 0.6 * valu) + rounds * 600.0;
    if (t < best) {
      best = t;
      *MT_out = mt;
      *NT_out = nt;
    }
  }
}

// Tiles per work item of a row layer: `chains` chains of `chain` vertical neighbours x FT filter tiles on eight waves;
// 0: it does not fit them.  A tall item reads fewer rows per tile, but two waves on a SIMD hide each other's waits:
// the sizes that keep all eight busy first.
int row_tiles(int stride, int cpt, int chain, int chains, int FT) {
  int best = 0, most = 0;
  for (int m : {8, 4, 2}) {
    if (chain % m != 0 || row_kind(stride, cpt, m) < 0) continue;
    const int items = chains * (chain / m) * FT;
    if (items <= kResRowWaves && items > most) {
      best = m;
      most = items;
    }
  }
  return best;
}

// Describes convolution `op` from ti to to as a row layer, given the layer's place in LDS; false: it is none.
bool describe_row(const fupr_op_desc& op, const TensorInfo& ti, const TensorInfo& to, const ResLayer& L, const PackedLayout& PL,
                  int in_ps, int out_ps, int res_ps, int halo, ResRow* r) {
  const fupr_conv_shape& s = op.conv;
  if (s.R != 3 || s.S != 3 || s.pad != 1 || halo != 1 || (s.stride != 1 && s.stride != 2) || PL.Kp > 64) return false;
  if (PL.Kp * 2 > out_ps) return false;         // all 16 channels of a filter tile are stored
  if (op.res >= 0 && s.stride != 1) return false;
  // a tile is 16 pixels of a row, or 8 of row t and 8 of row t + P / 2
  const bool halves = to.W == 8 && to.H % 2 == 0;
  if (!halves && to.W % 16 != 0) return false;
  const int chain = halves ? to.H / 2 : to.H, side = halves ? 1 : to.W / 16, cpt = PL.Cp / 8;
  const int m = row_tiles(s.stride, cpt, chain, side, L.FT);
  if (m == 0) return false;
  if (m == 8 && (row_swizzle_mask(in_ps) || row_swizzle_mask(out_ps) || row_swizzle_mask(res_ps))) return false;
  r->kind = row_kind(s.stride, cpt, m) + ((op.epilogue & FUPR_FUSE_RELU) ? kResRowRelu : 0) + (halves ? kResRowHalves : 0);
  r->wts_off = L.wts_off;
  r->kp16 = PL.Kp * 16;
  r->in_org = L.in_org;
  r->out_org = L.out_org;
  r->res_org = L.res_org;
  r->tap_row = L.in_row / s.stride;
  r->tap_col = in_ps;
  r->out_row = L.out_row;
  r->out_col = L.out_col;
  r->res_row = L.res_row;
  r->res_col = L.res_col;
  r->half_in = halves ? chain * L.in_row : 0;
  r->half_out = halves ? chain * L.out_row : 0;
  r->half_res = halves ? chain * L.res_row : 0;
  r->res_cs = L.res_cs;
  auto swizzle = [](int ps) { return row_swizzle_shift(ps) | row_swizzle_mask(ps) << 2; };
  r->swizzle = swizzle(in_ps) | swizzle(out_ps) << 4 | swizzle(res_ps) << 8;
  r->res_step = op.res_spatial_stride;
  for (int w = 0; w < kResRowWaves && w < side * (chain / m) * L.FT; ++w) {
    const int ft = w % L.FT, at = w / L.FT, col = at % side * 16, row = at / side * m;
    r->wave_in[w] = (uint16_t)((row * L.in_row + col * L.in_col) / 16 | ft << 14);
    r->wave_out[w] = (uint16_t)((row * L.out_row + col * L.out_col) / 16);
    r->wave_res[w] = (uint16_t)((row * L.res_row + col * L.res_col) / 16);
  }
  return true;
}

// A block of LDS with a lifetime in layers; blocks whose lifetimes intersect
// must not overlap.
struct LdsBlock {
  size_t units;       // 16-byte units
  int first, last;    // layers during which it is live (inclusive)
  size_t offset;
};

// Offset assignment: blocks are placed one by one at the lowest offset free
// over their whole lifetime.  The order matters; three orders are tried
// (largest first, earliest first, longest-lived first) and the tightest result
// is kept.
size_t place_in_order(std::vector<LdsBlock>& blocks, const std::vector<int>& order) {
  std::vector<int> placed;
  size_t extent = 0;
  for (int id : order) {
    LdsBlock& b = blocks[id];
    if (b.units == 0) { b.offset = 0; continue; }
    std::vector<std::pair<size_t, size_t>> busy;
    for (int other : placed) {
      const LdsBlock& o = blocks[other];
      if (o.first <= b.last && b.first <= o.last) busy.emplace_back(o.offset, o.offset + o.units);
    }
    std::sort(busy.begin(), busy.end());
    size_t at = 0;
    for (const auto& iv : busy) {
      if (at + b.units <= iv.first) break;
      at = std::max(at, iv.second);
    }
    b.offset = at;
    extent = std::max(extent, at + b.units);
    placed.push_back(id);
  }
  return extent;
}

size_t assign_offsets(std::vector<LdsBlock>& blocks) {
  std::vector<int> order(blocks.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
  std::vector<LdsBlock> best;
  size_t best_extent = ~size_t(0);
  for (int rule = 0; rule < 3; ++rule) {
    std::vector<int> o = order;
    std::stable_sort(o.begin(), o.end(), [&](int a, int b) {
      const LdsBlock &x = blocks[a], &y = blocks[b];
      if (rule == 0) return x.units > y.units;
      if (rule == 1) return x.first != y.first ? x.first < y.first : x.units > y.units;
      const int lx = x.last - x.first, ly = y.last - y.first;
      return lx != ly ? lx > ly : x.units > y.units;
    });
    std::vector<LdsBlock> trial = blocks;
    const size_t extent = place_in_order(trial, o);
    if (extent < best_extent) {
      best_extent = extent;
      best = trial;
    }
  }
  blocks = best;
  return best_extent;
}

// LDS pixel stride in bytes for tensors of cs 16-bit lanes.  The 16 pixels x 4
// chunks of one MFMA pixel fragment are read with one 16-byte access per lane;
// measured on gfx950 that access takes about 5 clocks of the LDS port when the
// pixel stride is an odd multiple of 32 bytes, 8.6 at other multiples of 16
// that are not multiples of 64, 8.7 at odd multiples of 64 and 16.7 at
// multiples of 128.  mode 0: the nearest odd multiple of 32; 1: the nearest
// stride that is not a multiple of 64; 2: dense.
constexpr int kRowStride = 3;   // mode of row layers (row_swizzle_mask)
int lds_pixel_stride(int cs, int mode) {
  const int dense = cs * 2;
  if (mode == kRowStride) return round_up(dense, 32);
  if (mode == 2) return dense;
  if (mode == 1) return dense % 64 == 0 ? dense + 16 : dense;
  int ps2 = dense;
  while (ps2 % 64 != 32) ps2 += 16;
  return ps2;
}

double lds_read_clocks(int ps2) {
  if (ps2 % 64 == 32) return 5.1;
  if (ps2 % 128 == 0) return 16.7;
  if (ps2 % 64 == 0) return 8.7;
  return 8.6;
}

// floor(v / d) = mulhi(v, reciprocal) for v < 2^16; 0 stands for d = 1
uint32_t reciprocal_u16(int d) { return d == 1 ? 0u : 0xffffffffu / (uint32_t)d + 1u; }

// Tries to lay the whole network out for resident_kernel: every per-image
// tensor (input included, final output excluded) and, for the current and the
// next layer, the tap table and the parameter blob, in LDS.
void plan_resident(fupr_model* m) {
  m->resident_ok = false;
  const int n = (int)m->ops.size();
  if (m->dt == FUPR_F32 || n > kResMaxLayers) return;
  for (const TensorInfo& t : m->tensors)
    if (t.H > 255 || t.W > 255 || t.cs > 4096) return;

  // every LDS tensor larger than 1 x 1 gets a ring of hp zero pixels
  int hp = 0;
  for (const fupr_op_desc& op : m->ops) {
    if (op.kind == FUPR_OP_CONV && (op.epilogue & (FUPR_FUSE_SCATTER | FUPR_FUSE_CAT))) return;   // per-operator kernels only
    if (op.kind == FUPR_OP_CONV) hp = std::max(hp, op.conv.pad);
    else if (op.kind != FUPR_OP_AVGPOOL) return;   // max-pool networks: images too large for LDS
  }
  for (const TensorInfo& t : m->tensors)
    if ((int64_t)(t.W + 2 * hp) * (t.H + 2 * hp) >= 65536) return;
  auto halo_of = [&](const TensorInfo& t) { return t.H * t.W > 1 ? hp : 0; };
  auto row_of = [&](const TensorInfo& t) { return t.W + 2 * halo_of(t); };

  const size_t budget_units = (kResLdsLimit - kResScratchBytes) / 16;

  // Tensors of one resolution share one pixel stride (that of the widest), so
  // that a tensor lands on the bytes of a dead tensor of the same geometry and
  // finds its halo still zero.  Per resolution the stride is the cheapest to
  // read that still lets the whole plan fit.
  struct Res { int H, W, cs, readers; };
  std::vector<Res> classes;
  std::vector<int> class_of(n + 1, -1);
  for (int tid = 0; tid <= n; ++tid) {
    const TensorInfo& t = m->tensors[tid];
    if (t.H * t.W <= 1 || tid == n) continue;
    size_t c = 0;
    while (c < classes.size() && !(classes[c].H == t.H && classes[c].W == t.W)) ++c;
    if (c == classes.size()) classes.push_back(Res{t.H, t.W, 0, 0});
    classes[c].cs = std::max(classes[c].cs, t.cs);
    class_of[tid] = (int)c;
  }
  for (const fupr_op_desc& op : m->ops)
    if (op.kind == FUPR_OP_CONV && class_of[op.in] >= 0) ++classes[class_of[op.in]].readers;
  // A block's output may be written over its shortcut tensor: the shortcut is
  // read by the lane that writes the same pixel and channels, before it writes,
  // and by nobody else; no convolution reads it in that layer.  home[t] is the
  // tensor whose LDS block t lives in.
  std::vector<int> home(n + 1);
  for (int tid = 0; tid <= n; ++tid) home[tid] = tid;
  for (int i = 0; i + 1 < n; ++i) {
    const fupr_op_desc& op = m->ops[i];
    if (op.kind != FUPR_OP_CONV || op.res < 0 || op.res == op.in) continue;
    const TensorInfo& tr = m->tensors[op.res];
    if (tr.last_use != i || op.res_spatial_stride != 1 || op.res_c_offset != 0) continue;
    if (class_of[op.res] < 0 || class_of[op.res] != class_of[i + 1]) continue;
    home[i + 1] = home[op.res];
  }
  const int k = (int)classes.size();
  std::vector<std::pair<double, std::vector<int>>> candidates;
  if (k <= 5) {
    int combos = 1;
    for (int c = 0; c < k; ++c) combos *= 3;
    for (int code = 0; code < combos; ++code) {
      std::vector<int> modes(k);
      double cost = 0.0;
      for (int c = 0, rest = code; c < k; ++c, rest /= 3) {
        modes[c] = rest % 3;
        const int ps2 = lds_pixel_stride(classes[c].cs, modes[c]);
        cost += classes[c].readers * lds_read_clocks(ps2) + 1e-6 * ps2;   // ties: the smaller stride
      }
      candidates.emplace_back(cost, modes);
    }
  } else {
    for (int mode = 0; mode < 3; ++mode) candidates.emplace_back((double)mode, std::vector<int>(k, mode));
  }
  std::stable_sort(candidates.begin(), candidates.end(),
                   [](const auto& a, const auto& b) { return a.first < b.first; });
  // first of all as row layers, which have the smallest strides
  if (!tuning_off("resident_rows")) candidates.insert(candidates.begin(), {-1.0, std::vector<int>(k, kRowStride)});

  // Parameter blocks by size, largest first: when nothing fits with every
  // layer's parameters staged one layer ahead, the largest ones are staged at
  // the start of their own layer instead (their global-memory latency is then
  // exposed, but they need LDS for one layer only).
  std::vector<int> by_size;
  for (int i = 1; i < n; ++i)
    if (m->ops[i].kind == FUPR_OP_CONV) by_size.push_back(i);
  std::stable_sort(by_size.begin(), by_size.end(), [&](int a, int b) {
    return packed_layout(m->ops[a].conv, m->dt).total_bytes >
           packed_layout(m->ops[b].conv, m->dt).total_bytes;
  });
  for (size_t n_late = 0; n_late <= by_size.size(); ++n_late) {
  std::vector<char> late(n, 0);
  for (size_t j = 0; j < n_late; ++j) late[by_size[j]] = 1;
  for (const auto& cand : candidates) {
    const bool as_rows = cand.first < 0.0;
    std::vector<int> ps2(n + 1);
    for (int tid = 0; tid <= n; ++tid) {
      const int c = class_of[tid];
      ps2[tid] = c >= 0 ? lds_pixel_stride(classes[c].cs, cand.second[c]) : m->tensors[tid].cs * 2;
    }
    std::vector<LdsBlock> blocks(2 * (size_t)n + 1);
    for (int tid = 0; tid <= n; ++tid) {
      const TensorInfo& t = m->tensors[tid];
      LdsBlock& b = blocks[tid];
      b.first = tid - 1;                       // produced by layer tid-1 (image: before layer 0)
      b.last = std::max(t.last_use, b.first);
      b.units = tid == n ? 0 : (size_t)(t.H + 2 * halo_of(t)) * row_of(t) * ps2[tid] / 16;
      if (home[tid] != tid) {                  // written over its shortcut: that block lives on
        blocks[home[tid]].last = std::max(blocks[home[tid]].last, b.last);
        b.units = 0;
      }
    }
    bool ok = true;
    for (int i = 0; i < n && ok; ++i) {
      LdsBlock& b = blocks[n + 1 + i];
      b.first = late[i] ? i : i - 1;           // lands while layer i-1 is running, unless late
      b.last = i;
      b.units = 0;
      if (m->ops[i].kind == FUPR_OP_CONV) {
        const PackedLayout PL = packed_layout(m->ops[i].conv, m->dt);
        if (PL.nchunk_pad / 4 + kResTablePad > 64) ok = false;   // one wave stages the table
        b.units = PL.total_bytes / 16;
        if (!as_rows || i + 1 == n) b.units += PL.nchunk_pad / 4 + kResTablePad;   // table (16 bytes per step), blob
      }
    }
    if (!ok && as_rows) continue;
    if (!ok) return;
    const size_t extent = assign_offsets(blocks);
    if (tuning_int("debug", 0)) {
      std::fprintf(stderr, "resident candidate: strides");
      for (int c = 0; c < k; ++c)
        std::fprintf(stderr, " %dx%d:%d", classes[c].H, classes[c].W,
                     lds_pixel_stride(classes[c].cs, cand.second[c]));
      std::fprintf(stderr, " late %zu -> %zu bytes (limit %zu)\n", n_late, extent * 16,
                   budget_units * 16);
    }
    if (extent > budget_units) continue;

    // LDS byte offset of pixel (row, col) counted from the halo's corner
    auto pixel_at = [&](int tid, int row, int col) {
      const TensorInfo& t = m->tensors[tid];
      return (int32_t)(blocks[home[tid]].offset * 16 + (size_t)(row * row_of(t) + col) * ps2[tid]);
    };

    // known-zero 16-byte units, to skip re-zeroing halos that are still clean
    std::vector<uint8_t> clean(extent, 0);
    auto mark = [&](size_t first, size_t count, uint8_t v) {
      std::fill(clean.begin() + first, clean.begin() + first + count, v);
    };
    auto halo_units = [&](int tid, auto&& fn) {   // fn(unit) for every channel chunk of the halo
      const TensorInfo& t = m->tensors[tid];
      const int h = halo_of(t), Wh = row_of(t);
      for (int row = 0; row < t.H + 2 * h; ++row)
        for (int col = 0; col < Wh; ++col) {
          if (row >= h && row < t.H + h && col >= h && col < t.W + h) continue;
          const size_t u = (size_t)pixel_at(tid, row, col) / 16;
          for (int c = 0; c < (as_rows ? ps2[tid] / 16 : t.cs / 8); ++c) fn(u + c);
        }
    };
    auto write_interior = [&](int tid) {
      const TensorInfo& t = m->tensors[tid];
      const int h = halo_of(t);
      for (int row = 0; row < t.H; ++row)
        mark((size_t)pixel_at(tid, row + h, h) / 16, (size_t)t.W * ps2[tid] / 16, 0);
    };

    ResParams& R = m->resident;
    R = ResParams{};
    const TensorInfo& t0 = m->tensors[0];
    R.in_H = t0.H;
    R.in_W = t0.W;
    R.in_Wh = row_of(t0);
    R.in_cs = t0.cs;
    R.in_ps2 = ps2[0];
    R.in_org = pixel_at(0, halo_of(t0), halo_of(t0));
    R.hp = hp;
    R.lds_bytes = (int)(kResScratchBytes + extent * 16);
    R.out_pixels = m->tensors[n].H * m->tensors[n].W;
    write_interior(0);
    halo_units(0, [&](size_t u) { clean[u] = 1; });
    if (blocks[n + 1].units) mark(blocks[n + 1].offset, blocks[n + 1].units, 0);

    std::array<int, 8> prev_geometry;
    prev_geometry.fill(-1);
    m->res_layers.clear();
    m->res_rows.clear();
    bool rows = as_rows && n >= 3;   // every layer so far is a row layer, or one of the last two
    m->res_tables.clear();
    m->res_table_at.clear();
    for (int i = 0; i < n; ++i) {
      const fupr_op_desc& op = m->ops[i];
      const TensorInfo& ti = m->tensors[op.in];
      const TensorInfo& to = m->tensors[i + 1];
      const bool last = i + 1 == n;
      ResLayer L{};
      ResRow no_row{};
      no_row.kind = kResNothing;
      std::fill(no_row.wave_in, no_row.wave_in + kResRowWaves, kResNoItem);
      ResRow row = no_row;
      size_t table_at = 0;
      L.flags = last ? kResLast : 0;
      if (late[i]) {
        // an entry that does nothing but stage this layer's parameters
        ResLayer stage{};
        stage.res_org = -1;
        stage.MT = stage.NT = stage.n_fgroups = stage.Q = stage.M = 1;   // a conv entry without work items
        m->res_layers.push_back(stage);
        m->res_rows.push_back(no_row);
        m->res_table_at.push_back(0);
        if (blocks[n + 1 + i].units) mark(blocks[n + 1 + i].offset, blocks[n + 1 + i].units, 0);
      }
      L.res_org = -1;
      L.out_org = last ? 0 : pixel_at(i + 1, halo_of(to), halo_of(to));
      L.cs_out = to.cs;
      L.M = to.H * to.W;
      L.Q = to.W;
      L.MT = L.NT = L.n_fgroups = 1;
      if (op.kind == FUPR_OP_AVGPOOL) {
        L.flags |= kResMean;
        L.in_org = pixel_at(op.in, halo_of(ti), halo_of(ti));
        L.in_row = row_of(ti) * ps2[op.in];
        L.in_col = ps2[op.in];
        L.M = ti.H * ti.W;       // the mean layer iterates over its INPUT extent
        L.Q = ti.W;
        // partial sums held in the scratch area: MT parts x cs_out floats
        L.MT = std::min(8, kResScratchBytes / 4 / to.cs);
        if (L.MT < 1 || L.MT * to.cs > kResThreads) return;
      } else {
        const fupr_conv_shape& s = op.conv;
        const PackedLayout PL = packed_layout(s, m->dt);
        if (halo_of(ti) < s.pad) return;   // a padded conv on a 1 x 1 image: not laid out here
        const int nsteps = PL.nchunk_pad / 4, cpt = PL.Cp / 8;
        L.packed = op.packed;
        L.blob_units = (int32_t)(PL.total_bytes / 16);
        L.tab_units = as_rows && !last ? 0 : nsteps + kResTablePad;
        L.tab_off = (int32_t)(blocks[n + 1 + i].offset * 16);
        L.w_off = L.tab_off + L.tab_units * 16;
        L.wts_off = L.w_off + (int32_t)PL.weight_offset;
        L.wstep = 4 * PL.Kp * 16;
        L.in_org = pixel_at(op.in, halo_of(ti) - s.pad, halo_of(ti) - s.pad);
        L.in_row = s.stride * row_of(ti) * ps2[op.in];
        L.in_col = s.stride * ps2[op.in];
        L.out_row = row_of(to) * ps2[i + 1];
        L.out_col = ps2[i + 1];
        L.nsteps = nsteps;
        L.FT = PL.Kp / 16;
        if (op.epilogue & FUPR_FUSE_RELU) L.flags |= kResRelu;
        if (op.res >= 0) {
          if (op.res_c_offset != 0) return;
          const TensorInfo& tr = m->tensors[op.res];
          L.res_org = pixel_at(op.res, halo_of(tr), halo_of(tr));
          L.res_cs = tr.cs;
          L.res_row = op.res_spatial_stride * row_of(tr) * ps2[op.res];
          L.res_col = op.res_spatial_stride * ps2[op.res];
        }
        int mt = 1, nt = 1;
        resident_item_shape(L.M, L.FT, nsteps, op.res >= 0, &mt, &nt);
        L.MT = mt;
        L.NT = nt;
        L.n_fgroups = (L.FT + nt - 1) / nt;
        L.n_items = ((L.M + 15) / 16 + mt - 1) / mt * L.n_fgroups;
        if (L.n_items >= 65536) return;
        if (L.M % (16 * mt) == 0) L.flags |= kResFullPixels;
        if (L.FT % nt == 0 && to.cs == PL.Kp && !last) L.flags |= kResFullFilters;
        if (op.res >= 0 && L.res_row == L.out_row && L.res_col == L.out_col) L.flags |= kResLikeOut;
        const std::array<int, 8> geometry = {L.M, L.Q, mt, L.n_fgroups, L.in_row, L.in_col, L.out_row, L.out_col};
        if (L.n_items <= kResThreads / 64) {
          if (geometry == prev_geometry && (L.flags & kResFullPixels) && !last && L.in_row == L.out_row &&
              L.in_col == L.out_col)
            L.flags |= kResReuse;
          prev_geometry = geometry;
        } else {
          prev_geometry.fill(-1);   // later work items overwrite what the first one left
        }
        // tap table: LDS byte offset of every chunk of output pixel (0, 0)'s
        // window; padding chunks (zero weights) and the padding steps after the
        // last one re-read the first chunk: finite data
        table_at = m->res_tables.size();
        for (int j = 0; j < L.tab_units * 4; ++j) {
          int32_t e = 0;
          if (j < PL.nchunk) {
            const int tap = j / cpt, c8 = j - tap * cpt;
            const int r = tap / s.S, sx = tap - r * s.S;
            e = (r * row_of(ti) + sx) * ps2[op.in] + c8 * 16;
          }
          m->res_tables.push_back(L.in_org + e);
        }
      }
      // (the mean and the convolution behind it run on the kernel's general path)
      const bool tail = i + 2 == n ? (L.flags & kResMean) != 0 && kResRowWaves * to.cs * 4 <= kResScratchBytes
                                   : last && op.kind == FUPR_OP_CONV && op.conv.R == 1 && op.conv.S == 1 && op.res < 0 &&
                                         L.MT == 1 && L.NT <= 2;
      if (op.kind == FUPR_OP_CONV && i + 2 < n)
        rows = rows && describe_row(op, ti, to, L, packed_layout(op.conv, m->dt), ps2[op.in], ps2[i + 1],
                                    ps2[op.res >= 0 ? op.res : op.in], halo_of(ti), &row);
      else
        rows = rows && tail, row.kind = kResTail;
      if (as_rows && !rows) break;
      L.magicQ = reciprocal_u16(L.Q);
      L.magicF = reciprocal_u16(L.n_fgroups);
      if (!last) {
        bool dirty = false;
        halo_units(i + 1, [&](size_t u) { dirty = dirty || !clean[u]; });
        if (dirty) {
          L.flags |= kResZeroHalo;
          L.hz_org = L.out_org;
          L.hz_P = to.H;
          L.hz_Q = to.W;
          L.hz_Wh = row_of(to);
          L.hz_ps2 = ps2[i + 1];
          L.hz_chunks = as_rows ? ps2[i + 1] / 16 : to.cs / 8;
          L.hz_hp = halo_of(to);
          halo_units(i + 1, [&](size_t u) { clean[u] = 1; });
        }
        if (halo_of(to) > 0) write_interior(i + 1);
        else mark(blocks[home[i + 1]].offset, blocks[home[i + 1]].units, 0);
      }
      if (i + 1 < n && !late[i + 1] && blocks[n + 2 + i].units)
        mark(blocks[n + 2 + i].offset, blocks[n + 2 + i].units, 0);
      m->res_layers.push_back(L);
      row.flags = L.flags;
      row.hz_org = L.hz_org;
      row.hz_P = L.hz_P;
      row.hz_Q = L.hz_Q;
      row.hz_Wh = L.hz_Wh;
      row.hz_ps2 = L.hz_ps2;
      row.hz_chunks = L.hz_chunks;
      row.hz_hp = L.hz_hp;
      m->res_rows.push_back(row);
      m->res_table_at.push_back(table_at);
      if (tuning_int("debug", 0))
        std::fprintf(stderr, "resident layer %d: M %d FT %d steps %d item %dx%d items %d ps2 in %d out %d "
                     "zero_halo %d res %d\n", i, L.M, L.FT, L.nsteps, L.MT, L.NT, L.n_items, ps2[op.in],
                     ps2[i + 1], (L.flags & kResZeroHalo) != 0, L.res_org >= 0);
    }
    if (as_rows && !rows) {
      m->res_rows.clear();
      continue;
    }
    if (m->res_layers.size() > (size_t)kResMaxLayers) return;
    R.n_layers = (int)m->res_layers.size();
    if (!as_rows) m->res_rows.clear();
    if (tuning_int("debug", 0))
      std::fprintf(stderr, "resident plan: %d bytes of LDS, %d table entries for %d layers\n",
                   R.lds_bytes, R.n_layers, n);
    m->resident_ok = true;
    return;
  }
  }
}

void release_side(fupr_model* m);   // below, with the forked schedule
bool conv_conv_pair(const fupr_model* m, size_t i);   // below, with the launch list
bool stem_pool_pair(const fupr_model* m, size_t i);
void find_blocks(fupr_model* m);                      // likewise
std::vector<Launch> list_launches(const fupr_model* m, int schedule);

// Sizes of the one-kernel schedule's table: the layer entries, then the tap tables.
size_t resident_layer_bytes(const fupr_model* m) {
  return round_up_sz(m->res_layers.size() * sizeof(ResLayer), 256);
}
size_t resident_table_bytes(const fupr_model* m) {
  return round_up_sz(m->res_tables.size() * sizeof(int32_t), 256) + 256;
}
// behind them, the table of row layers
size_t resident_rows_bytes(const fupr_model* m) { return round_up_sz(m->res_rows.size() * sizeof(ResRow), 256); }

}  // namespace

extern "C" fupr_status fupr_model_create(const fupr_graph_desc* g, fupr_model** out) {
  if (!g || !out || !g->ops) return FUPR_ERR_NULL;
  if (!dtype_ok((int)g->dt)) return FUPR_ERR_DTYPE;
  if (g->n_ops <= 0 || g->C <= 0 || g->H <= 0 || g->W <= 0) return FUPR_ERR_SHAPE;

  fupr_model* m = new (std::nothrow) fupr_model;
  if (!m) return FUPR_ERR_ARG;
  m->dt = g->dt;
  m->ops.assign(g->ops, g->ops + g->n_ops);
  m->tensors.resize(g->n_ops + 1);
  m->tensors[0] = TensorInfo{g->C, g->H, g->W, min_c_stride(g->C, g->dt), -1, -1};

  fupr_status err = FUPR_OK;
  for (int i = 0; i < g->n_ops && err == FUPR_OK; ++i) {
    const fupr_op_desc& op = m->ops[i];
    if (op.in < 0 || op.in > i) { err = FUPR_ERR_ARG; break; }
    const TensorInfo& tin = m->tensors[op.in];
    TensorInfo t{};
    t.buffer = -3;
    t.last_use = -1;
    if (op.kind == FUPR_OP_CONV) {
      const fupr_conv_shape& s = op.conv;
      if (!shape_ok(&s)) { err = FUPR_ERR_SHAPE; break; }
      if (!op.packed) { err = FUPR_ERR_NULL; break; }
      if (op.epilogue & ~uint32_t(FUPR_FUSE_RELU | FUPR_FUSE_ADD | FUPR_FUSE_SCATTER | FUPR_FUSE_CAT)) {
        err = FUPR_ERR_ARG; break;
      }
      const bool cat = (op.epilogue & FUPR_FUSE_CAT) != 0;
      int c_in = tin.C;
      if (cat) {
        // a 1 x 1 convolution over tensor `in` and tensor `in2` concatenated along the channels
        if (g->dt == FUPR_F32) { err = FUPR_ERR_DTYPE; break; }
        if (op.in2 < 0 || op.in2 > i || (op.in2_spatial_stride != 1 && op.in2_spatial_stride != 2) ||
            (op.epilogue & FUPR_FUSE_SCATTER)) {
          err = FUPR_ERR_ARG; break;
        }
        const TensorInfo& t2 = m->tensors[op.in2];
        if (s.R != 1 || s.S != 1 || s.stride != 1 || s.pad != 0 ||
            (int64_t)(tin.H - 1) * op.in2_spatial_stride >= t2.H ||
            (int64_t)(tin.W - 1) * op.in2_spatial_stride >= t2.W) {
          err = FUPR_ERR_SHAPE; break;
        }
        c_in = round_up(tin.C, FUPR_CAT_ALIGN) + t2.C;
      }
      if (s.C != c_in || tin.H + 2 * s.pad < s.R || tin.W + 2 * s.pad < s.S) {
        err = FUPR_ERR_SHAPE; break;
      }
      const bool scatter = (op.epilogue & FUPR_FUSE_SCATTER) != 0;
      if (scatter != (op.keep_idx != nullptr)) { err = scatter ? FUPR_ERR_NULL : FUPR_ERR_ARG; break; }
      t.C = s.K;
      t.H = out_extent(tin.H, s.R, s.stride, s.pad);
      t.W = out_extent(tin.W, s.S, s.stride, s.pad);
      const bool add = (op.epilogue & FUPR_FUSE_ADD) != 0;
      if (add != (op.res >= 0)) { err = FUPR_ERR_ARG; break; }
      if (add) {
        if (op.res > i) { err = FUPR_ERR_ARG; break; }
        const TensorInfo& tr = m->tensors[op.res];
        if (op.res_spatial_stride < 1 || op.res_c_offset < 0 || op.res_c_offset % 4 != 0) {
          err = FUPR_ERR_ARG; break;
        }
        if (scatter) {
          // the kept output filters add into tensor res in place; the output is that tensor
          if (g->dt == FUPR_F32) { err = FUPR_ERR_DTYPE; break; }
          if (op.res == 0 || i + 1 == g->n_ops || op.res_spatial_stride != 1 || op.res_c_offset != 0 ||
              op.res == op.in) {
            err = FUPR_ERR_ARG; break;
          }
          if (s.K > tr.C || tr.H != t.H || tr.W != t.W) { err = FUPR_ERR_SHAPE; break; }
          t.C = tr.C;
        } else if (op.res_c_offset + tr.C > s.K ||
                   (int64_t)(t.H - 1) * op.res_spatial_stride >= tr.H ||
                   (int64_t)(t.W - 1) * op.res_spatial_stride >= tr.W) {
          err = FUPR_ERR_SHAPE; break;
        }
      } else if (scatter) {
        err = FUPR_ERR_ARG; break;
      }
    } else if (op.kind == FUPR_OP_MAXPOOL) {
      const int k = op.conv.R;
      if (k <= 0 || op.conv.S != k || op.conv.stride <= 0 || op.conv.pad < 0 || op.conv.pad >= k) {
        err = FUPR_ERR_ARG; break;
      }
      if (op.res >= 0) { err = FUPR_ERR_ARG; break; }
      if (tin.H + 2 * op.conv.pad < k || tin.W + 2 * op.conv.pad < k) { err = FUPR_ERR_SHAPE; break; }
      t.C = tin.C;
      t.H = out_extent(tin.H, k, op.conv.stride, op.conv.pad);
      t.W = out_extent(tin.W, k, op.conv.stride, op.conv.pad);
    } else if (op.kind == FUPR_OP_AVGPOOL) {
      if (op.res >= 0) { err = FUPR_ERR_ARG; break; }
      t.C = tin.C;
      t.H = 1;
      t.W = 1;
    } else {
      err = FUPR_ERR_ARG; break;
    }
    t.cs = min_c_stride(t.C, g->dt);
    m->tensors[i + 1] = t;
  }
  if (err != FUPR_OK) {
    delete m;
    return err;
  }

  // Liveness and greedy buffer sharing.
  const int n = g->n_ops;
  for (int i = 0; i < n; ++i) {
    m->tensors[m->ops[i].in].last_use = i;
    if (m->ops[i].res >= 0) m->tensors[m->ops[i].res].last_use = i;
    if (m->ops[i].kind == FUPR_OP_CONV && (m->ops[i].epilogue & FUPR_FUSE_CAT))
      m->tensors[m->ops[i].in2].last_use = i;
  }
  // a tensor updated in place must have no reader after the update
  for (int i = 0; i < n; ++i) {
    if (!(m->ops[i].epilogue & FUPR_FUSE_SCATTER) || m->ops[i].kind != FUPR_OP_CONV) continue;
    if (m->tensors[m->ops[i].res].last_use != i) {
      delete m;
      return FUPR_ERR_ARG;
    }
  }
  // two operators that may run as one kernel: what the first reads must
  // outlive the second, whose output is written while the first still reads.
  // Which ones may does not depend on the switches of the moment: they can change
  // between here and a forward pass.
  m->pair_planned.assign(n, 0);
  {
    const WithoutTuning no_switches;
    for (int i = 0; i + 1 < n; ++i) m->pair_planned[i] = conv_conv_pair(m, (size_t)i) || stem_pool_pair(m, (size_t)i);
  }
  for (int i = 0; i + 1 < n; ++i) {
    if (!m->pair_planned[i]) continue;
    TensorInfo& tin = m->tensors[m->ops[i].in];
    tin.last_use = std::max(tin.last_use, i + 1);
    if (m->ops[i].res >= 0) {
      TensorInfo& tr = m->tensors[m->ops[i].res];
      tr.last_use = std::max(tr.last_use, i + 1);
    }
    if (m->ops[i].epilogue & FUPR_FUSE_CAT) {
      TensorInfo& t2 = m->tensors[m->ops[i].in2];
      t2.last_use = std::max(t2.last_use, i + 1);
    }
  }
  std::vector<int> holder;  // buffer -> tensor id it holds, -1 = free
  for (int i = 0; i < n; ++i) {
    const int tid = i + 1;
    TensorInfo& t = m->tensors[tid];
    if (tid == n) {
      t.buffer = -2;
    } else if (m->ops[i].kind == FUPR_OP_CONV && (m->ops[i].epilogue & FUPR_FUSE_SCATTER)) {
      // the operator's output is the tensor it updated: same buffer, new holder
      t.buffer = m->tensors[m->ops[i].res].buffer;
      holder[t.buffer] = tid;
    } else {
      const size_t need = (size_t)t.H * t.W * t.cs;
      int pick = -1;
      for (size_t b = 0; b < holder.size(); ++b) {
        if (holder[b] >= 0) continue;
        // prefer the free buffer whose size is closest to what is needed
        if (pick < 0) pick = (int)b;
        else {
          const size_t cur = m->buffer_elems[pick], cand = m->buffer_elems[b];
          const size_t dc = cur > need ? cur - need : need - cur;
          const size_t dn = cand > need ? cand - need : need - cand;
          if (dn < dc) pick = (int)b;
        }
      }
      if (pick < 0) {
        holder.push_back(-1);
        m->buffer_elems.push_back(0);
        pick = (int)holder.size() - 1;
      }
      holder[pick] = tid;
      m->buffer_elems[pick] = std::max(m->buffer_elems[pick], need);
      t.buffer = pick;
    }
    // tensors whose last reader is this operator become free afterwards
    for (size_t b = 0; b < holder.size(); ++b) {
      const int h = holder[b];
      if (h >= 0 && h != tid && m->tensors[h].last_use <= i) holder[b] = -1;
    }
  }
  plan_resident(m);
  const WithoutTuning no_switches;
  find_blocks(m);
  for (int schedule : {FUPR_SCHEDULE_AUTO, FUPR_SCHEDULE_PER_LAYER})
    m->launches[schedule] = list_launches(m, schedule);
  *out = m;
  return FUPR_OK;
}

extern "C" fupr_status fupr_model_set_schedule(fupr_model* m, int32_t schedule) {
  if (!m) return FUPR_ERR_NULL;
  if (schedule != FUPR_SCHEDULE_AUTO && schedule != FUPR_SCHEDULE_PER_LAYER) return FUPR_ERR_ARG;
  m->schedule = schedule;
  return FUPR_OK;
}

extern "C" fupr_status fupr_model_fuse_blocks(fupr_model* m, int32_t on) {
  if (!m) return FUPR_ERR_NULL;
  if (on != 0 && on != 1) return FUPR_ERR_ARG;
  m->blocks = on == 1;
  return FUPR_OK;
}

extern "C" size_t fupr_model_table_bytes(const fupr_model* m) {
  if (!m || !m->resident_ok) return 0;
  return resident_layer_bytes(m) + resident_table_bytes(m) + resident_rows_bytes(m);
}

extern "C" fupr_status fupr_model_table_write(const fupr_model* m, const void* dev_table,
                                              void* host_out) {
  if (!m || !dev_table || !host_out) return FUPR_ERR_NULL;
  if (!m->resident_ok) return FUPR_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(dev_table) & 255u) != 0) return FUPR_ERR_ALIGN;
  const size_t n = m->res_layers.size();
  const size_t layer_bytes = resident_layer_bytes(m);
  const char* base = reinterpret_cast<const char*>(dev_table);
  std::vector<ResLayer> layers = m->res_layers;
  for (size_t i = 0; i < n; ++i)
    layers[i].table = base + layer_bytes + m->res_table_at[i] * sizeof(int32_t);
  for (size_t i = 0; i + 1 < n; ++i) {
    layers[i].next_packed = layers[i + 1].packed;
    layers[i].next_table = layers[i + 1].table;
    layers[i].next_blob_units = layers[i + 1].blob_units;
    layers[i].next_tab_units = layers[i + 1].tab_units;
    layers[i].next_w_off = layers[i + 1].w_off;
    layers[i].next_tab_off = layers[i + 1].tab_off;
  }
  char* out = reinterpret_cast<char*>(host_out);
  std::fill(out, out + layer_bytes + resident_table_bytes(m) + resident_rows_bytes(m), 0);
  std::vector<ResRow> rows = m->res_rows;
  for (size_t i = 0; i + 1 < rows.size(); ++i) {
    rows[i].next_packed = layers[i].next_packed;
    rows[i].next_table = layers[i].next_table;
    rows[i].next_blob_units = layers[i].next_blob_units;
    rows[i].next_tab_units = layers[i].next_tab_units;
    rows[i].next_w_off = layers[i].next_w_off;
    rows[i].next_tab_off = layers[i].next_tab_off;
  }
  std::copy(reinterpret_cast<const char*>(rows.data()), reinterpret_cast<const char*>(rows.data() + rows.size()),
            out + layer_bytes + resident_table_bytes(m));
  std::copy(reinterpret_cast<const char*>(layers.data()),
            reinterpret_cast<const char*>(layers.data()) + n * sizeof(ResLayer), out);
  std::copy(reinterpret_cast<const char*>(m->res_tables.data()),
            reinterpret_cast<const char*>(m->res_tables.data()) + m->res_tables.size() * sizeof(int32_t),
            out + layer_bytes);
  return FUPR_OK;
}

extern "C" fupr_status fupr_model_set_table(fupr_model* m, const void* dev_table) {
  if (!m) return FUPR_ERR_NULL;
  if (dev_table && !m->resident_ok) return FUPR_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(dev_table) & 255u) != 0) return FUPR_ERR_ALIGN;
  m->res_dev = dev_table;
  return FUPR_OK;
}

extern "C" fupr_status fupr_model_set_side_streams(fupr_model* m, int32_t n, void* const* streams) {
  if (!m || (n > 0 && !streams)) return FUPR_ERR_NULL;
  if (n < 0 || n > kMaxSplit - 1) return FUPR_ERR_ARG;
  for (int k = 0; k < n; ++k)
    if (!streams[k]) return FUPR_ERR_NULL;   // the default stream cannot be forked into a capture
  std::lock_guard<std::mutex> lock(m->side_mutex);
  release_side(m);
  if (n == 0) return FUPR_OK;
  bool ok = hipEventCreateWithFlags(&m->fork_event, hipEventDisableTiming) == hipSuccess;
  for (int k = 0; ok && k < n; ++k)
    ok = hipEventCreateWithFlags(&m->join_event[k], hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    release_side(m);
    return FUPR_ERR_LAUNCH;
  }
  for (int k = 0; k < n; ++k) m->side_stream[k] = reinterpret_cast<hipStream_t>(streams[k]);
  m->n_side = n;
  return FUPR_OK;
}

extern "C" void fupr_model_destroy(fupr_model* m) {
  if (!m) return;
  release_side(m);
  delete m;
}

extern "C" int32_t fupr_model_num_ops(const fupr_model* m) { return m ? (int32_t)m->ops.size() : 0; }

extern "C" size_t fupr_model_workspace_bytes(const fupr_model* m, int32_t batch) {
  if (!m || batch <= 0) return 0;
  size_t total = 0;
  for (size_t e : m->buffer_elems) total += round_up_sz(e * (size_t)batch * elem_size(m->dt), 256);
  return std::max<size_t>(total, 256);
}

extern "C" fupr_status fupr_model_output_shape(const fupr_model* m, int32_t batch,
                                               fupr_tensor* out) {
  if (!m || !out) return FUPR_ERR_NULL;
  if (batch <= 0) return FUPR_ERR_SHAPE;
  const TensorInfo& t = m->tensors.back();
  out->N = batch;
  out->H = t.H;
  out->W = t.W;
  out->C = t.C;
  out->c_stride = t.cs;
  out->dt = m->dt;
  out->ptr = nullptr;
  return FUPR_OK;
}

namespace {

// The one-kernel schedule applies when the plan exists, the caller has not
// asked for per-layer kernels, and the caller's tensors have the strides the
// plan assumed.
bool use_resident(const fupr_model* m, const fupr_tensor* input, const fupr_tensor* output) {
  if (!m->resident_ok || !m->res_dev || m->schedule != FUPR_SCHEDULE_AUTO) return false;
  if (input->c_stride != m->tensors.front().cs) return false;
  const fupr_op_desc& last = m->ops.back();
  const int limit = last.kind == FUPR_OP_CONV ? round_up(last.conv.K, 16) : m->tensors[last.in].cs;
  return output->c_stride <= limit;
}

// Operator i is a 16-bit 7 x 7 stem convolution with ReLU whose only reader is
// the 3 x 3 max-pool right behind it: the two run as one kernel.
bool stem_pool_pair(const fupr_model* m, size_t i) {
  if (i + 1 >= m->ops.size()) return false;
  const fupr_op_desc& c = m->ops[i];
  const fupr_op_desc& q = m->ops[i + 1];
  if (c.kind != FUPR_OP_CONV || c.res >= 0 || c.epilogue != FUPR_FUSE_RELU) return false;
  if (q.kind != FUPR_OP_MAXPOOL || q.in != (int)i + 1) return false;
  if (m->tensors[i + 1].last_use != (int)i + 1) return false;
  const TensorInfo& tin = m->tensors[c.in];
  return stem_pool_applies(c.conv, m->dt, 1, tin.H, tin.W, tin.cs, m->tensors[i + 2].cs, q.conv.R,
                           q.conv.stride, q.conv.pad);
}

// First channel of y that the operator's shortcut adds to; -1: it has none.
int shortcut_offset(const fupr_op_desc& op) { return op.res >= 0 ? op.res_c_offset : -1; }

// Operator i is a 1 x 1 convolution whose whole output tile a wave holds, and
// operator i + 1 a 1 x 1 convolution of exactly that tensor (a bottleneck
// block's last convolution and the next block's first): one kernel computes
// both, the second from the first one's registers.
bool conv_conv_pair(const fupr_model* m, size_t i) {
  if (i + 1 >= m->ops.size()) return false;
  const fupr_op_desc& a = m->ops[i];
  const fupr_op_desc& b = m->ops[i + 1];
  if (a.kind != FUPR_OP_CONV || b.kind != FUPR_OP_CONV) return false;
  if ((a.epilogue | b.epilogue) & FUPR_FUSE_SCATTER) return false;
  if (b.epilogue & FUPR_FUSE_CAT) return false;
  if ((a.epilogue & FUPR_FUSE_CAT) && a.res >= 0) return false;
  if (b.in != (int)i + 1 || b.res >= 0) return false;
  const TensorInfo& tin = m->tensors[a.in];
  return conv_pair_fusable(a.conv, b.conv, m->dt, 1, tin.H, tin.W, shortcut_offset(a));
}

// Operators i and i + 1 are one launch under the switches of the moment: planned as one, and not refused now.
bool runs_as_pair(const fupr_model* m, size_t i) {
  return m->pair_planned[i] && (stem_pool_pair(m, i) || conv_conv_pair(m, i));
}

// Tensor t is read by one operator, as its input, and by nobody else.
bool read_once(const fupr_model* m, size_t t) {
  int readers = 0;
  for (const fupr_op_desc& o : m->ops) {
    const bool second = o.kind == FUPR_OP_CONV && (o.epilogue & FUPR_FUSE_CAT);
    readers += (o.in == (int)t) + (o.res == (int)t) + (second && o.in2 == (int)t);
  }
  return readers == 1;
}

// The bottleneck block that starts with operator i: a 3 x 3 convolution, the 1 x 1 convolution of its output
// that ends a bottleneck block, and, if the next operator is one, the 1 x 1 convolution of that
// output.  Returns its operators, 0 if there is none.
int bottleneck_at(const fupr_model* m, size_t i, BottleneckArgs* out) {
  const size_t n = m->ops.size();
  if (i + 2 >= n) return 0;            // (the network's output has strides of the caller's choice)
  const fupr_op_desc &a = m->ops[i], &b = m->ops[i + 1];
  if (a.kind != FUPR_OP_CONV || b.kind != FUPR_OP_CONV) return 0;
  if (a.in == 0 || a.res >= 0 || (a.epilogue & ~uint32_t(FUPR_FUSE_RELU)) || b.in != (int)i + 1) return 0;
  if (b.epilogue & FUPR_FUSE_SCATTER) return 0;
  BottleneckArgs g{};
  g.dt = m->dt;
  g.s1 = a.conv;
  g.s2 = b.conv;
  const TensorInfo &tx = m->tensors[a.in], &ty = m->tensors[i + 2];
  if (!read_once(m, i + 1)) return 0;
  g.H = tx.H; g.W = tx.W; g.xcs = tx.cs;
  if (b.epilogue & FUPR_FUSE_CAT) {
    if (b.res >= 0 || b.in2 == 0) return 0;
    const TensorInfo& t2 = m->tensors[b.in2];
    g.two = true;
    g.H2 = t2.H; g.W2 = t2.W; g.x2cs = t2.cs; g.stride2 = b.in2_spatial_stride;
  }
  if (b.res >= 0) {
    const TensorInfo& tr = m->tensors[b.res];
    if (b.res == 0 || b.res_spatial_stride != 1 || b.res_c_offset != 0 || tr.H != ty.H || tr.W != ty.W ||
        tr.C != ty.C)
      return 0;
    g.add = true;
  }
  g.relu1 = (a.epilogue & FUPR_FUSE_RELU) != 0;
  g.relu2 = (b.epilogue & FUPR_FUSE_RELU) != 0;
  g.ycs = ty.cs;
  int count = 2;
  if (i + 3 < n && m->ops[i + 2].kind == FUPR_OP_CONV) {
    const fupr_op_desc& c = m->ops[i + 2];
    if (c.in == (int)i + 2 && c.res < 0 && !(c.epilogue & ~uint32_t(FUPR_FUSE_RELU))) {
      BottleneckArgs third = g;
      third.third = true;
      third.s3 = c.conv;
      third.relu3 = (c.epilogue & FUPR_FUSE_RELU) != 0;
      third.hcs = m->tensors[i + 3].cs;
      if (bottleneck_applies(third)) {
        g = third;
        count = 3;
      }
    }
  }
  if (count == 2 && !bottleneck_applies(g)) return 0;
  *out = g;
  return count;
}

// The basic block that starts with operator i: two 3 x 3 convolutions, the second of the first one's
// output.  Returns its operators, 0 if there is none.
int basic_block_at(const fupr_model* m, size_t i, BasicBlockArgs* out) {
  const size_t n = m->ops.size();
  if (i + 1 >= n) return 0;
  const fupr_op_desc &a = m->ops[i], &b = m->ops[i + 1];
  if (a.kind != FUPR_OP_CONV || b.kind != FUPR_OP_CONV) return 0;
  if (a.res >= 0 || (a.epilogue & ~uint32_t(FUPR_FUSE_RELU)) || b.in != (int)i + 1 || b.res == (int)i + 1) return 0;
  if (b.epilogue & ~uint32_t(FUPR_FUSE_RELU | FUPR_FUSE_ADD)) return 0;
  if (!read_once(m, i + 1)) return 0;
  const TensorInfo& tx = m->tensors[a.in];
  BasicBlockArgs g{};
  g.dt = m->dt;
  g.s1 = a.conv;
  g.s2 = b.conv;
  g.H = tx.H;
  g.W = tx.W;
  g.add = b.res >= 0;
  g.alone = n == 2;
  if (!basic_block_applies(g)) return 0;
  *out = g;
  return 2;
}

// The plan with which a batch of N images runs the block that starts with operator i as one launch, -1: it does not.
int block_plan(const fupr_model* m, size_t i, int N) {
  const fupr_model::Block& b = m->block_args[i];
  if (b.kind == kBottleneck) return bottleneck_plan(b.bottleneck, N);
  if (b.kind != kBasic) return -1;
  // 32-bit byte offsets into every tensor
  for (int t : {m->ops[i].in, (int)i + 2, std::max(m->ops[i + 1].res, 0)}) {
    const TensorInfo& ti = m->tensors[t];
    if ((int64_t)N * ti.H * ti.W * ti.cs * (int64_t)elem_size(m->dt) >= (int64_t(1) << 31)) return -1;
  }
  return basic_block_plan(b.basic, N);
}

void find_blocks(fupr_model* m) {
  const int n = (int)m->ops.size();
  m->block_args.assign(n, fupr_model::Block{});
  for (int i = 0; i < n; ++i) {
    fupr_model::Block& b = m->block_args[i];
    if ((b.count = bottleneck_at(m, (size_t)i, &b.bottleneck)) > 0) {
      b.kind = kBottleneck;
      b.bottleneck.pair = m->pair_planned[i + 1] != 0;
    } else if ((b.count = basic_block_at(m, (size_t)i, &b.basic)) > 0) {
      b.kind = kBasic;
    }
  }
}

// Places the tensors anew in the buffers that the workspace has, for a batch of N images whose wanted
// blocks run as one launch each; blocks for which there is no room do not.  Empty if there is no block.
std::shared_ptr<fupr_model::Placement> place_blocks(const fupr_model* m, int N) {
  const int n = (int)m->ops.size();
  auto out = std::make_shared<fupr_model::Placement>();
  std::vector<char> chosen(n, 0);          // operators of the block that starts there
  std::vector<int> plan(n, -1);
  bool any = false;
  for (int i = 0; i < n; i += chosen[i] ? chosen[i] : 1)
    if ((plan[i] = block_plan(m, (size_t)i, N)) >= 0) {
      chosen[i] = (char)m->block_args[i].count;
      any = true;
    }
  auto reads = [&](int i, auto&& fn) {
    const fupr_op_desc& op = m->ops[i];
    fn(op.in);
    if (op.res >= 0) fn(op.res);
    if (op.kind == FUPR_OP_CONV && (op.epilogue & FUPR_FUSE_CAT)) fn(op.in2);
  };
  while (any) {
    // the launches, and the last operator that reads each tensor
    std::vector<int> last(n + 1, -1);
    std::vector<char> hidden(n + 1, 0);    // tensors that stay inside a launch
    out->launches.clear();
    for (int i = 0; i < n;) {
      Launch l{i, 1};
      if (chosen[i]) {
        l = Launch{i, chosen[i], m->block_args[i].kind, plan[i]};
        // (a block on the caller's own tensors can turn out to be two launches: their sizes and places
        // are known when it runs)
        hidden[i + 1] = m->ops[i].in != 0 && m->ops[i + 1].res != 0 && i + 2 != n;
      } else if (i + 1 < n && !chosen[i + 1] && runs_as_pair(m, (size_t)i)) {
        l.count = 2;
      }
      const bool together = l.block || m->pair_planned[i];
      for (int k = 0; k < l.count; ++k)
        reads(i + k, [&](int t) { last[t] = std::max(last[t], together && t <= i ? i + l.count - 1 : i + k); });
      out->launches.push_back(l);
      i += l.count;
    }
    // the smallest free buffer that holds a tensor first, the others where that leads nowhere
    out->buffer.assign(n + 1, -3);
    out->buffer[0] = -1;
    int failed = 0, tries = 20000;
    std::function<bool(int, const std::vector<int>&)> place = [&](int i, const std::vector<int>& held) {
      if (i == n) return true;
      if (--tries < 0) return false;
      failed = std::max(failed, i);
      const int tid = i + 1;
      const TensorInfo& t = m->tensors[tid];
      const size_t need = (size_t)t.H * t.W * t.cs;
      std::vector<int> choices;
      if (tid == n) {
        choices.push_back(-2);
      } else if (hidden[tid]) {
        choices.push_back(-3);
      } else if (m->ops[i].kind == FUPR_OP_CONV && (m->ops[i].epilogue & FUPR_FUSE_SCATTER)) {
        choices.push_back(out->buffer[m->ops[i].res]);
      } else {
        for (int b = 0; b < (int)held.size(); ++b)
          if (held[b] < 0 && m->buffer_elems[b] >= need) choices.push_back(b);
        std::stable_sort(choices.begin(), choices.end(),
                         [&](int x, int y) { return m->buffer_elems[x] < m->buffer_elems[y]; });
      }
      for (int b : choices) {
        std::vector<int> after = held;
        if (b >= 0) after[b] = tid;
        for (int& h : after)
          if (h >= 0 && h != tid && last[h] <= i) h = -1;
        out->buffer[tid] = b;
        if (place(i + 1, after)) return true;
      }
      return false;
    };
    if (place(0, std::vector<int>(m->buffer_elems.size(), -1))) return out;
    // no way past operator `failed`: the last block that starts at or before it keeps too much alive
    int drop = -1;
    any = false;
    for (int i = 0; i <= failed; ++i)
      if (chosen[i]) drop = i;
    if (drop >= 0) chosen[drop] = 0;
    for (int i = 0; drop >= 0 && i < n; ++i) any = any || chosen[i];
  }
  out->launches.clear();
  out->buffer.clear();
  return out;
}

std::vector<Launch> list_launches(const fupr_model* m, int schedule) {
  std::vector<Launch> v;
  for (size_t i = 0; i < m->ops.size();) {
    const int count = schedule == FUPR_SCHEDULE_AUTO && runs_as_pair(m, i) ? 2 : 1;
    v.push_back(Launch{(int)i, count});
    i += count;
  }
  return v;
}

// The list depends on the operators, the schedule and the tuning switches: the model keeps those
// without switches (3 us of host time for 52 operators otherwise, on every forward pass).
std::vector<Launch> launches_of(const fupr_model* m) {
  return tuning_any() ? list_launches(m, m->schedule) : m->launches[m->schedule];
}

// Of a pair of 1 x 1 convolutions whose tensors are small, two launches that fill the GPU are faster than
// one that walks it (nine images of 193 x 193, 49 x 49 pixels, 47 -> 256 -> 111 channels: 18 us in one,
// 12 in two; a launch more costs 1.7).
void adapt_pairs(const fupr_model* m, int N, std::vector<Launch>* list) {
  std::vector<Launch>& v = *list;
  for (size_t i = 0; i < v.size(); ++i) {
    const Launch l = v[i];
    if (l.count != 2 || l.block || m->ops[l.first + 1].kind != FUPR_OP_CONV) continue;
    const fupr_op_desc& op = m->ops[l.first];
    const TensorInfo& x = m->tensors[op.in];
    const bool cat = (op.epilogue & FUPR_FUSE_CAT) != 0;
    if (!conv_is_small(op.conv, m->dt, N, x.H, x.W, shortcut_offset(op), cat ? x.C : 0)) continue;
    v[i].count = 1;
    v.insert(v.begin() + ++i, Launch{l.first + 1, 1});
  }
  // A projection shortcut and its block's first convolution as one launch (with fupr_model_fuse_blocks: launch counts
  // are else as they were).  Neither's output may lie where the other reads or writes: what the first one writes has
  // to be read later, or its place would be free again.
  for (size_t i = 0; m->blocks && m->schedule == FUPR_SCHEDULE_AUTO && i + 1 < v.size(); ++i) {
    if (v[i].count != 1 || v[i + 1].count != 1 || v[i].block || v[i + 1].block) continue;
    const fupr_op_desc &a = m->ops[v[i].first], &b = m->ops[v[i + 1].first];
    if (a.kind == FUPR_OP_AVGPOOL && b.kind == FUPR_OP_CONV && b.in == v[i].first + 1 && b.res < 0 &&
        !(b.epilogue & ~uint32_t(FUPR_FUSE_RELU)) && m->tensors[b.in].last_use == v[i + 1].first &&
        mean_fc_applies(b.conv, m->dt, N, m->tensors[a.in].H, m->tensors[a.in].W)) {
      v[i] = Launch{v[i].first, 2, kMeanFc};
      v.erase(v.begin() + i + 1);
      continue;
    }
    if (a.kind != FUPR_OP_CONV || b.kind != FUPR_OP_CONV || a.in != b.in || a.res >= 0 || b.res >= 0) continue;
    if ((a.epilogue | b.epilogue) & ~uint32_t(FUPR_FUSE_RELU)) continue;
    if (m->tensors[v[i].first + 1].last_use <= v[i + 1].first) continue;
    const TensorInfo& x = m->tensors[a.in];
    if (!convs_beside(a.conv, b.conv, m->dt, N, x.H, x.W)) continue;
    v[i] = Launch{v[i].first, 2, kBeside};
    v.erase(v.begin() + i + 1);
  }
}

// What a batch of N images runs, with blocks as one launch; the placement's buffers are empty if there is none of these.
std::shared_ptr<const fupr_model::Placement> plan_batch(const fupr_model* m, int N) {
  auto p = place_blocks(m, N);
  if (p->buffer.empty()) p->launches = launches_of(m);
  adapt_pairs(m, N, &p->launches);
  return p;
}

// The same, kept by the model where no switch decides it too (2 us of host time for ResNet-18 otherwise, on every
// pass); null without fupr_model_fuse_blocks.
std::shared_ptr<const fupr_model::Placement> blocks_on(const fupr_model* m, int N) {
  if (!m->blocks || m->schedule != FUPR_SCHEDULE_AUTO) return nullptr;
  if (tuning_any()) return plan_batch(m, N);
  fupr_model* const keeper = const_cast<fupr_model*>(m);
  std::lock_guard<std::mutex> lock(keeper->placed_mutex);
  const auto known = m->placed.find(N);
  if (known != m->placed.end()) return known->second;
  const WithoutTuning no_switches;   // (one that another thread sets meanwhile has no place in what is kept)
  const auto p = plan_batch(m, N);
  if (m->placed.size() >= 256) keeper->placed.clear();
  keeper->placed.emplace(N, p);
  return p;
}

// The launches of a batch and the placement that they need, null for the model's own.  Looked up once
// for a pass: a launch is right only with the tensors where its list has them, and switches may change
// between two looks.
struct Scheduled {
  std::vector<Launch> launches;
  std::shared_ptr<const fupr_model::Placement> placed;
};

Scheduled scheduled_at(const fupr_model* m, int N) {
  Scheduled out;
  if (const auto kept = blocks_on(m, N)) {
    out.launches = kept->launches;
    if (!kept->buffer.empty()) out.placed = kept;
    return out;
  }
  out.launches = launches_of(m);
  adapt_pairs(m, N, &out.launches);
  return out;
}

// The plans of a batch's blocks for `count` of its images, per operator that starts one.
std::shared_ptr<const std::vector<int>> plans_of_part(const fupr_model* m, const fupr_model::Placement& placed, int count) {
  std::lock_guard<std::mutex> lock(placed.parts_mutex);
  std::shared_ptr<const std::vector<int>>& known = placed.parts[count];
  if (!known) {
    std::vector<int> plans(m->ops.size(), -1);
    for (const Launch& l : placed.launches) {
      const fupr_model::Block& b = m->block_args[l.first];
      if (l.block == kBottleneck) plans[l.first] = bottleneck_plan_part(b.bottleneck, l.plan, count);
      else if (l.block == kBasic) plans[l.first] = basic_block_plan_part(b.basic, l.plan, count);
    }
    known = std::make_shared<const std::vector<int>>(std::move(plans));
  }
  return known;
}

// Sub-batches of the per-operator schedule.  Two sub-batches side by side let one's
// memory-bound kernels run beside the other's arithmetic and fill launch gaps and tails.
// Measured on the ImageNet-size workloads (one / two / three / four sub-batches): the
// bottleneck network, whose 1 x 1 convolutions move 75 - 100 flops per byte, 3261 / 2988 /
// 3220 / 3320 us at 256 images and 922 / 888 / 960 / 1058 us at 64; the basic-block network
// (258 flops per byte, kernels that fill the compute units only at full batch) 417 / 448 us
// at 64.  So: two sub-batches from 192 images on, and from 64 images on for networks under
// 150 flops per byte; else one; never more than the caller has lent streams for.  The
// tuning switch split=<1..4> forces a count.
int split_count(const fupr_model* m, int N) {
  const int forced = std::min(std::max(tuning_int("split", 0), 0), kMaxSplit);
  int want = forced ? std::min(forced, std::max(N / 8, 1)) : (N >= 192 ? 2 : 1);
  if (!forced && want == 1 && N >= 64 && m->n_side > 0) {
    double flops = 0.0, bytes = 0.0;
    for (int32_t i = 0; i < (int32_t)m->ops.size(); ++i) {
      fupr_op_stats s;
      if (fupr_model_op_stats(m, N, i, &s) != FUPR_OK) return 1;
      flops += s.flops;
      bytes += s.bytes;
    }
    if (bytes > 0.0 && flops / bytes < 150.0) want = 2;
  }
  return std::min(want, m->n_side + 1);
}

void release_side(fupr_model* m) {
  if (m->fork_event) (void)hipEventDestroy(m->fork_event);
  m->fork_event = nullptr;
  for (int k = 0; k < kMaxSplit - 1; ++k) {
    if (m->join_event[k]) (void)hipEventDestroy(m->join_event[k]);
    m->join_event[k] = nullptr;
    m->side_stream[k] = nullptr;
  }
  m->n_side = 0;
}

// events: one before and one behind every launch, whose number is written to *n_launches.
fupr_status run(const fupr_model* m, const fupr_tensor* input, const fupr_tensor* output,
                void* workspace, size_t workspace_bytes, void* stream, hipEvent_t* events, size_t* n_launches) {
  if (!m || !input || !output || !workspace) return FUPR_ERR_NULL;
  if (!input->ptr || !output->ptr) return FUPR_ERR_NULL;
  if (input->dt != m->dt || output->dt != m->dt) return FUPR_ERR_DTYPE;
  const TensorInfo& t0 = m->tensors.front();
  const TensorInfo& tl = m->tensors.back();
  const int N = input->N;
  if (N <= 0 || input->C != t0.C || input->H != t0.H || input->W != t0.W) return FUPR_ERR_SHAPE;
  if (output->N != N || output->C != tl.C || output->H != tl.H || output->W != tl.W)
    return FUPR_ERR_SHAPE;
  if (input->c_stride < t0.C || input->c_stride % c_align(m->dt) != 0) return FUPR_ERR_ALIGN;
  if (output->c_stride < tl.C || output->c_stride % c_align(m->dt) != 0) return FUPR_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return FUPR_ERR_WORKSPACE;
  if (workspace_bytes < fupr_model_workspace_bytes(m, N)) return FUPR_ERR_WORKSPACE;
  for (const TensorInfo& t : m->tensors)
    if ((int64_t)N * t.H * t.W * t.cs >= (int64_t(1) << 31)) return FUPR_ERR_LIMIT;

  std::vector<char*> base(m->buffer_elems.size());
  size_t off = 0;
  for (size_t b = 0; b < base.size(); ++b) {
    base[b] = reinterpret_cast<char*>(workspace) + off;
    off += round_up_sz(m->buffer_elems[b] * (size_t)N * elem_size(m->dt), 256);
  }
  // images n0 .. n0 + count - 1 of a tensor; inside a workspace buffer every
  // sub-batch owns the slice its images would need at the buffer's largest tensor
  const size_t es = elem_size(m->dt);
  Scheduled schedule;
  const fupr_model::Placement* placed = nullptr;
  auto view = [&](int tid, int n0, int count) {
    const TensorInfo& t = m->tensors[tid];
    const int buffer = placed ? placed->buffer[tid] : t.buffer;
    fupr_tensor v;
    v.N = count; v.H = t.H; v.W = t.W; v.C = t.C; v.dt = m->dt;
    char* ptr;
    if (buffer == -1) {
      v.c_stride = input->c_stride;
      ptr = (char*)input->ptr + (size_t)n0 * t.H * t.W * input->c_stride * es;
    } else if (buffer == -2) {
      v.c_stride = output->c_stride;
      ptr = (char*)output->ptr + (size_t)n0 * t.H * t.W * output->c_stride * es;
    } else if (buffer < 0) {             // (a tensor that stays inside a launch)
      v.c_stride = t.cs;
      ptr = nullptr;
    } else {
      v.c_stride = t.cs;
      ptr = base[buffer] + (size_t)n0 * m->buffer_elems[buffer] * es;
    }
    v.ptr = ptr;
    return v;
  };

  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  if (events && hipEventRecord(events[0], hs) != hipSuccess) return FUPR_ERR_LAUNCH;
  if (use_resident(m, input, output)) {
    ResParams R = m->resident;
    R.layers = reinterpret_cast<const ResLayer*>(m->res_dev);
    R.rows = m->res_rows.empty() ? nullptr
                                 : reinterpret_cast<const ResRow*>(static_cast<const char*>(m->res_dev) + resident_layer_bytes(m) +
                                                                   resident_table_bytes(m));
    R.x = input->ptr;
    R.y = output->ptr;
    R.y_cs = output->c_stride;
    const fupr_status st = launch_resident(R, N, m->dt, stream);
    if (st != FUPR_OK) return st;
    if (events && hipEventRecord(events[1], hs) != hipSuccess) return FUPR_ERR_LAUNCH;
    if (n_launches) *n_launches = 1;
    return FUPR_OK;
  }
  schedule = scheduled_at(m, N);
  placed = schedule.placed.get();
  const std::vector<Launch>& launches = schedule.launches;
  if (n_launches) *n_launches = launches.size();
  auto residual = [&](const fupr_op_desc& op, int n0, int count) {
    fupr_residual r{};
    if (op.res >= 0) {
      r.t = view(op.res, n0, count);
      r.spatial_stride = op.res_spatial_stride;
      r.c_offset = op.res_c_offset;
    }
    return r;
  };
  // Operators i and i + 1 as one launch, after the checks that each of them gets by itself; as two
  // where tensors need more than 32-bit offsets or the output overlaps what the first reads (its own
  // launch reads it before the other's writes).
  auto basic_block = [&](size_t i, int plan, const fupr_tensor& x, const fupr_tensor& y, int n0, int count,
                         void* on) -> fupr_status {
    const fupr_op_desc &a = m->ops[i], &b = m->ops[i + 1];
    fupr_tensor mid = view((int)i + 1, n0, count);
    const bool hidden = mid.ptr == nullptr;
    // (a marker for the checks, that is never dereferenced)
    if (hidden) mid.ptr = reinterpret_cast<void*>(uintptr_t(256));
    const fupr_residual r = residual(b, n0, count);
    ConvArgs first, second;
    fupr_status st = conv_args(&a.conv, &x, a.packed, nullptr, a.epilogue, &mid, &first);
    if (st != FUPR_OK) return st;
    st = conv_args(&b.conv, &mid, b.packed, b.res >= 0 ? &r : nullptr, b.epilogue, &y, &second);
    if (st != FUPR_OK) return st;
    auto bytes = [&](const fupr_tensor& t) { return (size_t)t.N * t.H * t.W * t.c_stride * es; };
    const uintptr_t x0 = (uintptr_t)x.ptr, y0 = (uintptr_t)y.ptr;
    bool apart = x0 < y0 + bytes(y) && y0 < x0 + bytes(x);
    for (size_t size : {bytes(x), bytes(y), b.res >= 0 ? bytes(r.t) : 0}) apart = apart || size >= (size_t(1) << 31);
    if (hidden && apart) return FUPR_ERR_LIMIT;   // (block_plan takes no such sizes)
    if (!apart) return launch_basic_block(m->block_args[i].basic, first, second, plan, count, on);
    st = conv_fused_part(&a.conv, &x, nullptr, 0, a.packed, nullptr, a.epilogue, &mid, N, on);
    if (st != FUPR_OK) return st;
    return conv_fused_part(&b.conv, &mid, nullptr, 0, b.packed, b.res >= 0 ? &r : nullptr, b.epilogue, &y, N, on);
  };
  auto enqueue = [&](int n0, int count, void* on, bool record) -> fupr_status {
    const auto part = placed && count != N ? plans_of_part(m, *placed, count) : nullptr;
    for (size_t l = 0; l < launches.size(); ++l) {
      const size_t i = (size_t)launches[l].first;
      const fupr_op_desc& op = m->ops[i];
      const fupr_tensor x = view(op.in, n0, count);
      const fupr_tensor y = view((int)i + launches[l].count, n0, count);
      const int plan = part ? (*part)[i] : launches[l].plan;
      fupr_status st;
      if (launches[l].block == kMeanFc) {
        const fupr_op_desc& b = m->ops[i + 1];
        const fupr_tensor mean = view((int)i + 1, n0, count);
        st = mean_fc_part(&x, &mean, &b.conv, b.packed, b.epilogue, &y, N, on);
      } else if (launches[l].block == kBeside) {
        const fupr_op_desc& b = m->ops[i + 1];
        const fupr_tensor first = view((int)i + 1, n0, count);
        st = convs_beside_part(&op.conv, op.packed, op.epilogue, &first, &b.conv, b.packed, b.epilogue, &y, &x, N, on);
      } else if (launches[l].block == kBasic) {
        st = basic_block(i, plan, x, y, n0, count, on);
      } else if (launches[l].block) {
        BottleneckArgs g = m->block_args[i].bottleneck;
        const fupr_op_desc& b = m->ops[i + 1];
        g.x = x.ptr;
        g.packed1 = op.packed;
        g.packed2 = b.packed;
        g.y = view((int)i + 2, n0, count).ptr;
        if (g.two) g.x2 = view(b.in2, n0, count).ptr;
        if (g.add) g.res = view(b.res, n0, count).ptr;
        if (g.third) {
          g.packed3 = m->ops[i + 2].packed;
          g.h = y.ptr;
        }
        st = FUPR_OK;
        for (const void* blob : {g.packed1, g.packed2, g.packed3})
          if ((reinterpret_cast<uintptr_t>(blob) & 255u) != 0) st = FUPR_ERR_ALIGN;
        if (st == FUPR_OK) st = launch_bottleneck(g, plan, count, on);
      } else if (launches[l].count == 2 && m->ops[i + 1].kind == FUPR_OP_CONV) {
        const fupr_op_desc& second = m->ops[i + 1];
        const fupr_tensor mid = view((int)i + 1, n0, count);
        fupr_residual r;
        const bool add = op.res >= 0;
        if (add) {
          r.t = view(op.res, n0, count);
          r.spatial_stride = op.res_spatial_stride;
          r.c_offset = op.res_c_offset;
        }
        if (op.epilogue & FUPR_FUSE_CAT) {
          const fupr_tensor x2 = view(op.in2, n0, count);
          st = conv_cat_conv1x1_fused(&op.conv, &x, &x2, op.in2_spatial_stride, op.packed,
                                      op.epilogue & ~uint32_t(FUPR_FUSE_CAT), &mid, &second.conv,
                                      second.packed, second.epilogue, &y, on);
        } else {
          st = fupr_conv_conv1x1_fused(&op.conv, &x, op.packed, add ? &r : nullptr, op.epilogue, &mid,
                                       &second.conv, second.packed, second.epilogue, &y, on);
        }
      } else if (launches[l].count == 2) {
        const fupr_op_desc& pool = m->ops[i + 1];
        st = fupr_conv_maxpool_fused(&op.conv, &x, op.packed, pool.conv.R, pool.conv.stride,
                                     pool.conv.pad, &y, on);
      } else if (op.kind == FUPR_OP_CONV && (op.epilogue & FUPR_FUSE_SCATTER)) {
        st = conv_scatter_part(&op.conv, &x, op.packed, op.keep_idx, op.epilogue & FUPR_FUSE_RELU, &y, N, on);
      } else if (op.kind == FUPR_OP_CONV) {
        fupr_residual r;
        const bool add = op.res >= 0;
        if (add) {
          r.t = view(op.res, n0, count);
          r.spatial_stride = op.res_spatial_stride;
          r.c_offset = op.res_c_offset;
        }
        const bool cat = (op.epilogue & FUPR_FUSE_CAT) != 0;
        fupr_tensor x2;
        if (cat) x2 = view(op.in2, n0, count);
        st = conv_fused_part(&op.conv, &x, cat ? &x2 : nullptr, op.in2_spatial_stride, op.packed,
                             add ? &r : nullptr, op.epilogue & ~uint32_t(FUPR_FUSE_CAT), &y, N, on);
      } else if (op.kind == FUPR_OP_MAXPOOL) {
        st = fupr_maxpool(&x, op.conv.R, op.conv.stride, op.conv.pad, &y, on);
      } else {
        st = fupr_global_avgpool(&x, &y, on);
      }
      if (st != FUPR_OK) return st;
      if (record && hipEventRecord(events[l + 1], hs) != hipSuccess) return FUPR_ERR_LAUNCH;
    }
    return FUPR_OK;
  };
  // Timed runs and small batches stay on the caller's stream; otherwise the
  // batch is cut into sub-batches that run side by side (images are independent).
  const int split = events || m->schedule != FUPR_SCHEDULE_AUTO ? 1 : split_count(m, N);
  if (split <= 1) return enqueue(0, N, stream, events != nullptr);
  std::lock_guard<std::mutex> lock(const_cast<fupr_model*>(m)->side_mutex);
  if (hipEventRecord(m->fork_event, hs) != hipSuccess) return FUPR_ERR_LAUNCH;
  fupr_status result = FUPR_OK;
  int forked = 0;   // side streams that wait on the caller's stream and must be joined to it again
  for (int k = 1; k < split && result == FUPR_OK; ++k) {
    if (hipStreamWaitEvent(m->side_stream[k - 1], m->fork_event, 0) != hipSuccess) result = FUPR_ERR_LAUNCH;
    else ++forked;
  }
  for (int k = 0; k < split && result == FUPR_OK; ++k) {
    const int n0 = (int)((int64_t)N * k / split), n1 = (int)((int64_t)N * (k + 1) / split);
    result = enqueue(n0, n1 - n0, k == 0 ? stream : (void*)m->side_stream[k - 1], false);
  }
  // always join what was forked, so that the caller's stream (or capture) is whole again
  for (int k = 1; k <= forked; ++k) {
    if (hipEventRecord(m->join_event[k - 1], m->side_stream[k - 1]) != hipSuccess ||
        hipStreamWaitEvent(hs, m->join_event[k - 1], 0) != hipSuccess)
      result = FUPR_ERR_LAUNCH;
  }
  return result;
}

}  // namespace

extern "C" fupr_status fupr_forward(const fupr_model* m, const fupr_tensor* input,
                                    const fupr_tensor* output, void* workspace,
                                    size_t workspace_bytes, void* stream) {
  return run(m, input, output, workspace, workspace_bytes, stream, nullptr, nullptr);
}

extern "C" fupr_status fupr_forward_timed(const fupr_model* m, const fupr_tensor* input,
                                          const fupr_tensor* output, void* workspace,
                                          size_t workspace_bytes, void* stream, float* op_ms) {
  if (!m || !op_ms) return FUPR_ERR_NULL;
  const size_t n = m->ops.size();
  std::vector<hipEvent_t> ev(n + 1, nullptr);
  fupr_status st = FUPR_OK;
  for (size_t i = 0; i <= n; ++i)
    if (hipEventCreate(&ev[i]) != hipSuccess) { st = FUPR_ERR_LAUNCH; break; }
  size_t launches = 0;
  if (st == FUPR_OK) st = run(m, input, output, workspace, workspace_bytes, stream, ev.data(), &launches);
  if (st == FUPR_OK && hipStreamSynchronize(reinterpret_cast<hipStream_t>(stream)) != hipSuccess)
    st = FUPR_ERR_LAUNCH;
  if (st == FUPR_OK) {
    std::vector<float> ms(n, 0.0f);
    for (size_t i = 0; i < launches; ++i)
      if (hipEventElapsedTime(&ms[i], ev[i], ev[i + 1]) != hipSuccess) { st = FUPR_ERR_LAUNCH; break; }
    if (st == FUPR_OK) std::copy(ms.begin(), ms.end(), op_ms);
  }
  for (hipEvent_t e : ev)
    if (e) (void)hipEventDestroy(e);
  return st;
}

extern "C" fupr_status fupr_model_op_stats(const fupr_model* m, int32_t batch, int32_t op,
                                           fupr_op_stats* out) {
  if (!m || !out) return FUPR_ERR_NULL;
  if (batch <= 0 || op < 0 || op >= (int32_t)m->ops.size()) return FUPR_ERR_ARG;
  const fupr_op_desc& d = m->ops[op];
  const TensorInfo& ti = m->tensors[d.in];
  const TensorInfo& to = m->tensors[op + 1];
  const double es = (double)elem_size(m->dt);
  fupr_op_stats s{};
  s.first_op = op;
  s.n_ops = 1;
  s.M = (int64_t)batch * to.H * to.W;
  s.K = to.C;
  s.C = ti.C;
  const double in_b = es * batch * (double)ti.H * ti.W * ti.C;
  const double out_b = es * (double)s.M * to.C;
  if (d.kind == FUPR_OP_CONV) {
    s.R = d.conv.R; s.S = d.conv.S; s.stride = d.conv.stride;
    const double crs = (double)d.conv.C * d.conv.R * d.conv.S;
    s.flops = 2.0 * crs * d.conv.K * (double)s.M;
    double res_b = 0.0;
    if (d.res >= 0) res_b = es * (double)s.M * m->tensors[d.res].C;
    s.bytes = in_b + out_b + res_b + es * crs * d.conv.K + 4.0 * d.conv.K;
    if (d.epilogue & FUPR_FUSE_CAT) {
      // the second tensor's pixels that are read (one per output pixel); the zero
      // channels between the two tensors are neither read nor multiplied
      const double c2 = (double)m->tensors[d.in2].C;
      s.bytes += es * (double)s.M * c2 - es * ((double)d.conv.C - ti.C - c2) * d.conv.K;
      s.flops = 2.0 * (ti.C + c2) * d.conv.K * (double)s.M;
      s.C = ti.C + (int)c2;
    }
    const bool scatter = (d.epilogue & FUPR_FUSE_SCATTER) != 0;
    if (scatter)   // conv.K channels of the updated tensor read and written, and the index list
      s.bytes = in_b + 2.0 * es * (double)s.M * d.conv.K + es * crs * d.conv.K + 8.0 * d.conv.K;
    if (scatter) s.K = d.conv.K;
    s.kernel = conv_kernel_name(d.conv, m->dt, batch, ti.H, ti.W, scatter, shortcut_offset(d),
                                (d.epilogue & FUPR_FUSE_CAT) ? ti.C : 0);
  } else {
    s.R = s.S = d.kind == FUPR_OP_MAXPOOL ? d.conv.R : ti.H;
    s.stride = d.kind == FUPR_OP_MAXPOOL ? d.conv.stride : 1;
    s.flops = 0.0;
    s.bytes = in_b + out_b;
    s.kernel = d.kind == FUPR_OP_MAXPOOL ? "maxpool" : "global_avgpool";
  }
  *out = s;
  return FUPR_OK;
}

namespace {
// The one-kernel schedule will run (given tensors of the planned strides).
bool one_kernel(const fupr_model* m) {
  return m->resident_ok && m->res_dev && m->schedule == FUPR_SCHEDULE_AUTO;
}
}  // namespace

extern "C" int32_t fupr_model_num_launches(const fupr_model* m) {
  if (!m) return 0;
  return one_kernel(m) ? 1 : (int32_t)launches_of(m).size();
}

extern "C" int32_t fupr_model_num_launches_at(const fupr_model* m, int32_t batch) {
  if (!m || batch <= 0) return 0;
  return one_kernel(m) ? 1 : (int32_t)scheduled_at(m, batch).launches.size();
}

extern "C" fupr_status fupr_model_launch_stats(const fupr_model* m, int32_t batch, int32_t launch,
                                               fupr_op_stats* out) {
  if (!m || !out) return FUPR_ERR_NULL;
  if (batch <= 0 || launch < 0) return FUPR_ERR_ARG;
  if (one_kernel(m)) {
    if (launch > 0) return FUPR_ERR_ARG;
  } else {
    const std::vector<Launch> launches = scheduled_at(m, batch).launches;
    if ((size_t)launch >= launches.size()) return FUPR_ERR_ARG;
    const Launch l = launches[launch];
    fupr_status st = fupr_model_op_stats(m, batch, l.first, out);
    if (st != FUPR_OK || l.count == 1) return st;
    out->n_ops = l.count;
    if (l.block == kMeanFc) {
      // the mean is neither written nor read
      fupr_op_stats second;
      st = fupr_model_op_stats(m, batch, l.first + 1, &second);
      if (st != FUPR_OK) return st;
      out->flops += second.flops;
      out->bytes += second.bytes - 2.0 * (double)elem_size(m->dt) * batch * (double)m->tensors[l.first + 1].C;
      out->kernel = "mean_fc";
      return FUPR_OK;
    }
    if (l.block == kBeside) {
      // both outputs are written, the input is read once
      fupr_op_stats second;
      st = fupr_model_op_stats(m, batch, l.first + 1, &second);
      if (st != FUPR_OK) return st;
      const TensorInfo& x = m->tensors[m->ops[l.first].in];
      out->flops += second.flops;
      out->bytes += second.bytes - (double)elem_size(m->dt) * batch * (double)x.H * x.W * x.C;
      out->kernel = "conv_w+conv1x1p_w";
      return FUPR_OK;
    }
    if (l.block) {
      // the operators of a block in one kernel: the 3 x 3 convolution's output is not written, the
      // block's output is not read back
      const double es = (double)elem_size(m->dt);
      for (int k = 1; k < l.count; ++k) {
        fupr_op_stats o;
        st = fupr_model_op_stats(m, batch, l.first + k, &o);
        if (st != FUPR_OK) return st;
        const TensorInfo& t = m->tensors[l.first + k];
        out->flops += o.flops;
        out->bytes += o.bytes - (k == 1 ? 2.0 : 1.0) * es * batch * (double)t.H * t.W * t.C;
      }
      out->kernel = l.block == kBasic ? basic_block_name(l.plan) : bottleneck_name(l.plan);
      return FUPR_OK;
    }
    if (m->ops[l.first + 1].kind == FUPR_OP_CONV) {
      // two convolutions in one kernel: both outputs are written, the first one's
      // is not read back
      fupr_op_stats second;
      st = fupr_model_op_stats(m, batch, l.first + 1, &second);
      if (st != FUPR_OK) return st;
      const TensorInfo& mid = m->tensors[l.first + 1];
      out->flops += second.flops;
      out->bytes += second.bytes - (double)elem_size(m->dt) * batch * (double)mid.H * mid.W * mid.C;
      out->kernel = "conv1x1s_256f+conv1x1";
      return FUPR_OK;
    }
    // convolution + pool in one kernel: the convolution's flops; its input and
    // parameters read, the pool's output written
    fupr_op_stats pool;
    st = fupr_model_op_stats(m, batch, l.first + 1, &pool);
    if (st != FUPR_OK) return st;
    const double es = (double)elem_size(m->dt);
    const TensorInfo& mid = m->tensors[l.first + 1];
    const double mid_b = es * batch * (double)mid.H * mid.W * mid.C;
    out->bytes += pool.bytes - 2.0 * mid_b;
    out->kernel = "stem7x7_maxpool";
    return FUPR_OK;
  }
  // one kernel: all flops; the image in, the result out, every parameter once
  const double es = (double)elem_size(m->dt);
  const TensorInfo& t0 = m->tensors.front();
  const TensorInfo& tl = m->tensors.back();
  fupr_op_stats s{};
  s.first_op = 0;
  s.n_ops = (int32_t)m->ops.size();
  s.M = batch;
  s.C = t0.C;
  s.K = tl.C;
  s.R = t0.H;
  s.S = t0.W;
  s.stride = 1;
  s.bytes = es * batch * ((double)t0.C * t0.H * t0.W + (double)tl.C * tl.H * tl.W);
  for (size_t i = 0; i < m->ops.size(); ++i) {
    fupr_op_stats o;
    const fupr_status st = fupr_model_op_stats(m, batch, (int32_t)i, &o);
    if (st != FUPR_OK) return st;
    s.flops += o.flops;
    const fupr_op_desc& d = m->ops[i];
    if (d.kind == FUPR_OP_CONV)
      s.bytes += es * (double)d.conv.C * d.conv.R * d.conv.S * d.conv.K + 4.0 * d.conv.K;
  }
  s.kernel = m->res_rows.empty() ? "resident_network_taps" : "resident_network";
  *out = s;
  return FUPR_OK;
}

extern "C" fupr_status fupr_graph_create(const fupr_model* m, const fupr_tensor* input,
                                         const fupr_tensor* output, void* workspace,
                                         size_t workspace_bytes, void* stream, fupr_graph** out) {
  if (!out) return FUPR_ERR_NULL;
  if (!stream) return FUPR_ERR_ARG;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  fupr_graph* g = new (std::nothrow) fupr_graph;
  if (!g) return FUPR_ERR_ARG;
  if (hipStreamBeginCapture(hs, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    delete g;
    return FUPR_ERR_LAUNCH;
  }
  const fupr_status st = run(m, input, output, workspace, workspace_bytes, stream, nullptr, nullptr);
  const hipError_t e = hipStreamEndCapture(hs, &g->graph);
  if (st != FUPR_OK || e != hipSuccess || !g->graph) {
    if (g->graph) (void)hipGraphDestroy(g->graph);
    delete g;
    return st != FUPR_OK ? st : FUPR_ERR_LAUNCH;
  }
  if (hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0) != hipSuccess) {
    (void)hipGraphDestroy(g->graph);
    delete g;
    return FUPR_ERR_LAUNCH;
  }
  *out = g;
  return FUPR_OK;
}

extern "C" fupr_status fupr_graph_launch(const fupr_graph* g, void* stream) {
  if (!g || !g->exec) return FUPR_ERR_NULL;
  return hipGraphLaunch(g->exec, reinterpret_cast<hipStream_t>(stream)) == hipSuccess
             ? FUPR_OK
             : FUPR_ERR_LAUNCH;
}

extern "C" void fupr_graph_destroy(fupr_graph* g) {
  if (!g) return;
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  delete g;
}
