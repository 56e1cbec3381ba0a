// Process-wide tuning switches: a small table of named text values.  Each entry
// starts from the environment variable FUPR_<NAME IN CAPITALS>, read once when
// the table is first used, and changes afterwards only through fupr_tuning_set.
#include "tuning.h"

#include <atomic>
#include <cctype>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "fupr.h"

namespace fupr {
namespace {

constexpr size_t kValueBytes = 128;

struct Switch {
  const char* name;
  bool set;
  char value[kValueBytes];
};

Switch g_switches[] = {
    {"patch_tile", false, {0}},      // index of the 3 x 3 patch kernel's tile
    {"pipe_tile", false, {0}},       // index of the pipelined 1 x 1 kernel's tile
    {"pipe_order", false, {0}},      // that kernel's tiles: 0 a contiguous range per workgroup, 1 per XCD
    {"stream_tile", false, {0}},     // index of the streaming 1 x 1 kernel's tile
    {"stream_blocks", false, {0}},   // workgroups per compute unit that kernel is compiled for (1, 2)
    {"conv_tile", false, {0}},       // name of the general kernel's tile
    {"window_tile", false, {0}},     // <index>x<waves on filters>x<waves on the reduction>
    {"conv_window", false, {0}},     // 0: layers skip the kernel with weights straight into registers
    {"conv_two", false, {0}},        // 0: two convolutions of one tensor are two launches
    {"two_tap", false, {0}},         // index of the 1 x 1 convolution's tile in such a launch
    {"mean_fc", false, {0}},         // 0: a global mean and the layer behind it are two launches
    {"conv_patch", false, {0}},      // 0: 3 x 3 layers skip the patch kernel
    {"conv1x1_stream", false, {0}},  // 0: 1 x 1 layers skip the streaming kernel
    {"conv1x1_pipe", false, {0}},    // 0: 1 x 1 layers skip the pipelined kernel
    {"conv1x1_fuse", false, {0}},    // 0: no pairs of 1 x 1 convolutions in one launch
    {"pair_filters", false, {0}},    // most filters of such a pair's second convolution (up to 128)
    {"bottleneck_fuse", false, {0}},      // 0: bottleneck blocks run as several launches
    {"bottleneck_tile", false, {0}},      // index of the bottleneck kernel's tile
    {"basic_fuse", false, {0}},      // 0: basic blocks run as two launches
    {"basic_tile", false, {0}},      // <rectangle>x<waves along the filters> of the kernel that runs them
    {"split", false, {0}},           // sub-batches of the per-operator schedule
    {"resident_rows", false, {0}},   // 0: the one-kernel schedule without its kernel of row layers
    {"res_item", false, {0}},        // work-item shapes of the one-kernel schedule
    {"debug", false, {0}},           // non-empty: planner and HIP error text on stderr
};

std::mutex g_mutex;
std::once_flag g_env_once;
std::atomic<int> g_with_value{0};   // switches that have a value: launchers look at this first
thread_local int t_without = 0;     // WithoutTuning objects alive in this thread

void read_environment() {
  for (Switch& s : g_switches) {
    char var[64] = "FUPR_";
    size_t n = std::strlen(var);
    for (const char* c = s.name; *c && n + 1 < sizeof(var); ++c) var[n++] = (char)std::toupper((unsigned char)*c);
    var[n] = 0;
    const char* e = std::getenv(var);
    if (e && *e && std::strlen(e) < kValueBytes) {
      std::strcpy(s.value, e);
      s.set = true;
      g_with_value.fetch_add(1);
    }
  }
}

Switch* find(const char* name) {
  std::call_once(g_env_once, read_environment);
  for (Switch& s : g_switches)
    if (std::strcmp(s.name, name) == 0) return &s;
  return nullptr;
}

}  // namespace

WithoutTuning::WithoutTuning() { ++t_without; }
WithoutTuning::~WithoutTuning() { --t_without; }

bool tuning_any() {
  if (t_without > 0) return false;
  std::call_once(g_env_once, read_environment);
  return g_with_value.load(std::memory_order_acquire) != 0;
}

bool tuning_text(const char* name, char* out, size_t n) {
  if (!tuning_any()) return false;
  Switch* s = find(name);
  if (!s || n == 0) return false;
  std::lock_guard<std::mutex> lock(g_mutex);
  if (!s->set) return false;
  std::strncpy(out, s->value, n - 1);
  out[n - 1] = 0;
  return true;
}

int tuning_int(const char* name, int unset) {
  char buf[kValueBytes];
  return tuning_text(name, buf, sizeof(buf)) ? std::atoi(buf) : unset;
}

bool tuning_off(const char* name) {
  char buf[kValueBytes];
  return tuning_text(name, buf, sizeof(buf)) && buf[0] == '0';
}

}  // namespace fupr

extern "C" fupr_status fupr_tuning_set(const char* name, const char* value) {
  if (!name) return FUPR_ERR_NULL;
  fupr::Switch* s = fupr::find(name);
  if (!s) return FUPR_ERR_ARG;
  if (value && std::strlen(value) >= fupr::kValueBytes) return FUPR_ERR_ARG;
  std::lock_guard<std::mutex> lock(fupr::g_mutex);
  const bool set = value && *value;
  if (set) std::strcpy(s->value, value);
  fupr::g_with_value.fetch_add((set ? 1 : 0) - (s->set ? 1 : 0));
  s->set = set;
  return FUPR_OK;
}
