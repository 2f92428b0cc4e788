// Host-side internals shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "../../include/gx.h"
#include "gx_device.hpp"

namespace gx {

// Makes `device` the calling thread's current one while it lives: for calls
// that allocate memory or launch on the null stream for an object that may
// belong to another device than the current one.
class DeviceGuard {
 public:
  explicit DeviceGuard(int device) {
    ok_ = hipGetDevice(&before_) == hipSuccess;
    if (ok_ && before_ != device) switched_ = ok_ = hipSetDevice(device) == hipSuccess;
  }
  ~DeviceGuard() {
    if (switched_) (void)hipSetDevice(before_);
  }
  DeviceGuard(const DeviceGuard&) = delete;
  DeviceGuard& operator=(const DeviceGuard&) = delete;
  bool ok() const { return ok_; }

 private:
  int before_ = -1;
  bool ok_ = false, switched_ = false;
};

// Device workspace of the sorted lists (see gx_sort.hip); grow-only, freed
// with its owner.
struct SortSpace {
  uint32_t* words = nullptr;
  uint64_t cap = 0;
  SortSpace() = default;
  SortSpace(const SortSpace&) = delete;
  SortSpace& operator=(const SortSpace&) = delete;
  ~SortSpace();
  bool reserve(uint64_t n);  // room for lists of n records
};

}  // namespace gx

// Device buffers of the exploration driver, owned by a table and reused by
// every exploration into it (grow-only).
struct gx_explore_buffers {
  gx::SortSpace sort;
  uint32_t* img = nullptr;  // network image (in the control block, see ctr)
  uint32_t* img_global = nullptr;  // an image too large for LDS (own allocation)
  uint64_t img_global_cap = 0;     // words
  uint32_t* f[2] = {nullptr, nullptr};
  uint64_t f_cap[2] = {0, 0};  // states
  uint32_t* dead = nullptr;
  uint64_t dead_cap = 0;  // states
  uint32_t* log = nullptr;   // the first levels' states, as one workgroup found them
  uint64_t log_cap = 0;      // states
  // control block (device) and its pinned host mirror: the level counters
  // (one cache line each) and what the device leaves for the host (LevelCtl),
  // then the initial state's slot and the network image; one copy up per
  // exploration, the counters' part copied back by the last launch of a string
  // of levels (or read back where the host launches a level's slices)
  uint64_t* ctr = nullptr;
  uint64_t* ctr_host = nullptr;
  uint64_t* report = nullptr;  // host memory that level launches write (level_report)
  uint8_t* status = nullptr;
  uint32_t* key = nullptr;  // the initial state, 4 words (in the control block)
  // safety monitor: bad-state bitmask, violating states
  uint32_t* mon = nullptr;
  uint64_t mon_cap = 0;      // words
  uint32_t* viol = nullptr;
  uint64_t viol_cap = 0;     // states
};

struct gx_table {
  int device = 0;
  uint32_t w = 0;  // words per state
  uint32_t S = 0;  // slot words
  uint32_t B = 0;  // bucket words
  uint32_t G = 0;  // subgroup width
  uint32_t U = 1;  // keys in flight per subgroup
  uint32_t H = 8;  // hash functions
  uint64_t seed = 0;
  uint64_t n_buckets = 0;
  uint32_t* words = nullptr;     // n_buckets * B
  uint64_t* hc = nullptr;        // 2*H hash constants
  uint64_t* counters = nullptr;  // ctr_slots sets of gx::kNumCounters
  uint32_t ctr_slots = 1;
  uint64_t a0 = 0, c0 = 0;
  // something was inserted since creation or the last clear: gx_explore, whose
  // first levels place states assuming an empty table, refuses the table
  bool holds_states = false;
  uint32_t explorations = 0;  // begun on the table (a number for each, never 0)
  gx_explore_buffers eb;

  gx::TableDev dev() const {
    gx::TableDev t;
    t.words = words;
    t.n_buckets = n_buckets;
    t.hc = hc;
    t.seed = seed;
    t.a0 = a0;
    t.c0 = c0;
    t.H = H;
    t.counters = counters;
    t.ctr_slots = ctr_slots;
    return t;
  }
};

namespace gx {

inline uint32_t slot_words(uint32_t w) { return w == 3 ? 4u : w; }

// A 4-lane subgroup holds at most 8 words of a bucket per lane, so it pairs
// with buckets of up to 32 words.  An autotuned value gives way to an
// explicit one: an explicit 4-lane subgroup caps an autotuned bucket at 32
// words, an explicit 64-word bucket turns an autotuned 4-lane subgroup into 8.
inline void fit_subgroup(uint32_t* B, uint32_t* G, bool B_given) {
  if (*G == 4 && *B > 32) {
    if (B_given) *G = 8;
    else *B = 32;
  }
}

struct FopArgs {
  TableDev t;
  const uint32_t* keys;
  uint32_t w;
  uint64_t n;
  uint8_t* status;
  uint64_t* n_new;
  uint32_t cus;  // compute units of the device
  hipStream_t stream;
};

// Find-or-put dispatch over (B, G, U) for slot width S (one translation unit
// per S).
template <int S>
hipError_t dispatch_b(uint32_t B, uint32_t G, uint32_t U, const FopArgs& a);
extern template hipError_t dispatch_b<1>(uint32_t, uint32_t, uint32_t, const FopArgs&);
extern template hipError_t dispatch_b<2>(uint32_t, uint32_t, uint32_t, const FopArgs&);
extern template hipError_t dispatch_b<4>(uint32_t, uint32_t, uint32_t, const FopArgs&);

// Launch the find-or-put kernel specialised for the table's (S, B, G, U).
hipError_t launch_find_or_put(const gx_table* t, const uint32_t* keys, uint64_t n,
                              uint8_t* status, uint64_t* n_new, hipStream_t stream);

// Fill n_words (a multiple of 4, 16-byte aligned) with value, stream-ordered
// (a kernel, never a memset node, so it may be captured in a graph).
hipError_t fill_words(uint32_t* p, uint64_t n_words, uint32_t value, int device,
                      hipStream_t stream);

// Lists of fewer records, and storage of fewer words, are sorted on the host:
// a few kernels and a read-back take longer.
constexpr uint64_t kSortMin = 2048;
constexpr uint64_t kGatherMin = 32768;

// The keys stored in n_slots slots of S words on the device: their number to
// *n, and the first `cap` of them, in any order, to out (nullable).
// Synchronous.
gx_status gather_keys(uint32_t S, const uint32_t* words, uint64_t n_slots, uint32_t* out,
                      uint64_t cap, SortSpace& ws, uint64_t* n, hipStream_t stream);
// The n (< 2^32) keys that gather_keys has just put into a, sorted
// lexicographically, w words each, to host memory.  b: as large as a; both
// are overwritten.  Synchronous.
gx_status sort_gathered(uint32_t S, uint32_t w, uint32_t* a, uint32_t* b, uint64_t n,
                        SortSpace& ws, uint32_t* host, hipStream_t stream);
// The same for n records of S words in a.
gx_status sort_records(uint32_t S, uint32_t w, uint32_t* a, uint32_t* b, uint64_t n, SortSpace& ws,
                       uint32_t* host, hipStream_t stream);

// The keys stored in total_words words of bucket storage (slots of S words,
// keys of w words) on the device, sorted lexicographically, w words each, by
// the host.  Waits for all device work.  *n_out receives the number of keys.
gx_status sorted_keys(const uint32_t* dev_words, uint64_t total_words, uint32_t S, uint32_t w,
                      std::vector<uint32_t>* out, uint64_t* n_out);
// The same into a malloc'd array (for gx_explore_result.states), sorted on
// the device in a and b (buffers of `room` records each) where they hold the
// keys, else by the host.
gx_status sorted_keys_malloc(const uint32_t* dev_words, uint64_t total_words, uint32_t S,
                             uint32_t w, uint32_t* a, uint32_t* b, uint64_t room, SortSpace& ws,
                             hipStream_t stream, uint32_t** out);

// LDS bytes one workgroup may use on the device (queried once per device).
size_t lds_per_workgroup(int device);

// Number of workgroups that keep every CU busy for a grid-stride kernel.
uint32_t resident_grid(int device, uint32_t per_cu);

}  // namespace gx
