// Level-synchronous breadth-first exploration of the synchronous product of a
// network of LTSs (Sec. 3 of the paper), built on the bucketed find-or-put.
//
// A level is one launch of level_kernel: every wavefront walks its frontier
// states' transitions in the LDS-resident network image, puts the successors
// into the table 64 at a time and gathers the NEW ones for the next frontier.
// Levels whose successors fit the buffers in any case are strung together
// with no read-back between them; a level that might not fit is expanded in
// slices by the host, which grows the buffers.
// The paper's tool scans the hash table for states still to explore and keeps
// a per-block cache of new states (Sec. 3); here the next level is an explicit
// compacted frontier, so no scan of the table is needed.  With a safety
// monitor, every completed level is scanned once for states whose monitor
// process is in a bad state.
//
// The first levels of an exploration (all of a small one) are expanded on one
// workgroup by lds_levels_kernel, which decides NEW or SEEN from an LDS set of
// the states reached so far (the table holds nothing else yet) and puts them
// into the table at the end.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "gx_small_kernel.hpp"

namespace gx {
// instantiated in gx_explore_s1.hip, gx_explore_s2.hip and gx_explore_s4.hip
extern template hipError_t launch_level<1>(uint32_t, const LevelArgs&, bool, uint32_t, size_t,
                                             hipStream_t);
extern template uint32_t level_blocks_per_cu<1>(uint32_t, size_t);
extern template hipError_t launch_level<2>(uint32_t, const LevelArgs&, bool, uint32_t, size_t,
                                             hipStream_t);
extern template uint32_t level_blocks_per_cu<2>(uint32_t, size_t);
extern template hipError_t launch_level<4>(uint32_t, const LevelArgs&, bool, uint32_t, size_t,
                                             hipStream_t);
extern template uint32_t level_blocks_per_cu<4>(uint32_t, size_t);
extern template hipError_t launch_lds_levels<1>(uint32_t, SmallArgs, size_t, hipStream_t);
extern template hipError_t launch_lds_levels<2>(uint32_t, SmallArgs, size_t, hipStream_t);
extern template hipError_t launch_lds_levels<4>(uint32_t, SmallArgs, size_t, hipStream_t);
}  // namespace gx

namespace gx {

constexpr uint32_t kMaxSuccPerState = 1u << 20;
// Largest transition tables of any kernel: ones that exceed kImgMaxWords (the
// LDS budget) are read from global memory by the level kernel.
constexpr uint32_t kImgGlobalMaxWords = 1u << 26;

struct NetImage {
  std::vector<uint32_t> img;
  uint32_t words = 0;
  uint64_t table_words = 0;  // size of the transition tables, what the limits apply to
  std::vector<uint32_t> field;  // per process
  std::vector<uint32_t> initial;
  uint64_t max_succ = 0;  // transitions a state can have at most
  uint64_t max_out = 0;   // distinct successors formed for a state at most
};

namespace {

uint32_t field_bits(uint32_t n) {
  uint32_t b = 1;
  while (b < 32 && (uint64_t(1) << b) < n) ++b;
  return b;
}

gx_status compile_network(const gx_network* net, NetImage* out,
                          uint32_t max_words = kImgGlobalMaxWords) {
  if (!net || net->n_procs == 0 || !net->procs) return GX_EINVAL;
  if (net->n_rules && !net->rules) return GX_EINVAL;
  const uint32_t P = net->n_procs, R = net->n_rules, NL = net->n_labels;
  // packing plan
  std::vector<uint32_t> field(P);
  uint32_t word = 0, used = 0;
  for (uint32_t p = 0; p < P; ++p) {
    const gx_lts& l = net->procs[p];
    if (l.n_states == 0 || l.initial >= l.n_states) return GX_EINVAL;
    if (l.n_trans && (!l.src || !l.label || !l.dst)) return GX_EINVAL;
    const uint32_t b = field_bits(l.n_states);
    if (b > 31) return GX_EINVAL;
    if (used + b > 31) {
      ++word;
      used = 0;
    }
    field[p] = word | (used << 8) | (b << 16);
    used += b;
  }
  const uint32_t words = word + 1;
  if (words > 4) return GX_EINVAL;
  // which labels of each process are named by a rule at its position
  std::vector<std::vector<uint8_t>> governed(P, std::vector<uint8_t>(NL, 0));
  std::vector<std::vector<uint32_t>> parts(R);
  for (uint32_t r = 0; r < R; ++r) {
    for (uint32_t p = 0; p < P; ++p) {
      const int32_t a = net->rules[size_t(r) * P + p];
      if (a < -1 || a >= int32_t(NL)) return GX_EINVAL;
      if (a >= 0) {
        governed[p][a] = 1;
        parts[r].push_back(p);
      }
    }
    if (parts[r].empty()) return GX_EINVAL;
  }
  for (uint32_t p = 0; p < P; ++p) {
    const gx_lts& l = net->procs[p];
    for (uint32_t t = 0; t < l.n_trans; ++t)
      if (l.src[t] >= l.n_states || l.dst[t] >= l.n_states || l.label[t] >= NL) return GX_EINVAL;
  }

  std::vector<uint32_t> img(4 + 4 * (static_cast<size_t>(P) + R), 0);
  img[2] = slot_words(words);
  img[3] = words;
  // what the limits on a network's size count: a few words per process and
  // rule, an offset per local state and a word per transition of every
  // process and every rule participant
  uint64_t table_words = 4 + 2ull * P + R;
  for (uint32_t r = 0; r < R; ++r) table_words += 1 + 2ull * parts[r].size();
  // Lists of the targets selected by `keep` for process p (see the image's
  // layout): *max_deg receives the most transitions of a local state, *max_out
  // the most targets listed.  drop_self: targets equal to the source are only
  // counted.
  auto emit_csr = [&](uint32_t p, auto keep, bool drop_self, uint64_t* max_deg,
                      uint64_t* max_out) -> uint32_t {
    const gx_lts& l = net->procs[p];
    const uint32_t shift = (field[p] >> 8) & 0xFF;
    std::vector<uint32_t> start(static_cast<size_t>(l.n_states) + 1, 0);
    uint64_t n = 0;
    for (uint32_t t = 0; t < l.n_trans; ++t)
      if (keep(l.label[t])) {
        ++start[l.src[t] + 1];
        ++n;
      }
    table_words += l.n_states + 1ull + n;
    *max_deg = *max_out = 0;
    if (table_words > max_words || n == 0) return 0;
    for (uint32_t s = 0; s < l.n_states; ++s) {
      *max_deg = std::max<uint64_t>(*max_deg, start[s + 1]);
      start[s + 1] += start[s];
    }
    std::vector<uint32_t> dst(n), at(start.begin(), start.end() - 1);
    for (uint32_t t = 0; t < l.n_trans; ++t)
      if (keep(l.label[t])) dst[at[l.src[t]]++] = l.dst[t];
    const uint32_t off_at = static_cast<uint32_t>(img.size());
    img.resize(img.size() + l.n_states + 1);
    for (uint32_t s = 0; s < l.n_states; ++s) {
      const auto b = dst.begin() + start[s], e = dst.begin() + start[s + 1];
      std::sort(b, e);
      auto u = std::unique(b, e);
      if (drop_self) u = std::remove(b, u, s);
      const uint32_t listed = static_cast<uint32_t>(u - b), total = start[s + 1] - start[s];
      img[off_at + s] = static_cast<uint32_t>(img.size()) | (listed != total ? kListCounted : 0u);
      if (listed != total) img.push_back(total);
      for (auto d = b; d != u; ++d) img.push_back(*d << shift);
      *max_out = std::max<uint64_t>(*max_out, listed);
    }
    img[off_at + l.n_states] = static_cast<uint32_t>(img.size());
    return off_at;
  };
  uint64_t max_succ = 0, max_out = 0;
  uint32_t n_items = 0;
  auto item = [&]() { return 4 + 4 * static_cast<size_t>(n_items); };
  for (uint32_t p = 0; p < P && table_words <= max_words; ++p) {
    uint64_t md = 0, mo = 0;
    const uint32_t at = emit_csr(p, [&](uint32_t a) { return !governed[p][a]; }, true, &md, &mo);
    if (md == 0) continue;
    img[item() + 2] = field[p];
    img[item() + 3] = at;
    ++n_items;
    max_succ += md;
    max_out += mo;
  }
  for (uint32_t r = 0; r < R && table_words <= max_words; ++r) {
    const uint32_t np = static_cast<uint32_t>(parts[r].size());
    uint64_t prod = 1, prod_out = 1;
    std::vector<uint32_t> at(np, 0);
    for (uint32_t i = 0; i < np && table_words <= max_words; ++i) {
      const uint32_t want = static_cast<uint32_t>(net->rules[size_t(r) * P + parts[r][i]]);
      uint64_t md = 0, mo = 0;
      at[i] = emit_csr(parts[r][i], [&](uint32_t a) { return a == want; }, false, &md, &mo);
      prod = std::min<uint64_t>(prod * md, uint64_t(1) << 40);
      prod_out = std::min<uint64_t>(prod_out * mo, uint64_t(1) << 40);
    }
    if (prod == 0) continue;  // never enabled
    img[item() + 2] = field[parts[r][np - 1]];
    img[item() + 3] = at[np - 1];
    if (np == 2) {
      img[item()] = field[parts[r][0]];
      img[item() + 1] = at[0];
    } else if (np > 2) {
      img[item()] = kItemGeneral;
      img[item() + 1] = static_cast<uint32_t>(img.size());
      img.push_back(np - 1);
      for (uint32_t i = 0; i + 1 < np; ++i) {
        img.push_back(field[parts[r][i]]);
        img.push_back(at[i]);
      }
    }
    ++n_items;
    max_succ += prod;
    max_out += prod_out;
  }
  if (table_words > max_words) return GX_EINVAL;
  img[0] = n_items;
  if (max_succ > kMaxSuccPerState) return GX_EINVAL;
  out->img = std::move(img);
  out->words = words;
  out->table_words = table_words;
  out->field = std::move(field);
  out->initial.resize(P);
  for (uint32_t p = 0; p < P; ++p) out->initial[p] = net->procs[p].initial;
  out->max_succ = max_succ;
  out->max_out = max_out;
  return GX_OK;
}

void pack_host(const NetImage& ni, const uint32_t* local, uint32_t* out);

}  // namespace

gx_status compile_network_image(const gx_network* net, std::vector<uint32_t>* img,
                                uint32_t* words, std::vector<uint32_t>* packed_initial,
                                uint64_t* max_succ) {
  NetImage ni;
  // batches and the server keep every image in LDS
  const gx_status s = compile_network(net, &ni, kImgMaxWords);
  if (s != GX_OK) return s;
  packed_initial->assign(4, 0);
  pack_host(ni, ni.initial.data(), packed_initial->data());
  *img = std::move(ni.img);
  *words = ni.words;
  *max_succ = ni.max_succ;
  return GX_OK;
}

namespace {

void pack_host(const NetImage& ni, const uint32_t* local, uint32_t* out) {
  for (uint32_t k = 0; k < ni.words; ++k) out[k] = 0;
  for (size_t p = 0; p < ni.field.size(); ++p) {
    const uint32_t f = ni.field[p];
    out[f & 0xFF] |= local[p] << ((f >> 8) & 0xFF);
  }
}

}  // namespace

namespace {

// Safety monitor: the level just completed, states[0, n) of f[cur], searched
// for states whose monitor field (word | shift << 8 | width << 16) holds a
// local state marked in the bitmask `bad`.  They are counted in the kCtrViol
// counter and, below cap, copied to out (S words each); the first one ever
// leaves its level, plus one, in kCtrViolLevel.  With ctl (a string of levels,
// see LevelCtl) the level is the one that launch `link` has left, if it left
// one whose records fit; `stop` then ends the string at a violation.  One atomic add per
// workgroup and round that finds any.
struct ScanArgs {
  const uint32_t* f[2];
  uint64_t n;
  uint32_t cur;
  uint32_t field;
  const uint32_t* bad;
  uint32_t* out;
  uint64_t cap;
  uint64_t* ctr;
  uint64_t level;  // the level's number; in a string, its first level's
  LevelCtl* ctl;
  uint32_t link;
  uint32_t stop;
};

template <int S>
__global__ __launch_bounds__(256) void monitor_scan_kernel(ScanArgs a) {
  __shared__ uint32_t hits[4];
  __shared__ unsigned long long sh_base;
  uint64_t n = a.n, level = a.level;
  uint32_t cur = a.cur;
  LevelCtl::Entry* e = nullptr;
  if (a.ctl != nullptr) {
    e = &a.ctl->entry[(a.link & 1u) ^ 1u];
    if (e->scan != kScanHere) return;
    n = uniform64(e->n_in);
    cur = uniform32(static_cast<uint32_t>(e->cur));
    level = a.level + e->n_levels - 1;
  }
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  const uint32_t* states = a.f[cur];
  for (uint64_t base = static_cast<uint64_t>(blockIdx.x) * 256; base < n;
       base += static_cast<uint64_t>(gridDim.x) * 256) {
    const uint64_t i = base + threadIdx.x;
    uint32_t sw[S] = {};
    bool hit = false;
    if (i < n) {
      load_slot<S>(states + i * S, sw);
      const uint32_t l = get_field<S>(sw, a.field);
      hit = (a.bad[l >> 5] >> (l & 31)) & 1u;
    }
    const uint64_t m = __ballot(hit);
    if (lane == 0) hits[wave] = static_cast<uint32_t>(__popcll(m));
    __syncthreads();
    const uint32_t all = hits[0] + hits[1] + hits[2] + hits[3];
    if (threadIdx.x == 0 && all) {
      sh_base = atomicAdd(ctr_at(a.ctr, kCtrViol), static_cast<unsigned long long>(all));
      if (sh_base == 0) a.ctr[kCtrViolLevel * kCtrSpread] = level + 1;
      if (e != nullptr && a.stop) e->go = 0;
    }
    __syncthreads();
    if (hit) {
      uint64_t k = sh_base + lane_rank(m);
      for (uint32_t w = 0; w < wave; ++w) k += hits[w];
      if (k < a.cap) store_slot<S>(a.out + k * S, sw);
    }
    __syncthreads();  // hits and sh_base are rewritten by the next round
  }
}

hipError_t launch_monitor_scan(uint32_t S, const ScanArgs& a, uint32_t cus, hipStream_t s) {
  if (a.ctl == nullptr && a.n == 0) return hipSuccess;
  const uint64_t most = static_cast<uint64_t>(cus) * 4;
  const uint32_t grid =
      static_cast<uint32_t>(a.ctl ? most : std::min<uint64_t>((a.n + 255) / 256, most));
  switch (S) {
    case 1: hipLaunchKernelGGL(monitor_scan_kernel<1>, dim3(grid), dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL(monitor_scan_kernel<2>, dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL(monitor_scan_kernel<4>, dim3(grid), dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_level_of(const gx_table* t, const LevelArgs& a, bool filter, uint32_t grid,
                           size_t lds, hipStream_t s) {
  switch (t->S) {
    case 1: return launch_level<1>(t->B, a, filter, grid, lds, s);
    case 2: return launch_level<2>(t->B, a, filter, grid, lds, s);
    case 4: return launch_level<4>(t->B, a, filter, grid, lds, s);
  }
  return hipErrorInvalidValue;
}

// Level-kernel workgroups the table's device holds at once, and the LDS of
// each.
uint32_t level_grid(const gx_table* t, uint32_t img_stride, bool filter, uint32_t cus,
                    size_t* lds) {
  switch (t->S) {
    case 1:
      *lds = level_lds<1>(img_stride, filter);
      return cus * level_blocks_per_cu<1>(t->B, *lds);
    case 2:
      *lds = level_lds<2>(img_stride, filter);
      return cus * level_blocks_per_cu<2>(t->B, *lds);
    default:
      *lds = level_lds<4>(img_stride, filter);
      return cus * level_blocks_per_cu<4>(t->B, *lds);
  }
}

// Grow a device buffer of `cap` elements of `elem` bytes to at least `need`
// elements, keeping its first `keep` elements.  Waits for the stream first.
hipError_t grow(void** p, uint64_t* cap, uint64_t need, size_t elem, uint64_t keep,
                hipStream_t stream, uint64_t limit) {
  if (*cap >= need && *p) return hipSuccess;
  // at least half again the old size (amortised growth), never above limit
  const uint64_t nc = std::max<uint64_t>(need, std::min<uint64_t>(limit, *cap + *cap / 2));
  void* q = nullptr;
  hipError_t e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return e;
  e = hipMalloc(&q, nc * elem);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e;
  }
  if (keep && *p) {
    e = hipMemcpy(q, *p, keep * elem, hipMemcpyDeviceToDevice);
    if (e != hipSuccess) {
      (void)hipFree(q);
      return e;
    }
  }
  if (*p) (void)hipFree(*p);
  *p = q;
  *cap = nc;
  return hipSuccess;
}


}  // namespace
}  // namespace gx

namespace gx {

// The control block of an exploration's buffers: the level counters (one
// cache line each), what a small-level launch reports, the initial state's
// slot and the network image.
constexpr size_t kCtrWords = kCtrCount * kCtrSpread;
constexpr size_t kBlockWords = kCtrWords + sizeof(LevelCtl) / sizeof(uint64_t);
constexpr size_t kControlBytes =
    kBlockWords * sizeof(uint64_t) + 4 * sizeof(uint32_t) + kImgStoreWords * sizeof(uint32_t);

// Where gx_explore_noalloc puts its results.
struct FixedOut {
  uint64_t* level_counts;
  uint32_t max_levels;
  uint32_t* deadlocks;
  uint64_t max_deadlocks;
  gx_explore_summary* summary;
};

// Level counts: a growing host vector, or (fixed) the caller's array, which
// records an overflow instead of growing.
class LevelList {
 public:
  explicit LevelList(FixedOut* f) : f_(f) {}
  void push(uint64_t x) {
    if (f_) {
      if (n_ < f_->max_levels) f_->level_counts[n_] = x;
      else overflow_ = true;
    } else {
      vec_.push_back(x);
    }
    ++n_;
  }
  uint64_t size() const { return n_; }
  uint64_t at(uint64_t k) const { return f_ ? f_->level_counts[k] : vec_[k]; }
  bool overflow() const { return overflow_; }

 private:
  FixedOut* f_;
  std::vector<uint64_t> vec_;
  uint64_t n_ = 0;
  bool overflow_ = false;
};

template <int W>
int cmp_records(const void* a, const void* b) {
  const uint32_t* x = static_cast<const uint32_t*>(a);
  const uint32_t* y = static_cast<const uint32_t*>(b);
  for (int k = 0; k < W; ++k)
    if (x[k] != y[k]) return x[k] < y[k] ? -1 : 1;
  return 0;
}

// Results of a fixed (no-alloc) exploration into the caller's arrays: the
// deadlock records (S words each on the device) are copied into the caller's
// array in chunks through a small host buffer, cut to w words and sorted.
gx_status finish_fixed(FixedOut& f, const LevelList& levels, uint64_t n_dead,
                       uint64_t transitions, const uint32_t* dead, uint32_t S, uint32_t w) {
  if (levels.overflow() || n_dead > f.max_deadlocks) return GX_ENOMEM;
  constexpr uint64_t kChunk = 1024;
  static thread_local uint32_t chunk[kChunk * 4];
  for (uint64_t i0 = 0; i0 < n_dead; i0 += kChunk) {
    const uint64_t n = std::min<uint64_t>(kChunk, n_dead - i0);
    if (hipMemcpy(chunk, dead + i0 * S, n * S * sizeof(uint32_t), hipMemcpyDeviceToHost) !=
        hipSuccess)
      return GX_EDEVICE;
    for (uint64_t i = 0; i < n; ++i)
      for (uint32_t k = 0; k < w; ++k) f.deadlocks[(i0 + i) * w + k] = chunk[i * S + k];
  }
  static int (*const cmp[5])(const void*, const void*) = {nullptr, cmp_records<1>,
                                                          cmp_records<2>, cmp_records<3>,
                                                          cmp_records<4>};
  if (n_dead) std::qsort(f.deadlocks, n_dead, w * sizeof(uint32_t), cmp[w]);
  uint64_t n_states = 0;
  for (uint64_t k = 0; k < levels.size(); ++k) n_states += levels.at(k);
  f.summary->n_states = n_states;
  f.summary->n_transitions = transitions;
  f.summary->n_levels = static_cast<uint32_t>(levels.size());
  f.summary->words_per_state = w;
  f.summary->n_deadlocks = n_dead;
  return GX_OK;
}

}  // namespace gx

// ====================================================================== ABI
extern "C" {

gx_status gx_network_words(const gx_network* net, uint32_t* words) {
  if (!words) return GX_EINVAL;
  gx::NetImage ni;
  const gx_status s = gx::compile_network(net, &ni);
  if (s != GX_OK) return s;
  *words = ni.words;
  return GX_OK;
}

gx_status gx_network_pack(const gx_network* net, const uint32_t* local, uint64_t n,
                          uint32_t* out) {
  if ((n && (!local || !out))) return GX_EINVAL;
  gx::NetImage ni;
  const gx_status s = gx::compile_network(net, &ni);
  if (s != GX_OK) return s;
  const uint32_t P = net->n_procs;
  for (uint64_t i = 0; i < n; ++i) {
    for (uint32_t p = 0; p < P; ++p)
      if (local[i * P + p] >= net->procs[p].n_states) return GX_EINVAL;
  }
  for (uint64_t i = 0; i < n; ++i) gx::pack_host(ni, local + i * P, out + i * ni.words);
  return GX_OK;
}

void gx_explore_result_free(gx_explore_result* r) {
  if (!r) return;
  std::free(r->level_counts);
  std::free(r->deadlocks);
  std::free(r->violations);
  std::free(r->states);
  r->level_counts = nullptr;
  r->deadlocks = nullptr;
  r->violations = nullptr;
  r->states = nullptr;
}

// The exploration of gx_explore into table t, with its device buffers in eb.
// fixed == nullptr: eb is the table's resident set, grown on demand, and the
// result arrays are malloc'd into out.  fixed != nullptr (gx_explore_noalloc):
// eb views preallocated memory that never grows (a buffer that would have to
// is GX_ENOMEM), the control block's host side is plain memory, and the
// level counts and deadlocks go to the caller's arrays in fixed.
static gx_status explore_impl(const gx_network* net, gx_table* t, const gx_explore_opts* opts,
                              gx_explore_buffers& eb, gx::FixedOut* fixed,
                              gx_explore_result* out) {
  gx::NetImage ni;
  // (with preallocated buffers the image must fit the control block)
  gx_status s = gx::compile_network(net, &ni, fixed ? gx::kImgMaxWords : gx::kImgGlobalMaxWords);
  if (s != GX_OK) return s;
  if (ni.words != t->w) return GX_EINVAL;
  const bool monitor = opts && opts->monitor_bad;
  if (monitor && (fixed || opts->monitor_proc >= ni.field.size())) return GX_EINVAL;
  // the table must be empty: its first levels are placed assuming so
  if (t->holds_states) return GX_EINVAL;
  const uint32_t S = t->S;
  const size_t state_bytes = S * sizeof(uint32_t);
  // 0: limited only by device memory
  const uint64_t max_cap = opts && opts->frontier_capacity ? opts->frontier_capacity : ~0ull;
  const uint64_t max_dead = opts && opts->deadlock_capacity ? opts->deadlock_capacity : ~0ull;
  hipStream_t stream = opts ? static_cast<hipStream_t>(opts->hip_stream) : nullptr;
  const uint64_t max_succ = std::max<uint64_t>(1, ni.max_succ);
  const uint64_t max_out = std::max<uint64_t>(1, ni.max_out);

  auto grow_buf = [&](uint32_t** p, uint64_t* cap, uint64_t need, uint64_t keep,
                      uint64_t limit) -> gx_status {
    if (*cap >= need && *p) return GX_OK;
    if (need > limit || fixed) return GX_ENOMEM;
    const uint64_t want = std::min<uint64_t>(limit, std::max<uint64_t>(need, 1u << 16));
    const hipError_t e = gx::grow(reinterpret_cast<void**>(p), cap, want, state_bytes, keep,
                                  stream, limit);
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) return GX_ENOMEM;
    return e == hipSuccess ? GX_OK : GX_EDEVICE;
  };

  // resident buffers of the table (allocated on first use, grow-only)
  const uint32_t img_words = static_cast<uint32_t>(ni.img.size());
  // an image beyond the LDS budget stays in global memory (a buffer of its
  // own), read there by the level kernel; such networks' first levels are
  // not expanded in LDS (that kernel keeps the image there)
  const bool global_img =
      ni.table_words > gx::kImgMaxWords || img_words > gx::kImgStoreWords;
  const uint32_t img_stride = global_img ? 0u : (img_words + 3) & ~3u;
  // the control block: the level's counters, what a small-level launch
  // reports (read back together), the initial state's slot, the image
  constexpr size_t kCtrWords = gx::kCtrWords;
  constexpr size_t kBlockWords = gx::kBlockWords;
  constexpr size_t kControlBytes = gx::kControlBytes;
  if (global_img) {
    if (fixed) return GX_EINVAL;
    if (eb.img_global_cap < img_words) {
      if (eb.img_global) (void)hipFree(eb.img_global);
      eb.img_global = nullptr;
      eb.img_global_cap = 0;
      if (hipMalloc(&eb.img_global, img_words * sizeof(uint32_t)) != hipSuccess) {
        (void)hipGetLastError();
        return GX_ENOMEM;
      }
      eb.img_global_cap = img_words;
    }
    if (hipMemcpyAsync(eb.img_global, ni.img.data(), img_words * sizeof(uint32_t),
                       hipMemcpyHostToDevice, stream) != hipSuccess)
      return GX_EDEVICE;
  }
  if (!fixed &&
      ((!eb.ctr && hipMalloc(&eb.ctr, kControlBytes) != hipSuccess) ||
       (!eb.ctr_host && hipHostMalloc(&eb.ctr_host, kControlBytes,
                                      hipHostMallocMapped | hipHostMallocCoherent) !=
                            hipSuccess) ||
       (!eb.report && hipHostMalloc(&eb.report, gx::kReports * sizeof(uint64_t),
                                    hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) ||
       (!eb.status && hipMalloc(&eb.status, 8) != hipSuccess))) {
    (void)hipGetLastError();
    return GX_ENOMEM;
  }
  eb.key = reinterpret_cast<uint32_t*>(eb.ctr + kBlockWords);
  eb.img = eb.key + 4;
  // A level's NEW states are in the table, and there are no more states than
  // the product of the local ones: a frontier buffer that holds the smaller of
  // the two takes any level; likewise the deadlocks.  With tables of up to
  // kRoomyBytes buffers may grow to that, as the levels need it (see
  // make_room), so that levels follow each other on the device; with others
  // they grow with the levels.
  constexpr uint64_t kRoomyBytes = 256ull << 20;
  const uint64_t n_slots = t->n_buckets * (t->B / S);
  uint64_t most = 1;
  for (uint32_t p = 0; p < net->n_procs; ++p)
    most = net->procs[p].n_states > n_slots / most ? n_slots : most * net->procs[p].n_states;
  bool roomy = !fixed && n_slots * state_bytes <= kRoomyBytes;
  for (int k = 0; k < 2; ++k)
    if ((s = grow_buf(&eb.f[k], &eb.f_cap[k], 1, 0, max_cap)) != GX_OK) return s;
  if ((s = grow_buf(&eb.dead, &eb.dead_cap, 1, 0, max_dead)) != GX_OK) return s;
  // a state's successors never exceed a preallocated buffer
  if (fixed && max_succ > eb.log_cap) return GX_ENOMEM;
  // The first levels run on one workgroup (lds_levels_kernel) while a level
  // of `small_limit` states has room for all its successors in the frontier
  // buffer and the log; not with a safety monitor or the local duplicate
  // filter, whose per-level work that kernel does not do.
  const bool dedup = opts && opts->local_dedup;
  uint64_t small_limit = 0;
  if (!monitor && !dedup && !global_img) {
    if ((s = grow_buf(&eb.log, &eb.log_cap, 1, 0, ~0ull)) != GX_OK) return s;
    const uint64_t room = std::min<uint64_t>(
        std::min<uint64_t>(eb.f_cap[0], eb.f_cap[1]),
        std::min<uint64_t>(eb.log_cap, max_cap));
    small_limit = std::min<uint64_t>(
        gx::kSmallMaxLevel, std::min<uint64_t>(room, gx::kSmallSuccBudget) / max_out);
  }

  uint32_t init[4] = {0, 0, 0, 0};
  gx::pack_host(ni, ni.initial.data(), init);
  // the level's counters, spread over cache lines on the device, read back
  // into pinned host memory
  uint64_t* ctr_raw = eb.ctr_host;
  const gx::LevelCtl* ctl = reinterpret_cast<const gx::LevelCtl*>(ctr_raw + kCtrWords);
  auto ctr = [&](uint32_t k) { return ctr_raw[k * gx::kCtrSpread]; };
  t->holds_states = true;  // from here on the exploration writes the table
  if (++t->explorations == 0) t->explorations = 1;
  if (!fixed) std::memset(eb.report, 0, gx::kReports * sizeof(uint64_t));
  {
    // zeroed counters, the initial state's whole slot (a 3-word state's
    // fourth word is 0) and the image, up in one copy from pinned memory
    std::memset(ctr_raw, 0, kBlockWords * sizeof(uint64_t));
    uint32_t* hkey = reinterpret_cast<uint32_t*>(ctr_raw + kBlockWords);
    std::memcpy(hkey, init, 4 * sizeof(uint32_t));
    const uint32_t lds_img = global_img ? 0u : img_words;
    std::memcpy(hkey + 4, ni.img.data(), lds_img * sizeof(uint32_t));
    const size_t up = kBlockWords * sizeof(uint64_t) + (4 + lds_img) * sizeof(uint32_t);
    if (hipMemcpyAsync(eb.ctr, ctr_raw, up, hipMemcpyHostToDevice, stream) != hipSuccess)
      return GX_EDEVICE;
  }
  // the first level for the level kernel (lds_levels_kernel takes the initial
  // state from eb.key)
  if (small_limit == 0 &&
      hipMemcpyAsync(eb.f[0], eb.key, state_bytes, hipMemcpyDeviceToDevice, stream) != hipSuccess)
    return GX_EDEVICE;
  // the initial state must be new, i.e. the table must not hold it yet
  // (lds_levels_kernel puts it there itself)
  if (small_limit == 0) {
    if (gx::launch_find_or_put(t, eb.key, 1, eb.status, nullptr, stream) != hipSuccess)
      return GX_EDEVICE;
    uint8_t st0 = 0;
    if (hipMemcpyAsync(&st0, eb.status, 1, hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
      return GX_EDEVICE;
    if (st0 == gx::kFull) return GX_ETABLEFULL;
    if (st0 != gx::kNew) return GX_EINVAL;
  }

  // Safety monitor: a bitmask of the bad local states of the monitor
  // process; every completed level is scanned for states holding one.  The
  // initial state (level 0) is checked here.
  uint32_t mon_field = 0;
  std::vector<uint32_t> mon_mask;
  bool init_violates = false;
  uint32_t viol_level = 0xFFFFFFFFu;
  uint64_t viol_total = 0;  // violating states the device has recorded
  bool stop = false;
  if (monitor) {
    const uint32_t mp = opts->monitor_proc;
    const uint32_t n_local = net->procs[mp].n_states;
    mon_mask.assign((n_local + 31) / 32, 0u);
    for (uint32_t l = 0; l < n_local; ++l)
      if (opts->monitor_bad[l]) mon_mask[l >> 5] |= 1u << (l & 31);
    if (eb.mon_cap < mon_mask.size()) {
      if (eb.mon) (void)hipFree(eb.mon);
      eb.mon = nullptr;
      eb.mon_cap = 0;
      if (hipMalloc(&eb.mon, mon_mask.size() * sizeof(uint32_t)) != hipSuccess) {
        (void)hipGetLastError();
        return GX_ENOMEM;
      }
      eb.mon_cap = mon_mask.size();
    }
    if (hipMemcpy(eb.mon, mon_mask.data(), mon_mask.size() * sizeof(uint32_t),
                  hipMemcpyHostToDevice) != hipSuccess)
      return GX_EDEVICE;
    if (roomy && (s = grow_buf(&eb.viol, &eb.viol_cap, 1, 0, ~0ull)) != GX_OK) return s;
    mon_field = ni.field[mp];
    if (opts->monitor_bad[ni.initial[mp]]) {
      init_violates = true;
      viol_level = 0;
      stop = opts->stop_on_violation != 0;
    }
  }

  int cus = 256;
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device);
  // the counters and the control block, copied here, or by the stream's last
  // launch
  auto read_ctr = [&](bool copied = false) -> gx_status {
    if (!copied && (hipMemcpyAsync(ctr_raw, eb.ctr, kBlockWords * sizeof(uint64_t),
                                   hipMemcpyDeviceToHost, stream) != hipSuccess ||
                    hipStreamSynchronize(stream) != hipSuccess))
      return GX_EDEVICE;
    if (ctr(gx::kCtrFlags) & gx::kFlagTableFull) return GX_ETABLEFULL;
    if (ctr(gx::kCtrFlags) & gx::kFlagFrontierOverflow) return GX_ENOMEM;
    if (ctr(gx::kCtrFlags) & gx::kFlagNotEmpty) return GX_EINVAL;
    return GX_OK;
  };

  size_t lds = 0;
  const uint32_t grid_max = gx::level_grid(t, img_stride, dedup, static_cast<uint32_t>(cus), &lds);
  uint32_t max_qs = 0;
  while (max_qs < 6 && (1u << max_qs) < ni.img[0]) ++max_qs;
  gx::LevelArgs la{};
  la.t = t->dev();
  la.img = global_img ? eb.img_global : eb.img;
  la.img_words = img_words;
  la.img_stride = img_stride;
  la.ctr = eb.ctr;
  la.tail = gx::kCtrTail;
  la.waves = grid_max * (gx::kLevelBlock / 64);
  la.max_qs = max_qs;
  la.number = t->explorations;

  gx::ScanArgs scan{};
  scan.field = mon_field;
  scan.bad = eb.mon;
  scan.ctr = eb.ctr;
  scan.stop = opts && opts->stop_on_violation ? 1u : 0u;

  gx::LevelList levels(fixed);
  levels.push(1);
  uint64_t n_in = 1;
  int cur = 0;
  uint64_t dead_known = 0;
  // (the caller's limits on the buffers keep the plain bound of a level's
  // successors)
  const bool any_fits = !(opts && opts->frontier_capacity);
  const uint64_t slice_states = opts ? opts->slice_states : 0;

  // Levels whose successors fit whatever they are need nothing of the host:
  // launches follow each other on the stream, each taking the level the one
  // before left.  The arguments they share; false: level sizes beyond
  // `limit`, or than the deadlock buffer has room for, need the host.
  auto string_args = [&](uint64_t n) {
    la.f[0] = eb.f[0];
    la.f[1] = eb.f[1];
    la.cap_out = std::min<uint64_t>(std::min<uint64_t>(eb.f_cap[0], eb.f_cap[1]), max_cap);
    la.dead = eb.dead;
    la.dead_cap = std::min<uint64_t>(eb.dead_cap, max_dead);
    la.first = 0;
    la.ctl = reinterpret_cast<gx::LevelCtl*>(eb.ctr + kCtrWords);
    la.limit = any_fits && la.cap_out >= most ? ~0ull : la.cap_out / max_succ;
    if (slice_states) la.limit = std::min<uint64_t>(la.limit, slice_states);
    la.viol_cap = monitor ? static_cast<uint32_t>(std::min<uint64_t>(eb.viol_cap, gx::kNoMonitor - 1))
                          : gx::kNoMonitor;
    return (!monitor || eb.viol_cap) && n <= la.limit &&
           la.dead_cap - std::min(dead_known, la.dead_cap) >= n;
  };
  // Buffers that any level fits, once a level has outgrown the first ones (2^16
  // states): in one step, as every allocation takes longer than a level (a
  // first exploration of 3 M states: 1.70 ms with buffers of this size from
  // the start, 1.76 so, 3.4 in steps of four times the need).  False: no memory
  // for them.
  auto make_room = [&]() -> bool {
    const uint64_t f_want = std::min(most, max_cap), d_want = std::min(most, max_dead);
    return grow_buf(&eb.f[cur], &eb.f_cap[cur], f_want, n_in, max_cap) == GX_OK &&
           grow_buf(&eb.f[cur ^ 1], &eb.f_cap[cur ^ 1], f_want, 0, max_cap) == GX_OK &&
           grow_buf(&eb.dead, &eb.dead_cap, d_want, std::min(dead_known, eb.dead_cap), max_dead) ==
               GX_OK;
  };
  // Searches the level just completed, n_in states of buffer `buf`; if the
  // record buffer was short, grows it (keeping earlier levels' records) and
  // searches the level again.
  auto scan_level = [&](int buf) -> gx_status {
    const uint64_t prev = viol_total;
    for (int pass = 0; pass < 2; ++pass) {
      scan.f[buf] = eb.f[buf];
      scan.n = n_in;
      scan.cur = static_cast<uint32_t>(buf);
      scan.out = eb.viol;
      scan.cap = eb.viol_cap;
      scan.level = levels.size() - 1;
      scan.ctl = nullptr;
      if (gx::launch_monitor_scan(S, scan, static_cast<uint32_t>(cus), stream) != hipSuccess)
        return GX_EDEVICE;
      gx_status r = read_ctr();
      if (r != GX_OK) return r;
      viol_total = ctr(gx::kCtrViol);
      if (viol_total <= eb.viol_cap) break;
      if ((r = grow_buf(&eb.viol, &eb.viol_cap, viol_total, prev, ~0ull)) != GX_OK) return r;
      if (hipMemcpy(eb.ctr + gx::kCtrViol * gx::kCtrSpread, &prev, sizeof(prev),
                    hipMemcpyHostToDevice) != hipSuccess)
        return GX_EDEVICE;
    }
    if (viol_total > prev && opts->stop_on_violation) stop = true;
    return GX_OK;
  };
  auto launch_link = [&]() -> gx_status {
    if (gx::launch_level_of(t, la, dedup, grid_max, lds, stream) != hipSuccess) return GX_EDEVICE;
    if (!monitor) return GX_OK;
    scan.f[0] = eb.f[0];
    scan.f[1] = eb.f[1];
    scan.out = eb.viol;
    scan.cap = eb.viol_cap;
    scan.level = levels.size();
    scan.ctl = la.ctl;
    scan.link = la.link;
    return gx::launch_monitor_scan(S, scan, static_cast<uint32_t>(cus), stream) == hipSuccess
               ? GX_OK
               : GX_EDEVICE;
  };
  // A string that goes on until the exploration is over or the host is
  // needed.  kAhead launches are queued from the one on whose report is waited
  // for, and every launch says in host memory what it runs on: the device
  // never waits for the host, and the launches that turn out to have nothing
  // to do, 2 us each, are that many.  (Strings of 16 launches with a read-back
  // after each, about 25 us: a ring of 9 processes 654 us, 568 so; a small
  // random network 182, 151.  More launches ahead gain nothing.)
  // `given`: the first launch takes the level from la; the sizes of the
  // levels found go to `found`.
  constexpr uint32_t kAhead = 2;
  uint32_t link = 0;  // launches of all strings, the first of each an even one
  // The last launch's report is waited for, and it has copied the counters
  // and the control block by then: with a monitor the stream has to drain
  // (scans follow), else nothing is left that touches them.
  auto wait_report = [&](uint32_t k, uint64_t* w) -> gx_status {
    const uint64_t* word = eb.report + k % gx::kReports;
    const uint64_t want = (k + 1) & 0xFFFFu;
    for (uint32_t spins = 1;; ++spins) {
      *w = __hip_atomic_load(word, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
      if (*w >> 48 == want) return GX_OK;
      // (a stream that has nothing left to do has reported everything; asked
      // rarely: the question puts a marker into the stream's queue)
      if (spins % (1u << 22)) continue;
      const hipError_t q = hipStreamQuery(stream);
      if (q == hipErrorNotReady) continue;
      *w = __hip_atomic_load(word, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
      return q == hipSuccess && *w >> 48 == want ? GX_OK : GX_EDEVICE;
    }
  };
  auto run_string = [&](bool given, std::vector<uint64_t>* found) -> gx_status {
    link += link & 1u;
    uint32_t seen = link + (given ? 1u : 0u);  // the next launch to report
    la.report = eb.report;
    la.host_block = eb.ctr_host;
    la.block_words = kBlockWords;
    gx_status r = GX_OK;
    uint64_t w = 0;
    for (bool over = false; r == GX_OK && !over; ++seen) {
      for (; r == GX_OK && link < seen + kAhead; ++link) {
        la.link = link;
        la.given = given ? 1u : 0u;
        given = false;
        r = launch_link();
      }
      if (r != GX_OK || (r = wait_report(seen, &w)) != GX_OK) break;
      const uint64_t n = w & (gx::kReportFresh - 1);
      if ((w & gx::kReportFresh) && n) found->push_back(n);
      over = !(w & gx::kReportGo);
    }
    la.report = nullptr;
    if (r == GX_OK) r = wait_report(link - 1, &w);
    if ((r != GX_OK || monitor) && hipStreamSynchronize(stream) != hipSuccess) r = GX_EDEVICE;
    return r;
  };
  // what a string has left, read back: the level is in the entry given
  auto string_done = [&](uint32_t entry) -> gx_status {
    viol_total = ctr(gx::kCtrViol);
    if (viol_total && opts->stop_on_violation) stop = true;
    dead_known = ctr(gx::kCtrDead);
    if (dead_known > la.dead_cap) return GX_ENOMEM;
    const gx::LevelCtl::Entry& e = ctl->entry[entry & 1u];
    n_in = e.n_in;
    cur = static_cast<int>(e.cur);
    if (e.scan != gx::kScanHost) return GX_OK;
    // (with room for the levels to come as well, where there is memory for it)
    const uint64_t want = roomy ? most : viol_total + n_in;
    if (grow_buf(&eb.viol, &eb.viol_cap, want, viol_total, ~0ull) == GX_EDEVICE) return GX_EDEVICE;
    return scan_level(cur);
  };
  static_assert(kBlockWords <= gx::kLevelBlock, "one word a thread");
  std::vector<uint64_t> found;
  if (small_limit > 0) {
    // the first levels, LDS-resident while the table holds nothing else
    gx::SmallArgs sa{};
    sa.t = t->dev();
    sa.img = eb.img;
    sa.img_words = img_words;
    sa.img_stride = img_stride;
    sa.f = eb.f[0];
    sa.log = eb.log;
    sa.log_cap = eb.log_cap;
    sa.dead = eb.dead;
    sa.dead_cap = std::min<uint64_t>(eb.dead_cap, max_dead);
    sa.ctr = eb.ctr;
    sa.out = reinterpret_cast<gx::LevelCtl*>(eb.ctr + kCtrWords);
    sa.limit = small_limit;
    sa.init_key = eb.key;
    sa.max_succ = static_cast<uint32_t>(max_out);
    sa.max_qs = max_qs;
    const size_t lds_limit = gx::lds_per_workgroup(t->device);
    // a network of more states than the visited set may take goes on without
    // a read-back; one that is likely done has it at once
    uint32_t set_bits = 0;
    switch (S) {
      case 1: set_bits = gx::lds_set_bits<1>(img_stride, lds_limit); break;
      case 2: set_bits = gx::lds_set_bits<2>(img_stride, lds_limit); break;
      case 4: set_bits = gx::lds_set_bits<4>(img_stride, lds_limit); break;
    }
    uint64_t product = 1;
    for (uint32_t p = 0; p < net->n_procs && product < (uint64_t(1) << 31); ++p)
      product *= net->procs[p].n_states;
    const bool goes_on = !fixed && product > (uint64_t(3) << set_bits) / 4 && string_args(1);
    sa.next_limit = goes_on ? la.limit : 0;
    const bool placed =
        !fixed && (S == 1   ? gx::lds_places<1>(t->n_buckets, 1u << set_bits)
                   : S == 2 ? gx::lds_places<2>(t->n_buckets, 1u << set_bits)
                            : gx::lds_places<4>(t->n_buckets, 1u << set_bits));
    if (placed && !goes_on) {
      sa.report = eb.report;
      sa.host_block = eb.ctr_host;
      sa.block_words = kBlockWords;
    }
    sa.number = t->explorations;
    hipError_t e = hipErrorInvalidValue;
    switch (S) {
      case 1: e = gx::launch_lds_levels<1>(t->B, sa, lds_limit, stream); break;
      case 2: e = gx::launch_lds_levels<2>(t->B, sa, lds_limit, stream); break;
      case 4: e = gx::launch_lds_levels<4>(t->B, sa, lds_limit, stream); break;
    }
    if (e != hipSuccess) return GX_EDEVICE;
    uint64_t w = 0;
    if (goes_on && (s = run_string(false, &found)) != GX_OK) return s;
    if (sa.report && (s = wait_report(0, &w)) != GX_OK) return s;
    if (sa.report) link = 1;  // (report 0 is used)
    if ((s = read_ctr(goes_on || placed)) != GX_OK) return s;
    if (ctl->init_status == gx::kFull) return GX_ETABLEFULL;
    if (ctl->init_status != gx::kNew) return GX_EINVAL;
    for (uint64_t k = 0; k < ctl->n_levels; ++k) levels.push(ctl->levels[k]);
    dead_known = ctr(gx::kCtrDead);
    if (dead_known > std::min<uint64_t>(eb.dead_cap, max_dead)) return GX_ENOMEM;
    n_in = ctl->n_in;
    cur = static_cast<int>(ctl->cur);
    if (goes_on) {
      for (const uint64_t n : found) levels.push(n);
      if ((s = string_done(link - 1)) != GX_OK) return s;
    }
  }

  // 16384 workgroups' worth of states per launch unless the caller asks for
  // less
  const uint64_t kTargetSlice = slice_states ? slice_states : 1u << 22;
  constexpr uint64_t kMaxRoom = 1ull << 28;  // states of frontier room one slice may claim
  constexpr uint32_t kString = 16;           // launches between read-backs
  while (n_in > 0 && !stop) {
    if (roomy && !string_args(n_in) && !(slice_states && n_in > slice_states)) roomy = make_room();
    if (string_args(n_in)) {
      la.cur = static_cast<uint32_t>(cur);
      la.n_in = n_in;
      if (!fixed) {
        found.clear();
        if ((s = run_string(true, &found)) != GX_OK || (s = read_ctr(true)) != GX_OK) return s;
        for (const uint64_t n : found) levels.push(n);
        if ((s = string_done(link - 1)) != GX_OK) return s;
        continue;
      }
      // (no memory that the device writes and the host reads: read back after
      // every kString launches)
      for (la.link = 0; la.link < kString; ++la.link) {
        la.given = la.link == 0;
        if ((s = launch_link()) != GX_OK) return s;
      }
      if ((s = read_ctr()) != GX_OK) return s;
      for (uint64_t k = 0; k < ctl->entry[kString & 1u].n_levels; ++k) levels.push(ctl->levels[k]);
      if ((s = string_done(kString)) != GX_OK) return s;
      continue;
    }
    la.given = 1;
    // Otherwise the level is expanded in slices small enough that even if
    // every successor were new the next frontier could not overflow: slice *
    // max_succ <= free frontier room (and slice <= free deadlock room, one
    // record per state at most).  The room is tracked from these worst-case
    // bounds; only when it is short of a full slice is the exact fill read
    // back (one synchronisation), and the buffers grow, keeping their
    // contents, to hold a full slice.
    const int nxt = cur ^ 1;
    uint64_t tail_known = 0, bound = 0, dead_bound = dead_known, pos = 0;
    while (pos < n_in) {
      // full slices, but never more than kMaxRoom states of frontier room
      const uint64_t want = std::min<uint64_t>(
          n_in - pos, std::min<uint64_t>(kTargetSlice, std::max<uint64_t>(1, kMaxRoom / max_succ)));
      // usable capacities: a buffer left larger by an earlier call still
      // honours this call's limits
      auto f_cap = [&]() { return std::min<uint64_t>(eb.f_cap[nxt], max_cap); };
      auto d_cap = [&]() { return std::min<uint64_t>(eb.dead_cap, max_dead); };
      auto f_room = [&]() {
        return any_fits && f_cap() >= most ? ~0ull : (f_cap() - bound) / max_succ;
      };
      // a deadlock buffer at its limit no longer bounds the slice: records
      // past it are counted, not stored, and the call ends with GX_ENOMEM
      auto d_room = [&]() { return d_cap() >= max_dead ? ~0ull : d_cap() - dead_bound; };
      if (std::min<uint64_t>(f_room(), d_room()) < want) {
        if (bound != tail_known || dead_bound != dead_known) {
          if ((s = read_ctr()) != GX_OK) return s;
          tail_known = bound = ctr(la.tail);
          dead_known = dead_bound = ctr(gx::kCtrDead);
        }
        if (f_room() < want) {
          const uint64_t need = bound + want * max_succ;
          s = grow_buf(&eb.f[nxt], &eb.f_cap[nxt],
                       any_fits ? std::min<uint64_t>(need, most) : need, tail_known, max_cap);
          if (s == GX_ENOMEM)  // no room for a full slice: settle for one state
            s = grow_buf(&eb.f[nxt], &eb.f_cap[nxt], bound + max_succ, tail_known,
                         std::min<uint64_t>(max_cap, bound + max_succ));
          if (s != GX_OK) return s;
        }
        if (d_room() < want) {
          s = grow_buf(&eb.dead, &eb.dead_cap, std::min<uint64_t>(dead_bound + want, max_dead),
                       std::min<uint64_t>(dead_known, eb.dead_cap), max_dead);
          if (s != GX_OK) return s;
        }
      }
      const uint64_t run = std::min<uint64_t>(want, std::min<uint64_t>(f_room(), d_room()));
      if (run == 0) return GX_ENOMEM;
      la.f[cur] = eb.f[cur];
      la.f[nxt] = eb.f[nxt];
      la.cap_out = f_cap();
      la.dead = eb.dead;
      la.dead_cap = d_cap();
      la.cur = static_cast<uint32_t>(cur);
      la.first = pos;
      la.n_in = run;
      la.ctl = nullptr;
      const uint32_t qs = gx::lanes_per_state(run, la.waves, max_qs);
      const uint64_t per_group = (64u >> qs) * (gx::kLevelBlock / 64);
      const uint32_t grid = static_cast<uint32_t>(
          std::min<uint64_t>(grid_max, (run + per_group - 1) / per_group));
      if (gx::launch_level_of(t, la, dedup, grid, lds, stream) != hipSuccess) return GX_EDEVICE;
      pos += run;
      bound += std::min<uint64_t>(run * max_succ, most);
      dead_bound += run;
    }
    if ((s = read_ctr()) != GX_OK) return s;
    dead_known = ctr(gx::kCtrDead);
    n_in = ctr(la.tail);
    // (the level's launches have cleared the other tail for the next one)
    la.tail = la.tail == gx::kCtrTail ? gx::kCtrTailAlt : gx::kCtrTail;
    if (n_in) levels.push(n_in);
    if (monitor && n_in && (s = scan_level(nxt)) != GX_OK) return s;
    cur = nxt;
  }
  if (monitor && !init_violates && viol_total)
    viol_level = static_cast<uint32_t>(ctr(gx::kCtrViolLevel) - 1);
  const uint64_t n_dead = ctr(gx::kCtrDead);
  if (n_dead > std::min<uint64_t>(eb.dead_cap, max_dead)) return GX_ENOMEM;
  if (fixed) return gx::finish_fixed(*fixed, levels, n_dead, ctr(gx::kCtrTrans), eb.dead, S, t->w);
  // n records of S words at src, sorted, w words each, to dst
  auto sorted_out = [&](uint32_t* src, uint64_t n, uint32_t* dst) -> gx_status {
    if (n == 0) return GX_OK;
    if (n >= gx::kSortMin && n < (uint64_t(1) << 32) &&
        grow_buf(&eb.f[0], &eb.f_cap[0], n, 0, ~0ull) == GX_OK) {
      const gx_status r = gx::sort_records(S, t->w, src, eb.f[0], n, eb.sort, dst, stream);
      if (r != GX_ENOMEM) return r;
    }
    std::vector<uint32_t> raw(n * S);
    if (hipMemcpy(raw.data(), src, raw.size() * sizeof(uint32_t), hipMemcpyDeviceToHost) !=
        hipSuccess)
      return GX_EDEVICE;
    std::vector<std::array<uint32_t, 4>> v(n);
    for (uint64_t i = 0; i < n; ++i) {
      v[i] = {0, 0, 0, 0};
      for (uint32_t k = 0; k < t->w; ++k) v[i][k] = raw[i * S + k];
    }
    std::sort(v.begin(), v.end());
    for (uint64_t i = 0; i < n; ++i)
      for (uint32_t k = 0; k < t->w; ++k) dst[i * t->w + k] = v[i][k];
    return GX_OK;
  };

  uint64_t* lv = static_cast<uint64_t*>(std::malloc(sizeof(uint64_t) * levels.size()));
  uint32_t* dd = static_cast<uint32_t*>(std::malloc(sizeof(uint32_t) * (n_dead * t->w + 1)));
  s = lv && dd ? sorted_out(eb.dead, n_dead, dd) : GX_ENOMEM;
  if (s != GX_OK) {
    std::free(lv);
    std::free(dd);
    return s;
  }
  uint64_t n_states = 0;
  for (uint64_t k = 0; k < levels.size(); ++k) {
    lv[k] = levels.at(k);
    n_states += levels.at(k);
  }
  out->n_states = n_states;
  out->n_transitions = ctr(gx::kCtrTrans);
  out->words_per_state = t->w;
  out->n_levels = static_cast<uint32_t>(levels.size());
  out->level_counts = lv;
  out->n_deadlocks = n_dead;
  out->deadlocks = dd;
  out->local_duplicates = ctr(gx::kCtrDups);
  out->n_violations = 0;
  out->violations = nullptr;
  out->violation_level = viol_level;
  out->reserved = 0;
  out->states = nullptr;
  if (monitor) {
    const uint64_t n_viol = viol_total + (init_violates ? 1 : 0);
    uint32_t* vv = static_cast<uint32_t*>(std::malloc(sizeof(uint32_t) * (n_viol * t->w + 1)));
    s = vv ? sorted_out(eb.viol, viol_total, vv) : GX_ENOMEM;
    if (s != GX_OK) {
      std::free(vv);
      gx_explore_result_free(out);
      return s;
    }
    if (init_violates) {
      // the initial state to its place among the others
      uint64_t lo = 0, hi = viol_total;
      while (lo < hi) {
        const uint64_t mid = (lo + hi) / 2;
        if (std::lexicographical_compare(vv + mid * t->w, vv + (mid + 1) * t->w, init,
                                         init + t->w))
          lo = mid + 1;
        else
          hi = mid;
      }
      std::memmove(vv + (lo + 1) * t->w, vv + lo * t->w,
                   (viol_total - lo) * t->w * sizeof(uint32_t));
      std::copy(init, init + t->w, vv + lo * t->w);
    }
    out->n_violations = n_viol;
    out->violations = vv;
  }
  return GX_OK;
}

gx_status gx_explore(const gx_network* net, gx_table* t, const gx_explore_opts* opts,
                     gx_explore_result* out) {
  if (!t || !out) return GX_EINVAL;
  return explore_impl(net, t, opts, t->eb, nullptr, out);
}

}  // extern "C"

// ---------------------------------------------------- no-alloc exploration
// Every device buffer gx_explore_noalloc needs beyond the table: one array
// per GPU the library runs on, held until the process ends.  In host code
// the name `scratch` is only a stand-in; its device address comes from
// hipGetSymbolAddress (scratch_address below).
static __device__ __align__(256) uint8_t scratch[GX_NOALLOC_SCRATCH_BYTES];

namespace gx {
namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_dev[kMaxDevices] = {};

// The device address of this GPU's scratch array, looked up once per device
// (with that device current) and kept.
void* scratch_address(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_dev[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    scratch_dev[device] = p;
  }
  return scratch_dev[device];
}

}  // namespace
}  // namespace gx

extern "C" {

gx_status gx_explore_noalloc(const gx_network* net, gx_table* t, const gx_explore_opts* opts,
                             uint64_t* level_counts, uint32_t max_levels, uint32_t* deadlocks,
                             uint64_t max_deadlocks, gx_explore_summary* out) {
  if (!t || !out || !level_counts || max_levels == 0 || (max_deadlocks && !deadlocks))
    return GX_EINVAL;
  if (opts && opts->monitor_bad) return GX_EINVAL;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return GX_EDEVICE;
  if (dev != t->device) return GX_EINVAL;
  char* base = static_cast<char*>(gx::scratch_address(dev));
  if (!base) return GX_EDEVICE;
  // control block | status | frontier 0 | frontier 1 | log | deadlocks
  constexpr uint64_t kCtl = (gx::kControlBytes + 65535) / 65536 * 65536;
  constexpr uint64_t kRegion = (GX_NOALLOC_SCRATCH_BYTES - kCtl - 256) / 4 / 256 * 256;
  static_assert(kCtl + 256 + 4 * kRegion <= GX_NOALLOC_SCRATCH_BYTES, "scratch layout");
  const uint64_t cap = kRegion / (t->S * sizeof(uint32_t));
  alignas(64) static thread_local uint64_t host_block[(gx::kControlBytes + 7) / 8];
  gx_explore_buffers eb;  // views of the scratch array; never grown
  eb.ctr = reinterpret_cast<uint64_t*>(base);
  eb.ctr_host = host_block;
  eb.status = reinterpret_cast<uint8_t*>(base + kCtl);
  char* r = base + kCtl + 256;
  eb.f[0] = reinterpret_cast<uint32_t*>(r);
  eb.f[1] = reinterpret_cast<uint32_t*>(r + kRegion);
  eb.log = reinterpret_cast<uint32_t*>(r + 2 * kRegion);
  eb.dead = reinterpret_cast<uint32_t*>(r + 3 * kRegion);
  eb.f_cap[0] = eb.f_cap[1] = eb.log_cap = eb.dead_cap = cap;
  gx::FixedOut f{level_counts, max_levels, deadlocks, max_deadlocks, out};
  gx_explore_result unused{};
  return explore_impl(net, t, opts, eb, &f, &unused);
}

}  // extern "C"
