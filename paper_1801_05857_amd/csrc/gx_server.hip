// Exploration server: requests (networks with a declared size bound) are
// admitted when their HBM reservation fits the budget, get their table,
// frontiers and deadlock buffer as one block of a device arena allocated
// once with the server (a buddy allocator: reservations are powers of two,
// so admitting a request allocates nothing), and are advanced one BFS level
// per step by a multi-job launch over every active request (continuous
// batching: requests join and leave between steps).  A request whose table
// fills up is retried with four times its bound.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <set>
#include <thread>
#include <vector>

#include "gx_buddy.hpp"
#include "gx_serve_kernel.hpp"

namespace gx {

gx_status compile_network_image(const gx_network* net, std::vector<uint32_t>* img,
                                uint32_t* words, std::vector<uint32_t>* packed_initial,
                                uint64_t* max_succ);

// instantiated in gx_serve_s1.hip, gx_serve_s2.hip and gx_serve_s4.hip
extern template hipError_t serve_launch<1>(uint32_t, const ServeArgs&, uint32_t, size_t,
                                           hipStream_t);
extern template hipError_t admit_launch<1>(uint32_t, const TableDev&, const uint32_t*, uint32_t*,
                                            uint64_t*, uint32_t, hipStream_t);
extern template uint32_t step_blocks_per_cu<1>(uint32_t, size_t);
extern template hipError_t serve_launch<2>(uint32_t, const ServeArgs&, uint32_t, size_t,
                                           hipStream_t);
extern template hipError_t admit_launch<2>(uint32_t, const TableDev&, const uint32_t*, uint32_t*,
                                            uint64_t*, uint32_t, hipStream_t);
extern template uint32_t step_blocks_per_cu<2>(uint32_t, size_t);
extern template hipError_t serve_launch<4>(uint32_t, const ServeArgs&, uint32_t, size_t,
                                           hipStream_t);
extern template hipError_t admit_launch<4>(uint32_t, const TableDev&, const uint32_t*, uint32_t*,
                                            uint64_t*, uint32_t, hipStream_t);
extern template uint32_t step_blocks_per_cu<4>(uint32_t, size_t);

namespace {

using Clock = std::chrono::steady_clock;
constexpr uint32_t kMaxAttempts = 12;
// a job's counters: kCtrCount counters kCtrSpread words apart (one cache line each)
constexpr uint64_t kSlotCtrWords = uint64_t(kCtrCount) * kCtrSpread;

struct Request {
  uint64_t id = 0;
  std::vector<uint32_t> img, init;
  uint32_t w = 0;
  uint64_t declared = 0;
  uint32_t attempts = 0;
  Clock::time_point arrival;
  bool done = false;
  gx_status status = GX_OK;
  gx_explore_result result{};
  uint64_t latency_ns = 0;
};

uint64_t pow2_at_least(uint64_t x) {
  uint64_t p = 1;
  while (p < x) p <<= 1;
  return p;
}


// What goes up when a job is admitted, one copy: its initial state's slot and
// its network image (a region per job slot on the device).  Pinned staging has
// kStageSlots regions, used in turn: the copies of one round of admissions are
// done before the next (its steps' read-back follows them), and a round that
// admits more waits for them.
constexpr uint64_t kSlotWords = 4 + kImgStoreWords;
constexpr uint32_t kStageSlots = 64;

// Steps between read-backs, by the states of all jobs' levels: while levels
// are small a read-back (about 85 us) costs as much as a step, and a request
// that arrives meanwhile waits for a few short steps; from kLargeLevels on a
// step takes milliseconds, and every one is followed by a read-back.
constexpr uint32_t kSteps = 8;
constexpr uint64_t kSmallLevels = 1u << 20, kLargeLevels = 1u << 23;
uint32_t steps_for(uint64_t states) {
  return states < kSmallLevels ? kSteps : states < kLargeLevels ? kSteps / 2 : 1;
}

}  // namespace
}  // namespace gx

struct gx_server {
  struct Job {
    gx::Request* r = nullptr;
    gx_table* t = nullptr;   // a view of its arena block
    uint64_t reserved = 0;   // bytes of that block
    uint64_t block = 0;      // its offset in the arena
    uint64_t n_in = 0;
    int cur = 0;
    uint32_t slot = 0;
    std::vector<uint64_t> levels;
  };
  // configuration
  uint64_t budget = 0;
  uint32_t max_active = 0;
  bool keep_states = false;
  double load = 0.5;
  uint64_t seed = 0;
  uint32_t H = 8;
  uint32_t cfg[5][3] = {};  // per slot width: bucket words, subgroup, keys per subgroup
  int device = 0;
  hipStream_t stream = nullptr;
  // state, guarded by mu
  std::mutex mu;
  std::condition_variable cv_work, cv_done;
  bool stop = false;
  uint64_t next_id = 1;
  std::map<uint64_t, std::unique_ptr<gx::Request>> reqs;
  std::deque<gx::Request*> waiting;
  uint64_t reserved = 0;        // bytes reserved by active jobs
  // device arena of budget bytes, shared hash constants, per-slot small state
  char* arena = nullptr;
  uint64_t arena_bytes = 0;
  gx::Buddy buddy;
  uint64_t a0 = 0, c0 = 0;  // first hash constant pair (host copy)
  uint64_t* d_hc = nullptr;
  gx_server_stats stats{};
  // owned by the step thread
  gx::SortSpace sort;
  std::vector<Job> active;
  std::vector<uint32_t> free_slots;
  // per job slot: initial state and image (device, pinned staging), counters
  uint32_t* d_slot = nullptr;
  uint32_t* h_slot = nullptr;
  uint64_t* d_ctr = nullptr;
  uint64_t* h_ctr = nullptr;   // pinned host copy of d_ctr
  // per slot width: its steps' stream, descriptors and what they leave, as
  // the batch's classes
  struct Lane {
    hipStream_t stream = nullptr;
    hipEvent_t done = nullptr;
    char* d_step = nullptr;
    char* h_step = nullptr;
    gx::StepOut* d_out = nullptr;
    gx::StepOut* h_out = nullptr;
    std::vector<size_t> jobs;  // the string's, by their place in `active`
    uint32_t lds_for = 0, resident = 0;  // image stride the grid was sized for
  } lanes[3];
  hipEvent_t admitted = nullptr;
  std::thread th;
};

namespace gx {
namespace {

uint64_t table_bytes_for(uint32_t w, uint64_t slots) {
  // table + two frontiers + deadlock buffer, each slots x S words
  return 4ull * slots * slot_words(w) * sizeof(uint32_t);
}

void complete(gx_server* s, Request* r, gx_status st) {
  r->status = st;
  r->latency_ns = static_cast<uint64_t>(
      std::chrono::duration_cast<std::chrono::nanoseconds>(Clock::now() - r->arrival).count());
  r->done = true;
  r->img.clear();
  r->img.shrink_to_fit();
  if (st == GX_OK) ++s->stats.completed;
  else ++s->stats.failed;
}

// A table over the arena block at `off` for w words and `slots` slots (a
// power of two): the table, then the two frontiers and the deadlock buffer,
// slots states each; the server's shared hash constants.  Nothing is
// allocated on the device.  mu held.
gx_table* job_table(gx_server* s, uint32_t w, uint64_t slots, uint64_t off) {
  const uint32_t S = slot_words(w);
  const uint32_t* c = s->cfg[S];
  gx_table* t = new (std::nothrow) gx_table;
  if (!t) return nullptr;
  t->device = s->device;
  t->w = w;
  t->S = S;
  t->B = c[0];
  t->G = c[1];
  t->U = c[2];
  t->H = s->H;
  t->seed = s->seed;
  t->n_buckets = slots * S / c[0];
  t->a0 = s->a0;
  t->c0 = s->c0;
  const uint64_t T = slots * S * sizeof(uint32_t);
  char* base = s->arena + off;
  t->words = reinterpret_cast<uint32_t*>(base);
  t->hc = s->d_hc;
  t->counters = nullptr;  // job tables keep no statistics
  t->ctr_slots = 1;
  for (int k = 0; k < 2; ++k) {
    t->eb.f[k] = reinterpret_cast<uint32_t*>(base + (k + 1) * T);
    t->eb.f_cap[k] = slots;
  }
  t->eb.dead = reinterpret_cast<uint32_t*>(base + 3 * T);
  t->eb.dead_cap = slots;
  return t;
}

// Admit waiting requests while their reservations fit.  mu held.
void admit(gx_server* s) {
  uint32_t staged = 0;
  while (!s->waiting.empty() && !s->free_slots.empty()) {
    Request* r = s->waiting.front();
    const uint64_t slots = pow2_at_least(
        std::max<uint64_t>(64, static_cast<uint64_t>(static_cast<double>(r->declared) / s->load) + 1));
    const uint64_t need = table_bytes_for(r->w, slots);
    if (need > s->buddy.largest()) {  // can never fit
      s->waiting.pop_front();
      complete(s, r, GX_ENOMEM);
      s->cv_done.notify_all();
      continue;
    }
    const uint64_t off = s->buddy.alloc(need);
    if (off == ~0ull) break;  // wait for running jobs to finish
    const uint32_t slot = s->free_slots.back();
    gx_table* t = job_table(s, r->w, slots, off);
    if (!t) {
      s->buddy.release(off, need);
      break;
    }
    s->waiting.pop_front();
    gx_server::Job j;
    j.r = r;
    j.t = t;
    j.reserved = need;
    j.block = off;
    j.slot = slot;
    s->free_slots.pop_back();
    s->reserved += need;
    s->stats.reserved_peak = std::max(s->stats.reserved_peak, s->reserved);
    // reset the table, place the initial state, insert it: only enqueued (the
    // job's first step comes after it on the device)
    const uint64_t at = static_cast<uint64_t>(j.slot) * kSlotWords;
    bool ok = true;
    if (staged == kStageSlots) {
      ok = hipStreamSynchronize(s->stream) == hipSuccess;
      staged = 0;
    }
    uint32_t* up = s->h_slot + staged++ * kSlotWords;
    for (uint32_t x = 0; x < 4; ++x) up[x] = x < r->w ? r->init[x] : 0u;
    std::copy(r->img.begin(), r->img.end(), up + 4);
    uint64_t* ctr = s->d_ctr + kSlotCtrWords * j.slot;
    ok = ok && gx_table_clear(t, s->stream) == GX_OK &&
         hipMemcpyAsync(s->d_slot + at, up, (4 + r->img.size()) * sizeof(uint32_t),
                        hipMemcpyHostToDevice, s->stream) == hipSuccess;
    if (ok) {
      const uint32_t* key = s->d_slot + at;
      hipError_t e;
      switch (t->S) {
        case 1: e = admit_launch<1>(t->B, t->dev(), key, t->eb.f[0], ctr, kSlotCtrWords, s->stream); break;
        case 2: e = admit_launch<2>(t->B, t->dev(), key, t->eb.f[0], ctr, kSlotCtrWords, s->stream); break;
        default: e = admit_launch<4>(t->B, t->dev(), key, t->eb.f[0], ctr, kSlotCtrWords, s->stream); break;
      }
      ok = e == hipSuccess;
    }
    if (!ok) {
      s->reserved -= need;
      s->free_slots.push_back(j.slot);
      s->buddy.release(off, need);
      delete t;
      complete(s, r, GX_EDEVICE);
      s->cv_done.notify_all();
      continue;
    }
    j.n_in = 1;
    j.cur = 0;
    j.levels.assign(1, 1);
    s->active.push_back(std::move(j));
    s->stats.active_peak = std::max<uint64_t>(s->stats.active_peak, s->active.size());
  }
}

// Finish job k of s->active (mu held): store its result or retry it.
void finish_job(gx_server* s, size_t k, gx_status st, uint64_t transitions, uint64_t n_dead) {
  gx_server::Job& j = s->active[k];
  Request* r = j.r;
  if (st == GX_ETABLEFULL && r->attempts + 1 < kMaxAttempts) {
    ++r->attempts;
    // four times the bound, and at least twice the states already found
    uint64_t found = 0;
    for (uint64_t c : j.levels) found += c;
    r->declared = std::max<uint64_t>(r->declared * 4, 2 * found);
    ++s->stats.retried;
    s->waiting.push_front(r);
  } else if (st != GX_OK) {
    complete(s, r, st);
  } else {
    const uint32_t w = r->w, S = j.t->S;
    std::vector<uint32_t> raw(n_dead * S);
    gx_status rs = GX_OK;
    if (n_dead && hipMemcpy(raw.data(), j.t->eb.dead, raw.size() * sizeof(uint32_t),
                            hipMemcpyDeviceToHost) != hipSuccess)
      rs = GX_EDEVICE;
    std::vector<std::array<uint32_t, 4>> dl(n_dead);
    for (uint64_t i = 0; i < n_dead; ++i) {
      dl[i] = {0, 0, 0, 0};
      for (uint32_t x = 0; x < w; ++x) dl[i][x] = raw[i * S + x];
    }
    std::sort(dl.begin(), dl.end());
    uint64_t* L = static_cast<uint64_t*>(std::malloc(sizeof(uint64_t) * j.levels.size()));
    uint32_t* D = static_cast<uint32_t*>(std::malloc(sizeof(uint32_t) * (n_dead * w + 1)));
    uint32_t* V = nullptr;  // the table's contents, read before its block is released
    if (!L || !D) rs = GX_ENOMEM;
    if (rs == GX_OK && s->keep_states)
      // (the job's frontier buffers, free once it is over)
      rs = sorted_keys_malloc(j.t->words, j.t->n_buckets * j.t->B, S, w, j.t->eb.f[0],
                              j.t->eb.f[1], j.t->eb.f_cap[0], s->sort, s->stream, &V);
    if (rs == GX_OK) {
      uint64_t total = 0;
      for (size_t l = 0; l < j.levels.size(); ++l) {
        L[l] = j.levels[l];
        total += L[l];
      }
      for (uint64_t i = 0; i < n_dead; ++i)
        for (uint32_t x = 0; x < w; ++x) D[i * w + x] = dl[i][x];
      r->result.n_states = total;
      r->result.n_transitions = transitions;
      r->result.words_per_state = w;
      r->result.n_levels = static_cast<uint32_t>(j.levels.size());
      r->result.level_counts = L;
      r->result.n_deadlocks = n_dead;
      r->result.deadlocks = D;
      r->result.violation_level = 0xFFFFFFFFu;  // no safety monitor in the server
      r->result.states = V;
      s->stats.states += total;
    } else {
      std::free(L);
      std::free(D);
      std::free(V);
    }
    complete(s, r, rs);
  }
  s->reserved -= j.reserved;
  s->free_slots.push_back(j.slot);
  s->buddy.release(j.block, j.reserved);
  delete j.t;  // a view: its memory stays in the arena
  s->active.erase(s->active.begin() + k);
}

// Bytes of a class's header, job descriptors and first groups.
size_t step_bytes(uint32_t n_jobs) {
  return sizeof(StepHdr) + n_jobs * (sizeof(ServeJob) + sizeof(uint32_t));
}

// Enqueues a string of steps of the active jobs of slot width S on the
// class's stream, after the admissions; *steps receives its length.
hipError_t enqueue_steps(gx_server* s, uint32_t S, uint32_t cus, uint64_t all_states,
                         uint32_t n_steps, bool* any) {
  gx_server::Lane& ln = s->lanes[S == 1 ? 0 : S == 2 ? 1 : 2];
  ln.jobs.clear();
  uint64_t states = 0;
  uint32_t img_max = 0;
  for (size_t k = 0; k < s->active.size(); ++k) {
    const gx_server::Job& j = s->active[k];
    if (j.t->S != S) continue;
    ln.jobs.push_back(k);
    states += j.n_in;
    img_max = std::max<uint32_t>(img_max, static_cast<uint32_t>(j.r->img.size()));
  }
  *any = !ln.jobs.empty();
  if (!*any) return hipSuccess;
  const uint32_t n = static_cast<uint32_t>(ln.jobs.size());
  const uint32_t qs = step_lanes(states, cus);
  StepHdr* hdr = reinterpret_cast<StepHdr*>(ln.h_step);
  ServeJob* jobs = reinterpret_cast<ServeJob*>(ln.h_step + sizeof(StepHdr));
  uint32_t* begin = reinterpret_cast<uint32_t*>(jobs + n);
  uint64_t total = 0;
  for (uint32_t k = 0; k < n; ++k) {
    const gx_server::Job& j = s->active[ln.jobs[k]];
    ServeJob& x = jobs[k];
    x.t = j.t->dev();
    x.img_off = static_cast<uint32_t>(j.slot * kSlotWords + 4);
    x.img_words = static_cast<uint32_t>(j.r->img.size());
    x.f[0] = j.t->eb.f[0];
    x.f[1] = j.t->eb.f[1];
    x.n_in = j.n_in;
    x.cap_out = j.t->eb.f_cap[0];
    x.dead = j.t->eb.dead;
    x.dead_cap = j.t->eb.dead_cap;
    x.ctr = s->d_ctr + kSlotCtrWords * j.slot;
    x.dead_ctr = nullptr;
    x.dead_tag = nullptr;
    x.tag = 0;
    x.cur = static_cast<uint32_t>(j.cur);
    x.levels_left = 0xFFFFFFFFu;
    x.pad = 0;
    begin[k] = static_cast<uint32_t>(total);
    total += step_groups(j.n_in, qs);
  }
  if (total > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hdr->total = static_cast<uint32_t>(total);
  hdr->qs = qs;
  hdr->steps = 0;
  hdr->halt = 0;
  ServeJob* d_jobs = reinterpret_cast<ServeJob*>(ln.d_step + sizeof(StepHdr));
  uint32_t* d_begin = reinterpret_cast<uint32_t*>(d_jobs + n);
  StepHdr* d_hdr = reinterpret_cast<StepHdr*>(ln.d_step);
  ServeArgs a;
  a.jobs = d_jobs;
  a.begin = d_begin;
  a.n_jobs = n;
  a.hdr = d_hdr;
  a.img = s->d_slot;
  a.img_stride = (img_max + 3) & ~3u;
  const size_t lds = step_lds(S, a.img_stride);
  const uint32_t* c = s->cfg[S];
  if (ln.resident == 0 || ln.lds_for != a.img_stride) {
    switch (S) {
      case 1: ln.resident = cus * step_blocks_per_cu<1>(c[0], lds); break;
      case 2: ln.resident = cus * step_blocks_per_cu<2>(c[0], lds); break;
      default: ln.resident = cus * step_blocks_per_cu<4>(c[0], lds); break;
    }
    ln.lds_for = a.img_stride;
  }
  // the class's share of the device, a little more than its states' of all:
  // workgroups that hold the whole device would keep the others out for a step
  const double share =
      all_states ? static_cast<double>(states) / static_cast<double>(all_states) : 1.0;
  const uint32_t grid = std::min<uint32_t>(
      ln.resident, std::max<uint32_t>(cus, static_cast<uint32_t>(ln.resident * (share * 1.2))));
  hipError_t e = hipStreamWaitEvent(ln.stream, s->admitted, 0);
  if (e == hipSuccess)
    e = hipMemcpyAsync(ln.d_step, ln.h_step, step_bytes(n), hipMemcpyHostToDevice, ln.stream);
  for (uint32_t k = 0; k < n_steps && e == hipSuccess; ++k) {
    switch (S) {
      case 1: e = serve_launch<1>(c[0], a, grid, lds, ln.stream); break;
      case 2: e = serve_launch<2>(c[0], a, grid, lds, ln.stream); break;
      default: e = serve_launch<4>(c[0], a, grid, lds, ln.stream); break;
    }
    if (e != hipSuccess) break;
    hipLaunchKernelGGL(step_update_kernel, dim3(1), dim3(1024), 0, ln.stream, d_jobs, d_begin, n,
                       d_hdr, ln.d_out + static_cast<uint64_t>(k) * n, cus,
                       n_steps == 1      ? ~uint64_t(0)
                       : n_steps == kSteps ? 2 * kSmallLevels
                                           : 2 * kLargeLevels);
    e = hipGetLastError();
  }
  // the header tells how many steps were done
  if (e == hipSuccess)
    e = hipMemcpyAsync(ln.h_step, ln.d_step, sizeof(StepHdr), hipMemcpyDeviceToHost, ln.stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(ln.h_out, ln.d_out, sizeof(StepOut) * n_steps * n, hipMemcpyDeviceToHost,
                       ln.stream);
  if (e == hipSuccess) e = hipEventRecord(ln.done, ln.stream);
  return e;
}

void step_loop(gx_server* s) {
  (void)hipSetDevice(s->device);  // a new thread starts with device 0
  const uint32_t cus = resident_grid(s->device, 1);
  while (true) {
    {
      std::unique_lock<std::mutex> lock(s->mu);
      s->cv_work.wait(lock, [&] { return s->stop || !s->waiting.empty() || !s->active.empty(); });
      if (s->stop) return;
      admit(s);
      if (s->active.empty()) {
        // nothing admitted (budget held by nothing?) - wait for a new request
        if (!s->waiting.empty()) s->cv_work.wait_for(lock, std::chrono::milliseconds(1));
        continue;
      }
    }
    // a string of steps over every active job, the slot widths side by side
    uint64_t all = 0;
    for (const auto& j : s->active) all += j.n_in;
    const uint32_t n_steps = steps_for(all);
    bool ok = hipEventRecord(s->admitted, s->stream) == hipSuccess;
    bool any[3] = {false, false, false};
    for (int i = 0; i < 3 && ok; ++i)
      ok = enqueue_steps(s, i == 0 ? 1u : i == 1 ? 2u : 4u, cus, all, n_steps, &any[i]) ==
           hipSuccess;
    for (int i = 0; i < 3; ++i) {
      if (!any[i]) continue;
      if (ok) ok = hipEventSynchronize(s->lanes[i].done) == hipSuccess;
      if (!ok) (void)hipStreamSynchronize(s->lanes[i].stream);
    }
    // what became of each job: its levels, and its end
    struct End {
      size_t k;
      gx_status st;
    };
    std::vector<End> ends;
    uint64_t most = 0;
    if (ok) {
      for (int i = 0; i < 3; ++i) {
        if (!any[i]) continue;
        gx_server::Lane& ln = s->lanes[i];
        const uint32_t n = static_cast<uint32_t>(ln.jobs.size());
        const uint32_t steps = reinterpret_cast<const StepHdr*>(ln.h_step)->steps;
        most = std::max<uint64_t>(most, steps);
        for (uint32_t k = 0; k < n; ++k) {
          gx_server::Job& j = s->active[ln.jobs[k]];
          for (uint32_t st = 0; st < steps; ++st) {
            const StepOut& o = ln.h_out[static_cast<uint64_t>(st) * n + k];
            if (o.flags == 0 && o.n_next != 0) {
              j.levels.push_back(o.n_next);
              j.n_in = o.n_next;
              j.cur ^= 1;
              continue;
            }
            ends.push_back({ln.jobs[k], o.flags & kFlagTableFull ? GX_ETABLEFULL
                                        : o.flags                ? GX_ENOMEM
                                                                 : GX_OK});
            break;
          }
        }
      }
      // the counters of the jobs that have ended
      uint32_t n_slots = 0;
      for (const End& x : ends) n_slots = std::max(n_slots, s->active[x.k].slot + 1);
      if (n_slots &&
          (hipMemcpyAsync(s->h_ctr, s->d_ctr, kSlotCtrWords * n_slots * sizeof(uint64_t),
                          hipMemcpyDeviceToHost, s->stream) != hipSuccess ||
           hipStreamSynchronize(s->stream) != hipSuccess))
        ok = false;
    }
    std::lock_guard<std::mutex> lock(s->mu);
    s->stats.steps += std::max<uint64_t>(most, 1);
    if (!ok) {
      for (size_t k = s->active.size(); k-- > 0;) finish_job(s, k, GX_EDEVICE, 0, 0);
    } else {
      std::sort(ends.begin(), ends.end(), [](const End& x, const End& y) { return x.k > y.k; });
      for (const End& x : ends) {
        const uint64_t* c = &s->h_ctr[kSlotCtrWords * s->active[x.k].slot];
        if (x.st == GX_OK)
          finish_job(s, x.k, GX_OK, c[kCtrTrans * kCtrSpread], c[kCtrDead * kCtrSpread]);
        else
          finish_job(s, x.k, x.st, 0, 0);
      }
    }
    s->cv_done.notify_all();
  }
}

void destroy_server(gx_server* s) {
  if (!s) return;
  if (s->th.joinable()) {
    {
      std::lock_guard<std::mutex> lock(s->mu);
      s->stop = true;
    }
    s->cv_work.notify_all();
    s->th.join();
  }
  (void)hipDeviceSynchronize();
  for (auto& j : s->active) delete j.t;
  for (auto& kv : s->reqs) gx_explore_result_free(&kv.second->result);
  for (auto& ln : s->lanes) {
    if (ln.d_step) (void)hipFree(ln.d_step);
    if (ln.d_out) (void)hipFree(ln.d_out);
    if (ln.h_step) (void)hipHostFree(ln.h_step);
    if (ln.h_out) (void)hipHostFree(ln.h_out);
    if (ln.done) (void)hipEventDestroy(ln.done);
    if (ln.stream) (void)hipStreamDestroy(ln.stream);
  }
  if (s->admitted) (void)hipEventDestroy(s->admitted);
  if (s->d_slot) (void)hipFree(s->d_slot);
  if (s->h_slot) (void)hipHostFree(s->h_slot);
  if (s->d_ctr) (void)hipFree(s->d_ctr);
  if (s->h_ctr) (void)hipHostFree(s->h_ctr);
  if (s->arena) (void)hipFree(s->arena);
  if (s->d_hc) (void)hipFree(s->d_hc);
  if (s->stream) (void)hipStreamDestroy(s->stream);
  s->cv_done.notify_all();
  delete s;
}

}  // namespace
}  // namespace gx

// ====================================================================== ABI
extern "C" {

gx_status gx_server_create(const gx_server_opts* opts, gx_server** out) {
  if (!opts || !out || opts->budget_bytes == 0) return GX_EINVAL;
  const double load = opts->load_factor > 0 ? opts->load_factor : 0.5;
  if (load > 0.95) return GX_EINVAL;
  if (opts->bucket_words && !(opts->bucket_words == 8 || opts->bucket_words == 16 ||
                              opts->bucket_words == 32 || opts->bucket_words == 64))
    return GX_EINVAL;
  if (opts->subgroup && !(opts->subgroup == 4 || opts->subgroup == 8 || opts->subgroup == 16))
    return GX_EINVAL;
  if (opts->subgroup == 4 && opts->bucket_words > 32) return GX_EINVAL;
  if (opts->keys_per_subgroup && !(opts->keys_per_subgroup == 1 || opts->keys_per_subgroup == 2))
    return GX_EINVAL;
  gx_server* s = new (std::nothrow) gx_server;
  if (!s) return GX_ENOMEM;
  s->budget = opts->budget_bytes;
  s->max_active = opts->max_active ? opts->max_active : 256;
  s->keep_states = opts->keep_states != 0;
  s->load = load;
  s->seed = opts->hash_seed ? opts->hash_seed : 0x1801058570ull;
  s->H = opts->max_hashes ? opts->max_hashes : 8;
  if (hipGetDevice(&s->device) != hipSuccess) {
    delete s;
    return GX_EDEVICE;
  }
  for (uint32_t S : {1u, 2u, 4u}) {
    uint32_t B = opts->bucket_words, G = opts->subgroup, U = opts->keys_per_subgroup;
    if (!B || !G || !U) {
      uint32_t tb = 32, tg = 8, tu = 1;
      const gx_status st = gx_autotune(S, load, &tb, &tg, &tu);
      if (st != GX_OK) {
        delete s;
        return st;
      }
      B = B ? B : tb;
      G = G ? G : tg;
      U = U ? U : 1;
      gx::fit_subgroup(&B, &G, opts->bucket_words != 0);
    }
    if (B < 2 * S) B = 2 * S;
    s->cfg[S][0] = B;
    s->cfg[S][1] = G;
    s->cfg[S][2] = U;
  }
  s->cfg[3][0] = s->cfg[4][0];
  s->cfg[3][1] = s->cfg[4][1];
  s->cfg[3][2] = s->cfg[4][2];
  bool made =
      hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking) == hipSuccess &&
      hipEventCreateWithFlags(&s->admitted, hipEventDisableTiming) == hipSuccess &&
      hipMalloc(&s->d_slot, s->max_active * gx::kSlotWords * sizeof(uint32_t)) == hipSuccess &&
      hipHostMalloc(&s->h_slot, gx::kStageSlots * gx::kSlotWords * sizeof(uint32_t)) == hipSuccess &&
      hipMalloc(&s->d_ctr, gx::kSlotCtrWords * s->max_active * sizeof(uint64_t)) == hipSuccess &&
      hipHostMalloc(&s->h_ctr, gx::kSlotCtrWords * s->max_active * sizeof(uint64_t)) == hipSuccess;
  for (auto& ln : s->lanes)
    made = made && hipStreamCreateWithFlags(&ln.stream, hipStreamNonBlocking) == hipSuccess &&
           hipEventCreateWithFlags(&ln.done, hipEventDisableTiming) == hipSuccess &&
           hipMalloc(&ln.d_step, gx::step_bytes(s->max_active)) == hipSuccess &&
           hipHostMalloc(&ln.h_step, gx::step_bytes(s->max_active)) == hipSuccess &&
           hipMalloc(&ln.d_out, sizeof(gx::StepOut) * gx::kSteps * s->max_active) == hipSuccess &&
           hipHostMalloc(&ln.h_out, sizeof(gx::StepOut) * gx::kSteps * s->max_active) == hipSuccess;
  if (!made) {
    (void)hipGetLastError();
    gx::destroy_server(s);
    return GX_ENOMEM;
  }
  // the arena (allocated once: admission allocates nothing) and the hash
  // constants every job table shares
  {
    const uint64_t arena_bytes = s->budget & ~((uint64_t(1) << gx::Buddy::kMinShift) - 1);
    std::vector<uint64_t> hc(2 * s->H);
    for (uint32_t j = 0; j < s->H; ++j) gx::hash_constants(s->seed, j, &hc[2 * j], &hc[2 * j + 1]);
    s->a0 = hc[0];
    s->c0 = hc[1];
    if (arena_bytes == 0 || hipMalloc(&s->arena, arena_bytes) != hipSuccess ||
        hipMalloc(&s->d_hc, hc.size() * sizeof(uint64_t)) != hipSuccess) {
      (void)hipGetLastError();
      gx::destroy_server(s);
      return GX_ENOMEM;
    }
    if (hipMemcpy(s->d_hc, hc.data(), hc.size() * sizeof(uint64_t), hipMemcpyHostToDevice) !=
        hipSuccess) {
      gx::destroy_server(s);
      return GX_EDEVICE;
    }
    s->arena_bytes = arena_bytes;
    s->buddy.init(arena_bytes);
  }
  for (uint32_t k = s->max_active; k-- > 0;) s->free_slots.push_back(k);
  try {
    s->th = std::thread(gx::step_loop, s);
  } catch (...) {
    gx::destroy_server(s);
    return GX_ENOMEM;
  }
  *out = s;
  return GX_OK;
}

gx_status gx_server_submit(gx_server* s, const gx_network* net, uint64_t declared_states,
                           uint64_t* request_id) {
  if (!s || !request_id || declared_states == 0) return GX_EINVAL;
  auto r = std::unique_ptr<gx::Request>(new (std::nothrow) gx::Request);
  if (!r) return GX_ENOMEM;
  uint64_t ms = 0;
  const gx_status st = gx::compile_network_image(net, &r->img, &r->w, &r->init, &ms);
  if (st != GX_OK) return st;
  r->declared = declared_states;
  r->arrival = gx::Clock::now();
  {
    std::lock_guard<std::mutex> lock(s->mu);
    r->id = s->next_id++;
    *request_id = r->id;
    s->waiting.push_back(r.get());
    s->reqs.emplace(r->id, std::move(r));
    ++s->stats.submitted;
  }
  s->cv_work.notify_all();
  return GX_OK;
}

gx_status gx_server_poll(gx_server* s, uint64_t id, int wait, gx_explore_result* out,
                         gx_status* request_status, uint64_t* latency_ns) {
  if (!s || !out || !request_status) return GX_EINVAL;
  std::unique_lock<std::mutex> lock(s->mu);
  auto it = s->reqs.find(id);
  if (it == s->reqs.end()) return GX_EINVAL;
  if (!it->second->done) {
    if (!wait) return GX_EBUSY;
    s->cv_done.wait(lock, [&] { return it->second->done || s->stop; });
    if (!it->second->done) return GX_ECANCELED;
  }
  gx::Request* r = it->second.get();
  *out = r->result;
  r->result = gx_explore_result{};
  *request_status = r->status;
  if (latency_ns) *latency_ns = r->latency_ns;
  s->reqs.erase(it);
  return GX_OK;
}

gx_status gx_server_get_stats(gx_server* s, gx_server_stats* out) {
  if (!s || !out) return GX_EINVAL;
  std::lock_guard<std::mutex> lock(s->mu);
  *out = s->stats;
  out->reserved_now = s->reserved;
  out->pooled_bytes = s->arena_bytes - s->reserved;
  out->waiting = s->waiting.size();
  return GX_OK;
}

gx_status gx_server_destroy(gx_server* s) {
  gx::destroy_server(s);
  return GX_OK;
}

}  // extern "C"
