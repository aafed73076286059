// Every order in which one update of the serving queue and the claims of
// running workgroups can take effect -- TEST INFRASTRUCTURE ONLY.
//
// serve_claim and serve_publish (serve_queue.h) are the code that the kernels
// run; here their memory type hands each load, store and atomic to a scheduler
// that decides which takes effect next.  Loads issued together may be answered
// in any order, and stores may land in any order until settle() has waited for
// them.  The search is exhaustive up to the order of operations that do not
// touch the same word (sleep sets).
//
// Checked in every execution: a claimed item exists, belongs to the job whose
// record the slot holds, and is claimed once; the host is told "last item" for
// the last one only; the workgroup that claims an item sees the samples of its
// job (a word that stands for them is stored ahead of the update, and an
// acquire is a load of it); and, once the update has been applied, any one of
// the workgroups would claim all that is left in one turn of the list.
// Usage: serve_model SCENARIO; exit status 0 and the number of executions, or 1
// and the first faulty one.
#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "serve_queue.h"

using namespace corr;

namespace {

constexpr int kSlotsUsed = 4;
constexpr uint32_t kVersion = 7;   // of the list that the workgroups have seen; the update is the next one

// ------------------------------------------------------------------ scenario
struct JobSpec {
  int slot;
  uint32_t gen;
  int n_items;
};
struct Scenario {
  std::vector<JobSpec> before;   // jobs of the list that the workgroups have seen, all items claimed and done
  std::vector<JobSpec> live;     // jobs of that list with no item claimed yet
  std::vector<JobSpec> next;     // jobs that the update publishes
  std::vector<int> list;         // slots listed by the update
  int claimers, calls;           // workgroups, and claims that each tries
};

// ------------------------------------------------------------------- memory
struct Memory {
  ServeJob slots[kServeSlots];
  uint64_t claim[kServeSlots * kServeLine / 2];
  uint32_t done[kServeSlots * kServeLine];
  uint64_t active[1 + 2 * kServeSlots];
  uint64_t host[kServeSlots * kServeLine / 2];
  uint64_t last_claim;
  uint64_t samples;              // number of the latest update whose jobs' samples are in memory
  uint32_t closing, host_closing;
} mem;

ServeQueue queue() {
  ServeQueue q;
  std::memset(&q, 0, sizeof(q));
  q.slots = mem.slots;
  q.claim = mem.claim;
  q.done = mem.done;
  q.active = mem.active;
  q.last_claim = &mem.last_claim;
  q.closing = &mem.closing;
  q.host_closing = &mem.host_closing;
  q.host_claimed = mem.host;
  q.gen = 1;
  q.n_slots = kServeSlots;
  q.max_polls = 1;
  return q;
}

// ---------------------------------------------------------------- scheduler
enum Kind { kLoad, kStore, kAdd };
struct Op {
  int actor = 0, seq = 0;
  Kind kind = kLoad;
  uint64_t* addr = nullptr;
  uint64_t value = 0;
  uint64_t* out = nullptr;
};
struct Actor {
  ucontext_t ctx;
  std::vector<char> stack;
  std::function<void()> body;
  std::vector<Op> pending;
  int seq = 0;
  bool finished = false, barrier = false, publisher = false;
};
std::vector<Actor>* actors;
ucontext_t home;
int running = -1;               // the actor that runs; -1: operations take effect at once
std::vector<Op> trace;
std::string fault;

void fail(const std::string& what) {
  if (fault.empty()) fault = what;
}

void apply(const Op& o) {
  switch (o.kind) {
    case kLoad: *o.out = *o.addr; break;
    case kStore: *o.addr = o.value; break;
    case kAdd:
      *o.out = *o.addr;
      *o.addr += o.value;
      break;
  }
}

// Words whose order of access matters; anything else takes effect at once.
bool watched(const uint64_t* p) {
  if (p >= mem.active && p < mem.active + 1 + 2 * kServeSlots) return true;
  if (p >= mem.claim && p < mem.claim + kServeSlots * kServeLine / 2) return true;
  for (int s = 0; s < kSlotsUsed; ++s)
    if (p == &mem.slots[s].ident) return true;
  return p == &mem.samples;
}

void post(Kind k, const uint64_t* p, uint64_t value, uint64_t* out) {
  Op o;
  o.kind = k;
  o.addr = const_cast<uint64_t*>(p);
  o.value = value;
  o.out = out;
  if (running < 0 || !watched(p)) {
    apply(o);
    return;
  }
  Actor& a = (*actors)[running];
  o.actor = running;
  o.seq = a.seq++;
  a.pending.push_back(o);
}

void pause() {
  if (running < 0) return;
  Actor& a = (*actors)[running];
  swapcontext(&a.ctx, &home);
}
void wait_all() {
  while (running >= 0 && !(*actors)[running].pending.empty()) pause();
}

// The memory type of serve_claim and serve_publish.
struct ModelMemory {
  uint64_t load(const uint64_t* p) {
    uint64_t v = 0;
    post(kLoad, p, 0, &v);
    wait_all();
    return v;
  }
  uint32_t load_agent(const uint32_t* p) { return *p; }
  void load2(const uint64_t* p0, const uint64_t* p1, uint64_t& v0, uint64_t& v1) {
    post(kLoad, p0, 0, &v0);
    post(kLoad, p1, 0, &v1);
    wait_all();
  }
  void add_load(uint64_t* claim, const uint64_t* p, uint64_t& w, uint64_t& v) {
    post(kAdd, claim, 1, &w);
    post(kLoad, p, 0, &v);
    wait_all();
  }
  void store(uint64_t* p, uint64_t v) { post(kStore, p, v, nullptr); }
  void exchange(uint64_t* p, uint64_t v) { post(kStore, p, v, nullptr); }
  void exchange(uint32_t* p, uint32_t v) { *p = v; }
  void settle() {
    wait_all();
    if (running < 0) return;
    (*actors)[running].barrier = true;
    pause();
  }
  void claimed(const ServeQueue&) {}
  bool idle(const ServeQueue&) { return false; }
};

// ------------------------------------------------------------------- checks
struct Ledger {
  std::set<std::pair<int, uint64_t>> claims;   // (slot, claim word)
} ledger;
std::map<std::pair<int, uint32_t>, int> items_of;   // (slot, generation) -> items

void check_claim(int slot, uint64_t w) {
  const uint32_t gen = (uint32_t)(w >> 32), item = (uint32_t)w;
  char msg[160];
  const auto it = items_of.find({slot, gen});
  if (it == items_of.end() || item >= (uint32_t)it->second) {
    std::snprintf(msg, sizeof(msg), "item %u of slot %d generation %u claimed, which has %d items", item, slot, gen,
                  it == items_of.end() ? 0 : it->second);
    fail(msg);
  } else if (mem.slots[slot].x.n_items != it->second || (uint32_t)(mem.slots[slot].ident >> 32) != gen) {
    std::snprintf(msg, sizeof(msg), "slot %d generation %u claimed, but the record is another job's", slot, gen);
    fail(msg);
  }
  if (!ledger.claims.insert({slot, w}).second) {
    std::snprintf(msg, sizeof(msg), "item %u of slot %d generation %u claimed twice", item, slot, gen);
    fail(msg);
  }
}

void check_host() {
  for (int s = 0; s < kSlotsUsed; ++s) {
    const uint64_t gen = mem.host[s * (kServeLine / 2) + 1];
    const auto it = items_of.find({s, (uint32_t)gen});
    if (it == items_of.end()) continue;
    const uint64_t w = mem.claim[s * (kServeLine / 2)];
    if ((uint32_t)(w >> 32) == (uint32_t)gen && (uint32_t)w < (uint32_t)it->second)
      fail("the host is told that a job with unclaimed items is claimed");
  }
}

// ---------------------------------------------------------------- execution
ServeJob record(const JobSpec& j) {
  ServeJob r;
  std::memset(&r, 0, sizeof(r));
  r.x.n_items = j.n_items;
  r.ident = serve_ident(j.gen, j.n_items);
  return r;
}

ServeUpdate update;
const Scenario* scene;
std::vector<ServeView> views;

// All that is left goes to workgroup c, without another update.
void check_rest(int c) {
  const Memory saved = mem;
  const Ledger claims = ledger;
  ModelMemory m;
  const ServeQueue q = queue();
  ServeView v = views[c];
  uint64_t w = 0;
  for (int slot = serve_claim(m, q, v, &w); slot >= 0; slot = serve_claim(m, q, v, &w)) check_claim(slot, w);
  for (const JobSpec& j : scene->live)
    for (int k = 0; k < j.n_items; ++k)
      if (!ledger.claims.count({j.slot, (uint64_t)j.gen << 32 | (uint64_t)k})) fail("a workgroup ignores a listed job");
  for (const JobSpec& j : scene->next)
    for (int k = 0; k < j.n_items; ++k)
      if (!ledger.claims.count({j.slot, (uint64_t)j.gen << 32 | (uint64_t)k})) fail("a workgroup ignores a listed job");
  mem = saved;
  ledger = claims;
}

void claimer(int c) {
  ModelMemory m;
  const ServeQueue q = queue();
  uint64_t seen = kVersion;
  for (int k = 0; k < scene->calls; ++k) {
    uint64_t w = 0;
    const int slot = serve_claim(m, q, views[c], &w);
    if (slot < 0) continue;
    check_claim(slot, w);
    if (views[c].acquire) seen = m.load(&mem.samples);
    if (seen < (w >> 32)) fail("an item is multiplied without its job's samples having been acquired");
  }
  wait_all();
}

void setup(std::vector<Actor>& as) {
  std::memset(&mem, 0, sizeof(mem));
  std::memset(&update, 0, sizeof(update));
  ledger = Ledger{};
  items_of.clear();
  trace.clear();
  fault.clear();
  mem.samples = kVersion;
  int n = 0;
  std::map<int, JobSpec> jobs;
  for (const JobSpec& j : scene->before) jobs[j.slot] = j;
  for (const JobSpec& j : scene->live) jobs[j.slot] = j;
  for (auto& kv : jobs) {
    const JobSpec& j = kv.second;
    bool is_live = false;
    for (const JobSpec& l : scene->live) is_live = is_live || l.slot == j.slot;
    mem.slots[j.slot] = record(j);
    mem.claim[j.slot * (kServeLine / 2)] = (uint64_t)j.gen << 32 | (uint64_t)(is_live ? 0 : j.n_items);
    mem.active[1 + n++] = (uint64_t)j.slot;
    items_of[{j.slot, j.gen}] = j.n_items;
  }
  mem.active[0] = (uint64_t)kVersion << 32 | (uint64_t)n;
  for (size_t k = 0; k < scene->next.size(); ++k) {
    const JobSpec& j = scene->next[k];
    update.slot[k] = j.slot;
    update.job[k] = record(j);
    items_of[{j.slot, j.gen}] = j.n_items;
    jobs[j.slot] = j;
  }
  for (size_t k = 0; k < scene->list.size(); ++k) update.active[k] = (uint64_t)scene->list[k];
  views.assign(scene->claimers, ServeView{0, (uint32_t)n, kVersion, 0, kVersion, false, false});
  for (int c = 0; c < scene->claimers; ++c) views[c].turn = (uint32_t)c;

  const int nt = (int)std::max(scene->next.size(), scene->list.size()) + 1;
  as.clear();
  as.resize(nt + scene->claimers);
  for (int t = 0; t < nt; ++t) {
    as[t].publisher = true;
    as[t].body = [t, nt] {
      ModelMemory m;
      if (t == 0) m.store(&mem.samples, kVersion + 1);
      m.settle();   // the samples are there before the update's kernel starts
      serve_publish(m, &update, (int)scene->next.size(), (int)scene->list.size(), kVersion + 1, queue(), t, nt);
      wait_all();
    };
  }
  for (int c = 0; c < scene->claimers; ++c) as[nt + c].body = [c] { claimer(c); };
}

void entry_point(int k) {
  (*actors)[k].body();
  (*actors)[k].finished = true;
  running = -1;
  swapcontext(&(*actors)[k].ctx, &home);
}

void resume(int k) {
  running = k;
  swapcontext(&home, &(*actors)[k].ctx);
  running = -1;
}

// Publisher threads that have all arrived go on.
void barriers() {
  for (;;) {
    bool all = true, any = false;
    for (Actor& a : *actors)
      if (a.publisher) {
        all = all && a.barrier;
        any = any || a.barrier;
      }
    if (!any || !all) return;
    for (size_t k = 0; k < actors->size(); ++k)
      if ((*actors)[k].publisher) (*actors)[k].barrier = false;
    for (size_t k = 0; k < actors->size(); ++k)
      if ((*actors)[k].publisher) resume((int)k);
  }
}

void start(std::vector<Actor>& as) {
  actors = &as;
  for (size_t k = 0; k < as.size(); ++k) {
    as[k].stack.resize(64 << 10);
    getcontext(&as[k].ctx);
    as[k].ctx.uc_stack.ss_sp = as[k].stack.data();
    as[k].ctx.uc_stack.ss_size = as[k].stack.size();
    as[k].ctx.uc_link = &home;
    makecontext(&as[k].ctx, reinterpret_cast<void (*)()>(entry_point), 1, (int)k);
  }
  for (size_t k = 0; k < as.size(); ++k) resume((int)k);
  barriers();
}

std::vector<Op> enabled() {
  std::vector<Op> e;
  for (Actor& a : *actors) e.insert(e.end(), a.pending.begin(), a.pending.end());
  return e;
}

void step(const Op& o) {
  Actor& a = (*actors)[o.actor];
  for (size_t k = 0; k < a.pending.size(); ++k)
    if (a.pending[k].seq == o.seq) {
      const Op p = a.pending[k];
      apply(p);
      trace.push_back(p);
      a.pending.erase(a.pending.begin() + k);
      break;
    }
  if (a.pending.empty() && !a.finished && !a.barrier) resume(o.actor);
  barriers();
}

bool independent(const Op& a, const Op& b) { return a.addr != b.addr || (a.kind == kLoad && b.kind == kLoad); }

long executions = 0;
std::vector<Op> prefix;

std::string name_of(const uint64_t* p) {
  char s[64];
  if (p >= mem.active && p < mem.active + 1 + 2 * kServeSlots) {
    std::snprintf(s, sizeof(s), p == mem.active ? "head" : "list[%d]", (int)(p - mem.active) - 1);
  } else if (p >= mem.claim && p < mem.claim + kServeSlots * kServeLine / 2) {
    std::snprintf(s, sizeof(s), "claim[%d]", (int)((p - mem.claim) / (kServeLine / 2)));
  } else {
    std::snprintf(s, sizeof(s), p == &mem.samples ? "samples" : "identity");
  }
  return s;
}

bool report() {
  if (fault.empty()) return true;
  std::printf("FAULT after %ld executions: %s\n", executions, fault.c_str());
  for (const Op& o : trace)
    std::printf("  %s %d: %s %s\n", (*actors)[o.actor].publisher ? "update" : "workgroup", o.actor,
                o.kind == kLoad ? "load" : o.kind == kStore ? "store" : "add", name_of(o.addr).c_str());
  return false;
}

bool explore(std::vector<Op> sleep) {
  std::vector<Actor> as;
  setup(as);
  start(as);
  for (const Op& o : prefix) step(o);
  check_host();
  if (!report()) return false;
  const std::vector<Op> en = enabled();
  if (en.empty()) {
    ++executions;
    for (int c = 0; c < scene->claimers; ++c) check_rest(c);
    return report();
  }
  auto same = [](const Op& a, const Op& b) { return a.actor == b.actor && a.seq == b.seq; };
  for (const Op& t : en) {
    bool asleep = false;
    for (const Op& z : sleep) asleep = asleep || same(z, t);
    if (asleep) continue;
    std::vector<Op> child;
    for (const Op& z : sleep)
      if (independent(z, t)) child.push_back(z);
    prefix.push_back(t);
    const bool ok = explore(child);
    prefix.pop_back();
    if (!ok) return false;
    sleep.push_back(t);
  }
  return true;
}

const std::map<std::string, Scenario>& scenarios() {
  static const std::map<std::string, Scenario> all = {
      // a slot's next job in the same place of the list, with fewer, more and as many items
      {"shrinking", {{{3, 5, 4}}, {}, {{3, 8, 1}}, {3}, 2, 2}},
      {"growing", {{{3, 5, 1}}, {}, {{3, 8, 3}}, {3}, 2, 2}},
      {"equal", {{{3, 5, 2}}, {}, {{3, 8, 2}}, {3}, 2, 2}},
      // the place goes to another slot
      {"moved", {{{1, 5, 4}}, {}, {{2, 8, 2}}, {2}, 2, 2}},
      // the list grows in front of a job that has unclaimed items, and shrinks
      {"longer", {{{1, 4, 3}}, {{3, 5, 2}}, {{2, 8, 1}}, {2, 3}, 1, 4}},
      {"shorter", {{{1, 4, 3}, {2, 6, 4}}, {}, {{2, 8, 2}}, {2}, 1, 4}},
  };
  return all;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 2) {
    for (auto& kv : scenarios()) std::printf("%s\n", kv.first.c_str());
    return 0;
  }
  const auto it = scenarios().find(argv[1]);
  if (it == scenarios().end()) return 2;
  scene = &it->second;
  if (!explore({})) return 1;
  std::printf("%s: %ld executions\n", argv[1], executions);
  return 0;
}
