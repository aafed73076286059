// Host paths of libcorr that a GPU run shows too late or not at all, against
// the stand-in runtime of fake_hip.cpp -- TEST INFRASTRUCTURE ONLY.
// Usage: host_paths SCENARIO; exit status 0 when its checks hold.
#include <unistd.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <thread>

#include "corr.h"
#include "fake_hip.h"

namespace {

int fails = 0;
#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::fprintf(stderr, "line %d: %s\n", __LINE__, #c);            \
      ++fails;                                                        \
    }                                                                 \
  } while (0)

corr_config config(int n_in, int n_ch) {
  corr_config c;
  std::memset(&c, 0, sizeof(c));
  c.n_inputs = n_in;
  c.n_channels = n_ch;
  c.sample_type = CORR_CI8;
  c.engine = CORR_X_I8;
  c.max_abs = 7;
  return c;
}

struct Plan {
  corr_plan* plan = nullptr;
  void* ws = nullptr;
  void* samples = nullptr;
  size_t result = 0;
  explicit Plan(const corr_config& c) {
    size_t bytes = 0;
    CHECK(corr_workspace_bytes(&c, &bytes) == CORR_OK);
    ws = fake::device_alloc(bytes);
    CHECK(corr_create(&c, ws, bytes, nullptr, &plan) == CORR_OK);
    CHECK(corr_dump_bytes(plan, CORR_DUMP_INTEG, &result) == CORR_OK);
    samples = fake::device_alloc((size_t)c.n_channels * c.n_inputs * 64 * 2);
    CHECK(corr_correlate(plan, samples, 64, 0) == CORR_OK);
  }
};

// A device destination that is too small for the result is refused, as the
// runtime's copy refuses it, and nothing is stored past it.
void dump_range() {
  for (const size_t missing : {(size_t)0, (size_t)4, (size_t)256}) {
    Plan p(config(9, 5));
    uint8_t* d = static_cast<uint8_t*>(fake::device_alloc(p.result + 64 - missing));
    int64_t n = 0;
    const corr_status st = corr_dump(p.plan, CORR_DUMP_INTEG, d + 64, 1, &n, nullptr);
    CHECK(st == (missing ? CORR_E_HIP : CORR_OK));
    fake::set_last_error(hipSuccess);   // the program has taken note of it
    CHECK(fake::stores_outside() == 0);
    CHECK(corr_destroy(p.plan) == CORR_OK);
  }
}

// A plan whose dump failed while its check was still queued: the pinned page
// that the check will write to goes to no other plan before that.
void dump_failed_in_flight() {
  Plan a(config(9, 5));
  void* small = fake::device_alloc(16);
  fake::close_streams(true);
  std::thread late([] {   // the GPU gets on only later
    std::this_thread::sleep_for(std::chrono::milliseconds(200));
    fake::close_streams(false);
  });
  CHECK(corr_dump(a.plan, CORR_DUMP_INTEG, small, 1, nullptr, nullptr) == CORR_E_HIP);
  CHECK(corr_destroy(a.plan) == CORR_OK);
  CHECK(fake::queued() == 0);
  late.join();
}

// ---------------------------------------------------------------- scheduler
// A job's fill ends once its gate is open.
struct Gate {
  std::atomic<bool> open{true};
};
void fill(void* user, uint64_t, void*, int64_t, int64_t, int64_t, int64_t, void* stream) {
  fake::queue_gate(static_cast<hipStream_t>(stream), &static_cast<Gate*>(user)->open);
}

struct Serving {
  corr_sched* s = nullptr;
  size_t room = 0;   // arena bytes for jobs
  explicit Serving(size_t arena) {
    CHECK(corr_sched_create(fake::device_alloc(arena), arena, 1, &s) == CORR_OK);
    int64_t st[8];
    CHECK(corr_sched_stats(s, st) == CORR_OK);
    room = (size_t)st[7];
  }
  uint64_t submit(int n_ch, int64_t n_samples, Gate* g, corr_fill_fn f = fill) {
    corr_job_desc d;
    std::memset(&d, 0, sizeof(d));
    d.n_inputs = 16;
    d.n_channels = n_ch;
    d.n_samples = n_samples;
    d.max_abs = 7;
    d.fill = f;
    d.fill_user = g;
    d.dst = fake::device_alloc((size_t)n_ch * 136 * 8);
    d.dst_is_device = 1;
    uint64_t id = 0;
    CHECK(corr_sched_submit(s, &d, corr_sched_now(), &id) == CORR_OK);
    return id;
  }
  void until_admitted(int64_t n) {
    int64_t st[8] = {};
    while (corr_sched_stats(s, st) == CORR_OK && st[1] < n) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  }
  bool done(uint64_t id, double seconds) {
    const double t0 = corr_sched_now();
    do {
      const corr_status st = corr_sched_poll(s, id, nullptr, nullptr, nullptr, nullptr);
      if (st != CORR_E_BUSY) return st == CORR_OK;
      std::this_thread::sleep_for(std::chrono::milliseconds(1));
    } while (corr_sched_now() - t0 < seconds);
    return false;
  }
};

// A fill whose own calls left an error behind that it has dealt with.
void fill_with_error(void*, uint64_t, void*, int64_t, int64_t, int64_t, int64_t, void*) {
  fake::set_last_error(hipErrorInvalidValue);
}

// The process ends if what follows takes longer: a call that blocks would do so for good.
void limit(int seconds, const char* what) {
  std::thread([=] {
    std::this_thread::sleep_for(std::chrono::seconds(seconds));
    std::fprintf(stderr, "still waiting: %s\n", what);
    _exit(1);
  }).detach();
}

// Jobs whose fills take their time on the GPU, one update each: submission and
// the other calls go on while all 64 slots wait.
void submit_never_blocks() {
  Serving v(64 << 20);
  Gate g;
  g.open = false;
  uint64_t id[64];
  limit(20, "a call while the fills of admitted jobs are running");
  for (int k = 0; k < 64; ++k) {
    id[k] = v.submit(2, 64, &g);
    v.until_admitted(k + 1);
  }
  g.open = true;
  for (uint64_t j : id) CHECK(v.done(j, 15.0));
  CHECK(corr_sched_destroy(v.s) == CORR_OK);
}

// Two jobs admitted together: the first one runs while the second's fill does.
void fills_overlap() {
  Serving v(2 << 20);
  Gate first, quick, slow;
  first.open = false;
  slow.open = false;
  limit(30, "a job's turn");
  const uint64_t all = v.submit(8, (int64_t)(v.room / 2048 * 8), &first);   // 256 bytes a sample: the whole arena
  v.until_admitted(1);
  const uint64_t a = v.submit(2, 64, &quick), b = v.submit(2, 64, &slow);
  int64_t st[8] = {};
  CHECK(corr_sched_stats(v.s, st) == CORR_OK && st[1] == 1 && st[4] == 2);
  first.open = true;
  CHECK(v.done(all, 5.0));
  CHECK(v.done(a, 5.0));
  slow.open = true;
  CHECK(v.done(b, 5.0));
  CHECK(corr_sched_destroy(v.s) == CORR_OK);
}

// An update that was queued is not taken for one that was not.
void error_of_a_fill() {
  Serving v(2 << 20);
  limit(30, "a job's turn");
  for (int k = 0; k < 3; ++k) CHECK(v.done(v.submit(2, 64, nullptr, fill_with_error), 5.0));
  CHECK(corr_sched_destroy(v.s) == CORR_OK);
}

const std::map<std::string, void (*)()> kScenarios = {
    {"dump_range", dump_range},
    {"dump_failed_in_flight", dump_failed_in_flight},
    {"submit_never_blocks", submit_never_blocks},
    {"fills_overlap", fills_overlap},
    {"error_of_a_fill", error_of_a_fill},
};

}  // namespace

int main(int argc, char** argv) {
  const auto it = kScenarios.find(argc == 2 ? argv[1] : "");
  if (it == kScenarios.end()) return 2;
  it->second();
  std::fflush(stderr);
  _exit(fails ? 1 : 0);   // the stand-in's thread goes with the process
}
