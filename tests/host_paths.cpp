// Host paths of libcorr that a GPU run shows too late or not at all, against
// the stand-in runtime of fake_hip.cpp -- TEST INFRASTRUCTURE ONLY.
// Usage: host_paths SCENARIO; exit status 0 when its checks hold.
#include <unistd.h>

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

const std::map<std::string, void (*)()> kScenarios = {
    {"dump_range", dump_range},
    {"dump_failed_in_flight", dump_failed_in_flight},
};

}  // namespace

int main(int argc, char** argv) {
  const auto it = kScenarios.find(argc == 2 ? argv[1] : "");
  if (it == kScenarios.end()) return 2;
  it->second();
  std::fflush(stderr);
  _exit(fails ? 1 : 0);   // the stand-in's thread goes with the process
}
