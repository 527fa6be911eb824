// Which launches a call makes, on the CPU stand-in of the HIP runtime: every
// launch of the likelihood kernel is noted with its tile and whether it is the
// one-launch kernel of small thin batches.  Test infrastructure only.
//
//   1. the one-launch rule on both sides of each of its lines, from device and
//      host memory, on results over the rows and after fgl_set_tile;
//   2. the tuner times its candidates as three launches, where the tuned batch
//      itself is one launch too, and a tile of the bucket is the one it measured;
//   3. kernel timing covers the likelihood kernel alone;
//   4. cache entries of such buckets from timings of the one-launch kernel are
//      not used, others are.
// Prints "checks failed: 0" when all hold.
#define launch_main stand_in_launch_main
#include "launch_stub.cpp"
#undef launch_main

#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <unistd.h>

#include "../../include/fgl.h"
#include "../../paper_2603_13196_amd/csrc/fgl_host.h"

namespace {

struct Launch {
  int rows;            // thin_rows
  fgl::Tile tile;
};
std::vector<Launch> g_seen;
int g_slow_waves = 0;  // launches of other tiles take longer
long g_fail = 0;

#define CHECK(cond, ...)                          \
  do {                                            \
    if (!(cond)) {                                \
      std::fprintf(stderr, "FAIL line %d: ", __LINE__); \
      std::fprintf(stderr, __VA_ARGS__);          \
      std::fprintf(stderr, " (%s)\n", fgl_last_error()); \
      ++g_fail;                                   \
    }                                             \
  } while (0)

}  // namespace

namespace fgl {
hipError_t launch_main(Kind k, const DevModel& m, const Work& w, const Tile& tile, hipStream_t s) {
  g_seen.push_back({w.thin_rows, tile});
  if (g_slow_waves && !w.thin_rows && tile.waves != g_slow_waves) {
    const hipError_t e = stub_enqueue(s, [] { usleep(1500); });
    if (e != hipSuccess) return e;
  }
  return stand_in_launch_main(k, m, w, tile, s);
}
}  // namespace fgl

namespace {

fgl_model* model(int N, int F, int T) {
  std::vector<float> K((size_t)N * F * T, 0.5f);
  for (size_t k = 0; k < K.size(); ++k) K[k] += 0.25f * (float)(k % 7);
  std::vector<double> nu(F), D((size_t)F * T, 3.0);
  for (int f = 0; f < F; ++f) nu[f] = 50.0 + f;
  fgl_model* m = nullptr;
  CHECK(fgl_model_create(K.data(), nu.data(), D.data(), 100.0, N, F, T, 2.7, 0, &m) == FGL_OK, "create");
  CHECK(fgl_mixed_form(m) == FGL_FORM_THIN, "N%d T%d is not thin", N, T);
  return m;
}

// the launches of one call: rows per workgroup of its one launch, 0 for three
int host_call(fgl_model* m, int B) {
  const int P = fgl_model_nparams(m);
  std::vector<double> th((size_t)B * P, 0.5), out(B);
  g_seen.clear();
  CHECK(fgl_loglike_batch(m, th.data(), B, out.data(), FGL_PREC_MIXED) == FGL_OK, "host call");
  return g_seen.empty() ? 0 : g_seen.back().rows;    // a replayed graph launches nothing here
}
int device_call(fgl_model* m, int B, bool over = false) {
  const int P = fgl_model_nparams(m);
  double *th = nullptr, *out = nullptr;
  CHECK(hipMalloc(reinterpret_cast<void**>(&th), (size_t)B * P * 8) == hipSuccess, "alloc");
  CHECK(hipMalloc(reinterpret_cast<void**>(&out), (size_t)B * 8) == hipSuccess, "alloc");
  for (int k = 0; k < B * P; ++k) th[k] = 0.5;
  g_seen.clear();
  CHECK(fgl_loglike_batch_device(m, th, B, over ? th : out, FGL_PREC_MIXED, nullptr) == FGL_OK, "device call");
  CHECK(g_seen.size() == 1, "%zu likelihood launches", g_seen.size());
  (void)hipDeviceSynchronize();
  (void)hipFree(th);
  (void)hipFree(out);
  return g_seen.back().rows;
}

void rule() {
  struct Line { int N, F, T, B, device, host; };
  const Line lines[] = {
      {4, 151, 1, 1, 4, 4},     {4, 151, 1, 1024, 4, 4}, {4, 151, 1, 1025, 8, 8},
      {4, 151, 1, 2048, 8, 8},  {4, 151, 1, 2049, 0, 0},             // rows
      {16, 120, 10, 2000, 8, 8}, {4, 120, 30, 2000, 0, 0},           // a channel's cost, eight rows
      {16, 120, 20, 900, 4, 4}, {16, 151, 20, 900, 4, 4},            // and four
      {8, 120, 40, 900, 4, 4},  {8, 120, 45, 900, 0, 0},
      {32, 301, 1, 1000, 4, 4}, {8, 301, 20, 500, 0, 0},             // turns
      // faster in one launch only where the rows are copied otherwise
      {3, 395, 2, 1292, 0, 8},  {4, 301, 9, 300, 0, 4}, {4, 301, 8, 300, 4, 4}, {2, 200, 45, 1, 0, 4},
      {30, 301, 1, 1, 0, 4},    {12, 301, 7, 300, 0, 4}, {12, 301, 4, 300, 4, 4},
  };
  for (const Line& l : lines) {
    fgl_model* m = model(l.N, l.F, l.T);
    CHECK(device_call(m, l.B) == l.device, "N%d F%d T%d B%d: rows %d, not %d", l.N, l.F, l.T, l.B,
          g_seen.back().rows, l.device);
    CHECK(host_call(m, l.B) == l.host, "host N%d F%d T%d B%d", l.N, l.F, l.T, l.B);
    CHECK(device_call(m, l.B, true) == 0, "over the rows: N%d F%d T%d B%d", l.N, l.F, l.T, l.B);
    CHECK(fgl_model_destroy(m) == FGL_OK, "destroy");
  }
}

void chosen_tiles() {
  fgl_model* m = model(4, 151, 1);
  CHECK(device_call(m, 1000) == 4, "one launch");
  for (int waves : {1, 2, 4}) {
    CHECK(fgl_set_tile(m, 1000, FGL_PREC_MIXED, waves, 4, 2) == FGL_OK, "set_tile");
    CHECK(device_call(m, 1000) == 0 && g_seen.back().tile.waves == waves, "tile %d does not run", waves);
    CHECK(host_call(m, 900) == 0, "host call after set_tile");
    CHECK(device_call(m, 400) == 4, "another size class");
  }
  CHECK(fgl_tune(m, 1000, FGL_PREC_MIXED) == FGL_OK, "tune");
  CHECK(device_call(m, 1000) == 4, "one launch after a tuning");
  CHECK(fgl_model_destroy(m) == FGL_OK, "destroy");
  // the same where calls are replayed: a call captured as one launch, then the
  // default tile forced
  setenv("FGL_DEVICE_GRAPHS", "1", 1);
  m = model(4, 151, 1);
  unsetenv("FGL_DEVICE_GRAPHS");
  const int B = 1000, P = fgl_model_nparams(m);
  double *th = nullptr, *out = nullptr;
  CHECK(hipMalloc(reinterpret_cast<void**>(&th), (size_t)B * P * 8) == hipSuccess, "alloc");
  CHECK(hipMalloc(reinterpret_cast<void**>(&out), (size_t)B * 8) == hipSuccess, "alloc");
  for (int k = 0; k < B * P; ++k) th[k] = 0.5;
  auto calls = [&](int rows) {
    for (int c = 0; c < 4; ++c) {                     // eager, captured, replayed
      g_seen.clear();
      CHECK(fgl_loglike_batch_device(m, th, B, out, FGL_PREC_MIXED, nullptr) == FGL_OK, "replayed call");
      (void)hipDeviceSynchronize();
      CHECK(g_seen.size() == (c < 2 ? 1u : 0u) && (c > 1 || g_seen[0].rows == rows), "replayed call %d", c);
    }
  };
  calls(4);
  int waves = 0, chans = 0, occ = 0;
  CHECK(fgl_get_tile(m, B, FGL_PREC_MIXED, &waves, &chans, &occ) == FGL_OK, "get_tile");
  CHECK(fgl_set_tile(m, B, FGL_PREC_MIXED, waves, chans, occ) == FGL_OK, "set_tile");
  calls(0);
  CHECK(fgl_model_destroy(m) == FGL_OK, "destroy");
  (void)hipFree(th);
  (void)hipFree(out);
}

void tuning(const char* path) {
  std::remove(path);
  CHECK(fgl_tune_cache(path) == FGL_OK, "cache");
  for (int fast : {1, 2, 4}) {
    fgl_model* m = model(4, 151, 1);
    g_seen.clear();
    g_slow_waves = fast;
    CHECK(fgl_tune(m, 1000, FGL_PREC_MIXED) == FGL_OK, "tune");
    g_slow_waves = 0;
    for (const Launch& l : g_seen) CHECK(l.rows == 0, "a candidate was timed in one launch");
    int waves = 0;
    CHECK(fgl_get_tile(m, 1000, FGL_PREC_MIXED, &waves, nullptr, nullptr) == FGL_OK && waves == fast,
          "tuned to %d waves, not %d", waves, fast);
    CHECK(device_call(m, 1000) == 4, "one launch after a tuning");
    CHECK(device_call(m, 1000, true) == 0 && g_seen.back().tile.waves == fast, "its tile in three");
    CHECK(fgl_model_destroy(m) == FGL_OK, "destroy");
  }
}

void saved_tiles(const char* path) {
  std::string kept, line;
  FILE* f = std::fopen(path, "r");
  char buf[512];
  while (f && std::fgets(buf, sizeof buf, f))
    if (std::strstr(buf, "\"bucket\":1024")) line = buf;
  if (f) std::fclose(f);
  CHECK(line.find(",\"staged\":1,\"waves\":4") != std::string::npos, "cache line %s", line.c_str());
  // the same entry as an earlier library wrote it, and one of a bucket past the line
  std::string old = line;
  const size_t at = old.find(",\"staged\":1");
  if (at != std::string::npos) old.erase(at, std::strlen(",\"staged\":1"));
  std::string far = old;
  far.replace(far.find("1024"), 4, "4096");
  for (std::string* l : {&old, &far}) l->replace(l->find("\"F\":151"), 7, "\"F\":150");
  f = std::fopen(path, "w");
  std::fprintf(f, "%s%s", old.c_str(), far.c_str());
  std::fclose(f);
  CHECK(fgl_tune_cache(path) == FGL_OK, "cache");
  fgl_model* m = model(4, 150, 1);
  int w1 = 0, w4 = 0, d1 = 0;
  CHECK(fgl_get_tile(m, 1000, FGL_PREC_MIXED, &w1, nullptr, nullptr) == FGL_OK, "tile");
  CHECK(fgl_get_tile(m, 300, FGL_PREC_MIXED, &d1, nullptr, nullptr) == FGL_OK, "tile");
  CHECK(fgl_get_tile(m, 4000, FGL_PREC_MIXED, &w4, nullptr, nullptr) == FGL_OK, "tile");
  CHECK(w1 == d1 && w1 != 4, "the old entry was used: %d waves", w1);
  CHECK(w4 == 4, "an entry of three launches was not: %d waves", w4);
  CHECK(fgl_model_destroy(m) == FGL_OK, "destroy");
  CHECK(fgl_tune_cache(nullptr) == FGL_OK, "cache");
}

void timing() {
  fgl_model* m = model(4, 151, 1);
  CHECK(device_call(m, 500) == 4, "one launch");
  CHECK(fgl_kernel_timing(m, 2) == FGL_OK, "timing");
  for (int c = 0; c < 6; ++c) CHECK(device_call(m, 500) == (c % 2 ? 4 : 0), "timed call %d", c);
  for (int c = 0; c < 4; ++c) CHECK(host_call(m, 500) == (c % 2 ? 4 : 0), "timed host call %d", c);
  double ms = 0.0;
  int64_t n = 0;
  CHECK(fgl_kernel_time(m, &ms, &n) == FGL_OK && n == 5, "%lld recorded", (long long)n);
  CHECK(fgl_kernel_timing(m, 0) == FGL_OK, "timing");
  CHECK(device_call(m, 500) == 4, "one launch");
  CHECK(fgl_model_destroy(m) == FGL_OK, "destroy");
}

}  // namespace

int main(int argc, char** argv) {
  const std::string path = argc > 1 ? argv[1] : "route_tiles.jsonl";
  rule();
  chosen_tiles();
  tuning(path.c_str());
  saved_tiles(path.c_str());
  timing();
  std::printf("checks failed: %ld, stand-in reports: %ld\n", g_fail, stub_errors());
  return g_fail || stub_errors() ? 1 : 0;
}
