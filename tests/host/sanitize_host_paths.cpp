// Host-only exercise of libmona's boundary for a sanitizer build (AddressSanitizer + UndefinedBehaviorSanitizer
// on the host code; no GPU needed, see fake_hip.h): the arena layout over random lists of matrices, the argument checks
// of the entry points, and steps of states whose plan is kept, renewed and rebuilt as hyper-parameters, flags, iterations and the
// profiling level change from step to step.
// Build and run: tests/host/run_sanitizers.sh
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

static int failures = 0;
#define EXPECT(cond)                                                        \
  do {                                                                      \
    if (!(cond)) { std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); ++failures; } \
  } while (0)

// A state of random matrices through steps of every kind.
static void steps(std::mt19937& rng) {
  std::vector<mona_matrix> mats;
  const int groups = 1 + (int)(rng() % 12);
  for (int g = 0; g < groups; ++g) {
    auto side = [&] { return rng() % 2 ? 1 + (int)(rng() % 300) : 64 * (1 + (int)(rng() % (rng() % 8 ? 8 : 40))); };
    mona_matrix q;
    std::memset(&q, 0, sizeof q);
    q.m = side(); q.n = side(); q.w_dtype = rng() % 2; q.g_dtype = rng() % 2;
    q.w = reinterpret_cast<void*>((uintptr_t)16); q.g = q.w;
    mats.insert(mats.end(), 1 + rng() % (rng() % 2 ? 3 : 130), q);
  }
  const int n = (int)mats.size();
  mona_options o;
  std::memset(&o, 0, sizeof o);
  o.ns_precision = rng() % 4 == 0; o.state_dtype = rng() % 2; o.ns_schedule = rng() % 4;
  o.overlap = rng() % 2; o.max_streams = rng() % 5;
  size_t bytes = 0;
  EXPECT(mona_state_size(mats.data(), n, &o, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char stream;
  mona_state* st = nullptr;
  EXPECT(mona_init_state(mats.data(), n, &o, arena, bytes, &stream, &st) == MONA_OK);
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = 5; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  for (int k = 0; k < 10; ++k) {
    if (rng() % 2) hp.lr *= 0.9f;
    if (rng() % 3 == 0) hp.ns_steps = (int)(rng() % 70) / (rng() % 4 ? 10 : 1);
    if (rng() % 3 == 0) hp.flags = rng() % 8;
    if (rng() % 3 == 0) EXPECT(mona_set_profiling(st, rng() % 3) == MONA_OK);
    int64_t launches = 0;
    double flops = 0.0;
    EXPECT(mona_plan_info(st, hp.ns_steps, &launches, &flops, nullptr) == MONA_OK);
    EXPECT(mona_step(st, mats.data(), n, &hp, rng() % 4 ? &stream : nullptr) == MONA_OK);
    int32_t records = 0;
    if (mona_last_step_launches(st, nullptr, 0, &records) == MONA_OK) {
      std::vector<mona_launch_time> rec(records);
      EXPECT(mona_last_step_launches(st, rec.data(), records, &records) == MONA_OK);
    }
    if (rng() % 8 == 0) {            // a launch that fails half way, and the state after it
      fake::fail = "norm_finalize_kernel";
      EXPECT(mona_step(st, mats.data(), n, &hp, &stream) == MONA_EHIP);
      EXPECT(mona_step(st, mats.data(), n, &hp, &stream) == MONA_EHIP);
      size_t saved = 0;
      EXPECT(mona_state_export_size(st, &saved) == MONA_OK);
      std::vector<char> block(saved);
      EXPECT(mona_state_import(st, block.data(), saved, k, &stream) == MONA_OK);
    }
  }
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
  o.accel_form = 0;
  for (int k = 0; k < 3; ++k) {
    void* const any = reinterpret_cast<void*>((uintptr_t)256);
    const int rc = mona_step_noalloc(&mats[rng() % n], &o, any, any, any, &hp, k, &stream);
    EXPECT(rc == MONA_OK || rc == MONA_ENOMEM);
  }
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  std::mt19937 rng(12345);
  for (int round = 0; round < 60; ++round) steps(rng);
  auto dim = [&](int hi) { return 1 + (int)(rng() % hi); };
  for (int round = 0; round < 300; ++round) {
    const int count = 1 + (int)(rng() % 40);
    std::vector<mona_matrix> mats(count);
    for (auto& q : mats) {
      std::memset(&q, 0, sizeof q);
      const int kind = rng() % 4;
      q.m = kind == 0 ? dim(64) : kind == 1 ? dim(700) : 128 * dim(40);
      q.n = kind == 0 ? dim(64) : kind == 1 ? dim(700) : 128 * dim(40);
      q.w_dtype = rng() % 2;
      q.g_dtype = rng() % 2;
    }
    for (int variant = 0; variant < 12; ++variant) {
      mona_options o;
      std::memset(&o, 0, sizeof o);
      o.ns_precision = variant & 1;
      o.state_dtype = (variant >> 1) & 1;
      o.accel_form = variant % 3;
      o.ns_schedule = variant % 3;
      o.overlap = (variant >> 2) & 1;
      o.max_streams = variant % 5;
      size_t bytes = 0;
      EXPECT(mona_state_size(mats.data(), count, &o, &bytes) == MONA_OK);
      size_t least = 0;
      for (auto& q : mats) least += (size_t)q.m * q.n * 4;      // at least M itself
      EXPECT(bytes >= least);
    }
  }
  // argument checks
  size_t bytes = 0;
  mona_matrix one;
  std::memset(&one, 0, sizeof one);
  one.m = 8; one.n = 8;
  EXPECT(mona_state_size(nullptr, 1, nullptr, &bytes) == MONA_EINVAL);
  EXPECT(mona_state_size(&one, 0, nullptr, &bytes) == MONA_EINVAL);
  EXPECT(mona_state_size(&one, 1, nullptr, nullptr) == MONA_EINVAL);
  one.m = 0;
  EXPECT(mona_state_size(&one, 1, nullptr, &bytes) == MONA_EINVAL);
  one.m = 1 << 30; one.n = 4;
  EXPECT(mona_state_size(&one, 1, nullptr, &bytes) == MONA_EINVAL);
  one.m = 8; one.n = 8; one.w_dtype = 7;
  EXPECT(mona_state_size(&one, 1, nullptr, &bytes) == MONA_EINVAL);
  one.w_dtype = 0;
  mona_options bad;
  std::memset(&bad, 0, sizeof bad);
  bad.ns_schedule = 9;
  EXPECT(mona_state_size(&one, 1, &bad, &bytes) == MONA_EINVAL);
  EXPECT(std::strlen(mona_last_error()) > 0);
  mona_state* st = nullptr;
  EXPECT(mona_init_state(&one, 1, nullptr, nullptr, 0, nullptr, &st) == MONA_EINVAL && st == nullptr);
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  EXPECT(mona_step(nullptr, &one, 1, &hp, nullptr) == MONA_EINVAL);
  EXPECT(mona_step_streaming(nullptr, &one, nullptr, 1, &hp, nullptr) == MONA_EINVAL);
  EXPECT(mona_step_noalloc(&one, nullptr, nullptr, nullptr, nullptr, &hp, 0, nullptr) == MONA_EINVAL);
  EXPECT(mona_free_state(nullptr) == MONA_OK);
  mona_view v;
  EXPECT(mona_state_view(nullptr, 0, 0, &v) == MONA_EINVAL);
  EXPECT(mona_set_profiling(nullptr, 1) == MONA_EINVAL);
  mona_vector vec;
  std::memset(&vec, 0, sizeof vec);
  vec.n = 1000;
  EXPECT(mona_adamw_state_size(&vec, 1, &bytes) == MONA_OK && bytes >= 8000);
  vec.n = 0;
  EXPECT(mona_adamw_state_size(&vec, 1, &bytes) == MONA_EINVAL);
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
