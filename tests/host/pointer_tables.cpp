// Which parameter and gradient addresses the kernels of a step find: after a failed step, and with graphs replayed between
// eager steps.  Needs no GPU (fake_hip.h); built and run by tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>

using namespace mona;

static int failures = 0;
#define EXPECT(cond)                                                                                          \
  do {                                                                                                        \
    if (!(cond)) { std::printf("FAILED %s:%d: %s (%d tensors)\n", __FILE__, __LINE__, #cond, n); ++failures; } \
  } while (0)

// `n` made-up 16-byte aligned addresses for w and g; the kernels that read them are not carried out
static void name(mona_matrix* m, int n, int set) {
  for (int i = 0; i < n; ++i) {
    m[i].w = reinterpret_cast<void*>((uintptr_t)(1 + set) << 32 | (uintptr_t)(i + 1) << 8);
    m[i].g = reinterpret_cast<void*>((uintptr_t)(101 + set) << 32 | (uintptr_t)(i + 1) << 8);
  }
}

static int seen;   // the set of addresses that the last elementwise pass found, -1: none or a mixture
static void watch_matrices(int n) {
  fake::on_launch = [n](const fake::Launch& l) {
    if (l.name.find("state_update_kernel") == std::string::npos) return;
    const MatDynamic* dyn = *static_cast<const MatDynamic**>(l.args[1]);
    std::vector<mona_matrix> want(n);
    seen = -1;
    for (int set = 0; set < 20; ++set) {
      name(want.data(), n, set);
      bool all = true;
      for (int i = 0; i < n; ++i) all = all && dyn[i].w == want[i].w && dyn[i].g == want[i].g;
      if (all) seen = set;
    }
  };
}

static void matrices(int n) {
  std::vector<mona_matrix> m(n);
  std::memset(m.data(), 0, sizeof(mona_matrix) * n);
  for (auto& q : m) { q.m = 8; q.n = 16; q.w_dtype = MONA_F32; q.g_dtype = MONA_F32; }
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = 1; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  size_t bytes = 0;
  EXPECT(mona_state_size(m.data(), n, nullptr, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  void* stream = &one;
  mona_state* st = nullptr;
  EXPECT(mona_init_state(m.data(), n, nullptr, arena, bytes, stream, &st) == MONA_OK);
  watch_matrices(n);
  auto step = [&](int set) {
    name(m.data(), n, set);
    seen = -1;
    return mona_step(st, m.data(), n, &hp, stream);
  };
  for (int set : {0, 1, 1, 2, 3, 4, 5, 0}) EXPECT(step(set) == MONA_OK && seen == set);
  // the table of set 1 never gets on its way: the same call again must not take it for written
  for (const char* what : {"copy", "write_dyn"}) {
    fake::fail = what;
    const int rc = step(1);
    EXPECT(rc == MONA_EHIP || (!fake::fail.empty() && seen == 1));   // (a list uses one of the two ways)
    fake::fail.clear();
    EXPECT(step(1) == MONA_OK && seen == 1);
    EXPECT(step(0) == MONA_OK && seen == 0);
  }
  // recorded with the addresses of the last eager step, then eager steps with others around the replays
  for (int with : {0, 6}) {
    fake::clear_recorded();
    fake::capturing = true;
    EXPECT(step(with) == MONA_OK && seen == -1);
    fake::capturing = false;
    EXPECT(step(with) == MONA_OK && seen == with);   // recorded is not written
    for (int set : {1, 1, 2, 3, 4, 5, 7, 7}) {
      EXPECT(step(set) == MONA_OK && seen == set);
      seen = -1;
      fake::replay();
      EXPECT(seen == with);
    }
    EXPECT(step(0) == MONA_OK && seen == 0);
  }
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
}

static void vectors(int n) {
  std::vector<mona_vector> v(n);
  std::memset(v.data(), 0, sizeof(mona_vector) * n);
  for (auto& q : v) { q.n = 5; q.w_dtype = MONA_F32; q.g_dtype = MONA_F32; }
  size_t bytes = 0;
  EXPECT(mona_adamw_state_size(v.data(), n, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  void* stream = &one;
  mona_adamw_state* st = nullptr;
  EXPECT(mona_adamw_init_state(v.data(), n, arena, bytes, stream, &st) == MONA_OK);
  const mona_adamw_hparams hp = {0.1f, 0.9f, 0.9f, 1e-8f, 0.0f};
  struct Pair { void* w; const void* g; };
  bool right = false;
  fake::on_launch = [&](const fake::Launch& l) {
    if (l.name.find("adamw_kernel") == std::string::npos) return;
    // (stat, table in the arena, work, coefficients, dtypes, {count, table in the arguments})
    const int inline_n = *static_cast<const int*>(l.args[6]);
    const Pair* t = inline_n ? reinterpret_cast<const Pair*>(static_cast<const char*>(l.args[6]) + 8)
                             : *static_cast<const Pair**>(l.args[1]);
    right = true;
    for (int i = 0; i < n; ++i) right = right && t[i].w == v[i].w && t[i].g == v[i].g;
  };
  auto step = [&](int set) {
    std::vector<mona_matrix> m(n);
    name(m.data(), n, set);
    for (int i = 0; i < n; ++i) { v[i].w = m[i].w; v[i].g = m[i].g; }
    right = false;
    return mona_adamw_step(st, v.data(), n, &hp, stream);
  };
  for (int set : {0, 1, 1, 2, 3, 4, 5, 0}) EXPECT(step(set) == MONA_OK && right);
  fake::fail = "copy";
  const int rc = step(1);
  EXPECT(rc == MONA_EHIP || (!fake::fail.empty() && right));
  fake::fail.clear();
  EXPECT(step(1) == MONA_OK && right);
  fake::on_launch = nullptr;
  EXPECT(mona_adamw_free_state(st) == MONA_OK);
  std::free(arena);
}

int main() {
  for (int n : {1, 2, 96, 97, 193, 388}) matrices(n);
  for (int n : {1, 128, 129, 300}) vectors(n);
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
