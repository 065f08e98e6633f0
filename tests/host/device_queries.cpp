// When the device is asked for its architecture: never to size an arena, for the state's own device when a state is built, and
// again after a query that failed.  Needs no GPU (fake_hip.h); built and run by tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>

using namespace mona;

static int failures = 0;
#define EXPECT(cond)                                                                              \
  do {                                                                                            \
    if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); ++failures; }            \
  } while (0)

// launches of the kernels that are planned for this architecture only, in a step of matrices with a workgroup each, one of a
// chain, and one without allocation
static int particular_launches() {
  int seen = 0;
  fake::on_launch = [&](const fake::Launch& l) {
    seen += l.name.find("ns_matrix_kernel") != std::string::npos || l.name.find("ns_chain_kernel") != std::string::npos;
  };
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = 5; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  char stream;
  for (int n : {200, 1}) {
    mona_matrix q;
    std::memset(&q, 0, sizeof q);
    q.m = n == 1 ? 256 : 100; q.n = n == 1 ? 512 : 128;
    q.w = reinterpret_cast<void*>((uintptr_t)16); q.g = q.w;
    const std::vector<mona_matrix> m(n, q);
    size_t bytes = 0;
    const int before = fake::queries;
    EXPECT(mona_state_size(m.data(), n, nullptr, &bytes) == MONA_OK);
    EXPECT(fake::queries == before);
    char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
    mona_state* st = nullptr;
    EXPECT(mona_init_state(m.data(), n, nullptr, arena, bytes, &stream, &st) == MONA_OK);
    EXPECT(mona_step(st, m.data(), n, &hp, &stream) == MONA_OK);
    EXPECT(mona_free_state(st) == MONA_OK);
    std::free(arena);
    if (n > 1) continue;
    void* const any = reinterpret_cast<void*>((uintptr_t)256);
    EXPECT(mona_step_noalloc(&q, nullptr, any, any, any, &hp, 0, &stream) == MONA_OK);
  }
  fake::on_launch = nullptr;
  return seen;
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  fake::device = 3;
  fake::fail = "attribute";
  EXPECT(particular_launches() == 2);      // (the first state's query failed: products in launches there)
  EXPECT(fake::fail.empty());
  EXPECT(particular_launches() == 3);
  fake::device = 5;                        // another device, of another architecture
  fake::capability_minor = 4;
  EXPECT(particular_launches() == 0);
  fake::device = 3;
  EXPECT(particular_launches() == 3);
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
