// The plan that a state keeps takes up each step's hyper-parameters: the launches of a state whose hyper-parameters change from
// step to step against those of a fresh state.  Needs no GPU (fake_hip.h); built and run by tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <tuple>

using namespace mona;

static int failures = 0;
static std::string what;
#define EXPECT(cond)                                                                                   \
  do {                                                                                                 \
    if (!(cond)) { std::printf("FAILED line %d: %s (%s)\n", __LINE__, #cond, what.c_str()); ++failures; } \
  } while (0)

typedef std::vector<std::tuple<int, int, int>> Shapes;   // count, m, n

// everything of the product launches that hyper-parameters enter
static std::vector<float> figures;
static int kinds_seen[4];
static void note(const fake::Launch& l) {
  auto step = [&](const StepDesc& s) { figures.insert(figures.end(), {s.ns_a, s.ns_b, s.ns_c, s.w_keep}); };
  auto product = [&](const GemmArgs& a) {
    figures.insert(figures.end(), {a.alpha, a.beta, a.diag, a.w_keep, a.o_scale, (float)a.store_out, (float)a.epilogue, (float)a.K});
  };
  if (l.name.find("ns_matrix_kernel") != std::string::npos) {
    const MatrixBatch& b = *static_cast<const MatrixBatch*>(l.args[0]);
    step(b.step);
    figures.insert(figures.end(), {(float)b.steps, (float)b.store_o});
    for (int i = 0; i < b.n; ++i) figures.push_back(b.group[i].o_scale);
    ++kinds_seen[0];
  } else if (l.name.find("ns_chain_kernel") != std::string::npos) {
    const ChainArgs& c = *static_cast<const ChainArgs*>(l.args[0]);
    step(c.step);
    for (int i = 0; i < c.ops; ++i) {
      GemmArgs a;
      expand_op(c.step, c.group[c.op[i].code >> OPF_GROUP], c.op[i].code, a);
      product(a);
    }
    ++kinds_seen[1];
  } else if (l.name.find("ns_small_kernel") != std::string::npos) {
    const GemmBatch& b = *static_cast<const GemmBatch*>(l.args[0]);
    for (int i = 0; i < b.n; ++i) product(b.a[i]);
    ++kinds_seen[2];
  } else if (l.name.find("ns_gemm_bf16_dma_kernel") != std::string::npos) {
    product(*static_cast<const GemmArgs*>(l.args[0]));
    ++kinds_seen[3];
  }
}

static void run(const Shapes& shapes, int precision, int schedule, std::mt19937& rng) {
  std::vector<mona_matrix> m;
  what = "precision " + std::to_string(precision) + ", schedule " + std::to_string(schedule);
  for (auto [count, rows, cols] : shapes) {
    what += ", " + std::to_string(count) + "*" + std::to_string(rows) + "*" + std::to_string(cols);
    for (int i = 0; i < count; ++i) {
      mona_matrix q;
      std::memset(&q, 0, sizeof q);
      q.m = rows; q.n = cols; q.w_dtype = MONA_F32; q.g_dtype = MONA_F32;
      q.w = reinterpret_cast<void*>((uintptr_t)16); q.g = q.w;
      m.push_back(q);
    }
  }
  mona_options o;
  std::memset(&o, 0, sizeof o);
  o.ns_precision = precision; o.ns_schedule = schedule;
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = 5; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  const int n = (int)m.size();
  size_t bytes = 0;
  EXPECT(mona_state_size(m.data(), n, &o, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  auto fresh = [&]() {
    mona_state* st = nullptr;
    EXPECT(mona_init_state(m.data(), n, &o, arena, bytes, &one, &st) == MONA_OK);
    return st;
  };
  fake::on_launch = note;
  mona_state* const kept = fresh();
  for (int k = 0; k < 8; ++k) {
    auto value = [&] { return (float)(1 + rng() % 1000) / 256.0f; };
    if (rng() % 2) hp.lr = value();
    if (rng() % 2) hp.weight_decay = value();
    if (rng() % 2) hp.gamma_coeff = value();
    if (rng() % 2) { hp.ns_a = value(); hp.ns_b = -value(); hp.ns_c = value(); }
    if (rng() % 4 == 0) hp.ns_steps = 1 + (int)(rng() % 6);
    if (rng() % 4 == 0) hp.flags ^= MONA_FLAG_KEEP_O;
    figures.clear();
    EXPECT(mona_step(kept, m.data(), n, &hp, &one) == MONA_OK);
    const std::vector<float> got = figures;
    mona_state* const other = fresh();
    figures.clear();
    EXPECT(mona_step(other, m.data(), n, &hp, &one) == MONA_OK);
    EXPECT(!got.empty() && got == figures);
    EXPECT(mona_free_state(other) == MONA_OK);
  }
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(kept) == MONA_OK);
  std::free(arena);
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  std::mt19937 rng(17);
  run({{1, 256, 512}, {1, 64, 100}}, 0, 0, rng);
  run({{120, 256, 512}, {16, 1024, 1024}, {2, 300, 700}}, 0, 0, rng);
  run({{6, 512, 640}, {100, 40, 128}}, 1, 0, rng);
  run({{2, 1536, 4096}, {8, 1024, 2048}}, 0, 0, rng);
  run({{3, 500, 900}, {2, 1000, 1000}}, 0, 2, rng);
  for (int kind : kinds_seen) EXPECT(kind > 8);
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
