// What mona_plan_info says a step executes against the launches of that step, on a device for which chains and the kernel that
// gives a workgroup to each matrix are planned.  Needs no GPU (fake_hip.h); built and run by tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <tuple>

using namespace mona;

static int failures = 0, matrix_launches = 0, split_launches = 0, chain_launches = 0, other_launches = 0;
static std::string what;
#define EXPECT(cond)                                                                                   \
  do {                                                                                                 \
    if (!(cond)) { std::printf("FAILED line %d: %s (%s)\n", __LINE__, #cond, what.c_str()); ++failures; } \
  } while (0)

typedef std::vector<std::tuple<int, int, int>> Shapes;   // count, m, n

// A product's tiles times the K they go through: the long side of a Gram product's matrices, the short one of any other's, in whole slabs of 32
// on tiles of 32 and 64 (not those of split fp32 products), otherwise with all of its padding, to a multiple of 128.
static double product(const GemmArgs& a, const std::vector<mona_matrix>& mats, bool split) {
  const mona_matrix& q = mats[a.members[0]];
  const bool gram = a.symmetric && a.P == a.Q && !a.E;
  const int k = gram ? std::max(q.m, q.n) : std::min(q.m, q.n), unit = a.tile_m <= 64 && !split ? 32 : 128;
  return 2.0 * a.tile_m * a.tile_n * (double)((k + unit - 1) / unit * unit) * a.tiles_per_mat * a.count;
}

static void run(const Shapes& shapes, int precision, int steps) {
  std::vector<mona_matrix> m;
  what = "precision " + std::to_string(precision) + ", steps " + std::to_string(steps);
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
  o.ns_precision = precision;
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = steps; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  const int n = (int)m.size();
  size_t bytes = 0;
  EXPECT(mona_state_size(m.data(), n, &o, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  mona_state* st = nullptr;
  EXPECT(mona_init_state(m.data(), n, &o, arena, bytes, &one, &st) == MONA_OK);
  double flops = 0.0;
  int launches = 0;
  fake::on_launch = [&](const fake::Launch& l) {
    if (l.name.find("ns_") == std::string::npos) return;
    ++launches;
    if (l.name.find("ns_matrix_kernel") != std::string::npos) {
      // S = Y Y^T and Y' = a Y + B Y on a padded p x q matrix, S S on the whole square
      const MatrixBatch& b = *static_cast<const MatrixBatch*>(l.args[0]);
      for (int i = 0; i < b.n; ++i) {
        const double r = b.group[i].rows_pad, c = b.group[i].cols_pad, p = std::min(r, c), q = std::max(r, c);
        flops += b.steps * (2.0 * p * p * q + 2.0 * p * p * p + 2.0 * p * p * q) * b.group[i].count;
      }
      ++matrix_launches;
    } else if (l.name.find("ns_chain_kernel") != std::string::npos) {
      const ChainArgs& c = *static_cast<const ChainArgs*>(l.args[0]);
      for (int i = 0; i < c.ops; ++i) {
        GemmArgs a;
        expand_op(c.step, c.group[c.op[i].code >> OPF_GROUP], c.op[i].code, a);
        flops += product(a, m, false);
      }
      ++chain_launches;
    } else if (l.name.find("ns_small_kernel") != std::string::npos) {
      const bool split = l.name.find("ns_small_kernel_split") != std::string::npos;   // (an fp32 product counts once)
      const GemmBatch& b = *static_cast<const GemmBatch*>(l.args[0]);
      for (int i = 0; i < b.n; ++i) flops += product(b.a[i], m, split);
      ++(split ? split_launches : other_launches);
    } else {
      flops += product(*static_cast<const GemmArgs*>(l.args[0]), m, false);
      ++other_launches;
    }
  };
  int64_t plan_launches = 0;
  double plan_flops = 0.0;
  EXPECT(mona_plan_info(st, steps, &plan_launches, &plan_flops, nullptr) == MONA_OK);
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(launches == plan_launches);
  EXPECT(std::fabs(flops - plan_flops) <= 1e-9 * flops);
  // and what the records of launches timed one by one say
  EXPECT(mona_set_profiling(st, 2) == MONA_OK);
  flops = 0.0;
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  int32_t records = 0;
  EXPECT(mona_last_step_launches(st, nullptr, 0, &records) == MONA_OK);
  std::vector<mona_launch_time> record(records);
  EXPECT(mona_last_step_launches(st, record.data(), records, &records) == MONA_OK);
  double recorded = 0.0;
  for (const mona_launch_time& r : record) recorded += r.flops;
  EXPECT(std::fabs(flops - recorded) <= 1e-9 * flops);
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  run({{250, 70, 100}}, 0, 5);                                // 128 x 128 padded
  run({{111, 256, 512}}, 0, 5);
  run({{128, 768, 256}, {128, 256, 768}}, 0, 4);
  run({{4, 1024, 1024}, {1, 1024, 4096}}, 1, 5);              // fp32 products on the bf16 instructions
  run({{200, 64, 1000}}, 1, 5);                               // short K: on the fp32 instructions
  run({{1, 256, 512}}, 0, 5);
  run({{120, 256, 512}, {8, 2048, 2048}, {60, 100, 100}, {3, 30, 500}}, 0, 5);
  std::mt19937 rng(5);
  for (int round = 0; round < 40; ++round) {
    Shapes s;
    const int groups = 1 + (int)(rng() % 5);
    for (int g = 0; g < groups; ++g) {
      auto side = [&] { return rng() % 2 ? 1 + (int)(rng() % 300) : 64 * (1 + (int)(rng() % 8)); };
      s.emplace_back(1 + (int)(rng() % (rng() % 2 ? 3 : 200)), side(), side());
    }
    run(s, (int)(rng() % 4 == 0), 1 + (int)(rng() % 6));
  }
  EXPECT(matrix_launches > 4 && split_launches > 4 && chain_launches > 4 && other_launches > 4);
  std::printf("%s (%d failures; launches by matrix %d, split %d, chains %d, others %d)\n", failures ? "FAILED" : "ok", failures,
              matrix_launches, split_launches, chain_launches, other_launches);
  return failures ? 1 : 0;
}
