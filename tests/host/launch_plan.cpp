// The product launches of a step against what mona_plan_info says of it, and the products that profiling level 2 launches
// one by one against those of an ordinary step.  Needs no GPU (fake_hip.h); built and run by tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
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
// where a product's result goes, how many times that was the target before -> tile, K and kernel
typedef std::map<std::pair<const void*, int>, std::tuple<int, int, std::string>> Products;

static void run(const Shapes& shapes, int precision, int streams, int schedule, int want_launches) {
  std::vector<mona_matrix> m;
  what = "precision " + std::to_string(precision) + ", streams " + std::to_string(streams);
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
  o.ns_precision = precision; o.max_streams = streams; o.ns_schedule = schedule;
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = 5; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  const int n = (int)m.size();
  size_t bytes = 0;
  EXPECT(mona_state_size(m.data(), n, &o, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  mona_state* st = nullptr;
  EXPECT(mona_init_state(m.data(), n, &o, arena, bytes, &one, &st) == MONA_OK);
  int launches = 0;
  double flops = 0.0;
  Products products;
  fake::on_launch = [&](const fake::Launch& l) {
    const bool small = l.name.find("ns_small_kernel") != std::string::npos;
    if (!small && l.name.find("ns_gemm_bf16_dma_kernel") == std::string::npos) return;
    ++launches;
    const int k = small ? static_cast<const GemmBatch*>(l.args[0])->n : 1;
    const GemmArgs* a = small ? static_cast<const GemmBatch*>(l.args[0])->a : static_cast<const GemmArgs*>(l.args[0]);
    for (int i = 0; i < k; ++i) {
      // (tiles of 32 and 64 stop behind the last value of K that is no padding, in steps of 32, but for those of split products)
      const bool stops = a[i].tile_m <= 64 && l.name.find("ns_small_kernel_split") == std::string::npos;
      flops += 2.0 * a[i].tile_m * a[i].tile_n * (double)(stops ? (a[i].k_real + 31) / 32 * 32 : a[i].K) * a[i].tiles_per_mat * a[i].count;
      int again = 0;
      while (products.count({a[i].C, again})) ++again;
      products[{a[i].C, again}] = {a[i].tile_m, a[i].K, l.name};
    }
  };
  int64_t plan_launches = 0;
  double plan_flops = 0.0;
  EXPECT(mona_plan_info(st, 5, &plan_launches, &plan_flops, nullptr) == MONA_OK);
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(launches == plan_launches);
  EXPECT(want_launches == 0 || launches == want_launches);
  EXPECT(std::fabs(flops - plan_flops) <= 1e-9 * flops);
  // every product by itself
  const Products ordinary = products;
  products.clear(); launches = 0; flops = 0.0;
  EXPECT(mona_set_profiling(st, 2) == MONA_OK);
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(products == ordinary);
  EXPECT((size_t)launches == ordinary.size());
  int32_t records = 0;
  EXPECT(mona_last_step_launches(st, nullptr, 0, &records) == MONA_OK && records == launches);
  std::vector<mona_launch_time> rec(records);
  EXPECT(mona_last_step_launches(st, rec.data(), records, &records) == MONA_OK);
  double sum = 0.0;
  for (const auto& r : rec) sum += r.flops;
  EXPECT(std::fabs(sum - plan_flops) <= 1e-9 * sum);
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
}

int main() {
  // four bf16 shape groups in one launch, three fp32 ones (a short side of at most 64) in another
  const Shapes ragged = {{1, 100, 300}, {1, 333, 130}, {1, 257, 257}, {1, 3, 5}, {1, 1, 64}, {1, 70, 1}, {3, 192, 136}};
  run(ragged, 0, 0, 0, 30);
  run(ragged, 0, 1, 0, 30);
  run(ragged, 1, 0, 0, 15);
  run({{1, 256, 512}}, 0, 0, 0, 15);
  run({{1, 512, 1408}}, 0, 0, 0, 15);                       // the literal schedule
  // alone 64 x 64 tiles (20 and 30 of 128), 128 x 128 and two workgroups a CU in company
  run({{2, 500, 610}, {3, 500, 640}, {2, 640, 500}, {4, 512, 700}}, 0, 1, 0, 15);
  run({{4, 1000, 1000}, {2, 1000, 2666}, {1, 2666, 1000}}, 0, 0, 0, 0);
  run({{20, 512, 1536}, {3, 100, 100}, {2, 1024, 1024}}, 0, 0, 2, 0);
  std::mt19937 rng(7);
  for (int round = 0; round < 40; ++round) {
    Shapes s;
    const int groups = 1 + (int)(rng() % 11);
    for (int g = 0; g < groups; ++g) {
      auto side = [&] { return rng() % 2 ? 1 + (int)(rng() % 400) : 64 * (1 + (int)(rng() % 12)); };
      s.emplace_back(1 + (int)(rng() % (rng() % 4 ? 3 : 40)), side(), side());
    }
    run(s, (int)(rng() % 2), (int)(rng() % 5), (int)(rng() % 4), 0);
  }
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
