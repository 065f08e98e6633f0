// The chain launches of a step (ns_chain_kernel) followed on the host: their tasks carried out in number by any number of
// workgroups, latecomers among them, come to an end and respect the order of every chain, the rolls and flags they use are cleared before, and
// their products are those that are launched one by one at profiling level 2.  Needs no GPU (fake_hip.h); built and run by
// tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <set>
#include <tuple>

using namespace mona;

static int failures = 0, chains_seen = 0;
static std::string what;
#define EXPECT(cond)                                                                                   \
  do {                                                                                                 \
    if (!(cond)) { std::printf("FAILED line %d: %s (%s)\n", __LINE__, #cond, what.c_str()); ++failures; } \
  } while (0)

typedef std::vector<std::tuple<int, int, int>> Shapes;   // count, m, n

struct Task { int op, mat; };

// W workgroups, each with its tasks in order, one of those that can go on at a time.  late: so many more that come at any time,
// and all tasks behind the first W are drawn in order by whoever has finished one or has come.
static void carry_out(const ChainArgs& c, int workgroups, int late, std::mt19937& rng) {
  std::vector<Task> tasks;
  std::vector<int> first_of(c.ops), tiles_of(c.ops);
  for (int i = 0, first = 0; i < c.ops; first = c.op[i++].end) {
    GemmArgs a;
    expand_op(c.step, c.group[c.op[i].code >> OPF_GROUP], c.op[i].code, a);
    EXPECT(c.op[i].end - first == a.tiles_per_mat * a.count);
    EXPECT(a.tile_m == 32 || a.tile_m == 64);
    // the product before: the last one of the same group
    int before = -1;
    for (int j = 0; j < i; ++j)
      if (c.op[j].code >> OPF_GROUP == c.op[i].code >> OPF_GROUP) before = j;
    EXPECT(before < 0 ? c.op[i].before_per_mat == 0
                      : c.op[i].before == first_of[before] && c.op[i].before_per_mat == tiles_of[before]);
    first_of[i] = first;
    tiles_of[i] = a.tiles_per_mat;
    for (int t = first; t < c.op[i].end; ++t) tasks.push_back({i, (t - first) / a.tiles_per_mat});
  }
  EXPECT((int)tasks.size() == c.tasks);
  std::vector<char> done(tasks.size(), 0);
  std::vector<int> at(workgroups);
  for (int w = 0; w < workgroups; ++w) at[w] = w;
  int drawn = workgroups;
  size_t left = tasks.size();
  while (left > 0) {
    if (late > 0 && (int)at.size() < workgroups + late && rng() % 16 == 0) at.push_back(drawn++);
    std::vector<int> ready;
    for (int w = 0; w < (int)at.size(); ++w) {
      if (at[w] >= (int)tasks.size()) continue;
      const Task& t = tasks[at[w]];
      const ChainOp& op = c.op[t.op];
      bool go = true;
      for (int k = 0; k < op.before_per_mat; ++k) go = go && done[op.before + t.mat * op.before_per_mat + k];
      if (go) ready.push_back(w);
    }
    EXPECT(!ready.empty());
    if (ready.empty()) return;
    const int w = ready[rng() % ready.size()];
    done[at[w]] = 1;
    at[w] = late > 0 ? drawn++ : at[w] + workgroups;
    --left;
  }
}

static void run(const Shapes& shapes, int precision, int streams, int steps, int want_chains, std::mt19937& rng) {
  std::vector<mona_matrix> m;
  what = "precision " + std::to_string(precision) + ", streams " + std::to_string(streams) + ", steps " + std::to_string(steps);
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
  o.ns_precision = precision; o.max_streams = streams;
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
  // where a product's result goes, its tile, its K: in a chain or launched by itself
  typedef std::multiset<std::tuple<const void*, int, int>> Products;
  Products products;
  std::vector<ChainArgs> chains;
  const char* zero = nullptr;
  size_t zero_bytes = 0;
  fake::on_launch = [&](const fake::Launch& l) {
    if (l.name.find("norm_finalize_kernel") != std::string::npos) {
      zero = *static_cast<char**>(l.args[7]);
      zero_bytes = (size_t)*static_cast<int*>(l.args[8]) * 16;
    } else if (l.name.find("ns_chain_kernel") != std::string::npos) {
      const ChainArgs& c = *static_cast<const ChainArgs*>(l.args[0]);
      EXPECT(l.block == 512 && l.grid >= 1 && l.grid <= 256);
      EXPECT(c.patience == kPatience && c.roll_polls == kRollPolls);
      chains.push_back(c);
      for (int i = 0; i < c.ops; ++i) {
        GemmArgs a;
        expand_op(c.step, c.group[c.op[i].code >> OPF_GROUP], c.op[i].code, a);
        products.insert({a.C, a.tile_m, a.K});
      }
    } else if (l.name.find("ns_small_kernel") != std::string::npos) {
      const GemmBatch& b = *static_cast<const GemmBatch*>(l.args[0]);
      for (int i = 0; i < b.n; ++i) products.insert({b.a[i].C, b.a[i].tile_m, b.a[i].K});
    }
  };
  int64_t plan_launches = 0;
  EXPECT(mona_plan_info(st, steps, &plan_launches, nullptr, nullptr) == MONA_OK);
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(want_chains < 0 || (int)chains.size() == want_chains);
  EXPECT(chains.empty() || (int64_t)chains.size() == plan_launches);
  // rolls and flags: apart from each other, cleared, inside the arena
  std::vector<std::pair<const char*, const char*>> areas;
  for (const ChainArgs& c : chains) {
    areas.emplace_back(reinterpret_cast<const char*>(c.roll), reinterpret_cast<const char*>(c.roll + 1));
    areas.emplace_back(reinterpret_cast<const char*>(c.flags), reinterpret_cast<const char*>(c.flags + c.tasks));
  }
  std::sort(areas.begin(), areas.end());
  for (size_t i = 0; i < areas.size(); ++i) {
    EXPECT(areas[i].first >= zero && areas[i].second <= zero + zero_bytes);
    EXPECT(i == 0 || areas[i - 1].second <= areas[i].first);
  }
  EXPECT(chains.empty() || (zero >= arena && zero + zero_bytes <= arena + bytes));
  for (const ChainArgs& c : chains)
    for (int w : {1, 2, 7, 256})
      for (int late : {0, 1, 20}) carry_out(c, w, late, rng);
  chains_seen += (int)chains.size();
  const Products ordinary = products;
  products.clear();
  EXPECT(mona_set_profiling(st, 2) == MONA_OK);
  const bool chained = !chains.empty();
  chains.clear();
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(chains.empty());
  EXPECT(!chained || products == ordinary);
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  std::mt19937 rng(11);
  run({{1, 256, 512}}, 0, 0, 5, 1, rng);
  run({{1, 100, 300}, {1, 333, 130}, {1, 257, 257}, {1, 3, 5}, {1, 1, 64}, {1, 70, 1}, {3, 192, 136}}, 0, 0, 5, 1, rng);
  run({{1, 256, 512}}, 1, 0, 0, 0, rng);                       // no iterations, no products
  run({{1, 256, 512}}, 0, 0, 60, 0, rng);                      // more products than a chain takes
  run({{1, 1024, 1024}}, 0, 0, 5, 0, rng);                     // beyond the line
  run({{128, 768, 256}, {4, 128, 512}}, 0, 0, 5, 0, rng);      // beside large tiles
  run({{1, 70, 90}, {1, 83, 130}, {1, 96, 170}, {1, 109, 210}, {1, 122, 250}, {1, 135, 290}, {1, 148, 330}, {1, 161, 370},
       {1, 174, 410}}, 0, 1, 5, 2, rng);                       // nine groups, one stream
  for (int round = 0; round < 60; ++round) {
    Shapes s;
    const int groups = 1 + (int)(rng() % 11);
    for (int g = 0; g < groups; ++g) {
      auto side = [&] { return rng() % 2 ? 1 + (int)(rng() % 200) : 32 * (1 + (int)(rng() % 12)); };
      s.emplace_back(1 + (int)(rng() % 3), side(), side());
    }
    run(s, (int)(rng() % 2), (int)(rng() % 5), 1 + (int)(rng() % 8), -1, rng);
  }
  EXPECT(chains_seen > 40);
  std::printf("%s (%d failures, %d chains)\n", failures ? "FAILED" : "ok", failures, chains_seen);
  return failures ? 1 : 0;
}
