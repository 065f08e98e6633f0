// The launches that give a workgroup to each matrix (ns_matrix_kernel) followed on the host: beside whatever else a step launches,
// every shape group is carried through all its iterations exactly once, the workgroups of a launch are those of its
// groups one after the other, and profiling level 2 launches the same groups one by one.  Needs no GPU (fake_hip.h); built and
// run by tests/test_host_launches.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <set>
#include <tuple>

using namespace mona;

static int failures = 0, launches_seen = 0;
static std::string what;
#define EXPECT(cond)                                                                                   \
  do {                                                                                                 \
    if (!(cond)) { std::printf("FAILED line %d: %s (%s)\n", __LINE__, #cond, what.c_str()); ++failures; } \
  } while (0)

typedef std::vector<std::tuple<int, int, int>> Shapes;   // count, m, n

// want: launches of the kernel in an ordinary step (-1: any number)
static void run(const Shapes& shapes, int streams, int steps, uint32_t flags, int want) {
  std::vector<mona_matrix> m;
  std::set<std::pair<int, int>> kinds;
  what = "streams " + std::to_string(streams) + ", steps " + std::to_string(steps);
  for (auto [count, rows, cols] : shapes) {
    what += ", " + std::to_string(count) + "*" + std::to_string(rows) + "*" + std::to_string(cols);
    kinds.insert({rows, cols});
    for (int i = 0; i < count; ++i) {
      mona_matrix q;
      std::memset(&q, 0, sizeof q);
      q.m = rows; q.n = cols; q.w_dtype = MONA_BF16; q.g_dtype = MONA_F32;
      q.w = reinterpret_cast<void*>((uintptr_t)16); q.g = q.w;
      m.push_back(q);
    }
  }
  mona_options o;
  std::memset(&o, 0, sizeof o);
  o.max_streams = streams;
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = steps; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  hp.flags = flags;
  const int n = (int)m.size();
  size_t bytes = 0;
  EXPECT(mona_state_size(m.data(), n, &o, &bytes) == MONA_OK);
  char* arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  mona_state* st = nullptr;
  EXPECT(mona_init_state(m.data(), n, &o, arena, bytes, &one, &st) == MONA_OK);
  std::map<const int32_t*, int> updated;                       // members of a group -> times its parameters are updated
  std::map<const int32_t*, std::tuple<int, int, int>> whole;   // groups of the kernel: count, m, n
  int launches = 0, others = 0;
  size_t most_groups = 0;
  fake::on_launch = [&](const fake::Launch& l) {
    if (l.name.find("ns_matrix_kernel") != std::string::npos) {
      const MatrixBatch& b = *static_cast<const MatrixBatch*>(l.args[0]);
      ++launches;
      most_groups = std::max(most_groups, (size_t)b.n);
      EXPECT(b.n >= 1 && b.n <= kMaxMerged && b.steps == steps && b.store_o == ((flags & MONA_FLAG_KEEP_O) ? 1 : 0));
      int end = 0;
      for (int i = 0; i < b.n && i < kMaxMerged; ++i) {
        const GroupDesc& g = b.group[i];
        end += g.count;
        EXPECT(b.end[i] == end);
        EXPECT(g.rows_pad >= g.m && g.cols_pad >= g.n && g.rows_pad % 128 == 0 && g.cols_pad % 128 == 0);
        EXPECT(g.tall == (g.m > g.n));
        const int p = std::min(g.rows_pad, g.cols_pad);
        EXPECT(p == 128 || p == 256);
        for (int k = 0; k < g.count; ++k) EXPECT(m[g.members[k]].m == g.m && m[g.members[k]].n == g.n);
        whole[g.members] = {g.count, g.m, g.n};
        ++updated[g.members];
      }
      EXPECT((int)l.grid == end && l.block == 512);
      return;
    }
    auto product = [&](const GemmArgs& a) { if (a.epilogue == EPI_UPDATE) ++updated[a.members]; };
    if (l.name.find("ns_chain_kernel") != std::string::npos) {
      const ChainArgs& c = *static_cast<const ChainArgs*>(l.args[0]);
      for (int i = 0; i < c.ops; ++i) {
        GemmArgs a;
        expand_op(c.step, c.group[c.op[i].code >> OPF_GROUP], c.op[i].code, a);
        product(a);
      }
    } else if (l.name.find("ns_small_kernel") != std::string::npos) {
      const GemmBatch& b = *static_cast<const GemmBatch*>(l.args[0]);
      for (int i = 0; i < b.n; ++i) product(b.a[i]);
    } else if (l.name.find("ns_gemm_bf16_dma_kernel") != std::string::npos) {
      product(*static_cast<const GemmArgs*>(l.args[0]));
    } else {
      return;
    }
    ++others;
  };
  double plan_flops = 0.0;
  EXPECT(mona_plan_info(st, steps, nullptr, &plan_flops, nullptr) == MONA_OK);
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(want < 0 || launches == want);
  EXPECT(updated.size() == kinds.size());
  for (const auto& u : updated) EXPECT(u.second == 1);
  launches_seen += launches;
  // one by one
  const auto whole_ordinary = whole;
  updated.clear(); whole.clear(); launches = 0; others = 0; most_groups = 0;
  EXPECT(mona_set_profiling(st, 2) == MONA_OK);
  EXPECT(mona_step(st, m.data(), n, &hp, &one) == MONA_OK);
  EXPECT(whole == whole_ordinary && launches == (int)whole.size() && most_groups <= 1);
  for (const auto& u : updated) EXPECT(u.second == 1);
  int32_t records = 0;
  EXPECT(mona_last_step_launches(st, nullptr, 0, &records) == MONA_OK && records == launches + others);
  std::vector<mona_launch_time> rec(records);
  EXPECT(mona_last_step_launches(st, rec.data(), records, &records) == MONA_OK);
  double sum = 0.0;
  std::multiset<std::tuple<int, int, int>> seen, expected;
  for (const auto& r : rec) {
    sum += r.flops;
    if (r.kind != 4) continue;
    EXPECT(r.tile == (std::min(r.m, r.n) > 128 ? 256128 : 128128));
    seen.insert({r.count, r.m, r.n});
  }
  for (const auto& w : whole) expected.insert(w.second);
  EXPECT(seen == expected);
  EXPECT(std::fabs(sum - plan_flops) <= 1e-9 * sum);
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  run({{128, 768, 256}, {128, 256, 768}}, 0, 5, 0, 1);
  run({{1, 128, 128}}, 0, 5, MONA_FLAG_KEEP_O, 1);
  run({{300, 70, 100}}, 0, 1, 0, 1);
  // ten groups: eight in one launch, two in another
  Shapes ten;
  for (int i = 0; i < 10; ++i) ten.emplace_back(120, 66 + 5 * i, 130 + 37 * ((3 * i) % 7));
  run(ten, 0, 5, 0, 2);
  run(ten, 1, 6, 0, 2);
  // beside large tiles, merged small products of both precisions, and a group on a stream of its own
  run({{120, 256, 512}, {8, 2048, 2048}, {200, 100, 100}, {3, 30, 500}, {2, 300, 700}}, 0, 5, 0, 1);
  run({{120, 256, 512}, {8, 2048, 2048}, {200, 100, 100}, {3, 30, 500}, {2, 300, 700}}, 1, 5, 0, 1);
  run({{256, 4096, 1536}, {200, 256, 256}, {1, 2000, 2000}}, 0, 5, 0, 1);     // beside a group that keeps the caller's stream
  run({{2, 128, 128}, {1, 512, 1408}}, 0, 5, 0, 0);                           // all in a chain
  std::mt19937 rng(3);
  for (int round = 0; round < 40; ++round) {
    Shapes s;
    const int groups = 1 + (int)(rng() % 12);
    for (int g = 0; g < groups; ++g) {
      auto side = [&] { return rng() % 2 ? 65 + (int)(rng() % 191) : 64 * (1 + (int)(rng() % 12)); };
      s.emplace_back(1 + (int)(rng() % (rng() % 3 ? 200 : 3)), side(), side());
    }
    run(s, (int)(rng() % 5), 1 + (int)(rng() % 7), 0, -1);
  }
  EXPECT(launches_seen > 40);
  std::printf("%s (%d failures, %d launches)\n", failures ? "FAILED" : "ok", failures, launches_seen);
  return failures ? 1 : 0;
}
