// Chains whose products have a buffer each, followed on the host 16 bytes at a time: everything is written once, what is read has been
// written or filled with zeros, and states share no part of the pool.  Needs no GPU (fake_hip.h); built and run by
// tests/test_fresh_chains.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <tuple>

using namespace mona;

static int failures = 0, fresh_seen = 0, flagged_seen = 0;
static std::string what;
#define EXPECT(cond)                                                                                   \
  do {                                                                                                 \
    if (!(cond)) { std::printf("FAILED line %d: %s (%s)\n", __LINE__, #cond, what.c_str()); ++failures; } \
  } while (0)

typedef std::vector<std::tuple<int, int, int>> Shapes;   // count, m, n
constexpr size_t kPool = (size_t)128 << 20;
enum : char { kOutside = 0, kWaiting, kZero, kWritten };

struct State {
  std::vector<mona_matrix> m;
  char* arena = nullptr;
  size_t bytes = 0;
  mona_state* st = nullptr;
};

static State make(const Shapes& shapes, int precision) {
  State s;
  what = "precision " + std::to_string(precision);
  for (auto [count, rows, cols] : shapes) {
    what += ", " + std::to_string(count) + "*" + std::to_string(rows) + "*" + std::to_string(cols);
    for (int i = 0; i < count; ++i) {
      mona_matrix q;
      std::memset(&q, 0, sizeof q);
      q.m = rows; q.n = cols; q.w_dtype = MONA_F32; q.g_dtype = MONA_F32;
      q.w = reinterpret_cast<void*>((uintptr_t)16); q.g = q.w;
      s.m.push_back(q);
    }
  }
  mona_options o;
  std::memset(&o, 0, sizeof o);
  o.ns_precision = precision;
  size_t& bytes = s.bytes;
  EXPECT(mona_state_size(s.m.data(), (int)s.m.size(), &o, &bytes) == MONA_OK);
  s.arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char one;
  EXPECT(mona_init_state(s.m.data(), (int)s.m.size(), &o, s.arena, bytes, &one, &s.st) == MONA_OK);
  return s;
}
static void release(State& s) {
  EXPECT(mona_free_state(s.st) == MONA_OK);
  std::free(s.arena);
}

// a step; `pool` says of every 16 bytes what they hold
static void step(const State& s, int steps, int want_fresh, std::vector<char>& pool) {
  what += ", steps " + std::to_string(steps);
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 0.1f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.ns_steps = steps; hp.ns_a = hp.ns_b = hp.ns_c = hp.gamma_coeff = 1.0f;
  void* base = nullptr;
  (void)hipGetSymbolAddress(&base, nullptr);
  auto at = [&](const void* p) { return (size_t)(static_cast<const char*>(p) - static_cast<const char*>(base)); };
  std::fill(pool.begin(), pool.end(), kOutside);
  bool any = false, fresh = false;
  fake::on_launch = [&](const fake::Launch& l) {
    if (l.name.find("begin_norm_finalize_kernel") != std::string::npos) {
      const FillArgs& f = *static_cast<const FillArgs*>(l.args[9]);
      uint32_t groups = 0;
      for (int i = 0; i < f.n; ++i) {
        const FillItem& t = f.item[i];
        groups += (t.pieces + kFillPieces - 1) / kFillPieces;
        EXPECT(t.end == groups);
        for (uint32_t k = 0; k < t.pieces; ++k) {
          const uint32_t line = k / t.width, c = k % t.width, r = line % t.rows;
          const size_t to = at(t.at) + (size_t)(line / t.rows) * t.stride + (size_t)r * t.pitch + c * 16;
          EXPECT(to + 16 <= kPool);
          if (to + 16 > kPool) return;
          EXPECT(pool[to / 16] == kOutside);
          pool[to / 16] = r < t.cover_rows && c < t.cover ? kWaiting : kZero;
        }
      }
      EXPECT((int)groups == f.groups && l.grid == *static_cast<int*>(l.args[10]) + groups);
    } else if (l.name.find("ns_chain_kernel") != std::string::npos) {
      const ChainArgs& c = *static_cast<const ChainArgs*>(l.args[0]);
      any = true;
      fresh = c.fresh;
      if (!c.fresh) return;
      for (int i = 0; i < c.ops; ++i) {
        GemmArgs a;
        const GroupDesc& g = c.group[c.op[i].code >> OPF_GROUP];
        expand_op(c.step, g, c.op[i].code, a);
        const size_t es = g.f32 ? 4 : 2;
        const int k = (a.k_real + 31) / 32 * 32, T = a.tile_m;
        for (int mat = 0; mat < a.count; ++mat) {
          auto rows_of = [&](const void* p, int64_t stride, int ld, int r0, int r1, int c0, int c1, auto&& f) {
            const char* const from = static_cast<const char*>(p) + mat * stride * es;
            if (from >= s.arena && from < s.arena + s.bytes) return;      // X_0 or O
            const size_t first = at(from);
            EXPECT(first < kPool);
            if (first >= kPool) return;
            for (int r = r0; r < r1; ++r)
              for (size_t b = c0 * es; b < c1 * es; b += 16) f(pool[(first + (size_t)r * ld * es + b) / 16]);
          };
          auto read = [&](char& x) { EXPECT(x == kWritten || x == kZero); };
          const int m = a.tiles_m * T, n = a.tiles_n * T;
          if (a.trans_p) rows_of(a.P, a.strideP, a.ldp, 0, k, 0, m, read); else rows_of(a.P, a.strideP, a.ldp, 0, m, 0, k, read);
          if (a.trans_q) rows_of(a.Q, a.strideQ, a.ldq, 0, k, 0, n, read); else rows_of(a.Q, a.strideQ, a.ldq, 0, n, 0, k, read);
          if (a.E) rows_of(a.E, a.strideE, a.lde, 0, m, 0, n, read);
          // (a tile writes the zeros of padding again)
          rows_of(a.C, a.strideC, a.ldc, 0, m, 0, n, [&](char& x) { EXPECT(x == kWaiting || x == kZero); x = kWritten; });
        }
      }
    }
  };
  char one;
  EXPECT(mona_step(s.st, s.m.data(), (int)s.m.size(), &hp, &one) == MONA_OK);
  fake::on_launch = nullptr;
  EXPECT(want_fresh < 0 || (any && fresh == (want_fresh == 1)));
  if (any) ++(fresh ? fresh_seen : flagged_seen);
  if (fresh)
    for (size_t i = 0; i < pool.size(); ++i) {
      if (pool[i] != kWaiting) continue;
      EXPECT(!"filled and never written");
      break;
    }
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  std::vector<char> pool(kPool / 16);
  std::mt19937 rng(3);
  // the pool is in a source of its own: who needs another static array does not carry it too
  int pools = 0;
  for (const fake::Array& a : fake::arrays()) {
    if (a.bytes != kPool) continue;
    ++pools;
    EXPECT(std::count_if(fake::arrays().begin(), fake::arrays().end(), [&](const fake::Array& b) { return b.source == a.source; }) == 1);
  }
  EXPECT(pools == 1);
  for (int precision = 0; precision < 2; ++precision)
    for (int steps : {1, 2, 5, 6}) {
      State s = make({{1, 256, 512}}, precision);
      step(s, steps, steps <= kFreshSteps, pool);
      release(s);
    }
  {
    // of nine the last finds no room and runs with flags (eight fit where nothing lies between them); after the first has been
    // freed the next has its part
    std::vector<State> all;
    std::vector<char> used(pool.size(), 0);
    for (int i = 0; i < 9; ++i) {
      all.push_back(make({{1, 768, 768}}, 0));
      step(all.back(), 5, i < 6 ? 1 : i == 8 ? 0 : -1, pool);
      size_t shared = 0;
      for (size_t k = 0; k < pool.size(); ++k)
        if (pool[k] != kOutside) shared += used[k]++;
      EXPECT(shared == 0);
    }
    release(all.front());
    all.front() = make({{1, 768, 768}}, 0);
    step(all.front(), 5, 1, pool);
    for (State& s : all) release(s);
  }
  {
    // a recorded step may be replayed after its state has been freed: nobody else ever gets the part that its launches name
    State s = make({{1, 256, 512}}, 0);
    step(s, 5, 1, pool);
    const std::vector<char> recorded = pool;
    fake::capturing = true;
    step(s, 5, -1, pool);
    fake::capturing = false;
    fake::clear_recorded();
    release(s);
    std::vector<State> all;
    size_t fresh = 0;
    for (int i = 0; i < 70; ++i) {
      all.push_back(make({{1, 256, 512}}, 0));
      step(all.back(), 5, -1, pool);
      size_t shared = 0;
      for (size_t k = 0; k < pool.size(); ++k) shared += pool[k] != kOutside && recorded[k] != kOutside;
      EXPECT(shared == 0);
      fresh += std::count_if(pool.begin(), pool.end(), [](char c) { return c != kOutside; }) > 0;
    }
    EXPECT(fresh > 40 && fresh < 70);                  // (the pool was full in the end, and asked for parts given back)
    for (State& other : all) release(other);
  }
  for (int round = 0; round < 60; ++round) {
    Shapes shapes;
    const int groups = 1 + (int)(rng() % 6);
    for (int g = 0; g < groups; ++g) {
      auto side = [&] { return rng() % 2 ? 1 + (int)(rng() % 300) : 32 * (1 + (int)(rng() % 12)); };
      shapes.emplace_back(1 + (int)(rng() % 3), side(), side());
    }
    State s = make(shapes, (int)(rng() % 2));
    step(s, 1 + (int)(rng() % 6), -1, pool);
    release(s);
  }
  EXPECT(fresh_seen > 30 && flagged_seen > 3);
  std::printf("%s (%d failures, %d steps without flags, %d with)\n", failures ? "FAILED" : "ok", failures, fresh_seen, flagged_seen);
  return failures ? 1 : 0;
}
