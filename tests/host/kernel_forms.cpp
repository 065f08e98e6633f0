// Which form of a kernel a step takes where its host code chooses among several: what the elementwise pass leaves in the caches, and how the
// last product of large tiles takes the rows of W.  Needs no GPU (fake_hip.h); built and run by tests/test_kernel_forms.py.
#include "../../include/mona.h"
#include "fake_hip.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <tuple>

using namespace mona;

static int failures = 0;
static std::string what;
#define EXPECT(cond)                                                                                   \
  do {                                                                                                 \
    if (!(cond)) { std::printf("FAILED line %d: %s (%s)\n", __LINE__, #cond, what.c_str()); ++failures; } \
  } while (0)

// names of the kernels of one step of `count` matrices; of the parameters the first `f32` are fp32
static std::vector<std::string> kernels(int count, int m, int n, int f32, int schedule) {
  what = std::to_string(count) + "*" + std::to_string(m) + "*" + std::to_string(n) + ", " + std::to_string(f32) + " fp32, schedule " + std::to_string(schedule);
  std::vector<mona_matrix> mats;
  for (int i = 0; i < count; ++i) {
    mona_matrix q;
    std::memset(&q, 0, sizeof q);
    q.m = m; q.n = n; q.w_dtype = i < f32 ? MONA_F32 : MONA_BF16; q.g_dtype = MONA_F32;
    q.w = reinterpret_cast<void*>((uintptr_t)16); q.g = q.w;
    mats.push_back(q);
  }
  mona_options o;
  std::memset(&o, 0, sizeof o);
  o.ns_schedule = schedule;
  size_t bytes = 0;
  EXPECT(mona_state_size(mats.data(), count, &o, &bytes) == MONA_OK);
  char* const arena = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  char stream;
  mona_state* st = nullptr;
  EXPECT(mona_init_state(mats.data(), count, &o, arena, bytes, &stream, &st) == MONA_OK);
  std::vector<std::string> names;
  fake::on_launch = [&](const fake::Launch& l) { names.push_back(l.name); };
  mona_hparams hp;
  std::memset(&hp, 0, sizeof hp);
  hp.lr = 1e-3f; hp.momentum = 0.9f; hp.beta_a = 0.9f; hp.alpha = 0.5f; hp.ns_steps = 5;
  hp.ns_a = 3.0f; hp.ns_b = -3.0f; hp.ns_c = 1.0f; hp.ns_eps = 1e-7f; hp.gamma_coeff = 0.2f;
  EXPECT(mona_step(st, mats.data(), count, &hp, &stream) == MONA_OK);
  fake::on_launch = nullptr;
  EXPECT(mona_free_state(st) == MONA_OK);
  std::free(arena);
  return names;
}

static int count_of(const std::vector<std::string>& names, const std::string& piece) {
  int n = 0;
  for (const std::string& s : names) n += s.find(piece) != std::string::npos;
  return n;
}

int main() {
  fake::capability_major = 9;
  fake::capability_minor = 5;
  // fp32 gradients and state, two buffers (mode 1): the working copy is kept (1) of passes of 2 to 230 MB, whether or not all that they
  // move would fit into the caches, and nothing else
  for (auto [count, m, n] : {std::tuple{40, 128, 256}, {128, 128, 128}, {100, 128, 512}, {1, 1000, 1000}, {30, 300, 700}, {4, 16, 1024}}) {
    const auto names = kernels(count, m, n, 0, MONA_NS_SCHEDULE_AUTO);
    if (count_of(names, "begin_norm_finalize_kernel")) { EXPECT(count_of(names, "state_update_kernel") == 0); continue; }
    EXPECT(count_of(names, "state_update_kernel") == 1 && count_of(names, "state_update_kernelIffLi1ELi1EE") == 1);
  }
  // rows of whole pieces (0) where all parameters are bf16 and rows a multiple of 8, bf16 ends (1) where they are not, any (2) with fp32
  // parameters among them
  const std::string update = "ns_gemm_bf16_dma_kernelILi256ELi256ELi2ELi4ELi4ELi1ELb0ELb1ELb1ELb";
  for (int schedule : {MONA_NS_SCHEDULE_LITERAL, MONA_NS_SCHEDULE_FUSED})
    for (auto [n, f32, form] : {std::tuple{504, 0, 0}, {512, 0, 0}, {509, 0, 1}, {508, 0, 1}, {504, 1, 2}, {509, 1, 2}, {504, 44, 2}}) {
      const auto names = kernels(44, 505, n, f32, schedule);
      EXPECT(count_of(names, update) == 1);
      EXPECT(count_of(names, update + "0ELb0ELi" + std::to_string(form) + "EE") + count_of(names, update + "1ELb0ELi" + std::to_string(form) + "EE") == 1);
    }
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
