// Host side of libmona: argument checking, arena layout, shape grouping and the launch plan
// of one MONA step (Alg. 1).  All arithmetic happens in the kernels of state_update.hip,
// ns_gemm.hip and ns_small.hip; this file only decides what is launched on which buffers.
#include "../../include/mona.h"
#include "mona_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace mona;
static_assert(kStatusIncomplete == MONA_STATUS_INCOMPLETE, "the same bit");

namespace {
thread_local std::string g_err;
}

namespace mona {
int api_fail(int code, const char* fmt, va_list ap) {
  char buf[512];
  vsnprintf(buf, sizeof buf, fmt, ap);
  g_err = buf;
  return code;
}
}  // namespace mona

namespace {

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  const int rc = api_fail(code, fmt, ap);
  va_end(ap);
  return rc;
}

// (the error is taken off the runtime's record, where the check behind the next call's first launch would find it again)
#define HIP_TRY(expr)                                                     \
  do {                                                                    \
    hipError_t e__ = (expr);                                              \
    if (e__ != hipSuccess) {                                              \
      (void)hipGetLastError();                                            \
      return fail(MONA_EHIP, "%s: %s", #expr, hipGetErrorString(e__));    \
    }                                                                     \
  } while (0)

constexpr size_t kAlign = 256;
constexpr int kSmallSideF32 = 64;
constexpr double kFusedMaxStart = 0.0438;  // largest 1 / sqrt(p) + 1 / sqrt(q) for which the automatic choice fuses three iterations
constexpr int kPairsMinShortSide = 1024;   // padded short side from which it fuses pairs of iterations otherwise
size_t align_up(size_t v, size_t a = kAlign) { return (v + a - 1) / a * a; }
int round_up(int v, int a) { return (v + a - 1) / a * a; }

struct Group {
  int m = 0, n = 0;          // native shape
  bool tall = false;         // m > n: Gram matrix on the column side
  int rows_pad = 0, cols_pad = 0;  // padded native shape of the working copies
  int p_pad = 0;             // padded short side
  int gran = 128;            // padding granularity (largest tile usable)
  bool f32 = false;          // products of this group run in fp32 (else bf16 operands)
  bool large_with_company = false;  // 256 x 256 tiles even for launches of few tiles (set when the state is built)
  int esize = 2;             // bytes per element of this group's working copies
  std::vector<int> members;  // matrix indices
  int fused = 0;             // Newton-Schulz iterations taken in chunks on the p x p side (see OpBuilder):
                             // 0 literal, 1 chunks of two, 2 a chunk of three and then chunks of two
  int npp = 2;               // p x p working matrices: S and B (literal schedule) or S, S', U, Q, R, R' (fused)
  int o_buf = 1;             // which ping-pong buffer holds O_k of the last step
  size_t x_off[2] = {0, 0};  // byte offsets in the arena: ping-pong X buffers
  size_t pp_off[6] = {0, 0, 0, 0, 0, 0};
  size_t fresh_off = 0;      // byte offset of the group's part of a fresh chain's buffers
  size_t members_off = 0;
  int64_t x_stride = 0, s_stride = 0;  // elements per matrix
};

// Groups whose products are launched together: one group, or up to kMaxMerged groups that run small tiles only and
// share a launch per position in their chains of products.
struct Unit {
  std::vector<int> groups;
  bool merged = false;
  bool matrix = false;       // a workgroup for each matrix (ns_matrix_kernel)
  int lane = 0;              // stream: 0 is the caller's
};

struct Layout {
  int count = 0;
  bool gfx950 = false;       // the device's architecture: chains and ns_matrix_kernel are planned for this one only
  int ssize = 4;             // bytes per element of the stored G_{k-1}, A (or C)
  bool one_buffer = false;   // no G_{k-1}; acc_off holds C
  bool caller_slot = false;  // G_{k-1} is kept by the caller (streaming variant)
  bool external_state = false;  // G_{k-1}, A and M live in arrays of the caller's, not in the arena
  std::vector<size_t> gprev_off, acc_off, mom_off;
  size_t state_begin = 0, state_bytes = 0;     // persistent {G_prev, A, M}
  size_t work_begin = 0, work_bytes = 0;       // X, S, B of every group (zeroed once)
  size_t stat_off = 0, dyn_off = 0, scales_off = 0, partials_off = 0, blocks_off = 0, optr_off = 0, chain_off = 0;
  size_t total = 0;
  std::vector<Group> groups;
  std::vector<int> group_of, rank_in_group;
  std::vector<BlockWork> blocks;       // ordered: fp32-gradient matrices first, then bf16
  std::vector<int> first_block, num_blocks;
  int max_blocks = 0;                  // most blocks of any matrix
  int keep = 0;                        // what the caches are to keep of the elementwise pass
  // The block table is ordered: early groups (fp32-gradient matrices, then bf16), then the late group (same).
  int range_end[4] = {0, 0, 0, 0};     // ends of those four ranges of blocks
  std::vector<Unit> units;             // what the products of the groups are launched as, in launch order per lane
  int lanes = 1;
  bool small_enough = false;           // all groups together are as little as a chain takes
  size_t fresh_bytes = 0;              // ... what a buffer for every product of kFreshSteps literal iterations takes (0: not that)
  int late_group = -1;                 // group whose elementwise pass runs beside the products of the others
  std::vector<int32_t> order;          // matrix indices: early matrices, then those of the late group
  int num_early = 0;
  size_t order_off = 0;
};

int check_mats(const mona_matrix* mats, int32_t count, bool need_ptrs) {
  if (!mats) return fail(MONA_EINVAL, "mats is NULL");
  if (count < 1) return fail(MONA_EINVAL, "count must be >= 1 (got %d)", count);
  for (int i = 0; i < count; ++i) {
    const mona_matrix& q = mats[i];
    if (q.m < 1 || q.n < 1) return fail(MONA_EINVAL, "matrix %d: m and n must be >= 1 (got %d x %d)", i, q.m, q.n);
    if (q.m > (1 << 30) || q.n > (1 << 30))   // sides are rounded up to tile multiples in 32-bit arithmetic
      return fail(MONA_EINVAL, "matrix %d: m and n must each be at most 2^30 (got %d x %d)", i, q.m, q.n);
    if ((int64_t)q.m * q.n >= (int64_t)1 << 31)
      return fail(MONA_EINVAL, "matrix %d: m * n must be below 2^31 (got %d x %d)", i, q.m, q.n);
    if ((q.w_dtype != MONA_F32 && q.w_dtype != MONA_BF16) || (q.g_dtype != MONA_F32 && q.g_dtype != MONA_BF16))
      return fail(MONA_EINVAL, "matrix %d: dtype must be MONA_F32 or MONA_BF16", i);
    if (need_ptrs) {
      if (!q.w || !q.g) return fail(MONA_EINVAL, "matrix %d: w and g must not be NULL", i);
      if (((uintptr_t)q.w & 15) || ((uintptr_t)q.g & 15))
        return fail(MONA_EINVAL, "matrix %d: w and g must be 16-byte aligned", i);
    }
  }
  return MONA_OK;
}

int check_opts(const mona_options* o, mona_options* out) {
  mona_options z;
  memset(&z, 0, sizeof z);
  if (o) z = *o;
  if (z.ns_precision != 0 && z.ns_precision != 1) return fail(MONA_EINVAL, "ns_precision must be 0 or 1");
  if (z.state_dtype != MONA_F32 && z.state_dtype != MONA_BF16)
    return fail(MONA_EINVAL, "state_dtype must be MONA_F32 or MONA_BF16");
  if (z.accel_form != MONA_ACCEL_TWO_BUFFER && z.accel_form != MONA_ACCEL_ONE_BUFFER &&
      z.accel_form != MONA_ACCEL_CALLER_SLOT)
    return fail(MONA_EINVAL, "accel_form must be MONA_ACCEL_TWO_BUFFER, MONA_ACCEL_ONE_BUFFER or MONA_ACCEL_CALLER_SLOT");
  if (z.max_streams < 0 || z.max_streams > 8) return fail(MONA_EINVAL, "max_streams must lie in [0, 8]");
  if (z.ns_schedule != MONA_NS_SCHEDULE_AUTO && z.ns_schedule != MONA_NS_SCHEDULE_LITERAL &&
      z.ns_schedule != MONA_NS_SCHEDULE_FUSED && z.ns_schedule != MONA_NS_SCHEDULE_PAIRS)
    return fail(MONA_EINVAL, "ns_schedule must be MONA_NS_SCHEDULE_AUTO, _LITERAL, _FUSED or _PAIRS");
  if (z.overlap != MONA_OVERLAP_OFF && z.overlap != MONA_OVERLAP_LATE_GROUP)
    return fail(MONA_EINVAL, "overlap must be MONA_OVERLAP_OFF or MONA_OVERLAP_LATE_GROUP");
  for (int r : z.reserved)
    if (r != 0) return fail(MONA_EINVAL, "reserved option fields must be 0");
  *out = z;
  return MONA_OK;
}

constexpr int kRing = 4;
constexpr int kProfSets = 32;
constexpr int kDefaultLanes = 4;   // streams the shape groups of one step are spread over
// launches of at least this many tiles keep 256 CUs busy for six rounds or more.  Measured: with the limit at
// 512 or 768 mid-sized groups (a bank of 64 experts of 1024 x 2048) lose 4 % by waiting for each other; at
// 3072 the two expert groups of a 128-expert layer run side by side and lose 5 % to each other's L2 traffic.
constexpr long long kBigLaunchTiles = 1536;
constexpr long long kChipTiles = 256;      // one tile per CU
// 128 x 128 tiles up to which small groups share their launches.  Measured, us per step (three runs, within 0.3 %) with the
// line at 64 / 96 / 128 / 176: hidden size 512 (40, 20, 10 tiles) 187 / 173 / 173 / 173, hidden size 700 (84, 21)
// 223 / 223 / 232 / 232, 12 x 384 x 1000 and 4 x 500 x 500 (72, 40) 227 / 227 / 221 / 222, 5 x 520 x 640 and 3 x 640 x 520 (75, 45)
// 190 / 191 / 186 / 186, hidden size 640 (75, 30, 15) 265 / 274 / 268 / 268, hidden size 768 (84, 42, 21) 312 / 312 / 308 / 346,
// hidden size 1000 (144, 72, 36) 515 / 515 / 476 / 476, 16 x 512 x 768 both ways (160, 160) 365 on every line: 128 is best or within
// 1 % of it but for one.
constexpr long long kMergedTiles = 128;
// large tiles from which a product uses them; matrices from which it does where p is a single tile
constexpr long long kMinTiles256 = 128, kMinSingles256 = 112;
// what a chain of small products takes at most at one position: 64 x 64 tiles, and their K added up (chainable() has the figures)
constexpr long long kChainTiles = 448, kChainWork = 140000;
// CUs the late group's elementwise pass keeps to itself (a quarter of the chip): the HBM-bound pass still
// moves 2.8 TB/s there, and the power-limited products lose 13 % on the other three quarters (measured).
constexpr int kOverlapCuShare = 4;
constexpr double kSlowPassBytesPerSec = 2.8e12, kProductFlopPerSec = 1.0e15, kProductSlowdown = 1.13;

// whether one product of a group runs on the 256 x 256 kernel
bool large_tiles(const Group& g, int kind, int count) {
  if (g.f32 || g.gran < 256) return false;
  if (g.large_with_company) return true;
  long long tiles;
  if (kind == OP_APPLY) {
    tiles = (long long)(g.rows_pad / 256) * (g.cols_pad / 256) * count;
  } else {
    const long long t = g.p_pad / 256;
    tiles = t * (t + 1) / 2 * count;
  }
  // Too few large tiles to fill 256 CUs, unless groups running beside this one make up for it.  Measured, us per step
  // (three runs, within 0.3 %) with the line at 192 / 128 / 112 tiles: from 128 tiles on large tiles are faster, 4 x 2048 x 2048
  // (144 tiles a p x p product) 1043 / 847 / 847, 4096 x 4096 (136) 1816 / 1454 / 1452; below, they lose, 12 x 1024 x 2048 (120)
  // 748 / 748 / 768, 4 x 1792 x 1792 (112) 694 / 694 / 714, 8 x 1280 x 1280 (120) 568 / 568 / 580, 20 x 768 x 768 (120 and 180)
  // 461 / 431 / 429.  Where every symmetric product is a single tile the line lies at 112 (literal iterations of so many take
  // the kernel with a workgroup for each matrix, so this is for forced schedules): chunks of three / of two, 115 x 256 x 512
  // 424 / 421 on small tiles and 399 / 401 on large ones, 115 x 256 x 1024 619 / 645 and 597 / 630, 127 x 200 x 250 333 / 316 and 324 / 311, but
  // 120 x 256 x 256 322 / 306 and 331 / 318.
  return tiles >= kMinTiles256 || (g.p_pad == 256 && count >= kMinSingles256);
}
bool small_tiles_only(const Group& g) {
  const int count = (int)g.members.size();
  return !large_tiles(g, OP_GRAM, count) && !large_tiles(g, OP_APPLY, count);
}

// tiles one product launch of a group computes
long long launch_tiles(const Group& g, int kind, int tile, int count) {
  if (kind == OP_APPLY) return (long long)(g.rows_pad / tile) * (g.cols_pad / tile) * count;
  const long long t = g.p_pad / tile;
  return t * (t + 1) / 2 * count;
}

// Whether the matrices of a group get a workgroup each (ns_matrix_kernel), by what their iterations take that way and as
// products, us of a step.  Alone, products take as long as their launches at least; beside other groups, whose launches they share
// or run beside, only what they add.  Measured, us per step as products (launches, or a chain) / by matrix: 128 x 128 47 / 32,
// 8 x 128 x 128 46 / 33, 16 x 100 x 200 62 / 46, 24 x 128 x 512 80 / 76, 60 x 128 x 256 104 / 53, 250 x 70 x 100 161 / 45, 200 x 120 x 600 299 / 176,
// 250 x 128 x 4000 1983 / 1372, but 100 x 400 49 / 68, 4 x 128 x 1024 64 / 136, 40 x 128 x 2000 222 / 309; 256 x 256 x 256 440 / 232,
// 115 x 256 x 512 370 / 281, 128 x 768 x 256 both ways 831 / 611, but 60 x 256 x 512 231 / 239, 79 x 256 x 834 385 / 395; 4 x 171 x 66 beside
// 697 x 612 and 365 x 161 144 / 169; 50 x 256 x 256 170 / 143, 84 x 256 x 256 213 / 157, 70 x 130 x 200 141 / 130, 86 x 256 x 768 438 / 358, but
// 36 x 256 x 256 139 / 137, 28 x 256 x 256 114 / 132, 52 x 160 x 140 116 / 132, 50 x 140 x 380 150 / 171.  (The kernel with a padded short side
// of 256, 120 matrices with 4, 8, 16 panels: 208, 374, 679 us, 204, 360, 672 by the rule; of 128 with 4 and 16: 67 and 267, 55 and 243.)
bool by_matrix(const Group& g, bool alone) {
  if (g.f32 || g.fused || (g.p_pad != 128 && g.p_pad != 256)) return false;
  const double count = (double)g.members.size(), panels = std::max(g.rows_pad, g.cols_pad) / 128;
  const double units = count * panels, rounds = std::ceil(count / (double)kChipTiles);
  if (g.p_pad == 128) {    // (four panels stay in LDS)
    const double latency = alone ? std::min(50.0 + 0.4 * units, 100.0) : 0.0;
    return rounds * 5.0 * (2.2 + (panels <= 4 ? 2.2 : 2.9) * panels) < std::max(0.2 * units, latency);
  }
  const double unit = panels <= 4 ? 0.75 : count >= kMinSingles256 ? 0.45 : 0.55;
  // (products leave out 64 x 64 tiles of padding, this kernel does not)
  const double real = (double)(round_up(g.m, 64) * (int64_t)round_up(g.n, 64)) / ((double)g.rows_pad * g.cols_pad);
  const double latency = alone ? std::min(30.0 + units * real, 160.0) : 0.0;
  return rounds * 5.0 * (9.5 + 7.8 * panels) < std::max(unit * units, latency);
}

// Whether the groups of the step, all together, are as little as a chain takes (of five literal iterations: the exact check
// stands in chainable()).
bool all_in_a_chain(const Layout& L) {
  long long tiles[2] = {0, 0}, work[2] = {0, 0};
  for (const Group& g : L.groups) {
    const long long count = (long long)g.members.size(), p = (std::min(g.m, g.n) + 63) / 64;
    const long long of[2] = {p * (p + 1) / 2 * count, ((g.m + 63LL) / 64) * ((g.n + 63LL) / 64) * count};
    const long long k[2] = {std::max(g.rows_pad, g.cols_pad), g.p_pad};
    for (int i = 0; i < 2; ++i) { tiles[i] += of[i]; work[i] += of[i] * k[i]; }
  }
  return std::max(tiles[0], tiles[1]) <= kChainTiles && std::max(work[0], work[1]) <= kChainWork;
}

// What the elementwise pass moves: reads G, G_prev, A, M; writes G_prev, A, M and the working copy of M (one-buffer form: C in place of
// G_prev and A).
double pass_bytes(const Layout& L, const mona_matrix* mats) {
  double bytes = 0.0;
  for (int i = 0; i < L.count; ++i) {
    const double gsz = mats[i].g_dtype == MONA_BF16 ? 2 : 4, aux = (L.one_buffer ? 1 : 2) * L.ssize;
    bytes += (double)mats[i].m * mats[i].n * (gsz + aux + 4 + aux + 4 + L.groups[L.group_of[i]].esize);
  }
  return bytes;
}

// Streams and order of the step.
//
// Lanes.  A group whose every launch covers the chip many times over gains nothing from company (two
// persistent kernels sharing the CUs only disturb each other's L2 reuse: measured slower), so such groups
// stay in a row on the caller's stream; the others, sorted by work, each go to the least loaded lane, except that
// the groups that run small tiles only are merged first: their products are bound by the latency of a launch, and a
// launch takes as long for eight groups as for one (measured on nine ragged matrices: 982 us a step with a chain of
// launches for each group on four lanes).  They are merged only until their launches put a tile on half of the CUs:
// from there on a merged launch lasts longer with every group, and chains on lanes of their own fill each other's
// gaps (kMergedTiles has the figures).
//
// Late group (on request: mona_options.overlap).  The elementwise pass is bound by HBM and leaves the matrix
// units idle; the products are bound by the matrix units (and by power) and leave HBM half idle.  When the
// groups in the row are several, the elementwise pass of the one with the most elements is taken out of the
// common pass and runs on a stream of its own, confined to a quarter of the CUs, beside the products of the
// other groups, which keep to the remaining three quarters; its own products come last.  Taken only where
// the products of the other groups last about as long as that slowed-down pass, so that it is hidden
// completely.  Measured (388-matrix layer): the pass is hidden, but the products beside it run 10 % slower
// (13 % from the CUs they give up, the rest from sharing HBM), which leaves 3.6 % of the step; not the default.
void plan_lanes(Layout& L, const mona_options& opt) {
  const int want = opt.max_streams == 0 ? kDefaultLanes : opt.max_streams;
  L.late_group = -1;
  L.units.clear();
  const int ngroups = (int)L.groups.size();
  std::vector<long long> fewest_of(ngroups, 0);
  std::vector<double> work_of(ngroups, 0.0);
  std::vector<int> row, beside;
  bool any_big = false;
  for (int gi = 0; gi < ngroups; ++gi) {
    const Group& g = L.groups[gi];
    long long fewest = -1;
    for (int kind = OP_GRAM; kind <= OP_APPLY; ++kind) {
      const int tile = large_tiles(g, kind, (int)g.members.size()) ? 256 : 128;
      const long long t = launch_tiles(g, kind, tile, (int)g.members.size());
      if (fewest < 0 || t < fewest) fewest = t;
    }
    fewest_of[gi] = fewest;
    any_big = any_big || fewest >= kBigLaunchTiles;
    const double p = std::min(g.rows_pad, g.cols_pad), q = std::max(g.rows_pad, g.cols_pad);
    // flop of five iterations on the symmetric count: literal 5 (3 p^2 q + p^3), chunks (3, 2), chunks (2, 2, 1);
    // an fp32 product takes 16 times the time of a bf16 one
    const double per = g.fused == 2 ? 6.0 * p * p * q + 14.0 * p * p * p
                       : g.fused == 1 ? 9.0 * p * p * q + 11.0 * p * p * p : 5.0 * (3.0 * p * p * q + p * p * p);
    work_of[gi] = per * (double)g.members.size() * (g.f32 ? 16.0 : 1.0);
  }
  // A workgroup for each matrix: not where a chain that some groups need anyway takes all of them (the others cost it little).
  const bool only = L.gfx950 && std::all_of(L.groups.begin(), L.groups.end(), [](const Group& g) { return by_matrix(g, true); });
  std::vector<int> matrices;
  for (int gi = 0; gi < ngroups; ++gi) {
    if (only || (L.gfx950 && !L.small_enough && by_matrix(L.groups[gi], false))) { matrices.push_back(gi); continue; }
    // Beside a group that keeps the caller's stream, only groups too small to fill the chip by
    // themselves go to the side streams (their launch latency hides behind the large group); a
    // mid-sized group there gained 0.3 % at most (4 squares of 4096 beside 384 experts), and in a row
    // the per-launch times of a profile add up to the phase time.
    const bool in_row = fewest_of[gi] >= kBigLaunchTiles || (any_big && fewest_of[gi] >= kChipTiles);
    (in_row ? row : beside).push_back(gi);
  }
  std::stable_sort(beside.begin(), beside.end(), [&](int x, int y) { return work_of[x] > work_of[y]; });
  // The groups on the lanes run side by side.  When their launches, taken together, put a large tile
  // on at least half of the CUs, each of them uses the large-tile kernel even where its own launch
  // alone would be too small for it (measured on one dense block of hidden size 2048: 2.43 against
  // 2.80 ms per step).
  if (std::min(want, ngroups) > 1) {
    long long together = 0;
    for (int gi : beside) {
      const Group& g = L.groups[gi];
      if (g.f32 || g.gran < 256) continue;
      long long fewest = -1;
      for (int kind = OP_GRAM; kind <= OP_APPLY; ++kind) {
        const long long t = launch_tiles(g, kind, 256, (int)g.members.size());
        if (fewest < 0 || t < fewest) fewest = t;
      }
      together += fewest;
    }
    if (together >= 128)
      for (int gi : beside) L.groups[gi].large_with_company = true;
  }
  // Units: every group that uses the large-tile kernel by itself; the others merged, bf16 and fp32 apart (one kernel
  // per launch).
  auto add_unit = [&](bool merged) -> Unit& {
    L.units.emplace_back();
    L.units.back().merged = merged;
    return L.units.back();
  };
  for (int gi : row) add_unit(false).groups.push_back(gi);
  // (the most work a matrix first: the launch ends with the short ones)
  std::stable_sort(matrices.begin(), matrices.end(), [&](int x, int y) {
    return work_of[x] / (double)L.groups[x].members.size() > work_of[y] / (double)L.groups[y].members.size();
  });
  for (size_t i = 0; i < matrices.size(); ++i) {
    if (i % kMaxMerged == 0) add_unit(false).matrix = true;
    L.units.back().groups.push_back(matrices[i]);
  }
  const size_t first_beside = L.units.size();
  std::vector<long long> tiles_in(L.groups.size() + 1, 0);   // 128 x 128 tiles of each unit's smallest launches
  for (int gi : beside) {
    const Group& g = L.groups[gi];
    if (!small_tiles_only(g)) { add_unit(false).groups.push_back(gi); continue; }
    size_t u = first_beside;
    for (; u < L.units.size(); ++u) {
      const Unit& q = L.units[u];
      if (q.merged && L.groups[q.groups[0]].f32 == g.f32 && (int)q.groups.size() < kMaxMerged &&
          (want == 1 || tiles_in[u] + fewest_of[gi] <= kMergedTiles))
        break;
    }
    if (u == L.units.size()) add_unit(true);
    L.units[u].groups.push_back(gi);
    tiles_in[u] += fewest_of[gi];
  }
  const int parallel = (int)(L.units.size() - first_beside) + (row.empty() && matrices.empty() ? 0 : 1);
  L.lanes = std::max(1, std::min(want, parallel));
  std::vector<double> load(L.lanes, 0.0);
  for (int gi : row) load[0] += work_of[gi];
  for (int gi : matrices) load[0] += work_of[gi];
  std::vector<std::pair<double, size_t>> order;
  for (size_t u = first_beside; u < L.units.size(); ++u) {
    double work = 0.0;
    for (int gi : L.units[u].groups) work += work_of[gi];
    order.emplace_back(-work, u);
  }
  std::sort(order.begin(), order.end());
  for (auto& pr : order) {
    const int lane = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    L.units[pr.second].lane = lane;
    load[lane] -= pr.first;
  }
  if (opt.overlap == MONA_OVERLAP_LATE_GROUP && row.size() >= 2 && !L.external_state) {
    int late = -1;
    double most = 0.0, others = 0.0;
    auto elems = [&](int gi) { return (double)L.groups[gi].m * L.groups[gi].n * (double)L.groups[gi].members.size(); };
    for (int gi : row)
      if (elems(gi) > most) { most = elems(gi); late = gi; }
    for (int gi : row)
      if (gi != late) others += work_of[gi];
    const double slow_pass = 30.0 * most / kSlowPassBytesPerSec;
    if (kProductSlowdown * others / kProductFlopPerSec >= 0.95 * slow_pass && slow_pass >= 1.0e-3) L.late_group = late;
    // the late group comes last: its elementwise pass must have finished, and from then on the chip is free
    if (L.late_group >= 0)
      std::stable_partition(L.units.begin(), L.units.end(), [&](const Unit& u) { return u.groups[0] != L.late_group; });
  }
}

// `launches`: also what the products are launched as, for which the device is asked (nothing of it changes the sizes).
void build_layout(const mona_matrix* mats, int count, const mona_options& opt, bool external_state, bool launches, Layout& L) {
  L.count = count;
  L.external_state = external_state;
  L.ssize = opt.state_dtype == MONA_BF16 ? 2 : 4;
  L.one_buffer = opt.accel_form == MONA_ACCEL_ONE_BUFFER;
  L.caller_slot = opt.accel_form == MONA_ACCEL_CALLER_SLOT;
  size_t off = 0;
  // persistent state, contiguous: this block is what checkpoints carry
  L.state_begin = off;
  L.gprev_off.resize(count);
  L.acc_off.resize(count);
  L.mom_off.resize(count);
  for (int i = 0; i < count; ++i) {
    const size_t ne = (size_t)mats[i].m * mats[i].n;
    L.gprev_off[i] = off;
    if (external_state) { L.acc_off[i] = L.mom_off[i] = off; continue; }
    if (!L.one_buffer && !L.caller_slot) off = align_up(off + ne * L.ssize);
    L.acc_off[i] = off;   off = align_up(off + ne * L.ssize);
    L.mom_off[i] = off;   off = align_up(off + ne * 4);
  }
  L.state_bytes = off - L.state_begin;

  // groups of equal shape (order of first appearance)
  std::map<std::pair<int, int>, int> index;
  L.group_of.resize(count);
  L.rank_in_group.resize(count);
  for (int i = 0; i < count; ++i) {
    auto key = std::make_pair(mats[i].m, mats[i].n);
    auto it = index.find(key);
    int gi;
    if (it == index.end()) {
      gi = (int)L.groups.size();
      index[key] = gi;
      Group g;
      g.m = mats[i].m;
      g.n = mats[i].n;
      g.tall = g.m > g.n;
      const int r128 = round_up(g.m, 128), c128 = round_up(g.n, 128);
      // bf16 rounding errors of the p x p Gram entries average out over p singular directions;
      // below p = 64 they do not, and the products cost nothing there, so they run in fp32
      g.f32 = opt.ns_precision == 1 || std::min(g.m, g.n) <= kSmallSideF32;
      g.esize = g.f32 ? 4 : 2;
      g.gran = (!g.f32 && r128 % 256 == 0 && c128 % 256 == 0) ? 256 : 128;
      g.rows_pad = r128;
      g.cols_pad = c128;
      g.p_pad = g.tall ? g.cols_pad : g.rows_pad;
      // The fused schedule trades products with the long side q for products on the p x p side, so it pays
      // when q is well above p.  Advancing the Gram matrix on the p x p side is as accurate as recomputing
      // it from X while its eigenvalues are still small (the growth phase of the iteration) and less so
      // once they have reached the band around 1.  A full-rank matrix of this shape starts from singular
      // values up to about 1 / sqrt(p) + 1 / sqrt(q) and each early iteration multiplies them by a = 3.4445,
      // so the automatic choice fuses three iterations only where a^2 times that bound is still around one
      // half, and otherwise pairs of iterations, down to a short side of 1024.  Measured O error against the
      // float64 oracle on the benchmark's inputs, (3, 2) / (2, 2, 1) / literal: 1536 x 4096 7.1e-3 / 1.07e-2 /
      // 9.1e-3, 2048 x 8192 6.8e-3 / 1.07e-2 / 9.7e-3; 1024 x 2048 1.5e-2 / 1.2e-2 / 9.5e-3, 1024 x 4096
      // 1.4e-2 / 9.5e-3 / 9.1e-3; 512 x 4096 1.6e-2 / 1.3e-2 / 1.3e-2 (too small to gain: literal).
      const double q_pad = g.tall ? g.rows_pad : g.cols_pad;
      const double start = 1.0 / std::sqrt((double)g.p_pad) + 1.0 / std::sqrt(q_pad);
      g.fused = 0;
      if (!g.f32) {
        if (opt.ns_schedule == MONA_NS_SCHEDULE_FUSED) g.fused = 2;
        else if (opt.ns_schedule == MONA_NS_SCHEDULE_PAIRS) g.fused = 1;
        else if (opt.ns_schedule == MONA_NS_SCHEDULE_AUTO && 2.0 * q_pad >= 3.0 * g.p_pad)
          g.fused = start <= kFusedMaxStart ? 2 : (g.p_pad >= kPairsMinShortSide ? 1 : 0);
      }
      g.npp = g.fused ? 6 : 2;
      L.groups.push_back(g);
    } else {
      gi = it->second;
    }
    L.group_of[i] = gi;
    L.rank_in_group[i] = (int)L.groups[gi].members.size();
    L.groups[gi].members.push_back(i);
  }
  L.work_begin = off;
  for (Group& g : L.groups) {
    const size_t cnt = g.members.size();
    g.x_stride = (int64_t)g.rows_pad * g.cols_pad;
    g.s_stride = (int64_t)g.p_pad * g.p_pad;
    for (int b = 0; b < 2; ++b) { g.x_off[b] = off; off = align_up(off + cnt * g.x_stride * g.esize); }
    for (int b = 0; b < g.npp; ++b) { g.pp_off[b] = off; off = align_up(off + cnt * g.s_stride * g.esize); }
  }
  L.work_bytes = off - L.work_begin;
  L.small_enough = all_in_a_chain(L);
  if (L.small_enough && L.groups.size() <= (size_t)(kMaxMerged * kMaxChains) &&
      std::all_of(L.groups.begin(), L.groups.end(), [](const Group& g) { return !g.fused; }))
    for (Group& g : L.groups) {
      g.fresh_off = L.fresh_bytes;
      L.fresh_bytes += 2 * kFreshSteps * (g.pp_off[1] - g.pp_off[0]) + (kFreshSteps - 1) * (g.x_off[1] - g.x_off[0]);
    }

  if (launches) {
    L.gfx950 = device_is_gfx950();
    plan_lanes(L, opt);
  }

  double copies = 0.0;
  for (const Group& g : L.groups) copies += (double)g.m * g.n * (double)g.members.size() * g.esize;
  L.keep = choose_keep(copies);

  // elementwise work table
  L.first_block.assign(count, 0);
  L.num_blocks.assign(count, 0);
  for (int pass = 0; pass < 4; ++pass) {
    for (int i = 0; i < count; ++i) {
      if ((mats[i].g_dtype == MONA_BF16) != ((pass & 1) == 1)) continue;
      if ((L.group_of[i] == L.late_group) != (pass >= 2)) continue;
      const int64_t ne = (int64_t)mats[i].m * mats[i].n;
      const int nb = (int)((ne + kEwChunk - 1) / kEwChunk);
      L.first_block[i] = (int)L.blocks.size();
      L.num_blocks[i] = nb;
      L.max_blocks = std::max(L.max_blocks, nb);
      for (int c = 0; c < nb; ++c) L.blocks.push_back(BlockWork{i, c});
    }
    L.range_end[pass] = (int)L.blocks.size();
  }
  for (int late = 0; late < 2; ++late) {
    for (int i = 0; i < count; ++i)
      if ((L.group_of[i] == L.late_group) == (late == 1)) L.order.push_back(i);
    if (late == 0) L.num_early = (int)L.order.size();
  }

  // tables
  L.stat_off = off;     off = align_up(off + sizeof(MatStatic) * count);
  L.dyn_off = off;      off = align_up(off + sizeof(MatDynamic) * count);
  L.scales_off = off;   off = align_up(off + sizeof(MatScale) * count);
  L.optr_off = off;     off = align_up(off + sizeof(void*) * count);
  L.order_off = off;    off = align_up(off + sizeof(int32_t) * count);
  L.partials_off = off; off = align_up(off + sizeof(double) * L.blocks.size());
  L.blocks_off = off;   off = align_up(off + sizeof(BlockWork) * L.blocks.size());
  for (Group& g : L.groups) { g.members_off = off; off = align_up(off + sizeof(int32_t) * g.members.size()); }
  // (the static workspace has its own place for it, so that the matrices that fit are those they always were)
  if (external_state) L.chain_off = MONA_NOALLOC_SCRATCH_BYTES;
  else { L.chain_off = off; off = align_up(off + kChainBytes); }
  L.total = off;
}

constexpr int kWholeMatrices = 4;      // kind of a record that is no product (OpKind)
struct LaunchRecord {
  int kind, group, iter, tile;
  double flops;
  hipEvent_t e0, e1;
};

}  // namespace

// One product of the plan.
struct Op {
  GemmArgs a;         // what `code` stands for (expand_op)
  uint32_t code = 0;  // op code (OpField)
  int kind = 0;       // OpKind
  int group = 0;
  int iter = 0;       // Newton-Schulz iteration it belongs to
  bool large = false; // 256 x 256 kernel; otherwise the tile is chosen when the launch is put together
};

// One launch of the step: a product of one group, the products of a merged unit at one position of their chains, or
// (chain >= 0) whole chains.
struct Launch {
  int n = 0;
  Op* op[kMaxMerged];
  bool wide = false;   // small tiles: eight wavefronts a tile (see launch_ns_small)
  bool split = false;  // fp32 products on the bf16 matrix instructions (see launch_ns_split)
  int chain = -1;      // index in Plan::chains
  int matrix = -1;     // index in Plan::matrices
  int wgs = 0;         // workgroups of a chain launch
};

// The products of one step as they are launched, lane by lane: what enqueue_step issues and mona_plan_info counts.
struct Plan {
  StepDesc step;
  std::vector<GroupDesc> desc;              // by group
  std::vector<std::vector<Op>> ops;         // by group
  std::vector<int> o_buf;                   // by group: the ping-pong buffer that holds O_k afterwards
  std::vector<std::vector<Launch>> lanes;
  std::vector<ChainArgs> chains;
  std::vector<MatrixBatch> matrices;
  std::vector<std::vector<int>> chain_groups, matrix_groups;   // the groups of each, in order
  int32_t ns_steps = -1;                    // what it was built for
  uint32_t flags = 0;
  bool one_by_one = false;
  size_t chain_bytes = 0;                   // of rolls and flags, to be cleared before the products
  int chain_tasks = 0;
  bool fresh = false;                       // every product has a buffer of its own
  FillArgs fill;                            // what these are filled with before the products
};

struct mona_state {
  Layout L;
  mona_options opt;
  std::vector<mona_matrix> mats;   // shapes/dtypes given at init (pointers unused)
  char* arena = nullptr;
  int64_t k = 0;
  float last_beta_a = -1.0f;       // one-buffer form: beta_a of the previous step (< 0: none yet)
  // Shape groups are independent of each other, so their Newton-Schulz chains run on separate
  // streams: lane 0 is the caller's stream, lanes 1.. are side streams forked from it after the
  // elementwise pass and joined back before mona_step returns.
  std::vector<hipStream_t> side;       // lanes 1..
  std::vector<hipEvent_t> side_done;   // one per side stream
  hipEvent_t fork_ev = nullptr;
  // the late group's elementwise pass: a stream confined to a quarter of the CUs
  hipStream_t late_stream = nullptr;
  hipEvent_t late_fork = nullptr, late_done = nullptr;
  int late_cus = 0;                    // CUs that stream may use (0: no such stream)
  // pinned ring for the per-step pointer table of lists longer than kInlineMats
  MatDynamic* ring[kRing] = {nullptr, nullptr, nullptr, nullptr};
  hipEvent_t ring_ev[kRing];
  bool ring_used[kRing] = {false, false, false, false};
  int ring_next = 0;
  std::vector<MatDynamic> last_dyn;  // the pointer table enqueued last
  bool dyn_valid = false;            // last_dyn is what the device's table holds at this point of the stream
  bool captured = false;             // a step of this state was recorded into a graph (see step_impl)
  int device = 0;
  // profiling
  int profiling = 0;
  hipEvent_t ev[kProfSets][4];     // phase marks of the last kProfSets profiled steps, used in turn
  int64_t prof_steps = 0;          // profiled steps since mona_set_profiling
  bool ev_valid = false;
  bool times_ready = false;
  bool fused_update = false;
  bool failed = false;             // a launch failed half way through a step: the state arrays are not usable
  std::vector<LaunchRecord> records;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> event_pool;
  size_t pool_used = 0;

  struct Plan* plan = nullptr;     // of the last step (see plan_for)
  int chain_roll_polls = kRollPolls, chain_patience = kPatience;   // (see ChainArgs)
  char* fresh = nullptr;           // a buffer for every product of a chain: a part of the pool, or of the scratch of mona_step_noalloc
  bool from_pool = false;
  mona_state() = default;
  mona_state(const mona_state&) = delete;
  ~mona_state() { delete plan; }

  template <typename T> T* at(size_t off) const { return reinterpret_cast<T*>(arena + off); }
};

namespace {

// Flop that the matrix units execute, padding included (an fp32 product counts once, however it is carried out): of a
// product (tiles of 32 and 64 leave out the slabs of 32 along K that are padding alone, but for split ones), ...
double gemm_flops(const GemmArgs& a, bool split) {
  const int k = a.tile_m <= 64 && !split ? std::min(round_up(a.k_real, 32), a.K) : a.K;
  return 2.0 * a.tile_m * a.tile_n * (double)k * a.tiles_per_mat * a.count;
}
// ... of `steps` iterations of a group whose matrices get a workgroup each (both triangles of S and S S), ...
double matrix_flops(const GroupDesc& g, int steps) {
  const double p = g.tall ? g.cols_pad : g.rows_pad, q = g.tall ? g.rows_pad : g.cols_pad;
  return steps * (4.0 * p * p * q + 2.0 * p * p * p) * g.count;
}
// ... and of a launch.
double launch_flops(const Plan& plan, const Launch& l) {
  double flops = 0.0;
  if (l.matrix >= 0)
    for (int gi : plan.matrix_groups[l.matrix]) flops += matrix_flops(plan.desc[gi], plan.ns_steps);
  else if (l.chain >= 0)
    for (int gi : plan.chain_groups[l.chain])
      for (const Op& op : plan.ops[gi]) flops += gemm_flops(op.a, false);
  else
    for (int i = 0; i < l.n; ++i) flops += gemm_flops(l.op[i]->a, l.split);
  return flops;
}

void set_tile(const Plan& plan, Op& op, int tile) {
  op.code = (op.code & ~(3u << OPF_TILE)) | (tile == 32 ? 0u : tile == 64 ? 1u : tile == 128 ? 2u : 3u) << OPF_TILE;
  expand_op(plan.step, plan.desc[op.group], op.code, op.a);
}

// Tile of a launch of small tiles: 64 x 64 (four times the workgroups, each with a quarter of the work) until there
// are enough 128 x 128 tiles.  Measured, us per step with the limit at 64 / 128 / 256 tiles: 2 x 768 x 3072 both ways
// 464 / 409 / 409, one 2048 x 2048 404 / 404 / 457, a block of hidden size 1000 537 / 537 / 564.
// An fp32 tile takes 16 times as long, so there an even share for every CU matters more: 128 x 128 only from four such tiles
// per CU on.
constexpr long long kMinTiles128 = 128, kMinTiles128F32 = 1024;
constexpr int kShortK = 128;
// fp32 products (ns_small_kernel_split) keep a CU busy for long, so the rounds of the launch count: us a tile, measured, one workgroup
// a CU.
constexpr double kSplit128 = 0.042, kSplit64 = 0.0146, kSplitFixed = 4.0;   // per value of K; prologue and epilogue
void choose_small_tile(const Plan& plan, Op* const* ops, int n, bool split) {
  long long tiles = 0, tiles64 = 0;
  int k = 0;
  for (int i = 0; i < n; ++i) {
    set_tile(plan, *ops[i], 64);
    tiles64 += (long long)ops[i]->a.tiles_per_mat * ops[i]->a.count;
    set_tile(plan, *ops[i], 128);
    tiles += (long long)ops[i]->a.tiles_per_mat * ops[i]->a.count;
    k = std::max(k, ops[i]->a.K);
  }
  const long long cus = device_cu_count();
  const double t64 = (double)((tiles64 + cus - 1) / cus) * (k * kSplit64 + kSplitFixed);
  const double t128 = (double)((tiles + cus - 1) / cus) * (k * kSplit128 + kSplitFixed);
  for (int i = 0; i < n; ++i) {
    const bool f32 = plan.desc[ops[i]->group].f32 != 0;
    const long long t128_per_mat = ops[i]->a.tiles_per_mat;
    set_tile(plan, *ops[i], 64);
    // (a 64 x 64 tile costs about 0.3 of a 128 x 128 one: where 128 pads the sides that much, 64 is less work)
    if ((split ? t128 <= t64 : tiles >= (f32 ? kMinTiles128F32 : kMinTiles128)) && ops[i]->a.tiles_per_mat * 3 >= t128_per_mat * 10)
      set_tile(plan, *ops[i], 128);
  }
}

// Newton-Schulz iterations per chunk.  Literal schedule: one.  Fused schedules: three and then twos, or twos
// only (measured on bf16-rounded products: fusing the late iterations, or more than three of them, loses
// accuracy; three early ones and pairs afterwards do not).
std::vector<int> chunk_sizes(int T, int fused) {
  std::vector<int> out;
  if (!fused) { out.assign(T, 1); return out; }
  int left = T;
  if (fused == 2 && left >= 3) { out.push_back(3); left -= 3; }
  while (left >= 2) { out.push_back(2); left -= 2; }
  if (left) out.push_back(1);
  return out;
}

// Builds the product launches of one group for one step.
//
// Literal schedule, per iteration (Eq. newton_schulz with B = b S + c S S factored out):
//     S = X X^T;  B = b S + c S S;  X <- a X + B X            (tall: S = X^T X, X <- a X + X B)
// Fused schedule, per chunk of n iterations.  With Q_t = a I + b S_t + c S_t^2 one iteration is
// X_{t+1} = Q_t X_t and its Gram matrix is S_{t+1} = Q_t S_t Q_t = S_t Q_t^2 (polynomials of one symmetric
// matrix commute), so n iterations need X only at both ends:
//     S = X X^T;  for i < n:  Q_i = a I + b S + c S S;  (i < n - 1:  U = S Q_i;  S <- U Q_i);  R <- R Q_i  (R_0 = Q_0)
//     X <- R X
// The same polynomial of X in exact arithmetic, with 3 p^2 q + (4 n - 3) p^3 flop instead of n (3 p^2 q + p^3)
// on the symmetric count, i.e. fewer whenever q > p.  Every p x p result is computed on the upper block
// triangle and mirrored.  A chunk of one iteration is the literal iteration.
struct OpBuilder {
  const Group& g;
  int gi;
  const mona_hparams& hp;
  Plan& plan;
  std::vector<Op>& out;
  int cnt;

  OpBuilder(const Group& g_, int gi_, const mona_hparams& hp_, Plan& plan_)
      : g(g_), gi(gi_), hp(hp_), plan(plan_), out(plan_.ops[gi_]), cnt((int)g_.members.size()) {}
  void push(uint32_t code, int kind, int iter, bool tp, bool tq);
  void gram(int src, uint32_t S, bool first, int iter);
  void poly(uint32_t S, uint32_t dst, bool diag, int iter);
  void symprod(uint32_t P, uint32_t Q, uint32_t dst, int iter);
  void apply(int src, uint32_t Bm, bool with_e, bool first, bool last, int iter);
  int build();   // returns the ping-pong buffer that holds O_k afterwards
};

void OpBuilder::push(uint32_t code, int kind, int iter, bool tp, bool tq) {
  Op op;
  op.code = code | (uint32_t)kind << OPF_KIND | (uint32_t)tp << OPF_TP | (uint32_t)tq << OPF_TQ;
  op.kind = kind; op.group = gi; op.iter = iter;
  op.large = large_tiles(g, kind, cnt);
  set_tile(plan, op, op.large ? 256 : 64);
  out.push_back(op);
}

// The p x p matrices are symmetric bit for bit outside their diagonal tiles (mirrored tiles are copies), and
// inside a diagonal tile either triangle is the product to rounding, so as operands they may be read K-major
// as well as row-major.  The large-tile kernel fetches a K-major operand as 32 contiguous 512-byte rows
// instead of 64-byte pieces of 256 rows and runs 7-13 % faster per K step on it (measured).  The small-tile kernel
// gains the same way in bf16 (128- or 256-byte rows; us per step, row-major -> K-major: 1 x 2048 x 8192 716 -> 683,
// 3328 x 3328 1079 -> 1018, 3072 x 12288 1926 -> 1781, 512 x 256 unchanged) and nothing in fp32, where a product is
// bound by its multiplications (a block of hidden size 1024: 2353 row-major, 2373 K-major).

void OpBuilder::gram(int src, uint32_t S, bool first, int iter) {
  push(S << OPF_C | (uint32_t)src << OPF_SRC | (uint32_t)first << OPF_FIRST, OP_GRAM, iter, g.tall, g.tall);
}

void OpBuilder::poly(uint32_t S, uint32_t dst, bool diag, int iter) {
  push(S << OPF_P | S << OPF_Q | dst << OPF_C | (uint32_t)diag << OPF_DIAG, OP_POLY, iter, !g.f32, !g.f32);
}

void OpBuilder::symprod(uint32_t P, uint32_t Q, uint32_t dst, int iter) {
  push(P << OPF_P | Q << OPF_Q | dst << OPF_C, OP_SYMPROD, iter, !g.f32, !g.f32);
}

void OpBuilder::apply(int src, uint32_t Bm, bool with_e, bool first, bool last, int iter) {
  const bool symk = !g.f32;
  uint32_t code = Bm << OPF_P | Bm << OPF_Q | (uint32_t)src << OPF_SRC | (uint32_t)with_e << OPF_E |
                  (uint32_t)first << OPF_FIRST | (uint32_t)last << OPF_LAST;
  if (hp.flags & MONA_FLAG_KEEP_O) code |= 1u << OPF_STORE;
  // tall: X' = a X + X B, the Q operand is B; wide: X' = a X + B X, P is B and Q is X
  // (the large-tile launch with the update has no register for a K-major P)
  if (g.tall) push(code, OP_APPLY, iter, false, symk);
  else push(code, OP_APPLY, iter, symk && !(last && large_tiles(g, OP_APPLY, cnt)), true);
}

int OpBuilder::build() {
  const int T = hp.ns_steps;
  const std::vector<int> chunks = chunk_sizes(T, g.fused);
  int src = 0, iter = 0;
  for (size_t ci = 0; ci < chunks.size(); ++ci) {
    const int n = chunks[ci];
    const bool first = ci == 0, last = ci + 1 == chunks.size();
    if (n == 1) {
      gram(src, 0, first, iter);
      poly(0, 1, false, iter);
      apply(src, 1, true, first, last, iter);
    } else {
      uint32_t S = 0, S2 = 1, U = 2, Q = 3, R = 4, R2 = 5;
      gram(src, S, first, iter);
      for (int i = 0; i < n; ++i) {
        const uint32_t Qi = i == 0 ? R : Q;        // Q_0 is R_0
        poly(S, Qi, true, iter + i);
        if (i + 1 < n) {
          symprod(S, Qi, U, iter + i);
          symprod(U, Qi, S2, iter + i);
          std::swap(S, S2);
        }
        if (i > 0) {
          symprod(R, Q, R2, iter + i);
          std::swap(R, R2);
        }
      }
      apply(src, R, false, first, last, iter + n - 1);
    }
    src ^= 1;
    iter += n;
  }
  return T == 0 ? 1 : src;
}

// Tiles of the products of `groups` at position `pos` when all of them are `tile` wide.
long long tiles_at(Plan& plan, const std::vector<int>& groups, size_t pos, int tile) {
  long long tiles = 0;
  for (int gi : groups) {
    if (pos >= plan.ops[gi].size()) continue;
    Op& op = plan.ops[gi][pos];
    set_tile(plan, op, tile);
    tiles += (long long)op.a.tiles_per_mat * op.a.count;
  }
  return tiles;
}

// Whether the products of these groups may go out as one launch (ns_chain_kernel) instead of one launch per position.
//
// Where the line (kChainTiles, kChainWork) lies.  A chain saves 2 to 4 us of every product, but its workgroups are one to a CU and its tiles 64 x 64
// at most, dealt without regard to the die they are on.  Measured, us per step with launches / as a chain, with the work of the
// widest position (64 x 64 tiles times K, in thousands): 256 x 256 (4) 92 / 54, 512 x 512 (33) 109 / 74, 512 x 2048 (131) 145 / 104,
// 4 x 300 x 900 (115) 122 / 87, 200 x 64 x 128 (51, fp32) 127 / 124, 768 x 768 (110) 130 / 106, 4 x 512 x 512 (131) 117 / 97,
// 28 x 256 x 256 (115) 126 / 114.  Beyond it chains lose where the short side is 256 or less, 30 x 256 x 512 (245) 156 / 183, 20 x 256 x 512 (164)
// 128 / 128, 36 x 256 x 256 (147) 140 / 152, 250 x 70 x 100 (192, 1000 tiles) 166 / 223, and win where it is longer: 1024 x 1024 (262) 150 / 125,
// 6 x 384 x 1000 (221) 147 / 137, 700 x 2000 (270) 166 / 139, 2 x 640 x 1280 (256) 154 / 132.  The line is that of chains with flags and three
// launches in front, which lost 4 % at 1024 x 1024 and 6 x 384 x 1000; tiles and work alone do not part the two kinds.
// The tile a chain takes at one position: 32 x 32 as long as every one has a CU of its own.
int chain_tile(Plan& plan, const std::vector<int>& groups, size_t pos) {
  return tiles_at(plan, groups, pos, 32) <= device_cu_count() ? 32 : 64;
}
// Tasks of the chain, 0 if there is none.
int chainable(const Layout& L, Plan& plan, const std::vector<int>& groups) {
  if (!L.gfx950 || groups.size() > (size_t)kMaxMerged) return 0;
  size_t ops = 0, positions = 0;
  for (int gi : groups) {
    const Group& g = L.groups[gi];
    ops += plan.ops[gi].size();
    positions = std::max(positions, plan.ops[gi].size());
    // a matrix is addressed with 32-bit byte offsets
    if (std::max(g.x_stride, g.s_stride) * g.esize >= (int64_t)1 << 31) return 0;
  }
  if (ops == 0 || ops > (size_t)kMaxChainOps) return 0;
  long long tasks = 0;
  for (size_t pos = 0; pos < positions; ++pos) {
    if (tiles_at(plan, groups, pos, 64) > kChainTiles) return 0;
    long long work = 0;
    for (int gi : groups)
      if (pos < plan.ops[gi].size()) {
        const GemmArgs& a = plan.ops[gi][pos].a;
        work += (long long)a.tiles_per_mat * a.count * a.K;
      }
    if (work > kChainWork) return 0;
    const int tile = chain_tile(plan, groups, pos);
    // A 64 x 64 tile takes the fp32 instructions 14 us with K = 512, where launches take the bf16 ones.  Measured, us per step
    // with fp32 products as a chain / with launches: 512 x 512 (32 x 32) 139 / 186, 512 x 1408 199 / 245, but 768 x 768 323 / 238,
    // 2 x 512 x 512 239 / 191, 16 x 256 x 256 162 / 135.
    for (int gi : groups)
      if (tile == 64 && L.groups[gi].f32 && L.groups[gi].p_pad > 128 && pos < plan.ops[gi].size() && plan.ops[gi][pos].a.symmetric)
        return 0;
    tasks += tiles_at(plan, groups, pos, tile);
  }
  return tasks <= kMaxChainTasks ? (int)tasks : 0;
}

// Puts the chain of `groups` together: the tiles of every product, then the tasks in order.  `launches` receives the
// products position by position, as they are launched when each is timed by itself; returns the chain's own launch.
Launch build_chain(const mona_state* st, Plan& plan, const std::vector<int>& groups, std::vector<Launch>& launches) {
  const Layout& L = st->L;
  const int cus = device_cu_count();
  char* const area = st->arena + L.chain_off;
  ChainArgs c;
  memset(&c, 0, sizeof c);
  c.step = plan.step;
  c.roll_polls = st->chain_roll_polls;
  c.patience = st->chain_patience;
  c.fresh = plan.fresh;
  c.roll = reinterpret_cast<ChainRoll*>(area) + plan.chains.size();
  c.flags = reinterpret_cast<uint32_t*>(area + kMaxChains * sizeof(ChainRoll)) + plan.chain_tasks;
  struct Before { int32_t first = 0, per_mat = 0; };
  std::vector<Before> before(groups.size());
  long long tasks = 0, most = 0;
  for (size_t j = 0; j < groups.size(); ++j) c.group[j] = plan.desc[groups[j]];
  for (size_t pos = 0;; ++pos) {
    Launch l;
    const long long here = tiles_at(plan, groups, pos, chain_tile(plan, groups, pos));
    for (int gi : groups)
      if (pos < plan.ops[gi].size()) l.op[l.n++] = &plan.ops[gi][pos];
    if (l.n == 0) break;
    // the longest K first: its tiles are the last to finish
    std::stable_sort(l.op, l.op + l.n, [](const Op* x, const Op* y) { return x->a.K > y->a.K; });
    for (int i = 0; i < l.n; ++i) {
      const Op& op = *l.op[i];
      const size_t j = std::find(groups.begin(), groups.end(), op.group) - groups.begin();
      const int32_t first = (int32_t)tasks;
      tasks += (long long)op.a.tiles_per_mat * op.a.count;
      c.op[c.ops++] = ChainOp{(int32_t)tasks, before[j].first, before[j].per_mat, op.code | (uint32_t)j << OPF_GROUP};
      before[j].first = first;
      before[j].per_mat = op.a.tiles_per_mat;
    }
    most = std::max(most, here);
    l.wide = true;
    launches.push_back(l);
  }
  c.tasks = (int32_t)tasks;
  for (int i = c.ops; i < kMaxChainOps + 3; ++i) c.op[i].end = INT32_MAX;
  Launch chain;
  chain.wgs = (int)std::min<long long>(most, cus);
  chain.chain = (int)plan.chains.size();
  plan.chains.push_back(c);
  plan.chain_groups.push_back(groups);
  plan.chain_tasks += round_up((int)tasks, 4);
  plan.chain_bytes = kMaxChains * sizeof(ChainRoll) + plan.chain_tasks * sizeof(uint32_t);
  return chain;
}

// The hyper-parameters of a step that change nothing of its launches but their arguments.
void set_step(const mona_state* st, const mona_hparams& hp, Plan& plan) {
  const Layout& L = st->L;
  memset(&plan.step, 0, sizeof plan.step);
  plan.step.scales = st->at<MatScale>(L.scales_off);
  plan.step.stat = st->at<MatStatic>(L.stat_off);
  plan.step.dyn = st->at<MatDynamic>(L.dyn_off);
  plan.step.ns_a = hp.ns_a; plan.step.ns_b = hp.ns_b; plan.step.ns_c = hp.ns_c;
  plan.step.w_keep = 1.0f - hp.lr * hp.weight_decay;
}
float update_scale(const Group& g, const mona_hparams& hp) {
  return hp.lr * hp.gamma_coeff * sqrtf((float)std::max(g.m, g.n));
}

// What the products of `steps` iterations of a group write before the last one: X_1 .., and all S and B.
void add_fill(Plan& plan, const Group& g, size_t gi, int steps) {
  const GroupDesc& d = plan.desc[gi];
  int tile = 32;
  for (const Op& op : plan.ops[gi]) tile = std::max(tile, (int)op.a.tile_m);
  auto add = [&](char* at, int buffers, int64_t stride, int cols_pad, int rows, int cols) {
    if (buffers <= 0) return;
    FillItem& t = plan.fill.item[plan.fill.n++];
    t.at = at;
    t.stride = (uint32_t)(stride * g.esize);
    t.pitch = (uint32_t)(cols_pad * g.esize);
    t.rows = (uint32_t)round_up(rows, tile);
    t.width = (uint32_t)(round_up(cols, tile) * g.esize / 16);
    t.cover_rows = (uint32_t)round_up(rows, 32);
    t.cover = (uint32_t)(round_up(cols, 32) * g.esize / 16);
    t.pieces = (uint32_t)(buffers * d.count) * t.rows * t.width;
    plan.fill.groups += (int)((t.pieces + kFillPieces - 1) / kFillPieces);
    t.end = (uint32_t)plan.fill.groups;
  };
  const int p = std::min(g.m, g.n);
  // (the matrices of a buffer and the buffers follow each other without a gap)
  add(d.fresh, 2 * steps, g.s_stride, g.p_pad, p, p);
  add(d.fresh + 2 * kFreshSteps * d.pp_step, steps - 1, g.x_stride, g.cols_pad, g.m, g.n);
}

// `one_by_one`: every product as a launch of its own, on the tiles and with the split of K it has in the ordinary step, and every
// group whose matrices get a workgroup each as a launch of its own: that kernel has no products to take apart, and products in
// its place would sum and round in other places.
void build_plan(const mona_state* st, const mona_hparams& hp, Plan& plan, bool one_by_one) {
  const Layout& L = st->L;
  const size_t ngroups = L.groups.size();
  plan.ns_steps = hp.ns_steps; plan.flags = hp.flags; plan.one_by_one = one_by_one;
  memset(&plan.fill, 0, sizeof plan.fill);
  set_step(st, hp, plan);
  plan.ops.resize(ngroups);
  plan.lanes.resize(L.lanes);
  for (const Group& g : L.groups) {
    GroupDesc d;
    memset(&d, 0, sizeof d);
    d.x = st->arena + g.x_off[0];
    d.x_step = (int64_t)(g.x_off[1] - g.x_off[0]);
    d.pp = st->arena + g.pp_off[0];
    d.pp_step = (int64_t)(g.pp_off[1] - g.pp_off[0]);
    if (st->fresh) d.fresh = st->fresh + g.fresh_off;
    d.members = reinterpret_cast<const int32_t*>(st->arena + g.members_off);
    d.count = (int32_t)g.members.size();
    d.m = g.m; d.n = g.n; d.rows_pad = g.rows_pad; d.cols_pad = g.cols_pad;
    d.tall = g.tall; d.f32 = g.f32;
    const bool w_f32 = std::any_of(g.members.begin(), g.members.end(), [&](int i) { return st->mats[i].w_dtype == MONA_F32; });
    d.w_rows = w_f32 ? ROWS_ANY : g.n % 8 ? ROWS_BF16 : ROWS_WHOLE;
    d.o_scale = update_scale(g, hp);
    plan.desc.push_back(d);
  }
  for (size_t gi = 0; gi < ngroups; ++gi) plan.o_buf.push_back(OpBuilder(L.groups[gi], (int)gi, hp, plan).build());
  auto add = [&](std::vector<Launch>& lane, Launch l) {
    if (!l.op[0]->large) {
      // fp32 products of the shortest K gain nothing from the bf16 instructions (200 x 64 x 1000: 537 us a step without, 576
      // with them throughout)
      for (int i = 0; i < l.n; ++i) l.split = l.split || (plan.desc[l.op[i]->group].f32 && l.op[i]->a.K > kShortK);
      choose_small_tile(plan, l.op, l.n, l.split);
      // the longest chains of K first: their tiles are the last to finish
      std::stable_sort(l.op, l.op + l.n, [](const Op* x, const Op* y) { return x->a.K > y->a.K; });
      long long slots = 0;
      for (int i = 0; i < l.n; ++i) slots += slots_per_die(l.op[i]->a);
      // at most one workgroup per CU: eight wavefronts each, two per SIMD, so that one multiplies while the other reads
      l.wide = slots * kXcds <= device_cu_count();
    }
    lane.push_back(l);
  };
  // Chains, where all of the step fits into them: a chain's workgroups wait on their CUs, so beside launches that fill the
  // chip it takes more than it gives (128 x 768 x 256 and 4 x 128 x 512: 628 us a step with launches, 687 with a chain).
  std::vector<std::vector<int>> chains;
  bool all = L.small_enough && std::all_of(L.units.begin(), L.units.end(), [](const Unit& u) { return u.merged; });
  for (size_t u = 0; all && u < L.units.size(); ++u) {
    auto joined = [&](std::vector<int> chain) {
      chain.insert(chain.end(), L.units[u].groups.begin(), L.units[u].groups.end());
      return chain;
    };
    auto it = std::find_if(chains.begin(), chains.end(),
                           [&](const std::vector<int>& chain) { return chainable(L, plan, joined(chain)) > 0; });
    if (it != chains.end()) *it = joined(*it);
    else chains.push_back(joined({}));
    all = chains.size() <= (size_t)kMaxChains && chainable(L, plan, chains.back()) > 0;
  }
  int tasks = 0;
  for (const auto& groups : chains) tasks += all ? round_up(chainable(L, plan, groups), 4) : 0;
  all = all && tasks <= kMaxChainTasks;
  if (all) {
    plan.fresh = st->fresh != nullptr && hp.ns_steps <= kFreshSteps;
    for (size_t gi = 0; plan.fresh && gi < ngroups; ++gi) {
      for (Op& op : plan.ops[gi]) op.code |= (uint32_t)(op.iter + 1) << OPF_FRESH;
      plan.o_buf[gi] = 1;
    }
    for (size_t i = 0; i < chains.size(); ++i) {
      std::vector<Launch> singles;
      const Launch chain = build_chain(st, plan, chains[i], singles);
      std::vector<Launch>& lane = plan.lanes[i % plan.lanes.size()];
      if (one_by_one) lane.insert(lane.end(), singles.begin(), singles.end());
      else lane.push_back(chain);
    }
    for (size_t gi = 0; plan.fresh && gi < ngroups; ++gi) add_fill(plan, L.groups[gi], gi, hp.ns_steps);
    return;
  }
  for (const Unit& u : L.units) {
    std::vector<Launch>& lane = plan.lanes[u.lane];
    if (u.matrix && hp.ns_steps > 0) {
      const size_t most = one_by_one ? 1 : u.groups.size();
      for (size_t first = 0; first < u.groups.size(); first += most) {
        MatrixBatch b;
        memset(&b, 0, sizeof b);
        b.step = plan.step;
        b.steps = hp.ns_steps;
        b.store_o = (hp.flags & MONA_FLAG_KEEP_O) ? 1 : 0;
        const std::vector<int> groups(u.groups.begin() + first, u.groups.begin() + first + most);
        int matrices = 0;
        for (int gi : groups) {
          matrices += plan.desc[gi].count;
          b.group[b.n] = plan.desc[gi];
          b.end[b.n++] = matrices;
        }
        Launch l;
        l.matrix = (int)plan.matrices.size();
        plan.matrices.push_back(b);
        plan.matrix_groups.push_back(groups);
        lane.push_back(l);
      }
    } else if (u.merged) {
      for (size_t pos = 0;; ++pos) {
        Launch l;
        for (int gi : u.groups)
          if (pos < plan.ops[gi].size()) l.op[l.n++] = &plan.ops[gi][pos];
        if (l.n == 0) break;
        add(lane, l);
      }
    } else {
      for (int gi : u.groups)
        for (Op& op : plan.ops[gi]) {
          Launch l;
          l.n = 1; l.op[0] = &op;
          add(lane, l);
        }
    }
  }
}

// The plan of a step: the last one again, with this step's hyper-parameters, unless the number of iterations, the flags or the
// kind of launches differ (building it takes 10 to 40 us of host time with eight groups, this 1 to 4).
Plan& plan_for(mona_state* st, const mona_hparams& hp) {
  const bool one_by_one = st->profiling > 1;
  Plan* plan = st->plan;
  if (!plan || plan->ns_steps != hp.ns_steps || plan->flags != hp.flags || plan->one_by_one != one_by_one) {
    // (kept once it is whole: a caller may go on after an allocation that failed on the way)
    std::unique_ptr<Plan> fresh(new Plan());
    build_plan(st, hp, *fresh, one_by_one);
    delete plan;
    return *(st->plan = fresh.release());
  }
  const Layout& L = st->L;
  set_step(st, hp, *plan);
  for (size_t gi = 0; gi < L.groups.size(); ++gi) plan->desc[gi].o_scale = update_scale(L.groups[gi], hp);
  for (size_t i = 0; i < plan->chains.size(); ++i) {
    plan->chains[i].step = plan->step;
    for (size_t j = 0; j < plan->chain_groups[i].size(); ++j)
      plan->chains[i].group[j].o_scale = plan->desc[plan->chain_groups[i][j]].o_scale;
  }
  for (size_t i = 0; i < plan->matrices.size(); ++i) {
    plan->matrices[i].step = plan->step;
    for (size_t j = 0; j < plan->matrix_groups[i].size(); ++j)
      plan->matrices[i].group[j].o_scale = plan->desc[plan->matrix_groups[i][j]].o_scale;
  }
  for (auto& lane : plan->lanes)
    for (Launch& l : lane)
      for (int i = 0; i < l.n; ++i) expand_op(plan->step, plan->desc[l.op[i]->group], l.op[i]->code, l.op[i]->a);
  return *plan;
}

// Static description of matrix i: where its state arrays and its working copy live.
void fill_static(const Layout& L, const mona_matrix& q, int i, char* arena, void* g_prev, void* acc, void* mom,
                 MatStatic& ms, void*& o_ptr) {
  const Group& g = L.groups[L.group_of[i]];
  memset(&ms, 0, sizeof ms);
  ms.g_prev = (L.one_buffer || L.caller_slot) ? nullptr : g_prev;
  ms.acc = acc;
  ms.mom = static_cast<float*>(mom);
  ms.x = arena + g.x_off[0] + (size_t)L.rank_in_group[i] * g.x_stride * g.esize;
  ms.m = q.m;
  ms.n = q.n;
  ms.ldx = g.cols_pad;
  ms.w_dtype = q.w_dtype;
  ms.g_dtype = q.g_dtype;
  ms.first_block = L.first_block[i];
  ms.num_blocks = L.num_blocks[i];
  ms.x_f32 = g.f32 ? 1 : 0;
  o_ptr = arena + g.x_off[1] + (size_t)L.rank_in_group[i] * g.x_stride * g.esize;
}

// Theorem 1 assumes |alpha| < 1 / (1 - beta_a).  A step outside that range is taken all the same (the
// algorithm is defined for any alpha); the note is left where mona_last_error() finds it.
void note_unstable_alpha(const mona_hparams* hp) {
  if (hp->flags & MONA_FLAG_MUON_ONLY) return;
  const double bound = 1.0 / (1.0 - (double)hp->beta_a);
  if (std::fabs((double)hp->alpha) >= bound) {
    char buf[256];
    snprintf(buf, sizeof buf, "warning: |alpha| = %g is not below 1 / (1 - beta_a) = %g, the range the convergence "
             "theorem assumes; the step was taken", std::fabs((double)hp->alpha), bound);
    g_err = buf;
  }
}

int check_hparams(const mona_hparams* hp) {
  if (!hp) return fail(MONA_EINVAL, "hparams is NULL");
  if (!(hp->momentum >= 0.0f && hp->momentum < 1.0f)) return fail(MONA_EINVAL, "momentum must lie in [0, 1)");
  if (!(hp->beta_a >= 0.0f && hp->beta_a < 1.0f)) return fail(MONA_EINVAL, "beta_a must lie in [0, 1)");
  if (hp->ns_steps < 0) return fail(MONA_EINVAL, "ns_steps must be >= 0");
  if (!std::isfinite(hp->lr) || !std::isfinite(hp->alpha) || !std::isfinite(hp->weight_decay) ||
      !std::isfinite(hp->ns_a) || !std::isfinite(hp->ns_b) || !std::isfinite(hp->ns_c) ||
      !std::isfinite(hp->gamma_coeff) || !std::isfinite(hp->ns_eps) || hp->ns_eps < 0.0f)
    return fail(MONA_EINVAL, "hyper-parameters must be finite (and ns_eps >= 0)");
  if (hp->flags & ~(MONA_FLAG_FIRST_DIFF_ZERO | MONA_FLAG_KEEP_O | MONA_FLAG_MUON_ONLY)) return fail(MONA_EINVAL, "unknown flag bits");
  return MONA_OK;
}

bool get_event_pair(mona_state* st, hipEvent_t* a, hipEvent_t* b) {
  if (st->pool_used == st->event_pool.size()) {
    hipEvent_t x, y;
    if (hipEventCreate(&x) != hipSuccess) return false;
    if (hipEventCreate(&y) != hipSuccess) { (void)hipEventDestroy(x); return false; }
    st->event_pool.emplace_back(x, y);
  }
  *a = st->event_pool[st->pool_used].first;
  *b = st->event_pool[st->pool_used].second;
  ++st->pool_used;
  return true;
}

}  // namespace

extern "C" {

const char* mona_last_error(void) { return g_err.c_str(); }
const char* mona_version(void) { return "libmona 0.1 (gfx950)"; }

int mona_state_size(const mona_matrix* mats, int32_t count, const mona_options* opts, size_t* bytes_out) {
  if (!bytes_out) return fail(MONA_EINVAL, "bytes_out is NULL");
  int rc = check_mats(mats, count, false);
  if (rc) return rc;
  mona_options o;
  rc = check_opts(opts, &o);
  if (rc) return rc;
  Layout L;
  build_layout(mats, count, o, false, false, L);
  *bytes_out = L.total;
  return MONA_OK;
}

int mona_init_state(const mona_matrix* mats, int32_t count, const mona_options* opts, void* arena,
                    size_t arena_bytes, void* stream, mona_state** out) {
  if (!out) return fail(MONA_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_mats(mats, count, false);
  if (rc) return rc;
  mona_options o;
  rc = check_opts(opts, &o);
  if (rc) return rc;
  if (!arena) return fail(MONA_EINVAL, "arena is NULL");
  if ((uintptr_t)arena % kAlign) return fail(MONA_EINVAL, "arena must be 256-byte aligned");
  mona_state* st = new (std::nothrow) mona_state();
  if (!st) return fail(MONA_ENOMEM, "host allocation failed");
  build_layout(mats, count, o, false, true, st->L);
  const Layout& L = st->L;
  if (arena_bytes < L.total) {
    const size_t need = L.total;
    delete st;
    return fail(MONA_ENOMEM, "arena too small: %zu bytes given, %zu needed", arena_bytes, need);
  }
  st->opt = o;
  st->mats.assign(mats, mats + count);
  st->arena = static_cast<char*>(arena);
  hipStream_t s = static_cast<hipStream_t>(stream);

  auto cleanup = [&](int code) {
    for (int i = 0; i < kRing; ++i) {
      if (st->ring[i]) { (void)hipHostFree(st->ring[i]); (void)hipEventDestroy(st->ring_ev[i]); }
    }
    if (st->ev_valid)
      for (auto& set : st->ev)
        for (auto& e : set)
          if (e) (void)hipEventDestroy(e);
    for (hipStream_t q : st->side) (void)hipStreamDestroy(q);
    for (hipEvent_t e : st->side_done) (void)hipEventDestroy(e);
    if (st->fork_ev) (void)hipEventDestroy(st->fork_ev);
    if (st->late_stream) (void)hipStreamDestroy(st->late_stream);
    if (st->late_fork) (void)hipEventDestroy(st->late_fork);
    if (st->late_done) (void)hipEventDestroy(st->late_done);
    if (st->from_pool) give_back(st->device, st->fresh, L.fresh_bytes);
    delete st;
    (void)hipGetLastError();
    return code;
  };
#define INIT_TRY(expr)                                                                                   \
  do {                                                                                                   \
    hipError_t e__ = (expr);                                                                             \
    if (e__ != hipSuccess) return cleanup(fail(MONA_EHIP, "%s: %s", #expr, hipGetErrorString(e__)));     \
  } while (0)

  INIT_TRY(hipGetDevice(&st->device));
  if (L.gfx950 && L.fresh_bytes > 0) {
    st->fresh = take_from_pool(st->device, L.fresh_bytes);
    st->from_pool = st->fresh != nullptr;
  }
  for (int i = 0; i < kRing && count > kInlineMats; ++i) {   // shorter lists need no staging
    void* p = nullptr;
    INIT_TRY(hipHostMalloc(&p, sizeof(MatDynamic) * (size_t)count, hipHostMallocDefault));
    st->ring[i] = static_cast<MatDynamic*>(p);
    hipError_t e = hipEventCreateWithFlags(&st->ring_ev[i], hipEventDisableTiming);
    if (e != hipSuccess) {
      (void)hipHostFree(p);
      st->ring[i] = nullptr;
      return cleanup(fail(MONA_EHIP, "hipEventCreate: %s", hipGetErrorString(e)));
    }
  }
  for (auto& set : st->ev) for (auto& e : set) e = nullptr;
  st->ev_valid = true;             // from here on cleanup() destroys the events created so far
  for (auto& set : st->ev) for (auto& e : set) INIT_TRY(hipEventCreate(&e));
  {
    INIT_TRY(hipEventCreateWithFlags(&st->fork_ev, hipEventDisableTiming));
    for (int i = 1; i < L.lanes; ++i) {
      hipStream_t side = nullptr;
      INIT_TRY(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
      st->side.push_back(side);
      hipEvent_t done = nullptr;
      INIT_TRY(hipEventCreateWithFlags(&done, hipEventDisableTiming));
      st->side_done.push_back(done);
    }
    if (L.late_group >= 0) {
      // a stream that may use the first quarter of the CUs only (the mask's bits are dealt to the dies in
      // turn, so every die gives up the same number); default priority
      const int cus = device_cu_count();
      const int share = cus / kOverlapCuShare;
      std::vector<uint32_t> mask((cus + 31) / 32, 0u);
      for (int i = 0; i < share; ++i) mask[i / 32] |= 1u << (i % 32);
      INIT_TRY(hipExtStreamCreateWithCUMask(&st->late_stream, (uint32_t)mask.size(), mask.data()));
      INIT_TRY(hipEventCreateWithFlags(&st->late_fork, hipEventDisableTiming));
      INIT_TRY(hipEventCreateWithFlags(&st->late_done, hipEventDisableTiming));
      st->late_cus = share;
    }
  }

  // Alg. 1 initialisation: M_0 = A_0 = G_0 = 0; the padded working copies start (and stay) zero
  INIT_TRY(launch_fill_zero(st->arena + L.state_begin, L.state_bytes + L.work_bytes, s));
  INIT_TRY(launch_fill_zero(st->arena + L.scales_off, align_up(sizeof(MatScale) * count), s));

  std::vector<MatStatic> stat(count);
  std::vector<void*> optr(count);
  for (int i = 0; i < count; ++i) {
    fill_static(L, mats[i], i, st->arena, st->arena + L.gprev_off[i], st->arena + L.acc_off[i],
                st->arena + L.mom_off[i], stat[i], optr[i]);
  }
  INIT_TRY(hipMemcpyAsync(st->arena + L.stat_off, stat.data(), sizeof(MatStatic) * count, hipMemcpyHostToDevice, s));
  INIT_TRY(hipMemcpyAsync(st->arena + L.optr_off, optr.data(), sizeof(void*) * count, hipMemcpyHostToDevice, s));
  INIT_TRY(hipMemcpyAsync(st->arena + L.blocks_off, L.blocks.data(), sizeof(BlockWork) * L.blocks.size(),
                          hipMemcpyHostToDevice, s));
  INIT_TRY(hipMemcpyAsync(st->arena + L.order_off, L.order.data(), sizeof(int32_t) * L.order.size(),
                          hipMemcpyHostToDevice, s));
  for (const Group& g : L.groups) {
    std::vector<int32_t> mem(g.members.begin(), g.members.end());
    INIT_TRY(hipMemcpyAsync(st->arena + g.members_off, mem.data(), sizeof(int32_t) * mem.size(),
                            hipMemcpyHostToDevice, s));
    INIT_TRY(hipStreamSynchronize(s));   // `mem` leaves scope
  }
  INIT_TRY(hipStreamSynchronize(s));     // host vectors above leave scope
#undef INIT_TRY
  *out = st;
  return MONA_OK;
}

}  // extern "C"

namespace {
int step_impl(mona_state* st, const mona_matrix* mats, void* const* slots, int32_t count, const mona_hparams* hp,
              void* stream);
}

extern "C" {

int mona_step(mona_state* st, const mona_matrix* mats, int32_t count, const mona_hparams* hp, void* stream) {
  if (!st) return fail(MONA_EINVAL, "state is NULL");
  if (st->L.caller_slot)
    return fail(MONA_EINVAL, "this state keeps no G_{k-1} (MONA_ACCEL_CALLER_SLOT): use mona_step_streaming");
  return step_impl(st, mats, nullptr, count, hp, stream);
}

int mona_step_streaming(mona_state* st, const mona_matrix* mats, void* const* slots, int32_t count,
                        const mona_hparams* hp, void* stream) {
  if (!st) return fail(MONA_EINVAL, "state is NULL");
  if (!st->L.caller_slot)
    return fail(MONA_EINVAL, "mona_step_streaming needs a state built with MONA_ACCEL_CALLER_SLOT");
  if (!slots) return fail(MONA_EINVAL, "slots is NULL");
  if (count == st->L.count)
    for (int i = 0; i < count; ++i) {
      if (!slots[i]) return fail(MONA_EINVAL, "slot %d is NULL", i);
      if ((uintptr_t)slots[i] & 15) return fail(MONA_EINVAL, "slot %d must be 16-byte aligned", i);
    }
  return step_impl(st, mats, slots, count, hp, stream);
}

}  // extern "C"

namespace {

// Whether one launch does all that stands before the products (launch_begin): the step of a few small matrices.
bool begins_at_once(const mona_state* st, const Plan& plan) {
  return !plan.chains.empty() && st->profiling < 2 && st->L.count <= kBeginMats && st->L.max_blocks <= kBeginBlocks && st->L.late_group < 0;
}

// Enqueues the kernels of one step (Alg. 1 for every matrix) on `s` and the side streams.  The per-matrix
// tables in the arena must already name this step's w / g pointers, or (steps that begin at once) `table` does.
int enqueue_step(mona_state* st, const mona_hparams* hp, hipStream_t s, const BeginTable* table) {
  Layout& L = st->L;
  const int count = L.count;
  const MatStatic* stat = st->at<MatStatic>(L.stat_off);
  const MatDynamic* dyn = st->at<MatDynamic>(L.dyn_off);
  MatScale* scales = st->at<MatScale>(L.scales_off);
  double* partials = st->at<double>(L.partials_off);
  const BlockWork* blocks = st->at<BlockWork>(L.blocks_off);
  const int nblocks = (int)L.blocks.size();

  // A HIP call that fails once kernels of the step are in flight leaves the state arrays half updated:
  // join whatever was forked, mark the state unusable and say so.
  bool forked = false, late_forked = false;
  auto bail = [&](hipError_t e, const char* what) {
    if (late_forked) {
      (void)hipEventRecord(st->late_done, st->late_stream);
      (void)hipStreamWaitEvent(s, st->late_done, 0);
    }
    if (forked)
      for (size_t i = 0; i < st->side.size(); ++i) {
        (void)hipEventRecord(st->side_done[i], st->side[i]);
        (void)hipStreamWaitEvent(s, st->side_done[i], 0);
      }
    st->failed = true;
    (void)hipGetLastError();
    return fail(MONA_EHIP, "%s: %s (the step was abandoned half way: the state arrays are unusable until a checkpoint "
                "is imported with mona_state_import)", what, hipGetErrorString(e));
  };
#define STEP_TRY(expr)                                   \
  do {                                                   \
    hipError_t e__ = (expr);                             \
    if (e__ != hipSuccess) return bail(e__, #expr);      \
  } while (0)

  Plan& plan = plan_for(st, *hp);
  for (size_t gi = 0; gi < L.groups.size(); ++gi) L.groups[gi].o_buf = plan.o_buf[gi];

  const bool prof = st->profiling > 0;
  hipEvent_t* const ev = st->ev[st->prof_steps % kProfSets];
  st->times_ready = false;
  st->records.clear();
  st->pool_used = 0;
  if (prof) STEP_TRY(hipEventRecord(ev[0], s));

  // Alg. 1: difference, acceleration EMA, accelerated gradient, momentum, roll; sum of squares.
  // With a late group its pass goes to the stream that owns a quarter of the CUs and runs beside the
  // products of the other groups (not while every launch is timed on its own, and not under stream
  // capture, where the CU mask of a stream would not survive into the graph anyway).
  const bool muon_only = (hp->flags & MONA_FLAG_MUON_ONLY) != 0;
  const int use_prev = muon_only ? 2 : !((hp->flags & MONA_FLAG_FIRST_DIFF_ZERO) && st->k == 0);
  const int sbf = st->opt.state_dtype == MONA_BF16;
  const int one = L.one_buffer ? 1 : 0;
  const int T = hp->ns_steps;
  // (nor on the null stream: a stream with a CU mask can only be created as a blocking one, and the null
  // stream waits for every blocking stream, which would put the two passes in a row again)
  bool overlap = st->late_stream != nullptr && st->profiling < 2 && T > 0 && s != nullptr;
  if (overlap) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    STEP_TRY(hipStreamIsCapturing(s, &cap));
    overlap = cap == hipStreamCaptureStatusNone;
  }
  const int32_t* order = st->at<int32_t>(L.order_off);
  auto pass = [&](int r0, int r1, int g_bf16, hipStream_t q) {
    return launch_state_update(stat, dyn, blocks + r0, partials + r0, r1 - r0, g_bf16, sbf, one, hp->momentum,
                               hp->beta_a, hp->alpha, use_prev, L.keep, q);
  };
  if (overlap) {
    STEP_TRY(hipEventRecord(st->late_fork, s));
    late_forked = true;
    STEP_TRY(hipStreamWaitEvent(st->late_stream, st->late_fork, 0));
    STEP_TRY(pass(L.range_end[1], L.range_end[2], 0, st->late_stream));
    STEP_TRY(pass(L.range_end[2], L.range_end[3], 1, st->late_stream));
    STEP_TRY(launch_norm_finalize(stat, partials, scales, order + L.num_early, count - L.num_early,
                                  L.max_blocks, hp->ns_eps, nullptr, 0, nullptr, st->late_stream));
    STEP_TRY(hipEventRecord(st->late_done, st->late_stream));
  }
  const bool at_once = begins_at_once(st, plan);
  if (at_once) {
    const BeginTable none = {};
    STEP_TRY(launch_begin(stat, blocks, scales, partials, st->at<MatDynamic>(L.dyn_off), nblocks, sbf, one, hp->momentum, hp->beta_a,
                          hp->alpha, use_prev, hp->ns_eps, st->arena + L.chain_off, plan.chain_bytes, plan.fill, table ? *table : none, s));
  } else {
    STEP_TRY(pass(0, L.range_end[0], 0, s));
    STEP_TRY(pass(L.range_end[0], L.range_end[1], 1, s));
    if (!overlap) {
      STEP_TRY(pass(L.range_end[1], L.range_end[2], 0, s));
      STEP_TRY(pass(L.range_end[2], L.range_end[3], 1, s));
    }
  }
  if (L.one_buffer && !muon_only) st->last_beta_a = hp->beta_a;
  if (!at_once) STEP_TRY(launch_norm_finalize(stat, partials, scales, order, overlap ? L.num_early : count, L.max_blocks, hp->ns_eps,
                                st->arena + L.chain_off, plan.chain_bytes, &plan.fill, s));
  if (prof) STEP_TRY(hipEventRecord(ev[1], s));

  // Newton-Schulz (Eq. newton_schulz), T iterations per shape group
  st->fused_update = T > 0;
  // per-launch timing serialises the launches on the caller's stream so that each interval is one kernel
  bool fork = false;
  for (int lane = 1; lane < L.lanes; ++lane) fork = fork || !plan.lanes[lane].empty();
  fork = fork && st->profiling < 2;
  if (fork) {
    STEP_TRY(hipEventRecord(st->fork_ev, s));
    forked = true;
    for (hipStream_t q : st->side) STEP_TRY(hipStreamWaitEvent(q, st->fork_ev, 0));
  }
  const bool each = st->profiling > 1;
  // one product, or several as one launch
  auto launch = [&](const Launch& l, Op* const* op, int n, int cu_cap, hipStream_t q) {
    if (op[0]->large) return launch_ns_gemm(op[0]->a, cu_cap, q);
    GemmBatch batch;
    batch.n = n;
    for (int i = 0; i < n; ++i) batch.a[i] = op[i]->a;
    if (l.split) return launch_ns_split(batch, q);
    return launch_ns_small(batch, L.groups[op[0]->group].f32, l.wide, q);
  };
  // the lanes are fed in turn, so that no lane waits for the host to have enqueued all of another
  // (without side streams one lane after the other on the caller's)
  std::vector<size_t> at(L.lanes, 0);
  for (bool more = true; more;) {
    more = false;
    for (int lane = 0; lane < L.lanes; ++lane) {
      const std::vector<Launch>& queue = plan.lanes[lane];
      if (at[lane] == queue.size()) continue;
      if (!fork && lane > 0 && at[lane - 1] < plan.lanes[lane - 1].size()) break;
      more = true;
      const Launch& l = queue[at[lane]++];
      hipStream_t gs = lane == 0 || !fork ? s : st->side[lane - 1];
      if (l.matrix >= 0) {
        if (!each) {
          STEP_TRY(launch_ns_matrix(plan.matrices[l.matrix], gs));
          continue;
        }
        LaunchRecord rec;                        // (one group)
        if (!get_event_pair(st, &rec.e0, &rec.e1)) return bail(hipErrorOutOfMemory, "hipEventCreate");
        STEP_TRY(hipEventRecord(rec.e0, gs));
        STEP_TRY(launch_ns_matrix(plan.matrices[l.matrix], gs));
        STEP_TRY(hipEventRecord(rec.e1, gs));
        rec.kind = kWholeMatrices; rec.group = plan.matrix_groups[l.matrix][0]; rec.iter = 0;
        rec.tile = L.groups[rec.group].p_pad * 1000 + 128;
        rec.flops = launch_flops(plan, l);
        st->records.push_back(rec);
        continue;
      }
      if (l.chain >= 0) {
        STEP_TRY(launch_ns_chain(plan.chains[l.chain], l.wgs, gs));
        continue;
      }
      int cu_cap = 0;
      if (overlap && l.op[0]->group == L.late_group) {
        if (late_forked) STEP_TRY(hipStreamWaitEvent(s, st->late_done, 0));
        late_forked = false;
      } else if (overlap) {
        cu_cap = device_cu_count() - st->late_cus;
      }
      if (!each) {
        STEP_TRY(launch(l, l.op, l.n, cu_cap, gs));
        continue;
      }
      // each product timed by itself, on the tiles and with the split of K that it has in the common launch
      for (int i = 0; i < l.n; ++i) {
        const Op& op = *l.op[i];
        LaunchRecord rec;
        if (!get_event_pair(st, &rec.e0, &rec.e1)) return bail(hipErrorOutOfMemory, "hipEventCreate");
        STEP_TRY(hipEventRecord(rec.e0, gs));
        STEP_TRY(launch(l, l.op + i, 1, cu_cap, gs));
        STEP_TRY(hipEventRecord(rec.e1, gs));
        rec.kind = op.kind; rec.group = op.group; rec.iter = op.iter; rec.tile = op.a.tile_m * 1000 + op.a.tile_n;
        rec.flops = gemm_flops(op.a, l.split);
        st->records.push_back(rec);
      }
    }
  }
  if (fork) {
    for (size_t i = 0; i < st->side.size(); ++i) {
      STEP_TRY(hipEventRecord(st->side_done[i], st->side[i]));
      STEP_TRY(hipStreamWaitEvent(s, st->side_done[i], 0));
    }
    forked = false;
  }
  if (prof) STEP_TRY(hipEventRecord(ev[2], s));
  if (T == 0) {
    // O = X_0, then Eq. muon_update
    STEP_TRY(launch_plain_update(stat, dyn, scales, blocks, nblocks, st->at<void*>(L.optr_off), hp->lr,
                                 hp->weight_decay, hp->gamma_coeff, (hp->flags & MONA_FLAG_KEEP_O) ? 1 : 0, s));
  }
  if (prof) {
    STEP_TRY(hipEventRecord(ev[3], s));
    st->times_ready = true;
    st->prof_steps += 1;
  }
#undef STEP_TRY
  st->k += 1;
  return MONA_OK;
}

int step_impl(mona_state* st, const mona_matrix* mats, void* const* slots, int32_t count, const mona_hparams* hp,
              void* stream) {
  g_err.clear();
  if (st->failed)
    return fail(MONA_EHIP, "this state was left half updated by a failed launch in an earlier step: import a "
                "checkpoint with mona_state_import first");
  int rc = check_mats(mats, count, true);
  if (rc) return rc;
  rc = check_hparams(hp);
  if (rc) return rc;
  const Layout& L = st->L;
  if (count != L.count) return fail(MONA_ESHAPE, "count %d differs from %d at init", count, L.count);
  for (int i = 0; i < count; ++i) {
    const mona_matrix& a = mats[i];
    const mona_matrix& b = st->mats[i];
    if (a.m != b.m || a.n != b.n || a.w_dtype != b.w_dtype || a.g_dtype != b.g_dtype)
      return fail(MONA_ESHAPE, "matrix %d: shape or dtype differs from init (%d x %d vs %d x %d)", i, a.m, a.n, b.m,
                  b.n);
  }
  const bool muon_only = (hp->flags & MONA_FLAG_MUON_ONLY) != 0;
  if (L.one_buffer && !muon_only) {
    // C_{k+1} was formed with the previous step's beta_a: the identity A_k = C_k + (1 - beta_a) G_k
    // holds only if this step uses the same value
    if (st->last_beta_a >= 0.0f && st->last_beta_a != hp->beta_a)
      return fail(MONA_EINVAL, "one-buffer form: beta_a changed from %g to %g between steps", (double)st->last_beta_a,
                  (double)hp->beta_a);
  }
  hipStream_t s = static_cast<hipStream_t>(stream);

  // Per-step pointer table.  It is written again only when a pointer has changed since the last table that was enqueued;
  // from the first capture on it is written by every step, captured or not: a recorded write takes effect when the graph
  // is replayed, which this side does not see.  A recorded table travels in kernel arguments, whatever its length, because
  // a copy node would read the pinned ring at the time of the replay.
  if (s != nullptr) {                // (the null stream cannot be captured)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(s, &cap));
    if (cap != hipStreamCaptureStatusNone) st->captured = true;
  }
  BeginTable table;
  table.n = 0;
  bool changed = !st->dyn_valid || st->captured;
  if (!changed)
    for (int i = 0; i < count; ++i)
      if (st->last_dyn[i].w != mats[i].w || st->last_dyn[i].g != mats[i].g ||
          st->last_dyn[i].slot != (slots ? slots[i] : nullptr)) { changed = true; break; }
  if (changed) {
    st->dyn_valid = false;           // until the new table is on its way: a failure below must not leave a stale match
    st->last_dyn.resize(count);
    for (int i = 0; i < count; ++i) {
      st->last_dyn[i].w = mats[i].w;
      st->last_dyn[i].g = mats[i].g;
      st->last_dyn[i].slot = slots ? slots[i] : nullptr;
    }
    if (begins_at_once(st, plan_for(st, *hp))) {
      table.n = count;
      std::copy(st->last_dyn.begin(), st->last_dyn.end(), table.v);
    } else if (count <= kInlineMats || st->captured) {
      for (int first = 0; first < count; first += kInlineMats) {
        const int n = std::min(kInlineMats, count - first);
        DynTable t;
        memset(&t, 0, sizeof t);
        std::copy_n(st->last_dyn.begin() + first, n, t.v);
        HIP_TRY(launch_write_dyn(t, n, st->at<MatDynamic>(L.dyn_off) + first, s));
      }
    } else {
      const int slot = st->ring_next;
      if (st->ring_used[slot]) HIP_TRY(hipEventSynchronize(st->ring_ev[slot]));
      std::copy(st->last_dyn.begin(), st->last_dyn.end(), st->ring[slot]);
      HIP_TRY(hipMemcpyAsync(st->arena + L.dyn_off, st->ring[slot], sizeof(MatDynamic) * count, hipMemcpyHostToDevice,
                             s));
      HIP_TRY(hipEventRecord(st->ring_ev[slot], s));
      st->ring_used[slot] = true;
      st->ring_next = (slot + 1) % kRing;
    }
    st->dyn_valid = table.n == 0;
  }
  rc = enqueue_step(st, hp, s, &table);
  if (rc) return rc;
  st->dyn_valid = true;
  note_unstable_alpha(hp);
  return MONA_OK;
}

}  // namespace

// ---- the entry point that allocates nothing -------------------------------------------------------------
namespace {

// Workspace of mona_step_noalloc: what mona_step keeps in the caller's arena beyond the state arrays (the
// working copies X, the p x p matrices, per-block partial sums, scales and the small tables), here in a
// static device array.  Every GPU the library runs on holds its own copy, at its own address, until the
// process ends.
constexpr size_t kScratchBytes = MONA_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes + kChainBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, looked up once

// Device address of the scratch array on the current device.  In host code the array's name is only a
// handle for this lookup, never an address to hand to a kernel.
int scratch_on_current_device(char** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(MONA_EUNSUPPORTED, "device ordinal %d is beyond %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(MONA_EHIP, "hipGetSymbolAddress returned a null address for the scratch array");
    g_scratch_ptr[dev] = p;
  }
  *out = static_cast<char*>(g_scratch_ptr[dev]);
  return MONA_OK;
}

}  // namespace

extern "C" {

int mona_step_noalloc(const mona_matrix* mat, const mona_options* opts, void* g_prev, void* acc, void* mom,
                      const mona_hparams* hp, int64_t k, void* stream) {
  g_err.clear();
  int rc = check_mats(mat, 1, true);
  if (rc) return rc;
  rc = check_hparams(hp);
  if (rc) return rc;
  mona_options o;
  rc = check_opts(opts, &o);
  if (rc) return rc;
  if (o.accel_form != MONA_ACCEL_TWO_BUFFER)
    return fail(MONA_EUNSUPPORTED, "mona_step_noalloc takes the state arrays of Alg. 1 (MONA_ACCEL_TWO_BUFFER) only");
  if (k < 0) return fail(MONA_EINVAL, "k must be >= 0");
  if (!g_prev || !acc || !mom) return fail(MONA_EINVAL, "g_prev, acc and mom must not be NULL");
  if (((uintptr_t)g_prev & 15) || ((uintptr_t)acc & 15) || ((uintptr_t)mom & 15))
    return fail(MONA_EINVAL, "g_prev, acc and mom must be 16-byte aligned");
  // the same plan a one-matrix mona_init_state would build, laid out over the scratch array
  mona_state st;
  build_layout(mat, 1, o, true, true, st.L);
  const Layout& L = st.L;
  if (L.total > kScratchBytes)
    return fail(MONA_ENOMEM, "a %d x %d matrix needs %zu bytes of workspace; the static scratch of mona_step_noalloc "
                "holds %zu (use mona_step with an arena for larger matrices)", mat->m, mat->n, L.total, kScratchBytes);
  char* base = nullptr;
  rc = scratch_on_current_device(&base);
  if (rc) return rc;
  st.opt = o;
  st.mats.assign(mat, mat + 1);
  st.arena = base;
  if (L.gfx950 && L.fresh_bytes > 0 && align_up(L.total) + L.fresh_bytes <= kScratchBytes) st.fresh = base + align_up(L.total);
  st.k = k;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // The array keeps what the last call left in it: the padding of the working matrices and the scales must
  // start from zero (stores of a kernel, not a memset: the call may be under graph capture).  A matrix without padding
  // needs none of that: every buffer is written whole before it is read (us a step with and without the clearing: 512 x 1408
  // 118.5 and 115.6, 1024 x 1024 156 and 152).
  // (a fresh chain reads the first buffer of X and those that the step itself fills)
  const bool padded = L.groups[0].rows_pad != mat->m || L.groups[0].cols_pad != mat->n;
  const size_t clear = plan_for(&st, *hp).fresh ? L.groups[0].x_off[1] - L.groups[0].x_off[0] : L.work_bytes;
  MatStatic ms;
  void* o_ptr = nullptr;
  fill_static(L, *mat, 0, base, g_prev, acc, mom, ms, o_ptr);
  MatDynamic md;
  md.w = mat->w; md.g = mat->g; md.slot = nullptr;
  HIP_TRY(launch_single_prepare(ms, md, o_ptr, st.at<MatStatic>(L.stat_off), st.at<MatDynamic>(L.dyn_off),
                                st.at<void*>(L.optr_off), st.at<BlockWork>(L.blocks_off), (int)L.blocks.size(),
                                reinterpret_cast<int32_t*>(base + L.groups[0].members_off),
                                st.at<int32_t>(L.order_off), st.at<MatScale>(L.scales_off), base + L.work_begin,
                                padded ? clear : 0, s));
  rc = enqueue_step(&st, hp, s, nullptr);
  if (rc) return rc;
  note_unstable_alpha(hp);
  return MONA_OK;
}

}  // extern "C"

extern "C" {

int mona_free_state(mona_state* st) {
  if (!st) return MONA_OK;
  for (int i = 0; i < kRing; ++i) {
    if (st->ring_used[i]) (void)hipEventSynchronize(st->ring_ev[i]);
    if (st->ring[i]) { (void)hipHostFree(st->ring[i]); (void)hipEventDestroy(st->ring_ev[i]); }
  }
  if (st->ev_valid)
    for (auto& set : st->ev)
      for (auto& e : set)
        if (e) (void)hipEventDestroy(e);
  for (auto& pr : st->event_pool) { (void)hipEventDestroy(pr.first); (void)hipEventDestroy(pr.second); }
  for (hipStream_t q : st->side) { (void)hipStreamSynchronize(q); (void)hipStreamDestroy(q); }
  for (hipEvent_t e : st->side_done) (void)hipEventDestroy(e);
  if (st->fork_ev) (void)hipEventDestroy(st->fork_ev);
  if (st->late_stream) { (void)hipStreamSynchronize(st->late_stream); (void)hipStreamDestroy(st->late_stream); }
  if (st->late_fork) (void)hipEventDestroy(st->late_fork);
  if (st->late_done) (void)hipEventDestroy(st->late_done);
  if (st->from_pool && !st->captured) give_back(st->device, st->fresh, st->L.fresh_bytes);
  delete st;
  return MONA_OK;
}

int mona_state_view(mona_state* st, int32_t i, int32_t kind, mona_view* out) {
  if (!st || !out) return fail(MONA_EINVAL, "state or out is NULL");
  const Layout& L = st->L;
  if (i < 0 || i >= L.count) return fail(MONA_EINVAL, "matrix index %d out of range [0, %d)", i, L.count);
  const mona_matrix& q = st->mats[i];
  const Group& g = L.groups[L.group_of[i]];
  out->rows = q.m; out->cols = q.n; out->ld = q.n;
  switch (kind) {
    case MONA_VIEW_G_PREV:
      if (L.one_buffer) return fail(MONA_EUNSUPPORTED, "the one-buffer form stores no G_{k-1}");
      if (L.caller_slot) return fail(MONA_EUNSUPPORTED, "G_{k-1} is kept by the caller (MONA_ACCEL_CALLER_SLOT)");
      out->ptr = st->arena + L.gprev_off[i]; out->dtype = st->opt.state_dtype; break;
    case MONA_VIEW_A:
      if (L.one_buffer) return fail(MONA_EUNSUPPORTED, "the one-buffer form stores C, not A (use MONA_VIEW_C)");
      out->ptr = st->arena + L.acc_off[i]; out->dtype = st->opt.state_dtype; break;
    case MONA_VIEW_C:
      if (!L.one_buffer) return fail(MONA_EUNSUPPORTED, "MONA_VIEW_C exists only in the one-buffer form");
      out->ptr = st->arena + L.acc_off[i]; out->dtype = st->opt.state_dtype; break;
    case MONA_VIEW_M: out->ptr = st->arena + L.mom_off[i]; out->dtype = MONA_F32; break;
    case MONA_VIEW_NORM:
      out->ptr = reinterpret_cast<char*>(st->at<MatScale>(L.scales_off) + i) + offsetof(MatScale, norm);
      out->rows = out->cols = out->ld = 1; out->dtype = MONA_F32;
      break;
    case MONA_VIEW_O: {
      // every chunk of iterations reads one ping-pong buffer and writes the other (a fresh chain writes buffer 1); with T = 0 the
      // update kernel writes buffer 1
      out->ptr = st->arena + g.x_off[g.o_buf] + (size_t)L.rank_in_group[i] * g.x_stride * g.esize;
      out->ld = g.cols_pad;
      out->dtype = g.f32 ? MONA_F32 : MONA_BF16;
      break;
    }
    default: return fail(MONA_EINVAL, "unknown view kind %d", kind);
  }
  return MONA_OK;
}

int mona_state_export_size(mona_state* st, size_t* bytes_out) {
  if (!st || !bytes_out) return fail(MONA_EINVAL, "state or bytes_out is NULL");
  *bytes_out = st->L.state_bytes;
  return MONA_OK;
}

int mona_state_export(mona_state* st, void* dst, size_t dst_bytes, void* stream) {
  if (!st || !dst) return fail(MONA_EINVAL, "state or dst is NULL");
  if (dst_bytes < st->L.state_bytes) return fail(MONA_ENOMEM, "dst too small: %zu < %zu", dst_bytes, st->L.state_bytes);
  HIP_TRY(hipMemcpyAsync(dst, st->arena + st->L.state_begin, st->L.state_bytes, hipMemcpyDeviceToDevice,
                         static_cast<hipStream_t>(stream)));
  return MONA_OK;
}

int mona_state_import(mona_state* st, const void* src, size_t src_bytes, int64_t step_count, void* stream) {
  if (!st || !src) return fail(MONA_EINVAL, "state or src is NULL");
  if (src_bytes != st->L.state_bytes)
    return fail(MONA_ESHAPE, "checkpoint holds %zu bytes, this state needs %zu", src_bytes, st->L.state_bytes);
  if (step_count < 0) return fail(MONA_EINVAL, "step_count must be >= 0");
  HIP_TRY(hipMemcpyAsync(st->arena + st->L.state_begin, src, st->L.state_bytes, hipMemcpyDeviceToDevice,
                         static_cast<hipStream_t>(stream)));
  // The products rely on the padding of the working matrices being zero.  The steps themselves keep it so;
  // clearing it here as well makes an imported state independent of whatever the arena went through before.
  HIP_TRY(launch_fill_zero(st->arena + st->L.work_begin, st->L.work_bytes, static_cast<hipStream_t>(stream)));
  st->failed = false;
  st->k = step_count;
  st->last_beta_a = -1.0f;   // the checkpoint does not say which beta_a formed C
  return MONA_OK;
}

int mona_state_step_count(mona_state* st, int64_t* k_out) {
  if (!st || !k_out) return fail(MONA_EINVAL, "state or k_out is NULL");
  *k_out = st->k;
  return MONA_OK;
}

int mona_state_status(mona_state* st, uint32_t* host_out, int32_t count, void* stream) {
  if (!st || !host_out) return fail(MONA_EINVAL, "state or host_out is NULL");
  if (count != st->L.count) return fail(MONA_ESHAPE, "count %d differs from %d at init", count, st->L.count);
  std::vector<MatScale> tmp(count);
  hipStream_t s = static_cast<hipStream_t>(stream);
  HIP_TRY(hipMemcpyAsync(tmp.data(), st->arena + st->L.scales_off, sizeof(MatScale) * count, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  for (int i = 0; i < count; ++i) host_out[i] = tmp[i].status;
  return MONA_OK;
}

// Not part of the ABI: how often the chains of a state's steps poll the roll before they close it, and in one wait, for tests of
// chains that begin without some of their workgroups (with 0 most do) and of waits that do not end (with 0 none does).
int mona_internal_chain_polls(mona_state* st, int32_t roll, int32_t wait) {
  if (!st || roll < 0 || wait < 0) return fail(MONA_EINVAL, "state is NULL or a figure is negative");
  st->chain_roll_polls = roll;
  st->chain_patience = wait;
  delete st->plan;                 // (it holds the figures)
  st->plan = nullptr;
  return MONA_OK;
}
// Not part of the ABI: whether the chains of a state's last step had a buffer for every product (1), ran with flags (0), or it had none (-1).
int mona_internal_chain_kind(mona_state* st) { return !st || !st->plan || st->plan->chains.empty() ? -1 : st->plan->fresh ? 1 : 0; }

int mona_set_profiling(mona_state* st, int32_t on) {
  if (!st) return fail(MONA_EINVAL, "state is NULL");
  if (on < 0 || on > 2) return fail(MONA_EINVAL, "profiling level must be 0, 1 or 2");
  st->profiling = on;
  st->times_ready = false;
  st->prof_steps = 0;
  return MONA_OK;
}

int mona_last_step_times(mona_state* st, float* ms_out) {
  if (!st || !ms_out) return fail(MONA_EINVAL, "state or ms_out is NULL");
  if (!st->times_ready) return fail(MONA_EINVAL, "no profiled step yet (call mona_set_profiling(st, 1) first)");
  hipEvent_t* const ev = st->ev[(st->prof_steps - 1) % kProfSets];
  HIP_TRY(hipEventSynchronize(ev[3]));
  HIP_TRY(hipEventElapsedTime(&ms_out[0], ev[0], ev[1]));
  HIP_TRY(hipEventElapsedTime(&ms_out[1], ev[1], ev[2]));
  HIP_TRY(hipEventElapsedTime(&ms_out[2], ev[2], ev[3]));
  HIP_TRY(hipEventElapsedTime(&ms_out[3], ev[0], ev[3]));
  return MONA_OK;
}

int mona_mean_step_times(mona_state* st, float* ms_out, int32_t* steps_out) {
  if (!st || !ms_out || !steps_out) return fail(MONA_EINVAL, "state, ms_out or steps_out is NULL");
  if (!st->times_ready) return fail(MONA_EINVAL, "no profiled step yet (call mona_set_profiling(st, 1) first)");
  const int n = (int)std::min<int64_t>(st->prof_steps, kProfSets);
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b = 0; b < n; ++b) {
    hipEvent_t* const ev = st->ev[(st->prof_steps - 1 - b) % kProfSets];
    HIP_TRY(hipEventSynchronize(ev[3]));
    const int from[4] = {0, 1, 2, 0}, to[4] = {1, 2, 3, 3};
    for (int i = 0; i < 4; ++i) {
      float ms = 0.0f;
      HIP_TRY(hipEventElapsedTime(&ms, ev[from[i]], ev[to[i]]));
      sum[i] += ms;
    }
  }
  for (int i = 0; i < 4; ++i) ms_out[i] = (float)(sum[i] / n);
  *steps_out = n;
  return MONA_OK;
}

int mona_last_step_launches(mona_state* st, mona_launch_time* out, int32_t max_records, int32_t* n_out) {
  if (!st || !n_out) return fail(MONA_EINVAL, "state or n_out is NULL");
  if (st->profiling < 2 || !st->times_ready) return fail(MONA_EINVAL, "no step profiled at level 2 yet");
  HIP_TRY(hipEventSynchronize(st->ev[(st->prof_steps - 1) % kProfSets][3]));
  const int n = (int)st->records.size();
  *n_out = n;
  if (!out) return MONA_OK;
  for (int i = 0; i < n && i < max_records; ++i) {
    const LaunchRecord& r = st->records[i];
    out[i].kind = r.kind; out[i].group = r.group; out[i].iter = r.iter; out[i].tile = r.tile;
    out[i].flops = r.flops;
    const Group& g = st->L.groups[r.group];
    out[i].m = g.m; out[i].n = g.n; out[i].count = (int)g.members.size();
    HIP_TRY(hipEventElapsedTime(&out[i].ms, r.e0, r.e1));
  }
  return MONA_OK;
}

int mona_plan_info(mona_state* st, int32_t ns_steps, int64_t* launches_out, double* ns_flops_executed_out,
                   double* elementwise_bytes_out) {
  if (!st) return fail(MONA_EINVAL, "state is NULL");
  if (ns_steps < 0) return fail(MONA_EINVAL, "ns_steps must be >= 0");
  const Layout& L = st->L;
  mona_hparams hp;
  memset(&hp, 0, sizeof hp);
  hp.ns_steps = ns_steps;
  Plan plan;
  build_plan(st, hp, plan, false);
  double flops = 0.0;
  int64_t launches = 0;
  for (const auto& lane : plan.lanes) {
    launches += (int64_t)lane.size();
    for (const Launch& l : lane) flops += launch_flops(plan, l);
  }
  const double bytes = pass_bytes(L, st->mats.data());
  if (launches_out) *launches_out = launches;
  if (ns_flops_executed_out) *ns_flops_executed_out = flops;
  if (elementwise_bytes_out) *elementwise_bytes_out = bytes;
  return MONA_OK;
}

}  // extern "C"
