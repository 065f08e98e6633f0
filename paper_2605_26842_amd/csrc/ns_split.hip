// fp32-class Newton-Schulz products on the bf16 matrix instructions.
//
// What bounds the fp32 matrix instructions is their rate, a sixteenth of the bf16 ones'.  An fp32 value is the sum of three
// bf16 values to the last bit but two or so, x = h + m + l (each the rounding to nearest of what the ones before leave; 8 + 8 + 8
// significant bits and two signs), and the product of two of them the sum of
//     h h' + (h m' + m h') + (h l' + m m' + l h') + terms below 2^-26 |x x'|,
// six bf16 products with fp32 accumulation in place of one, at 16 times the rate.  The largest has accumulators of its own, so
// that it is rounded once for sixteen values of k (the fp32 instruction: eight times); the five small ones share a second set.
//
// Memory and LDS.  X, S and the other operands stay fp32 in memory.  A stage of K (32 values at 128 x 128 tiles, 64 at 64 x 64)
// goes through registers: every thread loads eight consecutive floats of each operand two stages ahead, splits them (eleven
// vector instructions for a pair) and writes three planes of bf16 in the layouts of the bf16 kernels, row-major or K-major, so
// that a value is split once for a whole tile and the fragment reads are those of bf16 products.  Two stages of 48 KB.
//
// Eight wavefronts, 64 x 64 (T = 128: 2 x 2 of them, twice over K) or 64 x 32 (T = 64: two, four times over K) each; 24 or 12
// products a stage and wavefront against 88 instructions of splitting.
//
// Measured against the fp32 instructions, us per step: a block of hidden size 1024 (4 x 1024 x 1024, 1024 x 4096 both ways)
// 2288 -> 1672, 2048 x 2048 1910 -> 1239, 64 x 1024 x 2048 21270 -> 15180 (there 1080 TFLOP/s of bf16 products, the rate
// the power limit leaves the large-tile kernel too), 42 x 256 x 207 303 -> 285; the relative error of the update against 64 bits
// on these shapes 0.9e-6 to 1.7e-6 -> 0.6e-6 to 1.0e-6.  Letting one wavefront of a SIMD split while the other multiplies, or
// weaving both into one stream by scheduling groups, is 16 and 5 % slower; a single set of accumulators is as fast.
#include "ns_small_tile.h"

namespace mona {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kSplitThreads = 512;

// Two floats -> two bf16 (to nearest even) as the hardware packs them; what is left of the floats stays in a and b.
__device__ __forceinline__ uint32_t split_pair(float& a, float& b) {
  uint32_t u;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(u) : "v"(a), "v"(b));   // (written as a conversion it is made two and three times)
  a -= __builtin_bit_cast(float, u << 16);
  b -= __builtin_bit_cast(float, u & 0xffff0000u);
  return u;
}

template <int T>
struct SplitGeo {
  static constexpr int KST = T == 128 ? 32 : 64;    // k values of a stage
  static constexpr int PLANE = T * KST * 2;         // bytes of one plane of one operand
  static constexpr int OPERAND = 3 * PLANE, STAGE = 2 * OPERAND;
  static constexpr int NBN = T == 128 ? 2 : 1;      // 32 x 32 blocks of a wavefront along the columns (two along the rows)
  static constexpr int SHARES = T == 128 ? 1 : 4;   // tiles staged by the epilogue
  static constexpr int STAGING = SHARES * T * staged_ld(T) * 4;
  static constexpr int LDS = 2 * STAGE > STAGING ? 2 * STAGE : STAGING;
  static_assert(T == 64 || T == 128, "64 or 128");
};

// where the 16-byte chunk c of row (or k-row) r stands in a plane
template <int T, bool TRANS>
__device__ __forceinline__ uint32_t plane_at(int r, int c) {
  if constexpr (!TRANS) return T == 128 ? r * 64 + ((c ^ ((r >> 2) & 3)) << 4) : r * 128 + ((c ^ ((r >> 1) & 7)) << 4);
  else return T == 128 ? r * 256 + ((c ^ ((r & 3) << 2)) << 4) : r * 128 + ((c ^ (((r >> 1) & 1) << 2)) << 4);
}

// one fragment: row-major one 16-byte read, K-major two transposing ones (k 0..3 and 4..7 of the lane's row)
template <bool TRANS, int PITCH4>
__device__ __forceinline__ bf16x8 read_fragment(const char* lds, uint32_t at) {
  if constexpr (!TRANS) return *reinterpret_cast<const bf16x8*>(lds + at);
  else {
    typedef MONA_AS3 s16x4* lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lds + at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lds + at + PITCH4));
    return frag(__builtin_bit_cast(u32x2, lo), __builtin_bit_cast(u32x2, hi));
  }
}

// C tile (ti, tj) of matrix t.mat.  lds: SplitGeo<T>::LDS bytes, 256-byte aligned.
template <int T, bool TP, bool TQ>
__device__ __forceinline__ void split_tile(const GemmArgs& a, const TileId& t, const TileMatrix& v, char* lds) {
  typedef SplitGeo<T> G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = T == 128 ? wave >> 2 : wave >> 1;                   // sixteen values of k of the stage
  const int wm = T == 128 ? (wave >> 1) & 1 : 0, wn = wave & 1;      // 64 rows, 64 or 32 columns of the tile
  const int m0 = t.ti * T, n0 = t.tj * T;

  // ---- a thread's eight values of each operand: chunk c8 of row (K-major: k-row) r8 ----
  constexpr int CPP = G::KST / 8, CPK = T / 8;       // chunks of eight to a row, to a k-row
  auto source = [&](const void* base, int64_t stride, int ld, int r0, bool trans) -> const float* {
    const float* src = static_cast<const float*>(base) + (size_t)t.mat * stride;
    return trans ? src + (size_t)(tid / CPK) * ld + r0 + (tid % CPK) * 8 : src + (size_t)(r0 + tid / CPP) * ld + (tid % CPP) * 8;
  };
  const float* const gp = source(a.P, a.strideP, a.ldp, m0, TP);
  const float* const gq = source(a.Q, a.strideQ, a.ldq, n0, TQ);
  const size_t incp = TP ? (size_t)G::KST * a.ldp : (size_t)G::KST, incq = TQ ? (size_t)G::KST * a.ldq : (size_t)G::KST;
  const uint32_t wp = plane_at<T, TP>(tid / (TP ? CPK : CPP), tid % (TP ? CPK : CPP));
  const uint32_t wq = G::OPERAND + plane_at<T, TQ>(tid / (TQ ? CPK : CPP), tid % (TQ ? CPK : CPP));
  f32x4 in[2][4];                                    // [stage parity][P low, P high, Q low, Q high]
  auto load = [&](auto s, int kt) {
    const f32x4* const p = reinterpret_cast<const f32x4*>(gp + kt * incp);
    const f32x4* const q = reinterpret_cast<const f32x4*>(gq + kt * incq);
    in[s][0] = p[0]; in[s][1] = p[1]; in[s][2] = q[0]; in[s][3] = q[1];
  };
  auto split = [&](auto s) {
    static_for<2>([&](auto o) {
      float x[8];
      static_for<8>([&](auto e) { x[e] = in[s][2 * o + e / 4][e % 4]; });
      static_for<3>([&](auto plane) {
        u32x4 w;
        static_for<4>([&](auto e) { w[(int)e] = split_pair(x[2 * e], x[2 * e + 1]); });
        *reinterpret_cast<u32x4*>(lds + s * G::STAGE + plane * G::PLANE + (o == 0 ? wp : wq)) = w;
      });
    });
  };

  // ---- fragment addresses, per lane, of stage 0, plane 0 ----
  const int frow = lane & 31, half = lane >> 5;
  const int tx = (lane & 15) >> 2, nl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  auto where = [&](auto trans, int first) -> uint32_t {      // first: first row or column of the block in the tile
    if constexpr (!trans) return plane_at<T, false>(first + frow, 2 * kq + half);
    else return plane_at<T, true>(kq * 16 + 8 * half + tx, (first + nl) >> 3) + (nl & 7) * 2;
  };
  constexpr int PITCH4 = 4 * T * 2;                  // bytes between k-row k and k-row k + 4
  uint32_t fa[2], fb[G::NBN];
  static_for<2>([&](auto i) { fa[i] = where(std::integral_constant<bool, TP>{}, wm * 64 + i * 32); });
  static_for<G::NBN>([&](auto j) { fb[j] = G::OPERAND + where(std::integral_constant<bool, TQ>{}, wn * 32 * G::NBN + j * 32); });

  f32x16 acc[2][G::NBN], low[2][G::NBN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < G::NBN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.0f;

  // (the operand roles are swapped, so a block is accumulated transposed: a lane holds one output row and, per group of four
  // registers, four consecutive columns)
  auto multiply = [&](auto s) {
    bf16x8 pa[3][2], qb[3][G::NBN];
    static_for<3>([&](auto plane) {
      static_for<2>([&](auto i) { pa[plane][i] = read_fragment<TP, PITCH4>(lds, s * G::STAGE + plane * G::PLANE + fa[i]); });
      static_for<G::NBN>([&](auto j) { qb[plane][j] = read_fragment<TQ, PITCH4>(lds, s * G::STAGE + plane * G::PLANE + fb[j]); });
    });
    auto product = [&](f32x16 (&to)[2][G::NBN], int x, int y) {
      static_for<2>([&](auto i) {
        static_for<G::NBN>([&](auto j) {
          to[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qb[y][j], pa[x][i], to[i][j], 0, 0, 0);
        });
      });
    };
    product(acc, 0, 0);
    product(low, 0, 1);
    product(low, 1, 0);
    product(low, 1, 1);
    product(low, 0, 2);
    product(low, 2, 0);
  };
  // stage kt + 1 is complete for every wavefront, and stage kt free (a fenced barrier would drain the loads in flight)
  auto meet = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  const int KT = a.K / G::KST;                       // K is a multiple of 128: a whole, even number of stages
  load(IC<0>{}, 0);
  load(IC<1>{}, 1);
  split(IC<0>{});
  if (KT > 2) load(IC<0>{}, 2);
  meet();
  auto stage = [&](auto s, int kt) {
    multiply(s);
    if (kt + 1 < KT) {
      split(IC<1 - s>{});
      if (kt + 3 < KT) load(IC<1 - s>{}, kt + 3);
    }
    meet();
  };
  for (int kt = 0; kt < KT; kt += 2) {
    stage(IC<0>{}, kt);
    stage(IC<1>{}, kt + 1);
  }

  // ---- epilogue ----
  f32x4 ev[TileChunks<float, T, kSplitThreads>::PER_LANE];
  load_e<float, T, kSplitThreads, false>(a, t, tid, ev);
  float* const sum = reinterpret_cast<float*>(lds);
  constexpr int LDW = staged_ld(T);
  float* const mine = sum + (T == 128 ? 0 : kq * T * LDW) + (wm * 64 + frow) * LDW + wn * 32 * G::NBN + 4 * half;
  auto each = [&](auto&& f) {
    static_for<2>([&](auto i) {
      static_for<G::NBN>([&](auto j) {
        static_for<4>([&](auto g) {
          f32x4 x;
          static_for<4>([&](auto e) { x[(int)e] = acc[i][j][g * 4 + e] + low[i][j][g * 4 + e]; });
          f(*reinterpret_cast<f32x4*>(mine + i * 32 * LDW + j * 32 + 8 * g), x);
        });
      });
    });
  };
  if (T == 64 || kq == 0) each([](f32x4& to, f32x4 x) { to = x; });
  __syncthreads();
  if constexpr (T == 128) {                          // the second half of K is added where the first one stands
    if (kq == 1) each([](f32x4& to, f32x4 x) { to += x; });
    __syncthreads();
  }
  finish_tile<float, T, G::SHARES, kSplitThreads, false>(a, t, v, tid, ev, sum);
}

// One workgroup per tile, dealt to the dies as for ns_small_kernel.
__global__ __launch_bounds__(kSplitThreads) void ns_small_kernel_split(const GemmBatch b) {
  constexpr int LDS = SplitGeo<64>::LDS > SplitGeo<128>::LDS ? SplitGeo<64>::LDS : SplitGeo<128>::LDS;
  __shared__ __attribute__((aligned(256))) char lds[LDS];
  const int die = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  int g = 0;
  while (g + 1 < b.n && slot >= b.slot_end[g]) ++g;
  const int first = g > 0 ? b.slot_end[g - 1] : 0;
  const GemmArgs& a = b.a[g];
  const int per_die = b.slot_end[g] - first, local = slot - first;
  const TileId t = decode_logical(a, die * per_die + local, local < per_die);
  if (!t.valid) return;
  const TileMatrix v = look_up(a, t);
  auto run = [&](auto tile) {
    if (!a.trans_p && !a.trans_q) split_tile<tile, false, false>(a, t, v, lds);
    else if (!a.trans_p) split_tile<tile, false, true>(a, t, v, lds);
    else split_tile<tile, true, true>(a, t, v, lds);
  };
  if (a.tile_m == 64) run(IC<64>{}); else run(IC<128>{});
}

}  // namespace

hipError_t launch_ns_split(GemmBatch& b, hipStream_t s) {
  long long slots = 0;
  for (int g = 0; g < b.n; ++g) {
    const GemmArgs& a = b.a[g];
    if ((a.tile_m != 64 && a.tile_m != 128) || a.tile_n != a.tile_m || (a.trans_p && !a.trans_q) || a.K % 128) return hipErrorInvalidValue;
    slots += slots_per_die(a);
    if (slots * kXcds > 0x7fffff00LL) return hipErrorInvalidValue;
    b.slot_end[g] = (int32_t)slots;
  }
  if (b.n < 1 || slots == 0) return hipSuccess;
  hipLaunchKernelGGL(ns_small_kernel_split, dim3((unsigned)(slots * kXcds)), dim3(kSplitThreads), 0, s, b);
  return hipGetLastError();
}

}  // namespace mona
