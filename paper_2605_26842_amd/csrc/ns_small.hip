// Newton-Schulz products for launches that do not fill the chip with 256 x 256 tiles, and all fp32-class products.
//
// What bounds these launches is latency: a handful of tiles, each a short chain of "fetch operands, multiply,
// store", repeated for 15 or 18 dependent launches per step.  Three things are done about it:
//   * all shape groups whose products are small share ONE launch per position in their chains of products
//     (GemmBatch: up to kMaxMerged groups per launch, each with its own shapes, operand layouts and scales), so a
//     step of many small groups costs the launches of one group;
//   * operands go from global memory straight into a ring of LDS stages, several stages ahead, so that a short K
//     is in flight at once and a long one never waits for a single round trip per stage;
//   * a launch of few tiles uses 64 x 64 tiles whose wavefronts split K between them (each its own slabs of LDS, no
//     workgroup barrier before the sum), a launch of more tiles 128 x 128 (the host decides, product by product).
// Measured, us per step, one chain of launches per group on a register-staged 128 x 128 kernel -> here: one 256 x 512
// matrix 170 -> 99, 512 x 1408 269 -> 137, nine ragged matrices 980 -> 180 to 194, a block of hidden size 1000 664 -> 509,
// one of hidden size 1024 with fp32 products 4583 -> 2283 (73 TFLOP/s; launches that fill the chip many times over 130 of 154).
// A launch costs 5 us (64 x 64) to 9 - 11 us (128 x 128) beside its K loop, and 1024 of K 4.7 and 9.4 us for a tile on a CU of
// its own, 8.6 and 19.4 us for two.
//
// One workgroup per tile, every wavefront 64 x 64 (2 x 2 blocks of 32 x 32, 64 accumulators); four wavefronts and 64 KB
// of ring, two workgroups per CU, or (launches of at most one workgroup per CU) eight and 128 KB:
//   T = 128: wavefronts 2 x 2 over the tile, one or two slabs of K per stage;
//   T =  64: wavefronts side by side in K, as many slabs per stage.
// A slab holds 64 bytes of K per operand row (32 bf16 or 16 fp32 values):
//   row-major operand: T rows x 4 chunks of 16 bytes, chunk c of row r at c ^ ((r >> 2) & 3); a fragment read is
//     one ds_read_b128 per lane, 16 consecutive rows fall on 16 different bank groups;
//   K-major operand: the slab's k-rows of T values; read with ds_read_b64_tr_b16 (bf16) or ds_read_b32 (fp32),
//     chunks XORed so that the rows one read touches lie on different banks.
#include "ns_tile.h"

namespace mona {

namespace {

template <typename E> struct Chunk;           // 16 bytes of E
template <> struct Chunk<bf16_t> { static constexpr int N = 8; typedef bf16x8 vec; };
template <> struct Chunk<float> { static constexpr int N = 4; typedef f32x4 vec; };

// ---- fragment reads ------------------------------------------------------------------------
// bf16, one stage (two k16 halves): a[half][block], b[half][block].  read_..() issues the reads of both halves in order
// and waits for the first half's; rest_..() waits for the second's, which travel while the first half is multiplied and
// whose registers nothing touches in between.
__device__ __forceinline__ void read_rr(u32x4 (&a)[2][2], u32x4 (&b)[2][2], uint32_t ra0, uint32_t ra1, uint32_t rb0,
                                        uint32_t rb1) {
  asm volatile(
      "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:2048\n\t"
      "ds_read_b128 %4, %10\n\tds_read_b128 %5, %10 offset:2048\n\t"
      "ds_read_b128 %2, %9\n\tds_read_b128 %3, %9 offset:2048\n\t"
      "ds_read_b128 %6, %11\n\tds_read_b128 %7, %11 offset:2048\n\t"
      "s_waitcnt lgkmcnt(4)"
      : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[1][0]), "=&v"(a[1][1]), "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[1][0]),
        "=&v"(b[1][1])
      : "v"(ra0), "v"(ra1), "v"(rb0), "v"(rb1)
      : "memory");
}
__device__ __forceinline__ void rest_rr(u32x4 (&a)[2][2], u32x4 (&b)[2][2]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[1][0]), "+v"(a[1][1]), "+v"(b[1][0]), "+v"(b[1][1]) : : "memory");
}
template <int T>
__device__ __forceinline__ void read_rt(u32x4 (&a)[2][2], u32x2 (&bl)[2][2], u32x2 (&bh)[2][2], uint32_t ra0, uint32_t ra1,
                                        uint32_t tb0, uint32_t tb1) {
  asm volatile(
      "ds_read_b128 %0, %12\n\tds_read_b128 %1, %12 offset:2048\n\t"
      "ds_read_b64_tr_b16 %4, %14\n\tds_read_b64_tr_b16 %8, %14 offset:%16\n\t"
      "ds_read_b64_tr_b16 %5, %15\n\tds_read_b64_tr_b16 %9, %15 offset:%16\n\t"
      "ds_read_b128 %2, %13\n\tds_read_b128 %3, %13 offset:2048\n\t"
      "ds_read_b64_tr_b16 %6, %14 offset:%17\n\tds_read_b64_tr_b16 %10, %14 offset:%18\n\t"
      "ds_read_b64_tr_b16 %7, %15 offset:%17\n\tds_read_b64_tr_b16 %11, %15 offset:%18\n\t"
      "s_waitcnt lgkmcnt(6)"
      : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[1][0]), "=&v"(a[1][1]), "=&v"(bl[0][0]), "=&v"(bl[0][1]),
        "=&v"(bl[1][0]), "=&v"(bl[1][1]), "=&v"(bh[0][0]), "=&v"(bh[0][1]), "=&v"(bh[1][0]), "=&v"(bh[1][1])
      : "v"(ra0), "v"(ra1), "v"(tb0), "v"(tb1), "n"(8 * T), "n"(32 * T), "n"(40 * T)
      : "memory");
}
__device__ __forceinline__ void rest_rt(u32x4 (&a)[2][2], u32x2 (&bl)[2][2], u32x2 (&bh)[2][2]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(a[1][0]), "+v"(a[1][1]), "+v"(bl[1][0]), "+v"(bl[1][1]), "+v"(bh[1][0]), "+v"(bh[1][1])
               :
               : "memory");
}
template <int T>
__device__ __forceinline__ void read_tt(u32x2 (&al)[2][2], u32x2 (&ah)[2][2], u32x2 (&bl)[2][2], u32x2 (&bh)[2][2],
                                        uint32_t ta0, uint32_t ta1, uint32_t tb0, uint32_t tb1) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %4, %16 offset:%20\n\t"
      "ds_read_b64_tr_b16 %1, %17\n\tds_read_b64_tr_b16 %5, %17 offset:%20\n\t"
      "ds_read_b64_tr_b16 %8, %18\n\tds_read_b64_tr_b16 %12, %18 offset:%20\n\t"
      "ds_read_b64_tr_b16 %9, %19\n\tds_read_b64_tr_b16 %13, %19 offset:%20\n\t"
      "ds_read_b64_tr_b16 %2, %16 offset:%21\n\tds_read_b64_tr_b16 %6, %16 offset:%22\n\t"
      "ds_read_b64_tr_b16 %3, %17 offset:%21\n\tds_read_b64_tr_b16 %7, %17 offset:%22\n\t"
      "ds_read_b64_tr_b16 %10, %18 offset:%21\n\tds_read_b64_tr_b16 %14, %18 offset:%22\n\t"
      "ds_read_b64_tr_b16 %11, %19 offset:%21\n\tds_read_b64_tr_b16 %15, %19 offset:%22\n\t"
      "s_waitcnt lgkmcnt(8)"
      : "=&v"(al[0][0]), "=&v"(al[0][1]), "=&v"(al[1][0]), "=&v"(al[1][1]), "=&v"(ah[0][0]), "=&v"(ah[0][1]),
        "=&v"(ah[1][0]), "=&v"(ah[1][1]), "=&v"(bl[0][0]), "=&v"(bl[0][1]), "=&v"(bl[1][0]), "=&v"(bl[1][1]),
        "=&v"(bh[0][0]), "=&v"(bh[0][1]), "=&v"(bh[1][0]), "=&v"(bh[1][1])
      : "v"(ta0), "v"(ta1), "v"(tb0), "v"(tb1), "n"(8 * T), "n"(32 * T), "n"(40 * T)
      : "memory");
}
__device__ __forceinline__ void rest_tt(u32x2 (&al)[2][2], u32x2 (&ah)[2][2], u32x2 (&bl)[2][2], u32x2 (&bh)[2][2]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(al[1][0]), "+v"(al[1][1]), "+v"(ah[1][0]), "+v"(ah[1][1]), "+v"(bl[1][0]), "+v"(bl[1][1]),
                 "+v"(bh[1][0]), "+v"(bh[1][1])
               :
               : "memory");
}
// fp32, one half of a stage (8 values of k): lane half h holds k = 4 h + e, e = 0..3, of both operands.
__device__ __forceinline__ void read32_rr(f32x4 (&a)[2], f32x4 (&b)[2], uint32_t ra, uint32_t rb) {
  asm volatile(
      "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:2048\n\t"
      "ds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:2048\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0]), "=&v"(b[1])
      : "v"(ra), "v"(rb)
      : "memory");
}
template <int T, int KK>
__device__ __forceinline__ void read32_rt(f32x4 (&a)[2], float (&b)[2][4], uint32_t ra, uint32_t tb0, uint32_t tb1) {
  asm volatile(
      "ds_read_b128 %0, %10\n\tds_read_b128 %1, %10 offset:2048\n\t"
      "ds_read_b32 %2, %11 offset:%13\n\tds_read_b32 %3, %11 offset:%14\n\t"
      "ds_read_b32 %4, %11 offset:%15\n\tds_read_b32 %5, %11 offset:%16\n\t"
      "ds_read_b32 %6, %12 offset:%13\n\tds_read_b32 %7, %12 offset:%14\n\t"
      "ds_read_b32 %8, %12 offset:%15\n\tds_read_b32 %9, %12 offset:%16\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[0][2]), "=&v"(b[0][3]), "=&v"(b[1][0]),
        "=&v"(b[1][1]), "=&v"(b[1][2]), "=&v"(b[1][3])
      : "v"(ra), "v"(tb0), "v"(tb1), "n"(KK * 32 * T), "n"((KK * 8 + 1) * 4 * T), "n"((KK * 8 + 2) * 4 * T),
        "n"((KK * 8 + 3) * 4 * T)
      : "memory");
}
template <int T, int KK>
__device__ __forceinline__ void read32_tt(float (&a)[2][4], float (&b)[2][4], uint32_t ta0, uint32_t ta1, uint32_t tb0,
                                          uint32_t tb1) {
  asm volatile(
      "ds_read_b32 %0, %16 offset:%20\n\tds_read_b32 %1, %16 offset:%21\n\t"
      "ds_read_b32 %2, %16 offset:%22\n\tds_read_b32 %3, %16 offset:%23\n\t"
      "ds_read_b32 %4, %17 offset:%20\n\tds_read_b32 %5, %17 offset:%21\n\t"
      "ds_read_b32 %6, %17 offset:%22\n\tds_read_b32 %7, %17 offset:%23\n\t"
      "ds_read_b32 %8, %18 offset:%20\n\tds_read_b32 %9, %18 offset:%21\n\t"
      "ds_read_b32 %10, %18 offset:%22\n\tds_read_b32 %11, %18 offset:%23\n\t"
      "ds_read_b32 %12, %19 offset:%20\n\tds_read_b32 %13, %19 offset:%21\n\t"
      "ds_read_b32 %14, %19 offset:%22\n\tds_read_b32 %15, %19 offset:%23\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[0][2]), "=&v"(a[0][3]), "=&v"(a[1][0]), "=&v"(a[1][1]),
        "=&v"(a[1][2]), "=&v"(a[1][3]), "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[0][2]), "=&v"(b[0][3]),
        "=&v"(b[1][0]), "=&v"(b[1][1]), "=&v"(b[1][2]), "=&v"(b[1][3])
      : "v"(ta0), "v"(ta1), "v"(tb0), "v"(tb1), "n"(KK * 32 * T), "n"((KK * 8 + 1) * 4 * T), "n"((KK * 8 + 2) * 4 * T),
        "n"((KK * 8 + 3) * 4 * T)
      : "memory");
}

__device__ __forceinline__ bf16x8 frag(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ bf16x8 frag(u32x2 lo, u32x2 hi) {
  const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ float elem(const f32x4& v, int e) { return v[e]; }
__device__ __forceinline__ float elem(const float (&v)[4], int e) { return v[e]; }

// ---- tile geometry ----------------------------------------------------------------------------
template <typename E, int T, bool WIDE>
struct Geo {
  static constexpr int ES = sizeof(E);
  static constexpr int KB = 64 / ES;                // k values of a slab
  static constexpr int WC = T / 64;                 // wavefronts along a side of the tile
  static constexpr int WAVES = WIDE ? 8 : 4, THREADS = 64 * WAVES;
  static constexpr int KS = WAVES / (WC * WC);      // wavefronts along K
  static constexpr int BK = KB * KS;                // k values of a stage
  static constexpr bool kPrivate = WC == 1;         // every wavefront loads what it alone reads
  static constexpr int SLAB = T * 64;               // bytes of one operand's slab
  static constexpr int STAGE = KS * 2 * SLAB;
  // wide: one workgroup per CU with 128 KB of ring; else two with 64 KB each
  static constexpr int STAGES = (WIDE ? 131072 : 65536) / STAGE;
  static constexpr int LDW = T + 4;                 // floats per staged row of the epilogue (+4: rows on different banks)
  static constexpr int RING = STAGES * STAGE, STAGING = KS * T * LDW * 4;
  static constexpr int LDS = RING > STAGING ? RING : STAGING;
  static_assert(T == 64 || T == 128, "64 or 128");
};

// C tile (ti, tj) of matrix t.mat.  lds: Geo<E, T, WIDE>::LDS bytes, 256-byte aligned.
template <typename E, int T, bool WIDE, bool TP, bool TQ>
__device__ __forceinline__ void small_tile(const GemmArgs& a, const TileId& t, char* lds) {
  typedef Geo<E, T, WIDE> G;
  constexpr int ES = G::ES, CH = Chunk<E>::N;
  typedef typename Chunk<E>::vec vec_t;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = G::kPrivate ? wave : wave >> 2, w4 = wave & 3;
  const int wm = G::kPrivate ? 0 : w4 >> 1, wn = G::kPrivate ? 0 : w4 & 1;
  const int m0 = t.ti * T, n0 = t.tj * T;

  // E operand of the epilogue: requested first, so that it has arrived long before it is used
  constexpr int CPR = T / CH;                       // chunks per tile row
  constexpr int U = T * T / CH / G::THREADS;          // chunks per lane
  const E* __restrict__ Eb = a.E ? static_cast<const E*>(a.E) + (size_t)t.mat * a.strideE : nullptr;
  vec_t ev[U];
  if (Eb) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = u * G::THREADS + tid;
      ev[u] = *reinterpret_cast<const vec_t*>(Eb + (size_t)(m0 + idx / CPR) * a.lde + n0 + (idx % CPR) * CH);
    }
  }

  // ---- direct loads: lane l of load q fetches unit S (16 bytes) of the slab ----
  constexpr int NL = G::kPrivate ? 4 : 2;           // loads per operand, wavefront and stage
  static_assert(NL * 64 * (G::kPrivate ? 1 : 4) == T * 4, "a slab is 4 T units");
  const E* gp[NL];
  const E* gq[NL];
  static_for<NL>([&](auto q) {
    const int S = (G::kPrivate ? 0 : w4 * NL * 64) + q * 64 + lane;
    auto addr = [&](const void* base, int64_t stride, int ld, int r0, bool trans) -> const E* {
      const E* src = static_cast<const E*>(base) + (size_t)t.mat * stride;
      if (!trans) {
        const int row = S >> 2, c = (S & 3) ^ ((row >> 2) & 3);
        return src + (size_t)(r0 + row) * ld + kg * G::KB + c * CH;
      }
      constexpr int CPK = T / CH;                   // chunks per k-row
      const int k = S / CPK;
      const int x = ES == 4 ? ((k >> 2) & 1) << 3 : (T == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2);
      return src + (size_t)(kg * G::KB + k) * ld + r0 + ((S % CPK) ^ x) * CH;
    };
    gp[q] = addr(a.P, a.strideP, a.ldp, m0, TP);
    gq[q] = addr(a.Q, a.strideQ, a.ldq, n0, TQ);
  });
  const size_t incp = TP ? (size_t)G::BK * a.ldp : (size_t)G::BK;
  const size_t incq = TQ ? (size_t)G::BK * a.ldq : (size_t)G::BK;
  auto issue = [&](int stage, int kt) {
    char* const sp = lds + stage * G::STAGE + kg * 2 * G::SLAB + (G::kPrivate ? 0 : w4 * NL * 1024);
    static_for<NL>([&](auto q) {
      __builtin_amdgcn_global_load_lds((const MONA_AS1 void*)(gp[q] + kt * incp), (MONA_AS3 void*)(sp + q * 1024), 16, 0, 0);
    });
    static_for<NL>([&](auto q) {
      __builtin_amdgcn_global_load_lds((const MONA_AS1 void*)(gq[q] + kt * incq),
                                       (MONA_AS3 void*)(sp + G::SLAB + q * 1024), 16, 0, 0);
    });
  };

  // ---- fragment addresses, per lane, of stage 0 ----
  const uint32_t base = (uint32_t)(uintptr_t)(MONA_AS3 const char*)lds + kg * 2 * G::SLAB;
  const int frow = lane & 31, half = lane >> 5;
  // row-major operand: one address per half of the stage; K-major: one per 32-row block
  auto frag_addr = [&](bool trans, int w, int operand, int which) -> uint32_t {
    const uint32_t b = base + operand * G::SLAB;
    if (!trans) return b + (w * 64 + frow) * 64 + (((2 * which + half) ^ ((frow >> 2) & 3)) << 4);
    if constexpr (ES == 4) {
      const int c = w * 16 + which * 8 + (frow >> 2);
      return b + 4 * half * (T * 4) + ((c ^ (half << 3)) << 4) + (frow & 3) * 4;
    } else {
      const int tx = (lane & 15) >> 2, nl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      const int c = w * 8 + which * 4 + (nl >> 3);
      const int x = T == 128 ? tx << 2 : (tx >> 1) << 2;
      return b + (8 * half + tx) * (T * 2) + ((c ^ x) << 4) + (nl & 7) * 2;
    }
  };
  uint32_t fa[2], fb[2];
  static_for<2>([&](auto i) {
    fa[i] = frag_addr(TP, wm, 0, i);
    fb[i] = frag_addr(TQ, wn, 1, i);
  });

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  // one stage: fragment reads and products (the operand roles are swapped, so a block is accumulated transposed:
  // a lane holds one output row and, per group of four registers, four consecutive columns)
  auto read_then = [&](int stage, auto&& after_reads) {
    const uint32_t so = stage * G::STAGE;
    if constexpr (ES == 2) {
      u32x4 ar[2][2], br[2][2];
      u32x2 al[2][2], ah[2][2], bl[2][2], bh[2][2];
      if constexpr (!TP && !TQ) read_rr(ar, br, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
      else if constexpr (!TP) read_rt<T>(ar, bl, bh, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
      else read_tt<T>(al, ah, bl, bh, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
      static_for<2>([&](auto kk) {
        if constexpr (kk == 1) {
          if constexpr (!TP && !TQ) rest_rr(ar, br);
          else if constexpr (!TP) rest_rt(ar, bl, bh);
          else rest_tt(al, ah, bl, bh);
          after_reads();
        }
        static_for<2>([&](auto i) {
          static_for<2>([&](auto j) {
            bf16x8 pa, qb;
            if constexpr (TP) pa = frag(al[kk][i], ah[kk][i]); else pa = frag(ar[kk][i]);
            if constexpr (TQ) qb = frag(bl[kk][j], bh[kk][j]); else qb = frag(br[kk][j]);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qb, pa, acc[i][j], 0, 0, 0);
          });
        });
      });
    } else {
      static_for<2>([&](auto kk) {
        f32x4 ar[2], br[2];
        float at[2][4], bt[2][4];
        if constexpr (!TP && !TQ) read32_rr(ar, br, fa[kk] + so, fb[kk] + so);
        else if constexpr (!TP) read32_rt<T, kk>(ar, bt, fa[kk] + so, fb[0] + so, fb[1] + so);
        else read32_tt<T, kk>(at, bt, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
        if constexpr (kk == 1) after_reads();
        static_for<4>([&](auto e) {
          static_for<2>([&](auto i) {
            static_for<2>([&](auto j) {
              float pa, qb;
              if constexpr (TP) pa = elem(at[i], e); else pa = elem(ar[i], e);
              if constexpr (TQ) qb = elem(bt[j], e); else qb = elem(br[j], e);
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(qb, pa, acc[i][j], 0, 0, 0);
            });
          });
        });
      });
    }
  };

  // stages this wavefront goes through: K is a multiple of 128, a whole number of slabs
  const int KT = G::kPrivate ? (a.K / G::KB - kg + G::KS - 1) / G::KS : a.K / G::BK;
  constexpr int S = G::STAGES, LPS = 2 * NL;
  // wait until at most min(later, MAX) stages' loads are outstanding
  auto wait_stages = [&](int later) {
    constexpr int MAX = G::kPrivate ? S - 1 : S - 2;
    static_assert(MAX * LPS < 64, "the load counter holds 6 bits");
    bool done = false;
    static_for<MAX>([&](auto i) {
      if (!done && later >= MAX - i) { MONA_WAIT_VM((MAX - i) * LPS); done = true; }
    });
    if (!done) MONA_WAIT_VM(0);
  };
  if constexpr (G::kPrivate) {
    // a stage slot is this wavefront's own: it may be refilled as soon as its fragment reads have returned
    static_for<S>([&](auto s) { if (s < KT) issue(s, s); });
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
      const int later = KT - 1 - kt;
      wait_stages(later);
      read_then(stage, [&]() { if (kt + S < KT) issue(stage, kt + S); });
      stage = stage + 1 == S ? 0 : stage + 1;
    }
  } else {
    // shared slots: after the barrier of step kt the loads of stage kt have landed for every wavefront (each has
    // waited for its own) and every wavefront has read stage kt - 1, whose slot takes chunk kt + S - 1
    static_for<S - 1>([&](auto s) { if (s < KT) issue(s, s); });
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
      const int later = KT - 1 - kt;
      wait_stages(later);
      __builtin_amdgcn_s_barrier();     // bare: a fence would drain the loads in flight
      if (kt + S - 1 < KT) issue(stage == 0 ? S - 1 : stage - 1, kt + S - 1);
      read_then(stage, []() {});
      stage = stage + 1 == S ? 0 : stage + 1;
    }
  }

  // ---- epilogue: the K shares of the tile meet in LDS, every global access is a 16-byte piece of a row ----
  const int mi = a.members ? a.members[t.mat] : t.mat;
  float post = 1.0f;
  if (a.post == POST_INV) post = a.scales[mi].inv;
  else if (a.post == POST_INV2) post = a.scales[mi].inv2;
  const bool mirror = a.symmetric && t.ti != t.tj, update = a.epilogue == EPI_UPDATE;
  bool skip_w = true;
  int wm_real = 0, wn_real = 0, w_is_bf16 = 0;
  void* wptr = nullptr;
  if (update) {
    const MatStatic& ms = a.stat[mi];
    wm_real = ms.m; wn_real = ms.n; w_is_bf16 = ms.w_dtype;
    wptr = a.dyn[mi].w;
    skip_w = (a.scales[mi].status & 2u) != 0;
  }
  const bool w_vec = wn_real % CH == 0;             // rows of W are whole chunks, 16-byte (fp32: 32-byte) aligned
  __syncthreads();                                  // every wavefront has finished reading operands
  float* const sum = reinterpret_cast<float*>(lds);
  {
    float* const mine = sum + kg * T * G::LDW + (wm * 64 + frow) * G::LDW + wn * 64 + 4 * half;
    static_for<2>([&](auto i) {
      static_for<2>([&](auto j) {
        static_for<4>([&](auto vg) {
          const f32x4 v = {acc[i][j][vg * 4 + 0], acc[i][j][vg * 4 + 1], acc[i][j][vg * 4 + 2], acc[i][j][vg * 4 + 3]};
          *reinterpret_cast<f32x4*>(mine + i * 32 * G::LDW + j * 32 + 8 * vg) = v;
        });
      });
    });
  }
  __syncthreads();
  E* __restrict__ C = static_cast<E*>(a.C) + (size_t)t.mat * a.strideC;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int idx = u * G::THREADS + tid;
    const int r = idx / CPR, ch = idx % CPR;
    const int grow = m0 + r, gcol = n0 + ch * CH;
    float val[CH];
#pragma unroll
    for (int e = 0; e < CH; ++e) val[e] = 0.0f;
    static_for<G::KS>([&](auto s) {
      static_for<CH / 4>([&](auto q) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(sum + (s * T + r) * G::LDW + ch * CH + q * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) val[q * 4 + e] = s == 0 ? p[e] : val[q * 4 + e] + p[e];
      });
    });
    if (Eb) {
#pragma unroll
      for (int e = 0; e < CH; ++e) val[e] = post * (a.alpha * val[e] + a.beta * (float)ev[u][e]);
    } else {
#pragma unroll
      for (int e = 0; e < CH; ++e) val[e] = post * (a.alpha * val[e]);
    }
    if (a.diag != 0.0f && grow < a.diag_n) {
      // not to the padding: that must be zero in every buffer, because a product whose tiles are 64 wide in this step may
      // leave out padding that a 128-wide tile wrote in another
#pragma unroll
      for (int e = 0; e < CH; ++e) val[e] += (grow == gcol + e) ? a.diag : 0.0f;
    }
    vec_t ov;
#pragma unroll
    for (int e = 0; e < CH; ++e) ov[e] = (E)val[e];
    if (!update || a.store_out) *reinterpret_cast<vec_t*>(C + (size_t)grow * a.ldc + gcol) = ov;
    if (mirror) {
      // the rounded result, for the transposed pass below, in place of the share this lane alone has read
      static_for<CH / 4>([&](auto q) {
        const f32x4 p = {(float)ov[q * 4 + 0], (float)ov[q * 4 + 1], (float)ov[q * 4 + 2], (float)ov[q * 4 + 3]};
        *reinterpret_cast<f32x4*>(sum + r * G::LDW + ch * CH + q * 4) = p;
      });
    }
    if (update && !skip_w && grow < wm_real) {
      // W <- (1 - eta lambda) W - eta gamma O, O as stored in the working precision
      const size_t wi = (size_t)grow * wn_real + gcol;
      if (w_vec && gcol + CH <= wn_real) {
        if (w_is_bf16) {
          typedef bf16_t wv_t __attribute__((ext_vector_type(CH)));
          wv_t* wp = reinterpret_cast<wv_t*>(static_cast<bf16_t*>(wptr) + wi);
          wv_t w = *wp;
#pragma unroll
          for (int e = 0; e < CH; ++e) w[e] = (bf16_t)(a.w_keep * (float)w[e] - a.o_scale * (float)ov[e]);
          *wp = w;
        } else {
          f32x4* wp = reinterpret_cast<f32x4*>(static_cast<float*>(wptr) + wi);
          static_for<CH / 4>([&](auto q) {
            f32x4 w = wp[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = a.w_keep * w[e] - a.o_scale * (float)ov[q * 4 + e];
            wp[q] = w;
          });
        }
      } else {
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          if (gcol + e < wn_real) {
            if (w_is_bf16) {
              bf16_t* w = static_cast<bf16_t*>(wptr) + wi + e;
              *w = (bf16_t)(a.w_keep * (float)*w - a.o_scale * (float)ov[e]);
            } else {
              float* w = static_cast<float*>(wptr) + wi + e;
              *w = a.w_keep * *w - a.o_scale * (float)ov[e];
            }
          }
        }
      }
    }
  }
  if (mirror) {
    // transposed copy: a wavefront writes 8 columns of the tile x 8 pieces of 16 bytes along its rows
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int grp = u * G::WAVES + wave;
      const int c = (grp % (T / 8)) * 8 + (lane >> 3), rc = (grp / (T / 8)) * 8 + (lane & 7);
      vec_t ov;
#pragma unroll
      for (int e = 0; e < CH; ++e) ov[e] = (E)sum[(rc * CH + e) * G::LDW + c];
      *reinterpret_cast<vec_t*>(C + (size_t)(n0 + c) * a.ldc + m0 + rc * CH) = ov;
    }
  }
}

// One workgroup per tile.  Group g of the batch owns the slots [slot_end[g - 1], slot_end[g]) of every die: workgroup
// L runs on die L % 8, and each die takes one contiguous eighth of every group's tiles, so that tiles that share
// operands share an L2 and no die gets all of the group with the longest K.
template <typename E, bool WIDE>
__global__ __launch_bounds__(WIDE ? 512 : 256) void ns_small_kernel(const GemmBatch b) {
  constexpr int L64 = Geo<E, 64, WIDE>::LDS, L128 = Geo<E, 128, WIDE>::LDS;
  __shared__ __attribute__((aligned(256))) char lds[L64 > L128 ? L64 : L128];
  const int die = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  int g = 0;
  while (g + 1 < b.n && slot >= b.slot_end[g]) ++g;
  const int first = g > 0 ? b.slot_end[g - 1] : 0;
  const GemmArgs& a = b.a[g];
  const int per_die = b.slot_end[g] - first, local = slot - first;
  const TileId t = decode_logical(a, die * per_die + local, local < per_die);
  if (!t.valid) return;
  auto run = [&](auto tile) {
    if (!a.trans_p && !a.trans_q) small_tile<E, tile, WIDE, false, false>(a, t, lds);
    else if (!a.trans_p) small_tile<E, tile, WIDE, false, true>(a, t, lds);
    else small_tile<E, tile, WIDE, true, true>(a, t, lds);
  };
  if (a.tile_m == 64) run(IC<64>{}); else run(IC<128>{});
}

}  // namespace

hipError_t launch_ns_small(GemmBatch& b, bool f32, bool wide, hipStream_t s) {
  if (b.n < 1 || b.n > kMaxMerged) return hipErrorInvalidValue;
  long long slots = 0;
  for (int g = 0; g < b.n; ++g) {
    const GemmArgs& a = b.a[g];
    if ((a.tile_m != 64 && a.tile_m != 128) || a.tile_n != a.tile_m || (a.trans_p && !a.trans_q)) return hipErrorInvalidValue;
    slots += slots_per_die(a);
    if (slots * kXcds > 0x7fffff00LL) return hipErrorInvalidValue;
    b.slot_end[g] = (int32_t)slots;
  }
  const dim3 grid((unsigned)(slots * kXcds));
  if (grid.x == 0) return hipSuccess;
  if (f32 && wide) hipLaunchKernelGGL((ns_small_kernel<float, true>), grid, dim3(512), 0, s, b);
  else if (f32) hipLaunchKernelGGL((ns_small_kernel<float, false>), grid, dim3(256), 0, s, b);
  else if (wide) hipLaunchKernelGGL((ns_small_kernel<bf16_t, true>), grid, dim3(512), 0, s, b);
  else hipLaunchKernelGGL((ns_small_kernel<bf16_t, false>), grid, dim3(256), 0, s, b);
  return hipGetLastError();
}

}  // namespace mona
