// Newton-Schulz products for launches that do not fill the chip with 256 x 256 tiles, in bf16 and (the shortest K, and
// chains; otherwise ns_split.hip) in fp32.
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
// Measured, us per step, one chain of launches per group on a register-staged 128 x 128 kernel -> here: a block of hidden size 1000
// 664 -> 505.  (Steps as small as one 256 x 512 matrix, 170 -> 99, or nine ragged ones, 980 -> 189, are one launch now: chains, below.)
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
#include "ns_small_tile.h"

#include <atomic>

namespace mona {

namespace {

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
// the same for a tile of a single block (T = 32: K-major rows of 64 bytes)
__device__ __forceinline__ void read1_rr(u32x4 (&a)[2], u32x4 (&b)[2], uint32_t ra0, uint32_t ra1, uint32_t rb0, uint32_t rb1) {
  asm volatile(
      "ds_read_b128 %0, %4\n\tds_read_b128 %2, %6\n\tds_read_b128 %1, %5\n\tds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0]), "=&v"(b[1])
      : "v"(ra0), "v"(ra1), "v"(rb0), "v"(rb1)
      : "memory");
}
__device__ __forceinline__ void read1_rt(u32x4 (&a)[2], u32x2 (&bl)[2], u32x2 (&bh)[2], uint32_t ra0, uint32_t ra1, uint32_t tb) {
  asm volatile(
      "ds_read_b128 %0, %6\n\tds_read_b64_tr_b16 %2, %8\n\tds_read_b64_tr_b16 %4, %8 offset:256\n\t"
      "ds_read_b128 %1, %7\n\tds_read_b64_tr_b16 %3, %8 offset:1024\n\tds_read_b64_tr_b16 %5, %8 offset:1280\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(bl[0]), "=&v"(bl[1]), "=&v"(bh[0]), "=&v"(bh[1])
      : "v"(ra0), "v"(ra1), "v"(tb)
      : "memory");
}
__device__ __forceinline__ void read1_tt(u32x2 (&al)[2], u32x2 (&ah)[2], u32x2 (&bl)[2], u32x2 (&bh)[2], uint32_t ta, uint32_t tb) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %2, %8 offset:256\n\t"
      "ds_read_b64_tr_b16 %4, %9\n\tds_read_b64_tr_b16 %6, %9 offset:256\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:1024\n\tds_read_b64_tr_b16 %3, %8 offset:1280\n\t"
      "ds_read_b64_tr_b16 %5, %9 offset:1024\n\tds_read_b64_tr_b16 %7, %9 offset:1280\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(al[0]), "=&v"(al[1]), "=&v"(ah[0]), "=&v"(ah[1]), "=&v"(bl[0]), "=&v"(bl[1]), "=&v"(bh[0]), "=&v"(bh[1])
      : "v"(ta), "v"(tb)
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

__device__ __forceinline__ void read32_1_rr(f32x4& a, f32x4& b, uint32_t ra, uint32_t rb) {
  asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(a), "=&v"(b) : "v"(ra), "v"(rb) : "memory");
}
template <int KK>
__device__ __forceinline__ void read32_1_rt(f32x4& a, float (&b)[4], uint32_t ra, uint32_t tb) {
  asm volatile(
      "ds_read_b128 %0, %5\n\tds_read_b32 %1, %6 offset:%7\n\tds_read_b32 %2, %6 offset:%8\n\t"
      "ds_read_b32 %3, %6 offset:%9\n\tds_read_b32 %4, %6 offset:%10\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(a), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
      : "v"(ra), "v"(tb), "n"(KK * 1024), "n"(KK * 1024 + 128), "n"(KK * 1024 + 256), "n"(KK * 1024 + 384)
      : "memory");
}
template <int KK>
__device__ __forceinline__ void read32_1_tt(float (&a)[4], float (&b)[4], uint32_t ta, uint32_t tb) {
  asm volatile(
      "ds_read_b32 %0, %8 offset:%10\n\tds_read_b32 %1, %8 offset:%11\n\t"
      "ds_read_b32 %2, %8 offset:%12\n\tds_read_b32 %3, %8 offset:%13\n\t"
      "ds_read_b32 %4, %9 offset:%10\n\tds_read_b32 %5, %9 offset:%11\n\t"
      "ds_read_b32 %6, %9 offset:%12\n\tds_read_b32 %7, %9 offset:%13\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
      : "v"(ta), "v"(tb), "n"(KK * 1024), "n"(KK * 1024 + 128), "n"(KK * 1024 + 256), "n"(KK * 1024 + 384)
      : "memory");
}

__device__ __forceinline__ float elem(const f32x4& v, int e) { return v[e]; }
__device__ __forceinline__ float elem(const float (&v)[4], int e) { return v[e]; }

// ---- tile geometry ----------------------------------------------------------------------------
template <typename E, int T, bool WIDE>
struct Geo {
  static constexpr int ES = sizeof(E);
  static constexpr int KB = 64 / ES;                // k values of a slab
  static constexpr int WC = T == 128 ? 2 : 1;       // wavefronts along a side of the tile
  static constexpr int NB = T == 32 ? 1 : 2;        // 32 x 32 blocks along a side of a wavefront's part of it
  static constexpr int WAVES = WIDE ? 8 : 4, THREADS = 64 * WAVES;
  static constexpr int KS = WAVES / (WC * WC);      // wavefronts along K
  static constexpr int BK = KB * KS;                // k values of a stage
  static constexpr bool kPrivate = WC == 1;         // every wavefront loads what it alone reads
  static constexpr int SLAB = T * 64;               // bytes of one operand's slab
  static constexpr int STAGE = KS * 2 * SLAB;
  // wide: one workgroup per CU with 128 KB of ring (T = 32: 96, the shares of the sum behind it); else two with 64 KB each
  static constexpr int STAGES = (T == 32 ? 98304 : WIDE ? 131072 : 65536) / STAGE;
  static constexpr int LDW = staged_ld(T);
  static constexpr int RING = STAGES * STAGE, STAGING = KS * T * LDW * 4;
  static constexpr int SUM_AT = T == 32 ? RING : 0;
  static constexpr int LDS = T == 32 ? RING + STAGING : RING > STAGING ? RING : STAGING;
  static_assert(T == 32 || T == 64 || T == 128, "32, 64 or 128");
};

// C tile (ti, tj) of matrix t.mat.  lds: Geo<E, T, WIDE>::LDS bytes, 256-byte aligned.  SHARED: other workgroups of this
// launch write the operands and read the result (Sharing).  FRESH: every wavefront fetches its operands again until all of them
// have been written, at most `patience` times; if one gives up, nothing is stored and the result is false.
template <typename E, int T, bool WIDE, bool TP, bool TQ, int SHARED>
__device__ __forceinline__ bool small_tile(const GemmArgs& a, const TileId& t, const TileMatrix& v, int tid, char* lds,
                                           int patience = 0, uint32_t* gave_up = nullptr) {
  typedef Geo<E, T, WIDE> G;
  constexpr int ES = G::ES, CH = Chunk<E>::N;
  typedef typename Chunk<E>::vec vec_t;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = G::kPrivate ? wave : wave >> 2, w4 = wave & 3;
  const int wm = G::kPrivate ? 0 : w4 >> 1, wn = G::kPrivate ? 0 : w4 & 1;
  const int m0 = t.ti * T, n0 = t.tj * T;

  // E operand of the epilogue: requested first, so that it has arrived long before it is used
  auto epilogue = [&]() {
    if constexpr (T == 32) return Finish32<E, G::KS, SHARED>(a, t, v, tid);
    else return FinishTile<E, T, G::KS, G::THREADS, SHARED>(a, t, tid);
  }();

  // ---- direct loads: lane l of load q fetches unit S (16 bytes) of the slab ----
  constexpr int NL = G::kPrivate ? T / 16 : 2;      // loads per operand, wavefront and stage
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
      const int x = T == 32 ? 0 : ES == 4 ? ((k >> 2) & 1) << 3 : (T == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2);
      return src + (size_t)(kg * G::KB + k) * ld + r0 + ((S % CPK) ^ x) * CH;
    };
    gp[q] = addr(a.P, a.strideP, a.ldp, m0, TP);
    gq[q] = addr(a.Q, a.strideQ, a.ldq, n0, TQ);
  });
  const size_t incp = TP ? (size_t)G::BK * a.ldp : (size_t)G::BK;
  const size_t incq = TQ ? (size_t)G::BK * a.ldq : (size_t)G::BK;
  auto issue_p = [&](int stage, int kt) {
    char* const sp = lds + stage * G::STAGE + kg * 2 * G::SLAB + (G::kPrivate ? 0 : w4 * NL * 1024);
    static_for<NL>([&](auto q) {
      __builtin_amdgcn_global_load_lds((const MONA_AS1 void*)(gp[q] + kt * incp), (MONA_AS3 void*)(sp + q * 1024), 16, 0,
                                       SHARED ? kDeviceScope : 0);
    });
  };
  auto issue_q = [&](int stage, int kt) {
    char* const sp = lds + stage * G::STAGE + kg * 2 * G::SLAB + (G::kPrivate ? 0 : w4 * NL * 1024);
    static_for<NL>([&](auto q) {
      __builtin_amdgcn_global_load_lds((const MONA_AS1 void*)(gq[q] + kt * incq),
                                       (MONA_AS3 void*)(sp + G::SLAB + q * 1024), 16, 0, SHARED ? kDeviceScope : 0);
    });
  };
  auto issue = [&](int stage, int kt) { issue_p(stage, kt); issue_q(stage, kt); };

  // ---- fragment addresses, per lane, of stage 0 ----
  const uint32_t base = (uint32_t)(uintptr_t)(MONA_AS3 const char*)lds + kg * 2 * G::SLAB;
  const int frow = lane & 31, half = lane >> 5;
  // row-major operand: one address per half of the stage; K-major: one per 32-row block
  auto frag_addr = [&](bool trans, int w, int operand, int which) -> uint32_t {
    const uint32_t b = base + operand * G::SLAB;
    if (!trans) return b + (w * 64 + frow) * 64 + (((2 * which + half) ^ ((frow >> 2) & 3)) << 4);
    if constexpr (ES == 4) {
      const int c = w * 16 + which * 8 + (frow >> 2);
      return b + 4 * half * (T * 4) + ((T == 32 ? c : c ^ (half << 3)) << 4) + (frow & 3) * 4;
    } else {
      const int tx = (lane & 15) >> 2, nl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      const int c = w * 8 + which * 4 + (nl >> 3);
      const int x = T == 32 ? 0 : T == 128 ? tx << 2 : (tx >> 1) << 2;
      return b + (8 * half + tx) * (T * 2) + ((c ^ x) << 4) + (nl & 7) * 2;
    }
  };
  uint32_t fa[2], fb[2];
  static_for<2>([&](auto i) {
    fa[i] = frag_addr(TP, wm, 0, i);
    fb[i] = frag_addr(TQ, wn, 1, i);
  });

  constexpr int NB = G::NB;
  f32x16 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  // one stage: fragment reads and products (the operand roles are swapped, so a block is accumulated transposed:
  // a lane holds one output row and, per group of four registers, four consecutive columns)
  // FRESH: what of a stage has been read again and again until it was whole
  auto whole = [&](int kt, int stage, auto&& read, auto&& look) {
    read();
    if constexpr (SHARED == FRESH) {
      for (;;) {
        Unwritten<E> p, q;
        look([&](const auto& x) { p.see(x); }, [&](const auto& x) { q.see(x); });
        const bool more_p = __any(p.any()), more_q = __any(q.any());
        if (!more_p && !more_q) break;
        if (patience <= 0) { *gave_up = 1u; break; }
        --patience;
        if (more_p) issue_p(stage, kt);
        if (more_q) issue_q(stage, kt);
        MONA_WAIT_VM(0);
        read();
      }
    }
  };
  auto read_then = [&](int kt, int stage, auto&& after_reads) {
    const uint32_t so = stage * G::STAGE;
    if constexpr (T == 32 && ES == 2) {
      u32x4 ar[2], br[2];
      u32x2 al[2], ah[2], bl[2], bh[2];
      whole(kt, stage, [&]() {
        if constexpr (!TP && !TQ) read1_rr(ar, br, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
        else if constexpr (!TP) read1_rt(ar, bl, bh, fa[0] + so, fa[1] + so, fb[0] + so);
        else read1_tt(al, ah, bl, bh, fa[0] + so, fb[0] + so);
      }, [&](auto&& p, auto&& q) {
        static_for<2>([&](auto kk) {
          if constexpr (TP) { p(al[kk]); p(ah[kk]); } else p(ar[kk]);
          if constexpr (TQ) { q(bl[kk]); q(bh[kk]); } else q(br[kk]);
        });
      });
      after_reads();
      static_for<2>([&](auto kk) {
        bf16x8 pa, qb;
        if constexpr (TP) pa = frag(al[kk], ah[kk]); else pa = frag(ar[kk]);
        if constexpr (TQ) qb = frag(bl[kk], bh[kk]); else qb = frag(br[kk]);
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qb, pa, acc[0][0], 0, 0, 0);
      });
    } else if constexpr (T == 32) {
      static_for<2>([&](auto kk) {
        f32x4 ar, br;
        float at[4], bt[4];
        whole(kt, stage, [&]() {
          if constexpr (!TP && !TQ) read32_1_rr(ar, br, fa[kk] + so, fb[kk] + so);
          else if constexpr (!TP) read32_1_rt<kk>(ar, bt, fa[kk] + so, fb[0] + so);
          else read32_1_tt<kk>(at, bt, fa[0] + so, fb[0] + so);
        }, [&](auto&& p, auto&& q) {
          if constexpr (TP) static_for<4>([&](auto e) { p(at[e]); }); else p(ar);
          if constexpr (TQ) static_for<4>([&](auto e) { q(bt[e]); }); else q(br);
        });
        if constexpr (kk == 1) after_reads();
        static_for<4>([&](auto e) {
          float pa, qb;
          pa = TP ? at[e] : elem(ar, e);
          qb = TQ ? bt[e] : elem(br, e);
          acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(qb, pa, acc[0][0], 0, 0, 0);
        });
      });
    } else if constexpr (ES == 2) {
      u32x4 ar[2][2], br[2][2];
      u32x2 al[2][2], ah[2][2], bl[2][2], bh[2][2];
      auto rest = [&]() {
        if constexpr (!TP && !TQ) rest_rr(ar, br);
        else if constexpr (!TP) rest_rt(ar, bl, bh);
        else rest_tt(al, ah, bl, bh);
      };
      whole(kt, stage, [&]() {
        if constexpr (!TP && !TQ) read_rr(ar, br, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
        else if constexpr (!TP) read_rt<T>(ar, bl, bh, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
        else read_tt<T>(al, ah, bl, bh, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
        if constexpr (SHARED == FRESH) rest();
      }, [&](auto&& p, auto&& q) {
        static_for<2>([&](auto kk) {
          static_for<2>([&](auto i) {
            if constexpr (TP) { p(al[kk][i]); p(ah[kk][i]); } else p(ar[kk][i]);
            if constexpr (TQ) { q(bl[kk][i]); q(bh[kk][i]); } else q(br[kk][i]);
          });
        });
      });
      static_for<2>([&](auto kk) {
        if constexpr (kk == 1) {
          if constexpr (SHARED != FRESH) rest();
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
        whole(kt, stage, [&]() {
          if constexpr (!TP && !TQ) read32_rr(ar, br, fa[kk] + so, fb[kk] + so);
          else if constexpr (!TP) read32_rt<T, kk>(ar, bt, fa[kk] + so, fb[0] + so, fb[1] + so);
          else read32_tt<T, kk>(at, bt, fa[0] + so, fa[1] + so, fb[0] + so, fb[1] + so);
        }, [&](auto&& p, auto&& q) {
          static_for<2>([&](auto i) {
            if constexpr (TP) static_for<4>([&](auto e) { p(at[i][e]); }); else p(ar[i]);
            if constexpr (TQ) static_for<4>([&](auto e) { q(bt[i][e]); }); else q(br[i]);
          });
        });
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

  // stages this wavefront goes through: K is a multiple of 128, a whole number of slabs; slabs of padding alone are left out where
  // every wavefront has its own
  const int KT = G::kPrivate ? ((a.k_real + 31) / 32 * 32 / G::KB - kg + G::KS - 1) / G::KS : a.K / G::BK;
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
      read_then(kt, stage, [&]() { if (kt + S < KT) issue(stage, kt + S); });
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
      read_then(kt, stage, []() {});
      stage = stage + 1 == S ? 0 : stage + 1;
    }
  }

  // ---- epilogue: the K shares of the tile meet in LDS, every global access is a piece of a row ----
  if constexpr (T != 32) __syncthreads();           // every wavefront has finished reading operands
  float* const sum = reinterpret_cast<float*>(lds + G::SUM_AT);
  {
    float* const mine = sum + kg * T * G::LDW + (wm * 64 + frow) * G::LDW + wn * 64 + 4 * half;
    static_for<NB>([&](auto i) {
      static_for<NB>([&](auto j) {
        static_for<4>([&](auto vg) {
          const f32x4 q = {acc[i][j][vg * 4 + 0], acc[i][j][vg * 4 + 1], acc[i][j][vg * 4 + 2], acc[i][j][vg * 4 + 3]};
          *reinterpret_cast<f32x4*>(mine + i * 32 * G::LDW + j * 32 + 8 * vg) = q;
        });
      });
    });
  }
  if constexpr (SHARED == FRESH) {
    // the E operand likewise, a wavefront's pieces at a time
    while (a.E) {
      Unwritten<E> u;
      epilogue.see(u);
      if (!__any(u.any())) break;
      if (patience <= 0) { *gave_up = 1u; break; }
      --patience;
      epilogue.load_e(a, t);
    }
  }
  __syncthreads();
  if constexpr (SHARED == FRESH)
    if (__builtin_amdgcn_readfirstlane(*gave_up) != 0u) return false;
  epilogue.run(a, t, v, sum);
  return true;
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
  const TileMatrix v = look_up(a, t);
  auto run = [&](auto tile) {
    if (!a.trans_p && !a.trans_q) small_tile<E, tile, WIDE, false, false, OWN_LAUNCH>(a, t, v, threadIdx.x, lds);
    else if (!a.trans_p) small_tile<E, tile, WIDE, false, true, OWN_LAUNCH>(a, t, v, threadIdx.x, lds);
    else small_tile<E, tile, WIDE, true, true, OWN_LAUNCH>(a, t, v, threadIdx.x, lds);
  };
  if constexpr (WIDE)
    if (a.tile_m == 32) { run(IC<32>{}); return; }
  if (a.tile_m == 64) run(IC<64>{}); else run(IC<128>{});
}

// All products of a step of several small groups in one launch.
//
// A chain of small products is bound by what every launch of its own costs: 5 to 7 us with 16 to 100 tiles, of which the
// products themselves are two to four.  Here the tiles of all products are tasks, numbered product by product in the
// order of the chains; workgroup w of W takes the tasks w, w + W, w + 2 W, ..., waits for the tiles of its matrix in the
// product before, computes the tile and says so.  How it waits:
//   * With a buffer for every product (NEW; the pool in chain_pool.hip) the data are their own flag: the buffers are filled beforehand with a
//     pattern that no result holds, and a wavefront fetches its share of the operands again until none of it is left (Unwritten, in
//     whole() below).  That takes the wait for the stores, the flag's way and the fetch behind it out of every product, and no barrier
//     stands before one.  A product of 256 x 512 takes 3.1 us then (1.2 to 1.5 from the last store to the last wavefront's operands, 2.8
//     where 128 workgroups ask for the same B), 4.2 with flags.
//   * Otherwise it polls a flag a task (ChainArgs::flags) of the tiles in the product before, and raises its own.
// Measured, us per step, with flags -> without (one launch in front of both): 256 x 512 71.3 -> 54.5, 512 x 1408 111.1 -> 89.9, 700 x 700 116.3 -> 90.9,
// 4 x 300 x 900 101.3 -> 87.6, 12 x 256 x 512 105.9 -> 95.3, 512 x 512 with fp32 products 131 -> 102.5, nine ragged matrices in both precisions
// 74.5 -> 71.5.  Filling is what many matrices and much padding pay for it: 28 x 256 x 256 (51 MB) 113.5 -> 113.5; the two lists found that
// lose are long ones (three launches in front), 40 x 160 x 140 (41 MB) 99.2 -> 101.1 and 100 x 60 x 60 with fp32 products (23 MB) 94.6 -> 98.3.
//   * No workgroup waits for one that does not run.  W is not the size of the grid but the number of workgroups that have
//     reported when the first of them closes the roll (all of the grid, unless the chip is busy with something else for
//     c.roll_polls polls).  Tasks wait for lower numbers only, and a workgroup takes its own in order, so the lowest unfinished
//     task always has all it needs.  (Numbers go by the order of reporting: a
//     workgroup begins its first task before the roll is closed.  Waiting for that, so as to give every die
//     neighbouring tiles by the workgroup's index, costs 6 to 7 us a step and gains at most 4 where the tiles are many.)
//   * Where the roll was closed without some, the tasks behind the first W are drawn from a counter instead, in order, so that
//     whoever comes later takes its share from then on: a chain that began on the few CUs another stream's kernels had left
//     would otherwise keep to them when the chip is free again.  Measured, us per step beside steps of 64 x 2048 x 1024 on
//     another stream, launches / chain without latecomers / with: 256 x 512 650 / 430 / 265, 512 x 1408 870 / 1400 to 4800 / 310, nine
//     ragged matrices 865 / 480 to 1100 / 270, 4 x 300 x 900 1060 / 1100 to 4400 / 355; alone the code costs nine ragged
//     matrices 1 us.
//   * The dies have an L2 each.  What one workgroup writes and another reads goes through device-scope (sc1) accesses, which
//     are coherent by themselves; a flag follows when the stores have completed (vmcnt 0 in every wavefront, then the
//     barrier).  Measured from the last store of a product to the first operands of the next: about 2 us, against 4 to 6 us
//     with the caches written back and invalidated (release and acquire fences); plain loads in their place would save
//     another 2 us a step.
//   * 32 x 32 tiles, K split between the eight wavefronts, where every one has a CU of its own: a tile of 64 x 64 takes 2.8 us
//     with K = 256 and 4.4 with 512, one of 32 x 32 2.1 and 2.5 (the CU's own 64 bytes a cycle from L2, and latency).
// Measured when all of them had flags, us per step, launches -> chain: one 256 x 512 matrix 99 -> 73, 512 x 1408 without allocation 137 -> 114, nine
// ragged matrices in both precisions 189 -> 84 (which had waited for the host).  Tickets instead of fixed numbers, drawn by an atomic
// operation for every task, and a counter of finished tiles instead of flags: 96, 189 and 133.
constexpr uint32_t kRollClosed = 0x80000000u;

__device__ __forceinline__ uint32_t device_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void device_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wait lasts microseconds.  Two steps on one workspace at the same time (which the entry points forbid) could clear each
// other's flags: a workgroup that has polled c.patience times in one wait marks the matrices of the chain and leaves, and so
// do, one after the other, those that wait for its tiles, so that every launch ends and no parameter is formed from an incomplete
// product.  (Looking whether wavefront 0 has given up costs every task an LDS read behind the barrier, 1 us of a step of 70 to
// 114; hidden behind the first loads, or looked at in front of the stores, it costs 2.)
//
// F32: some of the groups have fp32 products.  Both kinds of products together are 66 KB of code, bf16 alone 33 (256 x 512: 0.9 us a
// step less; a CU shares 64 KB of instruction cache with another).
template <bool F32, bool NEW>
__global__ __launch_bounds__(512) void ns_chain_kernel(const ChainArgs c) {
  constexpr int LB = Geo<bf16_t, 64, true>::LDS, LF = Geo<float, 64, true>::LDS;
  __shared__ __attribute__((aligned(256))) char lds[LB > LF ? LB : LF];
  __shared__ uint32_t shared, drawn, gave_up;
  if (threadIdx.x == 0) {
    ChainRoll* const roll = c.roll;
    gave_up = 0u;
    const uint32_t n = __hip_atomic_fetch_add(&roll->reported, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n == 0) {
      // the first to report closes the roll
      uint32_t seen = 1;
      for (int i = 0; i < c.roll_polls && (seen = device_load(&roll->reported)) < gridDim.x; ++i) __builtin_amdgcn_s_sleep(8);
      if (seen < gridDim.x)
        seen = __hip_atomic_fetch_or(&roll->reported, kRollClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      device_store(&roll->workgroups, seen);
    }
    shared = n;
  }
  __syncthreads();
  const uint32_t number = __builtin_amdgcn_readfirstlane(shared);
  __syncthreads();
  // step: 0 not known yet, < 0 where the tasks are drawn
  int workgroups = 0, step = 0;
  // the number of workgroups that had reported when the roll was closed (0: the wait did not end)
  auto ask = [&]() {
    if (threadIdx.x == 0) {
      ChainRoll* roll = c.roll;
      asm volatile("" : "+v"(roll));     // (looked up anew: kept from the beginning it would take registers of every task)
      uint32_t n = 0;
      for (int patience = c.patience; patience > 0 && (n = device_load(&roll->workgroups)) == 0u; --patience) __builtin_amdgcn_s_sleep(1);
      shared = n;
      if (n == 0u) gave_up = 1u;
    }
    __syncthreads();
    workgroups = (int)__builtin_amdgcn_readfirstlane(shared);
    step = workgroups == (int)gridDim.x ? workgroups : -1;
  };
  auto draw = [&]() -> int {
    if (threadIdx.x == 0) {
      ChainRoll* roll = c.roll;
      asm volatile("" : "+v"(roll));
      drawn = (uint32_t)workgroups + __hip_atomic_fetch_add(&roll->drawn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return (int)__builtin_amdgcn_readfirstlane(drawn);
  };
  int task = (int)number;
  if (number & kRollClosed) {        // a latecomer
    ask();
    task = workgroups != 0 ? draw() : c.tasks;
  }
  for (int i = 0; task < c.tasks;) {
    // (four products at a time: a position has one for each group, and each look is a round trip to the scalar cache; nine ragged
    // matrices in seven groups 81.0 -> 79.5 us a step)
    for (int passed = 4; passed == 4; i += passed)
      passed = (task >= c.op[i].end) + (task >= c.op[i + 1].end) + (task >= c.op[i + 2].end) + (task >= c.op[i + 3].end);
    const int first = i > 0 ? c.op[i - 1].end : 0;
    const uint32_t code = c.op[i].code;
    const GroupDesc& g = c.group[code >> OPF_GROUP];
    GemmArgs a;
    expand_op(c.step, g, code, a);
    const TileId t = decode_logical(a, task - first, true);
    const TileMatrix v = look_up(a, t);
    // the tiles of this matrix in the product before, 64 flags at a time
    const int per_mat = c.op[i].before_per_mat;
    const uint32_t* const before = c.flags + c.op[i].before + t.mat * per_mat;
    if constexpr (NEW) {
      if (per_mat > 0 && c.patience <= 0 && threadIdx.x == 0) gave_up = 1u;
    } else if (threadIdx.x < 64) {
      for (int at = 0; at < per_mat; at += 64) {
        const int k = at + (int)threadIdx.x;
        int patience = c.patience;
        while (patience > 0 && !__all(k >= per_mat || device_load(before + k) != 0u)) --patience;
        if (patience <= 0) { gave_up = 1u; break; }
      }
    }
    if constexpr (!NEW) {
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(gave_up) != 0u) break;
    }
    // opaque: what the bodies below derive from the thread's number is not to be hoisted out of the loop, where twelve of
    // them would share the registers
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    auto run = [&](auto element, auto tile) {
      typedef decltype(element) E;
      constexpr int SHARED = NEW ? FRESH : FLAGGED;
      if (!a.trans_p && !a.trans_q) return small_tile<E, tile, true, false, false, SHARED>(a, t, v, tid, lds, c.patience, &gave_up);
      if (!a.trans_p) return small_tile<E, tile, true, false, true, SHARED>(a, t, v, tid, lds, c.patience, &gave_up);
      return small_tile<E, tile, true, true, true, SHARED>(a, t, v, tid, lds, c.patience, &gave_up);
    };
    bool whole;
    if (F32 && g.f32) { if constexpr (F32) whole = a.tile_m == 32 ? run(0.0f, IC<32>{}) : run(0.0f, IC<64>{}); }
    else whole = a.tile_m == 32 ? run(bf16_t{}, IC<32>{}) : run(bf16_t{}, IC<64>{});
    if constexpr (NEW) {
      // (the stores need not be waited for: the next tile may begin as soon as LDS has been read)
      if (!whole) break;
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wavefront's stores are where every die sees them
      __syncthreads();
      if (threadIdx.x == 0) device_store(c.flags + task, 1u);
    }
    if (step <= 0) {
      if (step == 0) ask();
      if (workgroups == 0) break;
      if (step < 0) { task = draw(); continue; }
    }
    task += step;
  }
  if (gave_up != 0u)
    for (int j = 0; j < kMaxMerged; ++j)
      for (int i = threadIdx.x; i < c.group[j].count; i += 512)
        __hip_atomic_fetch_or(const_cast<uint32_t*>(&c.step.scales[c.group[j].members[i]].status), kStatusIncomplete,
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

hipError_t launch_ns_small(GemmBatch& b, bool f32, bool wide, hipStream_t s) {
  if (b.n < 1 || b.n > kMaxMerged) return hipErrorInvalidValue;
  long long slots = 0;
  for (int g = 0; g < b.n; ++g) {
    const GemmArgs& a = b.a[g];
    if ((a.tile_m != 64 && a.tile_m != 128 && !(a.tile_m == 32 && wide)) || a.tile_n != a.tile_m || (a.trans_p && !a.trans_q)) return hipErrorInvalidValue;
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

// The chain kernel stands on device-scope accesses that are coherent between the dies by themselves, ns_matrix_kernel on 160 KB of
// LDS, as gfx950 has them.
bool device_is_gfx950() {
  // by device: 0 not asked, 1 no, 2 yes (a query that failed says nothing of the next one)
  static std::atomic<int> known[64];
  int dev = -1, major = 0, minor = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0) {
    const bool kept = dev < 64;
    if (const int k = kept ? known[dev].load(std::memory_order_relaxed) : 0) return k == 2;
    if (hipDeviceGetAttribute(&major, hipDeviceAttributeComputeCapabilityMajor, dev) == hipSuccess &&
        hipDeviceGetAttribute(&minor, hipDeviceAttributeComputeCapabilityMinor, dev) == hipSuccess) {
      const bool yes = major == 9 && minor == 5;
      if (kept) known[dev].store(yes ? 2 : 1, std::memory_order_relaxed);
      return yes;
    }
  }
  (void)hipGetLastError();
  return false;
}

hipError_t launch_ns_chain(const ChainArgs& c, int wgs, hipStream_t s) {
  if (c.ops < 1 || c.ops > kMaxChainOps || c.tasks < 1 || wgs < 1) return hipErrorInvalidValue;
  bool f32 = false;
  for (int j = 0; j < kMaxMerged; ++j) f32 = f32 || c.group[j].f32;
  auto* const kernel = c.fresh ? (f32 ? ns_chain_kernel<true, true> : ns_chain_kernel<false, true>)
                               : (f32 ? ns_chain_kernel<true, false> : ns_chain_kernel<false, false>);
  hipLaunchKernelGGL(kernel, dim3(wgs), dim3(512), 0, s, c);
  return hipGetLastError();
}

}  // namespace mona
