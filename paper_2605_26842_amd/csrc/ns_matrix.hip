// All Newton-Schulz iterations of one matrix in one workgroup, for matrices with a short side of at most 256.
//
// As single products such matrices are bound by everything but the multiplications: a K of 128 or 256 is a handful of K
// steps between a prologue and an epilogue as long as they are, S and B travel through memory, and every one of 15 launches
// ends in a partial round.  Here a workgroup takes one matrix through all its iterations.  With Y the p x q matrix (X, or
// X^T where X is tall), cut into panels of 128 of the long side:
//     S = sum over panels Y_j Y_j^T       in accumulators, then bf16 in LDS
//     B = b S + c S S                     operands from LDS, back to LDS, then as fragments into registers
//     Y_j <- a Y_j + B Y_j                a panel at a time, in place in LDS: its own E operand, written to memory from there
// Nothing is exchanged between workgroups, so there is nothing to wait for but the workgroup's own barriers.
//
// P = 128: B takes 32 registers, so the S of the next iteration is accumulated from every panel while it is in LDS, and up to four
// panels (q <= 512) stay there from the first iteration to the last.  P = 256: B takes 128 registers, S 128 accumulators, so
// they take turns, the squares lie over the panels, and every iteration reads X twice and writes it once.  Eight wavefronts, one workgroup per CU.
//
// Panels that do not stay in LDS come from a die's 4 MB of L2, 128 KB for each of its 32 workgroups, or from behind it.  X is renewed
// in place, which halves what the steps touch, and passes go to and fro.  Measured, us per step, between two buffers and one way ->
// in place, to and fro: 250 x 128 x 4000 1505 -> 1367, 300 x 128 x 1000 559 -> 503, 256 x 200 x 700 644 -> 620, 128 x 256 x 1024 572 -> 541,
// 256 x 256 x 256 258 -> 243.  It is the place that counts: in place but one way, 0.3 % slower to 0.5 % faster, although to
// and fro 53 instead of 46 % of the requests find their line in L2 (128 x 768 x 256 both ways; 60 instead of 58 % at 250 x 128 x 4000) and
// 8 % less comes from behind it.  Letting the second panel of a pass arrive while the first is multiplied gains nothing on top.
//
// P = 256: nobody reads the renewed panel in LDS, so it is not renewed there: each wavefront turns its own values into rows in 4 KB of its
// own and stores them while the other one of its SIMD multiplies, and the workgroup meets once a panel instead of three times.  Cycles a
// panel of 768 x 256, the wait for it / multiplying / renewing / storing: 1.1k / 3.0k / 4.8k / 0.95k before, 2.6k / 3.0k / 1.8k / 1.4k now; what
// is left of the wait is the way from behind L2.  us per step: 128 x 768 x 256 both ways 622 -> 611, 128 x 256 x 1024 532 -> 513, 115 x 256 x 512
// 289 -> 278, 256 x 256 x 256 246 -> 236.  W in pieces of 8 values whatever the length of its rows: 256 x 200 x 700 558 -> 503,
// 250 x 70 x 100 49 -> 46.
//
// Measured, us per step, products in launches (or chains) -> here: 128 x 768 x 256 both ways 831 -> 611, 250 x 70 x 100 170 -> 45,
// 256 x 256 x 256 440 -> 232, 300 x 128 x 128 202 -> 82, one 128 x 128 47 (a chain) -> 32.  A panel costs an iteration 2.2 to 3.3 us (P = 128; the
// kernel takes 67 us of 120 x 128 x 512 and 267 of 120 x 128 x 2048) or, in both passes together, 7.6 to 8.3 (P = 256; 208, 374 and 679 us of 120 x
// 256 x 512, 1024 and 2048; 215, 388 and 718 while all panels were renewed in LDS), of which the multiplications are 1 and 4: the wavefronts
// meet three times a panel (P = 128), and the vector instructions of the epilogue (2.5 an element) do not run beside matrix instructions.
//
// LDS: rows of 256 or 512 bytes, chunk c (16 bytes) of row r at c ^ swizzle(r): 16 consecutive rows hit 16 different
// chunks (row-major fragments, one ds_read_b128), four consecutive rows four different groups of 64 bytes (K-major ones, two
// ds_read_b64_tr_b16).  A direct load writes its 64 lanes one after the other, so it is told which chunk to fetch.
#include "ns_small_tile.h"

namespace mona {

namespace {

constexpr int kMatThreads = 512, kMatWaves = 8;
constexpr int kPanel = 128;          // of the long side

template <int P>
struct MatGeo {
  static constexpr bool kFused = P == 128;                     // S of the next iteration beside the apply
  static constexpr int PANEL = P * kPanel * 2, SQUARE = P * P * 2;
  static constexpr int RESIDENT = P == 128 ? 4 : 0;            // panels that may stay in LDS
  static constexpr int PANELS_AT = P == 128 ? SQUARE : 0;      // where the panels begin
  static constexpr int STAGING_AT = 2 * PANEL, STAGING = 4096; // P = 256: 32 rows of 128 bytes for each wavefront
  static constexpr int LDS = P == 128 ? SQUARE + RESIDENT * PANEL : STAGING_AT + kMatWaves * STAGING;
  static constexpr int GM = P / 64, GN = P / 128;              // 32 x 32 blocks of a wavefront in a P x P product (2 x 4 wavefronts)
  static constexpr int RB = P / 128, CB = 2;                   // in the apply (4 wavefronts along p, 2 along the panel)
  static constexpr int KS = P / 16;                            // products along p
};

__device__ __forceinline__ int swizzle(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

// ---- fragment reads: every block issues its reads and waits for them ---------------------------------------------
template <int ST>   // ST: bytes between blocks of 32 rows
__device__ __forceinline__ void read_rows(u32x4 (&a)[4], u32x4 (&b)[2], uint32_t pa, uint32_t pb) {
  asm volatile(
      "ds_read_b128 %0, %6\n\tds_read_b128 %4, %7\n\tds_read_b128 %1, %6 offset:%8\n\tds_read_b128 %5, %7 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%9\n\tds_read_b128 %3, %6 offset:%10\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1])
      : "v"(pa), "v"(pb), "n"(ST), "n"(2 * ST), "n"(3 * ST)
      : "memory");
}
template <int ST>
__device__ __forceinline__ void read_rows(u32x4 (&a)[2], u32x4 (&b)[1], uint32_t pa, uint32_t pb) {
  asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %2, %4\n\tds_read_b128 %1, %3 offset:%5\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0])
               : "v"(pa), "v"(pb), "n"(ST)
               : "memory");
}
struct Pair { u32x2 lo, hi; };       // K-major fragment: k 0..3 and k 4..7 of the lane's row
template <int OFF>
__device__ __forceinline__ void read_cols(Pair (&a)[4], Pair (&b)[2], const uint32_t (&al)[4], const uint32_t (&ah)[4],
                                          const uint32_t (&bl)[2], const uint32_t (&bh)[2]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %12 offset:%24\n\tds_read_b64_tr_b16 %1, %13 offset:%24\n\t"
      "ds_read_b64_tr_b16 %8, %20 offset:%24\n\tds_read_b64_tr_b16 %9, %21 offset:%24\n\t"
      "ds_read_b64_tr_b16 %2, %14 offset:%24\n\tds_read_b64_tr_b16 %3, %15 offset:%24\n\t"
      "ds_read_b64_tr_b16 %10, %22 offset:%24\n\tds_read_b64_tr_b16 %11, %23 offset:%24\n\t"
      "ds_read_b64_tr_b16 %4, %16 offset:%24\n\tds_read_b64_tr_b16 %5, %17 offset:%24\n\t"
      "ds_read_b64_tr_b16 %6, %18 offset:%24\n\tds_read_b64_tr_b16 %7, %19 offset:%24\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(a[0].lo), "=&v"(a[0].hi), "=&v"(a[1].lo), "=&v"(a[1].hi), "=&v"(a[2].lo), "=&v"(a[2].hi), "=&v"(a[3].lo),
        "=&v"(a[3].hi), "=&v"(b[0].lo), "=&v"(b[0].hi), "=&v"(b[1].lo), "=&v"(b[1].hi)
      : "v"(al[0]), "v"(ah[0]), "v"(al[1]), "v"(ah[1]), "v"(al[2]), "v"(ah[2]), "v"(al[3]), "v"(ah[3]), "v"(bl[0]), "v"(bh[0]),
        "v"(bl[1]), "v"(bh[1]), "n"(OFF)
      : "memory");
}
template <int OFF>
__device__ __forceinline__ void read_cols(Pair (&a)[2], Pair (&b)[1], const uint32_t (&al)[2], const uint32_t (&ah)[2],
                                          const uint32_t (&bl)[1], const uint32_t (&bh)[1]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %6 offset:%12\n\tds_read_b64_tr_b16 %1, %7 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %10 offset:%12\n\tds_read_b64_tr_b16 %5, %11 offset:%12\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%12\n\tds_read_b64_tr_b16 %3, %9 offset:%12\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(a[0].lo), "=&v"(a[0].hi), "=&v"(a[1].lo), "=&v"(a[1].hi), "=&v"(b[0].lo), "=&v"(b[0].hi)
      : "v"(al[0]), "v"(ah[0]), "v"(al[1]), "v"(ah[1]), "v"(bl[0]), "v"(bh[0]), "n"(OFF)
      : "memory");
}
// two K steps of two blocks
template <int OFF, int STEP>
__device__ __forceinline__ void read_cols_2(Pair (&a)[2], Pair (&b)[2], const uint32_t (&l)[2], const uint32_t (&h)[2]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%12\n\tds_read_b64_tr_b16 %1, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %2, %10 offset:%12\n\tds_read_b64_tr_b16 %3, %11 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %8 offset:%13\n\tds_read_b64_tr_b16 %5, %9 offset:%13\n\t"
      "ds_read_b64_tr_b16 %6, %10 offset:%13\n\tds_read_b64_tr_b16 %7, %11 offset:%13\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(a[0].lo), "=&v"(a[0].hi), "=&v"(a[1].lo), "=&v"(a[1].hi), "=&v"(b[0].lo), "=&v"(b[0].hi), "=&v"(b[1].lo),
        "=&v"(b[1].hi)
      : "v"(l[0]), "v"(h[0]), "v"(l[1]), "v"(h[1]), "n"(OFF), "n"(OFF + STEP)
      : "memory");
}
template <int ST>
__device__ __forceinline__ void read_rows_2(u32x4 (&a)[2], u32x4 (&b)[2], uint32_t p, uint32_t q) {
  asm volatile(
      "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%6\n\tds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:%6\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0]), "=&v"(b[1])
      : "v"(p), "v"(q), "n"(ST)
      : "memory");
}
__device__ __forceinline__ bf16x8 frag(const Pair& p) { return frag(p.lo, p.hi); }

// LDS traffic of this wavefront done, then all wavefronts; loads into LDS may be in flight (a fence would drain them)
__device__ __forceinline__ void meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));

// What the phases derive from the lane's number is computed anew in each of them, a few instructions: hoisted out of the loops
// it would take registers that the accumulators and B need.
struct Lane {
  int lane, frow, half, tx, nl;
  __device__ __forceinline__ Lane() {
    lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    frow = lane & 31; half = lane >> 5;
    tx = (lane & 15) >> 2; nl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  }
};

template <int P, bool TALL>
__device__ __forceinline__ void run_matrix(const StepDesc& st, const GroupDesc& g, int steps, int store_o, int member, char* lds) {
#pragma clang fp contract(off)
  typedef MatGeo<P> G;
  constexpr int CPR = TALL ? P / 8 : kPanel / 8;              // chunks to a row of a panel
  constexpr int PITCH = CPR * 16, SPITCH = P * 2;             // bytes to a row of a panel, of a square
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(MONA_AS3 const char*)lds;
  const int ld = g.cols_pad;
  const int panels = (TALL ? g.rows_pad : g.cols_pad) / kPanel;
  const bool resident = panels <= G::RESIDENT;
  const int64_t x_stride = (int64_t)g.rows_pad * g.cols_pad;
  bf16_t* const x0 = reinterpret_cast<bf16_t*>(g.x) + member * x_stride;
  // (O goes where products one by one would leave it)
  bf16_t* const out_at = (steps & 1) ? reinterpret_cast<bf16_t*>(g.x + g.x_step) + member * x_stride : x0;
  const int mi = g.members[member];
  const MatScale sc = st.scales[mi];
  const bool skip_w = (sc.status & 2u) != 0;
  void* const wptr = st.dyn[mi].w;
  const int w_is_bf16 = st.stat[mi].w_dtype;

  // A pass goes over the panels forwards or (back) backwards, i counts them as they come.  Where they do not stay in LDS, passes
  // alternate and X is renewed in place: the panels that the pass before had last are still in L2 then.
  auto panel = [&](int i, bool back) { return back ? panels - 1 - i : i; };
  auto buffer = [&](int i) { return (uint32_t)(G::PANELS_AT + (resident ? i : i & 1) * G::PANEL); };
  // requests the i-th panel of a pass: every wavefront a share of its chunks
  // (unit u of a panel is chunk u % CPR of row u / CPR as it stands in LDS; a thread's units are 512 apart, a multiple of
  // sixteen rows, so they share their swizzle and are `rows` rows apart in memory)
  constexpr int UNITS = G::PANEL / 16 / kMatThreads, ROWS = kMatThreads / CPR;
  static_assert(ROWS % 16 == 0, "the swizzle has a period of 16 rows");
  auto unit_at = [&](const Lane& L, int j) -> size_t {       // element of X that unit 0 of this thread holds
    const int u = wave * 64 + L.lane, row = u / CPR, c = (u % CPR) ^ swizzle(row);
    return TALL ? (size_t)(j * kPanel + row) * ld + c * 8 : (size_t)row * ld + j * kPanel + c * 8;
  };
  auto request = [&](int i_th, bool back) {
    char* const to = lds + buffer(i_th) + wave * 1024;
    const Lane L;
    const bf16_t* const from = x0 + unit_at(L, panel(i_th, back));
    static_for<UNITS>([&](auto i) {
      __builtin_amdgcn_global_load_lds((const MONA_AS1 void*)(from + (size_t)(i * ROWS) * ld),
                                       (MONA_AS3 void*)(to + i * kMatThreads * 16), 16, 0, 0);
    });
  };

  // ---- P x P products: wavefront (wm, wn) has rows wm P / 2 .., columns wn P / 4 .. ----
  const int wm = wave >> 2, wn = wave & 3;
  const int ga = wm * (P / 2), gb = wn * (P / 4);             // first rows of the two operands
  f32x16 acc[G::GM][G::GN];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < G::GM; ++i)
#pragma unroll
      for (int j = 0; j < G::GN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  };
  // (roles swapped: a lane holds one row and, per group of four registers, four consecutive columns)
  auto multiply = [&](auto&& fa, auto&& fb) {
    static_for<G::GM>([&](auto i) {
      static_for<G::GN>([&](auto j) { acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb(j), fa(i), acc[i][j], 0, 0, 0); });
    });
  };
  // S += Y_j Y_j^T from the panel at `at`
  auto gram = [&](uint32_t at) {
    const uint32_t base = lds0 + at;
    const Lane L;
    if constexpr (!TALL) {
      const uint32_t pa = base + (ga + L.frow) * PITCH + ((L.half ^ swizzle(L.frow)) << 4);
      const uint32_t pb = base + (gb + L.frow) * PITCH + ((L.half ^ swizzle(L.frow)) << 4);
      static_for<kPanel / 16>([&](auto ks) {
        u32x4 a[G::GM], b[G::GN];
        read_rows<32 * PITCH>(a, b, pa ^ (ks << 5), pb ^ (ks << 5));
        multiply([&](auto i) { return frag(a[i]); }, [&](auto j) { return frag(b[j]); });
      });
    } else {
      uint32_t al[G::GM], ah[G::GM], bl[G::GN], bh[G::GN];
      auto where = [&](int first, int hi) -> uint32_t {
        const int row = 8 * L.half + L.tx + 4 * hi;
        return base + row * PITCH + ((((first + L.nl) >> 3) ^ swizzle(row)) << 4) + (L.nl & 7) * 2;
      };
      static_for<G::GM>([&](auto i) { al[i] = where(ga + i * 32, 0); ah[i] = where(ga + i * 32, 1); });
      static_for<G::GN>([&](auto j) { bl[j] = where(gb + j * 32, 0); bh[j] = where(gb + j * 32, 1); });
      static_for<kPanel / 16>([&](auto ks) {
        Pair a[G::GM], b[G::GN];
        read_cols<ks * 16 * PITCH>(a, b, al, ah, bl, bh);
        multiply([&](auto i) { return frag(a[i]); }, [&](auto j) { return frag(b[j]); });
      });
    }
  };
  // The four values of register group v of block (i, j) are 8 bytes of a square, at (square_at ^ xor_at(j, v)) + i 32 SPITCH: the
  // blocks and groups differ in bits of the chunk's number that are zero in the first one's, so one address serves all.
  auto square_at = [&](const Lane& L) -> uint32_t {
    return (ga + L.frow) * SPITCH + (((gb >> 3) ^ swizzle(L.frow)) << 4) + L.half * 8;
  };
  auto xor_at = [](int block, int v) -> uint32_t { return block << 6 | v << 4; };
  auto at8 = [&](uint32_t where) -> u32x2& { return *reinterpret_cast<u32x2*>(lds + where); };
  auto pack = [](float w, float x, float y, float z) {
    const bf16x4 r = {(bf16_t)w, (bf16_t)x, (bf16_t)y, (bf16_t)z};
    return __builtin_bit_cast(u32x2, r);
  };

  // W <- (1 - eta lambda) W - eta gamma O, O as stored in the working precision, of 8 values of a row
  auto update = [&](const bf16x8& o, int wr, int wc) {
    if (wr >= g.m || wc >= g.n) return;
    const size_t wi = (size_t)wr * g.n + wc;
    // (rows of any length: pieces are aligned like their elements, which the compiler makes one access of all the same)
    auto row = [&](auto* const p) {
      typedef std::remove_pointer_t<decltype(p + 0)> W;
      auto renewed = [&](W w, int e) { return (W)fmaf(st.w_keep, (float)w, -(g.o_scale * (float)o[e])); };
      auto some = [&](auto first, auto count) {
        constexpr int F = decltype(first)::value, N = decltype(count)::value;
        typedef W vec __attribute__((ext_vector_type(N)));
        typedef vec piece __attribute__((aligned(sizeof(W))));
        piece* const at = reinterpret_cast<piece*>(p + F);
        vec w = *at;
#pragma unroll
        for (int e = 0; e < N; ++e) w[e] = renewed(w[e], F + e);
        *at = w;
      };
      if (sizeof(W) == 2 && wc + 8 <= g.n) {
        if constexpr (sizeof(W) == 2) some(IC<0>{}, IC<8>{});
        return;
      }
      static_for<2>([&](auto h) {
        if (wc + 4 * h + 4 <= g.n) { some(IC<4 * h>{}, IC<4>{}); return; }
#pragma unroll
        for (int e = 4 * h; e < 4 * h + 4; ++e)
          if (wc + e < g.n) p[e] = renewed(p[e], e);
      });
    };
    if (w_is_bf16) row(static_cast<bf16_t*>(wptr) + wi); else row(static_cast<float*>(wptr) + wi);
  };

  // ---- apply: wavefront (rg, cg) has rows rg P / 4 .., columns 64 cg .. of the panel ----
  const int rg = wave >> 1, cg = wave & 1;
  const int pr = rg * (P / 4);

  request(0, false);
  if (panels > 1) request(1, false);
  if (resident)
    for (int i = 2; i < panels; ++i) request(i, false);
  for (int t = 0; t < steps; ++t) {
    const bool first = t == 0, last = t + 1 == steps;
    // direction of the apply: against the pass before it (P = 256: the S of this iteration, always forwards)
    const bool back = !resident && (!G::kFused || (t & 1) == 0);
    bf16_t* const to = last ? out_at : x0;
    // the loads of the panel (in issue order before the `later` newest accesses) have landed for every wavefront
    auto arrive = [&](auto later) { MONA_WAIT_VM(later); meet(); };
    if (first || !G::kFused) {
      clear();
      for (int i = 0; i < panels; ++i) {
        arrive(IC<0>{});
        if (i >= 1 && i + 1 < panels && !resident) request(i + 1, false);
        gram(buffer(i));
      }
    }
    // ---- S and B ----
    if constexpr (!G::kFused) meet();            // the squares lie over the panels
    {
      const Lane L;
      const uint32_t sq = square_at(L);
      if (first) {
        const float s = sc.inv2;
        static_for<G::GM>([&](auto i) {
          static_for<G::GN>([&](auto j) { static_for<16>([&](auto e) { acc[i][j][(int)e] *= s; }); });
        });
      }
      static_for<G::GM>([&](auto i) {
        static_for<G::GN>([&](auto j) {
          static_for<4>([&](auto v) {
            at8((sq ^ xor_at(j, v)) + i * 32 * SPITCH) =
                pack(acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]);
          });
        });
      });
    }
    meet();
    if (G::kFused && first && !resident) {       // the first pass has been over all panels
      request(0, back);
      request(1, back);
    }
    clear();
    {
      const Lane L;
      const uint32_t pa = lds0 + (ga + L.frow) * SPITCH + ((L.half ^ swizzle(L.frow)) << 4);
      const uint32_t pb = lds0 + (gb + L.frow) * SPITCH + ((L.half ^ swizzle(L.frow)) << 4);
      static_for<G::KS>([&](auto ks) {
        u32x4 a[G::GM], b[G::GN];
        read_rows<32 * SPITCH>(a, b, pa ^ (ks << 5), pb ^ (ks << 5));
        multiply([&](auto i) { return frag(a[i]); }, [&](auto j) { return frag(b[j]); });
      });
    }
    {
      const Lane L;
      const uint32_t sq = square_at(L);
      u32x2 out[G::GM][G::GN][4];
      static_for<G::GM>([&](auto i) {
        static_for<G::GN>([&](auto j) {
          static_for<4>([&](auto v) {
            const bf16x4 e = __builtin_bit_cast(bf16x4, at8((sq ^ xor_at(j, v)) + i * 32 * SPITCH));
            auto poly = [&](float x, bf16_t y) { return fmaf(st.ns_c, x, st.ns_b * (float)y); };
            out[i][j][v] = pack(poly(acc[i][j][4 * v], e.x), poly(acc[i][j][4 * v + 1], e.y), poly(acc[i][j][4 * v + 2], e.z),
                                poly(acc[i][j][4 * v + 3], e.w));
          });
          asm volatile("" ::: "memory");         // a block's values at a time: there is no room for those of all blocks
        });
      });
      meet();
      static_for<G::GM>([&](auto i) {
        static_for<G::GN>([&](auto j) {
          static_for<4>([&](auto v) { at8((sq ^ xor_at(j, v)) + i * 32 * SPITCH) = out[i][j][v]; });
        });
      });
    }
    meet();
    u32x4 B[G::RB][G::KS];
    {
      const Lane L;
      const char* const p = lds + (pr + L.frow) * SPITCH;
      static_for<G::RB>([&](auto i) {
        static_for<G::KS>([&](auto ks) {
          B[i][ks] = *reinterpret_cast<const u32x4*>(p + i * 32 * SPITCH + (((2 * ks + L.half) ^ swizzle(L.frow)) << 4));
        });
      });
    }
    if constexpr (!G::kFused) {
      meet();                                    // every wavefront has its B
      request(0, back);
      if (panels > 1) request(1, back);
    }
    if (G::kFused) clear();
    // ---- Y_j <- a Y_j + B Y_j ----
    for (int i_th = 0; i_th < panels; ++i_th) {
      const uint32_t at = buffer(i_th);
      const int j = panel(i_th, back);
      // (the stores of the panel before may still be on their way)
      if (i_th > 0 && !last && !resident) arrive(IC<UNITS>{}); else arrive(IC<0>{});
      if (i_th >= 1 && i_th + 1 < panels && !resident) request(i_th + 1, back);
      f32x16 y[G::RB][G::CB];
#pragma unroll
      for (int i = 0; i < G::RB; ++i)
#pragma unroll
        for (int c = 0; c < G::CB; ++c)
#pragma unroll
          for (int e = 0; e < 16; ++e) y[i][c][e] = 0.0f;
      // wide: a lane gets one row of p and consecutive columns; tall: one row of the panel and consecutive values of p
      auto step = [&](auto ks, auto&& f) {
        static_for<G::RB>([&](auto i) {
          static_for<G::CB>([&](auto c) {
            if constexpr (!TALL) y[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f(c), frag(B[i][ks]), y[i][c], 0, 0, 0);
            else y[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(B[i][ks]), f(c), y[i][c], 0, 0, 0);
          });
        });
      };
      const Lane L;
      if constexpr (!TALL) {
        uint32_t l[2], h[2];
        static_for<2>([&](auto c) {
          auto where = [&](int hi) -> uint32_t {
            const int row = 8 * L.half + L.tx + 4 * hi;
            return lds0 + at + row * PITCH + (((cg * 8 + c * 4 + (L.nl >> 3)) ^ swizzle(row)) << 4) + (L.nl & 7) * 2;
          };
          l[c] = where(0); h[c] = where(1);
        });
        static_for<G::KS / 2>([&](auto k2) {
          Pair a[2], b[2];
          read_cols_2<k2 * 32 * PITCH, 16 * PITCH>(a, b, l, h);
          step(IC<2 * k2>{}, [&](auto c) { return frag(a[c]); });
          step(IC<2 * k2 + 1>{}, [&](auto c) { return frag(b[c]); });
        });
      } else {
        const uint32_t p = lds0 + at + (cg * 64 + L.frow) * PITCH + ((L.half ^ swizzle(L.frow)) << 4);
        static_for<G::KS / 2>([&](auto k2) {
          u32x4 a[2], b[2];
          read_rows_2<32 * PITCH>(a, b, p ^ (k2 << 6), p ^ ((2 * k2 + 1) << 5));
          step(IC<2 * k2>{}, [&](auto c) { return frag(a[c]); });
          step(IC<2 * k2 + 1>{}, [&](auto c) { return frag(b[c]); });
        });
      }
      // the panel's own values, then the new ones in their place (addresses as in the squares)
      const Lane L2;
      const int row0 = TALL ? cg * 64 + L2.frow : pr + L2.frow, col0 = TALL ? pr : cg * 64;
      const uint32_t pan = at + row0 * PITCH + (((col0 >> 3) ^ swizzle(L2.frow)) << 4) + L2.half * 8;
      auto panel8 = [&](int i, int c, int v) -> u32x2& {
        return TALL ? at8((pan ^ xor_at(i, v)) + c * 32 * PITCH) : at8((pan ^ xor_at(c, v)) + i * 32 * PITCH);
      };
      u32x2 out[G::RB][G::CB][4];
      // The scale of the unscaled copy enters behind the sum, and every rounding is that of the large-tile kernel (at P = 256 these
      // are its bits).  In B and in a instead it rounds B in other places, which moves W by 2e-3 of its norm in a step.  (A
      // block's own values are read in front of the branch: read in both arms they cost 1 % of a step at P = 256.)
      const float post = first ? sc.inv : 1.0f, ce = post * st.ns_a;
      static_for<G::RB>([&](auto i) {
        static_for<G::CB>([&](auto c) {
          bf16x4 own[4];
          static_for<4>([&](auto v) { own[v] = __builtin_bit_cast(bf16x4, panel8(i, c, v)); });
          auto renew = [&](auto unit) {
            auto value = [&](bf16_t x, float sum) {
              return unit ? fmaf(ce, (float)x, sum) : fmaf(post, sum, ce * (float)x);
            };
            static_for<4>([&](auto v) {
              out[i][c][v] = pack(value(own[v].x, y[i][c][4 * v]), value(own[v].y, y[i][c][4 * v + 1]),
                                  value(own[v].z, y[i][c][4 * v + 2]), value(own[v].w, y[i][c][4 * v + 3]));
            });
          };
          if (post == 1.0f) renew(IC<1>{}); else renew(IC<0>{});
          asm volatile("" ::: "memory");
        });
      });
      if constexpr (G::kFused) {
        meet();
        static_for<G::RB>([&](auto i) {
          static_for<G::CB>([&](auto c) {
            static_for<4>([&](auto v) { panel8(i, c, v) = out[i][c][v]; });
          });
        });
        meet();
        // to memory, 16 bytes a lane along the rows (between iterations resident panels stay where they are)
        const char* const unit = lds + at + (wave * 64 + L2.lane) * 16;
        if (last ? store_o != 0 : !resident) {
          bf16_t* const p = to + unit_at(L2, j);
          static_for<UNITS>([&](auto i) {
            *reinterpret_cast<u32x4*>(p + (size_t)(i * ROWS) * ld) = *reinterpret_cast<const u32x4*>(unit + i * kMatThreads * 16);
          });
        }
        if (last && !skip_w) {
          static_for<UNITS>([&](auto i) {
            const int u = i * kMatThreads + wave * 64 + L2.lane, row = u / CPR, c = (u % CPR) ^ swizzle(row);
            update(__builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(unit + i * kMatThreads * 16)),
                   TALL ? j * kPanel + row : row, TALL ? c * 8 : j * kPanel + c * 8);
          });
        }
      } else {
        // Nobody reads the new values here, so the panel is left as it is and the wavefronts need not meet: each turns its own into rows
        // in a place of its own, 32 rows of 64 values at a time (chunk c of row r at c ^ (r mod 8)), and stores them, 8 rows of 128
        // bytes to an instruction, while the other one of its SIMD multiplies.
        char* const mine = lds + G::STAGING_AT + wave * G::STAGING;
        const int first_row = TALL ? j * kPanel + cg * 64 : pr, first_col = TALL ? pr : j * kPanel + cg * 64;
        static_for<2>([&](auto rb) {
          static_for<2>([&](auto cb) {
            static_for<4>([&](auto v) {
              const int chunk = (4 * cb + v) ^ (L2.frow & 7);
              *reinterpret_cast<u32x2*>(mine + L2.frow * 128 + chunk * 16 + L2.half * 8) = TALL ? out[cb][rb][v] : out[rb][cb][v];
            });
          });
          // (other lanes of the wavefront wrote what is read here; its LDS accesses keep the order they stand in)
          asm volatile("" ::: "memory");
          const int r8 = L2.lane >> 3, c8 = L2.lane & 7;
          u32x4 x[4];
          static_for<4>([&](auto k) { x[k] = *reinterpret_cast<const u32x4*>(mine + (8 * k + r8) * 128 + ((c8 ^ r8) << 4)); });
          asm volatile("" ::: "memory");
          const int row = first_row + rb * 32 + r8, col = first_col + c8 * 8;
          bf16_t* const p = to + (size_t)row * ld + col;
          if (!last || store_o) static_for<4>([&](auto k) { *reinterpret_cast<u32x4*>(p + (size_t)(8 * k) * ld) = x[k]; });
          if (last && !skip_w) static_for<4>([&](auto k) { update(__builtin_bit_cast(bf16x8, x[k]), row + 8 * k, col); });
        });
      }
      if (G::kFused && !last) gram(at);
    }
    if (!last && !resident) {
      MONA_WAIT_VM(0);                           // this wavefront's part of the new X is in memory
      meet();
      const bool next = G::kFused && !back;
      request(0, next);
      if (panels > 1) request(1, next);
    }
  }
}

// One workgroup per matrix; group i of the launch has the workgroups up to end[i].
__global__ __launch_bounds__(kMatThreads) void ns_matrix_kernel(const MatrixBatch b) {
  constexpr int LDS = MatGeo<128>::LDS > MatGeo<256>::LDS ? MatGeo<128>::LDS : MatGeo<256>::LDS;
  static_assert(LDS <= 160 * 1024, "LDS of one CU");
  __shared__ __attribute__((aligned(512))) char lds[LDS];
  int i = 0;
  while (i + 1 < b.n && (int)blockIdx.x >= b.end[i]) ++i;
  const int member = (int)blockIdx.x - (i > 0 ? b.end[i - 1] : 0);
  const GroupDesc& g = b.group[i];
  const int p = g.tall ? g.cols_pad : g.rows_pad;
  if (p == 128) {
    if (g.tall) run_matrix<128, true>(b.step, g, b.steps, b.store_o, member, lds);
    else run_matrix<128, false>(b.step, g, b.steps, b.store_o, member, lds);
  } else {
    if (g.tall) run_matrix<256, true>(b.step, g, b.steps, b.store_o, member, lds);
    else run_matrix<256, false>(b.step, g, b.steps, b.store_o, member, lds);
  }
}

}  // namespace

hipError_t launch_ns_matrix(const MatrixBatch& b, hipStream_t s) {
  if (b.n < 1 || b.n > kMaxMerged || b.steps < 1) return hipErrorInvalidValue;
  for (int i = 0; i < b.n; ++i) {
    const GroupDesc& g = b.group[i];
    const int p = g.tall ? g.cols_pad : g.rows_pad, q = g.tall ? g.rows_pad : g.cols_pad;
    if (g.f32 || (p != 128 && p != 256) || q % kPanel || b.end[i] - (i > 0 ? b.end[i - 1] : 0) != g.count) return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(ns_matrix_kernel, dim3((unsigned)b.end[b.n - 1]), dim3(kMatThreads), 0, s, b);
  return hipGetLastError();
}

}  // namespace mona
