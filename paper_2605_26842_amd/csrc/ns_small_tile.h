// What the kernels that give a tile to a workgroup share: what the epilogue knows of its matrix, the accesses to
// arrays that other workgroups of the same launch use too, and the epilogue itself.
#pragma once
#include "ns_tile.h"

namespace mona {
namespace {

template <typename E> struct Chunk;           // 16 bytes of E
template <> struct Chunk<bf16_t> { static constexpr int N = 8; typedef bf16x8 vec; };
template <> struct Chunk<float> { static constexpr int N = 4; typedef f32x4 vec; };

__device__ __forceinline__ bf16x8 frag(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ bf16x8 frag(u32x2 lo, u32x2 hi) {
  const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
  return __builtin_bit_cast(bf16x8, v);
}
// Who else uses the arrays of a tile: earlier and later launches only; other workgroups of the same launch, whose flags have been
// waited for; or these without flags, through arrays that held kUnwritten in every place before (FRESH).
enum Sharing : int { OWN_LAUNCH = 0, FLAGGED = 1, FRESH = 2 };

// Whether any 16 or 32 bits of what a lane has read are those of a place that has not been written.  16 bits each in bf16, because
// a K-major fragment holds values of two rows in one register.
template <typename E>
struct Unwritten {
  uint32_t most = 0, most_low = 0;
  __device__ __forceinline__ void see(uint32_t v) {
    most = most > v ? most : v;
    if constexpr (sizeof(E) == 2) { const uint32_t low = v << 16; most_low = most_low > low ? most_low : low; }
  }
  __device__ __forceinline__ void see(float v) { see(__builtin_bit_cast(uint32_t, v)); }
  __device__ __forceinline__ void see(const u32x2& v) { see(v.x); see(v.y); }
  __device__ __forceinline__ void see(const u32x4& v) { see(v.x); see(v.y); see(v.z); see(v.w); }
  __device__ __forceinline__ void see(const f32x4& v) { see(__builtin_bit_cast(u32x4, v)); }
  __device__ __forceinline__ bool any() const {
    if constexpr (sizeof(E) == 4) return most == kUnwritten;
    else return (most > most_low ? most : most_low) >= 0xffff0000u;
  }
  // (a NaN that would look like it becomes another)
  static __device__ __forceinline__ uint32_t avoid(uint32_t v) {
    if constexpr (sizeof(E) == 4) return v < 0xfffffffeu ? v : 0xfffffffeu;
    if (v >= 0xffff0000u) v &= 0xfffeffffu;
    if ((v & 0xffffu) == 0xffffu) v &= 0xfffffffeu;
    return v;
  }
};

// 16 bytes of such an array (SHARED: coherent across the dies at device scope, without any cache being written back or
// invalidated).  `bytes` from the start of the array, which is wavefront-uniform and smaller than 4 GB where it is shared.
constexpr int kDeviceScope = 16;   // sc1
template <typename E, int SHARED>
struct Array {
  char* p;
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Array(void* base, int64_t size) : p(static_cast<char*>(base)) {
    if constexpr (SHARED) r = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)(uint32_t)size, 0x00020000);
  }
  template <typename V> __device__ __forceinline__ V load(size_t bytes) const {
    if constexpr (SHARED) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(uint32_t)bytes, 0, kDeviceScope));
    else return *reinterpret_cast<const V*>(p + bytes);
  }
  template <typename V> __device__ __forceinline__ void store(size_t bytes, V v) const {
    if constexpr (SHARED) {
      u32x4 u = __builtin_bit_cast(u32x4, v);
      if constexpr (SHARED == FRESH) {
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = Unwritten<E>::avoid(u[i]);
      }
      __builtin_amdgcn_raw_buffer_store_b128(u, r, (int)(uint32_t)bytes, 0, kDeviceScope);
    } else {
      *reinterpret_cast<V*>(p + bytes) = v;
    }
  }
  // the same for two elements: 4 bytes in bf16, 8 in fp32
  typedef E pair_t __attribute__((ext_vector_type(2)));
  __device__ __forceinline__ pair_t load2(size_t bytes) const {
    if constexpr (!SHARED) return *reinterpret_cast<const pair_t*>(p + bytes);
    else if constexpr (sizeof(E) == 2)
      return __builtin_bit_cast(pair_t, __builtin_amdgcn_raw_buffer_load_b32(r, (int)(uint32_t)bytes, 0, kDeviceScope));
    else return __builtin_bit_cast(pair_t, __builtin_amdgcn_raw_buffer_load_b64(r, (int)(uint32_t)bytes, 0, kDeviceScope));
  }
  __device__ __forceinline__ void store2(size_t bytes, pair_t v) const {
    if constexpr (!SHARED) {
      *reinterpret_cast<pair_t*>(p + bytes) = v;
    } else if constexpr (sizeof(E) == 2) {
      uint32_t u = __builtin_bit_cast(uint32_t, v);
      if constexpr (SHARED == FRESH) u = Unwritten<E>::avoid(u);
      __builtin_amdgcn_raw_buffer_store_b32(u, r, (int)(uint32_t)bytes, 0, kDeviceScope);
    } else {
      u32x2 u = __builtin_bit_cast(u32x2, v);
      if constexpr (SHARED == FRESH) { u.x = Unwritten<E>::avoid(u.x); u.y = Unwritten<E>::avoid(u.y); }
      __builtin_amdgcn_raw_buffer_store_b64(u, r, (int)(uint32_t)bytes, 0, kDeviceScope);
    }
  }
};

// What the epilogue of a tile needs to know of its matrix: two or three loads that depend on each other, made before the
// first operand is waited for.
struct TileMatrix {
  float post;
  bool skip_w;
  int m, n, w_dtype;
  void* w;
};
__device__ __forceinline__ TileMatrix look_up(const GemmArgs& a, const TileId& t) {
  TileMatrix v = {1.0f, true, 0, 0, 0, nullptr};
  if (a.post == POST_NONE && a.epilogue != EPI_UPDATE) return v;
  const int mi = a.members[t.mat];
  if (a.post == POST_INV) v.post = a.scales[mi].inv;
  else if (a.post == POST_INV2) v.post = a.scales[mi].inv2;
  if (a.epilogue == EPI_UPDATE) {
    const MatStatic& ms = a.stat[mi];
    v.m = ms.m; v.n = ms.n; v.w_dtype = ms.w_dtype;
    v.w = a.dyn[mi].w;
    v.skip_w = (a.scales[mi].status & 2u) != 0;
  }
  return v;
}

// Chunks of 16 bytes that make up a tile, row by row, and how many a thread has of them.
template <typename E, int T, int THREADS>
struct TileChunks {
  static constexpr int CH = Chunk<E>::N, PER_ROW = T / CH, ALL = T * T / CH, PER_LANE = ALL / THREADS;
  static_assert(ALL % THREADS == 0, "as many for every thread");
};

// the E operand of this thread's chunks
template <typename E, int T, int THREADS, int SHARED>
__device__ __forceinline__ void load_e(const GemmArgs& a, const TileId& t, int tid,
                                       typename Chunk<E>::vec (&ev)[TileChunks<E, T, THREADS>::PER_LANE]) {
  typedef TileChunks<E, T, THREADS> N;
  if (!a.E) return;
  const Array<E, SHARED> Eb(static_cast<E*>(const_cast<void*>(a.E)) + (size_t)t.mat * a.strideE, a.strideE * sizeof(E));
#pragma unroll
  for (int u = 0; u < N::PER_LANE; ++u) {
    const int idx = u * THREADS + tid;
    ev[u] = Eb.template load<typename Chunk<E>::vec>(
        ((size_t)(t.ti * T + idx / N::PER_ROW) * a.lde + t.tj * T + (idx % N::PER_ROW) * N::CH) * sizeof(E));
  }
}

// floats per row of the staged tile (+4: rows on different banks)
constexpr int staged_ld(int T) { return T + 4; }

// The epilogue of a tile whose accumulators stand in LDS as SHARES tiles of T x staged_ld(T) floats that add up to the
// product: every global access is a 16-byte piece of a row.
template <typename E, int T, int SHARES, int THREADS, int SHARED>
__device__ __forceinline__ void finish_tile(const GemmArgs& a, const TileId& t, const TileMatrix& v, int tid,
                                            typename Chunk<E>::vec (&ev)[TileChunks<E, T, THREADS>::PER_LANE], float* sum) {
  // every contraction is written out: a product comes out the same, bit for bit, in whichever kernel it runs
#pragma clang fp contract(off)
  typedef TileChunks<E, T, THREADS> N;
  typedef typename Chunk<E>::vec vec_t;
  constexpr int ES = sizeof(E), CH = N::CH, CPR = N::PER_ROW, U = N::PER_LANE, LDW = staged_ld(T);
  const int lane = tid & 63, wave = tid >> 6;
  const int m0 = t.ti * T, n0 = t.tj * T;
  const bool mirror = a.symmetric && t.ti != t.tj, update = a.epilogue == EPI_UPDATE, skip_w = v.skip_w;
  const int wm_real = v.m, wn_real = v.n, w_is_bf16 = v.w_dtype;
  void* const wptr = v.w;
  const float post = v.post;
  const Array<E, SHARED> C(static_cast<E*>(a.C) + (size_t)t.mat * a.strideC, a.strideC * ES);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int idx = u * THREADS + tid;
    const int r = idx / CPR, ch = idx % CPR;
    const int grow = m0 + r, gcol = n0 + ch * CH;
    float val[CH];
#pragma unroll
    for (int e = 0; e < CH; ++e) val[e] = 0.0f;
    static_for<SHARES>([&](auto s) {
      static_for<CH / 4>([&](auto q) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(sum + (s * T + r) * LDW + ch * CH + q * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) val[q * 4 + e] = s == 0 ? p[e] : val[q * 4 + e] + p[e];
      });
    });
    if (a.E) {
#pragma unroll
      for (int e = 0; e < CH; ++e) val[e] = post * fmaf(a.alpha, val[e], a.beta * (float)ev[u][e]);
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
    if (!update || a.store_out) C.store(((size_t)grow * a.ldc + gcol) * ES, ov);
    if (mirror) {
      // the rounded result, for the transposed pass below, in place of the share this lane alone has read
      static_for<CH / 4>([&](auto q) {
        const f32x4 p = {(float)ov[q * 4 + 0], (float)ov[q * 4 + 1], (float)ov[q * 4 + 2], (float)ov[q * 4 + 3]};
        *reinterpret_cast<f32x4*>(sum + r * LDW + ch * CH + q * 4) = p;
      });
    }
    if (update && !skip_w && grow < wm_real) {
      // W <- (1 - eta lambda) W - eta gamma O, O as stored in the working precision
      const size_t wi = (size_t)grow * wn_real + gcol;
      if (gcol + CH <= wn_real) {
        // (rows of any length: pieces are aligned like their elements, which the compiler makes one access of all the same)
        if (w_is_bf16) {
          typedef bf16_t wv_t __attribute__((ext_vector_type(CH)));
          typedef wv_t piece __attribute__((aligned(2)));
          piece* wp = reinterpret_cast<piece*>(static_cast<bf16_t*>(wptr) + wi);
          wv_t w = *wp;
#pragma unroll
          for (int e = 0; e < CH; ++e) w[e] = (bf16_t)fmaf(a.w_keep, (float)w[e], -(a.o_scale * (float)ov[e]));
          *wp = w;
        } else {
          typedef f32x4 piece __attribute__((aligned(4)));
          piece* wp = reinterpret_cast<piece*>(static_cast<float*>(wptr) + wi);
          static_for<CH / 4>([&](auto q) {
            f32x4 w = wp[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = fmaf(a.w_keep, w[e], -(a.o_scale * (float)ov[q * 4 + e]));
            wp[q] = w;
          });
        }
      } else {
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          if (gcol + e < wn_real) {
            if (w_is_bf16) {
              bf16_t* w = static_cast<bf16_t*>(wptr) + wi + e;
              *w = (bf16_t)fmaf(a.w_keep, (float)*w, -(a.o_scale * (float)ov[e]));
            } else {
              float* w = static_cast<float*>(wptr) + wi + e;
              *w = fmaf(a.w_keep, *w, -(a.o_scale * (float)ov[e]));
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
      const int grp = u * (THREADS / 64) + wave;
      const int c = (grp % (T / 8)) * 8 + (lane >> 3), rc = (grp / (T / 8)) * 8 + (lane & 7);
      vec_t ov;
#pragma unroll
      for (int e = 0; e < CH; ++e) ov[e] = (E)sum[(rc * CH + e) * LDW + c];
      C.store(((size_t)(n0 + c) * a.ldc + m0 + rc * CH) * ES, ov);
    }
  }
}

// The same, with the E operand requested when the tile begins.
template <typename E, int T, int SHARES, int THREADS, int SHARED>
struct FinishTile {
  typedef TileChunks<E, T, THREADS> N;
  typename Chunk<E>::vec ev[N::PER_LANE];
  int tid;
  __device__ __forceinline__ FinishTile(const GemmArgs& a, const TileId& t, int tid_) : ev{}, tid(tid_) { load_e(a, t); }
  __device__ __forceinline__ void load_e(const GemmArgs& a, const TileId& t) { mona::load_e<E, T, THREADS, SHARED>(a, t, tid, ev); }
  __device__ __forceinline__ void see(Unwritten<E>& u) const {
#pragma unroll
    for (int c = 0; c < N::PER_LANE; ++c) u.see(__builtin_bit_cast(u32x4, ev[c]));
  }
  __device__ __forceinline__ void run(const GemmArgs& a, const TileId& t, const TileMatrix& v, float* sum) {
    finish_tile<E, T, SHARES, THREADS, SHARED>(a, t, v, tid, ev, sum);
  }
};

// The epilogue of a 32 x 32 tile whose accumulators stand in LDS as SHARES tiles, for 512 threads: a thread has two neighbours of
// a row and, where the tile is mirrored, two neighbours of a row of the mirrored tile, which it adds up for itself (the same sums in
// the same order, so the same bits).  Nothing is handed on between threads, and what does not depend on the product (E, W) is
// requested before it is waited for.
template <typename E, int SHARES, int SHARED>
struct Finish32 {
  typedef Array<E, SHARED> A;
  typedef typename A::pair_t pair_t;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  static constexpr int T = 32, LDW = staged_ld(T);
  int r, c;                     // row, first column
  pair_t e, em;                 // E at (r, c) of the tile, and of the mirrored one
  f32x2 w;
  bool mirror, update, w_pair;

  __device__ __forceinline__ Finish32(const GemmArgs& a, const TileId& t, const TileMatrix& v, int tid)
      : r(tid >> 4), c((tid & 15) * 2), e{}, em{}, w{0.0f, 0.0f} {
    mirror = a.symmetric && t.ti != t.tj;
    load_e(a, t);
    const int grow = t.ti * T + r, gcol = t.tj * T + c;
    update = a.epilogue == EPI_UPDATE && !v.skip_w && grow < v.m;
    w_pair = (v.n & 1) == 0 && gcol < v.n;           // (rows of W are whole pairs)
    if (update) {
      const size_t wi = (size_t)grow * v.n + gcol;
      if (w_pair) {
        if (v.w_dtype) {
          typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
          const bf16x2 x = *reinterpret_cast<const bf16x2*>(static_cast<const bf16_t*>(v.w) + wi);
          w = f32x2{(float)x.x, (float)x.y};
        } else {
          w = *reinterpret_cast<const f32x2*>(static_cast<const float*>(v.w) + wi);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (gcol + i < v.n) w[i] = v.w_dtype ? (float)static_cast<const bf16_t*>(v.w)[wi + i] : static_cast<const float*>(v.w)[wi + i];
      }
    }
  }
  __device__ __forceinline__ void load_e(const GemmArgs& a, const TileId& t) {
    if (!a.E) return;
    const A Eb(static_cast<E*>(const_cast<void*>(a.E)) + (size_t)t.mat * a.strideE, a.strideE * sizeof(E));
    e = Eb.load2(((size_t)(t.ti * T + r) * a.lde + t.tj * T + c) * sizeof(E));
    if (mirror) em = Eb.load2(((size_t)(t.tj * T + r) * a.lde + t.ti * T + c) * sizeof(E));
  }
  __device__ __forceinline__ void see(Unwritten<E>& u) const {
    if constexpr (sizeof(E) == 2) { u.see(__builtin_bit_cast(uint32_t, e)); u.see(__builtin_bit_cast(uint32_t, em)); }
    else { u.see(__builtin_bit_cast(u32x2, e)); u.see(__builtin_bit_cast(u32x2, em)); }
  }
  __device__ __forceinline__ void run(const GemmArgs& a, const TileId& t, const TileMatrix& v, const float* sum) const {
#pragma clang fp contract(off)
    f32x2 p[SHARES], q[SHARES];
    static_for<SHARES>([&](auto s) { p[s] = *reinterpret_cast<const f32x2*>(sum + (s * T + r) * LDW + c); });
    if (mirror)
      static_for<SHARES>([&](auto s) { q[s] = f32x2{sum[(s * T + c) * LDW + r], sum[(s * T + c + 1) * LDW + r]}; });
    const int grow = t.ti * T + r, gcol = t.tj * T + c;
    const A C(static_cast<E*>(a.C) + (size_t)t.mat * a.strideC, a.strideC * sizeof(E));
    auto result = [&](const f32x2 (&x)[SHARES], const pair_t& own, bool diagonal) {
      pair_t out;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float val = x[0][i];
        static_for<SHARES - 1>([&](auto s) { val = val + x[s + 1][i]; });
        val = a.E ? v.post * fmaf(a.alpha, val, a.beta * (float)own[i]) : v.post * (a.alpha * val);
        if (diagonal && a.diag != 0.0f && grow < a.diag_n) val += grow == gcol + i ? a.diag : 0.0f;
        out[i] = (E)val;
      }
      return out;
    };
    const pair_t out = result(p, e, true);
    if (a.epilogue != EPI_UPDATE || a.store_out) C.store2(((size_t)grow * a.ldc + gcol) * sizeof(E), out);
    if (mirror) C.store2(((size_t)(t.tj * T + r) * a.ldc + t.ti * T + c) * sizeof(E), result(q, em, false));
    if (update) {
      // W <- (1 - eta lambda) W - eta gamma O, O as stored in the working precision
      f32x2 x;
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = fmaf(a.w_keep, w[i], -(a.o_scale * (float)out[i]));
      const size_t wi = (size_t)grow * v.n + gcol;
      if (w_pair) {
        if (v.w_dtype) {
          typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
          *reinterpret_cast<bf16x2*>(static_cast<bf16_t*>(v.w) + wi) = bf16x2{(bf16_t)x.x, (bf16_t)x.y};
        } else {
          *reinterpret_cast<f32x2*>(static_cast<float*>(v.w) + wi) = x;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (gcol + i < v.n) {
            if (v.w_dtype) static_cast<bf16_t*>(v.w)[wi + i] = (bf16_t)x[i];
            else static_cast<float*>(v.w)[wi + i] = x[i];
          }
      }
    }
  }
};

}  // namespace
}  // namespace mona
