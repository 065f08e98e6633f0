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
// 16 bytes of an array that other workgroups of the same launch write or read (SHARED: coherent across the dies at device
// scope, without any cache being written back or invalidated), or that only earlier and later launches do.  `bytes` from
// the start of the array, which is wavefront-uniform and smaller than 4 GB where it is shared.
constexpr int kDeviceScope = 16;   // sc1
template <bool SHARED>
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
    if constexpr (SHARED) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)(uint32_t)bytes, 0, kDeviceScope);
    else *reinterpret_cast<V*>(p + bytes) = v;
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
  static constexpr int CH = Chunk<E>::N, PER_ROW = T / CH, ALL = T * T / CH;
  static constexpr int PER_LANE = (ALL + THREADS - 1) / THREADS;   // (where there are fewer: of the first threads only)
  static constexpr bool kAll = ALL % THREADS == 0;
};

// the E operand of this thread's chunks
template <typename E, int T, int THREADS, bool SHARED>
__device__ __forceinline__ void load_e(const GemmArgs& a, const TileId& t, int tid,
                                       typename Chunk<E>::vec (&ev)[TileChunks<E, T, THREADS>::PER_LANE]) {
  typedef TileChunks<E, T, THREADS> N;
  if (!a.E) return;
  const Array<SHARED> Eb(static_cast<E*>(const_cast<void*>(a.E)) + (size_t)t.mat * a.strideE, a.strideE * sizeof(E));
#pragma unroll
  for (int u = 0; u < N::PER_LANE; ++u) {
    const int idx = u * THREADS + tid;
    if (N::kAll || idx < N::ALL)
      ev[u] = Eb.template load<typename Chunk<E>::vec>(
          ((size_t)(t.ti * T + idx / N::PER_ROW) * a.lde + t.tj * T + (idx % N::PER_ROW) * N::CH) * sizeof(E));
  }
}

// floats per row of the staged tile (+4: rows on different banks)
constexpr int staged_ld(int T) { return T + 4; }

// The epilogue of a tile whose accumulators stand in LDS as SHARES tiles of T x staged_ld(T) floats that add up to the
// product: every global access is a 16-byte piece of a row.
template <typename E, int T, int SHARES, int THREADS, bool SHARED>
__device__ __forceinline__ void finish_tile(const GemmArgs& a, const TileId& t, const TileMatrix& v, int tid,
                                            typename Chunk<E>::vec (&ev)[TileChunks<E, T, THREADS>::PER_LANE], float* sum) {
  // every contraction is written out: a product comes out the same, bit for bit, in whichever kernel it runs
#pragma clang fp contract(off)
  typedef TileChunks<E, T, THREADS> N;
  typedef typename Chunk<E>::vec vec_t;
  constexpr int ES = sizeof(E), CH = N::CH, CPR = N::PER_ROW, CHUNKS = N::ALL, U = N::PER_LANE, LDW = staged_ld(T);
  constexpr bool kAll = N::kAll;
  const int lane = tid & 63, wave = tid >> 6;
  const int m0 = t.ti * T, n0 = t.tj * T;
  const bool mirror = a.symmetric && t.ti != t.tj, update = a.epilogue == EPI_UPDATE, skip_w = v.skip_w;
  const int wm_real = v.m, wn_real = v.n, w_is_bf16 = v.w_dtype;
  void* const wptr = v.w;
  const float post = v.post;
  const bool w_vec = wn_real % CH == 0;             // rows of W are whole chunks, 16-byte (fp32: 32-byte) aligned
  const Array<SHARED> C(static_cast<E*>(a.C) + (size_t)t.mat * a.strideC, a.strideC * ES);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int idx = u * THREADS + tid;
    if (!kAll && idx >= CHUNKS) break;
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
      if (w_vec && gcol + CH <= wn_real) {
        if (w_is_bf16) {
          typedef bf16_t wv_t __attribute__((ext_vector_type(CH)));
          wv_t* wp = reinterpret_cast<wv_t*>(static_cast<bf16_t*>(wptr) + wi);
          wv_t w = *wp;
#pragma unroll
          for (int e = 0; e < CH; ++e) w[e] = (bf16_t)fmaf(a.w_keep, (float)w[e], -(a.o_scale * (float)ov[e]));
          *wp = w;
        } else {
          f32x4* wp = reinterpret_cast<f32x4*>(static_cast<float*>(wptr) + wi);
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
      // (T = 32 in bf16: there are four pieces to a column, sixteen columns to a wavefront)
      const int grp = u * (THREADS / 64) + wave, idx = u * THREADS + tid;
      if (!kAll && idx >= CHUNKS) break;
      const int c = CPR < 8 ? idx / CPR : (grp % (T / 8)) * 8 + (lane >> 3);
      const int rc = CPR < 8 ? idx % CPR : (grp / (T / 8)) * 8 + (lane & 7);
      vec_t ov;
#pragma unroll
      for (int e = 0; e < CH; ++e) ov[e] = (E)sum[(rc * CH + e) * LDW + c];
      C.store(((size_t)(n0 + c) * a.ldc + m0 + rc * CH) * ES, ov);
    }
  }
}

}  // namespace
}  // namespace mona
