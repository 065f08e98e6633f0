// Elementwise part of the MONA step (Alg. 1: difference, acceleration EMA, accelerated
// gradient, momentum, state roll) fused with the sum of squares that the Newton-Schulz
// prescale X_0 = M / ||M||_F needs (Sec. 3.2).  One pass over the state: every array is
// read once and written once, 16 bytes per lane, so the kernel runs at HBM speed.
//
// Per element, with fp32 G and fp32 state: reads G, G_{k-1}, A, M (16 B), writes G_{k-1}, A, M
// (12 B) and the bf16 copy of M that the matrix products read (2 B): 30 B.  In the one-buffer form
// (no stored G_{k-1}: the bracket C_k = beta_a A_{k-1} - (1 - beta_a) G_{k-1} is carried instead of
// A and G_{k-1}, and A_k = C_k + (1 - beta_a) G_k) it reads G, C, M and writes C, M and the copy: 22 B.
#include "mona_internal.h"

#include <type_traits>

namespace mona {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));

// What of a pass the caches are to keep (choose_keep).  Non-temporal accesses leave nothing of an array that is read once and written
// once in the 256 MB cache behind the L2s.  Measured, us per pass, with nothing / the working copy kept: 64 x 1000 x 2000
// 725 / 676, 64 x 768 x 768 200 / 188, 128 x 768 x 256 both ways 261 / 247, 128 x 1000 x 2000 1452 / 1401, 256 x 1000 x 2000 2927 /
// 2897, 32 x 4096 x 4096 2896 / 2934.  Everything is kept by the launch that begins a small step only.  Elsewhere it pays where the next step
// of the same state finds its arrays still there, but a program's forward and backward passes stand in between.  us per step with the
// copy / everything kept, by states in turn that take 1.2 GB together: 128 x 128 x 128 42.4 / 48.5, 40 x 128 x 256 52.7 / 57.2, 24 x 128 x 512
// 81.6 / 85.9, 100 x 128 x 512 111 / 119, 200 x 128 x 256 84.8 / 92, 6 x 384 x 1000 149.9 / 153.4, 60 x 256 x 512 240 / 245, 30 x 300 x 700 237.6 /
// 241.3; by the same one or two, up to 100 MB of them, 1 to 2.5 % the other way (128 x 128 x 128 45.5 / 44.3, 6 x 384 x 1000 145 / 142).  It is the
// loads that cost: plain ones with non-temporal stores 48.2 and 152.8, the other way round 45.2 and 151.
enum Keep : int { KEEP_NOTHING = 0, KEEP_COPY = 1, KEEP_ALL = 2 };
template <bool STREAM, typename V> __device__ __forceinline__ V load(const V* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool STREAM, typename V> __device__ __forceinline__ void store(V* p, V v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <bool STREAM> __device__ __forceinline__ f32x4 load4(const float* p) { return load<STREAM>(reinterpret_cast<const f32x4*>(p)); }
template <bool STREAM> __device__ __forceinline__ f32x4 load4(const bf16_t* p) {
  bf16x4 v = load<STREAM>(reinterpret_cast<const bf16x4*>(p));
  f32x4 r = {(float)v.x, (float)v.y, (float)v.z, (float)v.w};
  return r;
}
template <bool STREAM> __device__ __forceinline__ void store4(float* p, f32x4 v) { store<STREAM>(reinterpret_cast<f32x4*>(p), v); }
template <bool STREAM> __device__ __forceinline__ void store4(bf16_t* p, f32x4 v) {
  bf16x4 r = {(bf16_t)v.x, (bf16_t)v.y, (bf16_t)v.z, (bf16_t)v.w};  // round to nearest even
  store<STREAM>(reinterpret_cast<bf16x4*>(p), r);
}
__device__ __forceinline__ float load1(const float* p) { return *p; }
__device__ __forceinline__ float load1(const bf16_t* p) { return (float)*p; }
__device__ __forceinline__ void store1(float* p, float v) { *p = v; }
__device__ __forceinline__ void store1(bf16_t* p, float v) { *p = (bf16_t)v; }

// value the stored state holds after rounding to its dtype (identity for fp32)
template <typename ST> __device__ __forceinline__ float stored(float v) { return v; }
template <> __device__ __forceinline__ float stored<bf16_t>(float v) { return (float)(bf16_t)v; }

struct Coef {
  float mu, beta, one_minus_beta, alpha;
  int use_prev;
};

// One element of Alg. 1's elementwise lines.  Returns M_k; updates a (A_k) in place.
__device__ __forceinline__ float mona_element(float g, float gp, float& a, float m, const Coef& c) {
  float d = c.use_prev ? (g - gp) : 0.0f;            // D_k = G_k - G_{k-1}
  a = c.beta * a + c.one_minus_beta * d;             // A_k = beta_a A_{k-1} + (1 - beta_a) D_k
  float gt = g + c.alpha * a;                        // Gt_k = G_k + alpha A_k
  return c.mu * m + gt;                              // M_k = mu M_{k-1} + Gt_k
}

// The squares are summed in double: M_ij^2 leaves the fp32 range once |M_ij| is below about 1e-19 or above
// 1e19 (a matrix that has received no gradient for a few hundred steps decays to such values), and the
// norm must still come out right there.  The kernel is bound by HBM; the fp64 operations are free.
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);   // within the wavefront
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wave] = v;                            // then across wavefronts in LDS
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < kEwThreads / 64; ++w) t += red[w];
  }
  return t;
}

// One element in the one-buffer form.  c holds C_k on entry and C_{k+1} on return; returns M_k.
// With use_prev == 0 (first step, "G_0 := G_1") A_1 = 0, i.e. C_1 = -(1 - beta_a) G_1.
__device__ __forceinline__ float mona_element_one_buffer(float g, float& cbuf, float m, const Coef& c) {
  const float a = c.use_prev ? (cbuf + c.one_minus_beta * g) : 0.0f;   // A_k
  const float gt = g + c.alpha * a;
  cbuf = c.beta * a - c.one_minus_beta * g;
  return c.mu * m + gt;
}

enum StateMode : int { MODE_MUON = 0, MODE_TWO_BUFFER = 1, MODE_ONE_BUFFER = 2 };

// An array whose values a later reader in the same launch may need (M and its working copy) goes through to memory (THROUGH: device
// scope, the array is below 4 GB).
constexpr int kDeviceScope = 16;   // sc1
template <bool THROUGH, bool STREAM>
struct Out {
  char* p;
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit Out(void* base) : p(static_cast<char*>(base)) {
    if constexpr (THROUGH) r = __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000);
  }
  __device__ __forceinline__ void put4(int64_t i, f32x4 v, bool f32) const {
    if constexpr (!THROUGH) {
      if (f32) store4<STREAM>(reinterpret_cast<float*>(p) + i, v); else store4<STREAM>(reinterpret_cast<bf16_t*>(p) + i, v);
    } else if (f32) {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)(uint32_t)(i * 4), 0, kDeviceScope);
    } else {
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      const bf16x4 h = {(bf16_t)v.x, (bf16_t)v.y, (bf16_t)v.z, (bf16_t)v.w};
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, h), r, (int)(uint32_t)(i * 2), 0, kDeviceScope);
    }
  }
  __device__ __forceinline__ void put2(int64_t i, float a, float b, bool f32) const {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    const bf16x2 h = {(bf16_t)a, (bf16_t)b};
    if constexpr (!THROUGH) {
      if (f32) *reinterpret_cast<f32x2*>(reinterpret_cast<float*>(p) + i) = v; else *reinterpret_cast<bf16x2*>(reinterpret_cast<bf16_t*>(p) + i) = h;
    } else if (f32) {
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)(uint32_t)(i * 4), 0, kDeviceScope);
    } else {
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, h), r, (int)(uint32_t)(i * 2), 0, kDeviceScope);
    }
  }
  __device__ __forceinline__ void put(int64_t i, float v, bool f32) const {
    if constexpr (!THROUGH) {
      if (f32) reinterpret_cast<float*>(p)[i] = v; else reinterpret_cast<bf16_t*>(p)[i] = (bf16_t)v;
    } else if (f32) {
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (int)(uint32_t)(i * 4), 0, kDeviceScope);
    } else {
      __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, (bf16_t)v), r, (int)(uint32_t)(i * 2), 0, kDeviceScope);
    }
  }
};

// MODE_MUON is plain Muon (Eq. muon_momentum fed with G_k itself): the acceleration buffers
// are neither read nor written.
// One chunk of a matrix by one workgroup; returns this thread's share of the sum of squares.
template <typename GT, typename ST, int MODE, int KEEP, bool THROUGH>
__device__ __forceinline__ double update_chunk(const MatStatic& ms, const MatDynamic& md, int chunk, const Coef& c) {
  const GT* __restrict__ g = static_cast<const GT*>(md.g);
  // G_{k-1} lives in the arena, or (streaming variant) in the slot the caller keeps
  ST* __restrict__ gp = static_cast<ST*>(ms.g_prev ? ms.g_prev : md.slot);
  ST* __restrict__ ac = static_cast<ST*>(ms.acc);
  float* __restrict__ mo = ms.mom;
  // working copy of M_k for the matrix products: bf16, or fp32 for matrices orthogonalised in fp32
  constexpr bool STREAM = KEEP != KEEP_ALL;
  const Out<THROUGH, STREAM> mom(ms.mom);
  const Out<THROUGH, KEEP == KEEP_NOTHING> x(ms.x);
  bf16_t* __restrict__ xh = static_cast<bf16_t*>(ms.x);
  float* __restrict__ xf = static_cast<float*>(ms.x);
  const bool xf32 = ms.x_f32 != 0;

  const int total = ms.m * ms.n;
  const int base = chunk * kEwChunk;
  const int count = min(kEwChunk, total - base);
  const int n = ms.n, ldx = ms.ldx;
  double ss = 0.0;

  // Groups of 4 elements as they lie in the arrays; where rows are no multiple of 4, a group may straddle two rows of the padded copy,
  // which it is stored to in pairs or one by one (element by element throughout, a chunk took sixteen round trips: nine ragged matrices 7.7 us)
  constexpr int kIter = kEwChunk / (kEwThreads * 4);
  constexpr int kBatch = 4;
  static_assert(kIter % kBatch == 0, "chunk must be a multiple of the batch");
  auto groups = [&](auto whole) {
    for (int it0 = 0; it0 < kIter; it0 += kBatch) {
      f32x4 vg[kBatch], vp[kBatch], va[kBatch], vm[kBatch];
      int idx[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int i = ((it0 + b) * kEwThreads + threadIdx.x) * 4;
        idx[b] = (i + 4 <= count) ? base + i : -1;
        if (idx[b] >= 0) {
          vg[b] = load4<STREAM>(g + idx[b]);
          if constexpr (MODE == MODE_TWO_BUFFER) vp[b] = load4<STREAM>(gp + idx[b]);
          if constexpr (MODE != MODE_MUON) va[b] = load4<STREAM>(ac + idx[b]);
          vm[b] = load4<STREAM>(mo + idx[b]);
        }
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        if (idx[b] >= 0) {
          float a4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, p4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          if constexpr (MODE != MODE_MUON) { a4[0] = va[b].x; a4[1] = va[b].y; a4[2] = va[b].z; a4[3] = va[b].w; }
          if constexpr (MODE == MODE_TWO_BUFFER) { p4[0] = vp[b].x; p4[1] = vp[b].y; p4[2] = vp[b].z; p4[3] = vp[b].w; }
          const float g4[4] = {vg[b].x, vg[b].y, vg[b].z, vg[b].w};
          const float m4[4] = {vm[b].x, vm[b].y, vm[b].z, vm[b].w};
          float n4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (MODE == MODE_TWO_BUFFER) n4[e] = mona_element(g4[e], p4[e], a4[e], m4[e], c);
            else if constexpr (MODE == MODE_ONE_BUFFER) n4[e] = mona_element_one_buffer(g4[e], a4[e], m4[e], c);
            else n4[e] = c.mu * m4[e] + g4[e];
          }
          const f32x4 a = {a4[0], a4[1], a4[2], a4[3]};
          const f32x4 mnew = {n4[0], n4[1], n4[2], n4[3]};
          ss += (double)mnew.x * mnew.x + (double)mnew.y * mnew.y + (double)mnew.z * mnew.z + (double)mnew.w * mnew.w;
          if constexpr (MODE == MODE_TWO_BUFFER) store4<STREAM>(gp + idx[b], vg[b]);   // G_{k-1} <- G_k
          if constexpr (MODE != MODE_MUON) store4<STREAM>(ac + idx[b], a);              // A_k, or C_{k+1}
          if constexpr (THROUGH) mom.put4(idx[b], mnew, true); else store4<STREAM>(mo + idx[b], mnew);
          // the padded copy can exceed 2^31 elements although m * n does not: 64-bit offset
          if constexpr (whole) {
            const int64_t xo = (ldx == n) ? (int64_t)idx[b] : (int64_t)(idx[b] / n) * ldx + (idx[b] % n);
            if constexpr (THROUGH) x.put4(xo, mnew, xf32);
            else if (xf32) store4<KEEP == KEEP_NOTHING>(xf + xo, mnew);
            else store4<KEEP == KEEP_NOTHING>(xh + xo, mnew);
          } else {
            const int row = idx[b] / n;
            int col = idx[b] - row * n;
            int64_t row_at = (int64_t)row * ldx;
            if ((n & 1) == 0) {
              x.put2(row_at + col, n4[0], n4[1], xf32);
              col += 2;
              if (col == n) { col = 0; row_at += ldx; }
              x.put2(row_at + col, n4[2], n4[3], xf32);
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (col == n) { col = 0; row_at += ldx; }
                x.put(row_at + col, n4[e], xf32);
                ++col;
              }
            }
          }
        }
      }
    }
  };
  if ((n & 3) == 0) groups(std::true_type{}); else groups(std::false_type{});
  // the last elements of a matrix
  if (const int i = (count & ~3) + (int)threadIdx.x; i < count) {
    const int id = base + i;
    const float gv = load1(g + id);
    float mnew;
    if constexpr (MODE == MODE_TWO_BUFFER) {
      float a = load1(ac + id);
      mnew = mona_element(gv, load1(gp + id), a, mo[id], c);
      store1(gp + id, gv);
      store1(ac + id, a);
    } else if constexpr (MODE == MODE_ONE_BUFFER) {
      float cb = load1(ac + id);
      mnew = mona_element_one_buffer(gv, cb, mo[id], c);
      store1(ac + id, cb);
    } else {
      mnew = c.mu * mo[id] + gv;
    }
    ss += (double)mnew * mnew;
    mom.put(id, mnew, true);
    const int64_t xo = (int64_t)(id / n) * ldx + (id % n);
    x.put(xo, mnew, xf32);
  }
  return ss;
}

template <typename GT, typename ST, int MODE, int KEEP>
__global__ __launch_bounds__(kEwThreads) void state_update_kernel(
    const MatStatic* __restrict__ stat, const MatDynamic* __restrict__ dyn,
    const BlockWork* __restrict__ work, double* __restrict__ partials, Coef c) {
  __shared__ double red[kEwThreads / 64];
  const BlockWork bw = work[blockIdx.x];
  const MatStatic ms = stat[bw.mat];
  const MatDynamic md = dyn[bw.mat];
  const double t = block_sum(update_chunk<GT, ST, MODE, KEEP, false>(ms, md, bw.chunk, c), red);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// ||M||_F per matrix from the per-block partial sums, added in a fixed order in fp64 so the
// result does not depend on scheduling, and the repair of the (rare) working copies that need one.
//
// The products that follow accumulate the unscaled working copy in fp32 and apply 1 / ||M||_F^2 afterwards,
// which is exact only while the squares stay inside the fp32 range.  A norm outside [2^-40, 2^40] therefore
// sets MONA_STATUS_RESCALED: that matrix's working copy is rewritten as M 2^e with
// ||M 2^e||_F in [1, 2), and the scale stored here is the one that belongs to the rewritten copy (a power
// of two moves no bit of any product, so the result is the one an unlimited exponent range would give).
// A matrix with a non-finite norm gets an all-zero copy (its products then stay zero, so no NaN ever reaches
// the zero padding the Gram matrices rely on; its parameter is left alone anyway).
//
// `per_mat` workgroups per matrix, every one of which adds up the partial sums for itself (the same order, the same
// bits): the first stores the scale, and all share the repair.  What bounds the kernel is the latency of the partial
// sums, one wavefront per matrix before: 34 us for the 7 696 partial sums of a 3328 x 9472 matrix, 6 us for 1 536, and
// 4 - 5 us more for a launch of its own that looked for flagged matrices; now 4 - 7 us in all where no matrix is flagged.
//
// The flags of the products that follow are cleared on the way, and (FILL) the buffers of fresh chains filled by workgroups behind
// those of the matrices (ns_chain_kernel).
//
// The repair has to stay wide whatever the length of the list: one expert without gradients in a long list would
// otherwise hold up every product behind it.  Where the list is too long for one workgroup to every kRepairBlocks
// blocks' worth of elements of every matrix, repair is 0 here and rescue_kernel does it (4 us of a step of 2 ms and more); small steps
// have it in their first launch (begin_norm_finalize_kernel).
constexpr double kNormLo = 9.094947017729282e-13;   // 2^-40
constexpr double kNormHi = 1099511627776.0;         // 2^40
constexpr int kRepairBlocks = 16, kRepairGroups = 2048;

// M as a repair reads it.  SHARED: other workgroups of the same launch have stored it (at device scope, Out), so it is read at device scope
// too: a line at the edge of two chunks may stand in this die's L2 as it was before the other chunk's workgroup stored its part (M is
// 16-byte aligned at least, chunks are 16 KB).
template <bool SHARED>
struct In {
  const float* p;
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit In(float* base) : p(base) {
    if constexpr (SHARED) r = __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000);
  }
  __device__ __forceinline__ f32x4 get4(uint32_t i) const {
    if constexpr (SHARED) return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(i * 4u), 0, kDeviceScope));
    else return *reinterpret_cast<const f32x4*>(p + i);
  }
  __device__ __forceinline__ float get(uint32_t i) const {
    if constexpr (SHARED) return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)(i * 4u), 0, kDeviceScope));
    else return p[i];
  }
};

// Rewrites a flagged working copy: the units (of 4 elements) first + thread, every step'th from there, below end.  Bound by HBM once wide
// enough: 16-byte loads of M, U in flight per lane; a unit's row and column follow from the one's before it.
template <int U, bool SHARED>
__device__ __forceinline__ void repair_units(const MatStatic& ms, const MatScale& r, uint32_t first, uint32_t end, uint32_t step) {
  const bool clear = (r.status & 2u) != 0;
  // m * n is below 2^31, and the walk passes its end by at most U x 2048 x 256 units: 32 bits hold every index
  const uint32_t n = (uint32_t)ms.n, total = (uint32_t)ms.m * n, whole = total / 4;
  bf16_t* __restrict__ xh = static_cast<bf16_t*>(ms.x);
  float* __restrict__ xf = static_cast<float*>(ms.x);
  const In<SHARED> mom(ms.mom);
  uint32_t u = first + threadIdx.x;
  uint32_t row = 4 * u / n, col = 4 * u - row * n;
  const uint32_t rows = 4 * step / n, cols = 4 * step - rows * n;
  for (; u < end; u += U * step) {
    f32x4 v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t at = u + j * step;
      v[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (clear || at >= end) continue;
      if (at < whole) v[j] = mom.get4(4 * at);
      else
        for (uint32_t e = 0; e < total - 4 * at; ++e) v[j][e] = mom.get(4 * at + e);
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t at = u + j * step;
      if (at < end) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = ldexpf(v[j][e], r.xexp);
        if (n % 4 == 0) {                            // the four elements are in one row, 16-byte aligned there
          const int64_t xo = (int64_t)row * ms.ldx + col;
          if (ms.x_f32) *reinterpret_cast<f32x4*>(xf + xo) = v[j];
          else *reinterpret_cast<bf16x4*>(xh + xo) = bf16x4{(bf16_t)v[j].x, (bf16_t)v[j].y, (bf16_t)v[j].z, (bf16_t)v[j].w};
        } else {
          int64_t row_at = (int64_t)row * ms.ldx;
          uint32_t c = col;
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) {
            if (at < whole || e < total - 4 * at) {
              if (ms.x_f32) xf[row_at + c] = v[j][e]; else xh[row_at + c] = (bf16_t)v[j][e];
            }
            if (++c == n) { c = 0; row_at += ms.ldx; }
          }
        }
      }
      row += rows;
      col += cols;
      if (col >= n) { col -= n; ++row; }
    }
  }
}
// ... the share of workgroup `part` of `parts`.
__device__ __forceinline__ void repair_copy(const MatStatic& ms, const MatScale& r, int part, int parts) {
  repair_units<4, false>(ms, r, (uint32_t)part * kEwThreads, ((uint32_t)ms.m * (uint32_t)ms.n + 3) / 4, (uint32_t)parts * kEwThreads);
}

// What a chain's buffers hold before its products, by one workgroup (of `block`): kFillPieces pieces, all of one item.  (The item is
// looked up by all lanes at once: one by one, each look is a round trip.)
__device__ __forceinline__ void fill_pieces(const FillArgs& f, uint32_t block) {
  const int lane = threadIdx.x & 63;
  const uint64_t before = __ballot(lane < f.n && f.item[lane].end <= block);
  const int i = __builtin_amdgcn_readfirstlane(__popcll(before));
  const FillItem t = f.item[i];
  const uint32_t first = i > 0 ? f.item[i - 1].end : 0u;
#pragma unroll
  for (int k = 0; k < kFillPieces / kEwThreads; ++k) {
    const uint32_t at = (block - first) * kFillPieces + k * kEwThreads + threadIdx.x;
    if (at >= t.pieces) break;
    const uint32_t line = at / t.width, c = at - line * t.width, buffer = line / t.rows, r = line - buffer * t.rows;
    const uint32_t v = r < t.cover_rows && c < t.cover ? kUnwritten : 0u;
    *reinterpret_cast<uint4*>(t.at + (size_t)buffer * t.stride + (size_t)r * t.pitch + c * 16) = uint4{v, v, v, v};
  }
}

// The scale of a matrix whose squares add up to s.
__device__ __forceinline__ MatScale scale_of(double s, float eps) {
  const double norm = sqrt(s);
  const double den = norm + (double)eps;
  MatScale r;
  r.norm = (float)fmin(norm, 3.402823466e38);
  r.status = 0u;
  r.xexp = 0;
  const bool finite = (s == s) && (s <= 1.7e308);
  if (!finite) {
    r.norm = (float)norm;
    r.inv = 0.0f;
    r.status = 2u;
  } else if (den <= 0.0) {
    r.inv = 0.0f;
    r.status = 1u;
  } else if (norm == 0.0 || (norm >= kNormLo && norm <= kNormHi)) {
    r.inv = 1.0f / ((float)norm + eps);
  } else {
    r.xexp = -ilogb(norm);
    r.inv = (float)ldexp(1.0 / den, -r.xexp);
    r.status = 4u;
  }
  r.inv2 = r.inv * r.inv;
  r.arrived = r.verdict = r.shares = 0u;
  return r;
}

struct NoFill {};
template <typename Fill>
__global__ __launch_bounds__(kEwThreads) void norm_finalize_kernel(const MatStatic* __restrict__ stat,
                                                                   const double* __restrict__ partials,
                                                                   MatScale* __restrict__ scales,
                                                                   const int32_t* __restrict__ list, float eps,
                                                                   int per_mat, int repair, uint4* __restrict__ zero,
                                                                   int n16, const Fill fill, int norm_groups) {
  if constexpr (!std::is_same_v<Fill, NoFill>) {
    if ((int)blockIdx.x >= norm_groups) {
      fill_pieces(fill, blockIdx.x - norm_groups);
      return;
    }
  }
  __shared__ double red[kEwThreads / 64];
  __shared__ double total_sum;
  const int li = blockIdx.x / per_mat, part = blockIdx.x % per_mat;
  const int mat = list ? list[li] : li;
  const MatStatic ms = stat[mat];
  const double* __restrict__ p = partials + ms.first_block;
  double s = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < ms.num_blocks; i += kEwThreads) s += p[i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) total_sum = s;
  __syncthreads();
  s = total_sum;
  const MatScale r = scale_of(s, eps);
  if (part == 0 && threadIdx.x == 0) scales[mat] = r;
  for (int i = blockIdx.x * kEwThreads + threadIdx.x; i < n16; i += norm_groups * kEwThreads) zero[i] = uint4{0u, 0u, 0u, 0u};
  if (repair && (r.status & 6u)) repair_copy(ms, r, part, per_mat);
}

// All that stands before the products of a small step in one launch (BeginTable: the pointers too): the elementwise pass, norms,
// scales, repair, what chains need cleared and filled.  Three launches of a few workgroups take 12 us, of which the work is a third.  The
// workgroup that finishes a matrix last (MatScale::arrived) adds up the partial sums, in the order of norm_finalize_kernel.
// Measured, us per step, three launches -> one: 256 x 512 58.8 -> 54.6, nine ragged matrices 75.0 -> 70.3, 512 x 1408 without allocation (two
// -> one) 96.0 -> 91.3.
//
// Repair: a workgroup that knows of a chunk whose squares alone put the norm out of range (its own, or ChainRoll::spoiled says so), or whose own
// chunk is too small to keep it within, stays until the last one has given its verdict, and those that have stayed share the repair with it,
// drawing pieces of the copy from a counter.  What they read of each other, at device scope, has gone through to memory before a workgroup
// counted itself.  Nobody has to stay (the chip may have no room for those that are still to come): after kStayPolls looks a workgroup
// leaves, and whoever is left does its share.  Whoever leaves last puts the counters back to zero.
// Bound by what a CU can have on its way beyond L2, so by the workgroups that share it.  Measured, us per step, ordinary / all tiny / all large /
// one value large / one not a number: 512 x 1408 90 / 104 / 108 / 101 / 96, 512 x 2048 104 / 120 / 128 / 116 / 112, 513 x 801 85 / 95 / 98 / 94 /
// 91, 256 x 512 54.5 / 60 / 62 / 60 / 57.  The last workgroup alone: 512 x 1408 90 / 320 / 319 / 319 / 281; three launches, a workgroup to every 16
// blocks: 115 / 142 / 142 / 142 / 123.  (`spoiled` beside the counters instead of on a line of its own cost ordinary steps 1 to 4 us.)
constexpr int kStayPolls = 64;                                       // about 50 us
constexpr double kSumLo = kNormLo * kNormLo, kSumHi = kNormHi * kNormHi;
constexpr uint32_t kStayed = 1u << 16;                               // MatScale::arrived, shares: a workgroup that stays, that leaves
// MatScale::verdict (not 0 once it is given): how many share the repair, whether there is any, what of MatScale it takes
constexpr uint32_t kVerdict = 1u << 31, kRepair = 1u << 30, kClear = 1u << 29;
constexpr int kExpAt = 16, kExpBias = 1024;

__device__ __forceinline__ uint32_t device_load(uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void device_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a workgroup does from the verdict on (0: it has not waited for it).  `word`: of LDS.
__device__ __forceinline__ void share_repair(const MatStatic& ms, MatScale* scale, uint32_t verdict, uint32_t* word) {
  if (verdict & kRepair) {
    MatScale r;
    r.status = verdict & kClear ? 2u : 4u;
    r.xexp = (int)(verdict >> kExpAt & 0x7ffu) - kExpBias;
    // (a copy to be cleared by its rows, 16 bytes a unit; their padding is zero as it is)
    const bool clear = (verdict & kClear) != 0;
    const uint32_t units = clear ? (uint32_t)((int64_t)ms.m * ms.ldx / (ms.x_f32 ? 4 : 8)) : ((uint32_t)ms.m * (uint32_t)ms.n + 3) / 4;
    const uint32_t pieces = min(2 * (verdict & 0xffffu), (uint32_t)ms.num_blocks), piece = (units + pieces - 1) / pieces;
    for (;;) {
      if (threadIdx.x == 0)
        *word = __hip_atomic_fetch_add(&scale->shares, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffffu;
      __syncthreads();
      const uint32_t mine = *word;
      __syncthreads();
      if (mine >= pieces) break;
      const uint32_t first = mine * piece, end = min(first + piece, units);
      if (!clear) repair_units<8, true>(ms, r, first, end, kEwThreads);
      else
        for (uint32_t u = first + threadIdx.x; u < end; u += kEwThreads) static_cast<uint4*>(ms.x)[u] = uint4{0u, 0u, 0u, 0u};
    }
  }
  if (threadIdx.x != 0) return;
  // (the verdict is in memory before the one who gave it has left, and looked up again by those who have not waited for it once they have)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const uint32_t left = __hip_atomic_fetch_add(&scale->shares, kStayed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  verdict = device_load(&scale->verdict);
  if (verdict == 0u || left + 1 != (verdict & 0xffffu)) return;
  device_store(&scale->arrived, 0u);
  device_store(&scale->verdict, 0u);
  device_store(&scale->shares, 0u);
}

template <typename ST, int MODE>
__global__ __launch_bounds__(kEwThreads) void begin_norm_finalize_kernel(
    const MatStatic* __restrict__ stat, const BlockWork* __restrict__ work, MatScale* scales, double* partials, MatDynamic* dyn,
    Coef c, float eps, uint4* __restrict__ zero, int n16, const FillArgs fill, int update_groups, const BeginTable table) {
  __shared__ double red[kEwThreads / 64];
  __shared__ double total_sum;
  __shared__ uint32_t count, word;
  for (int i = blockIdx.x * kEwThreads + threadIdx.x; i < n16; i += gridDim.x * kEwThreads) zero[i] = uint4{0u, 0u, 0u, 0u};
  if ((int)blockIdx.x >= update_groups) {
    fill_pieces(fill, blockIdx.x - update_groups);
    return;
  }
  const BlockWork bw = work[blockIdx.x];
  const MatStatic ms = stat[bw.mat];
  const MatDynamic md = table.n > 0 ? table.v[bw.mat] : dyn[bw.mat];
  if (table.n > 0 && bw.chunk == 0 && threadIdx.x == 0) dyn[bw.mat] = md;
  const double ss = ms.g_dtype ? update_chunk<bf16_t, ST, MODE, KEEP_ALL, true>(ms, md, bw.chunk, c)
                               : update_chunk<float, ST, MODE, KEEP_ALL, true>(ms, md, bw.chunk, c);
  MatScale* const scale = scales + bw.mat;
  double s = block_sum(ss, red);
  uint32_t spoiled = 0;
  if (threadIdx.x == 0) {
    // (only a hint: cleared above by workgroups that may still be to come, or that have not been heard of here)
    uint32_t* const hint = &reinterpret_cast<ChainRoll*>(zero)->spoiled;
    __hip_atomic_store(partials + blockIdx.x, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!(s <= kSumHi)) device_store(hint, 1u);
    spoiled = device_load(hint);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wavefront's stores are where every die sees them
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t stays = spoiled != 0u || !(s <= kSumHi) || (s > 0.0 && s < kSumLo) ? kStayed : 0u;
    count = __hip_atomic_fetch_add(&scale->arrived, 1u + stays, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word = stays;
  }
  __syncthreads();
  const uint32_t arrived = count;
  if ((int)(arrived & 0xffffu) != ms.num_blocks - 1) {
    if (word == 0u) return;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t v = 0;
      for (int i = 0; i < kStayPolls && (v = device_load(&scale->verdict)) == 0u; ++i) __builtin_amdgcn_s_sleep(8);
      word = v;
    }
  } else {
    s = 0.0;
    for (int i = threadIdx.x; i < ms.num_blocks; i += kEwThreads)
      s += __hip_atomic_load(partials + ms.first_block + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s = block_sum(s, red);
    if (threadIdx.x == 0) total_sum = s;
    __syncthreads();
    const MatScale r = scale_of(total_sum, eps);
    const bool repair = (r.status & 6u) != 0, alone = arrived < kStayed;
    if (threadIdx.x == 0) {
      scale->inv = r.inv;
      scale->inv2 = r.inv2;
      scale->norm = r.norm;
      scale->status = r.status;
      scale->xexp = r.xexp;
      if (alone && !repair) scale->arrived = 0u;
    }
    if (alone && !repair) return;
    if (threadIdx.x == 0) {
      word = kVerdict | (repair ? kRepair : 0u) | (r.status & 2u ? kClear : 0u) | (uint32_t)(r.xexp + kExpBias) << kExpAt |
             ((arrived >> 16) + 1u);
      device_store(&scale->verdict, word);
    }
  }
  __syncthreads();
  const uint32_t verdict = word;
  __syncthreads();
  share_repair(ms, scale, verdict, &word);
}

// The repair of a long list: every workgroup scans the flags, leaves at once when none is set, and takes its share of
// every flagged matrix.  Bound by the scan (4 us for 388 matrices) or, where it repairs, by HBM.
__global__ __launch_bounds__(kEwThreads) void rescue_kernel(const MatStatic* __restrict__ stat,
                                                            const MatScale* __restrict__ scales,
                                                            const int32_t* __restrict__ list, int count) {
  int any = 0;
  for (int i = threadIdx.x; i < count; i += kEwThreads) any |= (scales[list ? list[i] : i].status & 6u) != 0;
  if (!__syncthreads_or(any)) return;
  for (int li = 0; li < count; ++li) {
    const int mat = list ? list[li] : li;
    const MatScale r = scales[mat];
    if (r.status & 6u) repair_copy(stat[mat], r, blockIdx.x, gridDim.x);
  }
}

// The pointer table of a step whose pointers are new, for short lists.  What bounds it is the dispatch: a copy of the
// same bytes from pinned memory runs as a kernel too, but waits for what is before it and holds up what is behind it
// (one 256 x 512 matrix: 103.3 -> 98.3 us a step).
__global__ __launch_bounds__(128) void write_dyn_kernel(const DynTable t, int n, MatDynamic* __restrict__ dyn) {
  static_assert(kInlineMats <= 128, "one thread per entry");
  if ((int)threadIdx.x < n) dyn[threadIdx.x] = t.v[threadIdx.x];
}

// Prepares a state that holds ONE matrix, for the entry point that may neither allocate nor copy from host memory:
// clears [zero, zero + n16 x 16 bytes) and the scale, and writes the tables from kernel arguments.
__global__ __launch_bounds__(256) void single_prepare_kernel(MatStatic ms, MatDynamic md, void* o_ptr, MatStatic* stat,
                                                             MatDynamic* dyn, void** o_ptrs, BlockWork* work,
                                                             int num_blocks, int32_t* members, int32_t* order,
                                                             MatScale* scale, uint4* zero, size_t n16) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0) {
    stat[0] = ms; dyn[0] = md; o_ptrs[0] = o_ptr; members[0] = 0; order[0] = 0;
    scale[0] = MatScale{};
  }
  for (int b = i; b < num_blocks; b += gridDim.x * 256) work[b] = BlockWork{0, b};
  const uint4 z = {0u, 0u, 0u, 0u};
  for (size_t k = i; k < n16; k += (size_t)gridDim.x * 256) zero[k] = z;
}

// O = X_0 and the parameter update when no Newton-Schulz iteration is requested (T = 0),
// W <- (1 - eta lambda) W - eta gamma O   (Eq. muon_update).
template <typename WT>
__global__ __launch_bounds__(kEwThreads) void plain_update_kernel(
    const MatStatic* __restrict__ stat, const MatDynamic* __restrict__ dyn,
    const MatScale* __restrict__ scales, const BlockWork* __restrict__ work,
    void* const* __restrict__ o_ptrs, float lr, float wd, float gamma_coeff, int store_o, int want_w_dtype) {
  const BlockWork bw = work[blockIdx.x];
  const MatStatic ms = stat[bw.mat];
  if (ms.w_dtype != want_w_dtype) return;
  const MatScale sc = scales[bw.mat];
  if (sc.status & 2u) return;
  WT* __restrict__ w = static_cast<WT*>(dyn[bw.mat].w);
  const bool xf32 = ms.x_f32 != 0;
  const bf16_t* __restrict__ xh = static_cast<const bf16_t*>(ms.x);
  const float* __restrict__ xf = static_cast<const float*>(ms.x);
  bf16_t* __restrict__ oh = static_cast<bf16_t*>(o_ptrs[bw.mat]);
  float* __restrict__ of = static_cast<float*>(o_ptrs[bw.mat]);
  const int total = ms.m * ms.n;
  const int base = bw.chunk * kEwChunk;
  const int count = min(kEwChunk, total - base);
  const float gamma = gamma_coeff * sqrtf((float)max(ms.m, ms.n));
  const float keep = 1.0f - lr * wd, os = lr * gamma;
  for (int i = threadIdx.x; i < count; i += kEwThreads) {
    const int id = base + i;
    const int64_t xo = (int64_t)(id / ms.n) * ms.ldx + (id % ms.n);
    // O = X_0 in the working precision of this matrix
    const float ov = xf32 ? sc.inv * xf[xo] : stored<bf16_t>(sc.inv * (float)xh[xo]);
    if (store_o) {
      if (xf32) of[xo] = ov; else oh[xo] = (bf16_t)ov;
    }
    store1(w + id, keep * load1(w + id) - os * ov);
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint4* __restrict__ p, size_t n16) {
  const uint4 z = {0u, 0u, 0u, 0u};
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
    p[i] = z;
}

template <typename GT, typename ST, int MODE>
hipError_t launch_su(const MatStatic* stat, const MatDynamic* dyn, const BlockWork* work, double* partials,
                     int num_blocks, Coef c, int keep, hipStream_t s) {
  auto* const kernel = keep == KEEP_COPY ? state_update_kernel<GT, ST, MODE, KEEP_COPY> : state_update_kernel<GT, ST, MODE, KEEP_NOTHING>;
  // (long passes over four fp32 arrays with three workgroups to a CU instead of five, by LDS that nothing uses: the kernel, two runs of each,
  // 192 x 2048 x 1024 2154, 2160 -> 2135, 2148 us, 48 x 4096 x 4096 4384, 4405 -> 4357, 4326: 0.6 to 1.8 % of it, a quarter of that of a step.
  // Shorter ones gain and lose 1 %, a step with one bf16 array loses 0.8 %)
  const size_t lds = keep == KEEP_NOTHING && MODE == MODE_TWO_BUFFER && sizeof(ST) == 4 ? 160 * 1024 / 3 / 256 * 256 - 256 : 0;
  hipLaunchKernelGGL(kernel, dim3(num_blocks), dim3(kEwThreads), lds, s, stat, dyn, work, partials, c);
  return hipGetLastError();
}
template <int MODE>
hipError_t launch_su_mode(const MatStatic* stat, const MatDynamic* dyn, const BlockWork* work, double* partials,
                          int num_blocks, int g_bf16, int state_bf16, Coef c, int keep, hipStream_t s) {
  switch ((g_bf16 ? 2 : 0) | (state_bf16 ? 1 : 0)) {
    case 0: return launch_su<float, float, MODE>(stat, dyn, work, partials, num_blocks, c, keep, s);
    case 1: return launch_su<float, bf16_t, MODE>(stat, dyn, work, partials, num_blocks, c, keep, s);
    case 2: return launch_su<bf16_t, float, MODE>(stat, dyn, work, partials, num_blocks, c, keep, s);
    default: return launch_su<bf16_t, bf16_t, MODE>(stat, dyn, work, partials, num_blocks, c, keep, s);
  }
}

}  // namespace

// The working copies where these take at most twice what the cache holds: what the products read first is still there, and the copies' lines
// are not turned out one by one between the loads.
int choose_keep(double copy_bytes) {
  constexpr double kCache = 256.0 * 1024 * 1024;
  return copy_bytes <= 2.0 * kCache ? KEEP_COPY : KEEP_NOTHING;
}

// The gradient dtype may differ between matrices: the host orders the work table by gradient
// dtype and launches each dtype's range of blocks separately.
hipError_t launch_state_update(const MatStatic* stat, const MatDynamic* dyn, const BlockWork* work,
                               double* partials, int num_blocks, int g_bf16, int state_bf16, int one_buffer,
                               float mu, float beta_a, float alpha, int use_prev, int keep, hipStream_t s) {
  if (num_blocks <= 0) return hipSuccess;
  Coef c;
  c.mu = mu;
  c.beta = beta_a;
  c.one_minus_beta = 1.0f - beta_a;
  c.alpha = alpha;
  // use_prev: 0 = take D_k = 0 (first step with the first-difference flag), 1 = Alg. 1,
  //           2 = plain Muon (acceleration buffers untouched)
  c.use_prev = use_prev == 1;
  if (use_prev == 2) {
    // the state dtype does not matter: the acceleration buffers are not touched
    if (g_bf16) return launch_su<bf16_t, float, MODE_MUON>(stat, dyn, work, partials, num_blocks, c, keep, s);
    return launch_su<float, float, MODE_MUON>(stat, dyn, work, partials, num_blocks, c, keep, s);
  }
  if (one_buffer) return launch_su_mode<MODE_ONE_BUFFER>(stat, dyn, work, partials, num_blocks, g_bf16, state_bf16, c, keep, s);
  return launch_su_mode<MODE_TWO_BUFFER>(stat, dyn, work, partials, num_blocks, g_bf16, state_bf16, c, keep, s);
}

hipError_t launch_begin(const MatStatic* stat, const BlockWork* work, MatScale* scales, double* partials, MatDynamic* dyn, int num_blocks,
                        int state_bf16, int one_buffer, float mu, float beta_a, float alpha, int use_prev, float eps, void* zero,
                        size_t zero_bytes, const FillArgs& fill, const BeginTable& table, hipStream_t s) {
  const Coef c = {mu, beta_a, 1.0f - beta_a, alpha, use_prev == 1};
  auto* const kernel = use_prev == 2 ? begin_norm_finalize_kernel<float, MODE_MUON>
                       : one_buffer ? (state_bf16 ? begin_norm_finalize_kernel<bf16_t, MODE_ONE_BUFFER> : begin_norm_finalize_kernel<float, MODE_ONE_BUFFER>)
                       : state_bf16 ? begin_norm_finalize_kernel<bf16_t, MODE_TWO_BUFFER> : begin_norm_finalize_kernel<float, MODE_TWO_BUFFER>;
  hipLaunchKernelGGL(kernel, dim3(num_blocks + fill.groups), dim3(kEwThreads), 0, s, stat, work, scales, partials, dyn, c, eps,
                     static_cast<uint4*>(zero), (int)(zero_bytes / 16), fill, num_blocks, table);
  return hipGetLastError();
}

hipError_t launch_write_dyn(const DynTable& t, int n, MatDynamic* dyn, hipStream_t s) {
  if (n < 1 || n > kInlineMats) return hipErrorInvalidValue;
  hipLaunchKernelGGL(write_dyn_kernel, dim3(1), dim3(128), 0, s, t, n, dyn);
  return hipGetLastError();
}

hipError_t launch_norm_finalize(const MatStatic* stat, const double* partials, MatScale* scales,
                                const int32_t* list, int count, int max_blocks, float eps, void* zero, size_t zero_bytes,
                                const FillArgs* fill, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  // Workgroups of kRepairBlocks blocks' worth of elements each, as long as all of them are resident at once (eight to a
  // CU); otherwise one a matrix, and the repair in a launch of its own.  Measured, us per step without and with one
  // matrix out of range: 256 x 512 alone 102, 127 (one workgroup for 64 blocks: 349); 768 x 256 among 256 979, 995 (1349);
  // 2048 x 4096 behind 600 of 16 x 24 745, 835 (one workgroup a matrix and no launch of its own: 17409);
  // 4096 x 1536 among 388 13.78 ms, 13.80 (two workgroups: 21.36).
  int per_mat = (max_blocks + kRepairBlocks - 1) / kRepairBlocks;
  const bool apart = per_mat > 1 && (long long)count * per_mat > kRepairGroups;
  if (apart) per_mat = 1;
  const int groups = count * per_mat;
  if (fill && fill->groups > 0) {
    hipLaunchKernelGGL(norm_finalize_kernel<FillArgs>, dim3(groups + fill->groups), dim3(kEwThreads), 0, s, stat, partials, scales, list,
                       eps, per_mat, apart ? 0 : 1, static_cast<uint4*>(zero), (int)(zero_bytes / 16), *fill, groups);
  } else {
    hipLaunchKernelGGL(norm_finalize_kernel<NoFill>, dim3(groups), dim3(kEwThreads), 0, s, stat, partials, scales, list,
                       eps, per_mat, apart ? 0 : 1, static_cast<uint4*>(zero), (int)(zero_bytes / 16), NoFill{}, groups);
  }
  if (apart) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rescue_kernel, dim3(1024), dim3(kEwThreads), 0, s, stat, scales, list, count);
  }
  return hipGetLastError();
}

hipError_t launch_single_prepare(const MatStatic& ms, const MatDynamic& md, void* o_ptr, MatStatic* stat,
                                 MatDynamic* dyn, void** o_ptrs, BlockWork* work, int num_blocks, int32_t* members,
                                 int32_t* order, MatScale* scale, void* zero, size_t zero_bytes, hipStream_t s) {
  const size_t n16 = zero_bytes / 16;   // carved in multiples of 256 bytes
  size_t blocks = ((size_t)num_blocks > n16 ? (size_t)num_blocks : n16) / 256 + 1;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(single_prepare_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ms, md, o_ptr, stat, dyn, o_ptrs,
                     work, num_blocks, members, order, scale, static_cast<uint4*>(zero), n16);
  return hipGetLastError();
}

hipError_t launch_plain_update(const MatStatic* stat, const MatDynamic* dyn, const MatScale* scales,
                               const BlockWork* work, int num_blocks, void* const* o_ptrs, float lr, float wd,
                               float gamma_coeff, int store_o, hipStream_t s) {
  if (num_blocks <= 0) return hipSuccess;
  // one launch per parameter dtype; blocks of the other dtype return at once
  hipLaunchKernelGGL((plain_update_kernel<float>), dim3(num_blocks), dim3(kEwThreads), 0, s, stat, dyn, scales,
                     work, o_ptrs, lr, wd, gamma_coeff, store_o, 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((plain_update_kernel<bf16_t>), dim3(num_blocks), dim3(kEwThreads), 0, s, stat, dyn, scales,
                     work, o_ptrs, lr, wd, gamma_coeff, store_o, 1);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  const size_t n16 = bytes / 16;   // the arena is carved in multiples of 256 bytes
  const int blocks = (int)((n16 + 255) / 256 < 8192 ? (n16 + 255) / 256 : 8192);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, static_cast<uint4*>(p), n16);
  return hipGetLastError();
}

}  // namespace mona
