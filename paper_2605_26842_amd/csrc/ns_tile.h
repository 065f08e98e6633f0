// What the Newton-Schulz product kernels share: vector types, compile-time loops, the walk over the tiles of a
// batch of equal-shape products, the LDS fragment reads and the counted waits.
#pragma once
#include "mona_internal.h"

#include <type_traits>

namespace mona {
namespace {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// compile-time loop: f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>)
template <int I> struct IC { static constexpr int value = I; constexpr operator int() const { return I; } };
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IC<I>{});
    static_for<N, I + 1>(f);
  }
}

#define MONA_AS1 __attribute__((address_space(1)))
#define MONA_AS3 __attribute__((address_space(3)))
// s_waitcnt vmcnt(n), leaving the other counters alone (gfx9 encoding)
#define MONA_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// ---- tile decode ---------------------------------------------------------------------
constexpr int kBandRows = 6;

struct TileId {
  int mat, ti, tj;
  bool valid;
};

// Workgroup L runs on die L % 8.  Give every die one contiguous range of the logical tile
// order (matrix-major), so that tiles that share operands share that die's L2.
__device__ __forceinline__ TileId decode_logical(const GemmArgs& a, int logical, bool in_range) {
  TileId t;
  const int total = a.tiles_per_mat * a.count;
  t.valid = in_range && logical < total;
  t.mat = logical / a.tiles_per_mat;
  int r = logical - t.mat * a.tiles_per_mat;
  if (a.symmetric) {
    // row block ti holds the column blocks from its diagonal onwards
    int ti = 0, row = a.tiles_n;
    while (r >= row && row > 0) { r -= row; row -= 1; ++ti; }
    t.ti = ti;
    t.tj = ti + r;
  } else {
    // Bands of up to kBandRows tile rows, walked column by column: the 32 workgroups of a die then hold
    // a block of about 6 x 5 tiles at any time, which shares 11 operand panels in the die's L2 instead of
    // the 18 of two full tile rows.
    const int full = a.tiles_m / kBandRows;                 // complete bands
    const int in_full = full * kBandRows * a.tiles_n;
    int rows = kBandRows, first = 0;
    if (r >= in_full) { r -= in_full; rows = a.tiles_m - full * kBandRows; first = full * kBandRows; }
    else { const int b = r / (kBandRows * a.tiles_n); r -= b * kBandRows * a.tiles_n; first = b * kBandRows; }
    t.tj = r / rows;
    t.ti = first + (r - t.tj * rows);
  }
  return t;
}

}  // namespace
}  // namespace mona
