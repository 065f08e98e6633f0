// Buffers of chains whose products have one each (ns_chain_kernel).
#include "mona_internal.h"

#include <algorithm>
#include <mutex>

namespace mona {

namespace {

// The caller's arena holds two X and two p x p matrices to a matrix, which the products of a chain take in turn.  Where every product
// is to have a buffer of its own (ns_chain_kernel), the others come from a static array, of which every GPU the library runs on
// holds its own copy, like the one of mona_step_noalloc.  A state takes its part when it is built and gives it back when it is
// freed, unless a step of it has been captured: a graph may be replayed later on, on the arena that is the caller's, and its launches
// name the part.  A state that finds no room runs its chains with flags.  256 x 512 takes 2.3 MB, nine ragged matrices 14.
// (A source of its own: a static array takes its memory with the first use of any array or kernel of its source, and mona_step_noalloc needs
// its own only.)
constexpr size_t kPoolBytes = (size_t)128 << 20, kPoolUnit = (size_t)1 << 18;
constexpr int kPoolUnits = (int)(kPoolBytes / kPoolUnit);
static __device__ __align__(256) unsigned char chain_pool[kPoolBytes];
// A part that was given back may still be in use by steps on their way, on streams that this side does not know.
enum : uint8_t { UNIT_FREE = 0, UNIT_TAKEN = 1, UNIT_GIVEN_BACK = 2 };
struct Pool {
  char* base = nullptr;              // device address, looked up once
  uint8_t unit[kPoolUnits] = {};
};
std::mutex g_pool_mu;
Pool g_pool[kMaxDevices];

char* find_room(Pool& pool, int units) {
  for (int run = 0, i = 0; i < kPoolUnits; ++i) {
    run = pool.unit[i] == UNIT_FREE ? run + 1 : 0;
    if (run < units) continue;
    const int first = i + 1 - units;
    std::fill_n(pool.unit + first, units, (uint8_t)UNIT_TAKEN);
    return pool.base + (size_t)first * kPoolUnit;
  }
  return nullptr;
}

}  // namespace

// (a device without the array, or no room: nullptr, and no error)
char* take_from_pool(int device, size_t bytes) {
  const int units = (int)((bytes + kPoolUnit - 1) / kPoolUnit);
  if (device < 0 || device >= kMaxDevices || units < 1 || units > kPoolUnits) return nullptr;
  std::lock_guard<std::mutex> lock(g_pool_mu);
  Pool& pool = g_pool[device];
  if (!pool.base) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(chain_pool)) != hipSuccess || !p) { (void)hipGetLastError(); return nullptr; }
    pool.base = static_cast<char*>(p);
  }
  if (char* at = find_room(pool, units)) return at;
  if (std::find(pool.unit, pool.unit + kPoolUnits, (uint8_t)UNIT_GIVEN_BACK) == pool.unit + kPoolUnits) return nullptr;
  // freeing pinned memory waits for the device, and so for every step of a state that was freed
  void* mark = nullptr;
  if (hipHostMalloc(&mark, 64, hipHostMallocDefault) != hipSuccess || hipHostFree(mark) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  std::replace(pool.unit, pool.unit + kPoolUnits, (uint8_t)UNIT_GIVEN_BACK, (uint8_t)UNIT_FREE);
  return find_room(pool, units);
}
void give_back(int device, const char* at, size_t bytes) {
  std::lock_guard<std::mutex> lock(g_pool_mu);
  Pool& pool = g_pool[device];
  std::fill_n(pool.unit + (at - pool.base) / kPoolUnit, (bytes + kPoolUnit - 1) / kPoolUnit, (uint8_t)UNIT_GIVEN_BACK);
}

}  // namespace mona
