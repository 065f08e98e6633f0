// The part of the HIP runtime that libmona's host code calls, on host memory, so that what it enqueues can be followed
// without a GPU: "device" pointers are host pointers, the kernels that move pointers are carried out, launches of
// all of them are handed to a callback, captured work is kept and carried out by replay().
#pragma once
#include "../../paper_2605_26842_amd/csrc/mona_internal.h"

#include <functional>
#include <string>
#include <vector>

namespace fake {
struct Launch {
  std::string name;      // kernel name, mangled
  unsigned grid, block;
  void** args;           // valid during the callback only
};
extern std::function<void(const Launch&)> on_launch;   // called when a launch is carried out (not when it is recorded)
extern bool capturing;                                 // all streams but the null stream
extern std::string fail;                               // what to fail once: "copy", "attribute" or a piece of a kernel's name
extern int capability_major, capability_minor;         // of the device (those of none that exists, unless a test says so)
extern int device;                                     // the current device
extern int queries;                                    // what was asked of the devices so far
struct Array { const void* source; size_t bytes; };              // a static device array and the source it belongs to
std::vector<Array>& arrays();
void replay();                                         // carries out what was recorded since capturing was set
void clear_recorded();
}  // namespace fake
