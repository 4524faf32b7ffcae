// Pinned host buffers that kernels write the results of small reads to: a
// context takes one at its first read and gives it back at its end, for the
// next context of its device (at most kIdlePins lie idle, 2 MiB of host memory,
// until the process ends; safe from several threads).  Allocating one took 32 us
// of a context's first read, and freeing it 45 us of its end.
#pragma once
#include <cstddef>
#include <cstdint>

namespace micsa {

constexpr size_t kPinBytes = (size_t)256 << 10, kPinHead = 64;  // results, and what lies before them
constexpr size_t kIdlePins = 8;

uint8_t* take_pin(int device);           // null: no pinned memory
void give_pin(int device, uint8_t* pin);  // no kernel writes to it any more

}  // namespace micsa
