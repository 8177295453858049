// Division of small indices by a launch constant, for host and device.
#ifndef PRIEST_QUOTIENT_H_
#define PRIEST_QUOTIENT_H_

#include <cstdint>

namespace priest {

// ceil(2^31 / d): with 31 bits it fits a word for d = 1 too.
constexpr uint32_t inverse_of(uint32_t d) { return 0x7fffffffu / d + 1u; }

// i / d from inv = inverse_of(d): the high half of (2 i) inv.  inv exceeds
// 2^31 / d by less than 1, so that this is exact while i d < 2^31.
constexpr uint32_t quotient(uint32_t i, uint32_t inv) {
  return static_cast<uint32_t>((static_cast<uint64_t>(2u * i) * inv) >> 32);
}

}  // namespace priest

#endif  // PRIEST_QUOTIENT_H_
