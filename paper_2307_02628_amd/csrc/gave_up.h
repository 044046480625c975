// What the host learns of a kernel's bounded wait that ran out (host only, no HIP).
#pragma once
#include <cstdint>

namespace skd {

// A word that the host and the kernels of one state share, zero at first.  A kernel that had to go on without what it waited
// for writes it; what the state holds from then on is not to be used, so nothing sets it back.
struct GaveUp {
  volatile uint32_t *word = nullptr;  // null: the state has no kernels that wait
  bool seen() const { return word && *word != 0; }
};

}  // namespace skd
