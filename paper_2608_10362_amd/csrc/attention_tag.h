// Tags of the long-context attention's partial words, from the handle's pass
// count (no HIP needed: the arithmetic also compiles on the host).
#pragma once

#include <stdint.h>

namespace specdec {

// The pass count runs 0 .. P-1, P = (2^32 - 1) / n_layers, and starts over; a
// launch of layer l in pass p is tagged p * n_layers + l + 1.  So P * n_layers
// launches in a row (nearly 2^32) have different tags, and none has tag 0, which
// the zeroed words of a new handle hold.
constexpr uint32_t attention_pass_after(uint32_t pass, uint32_t n, uint32_t n_layers) {  // (n < P)
  return n < 0xffffffffu / n_layers - pass ? pass + n : pass - (0xffffffffu / n_layers - n);
}
constexpr uint32_t attention_tag(uint32_t pass, uint32_t n_layers, uint32_t layer) {
  return pass * n_layers + layer + 1u;
}

}  // namespace specdec
