// Transitions grouped by target, visited by `waves` waves one after the other.
#include "grouped_dev.h"

extern "C" void visit(uint32_t n, const uint32_t* in_ptr, uint32_t waves, uint32_t* target,
                      uint32_t* visits) {
  for (uint32_t w = 0; w < waves; ++w)
    lanes::run(64, w, [&]() {
      bisim::each_in_transition(n, in_ptr, w, waves, [&](uint32_t t, uint32_t e) {
        target[e] = t;
        ++visits[e];
      });
    });
}
