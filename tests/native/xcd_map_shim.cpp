// Host build of the library's workgroup renumbering, for the tests.
#include "xcd_map.h"

extern "C" void shim_xcd_slots(uint32_t nb, uint32_t run, uint32_t *out) {
    for (uint32_t b = 0; b < nb; ++b) out[b] = rcb::xcd_slot(b, nb, run);
}
