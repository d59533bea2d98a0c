// k_scan_any for bf16 storage with registers for 4 waves per SIMD.
#define COREY_SCAN_ANY_HERE
#include "corey_scan_impl.h"

namespace corey_scan {
COREY_SCAN_ANY(, uint16_t, 4)
}  // namespace corey_scan
