// k_scan_any for fp32 storage with registers for 4 waves per SIMD.
#define COREY_SCAN_ANY_HERE
#include "corey_scan_impl.h"

namespace corey_scan {
COREY_SCAN_ANY(, float, 4)
}  // namespace corey_scan
