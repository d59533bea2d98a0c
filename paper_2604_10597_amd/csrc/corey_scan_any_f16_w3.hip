// k_scan_any for fp16 storage with registers for 3 waves per SIMD.
#define COREY_SCAN_ANY_HERE
#include "corey_scan_impl.h"

namespace corey_scan {
COREY_SCAN_ANY(, _Float16, 3)
}  // namespace corey_scan
