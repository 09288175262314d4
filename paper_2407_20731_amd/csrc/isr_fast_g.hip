// Streaming passes of the FP64 orders 8..15 (workgroup tiles).
#include "isr_engine_g.cuh"

namespace isr {

hipError_t launch_fast_wide(int kind, const Job& j, int gx, hipStream_t s) { return launch_fast_g(kind, j, gx, s); }

int resident_fast_wide(int kind, int order) { return resident_fast_g(kind, order); }

}  // namespace isr
