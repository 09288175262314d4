// Streaming passes, decompression and quantisation of the FP64 orders 8..15
// (workgroup tiles).
#include "isr_engine_g.cuh"

namespace isr {

hipError_t launch_fast_wide(int kind, const Job& j, int gx, hipStream_t s) { return launch_fast_g(kind, j, gx, s); }

hipError_t launch_decomp_wide(const Job& j, int gx, int cus, hipStream_t s, void* out, int out_fp64) {
  return launch_decomp_g(j, gx, cus, s, out, out_fp64);
}

hipError_t launch_quant_wide(const Job& j, hipStream_t s) { return launch_quant_g(j, s); }

int resident_fast_wide(int kind, int order) { return resident_fast_g(kind, order); }

}  // namespace isr
