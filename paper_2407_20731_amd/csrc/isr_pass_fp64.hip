// Streaming passes and the persistent batch kernel instantiated for the
// FP64 transform path.
#include "isr_batch.cuh"
#include "isr_engine.cuh"
#include "isr_passes.cuh"

namespace isr {

hipError_t launch_pass_fp64(int kind, const Job& j, int grid, hipStream_t s, void* extra, int extra_i) {
  return launch_pass_prec<P_FP64>(kind, j, grid, s, extra, extra_i);
}

int resident_fp64(int kind, int order) { return resident_prec<P_FP64>(kind, order); }

hipError_t launch_batch_fp64(const BatchCtl& B, int grid, size_t lds, hipStream_t s) {
  return launch_batch_prec<P_FP64>(B, grid, lds, s);
}

size_t batch_lds_fp64() { return batch_lds_prec<P_FP64>(); }

int batch_resident_fp64(size_t lds) { return batch_resident_prec<P_FP64>(lds); }

hipError_t launch_fast_fp64(int kind, const Job& j, int gx, hipStream_t s) {
  return launch_fast_prec<P_FP64>(kind, j, gx, s);
}

hipError_t launch_decomp_wave_fp64(const Job& j, int gx, int cus, hipStream_t s, void* out, int out_fp64) {
  return launch_decompW_prec<P_FP64>(j, gx, cus, s, out, out_fp64);
}

hipError_t launch_quant_wave(const Job& j, hipStream_t s) { return launch_quantW(j, s); }

int resident_fast_fp64(int kind, int order) { return resident_fast_prec<P_FP64>(kind, order); }

}  // namespace isr
