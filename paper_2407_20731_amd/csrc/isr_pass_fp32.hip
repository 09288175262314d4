// Streaming passes and the persistent batch kernel instantiated for the
// FP32 transform path.
#include "isr_batch.cuh"
#include "isr_engine.cuh"
#include "isr_engine_l.cuh"
#include "isr_passes.cuh"

namespace isr {

hipError_t launch_pass_fp32(int kind, const Job& j, int grid, hipStream_t s, void* extra, int extra_i) {
  return launch_pass_prec<P_FP32>(kind, j, grid, s, extra, extra_i);
}

int resident_fp32(int kind, int order) { return resident_prec<P_FP32>(kind, order); }

hipError_t launch_batch_fp32(const BatchCtl& B, int grid, size_t lds, hipStream_t s) {
  return launch_batch_prec<P_FP32>(B, grid, lds, s);
}

size_t batch_lds_fp32() { return batch_lds_prec<P_FP32>(); }

int batch_resident_fp32(size_t lds) { return batch_resident_prec<P_FP32>(lds); }

hipError_t launch_fast_fp32(int kind, const Job& j, int gx, hipStream_t s) {
  if (j.order > FAST_MAX_ORDER) return launch_fast_l<P_FP32>(kind, j, gx, s);
  return launch_fast_prec<P_FP32>(kind, j, gx, s);
}

hipError_t launch_decomp_wave_fp32(const Job& j, int gx, int cus, hipStream_t s, void* out, int out_fp64) {
  if (j.order > FAST_MAX_ORDER) {
    // (one grid over the elements of every component)
    const long long all = (j.n_elem * j.ncomp + 3) / 4, most = (long long)cus * 8;
    return launch_decompL_prec<P_FP32>(j, (int)(all < most ? all : most), s, out, out_fp64);
  }
  return launch_decompW_prec<P_FP32>(j, gx, cus, s, out, out_fp64);
}

int resident_fast_fp32(int kind, int order) {
  return order > FAST_MAX_ORDER ? resident_fast_l<P_FP32>(kind, order) : resident_fast_prec<P_FP32>(kind, order);
}

}  // namespace isr
