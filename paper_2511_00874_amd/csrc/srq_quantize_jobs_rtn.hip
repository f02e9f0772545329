// Quantization jobs with round-to-nearest among them, in a translation unit of their own (compile time).
#include "srq_quantize_jobs.hpp"

namespace srq {

hipError_t launch_jobs_to_nearest(const QuantJobs& jobs, uint32_t blocks, bool cached, bool mixed, hipStream_t stream) {
  return mixed ? launch_jobs<MODE_MIXED>(jobs, blocks, cached, stream) : launch_jobs<MODE_RTN>(jobs, blocks, cached, stream);
}

}  // namespace srq
