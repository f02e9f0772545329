// Launch of a list of quantization jobs (the kernel is in srq_quantize_jobs.hpp).
#include "srq_quantize_jobs.hpp"

namespace srq {

// Requirements (checked by the callers): rows % 16 == 0 and cols % 16 == 0 for every job,
// store is STORE_BYTE or STORE_BF16.
hipError_t launch_quantize_jobs(QuantJobs& jobs, hipStream_t stream) {
  uint32_t first = 0;
  size_t bytes = jobs.other_bytes;
  int sr = 0, nearest = 0;  // quantizers by rounding mode
  for (int i = 0; i < jobs.njobs; ++i) {
    QuantJob& j = jobs.job[i];
    bytes += source_bytes((size_t)j.rows * j.cols, j.dtype);
    (j.round == SRQ_SR ? sr : nearest) += 1;
    if (j.transpose && j.out2 && j.kind2) (j.round2 == SRQ_SR ? sr : nearest) += 1;
    size_t nb;
    if (j.transpose) {
      const size_t tr = tile_rows(j.store == STORE_BF16, j.rows, j.cols);
      nb = (size_t)((j.cols + TC - 1) / TC) * ((j.rows + tr - 1) / tr);
    } else {
      const size_t groups = (size_t)j.rows * j.cols / 8;
      nb = (groups + FLAT_GROUPS_PER_BLOCK - 1) / FLAT_GROUPS_PER_BLOCK;
      if (nb > (1u << 20)) nb = 1u << 20;
    }
    j.first_block = first;
    j.nblocks = (uint32_t)nb;
    first += (uint32_t)nb;
  }
  if (first == 0) return hipSuccess;
  const bool cached = bytes <= JOBS_CACHED_BYTES;
  return nearest == 0 ? launch_jobs<MODE_SR>(jobs, first, cached, stream) : launch_jobs_to_nearest(jobs, first, cached, sr > 0, stream);
}

}  // namespace srq
