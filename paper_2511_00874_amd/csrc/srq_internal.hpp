// Launchers shared between the translation units of the library (host side).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/srq.h"
#include "srq_plan.hpp"

namespace srq {

// How a quantize launch stores its codes.
enum StoreMode {
  STORE_BYTE = 0,   // one byte per element (INT4 values sign-extended to the byte)
  STORE_NIBBLE = 1, // INT4 only: two elements per byte along the output's contiguous dim
  STORE_BF16 = 2    // the grid value itself as bfloat16 (two bytes per element)
};

// Cached or streaming loads of a source.  The scale of a tensor is found in one pass over it and its codes are made
// in another; whether the second pass finds the tensor in the last-level cache (256 MiB) depends on all that is touched in
// between, so both rules count a whole layer, not a tensor.
//   - An absmax call whose tensors take up to ABSMAX_CACHED_BYTES together reads them with cached loads: what it leaves is
//     found by cached and streaming loads alike.  Beyond, what it reads first is gone by the end and cached loads
//     only push out what the next kernels want.
//   - A quantizer launch reads with cached loads if A, W and Y or dY of its layer take up to JOBS_CACHED_BYTES together
//     (those it does not read counted as binary32): then the tensor is there again for the next pass, and the operands
//     fit beside it.  Beyond, streaming loads find what is there and leave the room to the codes and results.
// Training steps (scales of A and W, forward, scale of dY, backward), us with everything streamed, with both rules, and
// with cached absmax loads alone: 1024 x 2048 x 2048 (20 MiB a layer) 74.5, 71.3, 72.3; 2048 x 2048 x 2048 (40) 87.5, 82.6, 84.3;
// 4096 x 2048 x 2048 (72; absmax calls 40 and 32) 128.6, 124.7, 124.7, and 128 with cached quantizer loads; 16384 x 512 x
// 2048 (162) 185.9, 185.5, and 196 where the 32 MiB dY alone is read with cached loads by both passes; 6144 x 2048 x 2048 170.9, 168.5.
constexpr size_t ABSMAX_CACHED_BYTES = (size_t)88 << 20;
constexpr size_t JOBS_CACHED_BYTES = (size_t)56 << 20;
inline size_t source_bytes(size_t n, int dtype) { return n * (dtype == SRQ_F32 ? 4 : 2); }

// A value (a lane or thread index) as one the optimiser cannot see through.  Address arithmetic that is derived from it
// inside a loop is recomputed there (a few VALU operations) instead of being hoisted out of the loop and held in
// registers across it.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

struct QuantArgs {
  int kind, round, dtype, store;
  float scale;
  const float* scale_dev;
  uint64_t seed, counter_offset;
  const uint64_t* counter_dev;  // if not null: its value is added to counter_offset on the device
};

// codes: rows x cols (transpose_out = 0) or cols x rows (1), one byte each, INT4 two per byte.  Shapes already validated.
hipError_t launch_quantize(void* codes, const void* x, size_t rows, size_t cols, int transpose_out,
                           const QuantArgs& a, hipStream_t stream);

// Several quantizations in one launch (the operands of a product; in the fused backward pass
// the output gradient in both layouts).
constexpr int QUANT_JOBS_MAX = 3;
struct QuantJob {
  const void* x;
  uint8_t* out;    // rows x cols codes, or cols x rows when transpose
  uint8_t* out2;   // transpose only: optional extra rows x cols output, else nullptr:
                   //   kind2 == 0: the same codes again, in the source layout
                   //   kind2 == SRQ_INT8 / SRQ_INT4: the byte codes of a second, integer quantizer of the
                   //   same tensor (its own scale, rounding mode and stream position), source layout
  uint32_t rows, cols;
  int kind, round, dtype, store, transpose;
  float scale;
  const float* scale_dev;
  uint64_t seed, counter_offset;
  const uint64_t* counter_dev;   // if not null: its value is added to counter_offset on the device
  int kind2, round2;
  float scale2;
  const float* scale_dev2;
  uint64_t seed2, counter_offset2;
  const uint64_t* counter_dev2;
  // SRQ_INT4 from a binary32 source, transposing jobs: write the transposed output (pack_t) or the
  // same-codes output in the source layout (pack_2, kind2 == 0) two values per byte, in the form
  // gemm_takes_packed_x describes (runs of 16 along rows, respectively along columns)
  int pack_t, pack_2;
  uint32_t first_block, nblocks;  // filled by the launcher
};
struct QuantJobs {
  int njobs;
  size_t other_bytes = 0;  // of the layer's tensors that this launch does not read, in binary32 (for the load policy)
  QuantJob job[QUANT_JOBS_MAX];
};
hipError_t launch_quantize_jobs(QuantJobs& jobs, hipStream_t stream);
// Those of them whose jobs are all of one sort, which has a kernel of its own (srq_quantize_dual.hip): byte codes turned, rounding
// stochastically, in tiles of TURN_TILE_ROWS rows, alone, with the same codes as the source lies, or (8-bit floats) with the codes of a
// second, integer quantizer that rounds stochastically.  Not the E4M3 sub-grids, nor 4-bit values two per byte.
constexpr uint32_t TURN_TILE_ROWS = 128;
hipError_t launch_quantize_turned(const QuantJobs& jobs, uint32_t blocks, bool cached, hipStream_t stream);

// Several per-tensor scales in two launches: up to ABSMAX_MAX distinct tensors and
// ABSMAX_MAX scales (a tensor may feed several formats).
constexpr int ABSMAX_MAX = 8;
struct AbsmaxBatch {
  int ntensors, nouts;
  const void* x[ABSMAX_MAX];
  size_t n[ABSMAX_MAX];
  int dtype[ABSMAX_MAX];
  int cached;  // the load policy, filled by the launcher
  uint32_t first_block[ABSMAX_MAX], nblocks[ABSMAX_MAX];
  int out_tensor[ABSMAX_MAX], out_kind[ABSMAX_MAX];
  float out_qmax[ABSMAX_MAX];
  float* out[ABSMAX_MAX];
  uint32_t* partial;  // one word per launched block
};
size_t absmax_batch_plan(AbsmaxBatch& b);  // fills first_block / nblocks, returns the block count
hipError_t launch_absmax_batch(AbsmaxBatch& b, hipStream_t stream);

// Eq. 10 on bfloat16 weights, in place: w[i] <- Q(w[i] - eta * g[i]); element i takes slice i of
// the Philox stream that starts counter_offset blocks in.
hipError_t launch_update_bf16(uint16_t* w, const float* g, float eta, size_t n, int round, uint64_t seed,
                              uint64_t counter_offset, hipStream_t stream);

hipError_t launch_absmax_scale(float* scale_out_dev, const void* x, int dtype, size_t n, int kind,
                               hipStream_t stream);

// out[P][Q] = alpha_scale * sum_r X[p][r] Z[q][r] (+ out if accumulate); alpha_scale =
// alpha * (*sx_dev or sx) * (*sz_dev or sz), computed on the device in binary32.
struct GemmScale {
  float alpha;
  float sx, sz;
  const float* sx_dev;
  const float* sz_dev;
};
// R is the contraction length in elements; operand rows hold R bytes, or 2 R bytes (PIPE_BF16).
size_t gemm_workspace_bytes(size_t P, size_t Q, size_t R, int pipe);
// operand matrices must stay below 2 GiB (32-bit buffer offsets with an out-of-range sentinel)
bool gemm_operands_addressable(size_t P, size_t Q, size_t R, int pipe);
// pitch: bytes between consecutive operand rows (both operands), >= the row length.
// The sum of the contraction slices of a product (fixed order, then scale): run by the product's
// own launcher, or left to the caller (`defer`) who hands it to a LATER product launch (`carry`)
// whose last workgroups then do it -- memory-bound work beside the tiles of an unrelated product
// instead of a launch of its own.  total == 0: nothing to sum.
struct SliceSum {
  const uint32_t* partial;  // nsplit x total raw accumulators
  float* out;
  uint32_t nsplit;
  size_t total;
  GemmScale s;
  int accumulate, is_int;
};
// Which product of a layer a launch is.  It has a say in the kernel form, and in binary32 the form decides the order of a sum: a
// product must have the same role in every entry point that promises its result bit for bit (sr_linear_bwd, sr_linear_bwd_weight
// and sr_linear_bwd_data, the stash and phase calls), whether or not its sum is in fact deferred there.
enum ProductRole {
  ROLE_ANY = 0,
  ROLE_WEIGHT_GRADIENT = 1,  // sr_linear_bwd leaves its slice sum to the launch of the input gradient
  ROLE_INPUT_GRADIENT = 2    // (of either gradient it is known what pair sr_linear_bwd would make of the two)
};
hipError_t launch_gemm_codes(float* out, const uint8_t* X, int kindX, const uint8_t* Z, int kindZ,
                             size_t P, size_t Q, size_t R, size_t pitch, int pipe, const GemmScale& s,
                             bool accumulate, void* workspace, hipStream_t stream, ProductRole role = ROLE_ANY,
                             const SliceSum* carry = nullptr, SliceSum* defer = nullptr, bool x_packed = false,
                             const Plan* plan = nullptr);
// (plan: plan_for of this product, where the caller has it already)
// Both backward products of a layer in one launch where choose_pair says so (`done`; otherwise nothing is launched): the same
// results, bit for bit, as from launch_gemm_codes, the weight gradient with its role.  One byte per element, rows without gaps.
struct PairedProduct {
  float* out;
  const uint8_t *X, *Z;
  int kindZ;
  size_t P, Q, R;
  GemmScale s;
  bool accumulate;
  void* partial;  // room for its slices, as launch_gemm_codes takes it
  Plan plan;      // plan_for of it
};
hipError_t launch_gemm_pair(const PairedProduct& weight, const PairedProduct& data, int kindX, int pipe, hipStream_t stream, bool& done);
// x_packed: X holds 4-bit integers two per byte -- byte j of every 8 holds elements j (low nibble)
// and j + 8 (high nibble) of a run of 16 along the contraction -- in rows of pitch / 2 bytes, and
// s.alpha carries a factor 1/16 (the kernel multiplies 16 * value).  Only where
// gemm_takes_packed_x says so: the int8 pipeline on the 256 x 256 tiles.
bool gemm_takes_packed_x(size_t P, size_t Q, size_t R, int pipe);
// Weight-only objective (Sec. 3.2): out (P x Q) = X . Z^T, X binary32 as it is (P x R), Z bfloat16 (Q x R),
// R % 16 == 0; exact products, binary32 sums.  `partial`: room for slices of the contraction (as many as
// fit; none if partial_bytes is 0).  Operands below 2 GiB each (gemm_operands_addressable).
hipError_t launch_gemm_f32_bf16(float* out, const float* X, const uint16_t* Z, size_t P, size_t Q, size_t R,
                                const GemmScale& s, void* partial, size_t partial_bytes, hipStream_t stream);
// a deferred slice sum that found no later launch to ride on
hipError_t launch_slice_sum(const SliceSum& r, hipStream_t stream);

// Alg. 1 with the quantizers inside the product kernel (srq_fused.hip): out (P x Q) =
// Q(x)[P x R] . Q(z)[Q x R]^T from the source tensors, no codes in memory.  Formats: both integer,
// or both E5M2.
bool fused_pair_supported(int kind_x, int kind_z);
hipError_t launch_fused_fwd(float* out, const void* x, const QuantArgs& qx, const void* z, const QuantArgs& qz,
                            size_t P, size_t Q, size_t R, hipStream_t stream);

inline bool kind_is_int(int k) { return k == SRQ_INT8 || k == SRQ_INT4; }
// 8-bit float codes: E4M3, E5M2 and the sub-grids of E4M3 (stored as E4M3 codes)
inline bool kind_is_f8(int k) { return k >= SRQ_E4M3 && k <= SRQ_E4M0; }

}  // namespace srq
