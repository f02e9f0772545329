// The operand quantizers that write byte codes turned, rounding stochastically: of a forward pass that also saves its operands as 8-bit floats for
// the backward pass (every element of A and W goes through two quantizers, its integer code is written as the source lies), and of a
// backward pass (an output gradient in both layouts; A and W, turned only).  (Such launches of quantize_jobs_kernel, by conversion and by permutes; a
// kernel of its own because that one's registers have no room for it.)
//
// What bounds it is the vector ALU, one or two Philox blocks for eight elements, beside the loads.  The stochastic conversions
// (quantize_octet) take a third of the ALU work off, less where a tensor holds subnormals of the grid; codes go to LDS four at a time instead
// of one, and the same-layout codes leave in pieces of 8 bytes.  us, before and now:
//   two quantizers, E5M2 and E4M3 of normal tensors / E4M3 of an activation with 1 % of outliers / of one over 40 binades: GPT-2's second
//   linear (8192 x 3072 and 768 x 3072, 165 MB) 39.3 -> 32.3, 39.9 -> 33.0 / 39.7 -> 34.4 / 39.0 -> 35.2; 1008 x 768 and 3072 x 768
//   9.2 -> 6.6, 9.4 -> 6.8 / 9.4 -> 6.9 / 9.2 -> 6.8; 4096 x 2048 and 2048 x 2048 20.3 -> 16.5, 21.1 -> 16.9 / 20.0 -> 17.2 / 20.0 -> 17.1;
//   one quantizer in both layouts, E5M2, binary32 and bfloat16: 4096 x 2048 11.8 -> 10.3, 11.6 -> 9.2; 8192 x 2048 23.0 -> 19.1, 18.5 ->
//   14.3; 8192 x 3072 28.5 -> 27.1, 26.3 -> 21.4; 65536 x 256 20.8 -> 19.0, 19.9 -> 15.9; the three of a backward call, 1008 x 3072 and
//   3072 x 3072 16.7 -> 13.5, 8192 x 2048 and 2048 x 2048 38.6 -> 33.2, 16384 x 1024 and 1024 x 1024 35.4 -> 35.5 (bfloat16 16.6 -> 12.4,
//   35.9 -> 24.9, 31.9 -> 24.3).  E4M3 within 2 % of these.  Integers in both layouts, int8, binary32 and bfloat16: 2048 x 2048 8.9 -> 8.6,
//   9.0 -> 8.6; 4096 x 2048 10.6 -> 10.0, 10.0 -> 8.7; 8192 x 2048 22.0 -> 19.2, 16.1 -> 13.7; 15360 x 2048 37.2 -> 32.7, 32.1 -> 25.3.
//   Not so many binary32 rows 16 or 32 KiB apart (turn_strided).
// Not for large tensors (65536 x 2048, rows a power of two apart, int4 108 -> 143), nor two integer quantizers: they take 68 registers, and within
// 64 they spill (8192 x 2048 26.4 -> 26.6, 16384 x 1024 23.9 -> 27.9).
#include <cstddef>
#include <type_traits>

#include "srq_device.hpp"
#include "srq_internal.hpp"

namespace srq {
namespace {

constexpr int QBLOCK = 256;
constexpr uint32_t TC = 64, TR = TURN_TILE_ROWS;  // tile: TR source rows x TC source columns
constexpr uint32_t PITCH = TR + 4;                // the words a wave instruction writes to LDS fall on all 64 banks
constexpr uint32_t BAND_GROUP = 32;               // tile order as there

// The descriptor of a workgroup's job, in the kernel-argument segment (constant address space, scalar loads).  `again`: the fields that
// are used of it are loaded here and not kept from an earlier read (40 scalar registers of them do not fit beside the rest).
typedef __attribute__((address_space(4))) const uint32_t* job_words;
struct alignas(8) RawJob {
  uint32_t w[sizeof(QuantJob) / 4];
};
static_assert(sizeof(QuantJob) % 4 == 0 && offsetof(QuantJobs, job) % 4 == 0, "descriptor is read word-wise");
__device__ __forceinline__ QuantJob read_job(job_words at, bool again = false) {
  uint64_t a = (uint64_t)at;
  if (again) asm volatile("" : "+s"(a));
  const job_words p = (job_words)a;
  RawJob raw;
#pragma unroll
  for (unsigned k = 0; k < sizeof(QuantJob) / 4; ++k) raw.w[k] = p[k];
  return __builtin_bit_cast(QuantJob, raw);
}

// A value that is the same in all lanes, in scalar registers.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
  return (uint64_t)uniform((uint32_t)(v >> 32)) << 32 | uniform((uint32_t)v);
}
__device__ __forceinline__ InvScale uniform(InvScale s) {
  s.inv = __uint_as_float(uniform(__float_as_uint(s.inv)));
  s.inv16 = __uint_as_float(uniform(__float_as_uint(s.inv16)));
  return s;
}
// A pointer that is the same in all lanes, as the scalar base of an access whose 32-bit offset differs by lane.
template <class T>
__device__ __forceinline__ global_ptr<T> uniform_ptr(T* p) {
  uint64_t a = uniform((uint64_t)p);
  asm("" : "+s"(a));  // (or the sum is formed per lane)
  return (global_ptr<T>)a;
}

// A thread takes pieces of four neighbouring rows, neighbours in the output, so that codes go to LDS a word at a time, and loads a row of
// the next piece as soon as the present one has left its registers; the stores of a piece go out after those loads (a wave waits for
// loads and stores in the order they were issued).  The two steps are written out, one with those loads and one without: in a loop the
// compiler sees loads in flight at its end, too, and where the registers of the LDS reads fall together with theirs it waits
// for everything, the stores that write through included (8192 x 3072 and 768 x 3072 34.8 instead of 33.1 us).
// binary32: 4 columns; lanes L and L + 32 hold the two halves of each Philox group, so that a swap of wave halves hands out the random
// words of two rows and another one makes 8-byte pieces of the integer codes.  bfloat16: 8 columns, a group a row.
enum Second { SECOND_INT, SECOND_SAME, SECOND_NONE };  // what is written as the source lies: integer codes, the same codes, nothing
template <int KIND, bool F32, Second SECOND, bool CACHED>
__device__ __forceinline__ void turn_tile(job_words job, uint32_t local, uint8_t* tile) {
  const QuantJob j = read_job(job);
  const uint32_t tiles_x = (j.cols + TC - 1) / TC, tiles_y = (j.rows + TR - 1) / TR;
  const uint32_t band0 = local / (BAND_GROUP * tiles_x) * BAND_GROUP, within = local - band0 * tiles_x;
  const uint32_t bands = min(BAND_GROUP, tiles_y - band0);
  const uint32_t r0 = (band0 + within % bands) * TR, c0 = (within / bands) * TC;
  const uint32_t rows = j.rows, cols = j.cols;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, half = F32 ? lane >> 5 : 0u;
  constexpr uint32_t STEP = F32 ? 64 : 128;  // rows of the tile that the workgroup takes at a time
  const uint32_t cl = (lane & 7u) * 8 + half * 4, rl = F32 ? wave * 16 + ((lane >> 3) & 3u) * 4 : wave * 32 + (lane >> 3) * 4;
  using load_t = typename std::conditional<F32, f32x4, u32x4>::type;
  constexpr uint32_t ES = F32 ? 4 : 2;  // bytes of a source element
  // Addresses: a uniform part per row, and an offset of this lane below 2^32 (tiles of TR rows are for less than 2048 tiles of
  // twice the height, so less than 131072 columns)
  const size_t e_tile = (size_t)r0 * cols + c0;
  const uint32_t src_off = (rl * cols + cl) * ES, group_off = ((rl + half) * cols + cl) / 8;  // upper lanes draw for the row after
  // rows % 16 == 0 and cols % 16 == 0: a piece is inside or outside as a whole, and so is the group of a quad.  The first four
  // rows of a step are inside: lanes outside load the first element of those.
  const bool col_ok = c0 + cl < cols;
  load_t v[4];
  auto load = [&](uint32_t r, int i) {
    const uint32_t off = opaque(col_ok && r0 + rl + r < rows ? src_off : 0u);  // (not kept as 64 bits)
    v[i] = load_source<CACHED>(reinterpret_cast<global_ptr<const load_t>>(
        uniform_ptr(static_cast<const uint8_t*>(j.x) + (e_tile + (size_t)(r + i) * cols) * ES) + off));
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) load(0, i);
  // (the first loads are under way before the scales are waited for)
  const InvScale inv = uniform(inv_scale(j.scale, j.scale_dev, j.kind));
  const uint64_t ctr = uniform(first_block(j.counter_offset, j.counter_dev));
  InvScale inv2 = inv;
  uint64_t ctr2 = 0;
  if constexpr (SECOND == SECOND_INT) {
    inv2 = uniform(inv_scale(j.scale2, j.scale_dev2, j.kind2));
    ctr2 = uniform(first_block(j.counter_offset2, j.counter_dev2));
  }
  const uint32_t steps_end = min(TR, rows - r0);
  auto step = [&](uint32_t r, auto more) __attribute__((always_inline)) {
    const bool inside = col_ok && r0 + rl + r < rows;
    const QuantJob p = read_job(job, true);
    const uint32_t k0 = (uint32_t)p.seed, k1 = (uint32_t)(p.seed >> 32), m0 = (uint32_t)p.seed2, m1 = (uint32_t)(p.seed2 >> 32);
    const size_t group_step = (e_tile + (size_t)r * cols) / 8;
    const uint32_t gstep = cols / 8;  // groups of a row
    uint8_t* const dst = tile + cl * PITCH + rl + r;
    if constexpr (F32) {
      uint32_t c[4], out2[4];
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        __builtin_amdgcn_sched_barrier(0);  // (two pairs of rows at once would take more than 64 registers)
        const size_t group = group_step + (size_t)i * gstep;  // with group_off: of row i (lower lanes) or i + 1 (upper lanes)
        const float x[4] = {v[i].x, v[i].y, v[i].z, v[i].w}, y[4] = {v[i + 1].x, v[i + 1].y, v[i + 1].z, v[i + 1].w};
        uint32_t w[4];
        round_words_of_pair(ctr + group + group_off, k0, k1, w);
        const u32x2 q = quantize_octet<KIND>(x, y, inv, w, true);
        c[i] = q.x;
        c[i + 1] = q.y;
        if constexpr (SECOND == SECOND_INT) {
          round_words_of_pair(ctr2 + group + group_off, m0, m1, w);
          const u32x2 q2 = quantize_octet<SRQ_INTX>(x, y, inv2, w, true);
          out2[i] = q2.x;
          out2[i + 1] = q2.y;
        } else {
          out2[i] = q.x;
          out2[i + 1] = q.y;
        }
        if constexpr (more.value) {
          load(r + STEP, i);
          load(r + STEP, i + 1);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < (SECOND == SECOND_NONE ? 0 : 4); i += 2) {
        swap_halves(out2[i], out2[i + 1]);  // this lane: the whole group of its row
        const global_ptr<uint8_t> o = uniform_ptr(p.out2 + (group_step + (size_t)i * gstep) * 8) + group_off * 8;
        const u32x2 q2 = {out2[i], out2[i + 1]};
        if (inside) store_through8(o, q2);
      }
      uint32_t q[4];
      turn4x4(c[0], c[1], c[2], c[3], q);
#pragma unroll
      for (int e = 0; e < 4; ++e) *reinterpret_cast<uint32_t*>(dst + e * PITCH) = q[e];
    } else {
      u32x2 c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        const size_t group = group_step + (size_t)i * gstep;
        float f[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f[2 * e] = bf16_to_f32(v[i][e] & 0xFFFFu);
          f[2 * e + 1] = bf16_to_f32(v[i][e] >> 16);
        }
        c[i] = quantize_group_words<KIND>(f, inv, ctr + group + group_off, k0, k1, true);
        u32x2 q2 = c[i];
        if constexpr (SECOND == SECOND_INT) q2 = quantize_group_words<SRQ_INTX>(f, inv2, ctr2 + group + group_off, m0, m1, true);
        if (SECOND != SECOND_NONE && inside) *reinterpret_cast<global_ptr<u32x2>>(uniform_ptr(p.out2 + group * 8) + group_off * 8) = q2;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t q[4];
        turn4x4(c[0][h], c[1][h], c[2][h], c[3][h], q);
#pragma unroll
        for (int e = 0; e < 4; ++e) *reinterpret_cast<uint32_t*>(dst + (4 * h + e) * PITCH) = q[e];
      }
    }
  };
  static_assert(STEP == TR || 2 * STEP == TR, "one step or two");
  uint32_t r = 0;
  if constexpr (STEP < TR) {
    if (steps_end > STEP) {
      step(0u, std::true_type{});
      r = STEP;
    }
  }
  step(r, std::false_type{});
  __syncthreads();
  const QuantJob o = read_job(job, true);
#pragma unroll
  for (uint32_t it = 0; it < TC * TR / 16 / QBLOCK; ++it) {
    const uint32_t id = it * QBLOCK + threadIdx.x, ch = id % (TR / 16), cc = id / (TR / 16);
    const uint32_t col = c0 + cc, row = r0 + ch * 16;
    if (col >= o.cols || row >= o.rows) continue;  // rows % 16 == 0
    const uint32_t* const src = reinterpret_cast<const uint32_t*>(tile + cc * PITCH + ch * 16);
    const u32x4 w = {src[0], src[1], src[2], src[3]};
    uint8_t* const dst = o.out + (size_t)col * o.rows + row;
    store_through16(dst, w);
  }
}

template <int KIND, bool CACHED>
__device__ __forceinline__ void turn_job(const QuantJob& j, job_words job, uint32_t local, uint8_t* tile) {
  if (Grid<KIND>::is_float && j.out2 && j.kind2) {  // (two of integers take 68 registers)
    if constexpr (Grid<KIND>::is_float) {
      if (j.dtype == SRQ_F32) turn_tile<KIND, true, SECOND_INT, CACHED>(job, local, tile);
      else turn_tile<KIND, false, SECOND_INT, CACHED>(job, local, tile);
    }
  } else if (j.out2) {
    if (j.dtype == SRQ_F32) turn_tile<KIND, true, SECOND_SAME, CACHED>(job, local, tile);
    else turn_tile<KIND, false, SECOND_SAME, CACHED>(job, local, tile);
  } else {
    if (j.dtype == SRQ_F32) turn_tile<KIND, true, SECOND_NONE, CACHED>(job, local, tile);
    else turn_tile<KIND, false, SECOND_NONE, CACHED>(job, local, tile);
  }
}

// (Two quantizers was all it took at first, hence the name.)  At most 64 registers: a wave fits on a SIMD beside two of the persistent product kernel.
template <bool CACHED>
__global__ __launch_bounds__(QBLOCK) void quantize_dual_kernel(QuantJobs jobs) {
  __shared__ __attribute__((aligned(16))) uint8_t tile[TC * PITCH];
  int ji = 0;
#pragma unroll
  for (int i = 1; i < QUANT_JOBS_MAX; ++i)
    if (i < jobs.njobs && blockIdx.x >= jobs.job[i].first_block) ji = i;
  const job_words job = (job_words)__builtin_amdgcn_kernarg_segment_ptr() +  // the explicit arguments start at offset 0
                        (offsetof(QuantJobs, job) + (size_t)ji * sizeof(QuantJob)) / 4;
  const QuantJob j = read_job(job);
  const uint32_t local = blockIdx.x - j.first_block;
  if (j.kind == SRQ_E5M2) turn_job<SRQ_E5M2, CACHED>(j, job, local, tile);
  else if (j.kind == SRQ_E4M3) turn_job<SRQ_E4M3_CONV, CACHED>(j, job, local, tile);
  else turn_job<SRQ_INTX, CACHED>(j, job, local, tile);
}

}  // namespace

hipError_t launch_quantize_turned(const QuantJobs& jobs, uint32_t blocks, bool cached, hipStream_t stream) {
  if (cached) quantize_dual_kernel<true><<<blocks, QBLOCK, 0, stream>>>(jobs);
  else quantize_dual_kernel<false><<<blocks, QBLOCK, 0, stream>>>(jobs);
  return hipGetLastError();
}

}  // namespace srq
