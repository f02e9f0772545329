// Several tensor quantizations in ONE launch, for the linear entry points: the operands of a
// product (and, in the fused backward pass, the output gradient in both layouts at once) are
// independent element-wise jobs (Def. 3), so one grid serves them all and every tensor is
// read once.  A workgroup first finds its job, then runs the same-layout or the transposing
// path for that job's format; format, source dtype and rounding mode are uniform per
// workgroup, so the dispatch is scalar branches.
#pragma once
#include <cstddef>
#include <type_traits>

#include "srq_device.hpp"
#include "srq_internal.hpp"

namespace srq {
namespace {

constexpr int QBLOCK = 256;
constexpr int TC = 64;                  // transposing tile: tile_rows source rows x TC source columns
// Tile rows: 128, or 256 for one-byte codes of a tensor large enough to give every CU several such
// tiles (the same 16.6 KB of LDS as 128 rows of bfloat16 values).  A workgroup then writes 256 bytes
// of every transposed row (128 where two 4-bit values share a byte): whole cache lines.  Small
// tensors keep 128 rows: twice the workgroups (GPT-2 sizes lose 4 % of their step with 256).
__host__ __device__ inline int tile_rows(bool as_bf16, uint32_t rows, uint32_t cols) {
  return !as_bf16 && (size_t)((rows + 255u) / 256u) * ((cols + TC - 1) / TC) >= 2048u ? 256 : 128;
}
constexpr size_t STREAM_OUT_BYTES = 64u << 20;
constexpr int BAND_GROUP = 32;         // row bands whose tiles are walked together (tile order)
static_assert(BAND_GROUP % 8 == 0, "neighbouring column tiles of a band on one XCD");
constexpr int FLAT_GROUPS_PER_BLOCK = QBLOCK * 4;  // sixteen 512-element chunks: four per wave (measured best of 1, 2, 4, 8)

// The descriptor of a workgroup's job, in the kernel-argument segment (constant address space, scalar loads).  Indexing the
// by-value argument would make the compiler copy the whole argument to per-lane scratch memory.
typedef __attribute__((address_space(4))) const uint32_t* job_words;
struct alignas(8) RawJob {
  uint32_t w[sizeof(QuantJob) / 4];
};
static_assert(sizeof(QuantJob) % 4 == 0 && offsetof(QuantJobs, job) % 4 == 0, "descriptor is read word-wise");
// `again`: the fields that are used of it are loaded here and not kept from an earlier read (40 scalar registers of them do
// not fit beside the address arithmetic and the round keys of a transposing job)
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

// Rounding modes of a launch: all stochastic, all to nearest, or told job by job.
enum { MODE_SR, MODE_RTN, MODE_MIXED };
template <int MODE>
__device__ __forceinline__ bool is_sr(int round) {
  return MODE == MODE_SR || (MODE == MODE_MIXED && round == SRQ_SR);
}

template <int KIND, bool AS_BF16, int MODE>
__device__ __forceinline__ void job_quantize_group(uint32_t (&c)[8], const float (&v)[8], const InvScale& inv,
                                                   const QuantJob& j, uint64_t ctr, uint64_t g, uint32_t k0,
                                                   uint32_t k1) {
  if (is_sr<MODE>(j.round)) quantize_group<KIND, SRQ_SR, AS_BF16>(c, v, inv, ctr + g, k0, k1);
  else quantize_group<KIND, SRQ_RTN, AS_BF16>(c, v, inv, 0, 0, 0);
}

// one group, rounded and written to a row-major destination (elements 8 g .. 8 g + 7, all in range)
template <int KIND, bool AS_BF16, int MODE>
__device__ __forceinline__ void put_group(const QuantJob& j, const float (&v)[8], const InvScale& inv, uint64_t ctr, uint64_t g,
                                          uint32_t k0, uint32_t k1) {
  if constexpr (AS_BF16) {
    uint32_t c[8];
    job_quantize_group<KIND, true, MODE>(c, v, inv, j, ctr, g, k0, k1);
    *as_global(reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(j.out) + g * 8)) =
        u32x4{c[0] | (c[1] << 16), c[2] | (c[3] << 16), c[4] | (c[5] << 16), c[6] | (c[7] << 16)};
  } else {
    *as_global(reinterpret_cast<u32x2*>(j.out + g * 8)) = quantize_group_words<KIND>(v, inv, ctr + g, k0, k1, is_sr<MODE>(j.round));
  }
}

__device__ __forceinline__ void widen_bf16(float (&v)[8], const u32x4& raw) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[2 * e] = bf16_to_f32(raw[e] & 0xFFFFu);
    v[2 * e + 1] = bf16_to_f32(raw[e] >> 16);
  }
}

// same layout as the source; rows * cols is a multiple of 8 for the linear entry points.
// binary32 sources go chunk-wise (one fully coalesced 512-element chunk per wave at a time), what is
// left over group-wise.  A group of a bfloat16 source is one 16-byte load: a thread issues four of
// them, a block's width apart, before it rounds the first (11.5 M weights -> int8: 14.0 us, one after
// another 15.6).
template <int KIND, bool AS_BF16, bool CACHED, int MODE>
__device__ __forceinline__ void flat_path(const QuantJob& j, uint32_t local, uint32_t nblocks) {
  const InvScale inv = inv_scale(j.scale, j.scale_dev, j.kind);
  const uint64_t ctr = first_block(j.counter_offset, j.counter_dev);
  const uint32_t k0 = (uint32_t)j.seed, k1 = (uint32_t)(j.seed >> 32);
  const size_t n = (size_t)j.rows * j.cols, ngroups = n / 8;
  if (j.dtype == SRQ_F32) {
    const size_t nchunks = n / CHUNK, waves = (size_t)nblocks * (QBLOCK / 64);
    const float* x = static_cast<const float*>(j.x);
    for (size_t c = (size_t)local * (QBLOCK / 64) + (threadIdx.x >> 6); c < nchunks; c += waves) {
      quantize_chunk_f32<KIND, AS_BF16 ? 2 : 0, CACHED>(j.out, x, c, threadIdx.x & 63u, inv, k0, k1, ctr, is_sr<MODE>(j.round));
    }
    for (size_t g = nchunks * (CHUNK / 8) + (size_t)local * QBLOCK + threadIdx.x; g < ngroups; g += (size_t)nblocks * QBLOCK) {
      float v[8];
      load_group<SRQ_F32, CACHED>(v, j.x, g, n);
      put_group<KIND, AS_BF16, MODE>(j, v, inv, ctr, g, k0, k1);
    }
  } else {
    const u32x4* x = static_cast<const u32x4*>(j.x);
    for (size_t g0 = (size_t)local * FLAT_GROUPS_PER_BLOCK + threadIdx.x; g0 < ngroups;
         g0 += (size_t)nblocks * FLAT_GROUPS_PER_BLOCK) {
      u32x4 raw[FLAT_GROUPS_PER_BLOCK / QBLOCK];
#pragma unroll
      for (int i = 0; i < FLAT_GROUPS_PER_BLOCK / QBLOCK; ++i) {
        const size_t g = g0 + i * QBLOCK;
        raw[i] = load_source<CACHED>(x + (g < ngroups ? g : g0));
      }
#pragma unroll
      for (int i = 0; i < FLAT_GROUPS_PER_BLOCK / QBLOCK; ++i) {
        const size_t g = g0 + i * QBLOCK;
        if (g >= ngroups) break;
        float v[8];
        widen_bf16(v, raw[i]);
        put_group<KIND, AS_BF16, MODE>(j, v, inv, ctr, g, k0, k1);
      }
    }
  }
}

// Transposed output (cols x rows), optionally a same-layout output as well (out2): the same codes, or those of a second
// (integer) quantizer of the same values.
//
// Tile order: bands of TR source rows in groups of BAND_GROUP; inside a group the band index runs
// fastest, then the column tile.  Workgroups that run together then write BAND_GROUP * TR
// consecutive elements of every transposed row between them, and still read each source row in
// neighbouring pieces.
struct TileAt {
  uint32_t r0, c0;
};
__device__ __forceinline__ TileAt tile_at(const QuantJob& j, uint32_t local, uint32_t tr) {
  const uint32_t tiles_x = (j.cols + TC - 1) / TC, tiles_y = (j.rows + tr - 1) / tr;
  const uint32_t group = local / (BAND_GROUP * tiles_x), within = local % (BAND_GROUP * tiles_x);
  const uint32_t bands = min((uint32_t)BAND_GROUP, tiles_y - group * BAND_GROUP);
  return TileAt{(group * BAND_GROUP + within % bands) * tr, (within / bands) * TC};
}

// The output in the source layout leaves in pieces of 64 bytes of a row (32 where two values share a
// byte): half cache lines, completed by the workgroup of the next column tile, which the tile
// order puts on the same XCD (BAND_GROUP is a multiple of 8).  For a large tensor plain stores
// let that L2 put the halves together and leave the codes where the product that reads them
// next looks first (13.15 -> 13.02 ms per step of the Llama-shaped layer; streaming stores:
// 13.36); small ones keep the write-through form (GPT-2 sizes: 4 us per step better).
__device__ __forceinline__ void put8(bool big, global_ptr<uint8_t> p, const u32x2& v) {
  if (big) *reinterpret_cast<global_ptr<u32x2>>(p) = v;
  else store_through8(p, v);
}

// Byte codes.  A thread takes pieces four rows deep, so that the codes of neighbouring rows, neighbours in the output,
// go to LDS a word at a time, and loads a row of the next piece as soon as the present one has left its registers.  binary32: pieces of 4 columns; lanes L
// and L + 32 hold the two halves of each Philox group of their rows (as in quantize_chunk_f32), so that a swap of wave halves
// hands out the random words of two rows and another one makes the 8-byte pieces of the output in the source layout.
// bfloat16: pieces of 8 columns, a group a row.
// What bounds it is the vector ALU beside the loads (two Philox blocks for eight elements where two quantizers read the
// tensor).  Against element by element through LDS, neighbours trading random words, loads two rows ahead: 8192 x 3072 and 768 x 3072
// binary32 to E5M2 turned and int8 (forward pass of GPT-2's second linear, 165 MB) 46.0 -> 40.9 us.  At most 64 registers, so
// that a wave fits on a SIMD beside two of the persistent product kernel.
template <int KIND, bool F32, bool CACHED, int MODE>
__device__ __forceinline__ void transpose_bytes(job_words job, uint32_t local, uint8_t* tile) {
  const QuantJob j = read_job(job);
  const bool sr = is_sr<MODE>(j.round);
  const uint32_t tr = tile_rows(false, j.rows, j.cols);  // 128 or 256
  const uint32_t pitch = tr + 4;                         // the words a wave instruction writes fall on all 64 banks
  const bool dual = j.out2 && j.kind2;
  const InvScale inv = uniform(inv_scale(j.scale, j.scale_dev, j.kind));
  const InvScale inv2 = dual ? uniform(inv_scale(j.scale2, j.scale_dev2, j.kind2)) : inv;
  const uint64_t ctr = uniform(first_block(j.counter_offset, j.counter_dev));
  const uint64_t ctr2 = dual ? uniform(first_block(j.counter_offset2, j.counter_dev2)) : 0ull;
  const TileAt at = tile_at(j, local, tr);
  const uint32_t rows = j.rows, cols = j.cols;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, half = F32 ? lane >> 5 : 0u;
  const bool big = (size_t)rows * cols > STREAM_OUT_BYTES;
  constexpr uint32_t STEP = F32 ? 64 : 128;  // rows of the tile that the workgroup takes at a time
  const uint32_t cl = (lane & 7u) * 8 + half * 4, rl0 = F32 ? wave * 16 + ((lane >> 3) & 3u) * 4 : wave * 32 + (lane >> 3) * 4;
  using load_t = typename std::conditional<F32, f32x4, u32x4>::type;
  constexpr uint32_t ES = F32 ? 4 : 2;  // bytes of a source element
  // Addresses: a uniform part per step and row, and an offset of this lane below 2^32 (a tensor has less than 2^31 elements in at
  // least 272 rows, as the products' operands allow: 64 rows of binary32 or 128 of bfloat16 stay below)
  const size_t e_tile = (size_t)at.r0 * cols + at.c0;
  const uint32_t src_off = (rl0 * cols + cl) * ES;
  const uint32_t group_off = ((rl0 + half) * cols + cl) / 8;  // upper lanes draw for the row after
  // rows % 16 == 0 and cols % 16 == 0: a piece is inside or outside as a whole, and so is the group of a quad.  The first four
  // rows of a step that is not outside as a whole are inside: lanes outside load the first element of those.
  const bool col_ok = at.c0 + cl < cols;
  load_t v[4];
  auto load = [&](uint32_t r, int i) {
    const uint32_t off = opaque(col_ok && at.r0 + rl0 + r < rows ? src_off : 0u);  // (not kept as 64 bits)
    v[i] = load_source<CACHED>(reinterpret_cast<global_ptr<const load_t>>(
        uniform_ptr(static_cast<const uint8_t*>(j.x) + (e_tile + (size_t)(r + i) * cols) * ES) + off));
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) load(0, i);
  const uint32_t steps_end = min(tr, rows - at.r0);
#pragma unroll 1
  for (uint32_t r = 0; r < steps_end; r += STEP) {
    const bool more = r + STEP < steps_end, inside = col_ok && at.r0 + rl0 + r < rows;
    const size_t group_step = (e_tile + (size_t)r * cols) / 8;
    const uint32_t gstep = cols / 8;  // groups of a row
    uint8_t* const dst = tile + cl * pitch + rl0 + r;
    const QuantJob p = read_job(job, true);
    const uint32_t k0 = (uint32_t)p.seed, k1 = (uint32_t)(p.seed >> 32);
    const uint32_t m0 = (uint32_t)p.seed2, m1 = (uint32_t)(p.seed2 >> 32);
    const bool sr2 = is_sr<MODE>(p.round2);
    if constexpr (F32) {
      uint32_t c[4];
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        __builtin_amdgcn_sched_barrier(0);  // (two pairs of rows at once would take more than 64 registers)
        const size_t group = group_step + (size_t)i * gstep;  // with group_off: of row i (lower lanes) or i + 1 (upper lanes)
        uint32_t w[4];
        round_words_of_pair(sr, ctr + group + group_off, k0, k1, w);
        c[i] = quantize_word<KIND>(v[i].x, v[i].y, v[i].z, v[i].w, inv, w[0], w[1], sr);
        c[i + 1] = quantize_word<KIND>(v[i + 1].x, v[i + 1].y, v[i + 1].z, v[i + 1].w, inv, w[2], w[3], sr);
        if (p.out2) {
          uint32_t lo = c[i], hi = c[i + 1];
          if (p.kind2) {
            round_words_of_pair(sr2, ctr2 + group + group_off, m0, m1, w);
            lo = quantize_word<SRQ_INTX>(v[i].x, v[i].y, v[i].z, v[i].w, inv2, w[0], w[1], sr2);
            hi = quantize_word<SRQ_INTX>(v[i + 1].x, v[i + 1].y, v[i + 1].z, v[i + 1].w, inv2, w[2], w[3], sr2);
          }
          swap_halves(lo, hi);  // this lane: the whole group of its row
          if (KIND == SRQ_INTX && p.pack_2) {
            // two values per byte: two lanes hold a run of 16 columns (cols % 16 == 0: whole runs); byte j of its 8 takes
            // element j in the low and element j + 8 in the high nibble, so the lane with elements 0-7 takes the nibbles
            // of its neighbour
            lo &= 0x0F0F0F0Fu;
            hi &= 0x0F0F0F0Fu;
            const uint32_t nlo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0xB1, 0xF, 0xF, true);  // lane ^ 1
            const uint32_t nhi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0xB1, 0xF, 0xF, true);
            if (inside && !(lane & 1u)) put8(big, uniform_ptr(p.out2 + group * 4) + group_off * 4, u32x2{lo | (nlo << 4), hi | (nhi << 4)});
          } else if (inside) {
            put8(big, uniform_ptr(p.out2 + group * 8) + group_off * 8, u32x2{lo, hi});
          }
        }
        if (more) {
          load(r + STEP, i);
          load(r + STEP, i + 1);
        }
      }
      uint32_t q[4];
      turn4x4(c[0], c[1], c[2], c[3], q);
#pragma unroll
      for (int e = 0; e < 4; ++e) *reinterpret_cast<uint32_t*>(dst + e * pitch) = q[e];
    } else {
      u32x2 c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        const size_t group = group_step + (size_t)i * gstep;
        float f[8];
        widen_bf16(f, v[i]);
        c[i] = quantize_group_words<KIND>(f, inv, ctr + group + group_off, k0, k1, sr);
        if (p.out2) {
          const u32x2 d = p.kind2 ? quantize_group_words<SRQ_INTX>(f, inv2, ctr2 + group + group_off, m0, m1, sr2) : c[i];
          if (inside) *reinterpret_cast<global_ptr<u32x2>>(uniform_ptr(p.out2 + group * 8) + group_off * 8) = d;
        }
        if (more) load(r + STEP, i);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t q[4];
        turn4x4(c[0][h], c[1][h], c[2][h], c[3][h], q);
#pragma unroll
        for (int e = 0; e < 4; ++e) *reinterpret_cast<uint32_t*>(dst + (4 * h + e) * pitch) = q[e];
      }
    }
  }
  // The transposed output of a large tensor goes out with streaming stores (it is far bigger than the
  // caches and the write-through form left the wide gradients at 1 TB/s: 65536 x 5632, 450 -> 355 us);
  // a small one with write-through stores, which leave it in the last-level cache for the product
  // that reads it next (GPT-2 sizes: a few us per step).
  __syncthreads();
  const QuantJob o = read_job(job, true);
  const uint32_t shift = tr == 256 ? 4 : 3;  // log2 of the 16-byte pieces of a run
  for (uint32_t id = threadIdx.x; id < TC << shift; id += QBLOCK) {
    const uint32_t ch = id & ((1u << shift) - 1), c = id >> shift;
    const uint32_t col = at.c0 + c, row = at.r0 + ch * 16;
    if (col >= o.cols || row >= o.rows) continue;  // rows % 16 == 0 for the linear entry points
    const uint32_t* const src = reinterpret_cast<const uint32_t*>(tile + c * pitch + ch * 16);
    if (KIND == SRQ_INTX && o.pack_t) {
      // two values per byte along the transposed row: byte j of 8 = elements j and j + 8 of the 16
      const uint32_t m = 0x0F0F0F0Fu;
      const u32x2 w = {(src[0] & m) | ((src[2] & m) << 4), (src[1] & m) | ((src[3] & m) << 4)};
      uint8_t* const dst = o.out + (((size_t)col * o.rows + row) >> 1);
      if (big) __builtin_nontemporal_store(w, as_global(reinterpret_cast<u32x2*>(dst)));
      else store_through8(as_global(dst), w);
    } else {
      const u32x4 w = {src[0], src[1], src[2], src[3]};
      uint8_t* const dst = o.out + (size_t)col * o.rows + row;
      if (big) __builtin_nontemporal_store(w, as_global(reinterpret_cast<u32x4*>(dst)));
      else store_through16(dst, w);
    }
  }
}

// The grid values as bfloat16 numbers (small products with an E4M3-family operand, weights of the weight-only objective): tiles
// of 128 rows, element by element through LDS.
template <int KIND, bool CACHED, int MODE>
__device__ __forceinline__ void transpose_values(const QuantJob& j, uint32_t local, uint8_t* smem) {
  constexpr int TR = 128, PITCH = TR + 2;
  uint16_t* const tile = reinterpret_cast<uint16_t*>(smem);
  const InvScale inv = inv_scale(j.scale, j.scale_dev, j.kind);
  const bool dual = j.out2 && j.kind2;
  const InvScale inv2 = dual ? inv_scale(j.scale2, j.scale_dev2, j.kind2) : inv;
  const uint64_t ctr = first_block(j.counter_offset, j.counter_dev);
  const uint64_t ctr2 = dual ? first_block(j.counter_offset2, j.counter_dev2) : 0ull;
  const uint32_t k0 = (uint32_t)j.seed, k1 = (uint32_t)(j.seed >> 32);
  const uint32_t m0 = (uint32_t)j.seed2, m1 = (uint32_t)(j.seed2 >> 32);
  const TileAt at = tile_at(j, local, TR);
  const uint32_t rows = j.rows, cols = j.cols;
  const bool big = (size_t)rows * cols > STREAM_OUT_BYTES;
  if (j.dtype == SRQ_F32) {
    // lanes L and L + 32 hold the halves of each group, of row rA and of row rA + 64 (as in quantize_chunk_f32)
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, half = lane >> 5;
    const uint32_t cq = (lane & 7u) * 8 + half * 4, col = at.c0 + cq;  // first column of the quad
    const float* x = static_cast<const float*>(j.x);
#pragma unroll
    for (int it = 0; it < TR / 32; ++it) {
      const uint32_t rA = it * 16 + wave * 4 + ((lane >> 3) & 3u), rB = rA + TR / 2;
      const bool okA = at.r0 + rA < rows && col < cols, okB = at.r0 + rB < rows && col < cols;
      const size_t eA = (size_t)(at.r0 + rA) * cols + col, eB = (size_t)(at.r0 + rB) * cols + col;
      f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
      if (okA) a = load_source<CACHED>(reinterpret_cast<const f32x4*>(x + eA));
      if (okB) b = load_source<CACHED>(reinterpret_cast<const f32x4*>(x + eB));
      uint32_t addA[4], addB[4], ca[4], cb[4], w[4];
      round_words_of_pair(is_sr<MODE>(j.round), ctr + (half ? eB : eA) / 8, k0, k1, w);
      sr_addends(w[0], w[1], addA);
      sr_addends(w[2], w[3], addB);
      if (is_sr<MODE>(j.round)) {
        quantize_quad<KIND, SRQ_SR, true>(ca, a.x, a.y, a.z, a.w, inv, addA);
        quantize_quad<KIND, SRQ_SR, true>(cb, b.x, b.y, b.z, b.w, inv, addB);
      } else {
        quantize_quad<KIND, SRQ_RTN, true>(ca, a.x, a.y, a.z, a.w, inv, addA);
        quantize_quad<KIND, SRQ_RTN, true>(cb, b.x, b.y, b.z, b.w, inv, addB);
      }
      if (dual) {
        // the second quantizer: its own thresholds (same pairing of lanes and Philox blocks)
        const bool sr2 = is_sr<MODE>(j.round2);
        round_words_of_pair(sr2, ctr2 + (half ? eB : eA) / 8, m0, m1, w);
        const uint32_t da = quantize_word<SRQ_INTX>(a.x, a.y, a.z, a.w, inv2, w[0], w[1], sr2);
        const uint32_t db = quantize_word<SRQ_INTX>(b.x, b.y, b.z, b.w, inv2, w[2], w[3], sr2);
        if (okA) store_through4(j.out2 + eA, da);
        if (okB) store_through4(j.out2 + eB, db);
      } else if (j.out2) {
        uint16_t* const o = reinterpret_cast<uint16_t*>(j.out2);
        if (okA) put8(big, as_global(reinterpret_cast<uint8_t*>(o + eA)), u32x2{ca[0] | (ca[1] << 16), ca[2] | (ca[3] << 16)});
        if (okB) put8(big, as_global(reinterpret_cast<uint8_t*>(o + eB)), u32x2{cb[0] | (cb[1] << 16), cb[2] | (cb[3] << 16)});
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        tile[(cq + e) * PITCH + rA] = (uint16_t)ca[e];
        tile[(cq + e) * PITCH + rB] = (uint16_t)cb[e];
      }
    }
  } else {
#pragma unroll
    for (int it = 0; it < (TR * TC / 8) / QBLOCK; ++it) {
      const uint32_t id = it * QBLOCK + threadIdx.x;
      const uint32_t gc = id % (TC / 8), r = id / (TC / 8);
      const uint32_t row = at.r0 + r, col = at.c0 + gc * 8;
      if (row >= rows || col >= cols) continue;
      const size_t g = ((size_t)row * cols + col) / 8;
      float v[8];
      uint32_t c[8];
      widen_bf16(v, load_source<CACHED>(static_cast<const u32x4*>(j.x) + g));
      job_quantize_group<KIND, true, MODE>(c, v, inv, j, ctr, g, k0, k1);
      if (dual)
        *as_global(reinterpret_cast<u32x2*>(j.out2 + g * 8)) = quantize_group_words<SRQ_INTX>(v, inv2, ctr2 + g, m0, m1, is_sr<MODE>(j.round2));
      else if (j.out2)
        *as_global(reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(j.out2) + g * 8)) =
            u32x4{c[0] | (c[1] << 16), c[2] | (c[3] << 16), c[4] | (c[5] << 16), c[6] | (c[7] << 16)};
#pragma unroll
      for (int e = 0; e < 8; ++e) tile[(gc * 8 + e) * PITCH + r] = (uint16_t)c[e];
    }
  }
  const bool stream_out = (size_t)rows * cols * 2 > STREAM_OUT_BYTES;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < (TC * TR / 16) / QBLOCK; ++it) {
    const uint32_t id = it * QBLOCK + threadIdx.x;
    const uint32_t ch = id % (TR / 16), c = id / (TR / 16);
    const uint32_t col = at.c0 + c, row = at.r0 + ch * 16;
    if (col >= cols || row >= rows) continue;  // rows % 16 == 0 for the linear entry points
    const uint32_t* const src = reinterpret_cast<const uint32_t*>(&tile[c * PITCH + ch * 16]);
    u32x4* const dst = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(j.out) + (size_t)col * rows + row);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const u32x4 w = {src[4 * i], src[4 * i + 1], src[4 * i + 2], src[4 * i + 3]};
      if (stream_out) __builtin_nontemporal_store(w, as_global(dst + i));
      else store_through16(dst + i, w);
    }
  }
}

// KIND of bytes: SRQ_INTX stands for both integer formats
template <int KIND, bool CACHED, int MODE>
__device__ __forceinline__ void run_bytes(job_words job, const QuantJob& j, uint32_t local, uint8_t* smem) {
  if (!j.transpose) return flat_path<KIND, false, CACHED, MODE>(j, local, j.nblocks);
  if (j.dtype == SRQ_F32) transpose_bytes<KIND, true, CACHED, MODE>(job, local, smem);
  else transpose_bytes<KIND, false, CACHED, MODE>(job, local, smem);
}

template <int KIND, bool CACHED, int MODE>
__device__ __forceinline__ void run_values(const QuantJob& j, uint32_t local, uint8_t* smem) {
  if (j.transpose) transpose_values<KIND, CACHED, MODE>(j, local, smem);
  else flat_path<KIND, true, CACHED, MODE>(j, local, j.nblocks);
}

template <bool CACHED, int MODE>
__global__ __launch_bounds__(QBLOCK) __attribute__((amdgpu_num_vgpr(64))) void quantize_jobs_kernel(QuantJobs jobs) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[TC * (128 + 2) * 2];
  static_assert(TC * (256 + 4) <= (int)sizeof(smem), "the tile of 256 rows of bytes fits as well");
  int ji = 0;
#pragma unroll
  for (int i = 1; i < QUANT_JOBS_MAX; ++i)
    if (i < jobs.njobs && blockIdx.x >= jobs.job[i].first_block) ji = i;
  const job_words job = (job_words)__builtin_amdgcn_kernarg_segment_ptr() +  // the explicit arguments start at offset 0
                        (offsetof(QuantJobs, job) + (size_t)ji * sizeof(QuantJob)) / 4;
  const QuantJob j = read_job(job);
  const uint32_t local = blockIdx.x - j.first_block;
  const bool bf = j.store == STORE_BF16;
  switch (j.kind) {
    case SRQ_INT8: case SRQ_INT4:
      if (bf) run_values<SRQ_INTX, CACHED, MODE>(j, local, smem);
      else run_bytes<SRQ_INTX, CACHED, MODE>(job, j, local, smem);
      break;
    case SRQ_E4M3:
      if (bf) run_values<SRQ_E4M3, CACHED, MODE>(j, local, smem);
      else run_bytes<SRQ_E4M3, CACHED, MODE>(job, j, local, smem);
      break;
    case SRQ_E5M2:
      if (bf) run_values<SRQ_E5M2, CACHED, MODE>(j, local, smem);
      else run_bytes<SRQ_E5M2, CACHED, MODE>(job, j, local, smem);
      break;
    default:  // E4M2 / E4M1 / E4M0
      if (bf) run_values<SRQ_E4MX, CACHED, MODE>(j, local, smem);
      else run_bytes<SRQ_E4MX, CACHED, MODE>(job, j, local, smem);
      break;
  }
}

template <int MODE>
hipError_t launch_jobs(const QuantJobs& jobs, uint32_t blocks, bool cached, hipStream_t stream) {
  // decided for the launch (two forms inside one kernel cost more than they gave)
  if (cached) quantize_jobs_kernel<true, MODE><<<blocks, QBLOCK, 0, stream>>>(jobs);
  else quantize_jobs_kernel<false, MODE><<<blocks, QBLOCK, 0, stream>>>(jobs);
  return hipGetLastError();
}

}  // namespace
}  // namespace srq
