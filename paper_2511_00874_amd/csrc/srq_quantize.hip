// Tensor-level SR quantizer kernels (Def. 3: element-wise, independent thresholds) and the
// per-tensor absmax scale.  HBM-bound streaming kernels for gfx950: 128-bit loads, one
// Philox block per 8 consecutive elements, 64-bit (or 32-bit for nibbles) stores.
#include "srq_device.hpp"
#include "srq_internal.hpp"

namespace srq {
namespace {

constexpr int QBLOCK = 256;

// ---- same-layout output -------------------------------------------------------------------
template <int KIND, int SRC, int ROUND, int STORE>
__global__ __launch_bounds__(QBLOCK) void quantize_flat_kernel(uint8_t* __restrict__ out,
                                                               const void* __restrict__ x, size_t n,
                                                               float scale, const float* scale_dev, int kind,
                                                               uint64_t seed, uint64_t counter_host,
                                                               const uint64_t* counter_dev) {
  const InvScale inv = inv_scale(scale, scale_dev, kind);
  const uint64_t counter_offset = first_block(counter_host, counter_dev);
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const size_t ngroups = (n + 7) / 8;
  const size_t stride = (size_t)gridDim.x * QBLOCK;
  for (size_t g = (size_t)blockIdx.x * QBLOCK + threadIdx.x; g < ngroups; g += stride) {
    float v[8];
    load_group<SRC>(v, x, g, n);
    const u32x2 c = quantize_group_words<KIND>(v, inv, counter_offset + g, k0, k1, ROUND == SRQ_SR);
    const size_t base = g * 8;
    if constexpr (STORE == STORE_NIBBLE) {
      const uint32_t word = pack8_nibbles(c.x, c.y);
      if (base + 8 <= n) {
        __builtin_nontemporal_store(word, reinterpret_cast<uint32_t*>(out + base / 2));
      } else {
        for (size_t j = 0; base + 2 * j < n; ++j) out[base / 2 + j] = (uint8_t)(word >> (8 * j));
      }
    } else {
      if (base + 8 <= n) {
        __builtin_nontemporal_store(c, reinterpret_cast<u32x2*>(out + base));
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (base + j < n) out[base + j] = (uint8_t)(c[j / 4] >> (8 * (j % 4)));
      }
    }
  }
}

// binary32 source, whole 512-element chunks: one chunk per wave, fully coalesced (see
// quantize_chunk_f32); the ragged remainder goes to quantize_flat_kernel
template <int KIND, int ROUND, int STORE>
__global__ __launch_bounds__(QBLOCK) void quantize_flat_f32_kernel(uint8_t* __restrict__ out,
                                                                   const float* __restrict__ x, size_t nchunks,
                                                                   float scale, const float* scale_dev, int kind,
                                                                   uint64_t seed, uint64_t counter_host,
                                                                   const uint64_t* counter_dev) {
  const InvScale inv = inv_scale(scale, scale_dev, kind);
  const uint64_t counter_offset = first_block(counter_host, counter_dev);
  const uint32_t lane = threadIdx.x & 63u;
  const size_t waves = (size_t)gridDim.x * (QBLOCK / 64);
  for (size_t c = (size_t)blockIdx.x * (QBLOCK / 64) + (threadIdx.x >> 6); c < nchunks; c += waves)
    quantize_chunk_f32<KIND, STORE>(out, x, c, lane, inv, (uint32_t)seed, (uint32_t)(seed >> 32), counter_offset,
                                    ROUND == SRQ_SR);
}

// ---- transposed output --------------------------------------------------------------------
// A workgroup quantizes a tile of TR source rows x TC source columns (thresholds keyed by the
// row-major SOURCE index, so the codes equal those of the same-layout kernel), turns it through
// LDS, and writes TC runs of TR consecutive codes.  HBM-bound: what it is built around is whole
// lines on the store side.
//   - A thread takes a piece that is several rows deep, so the codes of neighbouring rows, which are
//     neighbours in the output, are packed in registers and go to LDS a word (or two) at a time.
//     binary32: 4 columns x 8 rows (a 16-byte load per row; lanes L and L + 32 hold the two halves of
//     each Philox group, the lower one draws the blocks of the even rows, the upper one those of the odd rows,
//     and they trade words by swaps of wave halves).  bfloat16: 8 columns x 4 rows.  All loads of
//     a piece are issued before its first code is made.
//   - A run whose length or place is not a multiple of 16 bytes (a row count that is not one) leaves
//     16 bytes at a time from the first multiple of four on, put together from LDS words by a byte
//     shift; only the up to 3 + 3 bytes at its ends go one by one.
//   - Tile order: XCD x takes a contiguous range of an order that walks groups of TBAND row bands,
//     band index fastest: workgroups that run together on one XCD write neighbouring runs of the
//     same output rows and read neighbouring columns of the same source rows, and the lines that two
//     tiles share are joined in that L2.  (Groups of 8 / 16 / 32 bands, binary32 -> int8: 12288 x 3080
//     40 / 41 / 42 us, 65536 x 4096 241 / 227 / 229.)
// Against the form before (a group of 8 codes per thread, byte-wise LDS writes, 128-row tiles, a ragged
// run byte by byte): 12289 x 3080 bfloat16 -> int8 82 -> 35 us, binary32 99 -> 47; 12288 x 3080 binary32
// 52 -> 41 (189 MB: 4.6 TB/s); 65536 x 4096 binary32 311 -> 227 (5.9 TB/s), bfloat16 162 -> 130.  With the codes of a quad made
// as one word: 12288 x 3080 bfloat16 -> E5M2 32.8 -> 28.6 us, 65536 x 4096 186 -> 151.
//   - At most 64 registers: a wave of it then fits on a SIMD beside two of the persistent product
//     kernel, so that on a second stream it runs beside a product and not behind it.  That takes no more than to
//     recompute the addresses of both sides (opaque) and to round a row at a time; alone it is as fast.  Six calls on 16384 x 4096
//     beside int8 products of 8192 cubed, us a call at 94 registers and at 64: binary32 490 and 177, bfloat16 478 and 145.
constexpr int TC = 64;
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at a multiple of four
constexpr uint32_t TBAND = 16;
constexpr uint32_t TRANSPOSE_GRID = 1u << 20;  // workgroups per launch at most; the rest of the tiles by a loop

template <int KIND, int SRC, int ROUND, int STORE, int TR>
__global__ __launch_bounds__(QBLOCK) void quantize_transpose_kernel(
    uint8_t* __restrict__ out, const void* __restrict__ x, uint32_t rows, uint32_t cols, float scale,
    const float* scale_dev, int kind, uint64_t seed, uint64_t counter_host, const uint64_t* counter_dev) {
  static_assert(STORE == STORE_BYTE || STORE == STORE_NIBBLE, "codes");
  constexpr bool F32 = SRC == SRQ_F32;
  constexpr int DIV = STORE == STORE_NIBBLE ? 2 : 1;  // codes per byte
  constexpr int SEG = TR / DIV;                       // bytes of a run
  // pitch: the pieces a wave instruction writes fall on all 64 banks (16 column quads x 4 row octets of
  // 8 bytes, or 8 column groups x 8 row quads of 4)
  constexpr int PITCH = SEG + (F32 ? 8 : 4);
  __shared__ __attribute__((aligned(16))) uint8_t tile[TC * PITCH + 8];
  const InvScale inv = inv_scale(scale, scale_dev, kind);
  const uint64_t ctr = first_block(counter_host, counter_dev);
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const uint32_t tiles_x = (cols + TC - 1) / TC, tiles_y = (rows + TR - 1) / TR;
  const uint32_t ntiles = tiles_x * tiles_y, chunk = (ntiles + 7u) >> 3;
  const uint32_t begin = (blockIdx.x & 7u) * chunk, end = min(ntiles, begin + chunk);
  const uint32_t orow = rows / DIV;  // bytes of an output row (rows is even where two codes share a byte)

  for (uint32_t work = begin + (blockIdx.x >> 3); work < end; work += gridDim.x >> 3) {
    const uint32_t band = work / (TBAND * tiles_x), band0 = band * TBAND;
    const uint32_t bands = min(TBAND, tiles_y - band0), within = work - band0 * tiles_x;
    const uint32_t r0 = (band0 + within % bands) * TR, c0 = (within / bands) * TC;

    constexpr int PR = F32 ? 8 : 4, PC = F32 ? 4 : 8;  // rows x columns of a thread's piece
    constexpr int PIECES = TR * TC / (PR * PC) / QBLOCK;
    static_assert(PIECES >= 1, "a piece per thread");
#pragma unroll 1
    for (int it = 0; it < PIECES; ++it) {
      // binary32: lanes L and L + 32 hold the two halves of each Philox group of their rows
      const uint32_t tid = opaque(threadIdx.x), id = it * QBLOCK + tid, lane = tid & 63u, half = lane >> 5;
      const uint32_t cl = F32 ? (lane & 7u) * 8 + half * 4 : (id % (TC / PC)) * PC;
      const uint32_t rl = F32 ? ((id >> 6) * 4 + ((lane >> 3) & 3u)) * PR : (id / (TC / PC)) * PR;
      const uint32_t col = c0 + cl, row = r0 + rl;
      const bool col_ok = col < cols;  // cols % 8 == 0: a piece never straddles the edge
      const size_t e0 = (size_t)row * cols + col;
      u32x4 raw[PR];
#pragma unroll
      for (int i = 0; i < PR; ++i) {
        const bool ok = col_ok && row + i < rows;
        const size_t e = ok ? e0 + (size_t)i * cols : 0;  // outside: element 0, and its code is dropped
        if constexpr (F32) raw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(static_cast<const float*>(x) + e));
        else raw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(x) + e));
      }
      if constexpr (F32) {
        uint32_t c[PR];
#pragma unroll
        for (int i = 0; i < PR; i += 2) {
          __builtin_amdgcn_sched_barrier(0);  // (two pairs of rows at once would not fit the registers)
          uint32_t w[4];
          if constexpr (ROUND == SRQ_SR) round_words_of_pair(ctr + (e0 + (size_t)(i + half) * cols) / 8, k0, k1, w);
          else w[0] = w[1] = w[2] = w[3] = RTN_WORD;
          const u32x2 q = quantize_octet<KIND>({__uint_as_float(raw[i].x), __uint_as_float(raw[i].y), __uint_as_float(raw[i].z),
                                                __uint_as_float(raw[i].w)},
                                               {__uint_as_float(raw[i + 1].x), __uint_as_float(raw[i + 1].y),
                                                __uint_as_float(raw[i + 1].z), __uint_as_float(raw[i + 1].w)},
                                               inv, w, ROUND == SRQ_SR);
          c[i] = q.x;
          c[i + 1] = q.y;
        }
        uint32_t upper[4], lower[4];
        turn4x4(c[0], c[1], c[2], c[3], upper);
        turn4x4(c[4], c[5], c[6], c[7], lower);
#pragma unroll
        for (int e = 0; e < PC; ++e) {
          uint8_t* const dst = tile + (cl + e) * PITCH + rl / DIV;
          if constexpr (STORE == STORE_NIBBLE) *reinterpret_cast<uint32_t*>(dst) = pack8_nibbles(upper[e], lower[e]);
          else *reinterpret_cast<u32x2*>(dst) = u32x2{upper[e], lower[e]};
        }
      } else {
        // by conversion: words of codes, turned; others: the codes, or the sums that hold them, of four rows, whose bytes are then
        // picked by column (24 byte permutes instead of 40)
        uint32_t sum[PR][2][4];
        u32x2 c[PR];
#pragma unroll
        for (int i = 0; i < PR; ++i) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[2 * e] = bf16_to_f32(raw[i][e] & 0xFFFFu);
            v[2 * e + 1] = bf16_to_f32(raw[i][e] >> 16);
          }
          const uint64_t block = ctr + (e0 + (size_t)i * cols) / 8;
          if constexpr (BY_CONVERSION<KIND>) {
            c[i] = quantize_group_words<KIND>(v, inv, block, k0, k1, ROUND == SRQ_SR);
          } else if constexpr (Grid<KIND>::is_float) {
            uint32_t code[8];
            quantize_group<KIND, ROUND, false>(code, v, inv, block, k0, k1);
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[i][e / 4][e % 4] = code[e];
          } else {
            uint32_t w[4];
            round_words(ROUND == SRQ_SR, block, k0, k1, w);
            integer_sums<KIND>(sum[i], {v[0], v[1], v[2], v[3]}, {v[4], v[5], v[6], v[7]}, inv, w, ROUND == SRQ_SR);
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t q[4];
          if constexpr (BY_CONVERSION<KIND>) {
            turn4x4(c[0][h], c[1][h], c[2][h], c[3][h], q);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const uint32_t col[4] = {sum[0][h][e], sum[1][h][e], sum[2][h][e], sum[3][h][e]};
              q[e] = Grid<KIND>::is_float ? pack4_bytes(col) : signed_bytes(col);
            }
          }
#pragma unroll
          for (int e = 0; e < 4; e += 2) {
            uint8_t* const dst = tile + (cl + 4 * h + e) * PITCH + rl / DIV;
            if constexpr (STORE == STORE_NIBBLE) {
              const uint32_t n = pack8_nibbles(q[e], q[e + 1]);
              *reinterpret_cast<uint16_t*>(dst) = (uint16_t)n;
              *reinterpret_cast<uint16_t*>(dst + PITCH) = (uint16_t)(n >> 16);
            } else {
              *reinterpret_cast<uint32_t*>(dst) = q[e];
              *reinterpret_cast<uint32_t*>(dst + PITCH) = q[e + 1];
            }
          }
        }
      }
    }
    __syncthreads();
    const uint32_t rb = r0 / DIV, nb = min((uint32_t)SEG, orow - rb);  // the runs of this tile, in bytes
    const uint32_t t = opaque(threadIdx.x);  // (addresses from here on are not kept over the loop)
    if ((orow & 15u) == 0) {
      // every run starts at a multiple of 16 bytes and is a multiple of 16 long
#pragma unroll
      for (int it = 0; it < TC * SEG / 16 / QBLOCK; ++it) {
        const uint32_t id = it * QBLOCK + t;
        const uint32_t ch = id % (SEG / 16), cl = id / (SEG / 16);
        if (c0 + cl >= cols || ch * 16 >= nb) continue;
        const uint32_t* src = reinterpret_cast<const uint32_t*>(tile + cl * PITCH + ch * 16);
        *reinterpret_cast<u32x4*>(out + (size_t)(c0 + cl) * orow + rb + ch * 16) = u32x4{src[0], src[1], src[2], src[3]};
      }
    } else {
      // one lane per four words of a run: h bytes up to the first aligned address, then whole words; the
      // last lane, whose words are never all there when a run has ends, takes the ends
      constexpr int LANES = SEG / 16;
#pragma unroll
      for (int it = 0; it < TC * LANES / QBLOCK; ++it) {
        const uint32_t id = it * QBLOCK + t;
        const uint32_t w = (id % LANES) * 4, cl = id / LANES;
        if (c0 + cl >= cols) continue;
        const uint8_t* const run = tile + cl * PITCH;
        uint8_t* const dst = out + (size_t)(c0 + cl) * orow + rb;
        const uint32_t h = min((0u - (uint32_t)(uintptr_t)dst) & 3u, nb), words = (nb - h) >> 2;
        const uint32_t* const src = reinterpret_cast<const uint32_t*>(run) + w;  // bytes h + 4 w ... of the run
        u32x4a4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_alignbyte(src[e + 1], src[e], h);
        if (w + 4 <= words) {
          *reinterpret_cast<u32x4a4*>(dst + h + 4 * w) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (w + e < words) *reinterpret_cast<uint32_t*>(dst + h + 4 * (w + e)) = v[e];
          if (id % LANES == LANES - 1) {
            for (uint32_t j = 0; j < h; ++j) dst[j] = run[j];
            for (uint32_t j = h + 4 * words; j < nb; ++j) dst[j] = run[j];
          }
        }
      }
    }
    __syncthreads();  // the tile is free for the next one
  }
}

// ---- absmax ---------------------------------------------------------------------------------
// max over the wave of non-negative bit patterns: DPP butterflies inside each row of 16
// lanes, then the four rows through scalar reads.
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));  // row_half_mirror
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));  // row_mirror
  const uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
  return max(max(a, b), max(c, d));
}

// |x| as bits, with Inf and NaN ignored (they do not take part in the scale).
__device__ __forceinline__ uint32_t abs_bits_finite(float f) {
  const uint32_t a = __float_as_uint(f) & 0x7FFFFFFFu;
  return a < 0x7F800000u ? a : 0u;
}

// The same order on a key that takes one instruction to make: the sign shifted out, and the largest exponent, of Inf and NaN,
// brought below every finite value by the carry that is lost.  Bits below those of a value, of the other bfloat16 of its word, only order equal
// values.  With the maximum of three values in one instruction an element costs 6.6 cycles of a wave instead of 15.6 (abs_bits_finite and
// max), which counts where one CU reads the tensor: GPU us of a call, 256 KiB, binary32 3.7 -> 3.1, bfloat16 5.8 -> 3.4; 4 MiB 6.5 ->
// 6.1 and 6.8 -> 6.3.
constexpr uint32_t FINITE_KEY = 0x01000000u;  // of zero
template <int SHIFT>
__device__ __forceinline__ uint32_t finite_key(uint32_t a) {
  return (a << SHIFT) + FINITE_KEY;
}
template <int SRC>
__device__ __forceinline__ uint32_t abs_bits_of_key(uint32_t k) {
  return k < FINITE_KEY ? 0u : (k - FINITE_KEY) >> 1 & (SRC == SRQ_F32 ? ~0u : 0xFFFF0000u);
}

// max of the finite |x_i| bit patterns over the 16-byte pieces [g0, g1) of x (4 binary32 or 8
// bfloat16 elements each; the last piece of the tensor may be partial): thread t of nt, eight loads in
// flight per lane, the pieces of a workgroup contiguous in memory
template <int SRC, bool CACHED>
__device__ __forceinline__ uint32_t absmax_pieces(const void* __restrict__ x, size_t n, size_t g0, size_t g1, uint32_t t,
                                                  uint32_t nt) {
  constexpr int PER = SRC == SRQ_F32 ? 4 : 8;
  uint32_t m = 0u;
  const size_t full = n / PER;  // pieces that lie wholly inside the tensor
  const size_t gf = g1 < full ? g1 : full;
  const u32x4* p = static_cast<const u32x4*>(x);
  auto fold = [&](const u32x4& a) {
#pragma unroll
    for (int j = 0; j < 4; j += SRC == SRQ_F32 ? 2 : 1) {
      if constexpr (SRC == SRQ_F32) m = max(max(m, finite_key<1>(a[j])), finite_key<1>(a[j + 1]));
      else m = max(max(m, finite_key<1>(a[j])), finite_key<17>(a[j]));
    }
  };
  size_t i = g0 + t;
  for (; i + 7 * (size_t)nt < gf; i += 8 * (size_t)nt) {
    u32x4 a[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = load_source<CACHED>(p + i + j * (size_t)nt);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // (all keys at once take registers)
      fold(a[j]);
    }
  }
  for (; i + 3 * (size_t)nt < gf; i += 4 * (size_t)nt) {
    const u32x4 a = load_source<CACHED>(p + i), b = load_source<CACHED>(p + i + nt);
    const u32x4 c = load_source<CACHED>(p + i + 2 * (size_t)nt), d = load_source<CACHED>(p + i + 3 * (size_t)nt);
    fold(a); fold(b); fold(c); fold(d);
  }
  for (; i < gf; i += nt) fold(load_source<CACHED>(p + i));
  m = abs_bits_of_key<SRC>(m);
  if (g1 > full && t < n - full * PER) {  // the partial last piece, element by element
    const size_t e = full * PER + t;
    m = max(m, abs_bits_finite(SRC == SRQ_F32 ? static_cast<const float*>(x)[e]
                                              : bf16_to_f32(static_cast<const uint16_t*>(x)[e])));
  }
  return m;
}

// The smallest step the quantizer takes (2^16 / step must stay finite in binary32): the absmax
// scale of a tensor of vanishing values is floored here instead of saturating every element.
constexpr float MIN_SCALE = 0x1p-100f;

__global__ void absmax_init_kernel(uint32_t* acc) { *acc = 0u; }

// The scale that belongs to max|x| (its bit pattern); an all-zero tensor gets 1.
__device__ __forceinline__ float scale_of(uint32_t amax_bits, float qmax) {
  const float amax = __uint_as_float(amax_bits);
  return amax == 0.0f ? 1.0f : fmaxf(__fdiv_rn(amax, qmax), MIN_SCALE);
}

// max over a workgroup of THREADS, valid in thread 0
template <int THREADS>
__device__ __forceinline__ uint32_t block_umax(uint32_t m) {
  __shared__ uint32_t part[THREADS / 64];
  m = wave_umax(m);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 1; i < THREADS / 64; ++i) m = max(m, part[i]);
  }
  return m;
}

// A tensor of up to 256 KiB: one workgroup reads it and writes the scale in one launch.  GPU us a call, against the three
// launches of larger ones (5.7): binary32 128 KiB 2.3, 256 KiB 3.1; bfloat16 2.4, 3.4.  (512 KiB 4.9 and 5.4, but see the next lines.)
// Latency bounds it, so it is as wide as a workgroup can be.  Beside a product on another stream it then waits for the
// end of the product kernel (256 KiB, beside int8 products of 8192 cubed, 150 us; of 256 threads 20 us, but alone 5.1 instead of
// 4.0): what follows such a call, the product of a small layer, waits for the same CUs anyway.
constexpr int ABSMAX_SMALL_BLOCK = 1024;
constexpr size_t ABSMAX_SMALL_BYTES = 256u << 10;
template <int SRC>
__global__ __launch_bounds__(ABSMAX_SMALL_BLOCK) void absmax_small_kernel(float* __restrict__ scale, const void* __restrict__ x,
                                                                          size_t n, float qmax) {
  constexpr size_t PER = SRC == SRQ_F32 ? 4 : 8;
  const uint32_t m = block_umax<ABSMAX_SMALL_BLOCK>(
      absmax_pieces<SRC, true>(x, n, 0, (n + PER - 1) / PER, threadIdx.x, ABSMAX_SMALL_BLOCK));
  if (threadIdx.x == 0) *scale = scale_of(m, qmax);
}

// A larger one: the maximum gathers in the scale's own word, between a launch that clears it and one
// that turns it into the scale.  Atomics on one address from eight XCDs are served one after
// another, about 30 ns each, so there are few of them: at most two workgroups per CU, and a workgroup
// whose maximum is not above what the word holds already does not ask.  (A stale word costs an
// atomic that changes nothing; the maximum is the same.)  Workgroups of 256 threads with 64 registers at most (the launch
// bounds) start on a CU that a persistent product kernel holds; of 1024 they waited for its end.
constexpr int ABSMAX_BLOCK = 256;
template <int SRC, bool CACHED>
__global__ __launch_bounds__(ABSMAX_BLOCK, 8) void absmax_kernel(uint32_t* __restrict__ acc,
                                                              const void* __restrict__ x, size_t n) {
  // every workgroup one contiguous share of the tensor
  constexpr size_t PER = SRC == SRQ_F32 ? 4 : 8;
  const size_t pieces = (n + PER - 1) / PER, share = (pieces + gridDim.x - 1) / gridDim.x;
  const size_t g0 = (size_t)blockIdx.x * share, g1 = g0 + share < pieces ? g0 + share : pieces;
  const uint32_t m = block_umax<ABSMAX_BLOCK>(g0 < pieces ? absmax_pieces<SRC, CACHED>(x, n, g0, g1, threadIdx.x, ABSMAX_BLOCK) : 0u);
  // bit patterns of non-negative floats order like the floats
  if (threadIdx.x == 0 && m > __hip_atomic_load(acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(acc, m);
}

__global__ void absmax_finish_kernel(float* scale, float qmax) {
  *scale = scale_of(__float_as_uint(*scale), qmax);  // the accumulator holds the bits of max|x|
}

// ---- several tensors, several scales, two launches -----------------------------------------
// Launch 1: every block reduces one contiguous slice of one tensor and writes its partial maximum
// to the workspace (plain stores: nothing to initialise).  Launch 2: one block per tensor folds
// that tensor's partials and writes the scales requested of it (several formats may share one
// tensor).
// At most 64 registers, as the scales are computed beside the products of another layer (70, the compiler's choice, cost 1.4 % of the
// two-stream step).
__global__ __launch_bounds__(QBLOCK, 8) void absmax_multi_kernel(AbsmaxBatch b) {
  int t = 0;
#pragma unroll
  for (int i = 1; i < ABSMAX_MAX; ++i)
    if (i < b.ntensors && blockIdx.x >= b.first_block[i]) t = i;
  const uint32_t local = blockIdx.x - b.first_block[t], nblk = b.nblocks[t];
  const size_t n = b.n[t];
  const void* x = b.x[t];
  const size_t per = b.dtype[t] == SRQ_F32 ? 4 : 8;
  const size_t pieces = (n + per - 1) / per, share = (pieces + nblk - 1) / nblk;
  const size_t g0 = (size_t)local * share, g1 = g0 + share < pieces ? g0 + share : pieces;
  uint32_t m = 0u;
  if (g0 < pieces) {
    if (b.dtype[t] == SRQ_F32)
      m = b.cached ? absmax_pieces<SRQ_F32, true>(x, n, g0, g1, threadIdx.x, QBLOCK)
                      : absmax_pieces<SRQ_F32, false>(x, n, g0, g1, threadIdx.x, QBLOCK);
    else
      m = b.cached ? absmax_pieces<SRQ_BF16, true>(x, n, g0, g1, threadIdx.x, QBLOCK)
                      : absmax_pieces<SRQ_BF16, false>(x, n, g0, g1, threadIdx.x, QBLOCK);
  }
  m = wave_umax(m);
  __shared__ uint32_t part[QBLOCK / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = part[0];
#pragma unroll
    for (int i = 1; i < QBLOCK / 64; ++i) r = max(r, part[i]);
    b.partial[blockIdx.x] = r;
  }
}

// 256 threads (one wave per SIMD, 20 registers): small enough to start on a CU that a product kernel
// occupies, when the scales are computed on a second stream beside the products of another layer (a
// workgroup of 1024 threads waited there for a product launch to end, 200-700 us)
constexpr int FINISH_BLOCK = 256;
__global__ __launch_bounds__(FINISH_BLOCK) void absmax_multi_finish_kernel(AbsmaxBatch b) {
  __shared__ uint32_t part[FINISH_BLOCK / 64];
  const int t = blockIdx.x;  // one block per tensor
  const uint32_t* p = b.partial + b.first_block[t];
  const uint32_t nb = b.nblocks[t];
  uint32_t m = 0u;
  uint32_t i = threadIdx.x;
  for (; i + 3 * FINISH_BLOCK < nb; i += 4 * FINISH_BLOCK)
    m = max(max(m, max(p[i], p[i + FINISH_BLOCK])), max(p[i + 2 * FINISH_BLOCK], p[i + 3 * FINISH_BLOCK]));
  for (; i < nb; i += FINISH_BLOCK) m = max(m, p[i]);
  m = wave_umax(m);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if ((int)threadIdx.x < b.nouts && b.out_tensor[threadIdx.x] == t) {
    uint32_t r = part[0];
    for (int w = 1; w < FINISH_BLOCK / 64; ++w) r = max(r, part[w]);
    *b.out[threadIdx.x] = scale_of(r, b.out_qmax[threadIdx.x]);
  }
}

int grid_for(size_t work_items, int per_block, int cap) {
  size_t blocks = (work_items + per_block - 1) / per_block;
  if (blocks < 1) blocks = 1;
  if (blocks > (size_t)cap) blocks = cap;
  return (int)blocks;
}

float qmax_of(int kind) {
  switch (kind) {
    case SRQ_INT8: return 127.0f;
    case SRQ_INT4: return 7.0f;
    case SRQ_E4M3: case SRQ_E4M2: return 448.0f;
    case SRQ_E4M1: return 384.0f;
    case SRQ_E4M0: return 256.0f;
    default: return 57344.0f;
  }
}

template <int KIND, int SRC, int ROUND, int STORE>
hipError_t launch_one(void* codes, const void* x, size_t rows, size_t cols, int transpose_out,
                      const QuantArgs& a, hipStream_t stream) {
  if (transpose_out) {
    // 256 rows (runs of 256 bytes) from 2^28 elements or so up, where the store side is the limit, else 128: twice the
    // workgroups.  us with 128 and 256, int8: 4096 x 4096 binary32 17.3 and 18.2, 8192 x 4096 34 and 37 (bfloat16 23.8 and 24.1), 16384 x
    // 4096 64 and 70 (38 and 42), 65536 x 2048 119 and 120 (74 and 75), 65536 x 4096 237 and 229 (136 and 138), 65537 x 4096 278 and 245
    // (186 and 154), 4096 x 65536 235 and 231 (157 and 146)
    const size_t tiles_x = (cols + TC - 1) / TC, big = tiles_x * ((rows + 255) / 256), small = tiles_x * ((rows + 127) / 128);
    auto launch = [&](auto kern, size_t ntiles) {
      const size_t per_xcd = (ntiles + 7) / 8;
      const unsigned grid = 8u * (unsigned)(per_xcd < TRANSPOSE_GRID / 8 ? per_xcd : TRANSPOSE_GRID / 8);
      kern<<<grid, QBLOCK, 0, stream>>>(static_cast<uint8_t*>(codes), x, (uint32_t)rows, (uint32_t)cols, a.scale,
                                        a.scale_dev, a.kind, a.seed, a.counter_offset, a.counter_dev);
    };
    if (big >= 16384) launch(&quantize_transpose_kernel<KIND, SRC, ROUND, STORE, 256>, big);
    else launch(&quantize_transpose_kernel<KIND, SRC, ROUND, STORE, 128>, small);
  } else {
    const size_t n = rows * cols;
    size_t done = 0;  // elements handled by the coalesced chunk kernel
    if constexpr (SRC == SRQ_F32) {
      const size_t nchunks = n / CHUNK;
      if (nchunks > 0) {
        const int grid = grid_for(nchunks, QBLOCK / 64, 1 << 22);
        quantize_flat_f32_kernel<KIND, ROUND, STORE><<<grid, QBLOCK, 0, stream>>>(
            static_cast<uint8_t*>(codes), static_cast<const float*>(x), nchunks, a.scale, a.scale_dev, a.kind, a.seed,
            a.counter_offset, a.counter_dev);
        done = nchunks * CHUNK;
      }
    }
    if (done < n) {
      // remainder (or a bfloat16 source, whose groups are one 16-byte load each already)
      const size_t es = SRC == SRQ_F32 ? 4 : 2;
      const size_t out_bytes = STORE == STORE_NIBBLE ? done / 2 : done;
      const int grid = grid_for((n - done + 7) / 8, QBLOCK * 4, 1 << 20);
      quantize_flat_kernel<KIND, SRC, ROUND, STORE><<<grid, QBLOCK, 0, stream>>>(
          static_cast<uint8_t*>(codes) + out_bytes, static_cast<const uint8_t*>(x) + done * es, n - done, a.scale,
          a.scale_dev, a.kind, a.seed, a.counter_offset + done / 8, a.counter_dev);
    }
  }
  return hipGetLastError();
}

template <int KIND, int STORE>
hipError_t dispatch_src_round(void* codes, const void* x, size_t rows, size_t cols, int tr,
                              const QuantArgs& a, hipStream_t s) {
  if (a.dtype == SRQ_F32) {
    return a.round == SRQ_SR ? launch_one<KIND, SRQ_F32, SRQ_SR, STORE>(codes, x, rows, cols, tr, a, s)
                             : launch_one<KIND, SRQ_F32, SRQ_RTN, STORE>(codes, x, rows, cols, tr, a, s);
  }
  return a.round == SRQ_SR ? launch_one<KIND, SRQ_BF16, SRQ_SR, STORE>(codes, x, rows, cols, tr, a, s)
                           : launch_one<KIND, SRQ_BF16, SRQ_RTN, STORE>(codes, x, rows, cols, tr, a, s);
}

// E4M3 by conversion (BY_CONVERSION) from here on, where a tensor of any values is no slower.  us without and with, for a normal tensor / one
// with 1 % of outliers / values over 40 binades: 2^20 elements binary32 turned 4.1 -> 3.8 / 4.1 -> 4.2 / 4.1 -> 4.2; 2^22, rows of 2048, binary32
// 5.2 -> 4.7 / 5.3 -> 5.1 / 5.3 -> 5.1, turned 5.9 -> 5.1 / 5.9 -> 5.6 / 5.9 -> 5.7, bfloat16 6.7 -> 6.0 / 6.7 -> 6.5 / 6.7 -> 6.5, turned 5.8 ->
// 4.9 / 5.8 -> 5.4 / 5.8 -> 5.4; 2^24, rows of 4096, binary32 17.2 -> 14.5 / 16.7 -> 15.0 / 15.5 -> 14.9, bfloat16 14.1 -> 11.3 / 14.2 -> 13.2 /
// 14.2 -> 13.2, turned 15.3 -> 12.3 / 15.3 -> 14.2 / 15.3 -> 14.2; 2^28 binary32 215 -> 217 / 218 -> 216 / 215 -> 220 (HBM; the times spread
// by 2 %), bfloat16 170 -> 140 / 173 -> 155 / 168 -> 161.
constexpr size_t E4M3_CONV_ELEMENTS = (size_t)1 << 22;

}  // namespace

hipError_t launch_quantize(void* codes, const void* x, size_t rows, size_t cols, int transpose_out,
                           const QuantArgs& a, hipStream_t stream) {
  if (rows * cols == 0) return hipSuccess;
  switch (a.kind) {
    case SRQ_INT8: return dispatch_src_round<SRQ_INT8, STORE_BYTE>(codes, x, rows, cols, transpose_out, a, stream);
    case SRQ_INT4: return dispatch_src_round<SRQ_INT4, STORE_NIBBLE>(codes, x, rows, cols, transpose_out, a, stream);
    case SRQ_E4M3:
      if (rows * cols >= E4M3_CONV_ELEMENTS)
        return dispatch_src_round<SRQ_E4M3_CONV, STORE_BYTE>(codes, x, rows, cols, transpose_out, a, stream);
      return dispatch_src_round<SRQ_E4M3, STORE_BYTE>(codes, x, rows, cols, transpose_out, a, stream);
    case SRQ_E5M2: return dispatch_src_round<SRQ_E5M2, STORE_BYTE>(codes, x, rows, cols, transpose_out, a, stream);
    case SRQ_E4M2: case SRQ_E4M1: case SRQ_E4M0:
      return dispatch_src_round<SRQ_E4MX, STORE_BYTE>(codes, x, rows, cols, transpose_out, a, stream);
    default: return hipErrorInvalidValue;
  }
}

size_t absmax_batch_plan(AbsmaxBatch& b) {
  // sixteen 16-byte loads per lane (64 KiB per workgroup: measured best between 16 and 128 KiB),
  // at most 32768 workgroups in all; at least one per tensor
  size_t total_groups = 0;
  for (int t = 0; t < b.ntensors; ++t) total_groups += (b.n[t] + 7) / 8;
  uint32_t first = 0;
  for (int t = 0; t < b.ntensors; ++t) {
    const size_t groups = (b.n[t] + 7) / 8;
    size_t nb = (groups + QBLOCK * 8 - 1) / (QBLOCK * 8);
    const size_t share = total_groups ? (32768 * groups + total_groups - 1) / total_groups : 1;
    if (nb > share) nb = share;
    if (nb < 1) nb = 1;
    b.first_block[t] = first;
    b.nblocks[t] = (uint32_t)nb;
    first += (uint32_t)nb;
  }
  return first;
}

hipError_t launch_absmax_batch(AbsmaxBatch& b, hipStream_t stream) {
  const size_t blocks = absmax_batch_plan(b);
  for (int i = 0; i < b.nouts; ++i) b.out_qmax[i] = qmax_of(b.out_kind[i]);
  size_t bytes = 0;
  for (int t = 0; t < b.ntensors; ++t) bytes += source_bytes(b.n[t], b.dtype[t]);
  b.cached = bytes <= ABSMAX_CACHED_BYTES;
  absmax_multi_kernel<<<(unsigned)blocks, QBLOCK, 0, stream>>>(b);
  absmax_multi_finish_kernel<<<b.ntensors, FINISH_BLOCK, 0, stream>>>(b);
  return hipGetLastError();
}

hipError_t launch_absmax_scale(float* scale_out_dev, const void* x, int dtype, size_t n, int kind,
                               hipStream_t stream) {
  const bool f32 = dtype == SRQ_F32;
  const float qmax = qmax_of(kind);
  const size_t pieces = (source_bytes(n, dtype) + 15) / 16;
  if (source_bytes(n, dtype) <= ABSMAX_SMALL_BYTES) {
    if (f32) absmax_small_kernel<SRQ_F32><<<1, ABSMAX_SMALL_BLOCK, 0, stream>>>(scale_out_dev, x, n, qmax);
    else absmax_small_kernel<SRQ_BF16><<<1, ABSMAX_SMALL_BLOCK, 0, stream>>>(scale_out_dev, x, n, qmax);
    return hipGetLastError();
  }
  uint32_t* acc = reinterpret_cast<uint32_t*>(scale_out_dev);
  absmax_init_kernel<<<1, 1, 0, stream>>>(acc);
  // 16 loads per thread, 64 to 512 workgroups.  GPU us a call, binary32 / bfloat16: 4 MiB 7.4 / 7.9, 16 MiB 9.7 / 11.3 (eight
  // loads and 512 workgroups 12.3 / 12.7), 64 MiB 20.6 / 20.3 (768 workgroups 24.8 / 23.1, 2048 36 / 36), 1 GiB 163 / 164 (178 / 175);
  // workgroups of 1024 threads 7.5 / 7.9, 9.4 / 11.6, 18.3 / 22.1, 167 / 165.  Six calls on 256 MiB beside int8 products of 8192
  // cubed on another stream 97 / 61 us each, with those 487 / 467.
  const int wide = grid_for(pieces, ABSMAX_BLOCK, 64), deep = grid_for(pieces, ABSMAX_BLOCK * 16, 512);
  const int grid = wide > deep ? wide : deep;
  const bool cached = source_bytes(n, dtype) <= ABSMAX_CACHED_BYTES;
  const auto kern = f32 ? (cached ? &absmax_kernel<SRQ_F32, true> : &absmax_kernel<SRQ_F32, false>)
                        : (cached ? &absmax_kernel<SRQ_BF16, true> : &absmax_kernel<SRQ_BF16, false>);
  kern<<<grid, ABSMAX_BLOCK, 0, stream>>>(acc, x, n);
  absmax_finish_kernel<<<1, 1, 0, stream>>>(scale_out_dev, qmax);
  return hipGetLastError();
}

}  // namespace srq
