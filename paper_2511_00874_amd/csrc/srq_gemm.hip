// Product of two code matrices on the gfx950 matrix cores (Sec. 2.2.2: low-precision
// multiplies, high-precision accumulation == exact product of the quantized matrices).
//
//   out[p][q] = s * sum_r val(X[p][r]) * val(Z[q][r])        X: P x R, Z: Q x R, R contiguous
//
// All three products of Alg. 1 / Alg. 2 have this form once the quantizer has written the
// operands with the contraction index contiguous.  Four matrix pipelines:
//   int8 codes          v_mfma_i32_16x16x64_i8, _32x32x32_i8        int32 accumulators, exact
//   E4M3/E5M2 as bf16   v_mfma_f32_16x16x32_bf16, _32x32x16_bf16    exact products, binary32 sums
//   E4M3/E5M2 as f16    v_mfma_f32_16x16x32_f16, _32x32x16_f16      the same, from one-byte codes: every value is a
//                                                                   binary16 number, the operands are widened in
//                                                                   registers
//   E4M3/E5M2 codes     v_mfma_f32_32x32x64_f8f6f4                  fp8 pipeline (aligns groups of 8 products)
// in MFMA tiles of 16 x 16, under which the chip clocks higher (srq_mma.hpp), or of 32 x 32, by the form of the product (launch_mma).
//
// Kernel shape.  A workgroup owns a BM x BN output tile, its waves a WGM x WGN grid of
// sub-tiles made of MFMA tiles.  The contraction advances BK = 128 bytes per stage.
// Operand tiles go from global memory straight into LDS (buffer_load ... lds, 16 bytes per
// lane, no registers in between) through a ring of STAGES buffers, so the loads of the next
// stages are in flight while the current one is multiplied; out-of-range rows and the tail of
// the contraction come back as zeros from the buffer bounds check.  LDS rows are 128 bytes
// with the 16-byte chunks XOR-swizzled by (row mod 8): the DMA writes 8 full rows per wave
// instruction and the MFMA operand reads (ds_read_b128, one row per lane) spread over all
// banks.  The product is computed transposed inside the wave (Z rows as the first MFMA
// operand) so that each lane ends up with 4 consecutive q of one p: 16-byte output stores.
#include <type_traits>

#include "srq_internal.hpp"
#include "srq_mma.hpp"
#include "srq_plan.hpp"

namespace srq {
namespace {

using namespace mma;
static_assert(BK == STAGE_BYTES, "the plan counts the kernels' stages");
typedef int v2i __attribute__((ext_vector_type(2)));

struct GemmParams {
  float* out;            // P x Q (final) -- or partial sums when nsplit > 1
  uint32_t* partial;     // nsplit x P x Q raw accumulators (nsplit > 1)
  const uint8_t* X;
  const uint8_t* Z;
  uint32_t P, Q, R;      // R: bytes per operand row (contraction length x element size)
  uint32_t pitch;        // bytes between operand rows (>= R, multiple of 16)
  uint32_t pitch_x;      // the same for X when its rows hold two 4-bit values per byte (else = pitch)
  uint32_t k_per_split;  // bytes of R per z-slice, multiple of BK / 2
  uint32_t nsplit;
  uint32_t tiles_p, tiles_q;
  float alpha, sx, sz;
  const float* sx_dev;
  const float* sz_dev;
  int accumulate;
};

__device__ __forceinline__ float total_scale(const GemmParams& g) {
  const float sx = g.sx_dev ? *g.sx_dev : g.sx;
  const float sz = g.sz_dev ? *g.sz_dev : g.sz;
  return __fmul_rn(g.alpha, __fmul_rn(sx, sz));
}

// Fixed-order sum of the slice partials of a product (deterministic), then scale: workgroup
// `block` of `nblocks`.  Integer partials are summed in int32, the others in binary32.
template <bool IS_INT>
__device__ __forceinline__ void slice_sum(const SliceSum& r, uint32_t block, uint32_t nblocks) {
  const float sx = r.s.sx_dev ? *r.s.sx_dev : r.s.sx, sz = r.s.sz_dev ? *r.s.sz_dev : r.s.sz;
  const float s = __fmul_rn(r.s.alpha, __fmul_rn(sx, sz));
  auto value = [&](uint32_t bits) {
    if constexpr (IS_INT) return (int)bits; else return __uint_as_float(bits);
  };
  const size_t nthreads = (size_t)nblocks * blockDim.x, tid = (size_t)block * blockDim.x + threadIdx.x;
  if ((r.total & 3u) == 0) {
    const size_t total4 = r.total / 4;
    const v4u* part = reinterpret_cast<const v4u*>(r.partial);
    v4f* out = reinterpret_cast<v4f*>(r.out);
    for (size_t i = tid; i < total4; i += nthreads) {
      const v4u p0 = part[i];
      auto a0 = value(p0[0]), a1 = value(p0[1]), a2 = value(p0[2]), a3 = value(p0[3]);
      for (uint32_t z = 1; z < r.nsplit; ++z) {
        const v4u p = part[z * total4 + i];
        a0 += value(p[0]); a1 += value(p[1]); a2 += value(p[2]); a3 += value(p[3]);
      }
      v4f v = {__fmul_rn((float)a0, s), __fmul_rn((float)a1, s), __fmul_rn((float)a2, s), __fmul_rn((float)a3, s)};
      if (r.accumulate) {
        const v4f o = out[i];
        v = v4f{__fadd_rn(v[0], o[0]), __fadd_rn(v[1], o[1]), __fadd_rn(v[2], o[2]), __fadd_rn(v[3], o[3])};
      }
      out[i] = v;
    }
  } else {
    for (size_t i = tid; i < r.total; i += nthreads) {
      auto a = value(r.partial[i]);
      for (uint32_t z = 1; z < r.nsplit; ++z) a += value(r.partial[z * r.total + i]);
      float v = __fmul_rn((float)a, s);
      if (r.accumulate) v = __fadd_rn(v, r.out[i]);
      r.out[i] = v;
    }
  }
}

constexpr uint32_t OOB = 0x80000000u;  // beyond any operand (operands are < 2 GiB): loads as zero

// s_waitcnt vmcnt(n) alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, others left at max)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// One wave-level LDS DMA: 64 lanes x 16 bytes from buffer `rsrc` at byte offset `voff` (per
// lane; out of range reads as zero) to LDS address `lds_addr` + lane * 16.  Written as inline
// assembly so that the compiler does not serialise the ring of stages behind vmcnt(0): the
// kernel counts outstanding DMAs itself (wait_vmcnt).
// M0 (the LDS base of the DMA) is written inside the asm.  It is a reserved register: the compiler
// neither allocates it nor honours it in a clobber list, and it writes M0 itself only for
// constructs this file does not contain (dynamic register indexing, messages, GWS, LDS-direct
// reads).  In the assembly generated for this file every write of m0 is the one below.
__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t rsrc, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(rsrc)
               : "memory");
}

// Four results of row p, columns q .. q + 3 (p and q inside the output), given as accumulator bits: a slice's partial
// sums as they are, final results scaled.
template <class MMA>
__device__ __forceinline__ void store_quad(const GemmParams& g, uint32_t* pbase, uint32_t p, uint32_t q, const v4u& raw,
                                           float s, bool q_vec) {
  const size_t idx = (size_t)p * g.Q + q;
  if (pbase) {
    if (q_vec) {
      // write-through: nothing of the partial tile stays dirty in the L2 when the kernel
      // ends, and the reduction launched next still finds it in the last-level cache
      asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" : : "v"(pbase + idx), "v"(raw) : "memory");
    } else {
      for (int e = 0; e < 4 && q + e < g.Q; ++e) pbase[idx + e] = raw[e];
    }
  } else {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __fmul_rn(MMA::to_f32(MMA::from_bits(raw[e])), s);
    float* dst = g.out + idx;
    if (q_vec) {
      if (g.accumulate) {
        const v4f o = *reinterpret_cast<const v4f*>(dst);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __fadd_rn(v[e], o[e]);
      }
      // the result is not read again by this kernel: a streaming store keeps it from pushing
      // operand panels out of the L2
      __builtin_nontemporal_store(v4f{v[0], v[1], v[2], v[3]}, reinterpret_cast<v4f*>(dst));
    } else {
      for (int e = 0; e < 4 && q + e < g.Q; ++e) dst[e] = g.accumulate ? __fadd_rn(v[e], dst[e]) : v[e];
    }
  }
}

// Epilogue of a wave: its TM x TN block of T x T MFMA results, first row p0 and column q0 of the output.
// MFMA result register r of lane l: MFMA row 4 * LG * (r / 4) + 4 * (l / T) + r % 4 (a q), MFMA column l % T (a p); LG = 64 / T.
// The wave turns its block through its own piece of LDS (`stage`), a band of 32 p-rows at a time (of
// at most 96 columns), so that every global store instruction writes whole rows of the band.
constexpr int epilogue_columns(int cols) { return cols <= 96 ? cols : cols % 96 == 0 ? 96 : 64; }
constexpr int epilogue_wave_bytes(int cols) { return 32 * (epilogue_columns(cols) + 4) * 4; }

template <class MMA, int TM, int TN>
__device__ __forceinline__ void write_wave_tile(const GemmParams& g, const typename MMA::acc_t (&acc)[TM][TN], uint8_t* stage,
                                                uint32_t lane, uint32_t p0, uint32_t q0, uint32_t slice) {
  constexpr int T = MMA::TILE, LG = 64 / T, IB = 32 / T;
  constexpr int COLS = epilogue_columns(TN * T), JB = COLS / T;
  static_assert(TN % JB == 0 && TM % IB == 0, "whole bands");
  constexpr int EP_PITCH = COLS + 4;                  // floats; +4 staggers the banks
  constexpr int CPR = COLS / 4;                       // 16-byte chunks per band row
  constexpr int EP_ITERS = 32 * CPR / 64;
  uint32_t* ep = reinterpret_cast<uint32_t*>(stage);
  const float s = total_scale(g);
  const bool q_vec = (g.Q & 3u) == 0;
  uint32_t* const pbase = g.nsplit > 1 ? g.partial + (size_t)slice * g.P * g.Q : nullptr;
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += IB) {
#pragma unroll
    for (int j0 = 0; j0 < TN; j0 += JB) {
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
          for (int gq = 0; gq < T / 4 / LG; ++gq) {
            const typename MMA::acc_t& sum = acc[i0 + i][j0 + j];
            *reinterpret_cast<v4u*>(ep + (i * T + lane % T) * EP_PITCH + j * T + 4 * (gq * LG + lane / T)) =
                v4u{MMA::bits(sum[4 * gq]), MMA::bits(sum[4 * gq + 1]), MMA::bits(sum[4 * gq + 2]), MMA::bits(sum[4 * gq + 3])};
          }
      const uint32_t pb = p0 + i0 * T, qb = q0 + j0 * T;
#pragma unroll
      for (int it = 0; it < EP_ITERS; ++it) {
        const uint32_t id = it * 64 + lane, row = id / CPR, c = id % CPR;
        const uint32_t p = pb + row, q = qb + c * 4;
        const v4u raw = *reinterpret_cast<const v4u*>(ep + row * EP_PITCH + c * 4);
        if (p >= g.P || q >= g.Q) continue;
        store_quad<MMA>(g, pbase, p, q, raw, s, q_vec);
      }
    }
  }
}

// One tile of a product: workgroup `block` of its tiles, `lds` a ring of STAGES stages.
// KG > 1: KG groups of WGM x WGN waves share the tile.  Each group multiplies its own sub-steps of every stage, and the
// groups' sums are added through LDS at the end.  For workgroups that are few: a CU with a single workgroup of four waves
// has one wave per SIMD, which nothing covers while it waits for LDS or at the barrier (2048 x 2048 x 4096 int8, with the
// loads of the stages left out 17.8 us, with the matrix work left out 24.0, together 25.4); the groups put two there and a
// longer ring of stages keeps more loads in flight (with four, 17.4 with the matrix work left out, 23.8 in all; with three 23.1).
// SETS = 2 (one group): two sets of accumulators, for the first and the second half of the sub-steps of every stage, added at the
// end: the sums of two groups of waves, in the same order.
template <class MMA, int BM, int BN, int WGM, int WGN, int STAGES, int KG, int SETS>
__device__ __forceinline__ void product_tile(const GemmParams& g, uint32_t block, uint8_t* lds) {
  constexpr int NG = WGM * WGN, NW = NG * KG;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;  // wave tile (p x q)
  constexpr int T = MMA::TILE, LG = 64 / T, TM = WTM / T, TN = WTN / T;
  constexpr int STAGE = (BM + BN) * BK;
  constexpr int XL = BM / 8 / NW, ZL = BN / 8 / NW;  // wave-level DMA instructions per stage
  constexpr int LPW = XL + ZL;
  static_assert(XL * 8 * NW == BM && ZL * 8 * NW == BN, "tile rows must split over the waves");
  static_assert((STAGES - 2) * LPW <= 63 && STAGES >= 2, "vmcnt range");
  using acc_t = typename MMA::acc_t;
  using frag_t = typename MMA::frag_t;
  using raw_t = typename MMA::raw_t;
  constexpr int FC = sizeof(raw_t) / 16;  // 16-byte chunks a lane reads per sub-step
  constexpr int KSUB = BK / MMA::KSTEP / KG;  // sub-steps of a stage that a wave multiplies
  static_assert(KSUB >= 1, "every group has a sub-step");
  static_assert(SETS == 1 || (KG == 1 && SETS == 2 && KSUB % 2 == 0), "two sets stand for two groups");

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);  // the same, known to be uniform
  const uint32_t kg = KG > 1 ? wave_u / NG : 0u;  // group
  const uint32_t wp = wave % NG / WGN, wq = wave % WGN;
  const uint32_t lds_base = (uint32_t)(size_t)(lds_void*)lds;
  // Workgroup -> tile.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs, each
  // with its own L2.  XCD x takes the contiguous range [x * chunk, (x+1) * chunk) of a tile
  // order that walks bands of GROUP tile rows column by column: the workgroups resident on one
  // XCD at a time (one or two per CU, 32 CUs) then cover a compact block of about GROUP x GROUP
  // tiles, and share GROUP X row panels and as many Z row panels in that L2 instead of one X
  // panel and a whole row of Z panels.
  // With the contraction cut into slices the order is slice-major (all tiles of slice 0, then
  // slice 1, ...): an XCD then works mostly inside one slice, i.e. on one range of the
  // contraction of a few panels, instead of on every slice of its tiles.
  constexpr uint32_t GROUP = 8;
  const uint32_t ntiles = g.tiles_p * g.tiles_q, nwork = ntiles * g.nsplit, chunk = (nwork + 7u) >> 3;
  const uint32_t work = (block & 7u) * chunk + (block >> 3);
  if (work >= nwork) return;  // padding of the last XCD's range (whole workgroup leaves)
  const uint32_t slice = work / ntiles, tile = work - slice * ntiles;
  const uint32_t band = tile / (GROUP * g.tiles_q), band_p = band * GROUP;
  const uint32_t band_rows = min(GROUP, g.tiles_p - band_p), in_band = tile - band * GROUP * g.tiles_q;
  const uint32_t tp = band_p + in_band % band_rows, tq = in_band / band_rows;
  const uint32_t p0 = tp * BM, q0 = tq * BN;
  const uint32_t kbeg = slice * g.k_per_split;
  const uint32_t kend = min(g.R, kbeg + g.k_per_split);
  const int ktiles = (int)((kend - kbeg + BK - 1) / BK);

  const __amdgpu_buffer_rsrc_t xrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.X), 0, (int)(g.P * g.pitch), 0x00020000);
  const __amdgpu_buffer_rsrc_t zrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.Z), 0, (int)(g.Q * g.pitch), 0x00020000);

  // LDS layout of a stage: tile row r at r * 128, its logical 16-byte chunk c at physical
  // chunk c ^ ((r >> 1) & 7).  The LDS has 64 banks (256 bytes per cycle) and serves a
  // ds_read_b128 sixteen lanes at a time: sixteen consecutive rows reading the same logical
  // chunk then touch sixteen different 16-byte slots (two rows per 256 bytes, eight swizzle
  // values per row parity), i.e. no bank conflicts.
  // DMA addressing: a wave instruction fills 8 tile rows (1 KiB of LDS, lane L at L*16); lane L
  // fetches row L/8 and the logical chunk whose physical slot is L%8.  (r >> 1) & 7 depends on
  // the parity of the 8-row block, hence two per-lane offsets.
  const uint32_t lrow = lane >> 3;
  const uint32_t lchunk = (lane & 7u) ^ (lane >> 4);  // of an even row block; ^ 4: of an odd one
  const uint32_t xchunk0 = lchunk ^ (XL % 2 ? (wave_u & 1u) * 4u : 0u), xchunk1 = xchunk0 ^ 4u;
  const uint32_t zchunk0 = lchunk ^ (ZL % 2 ? (wave_u & 1u) * 4u : 0u), zchunk1 = zchunk0 ^ 4u;
  const uint32_t xvoff = (p0 + wave * XL * 8 + lrow) * g.pitch + kbeg;
  const uint32_t zvoff = (q0 + wave * ZL * 8 + lrow) * g.pitch + kbeg;

  auto issue = [&](int kt, int buf) {
    const uint32_t koff = (uint32_t)kt * BK;
    // beyond the contraction the lane loads zeros (offset past the buffer)
    const uint32_t xc0 = koff + xchunk0 * 16, xc1 = koff + xchunk1 * 16;
    const uint32_t zc0 = koff + zchunk0 * 16, zc1 = koff + zchunk1 * 16;
    const bool xlive0 = kbeg + xc0 < kend, xlive1 = kbeg + xc1 < kend;
    const bool zlive0 = kbeg + zc0 < kend, zlive1 = kbeg + zc1 < kend;
    const uint32_t xs = lds_base + buf * STAGE + wave_u * XL * 1024;
    const uint32_t zs = lds_base + buf * STAGE + BM * BK + wave_u * ZL * 1024;
#pragma unroll
    for (int i = 0; i < XL; ++i)
      lds_dma16(xrsrc, xs + i * 1024,
                (i & 1) ? (xlive1 ? xvoff + xc1 + i * 8 * g.pitch : OOB) : (xlive0 ? xvoff + xc0 + i * 8 * g.pitch : OOB));
#pragma unroll
    for (int i = 0; i < ZL; ++i)
      lds_dma16(zrsrc, zs + i * 1024,
                (i & 1) ? (zlive1 ? zvoff + zc1 + i * 8 * g.pitch : OOB) : (zlive0 ? zvoff + zc0 + i * 8 * g.pitch : OOB));
  };

  // operand reads: lane (row = lane % T, group = lane / T) takes FC chunks per sub-step, logical chunk
  // (sub-step * LG + group) * FC + c; physical chunk = logical ^ ((row >> 1) & 7)
  const uint32_t swz = ((lane >> 1) & 7u) ^ ((kg * KSUB * LG + lane / T) * FC);
  const uint32_t xoff = (wp * WTM + lane % T) * BK + (swz << 4), zoff = BM * BK + (wq * WTN + lane % T) * BK + (swz << 4);
  auto load_frag = [&](const uint8_t* at, uint32_t off) {
    raw_t f;
#pragma unroll
    for (int c = 0; c < FC; ++c) {
      const v4i part = *reinterpret_cast<const v4i*>(at + (off ^ (c * 16u)));
      f[4 * c + 0] = part[0]; f[4 * c + 1] = part[1]; f[4 * c + 2] = part[2]; f[4 * c + 3] = part[3];
    }
    return f;
  };

  acc_t acc_set[SETS][TM][TN];
  auto& acc = acc_set[0];
#pragma unroll
  for (int h = 0; h < SETS; ++h)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < T * T / 64; ++r) acc_set[h][i][j][r] = 0;

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue(s, s);  // stages past the end load zeros

  // one stage
  auto compute = [&](int buf) {
    const uint8_t* const stage = lds + buf * STAGE;
    if constexpr (T == 16) {
      // After the MFMAs of an X fragment the next sub-step's fragments are read one by one into the registers that have
      // just come free.  Fragments that have to be widened (VALU) are, one ahead, between the MFMAs of the one before, those of Z
      // between the first ones that do without them.  The scheduling barriers pin that order.
      static_assert(!MMA::WIDENS || (TM >= 2 && TN >= 2), "the first fragments of a sub-step are read before they are widened at its turn");
      raw_t xf[TM], zf[2][TN];
      auto fetch_x = [&](int ks, int i) { xf[i] = load_frag(stage + i * T * BK, xoff ^ (ks * LG * FC * 16u)); };
      auto fetch_z = [&](int ks, int j) { zf[ks & 1][j] = load_frag(stage + j * T * BK, zoff ^ (ks * LG * FC * 16u)); };
      fetch_z(0, 0);
      fetch_x(0, 0);
#pragma unroll
      for (int j = 1; j < TN; ++j) fetch_z(0, j);
#pragma unroll
      for (int i = 1; i < TM; ++i) fetch_x(0, i);
      __builtin_amdgcn_sched_barrier(0);
      frag_t xe[2], ze[TN];  // (plain copies unless the pipeline widens its operands)
      if constexpr (MMA::WIDENS) {
        xe[0] = MMA::expand_x(xf[0]);
        ze[0] = MMA::expand_z(zf[0][0]);
      }
#pragma unroll
      for (int ks = 0; ks < KSUB; ++ks) {
        if constexpr (!MMA::WIDENS) {
#pragma unroll
          for (int j = 0; j < TN; ++j) ze[j] = MMA::expand_z(zf[ks & 1][j]);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int n = ks * TM + i;
          const bool turn = i + 1 == TM && ks + 1 < KSUB;
          if constexpr (MMA::WIDENS) {
            if (n + 1 < KSUB * TM) xe[(n + 1) & 1] = MMA::expand_x(xf[(i + 1) % TM]);
          } else {
            xe[n & 1] = MMA::expand_x(xf[i]);
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) {  // MFMA rows: q, columns: p
            acc_t& sum = acc_set[ks * SETS / KSUB][i][j];
            sum = MMA::mma(ze[j], xe[n & 1], sum);
            if constexpr (MMA::WIDENS) {
              if (i == 0 && j + 1 < TN) ze[j + 1] = MMA::expand_z(zf[ks & 1][j + 1]);
              if (turn && j == 0) ze[0] = MMA::expand_z(zf[(ks + 1) & 1][0]);
            }
          }
          if constexpr (MMA::WIDENS) {
            constexpr int N_MFMA = TN * MMA::MFMA_PER_MMA, V = MMA::VALU_PER_EXPAND;
            const int valu = V + (i == 0 ? (TN - 1) * V : 0) + (turn ? V : 0);
#pragma unroll
            for (int m = 0; m < N_MFMA; ++m) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              if (valu > 3 * N_MFMA) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
              else if (valu > N_MFMA) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
              else __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          if (ks + 1 < KSUB) {
            fetch_x(ks + 1, i);
#pragma unroll
            for (int j = i * TN / TM; j < (i + 1) * TN / TM; ++j) fetch_z(ks + 1, j);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    } else {
      // The fragments of the sub-steps up to PF ahead are fetched before sub-step ks is multiplied; the scheduling barriers
      // pin that order (the LDS latency then hides behind the MFMAs) and bound the number of live fragments (registers).
      constexpr int PF = KSUB > 2 ? 2 : 1;
      raw_t xf[PF + 1][TM], zf[PF + 1][TN];
      auto fetch = [&](int ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) xf[ks % (PF + 1)][i] = load_frag(stage + i * T * BK, xoff ^ (ks * LG * FC * 16u));
#pragma unroll
        for (int j = 0; j < TN; ++j) zf[ks % (PF + 1)][j] = load_frag(stage + j * T * BK, zoff ^ (ks * LG * FC * 16u));
      };
#pragma unroll
      for (int ks = 0; ks < PF && ks < KSUB; ++ks) fetch(ks);
      // Operands are widened in registers (VALU) before they are multiplied.  A wave issues in order, so widening a whole
      // sub-step and then multiplying it would leave the matrix pipe idle during the widening: instead the operands of
      // sub-step ks + 1 are widened while the MFMAs of sub-step ks are issued, a few VALU operations after each MFMA (the
      // scheduling groups below pin that interleaving).  Two widened operand sets fit the register file beside these wave tiles.
      constexpr int SETS_X = MMA::WIDENS ? 2 : 1;
      frag_t xe[SETS_X][TM], ze[SETS_X][TN];
      auto widen = [&](int ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) xe[ks % SETS_X][i] = MMA::expand_x(xf[ks % (PF + 1)][i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) ze[ks % SETS_X][j] = MMA::expand_z(zf[ks % (PF + 1)][j]);
      };
      if constexpr (MMA::WIDENS) widen(0);
#pragma unroll
      for (int ks = 0; ks < KSUB; ++ks) {
        if (ks + PF < KSUB) fetch(ks + PF);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!MMA::WIDENS) widen(ks);  // (plain copies)
        else if (ks + 1 < KSUB) widen(ks + 1);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc_t& sum = acc_set[ks * SETS / KSUB][i][j];
            sum = MMA::mma(ze[ks % SETS_X][j], xe[ks % SETS_X][i], sum);
          }
        if constexpr (MMA::WIDENS) {
          constexpr int N_MFMA = TM * TN * MMA::MFMA_PER_MMA, N_VALU = (TM + TN) * MMA::VALU_PER_EXPAND;
#pragma unroll
          for (int m = 0; m < N_MFMA; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                             // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, (N_VALU + N_MFMA - 1) / N_MFMA, 0);  // then a few VALU operations
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // ring of STAGES buffers, one barrier per stage: after the barrier of step kt every wave has
  // finished step kt-1, whose buffer is the one refilled now
  for (int kt0 = 0; kt0 < ktiles; kt0 += STAGES) {
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
      const int kt = kt0 + s;
      if (kt < ktiles) {
        wait_vmcnt<(STAGES - 2) * LPW>();
        __syncthreads();
        issue(kt + STAGES - 1, (s + STAGES - 1) % STAGES);
        compute(s);
      }
    }
  }

  wait_vmcnt<0>();   // the zero-filled stages issued past the end must have landed too
  __syncthreads();
  if constexpr (SETS == 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < T * T / 64; ++r) acc[i][j][r] = acc[i][j][r] + acc_set[SETS - 1][i][j][r];
  }
  if constexpr (KG == 1) {
    static_assert(NW * epilogue_wave_bytes(WTN) <= STAGES * STAGE, "epilogue staging must fit in the operand ring");
    write_wave_tile<MMA, TM, TN>(g, acc, lds + wave * epilogue_wave_bytes(WTN), lane, p0 + wp * WTM, q0 + wq * WTN, slice);
  } else {
    // The groups' sums meet in LDS, IP row blocks of every wave at a time, and are added in a fixed order by the threads
    // that write them out, whole rows of the tile per instruction.
    // Chunk c of 4 sums of row r lies at chunk c ^ (r mod CPR): a lane per row writes to all banks without padded rows.
    constexpr int CPR = BN / 4, RING = STAGES * STAGE;
    constexpr int IP = WTM % 64 == 0 && KG * WGM * 64 * BN * 4 <= RING ? 2 : 1, ROWS = WGM * IP * 32;
    static_assert(KG * ROWS * BN * 4 <= RING && ROWS * CPR % (NW * 64) == 0, "the sums must fit in the ring");
    static_assert(CPR == 16 || CPR == 32, "a power of two, rows of a wave in step with it");
    uint32_t* const ep = reinterpret_cast<uint32_t*>(lds);
    const float s = total_scale(g);
    const bool q_vec = (g.Q & 3u) == 0;
    uint32_t* const pbase = g.nsplit > 1 ? g.partial + (size_t)slice * g.P * g.Q : nullptr;
#pragma unroll
    for (int i0 = 0; i0 < WTM / 32; i0 += IP) {
      uint32_t* const mine = ep + (kg * ROWS + wp * IP * 32) * BN;
#pragma unroll
      for (int i = 0; i < IP * 32 / T; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int gq = 0; gq < T / 4 / LG; ++gq) {
            const acc_t& sum = acc[i0 * 32 / T + i][j];
            const uint32_t row = i * T + lane % T, c = wq * (WTN / 4) + j * (T / 4) + gq * LG + lane / T;
            *reinterpret_cast<v4u*>(mine + row * BN + 4 * (c ^ (row & (CPR - 1)))) =
                v4u{MMA::bits(sum[4 * gq]), MMA::bits(sum[4 * gq + 1]), MMA::bits(sum[4 * gq + 2]), MMA::bits(sum[4 * gq + 3])};
          }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < ROWS * CPR / (NW * 64); ++it) {
        const uint32_t id = it * NW * 64 + tid, row = id / CPR, c = id % CPR;
        const uint32_t p = p0 + row / (IP * 32) * WTM + i0 * 32 + row % (IP * 32), q = q0 + c * 4;
        const uint32_t* const at = ep + row * BN + 4 * (c ^ (row & (CPR - 1)));
        v4u raw = *reinterpret_cast<const v4u*>(at);
#pragma unroll
        for (int k = 1; k < KG; ++k) {
          const v4u more = *reinterpret_cast<const v4u*>(at + k * ROWS * BN);
#pragma unroll
          for (int e = 0; e < 4; ++e) raw[e] = MMA::bits(MMA::from_bits(raw[e]) + MMA::from_bits(more[e]));
        }
        if (p < g.P && q < g.Q) store_quad<MMA>(g, pbase, p, q, raw, s, q_vec);
      }
      if (i0 + IP < WTM / 32) __syncthreads();
    }
  }
}

// Besides its tiles a launch can carry the slice sum of an EARLIER product (`rider`, complete when
// this launch starts): memory-bound work that runs beside the matrix work, in the resident slots
// the tiles leave free and in the tail of the launch, instead of in a launch of its own.  (Its workgroups are given the LDS of a
// tile's: the launch chooses a form that leaves such slots, see choose_launch.)
// Workgroups [0, gemm_blocks) multiply, the rest sum.  (Measured against this: the rider groups
// spread through the launch, every fourth group of 8 -- slower.)
template <class MMA, int BM, int BN, int WGM, int WGN, int STAGES, int KG = 1, int SETS = 1>
__global__ __launch_bounds__(WGM* WGN* KG * 64, SETS) void gemm_nt_kernel(GemmParams g, SliceSum rider, uint32_t gemm_blocks) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  if (blockIdx.x >= gemm_blocks) {
    if (rider.is_int) slice_sum<true>(rider, blockIdx.x - gemm_blocks, gridDim.x - gemm_blocks);
    else slice_sum<false>(rider, blockIdx.x - gemm_blocks, gridDim.x - gemm_blocks);
    return;
  }
  product_tile<MMA, BM, BN, WGM, WGN, STAGES, KG, SETS>(g, blockIdx.x, lds);
}

// Two products in one launch: the uncut weight and input gradients of a layer.  Workgroups [0, blocks_a) multiply the first (the
// one with the longer tiles), the rest the second, in tiles of one size, so that both fill the same slots: the stores of one's tiles go out
// beside the matrix work of the other's, a product of few tiles leaves no CU idle, and there is one start and one end instead of two.
// choose_pair says where that is faster.  The results are bit for bit those of the products in launches of their own.
template <class MMA_, int WGM_, int WGN_, int KG_, int SETS_>
struct Waves {
  using MMA = MMA_;
  static constexpr int WGM = WGM_, WGN = WGN_, KG = KG_, SETS = SETS_, THREADS = WGM * WGN * KG * 64;
};
template <int BM, int BN, int STAGES, class WA, class WB>
__global__ __launch_bounds__(WA::THREADS, (WA::SETS > WB::SETS ? WA::SETS : WB::SETS)) void gemm_pair_kernel(GemmParams a, GemmParams b,
                                                                                                         uint32_t blocks_a) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  static_assert(WA::THREADS == WB::THREADS, "one launch");
  if (blockIdx.x < blocks_a)
    product_tile<typename WA::MMA, BM, BN, WA::WGM, WA::WGN, STAGES, WA::KG, WA::SETS>(a, blockIdx.x, lds);
  else
    product_tile<typename WB::MMA, BM, BN, WB::WGM, WB::WGN, STAGES, WB::KG, WB::SETS>(b, blockIdx.x - blocks_a, lds);
}

// ---- 256 x 256 tiles, workgroups that stay -------------------------------------------------------
// One workgroup per CU walks a list of tiles.  What that buys over one workgroup per tile:
//   - the operand loads of the next tile's first stage are issued during the last stage of the
//     current tile and land while its result is written, so no tile starts with an empty ring;
//   - the result stores of tile i drain while tile i + 1 is multiplied.
// The second point needs care on this chip: loads and stores of a wave share ONE in-order counter
// (vmcnt), so a wave that has result stores in flight cannot wait for a later operand load without
// waiting for those stores as well.  Waves 0-3 ("loaders") issue every operand DMA of the
// workgroup and are the only ones that wait on the counter; all eight multiply (wave tile
// 128 x 64) and every wave writes out its own part of a finished tile, band by band through its own
// piece of the staging area, without a barrier.  The loaders' one wait that can meet stores still
// in flight is the first of the next tile, and it costs less than what it replaced: a form in
// which only waves 4-7 stored -- the others handing them their bands through LDS and two barriers
// per band -- kept the loaders' counter exact and was 1.5 % slower on the Llama-shaped products.
// The ring has two stages of 64 KiB.  Stages are numbered through the whole tile list (`gs`): the
// loaders issue stage gs + 1 -- the next stage of this tile, or the first of the next tile -- at
// the barrier of stage gs, into the buffer that stage gs - 1 has just left.  When a tile is done,
// the buffer of its last stage is the staging area of the epilogue (the other one is receiving the
// next tile's first stage); it is handed back to the ring by the barrier of the next stage.
// Every loop bound below is uniform over the workgroup, so all waves meet at every barrier.
//
// What bounds it: the chip's power as much as its pipes (operands of zeros run 1.3 times as fast), and the operands on their
// way into LDS and out of it again (a stage is 64 KiB in and 192 KiB out for 2048 cycles of MFMAs a SIMD).  Hence MFMA
// tiles of 16 x 16, under which the clock is higher (the fp8 pipeline excepted), and LDS reads one at a time between the
// MFMAs.  int8, us before (32 x 32 tiles, all fragments of a sub-step read at its start) and now, Gaussian codes:
// 8192 x 2048 x 5632 84.9 -> 77.7 (79.2 -> 76.4 with the reads spread), 8192^3 450 -> 411, 65536 x 2048 x 5632 671 -> 645,
// 65536 x 2048 x 2048 264 -> 250, 65536 x 5632 x 2048 719 -> 683; with packed 4-bit X 65536 x 5632 x 2048 700 -> 680 (in the order of a
// step, beside a slice sum, 759 -> 752; it takes 2 to 3 % more cycles).  Whole steps:
// 65536 x 5632 x 2048 2834 -> 2768, 8192 x 2048 x 5632 E4M3 641 -> 603.  Errors against 64 bits of the 8-bit float products are what
// they were (0.9997 to 1.0003 of it over 8 large shapes).  Measured against it, all slower or equal: the two waves of a SIMD
// taking turns at LDS and at the MFMAs, a barrier between the turns, with half stages of 64 bytes (rows of 64 bytes
// come in at 0.75 of the rate of 128) or quarters of the tile, loads two and a half stages ahead: 0.98 to 1.05 of the time; operand
// rows stored in blocks of 8 or 256 so that a load is one piece, or 128 bytes apart beyond the row: 0.97 to 1.01.
struct TileItem {
  uint32_t valid, p0, q0, slice, kbeg, kend;
};

// XP: the X operand holds 4-bit integers, two per byte ("packed": byte j of every 8 holds elements j
// and j + 8 of a run of 16 along the contraction, low and high nibble).  Its rows take 64 bytes of
// a stage, half the DMA instructions, and half the LDS bytes per fragment; a fragment is widened in
// registers to the bytes 16 * value (shift / mask: the nibble's sign bit becomes the byte's), so
// the accumulators hold 16 times the sums and the caller passes alpha / 16 -- powers of two, the
// results are bit for bit those of the one-byte form.
template <class MMA, bool XP>
__global__ __launch_bounds__(512) void gemm_nt_persist_kernel(GemmParams g, SliceSum rider) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int BM = 256, BN = 256, WGN = 4, NW = 8, NLOAD = 4;
  constexpr int WTM = 128, WTN = 64, T = MMA::TILE, TM = WTM / T, TN = WTN / T, HM = TM / 2;
  constexpr int STAGE = (BM + BN) * BK;
  // DMA instructions per loader wave and stage (an instruction covers 8 rows of 128 bytes, or 16 packed rows of 64)
  constexpr int XL = XP ? BM / 16 / NLOAD : BM / 8 / NLOAD, ZL = BN / 8 / NLOAD;
  static_assert(XL % 2 == 0 && ZL % 2 == 0, "row blocks of a wave must start at an even block");
  static_assert(XL + ZL <= 63, "vmcnt range");
  using acc_t = typename MMA::acc_t;
  using frag_t = typename MMA::frag_t;
  using raw_t = typename MMA::raw_t;
  constexpr int FC = sizeof(raw_t) / 16;
  constexpr int KS = BK / MMA::KSTEP;  // sub-steps of a stage
  constexpr int LG = 64 / T;           // lane groups that read a sub-step
  static_assert(HM == TN, "a fragment of Z is fetched beside every fragment of half the X rows");
  static_assert(!XP || (FC == 1 && T == 16 && KS == 2 && sizeof(frag_t) == 16), "packed X: the int8 pipeline only");

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
  const bool loader = wave_u < NLOAD;
  const uint32_t wp = wave / WGN, wq = wave % WGN;
  const uint32_t lds_base = (uint32_t)(size_t)(lds_void*)lds;

  // Tile list of this workgroup.  As in gemm_nt_kernel, XCD x (workgroup ids = x mod 8) owns the
  // contiguous range [x * chunk, (x + 1) * chunk) of the banded, slice-major tile order; its
  // workgroups (slots) walk that range side by side, so the tiles in flight on one XCD at any time
  // are neighbours and share operand panels in that L2.
  constexpr uint32_t GROUP = 8;
  const uint32_t ntiles = g.tiles_p * g.tiles_q, nwork = ntiles * g.nsplit, chunk = (nwork + 7u) >> 3;
  const uint32_t xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3, nslots = gridDim.x >> 3;
  const uint32_t range_end = min(nwork, (xcd + 1) * chunk);
  auto item_at = [&](uint32_t n) {
    TileItem it;
    const uint32_t work = xcd * chunk + slot + n * nslots;
    it.valid = work < range_end ? 1u : 0u;
    const uint32_t w = it.valid ? work : 0u;
    const uint32_t slice = w / ntiles, tile = w - slice * ntiles;
    const uint32_t band = tile / (GROUP * g.tiles_q), band_p = band * GROUP;
    const uint32_t band_rows = min(GROUP, g.tiles_p - band_p), in_band = tile - band * GROUP * g.tiles_q;
    it.p0 = (band_p + in_band % band_rows) * BM;
    it.q0 = (in_band / band_rows) * BN;
    it.slice = slice;
    it.kbeg = slice * g.k_per_split;
    it.kend = min(g.R, it.kbeg + g.k_per_split);
    return it;
  };

  const __amdgpu_buffer_rsrc_t xrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.X), 0, (int)(g.P * g.pitch_x), 0x00020000);
  const __amdgpu_buffer_rsrc_t zrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.Z), 0, (int)(g.Q * g.pitch), 0x00020000);

  // DMA addressing (LDS layout of a stage as in gemm_nt_kernel: 128-byte rows, 16-byte chunk c of
  // row r at chunk c ^ ((r >> 1) & 7)); loader wave w fills tile rows [64 w, 64 w + 64) of X and of Z
  auto issue = [&](const TileItem& it, int kt, uint32_t buf) {
    const uint32_t ln = opaque(lane);
    const uint32_t lrow = ln >> 3;
    const uint32_t lchunk0 = (ln & 7u) ^ (ln >> 4), lchunk1 = lchunk0 ^ 4u;
    const uint32_t xvoff = (it.p0 + wave * XL * 8 + lrow) * g.pitch + it.kbeg;
    const uint32_t zvoff = (it.q0 + wave * ZL * 8 + lrow) * g.pitch + it.kbeg;
    const uint32_t koff = (uint32_t)kt * BK;
    const uint32_t kc0 = koff + lchunk0 * 16, kc1 = koff + lchunk1 * 16;
    const bool live0 = it.kbeg + kc0 < it.kend, live1 = it.kbeg + kc1 < it.kend;
    const uint32_t xs = lds_base + buf * STAGE + wave_u * XL * 1024;
    const uint32_t zs = lds_base + buf * STAGE + BM * BK + wave_u * ZL * 1024;
    if constexpr (XP) {
      // packed rows: 64 bytes of a row per stage, 16 rows per instruction; lane L fetches row L / 4
      // and the logical 16-byte chunk whose physical slot is L % 4 (chunk c of row r is stored at
      // chunk c ^ ((r >> 2) & 3)); a chunk holds 32 elements of the contraction
      const uint32_t pchunk = (ln & 3u) ^ ((ln >> 4) & 3u);
      const uint32_t xvp = (it.p0 + wave * XL * 16 + (ln >> 2)) * g.pitch_x + ((it.kbeg + koff) >> 1) + pchunk * 16;
      const bool livep = it.kbeg + koff + pchunk * 32 < it.kend;
#pragma unroll
      for (int i = 0; i < XL; ++i) lds_dma16(xrsrc, xs + i * 1024, livep ? xvp + i * 16 * g.pitch_x : OOB);
    } else {
#pragma unroll
      for (int i = 0; i < XL; ++i)
        lds_dma16(xrsrc, xs + i * 1024,
                  (i & 1) ? (live1 ? xvoff + kc1 + i * 8 * g.pitch : OOB) : (live0 ? xvoff + kc0 + i * 8 * g.pitch : OOB));
    }
#pragma unroll
    for (int i = 0; i < ZL; ++i)
      lds_dma16(zrsrc, zs + i * 1024,
                (i & 1) ? (live1 ? zvoff + kc1 + i * 8 * g.pitch : OOB) : (live0 ? zvoff + kc0 + i * 8 * g.pitch : OOB));
  };

  // Operand reads: lane (row = lane % T, group = lane / T) takes FC chunks of a sub-step, logical chunk
  // (ks * LG + group) * FC + c.  Packed X: the 16 bytes of a lane group are two runs of 16 elements, one for each
  // sub-step, so Z's chunk there is 2 * group + ks; row pitch 64, chunk c of row r at c ^ ((r >> 2) & 3).
  constexpr uint32_t KS_XOR = XP ? 16u : 16u * LG * FC;
  const uint32_t zoff = BM * BK + (wq * WTN + lane % T) * BK + ((((lane >> 1) & 7u) ^ ((lane / T) * (XP ? 2 : FC))) << 4);
  const uint32_t xoff = XP ? (wp * WTM + lane % T) * 64u + ((((lane / T) ^ (lane >> 2)) & 3u) << 4)
                           : (wp * WTM + lane % T) * BK + ((((lane >> 1) & 7u) ^ ((lane / T) * FC)) << 4);
  auto load_frag = [&](const uint8_t* at, uint32_t off) {
    raw_t f;
#pragma unroll
    for (int c = 0; c < FC; ++c) {
      const v4i part = *reinterpret_cast<const v4i*>(at + (off ^ (c * 16u)));
      f[4 * c + 0] = part[0]; f[4 * c + 1] = part[1]; f[4 * c + 2] = part[2]; f[4 * c + 3] = part[3];
    }
    return f;
  };

  acc_t acc[TM][TN];
  // A stage is a row of units: a sub-step of half the wave's X rows.  A unit's fragments of X are read one by one into the
  // registers that the unit before has just left, and the next sub-step's fragments of Z beside them: LDS reads spread
  // between the MFMAs, and few enough registers (int8 216, packed X and fp8 222, bfloat16 217) that two waves of this kernel leave a
  // SIMD 64, enough for one wave of the quantizer or absmax kernels: a memory-bound launch on another stream runs BESIDE this kernel
  // on the same CUs instead of behind it.  Widened codes take 230 and leave 48: room for the quantizers in the source layout and the
  // absmax of a binary32 tensor, not for the kernels of several tensors at once.  (With X read four ahead and all of Z before
  // the turn 242, beside which nothing fits: E5M2, both products of 8192 x 8192 x 2048 alone 368 us and 367 now, beside an int8
  // quantizer of 2^26 elements on another stream 431 and 404, beside their absmax 443 and 404.  With X two ahead and only the
  // first fragment of Z before the turn 222, but 1.02 to 1.04 of the time.)
  auto compute = [&](uint32_t buf) {
    const uint8_t* const stage = lds + buf * STAGE;
    if constexpr (!XP) {
      constexpr int AHEAD = MMA::WIDENS ? HM - 1 : HM, Z_LATE = MMA::WIDENS ? 2 : 0;  // (below)
      raw_t xf[HM], zf[2][TN];
      auto fetch_x = [&](int u, int i) { xf[i] = load_frag(stage + ((u & 1) * HM + i) * T * BK, xoff ^ ((u >> 1) * KS_XOR)); };
      auto fetch_z = [&](int ks, int j) { zf[ks & 1][j] = load_frag(stage + j * T * BK, zoff ^ (ks * KS_XOR)); };
      fetch_z(0, 0);
      fetch_x(0, 0);
#pragma unroll
      for (int j = 1; j < TN; ++j) fetch_z(0, j);
#pragma unroll
      for (int i = 1; i < AHEAD; ++i) fetch_x(0, i);
      __builtin_amdgcn_sched_barrier(0);
      frag_t xe[2], ze[TN];  // (plain copies unless the pipeline widens its operands)
      if constexpr (MMA::WIDENS) {
        xe[0] = MMA::expand_x(xf[0]);
        ze[0] = MMA::expand_z(zf[0][0]);
      }
#pragma unroll
      for (int u = 0; u < 2 * KS; ++u) {
        if (!MMA::WIDENS && (u & 1) == 0) {
#pragma unroll
          for (int j = 0; j < TN; ++j) ze[j] = MMA::expand_z(zf[(u >> 1) & 1][j]);
        }
#pragma unroll
        for (int i = 0; i < HM; ++i) {
          const bool first = (u & 1) == 0 && i == 0, turn = (u & 1) == 1 && i + 1 == HM && u + 1 < 2 * KS;
          if constexpr (MMA::WIDENS) {  // the next fragments are widened beside the MFMAs of these
            if (i + 1 < HM || u + 1 < 2 * KS) xe[(i + 1) & 1] = MMA::expand_x(xf[(i + 1) % HM]);
          } else {
            xe[i & 1] = MMA::expand_x(xf[i]);
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc_t& sum = acc[(u & 1) * HM + i][j];
            sum = MMA::mma(ze[j], xe[i & 1], sum);
            if constexpr (MMA::WIDENS) {
              if (first && j + 1 < TN) ze[j + 1] = MMA::expand_z(zf[(u >> 1) & 1][j + 1]);
              if (turn && j == 0) ze[0] = MMA::expand_z(zf[((u >> 1) + 1) & 1][0]);
            }
          }
          if constexpr (MMA::WIDENS) {
            constexpr int N_MFMA = TN * MMA::MFMA_PER_MMA;
#pragma unroll
            for (int m = 0; m < N_MFMA; ++m) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              if (first) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
              else if (turn) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
              else __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          // X: the fragment that takes the place just left, four ahead; three where widened ones take registers too.  Z: beside the
          // first unit's; where they are widened the last two at the turn, into the registers of the widened ones that it frees.
          const int n = u * HM + i + AHEAD;
          if (n < 2 * KS * HM) fetch_x(n / HM, n % HM);
          if ((u & 1) == 0 && u + 2 < 2 * KS && i < TN - Z_LATE) fetch_z((u >> 1) + 1, i);
          if (turn) {
#pragma unroll
            for (int j = TN - Z_LATE; j < TN; ++j) fetch_z((u >> 1) + 1, j);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
      // Packed X: 32 elements a lane and fragment, all of a stage's read at its start; the halves (h) and sub-steps (ks) in
      // the order (0,0) (1,0) (1,1) (0,1), so that Z is read once.  Fragment n + 1 of the sixteen is widened beside the
      // MFMAs of fragment n (widened a unit at a time, before its MFMAs: 6 % slower, as much as the tiles of 16 gain).
      raw_t xf[2][HM], zf[TN];
      auto fetch_z = [&](int ks, int j) { zf[j] = load_frag(stage + j * T * BK, zoff ^ (ks * KS_XOR)); };
      auto widen = [&](int n) {
        const int ks = n >> 3, h = ((n >> 2) & 1) ^ ks, i = n & 3;
        // byte j of the 8 of a run holds elements j (low nibble) and j + 8 (high nibble): four words of 16 * value
        const int x0 = xf[h][i][2 * ks], x1 = xf[h][i][2 * ks + 1], hi = (int)0xF0F0F0F0u;
        return frag_t{(x0 << 4) & hi, (x1 << 4) & hi, x0 & hi, x1 & hi};
      };
#pragma unroll
      for (int j = 0; j < TN; ++j) fetch_z(0, j);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < HM; ++i) xf[h][i] = load_frag(stage + (h * HM + i) * T * 64, xoff);
      __builtin_amdgcn_sched_barrier(0);
      frag_t xe[2];
      xe[0] = widen(0);
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        const int ks = n >> 3, h = ((n >> 2) & 1) ^ ks, i = n & 3;
        if (n < 15) xe[(n + 1) & 1] = widen(n + 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc_t& sum = acc[h * HM + i][j];
          sum = MMA::mma(zf[j], xe[n & 1], sum);
          if (n == 7) {  // the last MFMA that reads this fragment of the first sub-step
            __builtin_amdgcn_sched_barrier(0);
            fetch_z(1, j);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (n != 7) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // Epilogue staging: every wave owns 8 KiB, a band of 32 p-rows x 64 q as rows of 256 bytes
  // (16 chunks of 16 bytes); chunk c of row r is stored at chunk c ^ (r & 15), so that the
  // sixteen lanes an LDS instruction serves together -- sixteen rows with one chunk index when
  // the MFMA registers are written, sixteen chunks of one row when the rows are read back --
  // always fall on sixteen different 16-byte slots of the 64 banks.
  constexpr int EP_WAVE = 32 * WTN * 4;
  static_assert(NW * EP_WAVE <= STAGE, "epilogue staging must fit in one ring buffer");
  const float s = total_scale(g);
  const bool q_vec = (g.Q & 3u) == 0;

  TileItem cur = item_at(0);
  uint32_t n_item = 0, gs = 0;
  if (cur.valid) {
    if (loader) issue(cur, 0, 0);
    while (true) {
      const TileItem nxt = item_at(++n_item);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < T * T / 64; ++r) acc[i][j][r] = 0;
      const int ktiles = (int)((cur.kend - cur.kbeg + BK - 1) / BK);
      for (int kt = 0; kt < ktiles; ++kt) {
        if (loader) wait_vmcnt<0>();  // stage gs has landed (the only DMAs in flight)
        __syncthreads();              // ... for every wave; and every wave has left stage gs - 1
        if (loader) {
          if (kt + 1 < ktiles) issue(cur, kt + 1, (gs + 1) & 1u);
          else if (nxt.valid) issue(nxt, 0, (gs + 1) & 1u);
        }
        compute(gs & 1u);
        ++gs;
      }
      __syncthreads();  // the buffer of the last stage is free: it stages the result
      uint8_t* const stg = lds + ((gs - 1) & 1u) * STAGE;
      uint32_t* const pbase = g.nsplit > 1 ? g.partial + (size_t)cur.slice * g.P * g.Q : nullptr;
      // whole tile inside the output, rows 16-byte aligned, nothing to add to: plain row stores
      const bool fast = q_vec && !g.accumulate && cur.p0 + BM <= g.P && cur.q0 + BN <= g.Q;
#pragma unroll
      for (int i = 0; i < WTM / 32; ++i) {
        // MFMA result register r of lane l: q = 4 LG (r / 4) + 4 (l / T) + r % 4, p = l % T.
        // Final results are converted and scaled here, by the wave that computed them (all eight
        // share that work); partial results of a slice go out as raw accumulator bits.
        const uint32_t le = opaque(lane);
        uint8_t* const mine = stg + wave_u * EP_WAVE;
#pragma unroll
        for (int h = 0; h < 32 / T; ++h)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int gq = 0; gq < T / 4 / LG; ++gq) {
              const acc_t& sum = acc[i * (32 / T) + h][j];
              const uint32_t row = h * T + le % T, c = j * (T / 4) + gq * LG + le / T;
              v4u w;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                w[e] = pbase ? MMA::bits(sum[4 * gq + e]) : __float_as_uint(__fmul_rn(MMA::to_f32(sum[4 * gq + e]), s));
              *reinterpret_cast<v4u*>(mine + row * (WTN * 4) + ((c ^ (row & 15u)) << 4)) = w;
            }
        // the wave reads back what it has just written (its LDS instructions complete in order) and
        // writes whole rows of its band
        __builtin_amdgcn_wave_barrier();
        {
          {
            const uint32_t src = wave_u;
            const uint32_t pb = cur.p0 + (src / WGN) * WTM + i * 32, qw0 = cur.q0 + (src % WGN) * WTN;
            const uint8_t* const band = stg + src * EP_WAVE;
            const uint32_t ls = opaque(lane);
            const uint32_t r4 = ls >> 4, c = ls & 15u;
            if (fast) {
              // EB row reads in flight, then EB stores of four whole 256-byte rows each
              constexpr int EB = FC > 1 ? 4 : 8;  // (the pipeline with 32-byte fragments has fewer registers to spare)
              uint32_t* const dst0 = (pbase ? pbase : reinterpret_cast<uint32_t*>(g.out)) +
                                     (size_t)(pb + r4) * g.Q + qw0 + c * 4;
#pragma unroll
              for (int it0 = 0; it0 < 8; it0 += EB) {
                v4u raw[EB];
#pragma unroll
                for (int it = 0; it < EB; ++it) {
                  const uint32_t row = (it0 + it) * 4 + r4;
                  raw[it] = *reinterpret_cast<const v4u*>(band + row * (WTN * 4) + ((c ^ (row & 15u)) << 4));
                }
#pragma unroll
                for (int it = 0; it < EB; ++it) {
                  uint32_t* const dst = dst0 + (size_t)(it0 + it) * 4 * g.Q;
                  if (pbase) {
                    // write-through: the partial tile does not stay dirty in the L2, and the sum
                    // that reads it next still finds it in the last-level cache
                    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" : : "v"(dst), "v"(raw[it]) : "memory");
                  } else {
                    // not read again by this kernel: a streaming store keeps it from pushing
                    // operand panels out of the L2
                    __builtin_nontemporal_store(raw[it], reinterpret_cast<v4u*>(dst));
                  }
                }
              }
            } else {
#pragma unroll 2
              for (int it = 0; it < 8; ++it) {
                const uint32_t row = it * 4 + r4;
                const v4u raw = *reinterpret_cast<const v4u*>(band + row * (WTN * 4) + ((c ^ (row & 15u)) << 4));
                const uint32_t p = pb + row, q = qw0 + c * 4;
                if (p >= g.P || q >= g.Q) continue;
                const size_t idx = (size_t)p * g.Q + q;
                if (pbase) {
                  if (q_vec) {
                    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" : : "v"(pbase + idx), "v"(raw) : "memory");
                  } else {
                    for (int e = 0; e < 4 && q + e < g.Q; ++e) pbase[idx + e] = raw[e];
                  }
                } else {
                  float v[4];
#pragma unroll
                  for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(raw[e]);
                  float* dst = g.out + idx;
                  if (q_vec) {
                    if (g.accumulate) {
                      const v4f o = *reinterpret_cast<const v4f*>(dst);
#pragma unroll
                      for (int e = 0; e < 4; ++e) v[e] = __fadd_rn(v[e], o[e]);
                    }
                    __builtin_nontemporal_store(v4f{v[0], v[1], v[2], v[3]}, reinterpret_cast<v4f*>(dst));
                  } else {
                    for (int e = 0; e < 4 && q + e < g.Q; ++e) dst[e] = g.accumulate ? __fadd_rn(v[e], dst[e]) : v[e];
                  }
                }
              }
            }
          }
        }
      }
      if (!nxt.valid) break;
      cur = nxt;
    }
  }
  // the slice sum of an earlier product, if this launch carries one: every workgroup takes a share
  // once its tiles are done
  if (rider.total > 0) {
    if (rider.is_int) slice_sum<true>(rider, blockIdx.x, gridDim.x);
    else slice_sum<false>(rider, blockIdx.x, gridDim.x);
  }
}

// ---- binary32 rows times bfloat16 columns (the weight-only objective) ---------------------------
// X is binary32 as the caller has it; the bf16 pipeline multiplies it exactly once it is cut into three
// bfloat16 numbers that sum to it: p0 its top 8 significand bits, p1 the top 8 of the remainder, p2 what
// is left (binary32 has 24 bits; both subtractions are exact; a non-finite x gives a NaN part).  The
// cut is made in registers, between the LDS read and the MFMAs: 512 values cost a wave 44 vector
// operations and feed 3 TN MFMAs, so a wave owns 32 rows and ALL columns of the workgroup's tile (no
// other wave cuts the same values), and the vector work hides behind the matrix work of the other
// waves of the SIMD.  The matrix pipe bounds it: three products per value are what exactness costs.
// Compared with planes written to memory by a kernel of their own and one product over the tripled
// contraction (the earlier form) there is no 6-byte copy of X, no threefold copy of Z, and a Z
// fragment read from LDS serves three MFMAs.  Whole calls, int8 weights, us before and now: 8192 x 3072 x 768
// forward 136 -> 110, its input gradient 165 -> 121; 16384 x 4096 x 1024 374 -> 348 (1.2 PFLOP/s of MFMAs)
// and 457 -> 350; 272 x 4096 x 4096 93 -> 59; 256 x 256 x 256 19 -> 13.  Three stages in the ring (two
// workgroups per CU instead of three): 110 -> 113, 348 -> 365.
// A stage is 32 elements of the contraction: rows of 128 bytes of X (chunk c of row r at
// c ^ ((r >> 1) & 7), as above) and of 64 bytes of Z (chunk c of row r at c ^ ((r >> 2) & 3): sixteen
// consecutive rows reading one chunk fall on sixteen different 16-byte slots of the 64 banks).
// g.R, g.pitch, g.k_per_split: bytes of Z; a byte of Z stands for two of X.
__device__ __forceinline__ void cut3(const v4f (&x)[2], v4i (&plane)[3]) {
  uint32_t b0[8], b1[8], b2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = x[e >> 2][e & 3];
    b0[e] = __float_as_uint(v);
    const float r1 = __fsub_rn(v, __uint_as_float(b0[e] & 0xFFFF0000u));
    b1[e] = __float_as_uint(r1);
    b2[e] = __float_as_uint(__fsub_rn(r1, __uint_as_float(b1[e] & 0xFFFF0000u)));
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {  // the high halves of two neighbours
    plane[0][e] = (int)__builtin_amdgcn_perm(b0[2 * e + 1], b0[2 * e], 0x07060302u);
    plane[1][e] = (int)__builtin_amdgcn_perm(b1[2 * e + 1], b1[2 * e], 0x07060302u);
    plane[2][e] = (int)__builtin_amdgcn_perm(b2[2 * e + 1], b2[2 * e], 0x07060302u);
  }
}

// TWO: the large parts gather in one set of accumulators, the middle and small ones in another, and the two are added
// at the end.  A binary32 sum rounds at its own size whatever it is given, so one set over all three parts rounds
// three times for every 16 products instead of once: error over the 2-norm, 736 x 688 x 1744 2.5e-7 with one set,
// 7.1e-8 with two, 10976 x 1760 x 3312 5.4e-7 and 1.4e-7.  Twice the accumulators are 211 registers instead of 148
// (with MFMA tiles of 32 x 32 189 and 128), two workgroups per CU instead of three: with those 8192 x 3072 x 768 forward and input gradient 233 us against 253, 16384 x 4096
// x 1024 737 against 774.  Three stages in that ring (147 KiB of LDS): 251 and 767.  make_cut3_plan says which.
template <class MMA, int NW, int TN, int STAGES, bool TWO>
__global__ __launch_bounds__(NW * 64, TWO ? 2 : 1) void gemm_cut3_kernel(GemmParams g) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int BM = 32 * NW, BN = 32 * TN;
  constexpr int XROW = 128, ZROW = 64;  // bytes of a stage per row
  constexpr int STAGE = BM * XROW + BN * ZROW;
  constexpr int XL = BM / 8 / NW, ZL = BN / 16 / NW, LPW = XL + ZL;  // wave-level DMA instructions per stage
  static_assert(XL == 4 && ZL * 16 * NW == BN && (STAGES - 2) * LPW <= 63, "DMA split over the waves");
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds_base = (uint32_t)(size_t)(lds_void*)lds;
  // workgroup -> tile as in gemm_nt_kernel
  constexpr uint32_t GROUP = 8;
  const uint32_t ntiles = g.tiles_p * g.tiles_q, nwork = ntiles * g.nsplit, chunk = (nwork + 7u) >> 3;
  const uint32_t work = (blockIdx.x & 7u) * chunk + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= chunk || work >= nwork) return;
  const uint32_t slice = work / ntiles, tile = work - slice * ntiles;
  const uint32_t band = tile / (GROUP * g.tiles_q), band_p = band * GROUP;
  const uint32_t band_rows = min(GROUP, g.tiles_p - band_p), in_band = tile - band * GROUP * g.tiles_q;
  const uint32_t p0 = (band_p + in_band % band_rows) * BM, q0 = (in_band / band_rows) * BN;
  const uint32_t kbeg = slice * g.k_per_split, kend = min(g.R, kbeg + g.k_per_split);
  const int ktiles = (int)((kend - kbeg + ZROW - 1) / ZROW);

  const __amdgpu_buffer_rsrc_t xrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.X), 0, (int)(g.P * g.pitch_x), 0x00020000);
  const __amdgpu_buffer_rsrc_t zrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.Z), 0, (int)(g.Q * g.pitch), 0x00020000);

  // DMA: an instruction fills 8 rows of X (lane L: row L / 8, the chunk whose slot is L % 8; the swizzle
  // depends on the parity of the 8-row block) or 16 rows of Z (row L / 4, the chunk whose slot is L % 4)
  const uint32_t xc0 = ((lane & 7u) ^ (lane >> 4)) * 16, xc1 = xc0 ^ 64u;
  const uint32_t zc = ((lane & 3u) ^ ((lane >> 4) & 3u)) * 16;
  const uint32_t xvoff = (p0 + wave * 32 + (lane >> 3)) * g.pitch_x;
  const uint32_t zvoff = (q0 + wave * ZL * 16 + (lane >> 2)) * g.pitch;
  auto issue = [&](int kt, int buf) {
    const uint32_t zk = kbeg + (uint32_t)kt * ZROW, xk = 2 * zk;
    const uint32_t xs = lds_base + buf * STAGE + wave * 32 * XROW;
    const uint32_t zs = lds_base + buf * STAGE + BM * XROW + wave * ZL * 1024;
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const uint32_t k = xk + ((i & 1) ? xc1 : xc0);
      lds_dma16(xrsrc, xs + i * 1024, k < 2 * kend ? xvoff + i * 8 * g.pitch_x + k : OOB);
    }
    const uint32_t k = zk + zc;
#pragma unroll
    for (int i = 0; i < ZL; ++i) lds_dma16(zrsrc, zs + i * 1024, k < kend ? zvoff + i * 16 * g.pitch + k : OOB);
  };

  // operand reads: lane (row = lane % T, group = lane / T) takes 8 elements of the contraction.  A wave's 32 rows of a stage are
  // two fragments: two sub-steps (32 x 32 MFMA tiles) or two blocks of 16 rows (16 x 16, a stage deep)
  constexpr int T = MMA::TILE, KS = T / 16, RT = 32 / T, CN = BN / T;
  using acc_t = typename MMA::acc_t;
  uint32_t xoff[4], zoff[KS];
#pragma unroll
  for (int t = 0; t < 4; ++t)
    xoff[t] = (wave * 32 + (KS == 1 ? (t >> 1) * 16 : 0) + lane % T) * XROW +
              (((2 * (lane / T) + (t & 1) + (KS == 2 ? (t >> 1) * 4 : 0)) ^ ((lane >> 1) & 7u)) << 4);
#pragma unroll
  for (int t = 0; t < KS; ++t) zoff[t] = BM * XROW + (lane % T) * ZROW + (((2 * t + lane / T) ^ ((lane >> 2) & 3u)) << 4);

  acc_t acc[RT][CN], low[TWO ? RT : 1][TWO ? CN : 1];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CN; ++j)
#pragma unroll
      for (int r = 0; r < T * T / 64; ++r) acc[i][j][r] = low[TWO ? i : 0][TWO ? j : 0][r] = 0.0f;

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue(s, s);  // stages past the end load zeros
  for (int kt0 = 0; kt0 < ktiles; kt0 += STAGES) {
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
      const int kt = kt0 + s;
      if (kt < ktiles) {
        wait_vmcnt<(STAGES - 2) * LPW>();
        __syncthreads();
        issue(kt + STAGES - 1, (s + STAGES - 1) % STAGES);
        const uint8_t* const stage = lds + s * STAGE;
        v4f x[2][2];
        v4i z[KS][CN];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          x[n][0] = *reinterpret_cast<const v4f*>(stage + xoff[2 * n]);
          x[n][1] = *reinterpret_cast<const v4f*>(stage + xoff[2 * n + 1]);
          if (n < KS) {
#pragma unroll
            for (int j = 0; j < CN; ++j) z[n][j] = *reinterpret_cast<const v4i*>(stage + zoff[n] + j * T * ZROW);
          }
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const int i = n % RT, ks = n % KS;
          v4i plane[3];
          cut3(x[n], plane);
#pragma unroll
          for (int b = 2; b >= 0; --b)  // small parts first
#pragma unroll
            for (int j = 0; j < CN; ++j) {
              acc_t& sum = TWO && b > 0 ? low[TWO ? i : 0][TWO ? j : 0] : acc[i][j];
              sum = MMA::mma(z[ks][j], plane[b], sum);
            }
        }
      }
    }
  }
  wait_vmcnt<0>();
  __syncthreads();
  if constexpr (TWO) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CN; ++j)
#pragma unroll
        for (int r = 0; r < T * T / 64; ++r) acc[i][j][r] = __fadd_rn(acc[i][j][r], low[i][j][r]);
  }
  static_assert(NW * epilogue_wave_bytes(32 * TN) <= STAGES * STAGE, "epilogue staging must fit in the operand ring");
  write_wave_tile<MMA, RT, CN>(g, acc, lds + wave * epilogue_wave_bytes(32 * TN), lane, p0 + wave * 32, q0, slice);
}

// The slice sum in a launch of its own.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(SliceSum r) {
  if (r.is_int) slice_sum<true>(r, blockIdx.x, gridDim.x);
  else slice_sum<false>(r, blockIdx.x, gridDim.x);
}

// What a launch is asked to do about slice sums: carry the one of an earlier product (`carry`,
// may be null or empty), and either run its own afterwards or hand it to the caller (`defer`).
struct SliceSumPlan {
  const SliceSum* carry;
  SliceSum* defer;
};

// per_thread elements per thread where the vector path applies (a launch of its own wants many
// small workgroups, riders few and fat ones: each holds a tile's slot), at most 4096 workgroups
uint32_t slice_sum_blocks(const SliceSum& r, uint32_t threads, uint32_t per_thread) {
  const size_t per_block = (size_t)threads * ((r.total & 3u) == 0 ? per_thread : 1);
  size_t blocks = (r.total + per_block - 1) / per_block;
  if (blocks > 4096) blocks = 4096;
  return (uint32_t)(blocks < 1 ? 1 : blocks);
}

// The slice sum of a product (nothing to sum if it is not cut).
template <class MMA>
SliceSum own_slice_sum(const GemmParams& g) {
  SliceSum own{};
  if (g.nsplit > 1) {
    own.partial = g.partial; own.out = g.out; own.nsplit = g.nsplit; own.total = (size_t)g.P * g.Q;
    own.s = GemmScale{g.alpha, g.sx, g.sz, g.sx_dev, g.sz_dev};
    own.accumulate = g.accumulate;
    own.is_int = std::is_base_of<I8Mma, MMA>::value ? 1 : 0;
  }
  return own;
}

template <class MMA, int BM, int BN, int WGM, int WGN, int STAGES, int KG = 1, int SETS = 1>
hipError_t launch_tile(GemmParams g, const SliceSumPlan& ss, hipStream_t stream) {
  constexpr int LDS_BYTES = STAGES * (BM + BN) * BK;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
  auto kern = &gemm_nt_kernel<MMA, BM, BN, WGM, WGN, STAGES, KG, SETS>;
  // once per kernel (a function-local static: its initialisation is safe against concurrent
  // first calls from several host threads)
  static const hipError_t configured = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
  if (configured != hipSuccess) return configured;
  g.tiles_p = (g.P + BM - 1) / BM;
  g.tiles_q = (g.Q + BN - 1) / BN;
  const uint32_t gemm_blocks = ((g.tiles_p * g.tiles_q * g.nsplit + 7) / 8) * 8;
  SliceSum carry{};
  uint32_t carry_blocks = 0;
  if (ss.carry && ss.carry->total > 0) {
    carry = *ss.carry;
    carry_blocks = slice_sum_blocks(carry, WGM * WGN * KG * 64, 16);
  }
  kern<<<dim3(gemm_blocks + carry_blocks), WGM * WGN * KG * 64, LDS_BYTES, stream>>>(g, carry, gemm_blocks);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const SliceSum own = own_slice_sum<MMA>(g);
  if (ss.defer) {
    *ss.defer = own;
  } else if (own.total > 0) {
    splitk_reduce_kernel<<<slice_sum_blocks(own, 256, 4), 256, 0, stream>>>(own);
    e = hipGetLastError();
  }
  return e;
}

// The 256 x 256 tiles on workgroups that stay (gemm_nt_persist_kernel): one workgroup per CU, or
// fewer if there is less work.
template <class MMA32, bool XP = false>
hipError_t launch_persist(GemmParams g, const SliceSumPlan& ss, hipStream_t stream) {
  using MMA = typename Tiles16<MMA32>::type;
  constexpr int LDS_BYTES = 2 * (256 + 256) * BK;
  auto kern = &gemm_nt_persist_kernel<MMA, XP>;
  static const hipError_t configured = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
  if (configured != hipSuccess) return configured;
  g.tiles_p = (g.P + 255) / 256;
  g.tiles_q = (g.Q + 255) / 256;
  const uint32_t nwork = g.tiles_p * g.tiles_q * g.nsplit, chunk = (nwork + 7) / 8;
  const uint32_t slots = chunk < NUM_CU / 8 ? chunk : NUM_CU / 8;  // workgroups per XCD
  SliceSum carry{};
  if (ss.carry && ss.carry->total > 0) carry = *ss.carry;
  kern<<<dim3(8 * slots), 512, LDS_BYTES, stream>>>(g, carry);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const SliceSum own = own_slice_sum<MMA>(g);
  if (ss.defer) {
    *ss.defer = own;
  } else if (own.total > 0) {
    splitk_reduce_kernel<<<slice_sum_blocks(own, 256, 4), 256, 0, stream>>>(own);
    e = hipGetLastError();
  }
  return e;
}

// Which forms multiply in MFMA tiles of 16 x 16 (srq_mma.hpp): those whose workgroups fill the chip, so that its clock counts.  Where
// a CU has one workgroup, or its waves wait for each other's sums, it is the loads and the chain of a tile that count, and 32 x 32 ones are
// faster.  Kernels, us, 32 x 32 and 16 x 16:
//   128 x 128, one set of sums: int8 5552 x 1840 x 1184 with the other product of the call 47.2 -> 46.0, 2176 x 1232 x 8320 35.0 -> 33.1; bfloat16 values
//   1856 x 3312 x 1088 19.8 -> 18.5; widened codes 4368 x 8656 x 240 42.1 -> 40.0, pairs 0.95 to 1.0 of
//   the time.  One or two stages on a CU each: 6.2 and 6.3.
//   128 x 128, two groups: int8 2208 x 208 x 9248 16.2 -> 15.7, 3168 x 800 x 944 8.3 -> 8.4, 18 shapes 0.99 of the time; bfloat16
//   values 24.5 -> 26.5 at 3344 x 880 x 2944, 18 shapes 1.02; widened codes, half a stage a single sub-step with nothing to widen beside,
//   2048 x 2048 x 4096 38.5 -> 41.5 (with the groups taking turns at LDS and the MFMAs 43.5).  Two sets have the tiles of two groups, as
//   64 x 64 do, so that their binary32 sums stay the same bit for bit.
//   128 x 192: int8 4864 x 4960 x 624 32.5 -> 30.3; bfloat16 values 46.0 -> 42.6; widened codes, which are the most work between the
//   reads, 37.9 -> 35.5, with 458 tiles 29264 x 304 x 1648 4 less of 268 for its step, with 333 14160 x 528 x 272 21.7 -> 21.1; with a CU
//   for each tile 30.0 -> 31.5 at 1088 x 4576 x 2496 and 53.5 -> 56.4 at 4544 x 528 x 8688 in two slices (11 shapes 1.02 to 1.09 of the time).
//   64 x 64: int8 320 x 1552 x 4336 8.4 -> 8.8, bfloat16 values 448 x 1792 x 1152 6.0 -> 6.3.
// `large`: one set of sums of widened codes in MFMA tiles of 32 x 32 (sums_in_large_mfma, large_mfma_of_gradient).
template <class MMA>
hipError_t launch_mma(GemmParams g, const Launch& l, bool large, const SliceSumPlan& ss, hipStream_t stream) {
  constexpr bool IS_INT = std::is_same<MMA, I8Mma>::value;
  using Mma16 = typename Tiles16<MMA>::type;
  g.nsplit = l.nsplit;
  g.k_per_split = l.k_per_split;
  switch (l.form) {
    case FORM_256x256: return launch_persist<MMA>(g, ss, stream);                          // 8 waves of 128 x 64, persistent
    case FORM_128x128: return launch_tile<Mma16, 128, 128, 2, 2, 2>(g, ss, stream);        // 4 waves of 64 x 64
    case FORM_128x128_S2:  // binary32 sums only (choose_launch)
      if constexpr (!IS_INT) return launch_tile<MMA, 128, 128, 2, 2, 2, 1, 2>(g, ss, stream);
      break;
    case FORM_128x128_G2:                                                                  // 8 waves of 64 x 64
      return launch_tile<typename std::conditional<IS_INT, Mma16, MMA>::type, 128, 128, 2, 2, 3, 2>(g, ss, stream);
    case FORM_128x192:                                                                     // 4 waves of 64 x 96
      if constexpr (MMA::WIDENS) {
        if (large) return launch_tile<MMA, 128, 192, 2, 2, 2>(g, ss, stream);
      }
      return launch_tile<Mma16, 128, 192, 2, 2, 2>(g, ss, stream);
    case FORM_64x64_G2:                                                                    // 8 waves of 32 x 32
      return l.ring == 3 ? launch_tile<MMA, 64, 64, 2, 2, 3, 2>(g, ss, stream) : launch_tile<MMA, 64, 64, 2, 2, 4, 2>(g, ss, stream);
    case FORM_64x64_G4:  // 8 waves of 64 x 32; binary32 sums only (choose_launch)
      if constexpr (BK / MMA::KSTEP >= 4 && !IS_INT)
        return l.ring == 3 ? launch_tile<MMA, 64, 64, 1, 2, 3, 4>(g, ss, stream) : launch_tile<MMA, 64, 64, 1, 2, 5, 4>(g, ss, stream);
      break;
  }
  return hipErrorInvalidValue;
}

template <int BM, int BN, int STAGES, class WA, class WB>
hipError_t launch_pair(GemmParams a, GemmParams b, hipStream_t stream) {
  constexpr int LDS_BYTES = STAGES * (BM + BN) * BK;
  auto kern = &gemm_pair_kernel<BM, BN, STAGES, WA, WB>;
  static const hipError_t configured = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
  if (configured != hipSuccess) return configured;
  uint32_t blocks[2];
  GemmParams* const both[2] = {&a, &b};
  for (int i = 0; i < 2; ++i) {
    GemmParams& g = *both[i];
    g.tiles_p = (g.P + BM - 1) / BM;
    g.tiles_q = (g.Q + BN - 1) / BN;
    blocks[i] = (g.tiles_p * g.tiles_q * g.nsplit + 7) / 8 * 8;
  }
  kern<<<dim3(blocks[0] + blocks[1]), WA::THREADS, LDS_BYTES, stream>>>(a, b, blocks[0]);
  hipError_t e = hipGetLastError();
  for (int i = 0; i < 2 && e == hipSuccess; ++i)
    if (both[i]->nsplit > 1) e = launch_slice_sum(own_slice_sum<typename WA::MMA>(*both[i]), stream);
  return e;
}

// The forms of the two products: sets of accumulators (128 x 128 tiles) or groups of waves (64 x 64), in the MFMA tiles of launch_mma or
// choose_pair (of integers, any sums of which are the same, 16 x 16 on 64 x 64 as well: 3824 x 32 x 1872 12.5 -> 12.2 us).
template <class MMA>
hipError_t launch_pair_mma(const GemmParams& a, const GemmParams& b, PairForm form, const Paired& pa, const Paired& pb, hipStream_t stream) {
  constexpr bool IS_INT = std::is_same<MMA, I8Mma>::value;
  using Mma16 = typename Tiles16<MMA>::type;
  using One = Waves<Mma16, 2, 2, 1, 1>;
  using Two = Waves<MMA, 2, 2, 1, 2>;
  using G2 = Waves<typename std::conditional<IS_INT, Mma16, MMA>::type, 2, 2, 2, 1>;
  if (form == PAIR_128x128) {
    if constexpr (IS_INT) {
      return launch_pair<128, 128, 2, One, One>(a, b, stream);
    } else {
      if (pa.waves == 1 && pb.waves == 1) return launch_pair<128, 128, 2, One, One>(a, b, stream);
      if constexpr (MMA::WIDENS) {
        using Large = Waves<MMA, 2, 2, 1, 1>;
        if (pa.large_mfma) return launch_pair<128, 128, 2, Large, Two>(a, b, stream);
        if (pb.large_mfma) return launch_pair<128, 128, 2, Two, Large>(a, b, stream);
      }
      if (pa.waves == 1) return launch_pair<128, 128, 2, One, Two>(a, b, stream);
      return pb.waves == 1 ? launch_pair<128, 128, 2, Two, One>(a, b, stream) : launch_pair<128, 128, 2, Two, Two>(a, b, stream);
    }
  }
  if constexpr (BK / MMA::KSTEP >= 4 && !IS_INT) {
    using G4 = Waves<MMA, 1, 2, 4, 1>;
    if (pa.waves == 4) return pb.waves == 4 ? launch_pair<64, 64, 3, G4, G4>(a, b, stream) : launch_pair<64, 64, 3, G4, G2>(a, b, stream);
    if (pb.waves == 4) return launch_pair<64, 64, 3, G2, G4>(a, b, stream);
  }
  return launch_pair<64, 64, 3, G2, G2>(a, b, stream);
}

// Tiles and contraction slices of gemm_cut3_kernel, by the same model: 128 x 128 tiles of four waves,
// 64 x 64 of two for outputs too small to give every CU one; a stage is 32 elements.  per_cu: workgroups a CU holds
// (rings of 48 KiB, or registers with two sets of accumulators; rings of 36 KiB).
struct Cut3Kind {
  int waves, tn, per_cu;
  double rate_chip, fixed;
};
// (measured with MFMA tiles of 32 x 32; with those of 16 x 16 more than 256 large tiles take 0.93 to 1.0 of the time)
constexpr Cut3Kind CUT3_KINDS[2][2] = {{{4, 4, 3, 1.2e15, 8.0}, {2, 2, 4, 0.5e15, 8.0}},   // one set of accumulators
                                       {{4, 4, 2, 1.1e15, 8.0}, {2, 2, 4, 0.5e15, 8.0}}};  // two

struct Cut3Plan {
  int kind;
  bool two;
  uint32_t nsplit, k_per_split;  // bytes of Z
};
// Precision: no less than that of one bfloat16 product over the three parts side by side (a contraction of 3 R), for
// which a caller's workspace is sized.  Uncut, that product rounds its accumulators 3 R / 16 times, most of them at
// full size: one set of accumulators does no worse.  Cut, it sums the large parts in slices of their own, as long as
// its plan makes them: two sets of accumulators over slices no longer than those do no worse.  Cut in two, it has every large
// part and half of the next in one accumulator, and one set over two slices does no worse either; in more, one set does
// (six slices of 192 at 688 x 720 x 1152: 1.4e-7 against 8.3e-8, two sets over two slices 6.7e-8).  Error of that product and
// of this one: 736 x 688 x 1744, seven slices there, 1.1e-7 and 7.1e-8; 8192 x 3072 x 768, the input gradient in two, 3.8e-7
// and 3.7e-7; 16384 x 4096 x 1024, uncut, 8.3e-7 and 6.0e-7.
Cut3Plan make_cut3_plan(size_t P, size_t Q, size_t R, size_t partial_bytes) {
  const size_t ksteps = (2 * R + 63) / 64;
  const Plan whole = make_plan(P, Q, 6 * R);
  Cut3Plan best{};
  double best_time = -1.0;
  size_t best_n = 1;
  for (int two = whole.nsplit > 2; two < (whole.nsplit > 1 ? 2 : 1); ++two) {
    const size_t longest = whole.nsplit > 1 ? whole.k_per_split / (two ? 64 : 192) : ksteps;  // stages of a slice
    const size_t min_split = (ksteps + longest - 1) / longest;
    for (int kind = 0; kind < 2; ++kind) {
      const Cut3Kind& k = CUT3_KINDS[two][kind];
      const size_t bm = 32 * k.waves, bn = 32 * k.tn, t = ((P + bm - 1) / bm) * ((Q + bn - 1) / bn);
      size_t max_split = ksteps >= 32 ? ksteps / 16 : 1;
      if (max_split > 64) max_split = 64;
      if (max_split < min_split) max_split = min_split;
      for (size_t n = min_split; n <= max_split; ++n) {
        // (two sets over the fewest slices always fit: there are no more of them than that product has)
        if (n > 1 && n * P * Q * sizeof(uint32_t) > partial_bytes) break;
        const size_t per_cu = (t * n + NUM_CU - 1) / NUM_CU;  // items of the busiest CU
        const size_t stages = (ksteps + n - 1) / n;
        // a CU's rate with fewer workgroups than it holds
        const double share = per_cu >= (size_t)k.per_cu ? 1.0 : per_cu >= 2 ? 0.95 : 0.7;
        double time = (double)per_cu * ((double)stages + k.fixed) * 3.0 * 2.0 * bm * bn * 32 / (k.rate_chip / NUM_CU * share);
        if (n > 1) time += 2.0 * (double)n * (double)P * (double)Q * 4.0 / PARTIAL_BYTES_PER_SECOND + 3e-6;
        if (best_time < 0.0 || time < best_time) {
          best_time = time;
          best.kind = kind;
          best.two = two != 0;
          best_n = n;
        }
      }
    }
  }
  const size_t steps_per = (ksteps + best_n - 1) / best_n;
  best.k_per_split = (uint32_t)(steps_per * 64);
  best.nsplit = (uint32_t)((ksteps + steps_per - 1) / steps_per);
  return best;
}

template <class MMA, int NW, int TN, int STAGES, bool TWO>
hipError_t launch_cut3(GemmParams g, hipStream_t stream) {
  constexpr int LDS_BYTES = STAGES * (32 * NW * 128 + 32 * TN * 64);
  auto kern = &gemm_cut3_kernel<MMA, NW, TN, STAGES, TWO>;
  static const hipError_t configured = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
  if (configured != hipSuccess) return configured;
  g.tiles_p = (g.P + 32 * NW - 1) / (32 * NW);
  g.tiles_q = (g.Q + 32 * TN - 1) / (32 * TN);
  const uint32_t blocks = ((g.tiles_p * g.tiles_q * g.nsplit + 7) / 8) * 8;
  kern<<<blocks, NW * 64, LDS_BYTES, stream>>>(g);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || g.nsplit == 1) return e;
  SliceSum own{};
  own.partial = g.partial; own.out = g.out; own.nsplit = g.nsplit; own.total = (size_t)g.P * g.Q;
  own.s = GemmScale{g.alpha, g.sx, g.sz, g.sx_dev, g.sz_dev};
  return launch_slice_sum(own, stream);
}

}  // namespace

size_t gemm_workspace_bytes(size_t P, size_t Q, size_t R, int pipe) {
  return partial_bytes(plan_for(P, Q, R, pipe), P, Q);
}

bool gemm_takes_packed_x(size_t P, size_t Q, size_t R, int pipe) {
  return pipe == PIPE_I8 && make_plan(P, Q, R).tile == 0;
}

bool gemm_operands_addressable(size_t P, size_t Q, size_t R, int pipe) {
  const size_t rb = pipe == PIPE_BF16 || pipe == PIPE_F16W ? 2 * R : R;
  return (P + 256) * rb < (1ull << 31) && (Q + 256) * rb < (1ull << 31);
}

namespace {

// Runs f.template operator()<MMA>() with the matrix pipeline of `pipe` for operands of these kinds.
template <class F>
hipError_t with_pipeline(int pipe, int kindX, int kindZ, const F& f) {
  if (pipe == PIPE_I8) return f(I8Mma{});
  if (pipe == PIPE_BF16) return f(BF16Mma{});
  // the Z operand is the first MFMA operand, X the second
  const int fx = kindX == SRQ_E5M2, fz = kindZ == SRQ_E5M2;
  if (pipe == PIPE_F16C || pipe == PIPE_F16W) {
    if (!fz && !fx) return f(F8F16Mma<0, 0>{});
    if (!fz && fx) return f(F8F16Mma<0, 1>{});
    if (fz && !fx) return f(F8F16Mma<1, 0>{});
    return f(F8F16Mma<1, 1>{});
  }
  if (!fz && !fx) return f(F8Mma<0, 0>{});
  if (!fz && fx) return f(F8Mma<0, 1>{});
  if (fz && !fx) return f(F8Mma<1, 0>{});
  return f(F8Mma<1, 1>{});
}

GemmParams product_params(float* out, const uint8_t* X, const uint8_t* Z, size_t P, size_t Q, size_t row_bytes, size_t pitch,
                          const GemmScale& s, bool accumulate, void* workspace, bool x_packed) {
  GemmParams g;
  g.out = out;
  g.partial = static_cast<uint32_t*>(workspace);
  g.X = X; g.Z = Z;
  g.P = (uint32_t)P; g.Q = (uint32_t)Q; g.R = (uint32_t)row_bytes;
  g.pitch = (uint32_t)pitch;
  g.pitch_x = (uint32_t)(x_packed ? pitch / 2 : pitch);
  g.k_per_split = 0;
  g.nsplit = 1;
  g.tiles_p = g.tiles_q = 0;
  g.alpha = s.alpha; g.sx = s.sx; g.sz = s.sz; g.sx_dev = s.sx_dev; g.sz_dev = s.sz_dev;
  g.accumulate = accumulate ? 1 : 0;
  return g;
}

}  // namespace

hipError_t launch_gemm_codes(float* out, const uint8_t* X, int kindX, const uint8_t* Z, int kindZ,
                             size_t P, size_t Q, size_t R, size_t pitch, int pipe, const GemmScale& s,
                             bool accumulate, void* workspace, hipStream_t stream, ProductRole role,
                             const SliceSum* carry, SliceSum* defer, bool x_packed, const Plan* plan) {
  const SliceSumPlan ss{carry, defer};
  const size_t row_bytes = pipe == PIPE_BF16 ? 2 * R : R;
  const Plan pl = plan ? *plan : plan_for(P, Q, R, pipe);
  if (x_packed && !(pipe == PIPE_I8 && pl.tile == 0)) return hipErrorInvalidValue;  // see gemm_takes_packed_x
  GemmParams g = product_params(out, X, Z, P, Q, row_bytes, pitch, s, accumulate, workspace, x_packed);
  g.k_per_split = pl.k_per_split;
  g.nsplit = pl.nsplit;
  if (x_packed) return launch_persist<I8Mma, true>(g, ss, stream);
  // integer sums are the same in every form: there the launch counts, not the role
  const bool leaves = pipe == PIPE_I8 ? defer != nullptr : role == ROLE_WEIGHT_GRADIENT;
  const uint32_t rides = carry && carry->total > 0 ? carry->nsplit : 0;
  const Launch l = choose_launch(pl, P, Q, row_bytes, pipe, leaves, rides);
  const bool widens = pipe == PIPE_F16C || pipe == PIPE_F16W;
  const bool large = widens && (role == ROLE_ANY ? sums_in_large_mfma(l.form, P, Q, l.nsplit)
                                                 : large_mfma_of_gradient(pl, l, role == ROLE_WEIGHT_GRADIENT, P, Q, R, pipe));
  return with_pipeline(pipe, kindX, kindZ, [&](auto mma) { return launch_mma<decltype(mma)>(g, l, large, ss, stream); });
}

hipError_t launch_gemm_pair(const PairedProduct& w, const PairedProduct& d, int kindX, int pipe, hipStream_t stream, bool& done) {
  done = false;
  if (pipe == PIPE_BF16 || (pipe != PIPE_I8 && (w.kindZ == SRQ_E5M2) != (d.kindZ == SRQ_E5M2))) return hipSuccess;
  const Pair p = choose_pair(w.R, w.P, w.Q, pipe, w.plan, d.plan);  // M, N, K
  if (p.form == PAIR_NONE) return hipSuccess;
  GemmParams gw = product_params(w.out, w.X, w.Z, w.P, w.Q, w.R, w.R, w.s, w.accumulate, w.partial, false);
  GemmParams gd = product_params(d.out, d.X, d.Z, d.P, d.Q, d.R, d.R, d.s, d.accumulate, d.partial, false);
  gw.nsplit = p.w.nsplit;
  gw.k_per_split = p.w.k_per_split;
  gd.nsplit = p.d.nsplit;
  gd.k_per_split = p.d.k_per_split;
  done = true;
  return with_pipeline(pipe, kindX, w.kindZ, [&](auto mma) {
    using MMA = decltype(mma);
    if constexpr (std::is_same<MMA, BF16Mma>::value) return hipErrorInvalidValue;
    else return p.weight_first ? launch_pair_mma<MMA>(gw, gd, p.form, p.w, p.d, stream)
                               : launch_pair_mma<MMA>(gd, gw, p.form, p.d, p.w, stream);
  });
}

hipError_t launch_slice_sum(const SliceSum& r, hipStream_t stream) {
  if (r.total == 0) return hipSuccess;
  splitk_reduce_kernel<<<slice_sum_blocks(r, 256, 4), 256, 0, stream>>>(r);
  return hipGetLastError();
}

hipError_t launch_gemm_f32_bf16(float* out, const float* X, const uint16_t* Z, size_t P, size_t Q, size_t R,
                                const GemmScale& s, void* partial, size_t partial_bytes, hipStream_t stream) {
  const Cut3Plan pl = make_cut3_plan(P, Q, R, partial_bytes);
  GemmParams g{};
  g.out = out;
  g.partial = static_cast<uint32_t*>(partial);
  g.X = reinterpret_cast<const uint8_t*>(X);
  g.Z = reinterpret_cast<const uint8_t*>(Z);
  g.P = (uint32_t)P; g.Q = (uint32_t)Q; g.R = g.pitch = (uint32_t)(2 * R);
  g.pitch_x = (uint32_t)(4 * R);
  g.k_per_split = pl.k_per_split;
  g.nsplit = pl.nsplit;
  g.alpha = s.alpha; g.sx = s.sx; g.sz = s.sz; g.sx_dev = s.sx_dev; g.sz_dev = s.sz_dev;
  // MFMA tiles of 16 x 16 where CUs have more than one 128 x 128 tile and the clock counts.  With one, and the small ones, a tile waits
  // for LDS, the cut and its stores instead, and 32 x 32 are faster (int8 weights, us with 32 x 32 and 16 x 16; forward and input gradient
  // 8192 x 3072 x 768 220.7 and 208.9, 16384 x 4096 x 1024 696 and 646, 736 x 688 x 1744 46.5 and 48.2, 496 x 496 x 352 29.0 and
  // 30.2; forward calls, a tile a CU 192 x 5744 x 752 26.4 and 27.2, 544 x 976 x 4576 in slices 31.8 and 32.9, 16 shapes 0.97 to 1.03 of
  // the time of 16 x 16; 257 to 512 tiles 2112 x 3824 x 496 33.7 and 31.9, 944 x 2208 x 1664 37.9 and 36.3, 16 shapes 0.99 to 1.09;
  // error against 64 bits 3.68e-7 and 3.65e-7 at the first, 6.012e-7 and 5.989e-7 at the second)
  const size_t tiles = ((P + 127) / 128) * ((Q + 127) / 128) * pl.nsplit;
  const auto large_tiles = [&](auto two) {
    return tiles > NUM_CU ? launch_cut3<BF16Mma16, 4, 4, 2, two.value>(g, stream) : launch_cut3<BF16Mma, 4, 4, 2, two.value>(g, stream);
  };
  if (pl.two) return pl.kind == 0 ? large_tiles(std::true_type{}) : launch_cut3<BF16Mma, 2, 2, 3, true>(g, stream);
  return pl.kind == 0 ? large_tiles(std::false_type{}) : launch_cut3<BF16Mma, 2, 2, 3, false>(g, stream);
}

}  // namespace srq
