// Device-side building blocks of the SR quantizer: the counter-based random bits and the
// per-element threshold quantizer (Def. 1 / Eq. 1, Def. 2, Def. 3) on the four target grids.
// gfx950 only.
//
// Arithmetic.  The grid coordinate t = fl32(x * inv) is one binary32 multiply.  From there
// Eq. 1 is evaluated EXACTLY, in 16.16 fixed point: with y = t / D (a power-of-two scaling),
//     threshold eps = (r + 1/2) / 2^16,   y = f + frac,  f = floor(y)
//     round up  <=>  frac >= eps  <=>  frac * 2^16 >= r + 1/2  <=>  r < floor(frac * 2^16 + 1/2)
// and since floor(y * 2^16 + 1/2) = f * 2^16 + floor(frac * 2^16 + 1/2) =: U,
//     q = floor((U + 65535 - r) / 2^16)        (the carry out of the low 16 bits is "up").
// U is one v_cvt_rpi_i32_f32 (floor(x + 1/2), exact, saturating) of y * 2^16, which is itself
// exact.  Round-to-nearest (eps = 1/2) is  q = floor((floor(y * 2^16) + 32768) / 2^16).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/srq.h"

namespace srq {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// ---- Philox4x32-10 (Salmon et al., SC'11), counter (block_lo, block_hi, 0, 0) ----------
// The key schedule is wave-uniform, so it lives in scalar registers; only the two 32x32->64
// multiplies and the xors per round are vector work.
__device__ __forceinline__ void philox_block(uint64_t block, uint32_t k0, uint32_t k1,
                                             uint32_t (&w)[4]) {
  uint32_t c0 = (uint32_t)block, c1 = (uint32_t)(block >> 32), c2 = 0u, c3 = 0u;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);  // three-way xor
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}

// floor(x + 1/2) and floor(x) as int32: exact, saturating (NaN gives INT_MAX)
__device__ __forceinline__ int cvt_rpi(float x) {
  int r;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}
__device__ __forceinline__ int cvt_flr(float x) {
  int r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// u within [-q, q], q the same for the whole wave: one instruction, which the compiler forms only of constants
__device__ __forceinline__ int clamp_to(int u, int q) {
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(u), "s"(-q), "v"(q));
  return r;
}

// What is added to U before the shift: 65535 - r16 for stochastic rounding (r16 the element's
// 16 random bits), 32768 for round-to-nearest.
constexpr uint32_t RTN_ADDEND = 32768u;

// The four addends of two output words of a Philox block (elements 4h .. 4h+3 of a group,
// low half of the first word first).
__device__ __forceinline__ void sr_addends(uint32_t w0, uint32_t w1, uint32_t (&add)[4]) {
  const uint32_t n0 = ~w0, n1 = ~w1;  // 65535 - r in each half
  add[0] = n0 & 0xFFFFu; add[1] = n0 >> 16; add[2] = n1 & 0xFFFFu; add[3] = n1 >> 16;
}

template <int KIND> struct Grid;
template <> struct Grid<SRQ_INT8> { static constexpr bool is_float = false; static constexpr int qmax = 127; };
template <> struct Grid<SRQ_INT4> { static constexpr bool is_float = false; static constexpr int qmax = 7; };
template <> struct Grid<SRQ_E4M3> {
  static constexpr bool is_float = true; static constexpr float qmax = 448.0f;
  static constexpr int mbits = 3, emin = -6;
};
template <> struct Grid<SRQ_E5M2> {
  static constexpr bool is_float = true; static constexpr float qmax = 57344.0f;
  static constexpr int mbits = 2, emin = -14;
};
// E4M2 / E4M1 / E4M0: sub-grids of E4M3 whose fraction width and Qmax are run-time values (one
// instantiation serves the three); codes are written as E4M3 codes.
constexpr int SRQ_E4MX = 100;
template <> struct Grid<SRQ_E4MX> {
  static constexpr bool is_float = true; static constexpr float qmax = 0.0f;  // unused: InvScale::sub_qmax
  static constexpr int mbits = 0, emin = -6;                                  // mbits unused: InvScale::sub_m
};
__host__ __device__ constexpr bool kind_is_e4mx(int kind) { return kind >= SRQ_E4M2 && kind <= SRQ_E4M0; }
// INT8 / INT4 with the clamp as a run-time value (one instantiation serves both): used where a
// second, integer quantizer rides along with another format's pass over the same tensor.
constexpr int SRQ_INTX = 101;
template <> struct Grid<SRQ_INTX> { static constexpr bool is_float = false; static constexpr int qmax = 0; };  // InvScale::sub_qi
// E4M3 whose codes come out of the conversions (below); the same codes.
constexpr int SRQ_E4M3_CONV = 102;
template <> struct Grid<SRQ_E4M3_CONV> : Grid<SRQ_E4M3> {};

// Per-tensor constants of the multiply that produces the grid coordinate.
struct InvScale {
  float inv;    // fl32(1 / scale)
  float inv16;  // inv * 2^16 (exact): fl32(x * inv16) = fl32(x * inv) * 2^16
  int sub_m;        // SRQ_E4MX only: fraction bits (2, 1, 0)
  float sub_qmax;   // SRQ_E4MX only: 448, 384, 256
  int sub_qi;       // SRQ_INTX only: Qmax * 2^16 (127 or 7)
};

// One element through Eq. 1 on grid KIND.  Returns the code in the low 8 bits (integers:
// two's complement byte; INT4 values are in [-7,7], sign-extended to the byte).  With
// AS_BF16 it returns instead the bfloat16 bit pattern of the grid point q * D itself -- every
// grid value is a normal bfloat16 number -- which is what the exact (bf16 matrix pipeline)
// product consumes.
// FIX_NAN = false leaves the NaN rule to the caller (quantize_quad applies it per quad).
// Integer codes come back sign-extended to 32 bits: take the low byte (or nibble).
template <int KIND, int ROUND, bool AS_BF16 = false, bool FIX_NAN = true>
__device__ __forceinline__ uint32_t quantize_elem(float x, const InvScale& s, uint32_t addend) {
  using G = Grid<KIND>;
  uint32_t code;
  if constexpr (!G::is_float) {
    const int QI = KIND == SRQ_INTX ? s.sub_qi : (G::qmax << 16);
    const float y16 = __fmul_rn(x, s.inv16);                            // t * 2^16, D = 1
    int u = ROUND == SRQ_SR ? cvt_rpi(y16) : cvt_flr(y16);              // saturating
    u = clamp_to(u, QI);                                                // clamp t to +-Qmax
    const int q = (u + (int)addend) >> 16;
    code = AS_BF16 ? __float_as_uint((float)q) >> 16 : (uint32_t)q;     // (at most 7 significant bits)
    if (FIX_NAN && x != x) code = 0u;
  } else {
    const int m = KIND == SRQ_E4MX ? s.sub_m : G::mbits;
    const float qm = KIND == SRQ_E4MX ? s.sub_qmax : G::qmax;
    float t = __fmul_rn(x, s.inv);                                      // grid coordinate
    t = __builtin_amdgcn_fmed3f(t, -qm, qm);                            // saturate (NaN fixed up below)
    // spacing of the grid at t: D = 2^(e - m), e = max(floor(log2|t|), emin)
    const uint32_t a = __float_as_uint(t) & 0x7FFFFFFFu;
    const int eb = max((int)(a >> 23), G::emin + 127);                  // biased e (0 and subnormals clamp)
    const float up16 = __uint_as_float((uint32_t)(270 + m - eb) << 23);  // 2^(16 + m - e)
    const float y16 = __fmul_rn(t, up16);                               // (t / D) * 2^16, exact
    const int u = ROUND == SRQ_SR ? cvt_rpi(y16) : cvt_flr(y16);
    const int q = (u + (int)addend) >> 16;                              // |q| in [0, 2^(m+1)]
    if constexpr (AS_BF16) {
      const float d = __uint_as_float((uint32_t)(eb - m) << 23);        // D = 2^(e - m)
      code = __float_as_uint(__fmul_rn((float)q, d)) >> 16;             // exact, <= 4 significant bits
      if (FIX_NAN && x != x) code = 0x7FC0u;
    } else {
      // sign | ((e - emin) << m) + |q| : covers subnormals (field 0), normals (the hidden one
      // of |q| bumps the field) and the carry into the next binade
      uint32_t mag = ((uint32_t)(eb - (G::emin + 127)) << m) + (uint32_t)abs(q);
      if constexpr (KIND == SRQ_E4MX) mag <<= 3 - m;                    // the E4M3 code of the same value
      code = mag | (q < 0 ? 0x80u : 0u);
      if (FIX_NAN && x != x) code = 0x7Fu;
    }
  }
  return code;
}

// Four elements.  The NaN rule is tested for the quad as a whole (two unordered compares)
// and applied element-wise only on the rare lanes where it fires.
template <int KIND, int ROUND, bool AS_BF16>
__device__ __forceinline__ void quantize_quad(uint32_t (&c)[4], float x0, float x1, float x2, float x3,
                                              const InvScale& s, const uint32_t (&add)[4]) {
  c[0] = quantize_elem<KIND, ROUND, AS_BF16, false>(x0, s, add[0]);
  c[1] = quantize_elem<KIND, ROUND, AS_BF16, false>(x1, s, add[1]);
  c[2] = quantize_elem<KIND, ROUND, AS_BF16, false>(x2, s, add[2]);
  c[3] = quantize_elem<KIND, ROUND, AS_BF16, false>(x3, s, add[3]);
  if (__builtin_isunordered(x0, x1) || __builtin_isunordered(x2, x3)) {
    constexpr uint32_t NAN_CODE = !Grid<KIND>::is_float ? 0u : AS_BF16 ? 0x7FC0u : 0x7Fu;
    if (x0 != x0) c[0] = NAN_CODE;
    if (x1 != x1) c[1] = NAN_CODE;
    if (x2 != x2) c[2] = NAN_CODE;
    if (x3 != x3) c[3] = NAN_CODE;
  }
}

// low bytes of four codes -> one word (c0 in bits 7:0); upper bits of the inputs are ignored
__device__ __forceinline__ uint32_t pack4_bytes(const uint32_t (&c)[4]) {
  const uint32_t lo = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u);
  const uint32_t hi = __builtin_amdgcn_perm(c[3], c[2], 0x0c0c0400u);
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// ---- four elements to a word of four byte codes --------------------------------------------------
// r0 holds the random bits of elements 0 and 1 (low half first), r1 those of 2 and 3, as they come out of Philox; for
// round-to-nearest (sr = false) both are RTN_WORD, whose halves give the addend 32768.  (sr is uniform; where it is a constant the
// other form folds away.)
//
// What bounds the rounding is the vector ALU (a wave instruction is 2 to 2.7 cycles for plain binary32 and logic operations,
// 4.4 for most others, 5.2 for a 32 x 32 -> 64 multiply-add, 8.4 for the conversions below), so it is counted in cycles of a wave
// for 8 elements a lane, Philox (183) included: int8 513 -> 457 against code by code, E5M2 837 and E4M3 814 -> some 630, and 170 more
// where a lane holds one of the rare cases, which in many tensors no wave is without.
//
// Integers: the code is byte 2 of U + addend, so the byte permutes that pack the word also take the place of the shifts.
//
// E4M3 and E5M2: v_cvt_sr_fp8_f32 / v_cvt_sr_bf8_f32 add the top 20 / 21 bits of a seed to the fraction of |t| below the
// kept bits and cut.  That is Eq. 1 exactly where t is a normal number of the grid.  With F the 24-bit significand of |t| and
// 16 + b fraction bits below the kept ones (b = 5 for E5M2, 4 for E4M3), U of the rule above is (F + 2^(b-1)) >> b for t > 0 and
// -((F + 2^(b-1) - 1) >> b) for t < 0, hence
//     t > 0:  |q| = (F + ((65535 - r) << b) + 2^(b-1)) >> (16 + b)
//     t < 0:  |q| = (F + (r << b) + 2^(b-1) - 1) >> (16 + b)
// and the two seeds are each other's complement: (~r) << 16 | 0x8000, inverted where t is negative.  Round-to-nearest lacks the
// half of U: the seed 0x80000000 by the same rule.  (The bits of an inverted seed below the ones that are added do not matter.)
// Below the smallest normal number the spacing is one and the same, as for integers: those codes are made by the integers'
// few instructions (uniform_word), without a loop, and take their place in the word where the converted code has an exponent
// of 0 or 1, which covers the numbers that round up to a normal one.  How many elements that concerns is the tensor's: of a normal
// one of 2^28 elements E4M3 finds some in 6 % of the waves of 512, with 1 % of outliers fifty times as large in 97 %, of
// gradients over 40 binades or activations cut off at zero in all.  us of 2^26 elements code by code and by conversion, normal / outliers /
// 40 binades: E4M3 binary32 58 -> 56 / 58 -> 56 / 56 -> 57 (HBM), bfloat16 45 -> 37 / 45 -> 42 / 45 -> 42, turned 47 -> 40 / 47 -> 43 /
// 47 -> 44; E5M2 bfloat16 45 -> 36 / 45 -> 36 / 45 -> 42.
constexpr uint32_t RTN_WORD = 0x7FFF7FFFu;

// Formats whose codes come out of the conversions a word at a time.  E4M3's smallest normal number is 2^-15 of the largest, so a few
// waves of most tensors hold rare cases, and a launch of some microseconds waits for the first of them, whose code is not in the
// instruction cache: the quantizer of one tensor converts it from 2^22 elements on (E4M3_CONV_ELEMENTS), those of several operands at every
// size, where their small kernels save more than that costs (512 x 512 twice with 1 % of outliers 4.1 -> 3.7 us).  For E5M2 it is
// 2^-30 (1024 x 1024 binary32, turned: normal 4.15 -> 3.8 us, 40 binades 4.15 -> 4.25; bfloat16 4.1 -> 3.6 and 4.1).
template <int KIND>
constexpr bool BY_CONVERSION = KIND == SRQ_E4M3_CONV || KIND == SRQ_E5M2;

// Four elements by conversion; t: their clamped grid coordinates, least: the least magnitude of them, or NaN where one is.
template <int KIND>
__device__ __forceinline__ uint32_t convert_word(const float (&x)[4], float (&t)[4], float& least, const InvScale& s, uint32_t r0,
                                                 uint32_t r1, bool sr) {
  constexpr float QM = Grid<KIND>::qmax;
  const uint32_t n0 = ~r0, n1 = ~r1, add_half = sr ? 0x8000u : 0u;
  const uint32_t seed[4] = {(n0 << 16) | add_half, (n0 & 0xFFFF0000u) | add_half, (n1 << 16) | add_half,
                            (n1 & 0xFFFF0000u) | add_half};
  int sd[4], w = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float y = __builtin_fmaf(x[e], s.inv, 0.0f);
    least = e == 0 ? fabsf(y) : __builtin_elementwise_minimum(least, fabsf(y));
    t[e] = __builtin_amdgcn_fmed3f(y, -QM, QM);
    sd[e] = (int)seed[e] ^ ((int)__float_as_uint(t[e]) >> 31);
  }
  if constexpr (KIND == SRQ_E5M2) {
    w = __builtin_amdgcn_cvt_sr_bf8_f32(t[0], sd[0], w, 0);
    w = __builtin_amdgcn_cvt_sr_bf8_f32(t[1], sd[1], w, 1);
    w = __builtin_amdgcn_cvt_sr_bf8_f32(t[2], sd[2], w, 2);
    w = __builtin_amdgcn_cvt_sr_bf8_f32(t[3], sd[3], w, 3);
  } else {
    w = __builtin_amdgcn_cvt_sr_fp8_f32(t[0], sd[0], w, 0);
    w = __builtin_amdgcn_cvt_sr_fp8_f32(t[1], sd[1], w, 1);
    w = __builtin_amdgcn_cvt_sr_fp8_f32(t[2], sd[2], w, 2);
    w = __builtin_amdgcn_cvt_sr_fp8_f32(t[3], sd[3], w, 3);
  }
  return (uint32_t)w;
}

// 0xFF in the bytes whose top bit is set, 0 in the others.
__device__ __forceinline__ uint32_t bytes_of_sign(uint32_t w) { return __builtin_amdgcn_perm(w, w << 8, 0x0b090a08u); }

// Byte 2 of U + addend of four elements: the integers of the rule.
__device__ __forceinline__ uint32_t signed_bytes(const uint32_t (&c)[4]) {
  const uint32_t lo = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0602u), hi = __builtin_amdgcn_perm(c[3], c[2], 0x0c0c0602u);
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// Four elements of the other formats.
template <int KIND>
__device__ __forceinline__ uint32_t quantize_word(float x0, float x1, float x2, float x3, const InvScale& s, uint32_t r0,
                                                  uint32_t r1, bool sr) {
  static_assert(!BY_CONVERSION<KIND>, "quantize_octet");
  const float x[4] = {x0, x1, x2, x3};
  uint32_t add[4], c[4];
  sr_addends(r0, r1, add);
  if constexpr (Grid<KIND>::is_float) {
    if (sr) quantize_quad<KIND, SRQ_SR, false>(c, x0, x1, x2, x3, s, add);
    else quantize_quad<KIND, SRQ_RTN, false>(c, x0, x1, x2, x3, s, add);
    return pack4_bytes(c);
  } else {
    const int QI = KIND == SRQ_INTX ? s.sub_qi : (Grid<KIND>::qmax << 16);
    int u[4];
    if (sr) {
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = cvt_rpi(__fmul_rn(x[e], s.inv16));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = cvt_flr(__fmul_rn(x[e], s.inv16));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = (uint32_t)clamp_to(u[e], QI) + add[e];
    if (__builtin_isunordered(x0, x1) || __builtin_isunordered(x2, x3)) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (x[e] != x[e]) c[e] = 0u;
    }
    return signed_bytes(c);
  }
}

// Codes of four elements of E4M3 or E5M2 by the spacing of the subnormals, which the first normal binade shares: of those
// below twice the smallest normal number the codes of the rule (the magnitude of q is the code), of others any.
template <int KIND>
__device__ __forceinline__ uint32_t uniform_word(const float (&t)[4], uint32_t r0, uint32_t r1, bool sr) {
  constexpr float UP = KIND == SRQ_E5M2 ? 0x1p+32f : 0x1p+25f;  // 2^16 / D
  uint32_t add[4], c[4];
  sr_addends(r0, r1, add);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float y16 = __fmul_rn(t[e], UP);
    c[e] = (uint32_t)(sr ? cvt_rpi(y16) : cvt_flr(y16)) + add[e];
  }
  const uint32_t q = signed_bytes(c), negative = bytes_of_sign(q);
  return ((q ^ negative) + (negative & 0x01010101u)) | (negative & 0x80808080u);  // (no carry leaves a byte: none of these is zero)
}

// U + addend of eight elements for the integers, whose code is byte 2 of it; 0 of a NaN.  (One branch for all eight: 2^24 bfloat16 -> int4
// in their own layout 11.4 us with one for four, 10.5 so.)
template <int KIND>
__device__ __forceinline__ void integer_sums(uint32_t (&c)[2][4], const float (&x)[4], const float (&y)[4], const InvScale& s,
                                             const uint32_t (&r)[4], bool sr) {
  const int QI = KIND == SRQ_INTX ? s.sub_qi : (Grid<KIND>::qmax << 16);
  uint32_t add[2][4];
  sr_addends(r[0], r[1], add[0]);
  sr_addends(r[2], r[3], add[1]);
  int u[8];
  if (sr) {
#pragma unroll
    for (int e = 0; e < 8; ++e) u[e] = cvt_rpi(__fmul_rn(e < 4 ? x[e % 4] : y[e % 4], s.inv16));
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) u[e] = cvt_flr(__fmul_rn(e < 4 ? x[e % 4] : y[e % 4], s.inv16));
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) c[e / 4][e % 4] = (uint32_t)clamp_to(u[e], QI) + add[e / 4][e % 4];
  if (__builtin_isunordered(x[0], x[1]) || __builtin_isunordered(x[2], x[3]) || __builtin_isunordered(y[0], y[1]) ||
      __builtin_isunordered(y[2], y[3])) {
    asm volatile("");  // (a branch, no selects)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (x[e] != x[e]) c[0][e] = 0u;
      if (y[e] != y[e]) c[1][e] = 0u;
    }
  }
}

// Eight elements, x and y four each, with their four random words: two words of codes.  (One test for the rare cases of all eight,
// subnormals, zeros and NaN: branches keep the compiler from moving work across them.)
template <int KIND>
__device__ __forceinline__ u32x2 quantize_octet(const float (&x)[4], const float (&y)[4], const InvScale& s, const uint32_t (&r)[4],
                                                bool sr) {
  if constexpr (!Grid<KIND>::is_float) {
    uint32_t c[2][4];
    integer_sums<KIND>(c, x, y, s, r, sr);
    return u32x2{signed_bytes(c[0]), signed_bytes(c[1])};
  } else if constexpr (!BY_CONVERSION<KIND>) {
    return u32x2{quantize_word<KIND>(x[0], x[1], x[2], x[3], s, r[0], r[1], sr),
                 quantize_word<KIND>(y[0], y[1], y[2], y[3], s, r[2], r[3], sr)};
  } else {
    constexpr float LEAST = KIND == SRQ_E5M2 ? 0x1p-14f : 0x1p-6f;  // smallest normal number
    float t[2][4], least[2];
    uint32_t w[2] = {convert_word<KIND>(x, t[0], least[0], s, r[0], r[1], sr), convert_word<KIND>(y, t[1], least[1], s, r[2], r[3], sr)};
    const float lowest = __builtin_elementwise_minimum(least[0], least[1]);
    if (!(lowest >= LEAST)) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t small = uniform_word<KIND>(t[h], r[2 * h], r[2 * h + 1], sr);
        constexpr uint32_t EXPONENT = KIND == SRQ_E5M2 ? 0x78787878u : 0x70707070u;  // without its last bit
        const uint32_t normal = bytes_of_sign((w[h] & EXPONENT) + EXPONENT);
        w[h] = (w[h] & normal) | (small & ~normal);
      }
      if (lowest != lowest) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = e < 4 ? x[e % 4] : y[e % 4];
          if (v != v) w[e / 4] = (w[e / 4] & ~(0xFFu << (8 * (e % 4)))) | 0x7Fu << (8 * (e % 4));
        }
      }
    }
    return u32x2{w[0], w[1]};
  }
}

// Two words of byte codes -> one of nibbles (elements 0-7, element 0 in bits 3:0).
__device__ __forceinline__ uint32_t pack8_nibbles(uint32_t lo, uint32_t hi) {
  lo = (lo & 0x0F0F0F0Fu) | ((lo >> 4) & 0x00F000F0u);  // bytes 0 and 2 hold the pairs
  hi = (hi & 0x0F0F0F0Fu) | ((hi >> 4) & 0x00F000F0u);
  return __builtin_amdgcn_perm(hi, lo, 0x06040200u);
}

// Four words of four bytes, rows -> columns (eight byte permutes).
__device__ __forceinline__ void turn4x4(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3, uint32_t (&c)[4]) {
  const uint32_t a0 = __builtin_amdgcn_perm(r1, r0, 0x05010400u), a1 = __builtin_amdgcn_perm(r1, r0, 0x07030602u);
  const uint32_t b0 = __builtin_amdgcn_perm(r3, r2, 0x05010400u), b1 = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
  c[0] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
  c[1] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
  c[2] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
  c[3] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// 1 / scale, correctly rounded, from a host value or a device-resident one.
// `kind` is the srq_kind of the tensor (it fills the run-time grid parameters of SRQ_E4MX).
__device__ __forceinline__ InvScale inv_scale(float scale, const float* scale_dev, int kind) {
  const float sc = scale_dev ? *scale_dev : scale;
  InvScale s;
  s.inv = __fdiv_rn(1.0f, sc);
  s.inv16 = __fmul_rn(s.inv, 65536.0f);
  s.sub_m = SRQ_E4M0 - kind;  // E4M2 -> 2, E4M1 -> 1, E4M0 -> 0
  s.sub_qmax = kind == SRQ_E4M2 ? 448.0f : kind == SRQ_E4M1 ? 384.0f : 256.0f;
  s.sub_qi = (kind == SRQ_INT4 ? 7 : 127) << 16;
  return s;
}

// First Philox block of a tensor: a host value, plus the value of a device-resident counter if
// one is given (so that a captured launch can be replayed with fresh thresholds).
__device__ __forceinline__ uint64_t first_block(uint64_t counter_offset, const uint64_t* counter_dev) {
  return counter_offset + (counter_dev ? *counter_dev : 0ull);
}

// ---- groups of 8 consecutive elements (one Philox block) -----------------------------------
// A pointer that is known to point to global memory.  One that was read out of a structure in memory is generic to the compiler,
// whose flat instructions take no scalar base and are waited for together with those of the LDS.
template <class T>
using global_ptr = __attribute__((address_space(1))) T*;
template <class T>
__device__ __forceinline__ global_ptr<T> as_global(T* p) { return (global_ptr<T>)p; }

// A 16-byte load of a source tensor: streaming, or cached for one that is small enough to be met again in
// the last-level cache (the load policy in srq_internal.hpp).
template <bool CACHED, class T>
__device__ __forceinline__ T load_source(global_ptr<const T> p) {
  if constexpr (CACHED) return *p;
  else return __builtin_nontemporal_load(p);
}
template <bool CACHED, class T>
__device__ __forceinline__ T load_source(const T* p) { return load_source<CACHED, T>(as_global(p)); }

// Load the 8 elements of group g (element index 8g..8g+7) as binary32; lanes beyond n read 0.
template <int SRC, bool CACHED = false>
__device__ __forceinline__ void load_group(float (&v)[8], const void* x, size_t g, size_t n) {
  const size_t base = g * 8;
  if (base + 8 <= n) {
    if constexpr (SRC == SRQ_F32) {
      const f32x4* p = reinterpret_cast<const f32x4*>(static_cast<const float*>(x) + base);
      const f32x4 a = load_source<CACHED>(p);
      const f32x4 b = load_source<CACHED>(p + 1);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
      v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
      const u32x4 a = load_source<CACHED>(reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(x) + base));
      v[0] = bf16_to_f32(a.x & 0xFFFFu); v[1] = bf16_to_f32(a.x >> 16);
      v[2] = bf16_to_f32(a.y & 0xFFFFu); v[3] = bf16_to_f32(a.y >> 16);
      v[4] = bf16_to_f32(a.z & 0xFFFFu); v[5] = bf16_to_f32(a.z >> 16);
      v[6] = bf16_to_f32(a.w & 0xFFFFu); v[7] = bf16_to_f32(a.w >> 16);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float e = 0.0f;
      if (base + j < n) {
        if constexpr (SRC == SRQ_F32) e = static_cast<const float*>(x)[base + j];
        else e = bf16_to_f32(static_cast<const uint16_t*>(x)[base + j]);
      }
      v[j] = e;
    }
  }
}

// Quantize one group; c[j] = code of element j (integer codes sign-extended: use the low byte).
template <int KIND, int ROUND, bool AS_BF16>
__device__ __forceinline__ void quantize_group(uint32_t (&c)[8], const float (&v)[8], const InvScale& s,
                                               uint64_t block, uint32_t k0, uint32_t k1) {
  uint32_t add[8];
  if constexpr (ROUND == SRQ_SR) {
    uint32_t w[4];
    philox_block(block, k0, k1, w);
    uint32_t lo[4], hi[4];
    sr_addends(w[0], w[1], lo);
    sr_addends(w[2], w[3], hi);
#pragma unroll
    for (int j = 0; j < 4; ++j) { add[j] = lo[j]; add[4 + j] = hi[j]; }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) add[j] = RTN_ADDEND;  // Def. 2
  }
  uint32_t lo4[4], hi4[4];
  const uint32_t addlo[4] = {add[0], add[1], add[2], add[3]}, addhi[4] = {add[4], add[5], add[6], add[7]};
  quantize_quad<KIND, ROUND, AS_BF16>(lo4, v[0], v[1], v[2], v[3], s, addlo);
  quantize_quad<KIND, ROUND, AS_BF16>(hi4, v[4], v[5], v[6], v[7], s, addhi);
#pragma unroll
  for (int j = 0; j < 4; ++j) { c[j] = lo4[j]; c[4 + j] = hi4[j]; }
}

// The random words of a Philox block, or what stands for them in round-to-nearest.
__device__ __forceinline__ void round_words(bool sr, uint64_t block, uint32_t k0, uint32_t k1, uint32_t (&w)[4]) {
  if (sr) philox_block(block, k0, k1, w);
  else w[0] = w[1] = w[2] = w[3] = RTN_WORD;
}

// One group to two words of byte codes.
template <int KIND>
__device__ __forceinline__ u32x2 quantize_group_words(const float (&v)[8], const InvScale& s, uint64_t block, uint32_t k0,
                                                      uint32_t k1, bool sr) {
  uint32_t w[4];
  round_words(sr, block, k0, k1, w);
  return quantize_octet<KIND>({v[0], v[1], v[2], v[3]}, {v[4], v[5], v[6], v[7]}, s, w, sr);
}

// v_permlane32_swap: the upper 32 lanes of a and the lower 32 of b change places.
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// For lanes L and L + 32 that hold the two halves of each of two groups: the lower lane passes the block of the first
// group and the upper lane that of the second; w[0], w[1] become this lane's words of the first group, w[2], w[3] of the second.
__device__ __forceinline__ void round_words_of_pair(uint64_t block, uint32_t k0, uint32_t k1, uint32_t (&w)[4]) {
  philox_block(block, k0, k1, w);
  swap_halves(w[0], w[2]);
  swap_halves(w[1], w[3]);
}
// The same for neighbouring lanes: the even one passes the block of the first group, the odd one that of the second.
__device__ __forceinline__ void round_words_of_neighbours(uint64_t block, uint32_t k0, uint32_t k1, uint32_t (&w)[4], bool odd) {
  philox_block(block, k0, k1, w);
  const uint32_t n0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[0], 0xB1, 0xF, 0xF, true);  // lane ^ 1
  const uint32_t n1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[1], 0xB1, 0xF, 0xF, true);
  const uint32_t n2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[2], 0xB1, 0xF, 0xF, true);
  const uint32_t n3 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[3], 0xB1, 0xF, 0xF, true);
  w[0] = odd ? n2 : w[0];
  w[1] = odd ? n3 : w[1];
  w[2] = odd ? w[2] : n0;
  w[3] = odd ? w[3] : n1;
}

// ---- one wave, 512 consecutive binary32 elements ---------------------------------------------
// 64 groups of 8.  Lane L < 32 loads the first quad of groups L and 32 + L, lane 32 + L the second quads: two 16-byte
// loads, each a contiguous kilobyte across the wave.  The lower lane draws the Philox block of the first group, the upper one that
// of the second, and one swap of wave halves per word hands out the words (a swap is 8 cycles where trading between
// neighbouring lanes took two moves and two selects, 18).  The codes go the same way: after another swap
// a lane holds a whole group and writes 8 bytes.
constexpr int CHUNK = 512;

// Stores that write through the L2 (system-scope cache policy) without the streaming hint: the
// line does not stay dirty in the L2 (nothing left to flush when the kernel ends) but is still
// allocated in the last-level cache for the kernel that reads it next.
__device__ __forceinline__ void store_through16(void* p, const u32x4& v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through8(global_ptr<uint8_t> p, const u32x2& v) {
  asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through4(global_ptr<uint8_t> p, uint32_t v) {
  asm volatile("global_store_dword %0, %1, off sc0 sc1" : : "v"(p), "v"(v) : "memory");
}

// store modes: 0 one byte per element, 1 nibbles, 2 bfloat16 (values as in StoreMode)
template <int KIND, int STORE, bool CACHED = false>
__device__ __forceinline__ void quantize_chunk_f32(uint8_t* __restrict__ out, const float* __restrict__ x,
                                                   size_t chunk, uint32_t lane, const InvScale& s, uint32_t k0,
                                                   uint32_t k1, uint64_t counter_offset, bool sr) {
  if constexpr (STORE == 1) {
    // Two bytes a quad: quads of neighbouring lanes, which trade random words, in contiguous memory, instead of the order
    // below, in which a load is a kilobyte as well but four neighbouring lanes touch 128 bytes (2^24 elements SR 13.1 -> 12.0 us;
    // one-byte codes take 14.7 either way).
    const size_t e = chunk * CHUNK + 4 * lane;
    const bool odd = lane & 1u;
    const f32x4 a = load_source<CACHED>(reinterpret_cast<const f32x4*>(x + e));
    const f32x4 b = load_source<CACHED>(reinterpret_cast<const f32x4*>(x + e + 256));
    uint32_t w[4];
    if (sr) round_words_of_neighbours(counter_offset + chunk * (CHUNK / 8) + (odd ? 32u : 0u) + (lane >> 1), k0, k1, w, odd);
    else w[0] = w[1] = w[2] = w[3] = RTN_WORD;
    const u32x2 c = quantize_octet<KIND>({a.x, a.y, a.z, a.w}, {b.x, b.y, b.z, b.w}, s, w, sr);
    const uint32_t n = pack8_nibbles(c.x, c.y);
    uint16_t* const o = reinterpret_cast<uint16_t*>(out + e / 2);
    o[0] = (uint16_t)n;
    o[64] = (uint16_t)(n >> 16);
    return;
  }
  const uint32_t half = lane >> 5, l = lane & 31u;
  const size_t e0 = chunk * CHUNK + 8 * l + 4 * half;  // first element of this lane's first quad
  const f32x4 a = load_source<CACHED>(reinterpret_cast<const f32x4*>(x + e0));
  const f32x4 b = load_source<CACHED>(reinterpret_cast<const f32x4*>(x + e0 + 256));
  uint32_t w[4];
  if (sr) round_words_of_pair(counter_offset + chunk * (CHUNK / 8) + lane, k0, k1, w);
  else w[0] = w[1] = w[2] = w[3] = RTN_WORD;
  const size_t g0 = chunk * CHUNK + 8 * lane;  // the group this lane writes
  if constexpr (STORE == 2) {
    uint32_t addA[4], addB[4], ca[4], cb[4];
    sr_addends(w[0], w[1], addA);
    sr_addends(w[2], w[3], addB);
    if (sr) {
      quantize_quad<KIND, SRQ_SR, true>(ca, a.x, a.y, a.z, a.w, s, addA);
      quantize_quad<KIND, SRQ_SR, true>(cb, b.x, b.y, b.z, b.w, s, addB);
    } else {
      quantize_quad<KIND, SRQ_RTN, true>(ca, a.x, a.y, a.z, a.w, s, addA);
      quantize_quad<KIND, SRQ_RTN, true>(cb, b.x, b.y, b.z, b.w, s, addB);
    }
    uint32_t a0 = ca[0] | (ca[1] << 16), a1 = ca[2] | (ca[3] << 16), b0 = cb[0] | (cb[1] << 16), b1 = cb[2] | (cb[3] << 16);
    swap_halves(a0, b0);
    swap_halves(a1, b1);
    __builtin_nontemporal_store(u32x4{a0, a1, b0, b1}, as_global(reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out) + g0)));
  } else {
    const u32x2 c = quantize_octet<KIND>({a.x, a.y, a.z, a.w}, {b.x, b.y, b.z, b.w}, s, w, sr);
    uint32_t wa = c.x, wb = c.y;
    swap_halves(wa, wb);
    __builtin_nontemporal_store(u32x2{wa, wb}, as_global(reinterpret_cast<u32x2*>(out + g0)));
  }
}

}  // namespace srq
