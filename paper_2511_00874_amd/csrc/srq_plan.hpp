// How a product is cut into tiles and slices of the contraction, and which kernel form multiplies it.  Host arithmetic only
// (no GPU headers: a test compiles it by itself).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace srq {

// Which matrix pipeline multiplies the operands.
enum Pipe {
  PIPE_I8 = 0,   // int8 codes, int32 accumulators (exact)
  PIPE_F8 = 1,   // E4M3 / E5M2 codes on the fp8 pipeline (hardware aligns groups of 8 products)
  PIPE_BF16 = 2, // E4M3 / E5M2 grid values widened to bfloat16: exact products, binary32 sums
  PIPE_F16C = 3, // E4M3 / E5M2 codes widened to binary16 inside the kernel: the same arithmetic as PIPE_BF16
                 // from one byte per element
  PIPE_F16W = 4  // PIPE_F16C where small products take PIPE_BF16: slices of the contraction at most as long as
                 // PIPE_BF16 makes them (a sum's rounding errors grow with the slice), and its size limit
};

constexpr int STAGE_BYTES = 128;  // bytes of the contraction that a kernel takes per stage

struct Plan {
  int tile;  // 0: 256x256, 1: 128x128, 2: 64x64, 3: 128x192
  int bm, bn;
  uint32_t nsplit, k_per_split;
};

constexpr int NUM_CU = 256;

// Tile shape and number of contraction slices by a cost model (seconds, for ranking only):
//   time = rounds x (stages per item + fixed per-item stages) x operations per stage / rate
//          + the pass over the partial results that every extra slice adds.
// `rate` is what a CU sustains with that tile shape once its slots are full (measured with MFMA tiles of 32 x 32, int8: the
// other pipelines scale alike; those of 16 x 16 take 0.95 to 0.97 of the time on 256 x 256, 0.93 to 1.0 on 128-row tiles in full rounds): 256 x 256 tiles on workgroups that stay run one per CU and hide
// most of a tile's start and end; the 128-row tiles run two workgroups per CU (one alone gets
// about 0.85 of the CU's rate); 64 x 64 is for problems too small for anything else.
struct TileKind {
  int tile, bm, bn, per_cu;
  double rate_chip;   // operations per second over the whole chip, slots full
  double fixed;       // start + end of an item, in stages
};
constexpr TileKind TILE_KINDS[] = {
    {0, 256, 256, 1, 2.1e15, 6.0},
    {1, 128, 128, 2, 1.45e15, 3.0},
    {3, 128, 192, 2, 1.5e15, 3.0},
    {2, 64, 64, 4, 0.5e15, 4.0},
};
constexpr double PARTIAL_BYTES_PER_SECOND = 4.0e12;  // partial tiles out and back in

inline Plan make_plan(size_t P, size_t Q, size_t row_bytes) {
  const size_t ksteps = (row_bytes + STAGE_BYTES - 1) / STAGE_BYTES;
  Plan best{};
  double best_time = 0.0;
  bool have = false;
  for (const TileKind& k : TILE_KINDS) {
    const size_t t = ((P + k.bm - 1) / k.bm) * ((Q + k.bn - 1) / k.bn);
    // slices only for long contractions (at least 8 stages each), at most 64
    size_t max_split = ksteps >= 16 ? ksteps / 8 : 1;
    if (max_split > 64) max_split = 64;
    const double ops_stage = 2.0 * k.bm * k.bn * STAGE_BYTES;
    const double rate_cu = k.rate_chip / NUM_CU;
    for (size_t n = 1; n <= max_split; ++n) {
      const size_t items = t * n, slots = (size_t)NUM_CU * k.per_cu;
      const size_t rounds = (items + slots - 1) / slots;
      const size_t stages = (ksteps + n - 1) / n;
      // a workgroup's share of its CU: alone, or one of per_cu
      const double share = items <= (size_t)NUM_CU ? (k.per_cu > 1 ? 0.85 : 1.0) : 1.0 / k.per_cu;
      double time = (double)rounds * ((double)stages + k.fixed) * ops_stage / (rate_cu * share);
      if (n > 1) time += 2.0 * (double)n * (double)P * (double)Q * 4.0 / PARTIAL_BYTES_PER_SECOND;
      if (!have || time < best_time) {
        have = true;
        best_time = time;
        best.tile = k.tile; best.bm = k.bm; best.bn = k.bn;
        best.nsplit = (uint32_t)n;
      }
    }
  }
  const size_t steps_per = (ksteps + best.nsplit - 1) / best.nsplit;
  best.k_per_split = (uint32_t)(steps_per * STAGE_BYTES);
  best.nsplit = (uint32_t)((ksteps + steps_per - 1) / steps_per);
  return best;
}

// Bytes of the partial sums of a planned product.
inline size_t partial_bytes(const Plan& pl, size_t P, size_t Q) {
  return pl.nsplit > 1 ? (size_t)pl.nsplit * P * Q * sizeof(uint32_t) : 0;
}

// The plan of a product on one of the pipelines.  PIPE_F16W has half the row bytes of PIPE_BF16, and by its own
// count would cut long contractions into half as many slices: every accumulator would then sum twice as many
// products one after another, and round about 1.4 times as far from the exact result.  Where its slices would be longer
// than those of PIPE_BF16 it takes that plan, the same slices in half the bytes.  E4M3 steps, us and error of the
// results against 64 bits with its own slices and with those: 1472 x 1440 x 4448 129 (9.4e-8), 130 (7.0e-8), on PIPE_BF16
// 143; 224 x 1248 x 1792, where a slice sum is a launch more, 43 (5.9e-8), 47 (5.0e-8), on PIPE_BF16 51.  (These without
// groups of waves, with the error of PIPE_BF16.)
inline Plan plan_for(size_t P, size_t Q, size_t R, int pipe) {
  if (pipe == PIPE_BF16) return make_plan(P, Q, 2 * R);
  const Plan pl = make_plan(P, Q, R);
  if (pipe != PIPE_F16W) return pl;
  Plan wide = make_plan(P, Q, 2 * R);
  if (wide.nsplit == 1 || 2 * (size_t)pl.k_per_split <= wide.k_per_split) return pl;
  wide.k_per_split /= 2;
  return wide;
}

// One launch of 64 x 64 tiles over the whole contraction, with groups of waves, in place of the plan's slices or of its
// 128-row tiles, where the output is so small that the chip holds all of those tiles at once, two a CU: nothing is written
// out twice and no sum is left to a second launch.  Times of both in microseconds from straight lines through some 900
// products of random sizes, each repeated in a graph (st: stages; mb: megabytes of partial sums; `widens`: 8-bit floats on the
// f16 pipeline, twice the matrix work a stage), and 1.5 more for the second launch: in a graph it costs the GPU no more than its
// sum, but 3.5 us where small calls follow one another from the host and it is the host that they wait for.  As planned and
// this way, int8 and E5M2: 1008 x 768 x 3072 (three slices) 13.7 -> 7.1, 15.8 -> 10.2; 512 x 1024 x 4096 (four) 13.3 -> 8.1,
// 15.6 -> 12.2; 32 x 4240 x 2448 (64 x 64 tiles, two) 6.9 -> 6.0, 8.2 -> 8.7; 1024 x 2048 x 2048 (128 x 128 tiles, uncut)
// 12.9 -> 9.3, 17.4 -> 12.4.  The other side of the lines: more than a tile a CU (576 x 2048 x 6000 int8 22.2 -> 29.9).
// Whole calls with absmax and quantizers, in a row, waited for and in a graph: 48 x 1072 x 1664 E4M3 25.7, 37.4, 19.2 -> 20.9,
// 37.9, 20.2; 208 x 224 x 3248 int8 26.4, 36.9, 19.1 -> 22.7, 39.3, 22.0.  Over 420 random shapes the rule loses 0.35 us a call
// against the better form in a graph and 0.3 in a row (0.23 and 0.67 if the launch is not counted).
// Beyond some length the lines no longer hold and the slices stay: 64 stages where every row begins a cache line; otherwise
// 28 where 64 x 64 tiles are planned, 24 with codes to widen, and 40 where 128-row tiles are (3536 x 128 x 9696 int8 17.6 -> 24.3,
// 640 x 992 x 7168 17.2 -> 13.4, 1008 x 224 x 10240 14.7 -> 19.0; with the quantizers, whose codes come from beyond the L2,
// 496 x 304 x 6864 17.3 -> 32.3, 240 x 240 x 3984 19.8 -> 27.2, 848 x 320 x 3408 E5M2 17.2 -> 21.8; int8 at 28 to 36 and 36 to 48
// stages, the middle half: 64 x 64 tiles 2.3 to 4.8 and 4.2 to 8.7 us more, 128-row tiles 1.6 less to 1.2 more and 0.9 to 2.9 more).
// `leaves`: the sum of the slices is left to a later launch and runs beside its matrix work.  Slices of 64 x 64 tiles then
// always stay: the two products of E4M3 backward calls of up to 2^27 multiplications took 10 to 30 % longer otherwise (73 of 80
// random ones by more than 8 %), E5M2 2048 x 192 x 352 9.4 -> 11.8.  With 128-row tiles there is less to save: M, N, K 5824 x 960
// x 1216 int8 34.0 -> 39.3 and 4240 x 7360 x 224 E5M2 45.3 -> 50.0 stay in slices, 2736 x 432 x 1312 22.1 -> 17.8 does not.
inline bool small_in_one_pass(const Plan& pl, size_t P, size_t Q, size_t row_bytes, bool widens, bool leaves) {
  const size_t t64 = ((P + 63) / 64) * ((Q + 63) / 64);
  const size_t items = ((P + pl.bm - 1) / pl.bm) * ((Q + pl.bn - 1) / pl.bn) * pl.nsplit;
  const size_t stages = (row_bytes + STAGE_BYTES - 1) / STAGE_BYTES;
  if (pl.tile == 0 || t64 > 2 * NUM_CU || (pl.tile == 2 && pl.nsplit == 1)) return false;
  if (items > NUM_CU || (leaves && pl.tile == 2)) return false;
  if (pl.nsplit > 1 && stages > (row_bytes % STAGE_BYTES == 0 ? 64u : pl.tile != 2 ? 40u : widens ? 24u : 28u)) return false;
  const double st = (double)stages, slice = (double)(pl.k_per_split / STAGE_BYTES);
  const double mb = pl.nsplit > 1 ? 4e-6 * pl.nsplit * (double)P * (double)Q : 0.0;
  const double once = t64 <= NUM_CU ? (widens ? 3.2 + 0.285 * st : 2.75 + 0.18 * st)
                                    : (widens ? 4.0 + 0.49 * st : 2.5 + 0.44 * st);
  double planned = pl.tile == 2 ? 5.6 + (widens ? 0.22 : 0.085) * slice + 0.59 * mb
                                : (widens ? 5.8 : 4.0) + 0.73 * slice + 0.44 * mb;
  if (pl.nsplit > 1) planned += leaves ? -1.5 - 0.2 * mb : 1.5;
  return once < planned;
}

// The kernel form of a planned product, its slices and the stages of its LDS ring.  _G2, _G4: groups of waves share a tile;
// _S2: two sets of accumulators stand for two groups.
enum Form { FORM_256x256, FORM_128x128, FORM_128x128_S2, FORM_128x128_G2, FORM_128x192, FORM_64x64_G2, FORM_64x64_G4 };
struct Launch {
  Form form;
  uint32_t nsplit, k_per_split;
  int ring;
};
// Binary32 sums: an accumulator holds the part of a slice that its group of waves multiplies, half of it or a quarter, and no
// choice below makes the parts longer than the plan's slices.  Forms over the same slices in two halves, of 64 x 64 or
// 128 x 128 tiles, in groups or in sets, give the same result bit for bit: `rides`, which sr_linear_bwd has and
// sr_linear_bwd_data has not, may choose among them.
//
// The rings leave room on a CU for quantizer workgroups of another stream, and fewer stages are not slower alone: with eight
// waves on 128 x 128 tiles three take 0.97 to 1.0 of the time of four (2048 x 2048 x 4096 int8 23.3 and 23.1 us, E5M2
// 33.2 and 33.2), and beside the quantizer of another layer, M, N, K 2672 x 704 x 6128 E5M2, a step of 66.4 us with four takes 52.5
// (51.7 with four waves and two stages), 5792 x 592 x 5120 E5M2 77.5 and 66.9 (65.9), 2624 x 896 x 4288 int8 41.8 and 41.6
// (48.0).  64 x 64 tiles: three stages as well, 0.94 to 1.0 of the time of four or five alone.  Only longer contractions with a CU for
// a tile take four and five, as three are up to 1.2 times slower where the operands come from beyond the L2 (16 x 5632 x 5632
// int8 9.8 and 12.0): in one pass, and from eight stages on, except where the codes are widened, which covers the loads (quantizer
// and product, us, with three and four, at 8, 10, 11 and 16 stages: int8 128 x 1136 x 992 9.5 and 9.2, 128 x 1760 x 1280 10.5 and 10.3,
// 16 x 80 x 1296 9.1 and 8.4, bfloat16 values 16 x 224 x 1952 12.0 and 11.3; codes 64 x 1504 x 1616 12.9 and 13.1; at one to three
// stages four take 1.00 to 1.02 of the time of three).
//
// `rides`: slices of an earlier product whose sum the launch carries (0: none).  Its workgroups take as much LDS as a tile's, and
// where the tiles hold nearly all CUs they wait for them to finish instead of running beside them.
//   - Two groups on 128 x 128 tiles with such a sum: up to 192 of them, 224 from 16 stages on (both products of a backward
//     call, us without groups and with: E5M2 5328 x 3104 x 736, 252 tiles, 58.1 -> 64.1, 7296 x 1968 x 448, 228 tiles, 37.6 -> 41.5;
//     6784 x 4016 x 432, 212 tiles, 60.7 -> 56.9), or for integers 24 stages, beside which it ends in time (10304 x 5440 x 288,
//     243 tiles, 65.0 -> 61.9; at 16 and 19 stages 31.5 -> 33.8, 39.5 -> 41.9).  Instead four waves, a ring of 64 KiB, and for
//     binary32 sums two sets of accumulators (1.00 to 1.03 of the time of one).
//   - More than a 64 x 64 tile a CU: not over 12 stages or fewer beside a sum of more than three slices, a chain of as many
//     loads (int8 6064 x 1488 x 320, six, 25.1 -> 27.7; E4M3 8240 x 1152 x 160, 13, 27.7 -> 29.7; with two, 2816 x 272 x 368 int8
//     11.6 -> 10.0).  8-bit floats and sums of four to six slices: not over 6 stages (E5M2 6432 x 208 x 304 14.5 -> 15.8; at twelve,
//     4832 x 1488 x 320, 27.5 -> 23.6).
inline Launch choose_launch(const Plan& pl, size_t P, size_t Q, size_t row_bytes, int pipe, bool leaves, uint32_t rides) {
  const bool widens = pipe == PIPE_F16C || pipe == PIPE_F16W, is_int = pipe == PIPE_I8;
  const Form four_waves = is_int ? FORM_128x128 : FORM_128x128_S2;
  if (pl.tile == 0) return Launch{FORM_256x256, pl.nsplit, pl.k_per_split, 2};
  // (four groups stand for up to four slices of a binary32 sum; PIPE_F8 has two sub-steps a stage, no work for four groups)
  if (small_in_one_pass(pl, P, Q, row_bytes, widens, leaves)) {
    const uint32_t whole = (uint32_t)((row_bytes + STAGE_BYTES - 1) / STAGE_BYTES * STAGE_BYTES);
    const bool one_a_cu = ((P + 63) / 64) * ((Q + 63) / 64) <= NUM_CU;
    const bool waits = rides > 3 && pl.tile == 1 && pl.nsplit == 1 && !one_a_cu &&
                       row_bytes <= (size_t)(is_int || rides > 6 ? 12 : 6) * STAGE_BYTES;
    if (waits) return Launch{four_waves, 1, whole, 2};
    if (is_int || pl.nsplit <= 2) return Launch{FORM_64x64_G2, 1, whole, one_a_cu ? 4 : 3};
    if (pipe != PIPE_F8 && pl.nsplit <= 4) return Launch{FORM_64x64_G4, 1, whole, one_a_cu ? 5 : 3};
  }
  // 64 x 64 tiles: eight waves of 32 x 32 in two groups take 0.91 to 1.02 of the time of four waves (uncut one stage 1.0 to
  // 1.02, four 0.99, eight 0.95; slices 0.98).
  if (pl.tile == 2) {
    const bool one_a_cu = ((P + 63) / 64) * ((Q + 63) / 64) * pl.nsplit <= NUM_CU;
    const int ring = one_a_cu && !widens && rides == 0 && pl.k_per_split >= 8 * STAGE_BYTES ? 4 : 3;
    return Launch{FORM_64x64_G2, pl.nsplit, pl.k_per_split, ring};
  }
  if (pl.tile == 3) return Launch{FORM_128x192, pl.nsplit, pl.k_per_split, 2};
  // A workgroup that has a CU to itself: eight waves in two groups instead of four, and a longer ring.  2048 x 2048 x 4096 int8
  // 25.9 -> 23.1 us, E5M2 34.0 -> 33.2; 512 x 5632 x 5632 30.4 -> 24.0, 39.1 -> 35.9; at 8 to 15 stages int8 0.81 to 1.01 of the
  // time, E5M2 0.94 to 1.05; at three to seven 0.94 and 0.98, at one and two 8-bit floats 1.00 to 1.03.  (Codes of 8-bit floats
  // from as few terms on as their bfloat16 form, so that the sums of the two are as long.)
  const size_t items = ((P + 127) / 128) * ((Q + 127) / 128) * pl.nsplit, stages = pl.k_per_split / STAGE_BYTES;
  if (items > NUM_CU || stages < (widens ? 2 : 3)) return Launch{FORM_128x128, pl.nsplit, pl.k_per_split, 2};
  const bool room = rides == 0 || items <= (stages < 16 ? 192 : 224) || (is_int && stages >= 24);
  return room ? Launch{FORM_128x128_G2, pl.nsplit, pl.k_per_split, 3} : Launch{four_waves, pl.nsplit, pl.k_per_split, 2};
}

// One set of binary32 sums of widened codes: in MFMA tiles of 32 x 32 (true) or of 16 x 16, which round differently.  The larger ones
// where a product has at most `slots` tiles of 128 x 192: alone a CU for each (launch_mma says why); in a pair see choose_pair's end.
inline bool sums_in_large_mfma(Form form, size_t P, size_t Q, uint32_t nsplit, size_t slots = NUM_CU) {
  return form == FORM_128x192 && ((P + 127) / 128) * ((Q + 191) / 192) * nsplit <= slots;
}

// The two products of a backward call, dW (N x K, contraction M) and dA (M x K, contraction N), in one launch of tiles of
// one size, each over the slices that it is planned with (sums of slices follow in launches of their own).  Not where one takes
// the 256 x 256 tiles, and only forms in which an accumulator of a binary32 sum holds the same part of the contraction as in a
// launch of its own (sets of accumulators stand for two groups of waves on 128 x 128 tiles; 64 x 64 tiles have two or four groups): the
// results are the same bit for bit.
//
// Two launches leave the chip idle twice while their last tiles are written, and a product of few tiles leaves CUs idle for all of its
// time.  Both products from codes, us in two launches and in one: M, N, K 4096 x 2048 x 2048 int8 44.1 -> 39.5 (E5M2, not taken,
// 67.8 -> 69.9: three tiles a CU in one launch, 128 x 192 tiles in two); 2432 x 4240 x 1216 E5M2 59.3 -> 54.0; 1008 x 3072 x 768
// E5M2 22.1 -> 14.6 (64 x 64); 2048 x 1200 x 1200 E5M2 24.6 -> 18.0.  Straight lines fitted to 640 calls of random sizes say which is
// faster; 128 x 128 tiles that are not all on the chip at once have to gain more, as a round of few tiles at the end costs most (534 tiles
// of 12976 x 2384 x 384 int8 46.0 -> 54.7, not taken).
// Over 1440 other calls, 0.80 of the time of two launches on average where one is taken, 2 % of them more than 2 % slower.
// Beside the quantizers of another layer on a second stream (a graph each; the forms with two sets of accumulators leave these no
// registers, so that they wait for a workgroup's end, but that comes sooner) still 0.89 to 1.07 of the time of both streams, 0.975 on
// average of 48: N x K 3072 x 768, E5M2, at 1008, 2048, 3072, 4096 tokens 43.8, 58.1, 78.8, 93.8 -> 44.5, 52.5, 70.2, 89.7 (products alone
// 38.4, 50.1, 65.6, 74.2 -> 31.0, 42.8, 58.2, 66.8); the worst, 2048 x 2048 on the fp8 pipeline at 2048, 58.8 -> 63.1 (47.1 -> 42.0).
// Never 128 x 128 where a product has at most 128 rows (4144 x 80 x 784 E5M2 12.3 -> 15.0: alone it takes 64 x 64 tiles), nor where the
// results do not fit the last-level cache, whose writes then bound both (30656 x 112 x 5760 int8 170 -> 200).
// Where the results are written for longer than they are multiplied (integers; the line for 64 x 64 tiles has no term for that) larger
// tiles write faster.  With more than 64 MB of results a pair takes 128 x 128 tiles where it can (2496 x 192 x 10192, us apart, on 64 x 64 and
// on 128 x 128 tiles 44.0, 43.4, 33.4; 240 x 2928 x 6736 40.5, 37.2, 30.6; 33 calls 0.77 to 1.01 of the time of 64 x 64; with 30 to 60 MB
// 0.89 to 1.3).  With more than 96 MB no 64 x 64 tiles take the place of slices of 128 x 128 (5648 x 96 x 10688 69.5 -> 86.0, 16 x 8192 x 4096
// 39.0 -> 44.0; of 11 such calls 7 lost, 1.04 on average), but for weight gradients in 16 slices or more, whose sum would ride on the input
// gradient and delay it (32768 x 16 x 1024 64.2 -> 43.3, 99808 x 16 x 256 86.7 -> 47.0).
constexpr size_t PAIR_MAX_RESULTS = (size_t)64 << 20;  // of 4 bytes
constexpr double PAIR_LARGE_MB = 64.0, PAIR_LARGE_CUT_MB = 96.0;
enum PairForm { PAIR_NONE, PAIR_128x128, PAIR_64x64 };
struct Paired {
  int waves;  // sets of accumulators (128 x 128 tiles of four waves) or groups of waves (64 x 64 of eight)
  uint32_t nsplit, k_per_split;
  bool large_mfma = false;  // one set of widened codes: sums_in_large_mfma
};
struct Pair {
  PairForm form;
  bool weight_first;  // the product with the longer tiles goes first
  Paired w, d;
};
struct PairLines {  // microseconds: constant, per stage (of a tile, by form, or of all tiles a CU), of the last tiles to end beyond an even
                    // share, MB of results, MB of partial sums, a sum; most of the separate launches' time that is worth a pair of
                    // 128 x 128 tiles
  double apart, group128, group64_one, group64_two, load_apart128, last_apart128, load_apart192, last_apart192, out, partial, sum;
  double pair128, load128, last128, out128, partial128, sum128;
  double pair64, load64, partial64, sum64;
  double worth128;
};
// (Fitted with MFMA tiles of 32 x 32.  With those of 16 x 16 in one set of sums, pairs of 128 x 128 tiles take 0.97 to 1.03 of the time
// that they took, int8 0.996 on average of 10 shapes and widened codes 0.997 of 40, and the launches apart that others keep 0.95 to 1.02,
// 0.989 of 54 and 0.991 of 82: less than what a pair has to be worth.)
constexpr PairLines PAIR_LINES[2] = {
    {5.7, 0.51, 0.21, 0.42, 0.53, 0.56, 0.70, 0.51, 0.15, 0.55, 1.5, 3.2, 0.57, 0.44, 0.07, 0.43, 1.7, 4.2, 0.27, 0.42, 1.7, 0.93},
    {6.7, 0.77, 0.27, 0.46, 0.78, 0.82, 1.21, 0.39, 0.13, 0.38, 2.3, 3.7, 0.92, 0.24, 0.05, 0.34, 2.6, 4.8, 0.31, 0.36, 1.7, 0.88}};  // widened
// Stages until the last of n1 tiles of s1 stages and then n2 of s2 <= s1 ends, where `slots` of them run at a time.
inline uint64_t stages_to_end(uint64_t n1, uint64_t s1, uint64_t n2, uint64_t s2, uint64_t slots) {
  const uint64_t full = n1 / slots * s1, late = n1 % slots, first_end = full + (late ? s1 : 0);
  const uint64_t even = (n1 * s1 + n2 * s2 + slots - 1) / slots;
  uint64_t lo = even > first_end ? even : first_end, hi = lo + s2;  // (an even share and one tile are enough)
  while (lo < hi) {
    const uint64_t t = (lo + hi) / 2;
    if (late * ((t - first_end) / s2) + (slots - late) * ((t - full) / s2) >= n2) hi = t;
    else lo = t + 1;
  }
  return lo;
}
// plan_w, plan_d: the products' plans (plan_for), which take more time than the choice
inline Pair choose_pair(size_t M, size_t N, size_t K, int pipe, const Plan& plan_w, const Plan& plan_d) {
  const bool is_int = pipe == PIPE_I8;
  if (pipe == PIPE_BF16 || (M + N) * K > PAIR_MAX_RESULTS) return Pair{PAIR_NONE, false, {1, 1, 0}, {1, 1, 0}};
  const PairLines& c = PAIR_LINES[pipe == PIPE_F16C || pipe == PIPE_F16W];
  const Launch l[2] = {choose_launch(plan_w, N, K, M, pipe, true, 0), choose_launch(plan_d, M, K, N, pipe, false, 0)};
  Pair p{PAIR_NONE, l[0].k_per_split >= l[1].k_per_split, {1, l[0].nsplit, l[0].k_per_split}, {1, l[1].nsplit, l[1].k_per_split}};
  if (l[0].form == FORM_256x256 || l[1].form == FORM_256x256) return p;
  constexpr uint64_t SLOTS = 2 * NUM_CU;  // workgroups of four waves that are on the chip at a time
  const size_t rows[2] = {N, M};
  bool sets = M > 128 && N > 128, groups = true;  // the forms that keep the sums as they are
  int halves[2], parts[2];
  uint64_t n128[2], stages[2];
  double apart = c.apart, out = 0.0, partial = 0.0, sums = 0.0, load64 = 0.0;
  for (int i = 0; i < 2; ++i) {
    const Form f = l[i].form;
    const bool two = f == FORM_128x128_G2 || f == FORM_128x128_S2 || f == FORM_64x64_G2;
    halves[i] = two && !is_int ? 2 : 1;
    parts[i] = f == FORM_64x64_G4 ? 4 : 2;
    sets = sets && f != FORM_64x64_G4;
    groups = groups && (two || is_int || f == FORM_64x64_G4);
    stages[i] = (l[i].k_per_split + STAGE_BYTES - 1) / STAGE_BYTES;
    const auto tiles = [&](size_t bm, size_t bn) { return (uint64_t)((rows[i] + bm - 1) / bm) * ((K + bn - 1) / bn) * l[i].nsplit; };
    const uint64_t t64 = tiles(64, 64);
    n128[i] = tiles(128, 128);
    const double s = (double)stages[i], mb = 4e-6 * (double)rows[i] * (double)K;
    load64 += (double)t64 * s / NUM_CU;
    if (f == FORM_128x128_G2) apart += c.group128 * s;
    else if (f == FORM_64x64_G2 || f == FORM_64x64_G4)
      apart += (t64 <= NUM_CU ? c.group64_one : c.group64_two * (t64 > SLOTS ? (double)t64 / SLOTS : 1.0)) * s;
    else {
      const uint64_t t = f == FORM_128x192 ? tiles(128, 192) : n128[i];
      const double load = (double)t * s / NUM_CU, last = (double)((t + SLOTS - 1) / SLOTS) * s - 0.5 * load;
      apart += f == FORM_128x192 ? c.load_apart192 * load + c.last_apart192 * last : c.load_apart128 * load + c.last_apart128 * last;
    }
    out += mb;
    if (l[i].nsplit > 1) {
      partial += l[i].nsplit * mb;
      sums += 1.0;
      if (i == 1) apart += c.sum;  // (the other one's sum rides)
    }
  }
  const auto cut = [](const Launch& l) { return l.form == FORM_128x128_G2 && l.nsplit > 1; };
  if (out > PAIR_LARGE_CUT_MB && (cut(l[0]) || cut(l[1])) && l[0].nsplit < 16) groups = false;
  apart += c.out * out + c.partial * partial;
  const int a = p.weight_first ? 0 : 1, b = 1 - a;
  const double load128 = (double)(n128[0] * stages[0] + n128[1] * stages[1]) / NUM_CU;
  const double last = (double)stages_to_end(n128[a], stages[a], n128[b], stages[b], SLOTS) - 0.5 * load128;
  const double t128 = c.pair128 + c.load128 * load128 + c.last128 * last + c.out128 * out + c.partial128 * partial + c.sum128 * sums;
  const double t64 = c.pair64 + c.load64 * load64 + c.partial64 * partial + c.sum64 * sums;
  const bool at_once = n128[0] + n128[1] <= SLOTS;
  const bool small = groups && (!sets || (t64 <= t128 && out <= PAIR_LARGE_MB));
  const double worth = (small ? 0.95 : at_once ? 1.0 : c.worth128) * (sums > 0.0 ? 0.95 : 1.0);
  if (!(sets || groups) || (small ? t64 : t128) >= worth * apart) return p;
  p.form = small ? PAIR_64x64 : PAIR_128x128;
  p.w.waves = small ? parts[0] : halves[0];
  p.d.waves = small ? parts[1] : halves[1];
  // MFMA tiles of one set of widened codes.  Both products in one set: 16 x 16, their many tiles fill the chip (1104 x 4448 x 3888 E5M2,
  // whose input gradient has 189 tiles of 128 x 192 alone, 75.5 us with that in 32 x 32, 72.7 so; 10 random shapes 0.966 to 0.993 of the time).
  // Beside two sets, in 32 x 32 themselves: as well where the product has up to 512 tiles of 128 x 192 alone (160 x 5808 x 1776 21.4 ->
  // 20.0, 1152 x 448 x 4256 13.5 -> 12.6; 28 random shapes with others in 16 x 16 0.94 to 1.02, 0.985 on average; all in 32 x 32 0.94 to 1.06).
  if (p.form == PAIR_128x128 && p.w.waves != p.d.waves) {
    p.w.large_mfma = sums_in_large_mfma(l[0].form, N, K, l[0].nsplit, SLOTS);
    p.d.large_mfma = sums_in_large_mfma(l[1].form, M, K, l[1].nsplit, SLOTS);
  }
  return p;
}
// The same of a gradient in a call of its own: as in the pair that the whole backward call would make of both, so that its sums are the
// same bit for bit.
inline bool large_mfma_of_gradient(const Plan& pl, const Launch& l, bool weight, size_t P, size_t Q, size_t R, int pipe) {
  if (l.form != FORM_128x192) return false;
  const size_t M = weight ? R : P, N = weight ? P : R;
  const Plan other = weight ? plan_for(M, Q, N, pipe) : plan_for(N, Q, M, pipe);
  const Pair p = choose_pair(M, N, Q, pipe, weight ? pl : other, weight ? other : pl);
  return p.form == PAIR_NONE ? sums_in_large_mfma(l.form, P, Q, l.nsplit) : (weight ? p.w : p.d).large_mfma;
}

}  // namespace srq
