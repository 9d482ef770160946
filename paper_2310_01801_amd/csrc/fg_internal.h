// Host-side plumbing shared by the translation units of the FastGen HIP library:
// the context, the workspace carve-up and the kernel launchers. Not part of the ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "../../include/fastgen.h"

// ---------------------------------------------------------------- workspace layout
// Every region starts on a 256-byte boundary. Offsets are in bytes from the workspace base.
struct fg_layout {
  // profiling scratch
  size_t rowstat;   // [U * G, n] float2  per query row (m, 1/l): softmax row = 2^(c q.k - m) / l, with m a
                    //                    shift at or near the row's largest scaled logit (log2 domain)
  size_t colsum;    // [U, n] double  cumulative attention score of every prompt token
  size_t bandcol;   // [U, n] double  the part of colsum inside the local band
  size_t keep;      // [U, n] uint8   0 = dropped, else 4 | class bits of the kept token
  size_t slot;      // [U, n] int32   exclusive prefix sum of keep (slot in the cache)
  // per-unit results and cache bookkeeping
  size_t policy;    // [U] int32
  size_t recov;     // [U, 5] double
  size_t kcount;    // [U, 5] int32
  size_t cap;       // [U] int32      slots reserved for the unit
  size_t off;       // [U + 1] int64  first slot of each unit in the pool
  size_t len;       // [U] int32      tokens held
  size_t flags;     // [8] int32      [0] pool overflow, [1] decode steps done
  // ragged cache pool (pool_tokens slots)
  size_t ck;        // [pool, d] dtype
  size_t cv;        // [pool, d] dtype
  size_t cscore;    // [pool] double
  size_t cpos;      // [pool] int32
  size_t ccls;      // [pool] uint8
  size_t clogit;    // [pool, G] double  of every held token and query head, for the units whose cumulative scores are kept:
                    //                   this step's scaled logit; three to eight bf16 heads in one workgroup per unit:
                    //                   2^(logit - shift of its tile), a factor per tile and head turns it into attention
  // decode scratch
  size_t chunk_off; // [U + 1] int32  first chunk of each unit in the flat work list (per-unit form: its place by size)
  size_t item_unit; // [max_chunks, 8] int32  work-item records: unit, chunk, cap, tokens held, pool offset lo/hi, policy word, 0
                    //                        (per-unit form: one record per unit, longest reservations first)
  size_t part;      // [max_chunks, G, d + 2] float  split-KV partial (max, sum, o) per query head
  size_t total;
  int64_t pool_tokens;
  int64_t max_chunks;
  int chunk;        // tokens per decode work item (128 or 256)
  int unit_threads; // 0: split-KV decode step; else one workgroup of this size per unit
  int update_threads; // workgroup size of the split-KV step's update kernel
};

struct fastgen_ctx {
  fg_config cfg;
  fg_layout lay;
  char* ws;
  float scale;
  int w;            // local window
  int stage;        // 0 created, 1 profiled, 2 compacted / decoding
  int steps_done;
  char err[256];
  // optional device-time accounting
  // 0 off; 1 every kernel group; N > 1: the prompt-time phases always, a decode step when
  // its index is a multiple of N
  int timing;
  struct timed { int phase; int a, b; };   // indices into `events`
  std::vector<timed> pending;
  std::vector<hipEvent_t> events;          // recorded since the last read
  std::vector<hipEvent_t> spare;
};

// Tokens per split-KV work item of the decode kernels: 256 for long sequences, 128 when a unit
// can hold at most 4096 tokens (finer items balance short caches better; measured per shape).
inline int fg_decode_chunk(int prompt_len, int max_new_tokens) {
  return ((long long)prompt_len + max_new_tokens <= 4096) ? 128 : 256;
}

// Longest units (prompt and reserved tokens) of the kernels that hold a unit's bookkeeping in registers: the
// one-workgroup-per-unit step with 512 and with 256 threads, the update kernel with 256.
constexpr int FG_UNIT_TOKENS = 4608, FG_UNIT_TOKENS_256 = 2048, FG_UPDATE_TOKENS_256 = 3072;

// Form of the decode step: 0 = split-KV attention and a second launch for merge and update; else one
// workgroup of that many threads per unit. Measured per step, split / per unit (before the logits of the per-unit form stayed in
// LDS, which took 4 to 8 % off it: 1024 of 2048 tokens 102 us, 16384 of 1024 801):
//   1024 units of 2048 tokens, d = 128 bf16        120 / 112 us     (256 threads: 118)
//   4096 of 4096                                   831 / 790        (256 threads: 799)
//   16384 of 1024, 256 threads                     948 / 845        (512 threads: 857)
//   640 of 8192                                    250 / 283; 2560 of 8192: 989 / 1004
//   64 of 1000, float32 (1 MiB per unit)           17.2 / 16.7      and one launch less
//   128 of 1500 (0.75 MiB per unit)                20.1 / 17.3
//   32 of 2048 (1.02 MiB per unit)                 14.9 / 19.0
// Grouped heads (G heads share a unit's rows), two heads or float32 (bound by the float64 logits of the heads):
//   1024 of 700, G = 2                             71 / 52;  32 of 2000, G = 2: 23 / 31
// Three to eight bf16 heads, whose workgroups contract on the matrix cores:
//   256 units of 2048 tokens, G = 4                66 / 34 us;  16 of 300, G = 8: 37 / 17
//   300 of 3000, G = 8                             170 / 60;  64 of 3000, G = 8: 86 / 55, G = 3: 43 / 37
//   4 of 3000, G = 3                               28 / 33, G = 4: 33 / 34;  16 of 2500, G = 3: 27 / 30
// A few long units of theirs (per unit / split, d = 128; its time goes with the unit's bytes and with the four or eight
// columns that the heads are padded to, the split form's with the heads; full caches, which have no update, part earlier):
//   G = 5      1 of 4600 policy 3 66 / 50, full 1.57x; 12 of 3200 1.17x; 24 of 2600 1.11x; 32 of 4000 1.11x; 4 of 1600 1.0x, 64
//              of 3200 0.95x;  d = 64: 1 of 4600 full 1.10x, 4 of 3200 0.93x
//   G = 6      4 of 4000 policy 3 1.22x, full 1.21x; 12 of 2600 1.06x, 0.99x; 24 of 4000 1.01x, 0.95x;  G = 7 full 1 of 4600 1.20x,
//              of 3200 1.01x;  G = 8 full 4 of 4600 1.08x, of 4000 0.98x
//   G = 3      full 4 of 2000 1.45x, 24 of 1600 1.10x, 48 of 3200 1.12x, 64 of 3200 1.05x, 96 of 4000 0.96x; others 4 of 2000
//              1.09x, 32 of 3000 1.06x, 48 of 2600 1.02x;  G = 4 full 4 of 2000 1.18x, 24 of 2000 1.05x, 32 of 2600 1.00x
// So: long units stay split (a few of them decide how long the launch takes), and where there are
// fewer units than CUs a workgroup's own rate bounds the bytes (tokens times heads) per unit. The step
// is a one-dimensional launch: 512 threads per unit only while that stays below 2^32 threads.
// Above 256 units some CUs hold two and take twice as long. Units of different lengths even that out
// (300 of 3600 tokens, five kinds of heads: 57 split, 46 per unit; 320 of 4500: 90 / 102, 576 of 4500 143 /
// 150; all heads of one kind, which only the device knows: 300 of 3500 72 / 87), except float32 rows of 512
// bytes beyond 1856 tokens (400 of 2010: 84 / 93, 640 of 3500: 212 / 230; 400 of 1810: 84 / 88, 300 of 1220: 39 /
// 29). Under one forced policy all units are nearly alike, and the bytes that they hold decide:
//   full caches    257 of 2600 tokens 68 / 82, 300 of 2000 57 / 61, 300 of 4500 128 / 147; 400 of 2600 101 / 100,
//                  257 of 1500 36 / 36; G = 2, 300 of 2000, 66 / 69, G = 4, 300 of 4400, 198 / 176
//   policy 3       ratios 0.3, 257 of 2600 46 / 51, 513 of 4500 161 / 185, 900 of 4500 268 / 288; 513 of 3500 133 /
//                  138, 257 of 2000 40 / 41; policy 2, 257 of 3000 34 / 28
// With few units nothing else of the card is busy while a workgroup streams its unit, and a full cache
// has no update to merge the launches for: 4 full caches of 2000 tokens 8.7 / 13.7, 32 of 1000 8.7 / 9.6, float32
// with two heads 4 of 1000 13 / 18; 64 of 1000 11.3 / 9.9, float32 32 of 500 10.2 / 8.2.
inline double fg_forced_share(const fg_config& c) {   // of the tokens, in front of special and punctuation ones
  if (c.forced_policy == 4) return 1.0;
  const int eq2 = (c.forced_policy >= 2 ? FG_COMP_FREQUENT : 0) | (c.forced_policy == 3 ? FG_COMP_LOCAL : 0);
  const int comp = c.family[0] | c.family[1] | c.family[2] | c.family[3] ? c.family[c.forced_policy] : eq2;
  return ((comp & FG_COMP_FREQUENT) ? c.r_f : 0.0) + ((comp & FG_COMP_LOCAL) ? c.r_l : 0.0);
}
inline int fg_unit_threads(const fg_config& c) {
  const int U = c.num_units, group = c.group_size > 1 ? c.group_size : 1;
  const long long tokens = (long long)c.prompt_len + c.max_new_tokens;
  const int row_bytes = c.head_dim * (c.dtype == FG_BF16 ? 2 : 4);
  const long long unit_bytes = tokens * 2 * row_bytes;
  if (tokens > FG_UNIT_TOKENS || group > 8) return 0;
  if (group == 1 && U >= 2048 && tokens <= FG_UNIT_TOKENS_256) return 256;
  if (U > (1 << 22)) return 0;
  const bool matrix = c.dtype == FG_BF16 && group > 2;   // the grouped kernel on the matrix cores
  if (c.forced_policy >= 0) {
    const double held = fg_forced_share(c) * (double)unit_bytes;
    if (c.forced_policy == 4 && U < 48 && held > 0.4e6 && tokens > 900 && !matrix) return 0;   // 4 of 1000, G = 4: 16 / 15
    // (280 full caches of 3000 tokens, G = 3: 100 split, 108 per unit; 300 of 2000, G = 4: 81 / 70)
    if (U > 256 && U <= 360 && held > 0.8e6 && tokens * group <= (matrix && group > 3 ? 0 : 16000)) return 0;
    if (U > 256 && c.forced_policy < 4 && group == 1 && held > 1.2e6) return 0;
  }
  if (matrix) {
    // longest tokens at d = 128 for up to so many units, from there on growing with their square (three to eight heads)
    static const struct { int tokens, units; } line[2][6] = {
        {{1700, 28}, {FG_UNIT_TOKENS, 1}, {1700, 28}, {2400, 12}, {FG_UNIT_TOKENS, 1}, {FG_UNIT_TOKENS, 1}},
        {{1200, 40}, {1200, 20}, {1800, 20}, {2400, 20}, {3000, 16}, {4000, 16}}};   // full caches
    const auto& few = line[c.forced_policy == 4][group - 3];
    const double over = U > few.units ? (double)U / few.units : 1.0;
    // what one policy evicts counts less (policy 2, ratio 0.3: 2 of 1819, G = 5, 26 / 31; policy 0: 7 of 4590, G = 5, 8 / 24)
    const double share = c.forced_policy >= 0 ? fg_forced_share(c) : 1.0;
    const double held = (double)tokens * row_bytes * (share >= 0.6 ? 1.0 : share > 0.0 ? 0.4 + share : 0.0);
    if (held > few.tokens * 256.0 * over * over) return 0;
    return U < 32 && group <= 4 && tokens > 2200 ? 0 : 512;
  }
  if (group > 1) return tokens * group <= (U < 256 ? 2048 : 20000) ? 512 : 0;
  if (U < 256) return unit_bytes <= (1 << 20) ? 512 : 0;
  if (U > 256 && row_bytes > 256 && tokens > 1856) return 0;
  return 512;
}

// Threads per unit of the split-KV step's update kernel. Where there are more grouped units than
// 512-thread workgroups fit the card (two per CU), smaller ones take turns sooner, as long as they hold a
// unit in registers (256 threads: 3072 tokens). 512 / 256 threads, us per step: 600 units of 500 tokens, G =
// 16, 168 / 162, 2048 of 300, G = 16, 335 / 282, 1500 of 500, G = 9, 198 / 179, 700 of 1500, G = 16, 361 /
// 354 (full caches 420 / 400, forced policy 3 574 / 603); but 600 of 5000, G = 4, 286 / 340 and 300 of 500, G =
// 12, 83 / 85.
inline int fg_update_threads(const fg_config& c) {
  return c.group_size > 1 && c.num_units > 512 && c.prompt_len + c.max_new_tokens <= FG_UPDATE_TOKENS_256 ? 256 : 512;
}

// Form of a bf16 profiling sweep by its size: the split stream with 32 or 64 owner items per workgroup,
// or 256-owner blocks singly or in heavy / light pairs. The times of the split stream and of the blocks
// are estimated in microseconds by fits to about 300 shapes of 1 to 1000 units (rms 11 %), the cheaper one
// is taken (1.1 % above the best form of every shape in the mean).
//   split stream   fixed + contraction work + workgroups + one workgroup's chain. Units are dealt out over
//                  the eight XCDs, so fewer than eight leave XCDs idle and cost as much as eight.
//                  1 unit of 8192 tokens, split / pairs: 147 + 165 / 222 + 251 us (with 32 owners 242 + 303);
//                  of 12000: 280 + 355 / 314 + 360; of 16384: 493 + 598 / 431 + 498
//   blocks         fixed + tiles of the heaviest workgroup (a pair: the two blocks' tiles together).
//                  Singly at most three per CU and six per unit (64 x 1024 tokens: 43 -> 35, 256 x 333:
//                  26 -> 18; 256 x 1024: 57 -> 70); not in the second sweep at d = 128 (128 x 700: 39 -> 42),
//                  and not where four nearly full blocks per unit already fill the card as pairs in the
//                  first sweep (192 x 1000, d = 128: 59 -> 62; 128 x 1000, d = 64: 36 -> 39).
// 32 owners serve up to one workgroup per CU and 64 blocks per unit, beyond that they read too much (1 x
// 4096, 32 / 64 owners: 82 + 97 / 52 + 70). With one block per unit and four or more heads the chain of
// a second round of workgroups decides (200 x 230 tokens, G = 8: 88 split, 78 blocks).
enum fg_sweep_form { FG_SWEEP_SPLIT_32, FG_SWEEP_SPLIT_64, FG_SWEEP_BLOCKS, FG_SWEEP_PAIRS };
inline fg_sweep_form fg_sweep_form_of(int d, int pass, int U, int n, int G) {
  struct fit { double s0, work, groups, chain, pair0, pair, block0, block; };
  static const fit fits[2][2] = {
      {{7.0, 0.60, 0.0040, 0.055, 7.6, 0.67, 7.1, 0.70}, {6.0, 0.64, 0.0085, 0.20, 8.9, 0.85, 7.6, 0.90}},    // d = 64
      {{6.0, 0.96, 0.0083, 0.130, 9.5, 0.89, 7.8, 0.93}, {6.0, 0.89, 0.0165, 0.24, 11.0, 1.02, 0.0, 0.0}}};   // d = 128
  const fit& f = fits[d == 128][pass == 2];
  const double units = (double)U * (pass == 1 ? G : 1), heads = pass == 1 ? 1.0 : (double)G;
  const double nb32 = (n + 31) / 32, nb64 = (n + 63) / 64, nblk = (n + 255) / 256;
  const double spread = 8.0 * (double)(((long long)units + 7) / 8);
  bool single = (pass == 1 || d == 64) && nblk <= 6.0 && units * nblk <= 768.0;
  if (pass == 1 && nblk == 4.0 && n > 960 && units * nblk > (d == 128 ? 576.0 : 320.0)) single = false;
  const double tiles = heads * (single || nblk == 1.0 ? n : 2.0 * n - 256.0 * (nblk - 1.0)) / 32.0;
  const double split = f.s0 + f.work * spread * heads * nb64 * (nb64 + 1.0) / 1024.0 + f.groups * spread * nb64 + f.chain * heads * n / 32.0;
  const double blocks = single ? f.block0 + f.block * tiles : f.pair0 + f.pair * tiles;
  const bool second_round = nblk == 1.0 && heads >= 4.0 && units * nb64 > 512.0;
  if (split < blocks && !second_round) return units * nb32 <= 256.0 && nb32 <= 64.0 ? FG_SWEEP_SPLIT_32 : FG_SWEEP_SPLIT_64;
  return single ? FG_SWEEP_BLOCKS : FG_SWEEP_PAIRS;
}

// Scratch of fastgen_profile_static: the profiling regions of every shape that it takes.
constexpr size_t FG_STATIC_SCRATCH = (size_t)32 << 20;

// Room for the partial sums [parts, U, columns] of the one-pass kernels (a prompt's columns, up to 1024), two doubles each. The rules below choose within it by the
// shape alone, and a context's workspace as well as the static scratch always hold it, so that a shape gives
// the same bits with any cache pool and from either entry point. (Most chosen: all of it, 2048 units of 1792 tokens in two parts.)
constexpr size_t FG_PART_SUMS = (size_t)64 << 20;

// Both bf16 sweeps in one pass (profile_once.hip): waves of a workgroup and workgroups per unit, 0 waves where the two
// sweeps serve. A workgroup of 8 waves holds 1024 columns and fills a CU, one of 4 waves 512 and half a CU. Measured,
// two sweeps / one pass in us (random inputs, launches back to back; in brackets the workgroups per unit; the one pass
// before its shifts came from the rows before, which took another 5 to 15 % off it, 4096 units of 1024 tokens 1154, and before a
// single block, up to 64 tokens, had a kernel of its own, 1 us less and up to 45 %: every line lies on the side of the two sweeps,
// which keep shapes near it that one pass may serve faster by now):
//   d = 128    4096 units of 1024 tokens 1586 / 1324 (1), of 512 542 / 401 (1), 300 of 1000 152 / 110 (4), 64 of 1000 77 / 25
//              (4), 8 of 1000 22 / 15 (10), 128 of 512 49 / 19 (2), 32 of 333 16 / 10 (6), 64 of 64 7.2 / 5.4 (1)
//   d = 64     4096 of 1024 1116 / 1073 (1), 64 of 1000 49 / 23 (4), 32 of 400 13.5 / 10.2 (7), 4 of 1000 15.7 / 14.5 (10)
//   G = 4      d = 128: 32 of 512 48 / 24 (8), 200 of 333 107 / 55 (5), 64 of 64 10.4 / 12.4; d = 64: 16 of 200 13.7 / 16.3, 8 of
//              333 17.5 / 18.8; G = 8: 300 of 1000 973 / 787 (4), 128 of 64 16.8 / 23.3, d = 64: 32 of 256 25.4 / 27.9
// Parts, at most ten: the more of the places are taken in the last round the better, less 5 % for every further
// part's prologue and sums, which the selection adds; a single pair of blocks stays whole. The parts of a unit run
// on one XCD and units are dealt out over the eight, so the fullest XCD (an eighth of the units, rounded up) counts the
// rounds: 83 units of 519 tokens, d = 64, G = 16, in three parts each put 33 workgroups on 32 CUs (261), in five 185; two
// sweeps 194. Many units fill the places whole, and only parts with work enough gain (one part / several: 658 of 159, d = 64,
// G = 2, 31.9 / 36.6, 1746 of 365, d = 64, 80 / 92, 1667 of 290, G = 4, 305 / 329; but 1099 of 365, d = 64, G = 16, 851 /
// 761, 1804 of 965 618 / 593); above 2048 nothing is gained. Over 4070 shapes 2.0 % above the best form in the mean.
// A unit's G heads are one workgroup's work one after the other, where the first sweep alone has a workgroup for
// each: several heads need enough 64 x 64 tiles in all, single blocks of them enough units, and blocks that are mostly
// empty weigh more with them. Two sweeps / one pass, or the gain of one pass:
//   up to 32 tokens      d = 128: 576 of 22, G = 16, 56 / 85, 225 of 21, G = 4, 9.8 / 12.3, 27 of 10, G = 2, 6.4 / 7.6;
//                        but 482 of 32, G = 4, 18.4 / 13.1, 1277 of 16, G = 2, 23.3 / 19.7; d = 64: 3387 of 21 22.9 / 27.2
//   two blocks, G = 2    d = 64: 16 of 77 7.9 / 9.1, 97 of 95 10.7 / 9.1; d = 128: 40 of 86 9.5 / 9.9, 54 of 99 10.8 / 9.9
//   d = 64, > 512 units  549 of 78, G = 16, 105 / 121, 1368 of 83, G = 6, 84 / 92, 620 of 139, G = 12, 128 / 156; but 1398
//                        of 128, G = 4, 1.21x, 1161 of 229, G = 6, 1.13x
//   tiles (n < 512)      G > 8, d = 64: 119 of 84 (357) 0.76x, 361 of 96 (1083) 0.95x, 226 of 163 (1356) 1.54x; d = 128: 114
//                        of 143 (684) 0.87x, 338 of 92 (1014) 1.19x. G 5..8, d = 64: 57 of 135 (342) 0.95x, 213 of
//                        114 (639) 1.21x; d = 128: 104 of 135 (624) 0.97x, 56 of 158 (336) 1.06x, 59 of 237 (590) 1.46x
//   few units            d = 64: 2 of 534, G = 4, 29 / 31, 1 of 660, G = 5, 0.98x, 5 of 372, G = 8, 0.88x; G > 8: 3 of 378, d = 64,
//                        0.85x, 7 of 320 0.99x. From some 400 tiles on these would gain (5 of 894, d = 64, G = 8, 1.28x, 17 of
//                        873, G = 12, 219 / 88): the lines for few units leave that to the two sweeps
constexpr int FG_ONCE_TOKENS = 1024;   // columns that the one-pass kernels hold
constexpr double FG_ROW_SUM_LESS = 1.5;   // what a row sum of the columns behind them, between 1 and 2, is handed on less by
struct fg_once_form { int waves, parts; };
inline fg_once_form fg_once_of(int d, int U, int n, int G) {
  if (n > 1024 || U > (1 << 22)) return {0, 1};
  const int blocks = (n + 63) / 64;
  const double tiles = (double)U * blocks * (blocks + 1) / 2;
  if (G > 2 && blocks == 1 && (d == 64 || U < (G > 4 ? 256 : 192))) return {0, 1};
  // up to 32 tokens leave half of a block empty: with several heads one round of workgroups at most, which a few
  // units do not fill
  if (n <= 32 && (G > 1 ? U <= (G == 2 ? 200 : 320) || (U > 512 && (G > 2 || d == 64)) : d == 64 && U > 1024)) return {0, 1};
  if (blocks == 2 && G == 2 && U <= 66 && (d == 64 || n <= 96)) return {0, 1};
  if (d == 64 && U > 512 && ((blocks == 2 && G > 2 && n <= 96) || (blocks == 3 && G > 4 && n <= 160))) return {0, 1};
  if (d == 64 && G > 2 && U < 3 && n < 640) return {0, 1};
  if (n < 512 && blocks > 1) {
    const double least = G > 8 ? 1280 : G > 4 ? (d == 64 ? 640 : 400) : G > 2 ? (d == 64 ? 320 : 200) : G == 2 && d == 64 && blocks > 2 ? 320 : 0;
    if (tiles < least) return {0, 1};
  }
  if (G > 4 && d == 64 && U < 8) return {0, 1};
  if (G > 8 && U < 32) return {0, 1};
  const int waves = n > 512 || (U <= 128 && n > 128) ? 8 : 4, places = waves == 8 ? 256 : 512;
  int parts = 1;
  const bool enough = U <= 512 || (U <= 1024 ? G * blocks >= 8 : blocks > 3 && G * blocks >= (blocks > 12 ? 16 : 24));
  if (U <= 2048 && enough && (blocks > 2 || (blocks == 2 && G > 1))) {
    long long most = (long long)(FG_PART_SUMS / ((size_t)U * n * 16));
    if (most > 10) most = 10;
    if (most > blocks) most = blocks;
    double best = 0.0;
    for (int p = 1; p <= most; ++p) {
      const int rounds = ((U + 7) / 8 * p + places / 8 - 1) / (places / 8);
      const double score = (double)U * p / ((double)rounds * places) * (1.05 - 0.05 * p);
      if (score > best + 1e-9) { best = score; parts = p; }
    }
  }
  // a last round that is mostly empty and not filled: 2049 of 1000, d = 64: 559 / 585, 1330 of 923, d = 64: 332 / 337; but
  // 1447 of 926, d = 64: 362 / 340, 459 of 1002 156 / 121
  if (parts == 1 && U > 256 && n > 512 && (d == 64 || G > 1) &&
      (double)U < (d == 64 && n > 896 ? (U > 1024 ? 0.9 : 0.85) : 0.75) * (double)((U + places - 1) / places) * places)
    return {0, 1};
  // eight waves for little more than four hold, in two parts of unequal work: 1864 of 537, G = 3, 587 / 631, 1028 of 520, G =
  // 12, 1319 / 1451
  if (d == 64 && n > 512 && n <= 544 && U > 640 && parts == 2) return {0, 1};
  return {waves, parts};
}

// Longer bf16 prompts: workgroups per unit that take the first 1024 columns of all rows in one pass, 0 where the two sweeps
// serve the whole prompt. The triangle of rows and columns from 1024 on stays with the two sweeps: the first one leaves its
// rows' sums, which join the one pass, and the second one takes the rows' normalisers from there. Two sweeps / so, in us (in
// brackets the workgroups per unit of that run; for some the rule, fitted afterwards, picks more, 256 of 3000 one less: with its parts and the
// present kernels 1024 of 2048 1106, of 1337 497, 256 of 3000 610, 64 of 1060 43, 32 of 2048 86, d = 64, 1024 of 2048 801, 256 of 2048, G = 4, 1033):
//   d = 128    1024 units of 2048 tokens 1330 / 1159 (1), of 1337 688 / 554 (1), 256 of 3000 666 / 617 (4), 1024 of 4096 4654 / 4090 (3),
//              512 of 8192 8773 / 8430 (2), 64 of 1060 90 / 42 (4), 32 of 2048 130 / 85 (8), 16 of 2048 88 / 60 (16), 64 of 4096 343 / 343 (4)
//   d = 64     1024 of 2048 868 / 811 (1), 432 of 1337 254 / 206 (1), 700 of 2048 613 / 612 (1), 32 of 3000 142 / 120 (8), 180 of 2048 201 / 200 (4)
//   G > 1      256 of 2048, G = 4, 1370 / 1138 (1), 400 of 4000, G = 2, 3602 / 3240 (3), 64 of 4000, G = 8, 2491 / 2230 (4), 16 of 2048, G = 8, 391 / 303 (9)
// Parts: as above, the fullest XCD counts the rounds. A part's prologue and sums cost 5 % of a prompt of 1060 tokens (7 % at
// d = 64), 1 % of one of 2048; several workgroups that read a unit's keys from one L2 gain 2 to 3 % at d = 128 (1024 units of
// 4096 in one, two, three parts: 1.10x, 1.11x, 1.14x; of 1060 1.40x, 1.31x, 1.27x). Few units of long prompts stay: their
// sweeps spread over the card as well, and the share of the first columns falls (32 units of 4096 0.98x, 100 of 6000 0.94x, 67 of 3469 0.96x, 8 of
// 3000 1.09x, 0.94x at d = 64, 4 of 1060, d = 64, 0.80x; 8 of 1500 1.14x, 1.07x). At 8192 tokens 1.03x; beyond, nothing was measured.
inline int fg_once_long_parts(int d, int U, int n, int G) {
  (void)G;   // (heads lengthen a part; few units of many heads have not been measured and count as few)
  if (n <= FG_ONCE_TOKENS || n > 8192 || U > (1 << 22)) return 0;
  if (n > (U >= 180 ? 8192 : U >= 96 ? 5000 : U >= 12 ? 3200 : U >= 8 ? 1600 : 0)) return 0;
  long long most = (long long)(FG_PART_SUMS / ((size_t)U * FG_ONCE_TOKENS * 16));
  if (most > 16) most = 16;   // (a prompt of more than 1024 tokens has 17 blocks)
  const double part = (d == 64 ? 0.075 : 0.05) * (1024.0 / n) * (1024.0 / n);
  int parts = 1;
  double best = 0.0;
  for (int p = 1; p == 1 || p <= most; ++p) {
    const long long rounds = ((long long)(U + 7) / 8 * p + 31) / 32;
    const double shared = d == 128 && n >= 1700 ? (p > 2 ? 1.03 : p > 1 ? 1.02 : 1.0) : 1.0;
    const double score = (double)U * p / (256.0 * (double)rounds) * (1.0 - part * (p - 1)) * shared;
    if (score > best + 1e-9) { best = score; parts = p; }
  }
  return parts;
}

// Both float32 sweeps in one pass (profile_f32.hip): workgroups per unit, 0 where the two sweeps serve. Up to 2048
// workgroups in all (32 MiB of partial sums at most), at least two blocks of 16 rows each. Measured, two sweeps / one pass in us:
//   64 units of 1000 tokens, d = 128     464 / 253;  16 of 1000 134 / 78
//   64 of 128, d = 128                   25 / 16, d = 64, G = 4: 40 / 34;  128 of 64, d = 64, G = 2: 17 / 16
//   32 of 128, G = 4                     41 / 48;  4 of 700, G = 4: 127 / 117;  8 of 1000, G = 4 (248 workgroups): 276 / 173
// Fewer than 256 workgroups leave CUs idle, which the sweeps' workgroups of 16 rows do not; short prompts of several
// heads need more of them (two sweeps / one pass: 130 of 65, d = 64, G = 4, in 260 workgroups 37 / 48, 131 of 71, G = 16, in 262
// 225 / 266; but 114 of 95, G = 8, in 342 158 / 122, 83 of 120, G = 16, in 332 304 / 253, and 120 of 84, d = 64, G = 16, in 360 134 / 148).
inline int fg_once_f32_parts(int U, int n, int G) {
  if (n < 64 || n > 1024 || U > (1 << 22)) return 0;
  const long long blocks = (n + 15) / 16;
  long long parts = 2048 / U < blocks / 2 ? 2048 / U : blocks / 2;
  if (parts < 2) parts = 1;
  return U * parts >= (G > 2 && blocks < 6 ? 400 : 256) ? (int)parts : 0;
}

// Up to so many parts the selection adds them itself; more of them (float32) keep the card busy in a launch of their own
// (64 units of 1000 tokens in 31 parts: 32 MB, in the 64 workgroups of the selection 20 us, in all CUs 10).
constexpr int FG_SELECT_PARTS = 10;

// What serves a configuration without a supplied log-sum-exp (0 waves: the two sweeps), and the bytes of its partial sums.
inline fg_once_form fg_once_form_of(const fg_config& c) {
  const int G = c.group_size > 1 ? c.group_size : 1;
  if (c.dtype == FG_BF16) {
    if (c.prompt_len <= FG_ONCE_TOKENS) return fg_once_of(c.head_dim, c.num_units, c.prompt_len, G);
    const int parts = fg_once_long_parts(c.head_dim, c.num_units, c.prompt_len, G);
    return {parts ? 8 : 0, parts ? parts : 1};
  }
  const int parts = fg_once_f32_parts(c.num_units, c.prompt_len, G);
  return {parts ? 4 : 0, parts ? parts : 1};
}
inline size_t fg_part_bytes(const fg_config& c) {
  const fg_once_form f = fg_once_form_of(c);
  const int cols = c.prompt_len < FG_ONCE_TOKENS ? c.prompt_len : FG_ONCE_TOKENS;
  return f.waves && f.parts > 1 ? (size_t)f.parts * c.num_units * cols * 16 : 0;
}

// ---------------------------------------------------------------- launch arguments
struct fg_profile_args {
  const void* Q; const void* K;
  float2* rowstat; double* colsum; double* bandcol;
  int U, n, d, w;
  int stride;  // tokens from one unit to the next (of Q, K and all sums)
  int G;  // query heads per K/V unit: Q and rowstat hold U * G units
  float scale;
};

struct fg_select_args {
  double* colsum; const double* bandcol; const uint8_t* token_class;  // [B, n]
  uint8_t* keep; int32_t* slot;
  int32_t* policy; double* recov; int32_t* kcount; int32_t* cap; int32_t* len;
  int32_t* policy_out; double* recov_out; int32_t* kcount_out;  // optional caller copies
  int U, n, units_per_seq, w, S, G;
  double T, r_f;
  int forced_policy;
  int family[4];  // FG_COMP_* mask of policy ids 0..3 (0 = unused id)
};
// Where both sums still lie in parts [parts, U, n], of the selection that adds them alone: in fg_select_args they cost the others
// 0.2 of 7 us (in its middle 0.4), whose block size lies behind the arguments and then on one line more of them.
struct fg_part_sums { const double* col; const double* band; int parts; };
static_assert(sizeof(fg_select_args) + 8 + 16 <= 3 * 64, "a fourth line of arguments");

struct fg_compact_args {
  const void* K; const void* V;
  const double* colsum; const uint8_t* keep; const int32_t* slot;   // keep: 0, or 4 | class bits
  const int32_t* cap; int64_t* off; const int32_t* len; int32_t* flags;
  void* ck; void* cv; double* cscore; int32_t* cpos; uint8_t* ccls;
  int U, n, d, esize, units_per_seq;
  int64_t pool_tokens;
};

struct fg_decode_args {
  const void* q; const void* k_new; const void* v_new; const uint8_t* class_new; void* out;
  const int32_t* policy; const int32_t* cap; const int64_t* off; int32_t* len; int32_t* flags;
  void* ck; void* cv; double* cscore; int32_t* cpos; uint8_t* ccls; double* clogit;
  const int32_t* chunk_off; int32_t* item_unit; float* part;
  int U, n, d, dtype, units_per_seq, w, step, G;
  int family[4];   // FG_COMP_* mask of policy ids 0..3 (stability probe)
  double* probe;   // NULL, or [U, 5]: this step's attention mass on every family member
  double r_f;
  float scale;
  int64_t max_chunks;
  int chunk;       // tokens per work item (128 or 256)
  int unit_threads; // workgroup size of the one-workgroup-per-unit form
  int update_threads; // workgroup size of the update kernel of the split form
};

struct fg_export_args {
  const int64_t* off; const int32_t* len; const int32_t* flags;
  const void* ck; const void* cv; const double* cscore; const int32_t* cpos;
  int32_t* lengths; int64_t* offsets; int32_t* positions; double* scores; void* keys; void* values;
  int32_t* status;
  int U, d, esize, max_pos;  // max_pos = n + S
};

hipError_t fg_launch_profile_bf16(const fg_profile_args&, int pass, int from, hipStream_t);
// (several workgroups per unit leave their sums in `part_sums`: of the columns [parts, U, n or 1024], then of the band)
hipError_t fg_launch_profile_once(const fg_profile_args&, fg_once_form, double* part_sums, hipStream_t);
// sums over [parts, U, cols] in order, of two arrays, into [U, stride]
hipError_t fg_launch_part_sums(const double* pcol, const double* pband, double* col, double* band, int U, int cols, int stride, int parts, hipStream_t);
hipError_t fg_launch_profile_f32(const fg_profile_args&, int pass, hipStream_t);
hipError_t fg_launch_profile_once_f32(const fg_profile_args&, int parts, double* part_sums, hipStream_t);
hipError_t fg_launch_lse_to_rowstat(const float* lse_nat, float2* rowstat, size_t count, hipStream_t);
constexpr int FG_MAX_CLASS_IDS = 64;  // ids per list of fastgen_classify (passed by value)
struct fg_classify_args {
  const int32_t* token_ids; uint8_t* token_class; long long count;
  int num_special, num_punct;
  int32_t special[FG_MAX_CLASS_IDS], punct[FG_MAX_CLASS_IDS];
};
hipError_t fg_launch_classify(const fg_classify_args&, hipStream_t);
hipError_t fg_launch_select(const fg_select_args&, const fg_part_sums&, hipStream_t);   // parts = 1: the sums are whole
hipError_t fg_launch_compact(const fg_compact_args&, hipStream_t);
hipError_t fg_launch_offsets(const int32_t* cap, const int32_t* len, const int32_t* policy, int64_t* off,
                             int32_t* chunk_off, int32_t* item_unit, int32_t* flags, int U, int64_t pool_tokens,
                             int64_t max_chunks, int chunk, int max_cap, int row_bytes, bool by_unit, hipStream_t);
hipError_t fg_launch_decode_attn(const fg_decode_args&, hipStream_t);
hipError_t fg_launch_decode_update(const fg_decode_args&, hipStream_t);
hipError_t fg_launch_decode_unit(const fg_decode_args&, hipStream_t);
hipError_t fg_launch_decode_group(const fg_decode_args&, hipStream_t);
hipError_t fg_launch_decode_group_mfma(const fg_decode_args&, hipStream_t);
hipError_t fg_launch_export(const fg_export_args&, hipStream_t);
