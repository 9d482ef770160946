// Both profiling sweeps of a short bf16 prompt in one pass over Q and K (Alg. 1: A = softmax(Q K^T);
// Sec. 3.4 cumulative attention score; same outputs as the two sweeps of profile_mfma.hip).
//
// A workgroup walks the query rows of a unit in blocks of 64; where units are few, several workgroups share
// the blocks of each, dealt from the heavy end. The waves hold the whole block's exponentials in registers: the
// causal columns are dealt out in fragments of 32, fragment j to wave j mod NW, at most four per wave, so
// 4 * 32 * NW columns are the longest prompt. A value 2^(c q.k - m) is made once, with a shift m of its row that all
// waves share: from what the sum of the row 64 before came to, a whole number (fg_fits and below). No maximum is looked for, so a
// fragment's exponentials start with its last matrix instruction; whether the shift fits shows in the row's sum, and a
// block where one does not is done again with each wave's own maximum as its shift. The next block then starts with its own
// maxima if the shifts from before would not have fitted here either, and so does a workgroup's only block, which has
// none before it. The waves exchange the sums of the 64 rows through LDS, and the column sums take
// value / sum from the registers. One contraction and one exponential per score instead of two. Of the row statistics only
// those of longer prompts pass through memory: the sums of the columns behind the ones held here come from there, and the normalisers of
// the rows behind them and of a head's first 64 go back (for the second sweep over those columns). Workgroups that share a unit leave partial column sums, which are added in order.
//
// The row index is the lane index (Q is the B operand of v_mfma_f32_32x32x16_bf16), so row sums are
// private to a lane; the column sums cross the lanes once per block, after the block's two row fragments have been
// added (fg_cols_over_rows). A wave shares its keys with no other wave and waits for nobody's. Of its four fragments one
// stays in registers for the whole unit and one in LDS as the last one of a block and the first of the next; the other two
// take its place in LDS in turn, one ahead (d = 64: two in registers, two in LDS, each read once). The first two go
// through the matrix pipe together and share the reads of the query rows.
//
// Bound: two waves per SIMD in step. Per piece of 64 x 32 and wave, cycles, 16384 units of 1024 tokens, d = 128: 1010 of
// matrix instructions (512 alone), 885 of exponentials, 780 of column sums, and per block 680 for the exchange and 1500 at
// its barrier, where waves with a fragment less wait. 4096 units of 1024 tokens, d = 128, 1270 us with running maxima
// and all keys through LDS, 1154 with the row sums themselves for shifts (two sweeps 1586); of 512 385 -> 346, of 500, d = 64, 291 -> 254, 1024 of 1000, d =
// 64, 274 -> 241, 256 of 700, G = 4, 183 -> 157. The present shifts and a third float64 step take 1 to 3 % more than those (in turn, 1101 -> 1128,
// 308 -> 315, 229 -> 237, 217 -> 223, 137 -> 139). Heads whose rows never fit (60 powers of two up or down every 40 rows), with
// running maxima / so: 1024 of 1000 322 / 339, d = 64, 700 of 1000 191 / 207 (each block twice: 443 and 266), 256 of 2048 354 / 325. Relative error of a column sum against
// float64, running maxima / row sums for shifts / so: 512 units of 1000 tokens 1.85e-8 / 2.63e-8 / 1.92e-8, with queries a tenth as large 1.05e-8 / 1.97e-8 /
// 1.15e-8, three times 1.55e-7 / 1.59e-7 / 1.56e-7, 1000 of 512 in d = 64 2.01e-8 / 2.82e-8 / 1.96e-8, 50 of 435 2.42e-8 / 2.51e-8 / 2.31e-8; two
// float64 steps 2.03e-8, 1.34e-8, 1.56e-7, 2.15e-8, 2.47e-8. Tried without gain: all keys in registers with 32
// rows a block (1325) or 16 and the exchange under the next rows' products (1810), higher priority for half of the
// waves or for the matrix instructions (1115 to 1186 where 1114 without), keys for the registers straight from memory
// (1204 where 1154, and short prompts 0.6 us more), the first two fragments one by one in a first block (8 spills), the
// next block's first contraction under this one's column sums.
#include <type_traits>

#include "fg_common.h"
#include "fg_internal.h"

namespace {

constexpr int kFrag = 32;    // columns of a fragment
constexpr int kRows = 64;    // query rows of a block: two fragments
constexpr int kSlots = 4;    // fragments of a wave in one block: 128 registers
// Sums that row `row` may come to under the shift of the row 64 before, whose shift would have left the square root of its
// length (up to 2^6.5). An exponential's argument is rounded at its own size, beyond 16 by 2^-20 and more, which rows with a
// shift of their own do not pay (300 units of 500 tokens, exact products, rows 24 powers of two above the ones 64 before:
// accepted, column sums are 3.5e-7 off float64; redone, 4.2e-8). No argument is above its sum's power of two, and those of an even row
// lie below it by that of its length. A block done again costs 2 us, which few units cannot hide: with 2^-8 to 2^14 for all rows,
// products of 0 for a head's first shifts and each row's own sum for the next ones, one in three heads with favoured columns was
// (static calls of 50 units of 435 tokens 19.9 -> 22.1 us, 81 of 1023, d = 64, 38.0 -> 41.2; of 1110 such heads none is now, and the calls take 20.0 and 38.8).
__device__ __forceinline__ bool fg_fits(float sum, int row) { return sum >= (float)min(row + 1, 1024) * 0x1p-18f && sum <= 0x1p16f; }
constexpr float kFirstShift = 6.f;   // of a head's first block: a sum of 2^-12 (of one product) to 2^22 fits
constexpr float kBelowMost = 6.f;    // of the next one: no further below the largest, since a head's first rows are short

// 16 bytes per lane from memory straight into LDS, to `lds` + 16 * lane. Written out, because behind the builtin the
// compiler waits for the data at the next read of any LDS; here the waits below do, which every reader stands behind.
__device__ __forceinline__ void fg_load_lds16(__amdgpu_buffer_rsrc_t r, const void* lds, int voff, int soff) {
#ifdef __HIP_DEVICE_COMPILE__
  const unsigned at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)lds;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(__builtin_amdgcn_readfirstlane(at)), "v"(voff), "s"(r), "s"(soff) : "memory");   // (m0 holds nothing of the compiler's)
#endif
}
__device__ __forceinline__ void fg_load_lds4(__amdgpu_buffer_rsrc_t r, const void* lds, int voff, int soff) {   // 4 bytes per lane
#ifdef __HIP_DEVICE_COMPILE__
  const unsigned at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)lds;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               :: "s"(__builtin_amdgcn_readfirstlane(at)), "v"(voff), "s"(r), "s"(soff) : "memory");
#endif
}
__device__ __forceinline__ void fg_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }        // this wave's loads
__device__ __forceinline__ void fg_have_read() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }   // its LDS reads
__device__ __forceinline__ void fg_barrier() {   // all waves' loads and LDS accesses
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// a: the lower halves of both, b: the upper halves
__device__ __forceinline__ void fg_swap_halves(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void fg_swap_halves(double& a, double& b) {
  float al = __int_as_float(__double2loint(a)), ah = __int_as_float(__double2hiint(a));
  float bl = __int_as_float(__double2loint(b)), bh = __int_as_float(__double2hiint(b));
  fg_swap_halves(al, bl);
  fg_swap_halves(ah, bh);
  a = __hiloint2double(__float_as_int(ah), __float_as_int(al));
  b = __hiloint2double(__float_as_int(bh), __float_as_int(bl));
}

// 16 values per lane (columns) summed over the 32 lanes of its half (rows), in a fixed order. Every step
// halves the values a lane still carries: it ends with the sum of column number b4 b3 b2 b1 (bits of the lane).
// The last two steps run in float64: they would otherwise hold three quarters of the rounding of a 64-row sum. With THIRD the
// step before does, too: it holds half of the rest. Prompts beyond 1024 tokens go without, which saves 1 % of their
// profile: their column sums are closer to float64 than those of two sweeps either way (256 units of 2048 tokens, two
// sweeps / without / with: 1.47e-8, 1.15e-8, 1.06e-8).
template <bool THIRD>
__device__ __forceinline__ double fg_cols_over_rows(const float (&t)[16], int lane) {
  float a[8], b[4], f[2];
  double c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(t[i]), __float_as_uint(t[i + 8]), false, false);
    a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0, b1 = (lane & 2) != 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = (b3 ? a[i + 4] : a[i]) + fg_dpp<FG_DPP_MIRROR>(b3 ? a[i] : a[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b2 ? b[i + 2] : b[i], other = fg_dpp<FG_DPP_HALF_MIRROR>(b2 ? b[i] : b[i + 2]);
    if (THIRD) c[i] = (double)keep + (double)other;
    else f[i] = keep + other;
  }
  const double d = THIRD ? (b1 ? c[1] : c[0]) + fg_dpp_f64<FG_DPP_XOR2>(b1 ? c[0] : c[1])
                         : (double)(b1 ? f[1] : f[0]) + (double)fg_dpp<FG_DPP_XOR2>(b1 ? f[0] : f[1]);
  return d + fg_dpp_f64<FG_DPP_XOR1>(d);
}

// offset of accumulator i of a lane within its 32 items (matrix instruction layout, without the half's 4)
constexpr __device__ int fg_acc_item(int i) { return (i >> 2) * 8 + (i & 3); }

template <int D, int NW, bool LONG>
__global__ __launch_bounds__(NW * 64, 2) void fg_profile_once_kernel(
    const __bf16* __restrict__ Q, const __bf16* __restrict__ K, float2* rowstat, double* __restrict__ colsum,
    double* __restrict__ bandcol, int U, int n, int w, float c, int G, int P) {   // (64 bytes of arguments, one line)
  constexpr int KK = D / 16;
  constexpr int RB = D * 2;           // bytes of a row
  constexpr int PPR = D / 8;          // 16-byte pieces of a row
  constexpr int RPL = 1024 / RB;      // rows of one load of the wave (1 KiB)
  constexpr int NT = NW * 64;
  constexpr int QL = kRows * RB / 1024 / NW;   // loads of a row block per wave
  constexpr int KL = kFrag * RB / 1024;        // loads of a fragment of keys
  constexpr int COLS = kSlots * kFrag * NW;
  constexpr int HELD = 128 / D;       // fragments of a wave in registers, and as many in LDS
  constexpr auto in_registers = [](int p) { return p == 1 || (HELD == 2 && p == 2); };
  constexpr auto register_of = [](int p) { return HELD == 2 && p == 2 ? 1 : 0; };
  // Piece p of row r lies at place p ^ (r mod PPR): the lanes of a fragment, one row each, read different banks.
  __shared__ __attribute__((aligned(16))) unsigned char s_q[2][kRows * RB];
  __shared__ __attribute__((aligned(16))) unsigned char s_k[NW][HELD][kFrag * RB];
  __shared__ double s_l[2][NW][kRows];
  __shared__ float s_m[2][NW][kRows];
  __shared__ float2 s_x[2][LONG ? kRows : 1];   // of the columns beyond, per row: a whole number for its shift, and its sum less FG_ROW_SUM_LESS
  __shared__ double s_sum[2][COLS];   // column sums, and their part inside the band

  // parts of one unit on one XCD (its L2 then serves the keys)
  const int idx = blockIdx.x, xcd = idx & 7, rest = idx >> 3;
  const int unit = (rest / P) * 8 + xcd, part = rest % P;
  if (unit >= U) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int nblk = (n + kRows - 1) / kRows;
  for (int i = tid; i < 2 * COLS; i += NT) (&s_sum[0][0])[i] = 0.0;
  // blocks dealt out by weight from the heaviest, to the parts down, up, ...; walked from the lightest
  auto block = [&](int i) { return nblk - 1 - ((i & 1) ? (i + 1) * P - 1 - part : i * P + part); };
  int mine = 1;   // at most nblk parts
  while (block(mine) >= 0) ++mine;

  // the loads write LDS in lane order, so a lane picks the piece that belongs to its place; rows past the end of
  // the unit read as zeros (every use of them is masked)
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<__bf16*>(K + (size_t)unit * n * D), 0, n * RB, 0x00020000);
  const int lrow = lane / PPR, lplace = lane % PPR;
  auto source = [&](int load) { return lrow * RB + ((lplace ^ lrow ^ (load * RPL)) & (PPR - 1)) * 16; };
  auto load_k = [&](int slot, int to) {
#pragma unroll
    for (int i = 0; i < KL; ++i)
      fg_load_lds16(k_rsrc, &s_k[wave][to][i * 1024], source(i), (wave + NW * slot) * kFrag * RB + i * 1024);
  };
  const int frag = ln * RB + ((lh ^ ln) & (PPR - 1)) * 16;   // piece 2 kk + lh of row ln: frag ^ (32 kk)
  const int item = ((lane >> 4) & 1) * 16 + ((lane >> 3) & 1) * 8 + lh * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
  bf16x8 kf[HELD][KK];
  // (by LDS: from memory into the operands' registers, 32 cache lines an instruction, cost a short prompt 0.6 us)
#pragma unroll
  for (int s = 0; s < HELD; ++s) load_k(s, s);
  const int most = min(kSlots, ((n - 1) / kFrag - wave) / NW + 1);   // fragments of this wave in the last block (or below 1)
  int buf = 0, held = 1;   // the fragment in s_k (d = 128)
  for (int h = 0; h < G; ++h) {   // the query heads of the unit, one after the other over the same columns
    const __amdgpu_buffer_rsrc_t q_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(Q + ((size_t)unit * G + h) * n * D), 0, n * RB, 0x00020000);
    float2* stat = rowstat + ((size_t)unit * G + h) * n;
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(stat, 0, n * 8, 0x00020000);
    auto load_q = [&](int b, int to) {
#pragma unroll
      for (int i = 0; i < QL; ++i)
        fg_load_lds16(q_rsrc, &s_q[to][(wave * QL + i) * 1024], source(wave * QL + i), b * kRows * RB + (wave * QL + i) * 1024);
      if (LONG && wave < 2) fg_load_lds4(x_rsrc, &s_x[to][wave * kRows / 2], lane * 4, b * kRows * 8 + wave * kRows * 4);
    };
    load_q(block(mine - 1), buf);   // the last reads of this buffer lie behind a barrier
    fg_barrier();
    if (h == 0) {
#pragma unroll
      for (int s = 0; s < HELD; ++s)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) kf[s][kk] = *reinterpret_cast<const bf16x8*>(&s_k[wave][s][frag ^ (32 * kk)]);
      fg_have_read();
      if (most > HELD) load_k(HELD, 0);
      if (most > 3 && HELD == 2) load_k(3, 1);
    }
    float m_run[2] = {kFirstShift, kFirstShift};   // the shifts of this lane's rows, the same in all waves
    bool own = mine == 1;          // the next block starts with each wave's own maxima
    for (int i = mine - 1; i >= 0; --i, buf ^= 1) {
      const int b = block(i);
      const int r0 = b * kRows;
      const int jl = min(2 * b + 1, (n - 1) / kFrag);   // last column fragment
      const int cnt = jl >= wave ? min((jl - wave) / NW + 1, kSlots) : 0;   // fragments of this wave
      // (read before a barrier of the block: behind the last one the next block's load_q writes there)
      auto beyond = [&]() { return LONG && r0 >= COLS && r0 + lane < n ? s_x[buf][lane] : make_float2(FG_NEG_BIG, 0.f); };
      if (i > 0) load_q(block(i - 1), buf ^ 1);
      f32x16 e[kSlots][2];
      int at[kSlots];        // the fragments' slots
      double l_run[2];
      auto active = [&](int p) { return HELD == 1 ? cnt > (p == 0 ? 1 : p == 1 ? 0 : p) : cnt > at[p]; };
      // a fragment's products: MODE 0 become exponentials, with their sums over the row; MODE 1 give the rows' largest values
      auto rows = [&](auto md, int p) __attribute__((always_inline)) {
        constexpr int MODE = decltype(md)::value;
        auto half = [&](f32x16& ac, int f, bool diagonal) __attribute__((always_inline)) {
          const int lim = diagonal ? ln - lh * 4 : 32;   // column <= row
          float s[4];
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const bool ok = !diagonal || fg_acc_item(i) <= lim;
            if (MODE == 1) {   // (c > 0: the largest product gives the largest logit)
              const float x = ok ? ac[i] : -INFINITY;
              s[i & 3] = i < 4 ? x : fmaxf(s[i & 3], x);
            } else {
              const float v = fg_exp2(fmaf(ac[i], c, -m_run[f]));
              ac[i] = ok ? v : 0.f;
              s[i & 3] = i < 4 ? ac[i] : s[i & 3] + ac[i];
            }
          }
          if (MODE == 1) m_run[f] = fmaxf(m_run[f], fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c);
          else l_run[f] += (double)((s[0] + s[1]) + (s[2] + s[3]));
        };
        const int j = wave + NW * at[p];
        if (j < 2 * b) {
          half(e[p][0], 0, false);
          half(e[p][1], 1, false);
        } else if (j == 2 * b) {
          half(e[p][0], 0, true);
          half(e[p][1], 1, false);
        } else {   // above the diagonal for the first row fragment
#pragma unroll
          for (int i = 0; i < 16; ++i) e[p][0][i] = 0.f;
          half(e[p][1], 1, true);
        }
      };
      // the fragments' contractions, each followed by its rows
      auto sweep = [&](auto md) __attribute__((always_inline)) {
        // d = 128: the fragment in LDS, the one in registers, the others through LDS in turn; d = 64: all are at hand
        auto next = [&](int s) { return s >= cnt - 1 ? 1 : s + 1; };
        at[0] = HELD == 1 ? (held < cnt ? held : 1) : 2;
        at[1] = 0;
        at[2] = HELD == 1 ? next(at[0]) : 1;
        at[3] = HELD == 1 ? next(at[2]) : 3;
        // matrix instructions of one or two fragments, the operand reads three steps ahead of them
        auto contract = [&](auto first, auto second) __attribute__((always_inline)) {
          constexpr int pa = decltype(first)::value, pb = decltype(second)::value;   // second: none below 0
          constexpr bool ra = in_registers(pa), rb = pb < 0 || in_registers(pb);
          constexpr int reads = 2 + (ra ? 0 : 1) + (rb ? 0 : 1), AHEAD = 3;
          const unsigned char* ka = s_k[wave][HELD == 2 && pa == 3 ? 1 : 0];
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              e[pa][f][i] = 0.f;
              if (pb >= 0) e[pb & 3][f][i] = 0.f;
            }
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            const bf16x8 a = ra ? kf[register_of(pa)][kk] : *reinterpret_cast<const bf16x8*>(ka + (frag ^ (32 * kk)));
            const bf16x8 q0 = *reinterpret_cast<const bf16x8*>(&s_q[buf][frag ^ (32 * kk)]);
            const bf16x8 q1 = *reinterpret_cast<const bf16x8*>(&s_q[buf][32 * RB + (frag ^ (32 * kk))]);
            e[pa][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, q0, e[pa][0], 0, 0, 0);
            e[pa][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, q1, e[pa][1], 0, 0, 0);
            if (pb >= 0) {
              const bf16x8 o = kf[register_of(pb & 3)][kk];
              e[pb & 3][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o, q0, e[pb & 3][0], 0, 0, 0);
              e[pb & 3][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o, q1, e[pb & 3][1], 0, 0, 0);
            }
          }
          __builtin_amdgcn_sched_group_barrier(0x100, reads * AHEAD, 0);
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            __builtin_amdgcn_sched_group_barrier(0x8, pb < 0 ? 2 : 4, 0);
            if (kk + AHEAD < KK) __builtin_amdgcn_sched_group_barrier(0x100, reads, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        const std::integral_constant<int, -1> none;
        const std::integral_constant<int, 0> p0;
        const std::integral_constant<int, 1> p1;
        const std::integral_constant<int, 2> p2;
        const std::integral_constant<int, 3> p3;
        if (HELD == 1) {
          if (cnt > 1) {
            if (held != at[0]) load_k(at[0], 0);
            if (held != at[0] || i == mine - 1) fg_landed();   // (else it has landed before the last barrier)
            contract(p0, p1);
            held = at[0];
            if (cnt > 2) load_k(at[2], 0);   // the keys have been read: the next fragment takes their place
            rows(md, 0);
            rows(md, 1);
          } else if (cnt > 0) {
            contract(p1, none);
            rows(md, 1);
          }
          if (cnt > 2) {
            fg_landed();
            contract(p2, none);
            held = at[2];
            if (cnt > 3) load_k(at[3], 0);
            rows(md, 2);
          }
          if (cnt > 3) {
            fg_landed();
            contract(p3, none);
            held = at[3];
            rows(md, 3);
          }
        } else {
          if (cnt > 1) {
            contract(p2, p1);
            rows(md, 2);
            rows(md, 1);
          } else if (cnt > 0) {
            contract(p1, none);
            rows(md, 1);
          }
          if (cnt > 2) {
            if (i == mine - 1) fg_landed();
            contract(p0, none);
            rows(md, 0);
          }
          if (cnt > 3) {
            contract(p3, none);
            rows(md, 3);
          }
        }
      };
      // sums of row `lane` of the block: the halves of the wave (columns), then the waves
      auto put_sums = [&]() __attribute__((always_inline)) {
        double la = l_run[0], lb = l_run[1];
        fg_swap_halves(la, lb);
        s_l[buf][wave][lane] = la + lb;
      };
      double L = 0.0;
      const float given = lh ? m_run[1] : m_run[0];
      float M = given, share = 1.f;
      l_run[0] = l_run[1] = 0.0;
      bool again = own;
      if (!again) {
        sweep(std::integral_constant<int, 0>());
        put_sums();
        const float2 x = beyond();
        fg_barrier();
#pragma unroll
        for (int i = 0; i < NW; ++i) L += s_l[buf][i][lane];
        if (LONG) L = fma((double)x.y + FG_ROW_SUM_LESS, (double)fg_exp2(x.x - M), L);
        again = __any(r0 + lane < n && !fg_fits((float)L, r0 + lane));   // the same in all waves
        if (again) fg_barrier();   // s_l has been read
      }
      if (again) {   // the shifts do not fit, or hardly will, or there are none: this wave's own
        m_run[0] = m_run[1] = FG_NEG_BIG;
        sweep(std::integral_constant<int, 1>());
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          float o = m_run[f];
          fg_swap_halves(m_run[f], o);
          m_run[f] = rintf(fmaxf(m_run[f], o));
        }
        l_run[0] = l_run[1] = 0.0;
#pragma unroll
        for (int p = 0; p < kSlots; ++p)
          if (active(p)) rows(std::integral_constant<int, 0>(), p);
        put_sums();
        const float wave_m = lh ? m_run[1] : m_run[0];
        s_m[buf][wave][lane] = wave_m;
        const float2 x = beyond();
        fg_barrier();
        float mv[NW];
        M = x.x;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          mv[i] = s_m[buf][i][lane];
          M = fmaxf(M, mv[i]);
        }
        L = LONG ? ((double)x.y + FG_ROW_SUM_LESS) * (double)fg_exp2(x.x - M) : 0.0;
#pragma unroll
        for (int i = 0; i < NW; ++i) L = fma(s_l[buf][i][lane], (double)fg_exp2(mv[i] - M), L);
        share = fg_exp2(wave_m - M);
        // as far as this block tells; a head's first block, whose shifts are no row's, tells nothing
        own = mine == 1 || (i < mine - 1 && __any(r0 + lane < n && !fg_fits((float)(L * (double)fg_exp2(M - given)), r0 + lane)));
      }
      // The shifts of the next block: where these rows' sums would have been the square root of their length. What counts in
      // a row then lies on both sides of 0, be the row even (its terms would lie at -log2 n under the sum itself) or held
      // by few columns. (Its rows past the end stay at products of 0.)
      if (i > 0) {
        const float sum = (float)L * __builtin_amdgcn_rsqf((float)(r0 + lane + 1));
        float ma = M + rintf(__builtin_amdgcn_logf(sum));
        if (i == mine - 1) ma = fmaxf(ma, fg_wave_max(ma) - kBelowMost);
        if (block(i - 1) * kRows + lane >= n) ma = 0.f;
        float mb = ma;
        fg_swap_halves(ma, mb);
        m_run[0] = ma;
        m_run[1] = mb;
      }
      double inv = __builtin_amdgcn_rcp(L);
      inv = fma(inv, fma(-L, inv, 1.0), inv);
      // for the second sweep behind the columns held here, whose last tile of a head runs on into the next head's first rows
      if (LONG && wave == 0 && (r0 >= COLS || r0 == 0) && r0 + lane < n) stat[r0 + lane] = make_float2(M, (float)inv);
      float f0 = r0 + lane < n ? (float)inv * share : 0.f, f1 = f0;   // rows past the end count nothing
      fg_swap_halves(f0, f1);
#pragma unroll
      for (int p = 0; p < kSlots; ++p) {
        if (!active(p)) continue;
        const int j = wave + NW * at[p];
        const int d0 = r0 - j * kFrag;   // row - column of the fragment's corner
        const int to = j * kFrag + item;
        float t[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = fmaf(e[p][1][i], f1, e[p][0][i] * f0);
        // one wave adds to a column, in the order of the blocks; odd lanes carry the band
        const bool inside = d0 + 63 < w, outside = d0 - 31 >= w;
        const double v = fg_cols_over_rows<!LONG>(t, lane);
        if (!(lane & 1) || inside) unsafeAtomicAdd(&s_sum[lane & 1][to], v);
        if (!inside && !outside) {
          const int o0 = d0 + ln - lh * 4 - w;   // in the band: row - column < w, so the item's offset is above o0
          if (d0 + 1 >= w) {          // the second row fragment lies outside
#pragma unroll
            for (int i = 0; i < 16; ++i) t[i] = (fg_acc_item(i) > o0 ? e[p][0][i] : 0.f) * f0;
          } else if (d0 + 31 < w) {   // the first one inside
#pragma unroll
            for (int i = 0; i < 16; ++i) t[i] = fmaf(fg_acc_item(i) > o0 + 32 ? e[p][1][i] : 0.f, f1, e[p][0][i] * f0);
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i)
              t[i] = fmaf(fg_acc_item(i) > o0 + 32 ? e[p][1][i] : 0.f, f1, (fg_acc_item(i) > o0 ? e[p][0][i] : 0.f) * f0);
          }
          const double vb = fg_cols_over_rows<!LONG>(t, lane);
          if (lane & 1) unsafeAtomicAdd(&s_sum[1][to], vb);
        }
      }
    }
  }
  __syncthreads();
  const int stride = P > 1 ? min(n, FG_ONCE_TOKENS) : n;   // part sums are dense
  for (int i = tid; i < min(n, COLS); i += NT) {
    colsum[((size_t)part * U + unit) * stride + i] = s_sum[0][i];
    bandcol[((size_t)part * U + unit) * stride + i] = s_sum[1][i];
  }
}

// Prompts of a single block, up to 64 tokens: three waves take a tile of 32 rows and 32 columns each (the fourth only loads), with
// the tile's own row maxima for shifts. Bound: latency, so what counts is the one chain of load, matrix instructions, maxima,
// exponentials, exchange and column sums; in the kernel above it held the keys' way into registers, both row fragments one after
// the other and a second pass over the products. A call, with running maxima in one wave per 32 columns / in the kernel above / so:
// 4 units of 64 tokens, d = 128, 11.1 / 11.7 / 10.2 us, 4096 59.8 / 60.0 / 46.5, 4096 of 33, d = 64, 53 / 55 / 33, 300 of 64, G = 5,
// 26.6 / 27.3 / 19.2, 16000 of 64, d = 64, 200 / 202 / 113 (76 registers and 53 KB of LDS leave three to a CU).
template <int D>
__global__ __launch_bounds__(256) void fg_profile_block_kernel(
    const __bf16* __restrict__ Q, const __bf16* __restrict__ K, double* __restrict__ colsum, double* __restrict__ bandcol,
    int n, int w, float c, int G) {
  constexpr int KK = D / 16, RB = D * 2, PPR = D / 8, RPL = 1024 / RB;
  constexpr int LOADS = kRows * RB / 1024 / 4;   // per wave and matrix
  __shared__ __attribute__((aligned(16))) unsigned char s_q[2][kRows * RB];   // laid out as above
  __shared__ __attribute__((aligned(16))) unsigned char s_k[kRows * RB];
  __shared__ double s_l[2][4][32], s_sum[4][2][32];
  __shared__ float s_m[2][4][32];
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int lrow = lane / PPR, lplace = lane % PPR;
  auto load = [&](const __bf16* from, unsigned char* to) {   // rows past the end read as zeros
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(from), 0, n * RB, 0x00020000);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int at = wave * LOADS + i;
      fg_load_lds16(rsrc, to + at * 1024, lrow * RB + ((lplace ^ lrow ^ (at * RPL)) & (PPR - 1)) * 16, at * 1024);
    }
  };
  const int tr = wave > 0, tc = wave == 2;   // the wave's tile: (0, 0), (1, 0), (1, 1)
  const bool active = wave < 3 && tr * 32 < n;
  const int frag = ln * RB + ((lh ^ ln) & (PPR - 1)) * 16;
  const int row = tr * 32 + ln, d0 = (tr - tc) * 32;
  const bool inside = d0 + 31 < w, outside = d0 - 31 >= w;
  double sum = 0.0;   // of column tc * 32 + item; odd lanes carry the band
  load(Q + (size_t)unit * G * n * D, s_q[0]);
  load(K + (size_t)unit * n * D, s_k);
  fg_barrier();
  for (int h = 0, buf = 0; h < G; ++h, buf ^= 1) {
    if (h + 1 < G) load(Q + ((size_t)unit * G + h + 1) * n * D, s_q[buf ^ 1]);   // read last before the barrier of the head before
    f32x16 ac;
    float m = FG_NEG_BIG;
    double l = 0.0;
    if (active) {
#pragma unroll
      for (int i = 0; i < 16; ++i) ac[i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&s_k[tc * 32 * RB + (frag ^ (32 * kk))]);
        const bf16x8 q = *reinterpret_cast<const bf16x8*>(&s_q[buf][tr * 32 * RB + (frag ^ (32 * kk))]);
        ac = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, q, ac, 0, 0, 0);
      }
      const int lim = tr == tc ? ln - lh * 4 : 32;   // column <= row
      float s[4];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float x = fg_acc_item(i) <= lim ? ac[i] : -INFINITY;
        s[i & 3] = i < 4 ? x : fmaxf(s[i & 3], x);
      }
      m = fmaxf(FG_NEG_BIG, fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c);
      float o = m;
      fg_swap_halves(m, o);
      m = rintf(fmaxf(m, o));
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float e = fg_exp2(fmaf(ac[i], c, -m));
        ac[i] = fg_acc_item(i) <= lim ? e : 0.f;
        s[i & 3] = i < 4 ? ac[i] : s[i & 3] + ac[i];
      }
      l = (double)((s[0] + s[1]) + (s[2] + s[3]));
      double lo = l;
      fg_swap_halves(l, lo);
      l += lo;
      if (lh == 0) { s_m[buf][wave][ln] = m; s_l[buf][wave][ln] = l; }
    }
    fg_barrier();
    if (active) {
      float M = m;
      double L = l;
      if (tr) {   // the row's other tile
        const float mo = s_m[buf][3 - wave][ln];
        M = fmaxf(m, mo);
        L = fma(s_l[buf][3 - wave][ln], (double)fg_exp2(mo - M), l * (double)fg_exp2(m - M));
      }
      double inv = __builtin_amdgcn_rcp(L);
      inv = fma(inv, fma(-L, inv, 1.0), inv);
      const float f = row < n ? (float)inv * fg_exp2(m - M) : 0.f;   // rows past the end count nothing
      float t[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) t[i] = ac[i] * f;
      const double v = fg_cols_over_rows<true>(t, lane);
      if (!(lane & 1) || inside) sum += v;
      if (!inside && !outside) {
        const int o0 = d0 + ln - lh * 4 - w;   // in the band: row - column < w, so the item's offset is above o0
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = fg_acc_item(i) > o0 ? t[i] : 0.f;
        const double vb = fg_cols_over_rows<true>(t, lane);
        if (lane & 1) sum += vb;
      }
    }
  }
  const int item = ((lane >> 4) & 1) * 16 + ((lane >> 3) & 1) * 8 + lh * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
  s_sum[wave][lane & 1][item] = sum;   // 0 where the wave has no tile
  __syncthreads();
  const int which = tid >> 6, col = tid & 63;
  if (which < 2 && col < n) {
    const int o = col & 31;
    (which ? bandcol : colsum)[(size_t)unit * n + col] = col < 32 ? s_sum[0][which][o] + s_sum[1][which][o] : s_sum[2][which][o];
  }
}

template <int D>
hipError_t launch_block(const fg_profile_args& a, hipStream_t s) {
  hipLaunchKernelGGL((fg_profile_block_kernel<D>), dim3((unsigned)a.U), dim3(256), 0, s, static_cast<const __bf16*>(a.Q),
                     static_cast<const __bf16*>(a.K), a.colsum, a.bandcol, a.n, a.w, a.scale * FG_LOG2E, a.G);
  return hipGetLastError();
}

template <int D, int NW, bool LONG>
hipError_t launch(const fg_profile_args& a, int P, double* parts, hipStream_t s) {
  const int cols = a.n < FG_ONCE_TOKENS ? a.n : FG_ONCE_TOKENS;
  const size_t N = (size_t)a.U * cols;
  double* col = P > 1 ? parts : a.colsum;
  double* band = P > 1 ? parts + P * N : a.bandcol;
  hipLaunchKernelGGL((fg_profile_once_kernel<D, NW, LONG>), dim3((unsigned)(8 * P * ((a.U + 7) / 8))), dim3(NW * 64), 0, s,
                     static_cast<const __bf16*>(a.Q), static_cast<const __bf16*>(a.K), a.rowstat, col, band, a.U, a.n,
                     a.w, a.scale * FG_LOG2E, a.G, P);
  return hipGetLastError();
}

}  // namespace

hipError_t fg_launch_profile_once(const fg_profile_args& a, fg_once_form f, double* parts, hipStream_t s) {
  if ((a.n > kSlots * kFrag * f.waves && f.waves != 8) || f.parts > (a.n + kRows - 1) / kRows) return hipErrorInvalidValue;
  if (a.n <= kRows) return a.d == 128 ? launch_block<128>(a, s) : launch_block<64>(a, s);
  if (a.n > FG_ONCE_TOKENS) return a.d == 128 ? launch<128, 8, true>(a, f.parts, parts, s) : launch<64, 8, true>(a, f.parts, parts, s);
  if (f.waves == 8) return a.d == 128 ? launch<128, 8, false>(a, f.parts, parts, s) : launch<64, 8, false>(a, f.parts, parts, s);
  return a.d == 128 ? launch<128, 4, false>(a, f.parts, parts, s) : launch<64, 4, false>(a, f.parts, parts, s);
}
