// Both profiling sweeps of a short bf16 prompt in one pass over Q and K (Alg. 1: A = softmax(Q K^T);
// Sec. 3.4 cumulative attention score; same outputs as the two sweeps of profile_mfma.hip).
//
// A workgroup walks the query rows of a unit in blocks of 64; where units are few, several workgroups share
// the blocks of each, dealt from the heavy end. The waves hold the whole block's exponentials in registers: the
// causal columns are dealt out in fragments of 32, fragment j to wave j mod NW, at most four per wave, so
// 4 * 32 * NW columns are the longest prompt. A value p~ = 2^(c q.k - m) is
// made once, with the running shift m of its row in this wave (a whole number, so that every later rescaling
// is a power of two); the waves then exchange (m, l) of the 64 rows through LDS, and the column sums
// take p~ * 2^(m - M) / l from the registers. One contraction and one exponential per score instead of two, and
// no row statistics in memory. Q is read once, the causal keys once per block of rows but for the fragment that each wave
// still holds. Workgroups that share a unit leave partial column sums, which are added in order.
//
// The row index is the lane index (Q is the B operand of v_mfma_f32_32x32x16_bf16), so row maxima and sums are
// private to a lane; the column sums cross the lanes once per block, after the block's two row fragments have been
// added (fg_cols_over_rows). The fragments of K arrive by loads that write LDS directly, one ahead: a
// wave shares its keys with no other wave and waits for nobody's. Straight from memory into operand registers they
// would touch 32 cache lines per instruction (as fast measured, but 32 registers more).
//
// Bound: two waves per SIMD, whose waits (41 % of their cycles: the block's barrier, and keys from beyond L2) neither
// the vector ALU (about half busy: 282 instructions per wave-step, the two sweeps 141 + 132) nor the matrix pipe covers.
// 16384 units of 1024 tokens, d = 128, fetch 24.6 GB for 8.6 GB of Q and K (two sweeps 25.6), 4.4 to 4.8 TB/s:
// the traffic is part of the bound. 4096 units of 1024 tokens, d = 128, 1586 us in two sweeps, 1324 in one pass
// (the walk back and forth: 100 us more without); of 512 tokens 542 -> 401. Error of the column sums against
// float64: 1.66e-8 (two sweeps 1.91e-8), the same when shared. 64 units of 1000 tokens by four workgroups each 25
// (one each 66, two sweeps 77). Tried without gain: the next fragment's matrix instructions between this
// one's exponentials by hand (1410: more instructions, the same time), two to eight workgroups per unit that share
// its keys in L2 (1420, and partial sums), query operands in registers (51 spills), the next block's first
// contraction under this one's column sums (3 % slower, 12 % with many workgroups per unit).
#include "fg_common.h"
#include "fg_internal.h"

namespace {

constexpr int kFrag = 32;    // columns of a fragment
constexpr int kRows = 64;    // query rows of a block: two fragments
constexpr int kSlots = 4;    // fragments of a wave in one block: 128 registers

// 16 bytes per lane from memory straight into LDS, to `lds` + 16 * lane
__device__ __forceinline__ void fg_load_lds16(__amdgpu_buffer_rsrc_t r, void* lds, int voff, int soff) {
#ifdef __HIP_DEVICE_COMPILE__   // the host pass does not know the 16-byte form
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, soff, 0, 0);
#endif
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
// The last two steps run in float64: they would otherwise hold three quarters of the rounding of a 64-row sum.
__device__ __forceinline__ double fg_cols_over_rows(const float (&t)[16], int lane) {
  float a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(t[i]), __float_as_uint(t[i + 8]), false, false);
    a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0, b1 = (lane & 2) != 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = (b3 ? a[i + 4] : a[i]) + fg_dpp<FG_DPP_MIRROR>(b3 ? a[i] : a[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = (b2 ? b[i + 2] : b[i]) + fg_dpp<FG_DPP_HALF_MIRROR>(b2 ? b[i] : b[i + 2]);
  const double d = (double)(b1 ? c[1] : c[0]) + (double)fg_dpp<FG_DPP_XOR2>(b1 ? c[0] : c[1]);
  return d + fg_dpp_f64<FG_DPP_XOR1>(d);
}

// offset of accumulator i of a lane within its 32 items (matrix instruction layout, without the half's 4)
constexpr __device__ int fg_acc_item(int i) { return (i >> 2) * 8 + (i & 3); }

template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void fg_profile_once_kernel(
    const __bf16* __restrict__ Q, const __bf16* __restrict__ K, double* __restrict__ colsum,
    double* __restrict__ bandcol, int U, int n, int w, float c, int G, int P) {
  constexpr int KK = D / 16;
  constexpr int RB = D * 2;           // bytes of a row
  constexpr int PPR = D / 8;          // 16-byte pieces of a row
  constexpr int RPL = 1024 / RB;      // rows of one load of the wave (1 KiB)
  constexpr int NT = NW * 64;
  constexpr int QL = kRows * RB / 1024 / NW;   // loads of a row block per wave
  constexpr int KL = kFrag * RB / 1024;        // loads of a fragment
  constexpr int COLS = kSlots * kFrag * NW;
  // Piece p of row r lies at place p ^ (r mod PPR): the lanes of a fragment, one row each, read different banks.
  __shared__ __attribute__((aligned(16))) unsigned char s_q[2][kRows * RB];
  __shared__ __attribute__((aligned(16))) unsigned char s_k[NW][kFrag * RB];
  __shared__ double s_l[2][NW][kRows];
  __shared__ float s_m[2][NW][kRows];
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
  auto load_k = [&](int j) {
#pragma unroll
    for (int i = 0; i < KL; ++i) fg_load_lds16(k_rsrc, &s_k[wave][i * 1024], source(i), j * kFrag * RB + i * 1024);
  };
  const int frag = ln * RB + ((lh ^ ln) & (PPR - 1)) * 16;   // piece 2 kk + lh of row ln: frag ^ (32 kk)
  const int item = ((lane >> 4) & 1) * 16 + ((lane >> 3) & 1) * 8 + lh * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);

  // The columns are walked upwards in one block and downwards in the next: a block begins with the keys that the one
  // before has read last. The first fragment is then still in LDS, and more of the others in the XCD's L2.
  int buf = 0, held = -1;   // the fragment in s_k
  bool down = false;
  for (int h = 0; h < G; ++h) {   // the query heads of the unit, one after the other over the same columns
    const __amdgpu_buffer_rsrc_t q_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(Q + ((size_t)unit * G + h) * n * D), 0, n * RB, 0x00020000);
    auto load_q = [&](int b, int to) {
#pragma unroll
      for (int i = 0; i < QL; ++i)
        fg_load_lds16(q_rsrc, &s_q[to][(wave * QL + i) * 1024], source(wave * QL + i), b * kRows * RB + (wave * QL + i) * 1024);
    };
    load_q(block(mine - 1), buf);   // the last reads of this buffer lie behind a barrier
    __syncthreads();
    for (int i = mine - 1; i >= 0; --i, buf ^= 1, down = !down) {
      const int b = block(i);
      const int r0 = b * kRows;
      const int jl = min(2 * b + 1, (n - 1) / kFrag);   // last column fragment
      const int cnt = jl >= wave ? (jl - wave) / NW + 1 : 0;   // fragments of this wave
      auto fragment = [&](int s) { return wave + NW * (down ? cnt - 1 - s : s); };
      if (cnt > 0 && fragment(0) != held) load_k(fragment(0));
      f32x16 e[kSlots][2];
      float ms[kSlots][2];   // the shifts that e holds
      float m_run[2] = {FG_NEG_BIG, FG_NEG_BIG};
      double l_run[2] = {0.0, 0.0};
      // exponentials of 16 dot products in place, row statistics carried on
      auto full = [&](f32x16& ac, int f) __attribute__((always_inline)) {
        const float x0 = fmaxf(fmaxf(ac[0], ac[1]), ac[2]), x1 = fmaxf(fmaxf(ac[3], ac[4]), ac[5]);
        const float x2 = fmaxf(fmaxf(ac[6], ac[7]), ac[8]), x3 = fmaxf(fmaxf(ac[9], ac[10]), ac[11]);
        const float x4 = fmaxf(fmaxf(ac[12], ac[13]), ac[14]);
        const float y0 = fmaxf(fmaxf(x0, x1), x2), y1 = fmaxf(fmaxf(x3, x4), ac[15]);
        const float m_new = fmaxf(rintf(fmaxf(y0, y1) * c), m_run[f]);
        float s[2];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          ac[i] = fg_exp2(fmaf(ac[i], c, -m_new));
          s[i & 1] = i < 2 ? ac[i] : s[i & 1] + ac[i];
        }
        l_run[f] = fma(l_run[f], (double)fg_exp2(m_run[f] - m_new), (double)(s[0] + s[1]));
        m_run[f] = m_new;
      };
      auto diagonal = [&](f32x16& ac, int f) __attribute__((always_inline)) {   // column <= row
        const int lim = ln - lh * 4;
        float tmax = FG_NEG_BIG;
#pragma unroll
        for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, fg_acc_item(i) <= lim ? ac[i] * c : FG_NEG_BIG);
        const float m_new = fmaxf(m_run[f], rintf(tmax));
        float s[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float p = fg_exp2(fmaf(ac[i], c, -m_new));
          ac[i] = fg_acc_item(i) <= lim ? p : 0.f;
          s[i & 1] += ac[i];
        }
        l_run[f] = fma(l_run[f], (double)fg_exp2(m_run[f] - m_new), (double)(s[0] + s[1]));
        m_run[f] = m_new;
      };
#pragma unroll
      for (int s = 0; s < kSlots; ++s) {
        if (s >= cnt) continue;
        const int j = fragment(s);
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int i = 0; i < 16; ++i) e[s][f][i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(&s_k[wave][frag ^ (32 * kk)]);
          const bf16x8 q0 = *reinterpret_cast<const bf16x8*>(&s_q[buf][frag ^ (32 * kk)]);
          const bf16x8 q1 = *reinterpret_cast<const bf16x8*>(&s_q[buf][32 * RB + (frag ^ (32 * kk))]);
          e[s][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, q0, e[s][0], 0, 0, 0);
          e[s][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, q1, e[s][1], 0, 0, 0);
        }
        // operand reads three steps ahead of the matrix instructions
        constexpr int AHEAD = 3;
        __builtin_amdgcn_sched_group_barrier(0x100, 3 * AHEAD, 0);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
          if (kk + AHEAD < KK) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        held = j;
        if (s + 1 < kSlots && s + 1 < cnt) load_k(fragment(s + 1));   // the keys have been read
        else if (i > 0) load_q(block(i - 1), buf ^ 1);   // (at the block's barrier, which waits for it: 3 to 5 % slower)
        if (j < 2 * b) {
          full(e[s][0], 0);
          full(e[s][1], 1);
        } else if (j == 2 * b) {
          diagonal(e[s][0], 0);
          full(e[s][1], 1);
        } else {   // above the diagonal for the first row fragment
#pragma unroll
          for (int i = 0; i < 16; ++i) e[s][0][i] = 0.f;
          diagonal(e[s][1], 1);
        }
        ms[s][0] = m_run[0];
        ms[s][1] = m_run[1];
      }
      if (cnt == 0 && i > 0) load_q(block(i - 1), buf ^ 1);
      // (m, l) of row `lane` of the block: the halves of the wave (columns), then the waves
      {
        float ma = m_run[0], mb = m_run[1];
        double la = l_run[0], lb = l_run[1];
        fg_swap_halves(ma, mb);
        fg_swap_halves(la, lb);
        const float mm = fmaxf(ma, mb);
        s_m[buf][wave][lane] = mm;
        s_l[buf][wave][lane] = fma(la, (double)fg_exp2(ma - mm), lb * (double)fg_exp2(mb - mm));
      }
      __syncthreads();
      float mv[NW], M = FG_NEG_BIG;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        mv[i] = s_m[buf][i][lane];
        M = fmaxf(M, mv[i]);
      }
      double L = 0.0;
#pragma unroll
      for (int i = 0; i < NW; ++i) L = fma(s_l[buf][i][lane], (double)fg_exp2(mv[i] - M), L);
      double inv = __builtin_amdgcn_rcp(L);
      inv = fma(inv, fma(-L, inv, 1.0), inv);
      float M0 = M, M1 = M, i0 = r0 + lane < n ? (float)inv : 0.f, i1 = i0;   // rows past the end count nothing
      fg_swap_halves(M0, M1);
      fg_swap_halves(i0, i1);
#pragma unroll
      for (int s = 0; s < kSlots; ++s) {
        if (s >= cnt) continue;
        const int j = fragment(s);
        const float f0 = fg_exp2(ms[s][0] - M0) * i0, f1 = fg_exp2(ms[s][1] - M1) * i1;
        const int d0 = r0 - j * kFrag;   // row - column of the fragment's corner
        const int at = j * kFrag + item;
        float t[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = fmaf(e[s][1][i], f1, e[s][0][i] * f0);
        // one wave adds to a column, in the order of the blocks; odd lanes carry the band
        const bool inside = d0 + 63 < w, outside = d0 - 31 >= w;
        const double v = fg_cols_over_rows(t, lane);
        if (!(lane & 1) || inside) unsafeAtomicAdd(&s_sum[lane & 1][at], v);
        if (!inside && !outside) {
          const int o0 = d0 + ln - lh * 4 - w;   // in the band: row - column < w, so the item's offset is above o0
          if (d0 + 1 >= w) {          // the second row fragment lies outside
#pragma unroll
            for (int i = 0; i < 16; ++i) t[i] = (fg_acc_item(i) > o0 ? e[s][0][i] : 0.f) * f0;
          } else if (d0 + 31 < w) {   // the first one inside
#pragma unroll
            for (int i = 0; i < 16; ++i) t[i] = fmaf(fg_acc_item(i) > o0 + 32 ? e[s][1][i] : 0.f, f1, e[s][0][i] * f0);
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i)
              t[i] = fmaf(fg_acc_item(i) > o0 + 32 ? e[s][1][i] : 0.f, f1, (fg_acc_item(i) > o0 ? e[s][0][i] : 0.f) * f0);
          }
          const double vb = fg_cols_over_rows(t, lane);
          if (lane & 1) unsafeAtomicAdd(&s_sum[1][at], vb);
        }
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < n; i += NT) {
    colsum[((size_t)part * U + unit) * n + i] = s_sum[0][i];
    bandcol[((size_t)part * U + unit) * n + i] = s_sum[1][i];
  }
}

template <int D, int NW>
hipError_t launch(const fg_profile_args& a, int P, double* parts, hipStream_t s) {
  const size_t N = (size_t)a.U * a.n;
  double* col = P > 1 ? parts : a.colsum;
  double* band = P > 1 ? parts + P * N : a.bandcol;
  hipLaunchKernelGGL((fg_profile_once_kernel<D, NW>), dim3((unsigned)(8 * P * ((a.U + 7) / 8))), dim3(NW * 64), 0, s,
                     static_cast<const __bf16*>(a.Q), static_cast<const __bf16*>(a.K), col, band, a.U, a.n, a.w,
                     a.scale * FG_LOG2E, a.G, P);
  return hipGetLastError();
}

}  // namespace

hipError_t fg_launch_profile_once(const fg_profile_args& a, fg_once_form f, double* parts, hipStream_t s) {
  if (a.n > kSlots * kFrag * f.waves || f.parts > (a.n + kRows - 1) / kRows) return hipErrorInvalidValue;
  if (f.waves == 8) return a.d == 128 ? launch<128, 8>(a, f.parts, parts, s) : launch<64, 8>(a, f.parts, parts, s);
  return a.d == 128 ? launch<128, 4>(a, f.parts, parts, s) : launch<64, 4>(a, f.parts, parts, s);
}
