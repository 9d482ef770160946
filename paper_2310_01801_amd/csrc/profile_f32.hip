// Prompt-time attention profiling for float32 inputs (Alg. 1: A = softmax(Q K^T); Sec. 3.4
// cumulative attention score). Same two sweeps and the same outputs as the bf16 matrix-core
// kernel. This path spends its time on accuracy: dot products, exponentials and sums in float64
// (products of two floats are exact there), only the stored row statistics (m, 1/l) are floats.
//
// The contraction runs on the float64 matrix instructions (16x16x4). One workgroup of 4 waves
// owns 16 items (query rows in pass 1, key columns in pass 2) as the B operand; its waves take
// the streamed tiles of 16 items in turn (tile t goes to wave t mod 4), each straight from global
// memory into registers, and merge their statistics once at the end in a fixed order. A wave that
// shares nothing with its neighbours needs neither LDS tiles nor barriers, and four waves per 16
// owners give a short prompt enough waves. The order of the contraction index is free, so lane
// group g (16 lanes) takes the contiguous quarter g of a row: full cache lines, 16-byte loads.
//
// Bound: the float64 matrix pipe. Measured: 64 units of 1000 tokens, d = 128: 228 + 223 us for the
// two sweeps (one thread per owner with a serial float64 chain on the vector ALU, as before: 1543 +
// 1620 us), 37.6 TFLOP/s where a register-only loop of the instruction reaches 40 to 43; 4 units of
// 128 tokens, d = 64: 8 + 5 us (79 + 81). Tried without effect: two accumulator chains, two owner
// fragments per wave (5 % slower), a shorter polynomial for 2^x.
#include "fg_common.h"
#include "fg_internal.h"

namespace {

constexpr int kTile = 16;   // streamed items per tile = rows of the matrix instruction
constexpr int kWaves = 4;

typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int D, int PASS>
__global__ __launch_bounds__(256, 2) void fg_profile_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, float2* __restrict__ rowstat,
    double* __restrict__ colsum, double* __restrict__ bandcol, int unit0, int U, int n, int w,
    float c, int nblk, int G) {
  constexpr int PL = D / 4;        // elements of a row per lane
  constexpr int LV = PL / 4;       // 16-byte loads per row and lane
  __shared__ double s_a[kWaves][16];
  __shared__ double s_b[kWaves][16];

  // blocks of one unit on one XCD (its L2 then serves the streamed rows), heaviest first
  const int idx = blockIdx.x;
  const int xcd = idx & 7, rest = idx >> 3;
  const int unit = unit0 + (rest / nblk) * 8 + xcd;
  if (unit >= U) return;
  const int ord = rest % nblk;
  const int blk = (PASS == 1) ? nblk - 1 - ord : ord;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 15, g = lane >> 4;
  const int O0 = blk * 16;   // first owner item
  // G query heads share a K/V unit: sweep 1 runs per query head (U counts query heads, unit =
  // u * G + g) against K of u; sweep 2 runs per K/V unit and streams the rows of its G heads in turn
  const size_t mat = (size_t)n * D;
  const float* own_mat = (PASS == 1 ? Q : K) + (size_t)unit * mat;
  const float* str_base = (PASS == 1) ? K + (size_t)(unit / G) * mat : Q + (size_t)unit * G * mat;
  const float2* stat_base = rowstat + (size_t)unit * (PASS == 1 ? 1 : G) * n;

  // owner fragment (B operand): item O0 + ln, elements [g * D/4, +D/4), widened once. Items past
  // the end are clamped to the last one: their results are never stored.
  const int own_i = O0 + ln;
  double own[PL];
  {
    const float* src = own_mat + (size_t)min(own_i, n - 1) * D + g * PL;
#pragma unroll
    for (int i = 0; i < LV; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        own[4 * i + e] = (double)v[e];
        asm volatile("" : "+v"(own[4 * i + e]));   // keep the widened value, not the conversion
      }
    }
  }

  const int t_begin = (PASS == 1) ? 0 : O0 / kTile;
  const int t_end = (PASS == 1) ? (min(n, O0 + 16) + kTile - 1) / kTile : (n + kTile - 1) / kTile;

  float m_run = FG_NEG_BIG;
  double acc_a = 0.0, acc_b = 0.0;   // pass 1: l (acc_b unused); pass 2: column sum and its part in the band
  const double c_d = (double)c;

  const int heads = (PASS == 1) ? 1 : G;
  for (int h = 0; h < heads; ++h) {
    const float* str_mat = str_base + (size_t)h * mat;
    const float2* stat_row = stat_base + (size_t)h * n;
    f32x4 next[LV];
    auto load = [&](int t) {   // rows past the end are clamped: masked wherever they are used
      const float* src = str_mat + (size_t)min(t * kTile + ln, n - 1) * D + g * PL;
#pragma unroll
      for (int i = 0; i < LV; ++i) next[i] = *reinterpret_cast<const f32x4*>(src + 4 * i);
    };
    if (t_begin + wave < t_end) load(t_begin + wave);
    for (int t = t_begin + wave; t < t_end; t += kWaves) {
      f32x4 cur[LV];
#pragma unroll
      for (int i = 0; i < LV; ++i) cur[i] = next[i];
      const int t0 = t * kTile;
      float2 st[4];
      if (PASS == 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) st[i] = stat_row[min(t0 + 4 * i + g, n - 1)];
      }
      load(min(t + kWaves, t_end - 1));   // the last round re-reads the last tile
      __builtin_amdgcn_sched_barrier(0);
      f64x4 x = {0.0, 0.0, 0.0, 0.0};   // x[i] = q.k of streamed item t0 + 4 i + g with owner O0 + ln
#pragma unroll
      for (int i = 0; i < LV; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x = __builtin_amdgcn_mfma_f64_16x16x4f64((double)cur[i][e], own[4 * i + e], x, 0, 0, 0);
      if (PASS == 1) {
        // m is a shift near the row's largest logit (any float will do); most tiles keep it
        float m_new = m_run;
        bool ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ok[i] = t0 + 4 * i + g <= own_i;   // causal: column <= row (and so below n)
          x[i] *= c_d;
          m_new = fmaxf(m_new, ok[i] ? (float)x[i] : FG_NEG_BIG);
        }
        if (__any(m_new != m_run)) acc_a *= exp2((double)m_run - (double)m_new);
        m_run = m_new;
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) s += exp2(ok[i] ? x[i] - (double)m_new : -2000.0);   // masked: 0
        acc_a += s;
      } else {
        double s = 0.0, sb = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = t0 + 4 * i + g;
          const bool ok = row >= own_i && row < n;
          const double p = exp2(ok ? x[i] * c_d - (double)st[i].x : -2000.0) * (double)st[i].y;
          s += p;
          sb += row - own_i < w ? p : 0.0;
        }
        acc_a += s;
        acc_b += sb;
      }
    }
  }

  // ---- merge the lane groups of every owner, then the waves, in a fixed order
  if (PASS == 1) {
    float M = fmaxf(m_run, __shfl_xor(m_run, 16, 64));
    M = fmaxf(M, __shfl_xor(M, 32, 64));
    acc_a *= exp2((double)m_run - (double)M);   // a lane group without a tile has l = 0
    acc_b = (double)M;
  } else {
    acc_b += fg_shfl_xor_f64(acc_b, 16);
    acc_b += fg_shfl_xor_f64(acc_b, 32);
  }
  acc_a += fg_shfl_xor_f64(acc_a, 16);
  acc_a += fg_shfl_xor_f64(acc_a, 32);
  if (g == 0) { s_a[wave][ln] = acc_a; s_b[wave][ln] = acc_b; }
  __syncthreads();
  if (tid < 16 && own_i < n) {
    const size_t at = (size_t)unit * n + own_i;
    if (PASS == 1) {
      const double M = fmax(fmax(s_b[0][ln], s_b[1][ln]), fmax(s_b[2][ln], s_b[3][ln]));
      double L = 0.0;
#pragma unroll
      for (int i = 0; i < kWaves; ++i) L += s_a[i][ln] * exp2(s_b[i][ln] - M);
      rowstat[at] = make_float2((float)M, (float)(1.0 / L));
    } else {
      colsum[at] = (s_a[0][ln] + s_a[1][ln]) + (s_a[2][ln] + s_a[3][ln]);
      bandcol[at] = (s_b[0][ln] + s_b[1][ln]) + (s_b[2][ln] + s_b[3][ln]);
    }
  }
}

template <int D>
hipError_t launch(const fg_profile_args& a, int pass, hipStream_t s) {
  const int nblk = (a.n + 15) / 16;
  const int units = (pass == 1) ? a.U * a.G : a.U;   // sweep 1: one unit per query head
  const float c = a.scale * FG_LOG2E;
  const float* Q = static_cast<const float*>(a.Q);
  const float* K = static_cast<const float*>(a.K);
  // a launch holds fewer than 2^32 threads: very large inputs go in several ranges of units
  const int most = 8 * ((1 << 20) / nblk > 0 ? (1 << 20) / nblk : 1);
  for (int u0 = 0; u0 < units; u0 += most) {
    const int range = units - u0 < most ? units - u0 : most;
    const dim3 grid((unsigned)(8 * nblk * ((range + 7) / 8))), block(256);
    if (pass == 1)
      hipLaunchKernelGGL((fg_profile_f32_kernel<D, 1>), grid, block, 0, s, Q, K, a.rowstat, a.colsum,
                         a.bandcol, u0, u0 + range, a.n, a.w, c, nblk, a.G);
    else
      hipLaunchKernelGGL((fg_profile_f32_kernel<D, 2>), grid, block, 0, s, Q, K, a.rowstat, a.colsum,
                         a.bandcol, u0, u0 + range, a.n, a.w, c, nblk, a.G);
  }
  return hipGetLastError();
}

// A caller-supplied natural-log row log-sum-exp as (m, 1/l): m = the nearest integer to its
// log2 value, 1/l = 2^(m - log2 value) in [0.70, 1.42], so that no bits are lost to the
// magnitude of the log-sum-exp itself.
__global__ void fg_lse_to_rowstat_kernel(const float* __restrict__ in, float2* __restrict__ out, size_t count) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const double l2 = (double)in[i] * 1.4426950408889634074;
  const double m = rint(l2);
  out[i] = make_float2((float)m, (float)exp2(m - l2));
}

}  // namespace

hipError_t fg_launch_profile_f32(const fg_profile_args& a, int pass, hipStream_t s) {
  if (a.d == 128) return launch<128>(a, pass, s);
  return launch<64>(a, pass, s);
}

hipError_t fg_launch_lse_to_rowstat(const float* lse_nat, float2* rowstat, size_t count, hipStream_t s) {
  const unsigned blocks = (unsigned)((count + 255) / 256);
  hipLaunchKernelGGL(fg_lse_to_rowstat_kernel, dim3(blocks), dim3(256), 0, s, lse_nat, rowstat, count);
  return hipGetLastError();
}
