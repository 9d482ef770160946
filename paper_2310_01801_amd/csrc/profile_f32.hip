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

// Both sweeps in one pass over Q and K, for prompts of up to 64 * S tokens. Part p of a unit's P workgroups walks blocks
// of 16 query rows, dealt out back and forth from the heaviest down. Its waves take the tiles of 16 columns in turn and keep the
// exponentials of a block in registers, S tiles of four doubles; the waves exchange (m, l) of the rows, and the column
// sums take the exponentials from the registers. One contraction and one exponential per score instead of two, and
// no row statistics rounded to float32. A part's column sums meet in LDS (a column belongs to one wave) and
// leave as partial sums, which fg_part_sum_kernel adds in order.
// Bound: the float64 matrix pipe (52 % busy there). 64 units of 1000 tokens, d = 128: 464 us in two sweeps, 253 in one
// pass and the part sums; 16 of 1000: 134 -> 78. With 1024 columns at d = 128 the row's own elements are read back from LDS and the next keys asked
// for only behind the products, and still five registers spill; held as doubles the row alone takes 64.
template <int D, int S>
__global__ __launch_bounds__(256, 2) void fg_profile_once_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, double* __restrict__ colsum, double* __restrict__ bandcol,
    int U, int n, int w, float c, int G, int P) {
  constexpr int PL = D / 4;        // elements of a row per lane
  constexpr int LV = PL / 4;       // 16-byte loads per row and lane
  constexpr double kFar = 900.0;   // 2^x stays in range up to here
  constexpr bool EARLY = S <= 8 || D == 64;   // the next tile on its way during the products, else during the exponentials
  constexpr bool LDS_OWN = S > 8;  // the row's elements wait in LDS where the exponentials need the registers
  __shared__ __attribute__((aligned(16))) f32x4 s_own[LDS_OWN ? kWaves : 1][LDS_OWN ? LV : 1][64];
  __shared__ double s_l[2][kWaves][16], s_m[2][kWaves][16];
  __shared__ double s_sum[2][S * kWaves * kTile];   // column sums, and their part inside the band

  // parts of one unit on one XCD (its L2 then serves the keys)
  const int idx = blockIdx.x, xcd = idx & 7, rest = idx >> 3;
  const int unit = (rest / P) * 8 + xcd, part = rest % P;
  if (unit >= U) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 15, g = lane >> 4;
  const int nblk = (n + kTile - 1) / kTile;
  for (int i = tid; i < 2 * S * kWaves * kTile; i += 256) (&s_sum[0][0])[i] = 0.0;
  __syncthreads();
  const float* k_mat = K + (size_t)unit * n * D;
  const double c_d = (double)c;
  int buf = 0;
  for (int h = 0; h < G; ++h) {   // the query heads of the unit, over the same columns
    const float* q_mat = Q + ((size_t)unit * G + h) * n * D;
    for (int i = 0;; ++i) {
      const int place = (i & 1) ? (i + 1) * P - 1 - part : i * P + part;   // by weight: P down, P up, ...
      if (place >= nblk) break;   // every later one is further on
      const int blk = nblk - 1 - place;
      const int r0 = blk * kTile, row = r0 + ln;
      // rows past the end are clamped: they count nothing
      f32x4 own[LV], next[LV];
      {
        const float* src = q_mat + (size_t)min(row, n - 1) * D + g * PL;
#pragma unroll
        for (int v = 0; v < LV; ++v) {
          own[v] = *reinterpret_cast<const f32x4*>(src + 4 * v);
          if (LDS_OWN) s_own[LDS_OWN ? wave : 0][LDS_OWN ? v : 0][lane] = own[v];
        }
      }
      auto load = [&](int t) {
        const float* src = k_mat + (size_t)min(t * kTile + ln, n - 1) * D + g * PL;
#pragma unroll
        for (int v = 0; v < LV; ++v) next[v] = *reinterpret_cast<const f32x4*>(src + 4 * v);
      };
      if (wave <= blk) load(wave);
      double e[S][4];
      double m_run = 0.0, l_run = 0.0;   // of this lane's columns 4 i + g of the wave's tiles
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int t = wave + kWaves * s;
        if (t > blk) continue;
        f64x4 x = {0.0, 0.0, 0.0, 0.0};   // x[k] = q.k of column 16 t + 4 k + g with row ln
        f32x4 cur[LV];
#pragma unroll
        for (int v = 0; v < LV; ++v) cur[v] = next[v];
        if (EARLY && s + 1 < S) load(min(t + kWaves, blk));   // the last round re-reads the block's last tile
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < LV; ++v) {
          if (LDS_OWN) own[v] = s_own[LDS_OWN ? wave : 0][LDS_OWN ? v : 0][lane];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            asm volatile("" : "+v"(own[v][k]));   // widened here: held as doubles the row takes 64 registers
            x = __builtin_amdgcn_mfma_f64_16x16x4f64((double)cur[v][k], (double)own[v][k], x, 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!EARLY && s + 1 < S) load(min(t + kWaves, blk));
        bool ok[4];
        double far = -1.0e30;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          ok[k] = t < blk || 4 * k + g <= ln;   // causal
          x[k] *= c_d;
          far = fmax(far, ok[k] ? x[k] : -1.0e30);
        }
        // The shift only has to keep the exponentials in float64's range: it starts at 0, or at the first
        // tile's logit where that is far away, and hardly ever moves.
        if (__any(far > m_run + kFar) || (s == 0 && __any(far < m_run - kFar && far > -1.0e29))) {
          const double m_new = far > m_run + kFar || (s == 0 && far < m_run - kFar && far > -1.0e29) ? rint(far) : m_run;
          const double f = exp2(m_run - m_new);
          l_run = s == 0 ? 0.0 : l_run * f;
#pragma unroll
          for (int b = 0; b < s; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) e[b][k] *= f;
          m_run = m_new;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          e[s][k] = exp2(ok[k] ? x[k] - m_run : -2000.0);   // masked: 0
          l_run += e[s][k];
        }
      }
      // (m, l) of every row: its lane groups, then the waves, in a fixed order. A lane without a column has l = 0
      // and counts with any shift.
      double M = l_run > 0.0 ? m_run : -1.0e30;
      M = fmax(M, fg_shfl_xor_f64(M, 16));
      M = fmax(M, fg_shfl_xor_f64(M, 32));
      double L = l_run > 0.0 ? l_run * exp2(m_run - M) : 0.0;
      L += fg_shfl_xor_f64(L, 16);
      L += fg_shfl_xor_f64(L, 32);
      if (g == 0) { s_l[buf][wave][ln] = L; s_m[buf][wave][ln] = M; }
      __syncthreads();
      M = fmax(fmax(s_m[buf][0][ln], s_m[buf][1][ln]), fmax(s_m[buf][2][ln], s_m[buf][3][ln]));
      L = 0.0;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) L += s_l[buf][v][ln] * exp2(fmax(s_m[buf][v][ln] - M, -2000.0));
      buf ^= 1;
      const double f = row < n ? exp2(fmax(fmin(m_run - M, 1000.0), -2000.0)) / L : 0.0;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int t = wave + kWaves * s, t0 = t * kTile;
        if (t > blk) continue;
        double v[4], sum;
        float unused[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = e[s][k] * f;
        const int at = t0 + 4 * fg_sum4_index() + g;
        const bool inside = r0 + kTile - 1 - t0 < w, outside = r0 - (t0 + kTile - 1) >= w;
        fg_sum4_16(v, 1.0, &sum, unused);
        // one wave adds to a column, in the order of the blocks; every second lane of four carries the band
        if ((lane & 3) == 0 || ((lane & 3) == 1 && inside)) s_sum[lane & 3][at] += sum;
        if (!inside && !outside) {
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = row - (t0 + 4 * k + g) < w ? v[k] : 0.0;
          fg_sum4_16(v, 1.0, &sum, unused);
          if ((lane & 3) == 1) s_sum[1][at] += sum;
        }
      }
    }
  }
  __syncthreads();
  const size_t out = ((size_t)part * U + unit) * n;
  for (int i = tid; i < n; i += 256) {
    colsum[out + i] = s_sum[0][i];
    bandcol[out + i] = s_sum[1][i];
  }
}

// Sums of the parts [P, N] in order
__global__ void fg_part_sum_kernel(const double* __restrict__ pcol, const double* __restrict__ pband,
                                   double* __restrict__ col, double* __restrict__ band, int cols, int stride, size_t N, int P) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double a = pcol[i], b = pband[i];
  for (int p = 1; p < P; ++p) {
    a += pcol[p * N + i];
    b += pband[p * N + i];
  }
  const size_t to = i / cols * stride + i % cols;
  col[to] = a;
  band[to] = b;
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

template <int D, int S>
hipError_t launch_once(const fg_profile_args& a, int P, double* parts, hipStream_t s) {
  const size_t N = (size_t)a.U * a.n;
  double* col = P > 1 ? parts : a.colsum;
  double* band = P > 1 ? parts + P * N : a.bandcol;
  hipLaunchKernelGGL((fg_profile_once_f32_kernel<D, S>), dim3((unsigned)(8 * P * ((a.U + 7) / 8))), dim3(256), 0, s,
                     static_cast<const float*>(a.Q), static_cast<const float*>(a.K), col, band, a.U, a.n, a.w,
                     a.scale * FG_LOG2E, a.G, P);
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

hipError_t fg_launch_part_sums(const double* pcol, const double* pband, double* col, double* band, int U, int cols, int stride, int parts, hipStream_t s) {
  const size_t N = (size_t)U * cols;
  hipLaunchKernelGGL(fg_part_sum_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, pcol, pband, col, band, cols, stride, N, parts);
  return hipGetLastError();
}

hipError_t fg_launch_profile_f32(const fg_profile_args& a, int pass, hipStream_t s) {
  if (a.d == 128) return launch<128>(a, pass, s);
  return launch<64>(a, pass, s);
}

hipError_t fg_launch_profile_once_f32(const fg_profile_args& a, int P, double* parts, hipStream_t s) {
  if (a.n > 1024) return hipErrorInvalidValue;
  if (a.n <= 256) return a.d == 128 ? launch_once<128, 4>(a, P, parts, s) : launch_once<64, 4>(a, P, parts, s);
  if (a.n <= 512) return a.d == 128 ? launch_once<128, 8>(a, P, parts, s) : launch_once<64, 8>(a, P, parts, s);
  return a.d == 128 ? launch_once<128, 16>(a, P, parts, s) : launch_once<64, 16>(a, P, parts, s);
}

hipError_t fg_launch_lse_to_rowstat(const float* lse_nat, float2* rowstat, size_t count, hipStream_t s) {
  const unsigned blocks = (unsigned)((count + 255) / 256);
  hipLaunchKernelGGL(fg_lse_to_rowstat_kernel, dim3(blocks), dim3(256), 0, s, lse_nat, rowstat, count);
  return hipGetLastError();
}
