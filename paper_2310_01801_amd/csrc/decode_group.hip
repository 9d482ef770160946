// The per-unit decode step (decode_unit.hip) for grouped query heads: G heads share the unit's cache,
// its rows are loaded once and serve all of them. A wave converts a tile of keys to float64 once
// (units that keep scores) and goes through the heads with it, each head with its own running (max,
// sum, o). One workgroup of 512 threads per unit, longest units first.
// Serves two bf16 heads and float32; three to eight bf16 heads have a kernel on the matrix cores
// (decode_group_mfma.hip).
//
// Bound: the float64 logits on the vector ALU (per tile of 16 rows and head 32 multiply-adds and the
// sums over a row's 16 lanes, four sums at once). Two float32 heads spill 8 registers, and all spill some 45
// scalars; both are still faster than the split form.
#include <type_traits>

#include "fg_common.h"
#include "fg_internal.h"
#include "fg_rows.h"
#include "fg_update.h"

namespace {

constexpr int NT = 512;
constexpr int NW = NT / 64;

// GM: the most heads the instantiation holds. Two float32 heads fit 128 registers, and then two workgroups
// a CU.
template <int ESIZE, int D, int GM>
__global__ __launch_bounds__(NT, ESIZE == 4 && GM == 2 ? 4 : 2) void fg_decode_group_kernel(fg_decode_args a) {
  constexpr int RB = D * ESIZE;        // bytes per row
  constexpr int LPR = RB / 16;         // lanes per row
  constexpr int TPL = 64 / LPR;        // rows per wave load
  constexpr int EPL = 16 / ESIZE;      // elements per lane
  constexpr int ITERS = 4;
  constexpr int TW = ITERS * TPL;      // rows per tile, one wave's
  constexpr bool TILED = ESIZE == 4;   // a tile's values are summed by themselves before they join the total
  __shared__ fg_update_smem sh;
  __shared__ float s_m[NW + 1][GM], s_l[NW + 1][GM];   // partials of the waves, then of the new token
  __shared__ float s_o[NW + 1][GM][D];
  __shared__ double s_z[NW][GM];
  __shared__ __attribute__((aligned(16))) unsigned char s_q[GM * RB];

  // header: one 32-byte record per unit carries everything, the current length included
  int32_t* rec_p = a.item_unit + (size_t)blockIdx.x * 8;
  const int overflow = a.flags[0];
  const int4 rec = *reinterpret_cast<const int4*>(rec_p);
  const int4 rec_off = *reinterpret_cast<const int4*>(rec_p + 4);
  if (overflow != 0) return;
  const int u = __builtin_amdgcn_readfirstlane(rec.x), cap = __builtin_amdgcn_readfirstlane(rec.z);
  const int Lold = __builtin_amdgcn_readfirstlane(rec.w), L = Lold + 1;
  const int off_lo = __builtin_amdgcn_readfirstlane(rec_off.x), off_hi = __builtin_amdgcn_readfirstlane(rec_off.y);
  const int pword = __builtin_amdgcn_readfirstlane(rec_off.z);
  if (L > cap) {  // cannot happen while the host bounds the step count
    if (threadIdx.x == 0) a.flags[0] = 1;
    return;
  }
  const int64_t off = ((int64_t)off_hi << 32) | (uint32_t)off_lo;
  const int policy = pword & 0xff, comp = pword >> 8;
  const bool probing = a.probe != nullptr;
  const bool scored = (comp & FG_COMP_FREQUENT) != 0 || probing;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane % LPR, sub = lane / LPR;
  const float c = a.scale * FG_LOG2E;
  const double c_d = (double)a.scale * 1.4426950408889634074;
  const int G = a.G;

  // rows past the end read as zeros without touching memory
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      static_cast<char*>(a.ck) + off * RB, 0, Lold * RB, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      static_cast<char*>(a.cv) + off * RB, 0, Lold * RB, 0x00020000);
  const int voff = sub * RB + g * 16;
  u32x4 kv[ITERS], vv[ITERS];
  auto load = [&](const __amdgpu_buffer_rsrc_t& rsrc, u32x4 (&dst)[ITERS], int tile) {
#pragma unroll
    for (int it = 0; it < ITERS; ++it)
      dst[it] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, (tile * TW + it * TPL) * RB, 0));
  };
  const int ntile = (Lold + TW - 1) / TW;
  if (wave < ntile) {
    load(k_rsrc, kv, wave);
    load(v_rsrc, vv, wave);
  }
  // all G query vectors staged in LDS while the rows are in flight
  for (int i = tid; i < G * LPR; i += NT)
    *reinterpret_cast<u32x4*>(&s_q[i * 16]) = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.q) + (size_t)u * G * RB + (size_t)i * 16);
  __syncthreads();
  auto query = [&](int h) { return *reinterpret_cast<const u32x4*>(&s_q[h * RB + g * 16]); };

  float mw[GM], lsum[GM], oacc[GM][EPL];   // of the tokens of this lane group (the LPR lanes of a row)
#pragma unroll
  for (int h = 0; h < GM; ++h) {
    mw[h] = FG_NEG_BIG;
    lsum[h] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) oacc[h][e] = 0.f;
  }
  double* const clogit = a.clogit + off * G;
  auto stream = [&](auto keep) __attribute__((always_inline)) {
    constexpr bool KEEP = decltype(keep)::value;
    for (int tile = wave; tile < ntile; tile += NW) {
      const int slot0 = tile * TW + sub;
      const bool more = tile + NW < ntile;
      float x[GM][ITERS];
      float rescale[TILED ? GM : 1];
      if (KEEP) {
        double kd[ITERS][EPL];
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
          float kf[EPL];
          fg_unpack<ESIZE>(kv[it], kf);
#pragma unroll
          for (int e = 0; e < EPL; ++e) kd[it][e] = (double)kf[e];
        }
        if (more) load(k_rsrc, kv, tile + NW);   // in flight during the rest of the tile
#pragma unroll
        for (int h = 0; h < GM; ++h) {
          if (h >= G) break;
          float qv[EPL];
          fg_unpack<ESIZE>(query(h), qv);
          double dd[ITERS];
#pragma unroll
          for (int it = 0; it < ITERS; ++it) dd[it] = 0.0;
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            const double q = (double)qv[e];
#pragma unroll
            for (int it = 0; it < ITERS; ++it) dd[it] = fma(q, kd[it][e], dd[it]);
          }
          if (LPR == 16) {
            double v;
            fg_sum4_16(dd, c_d, &v, x[h]);
            const int slot = slot0 + fg_sum4_index() * TPL;   // every fourth lane stores one of the four logits
            if (slot < Lold && (lane & 3) == 0) clogit[(size_t)slot * G + h] = v;
#pragma unroll
            for (int it = 0; it < ITERS; ++it) x[h][it] = slot0 + it * TPL < Lold ? x[h][it] : FG_NEG_BIG;
          } else {
#pragma unroll
            for (int it = 0; it < ITERS; ++it) {
              const int slot = slot0 + it * TPL;
              const double v = fg_group_sum_f64<LPR>(dd[it]) * c_d;
              if (slot < Lold && g == 0) clogit[(size_t)slot * G + h] = v;
              x[h][it] = slot < Lold ? (float)v : FG_NEG_BIG;
            }
          }
        }
      } else {
#pragma unroll
        for (int h = 0; h < GM; ++h) {
          if (h >= G) break;
          const u32x4 q_raw = query(h);
#pragma unroll
          for (int it = 0; it < ITERS; ++it) {
            float dot = 0.f;
            if (ESIZE == 2) dot = fg_dot_bf16x8(q_raw, kv[it]);
            else {
              float qv[EPL], kf[EPL];
              fg_unpack<ESIZE>(q_raw, qv);
              fg_unpack<ESIZE>(kv[it], kf);
#pragma unroll
              for (int e = 0; e < EPL; ++e) dot = fmaf(qv[e], kf[e], dot);
            }
            dot = fg_group_sum<LPR>(dot) * c;
            x[h][it] = slot0 + it * TPL < Lold ? dot : FG_NEG_BIG;
          }
        }
        if (more) load(k_rsrc, kv, tile + NW);
      }
      // the heads' maxima, then the values of the tile once for all heads
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        if (h >= G) break;
        float mx = mw[h];
#pragma unroll
        for (int it = 0; it < ITERS; ++it) mx = fmaxf(mx, x[h][it]);
        const float f = fg_exp2(mw[h] - mx);
        mw[h] = mx;
        lsum[h] *= f;
        if (!TILED) {
#pragma unroll
          for (int e = 0; e < EPL; ++e) oacc[h][e] *= f;
        } else rescale[h] = f;
        float l_t = 0.f;
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
          x[h][it] = (slot0 + it * TPL < Lold) ? fg_exp2(x[h][it] - mx) : 0.f;
          l_t += x[h][it];
        }
        lsum[h] += l_t;
      }
      if (TILED) {
        // float32 outputs: the tile is summed by itself first, which keeps the chains of roundings
        // short (24 units of 1000 tokens, G = 2, d = 128: 2-norm error 1.89e-7, in one chain 2.22e-7)
#pragma unroll
        for (int h = 0; h < GM; ++h) {
          if (h >= G) break;
          float o_t[EPL];
#pragma unroll
          for (int it = 0; it < ITERS; ++it) {
            float vf[EPL];
            fg_unpack<ESIZE>(vv[it], vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) o_t[e] = it == 0 ? x[h][0] * vf[e] : fmaf(x[h][it], vf[e], o_t[e]);
          }
#pragma unroll
          for (int e = 0; e < EPL; ++e) oacc[h][e] = fmaf(oacc[h][e], rescale[h], o_t[e]);
        }
      } else {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
          float vf[EPL];
          fg_unpack<ESIZE>(vv[it], vf);
#pragma unroll
          for (int h = 0; h < GM; ++h) {
            if (h >= G) break;
#pragma unroll
            for (int e = 0; e < EPL; ++e) oacc[h][e] = fmaf(x[h][it], vf[e], oacc[h][e]);
          }
        }
      }
      if (more) load(v_rsrc, vv, tile + NW);
    }
  };
  if (scored) stream(std::true_type{});
  else stream(std::false_type{});

  // the new token: a partial of its own, and its row appended in the first free slot
  if (wave == NW - 1) {
    const u32x4 knew = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.k_new) + (size_t)u * RB + g * 16);
    const u32x4 vnew = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.v_new) + (size_t)u * RB + g * 16);
    float kf[EPL], vf[EPL];
    fg_unpack<ESIZE>(knew, kf);
    fg_unpack<ESIZE>(vnew, vf);
    if (sub == 0) {
      *reinterpret_cast<u32x4*>(static_cast<char*>(a.ck) + (off + Lold) * RB + g * 16) = knew;
      *reinterpret_cast<u32x4*>(static_cast<char*>(a.cv) + (off + Lold) * RB + g * 16) = vnew;
    }
    if (lane == 0) {
      a.cpos[off + Lold] = a.n + a.step;
      a.ccls[off + Lold] = a.class_new[u / a.units_per_seq];
      a.cscore[off + Lold] = 0.0;
    }
    for (int h = 0; h < G; ++h) {
      float qv[EPL];
      fg_unpack<ESIZE>(query(h), qv);
      double dd = 0.0;   // one token: float64 for every policy
#pragma unroll
      for (int e = 0; e < EPL; ++e) dd = fma((double)qv[e], (double)kf[e], dd);
      dd = fg_group_sum_f64<LPR>(dd) * c_d;
      if (sub == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) s_o[NW][h][g * EPL + e] = vf[e];
      }
      if (lane == 0) {
        if (scored) clogit[(size_t)Lold * G + h] = dd;
        s_m[NW][h] = (float)dd;
        s_l[NW][h] = 1.f;
      }
    }
  }
  // the row groups of the wave (lanes with equal g), then the waves
#pragma unroll
  for (int h = 0; h < GM; ++h) {
    if (h >= G) break;
    const float M = fg_wave_max(mw[h]), f = fg_exp2(mw[h] - M);   // a group without tokens has zero sums
    mw[h] = M;
    lsum[h] *= f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) oacc[h][e] *= f;
#pragma unroll
    for (int m = LPR; m < 64; m <<= 1) {
      lsum[h] += __shfl_xor(lsum[h], m, 64);
#pragma unroll
      for (int e = 0; e < EPL; ++e) oacc[h][e] += __shfl_xor(oacc[h][e], m, 64);
    }
    if (sub == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) s_o[wave][h][g * EPL + e] = oacc[h][e];
    }
    if (lane == 0) { s_m[wave][h] = mw[h]; s_l[wave][h] = lsum[h]; }
  }
  auto merge = [&]() -> float {
    __syncthreads();   // also orders the appended slot and the kept logits before the update
    for (int q = tid; q < G * D; q += NT) {
      const int h = q / D, e = q % D;
      float M = s_m[0][h];
#pragma unroll
      for (int i = 1; i <= NW; ++i) M = fmaxf(M, s_m[i][h]);
      // a wave without tokens carries the lowest max and zero sums: its factor is 0
      float o = 0.f, l = 0.f;
#pragma unroll
      for (int i = 0; i <= NW; ++i) {
        const float f = fg_exp2(s_m[i][h] - M);
        o += s_o[i][h][e] * f;
        l += s_l[i][h] * f;
      }
      fg_store_out<ESIZE>(a.out, (size_t)u * G * D + q, o * (1.0f / l));
    }
    if (scored) {
      // This step's attention (float64, as in fg_update.h) summed over the heads replaces head 0's
      // logit in place; each thread only touches the slots it owns in the update.
      double M[GM], z[GM];
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        if (h >= G) break;
        float m = s_m[0][h];
#pragma unroll
        for (int i = 1; i <= NW; ++i) m = fmaxf(m, s_m[i][h]);
        M[h] = (double)m;
        z[h] = 0.0;
      }
      for (int j = tid; j < L; j += NT) {
        double* lg = clogit + (size_t)j * G;
        double e[GM];
#pragma unroll
        for (int h = 0; h < GM; ++h) if (h < G) e[h] = lg[h];
#pragma unroll
        for (int h = 0; h < GM; ++h) {
          if (h >= G) break;
          e[h] = exp2(e[h] - M[h]);
          z[h] += e[h];
          lg[h] = e[h];
        }
      }
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        if (h >= G) break;
        z[h] = fg_wave_sum_f64(z[h]);
        if (lane == 0) s_z[wave][h] = z[h];
      }
      __syncthreads();
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        if (h >= G) break;
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < NW; ++i) t += s_z[i][h];
        z[h] = 1.0 / t;
      }
      for (int j = tid; j < L; j += NT) {
        double* lg = clogit + (size_t)j * G;
        double sum = 0.0;
#pragma unroll
        for (int h = 0; h < GM; ++h) if (h < G) sum += lg[h] * z[h];
        lg[0] = sum;
      }
    }
    return 0.f;   // the update takes the ready attention, no shift
  };
  auto set_len = [&](int v) {
    if (tid == 0) { a.len[u] = v; rec_p[3] = v; }
  };
  if (policy >= 4 && !probing) {
    (void)merge();
    set_len(L);
    return;
  }
  fg_update_unit<ESIZE, D, true, NT, FG_UNIT_TOKENS>(a, u, L, cap, off, policy, comp, sh, merge, set_len);
}

template <int GM>
hipError_t launch(const fg_decode_args& a, hipStream_t s) {
  const dim3 grid((unsigned)a.U), block(NT);
  if (a.dtype == FG_F32) {
    if (a.d == 128) hipLaunchKernelGGL((fg_decode_group_kernel<4, 128, GM>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((fg_decode_group_kernel<4, 64, GM>), grid, block, 0, s, a);
  } else {   // two heads
    if (a.d == 128) hipLaunchKernelGGL((fg_decode_group_kernel<2, 128, 2>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((fg_decode_group_kernel<2, 64, 2>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t fg_launch_decode_group(const fg_decode_args& a, hipStream_t s) {
  if (a.dtype == FG_BF16 && a.G > 2) return fg_launch_decode_group_mfma(a, s);
  if (a.G <= 2) return launch<2>(a, s);
  if (a.G <= 4) return launch<4>(a, s);
  return launch<8>(a, s);
}
