// One decode step, one workgroup per unit (Alg. 2: attend with K^,V^ plus the new token, then
// re-apply f with the head's policy; policies of Sec. 3.4): the form for units that a workgroup
// can stream by itself. Its waves take the unit's rows in turn, each with its own running (max,
// sum, o); the merge and the kept-set update then need neither a second launch nor partial results
// in memory, and the update of one unit (a chain of block reductions) runs while the other
// workgroups of the CU stream. Workgroups take the units longest first.
//
// Bound: HBM in the streaming part, the update's chain of latencies at the end of a launch.
// Measured against the split form (attention + update launch): 1024 units of 2048 tokens, d = 128
// bf16: 101 + 20 -> 102 us per step; 16384 of 1024: 835 -> 801 in this form; 432 of 1337, d = 64:
// 15 + 14 -> 18; 4 of 128, float32: 12 -> 5.9. The logits of the units that keep scores stay in LDS for the update
// (through memory their stores held up the merge's barrier and their loads the update), and the new token falls to
// a wave that ends early (the last one, behind its rows, kept the others waiting for 7 us): with both, and fewer barriers
// in the update, 110 -> 102, 19.4 -> 17.8, 6.4 -> 5.9, 4096 units of 1024 tokens 217 -> 205, 1600 of 4096 424 -> 403. Four loads of K and of V per lane and tile, the
// next tile's K on its way during the sums and its V during the logits, keep 109 to 126 vector
// registers (and spill 55 to 73 scalars into lanes of one): eight loads spill vectors (199 us at the first
// shape), 96 registers for five waves per SIMD too (190), 1024 threads are slower everywhere. By a clock trace
// of the first shape a scored unit of 1212 tokens streams for 54 to 62 us and holds its place for the update's 5, while
// only two workgroups fit a CU. Tried without gain: the last round's rows shared alike (104 -> 108), higher
// priority for the later waves (with this order 106) or for the update.
#include <type_traits>

#include "fg_common.h"
#include "fg_internal.h"
#include "fg_rows.h"
#include "fg_update.h"

namespace {

template <int ESIZE, int D, int NT>
__global__ __launch_bounds__(NT, 4) void fg_decode_unit_kernel(fg_decode_args a) {
  constexpr int RB = D * ESIZE;        // bytes per row
  constexpr int LPR = RB / 16;         // lanes per row
  constexpr int TPL = 64 / LPR;        // rows per wave load
  constexpr int EPL = 16 / ESIZE;      // elements per lane
  constexpr int ITERS = 4;             // loads per tile: K and V of a tile are 32 registers
  constexpr int TW = ITERS * TPL;      // rows per tile, one wave's
  constexpr int NW = NT / 64;
  __shared__ fg_update_smem sh;
  __shared__ float s_m[NW + 1], s_l[NW + 1];   // partials of the waves, then of the new token
  __shared__ float s_o[NW + 1][D];
  __shared__ double s_x[NT == 256 ? FG_UNIT_TOKENS_256 : FG_UNIT_TOKENS];   // logits of the units that keep scores

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
  // the float64 logits are kept where the update needs them: policies with `frequent` (cumulative
  // scores), or every unit when the step is probed
  const bool keep_logits = (comp & FG_COMP_FREQUENT) != 0 || probing;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane % LPR, sub = lane / LPR;
  const float c = a.scale * FG_LOG2E;
  const double c_d = (double)a.scale * 1.4426950408889634074;

  const u32x4 q_raw = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.q) + (size_t)u * RB + g * 16);
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
  float qv[EPL];
  fg_unpack<ESIZE>(q_raw, qv);

  // scaled logit (log2 domain) of the row piece held by a lane, the same in its LPR lanes
  auto logit64 = [&](const u32x4& k) {
    float kf[EPL];
    fg_unpack<ESIZE>(k, kf);
    double dd = 0.0;
#pragma unroll
    for (int e = 0; e < EPL; ++e) dd = fma((double)qv[e], (double)kf[e], dd);
    return fg_group_sum_f64<LPR>(dd) * c_d;
  };
  auto logit32 = [&](const u32x4& k) {
    float dot = 0.f;
    if (ESIZE == 2) dot = fg_dot_bf16x8(q_raw, k);
    else {
      float kf[EPL];
      fg_unpack<ESIZE>(k, kf);
#pragma unroll
      for (int e = 0; e < EPL; ++e) dot = fmaf(qv[e], kf[e], dot);
    }
    return fg_group_sum<LPR>(dot) * c;
  };

  float mw = FG_NEG_BIG, lsum = 0.f;       // of this wave's tokens; lsum and oacc per lane group
  float oacc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) oacc[e] = 0.f;
  auto stream = [&](auto keep) __attribute__((always_inline)) {
    for (int tile = wave; tile < ntile; tile += NW) {
      const int slot0 = tile * TW + sub;
      float x[ITERS];
      float mx = mw;
#pragma unroll
      for (int it = 0; it < ITERS; ++it) {
        const int slot = slot0 + it * TPL;
        const bool ok = slot < Lold;
        if (decltype(keep)::value) {
          const double dd = logit64(kv[it]);
          if (ok && g == 0) s_x[slot] = dd;
          x[it] = (float)dd;
        } else {
          x[it] = logit32(kv[it]);
        }
        x[it] = ok ? x[it] : FG_NEG_BIG;
        mx = fmaxf(mx, x[it]);
      }
      const bool more = tile + NW < ntile;
      if (more) load(k_rsrc, kv, tile + NW);  // in flight during the second half
      mx = fg_wave_max(mx);
      const float f = fg_exp2(mw - mx);
      mw = mx;
      // The tile is summed by itself first, which keeps the chains of roundings short: in a float32
      // replay of 2048 tokens over eight waves 1.4e-7 off 64 bits, in one chain 1.8e-7 (4096: 1.6 and 2.3).
      float l_t = 0.f, o_t[EPL];
#pragma unroll
      for (int it = 0; it < ITERS; ++it) {
        const float p = (slot0 + it * TPL < Lold) ? fg_exp2(x[it] - mx) : 0.f;
        l_t = it == 0 ? p : l_t + p;
        float vf[EPL];
        fg_unpack<ESIZE>(vv[it], vf);
#pragma unroll
        for (int e = 0; e < EPL; ++e) o_t[e] = it == 0 ? p * vf[e] : fmaf(p, vf[e], o_t[e]);
      }
      lsum = fmaf(lsum, f, l_t);
#pragma unroll
      for (int e = 0; e < EPL; ++e) oacc[e] = fmaf(oacc[e], f, o_t[e]);
      if (more) load(v_rsrc, vv, tile + NW);
    }
  };
  if (keep_logits) stream(std::true_type{});
  else stream(std::false_type{});

  // The new token: a partial of its own, and its row appended in the first free slot. By one of the waves that are through
  // first: the later half of them shares its SIMDs with older ones and ends 8 of 62 us after those.
  if (wave == NW / 2 - 1) {
    const u32x4 knew = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.k_new) + (size_t)u * RB + g * 16);
    const u32x4 vnew = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.v_new) + (size_t)u * RB + g * 16);
    const double dd = keep_logits ? logit64(knew) : (double)logit32(knew);
    if (sub == 0) {
      *reinterpret_cast<u32x4*>(static_cast<char*>(a.ck) + (off + Lold) * RB + g * 16) = knew;
      *reinterpret_cast<u32x4*>(static_cast<char*>(a.cv) + (off + Lold) * RB + g * 16) = vnew;
      float vf[EPL];
      fg_unpack<ESIZE>(vnew, vf);
#pragma unroll
      for (int e = 0; e < EPL; ++e) s_o[NW][g * EPL + e] = vf[e];
    }
    if (lane == 0) {
      a.cpos[off + Lold] = a.n + a.step;
      a.ccls[off + Lold] = a.class_new[u / a.units_per_seq];
      a.cscore[off + Lold] = 0.0;
      if (keep_logits) s_x[Lold] = dd;
      s_m[NW] = (float)dd;
      s_l[NW] = 1.f;
    }
  }
  // the row groups of the wave (lanes with equal g), then the waves
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1) {
    lsum += __shfl_xor(lsum, m, 64);
#pragma unroll
    for (int e = 0; e < EPL; ++e) oacc[e] += __shfl_xor(oacc[e], m, 64);
  }
  if (sub == 0) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) s_o[wave][g * EPL + e] = oacc[e];
  }
  if (lane == 0) { s_m[wave] = mw; s_l[wave] = lsum; }
  auto merge = [&]() -> float {
  __syncthreads();   // also orders the appended slot and the logits before the update
  float M = s_m[0];
#pragma unroll
  for (int i = 1; i <= NW; ++i) M = fmaxf(M, s_m[i]);
  if (tid < D) {
    // a wave without tokens carries the lowest max and zero sums: its factor is 0
    float o = 0.f, l = 0.f;
#pragma unroll
    for (int i = 0; i <= NW; ++i) {
      const float f = fg_exp2(s_m[i] - M);
      o += s_o[i][tid] * f;
      l += s_l[i] * f;
    }
    fg_store_out<ESIZE>(a.out, (size_t)u * D + tid, o * (1.0f / l));
  }
    return M;
  };
  auto set_len = [&](int v) {
    if (tid == 0) { a.len[u] = v; rec_p[3] = v; }
  };
  if (policy >= 4 && !probing) {
    (void)merge();
    set_len(L);
    return;
  }
  fg_update_unit<ESIZE, D, false, NT, NT == 256 ? FG_UNIT_TOKENS_256 : FG_UNIT_TOKENS>(a, u, L, cap, off, policy, comp, sh, merge, set_len,
      [&](int j) { return s_x[j]; });
}

template <int NT>
hipError_t launch(const fg_decode_args& a, hipStream_t s) {
  const dim3 grid((unsigned)a.U), block(NT);
  if (a.dtype == FG_BF16) {
    if (a.d == 128) hipLaunchKernelGGL((fg_decode_unit_kernel<2, 128, NT>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((fg_decode_unit_kernel<2, 64, NT>), grid, block, 0, s, a);
  } else {
    if (a.d == 128) hipLaunchKernelGGL((fg_decode_unit_kernel<4, 128, NT>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((fg_decode_unit_kernel<4, 64, NT>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t fg_launch_decode_unit(const fg_decode_args& a, hipStream_t s) {
  if (a.G > 1) return fg_launch_decode_group(a, s);
  if (a.unit_threads == 256) return launch<256>(a, s);
  return launch<512>(a, s);
}
