// The per-unit decode step (decode_group.hip) of bf16 caches with three to eight query heads per unit, its
// contractions on the matrix cores: 32 tokens per wave and tile.
//   logits   16x16x32 with the keys as rows and the heads as columns. The heads fill only part of the 16
//            columns, so the group is repeated: column n carries head n mod 4 (or 8) as its split n / 4 (n / 8).
//   values   the weights 2^(x - m) stay float32: cut into three pieces of 8 bits, which is exact, and column n's
//            lane holds piece number n / 4 of its head, in just the layout that the next instruction reads
//            as rows. The pieces' sums meet once, at the end. The rows of V pass through LDS and are read back
//            transposed (ds_read_b64_tr_b16).
//   scores   units that keep cumulative scores form their logits in float64 on the 4x4x4 float64 instruction
//            (four blocks of 4 tokens x 4 heads), from which the float32 ones are taken as well: 16 cycles for 256
//            multiply-adds where the vector ALU takes 8 to 12 for 64, and no sums over lanes. Their exponentials
//            are formed while the tiles stream as well.
// Bound: the rate at which one CU streams its unit (44.6 us for 256 full caches of 2048 tokens is 6.1 TB/s), with the
// update's chain behind it. Measured per step against the vector-ALU form (decode_group.hip): 256 units of 2048 tokens,
// G = 4: 48.8 -> 34.3 us (that form's score sums over memory kept: 39.4; each head's partials reduced by plain
// shuffles: 37.0); 256 of 1500, G = 8: 66 -> 38; 2048 of 64, G = 4: 75 -> 67; 4 of 64, G = 4: 10.2 -> 9.3. Two heads leave
// half of the columns idle and gain nothing (1024 of 700: 52 / 59); a few long units stay in the split form
// (fg_unit_threads), three and five heads first, which pay for four and eight columns.
#include <type_traits>

#include "fg_common.h"
#include "fg_internal.h"
#include "fg_rows.h"
#include "fg_update.h"

namespace {

constexpr int NT = 512;
constexpr int NW = NT / 64;

typedef int16_t i16x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Four rows by 16 columns of 16-bit elements per group of 16 lanes: a lane points at 8 bytes of its row and
// receives the four elements of its column.
__device__ __forceinline__ uint2 fg_read_transposed(const unsigned char* p) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) i16x4*)const_cast<unsigned char*>(p)));
#else
  return uint2{};
#endif
}

template <int D, int GM>
__global__ __launch_bounds__(NT, 2) void fg_decode_group_mfma_kernel(fg_decode_args a) {
  constexpr int RB = D * 2;            // bytes per row
  constexpr int TW = 32;               // tokens per tile, one wave's: two sets of 16 rows
  constexpr int KK = D / 32;           // steps of a 16x16x32 contraction over a row
  constexpr int NTL = D / 16;          // sets of 16 dimensions
  constexpr int LPR = RB / 16;         // lanes per row of V
  constexpr int TPL = 64 / LPR;        // rows of V per load
  constexpr int VL = TW / TPL;         // loads of V per tile
  constexpr int GP = GM <= 4 ? 4 : 8;  // columns of one split
  constexpr int GH = GP / 4;           // 4x4x4 instructions for all heads
  __shared__ fg_update_smem sh;
  __shared__ float s_m[NW + 1][GM], s_l[NW + 1][GM];   // partials of the waves, then of the new token
  __shared__ float s_o[NW + 1][GM][D];
  __shared__ double s_z[NW + 1][GM];
  __shared__ __attribute__((aligned(16))) unsigned char s_q[GM * RB];
  __shared__ __attribute__((aligned(16))) unsigned char s_v[NW][TW * RB];
  __shared__ __attribute__((aligned(16))) f64x2 s_qd[GH][KK * 4][16];   // query pairs of the float64 logits
  // Scores: a tile keeps 2^(x - m) of its float64 logits under its wave's shift m (a whole number); what is left for
  // the end is a factor 2^(m - M) / Z per tile and head. The last row is the new token's.
  constexpr int TILES = FG_UNIT_TOKENS / TW;
  __shared__ float s_shift[TILES][GP];
  __shared__ double s_factor[TILES + 1][GP];

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
  const int G = a.G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n16 = lane & 15, g = lane >> 4;
  const float c = a.scale * FG_LOG2E;
  const double c_d = (double)a.scale * 1.4426950408889634074;

  // rows past the end read as zeros without touching memory
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      static_cast<char*>(a.ck) + off * RB, 0, Lold * RB, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      static_cast<char*>(a.cv) + off * RB, 0, Lold * RB, 0x00020000);
  const int k_voff = n16 * RB + g * 16;                              // row n16 of 16, elements [32 kk + 8 g, + 8)
  const int v_row = lane / LPR, v_voff = v_row * RB + (lane % LPR) * 16;
  u32x4 kf[2][KK], vf[VL];
  auto load_k = [&](int tile) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        kf[st][kk] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, k_voff, (tile * TW + st * 16) * RB + kk * 64, 0));
  };
  auto load_v = [&](int tile) {
#pragma unroll
    for (int i = 0; i < VL; ++i)
      vf[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, v_voff, (tile * TW + i * TPL) * RB, 0));
  };
  const int ntile = (Lold + TW - 1) / TW;
  if (wave < ntile) {
    load_k(wave);
    load_v(wave);
  }
  // the query vectors: as they are, as columns of the logits, and as pairs of doubles
  const char* q_src = static_cast<const char*>(a.q) + (size_t)u * G * RB;
  for (int i = tid; i < G * LPR; i += NT)
    *reinterpret_cast<u32x4*>(&s_q[i * 16]) = *reinterpret_cast<const u32x4*>(q_src + (size_t)i * 16);
  if (scored) {
    for (int i = tid; i < GH * KK * 64; i += NT) {
      const int half = i / (KK * 64), step = (i / 16) % (KK * 4), gg = (i >> 2) & 3, h = half * 4 + (i & 3);
      f64x2 q = {0.0, 0.0};
      if (h < G) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(q_src + (size_t)h * RB + (step >> 2) * 64 + gg * 16 + (step & 3) * 4);
        q[0] = (double)fg_bf16_lo(w);
        q[1] = (double)fg_bf16_hi(w);
      }
      s_qd[half][step][i & 15] = q;
    }
  }
  __syncthreads();
  const int head = n16 % GP, split = n16 / GP;
  bf16x8 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (head < G) v = *reinterpret_cast<const u32x4*>(&s_q[head * RB + kk * 64 + g * 16]);
    qf[kk] = __builtin_bit_cast(bf16x8, v);
  }

  // V in LDS: 32-byte sets of a row swizzled by the row, so that the 16 rows of a transposed read spread over the banks
  auto v_place = [&](int row, int set) { return row * RB + (set ^ (D == 128 ? row & 7 : (row >> 1) & 3)) * 32; };
  // (a fourth split has no piece: nothing is left)
  const unsigned cut1 = split == 0 ? 0u : split == 3 ? 0xffffffffu : 0xffff0000u, cut2 = split >= 2 ? 0xffff0000u : 0u;

  float mw = FG_NEG_BIG, lsum = 0.f;   // of this lane's column (head); the sum is over this lane's tokens
  f32x4 acc[NTL];                      // row 4 g + i: piece and head, column: dimension
#pragma unroll
  for (int s = 0; s < NTL; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  double z[GH];                        // of head 4 hh + (lane & 3), this lane's tokens
#pragma unroll
  for (int hh = 0; hh < GH; ++hh) z[hh] = 0.0;
  double* const clogit = a.clogit + off * G;
  auto stream = [&](auto keep) __attribute__((always_inline)) {
    constexpr bool KEEP = decltype(keep)::value;
    for (int tile = wave; tile < ntile; tile += NW) {
      const bool more = tile + NW < ntile;
      float x[2][4];   // scaled logits of tokens 4 g + i of either set
      double xd[GH][2];
      if (KEEP) {
#pragma unroll
        for (int hh = 0; hh < GH; ++hh) xd[hh][0] = xd[hh][1] = 0.0;
#pragma unroll
        for (int step = 0; step < KK * 4; ++step) {
          double k0[2], k1[2];
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            const uint32_t w = kf[st][step >> 2][step & 3];
            k0[st] = (double)fg_bf16_lo(w);
            k1[st] = (double)fg_bf16_hi(w);
          }
#pragma unroll
          for (int hh = 0; hh < GH; ++hh) {
            const f64x2 q = s_qd[hh][step][g * 4 + (lane & 3)];
#pragma unroll
            for (int st = 0; st < 2; ++st) xd[hh][st] = __builtin_amdgcn_mfma_f64_4x4x4f64(k0[st], q[0], xd[hh][st], 0, 0, 0);
#pragma unroll
            for (int st = 0; st < 2; ++st) xd[hh][st] = __builtin_amdgcn_mfma_f64_4x4x4f64(k1[st], q[1], xd[hh][st], 0, 0, 0);
          }
          if ((step & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // not all steps' operands at once
        }
        if (more) load_k(tile + NW);   // in flight during the rest of the tile
        // lane j + 4 b + 16 i holds token 4 b + i, head j; wanted: lane of column n, tokens 4 g + i
        float xs[GH][2];
#pragma unroll
        for (int hh = 0; hh < GH; ++hh)
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            xd[hh][st] *= c_d;
            xs[hh][st] = (float)xd[hh][st];
          }
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int src = ((n16 & 3) + 4 * g + 16 * i) * 4;
            float v = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(xs[0][st])));
            if (GH == 2) {
              const float w = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(xs[GH - 1][st])));
              v = (n16 & 4) ? w : v;
            }
            x[st][i] = v;
          }
      } else {
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < KK; ++kk)
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[st][kk]), qf[kk], d, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) x[st][i] = d[i] * c;
        }
        if (more) load_k(tile + NW);
      }
      if (tile * TW + TW > Lold) {   // the last tile
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int i = 0; i < 4; ++i) x[st][i] = tile * TW + st * 16 + g * 4 + i < Lold ? x[st][i] : FG_NEG_BIG;
      }
      // The shift of a head moves when a logit exceeds it by more than 1: the large weights' exponents stay small
      // (and so their rounding), and the sums are rescaled a few times instead of once per tile.
      float mx = fmaxf(fmaxf(fmaxf(x[0][0], x[0][1]), fmaxf(x[0][2], x[0][3])), fmaxf(fmaxf(x[1][0], x[1][1]), fmaxf(x[1][2], x[1][3])));
      if (__any(mx > mw + 1.f)) {
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));   // over the lanes of the column
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = mx > mw + 1.f ? rintf(mx) : mw, f = fg_exp2(mw - m_new);
        mw = m_new;
        lsum *= f;
        if (KEEP) {
#pragma unroll
          for (int hh = 0; hh < GH; ++hh)
            z[hh] *= (double)__int_as_float(__builtin_amdgcn_ds_bpermute((hh * 4 + (lane & 3)) * 4, __float_as_int(f)));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float lo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), i));
          const float hi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), GP - 4 + i));
          const float fr = GP == 8 && (g & 1) ? hi : lo;
#pragma unroll
          for (int s = 0; s < NTL; ++s) acc[s][i] *= fr;
        }
      }
      if (KEEP) {
        if (lane < GP) s_shift[tile][lane] = mw;
#pragma unroll
        for (int hh = 0; hh < GH; ++hh) {
          const int h = hh * 4 + (lane & 3);
          const double m = (double)__int_as_float(__builtin_amdgcn_ds_bpermute(h * 4, __float_as_int(mw)));
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            const int slot = tile * TW + st * 16 + (n16 & 12) + g;
            const double e = exp2(xd[hh][st] - m);
            if (slot < Lold && h < G) {
              clogit[(size_t)slot * G + h] = e;
              z[hh] += e;
            }
          }
        }
      }
      // weights and the piece of each that this lane's row carries
      uint32_t piece[4], low[4];
      float l_t = 0.f;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          uint32_t b[2], r2[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float p = fg_exp2(x[st][i + e] - mw);
            l_t += p;
            const float r = p - __uint_as_float(__float_as_uint(p) & cut1);      // without the first 8 bits
            if (GP == 4) b[e] = __float_as_uint(r - __uint_as_float(__float_as_uint(r) & cut2));
            else {
              b[e] = __float_as_uint(r);
              r2[e] = __float_as_uint(r - __uint_as_float(__float_as_uint(r) & 0xffff0000u));
            }
          }
          piece[st * 2 + i / 2] = (b[0] >> 16) | (b[1] & 0xffff0000u);
          if (GP == 8) low[st * 2 + i / 2] = split ? (r2[0] >> 16) | (r2[1] & 0xffff0000u) : 0u;
        }
      lsum += l_t;
      const bf16x8 pa = __builtin_bit_cast(bf16x8, u32x4{piece[0], piece[1], piece[2], piece[3]});
      bf16x8 pl = pa;
      if (GP == 8) pl = __builtin_bit_cast(bf16x8, u32x4{low[0], low[1], low[2], low[3]});
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        const int row = i * TPL + v_row, p16 = lane % LPR;
        *reinterpret_cast<u32x4*>(&s_v[wave][v_place(row, p16 >> 1) + (p16 & 1) * 16]) = vf[i];
      }
      if (more) load_v(tile + NW);
#pragma unroll
      for (int s = 0; s < NTL; ++s) {
        const int row = 4 * g + (n16 >> 2);
        const uint2 v0 = fg_read_transposed(&s_v[wave][v_place(row, s) + (n16 & 3) * 8]);
        const uint2 v1 = fg_read_transposed(&s_v[wave][v_place(row + 16, s) + (n16 & 3) * 8]);
        const bf16x8 vb = __builtin_bit_cast(bf16x8, u32x4{v0.x, v0.y, v1.x, v1.y});
        acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, vb, acc[s], 0, 0, 0);
        if (GP == 8) acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl, vb, acc[s], 0, 0, 0);
      }
    }
  };
  if (scored) stream(std::true_type{});
  else stream(std::false_type{});

  // the new token: a partial of its own, and its row appended in the first free slot
  if (wave == NW - 1) {
    constexpr int EPL = 8;
    const int gl = lane % LPR, sub = lane / LPR;
    const u32x4 knew = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.k_new) + (size_t)u * RB + gl * 16);
    const u32x4 vnew = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.v_new) + (size_t)u * RB + gl * 16);
    float kn[EPL], vn[EPL];
    fg_unpack<2>(knew, kn);
    fg_unpack<2>(vnew, vn);
    if (sub == 0) {
      *reinterpret_cast<u32x4*>(static_cast<char*>(a.ck) + (off + Lold) * RB + gl * 16) = knew;
      *reinterpret_cast<u32x4*>(static_cast<char*>(a.cv) + (off + Lold) * RB + gl * 16) = vnew;
    }
    if (lane == 0) {
      a.cpos[off + Lold] = a.n + a.step;
      a.ccls[off + Lold] = a.class_new[u / a.units_per_seq];
      a.cscore[off + Lold] = 0.0;
    }
    for (int h = 0; h < G; ++h) {
      float qn[EPL];
      fg_unpack<2>(*reinterpret_cast<const u32x4*>(&s_q[h * RB + gl * 16]), qn);
      double dd = 0.0;   // one token: float64 for every policy
#pragma unroll
      for (int e = 0; e < EPL; ++e) dd = fma((double)qn[e], (double)kn[e], dd);
      dd = fg_group_sum_f64<LPR>(dd) * c_d;
      if (sub == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) s_o[NW][h][gl * EPL + e] = vn[e];
      }
      if (lane == 0) {
        s_m[NW][h] = (float)dd;
        s_l[NW][h] = 1.f;
        if (scored) {
          const double e = exp2(dd - (double)(float)dd);
          clogit[(size_t)Lold * G + h] = e;
          s_z[NW][h] = e;
        }
      }
    }
  }
  // this wave's partial
  if (wave < ntile) {
  lsum += __shfl_xor(lsum, 16, 64);
  lsum += __shfl_xor(lsum, 32, 64);
  if (lane < G) {   // columns of the first split
    s_m[wave][lane] = mw;
    s_l[wave][lane] = lsum;
  }
  if (scored) {
#pragma unroll
    for (int hh = 0; hh < GH; ++hh) {
#pragma unroll
      for (int m = 4; m < 64; m <<= 1) z[hh] += fg_shfl_xor_f64(z[hh], m);
      if (lane < 4 && hh * 4 + lane < G) s_z[wave][hh * 4 + lane] = z[hh];
    }
  }
  // The pieces lie in the four lane groups (two with eight heads): each exchange adds half of them and halves the
  // values a lane still carries.
  float half[NTL / 2][4];   // set 2 k in the lower groups, 2 k + 1 in the upper ones
#pragma unroll
  for (int k = 0; k < NTL / 2; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[2 * k][i]), __float_as_uint(acc[2 * k + 1][i]), false, false);
      half[k][i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      if (GP == 8) {
        const int h = 4 * (g & 1) + i;
        if (h < G) s_o[wave][h][(2 * k + (g >> 1)) * 16 + n16] = half[k][i];
      }
    }
  if (GP == 4) {
#pragma unroll
    for (int k = 0; k < NTL / 4; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(half[2 * k][i]), __float_as_uint(half[2 * k + 1][i]), false, false);
        const float o = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        if (i < G) s_o[wave][i][(4 * k + (g & 1) * 2 + (g >> 1)) * 16 + n16] = o;
      }
  }
  }
  auto merge = [&]() -> float {
    __syncthreads();   // also orders the appended slot and the kept exponentials before the update
    for (int q = tid; q < G * D; q += NT) {
      const int h = q / D, e = q % D;
      float M = s_m[NW][h];
#pragma unroll
      for (int i = 0; i < NW; ++i) if (i < ntile) M = fmaxf(M, s_m[i][h]);   // the others have had no tile
      const float f_new = fg_exp2(s_m[NW][h] - M);
      float o = s_o[NW][h][e] * f_new, l = s_l[NW][h] * f_new;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        if (i >= ntile) break;
        const float f = fg_exp2(s_m[i][h] - M);
        o += s_o[i][h][e] * f;
        l += s_l[i][h] * f;
      }
      fg_store_out<2>(a.out, (size_t)u * G * D + q, o * (1.0f / l));
    }
    if (scored) {
      for (int q = tid; q < (ntile + 1) * G; q += NT) {
        const int tile = q / G, h = q - tile * G;
        float m = rintf(s_m[NW][h]);
#pragma unroll
        for (int i = 0; i < NW; ++i) if (i < ntile) m = fmaxf(m, s_m[i][h]);
        const double fresh = exp2((double)s_m[NW][h] - (double)m);
        double sum = s_z[NW][h] * fresh;
#pragma unroll
        for (int i = 0; i < NW; ++i) if (i < ntile) sum += ldexp(s_z[i][h], (int)fmaxf(s_m[i][h] - m, -4096.f));
        const double inv = 1.0 / sum;
        if (tile == ntile) s_factor[TILES][h] = inv * fresh;
        else s_factor[tile][h] = ldexp(inv, (int)fmaxf(s_shift[tile][h] - m, -4096.f));
      }
      __syncthreads();
    }
    return 0.f;   // the update takes the ready attention, no shift
  };
  // this step's attention (float64) on a slot, summed over the heads
  auto attention = [&](int j) {
    const double* e = clogit + (size_t)j * G;
    const double* f = s_factor[j == Lold ? TILES : j / TW];
    double sum = 0.0;
#pragma unroll
    for (int h = 0; h < GM; ++h) if (h < G) sum = fma(e[h], f[h], sum);
    if (probing) clogit[(size_t)j * G] = sum;   // the probe reads it again, in the same thread
    return sum;
  };
  auto set_len = [&](int v) {
    if (tid == 0) { a.len[u] = v; rec_p[3] = v; }
  };
  if (policy >= 4 && !probing) {
    (void)merge();
    set_len(L);
    return;
  }
  fg_update_unit<2, D, true, NT, FG_UNIT_TOKENS>(a, u, L, cap, off, policy, comp, sh, merge, set_len, attention);
}

template <int GM>
hipError_t launch(const fg_decode_args& a, hipStream_t s) {
  const dim3 grid((unsigned)a.U), block(NT);
  if (a.d == 128) hipLaunchKernelGGL((fg_decode_group_mfma_kernel<128, GM>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((fg_decode_group_mfma_kernel<64, GM>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t fg_launch_decode_group_mfma(const fg_decode_args& a, hipStream_t s) {
  return a.G <= 4 ? launch<4>(a, s) : launch<8>(a, s);
}
