// The kept-set update of one unit after a decode step (Alg. 2: f again, with the head's policy):
// cumulative scores += this step's attention (policies with `frequent`, or every policy when the
// step is probed), kept = special | punct | TopK(score, k_f(L)) | window, in-place release of the
// evicted slots, and the probe's masses. Shared by the forms of a decode step (decode.hip, decode_unit.hip,
// decode_group.hip and decode_group_mfma.hip). One workgroup of NT threads calls it for its unit.
#pragma once
#include "fg_common.h"
#include "fg_internal.h"
#include "fg_select.h"

constexpr int FG_MOVE_LDS = 64;  // released slots per step whose move lists stay in shared memory

struct fg_update_smem {
  fg_select_smem sm;
  double dred[16];
  int ired[20];
  double zred[16];       // used once per step: no barrier in front of the write
  fg_evict_smem cut;
  int move[2 * FG_MOVE_LDS];
};

// Fast path (L <= NT * NC): each thread keeps its slots' updated scores and a "protected"
// bit (special / punctuation / window) in registers, so every later phase is register-only.
// The code below is straight-line per slot, i.e. executed once per workgroup and bound by
// instruction fetch: it is instantiated for a few sizes and the smallest one that fits is taken.
// Score path in float64 (Sec. 3.4, cumulative attention score): this step's attention on held slot
// j is a_j = 2^(x_j - M) / Z with the float64 logits x_j the attention kept and Z = sum_j 2^(x_j - M)
// summed here in float64 (M is only a shift: the float maximum). Grouped heads: `logit` gives the attention
// summed over the heads, from clogit[j, 0] or (three to eight bf16 heads in one workgroup per unit) as the sum of
// the slot's kept exponentials times its tile's factors, which it leaves in clogit[j, 0] for the probe.
// The bookkeeping of the held tokens is on its way while `merge` runs (the attention output and the
// maximum M of the scaled logits, from LDS or memory; it holds the barrier after which the logits
// and the appended slot of this step may be read). The new token's bookkeeping is known here.
template <int ESIZE, int D, bool GRP, int NT, int NC, bool LAST, class Merge, class SetLen, class Logit>
__device__ __forceinline__ void fg_update_kept(const fg_decode_args& a, int u, int L, int cap, int64_t off,
                                               int policy, int comp, fg_update_smem& sh, Merge merge,
                                               SetLen set_len, Logit logit) {
  constexpr int RB = D * ESIZE, CPR = RB / 16;
  const int tid = threadIdx.x;
  const int G = GRP ? a.G : 1;
  const bool freq = (comp & FG_COMP_FREQUENT) != 0;
  const bool probing = a.probe != nullptr;
  const bool scored = freq || probing;
  const int p_new = a.n + a.step;
  double* score = a.cscore + off;
  const int32_t* pos = a.cpos + off;
  const uint8_t* cls = a.ccls + off;
  const int cmask = ((comp & FG_COMP_SPECIAL) ? FG_CLASS_SPECIAL : 0) | ((comp & FG_COMP_PUNCT) ? FG_CLASS_PUNCT : 0);
  const int wlo = (comp & FG_COMP_LOCAL) ? p_new - a.w : 0x7fffffff;  // positions above wlo are inside the window

  uint64_t kc[NC];
  uint32_t prot = 0;
  const bool small = !LAST || L <= NT * NC;   // only the largest instantiation meets longer units
  double inv_d = 0.0;   // 1 / Z (without grouping)
  fg_topk tk;
  tk.mode = 0; tk.thr = 0; tk.pthr = 0;
  float M = 0.f;
  int evicted = -1;     // tokens that leave, where the shortcut below has found them out
  if (small) {
    // all loads first (they are independent), then the arithmetic, then the stores
    double lg[NC];
    double sc[NC];
    int cb[NC], pj[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      cb[i] = 0; pj[i] = 0; sc[i] = 0.0;
      if (j < L - 1) {
        cb[i] = cls[j];
        pj[i] = pos[j];
        if (scored) sc[i] = score[j];
      }
    }
    const int c_new = a.class_new[u / a.units_per_seq];
    M = merge();
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      lg[i] = 0.0;
      if (scored && j < L) lg[i] = logit(j);
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      kc[i] = 0;
      if (j == L - 1) { cb[i] = c_new; pj[i] = p_new; }
      if (j < L && ((cb[i] & cmask) != 0 || pj[i] > wlo)) prot |= 1u << i;
    }
    if (scored) {
      if (!GRP) {
        // 2^(x_j - M) in place of the logits, their float64 sum over the workgroup
        double z = 0.0;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int j = tid + NT * i;
          if (j < L) {
            lg[i] = exp2(lg[i] - (double)M);
            z += lg[i];
          }
        }
        z = fg_wave_sum_f64(z);
        if ((tid & 63) == 0) sh.zred[tid >> 6] = z;
        __syncthreads();
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) t += sh.zred[i];
        inv_d = 1.0 / t;
      }
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int j = tid + NT * i;
        if (j < L) {
          // cumulative attention score += this step's attention (Sec. 3.4, frequency policy)
          const double v = sc[i] + (GRP ? lg[i] : lg[i] * inv_d);
          score[j] = v;
          kc[i] = (uint64_t)__double_as_longlong(v);
        }
      }
    }
    if (scored) {
      const int k_f = fg_budget(a.r_f, p_new + 1);
      // without the probe only the unprotected tokens' membership matters: try the lowest ones
      bool done = false;
      if (!probing && k_f > 0 && k_f < L && L <= 0xffff)
        done = fg_evict_cut_regs<NT, NC>(kc, prot, L, k_f, sh.cut, sh.move, &evicted, &tk);
      if (!done) {
        evicted = -1;
        __syncthreads();  // score[] is re-read by other threads only if the boundary value is tied
        tk = fg_select_topk_regs<NT, NC>(kc, [&](int j) { return score[j]; },
                                     [&](int j) { return (uint32_t)pos[j]; }, L, k_f, &sh.sm);
      }
    }
  } else {
    M = merge();
  }
  if (!small && scored) {
    if (!GRP) {
      double z = 0.0;
      for (int j = tid; j < L; j += NT) z += exp2(a.clogit[off + j] - (double)M);
      inv_d = 1.0 / fg_block_sum_f64(z, sh.dred);
    }
    for (int j = tid; j < L; j += NT) {
      const double aj = GRP ? a.clogit[(off + j) * G] : exp2(a.clogit[off + j] - (double)M) * inv_d;
      score[j] += aj;
    }
    __syncthreads();
    const int k_f = fg_budget(a.r_f, p_new + 1);
    tk = fg_select_topk<NT>([&](int j) { return score[j]; }, [&](int j) { return (uint32_t)pos[j]; }, L, k_f, &sh.sm);
  }
  if (probing) {
    // Stability probe (Sec. 4): mass of this step's attention row on every family member's
    // tokens among the held ones (frequent = the top-k just selected, local = last w positions)
    double r[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int j = tid; j < L; j += NT) {
      // the mean of the G heads' rows
      const double aj = GRP ? a.clogit[(off + j) * G] / (double)G
                            : exp2(logit(j) - (double)M) * inv_d;
      const int c = cls[j];
      const bool top = fg_in_topk(tk, score[j], (uint32_t)pos[j]), recent = pos[j] > p_new - a.w;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int m = a.family[p];
        const bool in = ((m & FG_COMP_SPECIAL) && (c & FG_CLASS_SPECIAL)) || ((m & FG_COMP_PUNCT) && (c & FG_CLASS_PUNCT)) ||
                        ((m & FG_COMP_FREQUENT) && top) || ((m & FG_COMP_LOCAL) && recent);
        r[p] += in ? aj : 0.0;
      }
      r[4] += aj;
    }
#pragma unroll
    for (int p = 0; p < 5; ++p) {
      const double t = fg_block_sum_f64(r[p], sh.dred);
      if (tid == 0) a.probe[(size_t)u * 5 + p] = t;
    }
    if (policy >= 4) {
      set_len(L);
      return;
    }
  }
  char* ck = static_cast<char*>(a.ck) + off * RB;
  char* cv = static_cast<char*>(a.cv) + off * RB;
  // CPR lanes copy the row pair, one more moves score / position / class
  auto move_slot = [&](int ch, int dst, int src) {
    if (ch < CPR) {
      const u32x4 kr = *reinterpret_cast<const u32x4*>(ck + (size_t)src * RB + ch * 16);
      const u32x4 vr = *reinterpret_cast<const u32x4*>(cv + (size_t)src * RB + ch * 16);
      *reinterpret_cast<u32x4*>(ck + (size_t)dst * RB + ch * 16) = kr;
      *reinterpret_cast<u32x4*>(cv + (size_t)dst * RB + ch * 16) = vr;
    } else {
      const double sv = score[src];
      const int pv = pos[src];
      const uint8_t cb = cls[src];
      score[dst] = sv;
      a.cpos[off + dst] = pv;
      a.ccls[off + dst] = cb;
    }
  };
  if (small && freq && evicted >= 0) {
    // the usual step: sh.move holds the slots of the few tokens that leave
    const int new_len = L - evicted;
    set_len(new_len);
    if (evicted == 0) return;
    __syncthreads();   // also orders the updated scores before the moves
    if (evicted == 1) {
      // the last slot fills the hole
      if (sh.move[0] < new_len && tid <= CPR) move_slot(tid, sh.move[0], new_len);
      return;
    }
    // pair the holes below the new length with the kept slots above it
    if (tid == 0) {
      int moves = 0, src = new_len;
      for (int i = 0; i < evicted; ++i) {
        const int dst = sh.move[i];
        if (dst >= new_len) continue;
        for (bool out = true; out; ++src) {
          out = false;
          for (int k = 0; k < evicted; ++k) out = out || sh.move[k] == src;
        }
        sh.move[FG_MOVE_LDS + moves] = src - 1;
        sh.move[FG_MOVE_LDS + FG_EVICT_TRIES + moves] = dst;
        ++moves;
      }
      sh.ired[0] = moves;
    }
    __syncthreads();
    for (int q = tid; q < sh.ired[0] * (CPR + 1); q += NT) {
      const int i = q / (CPR + 1);
      move_slot(q % (CPR + 1), sh.move[FG_MOVE_LDS + FG_EVICT_TRIES + i], sh.move[FG_MOVE_LDS + i]);
    }
    return;
  }
  const bool tie_pos = (tk.mode == 2 && tk.pthr != 0xffffffffu);  // rare: boundary value shared
  auto kept = [&](int j) -> bool {  // from memory (large units and the tied case)
    bool k = (cls[j] & cmask) != 0 || pos[j] > wlo;
    if (freq) k = k || fg_in_topk(tk, score[j], (uint32_t)pos[j]);
    return k;
  };
  uint32_t keepbits = 0;  // fast path: bit i = slot tid + NT i stays
  int mine = 0;
  if (small) {
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      if (j < L) {
        bool k = (prot >> i) & 1u;
        if (freq && !k) {
          if (tk.mode == 1) k = true;
          else if (tk.mode == 2) k = tie_pos ? fg_in_topk(tk, __longlong_as_double((long long)kc[i]), (uint32_t)pos[j])
                                             : (kc[i] >= tk.thr);
        }
        if (k) { keepbits |= 1u << i; ++mine; }
      }
    }
  } else {
    for (int j = tid; j < L; j += NT) mine += kept(j) ? 1 : 0;
  }
  const int new_len = fg_block_sum_i32(mine, sh.ired);
  if (new_len == L) {
    set_len(L);
    return;
  }

  // ---- in-place release: i-th hole (evicted slot below new_len) <- i-th kept slot above it
  int* scratch = reinterpret_cast<int*>(a.clogit + off * G);  // logits are dead from here on (cap ints fit in cap doubles)
  int* s_move = sh.move;
  bool in_lds = false;
  __syncthreads();
  int run_h = 0, run_m = 0;
  if (small) {
    // any one-to-one pairing of holes and movers will do: number them thread by thread
    int nh = 0, nm = 0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      if (j < L) {
        const bool k = (keepbits >> i) & 1u;
        nh += (j < new_len && !k) ? 1 : 0;
        nm += (j >= new_len && k) ? 1 : 0;
      }
    }
    // one scan for both counts (each below 2^16: L <= NT * NC)
    int tot;
    const int at = fg_block_exscan_i32(nh | (nm << 16), sh.ired, &tot);
    int at_h = at & 0xffff, at_m = at >> 16;
    run_h = tot & 0xffff;
    run_m = tot >> 16;
    // a step releases very few slots: the two lists then stay in shared memory
    in_lds = run_h <= FG_MOVE_LDS;
    int* holes = in_lds ? s_move : scratch;
    int* movers_end = in_lds ? s_move + 2 * FG_MOVE_LDS - 1 : scratch + cap - 1;  // filled downwards
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      if (j < L) {
        const bool k = (keepbits >> i) & 1u;
        if (j < new_len && !k) holes[at_h++] = j;
        if (j >= new_len && k) *(movers_end - (at_m++)) = j;
      }
    }
    __syncthreads();
  } else {
    for (int base = 0; base < L; base += NT) {
      const int j = base + tid;
      int is_h = 0, is_m = 0;
      if (j < L) {
        const bool k = kept(j);
        is_h = (j < new_len && !k) ? 1 : 0;
        is_m = (j >= new_len && k) ? 1 : 0;
      }
      int tot_h, tot_m;
      const int ex_h = fg_block_exscan_i32(is_h, sh.ired, &tot_h);
      __syncthreads();
      const int ex_m = fg_block_exscan_i32(is_m, sh.ired, &tot_m);
      if (is_h) scratch[run_h + ex_h] = j;
      if (is_m) scratch[cap - 1 - (run_m + ex_m)] = j;
      run_h += tot_h;
      run_m += tot_m;
      __syncthreads();
    }
  }
  const int moves = run_h;  // == run_m
  // the kept() predicate of the large-unit path reads score/pos/cls from memory: there the
  // bookkeeping moves only after every thread is done with it
  if (!small) {
    for (int q = tid; q < moves * CPR; q += NT) {
      const int i = q / CPR, ch = q % CPR;
      const int dst = scratch[i], src = scratch[cap - 1 - i];
      *reinterpret_cast<u32x4*>(ck + (size_t)dst * RB + ch * 16) = *reinterpret_cast<const u32x4*>(ck + (size_t)src * RB + ch * 16);
      *reinterpret_cast<u32x4*>(cv + (size_t)dst * RB + ch * 16) = *reinterpret_cast<const u32x4*>(cv + (size_t)src * RB + ch * 16);
    }
    __syncthreads();
    for (int i = tid; i < moves; i += NT) {
      const int dst = scratch[i], src = scratch[cap - 1 - i];
      score[dst] = score[src];
      a.cpos[off + dst] = pos[src];
      a.ccls[off + dst] = cls[src];
    }
  } else {
    // rows and bookkeeping in one sweep
    for (int q = tid; q < moves * (CPR + 1); q += NT) {
      const int i = q / (CPR + 1);
      move_slot(q % (CPR + 1), in_lds ? s_move[i] : scratch[i],
                in_lds ? s_move[2 * FG_MOVE_LDS - 1 - i] : scratch[cap - 1 - i]);
    }
  }
  set_len(new_len);
}

// The smallest instantiation whose register slots hold the unit. MAX: the longest unit that the calling
// kernel can meet (0: any length, the part above the registers from memory).
// `logit` gives the logit of a slot that the thread owns (grouped heads: its attention).
template <int ESIZE, int D, bool GRP, int NT, int MAX, class Merge, class SetLen, class Logit>
__device__ __forceinline__ void fg_update_unit(const fg_decode_args& a, int u, int L, int cap, int64_t off,
                                               int policy, int comp, fg_update_smem& sh, Merge merge,
                                               SetLen set_len, Logit logit) {
#define FG_UPDATE(NC, LAST) fg_update_kept<ESIZE, D, GRP, NT, NC, LAST>(a, u, L, cap, off, policy, comp, sh, merge, set_len, logit)
  if (L <= NT * 1) FG_UPDATE(1, false);
  else if (L <= NT * 2) FG_UPDATE(2, false);
  else if (L <= NT * 4) FG_UPDATE(4, false);
  else if ((MAX != 0 && MAX <= NT * 8) || L <= NT * 8) FG_UPDATE(8, false);
  else FG_UPDATE(12, (MAX == 0 || MAX > NT * 12));
#undef FG_UPDATE
}
template <int ESIZE, int D, bool GRP, int NT, int MAX, class Merge, class SetLen>
__device__ __forceinline__ void fg_update_unit(const fg_decode_args& a, int u, int L, int cap, int64_t off,
                                               int policy, int comp, fg_update_smem& sh, Merge merge,
                                               SetLen set_len) {
  const int G = GRP ? a.G : 1;
  fg_update_unit<ESIZE, D, GRP, NT, MAX>(a, u, L, cap, off, policy, comp, sh, merge, set_len,
                                         [&](int j) { return a.clogit[(off + j) * G]; });
}
