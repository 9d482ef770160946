// Block-wide exact selection of the k largest of m non-negative doubles with the tie rule
// "equal score -> the smaller position is kept" (the frequent policy of Sec. 3.4 keeps the
// tokens with the largest cumulative attention score). MSB-first radix select on the IEEE
// bit patterns (monotone for non-negative doubles), 8 bits per pass:
//   * the caller hands the keys over in registers (fg_select_topk_regs) or they are re-read in each pass
//     (fg_select_topk);
//   * passes over the bits that all keys share are skipped (block-wide OR/AND of the keys);
//   * the scan stops as soon as the boundary bucket is taken whole;
//   * only if the boundary value is shared does a second select run on the positions.
// NT = blockDim.x: a power of two from 256 to 1024.
#pragma once
#include "fg_common.h"


struct fg_topk {
  uint64_t thr;   // keys above thr are in; keys equal to thr are in iff pos <= pthr
  uint32_t pthr;
  int mode;       // 0: nothing selected, 1: everything selected, 2: use (thr, pthr)
};

struct fg_select_smem {
  int hist[256];
  int red[20];
  unsigned long long w_or[16], w_and[16];
  int digit, rem, cnt;
};

__device__ __forceinline__ bool fg_in_topk(const fg_topk& t, double score, uint32_t pos) {
  if (t.mode != 2) return t.mode == 1;
  const uint64_t key = (uint64_t)__double_as_longlong(score);
  return key > t.thr || (key == t.thr && pos <= t.pthr);
}

// hist[digit] += 1 for every lane with `active`; lanes sharing the digit of the first active
// lane are counted with one atomic (keys cluster in few buckets during the first passes).
__device__ __forceinline__ void fg_hist_add(int* hist, bool active, int digit) {
  const unsigned long long act = __ballot(active);
  if (act == 0ull) return;
  const int leader = __ffsll((long long)act) - 1;
  const int d0 = __builtin_amdgcn_readlane(digit, leader);  // `leader` is wave-uniform
  const bool same = active && digit == d0;
  const unsigned long long grp = __ballot(same);
  if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[d0], (int)__popcll(grp));
  if (active && !same) atomicAdd(&hist[digit], 1);
}

// After the histogram of one digit is complete: locate the bucket that holds the rem-th
// largest. Thread t < 256 looks at bucket 255 - t (descending order).
__device__ __forceinline__ void fg_radix_locate(int rem, fg_select_smem* sm) {
  const int tid = threadIdx.x;
  const int h = tid < 256 ? sm->hist[255 - tid] : 0;
  int total;
  const int before = fg_block_exscan_i32(h, sm->red, &total);
  if (before < rem && before + h >= rem) {
    sm->digit = 255 - tid;
    sm->rem = rem - before;
    sm->cnt = h;
  }
  __syncthreads();
}

// NC > 0: element tid + NT i of the block is kc[i] (registers); NC == 0: keys come from score(j).
template <int NT, int NC, class ScoreFn, class PosFn>
__device__ __forceinline__ fg_topk fg_select_topk_impl(const uint64_t (&kc)[NC > 0 ? NC : 1], ScoreFn score,
                                                       PosFn pos, int m, int k, fg_select_smem* sm) {
  constexpr bool CACHED = NC > 0;
  fg_topk r;
  r.thr = 0; r.pthr = 0xffffffffu; r.mode = 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // ---- the bits the keys do not all share
  uint64_t k_or = 0, k_and = ~0ull;
  if (CACHED) {
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      if (j < m) {
        k_or |= kc[i];
        k_and &= kc[i];
      }
    }
  } else {
    for (int j = tid; j < m; j += NT) {
      const uint64_t key = (uint64_t)__double_as_longlong(score(j));
      k_or |= key;
      k_and &= key;
    }
  }
  {
    unsigned long long wo, wa;
    fg_wave_or_and_u64(k_or, k_and, &wo, &wa);
    k_or = wo;
    k_and = wa;
  }
  __syncthreads();
  if (lane == 0) { sm->w_or[wave] = k_or; sm->w_and[wave] = k_and; }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) { k_or |= sm->w_or[i]; k_and &= sm->w_and[i]; }
  const uint64_t diff = k_or ^ k_and;

  uint64_t prefix = 0, mask = 0;
  int rem = k, n_eq = m;
  if (diff != 0) {
    const int top = 63 - __clzll((long long)diff);  // highest bit in which two keys differ
    int shift = (top >> 3) << 3;
    mask = (shift + 8 >= 64) ? 0ull : ~((1ull << (shift + 8)) - 1ull);
    prefix = k_and & mask;
    for (; shift >= 0; shift -= 8) {
      if (tid < 256) sm->hist[tid] = 0;
      __syncthreads();
      if (CACHED) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int j = tid + NT * i;
          fg_hist_add(sm->hist, j < m && (kc[i] & mask) == prefix, (int)((kc[i] >> shift) & 255u));
        }
      } else {
        for (int j = tid; j < m; j += NT) {
          const uint64_t key = (uint64_t)__double_as_longlong(score(j));
          if ((key & mask) == prefix) atomicAdd(&sm->hist[(int)((key >> shift) & 255u)], 1);
        }
      }
      __syncthreads();
      fg_radix_locate(rem, sm);
      prefix |= (uint64_t)sm->digit << shift;
      mask |= (uint64_t)0xff << shift;
      rem = sm->rem;
      n_eq = sm->cnt;
      if (rem == n_eq) {  // the boundary bucket is taken whole: every key >= prefix is in
        r.thr = prefix;
        return r;
      }
    }
  } else {
    prefix = k_and;  // all keys are equal
  }
  r.thr = prefix;
  if (rem == n_eq) return r;
  // ties at the boundary value: keep the `rem` smallest positions among the tied elements,
  // i.e. select the rem-th largest of (~pos) over them
  const uint64_t thr = prefix;
  uint64_t p2 = 0, m2 = 0;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) sm->hist[tid] = 0;
    __syncthreads();
    for (int j = tid; j < m; j += NT) {
      if ((uint64_t)__double_as_longlong(score(j)) != thr) continue;
      const uint64_t key = (uint64_t)(0xffffffffu - pos(j));
      if ((key & m2) == p2) atomicAdd(&sm->hist[(int)((key >> shift) & 255u)], 1);
    }
    __syncthreads();
    fg_radix_locate(rem, sm);
    p2 |= (uint64_t)sm->digit << shift;
    m2 |= (uint64_t)0xff << shift;
    rem = sm->rem;
  }
  r.pthr = 0xffffffffu - (uint32_t)p2;
  return r;
}

// Keys already in registers (element tid + NT i is kc[i], i < NC, valid while < m).
// score(j) / pos(j) are only consulted if the boundary value is tied.
template <int NT, int NC, class ScoreFn, class PosFn>
__device__ __forceinline__ fg_topk fg_select_topk_regs(const uint64_t (&kc)[NC], ScoreFn score, PosFn pos,
                                                       int m, int k, fg_select_smem* sm) {
  fg_topk r;
  r.thr = 0; r.pthr = 0;
  if (k <= 0) { r.mode = 0; return r; }
  if (k >= m) { r.mode = 1; return r; }
  return fg_select_topk_impl<NT, NC>(kc, score, pos, m, k, sm);
}

// Shortcut for the per-step kept-set update. Only tokens that nothing else protects (`prot`
// bit clear) can leave, and they leave lowest score first: a token is outside the top k exactly
// if at least k scores are larger. So instead of locating the k-th largest score, test the
// lowest unprotected score, then the next one, ... until one stays (a step evicts very few
// tokens). Returns false when the shortcut does not apply -- two equal scores at a tested value,
// or more than FG_EVICT_TRIES evictions -- and the caller runs the full selection instead.
// On success every unprotected token with key >= out->thr is in the top k (mode 2, no position
// tie-break needed); left[0, *left_count) (shared memory, visible after the next barrier) are the
// slots of the tokens that leave. Keys of slot tid + NT i are kc[i] (valid while < m).
// Two barriers per test: the buffers of odd and even tests take turns, so that two barriers lie between a read and the next
// write (with one buffer four barriers, 256 units of 2048 tokens with four heads 37.3 us per step, 33.7 so; 4 units of 128,
// float32, 6.4 and 5.9). Two values per round, for half of the rounds, gained nothing: their minima cost as much.
#define FG_EVICT_TRIES 6
struct fg_evict_smem {
  double low[2][16];
  int count[2][16];
};
template <int NT, int NC>
__device__ __forceinline__ bool fg_evict_cut_regs(const uint64_t (&kc)[NC], uint32_t prot, int m, int k,
                                                  fg_evict_smem& sh, int* left, int* left_count,
                                                  fg_topk* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  double last = -1.0;  // every evicted score so far is <= last
  for (int it = 0; it < FG_EVICT_TRIES; ++it) {
    double loc = inf;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      const double v = __longlong_as_double((long long)kc[i]);
      if (j < m && !((prot >> i) & 1u) && v > last) loc = fmin(loc, v);
    }
    loc = fg_wave_min_f64(loc);
    if (lane == 0) sh.low[it & 1][wave] = loc;
    __syncthreads();
    double kmin = sh.low[it & 1][0];
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) kmin = fmin(kmin, sh.low[it & 1][i]);
    out->mode = 2; out->pthr = 0xffffffffu;
    if (kmin == inf) {  // no unprotected token is left: none of them is in the top k
      *left_count = it;
      out->thr = 0x7ff0000000000000ull;
      return true;
    }
    int cnt = 0;  // scores above kmin in the low half, scores equal to it in the high half
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = tid + NT * i;
      const double v = __longlong_as_double((long long)kc[i]);
      if (j < m) cnt += (v > kmin ? 1 : 0) + (v == kmin ? (1 << 16) : 0);
    }
    cnt = fg_wave_sum_i32(cnt);
    if (lane == 0) sh.count[it & 1][wave] = cnt;
    __syncthreads();
    int tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) tot += sh.count[it & 1][i];
    if ((tot >> 16) != 1) return false;       // a tie at the tested value: needs the position rule
    if ((tot & 0xffff) < k) {                  // fewer than k larger scores: it stays, and so do all above it
      *left_count = it;
      out->thr = (uint64_t)__double_as_longlong(kmin);
      return true;
    }
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if (tid + NT * i < m && __longlong_as_double((long long)kc[i]) == kmin) left[it] = tid + NT * i;
    last = kmin;                               // at least k larger scores: it leaves; test the next one
  }
  return false;
}

// Keys from score(j), re-read in every pass. ScoreFn(j) -> double (>= 0), PosFn(j) -> uint32 position
// (unique per element).
template <int NT, class ScoreFn, class PosFn>
__device__ __forceinline__ fg_topk fg_select_topk(ScoreFn score, PosFn pos, int m, int k,
                                                  fg_select_smem* sm) {
  fg_topk r;
  r.thr = 0; r.pthr = 0;
  if (k <= 0) { r.mode = 0; return r; }
  if (k >= m) { r.mode = 1; return r; }
  const uint64_t none[1] = {0ull};
  return fg_select_topk_impl<NT, 0>(none, score, pos, m, k, sm);
}
