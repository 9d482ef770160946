// Policy choice and compaction (Alg. 1: "C <- apply Eq. 1 to A", "K^,V^ <- f(K,V,C)").
//
//   fg_classify_kernel token ids -> class bytes (special / punctuation).
//   fg_select_kernel   per unit: the kept sets of the policy family (by default Eq. 2's:
//                      special, +punctuation, +frequent, +local; "+" = union; any table of
//                      component masks is accepted), their recoveries from the column /
//                      band sums, the cheapest policy reaching T (Eq. 1), kept flags and
//                      their prefix scan.
//   fg_offsets_kernel  exclusive scan of the per-unit slot reservations -> pool offsets,
//                      and the static work list of the decode kernels (split-KV items, or the
//                      units by size).
//   fg_gather_kernel   copies the kept rows of K, V with score, position, class.
//   fg_export_kernel   cache state read-back in ascending position order.
#include <type_traits>

#include "fg_common.h"
#include "fg_internal.h"
#include "fg_select.h"

namespace {

// Token ids -> class bytes (Sec. 3.4: which tokens C_special / C_punct. keep). The two id lists
// are small and arrive by value; every thread compares its token with all of them.
__global__ __launch_bounds__(256) void fg_classify_kernel(fg_classify_args a) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.count) return;
  const int32_t id = a.token_ids[i];
  int c = 0;
  for (int k = 0; k < a.num_special; ++k) c |= (id == a.special[k]) ? FG_CLASS_SPECIAL : 0;
  for (int k = 0; k < a.num_punct; ++k) c |= (id == a.punct[k]) ? FG_CLASS_PUNCT : 0;
  a.token_class[i] = (uint8_t)c;
}

// Latency-bound: one workgroup's chain of loads and block reductions per unit. With NC > 0 (n <= NT *
// NC) every token's column sum, band sum and class stay in registers (token tid + NT i in slot i),
// loaded once and all at once, and the prefix scan of the kept flags takes two barriers. Sums that several
// workgroups of a short prompt left in parts are added here, in order, three parts' loads in flight: a launch
// of their own, fg_part_sum_kernel, took 3.4 us of 32 units of 333 tokens in six parts.
struct fg_no_parts {};
template <int NT, int NC, class Parts>
__global__ __launch_bounds__(NT) void fg_select_kernel(fg_select_args a, Parts ps) {
  __shared__ fg_select_smem sm;
  __shared__ double part_r[NT / 64][4], sum_r[4];
  __shared__ int part_n[NT / 64][8], sum_n[8];
  __shared__ int ired[20];
  const int u = blockIdx.x, tid = threadIdx.x, n = a.n;
  const double* cs = a.colsum + (size_t)u * n;
  const double* bc = a.bandcol + (size_t)u * n;
  const uint8_t* cls = a.token_class + (size_t)(u / a.units_per_seq) * n;
  const int k_f = fg_budget(a.r_f, n);
  const int w = a.w;

  constexpr bool REGS = NC > 0;
  constexpr int NR = REGS ? NC : 1;
  uint64_t key[NR];
  double band[NR];
  int cl[NR];
  if constexpr (REGS && std::is_same<Parts, fg_part_sums>::value) {
    const size_t N = (size_t)a.U * n, at = (size_t)u * n;
    double sum[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = min(tid + NT * i, n - 1);
      sum[i] = ps.col[at + j];
      band[i] = ps.band[at + j];
      cl[i] = cls[j];
    }
    for (int p = 1; p < ps.parts; p += 3) {
      double s[3][NR], b[3][NR];
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          const size_t from = min(p + q, ps.parts - 1) * N + at + min(tid + NT * i, n - 1);
          s[q][i] = ps.col[from];
          b[q][i] = ps.band[from];
        }
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          sum[i] = p + q < ps.parts ? sum[i] + s[q][i] : sum[i];
          band[i] = p + q < ps.parts ? band[i] + b[q][i] : band[i];
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = tid + NT * i;
      if (j < n) a.colsum[at + j] = sum[i];   // the scores that the compaction hands on
      else { sum[i] = 0.0; band[i] = 0.0; cl[i] = 0; }
      key[i] = (uint64_t)__double_as_longlong(sum[i]);
    }
  } else if (REGS) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = tid + NT * i;
      key[i] = 0; band[i] = 0.0; cl[i] = 0;
      if (j < n) {
        key[i] = (uint64_t)__double_as_longlong(cs[j]);
        band[i] = bc[j];
        cl[i] = cls[j];
      }
    }
  }
  fg_topk tk;
  if (REGS) tk = fg_select_topk_regs<NT, NR>(key, [&](int j) { return cs[j]; }, [&](int j) { return (uint32_t)j; }, n, k_f, &sm);
  else tk = fg_select_topk<NT>([&](int j) { return cs[j]; }, [&](int j) { return (uint32_t)j; }, n, k_f, &sm);

  // Recovery of a policy = mean over rows of the kept attention mass. A column in the
  // policy's static set (special / punctuation / frequent) counts in every row: its column
  // sum; any other column is only seen through the local band, if the policy has one.
  double r[4] = {0.0, 0.0, 0.0, 0.0};
  int cnt[4] = {0, 0, 0, 0}, ccnt[4] = {0, 0, 0, 0};
  auto add_token = [&](int j, double s, double b, int c) {
    const bool top = fg_in_topk(tk, s, (uint32_t)j), tail = j >= n - w;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int m = a.family[p];
      const bool byclass = ((m & FG_COMP_SPECIAL) && (c & FG_CLASS_SPECIAL)) ||
                           ((m & FG_COMP_PUNCT) && (c & FG_CLASS_PUNCT));
      const bool st = byclass || ((m & FG_COMP_FREQUENT) && top);
      const bool loc = (m & FG_COMP_LOCAL) != 0;
      r[p] += st ? s : (loc ? b : 0.0);
      if (st || (loc && tail)) cnt[p]++;
      if (byclass) ccnt[p]++;
    }
  };
  if (REGS) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (tid + NT * i < n) add_token(tid + NT * i, __longlong_as_double((long long)key[i]), band[i], cl[i]);
  } else {
    for (int j = tid; j < n; j += NT) add_token(j, cs[j], bc[j], cls[j]);
  }
  // the twelve block sums in one round: waves first, then one thread per sum in wave order
  double R[5];
  int C[5], CC[4];
  {
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double rs = fg_wave_sum_f64(r[c]);
      const int n1 = fg_wave_sum_i32(cnt[c]), n2 = fg_wave_sum_i32(ccnt[c]);
      if (lane == 0) { part_r[wave][c] = rs; part_n[wave][c] = n1; part_n[wave][4 + c] = n2; }
    }
    __syncthreads();
    if (tid < 4) {
      double t = 0.0;
      for (int i = 0; i < NT / 64; ++i) t += part_r[i][tid];
      sum_r[tid] = t;
    } else if (tid < 12) {
      int t = 0;
      for (int i = 0; i < NT / 64; ++i) t += part_n[i][tid - 4];
      sum_n[tid - 4] = t;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      R[c] = sum_r[c] / ((double)n * (double)a.G);  // mean over the rows of all G query heads
      C[c] = sum_n[c];
      CC[c] = sum_n[4 + c];
    }
  }
  R[4] = 1.0;
  C[4] = n;
  // Eq. 1: the cheapest usable policy whose recovery reaches T; equal cost -> smaller id.
  // C_full always qualifies. (For the nested family of Eq. 2 this is the first id reaching T.)
  int policy = 4;
  for (int c = 3; c >= 0; --c)
    if (a.family[c] != 0 && R[c] >= a.T && C[c] <= C[policy]) policy = c;
  if (a.forced_policy >= 0) policy = a.forced_policy;
  const int comp = policy < 4 ? a.family[policy] : 0;

  // kept flags of the chosen policy and their exclusive scan (slot of each kept token)
  int running = 0;
  auto kept = [&](int j, double s, int c) {
    bool k = policy >= 4;
    if (comp & FG_COMP_SPECIAL) k = k || (c & FG_CLASS_SPECIAL) != 0;
    if (comp & FG_COMP_PUNCT) k = k || (c & FG_CLASS_PUNCT) != 0;
    if (comp & FG_COMP_FREQUENT) k = k || fg_in_topk(tk, s, (uint32_t)j);
    if (comp & FG_COMP_LOCAL) k = k || (j >= n - w);
    return k;
  };
  auto store = [&](int j, bool k, int c, int slot) {
    a.keep[(size_t)u * n + j] = (uint8_t)(k ? (4 | (c & 3)) : 0);  // kept flag plus the token's class bits
    a.slot[(size_t)u * n + j] = slot;
  };
  if (REGS) {
    // kept tokens per (slot i, wave) = per 64 consecutive positions, their scan by wave 0
    constexpr int NW = NT / 64;
    const int lane = tid & 63, wave = tid >> 6;
    __shared__ int s_count[NR * NW], s_total;
    unsigned long long flags[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = tid + NT * i;
      flags[i] = __ballot(j < n && kept(j, __longlong_as_double((long long)key[i]), cl[i]));
      if (lane == 0) s_count[i * NW + wave] = (int)__popcll(flags[i]);
    }
    __syncthreads();
    if (wave == 0) {
      int base = 0;
      for (int q = 0; q < NR * NW; q += 64) {
        const int v = q + lane < NR * NW ? s_count[q + lane] : 0;
        const int inc = fg_wave_incscan_i32(v);
        if (q + lane < NR * NW) s_count[q + lane] = base + inc - v;
        base += fg_readlane_i32(inc, 63);
      }
      if (lane == 0) s_total = base;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int j = tid + NT * i;
      if (j < n) store(j, (flags[i] >> lane) & 1ull, cl[i], s_count[i * NW + wave] + (int)__popcll(flags[i] & ((1ull << lane) - 1ull)));
    }
    running = s_total;
  } else {
    for (int base = 0; base < n; base += NT) {
      const int j = base + tid;
      const int c = j < n ? cls[j] : 0;
      const bool k = j < n && kept(j, cs[j], c);
      int total;
      const int ex = fg_block_exscan_i32(k ? 1 : 0, ired, &total);
      if (j < n) store(j, k, c, running + ex);
      running += total;
      __syncthreads();
    }
  }

  if (tid == 0) {
    // slots to reserve: the class-kept prompt tokens, and if a class component is present
    // every later token may be special/punctuation and stay (+S); the frequent budget follows
    // the sequence length; the window is fixed; one extra slot for the new token while it is
    // attended to. Never more than the uncompressed cache.
    const int S = a.S, full = n + S;
    long long cap;
    if (policy == 4) cap = full;
    else {
      cap = CC[policy];
      if (comp & (FG_COMP_SPECIAL | FG_COMP_PUNCT)) cap += S;
      if (comp & FG_COMP_FREQUENT) cap += fg_budget(a.r_f, full);
      if (comp & FG_COMP_LOCAL) cap += w;
      if (comp & (FG_COMP_FREQUENT | FG_COMP_LOCAL)) cap += 1;
      if (cap < running) cap = running;
    }
    if (cap > full) cap = full;
    if (cap < 1) cap = 1;
    a.cap[u] = (int)cap;
    a.len[u] = running;
    a.policy[u] = policy | (comp << 8);  // id in the low byte, component mask above
    if (a.policy_out) a.policy_out[u] = policy;
    for (int c = 0; c < 5; ++c) {
      a.recov[u * 5 + c] = R[c];
      a.kcount[u * 5 + c] = C[c];
      if (a.recov_out) a.recov_out[u * 5 + c] = R[c];
      if (a.kcount_out) a.kcount_out[u * 5 + c] = C[c];
    }
  }
}

// Unit records of the one-workgroup-per-unit decode step: record r = unit, 0, cap, tokens held (kept
// current by the step), off lo, off hi, policy word, 0.
__device__ __forceinline__ void fg_write_unit_record(int32_t* unit_rec, int r, int u, int cap, int len,
                                                     int64_t off, int policy) {
  int4* p = reinterpret_cast<int4*>(unit_rec + (size_t)r * 8);
  p[0] = make_int4(u, 0, cap, len);
  p[1] = make_int4((int32_t)(off & 0xffffffffll), (int32_t)(off >> 32), policy, 0);
}

// Adds 1 to counter[key] for every active lane and returns the lane's place among them (lanes
// that share a key are added by one atomic: the reservations take only a few different sizes).
__device__ __forceinline__ int fg_count_place(int* counter, bool active, int key) {
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(active);
  int place = 0;
  while (todo) {
    const int leader = __ffsll((long long)todo) - 1;
    const int k = __builtin_amdgcn_readlane(key, leader);
    const unsigned long long same = __ballot(active && key == k) & todo;
    int base = 0;
    if (lane == leader) base = atomicAdd(&counter[k], (int)__popcll(same));
    base = __builtin_amdgcn_readlane(base, leader);
    if ((same >> lane) & 1ull) place = base + (int)__popcll(same & ((1ull << lane) - 1ull));
    todo &= ~same;
  }
  return place;
}

// Whether the units are ordered by size. The order pays where the longest units would decide the end of
// a launch and costs one workgroup's counting sort in fastgen_compact (inside the offsets kernel's own time
// up to 1024 units). Unordered / ordered, compaction and decode step in us: 1024 units of 2000 tokens 221 +
// 125 / 224 + 117, 2048 of 1024 249 + 127 / 250 + 116, 4096 of 1024 495 + 228 / 506 + 221, 16384 of 1024
// (of 1536 reserved) 2317 + 1095 / 2310 + 1048; but 4096 of 150, d = 64, 59 + 30 / 66 + 30, 6000 of 400, d = 64,
// 166 + 72 / 181 + 72, 16384 of 600, d = 64, 666 + 252 / 700 + 262. So above 4096 units from 256 KiB each on.
constexpr int kSortUnits = 16384;
inline bool sorts_units(int U, int max_cap, int row_bytes) {
  if (U <= 4096) return U <= 1024 || max_cap >= 512;
  return U <= kSortUnits && (long long)max_cap * 2 * row_bytes >= (1 << 18);
}

// Single workgroup: off[u] = sum_{v<u} cap[v]. BY_UNIT false: chunk_off[u] = sum_{v<u} ceil(cap[v]/chunk).
// BY_UNIT true: chunk_off[u] = place of unit u among the units, with `ordered` longest reservations first
// (a counting sort into 64 classes; the order inside a class does not matter), and for few units their
// records too.
template <bool BY_UNIT>
__global__ __launch_bounds__(1024) void fg_offsets_kernel(const int32_t* __restrict__ cap,
                                                          int64_t* __restrict__ off,
                                                          int32_t* __restrict__ chunk_off,
                                                          int32_t* __restrict__ flags, int U,
                                                          int64_t pool_tokens, int64_t max_chunks, int chunk,
                                                          int max_cap, int32_t* __restrict__ unit_rec,
                                                          const int32_t* __restrict__ len,
                                                          const int32_t* __restrict__ policy, int ordered) {
  __shared__ int red[20];
  __shared__ long long wsum[16];
  __shared__ int class_at[64];
  __shared__ uint8_t s_class[BY_UNIT ? kSortUnits : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float to_class = 63.0f / (float)max_cap;
  const bool sorted = BY_UNIT && ordered != 0;
  if (BY_UNIT) {
    if (tid < 64) class_at[tid] = 0;
    __syncthreads();
  }
  long long run_off = 0;
  int run_chunk = 0;
  for (int base = 0; base < U; base += 1024) {
    const int u = base + tid;
    const int c = (u < U) ? cap[u] : 0;
    int exc = 0;
    if (!BY_UNIT) {
      int total;
      exc = fg_block_exscan_i32((c + chunk - 1) / chunk, red, &total) + run_chunk;
      run_chunk += total;
    } else if (sorted) {
      const int k = 63 - min(63, (int)((float)c * to_class));
      (void)fg_count_place(class_at, u < U, k);
      if (u < U) s_class[u] = (uint8_t)k;
    }
    // 64-bit scan of the capacities: wave scan + serial over the 16 waves
    long long inc = c;
    for (int o = 1; o < 64; o <<= 1) {
      long long t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    long long wbase = 0, wtot = 0;
    for (int i = 0; i < 16; ++i) {
      if (i < wave) wbase += wsum[i];
      wtot += wsum[i];
    }
    if (u < U) {
      off[u] = run_off + wbase + inc - c;
      if (!BY_UNIT) chunk_off[u] = exc;
    }
    run_off += wtot;
    __syncthreads();
  }
  if (tid == 0) {
    off[U] = run_off;
    if (!BY_UNIT) chunk_off[U] = run_chunk;
    flags[0] = (run_off > pool_tokens || (int64_t)run_chunk > max_chunks) ? 1 : 0;
    flags[1] = 0;
  }
  if (!BY_UNIT) return;
  if (sorted) {
    if (wave == 0) {
      const int count = class_at[lane];
      class_at[lane] = fg_wave_incscan_i32(count) - count;
    }
    __syncthreads();
  }
  for (int base = 0; base < U; base += 1024) {
    const int u = base + tid;
    const int r = sorted ? fg_count_place(class_at, u < U, u < U ? s_class[u] : 0) : u;
    if (u >= U) continue;
    if (U > 1024) chunk_off[u] = r;
    else fg_write_unit_record(unit_rec, r, u, cap[u], len[u], off[u], policy[u]);
  }
}

__global__ __launch_bounds__(256) void fg_unit_map_kernel(const int32_t* __restrict__ place,
                                                          const int32_t* __restrict__ cap,
                                                          const int64_t* __restrict__ off,
                                                          const int32_t* __restrict__ len,
                                                          const int32_t* __restrict__ policy,
                                                          int32_t* __restrict__ unit_rec, int U) {
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u < U) fg_write_unit_record(unit_rec, place[u], u, cap[u], len[u], off[u], policy[u]);
}

// Work-item records of the decode attention kernel: item c of unit u covers slots
// [chunk * (c - chunk_off[u]), +chunk) of that unit (chunk = 128 or 256 tokens). 8 ints per item: unit, chunk, cap, tokens held
// by the unit (kept current by the update kernel), off lo, off hi, policy word (id | component
// mask << 8), 0.
__global__ __launch_bounds__(256) void fg_item_map_kernel(const int32_t* __restrict__ chunk_off,
                                                          const int32_t* __restrict__ cap,
                                                          const int64_t* __restrict__ off,
                                                          const int32_t* __restrict__ len,
                                                          const int32_t* __restrict__ policy,
                                                          int32_t* __restrict__ item_rec,
                                                          const int32_t* __restrict__ flags, int U) {
  if (flags[0] != 0) return;
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u >= U) return;
  const int64_t o = off[u];
  const int c0 = chunk_off[u], c1 = chunk_off[u + 1];
  for (int c = c0; c < c1; ++c) {
    int32_t* r = item_rec + (size_t)c * 8;
    r[0] = u; r[1] = c - c0; r[2] = cap[u]; r[3] = len[u];
    r[4] = (int32_t)(o & 0xffffffffll); r[5] = (int32_t)(o >> 32); r[6] = policy[u]; r[7] = 0;
  }
}

// 16 prompt positions per workgroup; 16-byte chunks of the kept rows are copied by
// consecutive lanes (one 256-byte bf16 row = 16 lanes).
__global__ __launch_bounds__(256) void fg_gather_kernel(fg_compact_args a, int tiles_per_unit) {
  if (a.flags[0] != 0) return;
  const int u = blockIdx.x / tiles_per_unit, tile = blockIdx.x % tiles_per_unit;
  const int n = a.n, tid = threadIdx.x;
  const int rb = a.d * a.esize, cpr = rb / 16;
  const int64_t off = a.off[u];
  const char* Ku = static_cast<const char*>(a.K) + (size_t)u * n * rb;
  const char* Vu = static_cast<const char*>(a.V) + (size_t)u * n * rb;
  char* ck = static_cast<char*>(a.ck);
  char* cv = static_cast<char*>(a.cv);
  for (int q = tid; q < 16 * cpr; q += 256) {
    const int j = tile * 16 + q / cpr, ch = q % cpr;
    if (j >= n) continue;
    const int kb = a.keep[(size_t)u * n + j];
    if (!kb) continue;
    const int64_t dst = off + a.slot[(size_t)u * n + j];
    *reinterpret_cast<u32x4*>(ck + dst * rb + ch * 16) = *reinterpret_cast<const u32x4*>(Ku + (size_t)j * rb + ch * 16);
    *reinterpret_cast<u32x4*>(cv + dst * rb + ch * 16) = *reinterpret_cast<const u32x4*>(Vu + (size_t)j * rb + ch * 16);
    if (ch == 0) {
      a.cscore[dst] = a.colsum[(size_t)u * n + j];
      a.cpos[dst] = j;
      a.ccls[dst] = (uint8_t)(kb & 3);
    }
  }
}

// Single workgroup: offsets[u] = sum_{v<u} len[v].
__global__ __launch_bounds__(1024) void fg_len_scan_kernel(const int32_t* __restrict__ len,
                                                           int64_t* __restrict__ offsets,
                                                           int32_t* __restrict__ lengths,
                                                           const int32_t* __restrict__ flags,
                                                           int32_t* __restrict__ status, int U) {
  __shared__ long long wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  long long run = 0;
  for (int base = 0; base < U; base += 1024) {
    const int u = base + tid;
    const int c = (u < U) ? len[u] : 0;
    long long inc = c;
    for (int o = 1; o < 64; o <<= 1) {
      long long t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    long long wbase = 0, wtot = 0;
    for (int i = 0; i < 16; ++i) {
      if (i < wave) wbase += wsum[i];
      wtot += wsum[i];
    }
    if (u < U) {
      if (offsets) offsets[u] = run + wbase + inc - c;
      if (lengths) lengths[u] = c;
    }
    run += wtot;
    __syncthreads();
  }
  if (tid == 0) {
    if (offsets) offsets[U] = run;
    if (status) status[0] = flags[0] ? (int)FG_ECAP : 0;
  }
}

// `parts` workgroups per unit, each for its share of the unit's slots. Slots are unordered in the
// cache; the rank of a held position is the number of held positions below it, read off a bitmap
// of held positions that every workgroup builds for itself.
// Bound: HBM (rows read and written once) once enough loads are in flight; one workgroup per unit
// that took its rows 16 at a time with nothing in flight behind them needed 216 us for 256 units of
// 1850 tokens, d = 128 bf16, where a copy of the same bytes takes 95.
__global__ __launch_bounds__(256) void fg_export_kernel(fg_export_args a, const int64_t* __restrict__ dst_off, int parts) {
  extern __shared__ uint32_t smem[];  // words bitmap, then words prefix counts
  __shared__ int red[20];
  if (a.flags[0] != 0) return;
  const int u = blockIdx.x / parts, part = blockIdx.x % parts, tid = threadIdx.x;
  const int words = (a.max_pos + 31) / 32;
  uint32_t* bits = smem;
  uint32_t* pre = smem + words;
  const int L = a.len[u];
  const int64_t src = a.off[u], dst = dst_off[u];
  for (int i = tid; i < words; i += 256) bits[i] = 0u;
  __syncthreads();
  for (int j = tid; j < L; j += 256) {
    const int p = a.cpos[src + j];
    atomicOr(&bits[p >> 5], 1u << (p & 31));
  }
  __syncthreads();
  int run = 0;
  for (int base = 0; base < words; base += 256) {
    const int i = base + tid;
    const int count = i < words ? __popc(bits[i]) : 0;
    int total;
    const int before = fg_block_exscan_i32(count, red, &total);
    if (i < words) pre[i] = (uint32_t)(run + before);
    run += total;
    __syncthreads();
  }
  __syncthreads();
  auto rank_of = [&](int p) { return (int)pre[p >> 5] + __popc(bits[p >> 5] & ((1u << (p & 31)) - 1u)); };
  const int share = (L + parts - 1) / parts;
  const int j0 = min(L, part * share), j1 = min(L, j0 + share);
  for (int j = j0 + tid; j < j1; j += 256) {
    const int p = a.cpos[src + j];
    const int rank = rank_of(p);
    if (a.positions) a.positions[dst + rank] = p;
    if (a.scores) a.scores[dst + rank] = a.cscore[src + j];
  }
  if (!a.keys && !a.values) return;
  // rows: consecutive lanes take the 16-byte pieces of a row, four pieces per thread in flight
  const int rb = a.d * a.esize, cpr = rb / 16;
  const char* from[2] = {static_cast<const char*>(a.ck), static_cast<const char*>(a.cv)};
  char* to[2] = {static_cast<char*>(a.keys), static_cast<char*>(a.values)};
  constexpr int UN = 4;
  for (int q0 = j0 * cpr + tid; q0 < j1 * cpr; q0 += 256 * UN) {
    int64_t at[UN];
    int64_t get[UN];
#pragma unroll
    for (int i = 0; i < UN; ++i) {
      const int q = q0 + 256 * i;
      at[i] = -1;
      get[i] = 0;
      if (q < j1 * cpr) {
        const int j = q / cpr;
        get[i] = (src + j) * rb + (q % cpr) * 16;
        at[i] = (dst + rank_of(a.cpos[src + j])) * rb + (q % cpr) * 16;
      }
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv) {
      if (!to[kv]) continue;
      u32x4 v[UN];
#pragma unroll
      for (int i = 0; i < UN; ++i)
        if (at[i] >= 0) v[i] = *reinterpret_cast<const u32x4*>(from[kv] + get[i]);
#pragma unroll
      for (int i = 0; i < UN; ++i)
        if (at[i] >= 0) *reinterpret_cast<u32x4*>(to[kv] + at[i]) = v[i];
    }
  }
}

}  // namespace

hipError_t fg_launch_classify(const fg_classify_args& a, hipStream_t s) {
  const unsigned blocks = (unsigned)((a.count + 255) / 256);
  hipLaunchKernelGGL(fg_classify_kernel, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t fg_launch_select(const fg_select_args& a, const fg_part_sums& ps, hipStream_t s) {
  // More threads shorten a unit's chain while the card has room for them: 512 of them for few units,
  // 256 where many units of few tokens are bound by the workgroups in flight (512 / 256 threads
  // before the tokens stayed in registers: 256 units of 3000 tokens 27 / 38 us, 1024 of 2048
  // 44 / 37, 4096 of 1024 120 / 81), and as many as hold the prompt in at most 12 register slots.
  // Measured, us, with everything re-read per pass and twelve single block sums / now: 32 units of
  // 333 tokens 14.3 / 7.3, 1024 of 2048 37 / 29, 4096 of 1024 81 / 47, 256 of 3000 38 / 19, 640 of 8192
  // 137 / 80. Few workgroups of 1024 threads fit at once and twelve slots of 256 hold three waves per SIMD,
  // so many units take fewer slots or smaller workgroups where that is enough: 1024 x 8 / 512 x 12 slots,
  // 513 units of 4400 52 / 41, 1600 of 4400 125 / 83 (re-read 115), 1600 of 6000 139 / 91; 256 x 12 / x 10,
  // 1024 of 2100 39 / 28, 8192 of 2500 220 / 174 (re-read 213); 4096 of 3000 with twelve 134 (138).
  const fg_no_parts whole;
#define FG_SELECT(NT, NC, P) hipLaunchKernelGGL((fg_select_kernel<NT, NC, std::decay_t<decltype(P)>>), dim3((unsigned)a.U), dim3(NT), 0, s, a, P)
  if (ps.parts > 1) {   // (a kernel of its own: the parts' loads take 20 registers more)
    if (a.n > 1024) return hipErrorInvalidValue;
    if (a.U <= 512) { if (a.n <= 512) FG_SELECT(512, 1, ps); else FG_SELECT(512, 2, ps); }
    else if (a.n <= 512) FG_SELECT(256, 2, ps);
    else FG_SELECT(256, 4, ps);
  } else if (a.U <= 512 || a.n > 3072) {
    if (a.n <= 512) FG_SELECT(512, 1, whole);
    else if (a.n <= 1024) FG_SELECT(512, 2, whole);
    else if (a.n <= 2048) FG_SELECT(512, 4, whole);
    else if (a.n <= 4096) FG_SELECT(512, 8, whole);
    else if (a.n <= 6144 && a.U > 512) FG_SELECT(512, 12, whole);
    else if (a.n <= 8192) FG_SELECT(1024, 8, whole);
    else FG_SELECT(512, 0, whole);
  } else {
    if (a.n <= 512) FG_SELECT(256, 2, whole);
    else if (a.n <= 1024) FG_SELECT(256, 4, whole);
    else if (a.n <= 2048) FG_SELECT(256, 8, whole);
    else if (a.n <= 2560) FG_SELECT(256, 10, whole);
    else FG_SELECT(256, 12, whole);
  }
#undef FG_SELECT
  return hipGetLastError();
}

hipError_t fg_launch_compact(const fg_compact_args& a, hipStream_t s) {
  const int tiles = (a.n + 15) / 16;
  hipLaunchKernelGGL(fg_gather_kernel, dim3((unsigned)((size_t)a.U * tiles)), dim3(256), 0, s, a, tiles);
  return hipGetLastError();
}

hipError_t fg_launch_offsets(const int32_t* cap, const int32_t* len, const int32_t* policy, int64_t* off,
                             int32_t* chunk_off, int32_t* item_unit, int32_t* flags, int U, int64_t pool_tokens,
                             int64_t max_chunks, int chunk, int max_cap, int row_bytes, bool by_unit, hipStream_t s) {
  const dim3 blocks((unsigned)((U + 255) / 256));
  if (by_unit) {
    hipLaunchKernelGGL((fg_offsets_kernel<true>), dim3(1), dim3(1024), 0, s, cap, off, chunk_off, flags, U,
                       pool_tokens, max_chunks, chunk, max_cap, item_unit, len, policy, (int)sorts_units(U, max_cap, row_bytes));
    if (U > 1024) hipLaunchKernelGGL(fg_unit_map_kernel, blocks, dim3(256), 0, s, chunk_off, cap, off, len, policy, item_unit, U);
  } else {
    hipLaunchKernelGGL((fg_offsets_kernel<false>), dim3(1), dim3(1024), 0, s, cap, off, chunk_off, flags, U,
                       pool_tokens, max_chunks, chunk, max_cap, item_unit, len, policy, 0);
    hipLaunchKernelGGL(fg_item_map_kernel, blocks, dim3(256), 0, s, chunk_off, cap, off, len, policy, item_unit, flags, U);
  }
  return hipGetLastError();
}

hipError_t fg_launch_export(const fg_export_args& a, hipStream_t s) {
  // offsets are needed by the per-unit kernel even if the caller does not want them: the
  // caller-visible array is used when given, else positions cannot be packed
  hipLaunchKernelGGL(fg_len_scan_kernel, dim3(1), dim3(1024), 0, s, a.len, a.offsets, a.lengths,
                     a.flags, a.status, a.U);
  if (a.positions || a.scores || a.keys || a.values) {
    const int words = (a.max_pos + 31) / 32;
    const size_t smem = (size_t)(2 * words) * sizeof(uint32_t);
    // enough workgroups for the card (256 CUs, eight each), no share below 256 possible tokens
    int parts = (2048 + a.U - 1) / a.U;
    if (parts > a.max_pos / 256) parts = a.max_pos / 256;
    if (parts < 1) parts = 1;
    hipLaunchKernelGGL(fg_export_kernel, dim3((unsigned)a.U * (unsigned)parts), dim3(256), smem, s, a, a.offsets, parts);
  }
  return hipGetLastError();
}
