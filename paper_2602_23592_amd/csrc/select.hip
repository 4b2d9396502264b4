// Multi-hop importance propagation and selection (Section 4.2 of the paper:
// initialisation, importance propagation, convergence check) on the device.
//
// Every floating-point value that decides the selection is computed in binary32 in a fixed order (sums over
// candidates in ascending order, one division each), so the result is a pure function of S.
//
// Fewer than 64 candidates: one wave does all of it (k_select_small).  From 64 on k_row_totals (many workgroups: reading S
// once needs more than one CU) and k_select (one workgroup: what is left is a chain of small steps that depend on each
// other).  From 900 on the first selections are k_select_step and k_propagate in turn (the propagation on many workgroups),
// and k_select runs those that are left.
#include <algorithm>

#include "keep_internal.h"

namespace keep {

constexpr int SEL_THREADS = 1024;

// ---------------------------------------------------------------------------------------------
// Row totals of S, each summed one element after the other in ascending order.
//
// A workgroup owns 16 rows.  Waves 1..4 fetch the next 256 columns into LDS (consecutive threads on consecutive
// columns) while 16 lanes of wave 0 add the present ones, so the kernel costs the chain of m dependent additions and
// no memory latency beyond the first block's: 8 us at 1024 candidates on an idle chip (beside a product that fills the
// chip it waits for workgroups of that one to end).  It sums every row, also those a selection never reads; where scores
// are formed row by row some were not formed yet, and their totals mean nothing until a later launch.  The last workgroup
// instead forms the candidates' lengths and their total for callers that pass the memories' indices (`prep`).
// ---------------------------------------------------------------------------------------------
constexpr int RT_ROWS = 16, RT_COLS = 256, RT_LD = RT_COLS + 4;
constexpr int RT_THREADS = 64 + RT_COLS;

// Lengths of the candidates in candidate order and their total.  Indices are clamped into the length table so that a
// bad id cannot make the kernel read out of bounds.
__device__ void prepare_lengths(const SelectPrep& p, int m) {
  __shared__ int s_part[RT_THREADS / 64];
  int sum = 0;
  for (int i = threadIdx.x; i < m; i += RT_THREADS) {
    const int g = min(max(p.groups[i], 0), p.n_groups - 1);
    const int len = p.group_len[g];
    p.cand_len[i] = len;
    sum += len;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < RT_THREADS / 64; ++w) t += s_part[w];
    *p.cand_total = t;  // written, not accumulated: nothing of an earlier call survives
  }
}

__global__ void __launch_bounds__(RT_THREADS)
    k_row_totals(const float* __restrict__ S, int m, float* __restrict__ tot, SelectPrep prep) {
  if (prep.groups && blockIdx.x + 1 == gridDim.x) {
    prepare_lengths(prep, m);
    return;
  }
  __shared__ __attribute__((aligned(16))) float tile[2][RT_ROWS][RT_LD];
  const int tid = threadIdx.x;
  const int a0 = blockIdx.x * RT_ROWS;
  const int rows = min(RT_ROWS, m + 1 - a0);
  const int n_blocks = (m + RT_COLS - 1) / RT_COLS;
  const int c = tid - 64;  // loaders: the column
  float total = 0.f;
  for (int k = -1; k < n_blocks; ++k) {
    if (tid >= 64) {
      const int col = (k + 1) * RT_COLS + c;
      if (k + 1 < n_blocks && col < m) {
        const float* src = S + (size_t)a0 * m + col;
        float v[RT_ROWS];
#pragma unroll
        for (int r = 0; r < RT_ROWS; ++r) v[r] = r < rows ? src[(size_t)r * m] : 0.f;
#pragma unroll
        for (int r = 0; r < RT_ROWS; ++r) tile[(k + 1) & 1][r][c] = v[r];
      }
    } else if (k >= 0 && tid < rows) {
      const float* t = tile[k & 1][tid];
      const int cols = min(RT_COLS, m - k * RT_COLS);
      int j = 0;
      for (; j + 32 <= cols; j += 32) {
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const float4*>(t + j + 4 * q);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          total = total + v[q].x;
          total = total + v[q].y;
          total = total + v[q].z;
          total = total + v[q].w;
        }
      }
      for (; j < cols; ++j) total = total + t[j];
    }
    __syncthreads();
  }
  if (tid < rows) tot[a0 + tid] = total;
}

// ---------------------------------------------------------------------------------------------
// k_select
// ---------------------------------------------------------------------------------------------
// Sort key: ascending keys are (importance descending, index ascending).  -0 counts as +0; a NaN, which no score of
// attention mass is, comes behind every number.
__device__ __forceinline__ uint64_t sel_key(float v, int b) {
  uint32_t hi = 0xFFFFFFFFu;
  if (v == v) {
    const uint32_t u = v == 0.f ? 0u : __float_as_uint(v);
    hi = ~(u & 0x80000000u ? ~u : u | 0x80000000u);  // at most 0xFF800000 (-inf)
  }
  return (uint64_t)hi << 32 | (uint32_t)b;
}

// Bitonic sort of P keys (a power of two) in LDS, ascending.  A wave's pairs lie in 128 consecutive keys as long as
// partners are at most 64 apart, so only the wider steps need the workgroup's barrier.
__device__ void sel_sort(uint64_t* key, int P) {
  bool wide = true;  // the step before crossed waves (the caller's writes did)
  for (int k = 2; k <= P; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (wide || j > 64)
        __syncthreads();
      else
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      wide = j > 64;
      for (int p = threadIdx.x; p < (P >> 1); p += SEL_THREADS) {
        const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));
        const uint64_t x = key[i], y = key[i + j];
        if ((x > y) == ((i & k) == 0)) {
          key[i] = y;
          key[i + j] = x;
        }
      }
    }
  __syncthreads();
}

// A walk of up to 64 memories in rank order, one per lane: the ones that still fit, as a mask; `left` shrinks by them.
// Of those that fit what is left, all up to the first whose running sum does not are taken at once, that one is passed
// over, and so on; what does not fit once never will.
__device__ __forceinline__ uint64_t walk_chunk(bool valid, int l, int lane, int& left) {
  uint64_t cand = __ballot(valid && l <= left), got = 0;
  while (cand) {
    int64_t sum = cand >> lane & 1 ? l : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t t = __shfl_up((long long)sum, o, 64);
      if (lane >= o) sum += t;
    }
    const uint64_t over = __ballot((cand >> lane & 1) && sum > left);
    const int f = over ? __builtin_ctzll(over) : 64;  // the first that does not fit behind those before it
    got |= f < 64 ? cand & ((1ull << f) - 1) : cand;
    if (f > 0) left -= (int)__shfl((long long)sum, f - 1, 64);
    cand = f < 63 ? cand & ~((2ull << f) - 1) : 0;
    cand &= __ballot(l <= left);
  }
  return got;
}

// Mark what is taken of the order: its first k (count mode) or a walk of it that takes a memory iff it still fits the
// token budget (token mode).  key[b], b < m: the candidates' keys.
//
// Ranking by sorting: 1024 candidates against each other are 2^20 comparisons for one CU, the sort is 55 short steps.
// The walk goes in chunks of 64 through one wave.
__device__ void take(uint64_t* key, int m, int P, const int32_t* len, int k_count, int token_budget, int mode,
                     uint8_t* taken) {
  for (int b = m + threadIdx.x; b < P; b += SEL_THREADS) key[b] = ~0ull;
  sel_sort(key, P);
  if (mode == KEEP_BUDGET_GROUP_COUNT) {
    for (int i = threadIdx.x; i < m; i += SEL_THREADS) {
      const uint64_t e = key[i];
      // (nothing is greater than a NaN: its rank is 0)
      taken[(uint32_t)e] = (uint32_t)(e >> 32) == 0xFFFFFFFFu ? k_count > 0 : i < k_count;
    }
  } else if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int left = token_budget;
    for (int c0 = 0; c0 < m; c0 += 64) {
      const bool valid = c0 + lane < m;
      const int b = valid ? (int)(uint32_t)key[c0 + lane] : 0;
      const uint64_t got = walk_chunk(valid, valid ? len[b] : 0, lane, left);
      if (valid) taken[b] = got >> lane & 1;
    }
  }
  __syncthreads();
}

// The marked candidates in ascending order; returns how many.
__device__ int compact(const uint8_t* taken, int m, int32_t* list, int* s_cnt /*[SEL_THREADS / 64]*/) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int n = 0;
  for (int b0 = 0; b0 < m; b0 += SEL_THREADS) {
    const int b = b0 + threadIdx.x;
    const bool mine = b < m && taken[b];
    const uint64_t votes = __ballot(mine);
    if (lane == 0) s_cnt[wave] = __popcll(votes);
    __syncthreads();
    int at = n;
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
      at += w < wave ? s_cnt[w] : 0;
      n += s_cnt[w];
    }
    if (mine) list[at + __popcll(votes & ((1ull << lane) - 1))] = b;
    __syncthreads();
  }
  return n;
}

// What a selection that runs over several launches keeps between them, behind the m + 1 row totals
struct SelectState {
  int32_t* flags;  // [4]: selection ended, selections run, members of the set
  uint64_t* key;   // [m] importances as sort keys
  int32_t* list;   // [m] the set, ascending
  uint8_t* rel;    // [m] its members
};
static SelectState select_state(float* scratch, int m) {
  SelectState st;
  int32_t* w = reinterpret_cast<int32_t*>(scratch) + (m + 1 + 1) / 2 * 2;
  st.key = reinterpret_cast<uint64_t*>(w);
  st.flags = w + 2 * m;
  st.list = st.flags + 4;
  st.rel = reinterpret_cast<uint8_t*>(st.list + m);
  return st;
}

// The normalised score of (a, b) is S[a, b] / total_a with total_a the sum of row a in ascending order
// (0 where the row is empty); it is formed where it is used, only the row totals are kept.
//
// Bound by its chain of small steps.  It reads only the rows of S that the propagation averages, 16 loads in flight per
// thread.  768 candidates, 115 kept, three selections: 72 us; 1024 candidates, 308 kept: 118 us (k_propagate's now).
__global__ void __launch_bounds__(SEL_THREADS)
    k_select(const float* __restrict__ S, int m, int P, const int32_t* __restrict__ cand_len, int k_count,
             int token_budget, int mode, int hops, int set_only, const float* __restrict__ row_tot,
             int32_t* __restrict__ out, const int32_t* __restrict__ cand_total, const int32_t* __restrict__ id_map,
             int resume, SelectState st) {
  extern __shared__ __attribute__((aligned(16))) char sel_smem[];
  uint64_t* key = reinterpret_cast<uint64_t*>(sel_smem);  // [P]
  float* list_tot = reinterpret_cast<float*>(key + P);    // [m] row totals of the listed candidates
  int32_t* list = reinterpret_cast<int32_t*>(list_tot + m);  // [m] the relevant set, ascending
  int32_t* len = list + m;                                // [m]
  uint8_t* rel = reinterpret_cast<uint8_t*>(len + m);     // [m]
  uint8_t* rel2 = rel + m;                                // [m]
  __shared__ int s_diff, s_cnt[SEL_THREADS / 64];
  // Callers that could not classify the budget on the host pass the candidates' token total: a budget that
  // takes every candidate or none is settled here without a selection (0 selections run), as the host does
  // for the other callers.
  if (cand_total && !resume) {
    const bool all = m > 0 && (mode == KEEP_BUDGET_GROUP_COUNT ? k_count >= m : token_budget >= *cand_total);
    const bool none = m == 0 || (mode == KEEP_BUDGET_GROUP_COUNT ? k_count == 0 : token_budget <= 0);
    if (all || none) {
      const int n = all ? m : 0;
      for (int a = threadIdx.x; a < n; a += SEL_THREADS) out[2 + a] = id_map ? id_map[a] : a;
      if (threadIdx.x == 0) {
        out[0] = n;
        out[1] = 0;
      }
      return;
    }
  }
  if (resume && st.flags[0]) return;  // (the selection ended in the launches before)

  for (int b = threadIdx.x; b < m; b += SEL_THREADS) len[b] = cand_len[b];
  const float tq = row_tot[m];
  if (resume) {
    for (int b = threadIdx.x; b < m; b += SEL_THREADS) rel[b] = st.rel[b];
    __syncthreads();
  } else {
    for (int b = threadIdx.x; b < m; b += SEL_THREADS) key[b] = sel_key(tq > 0.f ? S[(size_t)m * m + b] / tq : 0.f, b);
    take(key, m, P, len, k_count, token_budget, mode, rel);
  }
  int n_rel = compact(rel, m, list, s_cnt);
  int runs = resume ? st.flags[1] : 1;
  const int max_runs = hops > 1 ? hops : 1;
  while (runs < max_runs) {
    for (int i = threadIdx.x; i < n_rel; i += SEL_THREADS) list_tot[i] = row_tot[list[i]];
    __syncthreads();
    // sources of the propagation: the query and the relevant set, or (set_only: the section's wording taken
    // literally) the relevant set alone; an empty source set leaves the importance at zero
    const int n_src = (set_only ? 0 : 1) + n_rel;
    const float denom = (float)n_src;
    for (int b = threadIdx.x; b < m; b += SEL_THREADS) {
      float acc = (!set_only && tq > 0.f) ? S[(size_t)m * m + b] / tq : 0.f;
      constexpr int U = 16;
      int i = 0;
      for (; i + U <= n_rel; i += U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = S[(size_t)list[i + u] * m + b];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float ta = list_tot[i + u];
          acc = acc + (ta > 0.f ? v[u] / ta : 0.f);
        }
      }
      for (; i < n_rel; ++i) {
        const float ta = list_tot[i];
        acc = acc + (ta > 0.f ? S[(size_t)list[i] * m + b] / ta : 0.f);
      }
      key[b] = sel_key(n_src > 0 ? acc / denom : acc, b);
    }
    if (threadIdx.x == 0) s_diff = 0;
    take(key, m, P, len, k_count, token_budget, mode, rel2);
    ++runs;
    int differs = 0;
    for (int a = threadIdx.x; a < m; a += SEL_THREADS) {
      differs |= rel[a] != rel2[a];
      rel[a] = rel2[a];
    }
    if (differs) s_diff = 1;  // (every writer writes the same value)
    __syncthreads();
    const int changed = s_diff;
    if (!changed) break;
    n_rel = compact(rel, m, list, s_cnt);  // (its barriers order this read of s_diff before the next clearing)
  }
  for (int i = threadIdx.x; i < n_rel; i += SEL_THREADS) out[2 + i] = id_map ? id_map[list[i]] : list[i];
  if (threadIdx.x == 0) {
    out[0] = n_rel;
    out[1] = runs;
  }
}

// ---------------------------------------------------------------------------------------------
// The same selection over several launches, where there are enough candidates that the propagation, one division per
// listed row and candidate, is worth more than one CU: k_select_step chooses and lists a set (one workgroup), and
// k_propagate forms the next importances (a workgroup per 64 candidates).  A step that finds the set it was given ends
// the selection: what is launched behind it returns at once.  That still costs a launch, so only the first selections run
// this way and k_select goes on from their state.  Same sums, divisions and orders as in k_select.
//
// k_propagate: lane = candidate.  Seven waves fetch the listed rows of a block of 112 and divide, the eighth adds the
// block before in ascending order: its chain of additions, 8 cycles each, is what bounds the kernel.
// ---------------------------------------------------------------------------------------------
constexpr int PR_WAVES = 8, PR_ROWS = 16 * (PR_WAVES - 1);

__global__ void __launch_bounds__(PR_WAVES * 64)
    k_propagate(const float* __restrict__ S, int m, int set_only, const float* __restrict__ row_tot, SelectState st) {
  __shared__ float s_q[2][PR_ROWS][64];
  if (st.flags[0]) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x * 64 + lane, bc = min(b, m - 1);
  const int n_rel = st.flags[2], n_src = (set_only ? 0 : 1) + n_rel;
  const int n_blocks = (n_rel + PR_ROWS - 1) / PR_ROWS;
  const float tq = row_tot[m];
  float acc = !set_only && tq > 0.f ? S[(size_t)m * m + bc] / tq : 0.f;
  for (int k = -1; k < n_blocks; ++k) {
    if (wave < PR_WAVES - 1) {
      const int i0 = (k + 1) * PR_ROWS + wave * 16;  // 16 consecutive rows of the next block
      if (i0 < n_rel) {
        float v[16], t[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int a = st.list[min(i0 + u, n_rel - 1)];
          t[u] = row_tot[a];
          v[u] = S[(size_t)a * m + bc];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) s_q[(k + 1) & 1][wave * 16 + u][lane] = t[u] > 0.f ? v[u] / t[u] : 0.f;
      }
    } else if (k >= 0) {
      const int rows = min(PR_ROWS, n_rel - k * PR_ROWS);
      int i = 0;
      for (; i + 16 <= rows; i += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = s_q[k & 1][i + u][lane];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc = acc + v[u];
      }
      for (; i < rows; ++i) acc = acc + s_q[k & 1][i][lane];
    }
    __syncthreads();
  }
  if (wave == PR_WAVES - 1 && b < m) st.key[b] = sel_key(n_src > 0 ? acc / (float)n_src : acc, b);
}

__global__ void __launch_bounds__(SEL_THREADS)
    k_select_step(const float* __restrict__ S, int m, int P, const int32_t* __restrict__ cand_len, int k_count,
                  int token_budget, int mode, int first, const float* __restrict__ row_tot, SelectState st,
                  int32_t* __restrict__ out, const int32_t* __restrict__ cand_total, const int32_t* __restrict__ id_map) {
  extern __shared__ __attribute__((aligned(16))) char sel_smem[];
  uint64_t* key = reinterpret_cast<uint64_t*>(sel_smem);  // [P]
  int32_t* list = reinterpret_cast<int32_t*>(key + P);    // [m]
  int32_t* len = list + m;                                // [m]
  uint8_t* rel = reinterpret_cast<uint8_t*>(len + m);     // [m]
  __shared__ int s_diff, s_cnt[SEL_THREADS / 64];
  if (!first && st.flags[0]) return;
  if (first && cand_total) {  // (as in k_select)
    const bool all = m > 0 && (mode == KEEP_BUDGET_GROUP_COUNT ? k_count >= m : token_budget >= *cand_total);
    const bool none = m == 0 || (mode == KEEP_BUDGET_GROUP_COUNT ? k_count == 0 : token_budget <= 0);
    if (all || none) {
      const int n = all ? m : 0;
      for (int a = threadIdx.x; a < n; a += SEL_THREADS) out[2 + a] = id_map ? id_map[a] : a;
      if (threadIdx.x == 0) {
        out[0] = n;
        out[1] = 0;
        st.flags[0] = 1;
      }
      return;
    }
  }
  const int runs = first ? 1 : st.flags[1] + 1;
  const float tq = row_tot[m];
  for (int b = threadIdx.x; b < m; b += SEL_THREADS) {
    len[b] = cand_len[b];
    key[b] = first ? sel_key(tq > 0.f ? S[(size_t)m * m + b] / tq : 0.f, b) : st.key[b];
  }
  if (threadIdx.x == 0) s_diff = first;
  take(key, m, P, len, k_count, token_budget, mode, rel);
  if (!first) {
    int differs = 0;
    for (int a = threadIdx.x; a < m; a += SEL_THREADS) differs |= rel[a] != st.rel[a];
    if (differs) s_diff = 1;  // (every writer writes the same value)
    __syncthreads();
  }
  if (!s_diff) {  // the set repeated: it is listed already
    if (threadIdx.x == 0) {
      out[1] = runs;
      st.flags[0] = 1;
    }
    return;
  }
  const int n_rel = compact(rel, m, list, s_cnt);
  for (int a = threadIdx.x; a < m; a += SEL_THREADS) st.rel[a] = rel[a];
  for (int i = threadIdx.x; i < n_rel; i += SEL_THREADS) {
    st.list[i] = list[i];
    out[2 + i] = id_map ? id_map[list[i]] : list[i];
  }
  if (threadIdx.x == 0) {
    out[0] = n_rel;
    out[1] = runs;
    st.flags[0] = 0;
    st.flags[1] = runs;
    st.flags[2] = n_rel;
  }
}

// ---------------------------------------------------------------------------------------------
// k_select_small: fewer than 64 candidates, one per lane of one wave.
//
// Bound by launches and barriers.  Four waves bring S (at most 64 x 63) to LDS, all loads in flight at once, and the
// first goes on alone, without a barrier: sets are 64-bit masks, ranks are counted.  The same sums, divisions and orders
// as in k_row_totals and k_select, so the same sets.  One wave holds up to 63 candidates and the query's row; from 64 on
// the two kernels above take over.  A call that is waited for, up to four selections: 9 candidates 22 us (36 with the two
// kernels), 63 candidates 37 us (64 with the two kernels: 51).
// ---------------------------------------------------------------------------------------------
constexpr int SEL_SMALL = 64;  // rows of S

__global__ void __launch_bounds__(256)
    k_select_small(const float* __restrict__ S, int m, const int32_t* __restrict__ cand_len, int k_count,
                   int token_budget, int mode, int hops, int set_only, int32_t* __restrict__ out, SelectPrep prep) {
  __shared__ float s_S[SEL_SMALL][SEL_SMALL + 1];
  __shared__ uint64_t s_key[SEL_SMALL];
  __shared__ int s_at[SEL_SMALL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool valid = lane < m;
  const bool classify = prep.cand_total;  // candidates given as indices, budget not classified by the caller
  {
    float v[SEL_SMALL / 4];
#pragma unroll
    for (int u = 0; u < SEL_SMALL / 4; ++u) v[u] = valid && wave + 4 * u <= m ? S[(size_t)(wave + 4 * u) * m + lane] : 0.f;
#pragma unroll
    for (int u = 0; u < SEL_SMALL / 4; ++u) s_S[wave + 4 * u][lane] = v[u];
  }
  int len = 0;
  if (wave == 0 && valid)
    len = classify ? prep.group_len[min(max(prep.groups[lane], 0), prep.n_groups - 1)] : cand_len[lane];
  __syncthreads();
  if (wave) return;
  uint64_t set = 0;
  int runs = 0;
  bool all = false, none = false;
  if (classify) {
    int sum = len;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    all = m > 0 && (mode == KEEP_BUDGET_GROUP_COUNT ? k_count >= m : token_budget >= sum);
    none = m == 0 || (mode == KEEP_BUDGET_GROUP_COUNT ? k_count == 0 : token_budget <= 0);
  }
  if (all) {
    set = (1ull << m) - 1;
  } else if (!none) {
    float total = 0.f;  // of the lane's row of S; the query's row is row m
    for (int j = 0; j < m; ++j) total = total + s_S[lane][j];
    auto choose = [&](float v) -> uint64_t {
      const uint64_t key = valid ? sel_key(v, lane) : ~0ull;
      s_key[lane] = key;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      int rank = 0;
      for (int c = 0; c < m; ++c) rank += s_key[c] < key;
      bool taken;
      if (mode == KEEP_BUDGET_GROUP_COUNT) {
        taken = (uint32_t)(key >> 32) == 0xFFFFFFFFu ? k_count > 0 : rank < k_count;  // (a NaN: as in take)
      } else {
        if (valid) s_at[rank] = lane;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int l = __shfl(len, valid ? s_at[lane] : 0, 64);
        int left = token_budget;
        taken = walk_chunk(valid, l, lane, left) >> rank & 1;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      return __ballot(valid && taken);
    };
    const float tq = __shfl(total, m, 64);
    const float query = tq > 0.f ? s_S[m][lane] / tq : 0.f;
    set = choose(query);
    runs = 1;
    while (runs < hops) {
      const int n_src = (set_only ? 0 : 1) + __popcll(set);
      float acc = set_only ? 0.f : query;
      for (uint64_t a = set; a; a &= a - 1) {
        const int i = __builtin_ctzll(a);
        const float ta = __shfl(total, i, 64);
        acc = acc + (ta > 0.f ? s_S[i][lane] / ta : 0.f);
      }
      const uint64_t next = choose(n_src > 0 ? acc / (float)n_src : acc);
      ++runs;
      if (next == set) break;
      set = next;
    }
  }
  if (set >> lane & 1) out[2 + __popcll(set & ((1ull << lane) - 1))] = classify ? prep.groups[lane] : lane;
  if (lane == 0) {
    out[0] = __popcll(set);
    out[1] = runs;
  }
}

// scratch of launch_select in words, for up to m candidates
size_t select_scratch_words(int32_t m) { return (size_t)(m + 1 + 1) / 2 * 2 + (size_t)3 * m + 4 + (size_t)(m + 3) / 4; }

// From here on the propagation gets workgroups of its own.  Back to back, us for a call of two / three / three / four
// selections that keep 5 / 10 / 15 / 40 % of the candidates: 512 candidates 31 / 53 / 54 / 110 in one workgroup against
// 34 / 56 / 52 / 89, 768: 40 / 74 / 72 / 170 against 42 / 71 / 65 / 112, 1024: 44 / 87 / 90 / 236 against
// 44 / 75 / 69 / 126, 4000: 202 / 581 / 741 / 2673 against 106 / 197 / 170 / 366.  (The line would lie lower for selections
// that go on longer and keep more, but how many are made is not known at the launch, and two lose below it.)
constexpr int SEL_SPREAD = 900;

// How many selections run this way before k_select goes on from their state, so that a caller who asks for the fixed point
// (any large `hops`) pays for few launches behind it.  Two empty launches cost 5 us.  A set that repeats at once, hops = 100,
// us in one workgroup / with 8 / with 30 spread selections: 1024 candidates 47 / 77 / 221, 2048: 97 / 90 / 224, 4000: 270 / 128 / 238;
// ten selections that keep 40 %: 638 / 391 / 317, 2164 / 884 / 511, 7658 / 2423 / 917.  With many candidates the empty launches
// may therefore take as long as one workgroup's second selection would, which grows with their square.
static int sel_spread_runs(int m) { return std::max(8, m * m / 450000); }

void launch_select(const float* S, int32_t m, const int32_t* d_cand_len, int32_t k_count, int32_t token_budget,
                   int32_t mode, int32_t hops, float* d_scratch, int32_t* d_out, hipStream_t s, bool set_only,
                   const SelectPrep* prep) {
  const SelectPrep pr = prep ? *prep : SelectPrep{};
  if (m < SEL_SMALL) {
    hipLaunchKernelGGL(k_select_small, dim3(1), dim3(256), 0, s, S, m, d_cand_len, k_count, token_budget, mode, hops,
                       set_only ? 1 : 0, d_out, pr);
    return;
  }
  int P = 2;
  while (P < m) P <<= 1;
  const int blocks = (m + 1 + RT_ROWS - 1) / RT_ROWS + (prep ? 1 : 0);
  hipLaunchKernelGGL(k_row_totals, dim3(blocks), dim3(RT_THREADS), 0, s, S, m, d_scratch, pr);
  const int max_runs = hops > 1 ? hops : 1;
  const int spread = m >= SEL_SPREAD && max_runs > 1 ? std::min(max_runs, sel_spread_runs(m)) : 0;
  const SelectState st = select_state(d_scratch, m);
  if (spread) {
    const size_t sh = (size_t)P * 8 + (size_t)m * (2 * 4 + 1);
    static std::atomic<uint64_t> attr_done{0};
    set_max_dyn_smem_once(attr_done, reinterpret_cast<const void*>(k_select_step), 160 * 1024 - 256);
    for (int run = 1; run <= spread; ++run) {
      if (run > 1)
        hipLaunchKernelGGL(k_propagate, dim3((m + 63) / 64), dim3(PR_WAVES * 64), 0, s, S, m, set_only ? 1 : 0, d_scratch, st);
      hipLaunchKernelGGL(k_select_step, dim3(1), dim3(SEL_THREADS), sh, s, S, m, P, d_cand_len, k_count, token_budget, mode,
                         run == 1 ? 1 : 0, d_scratch, st, d_out, pr.cand_total, pr.groups);
    }
    if (spread == max_runs) return;
  }
  const size_t sh = (size_t)P * 8 + (size_t)m * (3 * 4 + 2);  // <= 147 KB: m <= 6000
  static std::atomic<uint64_t> attr_done{0};
  set_max_dyn_smem_once(attr_done, reinterpret_cast<const void*>(k_select), 160 * 1024 - 256);
  hipLaunchKernelGGL(k_select, dim3(1), dim3(SEL_THREADS), sh, s, S, m, P, d_cand_len, k_count, token_budget, mode, hops,
                     set_only ? 1 : 0, d_scratch, d_out, pr.cand_total, pr.groups, spread ? 1 : 0, st);
}

}  // namespace keep
