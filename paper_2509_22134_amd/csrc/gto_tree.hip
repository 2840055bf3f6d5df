// Per-root kernels of the GTO hot path: layer-wise expansion, global re-rank, reward scan and
// greedy verification walk, group advantage, clipped surrogate forward.  All of them work on a
// few KB per root; they are latency-bound and tiny next to the row kernels.
//
// What bounds them is the chain of dependent steps in a root, so the usual sizes run as one wave per root: no
// barriers (a barrier also waits until every global store before it has been acknowledged), intermediate results in
// LDS or registers, global memory read in one or two rounds at the start and written once at the end.  Larger shapes
// take the workgroup-per-root kernels.
//
// Ranking everywhere is by the order-preserving bits of the fp32 score, then the inverted index, mostly packed into one
// key: keys are unique, so (score descending, index ascending) is realised exactly and deterministically whether the
// best are taken one after the other (expansion), a rank is found by counting the keys that beat mine (large k) or the
// keys are sorted (top-g).
#include <type_traits>

#include "gto_device.h"
#include "gto_kernels.h"

namespace gto {

constexpr int kTreeThreads = 256;
constexpr int kMaxPool = 4096;        // C

// ------------------------------------------------------------------------------ expansion
// Which rows feed which candidate is fixed by the shape (candidate c of the pool is child rk of slot j of
// level l), so every log-probability and token of the root is fetched up front in one round of loads; the
// level loop then runs out of LDS and only stores to memory.
// Dynamic LDS: k^2 keys rounded up to a multiple of eight (8 B each), C log-probabilities (4 B).
__global__ __launch_bounds__(kTreeThreads) void k_expand(ExpandArgs a) {
  const int r = blockIdx.x;
  const int k = a.k, d = a.d, kk = a.k * a.k, C = a.C;
  const int tid = threadIdx.x;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  const int kk8 = (kk + 7) & ~7;
  uint64_t *s_key = reinterpret_cast<uint64_t *>(s_dyn);
  float *s_lp = reinterpret_cast<float *>(s_key + kk8);
  __shared__ float s_score[2][64];
  __shared__ int s_cand[2][64];
  const int64_t pool0 = (int64_t)r * C;
  const int64_t slot0 = (int64_t)r * d * k;

  for (int t = kk + tid; t < kk8; t += kTreeThreads) s_key[t] = 0ull;
  for (int c = tid; c < C; c += kTreeThreads) {
    int l = 0, j = 0, rk = c;
    if (c >= k) {
      const int q = c - k;
      l = 1 + q / kk;
      const int t = q - (l - 1) * kk;
      j = t / k;
      rk = t - j * k;
    }
    const int64_t si = stat_index(r, l, j, d, k) * k + rk;
    s_lp[c] = a.top_logp[si];
    a.cand_tok[pool0 + c] = a.top_tok[si];
    a.cand_depth[pool0 + c] = l + 1;
    a.cand_pslot[pool0 + c] = j;
  }
  __syncthreads();
  // level 0: the root's k children, all expanded at level 1 in rank order
  for (int t = tid; t < k; t += kTreeThreads) {
    const float sc = __fadd_rn(0.f, s_lp[t]);
    a.cand_parent[pool0 + t] = -1;
    a.cand_score[pool0 + t] = sc;
    a.cand_slot[pool0 + t] = (d > 1) ? t : -1;
    a.slot_cand[slot0 + t] = -1;
    if (d > 1) a.slot_cand[slot0 + k + t] = t;
    s_score[1][t] = sc;
    s_cand[1][t] = t;
  }
  __syncthreads();
  for (int l = 1; l < d; ++l) {
    const int cur = l & 1, nxt = cur ^ 1;
    const int base = k + (l - 1) * kk;
    for (int t = tid; t < kk; t += kTreeThreads) {
      const int j = t / k;
      const float sc = __fadd_rn(s_score[cur][j], s_lp[base + t]);
      const int c = base + t;
      a.cand_parent[pool0 + c] = s_cand[cur][j];
      a.cand_score[pool0 + c] = sc;
      s_key[t] = rank_key(sc, t);
      if (l == d - 1) a.cand_slot[pool0 + c] = -1;
    }
    if (l == d - 1) break;
    __syncthreads();
    for (int t = tid; t < kk; t += kTreeThreads) {
      const uint64_t mine = s_key[t];
      int rank = 0;
      // eight keys per trip (the list is padded with zeros, which beat nothing): the reads of a trip are
      // independent, one key per trip would pay the LDS latency kk times
      for (int u = 0; u < kk8; u += 8) {
        uint64_t q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = s_key[u + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) rank += (q[e] > mine) ? 1 : 0;
      }
      const int c = base + t;
      if (rank < k) {
        // the same add as above gives the same bits; s_score[nxt] was last read before the previous barrier
        s_score[nxt][rank] = __fadd_rn(s_score[cur][t / k], s_lp[base + t]);
        s_cand[nxt][rank] = c;
        a.slot_cand[slot0 + (int64_t)(l + 1) * k + rank] = c;
        a.cand_slot[pool0 + c] = rank;
      } else {
        a.cand_slot[pool0 + c] = -1;
      }
    }
    __syncthreads();
  }
}

// One wave per root, k^2 <= 64 NT keys per level: lane t % 64 holds child t.  A level's k best come out one after the
// other by a wave-wide maximum of the score bits, the lowest child among equals first; lane j keeps the j-th, so the
// next level's parent scores are lane exchanges.  (Counting the keys that beat each key takes k^2 64-bit compares per
// lane and child.)  1024 roots with k = 10, d = 6: 14 us before, 12 now; 4 roots with k = 8, d = 7: 9.5 us, now 7.4.
// Dynamic LDS: C scores (4 B; they start as the log-probabilities), C parents and C slots (2 B each), d * k expanded
// candidates (2 B).
template <int NT>
__global__ __launch_bounds__(64) void k_expand_wave(ExpandArgs a) {
  const int r = blockIdx.x, lane = threadIdx.x;
  const int k = a.k, d = a.d, kk = a.k * a.k, C = a.C;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  float *s_sc = reinterpret_cast<float *>(s_dyn);
  int16_t *s_parent = reinterpret_cast<int16_t *>(s_sc + C);
  int16_t *s_slot = s_parent + C, *s_exp = s_slot + C;
  const int64_t pool0 = (int64_t)r * C;
  const int64_t row0 = (int64_t)r * d * kk;       // statistics of slot (0, 0)

  // candidate c is entry c of the root's slot, or entry c - k of the levels below, which follow each other
  for (int c0 = 0; c0 < C; c0 += 8 * 64) {
    float lp[8];
    int tok[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = min(c0 + u * 64 + lane, C - 1);
      const int64_t si = row0 + (c < k ? c : c - k + kk);
      lp[u] = a.top_logp[si];
      tok[u] = a.top_tok[si];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = c0 + u * 64 + lane;
      if (c < C) {
        s_sc[c] = lp[u];
        a.cand_tok[pool0 + c] = tok[u];
      }
    }
  }
  int jt[NT];                                     // slot of this lane's n-th child of a level
#pragma unroll
  for (int n = 0; n < NT; ++n) jt[n] = (n * 64 + lane) / k;
  __builtin_amdgcn_wave_barrier();
  // level 0: the root's k children, all expanded at level 1 in rank order
  float p_score = 0.f;                            // lane j: score and pool index of the node in slot j of the level
  int p_cand = lane;
  if (lane < k) {
    p_score = __fadd_rn(0.f, s_sc[lane]);
    s_sc[lane] = p_score;
    s_parent[lane] = -1;
    s_slot[lane] = (int16_t)((d > 1) ? lane : -1);
    s_exp[lane] = -1;
  }
  for (int l = 1; l < d; ++l) {
    const int base = k + (l - 1) * kk;
    if (lane < k) s_exp[l * k + lane] = (int16_t)p_cand;
    uint32_t o[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int t = n * 64 + lane;
      const float ps = __shfl(p_score, jt[n] & 63, kWave);
      const int pc = __shfl(p_cand, jt[n] & 63, kWave);
      o[n] = 0u;                                  // (no score has this image)
      if (t < kk) {
        const float sc = __fadd_rn(ps, s_sc[base + t]);
        s_sc[base + t] = sc;
        s_parent[base + t] = (int16_t)pc;
        s_slot[base + t] = -1;
        o[n] = ordered_bits(sc);
      }
    }
    if (l == d - 1) break;
    float n_score = 0.f;
    int n_cand = 0;
    for (int j = 0; j < k; ++j) {
      uint32_t m = o[0];
#pragma unroll
      for (int n = 1; n < NT; ++n) m = max(m, o[n]);
      m = wave_max_dpp(m);
      int at = 0;                                 // the lowest child that holds the maximum
#pragma unroll
      for (int n = NT - 1; n >= 0; --n) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(o[n] == m);
        if (mask != 0ull) at = n * 64 + __builtin_ctzll(mask);
      }
#pragma unroll
      for (int n = 0; n < NT; ++n)
        if (n * 64 + lane == at) o[n] = 0u;
      if (lane == j) {
        n_score = from_ordered_bits(m);
        n_cand = base + at;
      }
    }
    if (lane < k) {
      s_slot[n_cand] = (int16_t)lane;
      n_score = s_sc[n_cand];                     // (the image of -0 is that of 0: take the score itself)
    }
    p_score = n_score;
    p_cand = n_cand;
  }
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < C; c += 64) {
    a.cand_score[pool0 + c] = s_sc[c];
    a.cand_parent[pool0 + c] = s_parent[c];
    a.cand_slot[pool0 + c] = s_slot[c];
  }
  if (lane < k) {
    a.cand_depth[pool0 + lane] = 1;
    a.cand_pslot[pool0 + lane] = 0;
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int t = n * 64 + lane;
    if (t < kk)
      for (int l = 1; l < d; ++l) {
        a.cand_depth[pool0 + k + (l - 1) * kk + t] = l + 1;
        a.cand_pslot[pool0 + k + (l - 1) * kk + t] = jt[n];
      }
  }
  for (int i = lane; i < d * k; i += 64) a.slot_cand[(int64_t)r * d * k + i] = s_exp[i];
}

void launch_expand(const ExpandArgs &a, hipStream_t st) {
  const int kk = a.k * a.k;
  if (kk <= 256) {
    const size_t lds_wave = (size_t)a.C * 8 + (size_t)a.d * a.k * 2;
    if (kk <= 64) hipLaunchKernelGGL(k_expand_wave<1>, dim3(a.R), dim3(64), lds_wave, st, a);
    else if (kk <= 128) hipLaunchKernelGGL(k_expand_wave<2>, dim3(a.R), dim3(64), lds_wave, st, a);
    else hipLaunchKernelGGL(k_expand_wave<4>, dim3(a.R), dim3(64), lds_wave, st, a);
    return;
  }
  const size_t lds = (size_t)((a.k * a.k + 7) & ~7) * 8 + (size_t)a.C * 4;
  hipLaunchKernelGGL(k_expand, dim3(a.R), dim3(kTreeThreads), lds, st, a);
}

// ------------------------------------------------------------------------------ top-g
// The C candidates of a root are sorted by their (unique) keys with a bitonic network over the next power of
// two, padded with key 0 (below every real key: the low word of a real key is never 0).  Position i of the
// sorted list is rank i; comparing every key with every other one, as the expansion does for its k^2 keys,
// costs C^2 = 260 k compares per root at C = 510 and made this kernel ALU bound.
// Dynamic LDS: n_pad keys (8 B), C ranks (4 B), n_keep leaf flags, d * k need flags.
__device__ __forceinline__ int select_pad(int C) {
  int n = 2;
  while (n < C) n <<= 1;
  return n;
}

__global__ __launch_bounds__(kTreeThreads) void k_select(SelectArgs a) {
  const int r = blockIdx.x, tid = threadIdx.x;
  const int C = a.C, g = a.g;
  const int n_keep = (g < C) ? g : C;
  const int n_pad = select_pad(C);
  extern __shared__ __align__(16) unsigned char s_dyn[];
  uint64_t *s_key = reinterpret_cast<uint64_t *>(s_dyn);
  int *s_rank = reinterpret_cast<int *>(s_key + n_pad);
  unsigned char *s_leaf = reinterpret_cast<unsigned char *>(s_rank + C);
  unsigned char *s_need = s_leaf + n_keep;
  const int64_t pool0 = (int64_t)r * C;
  const int64_t sel0 = (int64_t)r * g;
  for (int c = tid; c < n_pad; c += kTreeThreads) s_key[c] = (c < C) ? rank_key(a.cand_score[pool0 + c], c) : 0ull;
  for (int i = tid; i < n_keep; i += kTreeThreads) s_leaf[i] = 1;
  for (int i = tid; i < a.d * a.k; i += kTreeThreads) s_need[i] = 0;
  __syncthreads();
  // descending bitonic sort
  for (int size = 2; size <= n_pad; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = tid; t < (n_pad >> 1); t += kTreeThreads) {
        const int lo = 2 * t - (t & (stride - 1));
        const int hi = lo + stride;
        const bool desc = (lo & size) == 0;
        const uint64_t x = s_key[lo], y = s_key[hi];
        if ((x < y) == desc) {
          s_key[lo] = y;
          s_key[hi] = x;
        }
      }
      __syncthreads();
    }
  }
  for (int i = tid; i < C; i += kTreeThreads) s_rank[(int)(0xffffffffu - (uint32_t)s_key[i])] = i;
  __syncthreads();
  for (int c = tid; c < C; c += kTreeThreads) {
    const int p = a.cand_parent[pool0 + c];
    if (s_rank[c] < n_keep && p >= 0) {
      const int pr = s_rank[p];
      if (pr < n_keep) s_leaf[pr] = 0;  // a kept child: the parent is not a leaf
    }
    // the row that produced a kept node is needed by the reward
    if (s_rank[c] < n_keep) s_need[(a.cand_depth[pool0 + c] - 1) * a.k + a.cand_pslot[pool0 + c]] = 1;
  }
  __syncthreads();
  // the kept candidates, straight from the sorted list
  for (int i = tid; i < n_keep; i += kTreeThreads) {
    const int c = (int)(0xffffffffu - (uint32_t)s_key[i]);
    const int p = a.cand_parent[pool0 + c];
    a.sel_cand[sel0 + i] = c;
    a.sel_tok[sel0 + i] = a.cand_tok[pool0 + c];
    // a parent always outranks its child (log-probabilities are <= 0); the range check only matters for
    // rows that held NaNs, whose values are unspecified but whose indices must stay inside the list
    a.sel_parent[sel0 + i] = (p >= 0 && s_rank[p] < i) ? s_rank[p] : -1;
    a.sel_depth[sel0 + i] = a.cand_depth[pool0 + c];
    a.sel_pslot[sel0 + i] = a.cand_pslot[pool0 + c];
    a.sel_slot[sel0 + i] = a.cand_slot[pool0 + c];
    a.sel_score[sel0 + i] = a.cand_score[pool0 + c];
    a.sel_leaf[sel0 + i] = s_leaf[i];
  }
  for (int i = n_keep + tid; i < g; i += kTreeThreads) {
    a.sel_cand[sel0 + i] = -1;
    a.sel_tok[sel0 + i] = -1;
    a.sel_parent[sel0 + i] = -1;
    a.sel_depth[sel0 + i] = 0;
    a.sel_pslot[sel0 + i] = 0;
    a.sel_slot[sel0 + i] = -1;
    a.sel_score[sel0 + i] = 0.f;
    a.sel_leaf[sel0 + i] = 0;
  }
  for (int i = tid; i < a.d * a.k; i += kTreeThreads) a.slot_need[(int64_t)r * a.d * a.k + i] = s_need[i];
  if (tid == 0) a.n_sel[r] = n_keep;
}

// One wave per root, C <= 64 NPL: the same network with NPL keys per lane (key index lane * NPL + e while sorting), so
// that short strides stay in a lane's registers and long ones are lane exchanges (DPP moves up to 8 lanes): 1024 roots
// with C = 510 take 12 us (workgroup per root: 17.6 us, 45 barriers), 4 roots 9 us (13).  The keys are doubles in [1, 2) whose mantissa
// holds the score's bits and the inverted index: the fp64 compare runs at full rate, the 64-bit integer one does not.
__device__ __forceinline__ double sort_key(float score, int index) {
  return __longlong_as_double(0x3ff0000000000000ull | ((uint64_t)ordered_bits(score) << 20) | (uint64_t)(0xfffff - index));
}
__device__ __forceinline__ int sort_index(double key) { return 0xfffff - (int)(__double_as_longlong(key) & 0xfffff); }

template <int NPL, int SIZE, int STRIDE>
__device__ __forceinline__ void bitonic_stage(double (&key)[NPL], int lane) {
  if constexpr (STRIDE >= NPL) {
    const bool desc = ((lane * NPL) & SIZE) == 0;              // (SIZE > STRIDE >= NPL: the same for all keys of a lane)
    const bool larger = desc != ((lane & (STRIDE / NPL)) != 0);
#pragma unroll
    for (int e = 0; e < NPL; ++e) {
      const double o = lane_xor<STRIDE / NPL>(key[e]);
      key[e] = ((key[e] < o) == larger) ? o : key[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < NPL; ++e) {
      if (e & STRIDE) continue;
      const bool desc = ((lane * NPL + e) & SIZE) == 0;
      const double x = key[e], y = key[e + STRIDE];
      const bool swap = (x < y) == desc;
      key[e] = swap ? y : x;
      key[e + STRIDE] = swap ? x : y;
    }
  }
  if constexpr (STRIDE > 1) bitonic_stage<NPL, SIZE, STRIDE / 2>(key, lane);
}
// descending sort of 64 NPL keys
template <int NPL, int SIZE = 2>
__device__ __forceinline__ void bitonic_sort(double (&key)[NPL], int lane) {
  bitonic_stage<NPL, SIZE, SIZE / 2>(key, lane);
  if constexpr (SIZE < 64 * NPL) bitonic_sort<NPL, SIZE * 2>(key, lane);
}
// Few kept nodes (SORT < NPL: n_keep <= 64 SORT): a threshold that n_keep to 64 SORT of the scores reach is bisected
// first, some ten rounds of compares and bit counts, and only those are sorted (1024 roots, 60 of 510: 12 us with all
// keys sorted, 9 so; 4 roots 9 us and 6).  More ties than that at the threshold: all keys are sorted.
// Dynamic LDS: 64 SORT keys (8 B, SORT < NPL), C ranks (2 B), n_keep candidates (2 B), n_keep leaf flags, d * k need
// flags (1 B each).
template <int NPL, int SORT>
__global__ __launch_bounds__(64) void k_select_wave(SelectArgs a) {
  const int r = blockIdx.x, lane = threadIdx.x;
  const int C = a.C, g = a.g;
  const int n_keep = (g < C) ? g : C;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  double *s_few = reinterpret_cast<double *>(s_dyn);
  int16_t *s_rank = reinterpret_cast<int16_t *>(s_few + (SORT < NPL ? 64 * SORT : 0));
  int16_t *s_sel = s_rank + C;
  unsigned char *s_leaf = reinterpret_cast<unsigned char *>(s_sel + n_keep);
  unsigned char *s_need = s_leaf + n_keep;
  const int64_t pool0 = (int64_t)r * C;
  const int64_t sel0 = (int64_t)r * g;
  double key[NPL];
#pragma unroll
  for (int e = 0; e < NPL; ++e) {
    const int c = e * 64 + lane;                  // (which lane starts with which key does not matter)
    const float sc = a.cand_score[pool0 + min(c, C - 1)];
    key[e] = (c < C) ? sort_key(sc, c) : 1.0;     // padding: below every real key
  }
  for (int c = lane; c < C; c += 64) s_rank[c] = 0x7fff;
  for (int i = lane; i < n_keep; i += 64) s_leaf[i] = 1;
  for (int i = lane; i < a.d * a.k; i += 64) s_need[i] = 0;
  auto emit = [&](auto &sorted, auto npl) {
#pragma unroll
    for (int e = 0; e < decltype(npl)::value; ++e) {
      const int i = lane * decltype(npl)::value + e;
      if (i < n_keep) {
        const int c = sort_index(sorted[e]);
        s_rank[c] = (int16_t)i;
        s_sel[i] = (int16_t)c;
      }
    }
  };
  bool few = SORT < NPL;
  if constexpr (SORT < NPL) {
    uint32_t o[NPL];                              // the scores' bits; padding: 0
#pragma unroll
    for (int e = 0; e < NPL; ++e) o[e] = (uint32_t)((uint64_t)__double_as_longlong(key[e]) >> 20);
    uint32_t lo = 0u, hi = 0xffffffffu;           // count(>= lo) >= n_keep > count(>= hi)
    int cnt = 64 * NPL;
    while (cnt > 64 * SORT && hi - lo > 1u) {
      const uint32_t mid = lo + (hi - lo) / 2;
      int c = 0;
#pragma unroll
      for (int e = 0; e < NPL; ++e) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(o[e] >= mid));
      if (c >= n_keep) {
        lo = mid;
        cnt = c;
      } else {
        hi = mid;
      }
    }
    few = cnt <= 64 * SORT;
    if (few) {
      int at = 0;
#pragma unroll
      for (int e = 0; e < NPL; ++e) {
        const bool on = o[e] >= lo;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(on);
        if (on) s_few[at + lanes_below(mask)] = key[e];
        at += __builtin_popcountll(mask);
      }
      __builtin_amdgcn_wave_barrier();
      double best[SORT];
#pragma unroll
      for (int e = 0; e < SORT; ++e) best[e] = (e * 64 + lane < cnt) ? s_few[e * 64 + lane] : 1.0;
      bitonic_sort<SORT>(best, lane);
      emit(best, std::integral_constant<int, SORT>{});
    }
  }
  if (!few) {
    bitonic_sort<NPL>(key, lane);
    emit(key, std::integral_constant<int, NPL>{});
  }
  __builtin_amdgcn_wave_barrier();
  for (int i = lane; i < n_keep; i += 64) {
    const int c = s_sel[i];
    const int p = a.cand_parent[pool0 + c], tok = a.cand_tok[pool0 + c], dep = a.cand_depth[pool0 + c];
    const int ps = a.cand_pslot[pool0 + c], sl = a.cand_slot[pool0 + c];
    const float sc = a.cand_score[pool0 + c];
    const int pr = (p >= 0) ? s_rank[p] : 0x7fff;
    if (pr < n_keep) s_leaf[pr] = 0;              // a kept child: the parent is not a leaf
    s_need[(dep - 1) * a.k + ps] = 1;             // the row that produced a kept node is needed by the reward
    a.sel_cand[sel0 + i] = c;
    a.sel_tok[sel0 + i] = tok;
    // a parent always outranks its child (log-probabilities are <= 0); the range check only matters for
    // rows that held NaNs, whose values are unspecified but whose indices must stay inside the list
    a.sel_parent[sel0 + i] = (pr < i) ? pr : -1;
    a.sel_depth[sel0 + i] = dep;
    a.sel_pslot[sel0 + i] = ps;
    a.sel_slot[sel0 + i] = sl;
    a.sel_score[sel0 + i] = sc;
  }
  __builtin_amdgcn_wave_barrier();
  for (int i = lane; i < g; i += 64) {
    a.sel_leaf[sel0 + i] = (i < n_keep) ? s_leaf[i] : 0;
    if (i >= n_keep) {
      a.sel_cand[sel0 + i] = -1;
      a.sel_tok[sel0 + i] = -1;
      a.sel_parent[sel0 + i] = -1;
      a.sel_depth[sel0 + i] = 0;
      a.sel_pslot[sel0 + i] = 0;
      a.sel_slot[sel0 + i] = -1;
      a.sel_score[sel0 + i] = 0.f;
    }
  }
  for (int i = lane; i < a.d * a.k; i += 64) a.slot_need[(int64_t)r * a.d * a.k + i] = s_need[i];
  if (lane == 0) a.n_sel[r] = n_keep;
}

template <int NPL, int SORT>
static void launch_select_wave(const SelectArgs &a, int n_keep, hipStream_t st) {
  const size_t lds = (SORT < NPL ? 64 * SORT * sizeof(double) : 0) + (size_t)a.C * 2 + (size_t)n_keep * 3 + (size_t)a.d * a.k;
  hipLaunchKernelGGL((k_select_wave<NPL, SORT>), dim3(a.R), dim3(64), lds, st, a);
}
template <int NPL>
static void launch_select_wave_n(const SelectArgs &a, int n_keep, int sort, hipStream_t st) {
  if (sort == 1) launch_select_wave<NPL, 1>(a, n_keep, st);
  else if (sort == 2) launch_select_wave<NPL, 2>(a, n_keep, st);
  else launch_select_wave<NPL, NPL>(a, n_keep, st);
}

void launch_select(const SelectArgs &a, hipStream_t st) {
  int n_pad = 2;
  while (n_pad < a.C) n_pad <<= 1;
  const int n_keep = (a.g < a.C) ? a.g : a.C;
  if (n_pad <= 1024) {
    const int sort = (n_keep <= 64) ? 1 : (n_keep <= 128) ? 2 : 16;
    if (n_pad <= 64) launch_select_wave<1, 1>(a, n_keep, st);
    else if (n_pad <= 128) sort == 1 ? launch_select_wave<2, 1>(a, n_keep, st) : launch_select_wave<2, 2>(a, n_keep, st);
    else if (n_pad <= 256) launch_select_wave_n<4>(a, n_keep, sort, st);
    else if (n_pad <= 512) launch_select_wave_n<8>(a, n_keep, sort, st);
    else launch_select_wave_n<16>(a, n_keep, sort, st);
    return;
  }
  const size_t lds = (size_t)n_pad * 8 + (size_t)a.C * 4 + (size_t)n_keep + (size_t)a.d * a.k;
  hipLaunchKernelGGL(k_select, dim3(a.R), dim3(kTreeThreads), lds, st, a);
}

// ------------------------------------------------------------------------------ reward
constexpr int kRewardThreads = 128;
constexpr int kMaxDepth = 32;

__device__ __forceinline__ double block_reduce(double v, double *scratch, bool is_max) {
  const int tid = threadIdx.x;
  scratch[tid] = v;
  __syncthreads();
  for (int off = kRewardThreads / 2; off >= 1; off >>= 1) {
    if (tid < off) {
      const double o = scratch[tid + off];
      scratch[tid] = is_max ? fmax(scratch[tid], o) : scratch[tid] + o;
    }
    __syncthreads();
  }
  const double out = scratch[0];
  __syncthreads();
  return out;
}

// most nodes a root can keep: min(g, C)
__host__ __device__ inline int reward_nodes(const RewardArgs &a) {
  const int C = a.k + (a.d - 1) * a.k * a.k;
  return a.g < C ? a.g : C;
}

template <typename T>
__global__ __launch_bounds__(kRewardThreads) void k_reward(RewardArgs a) {
  const int r = blockIdx.x, tid = threadIdx.x;
  const int d = a.d, k = a.k, g = a.g;
  const int n = a.n_sel[r];
  const int64_t sel0 = (int64_t)r * g;
  extern __shared__ __align__(16) unsigned char s_dyn[];     // min(g, C) doubles, then as many ints
  double *s_logt = reinterpret_cast<double *>(s_dyn);
  int *s_parent = reinterpret_cast<int *>(s_logt + reward_nodes(a));
  __shared__ double s_red[kRewardThreads];
  __shared__ int s_found;
  const T *logits = static_cast<const T *>(a.target_logits);

  // target log-probability of every kept token (one gather each)
  for (int i = tid; i < n; i += kRewardThreads) {
    const int lvl = a.sel_depth[sel0 + i] - 1;
    const int js = a.sel_pslot[sel0 + i];
    const int tok = min(max(a.sel_tok[sel0 + i], 0), a.V - 1);     // ids come from the row kernels: always in range
    const int64_t si = stat_index(r, lvl, js, d, k);
    const float x = a.node_logit ? a.node_logit[sel0 + i] : Elem<T>::load1(logits + si * a.row_stride + tok);
    s_logt[i] = (double)x - (double)a.t_lse[si];
    s_parent[i] = a.sel_parent[sel0 + i];
  }
  __syncthreads();

  // prefix products along each node's own ancestor chain (root first), Eq. 3-4
  double v_max = -1.0, v_sumL = 0.0, v_cnt = 0.0, v_q = 0.0;
  double myL[ (kMaxPool + kRewardThreads - 1) / kRewardThreads ];
  int nmine = 0;
  for (int i = tid; i < n; i += kRewardThreads) {
    int chain[kMaxDepth];
    int len = 0;
    for (int p = i; p >= 0 && len < kMaxDepth; p = s_parent[p]) chain[len++] = p;
    double lq = 0.0, cum = 0.0, q = 0.0;
    for (int s = len - 1; s >= 0; --s) {
      lq += s_logt[chain[s]];
      q = exp(lq);
      cum += q;
    }
    a.node_q[sel0 + i] = (float)q;
    a.node_cum[sel0 + i] = (float)cum;
    v_q += q;
    const bool leaf = a.sel_leaf[sel0 + i] != 0;
    if (leaf) {
      v_max = fmax(v_max, cum);
      v_sumL += cum;
      v_cnt += 1.0;
    }
    myL[nmine++] = leaf ? cum : -1.0;
  }
  for (int i = n + tid; i < g; i += kRewardThreads) {
    a.node_q[sel0 + i] = 0.f;
    a.node_cum[sel0 + i] = 0.f;
  }
  const double Lmax = block_reduce(v_max, s_red, true);
  double v_exp = 0.0;
  for (int q = 0; q < nmine; ++q)
    if (myL[q] >= 0.0) v_exp += exp((double)a.eta * (myL[q] - Lmax));
  const double sum_exp = block_reduce(v_exp, s_red, false);
  const double sumL = block_reduce(v_sumL, s_red, false);
  const double cnt = block_reduce(v_cnt, s_red, false);
  const double nodesum = block_reduce(v_q, s_red, false);
  if (tid == 0) {
    const double lse = (cnt > 0.0) ? Lmax + log(sum_exp) / (double)a.eta : 0.0;
    const double mx = (cnt > 0.0) ? Lmax : 0.0;
    const double mean = (cnt > 0.0) ? sumL / cnt : 0.0;
    float *aux = a.reward_aux + (int64_t)r * 4;
    aux[0] = (float)lse;
    aux[1] = (float)mx;
    aux[2] = (float)mean;
    aux[3] = (float)nodesum;
    const double pick = (a.reward_mode == 0) ? lse : (a.reward_mode == 1) ? mx : (a.reward_mode == 2) ? mean : nodesum;
    a.reward[r] = (float)pick;
    a.n_leaves[r] = (int)cnt;
  }

  if (a.path_mode == 1) {
    // alternative reading of "longest accepted sequence": the root-to-leaf sequence with the largest
    // expected acceptance length L_i (first one in kept order among equals)
    __syncthreads();
    for (int q = 0, i = tid; i < n; i += kRewardThreads, ++q) s_logt[i] = myL[q];   // -1 for non-leaves
    __syncthreads();
    if (tid == 0) {
      int best = -1;
      double bl = -1.0;
      for (int i = 0; i < n; ++i)
        if (s_logt[i] > bl) { bl = s_logt[i]; best = i; }
      int chain[kMaxDepth];
      int len = 0;
      for (int p = best; p >= 0 && len < kMaxDepth; p = s_parent[p]) chain[len++] = p;
      for (int t = 0; t < d; ++t) {
        const bool on = t < len;
        const int node = on ? chain[len - 1 - t] : -1;
        a.path_node[(int64_t)r * d + t] = node;
        a.path_slot[(int64_t)r * d + t] = on ? a.sel_pslot[sel0 + node] : -1;
      }
      a.path_len[r] = len;
    }
    return;
  }
  if (a.path_mode == 2) {
    // verification at temperature 1: the kept children of the current node are tried in kept order,
    // child x accepted with probability p_T(x) / (target mass not yet rejected at this node), decided
    // by the caller's uniform numbers; s_logt still holds log p_T of every kept token
    __syncthreads();
    if (tid == 0) {
      int cur = -1, slot = 0, len = 0;
      for (int t = 0; t < d; ++t) {
        double rest = 1.0;
        int j = 0, nxt = -1;
        for (int i = 0; i < n; ++i) {
          if (s_parent[i] != cur || a.sel_depth[sel0 + i] != t + 1) continue;
          const double p_tok = exp(s_logt[i]);
          const double acc = (rest > 0.0) ? p_tok / rest : 1.0;
          const double u = (double)a.accept_u[((int64_t)r * d + t) * k + j];
          if (u < acc) { nxt = i; break; }
          rest -= p_tok;
          ++j;
        }
        if (nxt < 0) break;
        a.path_node[(int64_t)r * d + t] = nxt;
        a.path_slot[(int64_t)r * d + t] = slot;
        len = t + 1;
        const int own = a.sel_slot[sel0 + nxt];
        if (own < 0) break;
        cur = nxt;
        slot = own;
      }
      for (int t = len; t < d; ++t) {
        a.path_node[(int64_t)r * d + t] = -1;
        a.path_slot[(int64_t)r * d + t] = -1;
      }
      a.path_len[r] = len;
    }
    return;
  }
  // greedy verification walk (T = 0): follow the kept child that equals the target argmax
  int cur = -1, slot = 0, len = 0;
  bool alive = true;
  for (int t = 0; t < d; ++t) {
    if (tid == 0) s_found = -1;
    __syncthreads();
    if (alive) {
      const int want = a.t_argmax[stat_index(r, t, slot, d, k)];
      for (int i = tid; i < n; i += kRewardThreads)
        if (s_parent[i] == cur && a.sel_depth[sel0 + i] == t + 1 && a.sel_tok[sel0 + i] == want) s_found = i;
    }
    __syncthreads();
    const int nxt = alive ? s_found : -1;
    __syncthreads();
    if (nxt >= 0) {
      if (tid == 0) {
        a.path_node[(int64_t)r * d + t] = nxt;
        a.path_slot[(int64_t)r * d + t] = slot;
      }
      len = t + 1;
      const int own = a.sel_slot[sel0 + nxt];
      if (own < 0) alive = false;
      cur = nxt;
      slot = own;
    } else {
      alive = false;
      if (tid == 0) {
        a.path_node[(int64_t)r * d + t] = -1;
        a.path_slot[(int64_t)r * d + t] = -1;
      }
    }
  }
  if (tid == 0) a.path_len[r] = len;
}

// One wave per root, at most 64 NN kept nodes, node i in lane i % 64: 1024 roots with 60 nodes take 7 us (workgroup
// per root: 14 to 18 us, of it the walk's dependent loads and barriers).  The prefix sums go level by level (a node
// adds its own term to its parent's sum, the order of the chain walk above).
// Dynamic LDS: per node the prefix sum and cumulative length (8 B each), parent (4 B); d * k target argmaxes.
template <typename T, int NN>
__global__ __launch_bounds__(64) void k_reward_wave(RewardArgs a) {
  const int r = blockIdx.x, lane = threadIdx.x;
  const int d = a.d, k = a.k, g = a.g;
  const int cap = reward_nodes(a);                // <= 64 NN
  const int64_t sel0 = (int64_t)r * g;
  const int64_t slot0 = (int64_t)r * d * k;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  double *s_lq = reinterpret_cast<double *>(s_dyn);
  double *s_cum = s_lq + cap;
  int *s_parent = reinterpret_cast<int *>(s_cum + cap);
  int *s_arg = s_parent + cap;
  const T *logits = static_cast<const T *>(a.target_logits);

  // everything that is addressed by the shape alone, in one round
  const int n = min(a.n_sel[r], cap);
  int dep[NN], par[NN], tok[NN], own[NN], ps[NN];
  bool leaf[NN], on[NN];
#pragma unroll
  for (int q = 0; q < NN; ++q) {
    const int64_t i = sel0 + min(q * 64 + lane, cap - 1);
    dep[q] = a.sel_depth[i];
    ps[q] = a.sel_pslot[i];
    tok[q] = a.sel_tok[i];
    par[q] = a.sel_parent[i];
    own[q] = a.sel_slot[i];
    leaf[q] = a.sel_leaf[i] != 0;
  }
  if (a.path_mode == 0)
    for (int i = lane; i < d * k; i += 64) s_arg[i] = a.t_argmax[slot0 + i];
  // target log-probability of every kept token (one gather each)
  double logt[NN];
#pragma unroll
  for (int q = 0; q < NN; ++q) {
    const int i = q * 64 + lane;
    on[q] = i < n;
    logt[q] = 0.0;
    if (on[q]) {
      const int t = min(max(tok[q], 0), a.V - 1);               // ids come from the row kernels: always in range
      const int64_t si = stat_index(r, dep[q] - 1, ps[q], d, k);
      const float x = a.node_logit ? a.node_logit[sel0 + i] : Elem<T>::load1(logits + si * a.row_stride + t);
      logt[q] = (double)x - (double)a.t_lse[si];
      s_parent[i] = par[q];
      s_lq[i] = 0.0;
      s_cum[i] = 0.0;
    }
  }
  __builtin_amdgcn_wave_barrier();
  // length of each node's ancestor chain
  int len[NN], deepest = 0;
#pragma unroll
  for (int q = 0; q < NN; ++q) {
    len[q] = 0;
    if (on[q])
      for (int p = q * 64 + lane; p >= 0 && len[q] < kMaxDepth; p = s_parent[p]) ++len[q];
  }
  // prefix products along each node's own ancestor chain (root first), Eq. 3-4
  double lq[NN], pq[NN], cum[NN];
#pragma unroll
  for (int q = 0; q < NN; ++q) lq[q] = cum[q] = 0.0;
  for (int s = 1; s <= kMaxDepth; ++s) {
    bool any = false;
#pragma unroll
    for (int q = 0; q < NN; ++q) {
      if (len[q] == s) {
        lq[q] = (par[q] >= 0 ? s_lq[par[q]] : 0.0) + logt[q];
        s_lq[q * 64 + lane] = lq[q];
      }
      any = any || len[q] == s;
    }
    if (__builtin_amdgcn_ballot_w64(any) == 0ull) break;        // chains are prefix-closed: none is longer
    deepest = s;
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int q = 0; q < NN; ++q) pq[q] = on[q] ? exp(lq[q]) : 0.0;
  for (int s = 1; s <= deepest; ++s) {
#pragma unroll
    for (int q = 0; q < NN; ++q)
      if (len[q] == s) {
        cum[q] = (par[q] >= 0 ? s_cum[par[q]] : 0.0) + pq[q];
        s_cum[q * 64 + lane] = cum[q];
      }
    __builtin_amdgcn_wave_barrier();
  }
  double v_max = -1.0, v_sumL = 0.0, v_cnt = 0.0, v_q = 0.0;
#pragma unroll
  for (int q = 0; q < NN; ++q) {
    const int i = q * 64 + lane;
    leaf[q] = leaf[q] && on[q];
    if (on[q]) {
      a.node_q[sel0 + i] = (float)pq[q];
      a.node_cum[sel0 + i] = (float)cum[q];
    }
    v_q += pq[q];
    if (leaf[q]) {
      v_max = fmax(v_max, cum[q]);
      v_sumL += cum[q];
      v_cnt += 1.0;
    }
  }
  for (int i = n + lane; i < g; i += 64) {
    a.node_q[sel0 + i] = 0.f;
    a.node_cum[sel0 + i] = 0.f;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v_max = fmax(v_max, __shfl_xor(v_max, off, kWave));
  const double Lmax = v_max;
  double v_exp = 0.0;
#pragma unroll
  for (int q = 0; q < NN; ++q)
    if (leaf[q]) v_exp += exp((double)a.eta * (cum[q] - Lmax));
  const double sum_exp = wave_sum_dpp(v_exp), sumL = wave_sum_dpp(v_sumL), cnt = wave_sum_dpp(v_cnt);
  const double nodesum = wave_sum_dpp(v_q);
  if (lane == 0) {
    const double lse = (cnt > 0.0) ? Lmax + log(sum_exp) / (double)a.eta : 0.0;
    const double mx = (cnt > 0.0) ? Lmax : 0.0;
    const double mean = (cnt > 0.0) ? sumL / cnt : 0.0;
    float *aux = a.reward_aux + (int64_t)r * 4;
    aux[0] = (float)lse;
    aux[1] = (float)mx;
    aux[2] = (float)mean;
    aux[3] = (float)nodesum;
    const double pick = (a.reward_mode == 0) ? lse : (a.reward_mode == 1) ? mx : (a.reward_mode == 2) ? mean : nodesum;
    a.reward[r] = (float)pick;
    a.n_leaves[r] = (int)cnt;
  }

  // the accepted sequence: lane t keeps its step t
  int p_node = -1, p_slot = -1, plen = 0;
  auto pick_of = [&](const int (&v)[NN], int i) {               // v of node i (uniform)
    int out = 0;
#pragma unroll
    for (int q = 0; q < NN; ++q)
      if ((i >> 6) == q) out = readlane(v[q], i & 63);
    return out;
  };
  if (a.path_mode == 1) {
    // the root-to-leaf sequence with the largest expected acceptance length L_i (first one in kept order among equals)
    int best = kNoId;
#pragma unroll
    for (int q = NN - 1; q >= 0; --q)
      if (leaf[q] && cum[q] == Lmax) best = q * 64 + lane;
    best = wave_min(best);
    if (best != kNoId) {
      plen = pick_of(len, best);
      for (int t = plen - 1, p = best; t >= 0; --t) {
        const int sl = pick_of(ps, p), up = pick_of(par, p);
        if (lane == t) { p_node = p; p_slot = sl; }
        p = up;
      }
    }
  } else if (a.path_mode == 2) {
    // verification at temperature 1: the kept children of the current node are tried in kept order,
    // child x accepted with probability p_T(x) / (target mass not yet rejected at this node), decided
    // by the caller's uniform numbers
    double p_tok[NN];
#pragma unroll
    for (int q = 0; q < NN; ++q) p_tok[q] = exp(logt[q]);
    int cur = -1, slot = 0;
    for (int t = 0; t < d; ++t) {
      const float u_lane = (lane < k) ? a.accept_u[((int64_t)r * d + t) * k + lane] : 0.f;
      double rest = 1.0;
      int j = 0, nxt = -1;
#pragma unroll
      for (int q = 0; q < NN; ++q) {
        uint64_t mask = __builtin_amdgcn_ballot_w64(on[q] && par[q] == cur && dep[q] == t + 1);
        for (; mask != 0ull && nxt < 0; mask &= mask - 1, ++j) {
          const int src = __builtin_ctzll(mask);
          const double pt = __shfl(p_tok[q], src, kWave);
          const double acc = (rest > 0.0) ? pt / rest : 1.0;
          const double u = (double)readlane(u_lane, min(j, 63));
          if (u < acc) nxt = q * 64 + src;
          rest -= pt;
        }
      }
      if (nxt < 0) break;
      if (lane == t) { p_node = nxt; p_slot = slot; }
      plen = t + 1;
      slot = pick_of(own, nxt);
      if (slot < 0) break;
      cur = nxt;
    }
  } else {
    // greedy verification walk (T = 0): follow the kept child that equals the target argmax
    int cur = -1, slot = 0;
    for (int t = 0; t < d; ++t) {
      const int want = s_arg[t * k + slot];
      int nxt = -1;
#pragma unroll
      for (int q = NN - 1; q >= 0; --q) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(on[q] && par[q] == cur && dep[q] == t + 1 && tok[q] == want);
        if (mask != 0ull) nxt = q * 64 + __builtin_ctzll(mask);
      }
      if (nxt < 0) break;
      if (lane == t) { p_node = nxt; p_slot = slot; }
      plen = t + 1;
      slot = pick_of(own, nxt);
      if (slot < 0) break;
      cur = nxt;
    }
  }
  if (lane < d) {
    a.path_node[(int64_t)r * d + lane] = p_node;
    a.path_slot[(int64_t)r * d + lane] = p_slot;
  }
  if (lane == 0) a.path_len[r] = plen;
}

template <typename T>
static void launch_reward_wave(const RewardArgs &a, int nodes, hipStream_t st) {
  const size_t lds = (size_t)nodes * 20 + (size_t)a.d * a.k * 4;
  if (nodes <= 64) hipLaunchKernelGGL((k_reward_wave<T, 1>), dim3(a.R), dim3(64), lds, st, a);
  else hipLaunchKernelGGL((k_reward_wave<T, 2>), dim3(a.R), dim3(64), lds, st, a);
}

void launch_reward(const RewardArgs &a, hipStream_t st) {
  if (reward_nodes(a) <= 128) {
    if (a.dtype == 0) launch_reward_wave<uint16_t>(a, reward_nodes(a), st);
    else launch_reward_wave<float>(a, reward_nodes(a), st);
    return;
  }
  const size_t lds = (size_t)reward_nodes(a) * 12;
  if (a.dtype == 0) hipLaunchKernelGGL(k_reward<uint16_t>, dim3(a.R), dim3(kRewardThreads), lds, st, a);
  else hipLaunchKernelGGL(k_reward<float>, dim3(a.R), dim3(kRewardThreads), lds, st, a);
}

// ------------------------------------------------------------------------------ advantage
// One wave per group: lane-strided fp64 sums and a fixed-shape wave reduction (deterministic for any m).
__global__ __launch_bounds__(64) void k_advantage(AdvArgs a) {
  const int grp = blockIdx.x, lane = threadIdx.x;
  const int i0 = grp * a.m;
  double sum = 0.0;
  for (int i = lane; i < a.m; i += 64)
    sum += (double)a.r_cur[i0 + i] - (a.r_ref ? (double)a.r_ref[i0 + i] : 0.0);
  const double mean = wave_sum(sum) / a.m;
  double var = 0.0;
  for (int i = lane; i < a.m; i += 64) {
    const double dv = ((double)a.r_cur[i0 + i] - (a.r_ref ? (double)a.r_ref[i0 + i] : 0.0)) - mean;
    var += dv * dv;
  }
  const double sd = sqrt(wave_sum(var) / a.m);
  for (int i = lane; i < a.m; i += 64) {
    const double dv = ((double)a.r_cur[i0 + i] - (a.r_ref ? (double)a.r_ref[i0 + i] : 0.0)) - mean;
    a.adv[i0 + i] = (float)(dv / (sd + (double)a.delta));
  }
}

void launch_advantage(const AdvArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(k_advantage, dim3(a.R / a.m), dim3(64), 0, st, a);
}

// ------------------------------------------------------------------------------ surrogate fwd
// Group losses (Eq. 12), then their mean, by one workgroup of 256; every sum has a fixed shape.
template <typename Term>
__device__ __forceinline__ void group_losses(const PpoFwdArgs &a, Term term) {
  const int K = a.R / a.m;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ double s_red[256];
  double part = 0.0;
  if (a.m <= 16) {
    // small groups: one thread per group
    for (int grp = threadIdx.x; grp < K; grp += 256) {
      double sum = 0.0;
      for (int i = 0; i < a.m; ++i) sum += (double)term(grp * a.m + i);
      const double lg = -sum / a.m;
      a.loss_group[grp] = (float)lg;
      part += lg;
    }
  } else {
    // large groups: one wave per group, lane-strided sum and wave reduction
    for (int grp = wave; grp < K; grp += 4) {
      double sum = 0.0;
      for (int i = lane; i < a.m; i += 64) sum += (double)term(grp * a.m + i);
      const double lg = -wave_sum(sum) / a.m;
      if (lane == 0) {
        a.loss_group[grp] = (float)lg;
        part += lg;
      }
    }
  }
  s_red[threadIdx.x] = part;
  __syncthreads();
  for (int off = 128; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) s_red[threadIdx.x] += s_red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.loss[0] = (float)(s_red[0] / K);
}

// 2^shift >= d lanes per root, one per step of the path: a step is three dependent loads (path entry, token and
// log-sum-exps, logits), which one thread per root paid once per step (1024 roots, two accepted tokens on average:
// 14.7 us, now 6).  ONE_BLOCK: all roots fit one workgroup, which then also takes the losses.
template <typename T, bool ONE_BLOCK>
__global__ __launch_bounds__(256) void k_ppo_root(PpoFwdArgs a, int shift) {
  const int r = (blockIdx.x * 256 + threadIdx.x) >> shift, t = threadIdx.x & ((1 << shift) - 1);
  __shared__ float s_term[ONE_BLOCK ? 256 : 1];
  if (r < a.R) {
    const int d = a.d, k = a.k;
    const int l = a.path_len[r];
    const T *dl = static_cast<const T *>(a.draft_logits);
    const T *rl = static_cast<const T *>(a.ref_logits);
    double lm = 0.0, lm0 = 0.0;
    if (t < l) {
      const int64_t rt = (int64_t)r * d + t;
      const int j = a.path_slot[rt];
      const int tok = min(max(a.sel_tok[(int64_t)r * a.g + a.path_node[rt]], 0), a.V - 1);
      const int64_t si = stat_index(r, t, j, d, k);
      const float xc = a.path_logit_cur ? a.path_logit_cur[rt] : Elem<T>::load1(dl + si * a.row_stride + tok);
      lm = (double)xc - (double)a.draft_lse[si];
      const double rlse = a.ref_lse_by_step ? (double)a.ref_lse[rt] : (double)a.ref_lse[si];
      const float xr = a.path_logit_ref ? a.path_logit_ref[rt] : Elem<T>::load1(rl + si * a.row_stride + tok);
      lm0 = (double)xr - rlse;
    }
    for (int off = 1; off < (1 << shift); off <<= 1) {
      lm += __shfl_xor(lm, off, kWave);
      lm0 += __shfl_xor(lm0, off, kWave);
    }
    if (t == 0) {
      const int lden = (l > 1) ? l : 1;
      const double s = exp((lm - lm0) / lden);
      const double A = (double)a.adv[r];
      const double lo = 1.0 - (double)a.eps, hi = 1.0 + (double)a.eps;
      const double clipped = fmax(lo, fmin(s, hi));
      const double term = fmin(s * A, clipped * A);
      const bool passes = (A >= 0.0) ? (s <= hi) : (s >= lo);
      const int active = (l > 0 && passes) ? 1 : 0;
      const int K = a.R / a.m;
      a.logM[r] = (float)lm;
      a.logM0[r] = (float)lm0;
      a.ratio[r] = (float)s;
      a.term[r] = (float)term;
      a.active[r] = active;
      a.coef[r] = (float)((double)a.grad_scale * (-A / ((double)a.m * K)) * active * s / lden);
      if (ONE_BLOCK) s_term[r] = (float)term;
    }
  }
  if (ONE_BLOCK) {
    __syncthreads();
    group_losses(a, [&](int i) { return s_term[i]; });
  }
}

__global__ __launch_bounds__(256) void k_ppo_loss(PpoFwdArgs a) {
  group_losses(a, [&](int i) { return a.term[i]; });
}

// (slot, token) pairs whose single logits the fused variant computes as dot products
__global__ void k_pairs(PairArgs a, int mode) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per = (mode == 0) ? a.g : a.d;
  if (p >= (int64_t)a.R * per) return;
  const int r = (int)(p / per), i = (int)(p - (int64_t)r * per);
  int64_t slot = -1;
  int tok = -1;
  if (mode == 0) {
    if (i < a.n_sel[r]) {
      slot = stat_index(r, a.sel_depth[p] - 1, a.sel_pslot[p], a.d, a.k);
      tok = a.sel_tok[p];
    }
  } else {
    const int j = a.path_slot[p];
    if (j >= 0) {
      slot = stat_index(r, i, j, a.d, a.k);
      tok = a.sel_tok[(int64_t)r * a.g + a.path_node[p]];
    }
  }
  a.slot[p] = slot;
  a.tok[p] = tok;
}

void launch_pairs(const PairArgs &a, int mode, hipStream_t st) {
  const int64_t n = (int64_t)a.R * ((mode == 0) ? a.g : a.d);
  hipLaunchKernelGGL(k_pairs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, mode);
}

template <typename T>
static void launch_ppo_fwd_t(const PpoFwdArgs &a, hipStream_t st) {
  int shift = 0;
  while ((1 << shift) < a.d) ++shift;
  const int64_t threads = (int64_t)a.R << shift;
  if (threads <= 256) {
    hipLaunchKernelGGL((k_ppo_root<T, true>), dim3(1), dim3(256), 0, st, a, shift);
    return;
  }
  hipLaunchKernelGGL((k_ppo_root<T, false>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a, shift);
  hipLaunchKernelGGL(k_ppo_loss, dim3(1), dim3(256), 0, st, a);
}

void launch_ppo_fwd(const PpoFwdArgs &a, hipStream_t st) {
  if (a.dtype == 0) launch_ppo_fwd_t<uint16_t>(a, st);
  else launch_ppo_fwd_t<float>(a, st);
}

}  // namespace gto
