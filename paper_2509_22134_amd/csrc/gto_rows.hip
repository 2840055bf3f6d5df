// Row-streaming kernels of the GTO hot path (gfx950, wave64).
//
//  k_row_stats : one workgroup per logits row.  Streams the row once with 16-byte loads and
//                produces max, log-sum-exp and the exact top-k (value descending, token id
//                ascending).  Used for draft rows (k = branching), target rows (k = 1 gives
//                the argmax) and for the reference rows on an accepted path.
//  k_ppo_bwd   : one workgroup per (root, path step).  Re-streams one draft row and writes
//                one fp32 gradient row  coef * (onehot - softmax).
//
// Both are HBM-bandwidth bound by design: per element they spend one conversion, one fused
// multiply-add, one exp2 and one add; the top-k costs one max per element, a few operations per
// group of them and a second read of the dozen groups that can hold it.
#include <type_traits>

#include "gto_device.h"
#include "gto_kernels.h"

namespace gto {

constexpr int kRowLoads = 4;   // 16-byte loads in flight per lane and tile (2 and 8 measured about 1 % slower)

// ----------------------------------------------------------------------------- top-k list
// A wave keeps the 64 best (value, id) pairs it has seen, sorted, one per lane (lane 0 = best).
// Inserting shifts the tail down by one lane with a single DPP move per register.
struct TopList {
  float v;
  int id;
  __device__ __forceinline__ void init() { v = neg_inf(); id = kNoId; }
  __device__ __forceinline__ void insert(float cv, int ci) {
    const bool b = better(cv, ci, v, id);
    const float uv = wave_shr1(v, __builtin_inff());
    const int ui = wave_shr1(id, -1);
    const bool bu = better(cv, ci, uv, ui);
    v = b ? (bu ? uv : cv) : v;
    id = b ? (bu ? ui : ci) : id;
  }
};

// k-th largest of the 64 lanes' values (k <= 64), the same in every lane: its ordered bits are built from the top,
// one compare and one scalar bit count per bit (BITS = 16 is exact for values that bf16 holds).
template <int BITS>
__device__ __forceinline__ float kth_largest_of_lanes(float x, int k) {
  const uint32_t o = ordered_bits(x);
  uint32_t t = 0;
#pragma unroll
  for (int b = 31; b > 31 - BITS; --b) {
    const uint32_t cand = t | (1u << b);
    if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(o >= cand)) >= k) t = cand;
  }
  // the low bits of a negative number's image are set
  if (BITS < 32 && (t & 0x80000000u) == 0u) t |= (1u << (32 - BITS)) - 1u;
  return from_ordered_bits(t);
}

// Streaming state of a wave: c, the log2-domain reference exponent all its lanes share, and per lane the running
// maximum m and s = sum 2^(x*log2(e) - c) over the elements the lane has seen.  c is an integer near the wave's
// maximum: it moves, rarely, when a tile exceeds it by more than 1 (exponents of the dominant terms stay small, whose
// rounding scales with them), and moving it scales s by an exact power of two.  A tile is summed in fp32 and then
// added to s in fp64: an fp32 running sum that already holds a dominant term would silently drop the many tiny ones
// added after it.  (A reference per lane instead costs an exp2 and fp64 products in every tile, fp64 adds per vector
// rather than per tile as much again: together a tenth of the loop's issue slots.)
struct WaveAcc {
  float m, c;
  double s;
  __device__ __forceinline__ void init() { m = neg_inf(); c = -3.402823466e+38f; s = 0.0; }
  __device__ __forceinline__ void refer(float cm) {
    if (__builtin_amdgcn_ballot_w64(__builtin_fmaf(cm, kLog2e, -c) > 1.f) == 0ull) return;
    const float cn = __builtin_rintf(wave_max_dpp(cm) * kLog2e);
    s = scale_pow2(s, c - cn);
    c = cn;
  }
};

// kDraftTopK: top-k collected at the end of the row (see LaneTop).  kDraftInsert: top-k kept in a sorted list while
// streaming (large k, or a row with more groups than LaneTop can number).
enum RowMode { kDraftTopK = 0, kTargetArgmax = 1, kLseOnly = 2, kDraftInsert = 3 };

// The exponents are taken with the fp32 log2(e), which is 1.3e-8 of itself too small: what a lane summed, whose terms
// lie near its maximum m, is that much times M - m too large against the row's maximum M, whose exponent the
// log-sum-exp corrects exactly.  Rows of N(0, 4), V = 128 256: the log-probabilities are 5.8e-8 too low on average
// without this, 2.3e-8 with it (26 112 rows of V = 32 000: 0.5 % slower; elsewhere the same).  (Lanes far below M, or
// without any finite value, hold nothing that counts.)
__device__ __forceinline__ double slope_fix(float m, float M) {
  constexpr double kSlope = 1.0 - (double)kLog2e * 0.69314718055994530942;
  return 1.0 + kSlope * (double)fmaxf(m - M, -256.f);
}

// Issues the LOADS 16-byte loads of one tile (lane l, load u: elements (u*64 + l)*EPV ...).
template <typename T, int LOADS, bool GUARD>
__device__ __forceinline__ void load_tile(const T *__restrict__ row, int tile_base, int V, int lane, u32x4 *q) {
  constexpr int EPV = Elem<T>::kPerVec;
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int e0 = tile_base + (u * kWave + lane) * EPV;
    if (!GUARD || e0 < V) {
      q[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row + e0));
    } else {
      const uint32_t none = (sizeof(T) == 2) ? 0xff80ff80u : 0xff800000u;      // -inf
      q[u] = u32x4{none, none, none, none};
    }
  }
}

// One tile as fp32 (entries beyond V: -inf) and its per-vector maxima.
template <typename T, int LOADS>
struct Tile {
  static constexpr int EPV = Elem<T>::kPerVec;
  float x[LOADS][EPV], mu[LOADS];
  template <bool GUARD>
  __device__ __forceinline__ void unpack(const u32x4 *q, int tile_base, int V, int lane) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      Elem<T>::unpack(q[u], x[u]);
      if (GUARD && V % EPV != 0) {             // the last vector is partly padding
        const int e0 = tile_base + (u * kWave + lane) * EPV;
#pragma unroll
        for (int e = 0; e < EPV; ++e)
          if (e0 + e >= V) x[u][e] = neg_inf();
      }
      mu[u] = x[u][0];
#pragma unroll
      for (int e = 1; e < EPV; ++e) mu[u] = fmaxf(mu[u], x[u][e]);
    }
  }
  __device__ __forceinline__ float max_of(int u0, int n) const {
    float m = mu[u0];
    for (int u = 1; u < n; ++u) m = fmaxf(m, mu[u0 + u]);
    return m;
  }
  // cm: the lane's maximum of the tile
  __device__ __forceinline__ void accumulate(WaveAcc &acc, float cm) const {
    acc.refer(cm);
    float p[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      p[u] = 0.f;
#pragma unroll
      for (int e = 0; e < EPV; ++e) p[u] += __builtin_amdgcn_exp2f(__builtin_fmaf(x[u][e], kLog2e, -acc.c));
    }
    static_assert(LOADS == 4, "sum of the vectors");
    acc.s += (double)((p[0] + p[1]) + (p[2] + p[3]));
    acc.m = fmaxf(acc.m, cm);
  }
  // inserts what beats the threshold (the k-th entry of the list, or a lower bound of it)
  template <bool GUARD>
  __device__ __forceinline__ void insert(int tile_base, int V, int lane, int ktop, TopList &top, float &thr_v, int &thr_i) const {
    const int lane_first = tile_base + lane * EPV;
    if (__builtin_amdgcn_ballot_w64(better(max_of(0, LOADS), lane_first, thr_v, thr_i)) == 0) return;
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      // skip a whole vector position when no lane's vector maximum can enter the list
      if (__builtin_amdgcn_ballot_w64(better(mu[u], tile_base + (u * kWave + lane) * EPV, thr_v, thr_i)) == 0) continue;
#pragma unroll
      for (int e = 0; e < EPV; ++e) {
        const int my_id = tile_base + (u * kWave + lane) * EPV + e;
        bool p = better(x[u][e], my_id, thr_v, thr_i);
        if (GUARD) p = p && (my_id < V);
        uint64_t mask = __builtin_amdgcn_ballot_w64(p);
        while (mask) {
          const int src = __builtin_ctzll(mask);
          mask &= mask - 1;
          const float cv = readlane(x[u][e], src);
          const int ci = tile_base + (u * kWave + src) * EPV + e;
          if (better(cv, ci, thr_v, thr_i)) {
            top.insert(cv, ci);
            const float nv = readlane(top.v, ktop - 1);
            const int ni = readlane(top.id, ktop - 1);
            if (better(nv, ni, thr_v, thr_i)) {
              thr_v = nv;
              thr_i = ni;
            }
          }
        }
      }
    }
  }
};

// ----------------------------------------------------------------------------- top-k at the end of the row
// While streaming, a lane only keeps the kTopGroups largest of its group maxima (a group: the kGroupVecs 16-byte
// vectors a lane holds of half a tile), each with the group's number.  At the end the wave takes T = the k-th largest
// of the lanes' best maxima: at least k elements reach T, so the top k lie in groups whose maximum reaches T, a dozen
// or so, which are read again and ranked.  A lane whose last entry reaches T may have had further such groups: all of
// that lane's groups are then read again (for k = 10 one wave in 10^4).
// Keeping a sorted list while streaming instead costs an insertion path in nearly every tile of a short row, and its
// serial latency where few waves are resident: 26 112 rows of V = 32 000 bf16 took 310 us, now 275 (a plain read of
// these rows takes 240); 196 rows of V = 151 936 41.8 us, now 14.1; 6528 fp32 rows of V = 32 003 147 us, now 134.
constexpr int kGroupVecs = 2;
constexpr int kTopGroups = 5;
constexpr int kDeferMaxK = 16;         // beyond, the lanes' lists hold the top k too rarely
template <typename T> struct LaneTop;
template <> struct LaneTop<uint16_t> {       // bf16: the group's number travels in the low half of its maximum
  float k[kTopGroups];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < kTopGroups; ++i) k[i] = neg_inf();
  }
  __device__ __forceinline__ void add(float m, int group) {
    // an infinity would turn into a NaN: the type's finite limits stand in for them
    m = __builtin_amdgcn_fmed3f(m, lowest(), __uint_as_float(0x7f7f0000u));
    m = __uint_as_float(__float_as_uint(m) | (uint32_t)group);
#pragma unroll
    for (int i = kTopGroups - 1; i > 0; --i) k[i] = __builtin_amdgcn_fmed3f(k[i - 1], k[i], m);
    k[0] = fmaxf(k[0], m);
  }
  __device__ __forceinline__ float value(int i) const { return __uint_as_float(__float_as_uint(k[i]) & 0xffff0000u); }
  __device__ __forceinline__ int group(int i) const { return (int)(__float_as_uint(k[i]) & 0xffffu); }
  __device__ static __forceinline__ float lowest() { return __uint_as_float(0xff7f0000u); }
};
template <> struct LaneTop<float> {
  float k[kTopGroups];
  int g[kTopGroups];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < kTopGroups; ++i) { k[i] = neg_inf(); g[i] = 0; }
  }
  __device__ __forceinline__ void add(float m, int group) {
    m = fmaxf(m, lowest());                  // above the empty entries' -inf, so that every group gets its number
    bool b[kTopGroups];
#pragma unroll
    for (int i = 0; i < kTopGroups; ++i) b[i] = m > k[i];
#pragma unroll
    for (int i = kTopGroups - 1; i > 0; --i) {
      k[i] = __builtin_amdgcn_fmed3f(k[i - 1], k[i], m);
      g[i] = b[i - 1] ? g[i - 1] : (b[i] ? group : g[i]);
    }
    k[0] = fmaxf(k[0], m);
    g[0] = b[0] ? group : g[0];
  }
  __device__ __forceinline__ float value(int i) const { return k[i]; }
  __device__ __forceinline__ int group(int i) const { return g[i]; }
  __device__ static __forceinline__ float lowest() { return -3.402823466e+38f; }
};

// What a wave's part of a row looks like: tiles first, first + step, ... below n_full, then (tail) the ragged one.
struct RowPart {
  int first, step, n_full;
  bool tail;
  __device__ __forceinline__ int full_tiles() const { return first < n_full ? (n_full - 1 - first) / step + 1 : 0; }
  __device__ __forceinline__ int tiles() const { return full_tiles() + (tail ? 1 : 0); }
  __device__ __forceinline__ int tile(int i) const { return i < full_tiles() ? first + i * step : n_full; }
};

// Sorted list of the wave's part by insertion, from the threshold (thr_v, thr_i) on; written to keys[0 .. ktop).
template <typename T, int LOADS>
__device__ __forceinline__ void insert_scan(const T *__restrict__ row, RowPart part, int V, int ktop, float thr_v, uint64_t *keys) {
  constexpr int TILE = kWave * LOADS * Elem<T>::kPerVec;
  const int lane = lane_id();
  TopList top;
  top.init();
  int thr_i = kNoId;
  Tile<T, LOADS> t;
  u32x4 q[LOADS];
  for (int i = part.first; i < part.n_full; i += part.step) {
    load_tile<T, LOADS, false>(row, i * TILE, V, lane, q);
    t.template unpack<false>(q, i * TILE, V, lane);
    t.template insert<false>(i * TILE, V, lane, ktop, top, thr_v, thr_i);
  }
  if (part.tail) {
    load_tile<T, LOADS, true>(row, part.n_full * TILE, V, lane, q);
    t.template unpack<true>(q, part.n_full * TILE, V, lane);
    t.template insert<true>(part.n_full * TILE, V, lane, ktop, top, thr_v, thr_i);
  }
  if (lane < ktop) keys[lane] = (top.id == kNoId) ? 0ull : rank_key(top.v, top.id);
}

// The top k of the wave's part from its lanes' group maxima: sorted keys[0 .. ktop), zeros behind the last one.
// groups: kTopGroups * 64 words of the wave's LDS; keys: 64.
template <typename T, int LOADS>
__device__ __forceinline__ void collect_topk(const T *__restrict__ row, const RowPart &part, int V, int ktop,
                                             const LaneTop<T> &lt, uint32_t *groups, uint64_t *keys) {
  constexpr int EPV = Elem<T>::kPerVec;
  constexpr int TILE = kWave * LOADS * EPV;
  constexpr int PER_TILE = LOADS / kGroupVecs;
  const int lane = lane_id();
  const int n_groups = part.tiles() * PER_TILE;                // per lane
  float T0 = kth_largest_of_lanes<(sizeof(T) == 2 ? 16 : 32)>(lt.value(0), ktop);
  if (T0 <= LaneTop<T>::lowest()) T0 = neg_inf();              // fewer than k lanes with a finite logit
  keys[lane] = 0ull;
  // lanes that may have more groups at T0 than they kept
  const bool over = n_groups > kTopGroups && lt.value(kTopGroups - 1) >= T0;
  uint64_t over_mask = __builtin_amdgcn_ballot_w64(over);
  int n = 0;
#pragma unroll
  for (int i = 0; i < kTopGroups; ++i) {
    const bool hit = (i < n_groups) && lt.value(i) >= T0 && !over;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(hit);
    if (hit) groups[n + lanes_below(mask)] = ((uint32_t)lt.group(i) << 6) | (uint32_t)lane;
    n += __builtin_popcountll(mask);
  }
  // read the groups again, kGroupVecs lanes each, and pack what reaches T0
  int n_keys = 0;
  auto pack = [&](bool on, int group, int l) {
    const int u = (group % PER_TILE) * kGroupVecs + lane % kGroupVecs;
    const int e0 = on ? (group / PER_TILE) * TILE + (u * kWave + l) * EPV : V;
    u32x4 q = {0u, 0u, 0u, 0u};
    if (e0 < V) q = *reinterpret_cast<const u32x4 *>(row + e0);
    float x[EPV];
    Elem<T>::unpack(q, x);
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
      const bool hit = (e0 + e < V) && x[e] >= T0;
      const uint64_t mask = __builtin_amdgcn_ballot_w64(hit);
      if (mask != 0ull) {
        const int at = n_keys + lanes_below(mask);
        if (hit && at < kWave) keys[at] = rank_key(x[e], e0 + e);
        n_keys += __builtin_popcountll(mask);
      }
    }
  };
  for (int base = 0; base < n; base += kWave / kGroupVecs) {
    const int idx = base + lane / kGroupVecs;
    const uint32_t gl = (idx < n) ? groups[idx] : 0u;
    pack(idx < n, (int)(gl >> 6), (int)(gl & 63u));
  }
  for (; over_mask != 0ull && n_keys <= kWave; over_mask &= over_mask - 1) {
    const int l = __builtin_ctzll(over_mask);
    for (int base = 0; base < n_groups; base += kWave / kGroupVecs) {
      const int idx = base + lane / kGroupVecs;
      const bool on = idx < n_groups;
      pack(on, on ? part.tile(idx / PER_TILE) * PER_TILE + idx % PER_TILE : 0, l);
    }
  }
  if (n_keys > kWave) {                                        // many ties at T0
    insert_scan<T, LOADS>(row, part, V, ktop, T0, keys);
    return;
  }
  // rank them: position i of the sorted list is the number of keys that beat mine (unused places hold 0)
  __builtin_amdgcn_wave_barrier();
  const uint64_t mine = keys[lane];
  int rank = 0;
  for (int i = 0; i < n_keys; i += 8) {
    uint64_t o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = keys[i + e];
#pragma unroll
    for (int e = 0; e < 8; ++e) rank += (o[e] > mine) ? 1 : 0;
  }
  __builtin_amdgcn_wave_barrier();
  keys[lane] = 0ull;
  __builtin_amdgcn_wave_barrier();
  if (mine != 0ull) keys[rank] = mine;
}

// Lowest id of the part's maximum m (each lane: its own first group that holds it).
template <typename T, int LOADS>
__device__ __forceinline__ int first_of_max(const T *__restrict__ row, int V, float m, float lane_m, int lane_tile) {
  constexpr int EPV = Elem<T>::kPerVec;
  constexpr int TILE = kWave * LOADS * EPV;
  const int lane = lane_id();
  int id = kNoId;
  if (lane_m == m) {
    u32x4 q[LOADS];
    load_tile<T, LOADS, true>(row, lane_tile * TILE, V, lane, q);
    float x[LOADS][EPV];
#pragma unroll
    for (int u = LOADS - 1; u >= 0; --u) {
      Elem<T>::unpack(q[u], x[u]);
      const int e0 = lane_tile * TILE + (u * kWave + lane) * EPV;
#pragma unroll
      for (int e = EPV - 1; e >= 0; --e)
        if (e0 + e < V && x[u][e] == m) id = e0 + e;
    }
  }
  return wave_min(id);
}

// What bounds it: memory, with the vector ALUs behind (6.7 issue slots per logit, 4 of them the quarter-rate exp2: 0.62
// of their time).  52 224 rows of V = 128 256 bf16 stream at 6.57 to 6.68 TB/s (target rows 6.86; a plain read reaches
// 7.0 to 7.1).  The next tile is requested before the current one is scanned, which matters where few waves
// share a compute unit (196 rows of V = 151 936: 16.1 us without, 14.1 with).
template <typename T, int WAVES, int LOADS, int MODE>
__global__ __launch_bounds__(WAVES *kWave) void k_row_stats(RowStatsArgs a) {
  constexpr int EPV = Elem<T>::kPerVec;
  constexpr int TILE = kWave * LOADS * EPV;
  constexpr int PER_TILE = LOADS / kGroupVecs;
  const int lane = lane_id();
  const int wave = (WAVES == 1) ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);

  // which row
  int r, l, j;
  int64_t oi;
  if (a.path_slot == nullptr) {
    r = blockIdx.x / a.rho;
    const int qq = blockIdx.x - r * a.rho;
    l = (qq == 0) ? 0 : 1 + (qq - 1) / a.kslots;
    j = (qq == 0) ? 0 : (qq - 1) % a.kslots;
    oi = stat_index(r, l, j, a.d, a.kslots);
    if (a.row_need != nullptr && a.row_need[oi] == 0) return;
  } else {  // rows on an accepted path: block = (root, step)
    r = blockIdx.x / a.d;
    l = blockIdx.x - r * a.d;
    j = a.path_slot[(int64_t)r * a.d + l];
    if (j < 0) return;
    oi = (int64_t)r * a.d + l;
  }
  const T *row = static_cast<const T *>(a.logits) + stat_index(r, l, j, a.d, a.kslots) * a.row_stride;
  const int V = a.V;
  const int n_full = V / TILE;
  const RowPart part{wave, WAVES, n_full, n_full * TILE < V && (n_full % WAVES) == wave};

  WaveAcc acc;
  acc.init();
  LaneTop<T> top_groups;
  top_groups.init();
  int best_t = wave;              // argmax: the first tile that holds this lane's maximum
  TopList top;                    // kDraftInsert
  top.init();
  float thr_v = neg_inf();
  int thr_i = kNoId;

  Tile<T, LOADS> t;
  auto scan = [&](const u32x4 *q, int i, auto guard) {
    constexpr bool GUARD = decltype(guard)::value;
    t.template unpack<GUARD>(q, i * TILE, V, lane);
    const float cm = t.max_of(0, LOADS);
    if (MODE == kTargetArgmax) best_t = (cm > acc.m) ? i : best_t;
    t.accumulate(acc, cm);
    if (MODE == kDraftTopK) {
#pragma unroll
      for (int h = 0; h < PER_TILE; ++h) top_groups.add(t.max_of(h * kGroupVecs, kGroupVecs), i * PER_TILE + h);
    } else if (MODE == kDraftInsert) {
      if (i == wave) {            // the first tile seeds the threshold: at least k of its elements reach it
        thr_v = kth_largest_of_lanes<32>(cm, a.ktop);
        thr_i = kNoId;
      }
      t.template insert<GUARD>(i * TILE, V, lane, a.ktop, top, thr_v, thr_i);
    }
  };
  // (the scheduling barriers keep a tile's loads in front of the scan of the one before)
  auto fetch = [&](int i, u32x4 *q) {
    load_tile<T, LOADS, false>(row, i * TILE, V, lane, q);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (MODE == kDraftInsert) {
    for (int i = wave; i < n_full; i += WAVES) {
      u32x4 q[LOADS];
      fetch(i, q);
      scan(q, i, std::false_type{});
    }
  } else if (wave < n_full) {
    u32x4 q0[LOADS], q1[LOADS];
    int i = wave;
    fetch(i, q0);
    for (; i + 2 * WAVES < n_full; i += 2 * WAVES) {
      fetch(i + WAVES, q1);
      scan(q0, i, std::false_type{});
      fetch(i + 2 * WAVES, q0);
      scan(q1, i + WAVES, std::false_type{});
    }
    if (i + WAVES < n_full) {
      fetch(i + WAVES, q1);
      scan(q0, i, std::false_type{});
      scan(q1, i + WAVES, std::false_type{});
    } else {
      scan(q0, i, std::false_type{});
    }
  }
  if (part.tail) {
    u32x4 q[LOADS];
    load_tile<T, LOADS, true>(row, n_full * TILE, V, lane, q);
    scan(q, n_full, std::true_type{});
  }

  const float Mw = wave_max_dpp(acc.m);
  const double Sw = wave_sum_dpp(acc.s * slope_fix(acc.m, Mw));

  __shared__ uint32_t sh_groups[WAVES * kTopGroups * kWave];
  __shared__ __align__(16) uint64_t sh_key[WAVES * kWave];      // each wave's sorted list
  __shared__ float sh_M[WAVES], sh_C[WAVES];
  __shared__ double sh_S[WAVES];
  if (MODE == kDraftTopK) {
    collect_topk<T, LOADS>(row, part, V, a.ktop, top_groups, sh_groups + wave * kTopGroups * kWave, sh_key + wave * kWave);
  } else if (MODE == kTargetArgmax) {
    const int id = part.tiles() ? first_of_max<T, LOADS>(row, V, Mw, acc.m, best_t) : kNoId;
    if (lane == 0) sh_key[wave * kWave] = (id == kNoId) ? 0ull : rank_key(Mw, id);
  } else if (MODE == kDraftInsert) {
    sh_key[wave * kWave + lane] = (top.id == kNoId) ? 0ull : rank_key(top.v, top.id);
  }
  if (WAVES > 1) {
    if (lane == 0) {
      sh_M[wave] = Mw;
      sh_C[wave] = acc.c;
      sh_S[wave] = Sw;
    }
    __syncthreads();
    if (wave != 0) return;
  }
  // the first wave finishes the row
  float M = Mw, C = acc.c;
  double S = Sw;
  if (WAVES > 1) {
    const bool on = lane < WAVES;
    const float wc = on ? sh_C[lane] : neg_inf();
    const float wm = on ? sh_M[lane] : neg_inf();
    M = wave_max_dpp(wm);
    C = wave_max_dpp(wc);
    S = wave_sum_dpp(on ? scale_pow2(sh_S[lane], wc - C) * slope_fix(wm, M) : 0.0);
  }
  // log2-domain total is C + log2(S); the row maximum contributes exactly M*log2e of it.
  const double lse = (double)M + kLn2 * (((double)C - (double)M * (double)kLog2e) + log2(S));
  if (lane == 0) {
    if (a.row_max) a.row_max[oi] = M;
    a.row_lse[oi] = (float)lse;
  }
  if (MODE == kLseOnly || a.top_tok == nullptr) return;
  const int ktop = (MODE == kTargetArgmax) ? 1 : a.ktop;
  // position `lane` of the row's list: of the only wave's, or by ranking the waves' candidates
  uint64_t key = 0ull;
  if (WAVES == 1) {
    __builtin_amdgcn_wave_barrier();
    key = sh_key[lane];
  } else {
    const int total = WAVES * ktop;
    __shared__ __align__(16) uint64_t sh_all[WAVES * kWave + 8], sh_out[kWave];
    sh_out[lane] = 0ull;
    for (int i = lane; i < total + 8; i += kWave) sh_all[i] = (i < total) ? sh_key[(i / ktop) * kWave + i % ktop] : 0ull;
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < total; i += kWave) {
      const uint64_t mine = sh_all[i];
      int rank = 0;
      for (int u = 0; u < total; u += 8) {
        uint64_t o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = sh_all[u + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) rank += (o[e] > mine) ? 1 : 0;
      }
      if (mine != 0ull && rank < ktop) sh_out[rank] = mine;
    }
    __builtin_amdgcn_wave_barrier();
    key = sh_out[lane];
  }
  if (lane < ktop) {
    // A row that holds NaNs can leave ranks unclaimed (a NaN wins no comparison).  Such a row's values are
    // unspecified, but every id written must be a token of the vocabulary: unclaimed ranks get token `rank`
    // (V >= ktop) with probability zero.
    const bool ok = key != 0ull;
    a.top_tok[oi * ktop + lane] = ok ? key_index(key) : lane;
    // clamped: rounding must never make a log-probability positive (a child may not outrank its parent)
    if (a.top_logp) a.top_logp[oi * ktop + lane] = ok ? fminf((float)((double)key_score(key) - lse), 0.f) : neg_inf();
  }
}

// Four consecutive elements of a row, at element index 4 * q4, as fp32: one 8-byte (bf16) or 16-byte (fp32)
// nontemporal load.  A wave's 64 such loads are contiguous, and so are the 64 16-byte stores of the four
// fp32 results: every store instruction fills whole cache lines (two 16-byte stores per lane, 32 bytes
// apart between lanes, leave every line half written and cost ~1.7x the write traffic, measured).
template <typename T>
__device__ __forceinline__ void load4(const T *row, int q4, float *x);
template <>
__device__ __forceinline__ void load4<uint16_t>(const uint16_t *row, int q4, float *x) {
  const u32x2 q = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(row) + q4);
  x[0] = __uint_as_float(q.x << 16); x[1] = __uint_as_float(q.x & 0xffff0000u);
  x[2] = __uint_as_float(q.y << 16); x[3] = __uint_as_float(q.y & 0xffff0000u);
}
template <>
__device__ __forceinline__ void load4<float>(const float *row, int q4, float *x) {
  const u32x4 q = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row) + q4);
  x[0] = __uint_as_float(q.x); x[1] = __uint_as_float(q.y); x[2] = __uint_as_float(q.z); x[3] = __uint_as_float(q.w);
}
// The same four elements as they come from memory (to be carried across loop trips without the unpacking
// being scheduled right behind the load), and their conversion.
template <typename T> struct Raw4;
template <> struct Raw4<uint16_t> {
  typedef u32x2 type;
  __device__ static __forceinline__ type load(const uint16_t *row, int q4) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(row) + q4);
  }
  __device__ static __forceinline__ void unpack(const type &q, float *x) {
    x[0] = __uint_as_float(q.x << 16); x[1] = __uint_as_float(q.x & 0xffff0000u);
    x[2] = __uint_as_float(q.y << 16); x[3] = __uint_as_float(q.y & 0xffff0000u);
  }
};
template <> struct Raw4<float> {
  typedef u32x4 type;
  __device__ static __forceinline__ type load(const float *row, int q4) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row) + q4);
  }
  __device__ static __forceinline__ void unpack(const type &q, float *x) {
    x[0] = __uint_as_float(q.x); x[1] = __uint_as_float(q.y); x[2] = __uint_as_float(q.z); x[3] = __uint_as_float(q.w);
  }
};

// N consecutive elements at element index N * idx: N == 4 as above; N == the elements of a 16-byte
// vector for kernels that only read (16-byte loads stream ~20 % faster than 8-byte ones, measured).
template <typename T, int N>
__device__ __forceinline__ void load_group(const T *row, int idx, float *x) {
  if constexpr (N == 4) {
    load4<T>(row, idx, x);
  } else {
    static_assert(N == Elem<T>::kPerVec, "group is four elements or one 16-byte vector");
    Elem<T>::unpack(__builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row) + idx), x);
  }
}

// ------------------------------------------------------------------------------- backward
// One workgroup of 16 waves per (root, step): only the few hundred rows on accepted paths do any work,
// so the parallelism has to come from inside the row.
constexpr int kBwdThreads = 1024;
template <typename T, bool VEC>
__global__ __launch_bounds__(kBwdThreads) void k_ppo_bwd(PpoBwdArgs a) {
  // step-major order: the rows that carry a gradient (short paths: mostly the first steps) then sit densely at
  // the front of the grid and spread over the compute units (root-major order: 106 us instead of 80)
  const int n_roots = gridDim.x / a.d;
  const int t = blockIdx.x / n_roots;
  const int r = blockIdx.x - t * n_roots;
  const int64_t rt = (int64_t)r * a.d + t;
  const int j = a.path_slot[rt];
  const float coef = a.coef[r];
  const bool valid = (j >= 0) && (coef != 0.f);
  if (threadIdx.x == 0) a.grad_slot[rt] = valid ? j : -1;
  float *__restrict__ out = a.grad_rows + rt * (int64_t)a.V;
  const int V = a.V;
  if (!valid) {
    if (a.zero_fill) {
      if (VEC) {
        f32x4 *o4 = reinterpret_cast<f32x4 *>(out);
        for (int i = threadIdx.x; i < V / 4; i += blockDim.x) o4[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      } else {
        for (int i = threadIdx.x; i < V; i += blockDim.x) out[i] = 0.f;
      }
    }
    return;
  }
  const int tok = a.sel_tok[(int64_t)r * a.g + a.path_node[rt]];
  const float lse = a.row_lse[stat_index(r, t, j, a.d, a.k)];
  const T *__restrict__ row = static_cast<const T *>(a.logits) + stat_index(r, t, j, a.d, a.k) * a.row_stride;
  // Every entry but the token's is -coef * p_v.  The token's entry coef * (1 - p_tok) is formed as
  // coef * (sum of the other probabilities): when p_tok is close to 1 the subtraction would cancel.
  float others = 0.f;
  bool own_tok = false;
  if (VEC) {
    // Groups of four elements, kBwdUnroll groups per step and lane.  The loads of the next step are issued
    // before the stores of this one: loads and stores share one in-order counter, so a wait for loads that
    // were issued after a batch of stores would also wait for those stores to be acknowledged by memory.
    constexpr int kBwdUnroll = 8;
    const int n4 = V / 4;
    typedef typename Raw4<T>::type raw_t;
    raw_t x[kBwdUnroll], xn[kBwdUnroll];
    // (past the end of the row the last group is fetched again: a branch around a load would end in a wait
    // for everything outstanding)
    auto fetch = [&](raw_t (&dst)[kBwdUnroll], int i0) {
#pragma unroll
      for (int u = 0; u < kBwdUnroll; ++u) dst[u] = Raw4<T>::load(row, min(i0 + u * kBwdThreads, n4 - 1));
    };
    auto emit = [&](const raw_t (&src)[kBwdUnroll], int i0) {
#pragma unroll
      for (int u = 0; u < kBwdUnroll; ++u) {
        const int i = i0 + u * kBwdThreads;
        if (i >= n4) continue;
        float xv[4];
        Raw4<T>::unpack(src[u], xv);
        float gq[4];
        float part = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = __builtin_amdgcn_exp2f((xv[e] - lse) * kLog2e);
          gq[e] = -coef * p;
          const bool is_tok = (i * 4 + e == tok);
          own_tok = own_tok || is_tok;
          part += is_tok ? 0.f : p;
        }
        others += part;
        const f32x4 o = {gq[0], gq[1], gq[2], gq[3]};
        __builtin_nontemporal_store(o, reinterpret_cast<f32x4 *>(out) + i);
      }
    };
    // two steps per trip, the two register sets swapping roles (no copies between them)
    constexpr int kStep = kBwdUnroll * kBwdThreads;
    fetch(x, threadIdx.x);
    for (int i0 = threadIdx.x; i0 < n4; i0 += 2 * kStep) {
      fetch(xn, i0 + kStep);
      emit(x, i0);
      fetch(x, i0 + 2 * kStep);
      emit(xn, i0 + kStep);
    }
  } else {
    for (int i = threadIdx.x; i < V; i += blockDim.x) {
      const float xv = Elem<T>::load1(row + i);
      const float p = __builtin_amdgcn_exp2f((xv - lse) * kLog2e);
      const bool is_tok = (i == tok);
      own_tok = own_tok || is_tok;
      others += is_tok ? 0.f : p;
      out[i] = -coef * p;
    }
  }
  __shared__ double s_part[kBwdThreads];
  s_part[threadIdx.x] = (double)others;
  __syncthreads();
  for (int off = kBwdThreads / 2; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) s_part[threadIdx.x] += s_part[threadIdx.x + off];
    __syncthreads();
  }
  // the thread that stored the token's entry overwrites it (same thread, program order)
  if (own_tok) out[tok] = (float)((double)coef * s_part[0]);
}

// ------------------------------------------------------------------------------- token-level loss
// One workgroup per root: streams the root rows (slot (0,0)) of the draft and the target logits
// together.  Forward: H = lse_M - sum_v p_T(v) d_v.  Backward: scale * (p_M - p_T) as an fp32 row.
constexpr int kTokThreads = 256;
template <typename T, bool BWD, bool VEC>
__global__ __launch_bounds__(kTokThreads) void k_token_loss(TokenLossArgs a) {
  const int r = blockIdx.x;
  const float w = a.weight ? a.weight[r] : 1.f;
  const int64_t si = stat_index(r, 0, 0, a.d, a.k);
  const int64_t lo = a.root_stride ? (int64_t)r * a.root_stride : si * a.row_stride;
  const T *__restrict__ drow = static_cast<const T *>(a.draft_logits) + lo;
  const T *__restrict__ trow = static_cast<const T *>(a.target_logits) + lo;
  const float d_lse = a.d_lse[si], t_lse = a.t_lse[si];
  const int V = a.V;
  float *__restrict__ out = BWD ? a.grad + (int64_t)r * V : nullptr;
  const float scale = BWD ? a.grad_scale * w * a.inv_count[0] : 0.f;
  double acc = 0.0;
  // Groups of kGroup elements, kUnroll groups of each row in flight per lane.  The backward takes
  // groups of four so that its stores fill whole lines (see load4); the forward, which stores nothing,
  // takes whole 16-byte vectors.  VEC: V % kGroup == 0 and, for the backward, 16-byte aligned output
  // rows; otherwise one element at a time.
  constexpr int kGroup = BWD ? 4 : Elem<T>::kPerVec;
  constexpr int kUnroll = BWD ? 4 : 2;
  const int n4 = VEC ? V / kGroup : 0;
  for (int i0 = threadIdx.x; i0 < n4; i0 += kUnroll * kTokThreads) {
    float xd[kUnroll][kGroup], xt[kUnroll][kGroup];
    // past the end of the rows the last group is fetched again (a branch around a load would end in a wait
    // for everything outstanding)
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int i = min(i0 + u * kTokThreads, n4 - 1);
      load_group<T, kGroup>(drow, i, xd[u]);
      load_group<T, kGroup>(trow, i, xt[u]);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int i = i0 + u * kTokThreads;
      if (i >= n4) continue;
      if constexpr (BWD) {
        float gq[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pm = __builtin_amdgcn_exp2f((xd[u][e] - d_lse) * kLog2e);
          const float pt = __builtin_amdgcn_exp2f((xt[u][e] - t_lse) * kLog2e);
          gq[e] = scale * (pm - pt);
        }
        const f32x4 o = {gq[0], gq[1], gq[2], gq[3]};
        __builtin_nontemporal_store(o, reinterpret_cast<f32x4 *>(out) + i);
      } else {
        float part = 0.f;
#pragma unroll
        for (int e = 0; e < kGroup; ++e) {
          const float pt = __builtin_amdgcn_exp2f((xt[u][e] - t_lse) * kLog2e);
          part += (pt > 0.f) ? pt * (xd[u][e] - d_lse) : 0.f;      // 0 * log 0 := 0
        }
        acc += (double)part;
      }
    }
  }
  if (!VEC) {
    for (int i = threadIdx.x; i < V; i += kTokThreads) {
      const float dv = Elem<T>::load1(drow + i), tv = Elem<T>::load1(trow + i);
      const float pt = __builtin_amdgcn_exp2f((tv - t_lse) * kLog2e);
      if (BWD) out[i] = scale * (__builtin_amdgcn_exp2f((dv - d_lse) * kLog2e) - pt);
      else acc += (double)((pt > 0.f) ? pt * (dv - d_lse) : 0.f);
    }
  }
  if (BWD) return;
  __shared__ double s_red[kTokThreads];
  s_red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = kTokThreads / 2; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) s_red[threadIdx.x] += s_red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.loss_rows[r] = (float)(-(double)w * s_red[0]);
}

// single workgroup: |I| = sum of weights, loss = sum of rows / |I| (fixed-shape tree reductions)
__global__ __launch_bounds__(256) void k_token_loss_mean(TokenLossArgs a) {
  __shared__ double s_a[256], s_b[256];
  double sa = 0.0, sb = 0.0;
  for (int r = threadIdx.x; r < a.R; r += 256) {
    sa += (double)a.loss_rows[r];
    sb += a.weight ? (double)a.weight[r] : 1.0;
  }
  s_a[threadIdx.x] = sa;
  s_b[threadIdx.x] = sb;
  __syncthreads();
  for (int off = 128; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) {
      s_a[threadIdx.x] += s_a[threadIdx.x + off];
      s_b[threadIdx.x] += s_b[threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double n = s_b[0];
    a.loss[0] = (n > 0.0) ? (float)(s_a[0] / n) : 0.f;
    a.inv_count_out[0] = (n > 0.0) ? (float)(1.0 / n) : 0.f;
  }
}

void launch_token_loss(const TokenLossArgs &a, int dtype, bool bwd, hipStream_t st) {
  const dim3 grid(a.R), block(kTokThreads);
  // rows start 16-byte aligned; the backward walks groups of four elements, the forward 16-byte vectors
  const int group = bwd ? 4 : (dtype == 0 ? 8 : 4);
  const bool vec = (a.V % group == 0) && (!bwd || (reinterpret_cast<uintptr_t>(a.grad) & 15) == 0);
  if (bwd) {
    if (dtype == 0) {
      if (vec) hipLaunchKernelGGL((k_token_loss<uint16_t, true, true>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((k_token_loss<uint16_t, true, false>), grid, block, 0, st, a);
    } else {
      if (vec) hipLaunchKernelGGL((k_token_loss<float, true, true>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((k_token_loss<float, true, false>), grid, block, 0, st, a);
    }
    return;
  }
  if (dtype == 0) {
    if (vec) hipLaunchKernelGGL((k_token_loss<uint16_t, false, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_token_loss<uint16_t, false, false>), grid, block, 0, st, a);
  } else {
    if (vec) hipLaunchKernelGGL((k_token_loss<float, false, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_token_loss<float, false, false>), grid, block, 0, st, a);
  }
  hipLaunchKernelGGL(k_token_loss_mean, dim3(1), dim3(256), 0, st, a);
}

// ------------------------------------------------------------------------------- calibration copy
// Plain 16-byte-per-lane copy of a known size: the yardstick that hardware HBM counters of the
// row kernels are scaled by.
__global__ __launch_bounds__(256) void k_copy16(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int64_t nvec) {
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += step) dst[i] = src[i];
}

void launch_copy16(const void *src, void *dst, int64_t bytes, hipStream_t st) {
  hipLaunchKernelGGL(k_copy16, dim3(16384), dim3(256), 0, st, static_cast<const u32x4 *>(src),
                     static_cast<u32x4 *>(dst), bytes / 16);
}

// ------------------------------------------------------------------------------- launchers
// One wave per row streams best when rows are long and plentiful (one threshold, one list per
// row).  With few rows, or short ones, split a row over more waves so the chip stays full.
static int choose_waves(int forced, int V, int blocks, int elems_per_tile) {
  if (forced) return forced;
  const int64_t wave_slots = 256 * 28;   // CUs x resident waves per CU at this kernel's register use
  int w = 1;
  while (w < 8 && (int64_t)blocks * w < wave_slots && V / (2 * w) >= 2 * elems_per_tile) w *= 2;
  return w;
}


template <typename T, int MODE>
static void launch_row_stats_m(const RowStatsArgs &a, int blocks, hipStream_t st) {
  const int w = choose_waves(a.waves, a.V, blocks, kWave * kRowLoads * Elem<T>::kPerVec);
  switch (w) {
    case 1: hipLaunchKernelGGL((k_row_stats<T, 1, kRowLoads, MODE>), dim3(blocks), dim3(64), 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_row_stats<T, 2, kRowLoads, MODE>), dim3(blocks), dim3(128), 0, st, a); break;
    case 8: hipLaunchKernelGGL((k_row_stats<T, 8, kRowLoads, MODE>), dim3(blocks), dim3(512), 0, st, a); break;
    default: hipLaunchKernelGGL((k_row_stats<T, 4, kRowLoads, MODE>), dim3(blocks), dim3(256), 0, st, a); break;
  }
}

template <typename T>
static void launch_row_stats_t(const RowStatsArgs &a, int blocks, hipStream_t st) {
  if (a.top_tok == nullptr) launch_row_stats_m<T, kLseOnly>(a, blocks, st);
  else if (a.ktop == 1) launch_row_stats_m<T, kTargetArgmax>(a, blocks, st);
  // the deferred top-k numbers a row's groups in 16 bits
  else if (a.ktop <= kDeferMaxK && (int64_t)a.V / (kWave * Elem<T>::kPerVec * kGroupVecs) < 65000)
    launch_row_stats_m<T, kDraftTopK>(a, blocks, st);
  else launch_row_stats_m<T, kDraftInsert>(a, blocks, st);
}

void launch_row_stats(const RowStatsArgs &a, int dtype, int blocks, hipStream_t st) {
  if (dtype == 0) launch_row_stats_t<uint16_t>(a, blocks, st);
  else launch_row_stats_t<float>(a, blocks, st);
}

void launch_ppo_bwd(const PpoBwdArgs &a, int dtype, int blocks, hipStream_t st) {
  const bool vec = (a.V % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.grad_rows) & 15) == 0);
  if (dtype == 0) {
    if (vec) hipLaunchKernelGGL((k_ppo_bwd<uint16_t, true>), dim3(blocks), dim3(kBwdThreads), 0, st, a);
    else hipLaunchKernelGGL((k_ppo_bwd<uint16_t, false>), dim3(blocks), dim3(kBwdThreads), 0, st, a);
  } else {
    if (vec) hipLaunchKernelGGL((k_ppo_bwd<float, true>), dim3(blocks), dim3(kBwdThreads), 0, st, a);
    else hipLaunchKernelGGL((k_ppo_bwd<float, false>), dim3(blocks), dim3(kBwdThreads), 0, st, a);
  }
}

}  // namespace gto
