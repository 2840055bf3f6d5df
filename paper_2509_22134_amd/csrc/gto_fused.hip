// Fused LM-head variant: logits = hidden . W^T are produced tile by tile on the matrix cores and
// reduced to the row statistics (max, log-sum-exp, exact top-k) in the epilogue, so the logits
// never reach HBM.
//
//  k_fused_rows  : 256 x 256 output tile per workgroup iteration: 8 waves, two per SIMD, each 128 x 64
//                  as 8 x 4 MFMA 16x16x32 bf16 tiles with fp32 accumulators.  K slabs of 64 go from
//                  global memory straight into one of two LDS stages; the two waves of a SIMD take turns
//                  between the matrix cores and everything else (see the main loop).  The launch is
//                  persistent (one workgroup per compute unit); a workgroup keeps its 256 rows while it
//                  moves along a patch row of the tile grid.  After each tile the accumulators are staged
//                  through LDS column-major; in the statistics passes threads t and t + 256 own row t
//                  (half of the columns each) and fold the new logits into a running (max, sum, top-k
//                  list) in registers; in the writing passes (gradient rows, bf16 planes, stored logits)
//                  the eight lanes of a row write contiguous bytes.
//  k_fused_merge : combines the partial results of a row (one per group and column phase) into the
//                  final statistics.
//  k_gather_dot  : single logits (hidden row . W row) for the few (row, token) pairs the reward
//                  and the surrogate need.
#include <algorithm>

#include "gto_device.h"
#include "gto_kernels.h"

namespace gto {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int FBM = 256, FBN = 256;
constexpr int FTHREADS = 512;                      // 8 waves: two groups of four, one wave of each group per SIMD
constexpr int FBK = 64;                            // k extent of one LDS stage (a whole 128-byte line per row)
constexpr int FROWB = FBK * 2;                     // bytes per staged row (bf16)
constexpr int FOP_B = FBM * FROWB;                 // bytes of one operand in a stage
constexpr int FSTAGE_B = 2 * FOP_B;                // 256 hidden rows, then 256 W rows
constexpr int FKT = 16;                            // capacity of the per-thread top list
constexpr int FSTG_CM = FBM + 4;                   // staging column stride (floats), column-major staging
constexpr size_t kFusedLdsBytes = (size_t)2 * FSTAGE_B;
static_assert(FBM == FBN, "the two operands share one stage layout");
static_assert(kFusedLdsBytes >= (size_t)64 * FSTG_CM * sizeof(float), "staging area must fit");
static_assert(63 * FSTG_CM * sizeof(float) < 65536, "a row's 64 staged columns are reached with immediate offsets");
static_assert(kFusedLdsBytes >= (size_t)FBM * (sizeof(double) + 8 + FKT * 8), "a flush hands 256 row states over");

// 16 bytes per lane from global memory straight into LDS: lane l of the wave lands at lds_addr + 16 l
// (lds_addr is wave-uniform; the compiler moves it into M0); counted by vmcnt.
__device__ __forceinline__ void load_to_lds16(unsigned lds_addr, const void *g) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                   (__attribute__((address_space(3))) void *)(uintptr_t)lds_addr, 16, 0, 0);
}

// index of the statistics entry (= logits slot) of the q-th used row of root r
__device__ __forceinline__ int64_t used_slot_index(int64_t gidx, int rho, int d, int k) {
  const int64_t r = gidx / rho;
  const int q = (int)(gidx - r * rho);
  return r * d * k + (q ? k + q - 1 : 0);
}

template <int KT>
struct RowState {
  float m, c;
  double s;
  float v[KT];
  int id[KT];
};

template <int KT>
__device__ __forceinline__ void list_insert(float (&v)[KT], int (&id)[KT], float x, int xi) {
  // v/id sorted best first; branch-free shift-insert
  bool prev = false;   // "x beats entry i-1"
  float pv = 0.f;
  int pi = 0;
#pragma unroll
  for (int i = 0; i < KT; ++i) {
    const bool b = better(x, xi, v[i], id[i]);
    const float cv = v[i];
    const int ci = id[i];
    v[i] = b ? (prev ? pv : x) : cv;
    id[i] = b ? (prev ? pi : xi) : ci;
    prev = b;
    pv = cv;
    pi = ci;
  }
}

// ---- the GEMM main loop: acc += A . B^T over n_slabs k slabs of 64, for the 256 x 256 tile of the workgroup.
// Wave (wm, wn) = (wave / 4, wave % 4) owns rows 128 wm .. + 127 and 64 columns as 8 x 4 MFMA 16x16x32 tiles; its
// tile (i, j) holds rows 128 wm + 16 i and columns 64 j + 16 wn (the callers lay the column operand out so): the
// j-th column tiles of the four column waves are 64 consecutive columns, what one epilogue phase takes.
//
// What bounds it: the matrix pipe, as long as nothing else stands in its way.  One wave per SIMD that issues
// fragment reads and loads between its MFMAs stalls the pipe whenever one of those instructions is held up
// (measured: 0.66 busy, 110 ms for 58 368 x 8192 x 128 256).  So two waves share a SIMD and take turns: the waves of
// group 0 (wm = 0) and of group 1 are half a phase apart, and between two barriers one group issues 32 MFMAs (512
// matrix-pipe cycles) while the other reads fragments and requests loads for its next 32.  A slab is two such phases:
//     phase   MFMAs       fragments read before them    loads requested before them
//       0     A0 x B      B (8 reads), A0 (8)           A1 of slab s + 1
//       1     A1 x B      A1 (8)                        B, A0 of slab s + 2
// (A0 / A1: the first and second 64 rows of each row half; B: the wave's 64 columns.)  A part of a stage is requested
// again as soon as both groups have read it, so two stages of 64 KB keep every load in flight for one and a half
// slabs (about 3000 clocks).  Every phase ends its reading part with `vmcnt(8)`: the eight newest load instructions
// are exactly what the next phase does not read; the barrier extends that to the other waves' shares.
// Measured with the statistics epilogue: 16 359 x 8192 x 128 256 in 24.4 ms (1.41 PFLOP/s at 1.60 GHz with the matrix
// pipe 0.83 busy: the power limit holds the clock; the library's GEMM reaches 1.55 in the same process), 58 368 rows
// in 89 to 93 ms.  Phases of 16 MFMAs, four a slab, lose more to the barriers (0.77 busy at 1.80 GHz): 2.5 % slower
// in a run of 25 ms, the same in one of 90.  Four waves of 128 x 128 with accumulators pinned to the accumulation
// registers read a third less LDS but reach 1.31 PFLOP/s without an epilogue.
struct Slab {
  unsigned wA, wB;               // LDS byte address of this wave's share of A0 / B0 in stage 0
  const unsigned char *ldsb;     // the stages
  int fA, fB;                    // byte offset of this lane's fragments in stage 0, k step 0 (k step 1: offset ^ 64)
};

template <int VM>
__device__ __forceinline__ void end_of_reads() {
  // all fragment reads have returned (the other group may request over what they read), loads as counted
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(VM) : "memory");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

template <int I0>
__device__ __forceinline__ void half_tile(f32x4 (&acc)[8][4], const bf16x8 (&fa)[2][4], const bf16x8 (&fb)[2][4]) {
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int j = (i & 1) ? 3 - jj : jj;        // one operand changes per MFMA
        acc[I0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][j], acc[I0 + i][j], 0, 0, 0);
      }
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// N 16-row fragment tiles from `off` bytes behind this lane's fragment offset (both k steps)
template <int N>
__device__ __forceinline__ void read_frags(bf16x8 (&f)[2][N], const unsigned char *ldsb, int frag, int off) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < N; ++t)
      f[h][t] = *reinterpret_cast<const bf16x8 *>(ldsb + (frag ^ (64 * h)) + off + t * 16 * FROWB);
}
// this wave's two load instructions of one quarter of a stage; the pointers move on by one slab
__device__ __forceinline__ void request(unsigned lds_addr, const uint16_t *&p0, const uint16_t *&p1) {
  load_to_lds16(lds_addr, p0);
  load_to_lds16(lds_addr + 1024, p1);
  p0 += FBK;
  p1 += FBK;
}

// One slab.  LOAD_A1: slab s + 1 exists and the second half of its row operand is requested.  LOAD: slab s + 2 exists
// and the rest of it is requested.  V0, V1: outstanding load instructions allowed at the end of each phase's reads.
template <bool LOAD_A1, bool LOAD, int V0, int V1>
__device__ __forceinline__ void slab_step(f32x4 (&acc)[8][4], const Slab &r, const uint16_t *(&ap)[4],
                                          const uint16_t *(&bp)[4], int stage) {
  const int off = stage * FSTAGE_B, nxt = FSTAGE_B - off;
  bf16x8 fa[2][4], fb[2][4];
  read_frags<4>(fb, r.ldsb, r.fB, off);
  read_frags<4>(fa, r.ldsb, r.fA, off);
  if (LOAD_A1) request(r.wA + nxt + 64 * FROWB, ap[2], ap[3]);
  end_of_reads<V0>();
  half_tile<0>(acc, fa, fb);
  read_frags<4>(fa, r.ldsb, r.fA, off + 64 * FROWB);
  if (LOAD) {
    request(r.wB + off, bp[0], bp[1]);
    request(r.wA + off, ap[0], ap[1]);
    request(r.wB + off + 32 * FROWB, bp[2], bp[3]);
  }
  end_of_reads<V1>();
  half_tile<4>(acc, fa, fb);
}

// Which rows of the two operands this lane fetches: load i of quarter A0 is tile row a_row(i), of A1 a_row(i) + 64;
// of B0 staged column b_row(i), of B1 b_row(i) + 32; staged column c is the operand's row b_col(c).  The 16 bytes
// at k unit k_unit(i) of that row land at unit lane % 8, which spreads the fragment reads (16 rows at one k unit)
// over all LDS banks.
struct LaneMap {
  int wave, lane;
  __device__ __forceinline__ int a_row(int i) const { return (wave >> 2) * 128 + (wave & 3) * 16 + 8 * i + (lane >> 3); }
  __device__ __forceinline__ int b_row(int i) const { return (wave >> 1) * 64 + (wave & 1) * 16 + 8 * i + (lane >> 3); }
  __device__ __forceinline__ int k_unit(int i) const { return (lane & 7) ^ (4 * i + (lane >> 4)); }
  // staged column 64 wn + 16 j + t <-> operand row 64 j + 16 wn + t
  __device__ static __forceinline__ int b_col(int c) { return ((c >> 4) & 3) * 64 + (c >> 6) * 16 + (c & 15); }
};

// ap / bp: this lane's global addresses, in slab 0, of loads A0.0, A0.1, A1.0, A1.1 and B0.0, B0.1, B1.0, B1.1.
// Every wave of the workgroup calls this with the same n_slabs >= 1; on return all waves' fragment reads are done
// and nothing of this call is in flight.
__device__ __forceinline__ void tile_mainloop(f32x4 (&acc)[8][4], uint16_t *lds, int wave, int lane, int n_slabs,
                                              const uint16_t *(&ap)[4], const uint16_t *(&bp)[4]) {
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)lds;
  const int wm = wave >> 2, wn = wave & 3;
  Slab r;
  r.wA = __builtin_amdgcn_readfirstlane(lds_base + (unsigned)(wm * 128 + (wave & 3) * 16) * FROWB);
  r.wB = __builtin_amdgcn_readfirstlane(lds_base + FOP_B + (unsigned)((wave >> 1) * 64 + (wave & 1) * 16) * FROWB);
  const int fl = (lane & 15) * FROWB + (((lane >> 4) ^ (lane >> 1)) & 3) * 16 + (lane & 8) * 8;
  r.ldsb = reinterpret_cast<const unsigned char *>(lds);
  r.fA = wm * 128 * FROWB + fl;
  r.fB = FOP_B + wn * 64 * FROWB + fl;
  __syncthreads();                           // the previous user of the stages (an epilogue's staging area) is done
  request(r.wB, bp[0], bp[1]);
  request(r.wA, ap[0], ap[1]);
  request(r.wB + 32 * FROWB, bp[2], bp[3]);
  request(r.wA + 64 * FROWB, ap[2], ap[3]);
  if (n_slabs > 1) {
    request(r.wB + FSTAGE_B, bp[0], bp[1]);
    request(r.wA + FSTAGE_B, ap[0], ap[1]);
    request(r.wB + FSTAGE_B + 32 * FROWB, bp[2], bp[3]);
    end_of_reads<8>();                       // all of slab 0 but A1 has landed
  } else {
    end_of_reads<2>();
  }
  if (wm) __builtin_amdgcn_s_barrier();      // group 1 runs half a phase behind group 0
  int s = 0;
  for (; s + 2 < n_slabs; ++s) slab_step<true, true, 8, 8>(acc, r, ap, bp, s & 1);
  if (n_slabs > 1) slab_step<true, false, 8, 2>(acc, r, ap, bp, s++ & 1);
  slab_step<false, false, 0, 0>(acc, r, ap, bp, s & 1);
  if (!wm) __builtin_amdgcn_s_barrier();
}

// ---- work distribution of the row pass
// The 256 x 256 output tiles form an (m_blocks x n_tiles) grid; it is cut into patches of pr row blocks x
// pc column tiles: PR patch rows of QC patches ("patch steps").  The launch has G groups of kCells
// workgroups; workgroup (dr, dc) of a group computes tile (row block P pr + dr, column tile Q pc + dc) of
// every step (P, Q) its group owns, one after the other.  A group owns
//   - base = PR / G whole patch rows (group x: rows x base .. (x+1) base - 1), swept left to right, and
//   - an equal share of the steps of the remaining PR % G patch rows (row-major, contiguous).
// Consecutive steps of a patch row keep the row block, so a workgroup's 256 rows carry their statistics in
// registers from tile to tile and write one partial result per (row, group, dc) when a patch row (or the
// group's share of it) ends.
//   - Workgroup i of a launch runs on XCD i % 8, so with G = 8 a group is the 32 compute units of one XCD:
//     at any time its L2 serves pr row-operand streams and pc column-operand streams to pr * pc workgroups.
//   - While the groups sweep their whole patch rows they all sit at about the same column position, so a
//     column-operand tile is fetched from HBM by the first group and from the memory-side cache by the others.
//   - Every group gets the same number of steps to within one, whatever the shape: no tail of idle
//     compute units, and nothing depends on the row count being known on the host (a launch over a
//     device-side row list reads its count here).
//   - The patch follows the numbers of row blocks and column tiles: the shape pr x (32 / pr) that covers them in the
//     fewest steps of a group, the tallest among equals.  With a fixed 8 x 4 patch one row block kept an eighth of the
//     chip busy and two a quarter (456 rows x 8192 x 128 256: 2.37 ms, now 0.8 to 1.1; 1024 rows: 2.28 ms, now 1.6),
//     and 57 row blocks left seven eighths of the eighth patch row empty (24.0 ms with pr = 8, 23.1 with 4).  A step
//     takes about the same time with pr = 2, 4 and 8 (64 row blocks: 24.3, 24.3, 24.4 ms), so a lower patch has to
//     save 2.5 %; with pr = 1 nobody shares a column tile, which costs a tenth, in the passes that write a quarter.
//     Many row blocks waste little either way and stay at pr >= 4, which bounds the partial results.
constexpr int kCells = 32;        // workgroups of a group
constexpr int kFewBlocks = 16;    // up to here any height is considered
__host__ __device__ inline void patch_shape(int64_t m_blocks, int64_t n_tiles, int groups, int &pr, int &pc) {
  const int64_t mb = m_blocks < 1 ? 1 : m_blocks;
  int64_t best = 0;
  for (int h = 8; h >= (mb <= kFewBlocks ? 1 : 4); --h) {
    if (h > mb) continue;
    const int w = kCells / h;
    const int64_t steps = (((mb + h - 1) / h) * ((n_tiles + w - 1) / w) + groups - 1) / groups;
    const int64_t cost = steps * ((h == 1 && mb > 1) ? 50 : h <= 4 ? 41 : 40);
    if (best == 0 || cost < best) { best = cost; pr = h; pc = w; }
  }
}
struct RowSched {
  int m_blocks, n_tiles, PR, QC, pr, pc, G;
  int base;         // whole patch rows per group
  int64_t Tr;       // steps of the remaining patch rows, shared out evenly
};
// pr == 0: the patch shape is the library's choice
__device__ __forceinline__ RowSched make_sched(int64_t M, int n_tiles, int G, int pr, int pc) {
  RowSched s;
  s.m_blocks = (int)((M + FBM - 1) / FBM);
  if (pr == 0) patch_shape(s.m_blocks, n_tiles, G, pr, pc);
  s.n_tiles = n_tiles;
  s.pr = pr; s.pc = pc; s.G = G;
  s.PR = (s.m_blocks + pr - 1) / pr;
  s.QC = (n_tiles + pc - 1) / pc;
  s.base = s.PR / G;
  s.Tr = (int64_t)(s.PR - s.base * G) * s.QC;
  return s;
}
__device__ __forceinline__ int64_t rest_begin(const RowSched &s, int x) {
  if (s.Tr < (1 << 26)) return (uint32_t)s.Tr * (uint32_t)x / (uint32_t)s.G;     // x <= G <= 16: the usual sizes in 32 bits
  return s.Tr * x / s.G;
}
// number of steps of group x, and its i-th step as (patch row, patch column)
__device__ __forceinline__ int64_t group_steps(const RowSched &s, int x) {
  return (int64_t)s.base * s.QC + (rest_begin(s, x + 1) - rest_begin(s, x));
}
__device__ __forceinline__ void group_step(const RowSched &s, int x, int64_t i, int &P, int &Q) {
  const int64_t n1 = (int64_t)s.base * s.QC;
  if (i < n1) {
    P = x * s.base + (int)(i / s.QC);
    Q = (int)(i % s.QC);
  } else {
    const int64_t r = rest_begin(s, x) + (i - n1);
    P = s.base * s.G + (int)(r / s.QC);
    Q = (int)(r % s.QC);
  }
}
// does partial slot (group x, column phase dc) of row block `mblock` hold a result?
__device__ __forceinline__ bool slot_valid(const RowSched &s, int mblock, int slot) {
  const int x = slot / s.pc, dc = slot - x * s.pc;
  if (x >= s.G) return false;
  const int P = mblock / s.pr;
  if (P < s.base * s.G) return x == P / s.base && dc < s.n_tiles;
  const int64_t row_lo = (int64_t)(P - s.base * s.G) * s.QC;
  const int64_t lo = max(rest_begin(s, x), row_lo), hi = min(rest_begin(s, x + 1), row_lo + s.QC);
  if (lo >= hi) return false;
  return (int)(lo - row_lo) * s.pc + dc < s.n_tiles;   // the first tile of the segment exists (later ones lie further right)
}

enum FusedMode { kFusedStats = 0, kFusedBwd = 1, kFusedPlanes = 2, kFusedStore = 3 };

constexpr float kNoRef = -3.402823466e+38f;         // reference of an empty sum: below every real one

// exponent reference of a chunk: the maximum's, rounded to an integer, so that partial sums with different
// references combine by exact powers of two
__device__ __forceinline__ float chunk_ref(float cm) { return (cm == neg_inf()) ? 0.f : __builtin_rintf(cm * kLog2e); }

// s (reference c) += p (reference pc); c becomes the larger one.  The references are integers: no rounding but
// that of the fp64 add, so the result does not depend on how a row's chunks are grouped or ordered.
__device__ __forceinline__ void add_sum(double &s, float &c, double p, float pc) {
  const float cn = fmaxf(c, pc);
  s = scale_pow2(s, c - cn) + scale_pow2(p, pc - cn);
  c = cn;
}

template <int KT, int MODE>
__global__ __launch_bounds__(FTHREADS, 2) void k_fused_rows(FusedArgs a) {
  extern __shared__ __align__(1024) uint16_t lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int trow = tid & 255, half = tid >> 8;        // statistics: this thread's row, and which half of the columns

  const int64_t M = a.m_dev ? min((int64_t)*a.m_dev, a.M) : a.M;   // row count may live on the device
  const RowSched sc = make_sched(M, a.n_tiles, a.groups, a.patch_rows, a.patch_cols);
  const int grp = blockIdx.x % sc.G, cell = blockIdx.x / sc.G;       // workgroup (dr, dc) of group grp
  if (cell >= sc.pr * sc.pc) return;
  const int dr = cell / sc.pc, dc = cell - dr * sc.pc;
  const int slot = grp * sc.pc + dc;                                  // partial-result slot of a row
  const int n_slots = sc.G * sc.pc;
  const int64_t n_steps = group_steps(sc, grp);
  const int HD = a.hidden_dim;
  const uint16_t *__restrict__ Hp = static_cast<const uint16_t *>(a.hidden);
  const uint16_t *__restrict__ Wp = static_cast<const uint16_t *>(a.w);

  const LaneMap lm{wave, lane};
  // the list keeps the KT >= ktop best of the row; its last entry is the insertion threshold
  RowState<KT> st;
  const int ktop = a.ktop;
  // Writing modes (backward, planes, store): a wave writes the rows 32 wave .. 32 wave + 31 of the tile, eight
  // at a time; lane l then holds four consecutive columns (4 (l % 8) ..) of row 8 it + l / 8, so that the eight
  // lanes of a row write 128 contiguous bytes of an fp32 row (64 of a bf16 plane) per store instruction.  A
  // lane therefore keeps the parameters of its four rows (it = 0..3) for the whole patch row.
  constexpr bool kWrites = (MODE != kFusedStats);
  constexpr int NR = kWrites ? 4 : 1;
  float e_lse[NR], e_coef[NR];
  int e_tok[NR];
  int64_t e_base[NR];        // element offset of the row in the output (gradient rows / planes / stored rows); -1: no row
  double e_others[NR];       // backward and planes: sum of the probabilities of all tokens but the accepted one
#pragma unroll
  for (int it = 0; it < NR; ++it) { e_lse[it] = 0.f; e_coef[it] = 0.f; e_tok[it] = -1; e_base[it] = -1; e_others[it] = 0.0; }
  const uint16_t *a_ptr[4] = {nullptr, nullptr, nullptr, nullptr};
  int64_t row0 = 0;
  int cur_P = -1;
  bool rows_live = false;      // this workgroup's row block of the current patch row exists

  // partial results of the row-block segment that ends (patch row finished, or the group's range did)
  auto flush = [&]() {
    if constexpr (MODE == kFusedStore) {
      return;
    } else if constexpr (kWrites) {
      // the eight lanes of a row add up their column groups (fixed order), lane 0 of the eight writes
#pragma unroll
      for (int it = 0; it < NR; ++it) {
        double v = e_others[it];
        v += __shfl_xor(v, 1, kWave);
        v += __shfl_xor(v, 2, kWave);
        v += __shfl_xor(v, 4, kWave);
        const int64_t g = row0 + wave * 32 + 8 * it + (lane >> 3);
        if ((lane & 7) == 0 && g < M) a.part_s[g * n_slots + slot] = v;
      }
    } else {
      // the two threads of a row: the second hands its state over, the first merges and writes
      double *x_s = reinterpret_cast<double *>(lds);
      float *x_m = reinterpret_cast<float *>(x_s + FBM), *x_c = x_m + FBM, *x_v = x_c + FBM;
      int *x_i = reinterpret_cast<int *>(x_v + KT * FBM);
      __syncthreads();
      if (half) {
        x_s[trow] = st.s;
        x_m[trow] = st.m;
        x_c[trow] = st.c;
#pragma unroll
        for (int i = 0; i < KT; ++i) {
          x_v[i * FBM + trow] = st.v[i];
          x_i[i * FBM + trow] = st.id[i];
        }
      }
      __syncthreads();
      if (!half) {
        st.m = fmaxf(st.m, x_m[trow]);
        add_sum(st.s, st.c, x_s[trow], x_c[trow]);
#pragma unroll 1
        for (int i = 0; i < KT; ++i) {
          const float xv = x_v[i * FBM + trow];
          const int xi = x_i[i * FBM + trow];
          if (better(xv, xi, st.v[KT - 1], st.id[KT - 1])) list_insert<KT>(st.v, st.id, xv, xi);
        }
        const int64_t g = row0 + trow;
        if (g < M) {
          const int64_t pi = g * n_slots + slot;
          a.part_m[pi] = st.m;
          a.part_c[pi] = st.c;
          a.part_s[pi] = st.s;
#pragma unroll
          for (int i = 0; i < KT; ++i) {
            if (i < ktop) {
              a.part_v[pi * ktop + i] = st.v[i];
              a.part_i[pi * ktop + i] = st.id[i];
            }
          }
        }
      }
    }
  };

  for (int64_t step = 0; step < n_steps; ++step) {
    int P, Q;
    group_step(sc, grp, step, P, Q);
    if (P != cur_P) {
      if (rows_live) flush();
      cur_P = P;
      const int mblock = P * sc.pr + dr;
      rows_live = mblock < sc.m_blocks;
      row0 = (int64_t)mblock * FBM;
      st.m = neg_inf(); st.c = kNoRef; st.s = 0.0;
#pragma unroll
      for (int i = 0; i < KT; ++i) { st.v[i] = neg_inf(); st.id[i] = kNoId; }
#pragma unroll
      for (int it = 0; it < NR; ++it) { e_base[it] = -1; e_others[it] = 0.0; e_tok[it] = -1; }
      if (rows_live) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int64_t g = row0 + lm.a_row(j & 1) + 64 * (j >> 1);
          if (g >= M) g = M - 1;
          const int64_t hs = a.row_list ? (int64_t)a.row_list[g] : used_slot_index(g, a.rho, a.d, a.kslots);
          a_ptr[j] = Hp + hs * HD + lm.k_unit(j & 1) * 8;
        }
        if constexpr (kWrites) {
#pragma unroll
          for (int it = 0; it < NR; ++it) {
            const int64_t gme = row0 + wave * 32 + 8 * it + (lane >> 3);
            if (gme < M) {
              if constexpr (MODE == kFusedStore) {
                e_base[it] = gme * a.store_pitch;
              } else {
                const int pidx = a.list_p[gme];
                const int rr = pidx / a.d;
                e_lse[it] = a.lse_by_slot[a.row_list[gme]];
                e_coef[it] = a.coef[rr];
                e_tok[it] = a.sel_tok[(int64_t)rr * a.g + a.path_node[pidx]];
                e_base[it] = (MODE == kFusedBwd) ? (int64_t)pidx * a.V : gme * a.plane_pitch;
              }
            }
          }
        }
      }
    }
    const int tile = Q * sc.pc + dc;
    if (!rows_live || tile >= sc.n_tiles) continue;     // uniform over the workgroup
    const int n0 = tile * FBN;
    f32x4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
      const uint16_t *ap[4], *bp[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ap[j] = a_ptr[j];
        int n = n0 + LaneMap::b_col(lm.b_row(j & 1) + 32 * (j >> 1));
        if (n >= a.V) n = a.V - 1;
        bp[j] = Wp + (int64_t)n * HD + lm.k_unit(j & 1) * 8;
      }
      tile_mainloop(acc, lds, wave, lane, HD / FBK, ap, bp);
    }
    __syncthreads();                           // all fragment reads done before the staging area is written

    float *stg = reinterpret_cast<float *>(lds);
    if constexpr (MODE == kFusedStats) {
      // ---- epilogue of the statistics pass: threads t and t + 256 own row t.  Four phases; phase nt takes
      // column tile nt of every wave (64 consecutive columns) through a column-major staging area: the four
      // consecutive rows a lane holds of a column leave as one 16-byte write (8 per wave and phase,
      // conflict-free with the column stride FSTG_CM), and a thread then reads half of its row with one 4-byte
      // read per column, all 32 issued back to back.
      const bool full_tile = (n0 + FBN <= a.V);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        {
          float *wcol = stg + (wn * 16 + (lane & 15)) * FSTG_CM + wm * 128 + 4 * (lane >> 4);
#pragma unroll
          for (int mt = 0; mt < 8; ++mt) *reinterpret_cast<f32x4 *>(wcol + mt * 16) = acc[mt][nt];
        }
        __syncthreads();
        const int cid0 = n0 + nt * 64 + half * 32;     // vocabulary entry of this thread's first column
        const float *src = stg + (half * 32) * FSTG_CM + trow;
        float x[32];
#pragma unroll
        for (int c = 0; c < 32; ++c) x[c] = src[c * FSTG_CM];
        if (!full_tile) {
#pragma unroll
          for (int c = 0; c < 32; ++c)
            if (cid0 + c >= a.V) x[c] = neg_inf();     // adds nothing to max and sum
        }
        // The 32 logits' maximum, then their sum of exp2 against a reference of their own: an integer, so that
        // it joins the row's sum by an exact power of two and the result is the same for every launch geometry.
        float cm = x[0];
#pragma unroll
        for (int c = 1; c < 32; ++c) cm = fmaxf(cm, x[c]);
        const float c_ref = chunk_ref(cm);
        float p = 0.f;
#pragma unroll
        for (int c = 0; c < 32; ++c) p += __builtin_amdgcn_exp2f(__builtin_fmaf(x[c], kLog2e, -c_ref));
        // top-k insertions.  Some row of the workgroup reaches its threshold in almost every phase, and
        // the other waves wait for that wave at the barrier, so the search for the candidates must not walk
        // the columns one by one: a row first marks, from registers, the columns that reach the threshold
        // it had on entry (later thresholds are higher), then visits only those (typically one or two).
        if (cm >= st.v[KT - 1]) {
          const float thr = st.v[KT - 1];
          uint32_t mask = 0;
#pragma unroll
          for (int c = 0; c < 32; ++c) mask |= (x[c] >= thr) ? (1u << c) : 0u;
          if (!full_tile) {      // masked columns hold -inf, which reaches the threshold of a list that is not full yet
            const int left = a.V - cid0;                      // valid columns from cid0 on
            mask &= (left >= 32) ? ~0u : (left <= 0 ? 0u : (1u << left) - 1u);
          }
          while (mask != 0u) {
            const int c = __builtin_ctz(mask);
            mask &= mask - 1u;
            const float xv = src[c * FSTG_CM];
            if (better(xv, cid0 + c, st.v[KT - 1], st.id[KT - 1])) list_insert<KT>(st.v, st.id, xv, cid0 + c);
          }
        }
        if (cm != neg_inf()) add_sum(st.s, st.c, (double)p, c_ref);
        st.m = fmaxf(st.m, cm);
        __syncthreads();
      }
    } else {
      // ---- epilogue of the writing modes: the same four phases and the same column-major staging; then
      // every wave walks its 32 rows eight at a time (see the lane mapping above), two pieces of 32 columns each
      const bool vec4 = ((a.V & 3) == 0) && (MODE != kFusedStore || (a.store_pitch & 3) == 0);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        {
          float *wcol = stg + (wn * 16 + (lane & 15)) * FSTG_CM + wm * 128 + 4 * (lane >> 4);
#pragma unroll
          for (int mt = 0; mt < 8; ++mt) *reinterpret_cast<f32x4 *>(wcol + mt * 16) = acc[mt][nt];
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < NR; ++it) {
          const float *src = stg + wave * 32 + 8 * it + (lane >> 3);
#pragma unroll
          for (int piece = 0; piece < 2; ++piece) {
            const int c0 = piece * 32 + 4 * (lane & 7);                       // staged column of this lane's first element
            const int col = n0 + nt * 64 + c0;                                // its vocabulary entry
            if (e_base[it] < 0 || col >= (MODE == kFusedPlanes ? a.plane_pitch : a.V)) continue;
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = src[(c0 + e) * FSTG_CM];
            const bool whole = vec4 && (col + 3 < a.V);
            if constexpr (MODE == kFusedStore) {
              float *o = a.store_rows + e_base[it] + col;
              if (whole) {
                const f32x4 q = {x[0], x[1], x[2], x[3]};
                *reinterpret_cast<f32x4 *>(o) = q;
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (col + e < a.V) o[e] = x[e];
              }
            } else {
              // -coef * softmax; the accepted token's probability is left out of the sum (and, in the planes, out
              // of the entry) so that its coefficient coef * (1 - p_token) can be formed without cancellation
              float gq[4], part = 0.f;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const bool is_tok = (col + e == e_tok[it]);
                float pv = (col + e < a.V) ? __builtin_amdgcn_exp2f((x[e] - e_lse[it]) * kLog2e) : 0.f;
                if (MODE == kFusedPlanes && is_tok) pv = 0.f;
                part += is_tok ? 0.f : pv;
                gq[e] = -e_coef[it] * pv;
              }
              e_others[it] += (double)part;
              if constexpr (MODE == kFusedBwd) {
                float *o = a.grad_rows + e_base[it] + col;
                if (whole) {
                  const f32x4 q = {gq[0], gq[1], gq[2], gq[3]};
                  __builtin_nontemporal_store(q, reinterpret_cast<f32x4 *>(o));
                } else {
#pragma unroll
                  for (int e = 0; e < 4; ++e)
                    if (col + e < a.V) o[e] = gq[e];
                }
              } else {
                // planes: value = hi + lo in bf16 (V is a multiple of 32 and the pitch of 64: whole 8-byte stores, zeros
                // in the padding)
                uint16_t hq[4], lq[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const __bf16 hb = (__bf16)gq[e];
                  const __bf16 lb = (__bf16)(gq[e] - (float)hb);
                  hq[e] = __builtin_bit_cast(uint16_t, hb);
                  lq[e] = __builtin_bit_cast(uint16_t, lb);
                }
                const u32x2 ho = {(uint32_t)hq[0] | ((uint32_t)hq[1] << 16), (uint32_t)hq[2] | ((uint32_t)hq[3] << 16)};
                const u32x2 lo = {(uint32_t)lq[0] | ((uint32_t)lq[1] << 16), (uint32_t)lq[2] | ((uint32_t)lq[3] << 16)};
                *reinterpret_cast<u32x2 *>(a.plane_hi + e_base[it] + col) = ho;
                *reinterpret_cast<u32x2 *>(a.plane_lo + e_base[it] + col) = lo;
              }
            }
          }
        }
        __syncthreads();
      }
    }
  }

  if (rows_live) flush();
}

// One wave per row: merge the partial results of the row's segments into the final statistics (a lane takes
// every 64th slot).  Which slots hold a result follows from the launch geometry alone (slot_valid).
// The k best of the slots' lists come out in k rounds of a wave-wide maximum over candidates kept in registers
// (entries beyond kMergeReg * 64 are read again in every round): a few row blocks leave up to 512 slots a row, and
// ranking every candidate against every other one takes (512 k)^2 steps.
constexpr int kMergeReg = 16;
__global__ __launch_bounds__(64) void k_fused_merge(FusedArgs a) {
  const int64_t g = blockIdx.x;
  const int64_t M = a.m_dev ? min((int64_t)*a.m_dev, a.M) : a.M;
  if (g >= M) return;
  const int lane = threadIdx.x;
  const int ktop = a.ktop;
  const RowSched sc = make_sched(M, a.n_tiles, a.groups, a.patch_rows, a.patch_cols);
  const int n_slots = sc.G * sc.pc;
  const int mblock = (int)(g / FBM);
  const int64_t oi = a.row_list ? (a.out_by_list ? g : (int64_t)a.row_list[g])
                                : used_slot_index(g, a.rho, a.d, a.kslots);
  __shared__ int16_t s_slot[16 * kCells];
  int n_valid = 0;
  float m = neg_inf(), c = kNoRef;
  double s = 0.0;
  for (int q0 = 0; q0 < n_slots; q0 += 64) {
    const int q = q0 + lane;
    const bool ok = q < n_slots && slot_valid(sc, mblock, q);
    const uint64_t mask = __builtin_amdgcn_ballot_w64(ok);
    if (ok) s_slot[n_valid + lanes_below(mask)] = (int16_t)q;
    n_valid += __builtin_popcountll(mask);
    if (!ok) continue;
    const float pm = a.part_m[g * n_slots + q];
    if (pm == neg_inf()) continue;
    m = fmaxf(m, pm);
    add_sum(s, c, a.part_s[g * n_slots + q], a.part_c[g * n_slots + q]);
  }
  const float Mx = wave_max_dpp(m);
  const float C = wave_max_dpp(c);
  const double S = wave_sum_dpp(scale_pow2(s, c - C));
  const double lse = (double)Mx + kLn2 * (((double)C - (double)Mx * (double)kLog2e) + log2(S));
  if (lane == 0) {
    if (a.row_max) a.row_max[oi] = Mx;
    a.row_lse[oi] = (float)lse;
  }
  if (a.top_tok == nullptr) return;
  const float *pv = a.part_v + g * n_slots * ktop;
  const int32_t *pi = a.part_i + g * n_slots * ktop;
  const int total = n_valid * ktop;
  __builtin_amdgcn_wave_barrier();
  auto fetch = [&](int j, float &v, int &id) {
    const int q = min(j, total - 1) / ktop;
    const int at = s_slot[q] * ktop + (min(j, total - 1) - q * ktop);
    v = (j < total) ? pv[at] : neg_inf();
    id = (j < total) ? pi[at] : kNoId;
  };
  float cv[kMergeReg];
  int ci[kMergeReg];
#pragma unroll
  for (int u = 0; u < kMergeReg; ++u) {
    cv[u] = neg_inf();
    ci[u] = kNoId;
    if (u * 64 < total) fetch(u * 64 + lane, cv[u], ci[u]);
  }
  float last_v = __builtin_inff(), my_v = neg_inf();
  int last_i = -1, my_i = kNoId;
  for (int r = 0; r < ktop; ++r) {
    float bv = neg_inf();
    int bi = kNoId;
#pragma unroll
    for (int u = 0; u < kMergeReg; ++u) {
      if (u * 64 < total && better(cv[u], ci[u], bv, bi)) { bv = cv[u]; bi = ci[u]; }
    }
    for (int j = kMergeReg * 64 + lane; j < total; j += 64) {
      float v;
      int id;
      fetch(j, v, id);
      if (better(last_v, last_i, v, id) && better(v, id, bv, bi)) { bv = v; bi = id; }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const float ov = __shfl_xor(bv, off, kWave);
      const int oid = __shfl_xor(bi, off, kWave);
      if (better(ov, oid, bv, bi)) { bv = ov; bi = oid; }
    }
#pragma unroll
    for (int u = 0; u < kMergeReg; ++u)
      if (ci[u] == bi) { cv[u] = neg_inf(); ci[u] = kNoId; }
    last_v = bv;
    last_i = bi;
    if (lane == r) { my_v = bv; my_i = bi; }
  }
  if (lane < ktop) {
    // ranks no entry claimed (possible only when the row held NaNs): a valid token id with probability zero
    const bool ok = my_i != kNoId;
    a.top_tok[oi * ktop + lane] = ok ? my_i : lane;
    if (a.top_logp) a.top_logp[oi * ktop + lane] = ok ? fminf((float)((double)my_v - lse), 0.f) : neg_inf();
    if (a.top_logit) a.top_logit[oi * ktop + lane] = ok ? my_v : neg_inf();
  }
}

// sum, over the valid slots of row g, of the per-segment sums of the non-token probabilities; the same in every
// lane of the (whole, converged) wave that calls it
__device__ __forceinline__ double sum_others(const double *part_s, int64_t g, const RowSched &sc) {
  const int n_slots = sc.G * sc.pc;
  double tot = 0.0;
  for (int c = lane_id(); c < n_slots; c += 64)
    if (slot_valid(sc, (int)(g / FBM), c)) tot += part_s[g * n_slots + c];
  return wave_sum_dpp(tot);
}

// Backward fix-up, one wave per processed row: the accepted token's entry is coef times the sum
// of all other probabilities (summed in a fixed order).
__global__ __launch_bounds__(64) void k_fused_bwd_fixup(FusedArgs a) {
  const int64_t g = blockIdx.x;
  const int64_t M = a.m_dev ? min((int64_t)*a.m_dev, a.M) : a.M;
  if (g >= M) return;
  const double tot = sum_others(a.part_s, g, make_sched(M, a.n_tiles, a.groups, a.patch_rows, a.patch_cols));
  const int pidx = a.list_p[g];
  const int rr = pidx / a.d;
  const int tok = a.sel_tok[(int64_t)rr * a.g + a.path_node[pidx]];
  if (threadIdx.x == 0 && tok >= 0 && tok < a.V)
    a.grad_rows[(int64_t)pidx * a.V + tok] = (float)((double)a.coef[rr] * tot);
}

// Ordered compaction by a single workgroup of 1024: wave w takes the w-th part of the entries, counts them, learns its
// place from the other waves' counts and writes; valid(p), emit(p, position); returns the total in every thread.
// (65 536 flags with a scan over the workgroup per 1024 entries: 62 us.)
// kU: entries per lane and trip, independent loads.
template <int kU, typename Valid, typename Emit>
__device__ __forceinline__ int compact_ordered(int n, Valid valid, Emit emit) {
  __shared__ int s_wave[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int part = ((n + 1023) / 1024) * 64;
  const int p0 = min(wave * part, n), p1 = min(p0 + part, n);
  auto trip = [&](int p, uint64_t (&mask)[kU]) {
    bool v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = valid(min(p + u * 64 + lane, n - 1));
#pragma unroll
    for (int u = 0; u < kU; ++u) mask[u] = __builtin_amdgcn_ballot_w64(v[u] && p + u * 64 + lane < p1);
  };
  int cnt = 0;
  uint64_t mask[kU];
  for (int p = p0; p < p1; p += kU * 64) {
    trip(p, mask);
#pragma unroll
    for (int u = 0; u < kU; ++u) cnt += __builtin_popcountll(mask[u]);
  }
  if (lane == 0) s_wave[wave] = cnt;
  __syncthreads();
  int at = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    at += (w < wave) ? s_wave[w] : 0;
    total += s_wave[w];
  }
  for (int p = p0; p < p1; p += kU * 64) {
    if (p1 - p0 > kU * 64) trip(p, mask);    // (a single trip's masks are still there)
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if ((mask[u] >> lane) & 1ull) emit(p + u * 64 + lane, at + lanes_below(mask[u]));
      at += __builtin_popcountll(mask[u]);
    }
  }
  return total;
}

// The (root, step) pairs that carry a gradient, their hidden-row slots, and grad_slot for every pair.
__global__ __launch_bounds__(1024) void k_bwd_rows(BwdRowsArgs a) {
  const int total = compact_ordered<4>(
      a.R * a.d,
      [&](int p) {
        const int j = (a.coef[p / a.d] != 0.f) ? max(a.path_slot[p], -1) : -1;
        a.grad_slot[p] = j;                  // (by every trip that looks: the same value)
        return j >= 0;
      },
      [&](int p, int at) {
        const int r = p / a.d, t = p - r * a.d;
        a.list_p[at] = p;
        a.list_slot[at] = (int)stat_index(r, t, a.path_slot[p], a.d, a.k);
      });
  if (threadIdx.x == 0) *a.count = total;
}

// The slots whose flag is set: list of slot indices + count.
__global__ __launch_bounds__(1024) void k_compact_flags(const int32_t *flags, int n, int32_t *list, int32_t *count) {
  const int total = compact_ordered<16>(n, [&](int p) { return flags[p] != 0; }, [&](int p, int at) { list[at] = p; });
  if (threadIdx.x == 0) *count = total;
}

void launch_compact_flags(const int32_t *flags, int n, int32_t *list, int32_t *count, hipStream_t st) {
  hipLaunchKernelGGL(k_compact_flags, dim3(1), dim3(1024), 0, st, flags, n, list, count);
}

__global__ void k_zero_rows(float *grad_rows, const int32_t *grad_slot, int V) {
  if (grad_slot[blockIdx.x] >= 0) return;
  float *o = grad_rows + (int64_t)blockIdx.x * V;
  for (int i = threadIdx.x; i < V; i += blockDim.x) o[i] = 0.f;
}

// One wave per (row slot, token): fp32 dot product of a hidden row and a W row.
__global__ __launch_bounds__(64) void k_gather_dot(GatherDotArgs a) {
  const int64_t p = blockIdx.x;
  const int lane = threadIdx.x;
  const int64_t slot = a.slot[p];
  const int tok = a.tok[p];
  if (slot < 0 || tok < 0 || tok >= a.V) {
    if (lane == 0) a.out[p] = 0.f;
    return;
  }
  const uint16_t *h = static_cast<const uint16_t *>(a.hidden) + slot * a.hidden_dim;
  const uint16_t *w = static_cast<const uint16_t *>(a.w) + (int64_t)tok * a.hidden_dim;
  float acc = 0.f;
  for (int e0 = lane * 8; e0 < a.hidden_dim; e0 += 64 * 8) {
    const u32x4 hq = *reinterpret_cast<const u32x4 *>(h + e0);
    const u32x4 wq = *reinterpret_cast<const u32x4 *>(w + e0);
    float hx[8], wx[8];
    Elem<uint16_t>::unpack(hq, hx);
    Elem<uint16_t>::unpack(wq, wx);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = __builtin_fmaf(hx[e], wx[e], acc);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (lane == 0) a.out[p] = acc;
}

// Hidden-state gradient, one 256 (rows of the list) x 256 (hidden columns) tile per workgroup and split of
// the contraction: partial[split] = sum over the split's k slabs of G . W, G = [plane_hi | plane_lo]
// (contraction length 2 V), W hidden-major so that both operands are contiguous along the vocabulary.
__global__ __launch_bounds__(FTHREADS, 2) void k_fused_dh(FusedDhArgs a) {
  extern __shared__ __align__(1024) uint16_t lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  // Workgroup i runs on XCD i % 8: with eight splits an XCD keeps to one k range, and the row blocks of a column block
  // run next to each other, so that its L2 serves a head tile to all of them (910 rows x 8192: 3.17 ms with the
  // column blocks next to each other, now 2.75).
  const int64_t M = min((int64_t)*a.m_dev, a.M);
  const int m_blocks = (int)((M + FBM - 1) / FBM);
  const int split = blockIdx.x % a.n_splits;
  const int rest = blockIdx.x / a.n_splits;
  if (rest >= m_blocks * a.h_blocks) return;
  const int mblock = rest % m_blocks, hblock = rest / m_blocks;
  const int64_t row0 = (int64_t)mblock * FBM;
  const int nks = (int)(a.plane_pitch / FBK);                 // slabs per plane (the last one may be half padding)
  const int s0 = split * a.slabs_per_split;
  const int s1 = min(s0 + a.slabs_per_split, 2 * nks);
  const int h0 = hblock * FBN;
  const LaneMap lm{wave, lane};
  int64_t a_off[4];
  const uint16_t *b_ptr[4];
  const uint16_t *Wp = static_cast<const uint16_t *>(a.w_hv);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int64_t g = row0 + lm.a_row(j & 1) + 64 * (j >> 1);
    if (g >= M) g = M - 1;
    a_off[j] = g * a.plane_pitch + lm.k_unit(j & 1) * 8;
    int n = h0 + LaneMap::b_col(lm.b_row(j & 1) + 32 * (j >> 1));
    if (n >= a.hidden_dim) n = a.hidden_dim - 1;
    b_ptr[j] = Wp + (int64_t)n * a.V + lm.k_unit(j & 1) * 8;
  }
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // The split's slabs [s0, s1) of the contraction over [hi plane | lo plane], in up to four contiguous k ranges of
  // both operands: whole slabs of the hi plane, its last slab if that is half padding, and the same of the lo
  // plane.  In a half slab the head's rows end in the middle: the lanes beyond fetch the slab's first half again,
  // which the planes' zeros take out of the sum.
  const int whole = a.V / FBK;
#pragma unroll 1
  for (int part = 0; part < 4; ++part) {
    const int base = (part >> 1) * nks;
    const bool tail = part & 1;
    const int lo = max(s0, base + (tail ? whole : 0)), hi = min(s1, base + (tail ? nks : whole));
    if (lo >= hi) continue;
    const uint16_t *plane = (part >> 1) ? a.plane_lo : a.plane_hi;
    const int64_t k0 = (int64_t)(lo - base) * FBK;
    const uint16_t *ap[4], *bp[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      ap[j] = plane + a_off[j] + k0;
      bp[j] = b_ptr[j] + k0 - ((tail && lm.k_unit(j & 1) >= 4) ? FBK / 2 : 0);
    }
    tile_mainloop(acc, lds, wave, lane, hi - lo, ap, bp);
  }
  float *out = a.partial + (int64_t)split * a.M * a.hidden_dim;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t row = row0 + wm * 128 + i * 16 + 4 * (lane >> 4) + e;
        const int col = h0 + j * 64 + wn * 16 + (lane & 15);
        if (row < M && col < a.hidden_dim) out[row * a.hidden_dim + col] = acc[i][j][e];
      }
}

// dH row of list entry g: the splits in a fixed order, plus the accepted token's own term
// coef * (1 - p_token) * W[token, :], with 1 - p_token taken as the sum of the other probabilities.
__global__ __launch_bounds__(256) void k_fused_dh_reduce(FusedDhArgs a) {
  const int64_t g = blockIdx.x;
  if (g >= (int64_t)*a.m_dev) return;
  const int pidx = a.list_p[g];
  const int rr = pidx / a.d;
  const int tok = min(max(a.sel_tok[(int64_t)rr * a.g + a.path_node[pidx]], 0), a.V - 1);
  const float coef = a.coef[rr];
  const uint16_t *wrow = static_cast<const uint16_t *>(a.w_vh) + (int64_t)tok * a.hidden_dim;
  // sum of the probabilities of all tokens but the accepted one, from the plane pass's segments
  const int64_t M = min((int64_t)*a.m_dev, a.M);
  const double others = sum_others(a.part_s, g, make_sched(M, a.n_tiles, a.groups, a.patch_rows, a.patch_cols));
  const float ctok = (float)((double)coef * others);
  // four columns a thread (hidden_dim is a multiple of 64), eight splits at a time
  for (int h = threadIdx.x * 4; h < a.hidden_dim; h += 1024) {
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < a.n_splits; s0 += 8) {
      f32x4 q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        q[u] = *reinterpret_cast<const f32x4 *>(a.partial + ((int64_t)min(s0 + u, a.n_splits - 1) * a.M + g) * a.hidden_dim + h);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < a.n_splits) sum += q[u];
    }
    float *o = a.dh_rows + (int64_t)pidx * a.hidden_dim + h;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(ctok, Elem<uint16_t>::load1(wrow + h + e), sum[e]);
  }
}

template <typename K>
static void set_lds_attr(K kern) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kFusedLdsBytes);
}

int64_t fused_partials(int64_t rows, int n_tiles, int groups, int pr, int pc) {
  if (pr != 0) return rows * groups * pc;
  int64_t most = rows * (kCells / 4);                     // beyond kFewBlocks the patch is at most eight tiles wide
  for (int64_t mb = 1; mb <= kFewBlocks && (mb - 1) * FBM < rows; ++mb) {
    patch_shape(mb, n_tiles, groups, pr, pc);
    most = std::max(most, std::min(rows, mb * FBM) * pc);
  }
  return groups * most;
}

static int fused_grid(const FusedArgs &a) { return a.groups * kCells; }

// the kernels that use the whole slab ring need the dynamic LDS limit raised once per process
// (initialisation of a function-local static is thread-safe)
static void ensure_lds_attrs() {
  static const bool done = [] {
    set_lds_attr(k_fused_rows<1, kFusedStats>);
    set_lds_attr(k_fused_rows<8, kFusedStats>);
    set_lds_attr(k_fused_rows<16, kFusedStats>);
    set_lds_attr(k_fused_rows<1, kFusedBwd>);
    set_lds_attr(k_fused_rows<1, kFusedPlanes>);
    set_lds_attr(k_fused_rows<1, kFusedStore>);
    set_lds_attr(k_fused_dh);
    return true;
  }();
  (void)done;
}

void launch_fused_rows(const FusedArgs &a, hipStream_t st) {
  ensure_lds_attrs();
  const int blocks = fused_grid(a);
  if (a.store_rows != nullptr)
    hipLaunchKernelGGL((k_fused_rows<1, kFusedStore>), dim3(blocks), dim3(FTHREADS), kFusedLdsBytes, st, a);
  else if (a.plane_hi != nullptr)
    hipLaunchKernelGGL((k_fused_rows<1, kFusedPlanes>), dim3(blocks), dim3(FTHREADS), kFusedLdsBytes, st, a);
  else if (a.grad_rows != nullptr)
    hipLaunchKernelGGL((k_fused_rows<1, kFusedBwd>), dim3(blocks), dim3(FTHREADS), kFusedLdsBytes, st, a);
  else if (a.ktop <= 1)
    hipLaunchKernelGGL((k_fused_rows<1, kFusedStats>), dim3(blocks), dim3(FTHREADS), kFusedLdsBytes, st, a);
  else if (a.ktop <= 8)
    hipLaunchKernelGGL((k_fused_rows<8, kFusedStats>), dim3(blocks), dim3(FTHREADS), kFusedLdsBytes, st, a);
  else
    hipLaunchKernelGGL((k_fused_rows<16, kFusedStats>), dim3(blocks), dim3(FTHREADS), kFusedLdsBytes, st, a);
}

void launch_fused_dh(const FusedDhArgs &a, hipStream_t st) {
  ensure_lds_attrs();
  hipLaunchKernelGGL(k_fused_dh, dim3((unsigned)(a.m_blocks * a.h_blocks * a.n_splits)), dim3(FTHREADS), kFusedLdsBytes, st, a);
  hipLaunchKernelGGL(k_fused_dh_reduce, dim3((unsigned)a.M), dim3(256), 0, st, a);
}

void launch_fused_bwd_fixup(const FusedArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(k_fused_bwd_fixup, dim3((unsigned)a.M), dim3(64), 0, st, a);
}

void launch_bwd_rows(const BwdRowsArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(k_bwd_rows, dim3(1), dim3(1024), 0, st, a);
}

void launch_zero_rows(float *grad_rows, const int32_t *grad_slot, int rows, int V, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_rows, dim3(rows), dim3(256), 0, st, grad_rows, grad_slot, V);
}

void launch_fused_merge(const FusedArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(k_fused_merge, dim3((unsigned)a.M), dim3(64), 0, st, a);
}

void launch_gather_dot(const GatherDotArgs &a, hipStream_t st) {
  if (a.n > 0) hipLaunchKernelGGL(k_gather_dot, dim3((unsigned)a.n), dim3(64), 0, st, a);
}

}  // namespace gto
