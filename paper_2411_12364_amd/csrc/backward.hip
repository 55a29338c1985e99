// Backward of the gather-sum (eq. (1), eq. (15) per virtual block, eq. (17) per column slice):
// the weight gradients dw[e] = <d_pooled[t_e, p_e], V[row_e]> (per slice with multi-core
// scoring) and the value-row gradients dV[row] += sum over the entries e on that row of
// w_e d_pooled[t_e, p_e].
//
// The T * bag entries are keyed by physical row and stably sorted (sort.hip), so the entries of
// one row form a run in their original order.  Most rows of a large table are chosen once, some
// by thousands of tokens, and the two are separate work:
//  * token_bwd_kernel walks the entries that are alone on their row token by token, with the token's
//    d_pooled row in registers: it reads the entry's value row for the weight gradient and writes its
//    gradient row (w_e d_pooled) there and then;
//  * the runs of several entries are cut into pieces of at most 64 entries; the row kernels read a
//    piece's value row once, and each entry's d_pooled row for the entry's weight gradient and for the
//    row's sum (row_dot).  A piece adds its sum into its row, or, where it continues a run, stores a
//    partial row that seg_join_kernel adds in order.
// Where rows repeat in few pieces or stay in the L2s (RowRule), and for narrow rows, token_bwd_kernel takes
// the weight gradients of all entries, and the rows are summed by another walk, a few columns at a time
// (row_walk).
// Every row has one writer and a fixed summation order: the result does not depend on timing, and
// no float atomics are needed.  The compact form writes one gradient row per run (distinct row)
// from zero instead of adding into a dense table.
//
// Backward of the scores (eqs. (2)-(4), (10), (16)) with the selection held fixed: one wave
// per (token, head) turns the weight gradients into grid-score gradients (SoftMax Jacobian where
// eq. (3)'s SoftMax weights), finds the distinct rows and columns of its slots (ballots over the
// key bits), recomputes their per-slice scores (Tucker), forms each slot's contribution to
// dS_row / dS_col and to dC, adds the contributions of slots that share a row (or column) in
// slot order, and writes dq = sum_i dS[i] K[i].  The key
// gradients dK[i] += dS[i] q are sums over tokens: each (token, head, axis) emits one entry per
// distinct key, the entries are stably sorted by key, and the key's pieces are summed in a fixed
// order as above.  dC sums its per-token partials in a fixed order (per thread, then a tree over
// the threads).
#include <algorithm>

#include "umem_internal.h"

namespace umem {
namespace {

constexpr int THREADS = 256;
constexpr int NWAVES = THREADS / kWave;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Each entry's physical row as the sort's key, its d_pooled row into prow[e], and the tile's
// histogram of its first digit (the sort's first counting pass, for which the keys need not be
// read again).
__global__ __launch_bounds__(kSortThreads) void bwd_keys_kernel(const int32_t* __restrict__ idx,
                                                                const int32_t* __restrict__ perm,
                                                                uint32_t n_values, int bag, int expand,
                                                                uint32_t* __restrict__ prow, SortPlan sp) {
  __shared__ uint32_t cnt[1 << kSortMaxDigitBits];
  const int nd = 1 << sp.dbits;
  const uint32_t mask = static_cast<uint32_t>(nd - 1);
  for (int d = threadIdx.x; d < nd; d += kSortThreads) cnt[d] = 0;
  __syncthreads();
  const int base = blockIdx.x * sp.tile, end = min(base + sp.tile, sp.M);
  for (int e = base + static_cast<int>(threadIdx.x); e < end; e += kSortThreads) {
    const int32_t x = idx[e];
    const uint32_t v = perm != nullptr ? static_cast<uint32_t>(perm[x]) : static_cast<uint32_t>(x);
    const uint32_t p = perm != nullptr ? v / n_values : 0u;
    const uint32_t row = v - p * n_values;
    sp.keys[e] = row;
    prow[e] = static_cast<uint32_t>(e / bag) * expand + p;
    atomicAdd(&cnt[row & mask], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < nd; d += kSortThreads)
    sp.hist[static_cast<size_t>(d) * sp.tiles + blockIdx.x] = cnt[d];
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

template <typename Elem>
struct Chunk;
template <>
struct Chunk<float> {
  static constexpr int kElems = 4;
  __device__ static inline void widen(const u32x4& r, float* x) {
    x[0] = __uint_as_float(r.x);
    x[1] = __uint_as_float(r.y);
    x[2] = __uint_as_float(r.z);
    x[3] = __uint_as_float(r.w);
  }
};
template <>
struct Chunk<uint16_t> {   // bf16 bit patterns
  static constexpr int kElems = 8;
  __device__ static inline void widen(const u32x4& r, float* x) {
    const uint32_t q[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(q[i] << 16);
      x[2 * i + 1] = __uint_as_float(q[i] & 0xFFFF0000u);
    }
  }
};

// ---------------------------------------------------------------- runs and pieces

// A run: the sorted entries of one key.  Runs are cut into pieces at every kSeg-th position, and
// each piece is one wave's work, so that a row chosen by thousands of tokens does not leave one
// wave walking them all.  The piece starts are listed in order (counted per chunk, then written
// from the sum of the earlier chunks' counts), and a fixed grid of waves walks the list.  A piece
// that is a whole run adds its sum into its row; one that continues its run (the first piece of
// segment g = positions [g kSeg, (g + 1) kSeg)) stores its partial row in slot g; one that starts a
// run that goes on stores its partial row in the gradient row itself where that is written from
// zero (compact form), else in slot g of its own (`heads_part`), so that what the row held takes one
// rounding.  seg_join_kernel adds, for each run spanning segments, its head and the partial rows of
// its later segments, in order, into the row.
constexpr int kSeg = kWave;

// Where sorted position i (< n) stands in its run.
struct Place {
  uint32_t key;
  bool starts, alone;      // first of its run; the only entry of its run
};
__device__ __forceinline__ Place place_at(const uint2* __restrict__ sorted, int i, int n) {
  Place p;
  p.key = sorted[i].x;
  p.starts = i == 0 || sorted[i - 1].x != p.key;
  p.alone = p.starts && (i + 1 == n || sorted[i + 1].x != p.key);
  return p;
}

// The end of the piece that starts at sorted position i of key `key`, and whether its run ends
// there.  Wave-uniform.
__device__ __forceinline__ int piece_end(const uint2* __restrict__ sorted, int i, int n, uint32_t key,
                                         bool* ends_run) {
  const int lane = threadIdx.x & (kWave - 1);
  const int seg_end = min(n, (i / kSeg + 1) * kSeg);
  const int pos = i + 1 + lane;
  const uint64_t diff = __ballot(pos < seg_end && sorted[pos].x != key);
  const int pe = diff != 0ull ? i + 1 + __builtin_ctzll(diff) : seg_end;
  *ends_run = pe == n || sorted[pe].x != key;
  return pe;
}

// The end of the run that holds sorted position i (wave-uniform).
__device__ __forceinline__ int run_end(const uint2* __restrict__ sorted, int i, int n, uint32_t key) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int base = i + 1; base < n; base += kWave) {
    const int pos = base + lane;
    const uint64_t same = __ballot(pos < n && sorted[pos].x == key);
    if (same != ~0ull) return base + __builtin_ctzll(~same);
  }
  return n;
}

constexpr int kListSteps = 4;                           // positions per thread, THREADS apart
constexpr int kListChunk = THREADS * kListSteps;        // positions per workgroup

// ROWS (value rows): only runs of several entries are cut into pieces, the entries alone on their
// row being the token kernel's; otherwise (keys) every run is.
template <bool ROWS>
__device__ __forceinline__ bool starts_piece(const Place& p, int i) {
  return (!ROWS || !p.alone) && (p.starts || i % kSeg == 0);
}

// Per chunk of kListChunk positions: the pieces (x) and runs (y) that start in it.
template <bool ROWS>
__global__ __launch_bounds__(THREADS) void piece_count_kernel(const uint2* __restrict__ sorted,
                                                              const uint32_t* __restrict__ n_sorted,
                                                              uint2* __restrict__ cnt) {
  __shared__ uint32_t wp[NWAVES], wr[NWAVES];
  const int n = static_cast<int>(*n_sorted);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t c = 0, cr = 0;
#pragma unroll
  for (int q = 0; q < kListSteps; ++q) {
    const int i = blockIdx.x * kListChunk + q * THREADS + threadIdx.x;
    bool piece = false, run = false;
    if (i < n) {
      const Place p = place_at(sorted, i, n);
      piece = starts_piece<ROWS>(p, i);
      run = p.starts;
    }
    c += __popcll(__ballot(piece));
    cr += __popcll(__ballot(run));
  }
  if (lane == 0) {
    wp[wave] = c;
    wr[wave] = cr;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c = cr = 0;
#pragma unroll
    for (int v = 0; v < NWAVES; ++v) {
      c += wp[v];
      cr += wr[v];
    }
    cnt[blockIdx.x] = make_uint2(c, cr);
  }
}

// What the ROWS form of piece_write_kernel leaves for the two gradient kernels.
constexpr uint32_t kAlone = 0x80000000u;
struct RowInfo {
  uint32_t* entry;          // [M] by entry: its d_pooled row (below 2^31), replaced by its run's
                            // number with kAlone where it is the run, without at a piece's start
  uint2* rec;               // [M] by sorted position, runs of several entries: the d_pooled row and
                            // the weight's bits (one core) or the entry (several)
  const float* w;           // the weights with one core, else NULL
  int32_t* rows_out;        // each run's row (compact form, else NULL)
  int32_t* n_runs;          // their number (compact form, else NULL)
};

// cnt: the counts of piece_count_kernel.  Writes the pieces' first sorted positions in order into
// list, their number into counts[0] and that of the runs into counts[2], and clears counts[1] (the
// spanning runs, appended later).
template <bool ROWS>
__global__ __launch_bounds__(THREADS) void piece_write_kernel(
    const uint2* __restrict__ sorted, const uint32_t* __restrict__ n_sorted,
    const uint2* __restrict__ cnt, uint32_t* __restrict__ list, uint32_t* __restrict__ counts,
    RowInfo info) {
  __shared__ uint2 wsum[NWAVES];
  __shared__ uint2 wcnt[kListSteps][NWAVES];
  const int n = static_cast<int>(*n_sorted);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t bp = 0, br = 0;
  for (int j = threadIdx.x; j < static_cast<int>(blockIdx.x); j += THREADS) {
    const uint2 c = cnt[j];
    bp += c.x;
    br += c.y;
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    bp += __shfl_xor(bp, off, kWave);
    br += __shfl_xor(br, off, kWave);
  }
  if (lane == 0) wsum[wave] = make_uint2(bp, br);
  Place pl[kListSteps];
  bool piece[kListSteps];
  uint64_t mp[kListSteps], mr[kListSteps];
#pragma unroll
  for (int q = 0; q < kListSteps; ++q) {
    const int i = blockIdx.x * kListChunk + q * THREADS + threadIdx.x;
    piece[q] = false;
    pl[q] = Place{0u, false, false};
    if (i < n) {
      pl[q] = place_at(sorted, i, n);
      piece[q] = starts_piece<ROWS>(pl[q], i);
    }
    mp[q] = __ballot(piece[q]);
    mr[q] = __ballot(pl[q].starts);
    if (lane == 0) wcnt[q][wave] = make_uint2(__popcll(mp[q]), __popcll(mr[q]));
  }
  __syncthreads();
  bp = br = 0;
#pragma unroll
  for (int v = 0; v < NWAVES; ++v) {
    bp += wsum[v].x;
    br += wsum[v].y;
  }
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int q = 0; q < kListSteps; ++q) {
    uint32_t ap = bp, ar = br;                            // before this wave's positions
#pragma unroll
    for (int v = 0; v < NWAVES; ++v) {
      const uint2 c = wcnt[q][v];
      ap += v < wave ? c.x : 0u;
      ar += v < wave ? c.y : 0u;
      bp += c.x;
      br += c.y;
    }
    const int i = blockIdx.x * kListChunk + q * THREADS + threadIdx.x;
    if (i >= n) continue;
    const uint32_t run = ar + __popcll(mr[q] & lt) + (pl[q].starts ? 0u : ~0u);   // starts, less one
    if (piece[q]) list[ap + __popcll(mp[q] & lt)] = static_cast<uint32_t>(i);
    if (ROWS) {
      const int ent = static_cast<int>(sorted[i].y);
      if (!pl[q].alone)
        info.rec[i] = make_uint2(info.entry[ent], info.w != nullptr ? __float_as_uint(info.w[ent]) : static_cast<uint32_t>(ent));
      if (pl[q].alone || piece[q]) info.entry[ent] = run | (pl[q].alone ? kAlone : 0u);
      if (info.rows_out != nullptr && pl[q].starts) info.rows_out[run] = static_cast<int32_t>(pl[q].key);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    counts[0] = bp;
    counts[1] = 0u;
    counts[2] = br;
    if (ROWS && info.n_runs != nullptr) *info.n_runs = static_cast<int32_t>(br);
  }
}

int list_chunks(int M) { return (M + kListChunk - 1) / kListChunk; }

// Whether the token kernel takes the weight gradients of the runs of several entries too, and their rows are
// summed by columns (row_walk); otherwise a row is read once for its run (row_dot) and not for each of its
// entries.  By token where a call touches few distinct rows (at most `few`, kFewBytes of them: the entries find
// them in the L2s) and d_pooled lies by slice, and where rows repeat (four entries a row, of `entries`) in few
// pieces: a wave each, which goes through all columns of a wide row, they leave the chip short of waves.  Calls
// of at most kTinyCall entries, where nothing but the chain of loads counts, all go by token (a row to a wave).
// Compact form, by token / row_dot (us): 4,096 tokens of 256 entries on rows of 1 KiB, 4,096 rows 351 / 395,
// 7,600 in clusters 383 / 392, 16,384 561 / 446, 32,768 529 / 453, 65,536 588 / 453, 262,144 714 / 571; 2,048
// tokens of 64 entries on rows of 2 KiB, 2,048 rows in clusters 115 / 153, 4,096 117 / 140, 16,384 (18,000
// pieces) 148 / 126; 4,096 tokens of 64 on 8,192 rows (12,300 pieces) 193 / 226; 512 tokens of 84 on rows of 7
// KiB, 2,688 rows in clusters (3,400 pieces) 161 / 252; of 8 KiB in four blocks (d_pooled as it is), 1,000 rows
// 112 / 242, 2,688 154 / 187, but 88,000 (7,500 pieces of two entries) 284 / 182 on rows of 7 KiB.
constexpr uint32_t kFewBytes = 8u << 20, kFewPieces = 14336;
constexpr int kTinyCall = 4096;
struct RowRule {
  uint32_t few, entries;
  __device__ __forceinline__ bool repeats(const uint32_t* __restrict__ counts) const { return 4 * counts[2] <= entries; }
  __device__ __forceinline__ bool by_token(const uint32_t* __restrict__ counts) const {
    return counts[2] <= few || (counts[0] <= kFewPieces && repeats(counts));
  }
};

// ---------------------------------------------------------------- value rows, token by token

constexpr int kTokenWaves = 8192;       // waves the launch aims at (eight per SIMD)

// Sum over the aligned group of L lanes that a lane belongs to, valid in its last lane: DPP row
// shifts within 16 lanes, then the row broadcasts (L > 16).
template <int L>
__device__ __forceinline__ float group_total(float x) {
  int r = __builtin_bit_cast(int, x);
#define UMEM_ADD(CTRL, ROWS)                                                                   \
  r = __builtin_bit_cast(int, __builtin_bit_cast(float, r) +                                    \
                         __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, r, CTRL, ROWS, 0xF, true)))
  if (L >= 2) UMEM_ADD(0x111, 0xF);      // row_shr:1
  if (L >= 4) UMEM_ADD(0x112, 0xF);      // row_shr:2
  if (L >= 8) UMEM_ADD(0x114, 0xF);      // row_shr:4
  if (L >= 16) UMEM_ADD(0x118, 0xF);     // row_shr:8
  if (L >= 32) UMEM_ADD(0x142, 0xA);     // row_bcast:15 into rows 1 and 3
  if (L >= 64) UMEM_ADD(0x143, 0xC);     // row_bcast:31 into rows 2 and 3
#undef UMEM_ADD
  return __builtin_bit_cast(float, r);
}

// One workgroup per token (gridDim.y of them share a bag); entries ordered by virtual block, CW
// waves taking one entry's columns together (64 lanes x CPL chunks of 16 bytes each), the
// workgroup's NWAVES / CW groups of waves contiguous ranges of its share of the bag.  For rows of
// 1 KiB and more a wave keeps its columns of the block's d_pooled row in registers and reloads them
// where the block changes; narrower rows are read L lanes each, 64 / L entries at once, with their
// d_pooled rows from cache.  Entry j of a group's current 64 leaves its partial weight gradients in
// LDS ([group][wave][core][j]), which are added in wave order behind a barrier per 64 entries.
// SLICED, where all weight gradients are taken here: the wave that takes a block's first entry also leaves
// its d_pooled columns in `sliced`, by column slice (row_walk).  Wide rows are split between waves (CW = 4
// at 4096 bf16 columns) because the d_pooled row of a whole one takes 64 registers beside the value row:
// three waves per SIMD, one row in flight each.  (Rows of 5 and 7 KiB, which do not split evenly, stay whole
// all the same: 512 tokens of 84 lone rows 198 and 266 us the call, 300 and 368 in one kernel with the sums.)
// Bound by HBM: each value row is read once and each lone entry's gradient row written once.  At
// 2,048 tokens of 64 rows of 2 KiB (121,600 distinct) it moves 764 MB in 158 us, 4.8 TB/s, the rate
// of a large device copy; at 512 tokens of 84 rows of 8 KiB 1.06 GB in 224 us.  A wave per row read
// d_pooled again for each of them, from the MALL: 268 and 332 us.  Nontemporal stores of the
// gradient rows took 274 us at 8 KiB rows (the same at 2 KiB), nontemporal row loads 192 at 2 KiB;
// eight or two loads in flight a lane instead of four 163 and 161 us.
template <typename Elem, int L, int CPL, int CW, bool SLICED, bool DENSE>
__global__ __launch_bounds__(THREADS) void token_bwd_kernel(
    const Elem* __restrict__ values, int dv, int bag, const int32_t* __restrict__ idx,
    const float* __restrict__ w, const int32_t* __restrict__ perm, uint32_t n_values, int expand,
    int cores, const float* __restrict__ d_pooled, const uint32_t* __restrict__ info,
    float* __restrict__ d_rows, float* __restrict__ dw, float* __restrict__ sliced,
    int slice_cols, const uint32_t* __restrict__ counts, RowRule rule) {
  using TR = Chunk<Elem>;
  constexpr int EPC = TR::kElems;
  constexpr int SUB = kWave / L;                   // entries a wave reads at once
    constexpr int U = CPL >= 4 ? 1 : 4 / CPL;        // batches of them in flight
  constexpr int NG = NWAVES / CW;                  // groups of waves
  static_assert(L == kWave || (CW == 1 && CPL == 1 && !SLICED), "several entries at once only in narrow rows");
  extern __shared__ __align__(16) int32_t lds[];   // [NWAVES][cores][64] sums, then [3][bag]
  float* const sums = reinterpret_cast<float*>(lds);
  const int t = blockIdx.x;
  const int32_t* __restrict__ idx_t = idx + static_cast<size_t>(t) * bag;
  const float* __restrict__ w_t = w + static_cast<size_t>(t) * bag * cores;
  const uint32_t* __restrict__ info_t = info + static_cast<size_t>(t) * bag;
  float* __restrict__ dw_t = dw + static_cast<size_t>(t) * bag * cores;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  int32_t *rows = lds + NWAVES * cores * kWave, *blk = rows + bag, *order = blk + bag;
  // which entries: all where the others' rows are summed without the value rows, else those alone on theirs
  const bool all = L != kWave || rule.by_token(counts);
  int n_mine = bag;
  if (expand > 1) {
    __shared__ int bcount[kMaxExpand], total;
    for (int p = tid; p < expand; p += THREADS) bcount[p] = 0;
    __syncthreads();
    for (int s = tid; s < bag; s += THREADS) {
      const uint32_t v = static_cast<uint32_t>(perm[idx_t[s]]);
      const uint32_t p = v / n_values;
      const bool mine = all || (info_t[s] & kAlone) != 0u;
      rows[s] = static_cast<int32_t>(v - p * n_values);
      blk[s] = mine ? static_cast<int32_t>(p) : -1;
      if (mine) atomicAdd(&bcount[p], 1);
    }
    __syncthreads();
    // entries by block, stably (the workgroups that share a bag must agree on the order): wave 0
    // places 64 at a time, each after its block's earlier ones
    if (wave == 0) {
      const int c = lane < expand ? bcount[lane] : 0;
      const int incl = wave_inclusive_scan(c);
      wave_lds_order();
      if (lane < expand) bcount[lane] = incl - c;
      if (lane == kWave - 1) total = incl;
      wave_lds_order();
      const uint64_t lt = lanemask_lt();
      for (int s0 = 0; s0 < bag; s0 += kWave) {
        const int s = s0 + lane;
        const int p = s < bag ? blk[s] : -1;
        uint64_t peers = __ballot(p >= 0);
        for (int b = 0; (1 << b) < expand; ++b) {
          const bool one = (p >> b) & 1;
          const uint64_t ones = __ballot(one);
          peers &= one ? ones : ~ones;
        }
        const int at = bcount[max(p, 0)];
        const int rank = __popcll(peers & lt);
        if (p >= 0) order[at + rank] = s;
        wave_lds_order();
        if (p >= 0 && rank == 0) bcount[p] = at + __popcll(peers);
        wave_lds_order();
      }
    }
    __syncthreads();
    n_mine = __builtin_amdgcn_readfirstlane(total);
  } else {                                         // the bag as it is, others' entries passed over
    for (int s = tid; s < bag; s += THREADS) {
      rows[s] = idx_t[s];
      blk[s] = all || (info_t[s] & kAlone) != 0u ? 0 : -1;
      order[s] = s;
    }
    __syncthreads();
  }
  const int parts = NG * gridDim.y, group = wave / CW;
  const int per = (n_mine + parts - 1) / parts;
  const int part = blockIdx.y * NG + group;
  const int beg = min(n_mine, part * per), end = min(n_mine, beg + per);
  const int sub = lane / L, cl = lane % L;
  const int chunk0 = (wave % CW) * CPL * kWave + cl;    // the lane's first 16-byte chunk of the row
  const int per_core = dv / cores;
  int slice[CPL];                                  // this lane's chunks' core (0 with one core)
#pragma unroll
  for (int c = 0; c < CPL; ++c) slice[c] = cores > 1 ? ((chunk0 + L * c) * EPC) / per_core : 0;
  // the cores this wave's columns belong to
  const int core_lo = L == kWave ? __builtin_amdgcn_readfirstlane(slice[0]) : 0;
  const int core_hi = L == kWave ? __builtin_amdgcn_readlane(slice[CPL - 1], kWave - 1) : cores - 1;
  float dp[CPL][EPC];                              // L == 64: the current block's d_pooled columns
  int held = -1;
  for (int r0 = 0; r0 < per; r0 += kWave) {        // rounds of up to 64 entries a group
    for (int k = 0; k < cores; ++k) sums[(wave * cores + k) * kWave + lane] = 0.0f;
    wave_lds_order();
    const int rbeg = beg + r0, rend = min(end, rbeg + kWave);
    for (int j0 = rbeg; j0 < rend; j0 += SUB * U) {
      u32x4 raw[U][CPL];
      int ent[U], row[U], blk_of[U];
      uint32_t inf[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + SUB * u + sub;
        ent[u] = -1;
        row[u] = blk_of[u] = 0;
        inf[u] = 0u;
#pragma unroll
        for (int c = 0; c < CPL; ++c) raw[u][c] = u32x4{0u, 0u, 0u, 0u};
        if (j < rend) {
          int s = order[j];
          if (L == kWave) s = __builtin_amdgcn_readfirstlane(s);    // one entry for the wave
          int r = rows[s];
          int p = blk[s];
          if (L == kWave) {
            r = __builtin_amdgcn_readfirstlane(r);
            p = __builtin_amdgcn_readfirstlane(p);
          }
          if (p >= 0) {                            // (wave-uniform where a wave takes one entry)
            ent[u] = s;
            row[u] = r;
            blk_of[u] = p;
            inf[u] = info_t[s];
            const Elem* src = values + static_cast<size_t>(r) * dv;
#pragma unroll
            for (int c = 0; c < CPL; ++c)
              raw[u][c] = *reinterpret_cast<const u32x4*>(src + (chunk0 + L * c) * EPC);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (L == kWave && j0 + u >= rend) break;   // (wave-uniform)
        if (L == kWave && ent[u] < 0) continue;
        const bool on = ent[u] >= 0;
        const int p = blk_of[u];
        if (L != kWave || p != held) {
          const float* src = d_pooled + (static_cast<size_t>(t) * expand + p) * dv;
#pragma unroll
          for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int e = 0; e < EPC; e += 4) {
              const f32x4 v = *reinterpret_cast<const f32x4*>(src + (chunk0 + L * c) * EPC + e);
              dp[c][e] = v.x;
              dp[c][e + 1] = v.y;
              dp[c][e + 2] = v.z;
              dp[c][e + 3] = v.w;
              if (SLICED && all && (j0 + u == 0 || blk[order[max(j0 + u - 1, 0)]] != p)) {
                const int col = (chunk0 + L * c) * EPC + e;       // slices are whole 16-byte pieces
                const size_t at = (static_cast<size_t>(col / slice_cols) * gridDim.x + t) * expand + p;
                *reinterpret_cast<f32x4*>(sliced + at * slice_cols + col % slice_cols) = v;
              }
            }
          held = p;
        }
        float dot[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          float x[EPC];
          TR::widen(raw[u][c], x);
          dot[c] = 0.0f;
#pragma unroll
          for (int e = 0; e < EPC; ++e) dot[c] = fmaf(dp[c][e], x[e], dot[c]);
        }
        for (int k = core_lo; k <= core_hi; ++k) {
          float v = 0.0f;                          // (chunk by chunk, as row_dot adds them)
#pragma unroll
          for (int c = 0; c < CPL; ++c) v += group_total<L>(slice[c] == k ? dot[c] : 0.0f);
          if (cl == L - 1 && on) sums[(wave * cores + k) * kWave + (j0 + SUB * u + sub - rbeg)] = v;
        }
        if (on && (inf[u] & kAlone) != 0u) {       // alone on its row: the gradient row is here
          float* dst = d_rows + static_cast<size_t>(DENSE ? static_cast<uint32_t>(row[u]) : inf[u] & ~kAlone) * dv;
          f32x4 old[DENSE ? CPL : 1][EPC / 4];
          if constexpr (DENSE) {
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
              for (int e = 0; e < EPC; e += 4)
                old[c][e / 4] = *reinterpret_cast<const f32x4*>(dst + (chunk0 + L * c) * EPC + e);
          }
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            const float wt = w_t[static_cast<size_t>(ent[u]) * cores + slice[c]];
#pragma unroll
            for (int e = 0; e < EPC; e += 4) {
              f32x4 v = DENSE ? old[DENSE ? c : 0][e / 4] : f32x4{0.f, 0.f, 0.f, 0.f};
              v.x += wt * dp[c][e];
              v.y += wt * dp[c][e + 1];
              v.z += wt * dp[c][e + 2];
              v.w += wt * dp[c][e + 3];
              *reinterpret_cast<f32x4*>(dst + (chunk0 + L * c) * EPC + e) = v;
            }
          }
        }
      }
    }
    if (CW > 1) __syncthreads();                   // (every wave takes every round)
    else wave_lds_order();
    // the group's waves share its entries' sums out: lane = entry, wave % CW, + CW, ... = core
    for (int k = wave % CW; k < cores; k += CW) {
      const int j = rbeg + lane;
      if (j < rend && blk[order[j]] >= 0) {
        float v = sums[(group * CW * cores + k) * kWave + lane];
#pragma unroll
        for (int x = 1; x < CW; ++x) v += sums[((group * CW + x) * cores + k) * kWave + lane];
        const int s = order[j];
        dw_t[static_cast<size_t>(s) * cores + k] = v;
      }
    }
    if (CW > 1) __syncthreads();                   // before the next round clears the sums
    else wave_lds_order();
  }
}

// ---------------------------------------------------------------- value rows of several entries

constexpr int kListWaves = 8192;        // waves of the grids that walk the key lists (b2)
constexpr int kRowWaves = 16384;         // ... and the row lists
constexpr int kJoinWaves = 4096;        // ... and of the join
constexpr int kInFlight = 4;            // a key piece's entries whose loads are issued together
constexpr int kRowInFlight = 4;         // a row piece's

// A row piece before it is walked: where it starts, its rows and entries and their records (one per
// lane), and the rows on either side.
struct RowPiece {
  uint32_t at;           // first sorted position
  uint2 own;             // lane: (row, entry) of position first + lane
  uint2 rec;             // lane: its RowInfo::rec
  uint32_t prev, next;   // the rows at first - 1 and first + 64
};

// A piece as the walks below take it: its entries n_e, whether it starts and ends its run.
struct PieceEnds {
  uint32_t row;
  int n_e;
  bool starts, ends;
};

// The pieces k = first, first + step, ... of the list in turn, to body(k, piece, ends).  The next piece's
// record is read two pieces ahead and its entries one piece ahead.
template <typename Body>
__device__ __forceinline__ void walk_pieces(const uint2* __restrict__ sorted, int n, const uint2* __restrict__ rec,
                                            const uint32_t* __restrict__ list, uint32_t n_pieces,
                                            uint32_t first, uint32_t step, Body body) {
  const int lane = threadIdx.x & (kWave - 1);
  auto fetch = [&](uint32_t at, RowPiece& p) {
    p.at = at;
    const int ps = static_cast<int>(at);
    const int pos = min(ps + lane, n - 1);
    p.own = sorted[pos];
    p.rec = rec[pos];
    p.prev = sorted[max(ps - 1, 0)].x;
    p.next = sorted[min(ps + kWave, n - 1)].x;
  };
  if (first >= n_pieces) return;
  RowPiece nxt;
  fetch(list[first], nxt);
  uint32_t after = first + step < n_pieces ? list[first + step] : 0u;
  for (uint32_t k = first; k < n_pieces; k += step) {  // wave-uniform
    const RowPiece cur = nxt;
    if (k + step < n_pieces) fetch(after, nxt);
    if (k + 2 * step < n_pieces) after = list[k + 2 * step];
    const int ps = static_cast<int>(cur.at);
    PieceEnds e;
    e.row = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(cur.own.x)));
    e.starts = ps == 0 || cur.prev != e.row;
    const int seg_end = min(n, (ps / kSeg + 1) * kSeg);
    const uint64_t other = __ballot(ps + lane < seg_end && cur.own.x != e.row);
    e.n_e = other != 0ull ? __builtin_ctzll(other) : seg_end - ps;
    // the row after the piece (a piece that stops before its segment's end stops at another row)
    const uint32_t past = e.n_e == kWave ? cur.next : static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(cur.own.x), e.n_e & (kWave - 1)));
    e.ends = ps + e.n_e >= n || past != e.row;
    body(k, cur, e);
  }
}

// What the walks read and write.
struct RowArgs {
  const uint2* sorted;
  const uint32_t* n_sorted;
  const uint2* rec;
  const uint32_t *info, *list;
  uint32_t *counts, *heads;
  const float* w;
  int cores, dv, compact;
  size_t pooled_rows;
  const float *d_pooled, *sliced;
  float *out, *dw, *partial, *heads_part;

  __device__ __forceinline__ float* row_of(const RowPiece& p, const PieceEnds& e) const {
    const uint32_t r = compact ? info[__builtin_amdgcn_readfirstlane(static_cast<int>(p.own.y))] & ~kAlone : e.row;
    return out + static_cast<size_t>(r) * dv;
  }
  // where a piece's sum goes: its row (after what that held, where the run is whole) or a partial row
  __device__ __forceinline__ float* sum_at(const RowPiece& p, const PieceEnds& e, float* dst) const {
    if (e.starts && (e.ends || compact)) return dst;
    return (e.starts ? heads_part : partial) + static_cast<size_t>(p.at / kSeg) * dv;
  }
};

// The pieces of the runs of several entries: their w_e d_pooled rows summed.  The entries j, j + S,
// j + 2 S, ... of a piece are one group's, added in order; the S groups then meet by a fixed tree.  GL
// lanes of 16 bytes take an entry, 64 / GL = S groups at once.
// Bound by the re-reads of d_pooled: a run's tokens are random, so its rows come from all over.
// COLUMNS: 4 GL columns at a time, slice s of them by XCD s % 8 (workgroups go to XCDs round-robin), from the
// copy that token_bwd_kernel left by column slice, [slice][pooled row][4 GL columns], where there is one: an
// XCD then reads a few columns of every row, a contiguous block that its 4 MiB L2 holds.  (The same
// slices of d_pooled itself lie a row apart, on two of the L2's sixteen channels.  Where pieces are few they
// still leave more waves to the chip than whole rows: 512 tokens of 84 entries on 1,000 rows of 8 KiB 112
// us the call, 177 with a wave to a whole row.)  Otherwise (rows below 1 KiB, tiny calls) a wave walks all
// columns of its piece.  At 4,096 tokens of 256 entries on 7,600 rows
// (2 KiB of d_pooled an entry): 146 us beside the token kernel's 108, against 342 us for one kernel that
// did both from d_pooled as it is.  8,192 waves 169 us, 32,768 146; two entries in flight a lane group
// 252, eight 153; slices of half the columns (2 MiB of d_pooled an XCD) no faster.
template <int GL, bool COLUMNS>
__device__ __forceinline__ void row_walk(const RowArgs& A) {
  constexpr int S = kWave / GL, kCols = 4 * GL;
  const int lane = threadIdx.x & (kWave - 1);
  const int sub = lane / GL;
  const int dv = A.dv, cores = A.cores, per_core = dv / cores;
  // by columns: each XCD walks the whole list for its own slices
  const uint32_t xcds = COLUMNS ? 8u : 1u;
  const uint32_t first = (blockIdx.x / xcds) * NWAVES + threadIdx.x / kWave;
  const uint32_t step = (gridDim.x / xcds) * NWAVES;
  const int c_first = COLUMNS ? static_cast<int>(blockIdx.x & 7u) * kCols : 0;
  const uint32_t n_pieces = A.counts[0];
  for (int c0 = c_first; c0 < (COLUMNS ? dv : 1); c0 += 8 * kCols) {
    walk_pieces(A.sorted, static_cast<int>(*A.n_sorted), A.rec, A.list, n_pieces, first, step,
                [&](uint32_t k, const RowPiece& cur, const PieceEnds& e) {
      const int n_e = e.n_e;
      if (c0 == 0 && e.starts && !e.ends && lane == 0) A.heads[atomicAdd(A.counts + 1, 1u)] = k;
      const int my_prow = static_cast<int>(cur.rec.x);
      const int my_we = static_cast<int>(cur.rec.y);
      float* row = A.row_of(cur, e);
      for (int c = c0; c < (COLUMNS ? c0 + 1 : dv); c += kCols) {
        const int col = c + (lane % GL) * 4;
        const int core = cores > 1 ? col / per_core : 0;   // four columns lie in one core's slice
        const bool copy = COLUMNS && A.sliced != nullptr;
        const float* src = copy ? A.sliced + static_cast<size_t>(c0 / kCols) * A.pooled_rows * kCols + (col - c0)
                                : A.d_pooled + col;
        const int pitch = copy ? kCols : dv;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        f32x4 old = {0.f, 0.f, 0.f, 0.f};
        if (e.starts && e.ends && !A.compact && sub == 0) old = *reinterpret_cast<const f32x4*>(row + col);
        for (int j0 = 0; j0 < n_e; j0 += S * kRowInFlight) {  // wave-uniform
          f32x4 v[kRowInFlight];
          float wt[kRowInFlight];
#pragma unroll
          for (int u = 0; u < kRowInFlight; ++u) {         // all loads first
            const int j = j0 + S * u + sub;
            const int jj = min(j, n_e - 1);
            const int pr = __shfl(my_prow, jj, kWave);
            const int we = __shfl(my_we, jj, kWave);
            v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            wt[u] = __int_as_float(we);
            if (cores > 1) wt[u] = j < n_e ? A.w[static_cast<size_t>(we) * cores + core] : 0.0f;
            if (j < n_e) v[u] = *reinterpret_cast<const f32x4*>(src + static_cast<size_t>(pr) * pitch);
          }
#pragma unroll
          for (int u = 0; u < kRowInFlight; ++u) {         // then this group's entries in order
            const int j = j0 + S * u + sub;
            if (j >= n_e) continue;                        // (no product with a row that is not there)
            acc.x = fmaf(wt[u], v[u].x, acc.x);
            acc.y = fmaf(wt[u], v[u].y, acc.y);
            acc.z = fmaf(wt[u], v[u].z, acc.z);
            acc.w = fmaf(wt[u], v[u].w, acc.w);
          }
        }
#pragma unroll
        for (int off = GL; off < kWave; off <<= 1) {
          acc.x += __shfl_xor(acc.x, off, kWave);
          acc.y += __shfl_xor(acc.y, off, kWave);
          acc.z += __shfl_xor(acc.z, off, kWave);
          acc.w += __shfl_xor(acc.w, off, kWave);
        }
        if (sub == 0) *reinterpret_cast<f32x4*>(A.sum_at(cur, e, row) + col) = old + acc;
      }
    });
  }
}

// The same pieces with their weight gradients, rows of 1 KiB and more: a wave takes 64 16-byte chunks of
// the piece's value row at a time and reads each entry's d_pooled columns once, for the dot and for the
// sum.  S groups of entries as row_walk's (S of them in a lane's registers), and the dots added chunk
// by chunk and, after every `cpl` chunks, between the waves' shares, as token_bwd_kernel adds them: dense
// and compact form give the same bits whichever kernel a call takes.
// Bound by the re-reads of d_pooled, one an entry.  With the weight gradients left to the token kernel,
// which reads a value row for each entry, calls whose rows repeat a few times were slower than the
// one-kernel form of old: dense, 4,096 tokens of 256 entries (rows of 1 KiB, 2 KiB of d_pooled an entry) on
// 262,144 / 65,536 rows 781 / 609 us the whole call, 647 / 466 now, 687 / 503 then; compact 934 / 588, 636 / 453,
// 665 / 492.  Four waves per SIMD for S = 4 (128 registers, two of them in scratch): 612 / 484.
template <typename Elem, int S>
__device__ __forceinline__ void row_dot(const RowArgs& A, const Elem* __restrict__ values, int cpl) {
  constexpr int EPC = Chunk<Elem>::kElems, Q = EPC / 4;
  constexpr int U = kRowInFlight, kTurns = S > U ? S / U : 1;  // entries in flight; batches until the groups recur
  const int lane = threadIdx.x & (kWave - 1);
  const int dv = A.dv, cores = A.cores, per_core = dv / cores;
  const uint32_t first = blockIdx.x * NWAVES + threadIdx.x / kWave;
  walk_pieces(A.sorted, static_cast<int>(*A.n_sorted), A.rec, A.list, A.counts[0], first, gridDim.x * NWAVES,
              [&](uint32_t k, const RowPiece& cur, const PieceEnds& e) {
    const int n_e = e.n_e;
    if (e.starts && !e.ends && lane == 0) A.heads[atomicAdd(A.counts + 1, 1u)] = k;
    const int my_prow = static_cast<int>(cur.rec.x);
    const int my_we = static_cast<int>(cur.rec.y);
    float* row = A.row_of(cur, e);
    float my_dw[kMaxCores], share[kMaxCores];                // lane j: entry j's, by core
#pragma unroll
    for (int c = 0; c < kMaxCores; ++c) my_dw[c] = share[c] = 0.0f;
    int chunk = 0;
    for (int c0 = 0; c0 < dv; c0 += kWave * EPC) {
      const int col = c0 + lane * EPC;
      const int core = cores > 1 ? col / per_core : 0;       // a chunk lies in one core's slice
      const u32x4 raw = *reinterpret_cast<const u32x4*>(values + static_cast<size_t>(e.row) * dv + col);
      f32x4 acc[S][Q], old[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        old[q] = e.starts && e.ends && !A.compact ? *reinterpret_cast<const f32x4*>(row + col + 4 * q)
                                                  : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < S; ++i) acc[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      float x[EPC];
      Chunk<Elem>::widen(raw, x);
      for (int jt = 0; jt < n_e; jt += U * kTurns) {         // wave-uniform
#pragma unroll
       for (int turn = 0; turn < kTurns; ++turn) {
        const int j0 = jt + U * turn;
        if (j0 >= n_e) break;
        f32x4 v[U][Q];
        float wt[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {                        // all loads first
          const int j = min(j0 + u, n_e - 1);
          const int pr = __builtin_amdgcn_readlane(my_prow, j);
          const int we = __builtin_amdgcn_readlane(my_we, j);
          wt[u] = cores > 1 ? A.w[static_cast<size_t>(we) * cores + core] : __int_as_float(we);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            v[u][q] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (j0 + u < n_e) v[u][q] = *reinterpret_cast<const f32x4*>(A.d_pooled + static_cast<size_t>(pr) * dv + col + 4 * q);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {                        // then each group's entries in order
          if (j0 + u >= n_e) break;
          float dot = 0.0f;
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            f32x4& a = acc[(U * turn + u) % S][q];
            dot = fmaf(v[u][q].x, x[4 * q], dot);
            dot = fmaf(v[u][q].y, x[4 * q + 1], dot);
            dot = fmaf(v[u][q].z, x[4 * q + 2], dot);
            dot = fmaf(v[u][q].w, x[4 * q + 3], dot);
            a.x = fmaf(wt[u], v[u][q].x, a.x);
            a.y = fmaf(wt[u], v[u][q].y, a.y);
            a.z = fmaf(wt[u], v[u][q].z, a.z);
            a.w = fmaf(wt[u], v[u][q].w, a.w);
          }
          const int lo = __builtin_amdgcn_readfirstlane(core), hi = __builtin_amdgcn_readlane(core, kWave - 1);
#pragma unroll
          for (int c = 0; c < kMaxCores; ++c) {
            if (c < lo || c > hi) continue;                  // (wave-uniform)
            const float t = group_total<kWave>(core == c ? dot : 0.0f);
            const float sum = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), kWave - 1));
            if (lane == j0 + u) share[c] += sum;
          }
        }
       }
      }
#pragma unroll
      for (int off = 1; off < S; off <<= 1)
#pragma unroll
        for (int i = 0; i < S; i += 2 * off)
#pragma unroll
          for (int q = 0; q < Q; ++q) acc[i][q] += acc[i + off][q];
      float* dst = A.sum_at(cur, e, row) + col;
#pragma unroll
      for (int q = 0; q < Q; ++q) *reinterpret_cast<f32x4*>(dst + 4 * q) = old[q] + acc[0][q];
      if (++chunk == cpl) {
        chunk = 0;
#pragma unroll
        for (int c = 0; c < kMaxCores; ++c) {
          my_dw[c] += share[c];
          share[c] = 0.0f;
        }
      }
    }
    if (lane < n_e) {                                        // this wave is the entries' only writer
      float* dw = A.dw + static_cast<size_t>(cur.own.y) * cores;
#pragma unroll
      for (int c = 0; c < kMaxCores; ++c)
        if (c < cores) dw[c] = my_dw[c];
    }
  });
}

// Rows of 1 KiB and more: with their weight gradients, or, where these are the token kernel's, by columns.
// In one launch with one group of entries (110 registers at most); an empty launch takes 3 us.
template <typename Elem, int GL>
__global__ __launch_bounds__(THREADS) void row_bwd_kernel(RowArgs A, const Elem* __restrict__ values, int cpl,
                                                          RowRule rule) {
  if (rule.by_token(A.counts)) row_walk<GL, true>(A);
  else row_dot<Elem, 1>(A, values, cpl);
}

// d_pooled by slice: row_dot's registers for S groups would leave the walk three waves per SIMD of five.
template <typename Elem, int S>
__global__ __launch_bounds__(THREADS) void row_bwd_dots_kernel(RowArgs A, const Elem* __restrict__ values, int cpl,
                                                               RowRule rule) {
  if (!rule.by_token(A.counts)) row_dot<Elem, S>(A, values, cpl);
}
template <int GL>
__global__ __launch_bounds__(THREADS) void row_bwd_sliced_kernel(RowArgs A, RowRule rule) {
  if (rule.by_token(A.counts)) row_walk<GL, true>(A);
}

// Narrower rows, GL lanes an entry; and tiny calls' rows of any width.
template <int GL>
__global__ __launch_bounds__(THREADS) void row_bwd_narrow_kernel(RowArgs A) {
  row_walk<GL, false>(A);
}

// One wave per run that spans segments: its head (heads_part, or what the row holds: compact form)
// and the partial rows of its later segments, in order, added into the row.
// heads: the places in list of those runs' first pieces.
__global__ __launch_bounds__(THREADS) void seg_join_kernel(const uint2* __restrict__ sorted,
                                                           const uint32_t* __restrict__ n_sorted,
                                                           int width, const float* __restrict__ partial,
                                                           const float* __restrict__ heads_part,
                                                           float* __restrict__ out,
                                                           const uint32_t* __restrict__ list,
                                                           const uint32_t* __restrict__ heads,
                                                           const uint32_t* __restrict__ counts,
                                                           int H, int n, float* __restrict__ out2,
                                                           const uint32_t* __restrict__ info) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t n_heads = counts[1];
  for (uint32_t hk = blockIdx.x * NWAVES + threadIdx.x / kWave; hk < n_heads;
       hk += gridDim.x * NWAVES) {
    const int i = static_cast<int>(list[heads[hk]]);
    const uint32_t key = sorted[i].x;
    const int g0 = i / kSeg;
    const int end = run_end(sorted, i, static_cast<int>(*n_sorted), key);
    const int g1 = (end - 1) / kSeg;
    // the row of this key: value rows directly, or (out2 given) key rows of the two axes
    float* dst;
    if (info != nullptr) {                             // compact rows: by run
      dst = out + static_cast<size_t>(info[sorted[i].y] & ~kAlone) * width;
    } else if (out2 == nullptr) {
      dst = out + static_cast<size_t>(key) * width;
    } else {
      const int axis = static_cast<int>(key / (static_cast<uint32_t>(H) * n));
      dst = (axis ? out2 : out) + static_cast<size_t>(key - static_cast<uint32_t>(axis) * H * n) * width;
    }
    for (int c = lane * 4; c < width; c += kWave * 4) {
      f32x4* d = reinterpret_cast<f32x4*>(dst + c);
      const f32x4 held = *d;
      f32x4 acc = info != nullptr ? held : *reinterpret_cast<const f32x4*>(heads_part + static_cast<size_t>(g0) * width + c);
      for (int g = g0 + 1; g <= g1; ++g)
        acc += *reinterpret_cast<const f32x4*>(partial + static_cast<size_t>(g) * width + c);
      *d = info != nullptr ? acc : held + acc;
    }
  }
}

// ---------------------------------------------------------------- score backward

// One wave per (token, head); slot s = g * 64 + lane for the NG groups g of a lane.  The waves
// of a workgroup share nothing, so the kernel has no workgroup barrier; each wave's own LDS
// traffic is ordered by wave_lds_order.
template <int NG>
struct ScoreBwdLds {
  int dist[2][NG * kWave];                     // distinct rows / columns, in slot order
  float sd[2][NG * kWave][kMaxRank];           // per distinct key: its per-slice score, then its dS
  float cs[2][NG * kWave][kMaxRank];           // per slot: its dS_row / dS_col term
};

template <int NG>
constexpr int score_bwd_waves() { return NG >= 4 ? 2 : 4; }

// The lanes whose key_other (valid_other) equals this lane's key: one ballot per key bit.
__device__ __forceinline__ uint64_t key_match(uint32_t key, uint32_t key_other, bool valid_other,
                                              int bits) {
  uint64_t mask = __ballot(valid_other);
  for (int b = 0; b < bits; ++b) {
    const uint64_t ones = __ballot(valid_other && ((key_other >> b) & 1u));
    mask &= ((key >> b) & 1u) ? ones : ~ones;
  }
  return mask;
}

template <int NG>
__global__ __launch_bounds__(score_bwd_waves<NG>() * kWave) void score_bwd_kernel(
    const float* __restrict__ q_row, const float* __restrict__ q_col,
    const float* __restrict__ k_row, const float* __restrict__ k_col,
    const float* __restrict__ core_all, const int32_t* __restrict__ idx,
    const float* __restrict__ w, const float* __restrict__ dw, int T, int H, int n, int key_bits,
    int dk, int rank, int m, int tucker, int softmax, int hc, float* __restrict__ dq_row,
    float* __restrict__ dq_col, uint32_t* __restrict__ ekeys, float* __restrict__ edS,
    float* __restrict__ dc_part) {
  constexpr int W = score_bwd_waves<NG>();
  __shared__ ScoreBwdLds<NG> lds[W];
  const int lane = threadIdx.x & (kWave - 1);
  ScoreBwdLds<NG>& sh = lds[threadIdx.x / kWave];
  // (token, head) pairs in head-major order, dealt to the eight XCDs in contiguous runs
  // (workgroups go to XCDs round-robin): an XCD's pairs then share few heads, and their key rows
  // stay in its L2 for the two passes over them below
  const int64_t pairs = static_cast<int64_t>(T) * H;
  const int64_t nwg = gridDim.x, per = nwg >> 3, extra = nwg & 7;
  const int64_t xcd = blockIdx.x & 7;
  const int64_t wg = xcd * per + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
  const int64_t q = wg * W + threadIdx.x / kWave;
  if (q >= pairs) return;                             // wave-uniform
  const int h = static_cast<int>(q / T);
  const size_t th = static_cast<size_t>(q % T) * H + h;
  const int R = tucker ? rank : 1;
  bool valid[NG];
  uint32_t key[2][NG];                                 // row, column of each slot
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int s = g * kWave + lane;
    valid[g] = s < m;
    const uint32_t flat = valid[g] ? static_cast<uint32_t>(idx[th * m + s]) : 0u;
    key[0][g] = flat / static_cast<uint32_t>(n);
    key[1][g] = flat % static_cast<uint32_t>(n);
  }
  // ---- weight gradients -> grid-score gradients (SoftMax Jacobian where eq. (3) weights)
  float dg[NG][kMaxCores];
  if (softmax) {
    float p = 0.0f;
#pragma unroll
    for (int g = 0; g < NG; ++g)
      if (valid[g]) p = fmaf(w[th * m + g * kWave + lane], dw[th * m + g * kWave + lane], p);
    const float wdot = wave_sum(p);                    // identical in every lane
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const size_t x = th * m + g * kWave + lane;
      dg[g][0] = valid[g] ? w[x] * (dw[x] - wdot) : 0.0f;
    }
  } else {
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int c = 0; c < kMaxCores; ++c)
        dg[g][c] = valid[g] && c < hc ? dw[(th * m + g * kWave + lane) * hc + c] : 0.0f;
  }
  // ---- distinct keys per axis: a slot leads its key when no earlier slot holds it; pos is the
  // number of leaders before the key's leader
  int first[2][NG], pos[2][NG], nd[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    uint64_t lead[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      int f = -1;
#pragma unroll
      for (int g2 = 0; g2 <= g; ++g2) {
        const uint64_t mm = key_match(key[a][g], key[a][g2], valid[g2], key_bits);
        if (f < 0 && mm != 0ull) f = g2 * kWave + __builtin_ctzll(mm);
      }
      first[a][g] = f;
      lead[g] = __ballot(valid[g] && f == g * kWave + lane);
    }
    int total = 0;
#pragma unroll
    for (int g = 0; g < NG; ++g) total += __popcll(lead[g]);
    nd[a] = total;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int f = valid[g] ? first[a][g] : 0;
      int p = 0;
#pragma unroll
      for (int g2 = 0; g2 < NG; ++g2) {
        if (g2 < f / kWave) p += __popcll(lead[g2]);
        if (g2 == f / kWave) p += __popcll(lead[g2] & ((1ull << (f % kWave)) - 1ull));
      }
      pos[a][g] = p;
      if (valid[g] && f == g * kWave + lane) sh.dist[a][p] = static_cast<int>(key[a][g]);
    }
  }
  wave_lds_order();
  // ---- Tucker: per-slice scores of the distinct keys, four lanes per key row.  The quad is
  // split into one group per slice (4, 2 or 1 lanes for rank 1, 2, 3-4; rank 3 leaves a lane
  // idle); a lane strides its slice's 16-byte pieces by the group width, eight loads in flight,
  // and the group's partial sums meet through DPP in a fixed order.
  float sr[NG][kMaxRank] = {}, sc[NG][kMaxRank] = {};
  if (tucker) {
    constexpr int kPieces = 8;
    const int n4 = dk >> 2, wp = n4 / rank;                   // pieces per row, per slice
    const int part = lane & 3;
    const int ls = rank == 1 ? 2 : (rank == 2 ? 1 : 0);       // log2 lanes per slice
    const int rho = part >> ls, sub = part & ((1 << ls) - 1);
    const int cnt = rho < rank ? (wp - sub + (1 << ls) - 1) >> ls : 0;
    const int first = rho * wp + sub;
    const int jobs = nd[0] + nd[1];
    for (int j0 = 0; j0 < jobs; j0 += kWave / 4) {     // wave-uniform trip count
      const int kk = j0 + lane / 4;
      const bool ok = kk < jobs;                       // uniform across each quad
      const int a = kk >= nd[0] ? 1 : 0;
      const int k = kk - (a ? nd[0] : 0);
      float acc = 0.0f;
      if (ok) {
        const float4* kr = reinterpret_cast<const float4*>(
            (a ? k_col : k_row) + (static_cast<size_t>(h) * n + sh.dist[a][k]) * dk) + first;
        const float4* qr = reinterpret_cast<const float4*>((a ? q_col : q_row) + th * dk) + first;
        for (int i0 = 0; i0 < cnt; i0 += kPieces) {
          float4 kv[kPieces];
#pragma unroll
          for (int i = 0; i < kPieces; ++i)
            if (i0 + i < cnt) kv[i] = kr[(i0 + i) << ls];
#pragma unroll
          for (int i = 0; i < kPieces; ++i)
            if (i0 + i < cnt) {
              const float4 qv = qr[(i0 + i) << ls];
              acc = fmaf(kv[i].x, qv.x, acc);
              acc = fmaf(kv[i].y, qv.y, acc);
              acc = fmaf(kv[i].z, qv.z, acc);
              acc = fmaf(kv[i].w, qv.w, acc);
            }
        }
      }
      // the slice group's sum (every lane takes part)
      if (ls >= 1) acc += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, acc), 0xB1, 0xF, 0xF, false));
      if (ls >= 2) acc += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, acc), 0x4E, 0xF, 0xF, false));
      if (ok && rho < rank && sub == 0) sh.sd[a][k][rho] = acc;
      if (ok && part == 0)
        for (int r = rank; r < kMaxRank; ++r) sh.sd[a][k][r] = 0.0f;
    }
    wave_lds_order();
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int r = 0; r < kMaxRank; ++r) {
        sr[g][r] = valid[g] ? sh.sd[0][pos[0][g]][r] : 0.0f;
        sc[g][r] = valid[g] ? sh.sd[1][pos[1][g]][r] : 0.0f;
      }
  }
  // ---- each slot's dS terms: d score / d s_row = C s_col, d score / d s_col = C^T s_row (eq. (10))
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (!valid[g]) continue;
    const int s = g * kWave + lane;
    if (!tucker) {
      sh.cs[0][s][0] = dg[g][0];
      sh.cs[1][s][0] = dg[g][0];
      continue;
    }
    for (int r = 0; r < rank; ++r) {
      float x0 = 0.0f, x1 = 0.0f;
#pragma unroll
      for (int c = 0; c < kMaxCores; ++c) {
        if (c >= hc) break;
        const float* C = core_all + (static_cast<size_t>(h) * hc + c) * rank * rank;
        float ca = 0.0f, cb = 0.0f;
#pragma unroll
        for (int x = 0; x < kMaxRank; ++x) {
          if (x >= rank) break;
          ca = fmaf(C[r * rank + x], sc[g][x], ca);
          cb = fmaf(C[x * rank + r], sr[g][x], cb);
        }
        x0 = fmaf(dg[g][c], ca, x0);
        x1 = fmaf(dg[g][c], cb, x1);
      }
      sh.cs[0][s][r] = x0;
      sh.cs[1][s][r] = x1;
    }
  }
  // ---- dC partial of this (token, head): sum over slots of dg s_row s_col^T (a wave sum)
  if (tucker) {
    for (int x = 0; x < hc * rank * rank; ++x) {    // wave-uniform
      const int c = x / (rank * rank), r = (x / rank) % rank, z = x % rank;
      float v = 0.0f;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float d = 0.0f, a = 0.0f, b = 0.0f;
#pragma unroll
        for (int cc = 0; cc < kMaxCores; ++cc) d = cc == c ? dg[g][cc] : d;
#pragma unroll
        for (int q = 0; q < kMaxRank; ++q) {
          a = q == r ? sr[g][q] : a;
          b = q == z ? sc[g][q] : b;
        }
        v = fmaf(d, a * b, v);
      }
      v = wave_sum(v);
      if (lane == 0) dc_part[th * hc * rank * rank + x] = v;
    }
  }
  wave_lds_order();
  // ---- dS per distinct key: its slots' terms in slot order, summed by the leading slot
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const bool leads = valid[g] && first[a][g] == g * kWave + lane;
      float acc[kMaxRank] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int g2 = g; g2 < NG; ++g2) {
        uint64_t mm = key_match(key[a][g], key[a][g2], valid[g2], key_bits);
        if (!leads) continue;
        while (mm != 0ull) {
          const int x = g2 * kWave + __builtin_ctzll(mm);
          mm &= mm - 1ull;
#pragma unroll
          for (int r = 0; r < kMaxRank; ++r)
            if (r < R) acc[r] += sh.cs[a][x][r];
        }
      }
      if (leads)
#pragma unroll
        for (int r = 0; r < kMaxRank; ++r) sh.sd[a][pos[a][g]][r] = acc[r];
    }
  wave_lds_order();
  // ---- dq = sum over distinct keys of dS K (eqs. (2) / (4) transposed)
  const int width = dk / R;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const float* Kh = (a ? k_col : k_row) + static_cast<size_t>(h) * n * dk;
    float* dq = (a ? dq_col : dq_row) + th * dk;
    const int nk = nd[a];
    if (dk % 4 == 0 && (dk > 2 * kWave || (dk & (dk - 1)) == 0) &&
        (reinterpret_cast<uintptr_t>(dq) & 15u) == 0) {
      // four dims per lane (16-byte loads); rows of at most 128 dims take S = 64 / (dk / 4) keys
      // per load, lane group s summing keys s, s + S, ... in order, the groups then meeting by a
      // fixed butterfly of shuffles; wider rows go in passes of 256 dims, each lane's sum in key
      // order
      const int G = dk <= 2 * kWave ? dk / 4 : kWave, S = kWave / G;
      const int sub = lane / G;
      for (int d0 = 0; d0 < dk; d0 += 4 * G) {
        const int e = d0 + (lane % G) * 4;
        const bool active = e < dk;
        const int r = active ? e / width : 0;         // four consecutive dims lie in one slice
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < nk; k0 += 4 * S) {      // four 16-byte loads in flight per lane
          f32x4 kv[4];
          float sd[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int k = k0 + S * u + sub;
            const bool ok = active && k < nk;
            kv[u] = ok ? *reinterpret_cast<const f32x4*>(Kh + static_cast<size_t>(sh.dist[a][k]) * dk + e)
                       : f32x4{0.f, 0.f, 0.f, 0.f};
            sd[u] = ok ? sh.sd[a][k][r] : 0.0f;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (k0 + S * u >= nk) break;              // wave-uniform: no key for any group
            acc.x = fmaf(sd[u], kv[u].x, acc.x);
            acc.y = fmaf(sd[u], kv[u].y, acc.y);
            acc.z = fmaf(sd[u], kv[u].z, acc.z);
            acc.w = fmaf(sd[u], kv[u].w, acc.w);
          }
        }
        for (int off = G; off < kWave; off <<= 1) {
          acc.x += __shfl_xor(acc.x, off, kWave);
          acc.y += __shfl_xor(acc.y, off, kWave);
          acc.z += __shfl_xor(acc.z, off, kWave);
          acc.w += __shfl_xor(acc.w, off, kWave);
        }
        if (sub == 0 && active) *reinterpret_cast<f32x4*>(dq + e) = acc;
      }
      continue;
    }
    for (int e = lane; e < dk; e += kWave) {
      const int r = e / width;
      float acc = 0.0f;
      int k = 0;
      for (; k + 8 <= nk; k += 8) {     // eight key loads in flight, the sum still in key order
        float kv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) kv[u] = Kh[static_cast<size_t>(sh.dist[a][k + u]) * dk + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fmaf(sh.sd[a][k + u][r], kv[u], acc);
      }
      for (; k < nk; ++k) acc = fmaf(sh.sd[a][k][r], Kh[static_cast<size_t>(sh.dist[a][k]) * dk + e], acc);
      dq[e] = acc;
    }
  }
  // ---- key-gradient entries: slot ((t H + h) 2 + axis) m + k for the k-th distinct key; the
  // rest of the axis' m slots hold the sentinel, which the sort drops
  const uint32_t sentinel = static_cast<uint32_t>(2 * H) * n;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (!valid[g]) continue;
      const int s = g * kWave + lane;
      const size_t base = (th * 2 + a) * m;
      if (first[a][g] == s) {
        const size_t slot = base + pos[a][g];
        ekeys[slot] = static_cast<uint32_t>((a * H + h) * n) + key[a][g];
        for (int r = 0; r < rank; ++r) edS[slot * rank + r] = sh.sd[a][pos[a][g]][r];
      }
      if (s >= nd[a]) ekeys[base + s] = sentinel;
    }
}

// Key gradients by segments of sorted entries (as the value rows): dK[key] += sum over the
// entries of its run, in order, of dS[entry][slice] q[t, h, :]; pieces cut by a segment store
// their partial row for seg_join_kernel.
__global__ __launch_bounds__(THREADS) void key_bwd_seg_kernel(
    const uint2* __restrict__ sorted, const uint32_t* __restrict__ n_sorted,
    const float* __restrict__ edS, const float* __restrict__ q_row, const float* __restrict__ q_col,
    float* __restrict__ dk_row, float* __restrict__ dk_col, int H, int n, int dk, int rank, int m,
    float* __restrict__ partial, float* __restrict__ heads_part, const uint32_t* __restrict__ list,
    uint32_t* __restrict__ counts, uint32_t* __restrict__ heads) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t n_pieces = counts[0];
  const int M = static_cast<int>(*n_sorted);
  // The pieces (in (axis, head, key) order) are split into eight contiguous ranges, one per XCD
  // (workgroups go to XCDs round-robin), so that an XCD's waves read the query rows of few
  // (axis, head) blocks and find them in its L2.
  const uint32_t xcd = blockIdx.x & 7u, groups = gridDim.x < 8u ? gridDim.x : 8u;
  const uint32_t lo = static_cast<uint32_t>(static_cast<uint64_t>(n_pieces) * xcd / groups);
  const uint32_t hi = static_cast<uint32_t>(static_cast<uint64_t>(n_pieces) * (xcd + 1) / groups);
  const uint32_t xcd_waves = ((gridDim.x - xcd + 7u) >> 3) * NWAVES;   // this XCD's waves
  for (uint32_t pk = lo + (blockIdx.x >> 3) * NWAVES + threadIdx.x / kWave; pk < hi;
       pk += xcd_waves) {
  const int ps = static_cast<int>(list[pk]);
  const uint32_t key = sorted[ps].x;
  const bool run_start = ps == 0 || sorted[ps - 1].x != key;
  bool run_end;
  const int pe = piece_end(sorted, ps, M, key, &run_end);
  if (run_start && !run_end && lane == 0) heads[atomicAdd(counts + 1, 1u)] = pk;
  const int axis = static_cast<int>(key / (static_cast<uint32_t>(H) * n));
  const int rem = static_cast<int>(key - static_cast<uint32_t>(axis) * H * n);
  const int h = rem / n;
  const float* q = axis ? q_col : q_row;
  float* dK = (axis ? dk_col : dk_row) + static_cast<size_t>(rem) * dk;
  const int width = dk / rank;
  const int n_e = pe - ps;
  const uint32_t my_slot = lane < n_e ? sorted[ps + lane].y : 0u;   // one entry per lane
  const bool whole = run_start && run_end;
  float* const part_row = (run_start ? heads_part : partial) + static_cast<size_t>(ps / kSeg) * dk;
  if (dk <= 2 * kWave && (dk & (dk - 1)) == 0) {
    // Rows of at most 128 dims fill a fraction of the wave: G = dk / 4 lanes take one entry, and
    // the wave's S = 64 / G lane groups take entries s, s + S, s + 2 S, ... of the piece, each
    // group in order; the groups' sums then meet by a fixed butterfly of shuffles.
    const int G = dk / 4, S = kWave / G;
    const int sub = lane / G, d = (lane % G) * 4;
    const int r = d / width;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const f32x4 old = (whole && sub == 0) ? *reinterpret_cast<const f32x4*>(dK + d) : f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < n_e; j0 += S * kInFlight) {   // wave-uniform
      f32x4 qv[kInFlight];
      float ds[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {              // all loads first
        const int j = j0 + S * u + sub;
        const size_t slot = static_cast<uint32_t>(__shfl(static_cast<int>(my_slot), min(j, n_e - 1), kWave));
        const size_t t = slot / (static_cast<size_t>(2) * H * m);
        qv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        ds[u] = 0.0f;
        if (j < n_e) {
          qv[u] = *reinterpret_cast<const f32x4*>(q + (t * H + h) * dk + d);
          ds[u] = edS[slot * rank + r];
        }
      }
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {              // then this group's entries in order
        acc.x = fmaf(ds[u], qv[u].x, acc.x);
        acc.y = fmaf(ds[u], qv[u].y, acc.y);
        acc.z = fmaf(ds[u], qv[u].z, acc.z);
        acc.w = fmaf(ds[u], qv[u].w, acc.w);
      }
    }
    for (int off = G; off < kWave; off <<= 1) {
      acc.x += __shfl_xor(acc.x, off, kWave);
      acc.y += __shfl_xor(acc.y, off, kWave);
      acc.z += __shfl_xor(acc.z, off, kWave);
      acc.w += __shfl_xor(acc.w, off, kWave);
    }
    if (sub == 0) {
      if (whole) *reinterpret_cast<f32x4*>(dK + d) = old + acc;
      else *reinterpret_cast<f32x4*>(part_row + d) = acc;
    }
    continue;
  }
  for (int d0 = 0; d0 < dk; d0 += kWave * 4) {
    const int d = d0 + lane * 4;
    const bool active = d < dk;
    const int r = active ? d / width : 0;             // four consecutive dims lie in one slice
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // a whole run adds into its key's gradient row: read it now, under the entries' loads
    const f32x4 old = (active && whole) ? *reinterpret_cast<const f32x4*>(dK + d) : f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < n_e; j0 += 2 * kInFlight) {  // wave-uniform
      f32x4 qv[2 * kInFlight];
      float ds[2 * kInFlight];
#pragma unroll
      for (int u = 0; u < 2 * kInFlight; ++u) {      // all loads first
        const size_t slot = static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(my_slot), min(j0 + u, n_e - 1)));
        const size_t t = slot / (static_cast<size_t>(2) * H * m);
        qv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        ds[u] = 0.0f;
        if (active && j0 + u < n_e) {                 // (past the piece's end: no loads)
          qv[u] = *reinterpret_cast<const f32x4*>(q + (t * H + h) * dk + d);
          ds[u] = edS[slot * rank + r];
        }
      }
#pragma unroll
      for (int u = 0; u < 2 * kInFlight; ++u) {      // then the entries in order
        if (j0 + u >= n_e) break;
        acc.x = fmaf(ds[u], qv[u].x, acc.x);
        acc.y = fmaf(ds[u], qv[u].y, acc.y);
        acc.z = fmaf(ds[u], qv[u].z, acc.z);
        acc.w = fmaf(ds[u], qv[u].w, acc.w);
      }
    }
    if (!active) continue;
    if (whole) *reinterpret_cast<f32x4*>(dK + d) = old + acc;
    else *reinterpret_cast<f32x4*>(part_row + d) = acc;
  }
  }
}

// out[c] += sum over the R rows of in[.][c]: one workgroup per column, thread i adding rows i,
// i + 256, ... in order, then a fixed tree over the threads.
__global__ __launch_bounds__(THREADS) void sum_cols_kernel(const float* __restrict__ in,
                                                           float* __restrict__ out, int R, int C) {
  __shared__ float red[THREADS];
  const int c = blockIdx.x, tid = threadIdx.x;
  float a = 0.0f;
  for (int j = tid; j < R; j += THREADS) a += in[static_cast<size_t>(j) * C + c];
  red[tid] = a;
  __syncthreads();
  for (int off = THREADS / 2; off > 0; off >>= 1) {
    if (tid < off) red[tid] += red[tid + off];
    __syncthreads();
  }
  if (tid == 0) out[c] += red[0];
}

size_t round_up256(size_t x) { return (x + 255) / 256 * 256; }

int bits_for(int64_t n) {
  int b = 0;
  while (b < 31 && (INT64_C(1) << b) < n) ++b;
  return b;
}

}  // namespace

// [entry info: M words][segment heads][counts][chunk counts][partial rows][as many again: the heads'
// partial rows (dense form) or d_pooled by column slice (compact form)][sort: its pairs, the dead half of which holds the entries' records, and
// M spare words, which hold the piece list: runs of several entries alone are cut into pieces, at
// most M / 2 + nseg of them]
size_t gather_backward_workspace_bytes(int T, int bag, int dv) {
  const int M = T * bag;
  if (M == 0) return 0;
  const size_t nseg = (static_cast<size_t>(M) + kSeg - 1) / kSeg;
  return round_up256(static_cast<size_t>(M) * sizeof(uint32_t)) + round_up256(nseg * sizeof(uint32_t)) +
         256 + round_up256(list_chunks(M) * sizeof(uint2)) +
         2 * round_up256(nseg * dv * sizeof(float)) + round_up256(sort_workspace_bytes(M));
}

namespace {

template <typename Elem>
hipError_t launch_tokens(const Elem* values, uint32_t n_values, int dv, int T, int bag,
                         const int32_t* idx, const float* w, const int32_t* perm, int expand, int cores,
                         const float* d_pooled, const uint32_t* info, float* d_rows, bool dense,
                         float* dw, float* sliced, int slice_cols, const uint32_t* counts, RowRule rule,
                         hipStream_t s) {
  const int chunks = dv * static_cast<int>(sizeof(Elem)) / 16;
  const size_t lds = static_cast<size_t>(NWAVES) * cores * kWave * 4 + static_cast<size_t>(bag) * 12;
  const dim3 block(THREADS);
  // few tokens: several workgroups share a bag, until the launch has its waves or a group of waves
  // would fall below four entries
#define UMEM_TOKENS_AS(LL, CC, CW, SLICED, DENSE)                                                  \
  hipLaunchKernelGGL((token_bwd_kernel<Elem, LL, CC, CW, SLICED, DENSE>), grid, block, lds, s, values, \
                     dv, bag, idx, w, perm, n_values, expand, cores, d_pooled, info, d_rows, dw,  \
                     sliced, slice_cols, counts, rule)
#define UMEM_TOKENS(LL, CC, CW)                                                                   \
  do {                                                                                            \
    int split = 1;                                                                                \
    while (T * NWAVES * split < kTokenWaves && bag * CW >= 4 * NWAVES * 2 * split) split *= 2;    \
    const dim3 grid(T, split);                                                                    \
    constexpr bool SL = LL == kWave;                                                              \
    if (dense) UMEM_TOKENS_AS(LL, CC, CW, false, true);                                           \
    else if (SL && sliced != nullptr) UMEM_TOKENS_AS(LL, CC, CW, SL, false);                      \
    else UMEM_TOKENS_AS(LL, CC, CW, false, false);                                                \
  } while (0)
  switch (chunks) {
    case 1: UMEM_TOKENS(1, 1, 1); break;
    case 2: UMEM_TOKENS(2, 1, 1); break;
    case 4: UMEM_TOKENS(4, 1, 1); break;
    case 8: UMEM_TOKENS(8, 1, 1); break;
    case 16: UMEM_TOKENS(16, 1, 1); break;
    case 32: UMEM_TOKENS(32, 1, 1); break;
    case 64: UMEM_TOKENS(64, 1, 1); break;
    case 128: UMEM_TOKENS(64, 2, 1); break;
    case 192: UMEM_TOKENS(64, 3, 1); break;
    case 256: UMEM_TOKENS(64, 2, 2); break;
    case 320: UMEM_TOKENS(64, 5, 1); break;
    case 384: UMEM_TOKENS(64, 3, 2); break;
    case 448: UMEM_TOKENS(64, 7, 1); break;
    case 512: UMEM_TOKENS(64, 2, 4); break;
    default: return hipErrorInvalidValue;
  }
#undef UMEM_TOKENS
#undef UMEM_TOKENS_AS
  return hipGetLastError();
}

// The runs of several entries.  slices: RowRule's forms may differ between dense and compact form; cols: the
// columns that row_walk takes at a time; a wave's share of a wide row's chunks as launch_tokens deals them.
template <typename Elem>
hipError_t launch_rows(const RowArgs& A, const Elem* values, int M, bool slices, int cols, RowRule rule,
                       hipStream_t s) {
  const dim3 grid(kRowWaves / NWAVES), block(THREADS);
  const int chunks = A.dv * static_cast<int>(sizeof(Elem)) / 16;
  const int cpl = chunks == 256 ? 2 : chunks == 384 ? 3 : chunks == 512 ? 2 : chunks / kWave;
#define UMEM_NARROW(GL) hipLaunchKernelGGL(row_bwd_narrow_kernel<GL>, grid, block, 0, s, A)
#define UMEM_ROWS(S, GL)                                                                          \
  do {                                                                                            \
    if (slices) {                                                                                 \
      hipLaunchKernelGGL((row_bwd_dots_kernel<Elem, S>), grid, block, 0, s, A, values, cpl, rule); \
      hipLaunchKernelGGL(row_bwd_sliced_kernel<GL>, grid, block, 0, s, A, rule);                  \
    } else {                                                                                      \
      hipLaunchKernelGGL((row_bwd_kernel<Elem, GL>), grid, block, 0, s, A, values, cpl, rule);    \
    }                                                                                             \
  } while (0)
  if (chunks >= kWave && M > kTinyCall) {
    switch (cols) {
      case 32: UMEM_ROWS(8, 8); break;
      case 64: UMEM_ROWS(4, 16); break;
      case 128: UMEM_ROWS(2, 32); break;
      default: UMEM_ROWS(1, 64); break;
    }
  } else if (chunks >= kWave) {
    UMEM_NARROW(64);
  } else {
    switch (A.dv / 4) {                                     // dv a power of two
      case 1: UMEM_NARROW(1); break;
      case 2: UMEM_NARROW(2); break;
      case 4: UMEM_NARROW(4); break;
      case 8: UMEM_NARROW(8); break;
      case 16: UMEM_NARROW(16); break;
      case 32: UMEM_NARROW(32); break;
      case 64: UMEM_NARROW(64); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef UMEM_ROWS
#undef UMEM_NARROW
  return hipGetLastError();
}

// Columns of row_bwd_kernel's slices (dv a multiple of 256): a multiple of eight slices of 32 to 256
// columns, as wide as leaves each XCD no more than kSliceBytes of d_pooled to keep in its 4 MiB L2
// at a time.
constexpr int64_t kSliceBytes = 9 << 19;
int slice_columns(int64_t pooled_rows, int dv) {
  int cols = 32;
  while (cols < 256 && dv % (16 * cols) == 0 && pooled_rows * 2 * cols * 4 <= kSliceBytes) cols *= 2;
  return cols;
}

}  // namespace

// rows_out == nullptr: d_values is the dense [n_values, dv] gradient, added into.  Otherwise the
// compact form: d_values is [T * bag, dv], row r the gradient of rows_out[r], the r-th distinct
// row (ascending), and *n_rows the number of distinct rows.
hipError_t launch_gather_backward(int64_t n_values, int dv, int vdtype, const void* values, int T,
                                  int bag, const int32_t* idx, const float* w, const int32_t* perm,
                                  int expand, int cores, const float* d_pooled, float* d_values,
                                  float* dw, int32_t* rows_out, int32_t* n_rows, void* ws,
                                  hipStream_t s) {
  clear_stale_error();
  const int M = T * bag;
  if (M == 0) return hipSuccess;
  char* base = static_cast<char*>(ws);
  uint32_t* info = reinterpret_cast<uint32_t*>(base);
  base += round_up256(static_cast<size_t>(M) * sizeof(uint32_t));
  const size_t nseg = (static_cast<size_t>(M) + kSeg - 1) / kSeg;
  uint32_t* heads = reinterpret_cast<uint32_t*>(base);
  base += round_up256(nseg * sizeof(uint32_t));
  uint32_t* counts = reinterpret_cast<uint32_t*>(base);
  base += 256;
  uint2* chunk_cnt = reinterpret_cast<uint2*>(base);
  base += round_up256(list_chunks(M) * sizeof(uint2));
  float* partial = reinterpret_cast<float*>(base);
  base += round_up256(nseg * dv * sizeof(float));
  float* const heads_part = reinterpret_cast<float*>(base);
  float* sliced = heads_part;
  base += round_up256(nseg * dv * sizeof(float));
  const SortPlan sp = sort_plan(M, bits_for(n_values), base);
  const int32_t* pm = expand > 1 ? perm : nullptr;
  const uint32_t nv = static_cast<uint32_t>(n_values);              // at most 2^31
  const int c = cores > 1 ? cores : 1;
  const bool compact = rows_out != nullptr;
  hipLaunchKernelGGL(bwd_keys_kernel, dim3(sp.tiles), dim3(kSortThreads), 0, s, idx, pm, nv, bag, expand,
                     info, sp);
  uint2 *sorted, *rec;
  uint32_t* list = sp.spare;
  // (row indices are below 2^31: no key is skipped)
  hipError_t e = sort_run(sp, 0xFFFFFFFFu, true, s, &sorted, &rec);
  if (e != hipSuccess) return e;
  const RowInfo ri{info, rec, c == 1 ? w : nullptr, rows_out, n_rows};
  hipLaunchKernelGGL(piece_count_kernel<true>, dim3(list_chunks(M)), dim3(THREADS), 0, s, sorted, sp.n,
                     chunk_cnt);
  hipLaunchKernelGGL(piece_write_kernel<true>, dim3(list_chunks(M)), dim3(THREADS), 0, s, sorted, sp.n,
                     chunk_cnt, list, counts, ri);
  // rows repeat from a quarter as many entries as rows on (the gather's rule for cached loads).  The
  // copy by column slice pays where rows repeat and d_pooled is beyond an L2; it needs rows of 64
  // lanes (1 KiB) and room beside the partial rows (which the dense form's heads take)
  const bool keep = 4 * static_cast<int64_t>(M) >= n_values;
  const int64_t pooled_rows = static_cast<int64_t>(T) * expand;
  const bool slices = keep && M > kTinyCall && dv * (vdtype == UMEM_F32 ? 4 : 2) >= 1024 && pooled_rows <= static_cast<int64_t>(nseg) &&
                      pooled_rows * dv * 4 > (INT64_C(4) << 20);
  if (!(slices && compact)) sliced = nullptr;
  // Where one form may take the other kernel than the other form, both add in the same groups of entries:
  // the same sums, bit for bit.
  const int cols = slice_columns(pooled_rows, dv);
  // (with several cores the walk by slices gathers an entry's weight anew for every slice: 4,096 tokens of 256
  // entries on 7,600 rows of 1 KiB, two cores, 548 us, by row_dot 424)
  const RowRule rule{M <= kTinyCall ? ~0u : sliced == nullptr || c > 1 ? 0u : kFewBytes / (static_cast<uint32_t>(dv) * (vdtype == UMEM_F32 ? 4 : 2)),
                     static_cast<uint32_t>(M)};
  e = vdtype == UMEM_F32
          ? launch_tokens(static_cast<const float*>(values), nv, dv, T, bag, idx, w, pm, expand, c,
                          d_pooled, info, d_values, !compact, dw, sliced, cols, counts, rule, s)
          : launch_tokens(static_cast<const uint16_t*>(values), nv, dv, T, bag, idx, w, pm, expand, c,
                          d_pooled, info, d_values, !compact, dw, sliced, cols, counts, rule, s);
  if (e != hipSuccess) return e;
  const RowArgs ra{sorted, sp.n, rec, info, list, counts, heads, w, c, dv, compact ? 1 : 0,
                   static_cast<size_t>(pooled_rows), d_pooled, sliced, d_values, dw, partial, heads_part};
  e = vdtype == UMEM_F32 ? launch_rows(ra, static_cast<const float*>(values), M, slices, cols, rule, s)
                         : launch_rows(ra, static_cast<const uint16_t*>(values), M, slices, cols, rule, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(seg_join_kernel, dim3(kJoinWaves / NWAVES), dim3(THREADS), 0, s, sorted, sp.n, dv,
                     partial, heads_part, d_values, list, heads, counts, 0, 0, nullptr, compact ? info : nullptr);
  return hipGetLastError();
}

size_t score_backward_workspace_bytes(const umem_desc& d, int T) {
  if (T == 0) return 0;
  const size_t th = static_cast<size_t>(T) * d.heads;
  const int Mk = static_cast<int>(th * 2 * d.topm);
  const int hc = d.cores > 1 ? d.cores : 1;
  const size_t dc = d.grid == UMEM_GRID_TUCKER ? static_cast<size_t>(hc) * d.rank * d.rank : 0;
  const size_t nseg = (static_cast<size_t>(Mk) + kSeg - 1) / kSeg;
  return round_up256(nseg * sizeof(uint32_t)) + 256 + round_up256(list_chunks(Mk) * sizeof(uint2)) +
         round_up256(static_cast<size_t>(Mk) * d.rank * sizeof(float)) +
         2 * round_up256(nseg * d.dk * sizeof(float)) + round_up256(th * dc * sizeof(float)) +
         round_up256(sort_workspace_bytes(Mk));
}

hipError_t launch_score_backward(const umem_desc& d, int T, const float* q_row, const float* q_col,
                                 const float* k_row, const float* k_col, const float* core,
                                 const int32_t* idx, const float* w, const float* dw,
                                 float* dq_row, float* dq_col, float* dk_row, float* dk_col,
                                 float* dcore, void* ws, hipStream_t s) {
  clear_stale_error();
  if (T == 0) return hipSuccess;
  const int H = d.heads, m = d.topm, r = d.rank;
  const size_t th = static_cast<size_t>(T) * H;
  const int Mk = static_cast<int>(th * 2 * m);
  const bool tucker = d.grid == UMEM_GRID_TUCKER;
  const int hc = d.cores > 1 ? d.cores : 1;
  const int dc = tucker ? hc * r * r : 0;
  char* base = static_cast<char*>(ws);
  float* edS = reinterpret_cast<float*>(base);
  base += round_up256(static_cast<size_t>(Mk) * r * sizeof(float));
  const size_t nseg = (static_cast<size_t>(Mk) + kSeg - 1) / kSeg;
  float* kpart = reinterpret_cast<float*>(base);
  base += round_up256(nseg * d.dk * sizeof(float));
  float* kheads = reinterpret_cast<float*>(base);
  base += round_up256(nseg * d.dk * sizeof(float));
  uint32_t* heads = reinterpret_cast<uint32_t*>(base);
  base += round_up256(nseg * sizeof(uint32_t));
  uint32_t* counts = reinterpret_cast<uint32_t*>(base);
  base += 256;
  uint2* chunk_cnt = reinterpret_cast<uint2*>(base);
  base += round_up256(list_chunks(Mk) * sizeof(uint2));
  float* dc_part = reinterpret_cast<float*>(base);
  base += round_up256(th * dc * sizeof(float));
  const uint32_t sentinel = static_cast<uint32_t>(2 * H) * d.n_keys;
  const SortPlan sp = sort_plan(Mk, bits_for(sentinel), base);
  const int key_bits = bits_for(d.n_keys);
  const int sm = d.weight == UMEM_W_SOFTMAX ? 1 : 0;
#define UMEM_SCORE_BWD(NG)                                                                       \
  hipLaunchKernelGGL(score_bwd_kernel<NG>,                                                      \
                     dim3(static_cast<unsigned>((th + score_bwd_waves<NG>() - 1) / score_bwd_waves<NG>())), \
                     dim3(score_bwd_waves<NG>() * kWave), 0, s, q_row, q_col, k_row, k_col, core, \
                     idx, w, dw, T, H, d.n_keys, key_bits, d.dk, r, m, tucker ? 1 : 0, sm, hc,   \
                     dq_row, dq_col, sp.keys, edS, dc_part)
  if (m <= kWave) UMEM_SCORE_BWD(1);
  else if (m <= 2 * kWave) UMEM_SCORE_BWD(2);
  else UMEM_SCORE_BWD(4);
#undef UMEM_SCORE_BWD
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  uint2 *sorted, *dead;
  e = sort_run(sp, sentinel, false, s, &sorted, &dead);
  uint32_t* list = reinterpret_cast<uint32_t*>(dead);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(piece_count_kernel<false>, dim3(list_chunks(Mk)), dim3(THREADS), 0, s, sorted,
                     sp.n, chunk_cnt);
  hipLaunchKernelGGL(piece_write_kernel<false>, dim3(list_chunks(Mk)), dim3(THREADS), 0, s, sorted,
                     sp.n, chunk_cnt, list, counts, RowInfo{});
  hipLaunchKernelGGL(key_bwd_seg_kernel, dim3(kListWaves / NWAVES), dim3(THREADS), 0, s, sorted, sp.n,
                     edS, q_row, q_col, dk_row, dk_col, H, d.n_keys, d.dk, r, m, kpart, kheads, list, counts,
                     heads);
  hipLaunchKernelGGL(seg_join_kernel, dim3(kJoinWaves / NWAVES), dim3(THREADS), 0, s, sorted, sp.n,
                     d.dk, kpart, kheads, dk_row, list, heads, counts, H, d.n_keys, dk_col, nullptr);
  if (tucker)   // dC: the per-token partials [T][H dc], summed over tokens into dcore
    hipLaunchKernelGGL(sum_cols_kernel, dim3(H * dc), dim3(THREADS), 0, s, dc_part, dcore, T, H * dc);
  return hipGetLastError();
}

}  // namespace umem
