// a3 + a4 + a5: per-axis top-k, grid scores of the candidates, global top-m and weights.
//
// One workgroup of eight waves per (token, head): waves 0-3 select on the row axis and waves
// 4-7 on the column axis, at the same time.  Every selection is exact under the order
// (score desc, index asc), in three steps:
//
//  1. Threshold.  Each thread holds its elements in registers and takes their maximum; the
//     maxima of four threads are merged per lane, and L is the largest value whose low 16 key
//     bits are zero such that at least k of those 64 merged maxima are >= L (8 radix-4 steps of
//     ballots, which each wave of the axis runs for itself).  They are maxima of disjoint sets, so at least k elements are >= L:
//     the whole top-k is >= L.
//  2. Survivors {x >= L} (typically a few dozen) are compacted into LDS: a DPP wave scan places
//     them within the wave's range, which one LDS atomic reserves (the ranks below do not depend
//     on the order of the ranges, so the result is deterministic).
//  3. A survivor's rank is the number of survivors ordered before it, counted by P threads per
//     survivor (as many as the group has to spare) and summed over those lanes; ranks < k are
//     the answer, already sorted.
//  If an axis's survivors overflow their buffer (massive ties), an exact threshold search over
//  all elements of the axis (32 steps of group-wide counts) takes over.
//
// Additive grid (eq. (3)): with both axis lists sorted, candidate (a, b) (a-th best row, b-th
// best column) is preceded in the order by the (a+1)(b+1)-1 candidates (a' <= a, b' <= b), so
// only (a+1)(b+1) <= m can reach the top-m.  Candidate scores are summed in fp64, where the sum
// of two fp32 scores is exact (or monotone), so this dominance holds.  Further, for r <= k rows
// and c = ceil(m / r) <= k columns the r x c corner of the grid holds at least m pairs, all
// scoring >= A[r-1] + B[c-1]: theta, the largest such bound over r, is <= the m-th best score,
// and only candidates >= theta are ranked (typically a third of them).
// For the forward without expansion (at most two heads, rows of 1 or 2 KiB) the workgroup also
// pools its m rows (eq. (1)) and adds them into the token's output: the decode path then needs
// no separate gather launch.
// With multi-core scoring (eqs. (16), (17)) the selection runs on the summed core and, for the
// m selected slots, each component core's exact score is computed (fp64) as its weight.
// Tucker grid (eq. (10)): all k*k candidates, the exact per-slice scores recomputed for the
// selected keys, candidate scores in fp64; the threshold of step 1 runs on their fp32 roundings
// (rounding is monotone, so the survivors still contain the top-m) and the ranks on fp64.
#include "umem_internal.h"

namespace umem {
namespace {

constexpr int THREADS = 512;
constexpr int NWAVES = THREADS / kWave;
constexpr int GROUP = 256;          // threads per axis
constexpr int SMAX_AX = 512;        // survivors per axis
constexpr int SMAX_S = 512;         // grid survivors (Tucker)
constexpr int KK_MAX = 4096;        // Tucker: k*k candidates
constexpr int ADD_MAX = 2048;       // additive candidates (a+1)(b+1) <= m, a, b < k
constexpr int CPT = KK_MAX / THREADS;   // Tucker candidates per thread

// Kernel variants: kModePool pools the value rows when given them and takes the grid from its
// argument; its row loads in flight take many registers.  kModeAdd and kModeTucker never pool
// and are specialised to one grid: fewer registers, more workgroups per CU for many tokens.
constexpr int kModePool = 0, kModeAdd = 1, kModeTucker = 2;

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SelectShared {
  uint32_t mx[THREADS];               // thread maxima (both axes, or the grid)
  int wave_tot[NWAVES];
  int ax_cnt[2];                      // survivors of each axis (LDS-atomic ranges per wave)
  uint32_t thr[2];
  int32_t ax_idx[2][kMaxTopK];        // axis top-k, sorted by (score desc, index asc)
  float ax_sc[2][kMaxTopK];
  int grid_cnt;                       // additive grid: candidates kept for ranking
  int grid_total;                     // additive grid: (a+1)(b+1) <= m candidates
  uint16_t grid_ab[ADD_MAX];          // ... their (a << 8) | b, row by row
  uint8_t th_col[kMaxTopK + 1];       // ceil(m / r) for the corner bound of r rows (0: beyond k)
  float s_ex[2][kMaxRank][kMaxTopK];  // Tucker: exact per-slice scores of the selected keys
  double p_col[kMaxRank][kMaxTopK];   // Tucker: (C S_col)[rho, b] in fp64
  double core[kMaxRank * kMaxRank];              // Tucker: the core (sum of its components)
  float core_parts[kMaxCores][kMaxRank * kMaxRank];   // multi-core scoring: the components
  int32_t out_ab[kMaxTopM];                      // Tucker: (a << 8) | b of each selected slot
  float w_core[kMaxTopM * kMaxCores];            // multi-core scoring: weights [m][cores]
  int32_t out_flat[kMaxTopM];         // final top-m, by rank
  double out_g[kMaxTopM];
  float e[kMaxTopM];
  float esum;
};

__device__ __forceinline__ uint64_t order_key64(double x) {
  if (x != x) return 0ull;
  if (x == 0.0) x = 0.0;                      // -0.0 ranks as +0.0
  const uint64_t u = static_cast<uint64_t>(__double_as_longlong(x));
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ __forceinline__ double key64_value(uint64_t k) {
  const uint64_t raw = (k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k;
  return __longlong_as_double(static_cast<long long>(raw));
}

// Composite key of an axis element: larger = earlier in (score desc, index asc).
__device__ __forceinline__ uint64_t axis_comp(uint32_t key, int idx) {
  return (static_cast<uint64_t>(key) << 32) |
         static_cast<uint64_t>(0xFFFFFFFFu - static_cast<uint32_t>(idx));
}

// Inclusive prefix sum over the 64 lanes of a wave (DPP row shifts and row broadcasts).
__device__ __forceinline__ int wave_scan_dpp(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return x;
}

// Maximum of a 64-bit value over the 64 lanes of a wave (DPP row shifts and row broadcasts on
// both halves; lanes outside a step's source read 0, the identity), returned to every lane.
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t x) {
#define UMEM_MAX_STEP(CTRL, ROWS, BC)                                                        \
  {                                                                                          \
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(x), CTRL, ROWS, 0xF, BC);  \
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(x >> 32), CTRL, ROWS, 0xF, BC); \
    const uint64_t y = (static_cast<uint64_t>(hi) << 32) | lo;                               \
    x = y > x ? y : x;                                                                       \
  }
  UMEM_MAX_STEP(0x111, 0xF, true)    // row_shr:1
  UMEM_MAX_STEP(0x112, 0xF, true)    // row_shr:2
  UMEM_MAX_STEP(0x114, 0xF, true)    // row_shr:4
  UMEM_MAX_STEP(0x118, 0xF, true)    // row_shr:8
  UMEM_MAX_STEP(0x142, 0xA, false)   // row_bcast:15
  UMEM_MAX_STEP(0x143, 0xC, false)   // row_bcast:31
#undef UMEM_MAX_STEP
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(x), kWave - 1);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(x >> 32), kWave - 1);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Sum over aligned groups of 2^lp consecutive lanes (every lane of a group gets the sum): the
// quad swaps, the half-row and row mirrors of DPP, then shuffles across rows.
__device__ __forceinline__ int group_sum(int r, int lp) {
  if (lp >= 1) r += __builtin_amdgcn_update_dpp(0, r, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
  if (lp >= 2) r += __builtin_amdgcn_update_dpp(0, r, 0x4E, 0xF, 0xF, false);   // quad_perm 2,3,0,1
  if (lp >= 3) r += __builtin_amdgcn_update_dpp(0, r, 0x141, 0xF, 0xF, false);  // row_half_mirror
  if (lp >= 4) r += __builtin_amdgcn_update_dpp(0, r, 0x140, 0xF, 0xF, false);  // row_mirror
  if (lp >= 5) r += __shfl_xor(r, 16, kWave);
  if (lp >= 6) r += __shfl_xor(r, 32, kWave);
  return r;
}

// The same for floats (IEEE addition commutes, so every lane of a group gets the same bits).
__device__ __forceinline__ float group_sum_f(float x, int lp) {
  int r = __builtin_bit_cast(int, x);
#define UMEM_FSTEP(CTRL) \
  r = __builtin_bit_cast(int, __builtin_bit_cast(float, r) + \
                         __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, r, CTRL, 0xF, 0xF, false)))
  if (lp >= 1) UMEM_FSTEP(0xB1);
  if (lp >= 2) UMEM_FSTEP(0x4E);
  if (lp >= 3) UMEM_FSTEP(0x141);
  if (lp >= 4) UMEM_FSTEP(0x140);
#undef UMEM_FSTEP
  return __builtin_bit_cast(float, r);
}

// Exclusive offset of each thread's count within waves [w0, w0 + nw), and their total.
// Called by every thread of the workgroup (it holds two barriers).
__device__ __forceinline__ int2 group_offsets(int cnt, int w0, int nw, SelectShared& sh) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int incl = wave_scan_dpp(cnt);
  if (lane == kWave - 1) sh.wave_tot[wave] = incl;
  __syncthreads();
  int base = 0, total = 0;
  for (int w = w0; w < w0 + nw; ++w) {
    const int tw = sh.wave_tot[w];
    base += (w < wave) ? tw : 0;
    total += tw;
  }
  __syncthreads();
  return make_int2(base + incl - cnt, total);
}

// Largest L with zero low 16 bits such that at least k of the wave's 64 G values v[] are
// >= L (k <= 64 G): eight radix-4 steps, each of three independent ballots.
template <int G>
__device__ __forceinline__ uint32_t wave_kth_largest16(const uint32_t (&v)[G], int k) {
  uint32_t p = 0u;
  for (int b = 30; b >= 16; b -= 2) {
    const uint32_t c1 = p | (1u << b), c2 = p | (2u << b), c3 = p | (3u << b);
    int n1 = 0, n2 = 0, n3 = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      n1 += __popcll(__ballot(v[g] >= c1));
      n2 += __popcll(__ballot(v[g] >= c2));
      n3 += __popcll(__ballot(v[g] >= c3));
    }
    p = n3 >= k ? c3 : (n2 >= k ? c2 : (n1 >= k ? c1 : p));
  }
  return p;
}

// A valid threshold for a top-k from V maxima per lane (maxima of disjoint sets) in LDS:
// lane-wise they are merged into G = ceil(k / 32) (at most V) maxima of unions (still disjoint
// sets), and L, the k-th largest of those 64 G values with its low 16 bits cleared, has at
// least k elements >= L.  With at least two groups per wanted element L stays close to the
// k-th largest element (with one, it falls to the best of the worst group).  One wave.
template <int V>
__device__ __forceinline__ uint32_t threshold_from_maxima(const uint32_t* vals, int k) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t v[V];
#pragma unroll
  for (int q = 0; q < V; ++q) v[q] = vals[lane + kWave * q];
  if (k <= kWave / 2) {
    uint32_t r[1] = {0u};
#pragma unroll
    for (int q = 0; q < V; ++q) r[0] = max(r[0], v[q]);
    return wave_kth_largest16<1>(r, k);
  }
  if (V >= 4 && k <= kWave) {
    uint32_t r[2] = {0u, 0u};
#pragma unroll
    for (int q = 0; q < V; ++q) r[q & 1] = max(r[q & 1], v[q]);
    return wave_kth_largest16<2>(r, k);
  }
  uint32_t r[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int q = 0; q < V; ++q) r[q & 3] = max(r[q & 3], v[q]);
  return wave_kth_largest16<4>(r, k);
}

// ---------------------------------------------------------------- per-axis top-k

// Element i of an axis is held by thread g of its group (g = threadIdx.x % 256) as key[j]:
// VEC == 4 (n % 4 == 0): i = 1024 j + 4 g + e, key[4 j + e]; VEC == 1: i = 256 j + g.
template <int VEC>
__device__ __forceinline__ int elem_index(int g, int j, int e) {
  return VEC == 4 ? 1024 * j + 4 * g + e : GROUP * j + g;
}

// Rank the S survivors of one axis in comp[0, S) with the axis's 256 threads: P = 2^lp threads
// per survivor (consecutive lanes), each counting the survivors before it among every P-th
// entry; ranks < k go to the axis list.
__device__ __forceinline__ void rank_axis(const uint64_t* comp, int S, int axis, int k, int g,
                                          SelectShared& sh) {
  int lp = 0;
  while (lp < 6 && (S << (lp + 1)) <= GROUP) ++lp;
  const int P = 1 << lp;
  for (int base = 0; base < (S << lp); base += GROUP) {
    const int slot = base + g;
    const int e = slot >> lp, part = slot & (P - 1);
    uint64_t me = 0ull;
    int r = 0;
    if (e < S) {
      me = comp[e];
      int u = part;
      for (; u + 3 * P < S; u += 4 * P) {
        const uint64_t b0 = comp[u], b1 = comp[u + P], b2 = comp[u + 2 * P], b3 = comp[u + 3 * P];
        r += static_cast<int>(b0 > me) + static_cast<int>(b1 > me) + static_cast<int>(b2 > me) +
             static_cast<int>(b3 > me);
      }
      for (; u < S; u += P) r += comp[u] > me;
    }
    r = group_sum(r, lp);
    if (part == 0 && e < S && r < k) {
      sh.ax_idx[axis][r] = static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(me & 0xFFFFFFFFull));
      sh.ax_sc[axis][r] = key32_value(static_cast<uint32_t>(me >> 32));
    }
  }
}

// The additive grid's corner bound as a limit of its candidates.  +inf on one axis with -inf on the other is
// NaN, below the corners that it stands before; those are -inf then (or NaN), and as a bound -inf may leave fewer
// than m candidates: all are kept.
__device__ __forceinline__ uint64_t additive_limit(uint64_t th) {
  constexpr uint64_t kNegInf = 0x000FFFFFFFFFFFFFull;     // order_key64(-inf)
  return th > kNegInf ? th : 0ull;
}

// The additive grid's candidates (a+1)(b+1) <= m as a table, row by row, and ceil(m / r) for
// the corner bound; one wave, while the score loads are in flight.
__device__ __forceinline__ void additive_tables(int k, int m, SelectShared& sh) {
  const int lane = threadIdx.x & (kWave - 1);
  const int R = min(k, m);
  int carry = 0;
  for (int a0 = 0; a0 < R; a0 += kWave) {
    const int a = a0 + lane;
    const int len = a < R ? min(k, m / (a + 1)) : 0;
    const int first = carry + wave_scan_dpp(len) - len;
    for (int b = 0; b < len; ++b) sh.grid_ab[first + b] = static_cast<uint16_t>((a << 8) | b);
    if (a < R) {
      const int c = (m + a) / (a + 1);                   // ceil(m / r), r = a + 1
      sh.th_col[a + 1] = static_cast<uint8_t>(c <= k ? c : 0);
    }
    carry = __shfl(first + len, kWave - 1, kWave);   // first already counts the earlier rows
  }
  if (lane == 0) sh.grid_total = carry;
}

// MODE only gives each kernel variant its own copy (with a single caller, the inliner treats it
// as it would in a single-variant build).
template <int NV, int VEC, int MODE>
__device__ void select_axes(const float* __restrict__ sel, int T, int H, int t, int h, int n, int k,
                            int m, bool tables, uint64_t* comp_all, SelectShared& sh) {
  constexpr int NE = NV * VEC;
  const int tid = threadIdx.x;
  const int axis = tid / GROUP;
  const int g = tid % GROUP;
  const int lane = tid & (kWave - 1);
  const float* src = sel + ((static_cast<size_t>(axis) * T + t) * H + h) * n;
  uint64_t* comp = comp_all + axis * SMAX_AX;
  uint32_t key[NE];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    // the scores are read nontemporally: they stream through once (the keys the Tucker grid
    // reads back should stay in L2), and they were written from other XCDs (measured at decode:
    // 10.32 -> 10.06 us against plain loads)
    if (VEC == 4) {
      const f32x4* p = reinterpret_cast<const f32x4*>(src + min(1024 * j + 4 * g, n - 4));
      const f32x4 v = __builtin_nontemporal_load(p);
      key[4 * j + 0] = order_key(v.x);
      key[4 * j + 1] = order_key(v.y);
      key[4 * j + 2] = order_key(v.z);
      key[4 * j + 3] = order_key(v.w);
    } else {
      const float* p = src + min(GROUP * j + g, n - 1);
      key[j] = order_key(__builtin_nontemporal_load(p));
    }
  }
  if (tables && tid < kWave) additive_tables(k, m, sh);
  uint32_t mx = 0u;
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const bool ok = elem_index<VEC>(g, j, e) < n;
      key[j * VEC + e] = ok ? key[j * VEC + e] : 0u;      // masked tail: below every element
      mx = ok ? max(mx, key[j * VEC + e]) : mx;
    }
  sh.mx[tid] = mx;
  __syncthreads();
  const uint32_t L = threshold_from_maxima<4>(sh.mx + axis * GROUP, k);   // in every wave
  uint32_t hit = 0u;                                      // bit j*VEC+e: element survives
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      hit |= static_cast<uint32_t>((elem_index<VEC>(g, j, e) < n) & (key[j * VEC + e] >= L)) << (j * VEC + e);
  const int cnt = __popc(hit);
  const int incl = wave_scan_dpp(cnt);
  const int tot = __shfl(incl, kWave - 1, kWave);
  int wbase = 0;
  if (lane == 0) wbase = atomicAdd(&sh.ax_cnt[axis], tot);
  wbase = __shfl(wbase, 0, kWave);
  if (wbase + tot <= SMAX_AX) {
    int pos = wbase + incl - cnt;
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if ((hit >> (j * VEC + e)) & 1u) comp[pos++] = axis_comp(key[j * VEC + e], elem_index<VEC>(g, j, e));
  }
  __syncthreads();
  int S = sh.ax_cnt[axis];
  if (max(sh.ax_cnt[0], sh.ax_cnt[1]) > SMAX_AX) {
    // Massive ties on one axis: the exact k-th largest key theta over all its elements, then
    // the elements above it and the lowest-indexed elements equal to it.  Both groups run the
    // loop (its barriers are shared); only an overflowing axis writes.
    const bool overflow = S > SMAX_AX;
    uint32_t prefix = 0u;
    for (int b = 31; b >= 0; --b) {
      const uint32_t c = prefix | (1u << b);
      int cl = 0;
#pragma unroll
      for (int j = 0; j < NE; ++j) cl += key[j] >= c;       // masked keys are 0
      if (group_offsets(cl, axis * 4, 4, sh).y >= k) prefix = c;
    }
    const uint32_t theta = prefix;
    int gl = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) gl += key[j] > theta;
    const int need = k - group_offsets(gl, axis * 4, 4, sh).y;
    int pos = 0, eq_seen = 0;
    // element order: chunk j, then thread g, then e
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      int eq_l = 0;
#pragma unroll
      for (int e = 0; e < VEC; ++e) eq_l += (elem_index<VEC>(g, j, e) < n) & (key[j * VEC + e] == theta);
      const int2 oe = group_offsets(eq_l, axis * 4, 4, sh);
      int eq_rank = eq_seen + oe.x;
      int take_l = 0;
      bool take[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const bool ok = elem_index<VEC>(g, j, e) < n;
        const bool eq = ok & (key[j * VEC + e] == theta);
        take[e] = (ok & (key[j * VEC + e] > theta)) | (eq & (eq_rank < need));
        eq_rank += eq;
        take_l += take[e];
      }
      const int2 otk = group_offsets(take_l, axis * 4, 4, sh);
      if (overflow) {
        int p = pos + otk.x;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
          if (take[e]) comp[p++] = axis_comp(key[j * VEC + e], elem_index<VEC>(g, j, e));
      }
      pos += otk.y;
      eq_seen += oe.y;
    }
    if (overflow) S = k;
    __syncthreads();
  }
  rank_axis(comp, S, axis, k, g, sh);
  __syncthreads();
}

// ---------------------------------------------------------------- top-m of candidates

// A candidate: its fp64 order key and its flat slot, in one 16-byte LDS record.
struct Cand {
  uint64_t key;
  int32_t id;
  int32_t pad;
};

__device__ __forceinline__ int before(const Cand& a, uint64_t ks, int is) {
  return static_cast<int>(a.key > ks) + static_cast<int>((a.key == ks) & (a.id < is));
}

// Rank the S candidates (key desc, id asc) with the whole workgroup: P = 2^lp threads per
// candidate (consecutive lanes), each counting the candidates before it among every P-th one;
// ranks < m go to sh.out_flat / sh.out_g.
__device__ __forceinline__ void rank_candidates(const Cand* cand, int S, int m, SelectShared& sh) {
  int lp = 0;
  while (lp < 6 && (S << (lp + 1)) <= THREADS) ++lp;
  const int P = 1 << lp;
  for (int base = 0; base < (S << lp); base += THREADS) {
    const int slot = base + static_cast<int>(threadIdx.x);
    const int e = slot >> lp, part = slot & (P - 1);
    uint64_t ks = 0ull;
    int is = 0, ab = 0, r = 0;
    if (e < S) {
      ks = cand[e].key;
      is = cand[e].id;
      ab = cand[e].pad;
      int u = part;
      for (; u + 3 * P < S; u += 4 * P) {
        const Cand b0 = cand[u], b1 = cand[u + P], b2 = cand[u + 2 * P], b3 = cand[u + 3 * P];
        r += before(b0, ks, is) + before(b1, ks, is) + before(b2, ks, is) + before(b3, ks, is);
      }
      for (; u < S; u += P) r += before(cand[u], ks, is);
    }
    r = group_sum(r, lp);
    if (part == 0 && e < S && r < m) {
      sh.out_flat[r] = is;
      sh.out_g[r] = key64_value(ks);
      sh.out_ab[r] = ab;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------- a7 fused (decode)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kPoolRowsPerWave = kMaxPoolTopM / NWAVES;

// This (token, head)'s m rows pooled into out_t[0, dv) with fp32 atomic adds.  Wave v reads rows
// v, v + 8, ... with 16-byte nontemporal loads (64 lanes x cpl chunks of a 1 or 2 KiB row, all
// of the wave's rows in flight), the 8 partial rows meet in LDS and are added in wave order, and
// each element takes one atomic add per head.
template <bool BF16>
__device__ void pool_rows(const void* __restrict__ values, int dv, int m, bool softmax, int cores,
                          const SelectShared& sh, float* red, float* __restrict__ out_t) {
  constexpr int EPC = BF16 ? 8 : 4;                  // elements per 16-byte chunk
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int cpl = dv * (BF16 ? 2 : 4) / 1024;        // 16-byte chunks per lane: 1 or 2
  const char* base = static_cast<const char*>(values);
  const size_t row_bytes = static_cast<size_t>(dv) * (BF16 ? 2 : 4);
  // with multi-core scoring a lane's chunk c takes the weight of the column slice it lies in
  // (a second chunk past a 1 KiB row is never loaded; its slice is clamped to a real one)
  int slice[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
    slice[c] = cores > 1 ? min(((kWave * c + lane) * EPC) / (dv / cores), cores - 1) : 0;
  u32x4 raw[kPoolRowsPerWave][2];
  float wt[kPoolRowsPerWave][2];
#pragma unroll
  for (int i = 0; i < kPoolRowsPerWave; ++i) {
    const int r = wave + NWAVES * i;
    wt[i][0] = wt[i][1] = 0.0f;
    raw[i][0] = raw[i][1] = u32x4{0u, 0u, 0u, 0u};
    if (r < m) {
      if (cores > 1) {
        wt[i][0] = sh.w_core[r * cores + slice[0]];
        wt[i][1] = sh.w_core[r * cores + slice[1]];
      } else {
        wt[i][0] = wt[i][1] = softmax ? sh.e[r] / sh.esum : static_cast<float>(sh.out_g[r]);
      }
      const u32x4* src = reinterpret_cast<const u32x4*>(base + static_cast<size_t>(sh.out_flat[r]) * row_bytes);
      raw[i][0] = __builtin_nontemporal_load(src + lane);
      if (cpl > 1) raw[i][1] = __builtin_nontemporal_load(src + kWave + lane);
    }
  }
  float acc[2][EPC];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[c][e] = 0.0f;
#pragma unroll
  for (int i = 0; i < kPoolRowsPerWave; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const uint32_t q[4] = {raw[i][c].x, raw[i][c].y, raw[i][c].z, raw[i][c].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (BF16) {
          acc[c][2 * e] = fmaf(wt[i][c], __uint_as_float(q[e] << 16), acc[c][2 * e]);
          acc[c][2 * e + 1] = fmaf(wt[i][c], __uint_as_float(q[e] & 0xFFFF0000u), acc[c][2 * e + 1]);
        } else {
          acc[c][e] = fmaf(wt[i][c], __uint_as_float(q[e]), acc[c][e]);
        }
      }
    }
  // lane holds elements (64 c + lane) * EPC .. + EPC - 1 of chunk c
#pragma unroll
  for (int c = 0; c < 2; ++c)
    if (c < cpl) {
#pragma unroll
      for (int e = 0; e < EPC; e += 4)
        *reinterpret_cast<float4*>(red + wave * dv + (kWave * c + lane) * EPC + e) =
            make_float4(acc[c][e], acc[c][e + 1], acc[c][e + 2], acc[c][e + 3]);
    }
  __syncthreads();
  for (int col = tid; col < dv; col += THREADS) {
    float v = red[col];
#pragma unroll
    for (int u = 1; u < NWAVES; ++u) v += red[u * dv + col];
    atomicAdd(out_t + col, v);
  }
}

// ---------------------------------------------------------------- the kernel

template <int NV, int VEC, int MODE>
__global__ __launch_bounds__(THREADS) void select_kernel(
    const float* __restrict__ sel, const float* __restrict__ q_row,
    const float* __restrict__ q_col, const float* __restrict__ k_row,
    const float* __restrict__ k_col, const float* __restrict__ core_all,
    int32_t* __restrict__ idx_out, float* __restrict__ w_out, int32_t* __restrict__ axis_out,
    const void* __restrict__ values, int vbf16, int dv, float* __restrict__ pooled,
    int T, int H, int n, int dk, int rank, int k, int m, int grid_tucker, int softmax, int n_cand,
    int cores) {
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ SelectShared sh;
  const int tucker = MODE == kModePool ? grid_tucker : MODE == kModeTucker;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int t = blockIdx.x / H;
  const int h = blockIdx.x % H;

  // ---- a3: the two axes, four waves each
  if (tucker && tid < rank * rank) {
    const float* ch = core_all + static_cast<size_t>(h) * cores * rank * rank;
    double c = 0.0;
    for (int i = 0; i < cores; ++i) {
      const float x = ch[i * rank * rank + tid];
      c += static_cast<double>(x);                 // eq. (16): the core is the sum
      if (cores > 1) sh.core_parts[i][tid] = x;
    }
    sh.core[tid] = c;
  }
  if (tid < 2) sh.ax_cnt[tid] = 0;
  if (tid == 0) sh.grid_cnt = 0;
  // Tucker: the token's two query rows (2 dk / 4 <= THREADS 16-byte pieces), loaded now, staged
  // in LDS for the exact per-slice scores once the axes are done with it
  const int n4 = dk >> 2;
  f32x4 q_piece = {0.0f, 0.0f, 0.0f, 0.0f};
  if (tucker && tid < 2 * n4) {
    const int ax = tid >= n4;
    q_piece = reinterpret_cast<const f32x4*>((ax ? q_col : q_row) + (static_cast<size_t>(t) * H + h) * dk)[tid - (ax ? n4 : 0)];
  }
  select_axes<NV, VEC, MODE>(sel, T, H, t, h, n, k, m, !tucker, reinterpret_cast<uint64_t*>(dyn), sh);
  if (axis_out != nullptr)
    for (int a = tid; a < 2 * k; a += THREADS)
      axis_out[((static_cast<size_t>(a / k) * T + t) * H + h) * k + a % k] = sh.ax_idx[a / k][a % k];

  Cand* cand = reinterpret_cast<Cand*>(dyn);                 // candidates, after the axes
  int S;
  if (!tucker) {
    // ---- a4 (additive): (a, b) with a, b < k and (a+1)(b+1) <= m, scores exact in fp64; every
    // wave first takes theta, the corner bound, itself
    const int R = min(k, m);
    uint64_t th = 0ull;
    for (int r0 = 1; r0 <= R; r0 += kWave) {
      const int r = r0 + lane;
      const int c = r <= R ? sh.th_col[r] : 0;
      if (c > 0)
        th = max(th, order_key64(static_cast<double>(sh.ax_sc[0][r - 1]) + static_cast<double>(sh.ax_sc[1][c - 1])));
    }
    th = additive_limit(wave_max_u64(th));
    const int C = sh.grid_total;
    for (int c0 = wave * kWave; c0 < C; c0 += THREADS) {
      const int c = c0 + lane;
      uint64_t key = 0ull;
      bool keep = false;
      int a = 0, b = 0;
      if (c < C) {
        const int ab = sh.grid_ab[c];
        a = ab >> 8;
        b = ab & 0xFF;
        key = order_key64(static_cast<double>(sh.ax_sc[0][a]) + static_cast<double>(sh.ax_sc[1][b]));
        keep = key >= th;
      }
      const uint64_t bal = __ballot(keep);
      int wbase = 0;
      if (lane == 0 && bal) wbase = atomicAdd(&sh.grid_cnt, static_cast<int>(__popcll(bal)));
      wbase = __shfl(wbase, 0, kWave);
      if (keep) {
        const int pos = wbase + static_cast<int>(__popcll(bal & lanemask_lt()));
        cand[pos].key = key;
        cand[pos].id = sh.ax_idx[0][a] * n + sh.ax_idx[1][b];
      }
    }
    __syncthreads();
    S = sh.grid_cnt;
  } else {
    // ---- a4 (Tucker): exact per-slice scores of the selected keys (eq. (4)), in fp32.  G = 4, 8
    // or 16 lanes per (axis, key) row, as many as 2k rows leave in the workgroup (one pass), and
    // L = G / 4, G / 2 or G lanes per slice of the row (rank 3 or 4, 2, 1): lane sub of a slice
    // takes its 16-byte pieces sub, sub + L, ... (the L lanes read contiguous 16L-byte runs),
    // eight loads in flight before any is used, and the L partial sums meet through DPP.
    {
      const f32x4* qs = reinterpret_cast<const f32x4*>(dyn);          // [2][n4] query pieces
      if (tid < 2 * n4) reinterpret_cast<f32x4*>(dyn)[tid] = q_piece;
      __syncthreads();
      constexpr int kPieces = 8;
      const int wp = n4 / rank;                                        // pieces per slice
      const int lg = 2 * k <= 32 ? 4 : (2 * k <= 64 ? 3 : 2);
      const int ls = rank == 1 ? lg : (rank == 2 ? lg - 1 : lg - 2);
      for (int job = tid; job < (2 * k) << lg; job += THREADS) {   // whole groups: G | THREADS
        const int part = job & ((1 << lg) - 1), row = job >> lg;
        const int axis = row >= k, a = row - (axis ? k : 0);
        const int rho = part >> ls, sub = part & ((1 << ls) - 1);
        const int cnt = rho < rank ? (wp - sub + (1 << ls) - 1) >> ls : 0;
        const int first = rho * wp + sub;
        const f32x4* kr = reinterpret_cast<const f32x4*>(
            (axis ? k_col : k_row) + (static_cast<size_t>(h) * n + sh.ax_idx[axis][a]) * dk) + first;
        const f32x4* qr = qs + axis * n4 + first;
        float acc = 0.0f;
        for (int i0 = 0; i0 < cnt; i0 += kPieces) {
          f32x4 kv[kPieces];
#pragma unroll
          for (int i = 0; i < kPieces; ++i)
            if (i0 + i < cnt) kv[i] = kr[(i0 + i) << ls];
#pragma unroll
          for (int i = 0; i < kPieces; ++i)
            if (i0 + i < cnt) {
              const f32x4 qv = qr[(i0 + i) << ls];
              acc = fmaf(kv[i].x, qv.x, acc);
              acc = fmaf(kv[i].y, qv.y, acc);
              acc = fmaf(kv[i].z, qv.z, acc);
              acc = fmaf(kv[i].w, qv.w, acc);
            }
        }
        acc = group_sum_f(acc, ls);
        if (rho < rank && sub == 0) sh.s_ex[axis][rho][a] = acc;
      }
    }
    __syncthreads();
    for (int job = tid; job < rank * k; job += THREADS) {
      const int rho = job / k, b = job % k;
      double p = 0.0;
      for (int sg = 0; sg < rank; ++sg)
        p += sh.core[rho * rank + sg] * static_cast<double>(sh.s_ex[1][sg][b]);
      sh.p_col[rho][b] = p;
    }
    __syncthreads();
    // Candidates in registers: thread tid < R k takes column b = tid mod k and rows a0 + R j
    // (a0 = tid / k, R = 512 / k, j < CPT; R >= 8 as k <= 64, so CPT = 8 rows cover a column).
    const int R = THREADS / k;
    const int b = tid % k, a0 = tid / k;
    const bool on = tid < R * k;
    double pc[kMaxRank];
#pragma unroll
    for (int r = 0; r < kMaxRank; ++r) pc[r] = (on && r < rank) ? sh.p_col[r][b] : 0.0;
    uint64_t k64[CPT];
    uint32_t k32[CPT];
    uint32_t valid = 0u;                              // bit j: row a0 + R j exists
    uint32_t mx = 0u;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int a = a0 + R * j;
      k64[j] = 0ull;
      k32[j] = 0u;
      if (on && a < k) {
        double gv = 0.0;
#pragma unroll
        for (int rho = 0; rho < kMaxRank; ++rho)            // pc[] indexed at compile time
          if (rho < rank) gv += static_cast<double>(sh.s_ex[0][rho][a]) * pc[rho];
        k64[j] = order_key64(gv);
        k32[j] = order_key(static_cast<float>(gv));
        mx = max(mx, k32[j]);
        valid |= 1u << j;
      }
    }
    sh.mx[tid] = mx;
    __syncthreads();
    // The threshold from all 512 thread maxima, unmerged (each covers up to 8 candidates of one
    // column): their m-th largest lies close to the m-th largest candidate.  Merged lane-wise
    // they would be column maxima, whose m-th largest (m = k) is the best score of the worst
    // column, below most of the grid.  One wave takes it, the others wait at the barrier.
    if (wave == 0) {
      uint32_t mxs[CPT];
#pragma unroll
      for (int q = 0; q < CPT; ++q) mxs[q] = sh.mx[lane + kWave * q];
      const uint32_t L0 = wave_kth_largest16<CPT>(mxs, m);
      if (lane == 0) sh.thr[0] = L0;
    }
    __syncthreads();
    const uint32_t L = sh.thr[0];
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < CPT; ++j) cnt += ((valid >> j) & 1u) & (k32[j] >= L);
    const int2 o = group_offsets(cnt, 0, NWAVES, sh);
    if (o.y <= SMAX_S) {
      int pos = o.x;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const int a = a0 + R * j;
        if (((valid >> j) & 1u) && k32[j] >= L) {
          cand[pos].key = k64[j];
          cand[pos].id = sh.ax_idx[0][a] * n + sh.ax_idx[1][b];
          cand[pos].pad = (a << 8) | b;
          ++pos;
        }
      }
      __syncthreads();
      S = o.y;
    } else {
      // Massive ties: exact m-th largest fp64 key theta, then the lowest flat indices among
      // the candidates equal to it.
      int32_t fl[CPT];
#pragma unroll
      for (int j = 0; j < CPT; ++j)
        fl[j] = ((valid >> j) & 1u) ? sh.ax_idx[0][a0 + R * j] * n + sh.ax_idx[1][b] : 0x7FFFFFFF;
      uint64_t prefix = 0ull;
      for (int bit = 63; bit >= 0; --bit) {
        const uint64_t cb = prefix | (1ull << bit);
        int cl = 0;
#pragma unroll
        for (int j = 0; j < CPT; ++j) cl += ((valid >> j) & 1u) & (k64[j] >= cb);
        if (group_offsets(cl, 0, NWAVES, sh).y >= m) prefix = cb;
      }
      const uint64_t theta = prefix;
      int gl = 0;
#pragma unroll
      for (int j = 0; j < CPT; ++j) gl += ((valid >> j) & 1u) & (k64[j] > theta);
      const int need = m - group_offsets(gl, 0, NWAVES, sh).y;
      uint32_t ylim = 0u;     // the need-th smallest flat index among the keys equal to theta
      for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cb = ylim | (1u << bit);
        int cl = 0;
#pragma unroll
        for (int j = 0; j < CPT; ++j)
          cl += ((valid >> j) & 1u) & (k64[j] == theta) & (static_cast<uint32_t>(fl[j]) < cb);
        if (group_offsets(cl, 0, NWAVES, sh).y < need) ylim = cb;
      }
      int tk = 0;
      uint32_t take = 0u;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const bool ok = ((valid >> j) & 1u) &&
                        ((k64[j] > theta) | ((k64[j] == theta) & (static_cast<uint32_t>(fl[j]) <= ylim)));
        take |= static_cast<uint32_t>(ok) << j;
        tk += ok;
      }
      const int2 ot = group_offsets(tk, 0, NWAVES, sh);
      int pos = ot.x;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        if ((take >> j) & 1u) {
          cand[pos].key = k64[j];
          cand[pos].id = fl[j];
          cand[pos].pad = ((a0 + R * j) << 8) | b;
          ++pos;
        }
      }
      __syncthreads();
      S = m;
    }
  }

  // ---- a5: rank the candidates by (score desc, flat index asc); ranks < m are the answer
  rank_candidates(cand, S, m, sh);
  if (softmax) {
    for (int j = tid; j < m; j += THREADS) sh.e[j] = __expf(static_cast<float>(sh.out_g[j] - sh.out_g[0]));
    __syncthreads();
    if (wave == 0) {
      float s = 0.0f;
      for (int j = lane; j < m; j += kWave) s += sh.e[j];
      s = wave_sum(s);
      if (lane == 0) sh.esum = s;
    }
    __syncthreads();
  }
  for (int j = tid; j < m; j += THREADS) {
    const size_t o = (static_cast<size_t>(t) * H + h) * m + j;
    idx_out[o] = sh.out_flat[j];
    if (cores == 1) w_out[o] = softmax ? sh.e[j] / sh.esum : static_cast<float>(sh.out_g[j]);
  }
  if (cores > 1) {
    // multi-core scoring (eq. (16)): each core's exact score of every selected slot, in fp64
    for (int x = tid; x < m * cores; x += THREADS) {
      const int j = x / cores, i = x - (x / cores) * cores;
      const int a = sh.out_ab[j] >> 8, b = sh.out_ab[j] & 0xFF;
      double g = 0.0;
      for (int rho = 0; rho < rank; ++rho) {
        double p = 0.0;
        for (int sg = 0; sg < rank; ++sg)
          p += static_cast<double>(sh.core_parts[i][rho * rank + sg]) * static_cast<double>(sh.s_ex[1][sg][b]);
        g += static_cast<double>(sh.s_ex[0][rho][a]) * p;
      }
      sh.w_core[x] = static_cast<float>(g);
      w_out[((static_cast<size_t>(t) * H + h) * m + j) * cores + i] = static_cast<float>(g);
    }
    __syncthreads();
  }
  // ---- a7 fused: pool this head's rows into the token's output (the axes' LDS is free now)
  // (a run-time test also in the pooling variant: the decode kernel measured faster with it than
  // with the branch resolved at compile time)
  if (MODE == kModePool && pooled != nullptr) {
    float* red = reinterpret_cast<float*>(dyn);
    float* out_t = pooled + static_cast<size_t>(t) * dv;
    if (vbf16) pool_rows<true>(values, dv, m, softmax, cores, sh, red, out_t);
    else pool_rows<false>(values, dv, m, softmax, cores, sh, red, out_t);
  }
}

// ---------------------------------------------------------------- a wave per (token, head)
//
// Many (token, head) pairs: one wave takes a pair from its scores to its slots.  With a workgroup to
// a pair the vector ALUs' issue was the bound (1,230 instructions in each of eight waves at 2,048
// keys, k = m = 64: every phase's counts, scans and thresholds are repeated by waves that each hold
// a part), and six barriers stand in its chain.  A wave alone needs none of either: thresholds and
// ranks run once, on 64 lanes, and its arrays are its own part of LDS, ordered by wave_lds_order.
//  * Axis scores sit in registers (NV 16-byte pieces a lane).  The threshold of step 1 is the k-th
//    largest of 64 G lane maxima (G = 2 for k <= 32, else 4); survivors go to LDS by ballot.
//  * The Tucker grid needs the top-k only as a set: the k-th key of the survivors is found by a
//    ballot per key bit.  The additive grid needs it in order: every lane counts the keys above its
//    own (32-bit compares; equal keys are found by two lanes claiming one rank, and the lower indices
//    among them counted too).  More than 128 survivors are first cut to the top-k as a set.
//  * Tucker: exact per-slice scores as in the workgroup kernel (the same lanes per row and the same
//    order of additions); a lane then takes a column and walks the rows, whose scores it reads from
//    LDS as doubles; the threshold is the m-th largest of the 512 maxima over eight rows of a column,
//    and only the columns' sets of eight rows that reach it are looked into.
//  * The final rank compares fp64 scores, and counts the lower slots among equal scores where claims
//    (as above) show any; with NaNs it takes the ordered compare by (key, slot).
// Whatever the fast steps cannot hold (more than kWaveCap survivors, fewer than k or m numbers) goes
// to exact searches over all elements, as in the workgroup kernel.
constexpr int kWaveCap = 256;            // survivors of an axis or of the grid
constexpr int kWavePieces = 128;         // 16-byte pieces of an axis (sets of the grid) that hold them
// Pairs (waves) per workgroup: alone where a pair's rare slow steps would hold its neighbours' LDS
// (16,384 Tucker pairs 161 us, 166 with two, 162 - 173 with four; now 141), four where they share a table.
constexpr int wave_items(bool tucker) { return tucker ? 1 : 4; }
constexpr int kWaveMaxK = 64, kWaveMaxM = 64;
constexpr int kWaveMaxKeys = 18 * 256;

// One pair's LDS: the survivors (8 bytes each: key and index of an axis, then fp64 scores of the
// grid), claims of ranks, the grid survivors' (a << 8) | b, the axes' indices, the additive grid's
// sorted scores or the Tucker per-slice scores, and the two query rows.
struct WaveLds {
  uint32_t* skey;        // [kWaveCap]
  uint32_t* sidx;        // [kWaveCap]
  double* cg;            // [kWaveCap], in their place
  uint32_t* code;        // [kWaveCap]: claims; the exponentials
  uint16_t* ab;          // [8 kWavePieces]: the grid survivors
  f32x4* piece;          // [kWavePieces], with piece_at: before the Tucker scores, in their place
  uint32_t* piece_at;    // [kWavePieces]
  int32_t* ax_idx;       // [2][64]
  float* ax_sc;          // [2][64] (additive)
  float* s_ex;           // [2][rank][64] (Tucker)
  double* srow;          // [64][2]: row scores (the second 0 with rank 1)
  double* pcol;          // [2][64]: column factors
  f32x4* q;              // [2][dk / 4]
};

constexpr int kWaveRank = 2;             // the largest Tucker rank here

__host__ __device__ inline size_t wave_lds_bytes(bool tucker, int rank, int dk) {
  const size_t base = kWaveCap * 8 + kWaveCap * 4 + 8 * kWavePieces * 2 + 2 * 64 * 4, pieces = kWavePieces * 20;
  const size_t scores = tucker ? 2 * rank * 64 * 4 + 2 * 64 * kWaveRank * 8 : 2 * 64 * 4;
  return base + (scores > 2 * 64 * 4 + pieces ? scores : 2 * 64 * 4 + pieces) +
         (tucker ? static_cast<size_t>(2) * dk * 4 : 0);
}

__device__ __forceinline__ WaveLds wave_lds(unsigned char* p, bool tucker, int rank) {
  WaveLds s;
  s.cg = reinterpret_cast<double*>(p);
  s.skey = reinterpret_cast<uint32_t*>(p);
  s.sidx = s.skey + kWaveCap;
  s.code = s.sidx + kWaveCap;
  s.ab = reinterpret_cast<uint16_t*>(s.code + kWaveCap);
  s.ax_idx = reinterpret_cast<int32_t*>(s.ab + 8 * kWavePieces);
  s.ax_sc = reinterpret_cast<float*>(s.ax_idx + 2 * 64);
  s.piece = reinterpret_cast<f32x4*>(s.ax_sc + 2 * 64);
  s.piece_at = reinterpret_cast<uint32_t*>(s.piece + kWavePieces);
  s.srow = reinterpret_cast<double*>(s.ax_sc);
  s.pcol = s.srow + 64 * kWaveRank;
  s.s_ex = reinterpret_cast<float*>(s.pcol + 64 * kWaveRank);
  s.q = reinterpret_cast<f32x4*>(p + wave_lds_bytes(tucker, rank, 0));
  return s;
}

// Lanes before this one among those of the mask.
__device__ __forceinline__ int mask_rank(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// Largest L with zero low 16 bits such that at least k of the wave's 64 G values are >= L, one bit
// and G ballots a step (fewer vector instructions than radix-4 steps; other waves fill the chain).
template <int G>
__device__ __forceinline__ uint32_t wave_kth16(const uint32_t (&v)[G], int k) {
  uint32_t p = 0u;
#pragma unroll 1
  for (int b = 31; b >= 16; --b) {
    const uint32_t c = p | (1u << b);
    int cnt = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) cnt += __popcll(__ballot(v[g] >= c));
    p = cnt >= k ? c : p;
    if (cnt == k) break;
  }
  return p;
}

// A key that exactly k of the wave's 64 R keys reach, or, where equal keys allow none, the k-th
// largest.
template <int R>
__device__ __forceinline__ uint32_t wave_kth32(const uint32_t (&v)[R], int k) {
  uint32_t p = 0u;
#pragma unroll 1
  for (int b = 31; b >= 0; --b) {
    const uint32_t c = p | (1u << b);
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) cnt += __popcll(__ballot(v[r] >= c));
    p = cnt >= k ? c : p;
    if (cnt == k) break;
  }
  return p;
}

// The set of the k largest of the S survivors (key desc, index asc), in survivor order: their indices to
// ax[0, k), or, without ax, they become the survivors [0, k).
template <int R>
__device__ __forceinline__ void wave_top_set(const WaveLds& s, int S, int k, int32_t* ax) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t key[R], idx[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = lane + kWave * r;
    key[r] = e < S ? s.skey[e] : 0u;
    idx[r] = e < S ? s.sidx[e] : 0xFFFFFFFFu;
  }
  uint32_t theta = 0u, ylim = 0xFFFFFFFEu;               // (index of no survivor: above ylim)
  if (S > k) {
    theta = wave_kth32<R>(key, k);
    int gt = 0, ge = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      gt += __popcll(__ballot(key[r] > theta));
      ge += __popcll(__ballot(key[r] >= theta && idx[r] <= ylim));
    }
    if (ge > k) {                                         // ties: the lowest indices among them
      const int need = k - gt;
      ylim = 0u;
      for (int b = 15; b >= 0; --b) {                     // largest y with fewer than need below it
        const uint32_t c = ylim | (1u << b);
        int below = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) below += __popcll(__ballot(key[r] == theta && idx[r] < c));
        if (below < need) ylim = c;
      }
    }
  }
  int pos = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool take = idx[r] != 0xFFFFFFFFu && (key[r] > theta || (key[r] == theta && idx[r] <= ylim));
    const uint64_t m = __ballot(take);
    if (take && ax != nullptr) ax[pos + mask_rank(m)] = static_cast<int32_t>(idx[r]);
    if (take && ax == nullptr) {
      s.skey[pos + mask_rank(m)] = key[r];
      s.sidx[pos + mask_rank(m)] = idx[r];
    }
    pos += __popcll(m);
  }
}

// Ranks among equal scores, by id: rank[] counts the greater scores, so that c equal ones have the places rank
// .. rank + c - 1 to themselves.  Each round the lowest id that claims a place keeps it, the others go on to
// the next.  Places from `limit` on are not told apart.  `lost`: the lanes that are not the only ones of their
// score, but for one of each.  False where they are over three quarters of the S or some score has more than
// kClaimRounds + 1 (many equal scores: a round is a trip to LDS and back, and comparing all is as fast); rank[]
// is then as it was.  Scores rounded to bf16, 2,049 pairs of 2,044 keys, k = 60, m = 40: 24.6 us, 31.7 where all
// were compared, the workgroup kernel 25.8; 2,048 of 1,024, k = m = 32: 15.3, 18.2, 19.1.
constexpr int kClaimRounds = 12;
template <int R, typename Id>
__device__ __forceinline__ bool wave_claim_places(const WaveLds& s, int S, int limit, const uint64_t (&lost)[R],
                                                  const Id (&id)[R], int (&rank)[R]) {
  int n_lost = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) n_lost += __popcll(lost[r]);
  if (4 * n_lost > 3 * S) return false;
  const int lane = threadIdx.x & (kWave - 1);
  int at[R];
  bool open[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    at[r] = rank[r];
    open[r] = lane + kWave * r < S && at[r] < limit;
    s.code[lane + kWave * r] = ~0u;
  }
  wave_lds_order();
#pragma unroll 1
  for (int round = 0; round <= kClaimRounds; ++round) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (open[r]) atomicMin(s.code + at[r], static_cast<uint32_t>(id[r]));
    wave_lds_order();
    bool any = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (open[r] && s.code[at[r]] != static_cast<uint32_t>(id[r])) ++at[r];
      else open[r] = false;
      open[r] = open[r] && at[r] < limit;
      any |= open[r];
    }
    if (__ballot(any) == 0ull) {
#pragma unroll
      for (int r = 0; r < R; ++r) rank[r] = at[r];
      return true;
    }
    wave_lds_order();
  }
  return false;
}

// The S survivors ranked (key desc, index asc): ranks < k to ax / sc.
template <int R>
__device__ __forceinline__ void wave_top_sorted(const WaveLds& s, int S, int k, int32_t* ax, float* sc) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t key[R], idx[R];
  int rank[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = lane + kWave * r;
    key[r] = e < S ? s.skey[e] : 0u;
    idx[r] = e < S ? s.sidx[e] : 0u;
    rank[r] = 0;
  }
  if (lane < 4 && S + lane < kWaveCap) {                  // the last group of four compares
    s.skey[S + lane] = 0u;
    s.sidx[S + lane] = 0xFFFFFFFFu;
  }
  wave_lds_order();
#pragma unroll 4
  for (int u = 0; u < S; u += 4) {
    const uint4 o = *reinterpret_cast<const uint4*>(s.skey + u);
#pragma unroll
    for (int r = 0; r < R; ++r)
      rank[r] += static_cast<int>(o.x > key[r]) + static_cast<int>(o.y > key[r]) +
                 static_cast<int>(o.z > key[r]) + static_cast<int>(o.w > key[r]);
  }
  // equal keys claim one rank: the claim's last writer is one of them, the others see it.  (One pair with
  // a tie holds up its launch: 2,048 additive pairs of 1,024 normal scores took 27.1 us where this and the
  // grid's ranks below went entry by entry over up to 256 survivors in four registers a lane, 14.2 now, the
  // workgroup kernel 18.3; scores in steps of 1/4 44 -> 22, 20 there.)
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane + kWave * r < S) s.code[rank[r]] = lane + kWave * r;
  wave_lds_order();
  uint64_t lost[R], any = 0ull;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    lost[r] = __ballot(lane + kWave * r < S && s.code[rank[r]] != static_cast<uint32_t>(lane + kWave * r));
    any |= lost[r];
  }
  if (any != 0ull && !wave_claim_places<R>(s, S, k, lost, idx, rank)) {
#pragma unroll 2
    for (int u = 0; u < S; u += 4) {
      const uint4 ok = *reinterpret_cast<const uint4*>(s.skey + u), oi = *reinterpret_cast<const uint4*>(s.sidx + u);
#pragma unroll
      for (int r = 0; r < R; ++r)
        rank[r] += static_cast<int>((ok.x == key[r]) & (oi.x < idx[r])) + static_cast<int>((ok.y == key[r]) & (oi.y < idx[r])) +
                   static_cast<int>((ok.z == key[r]) & (oi.z < idx[r])) + static_cast<int>((ok.w == key[r]) & (oi.w < idx[r]));
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane + kWave * r < S && rank[r] < k) {
      ax[rank[r]] = static_cast<int32_t>(idx[r]);
      sc[rank[r]] = key32_value(key[r]);
    }
}

// The k largest of src[0, n) (score desc, index asc) to s.skey / s.sidx[0, k), in no order: the k-th key
// by histograms of its four bytes in LDS, then the elements above it and the lowest-indexed ones equal
// to it.  Bound by latency: five passes over scores that the caches hold, four 16-byte loads in flight
// a lane (in registers they would set the whole kernel's).  2,048 Tucker pairs of 2,048 keys with all but
// 100 masked: 55 us (32 with no key masked; 81 in the workgroup kernel), 508 when the search took a pass
// of single loads a bit; 8,192 additive pairs of 4,480 keys 277 us (299), before 5,914.  A pass that finds
// one key among the candidates (all equal, few distinct scores) ends the search: those pairs with equal
// scores 463 -> 243 us (312).
__device__ __forceinline__ void wave_axis_exact(const float* __restrict__ src, int n, int k, const WaveLds& s) {
  constexpr int kLoads = 4;
  int lane = threadIdx.x & (kWave - 1);
  asm("" : "+v"(lane));                                   // (no address of the caller's kept for this)
  const int steps = (n + 255) / 256;
  uint32_t* const bins = s.skey;                          // [256]
  uint32_t theta = 0u;                                    // the k-th key's bytes so far
  int want = k;                                           // its rank among the keys of these bytes
  auto load = [&](int j0, f32x4 (&x)[kLoads]) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
      x[u] = *reinterpret_cast<const f32x4*>(src + min(256 * (j0 + u) + 4 * lane, n - 4));
  };
  bool all = false;                                       // exactly k keys reach theta
#pragma unroll 1
  for (int shift = 24; shift >= 0 && !all; shift -= 8) {
    const uint32_t known = shift == 24 ? 0u : ~0u << (shift + 8);
    uint32_t hi = 0u, nlo = 0u;                           // the largest of these keys, ~ the smallest
    *reinterpret_cast<uint4*>(bins + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_order();
#pragma unroll 1
    for (int j0 = 0; j0 < steps; j0 += kLoads) {
      f32x4 x[kLoads];
      load(j0, x);
#pragma unroll
      for (int u = 0; u < kLoads; ++u) {
        const bool in = 256 * (j0 + u) + 4 * lane < n;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t key = order_key(x[u][e]), digit = (key >> shift) & 255u;
          const bool mine = in && ((key ^ theta) & known) == 0u;
          const uint64_t m = __ballot(mine);
          if (m == 0ull) continue;                        // (wave-uniform)
          hi = max(hi, mine ? key : 0u);
          nlo = max(nlo, mine ? ~key : 0u);
          // equal digits (ties, a mask) add once
          const int lead = __builtin_ctzll(m);
          const uint32_t d0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(digit), lead));
          if ((__ballot(digit != d0) & m) == 0ull) {
            if (lane == lead) atomicAdd(bins + d0, static_cast<uint32_t>(__popcll(m)));
          } else if (mine) {
            atomicAdd(bins + digit, 1u);
          }
        }
      }
    }
    hi = static_cast<uint32_t>(wave_max_u64(hi));
    if (hi == ~static_cast<uint32_t>(wave_max_u64(nlo))) {         // one key
      theta = hi;
      break;
    }
    wave_lds_order();
    const uint4 c = *reinterpret_cast<const uint4*>(bins + 4 * lane);
    const int sum = static_cast<int>(c.x + c.y + c.z + c.w);
    const int incl = wave_scan_dpp(sum), total = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int at = __builtin_ctzll(__ballot(total - incl < want && total - incl + sum >= want));
    int over = total - __builtin_amdgcn_readlane(incl, at);       // keys of these bytes in higher bins
    int bin = 3, held = __builtin_amdgcn_readlane(static_cast<int>(c.w), at);
    if (over + held < want) over += held, bin = 2, held = __builtin_amdgcn_readlane(static_cast<int>(c.z), at);
    if (over + held < want) over += held, bin = 1, held = __builtin_amdgcn_readlane(static_cast<int>(c.y), at);
    if (over + held < want) over += held, bin = 0, held = __builtin_amdgcn_readlane(static_cast<int>(c.x), at);
    theta |= static_cast<uint32_t>(4 * at + bin) << shift;
    want -= over;
    all = held == want;
    wave_lds_order();                                     // before the next pass clears the bins
  }
  // greater keys from the front, equal ones from the back (their ranks in index order)
  const int need = all ? k : want;
  int pos = 0, seen = 0;
#pragma unroll 1
  for (int j0 = 0; j0 < steps; j0 += kLoads) {
    f32x4 x[kLoads];
    load(j0, x);
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int i = 256 * (j0 + u) + 4 * lane;
      uint32_t key[4];
      uint64_t eq[4];
      int rank = seen;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        key[e] = order_key(x[u][e]);
        const bool hit = i < n && key[e] > theta;
        const uint64_t m = __ballot(hit);
        if (hit) {
          const int at = pos + mask_rank(m);
          s.skey[at] = key[e];
          s.sidx[at] = static_cast<uint32_t>(i + e);
        }
        pos += __popcll(m);
        eq[e] = __ballot(i < n && key[e] == theta);
        rank += mask_rank(eq[e]);
        seen += __popcll(eq[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool mine = (eq[e] >> lane) & 1ull;
        if (mine && rank < need) {
          s.skey[k - 1 - rank] = theta;
          s.sidx[k - 1 - rank] = static_cast<uint32_t>(i + e);
        }
        rank += mine;
      }
    }
  }
}

// One axis: the top-k of src[0, n), which is in v, to ax (a set, or in order with their scores to sc).
// Once the survivors' pieces are in LDS v takes the next axis's scores, which land under the rest.
template <int NV>
__device__ __forceinline__ void wave_load(const float* __restrict__ src, int n, f32x4 (&v)[NV]) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int j = 0; j < NV; ++j)
    v[j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + min(256 * j + 4 * lane, n - 4)));
}
template <int NV, bool TUCKER>
__device__ __forceinline__ void wave_axis(f32x4 (&v)[NV], const float* __restrict__ src,
                                          const float* __restrict__ next, int n, int k, bool sorted,
                                          const WaveLds& s, int32_t* ax, float* sc) {
  const int lane = threadIdx.x & (kWave - 1);
  const float nan = __builtin_nanf("");
  float mx[4] = {nan, nan, nan, nan};                     // fmaxf takes the number
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (256 * (j + 1) > n && 256 * j + 4 * lane >= n) v[j] = f32x4{nan, nan, nan, nan};
    mx[j & 3] = fmaxf(mx[j & 3], fmaxf(fmaxf(v[j].x, v[j].y), fmaxf(v[j].z, v[j].w)));
  }
  uint32_t L;
  if (k <= kWave / 2 || NV < 4) {
    const uint32_t g[2] = {order_key(fmaxf(mx[0], mx[2])), order_key(fmaxf(mx[1], mx[3]))};
    L = wave_kth16<2>(g, k);
  } else {
    const uint32_t g[4] = {order_key(mx[0]), order_key(mx[1]), order_key(mx[2]), order_key(mx[3])};
    L = wave_kth16<4>(g, k);
  }
  // (an L up to -inf's key, where that many groups hold no number above it, bounds nothing: exact search)
  const bool limit = key32_is_limit(L);
  int S = 0, Q = 0;
  if (limit) {
    // first the 16-byte pieces that hold a survivor, then, a piece to a lane, the survivors
    const float lim = key32_value(L);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const bool hit = fmaxf(fmaxf(v[j].x, v[j].y), fmaxf(v[j].z, v[j].w)) >= lim;
      const uint64_t m = __ballot(hit);
      if (m != 0ull) {                                    // (wave-uniform)
        const int at = Q + mask_rank(m);
        if (hit && at < kWavePieces) {
          s.piece[at] = v[j];
          s.piece_at[at] = static_cast<uint32_t>(256 * j + 4 * lane);
        }
        Q += __popcll(m);
      }
    }
  }
  if (next != nullptr) wave_load<NV>(next, n, v);
  if (limit) {
    const float lim = key32_value(L);
    wave_lds_order();
    if (Q <= kWavePieces) {
      for (int q0 = 0; q0 < Q; q0 += kWave) {             // (wave-uniform)
        const int q = q0 + lane;
        const f32x4 x = q < Q ? s.piece[q] : f32x4{nan, nan, nan, nan};
        const uint32_t i = q < Q ? s.piece_at[q] : 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool hit = x[e] >= lim;
          const uint64_t m = __ballot(hit);
          const int at = S + mask_rank(m);
          if (hit && at < kWaveCap) {
            s.skey[at] = order_key(x[e]);
            s.sidx[at] = i + e;
          }
          S += __popcll(m);
        }
      }
    }
  }
  if (S < k || Q > kWavePieces || S > kWaveCap) {
    // too many survivors (massive ties) or too few (S stays 0 without a limit)
    wave_axis_exact(src, n, k, s);
    S = k;
  }
  S = __builtin_amdgcn_readfirstlane(S);
  wave_lds_order();
  if (TUCKER && !sorted) {
    if (S <= 2 * kWave) wave_top_set<2>(s, S, k, ax);
    else wave_top_set<4>(s, S, k, ax);
  } else {
    if (S > (TUCKER ? 1 : 2) * kWave) {                   // fewer first: a rank costs S compares
      wave_top_set<4>(s, S, k, nullptr);
      S = k;
      wave_lds_order();
    }
    if (TUCKER || S <= kWave) wave_top_sorted<1>(s, S, k, ax, sc);
    else wave_top_sorted<2>(s, S, k, ax, sc);
  }
  wave_lds_order();
}

// The S grid survivors (fp64 scores in s.cg, lane + 64 r's slot in id[r]) ranked (score desc, slot
// asc), the first m of them exactly.
template <int R>
__device__ __forceinline__ void wave_rank_grid(const WaveLds& s, int S, int m, const double (&g)[R],
                                               const int32_t (&id)[R], int (&rank)[R]) {
  const int lane = threadIdx.x & (kWave - 1);
  bool nan = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    rank[r] = 0;
    nan |= lane + kWave * r < S && g[r] != g[r];
  }
  if (lane == 0 && (S & 1) != 0) s.cg[S] = __builtin_nan("");    // (S < kWaveCap: the second of a pair)
  wave_lds_order();
#pragma unroll 4
  for (int u = 0; u < S; u += 2) {
    const double2 o = *reinterpret_cast<const double2*>(s.cg + u);
#pragma unroll
    for (int r = 0; r < R; ++r) rank[r] += static_cast<int>(o.x > g[r]) + static_cast<int>(o.y > g[r]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane + kWave * r < S) s.code[rank[r]] = lane + kWave * r;
  wave_lds_order();
  uint64_t lost[R], any = 0ull;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    lost[r] = __ballot(lane + kWave * r < S && s.code[rank[r]] != static_cast<uint32_t>(lane + kWave * r));
    any |= lost[r];
  }
  const bool nans = __ballot(nan) != 0ull;
  if (!nans && any == 0ull) return;
  wave_lds_order();
  if (!nans && wave_claim_places<R>(s, S, m, lost, id, rank)) return;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane + kWave * r < S) s.code[lane + kWave * r] = static_cast<uint32_t>(id[r]);
  wave_lds_order();
  if (!nans) {                                            // equal scores: the lower slots first
#pragma unroll 4
    for (int u = 0; u < S; u += 2) {                      // (the NaN past an odd S equals nothing)
      const double2 o = *reinterpret_cast<const double2*>(s.cg + u);
      const int2 oi = *reinterpret_cast<const int2*>(s.code + u);
#pragma unroll
      for (int r = 0; r < R; ++r)
        rank[r] += (static_cast<int>(o.x == g[r]) & static_cast<int>(oi.x < id[r])) +
                   (static_cast<int>(o.y == g[r]) & static_cast<int>(oi.y < id[r]));
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) rank[r] = 0;
  for (int u = 0; u < S; ++u) {
    const uint64_t ok = order_key64(s.cg[u]);
    const int32_t oi = static_cast<int32_t>(s.code[u]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint64_t me = order_key64(g[r]);
      rank[r] += static_cast<int>(ok > me) + static_cast<int>((ok == me) & (oi < id[r]));
    }
  }
}

// The S > 2 kWave survivors of the additive grid, whose codes are in s.ab, cut to the m best where those
// equal to the m-th in fp32 are one score (ties of many: quantised or repeated scores), else to those that
// reach it in fp32.  Their new number.  2,060 pairs of 1,024 normal scores, k = 33, m = 64: 19.2 us, 27.6 where
// all were ranked (the workgroup kernel 29.9); scores in steps of 1/4 28, 43 (33.5).
__device__ __forceinline__ int wave_cut_additive(const WaveLds& s, int S, int n, int m) {
  constexpr int R = kWaveCap / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t code[R], key[R];
  double g[R];
  int id[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool on = lane + kWave * r < S;
    code[r] = on ? s.ab[lane + kWave * r] : 0u;
    const int a = static_cast<int>(code[r] >> 8), b = static_cast<int>(code[r] & 0xFFu);
    g[r] = static_cast<double>(s.ax_sc[a]) + static_cast<double>(s.ax_sc[64 + b]);
    key[r] = on ? order_key(static_cast<float>(g[r])) : 0u;
    id[r] = on ? s.ax_idx[a] * n + s.ax_idx[64 + b] : 0x7FFFFFFF;
  }
  const uint32_t theta = wave_kth32<R>(key, m);
  int gt = 0, ge = 0;
  double at = __builtin_nan("");                          // a score equal to the m-th in fp32
  uint64_t eq[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool on = lane + kWave * r < S;
    gt += __popcll(__ballot(on && key[r] > theta));
    eq[r] = __ballot(on && key[r] == theta);
    ge += __popcll(eq[r]);
    if (eq[r] != 0ull) {                                  // (wave-uniform)
      const uint64_t v = __builtin_bit_cast(uint64_t, g[r]);
      const int from = __builtin_ctzll(eq[r]);
      const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(v), from);
      const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), from);
      at = __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
    }
  }
  ge += gt;
  int lim = 0x7FFFFFFE;                                   // the highest slot taken among the equal ones
  bool one = ge > m;
#pragma unroll
  for (int r = 0; r < R; ++r)
    one = one && (__ballot(g[r] == at || (g[r] != g[r] && at != at)) & eq[r]) == eq[r];
  if (one) {                                              // the lowest slots among them
    const int need = m - gt;
    lim = 0;
    for (int b = 25; b >= 0; --b) {                       // largest y with fewer than need below it
      const int c = lim | (1 << b);
      int below = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) below += __popcll(__ballot(id[r] < c) & eq[r]);
      if (below < need) lim = c;
    }
  }
  wave_lds_order();
  int pos = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool take = lane + kWave * r < S && (key[r] > theta || (key[r] == theta && id[r] <= lim));
    const uint64_t mk = __ballot(take);
    if (take) s.ab[pos + mask_rank(mk)] = static_cast<uint16_t>(code[r]);
    pos += __popcll(mk);
  }
  wave_lds_order();
  return pos;
}

struct WaveArgs {
  const float *sel, *q_row, *q_col, *k_row, *k_col, *core;
  int32_t* idx_out;
  float* w_out;
  int32_t* axis_out;
  int T, H, n, dk, rank, k, m, softmax, cores;
};

// Ranks the S grid survivors, whose codes are in s.ab, and writes the m best.
template <int R, bool TUCKER>
__device__ __forceinline__ void wave_finish(const WaveArgs& A, const WaveLds& s, int S, size_t pair, int h) {
  const int lane = threadIdx.x & (kWave - 1);
  double g[R];
  int32_t id[R];
  int rank[R], a[R], b[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = lane + kWave * r;
    const uint32_t c = e < S ? s.ab[e] : 0u;
    a[r] = static_cast<int>(c >> 8);
    b[r] = static_cast<int>(c & 0xFFu);
    if (TUCKER) {
      g[r] = 0.0;
      g[r] += s.srow[2 * a[r]] * s.pcol[b[r]];
      g[r] += s.srow[2 * a[r] + 1] * s.pcol[64 + b[r]];
    } else {
      g[r] = static_cast<double>(s.ax_sc[a[r]]) + static_cast<double>(s.ax_sc[64 + b[r]]);
    }
    id[r] = s.ax_idx[a[r]] * A.n + s.ax_idx[64 + b[r]];
  }
  wave_lds_order();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane + kWave * r < S) s.cg[lane + kWave * r] = g[r];
  wave_lds_order();
  wave_rank_grid<R>(s, S, A.m, g, id, rank);
  const size_t o = pair * A.m;
  float e_of[R];
  float inv_of = 1.0f;
  if (A.softmax) {
    // the exponentials by rank (a lane each, as they are summed), then their sum
    wave_lds_order();
    float* ex = reinterpret_cast<float*>(s.code);
    double* best = s.cg;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (lane + kWave * r < S && rank[r] == 0) best[0] = g[r];
    wave_lds_order();
    const double g0 = best[0];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      e_of[r] = __expf(static_cast<float>(g[r] - g0));
      if (lane + kWave * r < S && rank[r] < A.m) ex[rank[r]] = e_of[r];
    }
    wave_lds_order();
    inv_of = wave_sum(lane < A.m ? ex[lane] : 0.0f);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (!(lane + kWave * r < S && rank[r] < A.m)) continue;
    A.idx_out[o + rank[r]] = id[r];
    if (!TUCKER || A.cores == 1) {
      A.w_out[o + rank[r]] = A.softmax ? e_of[r] / inv_of : static_cast<float>(g[r]);
    } else {
      // multi-core scoring (eq. (16)): each core's exact score of the slot, in fp64
      const float* parts = A.core + static_cast<size_t>(h) * A.cores * A.rank * A.rank;
      for (int i = 0; i < A.cores; ++i) {
        double gi = 0.0;
        for (int rho = 0; rho < A.rank; ++rho) {
          double p = 0.0;
          for (int sg = 0; sg < A.rank; ++sg)
            p += static_cast<double>(parts[(i * A.rank + rho) * A.rank + sg]) *
                 static_cast<double>(s.s_ex[(A.rank + sg) * 64 + b[r]]);
          gi += s.srow[2 * a[r] + rho] * p;
        }
        A.w_out[(o + rank[r]) * A.cores + i] = static_cast<float>(gi);
      }
    }
  }
}

template <int NV, bool TUCKER>
__global__ __launch_bounds__(wave_items(TUCKER) * kWave, NV <= 12 ? 4 : 3) void select_wave_kernel(WaveArgs A) {
  constexpr int kItems = wave_items(TUCKER);
  extern __shared__ __align__(16) unsigned char dyn[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = kItems == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // pairs in head-major order, dealt to the eight XCDs in contiguous runs (workgroups go to XCDs
  // round-robin): an XCD's waves re-read the key rows of few heads, from its own L2
  const int64_t pairs = static_cast<int64_t>(A.T) * A.H;
  const int64_t nwg = gridDim.x, per = nwg >> 3, extra = nwg & 7, xcd = blockIdx.x & 7;
  const int64_t wg = xcd * per + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
  const int64_t item = wg * kItems + wave;
  const int k = A.k, m = A.m;
  const size_t part = wave_lds_bytes(TUCKER, A.rank, A.dk);
  const WaveLds s = wave_lds(dyn + wave * part, TUCKER, A.rank);
  if (!TUCKER) {
    // the workgroup's table of the additive grid's candidates (a+1)(b+1) <= m, row by row, and
    // ceil(m / r) for the corner bound of r rows, after the waves' parts
    uint16_t* ab = reinterpret_cast<uint16_t*>(dyn + kItems * part);
    if (wave == 0) {
      const int rows = min(k, m);
      const int len = lane < rows ? min(k, m / (lane + 1)) : 0;
      const int first = wave_scan_dpp(len) - len;
      for (int b = 0; b < len; ++b) ab[first + b] = static_cast<uint16_t>((lane << 8) | b);
    }
    __syncthreads();
  }
  if (item >= pairs) return;                              // (no barrier beyond)
  const int h = static_cast<int>(item / A.T);
  const size_t pair = static_cast<size_t>(item % A.T) * A.H + h;
  if (TUCKER) {                                           // the two query rows to LDS
    const int n4 = A.dk >> 2;
    for (int x = lane; x < 2 * n4; x += kWave)
      s.q[x] = reinterpret_cast<const f32x4*>((x >= n4 ? A.q_col : A.q_row) + pair * A.dk)[x - (x >= n4 ? n4 : 0)];
  }
  const bool sorted = !TUCKER || A.axis_out != nullptr;
  const float* const src0 = A.sel + pair * A.n;
  const float* const src1 = src0 + static_cast<size_t>(A.T) * A.H * A.n;
  f32x4 v[NV];
  wave_load<NV>(src0, A.n, v);
#pragma unroll 1
  for (int axis = 0; axis < 2; ++axis) {
    // (the Tucker per-slice scores come later: their place takes the axis scores nobody reads)
    wave_axis<NV, TUCKER>(v, axis ? src1 : src0, axis ? nullptr : src1, A.n, k, sorted, s,
                          s.ax_idx + axis * 64, s.ax_sc + axis * 64);
    if (A.axis_out != nullptr && lane < k)
      A.axis_out[(static_cast<size_t>(axis) * A.T * A.H + pair) * k + lane] = s.ax_idx[axis * 64 + lane];
  }
  int S = 0;
  if (!TUCKER) {
    const uint16_t* ab = reinterpret_cast<const uint16_t*>(dyn + kItems * part);
    // theta: the best lower bound on the m-th score that a corner of r x ceil(m / r) pairs gives
    // (a NaN corner bounds nothing; none at all keeps every candidate)
    const int rows = min(k, m);
    uint64_t th = 0ull;
    if (lane < rows) {
      const int c = (m + lane) / (lane + 1);
      if (c <= k) th = order_key64(static_cast<double>(s.ax_sc[lane]) + static_cast<double>(s.ax_sc[64 + c - 1]));
    }
    th = additive_limit(wave_max_u64(th));
    const int len = lane < rows ? min(k, m / (lane + 1)) : 0;
    const int C = __shfl(wave_scan_dpp(len), kWave - 1, kWave);
    for (int c0 = 0; c0 < C; c0 += kWave) {
      const int c = c0 + lane;
      bool keep = false;
      uint32_t code = 0u;
      if (c < C) {
        code = ab[c];
        keep = order_key64(static_cast<double>(s.ax_sc[code >> 8]) + static_cast<double>(s.ax_sc[64 + (code & 0xFFu)])) >= th;
      }
      const uint64_t mk = __ballot(keep);
      if (keep) s.ab[S + mask_rank(mk)] = static_cast<uint16_t>(code);
      S += __popcll(mk);
    }
    wave_lds_order();
    // (a rank of that many costs more)
    if (S > 2 * kWave) S = wave_cut_additive(s, S, A.n, m);
  } else {
    // ---- exact per-slice scores of the selected keys (eq. (4)), fp32: G = 4, 8 or 16 lanes to an
    // (axis, key) row, L of them to a slice, each striding its slice's 16-byte pieces by L, eight
    // loads in flight; the partial sums meet through DPP
    const int rank = A.rank;
    {
      constexpr int kPieces = 8;
      const int n4 = A.dk >> 2, wp = n4 / rank;
      const int lg = 2 * k <= 32 ? 4 : (2 * k <= 64 ? 3 : 2);
      const int ls = rank == 1 ? lg : lg - 1;
      const int part_of = lane & ((1 << lg) - 1);
      const int rho = part_of >> ls, sub = part_of & ((1 << ls) - 1);
      const int cnt = (wp - sub + (1 << ls) - 1) >> ls;
      const int first = rho * wp + sub;
      const int most = (wp + (1 << ls) - 1) >> ls, least = wp >> ls;    // of cnt
      for (int row0 = 0; row0 < 2 * k; row0 += kWave >> lg) {
        const int row = row0 + (lane >> lg);
        const bool on = row < 2 * k;
        const int axis = row >= k && on, a = on ? row - (axis ? k : 0) : 0;
        const f32x4* kr = reinterpret_cast<const f32x4*>(
            (axis ? A.k_col : A.k_row) + (static_cast<size_t>(h) * A.n + s.ax_idx[axis * 64 + a]) * A.dk) + first;
        const f32x4* qr = s.q + axis * n4 + first;
        float acc = 0.0f;
        int i0 = 0;
        for (; i0 + kPieces <= least; i0 += kPieces) {    // whole batches in every lane
          f32x4 kv[kPieces];
#pragma unroll
          for (int i = 0; i < kPieces; ++i) kv[i] = kr[(i0 + i) << ls];
#pragma unroll
          for (int i = 0; i < kPieces; ++i) {
            const f32x4 qv = qr[(i0 + i) << ls];
            acc = fmaf(kv[i].x, qv.x, acc);
            acc = fmaf(kv[i].y, qv.y, acc);
            acc = fmaf(kv[i].z, qv.z, acc);
            acc = fmaf(kv[i].w, qv.w, acc);
          }
        }
        for (; i0 < most; i0 += kPieces) {
          f32x4 kv[kPieces];
#pragma unroll
          for (int i = 0; i < kPieces; ++i)
            if (i0 + i < cnt) kv[i] = kr[(i0 + i) << ls];
#pragma unroll
          for (int i = 0; i < kPieces; ++i)
            if (i0 + i < cnt) {
              const f32x4 qv = qr[(i0 + i) << ls];
              acc = fmaf(kv[i].x, qv.x, acc);
              acc = fmaf(kv[i].y, qv.y, acc);
              acc = fmaf(kv[i].z, qv.z, acc);
              acc = fmaf(kv[i].w, qv.w, acc);
            }
        }
        acc = group_sum_f(acc, ls);
        if (on && sub == 0) {
          s.s_ex[(axis * rank + rho) * 64 + a] = acc;
          if (axis == 0) {
            s.srow[2 * a + rho] = static_cast<double>(acc);
            if (rank == 1) s.srow[2 * a + 1] = 0.0;
          }
        }
      }
    }
    // rows up to the next eight score NaN: never above a threshold
    const double nan64 = __builtin_nan("");
    if (lane >= k && lane < ((k + 7) & ~7))
      s.srow[2 * lane] = s.srow[2 * lane + 1] = nan64;
    wave_lds_order();
    // column factors p = C S_col[:, b], lane b's own and in LDS
    double pc[kWaveRank];
    {
      const float* ch = A.core + static_cast<size_t>(h) * A.cores * rank * rank;
#pragma unroll
      for (int rho = 0; rho < kWaveRank; ++rho) {
        double p = 0.0;
        for (int sg = 0; sg < rank; ++sg) {
          double c = 0.0;
          if (rho < rank)
            for (int i = 0; i < A.cores; ++i) c += static_cast<double>(ch[(i * rank + rho) * rank + sg]);
          p += c * static_cast<double>(s.s_ex[(rank + sg) * 64 + min(lane, k - 1)]);
        }
        if (rho >= rank) p = 0.0;
        s.pcol[rho * 64 + lane] = p;
        pc[rho] = lane < k ? p : nan64;
      }
    }
    wave_lds_order();
    // row a's score in the column of factors p0, p1, exact in fp64; this lane's column
    auto score_at = [&](int a, double p0, double p1) {
      const double2 sr = *reinterpret_cast<const double2*>(s.srow + 2 * a);
      double g = 0.0;
      g += sr.x * p0;
      g += sr.y * p1;
      return g;
    };
    auto score = [&](int a) { return score_at(a, pc[0], pc[1]); };
    // sets of eight rows of a column: their maxima (fp32 roundings: rounding is monotone)
    uint32_t mxk[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      double mx = nan64;
      if (8 * c < k) {                                    // (wave-uniform)
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmax(mx, score(8 * c + i));
      }
      mxk[c] = order_key(static_cast<float>(mx));
    }
    const uint32_t L = wave_kth16<8>(mxk, m);
    const bool limit = key32_is_limit(L);                 // (else the exact search, as for an axis)
    int Q = 0;
    if (limit) {
      // first the sets that hold a survivor, then, a set to a lane, the survivors
      const float lim = key32_value(L);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const bool hit = mxk[c] >= L;
        const uint64_t mk = __ballot(hit);
        const int at = Q + mask_rank(mk);
        if (hit && at < kWavePieces) s.sidx[at] = static_cast<uint32_t>((c << 11) | lane);
        Q += __popcll(mk);
      }
      wave_lds_order();
      if (Q <= kWavePieces) {
        for (int q0 = 0; q0 < Q; q0 += kWave) {           // (wave-uniform)
          const bool on = q0 + lane < Q;
          const uint32_t set = on ? s.sidx[q0 + lane] : 0u;
          const int a0 = static_cast<int>(set >> 8), b = static_cast<int>(set & 0xFFu);
          const double p0 = on ? s.pcol[b] : nan64, p1 = s.pcol[64 + b];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const bool hit = static_cast<float>(score_at(a0 + i, p0, p1)) >= lim;
            const uint64_t mk = __ballot(hit);
            const int at = S + mask_rank(mk);
            if (hit) s.ab[at] = static_cast<uint16_t>(set + (i << 8));
            S += __popcll(mk);
          }
        }
      }
    }
    if (limit && Q <= kWavePieces && S > kWaveCap && S <= 2 * kWaveCap) {
      // sets of a few columns that hold most of the grid's best (a core close to rank one): the m-th
      // largest rounding of all survivors takes the threshold's place
      constexpr int kPer = 2 * kWaveCap / kWave;
      wave_lds_order();
      uint32_t key[kPer], code[kPer];
#pragma unroll
      for (int r = 0; r < kPer; ++r) {
        const int e = lane + kWave * r;
        code[r] = e < S ? s.ab[e] : 0u;
        const uint32_t b = code[r] & 0xFFu;
        key[r] = e < S ? order_key(static_cast<float>(score_at(code[r] >> 8, s.pcol[b], s.pcol[64 + b]))) : 0u;
      }
      const uint32_t theta = wave_kth32<kPer>(key, m);    // (above 0: they are all numbers)
      wave_lds_order();
      S = 0;
#pragma unroll
      for (int r = 0; r < kPer; ++r) {
        const bool hit = key[r] >= theta;
        const uint64_t mk = __ballot(hit);
        if (hit) s.ab[S + mask_rank(mk)] = static_cast<uint16_t>(code[r]);
        S += __popcll(mk);
      }
    }
    if (S < m || Q > kWavePieces || S > kWaveCap) {
      // Massive ties, or fewer than m sets with a number above fp32's -inf: the exact m-th largest
      // score, then the lowest slots among the candidates equal to it.  The search for its key starts at
      // the highest bit in which any two keys differ, and compares the scores as numbers (of NaNs it
      // knows only how many there are); slots go by row index, then column index.  2,048 Tucker pairs of
      // k = m = 64 with keys of zeros 77 us (32 with scores all different, 184 in the workgroup kernel),
      // 394 when every step made 64-bit keys anew and the slots were searched bit by bit.
      const bool on = lane < k;
      double hi = nan64, lo = nan64;
      int numbers = 0;
      for (int a = 0; a < k; ++a) {
        const double g = score(a);
        hi = fmax(hi, g);
        lo = fmin(lo, g);
        numbers += __popcll(__ballot(g == g));
      }
      const uint64_t hi_key = wave_max_u64(order_key64(hi)), lo_key = ~wave_max_u64(lo == lo ? ~order_key64(lo) : 0ull);
      const bool nans = numbers < m;                      // NaNs among the top-m, after every number
      double theta_at = nan64;
      if (!nans) {
        const int top = hi_key == lo_key ? -1 : 63 - __builtin_clzll(hi_key ^ lo_key);
        uint64_t theta = top < 0 ? hi_key : (top == 63 ? 0ull : hi_key >> (top + 1) << (top + 1));
#pragma unroll 1
        for (int bit = top; bit >= 0; --bit) {
          // (a key below the lowest score's is reached by all; one above the highest's, a number or
          // not, by none)
          const uint64_t c = theta | (1ull << bit);
          const double at = key64_value(c < lo_key ? lo_key : c);
          int cnt = 0;
          for (int a = 0; a < k; ++a) cnt += __popcll(__ballot(score(a) >= at));
          theta = cnt >= m ? c : theta;
          if (cnt == m) break;
        }
        theta_at = key64_value(theta < lo_key ? lo_key : theta);
      }
      int above = 0, ties = 0;                            // lane a: row a's candidates equal to theta
      for (int a = 0; a < k; ++a) {
        const double g = score(a);
        above += __popcll(__ballot(nans ? g == g : g > theta_at));
        const int row_ties = __popcll(__ballot(on && (nans ? g != g : g == theta_at)));
        ties = lane == a ? row_ties : ties;
      }
      const int row = s.ax_idx[min(lane, k - 1)], col = s.ax_idx[64 + min(lane, k - 1)];
      int before = 0;                                     // ties in rows of lower index
      for (int a = 0; a < k; ++a)
        before += __builtin_amdgcn_readlane(row, a) < row ? __builtin_amdgcn_readlane(ties, a) : 0;
      const int quota = max(0, min(ties, m - above - before));
      S = 0;
      for (int a = 0; a < k; ++a) {
        const double g = score(a);
        const bool tie = on && (nans ? g != g : g == theta_at);
        const uint64_t mt = __ballot(tie);
        const int n_take = __builtin_amdgcn_readlane(quota, a);
        bool take = nans ? g == g : g > theta_at;
        if (n_take == __popcll(mt)) {                     // (wave-uniform)
          take = take || tie;
        } else if (n_take > 0) {                          // the row with the last of them: by column
          int rank = 0;
          for (uint64_t x = mt; x != 0ull; x &= x - 1ull)
            rank += static_cast<int>(__builtin_amdgcn_readlane(col, __builtin_ctzll(x)) < col);
          take = take || (tie && rank < n_take);
        }
        const uint64_t mk = __ballot(take);
        if (take) s.ab[S + mask_rank(mk)] = static_cast<uint16_t>((a << 8) | lane);
        S += __popcll(mk);
      }
    }
    wave_lds_order();
  }
  S = __builtin_amdgcn_readfirstlane(S);
  // (about 100 survivors of the Tucker grid, 60 of the additive one)
  if (!TUCKER && S <= kWave) wave_finish<1, TUCKER>(A, s, S, pair, h);
  else if (S <= 2 * kWave) wave_finish<2, TUCKER>(A, s, S, pair, h);
  else wave_finish<4, TUCKER>(A, s, S, pair, h);
}

}  // namespace

int additive_candidates(int k, int m) {
  int c = 0;
  for (int a = 0; a < k && a < m; ++a) c += min(k, m / (a + 1));
  return c;
}

size_t select_lds_bytes(int n_cand, int tucker, int pool_dv) {
  const size_t axes = 2 * static_cast<size_t>(SMAX_AX) * 8;
  const size_t grid = static_cast<size_t>(tucker ? SMAX_S : 2 * n_cand) * sizeof(Cand);
  const size_t pool = static_cast<size_t>(NWAVES) * pool_dv * 4;
  return axes > grid ? (axes > pool ? axes : pool) : (grid > pool ? grid : pool);
}

bool select_pools(const umem_desc& d) {
  const int row_bytes = d.dv * (d.vdtype == UMEM_F32 ? 4 : 2);
  return d.expand == 1 && d.heads <= 2 && d.topm <= kMaxPoolTopM &&
         (row_bytes == 1024 || row_bytes == 2048);
}

hipError_t launch_select(const umem_desc& d, int T, const float* sel, const float* q_row,
                         const float* q_col, const float* k_row, const float* k_col,
                         const float* core, int32_t* idx, float* w, int32_t* axis_idx,
                         const void* values, float* pooled, hipStream_t s) {
  clear_stale_error();
  if (pooled != nullptr && !select_pools(d)) return hipErrorInvalidValue;
  if (T == 0) return hipSuccess;
  const int tucker = d.grid == UMEM_GRID_TUCKER;
  const int n_cand = tucker ? d.topk * d.topk : additive_candidates(d.topk, d.topm);
  if (tucker && n_cand > KK_MAX) return hipErrorInvalidValue;
  const size_t lds = select_lds_bytes(n_cand, tucker, pooled ? d.dv : 0);
  const int64_t pairs = static_cast<int64_t>(T) * d.heads;
  // A wave per pair from two waves per SIMD on: fewer leave its chain of steps (about 11 us, 23 with
  // the Tucker grid) longer than the workgroup kernel's, which spreads a pair over eight waves.
  // Measured (us, wave / workgroup kernel): additive, k = m = 32, 1,024 keys, 512 / 1,024 / 2,048 / 4,096
  // pairs 11.4 / 8.9, 11.8 / 11.6, 13.0 / 19.4, 17.2 / 33.6; 4,480 keys 15.7 / 10.3, 16.8 / 16.3, 23.1 / 27.0,
  // 40.9 / 48.3; Tucker, k = m = 64, 2,048 keys 23.5 / 17.5, 26.1 / 30.0, 30.7 / 49.7, 41.9 / 91.5; k = m = 42,
  // 448 dims 33.8 / 21.7, 36.3 / 35.8, 46.1 / 57.7, 87.7 / 106.  Beyond 2,048 keys the scores take 48 to 72
  // registers (four waves per SIMD up to 3,072 keys, three beyond, and the additive forms keep two or three
  // registers in scratch) and too few loads are in flight where the scores come from HBM: there the
  // 1,024-token decode forward (2,048 pairs of 4,480 keys) took 76.0 against 71.6; 8,192 pairs 69.2 / 90.6.
  const int64_t wave_pairs = d.n_keys > 2048 ? 8192 : 2048;
  if (pooled == nullptr && pairs >= wave_pairs && d.n_keys % 4 == 0 && d.n_keys <= kWaveMaxKeys &&
      d.topk <= kWaveMaxK && d.rank <= kWaveRank && d.n_keys >= 8 * d.topk && d.topm <= kWaveMaxM &&
      (tucker || n_cand <= kWaveCap)) {
    const WaveArgs A{sel, q_row, q_col, k_row, k_col, core, idx, w, axis_idx, T, d.heads, d.n_keys, d.dk,
                     d.rank, d.topk, d.topm, d.weight == UMEM_W_SOFTMAX, n_cores(d)};
    const int items = wave_items(tucker);
    const size_t bytes = items * wave_lds_bytes(tucker, d.rank, d.dk) + (tucker ? 0 : 2 * static_cast<size_t>(kWaveCap));
    const dim3 wgrid(static_cast<unsigned>((pairs + items - 1) / items)), wblock(items * kWave);
#define UMEM_SELECT_WAVE(NV)                                                                        \
  do {                                                                                            \
    if (tucker) hipLaunchKernelGGL((select_wave_kernel<NV, true>), wgrid, wblock, bytes, s, A);   \
    else hipLaunchKernelGGL((select_wave_kernel<NV, false>), wgrid, wblock, bytes, s, A);         \
  } while (0)
    const int nv = (d.n_keys + 255) / 256;
    if (nv <= 2) UMEM_SELECT_WAVE(2);
    else if (nv <= 4) UMEM_SELECT_WAVE(4);
    else if (nv <= 8) UMEM_SELECT_WAVE(8);
    else if (nv <= 12) UMEM_SELECT_WAVE(12);
    else UMEM_SELECT_WAVE(18);
#undef UMEM_SELECT_WAVE
    return hipGetLastError();
  }
  const dim3 grid(static_cast<unsigned>(T) * d.heads), block(THREADS);
#define UMEM_SELECT_P(NV, VEC, MODE)                                                              \
  hipLaunchKernelGGL((select_kernel<NV, VEC, MODE>), grid, block, lds, s, sel, q_row, q_col,     \
                     k_row, k_col, core, idx, w, axis_idx, values, d.vdtype == UMEM_BF16, d.dv,   \
                     pooled, T, d.heads, d.n_keys, d.dk, d.rank, d.topk,                         \
                     d.topm, tucker, d.weight == UMEM_W_SOFTMAX, n_cand, n_cores(d))
#define UMEM_SELECT(NV, VEC)                                                                      \
  do {                                                                                            \
    if (pooled != nullptr) UMEM_SELECT_P(NV, VEC, kModePool);                                     \
    else if (tucker) UMEM_SELECT_P(NV, VEC, kModeTucker);                                         \
    else UMEM_SELECT_P(NV, VEC, kModeAdd);                                                        \
  } while (0)
  const int n = d.n_keys;
  if (n % 4 == 0) {
    const int nv = (n + 1023) / 1024;
    if (nv <= 1) UMEM_SELECT(1, 4);
    else if (nv <= 2) UMEM_SELECT(2, 4);
    else if (nv <= 3) UMEM_SELECT(3, 4);
    else if (nv <= 4) UMEM_SELECT(4, 4);
    else if (nv <= 5) UMEM_SELECT(5, 4);
    else if (nv <= 6) UMEM_SELECT(6, 4);
    else if (nv <= 8) UMEM_SELECT(8, 4);
    else return hipErrorInvalidValue;
  } else {
    const int nv = (n + GROUP - 1) / GROUP;
    if (nv <= 1) UMEM_SELECT(1, 1);
    else if (nv <= 2) UMEM_SELECT(2, 1);
    else if (nv <= 4) UMEM_SELECT(4, 1);
    else if (nv <= 8) UMEM_SELECT(8, 1);
    else if (nv <= 16) UMEM_SELECT(16, 1);
    else if (nv <= 24) UMEM_SELECT(24, 1);
    else if (nv <= 32) UMEM_SELECT(32, 1);
    else return hipErrorInvalidValue;
  }
#undef UMEM_SELECT
#undef UMEM_SELECT_P
  return hipGetLastError();
}

}  // namespace umem
