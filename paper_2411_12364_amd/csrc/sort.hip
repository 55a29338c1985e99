// Stable sort of the positions 0 .. M-1 by a 32-bit unsigned key each: least-significant-digit
// radix sort in as few passes of at most 11-bit digits as the key width needs (ceil(bits / 11)
// passes of ceil(bits / passes) bits: 20-bit row keys in two passes of 10).  The backward passes
// use it to bring all contributions to one value row (or key row) together, in their original
// order, so that each row is summed in a fixed order and the gradient does not depend on timing.
// A skip key drops its positions on the way: they are neither counted nor written.
//
// The arrays are small (tens of thousands to a few million pairs), so each pass is a chain of
// short, latency-bound kernels, and what counts is how few round trips and barriers each holds.
// Per pass, over tiles of 8 waves x steps x 64 pairs, with 2^D digit values:
//  * sort_hist_kernel: the tile's digit histogram (LDS atomics), stored digit-major
//    [2^D][tiles].  The caller may fold the first one into the kernel that makes the keys
//    (sort_tile_hist);
//  * sort_scan_kernel: a wave per digit turns its row of tile counts into exclusive offsets
//    within the digit and leaves the digit's total;
//  * sort_scatter_kernel: every workgroup scans the 2^D totals itself (LDS), so no kernel stands
//    between; each wave then ranks its own 64 x steps consecutive pairs without a barrier: a
//    pair's rank is its wave's running count of the digit (LDS, the wave's own row) + its rank
//    among equal digits of its step (D ballots match the digit).  Two barriers and a prefix over
//    the eight waves' counts later every pair knows its place and leaves as one 8-byte
//    (key, position) store.
// Before, every step of 256 pairs ended in two workgroup barriers, the counts were scanned by two
// kernels and keys and values left as two stores: one pass (histogram, scan, scatter) took 33.5 us
// for 131,072 pairs of 10-bit digits and 42 us for 1,048,576; it now takes 18 us and 23 - 29 us.
#include <algorithm>

#include "umem_internal.h"

namespace umem {
namespace {

constexpr int kThreads = kSortThreads;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxDigits = 1 << kSortMaxDigitBits;

__device__ __forceinline__ uint64_t lanes_below() {
  const unsigned lane = threadIdx.x & (kWave - 1);
  return lane == 0 ? 0ull : (~0ull >> (kWave - lane));
}

__global__ __launch_bounds__(kThreads) void sort_hist_kernel(const uint2* __restrict__ pairs,
                                                             const uint32_t* __restrict__ keys,
                                                             int M, const uint32_t* __restrict__ n,
                                                             uint32_t skip, int shift, int dbits,
                                                             uint32_t* __restrict__ hist, int tiles,
                                                             int tile) {
  __shared__ uint32_t cnt[kMaxDigits];
  const int nd = 1 << dbits;
  const uint32_t mask = static_cast<uint32_t>(nd - 1);
  const int count = n != nullptr ? static_cast<int>(*n) : M;      // of a later pass: without the skipped
  for (int d = threadIdx.x; d < nd; d += kThreads) cnt[d] = 0;
  __syncthreads();
  const int base = blockIdx.x * tile, end = min(base + tile, count);
  for (int pos = base + static_cast<int>(threadIdx.x); pos < end; pos += kThreads) {
    const uint32_t key = pairs != nullptr ? pairs[pos].x : keys[pos];
    if (pairs != nullptr || key != skip) atomicAdd(&cnt[(key >> shift) & mask], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < nd; d += kThreads)
    hist[static_cast<size_t>(d) * tiles + blockIdx.x] = cnt[d];
}

// Digit d's tile counts hist[d][0, tiles) to exclusive prefix sums, their total to tot[d]; a wave
// per digit, 64 tiles per step.
__global__ __launch_bounds__(256) void sort_scan_kernel(uint32_t* __restrict__ hist, int nd, int tiles,
                                                        uint32_t* __restrict__ tot) {
  const int lane = threadIdx.x & (kWave - 1);
  const int d = blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
  if (d >= nd) return;                                    // whole waves: no barrier in this kernel
  uint32_t* row = hist + static_cast<size_t>(d) * tiles;
  uint32_t run = 0;
  for (int t0 = 0; t0 < tiles; t0 += kWave) {
    const int t = t0 + lane;
    const uint32_t c = t < tiles ? row[t] : 0u;
    const uint32_t incl = static_cast<uint32_t>(wave_inclusive_scan(static_cast<int>(c)));
    if (t < tiles) row[t] = run + incl - c;
    run += static_cast<uint32_t>(__shfl(static_cast<int>(incl), kWave - 1, kWave));
  }
  if (lane == 0) tot[d] = run;
}

// FIRST: from keys[0, M), the pair of position pos being (keys[pos], pos); else from *n pairs.
template <int STEPS, bool FIRST>
__global__ __launch_bounds__(kThreads) void sort_scatter_kernel(
    const uint32_t* __restrict__ keys, const uint2* __restrict__ in, uint2* __restrict__ out, int M,
    uint32_t* __restrict__ n, uint32_t skip, int shift, int dbits, const uint32_t* __restrict__ offs,
    const uint32_t* __restrict__ tot, int tiles) {
  __shared__ uint32_t base[kMaxDigits];                   // the tile's first place of each digit
  __shared__ uint16_t wcnt[kWaves][kMaxDigits];           // counts, then places before each wave
  __shared__ uint32_t wsum[kWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int nd = 1 << dbits;
  const uint32_t mask = static_cast<uint32_t>(nd - 1);
  const int count = FIRST ? M : static_cast<int>(*n);
  const int first = (blockIdx.x * kWaves + wave) * (STEPS * kWave) + lane;
  uint2 pr[STEPS];
  bool valid[STEPS];
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const int pos = first + q * kWave;
    valid[q] = pos < count;
    if (FIRST) {
      pr[q] = make_uint2(valid[q] ? keys[pos] : 0u, static_cast<uint32_t>(pos));
      valid[q] = valid[q] && pr[q].x != skip;
    } else {
      pr[q] = valid[q] ? in[pos] : make_uint2(0u, 0u);
    }
  }
  // the digits' first places: an exclusive scan of the totals, kPer consecutive digits a thread
  constexpr int kPer = kMaxDigits / kThreads;
  uint32_t loc[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int d = tid * kPer + k;
    loc[k] = d < nd ? tot[d] : 0u;
    sum += loc[k];
  }
  const uint32_t incl = static_cast<uint32_t>(wave_inclusive_scan(static_cast<int>(sum)));
  if (lane == kWave - 1) wsum[wave] = incl;
  for (int d = lane; d < nd; d += kWave) wcnt[wave][d] = 0;       // the wave's own row
  __syncthreads();
  uint32_t run = incl - sum;
  uint32_t total = 0;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) {
    run += v < wave ? wsum[v] : 0u;
    total += wsum[v];
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int d = tid * kPer + k;
    if (d < nd) base[d] = run + (tiles > 1 ? offs[static_cast<size_t>(d) * tiles + blockIdx.x] : 0u);
    run += loc[k];
  }
  if (FIRST && blockIdx.x == 0 && tid == 0) *n = total;
  uint32_t rank[STEPS];
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const uint32_t digit = (pr[q].x >> shift) & mask;
    uint64_t peers = __ballot(valid[q]);
    for (int b = 0; b < dbits; ++b) {
      const bool one = (digit >> b) & 1u;
      const uint64_t ones = __ballot(one);
      peers &= one ? ones : ~ones;
    }
    const uint32_t before = static_cast<uint32_t>(__popcll(peers & lanes_below()));
    const uint32_t have = wcnt[wave][digit];
    rank[q] = have + before;
    wave_lds_order();
    if (valid[q] && before == 0) wcnt[wave][digit] = static_cast<uint16_t>(have + __popcll(peers));
    wave_lds_order();
  }
  __syncthreads();
  for (int d = tid; d < nd; d += kThreads) {
    uint32_t at = 0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      const uint32_t c = wcnt[v][d];
      wcnt[v][d] = static_cast<uint16_t>(at);             // below a tile's 4096 pairs
      at += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const uint32_t digit = (pr[q].x >> shift) & mask;
    if (valid[q]) out[base[digit] + wcnt[wave][digit] + rank[q]] = pr[q];
  }
}

// Tiles of 2048 pairs (half the steps in each wave's chain, twice the workgroups) where there are
// several; up to 4096 pairs one tile needs no scan, and from 2^19 pairs on the chip is full either
// way and tiles of 4096 halve the counts to scan.
int sort_steps(int M) { return M > 4096 && M < (1 << 19) ? 4 : 8; }

// One tile's counts are its totals: they share their place, and no scan runs.
size_t count_words(int tiles) {
  return tiles > 1 ? static_cast<size_t>(kMaxDigits) * (tiles + 1) : kMaxDigits;
}

}  // namespace

SortPlan sort_plan(int M, int bits, void* ws) {
  SortPlan p;
  p.M = M;
  p.tile = kSortThreads * sort_steps(M);
  p.tiles = (M + p.tile - 1) / p.tile;
  p.passes = bits <= 0 ? 1 : (bits + kSortMaxDigitBits - 1) / kSortMaxDigitBits;
  p.dbits = bits <= 0 ? 1 : (bits + p.passes - 1) / p.passes;     // <= kSortMaxDigitBits
  p.a = static_cast<uint2*>(ws);
  p.b = p.a + M;
  p.keys = reinterpret_cast<uint32_t*>(p.b);
  p.n = reinterpret_cast<uint32_t*>(p.b + M);
  p.tot = p.n + 16;
  p.hist = p.tiles > 1 ? p.tot + kMaxDigits : p.tot;
  p.spare = p.n + 16;
  return p;
}

size_t sort_workspace_bytes(int M) {
  const int tile = kSortThreads * sort_steps(M);
  const size_t words = std::max(count_words((M + tile - 1) / tile), static_cast<size_t>(M));
  return 2 * static_cast<size_t>(M) * sizeof(uint2) + (16 + words) * sizeof(uint32_t);
}

hipError_t sort_run(const SortPlan& p, uint32_t skip, bool have_hist, hipStream_t s, uint2** sorted,
                    uint2** dead) {
  uint2 *in = p.b, *out = p.a;                            // the first pass reads p.keys, not p.b
  const int nd = 1 << p.dbits;
  for (int pass = 0; pass < p.passes; ++pass) {
    const int shift = p.dbits * pass;
    const bool first = pass == 0;
    if (!first || !have_hist)
      hipLaunchKernelGGL(sort_hist_kernel, dim3(p.tiles), dim3(kThreads), 0, s, first ? nullptr : in,
                         p.keys, p.M, first ? nullptr : p.n, skip, shift, p.dbits, p.hist, p.tiles, p.tile);
    if (p.tiles > 1)
      hipLaunchKernelGGL(sort_scan_kernel, dim3((nd + 3) / 4), dim3(256), 0, s, p.hist, nd, p.tiles, p.tot);
#define UMEM_SCATTER(STEPS, FIRST)                                                                  \
  hipLaunchKernelGGL((sort_scatter_kernel<STEPS, FIRST>), dim3(p.tiles), dim3(kThreads), 0, s, p.keys, \
                     in, out, p.M, p.n, skip, shift, p.dbits, p.hist, p.tot, p.tiles)
    if (p.tile == kThreads * 4) {
      if (first) UMEM_SCATTER(4, true);
      else UMEM_SCATTER(4, false);
    } else {
      if (first) UMEM_SCATTER(8, true);
      else UMEM_SCATTER(8, false);
    }
#undef UMEM_SCATTER
    uint2* t = in;
    in = out;
    out = t;
  }
  *sorted = in;
  *dead = out;
  return hipGetLastError();
}

}  // namespace umem
