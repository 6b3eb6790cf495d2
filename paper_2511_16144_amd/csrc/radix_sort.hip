// Stable LSD radix sort of (u32 key, u32 value) pairs on the device: the sort
// of visible Gaussians by depth and of (tile, Gaussian) pairs by tile that put
// every tile's list in front-to-back (depth, index) order.
//
// A pass is a digit histogram per block of keys, the sums of the blocks before
// each block, and a stable scatter.  Three forms:
//
// small (count bound <= the caller's small_max): what bounds so few keys is
//   launches, so there are as few as can be: digits of up to 11 bits, and two
//   launches a pass, the scatter adding up the histograms of the blocks before
//   its own by itself (2048 keys to a block).
// middle: digits of up to 8 bits, 1024 keys to a block (the more blocks, the
//   shorter each one's chain of loads, ballots and writes); a kernel between
//   the two turns each digit's row of block counts into its exclusive scan and
//   the digit's total.
// large (> kMiddleMax): the same with 4096 keys to a block, so that a block has
//   more keys to a digit and a line of the output is written in fewer parts.
//
// Inside a block the rank of a key among equal digits comes from wave64 match
// masks: one ballot per digit bit gives each lane the set of lanes holding its
// digit, the popcount of that set below the lane is its rank, and one leader
// lane per digit updates the wave's running count.  The histograms' atomics only
// count, so the order is that of the input for equal digits: deterministic and
// stable.
//
// Both sorts of a forward, with all launches (before: digits of 8 bits, 1024
// keys to a block, three launches a pass): 2000 ids, 4.8k pairs: 71 -> 50 us;
// 31k visible of 2^19, 0.61 M pairs: 86 -> 60; eight views, 1.04 M visible, 3.9 M
// pairs: 198 -> 150.  The lines: the small form on 100k visible takes 53 us and
// the middle one 50, on 30k 36 and 48; 4096 keys to a block take 9 us a pass in
// place of 5 for 0.4 M pairs, 16 in place of 21 for 3.9 M.
#include "lgs_internal.h"

#include <algorithm>
#include <utility>

namespace lgs {
namespace {

constexpr int kIters = 4;               // 64-key rows per wave
constexpr int kWaveKeys = 64 * kIters;  // 256
constexpr int kSmallThreads = 512, kMiddleThreads = 256, kLargeThreads = 1024;
constexpr int64_t kMiddleMax = 1ll << 20;
constexpr int kSmallBits = 11, kBits = 8;

// a pass's digits: 2^bits of them, rows of D >= 4 counts
struct Digits {
  int shift, bits, D;
};

__device__ __forceinline__ uint32_t digit_of(uint32_t k, const Digits& g) {
  return (k >> g.shift) & ((1u << g.bits) - 1u);
}

// lanes of `valid` whose digit equals this lane's (bits: digit width)
template <int MAXBITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t valid, int bits) {
  uint64_t peers = valid;
#pragma unroll
  for (int b = 0; b < MAXBITS; ++b)
    if (b < bits) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bal = __builtin_amdgcn_ballot_w64(bit);
      peers &= bit ? bal : ~bal;
    }
  return peers;
}

__device__ __forceinline__ int64_t count_of(const uint32_t* n_dev, int64_t n_max) {
  return n_dev ? (int64_t)*n_dev : n_max;
}

// exclusive scan over the threads of a block of THREADS, in thread order
template <int THREADS>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* sh, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(inc, off, 64);
    if (lane >= off) inc += y;
  }
  if (lane == 63) sh[wave] = inc;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    const uint32_t v = sh[w];
    if (w < wave) pre += v;
    tot += v;
  }
  __syncthreads();
  total = tot;
  return pre + inc - x;
}

// hist: [block][digit] when DIRECT, else [digit][block]
template <int THREADS, int MAXBITS, bool DIRECT>
__global__ void __launch_bounds__(THREADS) k_hist(const uint32_t* __restrict__ keys, const uint32_t* n_dev,
                                                  int64_t n_max, Digits g, uint32_t* __restrict__ hist) {
  constexpr int kTile = THREADS * kIters;
  __shared__ uint32_t cnt[1 << MAXBITS];
  const int64_t n = count_of(n_dev, n_max);
  const int64_t nb = (n + kTile - 1) / kTile;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  if (base >= n) return;
  // every key requested before the first is counted (unconditional loads at
  // indices clamped to the last key)
  uint32_t kr[kIters];
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int64_t i = base + it * THREADS + threadIdx.x;
    kr[it] = keys[i < n ? i : n - 1];
  }
  for (int d = threadIdx.x; d < g.D; d += THREADS) cnt[d] = 0u;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kIters; ++it)
    if (base + it * THREADS + threadIdx.x < n) atomicAdd(&cnt[digit_of(kr[it], g)], 1u);
  __syncthreads();
  for (int d = threadIdx.x; d < g.D; d += THREADS)
    hist[DIRECT ? (int64_t)blockIdx.x * g.D + d : (int64_t)d * nb + blockIdx.x] = cnt[d];
}

constexpr int kRowThreads = 256;
constexpr int kRowItems = 8;

// One work-group per digit d: the row hist[d][0 .. nb) becomes its exclusive
// scan in place (the number of keys with digit d in the blocks before each
// block) and dtot[d] the digit's total.
__global__ void __launch_bounds__(kRowThreads) k_row_scan(const uint32_t* n_dev, int64_t n_max, int tile,
                                                          uint32_t* __restrict__ hist, uint32_t* __restrict__ dtot) {
  __shared__ uint32_t sh[kRowThreads / 64];
  const int64_t n = count_of(n_dev, n_max);
  const int64_t nb = (n + tile - 1) / tile;
  uint32_t* row = hist + (int64_t)blockIdx.x * nb;
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += (int64_t)kRowThreads * kRowItems) {
    const int64_t i0 = b0 + (int64_t)threadIdx.x * kRowItems;
    // every item requested before any is added (clamped unconditional loads)
    uint32_t v[kRowItems];
#pragma unroll
    for (int k = 0; k < kRowItems; ++k) v[k] = row[i0 + k < nb ? i0 + k : nb - 1];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kRowItems; ++k) {
      v[k] = i0 + k < nb ? v[k] : 0u;
      sum += v[k];
    }
    uint32_t tot;
    uint32_t run = carry + block_excl_scan<kRowThreads>(sum, sh, tot);
#pragma unroll
    for (int k = 0; k < kRowItems; ++k) {
      if (i0 + k < nb) row[i0 + k] = run;
      run += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

// hist, dtot: the row scan's; when DIRECT, the histograms themselves
template <int THREADS, int MAXBITS, bool DIRECT>
__global__ void __launch_bounds__(THREADS) k_scatter(const uint32_t* __restrict__ kin,
                                                     const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                     uint32_t* __restrict__ vout, const uint32_t* n_dev,
                                                     int64_t n_max, Digits g, const uint32_t* __restrict__ hist,
                                                     const uint32_t* __restrict__ dtot) {
  constexpr int kTile = THREADS * kIters, kWaves = THREADS / 64;
  constexpr int kOwn = 4;   // digits to a thread
  static_assert(kOwn * THREADS >= (1 << MAXBITS), "every digit has its thread");
  // a wave's keys of a digit, then those of the waves before it (two counts to a word where that pays)
  __shared__ alignas(16) uint16_t cnt[kWaves][1 << MAXBITS];
  __shared__ uint32_t first[1 << MAXBITS];         // position of the block's first key of a digit
  __shared__ uint32_t sh[kWaves];
  const int64_t n = count_of(n_dev, n_max);
  const int64_t nb = (n + kTile - 1) / kTile;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  if (base >= n) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t kk[kIters], vv[kIters];
  // all of the wave's keys and values are requested before the first key is
  // ranked (unconditional loads at indices clamped to the last key)
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int64_t i = base + wave * kWaveKeys + it * 64 + lane;
    const int64_t ic = i < n ? i : n - 1;
    kk[it] = kin[ic];
    vv[it] = vin[ic];
  }
  // this thread's digits d0 .. d0 + kOwn - 1: their totals and their keys in
  // the blocks before this one
  const int d0 = kOwn * (int)threadIdx.x;
  const bool owner = d0 < g.D;
  uint32_t tot[kOwn] = {}, pre[kOwn] = {};
  if (owner) {
    if constexpr (DIRECT) {
      constexpr int kRows = 8;
      for (int64_t b0 = 0; b0 < nb; b0 += kRows) {
        uint4 v[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) v[r] = *(const uint4*)(hist + (b0 + r < nb ? b0 + r : nb - 1) * g.D + d0);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
          const bool in = b0 + r < nb, before = b0 + r < (int64_t)blockIdx.x;
          const uint32_t x[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            tot[k] += in ? x[k] : 0u;
            pre[k] += before ? x[k] : 0u;
          }
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {
        tot[k] = dtot[d0 + k];
        pre[k] = hist[(int64_t)(d0 + k) * nb + blockIdx.x];
      }
    }
  }
  for (int d = lane; d < g.D / 2; d += 64) ((uint32_t*)cnt[wave])[d] = 0u;
  // (words and halves are distinct types to the compiler: without the fence it
  // may count before it clears)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint64_t peers[kIters];
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int64_t i = base + wave * kWaveKeys + it * 64 + lane;
    const bool ok = i < n;
    const uint32_t d = digit_of(kk[it], g);
    peers[it] = match_digit<MAXBITS>(d, __builtin_amdgcn_ballot_w64(ok), g.bits);
    if (ok && (peers[it] & lt) == 0ull) cnt[wave][d] += (uint16_t)__popcll(peers[it]);
    __builtin_amdgcn_wave_barrier();
  }
  uint32_t all, mine = 0u;
#pragma unroll
  for (int k = 0; k < kOwn; ++k) mine += tot[k];
  uint32_t run = block_excl_scan<THREADS>(mine, sh, all);
  if (owner) {
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      first[d0 + k] = run + pre[k];
      run += tot[k];
    }
#pragma unroll
    for (int k = 0; k < kOwn; k += 2) {   // (two digits to a word: a block's counts stay below 2^16)
      uint32_t a = 0u, b = 0u;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        uint32_t* at = (uint32_t*)&cnt[w][d0 + k];
        const uint32_t c = *at;
        *at = a | b << 16;
        a += c & 0xffffu;
        b += c >> 16;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int64_t i = base + wave * kWaveKeys + it * 64 + lane;
    const bool ok = i < n;
    const uint32_t d = digit_of(kk[it], g);
    const uint32_t rank = (uint32_t)__popcll(peers[it] & lt);
    const uint32_t c = cnt[wave][d];
    __builtin_amdgcn_wave_barrier();
    if (ok) {
      const uint32_t pos = first[d] + c + rank;
      kout[pos] = kk[it];
      vout[pos] = vv[it];
      if (rank == 0u) cnt[wave][d] = (uint16_t)(c + (uint32_t)__popcll(peers[it]));
    }
    __builtin_amdgcn_wave_barrier();
  }
}

int64_t blocks_of(int64_t n_max, int threads) {
  const int64_t tile = (int64_t)threads * kIters;
  return n_max > 0 ? (n_max + tile - 1) / tile : 1;
}

// block counts (2^bits x blocks) and the digits' totals
size_t temp_words(int64_t n_max, int threads, int bits) { return ((size_t)blocks_of(n_max, threads) + 1) << bits; }

// a sort's buffers; run: its passes in one form, whether the result is in the
// alternate buffers
struct Sort {
  uint32_t *keys, *vals, *keys_alt, *vals_alt;
  const uint32_t* n_dev;
  int64_t n_max;
  uint32_t* temp;
  hipStream_t s;

  template <int THREADS, int BITS, bool DIRECT>
  bool run(int begin_bit, int end_bit) {
    const int total = end_bit - begin_bit, passes = (total + BITS - 1) / BITS;
    const dim3 nb((unsigned)blocks_of(n_max, THREADS));
    uint32_t* const dtot = temp + ((size_t)nb.x << BITS);
    for (int p = 0; p < passes; ++p) {
      const int lo = begin_bit + total * p / passes, hi = begin_bit + total * (p + 1) / passes;   // in equal parts
      const Digits g{lo, hi - lo, std::max(1 << (hi - lo), 4)};
      hipLaunchKernelGGL((k_hist<THREADS, BITS, DIRECT>), nb, dim3(THREADS), 0, s, (const uint32_t*)keys, n_dev,
                         n_max, g, temp);
      if (!DIRECT)
        hipLaunchKernelGGL(k_row_scan, dim3((unsigned)g.D), dim3(kRowThreads), 0, s, n_dev, n_max, THREADS * kIters,
                           temp, dtot);
      hipLaunchKernelGGL((k_scatter<THREADS, BITS, DIRECT>), nb, dim3(THREADS), 0, s, (const uint32_t*)keys,
                         (const uint32_t*)vals, keys_alt, vals_alt, n_dev, n_max, g, (const uint32_t*)temp,
                         (const uint32_t*)dtot);
      std::swap(keys, keys_alt);
      std::swap(vals, vals_alt);
    }
    return passes % 2 != 0;
  }
};

}  // namespace

size_t radix_temp_bytes(int64_t n_max, int64_t small_max) {
  return sizeof(uint32_t) * (n_max <= small_max    ? temp_words(n_max, kSmallThreads, kSmallBits)
                             : n_max <= kMiddleMax ? temp_words(n_max, kMiddleThreads, kBits)
                                                   : temp_words(n_max, kLargeThreads, kBits));
}

void radix_sort_u32(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                    const uint32_t* n_dev, int64_t n_max, int64_t small_max, int begin_bit, int end_bit, void* temp,
                    hipStream_t s, bool* in_alt) {
  *in_alt = false;
  if (n_max <= 0 || end_bit <= begin_bit) return;
  Sort t{keys, vals, keys_alt, vals_alt, n_dev, n_max, (uint32_t*)temp, s};
  *in_alt = n_max <= small_max    ? t.run<kSmallThreads, kSmallBits, true>(begin_bit, end_bit)
            : n_max <= kMiddleMax ? t.run<kMiddleThreads, kBits, false>(begin_bit, end_bit)
                                  : t.run<kLargeThreads, kBits, false>(begin_bit, end_bit);
}

}  // namespace lgs
