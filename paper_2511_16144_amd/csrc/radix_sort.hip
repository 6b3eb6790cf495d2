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
//   its own by itself (2048 keys to a block).  So that this stays short for any
//   count, threads with no digits of their own share the rows, and past some
//   100k keys the histogram kernel adds up groups of blocks.
// middle: digits of up to 8 bits, 1024 keys to a block (the more blocks, the
//   shorter each one's chain of loads, ballots and writes); a kernel between
//   the two turns each digit's row of block counts into its exclusive scan and
//   the digit's total.
// large (> kMiddleMax): the same with up to 4096 keys to a block, so that a block
//   has more keys to a digit and a line of the output is written in fewer parts;
//   fewer where the count, of which the host knows only the bound, is small.
//
// Inside a block the rank of a key among equal digits comes from wave64 match
// masks: one ballot per digit bit gives each lane the set of lanes holding its
// digit, the popcount of that set below the lane is its rank, and one leader
// lane per digit updates the wave's running count.  The histograms' atomics only
// count, so the order is that of the input for equal digits: deterministic and
// stable.
//
// Times of a sort with all launches, us, in this form and in the middle one (by
// itself, which is the form of 8 bits, 1024 keys and three launches a pass for
// every count):
//   ids (32 bits), visible of bound:  2.6k of 2^17 28, 38; 52k of 2^19 39, 45;
//     131k of 2^19 43, 49; 262k of 2^19 53, 56; 2^19 of 2^19 71, 70;
//     2^20 of 2^20 (middle) 106, 111;
//     84k of 2^22 47, 49; 419k of 2^22 62, 66; 2.1 M of 2^22 139, 179; all of 2^22 235, 297
//   pairs: 30k of 11 bits 11, 22; 127k of 8 bits 11, 12, of 11 17, 23, of 14 20, 23;
//     500k of 11 bits 25, 30; 4 M of 11 bits 80, 92
// (A scatter that reads all blocks' histograms takes 122 us for all of 2^19 ids
// and 26 for 127k pairs of 14 bits; blocks of 4096 keys at any count 61 us for 84k
// of 2^22.)
#include "lgs_internal.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace lgs {
namespace {

constexpr int kIters = 4;               // 64-key rows per wave
constexpr int kSmallThreads = 512, kMiddleThreads = 256, kLargeThreads = 1024;
constexpr int64_t kMiddleMax = 1ll << 20;
constexpr int kSmallBits = 11, kBits = 8;
constexpr int kOwn = 4;                 // a thread's digits in the scatter

// a pass's digits: 2^bits of them, rows of D >= 4 counts
struct Digits {
  int shift, bits, D;
  __device__ __forceinline__ int log2_quads() const { return max(bits, 2) - 2; }   // of D / kOwn
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

// How the count decides a pass, alike in all of its kernels.
//
// DIRECT: tiles of 2048 keys.  Threads that share the rows of a digit in the
// scatter: where a row has digits for a quarter of the threads or fewer, and
// more rows than two of a thread's batches (127k pairs, 8 bits: 13.7 -> 11.0 us;
// 16 tiles: 9.7, with them 10.3).  Tiles that a block of the histogram takes: one
// while a thread has at most 48 rows to add up (64 rows: 131k ids 50 us, in fours
// 43; 32 rows: 38 and 39), eights past 128 (256 tiles: 71, in fours 76).  Both as
// powers of two.
constexpr int kMinTiles = 4;
__device__ __forceinline__ int log2_sharers(uint32_t tiles, const Digits& g) {
  constexpr int kLog2Threads = 9;
  static_assert(1 << kLog2Threads == kSmallThreads, "a power of two");
  const int s = kLog2Threads - g.log2_quads();
  return tiles <= 16u || s < 2 ? 0 : s;
}
__device__ __forceinline__ int log2_tiles(uint32_t tiles, const Digits& g) {
  const uint32_t rows = tiles >> log2_sharers(tiles, g);
  return rows <= 48u ? 0 : rows <= 128u ? 2 : 3;
}
// Else: rows of 64 keys to a wave; blocks of 1024 threads take as many as leave
// the chip full (419k keys: one row 74 us, two 62, four 68; 210k: 51 with one, 63
// with four).
constexpr int64_t kOneRow = 1ll << 18, kTwoRows = 1ll << 19;
template <int THREADS>
__host__ __device__ constexpr int iters_of(int64_t n) {
  return THREADS != kLargeThreads ? kIters : n <= kOneRow ? 1 : n <= kTwoRows ? 2 : kIters;
}
// f(the iterations, known to the compiler)
template <int THREADS, class F>
__device__ __forceinline__ void with_iters(int64_t n, F f) {
  const int iters = iters_of<THREADS>(n);
  if constexpr (THREADS == kLargeThreads) {
    if (iters == 1) return f(std::integral_constant<int, 1>());
    if (iters == 2) return f(std::integral_constant<int, 2>());
  }
  f(std::integral_constant<int, kIters>());
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

// hist: [digit][block]; when DIRECT [block][digit] and, in groups of tiles, the
// keys of the group's tiles before each tile, followed by the groups' totals
template <int THREADS, int MAXBITS, bool DIRECT>
__global__ void __launch_bounds__(THREADS) k_hist(const uint32_t* __restrict__ keys, const uint32_t* n_dev,
                                                  int64_t n_max, Digits g, uint32_t* __restrict__ hist) {
  __shared__ uint32_t cnt[1 << MAXBITS];
  const int64_t n = count_of(n_dev, n_max);
  with_iters<THREADS>(n, [&](auto iters_tag) {
    constexpr int iters = decltype(iters_tag)::value, kTile = THREADS * iters;
    const int64_t nb = (n + kTile - 1) / kTile;
    const int per = DIRECT ? 1 << log2_tiles((uint32_t)nb, g) : 1;
    const int64_t first = (int64_t)blockIdx.x * per;
    if (first >= nb) return;
    // every key of a tile requested before the first is counted (unconditional
    // loads at indices clamped to the last key)
    uint32_t kr[iters];
    auto request = [&](int64_t t) {
#pragma unroll
      for (int it = 0; it < iters; ++it) {
        const int64_t i = t * kTile + it * THREADS + threadIdx.x;
        kr[it] = keys[i < n ? i : n - 1];
      }
    };
    auto count = [&](int64_t t) {
#pragma unroll
      for (int it = 0; it < iters; ++it)
        if (t * kTile + it * THREADS + threadIdx.x < n) atomicAdd(&cnt[digit_of(kr[it], g)], 1u);
    };
    auto store = [&](int64_t row) {
      for (int d = threadIdx.x; d < g.D; d += THREADS) hist[DIRECT ? row * g.D + d : (int64_t)d * nb + row] = cnt[d];
    };
    request(first);
    for (int d = threadIdx.x; d < g.D; d += THREADS) cnt[d] = 0u;
    __syncthreads();
    if (!DIRECT || per == 1) {
      count(first);
      __syncthreads();
      store(first);
      return;
    }
    const int64_t end = first + per < nb ? first + per : nb;
    for (int64_t t = first; t < end; ++t) {
      store(t);
      __syncthreads();
      count(t);
      if (t + 1 < end) request(t + 1);
      __syncthreads();
    }
    store(nb + blockIdx.x);
  });
}

constexpr int kRowThreads = 256;
constexpr int kRowItems = 8;

// One work-group per digit d: the row hist[d][0 .. nb) becomes its exclusive
// scan in place (the number of keys with digit d in the blocks before each
// block) and dtot[d] the digit's total.
template <int THREADS>
__global__ void __launch_bounds__(kRowThreads) k_row_scan(const uint32_t* n_dev, int64_t n_max,
                                                          uint32_t* __restrict__ hist, uint32_t* __restrict__ dtot) {
  __shared__ uint32_t sh[kRowThreads / 64];
  const int64_t n = count_of(n_dev, n_max), tile = (int64_t)THREADS * iters_of<THREADS>(n);
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

// The sums of a digit's rows before and over all tiles, for the kOwn digits of a
// thread of the DIRECT scatter.
template <int THREADS>
__device__ __forceinline__ void add_rows(const Digits& g, const uint32_t* __restrict__ hist, uint32_t nb,
                                         uint32_t (*part)[THREADS], uint32_t (&tot)[kOwn], uint32_t (&pre)[kOwn]) {
  constexpr uint32_t kRows = 8;
  const int per = log2_tiles(nb, g);
  const uint32_t share = 1u << log2_sharers(nb, g), from = threadIdx.x >> g.log2_quads();
  const uint32_t q = threadIdx.x & ((1u << g.log2_quads()) - 1u);
  // the tiles' histograms, or the groups' and what the own group has before this tile
  const uint32_t rows = (nb + (1u << per) - 1u) >> per, own = blockIdx.x >> per;
  const uint4* h = (const uint4*)(hist + (per ? (size_t)nb * g.D : 0)) + q;
  if (from < share) {
    if (per && from == 0u) {
      const uint4 v = ((const uint4*)(hist + (size_t)blockIdx.x * g.D))[q];
      pre[0] = v.x, pre[1] = v.y, pre[2] = v.z, pre[3] = v.w;
    }
    for (uint32_t b0 = from; b0 < rows; b0 += kRows * share) {
      uint4 v[kRows];
#pragma unroll
      for (uint32_t r = 0; r < kRows; ++r) v[r] = h[(size_t)min(b0 + r * share, rows - 1u) << g.log2_quads()];
#pragma unroll
      for (uint32_t r = 0; r < kRows; ++r) {
        const uint32_t b = b0 + r * share;
        const bool in = b < rows, before = b < own;
        const uint32_t x[kOwn] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
          tot[k] += in ? x[k] : 0u;
          pre[k] += before ? x[k] : 0u;
        }
      }
    }
  }
  if (share == 1u) return;
  for (int d = threadIdx.x; d < g.D; d += THREADS) part[0][d] = part[1][d] = 0u;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    if (from < share) {
      atomicAdd(&part[0][kOwn * q + k], tot[k]);
      atomicAdd(&part[1][kOwn * q + k], pre[k]);
    }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {   // (of threads without digits of their own: not used, but tot)
    tot[k] = from == 0u ? part[0][kOwn * q + k] : 0u;
    pre[k] = part[1][kOwn * q + k];
  }
}

// hist, dtot: the row scan's; when DIRECT, the histograms themselves
template <int THREADS, int MAXBITS, bool DIRECT>
__global__ void __launch_bounds__(THREADS) k_scatter(const uint32_t* __restrict__ kin,
                                                     const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                     uint32_t* __restrict__ vout, const uint32_t* n_dev,
                                                     int64_t n_max, Digits g, const uint32_t* __restrict__ hist,
                                                     const uint32_t* __restrict__ dtot) {
  constexpr int kWaves = THREADS / 64;
  static_assert(kOwn * THREADS >= (1 << MAXBITS), "every digit has its thread");
  // a wave's keys of a digit, then those of the waves before it (two counts to a word where that pays)
  __shared__ alignas(16) uint16_t cnt[kWaves][1 << MAXBITS];
  __shared__ uint32_t first[1 << MAXBITS];         // position of the block's first key of a digit
  __shared__ uint32_t sh[kWaves];
  __shared__ uint32_t part[2][DIRECT ? THREADS : 1];
  const int64_t n = count_of(n_dev, n_max);
  with_iters<THREADS>(n, [&](auto iters_tag) {
    constexpr int iters = decltype(iters_tag)::value, kTile = THREADS * iters;
    const int64_t nb = (n + kTile - 1) / kTile;
    const int64_t base = (int64_t)blockIdx.x * kTile;
    if (base >= n) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t kk[iters], vv[iters];
    // all of the wave's keys and values are requested before the first key is
    // ranked (unconditional loads at indices clamped to the last key)
    auto index = [&](int it) { return base + wave * 64 * iters + it * 64 + lane; };
#pragma unroll
    for (int it = 0; it < iters; ++it) {
      const int64_t i = index(it), ic = i < n ? i : n - 1;
      kk[it] = kin[ic];
      vv[it] = vin[ic];
    }
    // this thread's digits d0 .. d0 + kOwn - 1: their totals and their keys in
    // the blocks before this one
    const int d0 = kOwn * (int)threadIdx.x;
    const bool owner = d0 < g.D;
    uint32_t tot[kOwn] = {}, pre[kOwn] = {};
    if constexpr (DIRECT) {
      add_rows<THREADS>(g, hist, (uint32_t)nb, part, tot, pre);
    } else if (owner) {
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {
        tot[k] = dtot[d0 + k];
        pre[k] = hist[(int64_t)(d0 + k) * nb + blockIdx.x];
      }
    }
    for (int d = lane; d < g.D / 2; d += 64) ((uint32_t*)cnt[wave])[d] = 0u;
    // (words and halves are distinct types to the compiler: without the fence it
    // may count before it clears)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t peers[iters];
#pragma unroll
    for (int it = 0; it < iters; ++it) {
      const bool ok = index(it) < n;
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
    for (int it = 0; it < iters; ++it) {
      const bool ok = index(it) < n;
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
  });
}

// blocks for any count up to n_max
template <int THREADS>
int64_t blocks_of(int64_t n_max) {
  auto at = [](int64_t n) { return (n + THREADS * iters_of<THREADS>(n) - 1) / (THREADS * iters_of<THREADS>(n)); };
  return std::max<int64_t>(1, std::max({at(n_max), at(std::min(n_max, kOneRow)), at(std::min(n_max, kTwoRows))}));
}

// block counts (2^bits x blocks), and the digits' totals or the groups'
template <int THREADS>
size_t temp_words(int64_t n_max, int bits) {
  const int64_t nb = blocks_of<THREADS>(n_max);
  return (size_t)(nb + (nb + kMinTiles - 1) / kMinTiles) << bits;
}

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
    const dim3 nb((unsigned)blocks_of<THREADS>(n_max));
    uint32_t* const dtot = temp + ((size_t)nb.x << BITS);
    for (int p = 0; p < passes; ++p) {
      const int lo = begin_bit + total * p / passes, hi = begin_bit + total * (p + 1) / passes;   // in equal parts
      const Digits g{lo, hi - lo, std::max(1 << (hi - lo), 4)};
      hipLaunchKernelGGL((k_hist<THREADS, BITS, DIRECT>), nb, dim3(THREADS), 0, s, (const uint32_t*)keys, n_dev,
                         n_max, g, temp);
      if (!DIRECT)
        hipLaunchKernelGGL(k_row_scan<THREADS>, dim3((unsigned)g.D), dim3(kRowThreads), 0, s, n_dev, n_max, temp,
                           dtot);
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
  return sizeof(uint32_t) * (n_max <= small_max    ? temp_words<kSmallThreads>(n_max, kSmallBits)
                             : n_max <= kMiddleMax ? temp_words<kMiddleThreads>(n_max, kBits)
                                                   : temp_words<kLargeThreads>(n_max, kBits));
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
