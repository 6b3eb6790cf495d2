// Tile binning (the step between projection and compositing): device-wide
// exclusive scans, compaction of the visible (view, Gaussian) ids, the
// load-balanced emission of (tile, Gaussian) pairs in depth order, and the
// per-tile [start, end) ranges of the tile-sorted pair list.
//
// Every kernel reads its element count from device memory, so the same
// launches serve the eager path (grid sized to the exact count) and the
// captured graph (grid sized to a capacity; blocks past the count exit).
#include "lgs_internal.h"

namespace lgs {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;   // 2048

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, int lane) {
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  return x;
}

// exclusive scan of one value per thread over a 256-thread block
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* sh, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(x, lane);
  if (lane == 63) sh[wave] = inc;
  __syncthreads();
  uint32_t wsum = 0, tot = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) {
    uint32_t s = sh[w];
    if (w < wave) wsum += s;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return wsum + inc - x;
}

__device__ __forceinline__ int64_t count_of(const uint32_t* n_dev, int64_t n_max) {
  return n_dev ? (int64_t)*n_dev : n_max;
}

// A gather scan reads src[idx[i]] at random once: the reduce pass leaves
// each gathered value in out[i], where the down-sweep reads it in order
// (and then overwrites it with the item's prefix).
//
// In both passes a thread requests all of its items' words before it uses
// any (unconditional loads at indices clamped to the last item, validity
// applied afterwards): a load under a bounds test that is used at once
// costs one memory round trip per item.
//
// A launch takes two scans of the same bound (blockIdx.y): the step's two
// gather scans share their two launches (a launch of any size takes some 4.5 us
// of a busy queue: 21 -> 15 us for 31k visible of 2^19 ids).
struct ScanArgs {
  const uint32_t *src, *idx;
  const uint32_t* n_dev;
  uint32_t *out, *total, *bsum, *out_at_idx;
  Compact cp;
};

template <int MODE>
__global__ void __launch_bounds__(kScanThreads) k_scan_reduce(ScanArgs first, ScanArgs second, int64_t n_max) {
  const ScanArgs& A = blockIdx.y ? second : first;
  const uint32_t *__restrict__ src = A.src, *__restrict__ idx = A.idx, *n_dev = A.n_dev;
  uint32_t *__restrict__ bsum = A.bsum, *__restrict__ stash = A.out;
  __shared__ uint32_t sh[4];
  const int64_t n = count_of(n_dev, n_max);
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  if (base >= n) return;
  auto item = [&](int k) { return base + (int64_t)k * kScanThreads + threadIdx.x; };
  auto clamp = [&](int64_t i) { return i < n ? i : n - 1; };
  uint32_t x[kScanItems];
  if constexpr (MODE == SCAN_GATHER) {
    uint32_t id[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) id[k] = idx[clamp(item(k))];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) x[k] = src[id[k]];
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) x[k] = src[clamp(item(k))];
  }
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = item(k);
    uint32_t v = MODE == SCAN_FLAG_NONZERO ? (x[k] != 0u ? 1u : 0u) : x[k];
    v = i < n ? v : 0u;
    if constexpr (MODE == SCAN_GATHER) {
      if (i < n) stash[i] = v;
    }
    s += v;
  }
  uint32_t total;
  block_excl_scan(s, sh, total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

template <int MODE>
__global__ void __launch_bounds__(kScanThreads) k_scan_down(ScanArgs first, ScanArgs second, int64_t n_max) {
  const ScanArgs& A = blockIdx.y ? second : first;
  const uint32_t *__restrict__ src = A.src, *__restrict__ idx = A.idx, *n_dev = A.n_dev, *__restrict__ bsum = A.bsum;
  uint32_t *__restrict__ out = A.out, *__restrict__ total = A.total, *__restrict__ out_at_idx = A.out_at_idx;
  const Compact& cp = A.cp;
  __shared__ uint32_t sh[4];
  const int64_t n = count_of(n_dev, n_max);
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  if (n == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *total = 0u;
    return;
  }
  if (base >= n) return;
  // thread t owns the contiguous items [base + t*8, base + t*8 + 8); their
  // words (the value, and the source index or depth key the writes below
  // need) are requested before the block sums, so all are in flight at once
  auto item = [&](int k) { return base + (int64_t)threadIdx.x * kScanItems + k; };
  auto clamp = [&](int64_t i) { return i < n ? i : n - 1; };
  // (16 bytes a request, but in a last part-filled block: a 4-byte request of a
  // wave over items 32 bytes apart touches as many lines for an eighth of
  // them.  4.2 M ids of 8 views: 34 -> 17 us, the offsets of their 1.04 M visible
  // ones 23 -> 18)
  const bool full = base + kScanTile <= n;
  auto load_items = [&](const uint32_t* p, uint32_t (&x)[kScanItems]) {
    if (full) {
      static_assert(kScanItems == 8, "two 16-byte requests");
      const uint4 a = ((const uint4*)(p + item(0)))[0], b = ((const uint4*)(p + item(0)))[1];
      x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w;
      x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
    } else {
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) x[k] = p[clamp(item(k))];
    }
  };
  uint32_t raw[kScanItems], aux[kScanItems];
  load_items(MODE == SCAN_GATHER ? out : src, raw);
  if (out_at_idx) {
    load_items(idx, aux);
  } else if (cp.ent) {
    load_items(cp.key_src, aux);
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) aux[k] = 0u;
  }
  asm volatile("" ::: "memory");
  // offset of this block: the sum of the block sums before it (each block
  // adds them up itself, so no separate pass over the block sums is needed)
  uint32_t pre = 0;
  for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += kScanThreads) pre += bsum[b];
  uint32_t boff;
  block_excl_scan(pre, sh, boff);
  uint32_t v[kScanItems];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint32_t x = MODE == SCAN_FLAG_NONZERO ? (raw[k] != 0u ? 1u : 0u) : raw[k];
    v[k] = item(k) < n ? x : 0u;
    s += v[k];
  }
  uint32_t btot;
  uint32_t run = block_excl_scan(s, sh, btot) + boff;
  if (full) {
    uint32_t at[kScanItems];
    at[0] = run;
#pragma unroll
    for (int k = 1; k < kScanItems; ++k) at[k] = at[k - 1] + v[k - 1];
    ((uint4*)(out + item(0)))[0] = make_uint4(at[0], at[1], at[2], at[3]);
    ((uint4*)(out + item(0)))[1] = make_uint4(at[4], at[5], at[6], at[7]);
  }
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = item(k);
    if (i < n) {
      if (!full) out[i] = run;
      if (out_at_idx) out_at_idx[aux[k]] = run;   // gather scans: the value also at its source index
      if (cp.ent && v[k] != 0u) {                  // flag scans: compaction of the flagged items
        cp.ent[run] = (uint32_t)i;
        cp.ent_copy[run] = (uint32_t)i;
        cp.keys[run] = aux[k];
      }
    }
    run += v[k];
  }
  if (cp.big) {   // one atomic per wave that holds such items
    uint32_t nbig = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) nbig += v[k] > cp.big_min ? 1u : 0u;
    if (__builtin_amdgcn_ballot_w64(nbig != 0u) != 0ull) {
      const int lane = threadIdx.x & 63;
      const uint32_t inc = wave_incl_scan(nbig, lane);
      uint32_t at = 0;
      if (lane == 63) at = atomicAdd(cp.n_big, inc);
      at = (uint32_t)__shfl((int)at, 63) + inc - nbig;
#pragma unroll
      for (int k = 0; k < kScanItems; ++k)
        if (v[k] > cp.big_min) cp.big[at++] = (uint32_t)item(k);
    }
  }
  if (base + kScanTile >= n && threadIdx.x == 0) *total = boff + btot;   // the last block
}

// reduce kernel must sum the same items as the down-sweep: both cover the
// block's 2048 items, only the assignment to threads differs.

// The lists of a small front end by one work-group of 16 waves, in LDS: ten
// launches become one.  Thread t owns the ids 4 t .. 4 t + 3 in the scans.  The
// depth sort is the radix sort's (stable, ranks from match masks, a wave's keys
// contiguous), with the keys in LDS between four passes of 8 bits (three of 11
// clear and scan eight times the counters: 21 us in place of 18 for 2000).  What
// bounds it is one work-group's chain of loads, barriers and LDS accesses.
// 2000 visible ids: 44 us and nine more launches -> 18 us (a captured step 134 ->
// 109); 4000: 57 -> 28.  The line: with room for 8192 ids, 8000 take 65 us in
// place of some 60, and 2000 take 23.
constexpr int kFrontThreads = 1024, kFrontWaves = kFrontThreads / 64;
constexpr int kFrontItems = (int)(kSmallFront / kFrontThreads);   // 4
constexpr int kFrontBits = 8, kFrontPasses = 32 / kFrontBits;
struct alignas(16) FrontLds {   // (cnt is cleared 16 bytes at a time)
  uint32_t key[kSmallFront];
  uint16_t id[kSmallFront];
  uint16_t cnt[kFrontWaves][1 << kFrontBits];   // a wave's keys of a digit, then those of the waves before it
  uint32_t first[1 << kFrontBits];
  uint32_t sh[2][kFrontWaves];
};
static_assert(sizeof(FrontLds) <= 160 * 1024, "the lists fit in LDS");
static_assert(offsetof(FrontLds, cnt) % 16 == 0 && sizeof(FrontLds::cnt) % 16 == 0, "16-byte stores");

// exclusive scans of two values per thread over the work-group
__device__ __forceinline__ uint2 front_scan2(uint32_t x, uint32_t y, uint32_t (*sh)[kFrontWaves], uint2& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t ix = wave_incl_scan(x, lane), iy = wave_incl_scan(y, lane);
  __syncthreads();
  if (lane == 63) {
    sh[0][wave] = ix;
    sh[1][wave] = iy;
  }
  __syncthreads();
  uint2 pre = make_uint2(0u, 0u);
  total = make_uint2(0u, 0u);
#pragma unroll
  for (int w = 0; w < kFrontWaves; ++w) {
    const uint32_t a = sh[0][w], b = sh[1][w];
    if (w < wave) {
      pre.x += a;
      pre.y += b;
    }
    total.x += a;
    total.y += b;
  }
  return make_uint2(pre.x + ix - x, pre.y + iy - y);
}

__global__ void __launch_bounds__(kFrontThreads) k_small_front(FrontLists f, uint32_t n, Counters* __restrict__ out) {
  __shared__ FrontLds S;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t ct[kFrontItems], cb[kFrontItems], dk[kFrontItems];
#pragma unroll
  for (int k = 0; k < kFrontItems; ++k) {
    const uint32_t i = min((uint32_t)(kFrontItems * t + k), n - 1u);
    ct[k] = f.cnt_t[i];
    cb[k] = f.cnt_b[i];
    dk[k] = f.dkey[i];
  }
  asm volatile("" ::: "memory");
  uint32_t vis = 0u, slots = 0u;
#pragma unroll
  for (int k = 0; k < kFrontItems; ++k) {
    const bool v = (uint32_t)(kFrontItems * t + k) < n && ct[k] != 0u;
    vis += v ? 1u : 0u;
    slots += v ? cb[k] : 0u;
  }
  uint2 total;
  uint2 at = front_scan2(vis, slots, S.sh, total);
  const uint32_t m = total.x;
#pragma unroll
  for (int k = 0; k < kFrontItems; ++k) {
    const uint32_t i = (uint32_t)(kFrontItems * t + k);
    if (i >= n) continue;
    f.cidx[i] = at.x;
    if (ct[k] == 0u) continue;
    f.ent[at.x] = i;
    f.slot_off[at.x] = at.y;
    f.slot_base[i] = at.y;
    if (cb[k] > kLongSlots) f.long_ids[atomicAdd(&out->n_long, 1u)] = at.x;
    S.key[at.x] = dk[k];
    S.id[at.x] = (uint16_t)i;
    ++at.x;
    at.y += cb[k];
  }
  // depth sort of the m keys; a wave takes iters rows of 64
  const int iters = (int)((m + kFrontThreads - 1) / kFrontThreads);
  const uint32_t base = (uint32_t)(wave * iters * 64 + lane);
#pragma unroll 1
  for (int pass = 0; pass < kFrontPasses; ++pass) {
    const int shift = kFrontBits * pass;
    constexpr uint32_t mask = (1u << kFrontBits) - 1u;
    for (int d = t; d < (int)(sizeof(S.cnt) / 16); d += kFrontThreads) ((uint4*)S.cnt)[d] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();   // (the keys are complete, too)
    uint32_t kk[kFrontItems];
    uint16_t vv[kFrontItems];
    uint64_t peers[kFrontItems];
#pragma unroll
    for (int it = 0; it < kFrontItems; ++it)
      if (it < iters) {
        const uint32_t i = base + 64u * it;
        const bool ok = i < m;
        kk[it] = S.key[ok ? i : 0u];
        vv[it] = S.id[ok ? i : 0u];
        const uint32_t d = (kk[it] >> shift) & mask;
        uint64_t p = __builtin_amdgcn_ballot_w64(ok);
#pragma unroll
        for (int b = 0; b < kFrontBits; ++b) {
          const bool bit = (d >> b) & 1u;
          const uint64_t bal = __builtin_amdgcn_ballot_w64(bit);
          p &= bit ? bal : ~bal;
        }
        peers[it] = p;
        if (ok && (p & lt) == 0ull) S.cnt[wave][d] += (uint16_t)__popcll(p);
        __builtin_amdgcn_wave_barrier();
      }
    __syncthreads();
    uint32_t a = 0u, b = 0u;   // digits 2 t, 2 t + 1
    const bool owner = 2 * t < (1 << kFrontBits);
    if (owner) {
#pragma unroll
      for (int w = 0; w < kFrontWaves; ++w) {
        uint32_t* q = (uint32_t*)&S.cnt[w][2 * t];
        const uint32_t c = *q;
        *q = a | b << 16;
        a += c & 0xffffu;
        b += c >> 16;
      }
    }
    uint2 all;
    const uint2 pre = front_scan2(a + b, 0u, S.sh, all);
    if (owner) {
      S.first[2 * t] = pre.x;
      S.first[2 * t + 1] = pre.x + a;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kFrontItems; ++it)
      if (it < iters) {
        const bool ok = base + 64u * it < m;
        const uint32_t d = (kk[it] >> shift) & mask, rank = (uint32_t)__popcll(peers[it] & lt), c = S.cnt[wave][d];
        __builtin_amdgcn_wave_barrier();
        if (ok) {
          const uint32_t pos = S.first[d] + c + rank;
          S.key[pos] = kk[it];
          S.id[pos] = vv[it];
          if (rank == 0u) S.cnt[wave][d] = (uint16_t)(c + (uint32_t)__popcll(peers[it]));
        }
        __builtin_amdgcn_wave_barrier();
      }
    __syncthreads();
  }
  // pair offsets in depth order
  uint32_t id[kFrontItems], np[kFrontItems], pairs = 0u;
#pragma unroll
  for (int k = 0; k < kFrontItems; ++k) {
    const uint32_t j = (uint32_t)(kFrontItems * t + k);
    id[k] = S.id[j < m ? j : 0u];
    np[k] = f.cnt_t[m ? id[k] : 0u];
  }
#pragma unroll
  for (int k = 0; k < kFrontItems; ++k) {
    np[k] = (uint32_t)(kFrontItems * t + k) < m ? np[k] : 0u;
    pairs += np[k];
  }
  uint2 n_pairs;
  uint32_t run = front_scan2(pairs, 0u, S.sh, n_pairs).x;
#pragma unroll
  for (int k = 0; k < kFrontItems; ++k) {
    const uint32_t j = (uint32_t)(kFrontItems * t + k);
    if (j < m) {
      f.srid[j] = id[k];
      f.off_t[j] = run;
    }
    run += np[k];
  }
  if (t == 0) {
    out->n_visible = m;
    out->n_pairs = n_pairs.x;
    out->n_slots = total.y;
  }
}

constexpr int kEmitThreads = 256;
constexpr int kEmitPerThread = 4;
constexpr int kEmitTile = kEmitThreads * kEmitPerThread;   // 1024 pairs per block
constexpr int kEmitZero = kEmitThreads * 16;               // words zeroed per block, at most

// The first index i with a[i] > x (n if none) of a non-decreasing array,
// found by one wave: each step the 64 lanes probe 64 evenly
// spaced positions of the remaining range [lo, hi) and a ballot keeps the
// part holding the first element > x (hi stays a candidate: a[hi] > x or
// hi == n): about log64(n) dependent loads, where a one-thread binary
// search takes log2(n).
__device__ __forceinline__ int64_t wave_upper_bound_u32(const uint32_t* a, int64_t n, uint32_t x) {
  const int lane = threadIdx.x & 63;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t i = lo + (int64_t)lane * step;
    const bool valid = i < hi;
    const bool gt = valid && a[i] > x;
    const uint64_t m = __builtin_amdgcn_ballot_w64(gt);
    if (m != 0ull) {
      const int f = __builtin_ctzll(m);
      hi = lo + (int64_t)f * step;
      if (f > 0) lo += (int64_t)(f - 1) * step + 1;
    } else {
      const int last = 63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(valid));
      lo += (int64_t)last * step + 1;
    }
  }
  return lo;
}

// Also the step's overflow flag and effective counts (block 0), and a range of
// words zeroed for the stages that follow (nothing here reads any of them).
// The box and its view are read once per entry and kept in LDS, a thread's
// pairs are looked up together and the place in the box is divided by its width
// through a reciprocal: 2 M Gaussians at 1296 x 968 (4.3 M pairs) 26 -> 20 us,
// 300k at 640 x 480 8.5 -> 6.4, 2k 7.4 -> 5.8; eight views of 640 x 480 (3.9 M
// pairs of 1.04 M entries, whose scattered boxes bound it) 38.5 -> 36.5.
__global__ void __launch_bounds__(kEmitThreads) k_emit(
    const GeomRec* __restrict__ geom, const ViewDesc* __restrict__ views,
    const uint32_t* __restrict__ srid, const uint32_t* __restrict__ off_t,
    Counters* __restrict__ cnt, int64_t cap_pairs, int64_t cap_slots, int npad_shift, int tile_shift,
    uint32_t* __restrict__ keys, uint32_t* __restrict__ vals, uint32_t* __restrict__ zero, int64_t n_zero) {
  __shared__ uint32_t s_off[kEmitTile + 2];
  __shared__ uint32_t s_rid[kEmitTile + 2];
  __shared__ uint32_t s_key[kEmitTile + 2], s_row[kEmitTile + 2];   // first tile; tiles per row | tiles_x << 16
  __shared__ int64_t s_j[2];
  const int64_t M = cnt->n_visible;
  const int64_t P = cnt->n_pairs;
  for (int64_t i = (int64_t)blockIdx.x * kEmitThreads + threadIdx.x; i < n_zero; i += (int64_t)gridDim.x * kEmitThreads)
    zero[i] = 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const bool ov = P > cap_pairs || (int64_t)cnt->n_slots > cap_slots;
    cnt->overflow = ov ? 1u : 0u;
    cnt->n_pairs_eff = ov ? 0u : cnt->n_pairs;
  }
  if (P > cap_pairs) return;                 // overflow: nothing valid is written
  const int64_t p0 = (int64_t)blockIdx.x * kEmitTile;
  if (p0 >= P) return;
  const int64_t p1 = (p0 + kEmitTile < P ? p0 + kEmitTile : P) - 1;   // last pair of the block
  // the entries owning the block's first and last pair: wave 0 and wave 1
  if (threadIdx.x < 128) {
    const int w = threadIdx.x >> 6;
    const int64_t j = wave_upper_bound_u32(off_t, M, (uint32_t)(w == 0 ? p0 : p1)) - 1;
    if ((threadIdx.x & 63) == 0) s_j[w] = j;
  }
  __syncthreads();
  const int64_t j0 = s_j[0], j1 = s_j[1];
  const int nj = (int)(j1 - j0 + 1);         // <= kEmitTile: every entry owns >= 1 pair
  for (int t = threadIdx.x; t < nj; t += kEmitThreads) {
    const uint32_t rid = srid[j0 + t];
    s_off[t] = off_t[j0 + t];
    s_rid[t] = rid;
    const uint32_t bb = geom[rid].bbox;
    const ViewDesc& V = views[rid >> npad_shift];
    const uint32_t tx0 = (bb & 255u) >> tile_shift, tx1 = ((bb >> 8) & 255u) >> tile_shift;
    const uint32_t ty0 = ((bb >> 16) & 255u) >> tile_shift, tiles_x = (uint32_t)V.tiles_x;
    s_key[t] = (uint32_t)V.tile_off + ty0 * tiles_x + tx0;
    s_row[t] = (tx1 - tx0 + 1u) | (tiles_x << 16);
  }
  __syncthreads();
  // each pair's entry, the largest t with s_off[t] <= pi: one search for all
  // of a thread's pairs, step by step, so that their LDS reads overlap
  int own[kEmitPerThread];
#pragma unroll
  for (int k = 0; k < kEmitPerThread; ++k) own[k] = 0;
  for (int step = nj > 1 ? 1 << (31 - __builtin_clz(nj - 1)) : 0; step > 0; step >>= 1)
#pragma unroll
    for (int k = 0; k < kEmitPerThread; ++k) {
      const int mid = min(own[k] + step, nj - 1);
      own[k] = (int64_t)s_off[mid] <= p0 + k * kEmitThreads + (int)threadIdx.x ? mid : own[k];
    }
#pragma unroll
  for (int k = 0; k < kEmitPerThread; ++k) {
    const int64_t pi = p0 + k * kEmitThreads + threadIdx.x;
    const uint32_t local = (uint32_t)(pi - s_off[own[k]]), row = s_row[own[k]], w = row & 0xffffu;
    // local / w: at most 2^16 tiles, so the quotient's fraction is at least
    // 2^-17 of it away from an integer, far more than the reciprocal's error
    const uint32_t q = (uint32_t)(((float)local + 0.5f) * __builtin_amdgcn_rcpf((float)w));
    if (pi <= p1) {
      keys[pi] = s_key[own[k]] + q * (row >> 16) + (local - q * w);
      vals[pi] = s_rid[own[k]];
    }
  }
}

__global__ void __launch_bounds__(256) k_fill_u32(uint32_t* __restrict__ p, uint32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void __launch_bounds__(256) k_zero(ZeroRanges r) {
#pragma unroll
  for (int k = 0; k < ZeroRanges::kMax; ++k)
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < r.n[k]; i += (int64_t)gridDim.x * 256) r.p[k][i] = 0u;
}

__global__ void __launch_bounds__(256) k_tile_ranges(const uint32_t* __restrict__ keys,
                                                     const Counters* __restrict__ cnt,
                                                     uint2* __restrict__ ranges) {
  const int64_t P = cnt->overflow ? 0 : (int64_t)cnt->n_pairs;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= P) return;
  const uint32_t k = keys[i];
  if (i == 0 || keys[i - 1] != k) ranges[k].x = (uint32_t)i;
  if (i == P - 1 || keys[i + 1] != k) ranges[k].y = (uint32_t)(i + 1);
}

// Work items grouped by queue and, inside a queue, by descending list length
// (longest first): one work-group per queue, a counting sort of the queue's
// tiles on 256 length buckets (255 - bucket, bucket = 4 sqrt(length)
// clamped at 255) into the queue's segment of the output (a queue's items
// keep the segment the static table gives them).  Tiles of one bucket may
// come out in any order; the order only affects scheduling, not results.
constexpr int kOrderThreads = 256;
constexpr uint32_t kMaxTileItems = 16;   // 8x8 blocks of a 32-pixel tile

__device__ __forceinline__ uint32_t tile_bin(const uint2* __restrict__ ranges, const TileItems& T) {
  const uint2 r = ranges[T.tile];
  const uint32_t bucket = min(255u, (uint32_t)(4.f * sqrtf((float)(r.y - r.x))));
  return 255u - bucket;
}

// Work-group q: tiles tq[q] .. tq[q + 1] of the queue-major tile table, items
// to out[qoff[q] ..]; each tile's blocks are copied as a run, so they stay
// together in the output and are taken up by the queue's waves side by side.
__global__ void __launch_bounds__(kOrderThreads) k_order_items(const uint2* __restrict__ ranges,
                                                             const uint32_t* __restrict__ items,
                                                             const uint32_t* __restrict__ qoff,
                                                             const TileItems* __restrict__ tiles,
                                                             const uint32_t* __restrict__ tq,
                                                             uint32_t* __restrict__ out) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t wsum[kOrderThreads / 64];
  const uint32_t q = blockIdx.x, t0 = tq[q], t1 = tq[q + 1], base = qoff[q];
  hist[threadIdx.x] = 0u;
  __syncthreads();
  for (uint32_t i = t0 + threadIdx.x; i < t1; i += kOrderThreads) {
    const TileItems T = tiles[i];
    atomicAdd(&hist[tile_bin(ranges, T)], T.count);
  }
  __syncthreads();
  // exclusive scan of the 256 bins, one per thread
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t a = hist[threadIdx.x];
  uint32_t inc = a;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(inc, off, 64);
    if (lane >= off) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t pre = 0;
  for (int w = 0; w < wave; ++w) pre += wsum[w];
  hist[threadIdx.x] = base + pre + inc - a;
  __syncthreads();
  // a tile has at most kMaxTileItems blocks: all of its loads are issued
  // before the first store (one memory round trip per tile)
  for (uint32_t i = t0 + threadIdx.x; i < t1; i += kOrderThreads) {
    const TileItems T = tiles[i];
    const uint32_t pos = atomicAdd(&hist[tile_bin(ranges, T)], T.count);
    uint32_t v[kMaxTileItems];
#pragma unroll
    for (uint32_t k = 0; k < kMaxTileItems; ++k) v[k] = k < T.count ? items[T.first + k] : 0u;
#pragma unroll
    for (uint32_t k = 0; k < kMaxTileItems; ++k)
      if (k < T.count) out[pos + k] = v[k];
  }
}

}  // namespace

size_t scan_temp_bytes(int64_t n) {
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  return (size_t)(nb > 0 ? nb : 1) * 2 * sizeof(uint32_t);   // (two scans' block sums)
}

template <int MODE>
static void launch_scan_t(const ScanArgs& a, const ScanArgs& b, unsigned count, int64_t n_max, hipStream_t s) {
  const int64_t nb = (n_max + kScanTile - 1) / kScanTile;
  if (nb > 0)
    hipLaunchKernelGGL(k_scan_reduce<MODE>, dim3((unsigned)nb, count), dim3(kScanThreads), 0, s, a, b, n_max);
  hipLaunchKernelGGL(k_scan_down<MODE>, dim3((unsigned)(nb > 0 ? nb : 1), count), dim3(kScanThreads), 0, s, a, b,
                     n_max);
}

void launch_scan(int mode, const uint32_t* src, uint32_t* out, uint32_t* total, int64_t n, void* temp, hipStream_t s,
                 Compact cp) {
  const ScanArgs a{src, nullptr, nullptr, out, total, (uint32_t*)temp, nullptr, cp};
  if (mode == SCAN_FLAG_NONZERO) launch_scan_t<SCAN_FLAG_NONZERO>(a, a, 1, n, s);
  else launch_scan_t<SCAN_VALUE>(a, a, 1, n, s);
}

void launch_gather_scans(const GatherScan& a, const GatherScan& b, const uint32_t* n_dev, int64_t n_max, void* temp,
                         hipStream_t s) {
  const size_t nb = (size_t)std::max<int64_t>(1, (n_max + kScanTile - 1) / kScanTile);
  auto args = [&](const GatherScan& g, uint32_t* bsum) {
    return ScanArgs{g.src, g.idx, n_dev, g.out, g.total, bsum, g.out_at_idx, g.cp};
  };
  launch_scan_t<SCAN_GATHER>(args(a, (uint32_t*)temp), args(b, (uint32_t*)temp + nb), 2, n_max, s);
}

void launch_small_front(const FrontLists& f, int64_t n_rid, Counters* cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_small_front, dim3(1), dim3(kFrontThreads), 0, s, f, (uint32_t)n_rid, cnt);
}

void launch_emit(const GeomRec* geom, const ViewDesc* views, const uint32_t* srid, const uint32_t* off_t,
                 Counters* cnt, int64_t cap_pairs, int64_t cap_slots, int npad_shift,
                 int tile_shift, uint32_t* keys, uint32_t* vals, uint32_t* zero, int64_t n_zero, hipStream_t s) {
  // enough blocks for the words to be zeroed, too (no pairs over the tiles of 8
  // of eight views of 2048 x 2048: 107 -> 5 us)
  const int64_t blocks = std::max<int64_t>({1, (cap_pairs + kEmitTile - 1) / kEmitTile,
                                            (n_zero + kEmitZero - 1) / kEmitZero});
  hipLaunchKernelGGL(k_emit, dim3((unsigned)blocks), dim3(kEmitThreads), 0, s, geom, views, srid, off_t,
                     cnt, cap_pairs, cap_slots, npad_shift, tile_shift, keys, vals, zero, n_zero);
}

void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
}

void launch_zero(const ZeroRanges& r, hipStream_t s) {
  int64_t n = 0;
  for (int k = 0; k < ZeroRanges::kMax; ++k) n = std::max(n, r.n[k]);
  if (n <= 0) return;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), dim3(256), 0, s, r);
}

void launch_tile_ranges(const uint32_t* keys, const Counters* cnt, int64_t grid_max, uint2* ranges,
                        hipStream_t s) {
  if (grid_max <= 0) return;
  hipLaunchKernelGGL(k_tile_ranges, dim3((unsigned)((grid_max + 255) / 256)), dim3(256), 0, s, keys,
                     cnt, ranges);
}


uint32_t* launch_order_items(const uint2* ranges, const uint32_t* items, const uint32_t* qoff, const TileItems* tiles,
                             const uint32_t* tq, int64_t n_tiles, uint32_t* out, hipStream_t s) {
  if (n_tiles <= 0) return out;
  hipLaunchKernelGGL(k_order_items, dim3(kQueues), dim3(kOrderThreads), 0, s, ranges, items, qoff, tiles, tq, out);
  return out;
}

}  // namespace lgs
