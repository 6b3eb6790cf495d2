// Language-guided pruning (Sec. III-C, Eq. (4)) and the geometric criteria
// it is combined with.  For each Gaussian i, its K nearest other Gaussians
// (Euclidean distance of the means, ties by index) are examined; a
// neighbour j is redundant when |p_i - p_j| < tau_dist, the cosine
// similarity of their language features exceeds tau_sim, and i dominates j
// (larger opacity logit, or equal logits and i < j), so that one Gaussian of
// a redundant pair survives.  Geometric: opacity below min_opacity, largest
// scale above max_scale, or a non-finite mean / logit / log-scale.
//
// Only neighbours closer than tau_dist can be redundant, so the K nearest
// that matter are the K nearest among those within tau_dist.  The means are
// bucketed by cells of side tau_dist, folded onto a table of m buckets:
//   bucket = (cx * kFoldX + cy * kFoldY + cz) mod m,  2 n <= m < 4 n.
// Three cells (ux, uy, cz - 1 .. cz + 1) are then three buckets in a row, and
// the 27 cells around a Gaussian 9 runs of the positions laid out in bucket
// order, of which no two share a bucket (checked below for every m).  A first
// pass counts the buckets (the count before it is a Gaussian's place in its
// bucket) and packs what a neighbour's test reads into one record per
// Gaussian; a scan of the counts and a pass that puts each position in its
// place complete the table.  (A sort by cell takes four to eight passes of
// three kernels, and every lookup a binary search.)  Other cells that fold onto
// a run's buckets add candidates that the distance drops.
//
// A Gaussian's candidates are first held against tau_dist^2 in FP32, with a
// margin above its rounding.  While no more than K pass, the K nearest are
// among them without any ordering: each pair's distance is evaluated in FP64
// (no contraction: (dx^2 + dy^2) + dz^2), and a dominated one's similarity in
// FP64; a Gaussian with more goes to a list, which a second kernel works
// through with a register-resident sorted list of the K best (FP64 distance,
// index) pairs.  A dominated similar neighbour's byte is set to 1 (every
// writer stores the same value), so the order inside a bucket, which the
// atomics leave open, does not show in the mask.
//
// What bounds the neighbour search: its vector instructions.  500k Gaussians
// on the surfaces of a 6 m room, 2.3 neighbours within 2 cm each: 44 us in
// place of 767 (sorted cells, 9 binary searches per Gaussian, every candidate
// in the sorted list), of which the FP32 test first is 77 -> 44; the table
// (count, scan, fill) 45 us in place of 141 for the sort; bytes moved: record
// and table 0.15 GB, 30 us at the rate of a large copy.
#include "lgs_internal.h"

namespace lgs {
namespace {

constexpr int kPruneKMax = 32;
constexpr int64_t kCellBias = 1ll << 20;   // cell coordinates in [-2^20, 2^20)
constexpr int kRuns = 9;
constexpr uint32_t kFoldX = 1986774811u, kFoldY = 1320501587u;
constexpr uint32_t kMinBuckets = 256u;
constexpr uint32_t kNoPlace = 0xffffffffu;

// whether the 9 runs of three buckets are disjoint in a table of m
constexpr bool runs_disjoint(uint32_t m) {
  for (uint32_t dx = 0; dx < 5; ++dx)
    for (uint32_t dy = 0; dy < 5; ++dy) {
      const uint32_t d = ((dx - 2u) * kFoldX + (dy - 2u) * kFoldY) & (m - 1u);
      if ((dx != 2u || dy != 2u) && (d < 3u || m - d < 3u)) return false;
    }
  return m == 1u << 31 || runs_disjoint(2u * m);
}
static_assert(runs_disjoint(kMinBuckets), "two runs around a Gaussian share a bucket");

__device__ __forceinline__ bool finite3(float x, float y, float z) {
  return isfinite(x) && isfinite(y) && isfinite(z);
}

// cell coordinates of a finite mean; false when out of the grid's range
__device__ __forceinline__ bool cell_of(const PruneArgs& a, float x, float y, float z, int32_t c[3]) {
  const int64_t cx = (int64_t)floor((double)x * a.inv_cell), cy = (int64_t)floor((double)y * a.inv_cell),
                cz = (int64_t)floor((double)z * a.inv_cell);
  const int64_t v[3] = {cx, cy, cz};
  bool ok = true;
  for (int k = 0; k < 3; ++k) {
    ok &= v[k] >= -kCellBias && v[k] < kCellBias;
    c[k] = (int32_t)v[k];
  }
  return ok;
}

__device__ __forceinline__ uint32_t bucket_of(const PruneArgs& a, int32_t cx, int32_t cy, int32_t cz) {
  return ((uint32_t)cx * kFoldX + (uint32_t)cy * kFoldY + (uint32_t)cz) & (a.buckets - 1u);
}

// what a neighbour's test reads: position and logit, the features' norm
// (FP64), the features (stored type)
template <bool BF16>
struct Rec {
  float4 p;          // x, y, z, opacity logit
  double norm;
  double pad;
  uint4 f[BF16 ? 2 : 4];
};

__device__ __forceinline__ void feats(const Rec<true>& r, double f[16]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t w[4] = {r.f[q].x, r.f[q].y, r.f[q].z, r.f[q].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[8 * q + 2 * k] = (double)__uint_as_float(w[k] << 16);
      f[8 * q + 2 * k + 1] = (double)__uint_as_float(w[k] & 0xffff0000u);
    }
  }
}
__device__ __forceinline__ void feats(const Rec<false>& r, double f[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t w[4] = {r.f[q].x, r.f[q].y, r.f[q].z, r.f[q].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) f[4 * q + k] = (double)__uint_as_float(w[k]);
  }
}

#pragma clang fp contract(off)
// Per Gaussian: its record, the geometric flag, the semantic one cleared, and
// its place in its bucket (kNoPlace without a cell).
template <bool BF16>
__global__ void __launch_bounds__(256) k_prune_pack(PruneArgs a, Rec<BF16>* __restrict__ rec,
                                                    uint8_t* __restrict__ geo, uint8_t* __restrict__ sem,
                                                    uint32_t* __restrict__ count, uint32_t* __restrict__ place,
                                                    PruneCounters* __restrict__ pc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const float x = a.means[i], y = a.means[a.n + i], z = a.means[2 * a.n + i];
  const float lam = a.logits[i];
  const float s0 = a.log_scales[i], s1 = a.log_scales[a.n + i], s2 = a.log_scales[2 * a.n + i];
  uint32_t w[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int64_t at = (int64_t)(k < a.planes ? k : 0) * a.n + i;
    w[k] = BF16 ? (uint32_t)((const unsigned short*)a.feat)[at] : ((const uint32_t*)a.feat)[at];
  }
  uint32_t at = kNoPlace;
  if (finite3(x, y, z)) {
    int32_t c[3];
    if (cell_of(a, x, y, z, c)) at = atomicAdd(&count[bucket_of(a, c[0], c[1], c[2])], 1u);
    else pc->range_err = 1u;
  }
  const bool fin = finite3(x, y, z) && isfinite(lam) && finite3(s0, s1, s2);
  const double smax = fmax(fmax((double)s0, (double)s1), (double)s2);
  geo[i] = (!fin || (double)lam < a.logit_min || smax > a.log_scale_max) ? 1 : 0;
  sem[i] = 0;
#pragma unroll
  for (int k = 8; k < 16; ++k) w[k] = k < a.planes ? w[k] : 0u;
  Rec<BF16> r;
  r.p = make_float4(x, y, z, lam);
  r.pad = 0.0;
#pragma unroll
  for (int q = 0; q < (BF16 ? 2 : 4); ++q)
    r.f[q] = BF16 ? make_uint4(w[(8 * q) & 15] | (w[(8 * q + 1) & 15] << 16), w[(8 * q + 2) & 15] | (w[(8 * q + 3) & 15] << 16),
                               w[(8 * q + 4) & 15] | (w[(8 * q + 5) & 15] << 16), w[(8 * q + 6) & 15] | (w[(8 * q + 7) & 15] << 16))
                  : make_uint4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
  double f[16], n2 = 0.0;
  feats(r, f);
#pragma unroll
  for (int k = 0; k < 16; ++k) n2 += f[k] * f[k];
  r.norm = sqrt(n2);
  rec[i] = r;
  place[i] = at;
}

// positions (and indices) in bucket order; start[b]: the bucket's first
__global__ void __launch_bounds__(256) k_prune_fill(PruneArgs a, const uint32_t* __restrict__ start,
                                                    const uint32_t* __restrict__ place, float4* __restrict__ pos) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const float x = a.means[i], y = a.means[a.n + i], z = a.means[2 * a.n + i];
  const uint32_t at = place[i];
  int32_t c[3];
  if (at == kNoPlace || !cell_of(a, x, y, z, c)) return;
  pos[start[bucket_of(a, c[0], c[1], c[2])] + at] = make_float4(x, y, z, __uint_as_float((uint32_t)i));
}

// Run r around cell c: its first position, and its end (past n_pos where it
// goes on at position 0).
__device__ __forceinline__ void run_of(const PruneArgs& a, const int32_t c[3], int r,
                                       const uint32_t* __restrict__ start, uint32_t n_pos, uint32_t& lo, uint32_t& hi) {
  const uint32_t b = bucket_of(a, c[0] + r / 3 - 1, c[1] + r % 3 - 1, c[2] - 1);
  lo = start[b];
  hi = start[((b + 2u) & (a.buckets - 1u)) + 1u] + (b + 2u >= a.buckets ? n_pos : 0u);   // start[buckets] = n_pos
}

__device__ __forceinline__ double dist2(const float4& p, const float4& q) {
  const double ex = (double)q.x - (double)p.x, ey = (double)q.y - (double)p.y, ez = (double)q.z - (double)p.z;
  return (ex * ex + ey * ey) + ez * ez;
}

// j is set when i, closer than tau_dist, dominates it and their features are
// similar
template <bool BF16>
__device__ __forceinline__ void mark_if_redundant(const PruneArgs& a, const Rec<BF16>* __restrict__ rec, uint32_t i,
                                                  uint32_t j, uint8_t* __restrict__ sem) {
  const Rec<BF16> p = rec[i], q = rec[j];
  const float li = p.p.w, lj = q.p.w;
  if (!(li > lj || (li == lj && i < j)) || !(dist2(p.p, q.p) < a.tau2)) return;
  double fi[16], fj[16], dot = 0.0;
  feats(p, fi);
  feats(q, fj);
#pragma unroll
  for (int k = 0; k < 16; ++k) dot += fi[k] * fj[k];
  const double den = p.norm * q.norm;
  const double sim = den > 0.0 ? dot / den : 0.0;
  if (sim > a.tau_sim) sem[j] = 1;
}

constexpr int kPairThreads = 128;
constexpr int kRunWords = 2 * (kRuns + 1);

// One thread per Gaussian in bucket order.  LDS per thread: the runs that hold
// a candidate and the neighbours found (at most k).  The similarities are taken
// by the wave together, a lane to each pair that its 64 Gaussians have (lists
// of 0 to 16 leave most lanes idle: 13 us of 62).
template <bool BF16>
__global__ void __launch_bounds__(kPairThreads) k_prune_pairs(PruneArgs a, const uint32_t* __restrict__ start,
                                                              const float4* __restrict__ pos,
                                                              const Rec<BF16>* __restrict__ rec,
                                                              uint8_t* __restrict__ sem, uint32_t* __restrict__ heavy,
                                                              PruneCounters* __restrict__ pc) {
  extern __shared__ uint32_t lds[];
  uint32_t* run = lds + threadIdx.x;                                   // [10][2] words, kPairThreads apart
  uint32_t* near = lds + kRunWords * kPairThreads + threadIdx.x;       // [k]
  uint8_t* owner = (uint8_t*)(lds + (kRunWords + a.k) * kPairThreads) + (threadIdx.x >> 6) * (64 * a.k);
  const uint32_t n_pos = start[a.buckets];
  const uint32_t s = blockIdx.x * (uint32_t)kPairThreads + threadIdx.x;
  if ((s & ~63u) >= n_pos) return;
  const bool live = s < n_pos;
  const uint32_t self = live ? s : n_pos - 1u;
  const float4 p = pos[self];
  const uint32_t i = __float_as_uint(p.w);
  // runs with a candidate, and one without end, so that the walk below never
  // runs out of them
  int32_t left = 0;
  {
    int32_t c[3];
    cell_of(a, p.x, p.y, p.z, c);
    uint32_t lo[kRuns], hi[kRuns];
#pragma unroll
    for (int r = 0; r < kRuns; ++r) run_of(a, c, r, start, n_pos, lo[r], hi[r]);
    uint32_t* w = run;
#pragma unroll
    for (int r = 0; r < kRuns; ++r)
      if (live && hi[r] > lo[r]) {
        w[0] = lo[r];
        w[kPairThreads] = hi[r];
        w += 2 * kPairThreads;
        left += (int32_t)(hi[r] - lo[r]);
      }
    w[0] = 0u;
    w[kPairThreads] = 0xffffffffu;
  }
  // candidates, eight requested at a time (past the last: the Gaussian itself)
  constexpr int kAhead = 8;
  int cnt = 0;
  uint32_t t = 0u, te = 0u;
  const uint32_t* w = run;
  for (; left > 0 && cnt <= a.k; left -= kAhead) {
    uint32_t at[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      if (t == te) {
        t = w[0];
        te = w[kPairThreads];
        w += 2 * kPairThreads;
      }
      at[q] = q < left ? min(t, t - n_pos) : self;   // (t - n_pos: large below n_pos)
      ++t;
    }
    float4 v[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) v[q] = pos[at[q]];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const float ex = v[q].x - p.x, ey = v[q].y - p.y, ez = v[q].z - p.z;
      const float d2 = fmaf(ex, ex, fmaf(ey, ey, ez * ez));
      if (at[q] != self && !(d2 > a.tau2_above)) {
        if (cnt < a.k) near[cnt * kPairThreads] = __float_as_uint(v[q].w);
        ++cnt;
      }
    }
  }
  if (cnt > a.k) {   // which are the K nearest has to be found out
    heavy[atomicAdd(&pc->n_heavy, 1u)] = s;
    cnt = 0;
  }
  const int lane = threadIdx.x & 63;
  int end = cnt;
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(end, o);
    if (lane >= o) end += up;
  }
  const int first = end - cnt, total = __shfl(end, 63);
  for (int q = 0; q < cnt; ++q) owner[first + q] = (uint8_t)lane;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int b0 = 0; b0 < total; b0 += 64) {
    const int at = min(b0 + lane, total - 1);
    const int o = owner[at];
    const int q = at - __shfl(first, o);
    const uint32_t io = (uint32_t)__shfl((int)i, o);
    const uint32_t j = near[q * kPairThreads + o - lane];
    if (b0 + lane >= total) continue;
    mark_if_redundant(a, rec, io, j, sem);
  }
}

// The listed Gaussians, which have more than K neighbours within tau_dist: one
// thread each, the K best (squared distance, index) pairs in a sorted list of
// KMAX.  What bounds it is the chain of one thread, and in it the list's (a
// candidate is carried past every entry): so candidates are read eight at a
// time, those within tau_dist wait in LDS, and the wave inserts when a lane has
// no more room, each lane its own next one.  A round for every candidate, which
// one of 64 lanes is always near, takes three times as many.  One wave to a
// work-group, as there may be few.  The whole pass, us, with cells sorted and a list
// for every Gaussian / with a round for every candidate here / so: 60k of 10
// neighbours each, K = 16 490, 590, 162; of 40, K = 32 940, 1090, 450; 20k of 1000,
// K = 16 10930, 11040, 2710; 200k of 200, K = 16 5430, 4510, 1820.  (Room for 64
// waiting: the last 2630, as fewer waves fit.)
constexpr int kHeavyThreads = 64, kHeavyRoom = 32;
template <bool BF16, int KMAX>
__global__ void __launch_bounds__(kHeavyThreads) k_prune_heavy(PruneArgs a, const uint32_t* __restrict__ start,
                                                               const float4* __restrict__ pos,
                                                               const Rec<BF16>* __restrict__ rec,
                                                               uint8_t* __restrict__ sem,
                                                               const uint32_t* __restrict__ heavy,
                                                               const PruneCounters* __restrict__ pc) {
  constexpr uint32_t kAhead = 8;
  __shared__ double wait_d[kHeavyRoom][kHeavyThreads];
  __shared__ uint32_t wait_j[kHeavyRoom][kHeavyThreads];
  const uint32_t nh = pc->n_heavy, n_pos = start[a.buckets];
  const int lane = threadIdx.x;
  for (uint32_t h0 = blockIdx.x * kHeavyThreads; h0 < nh; h0 += gridDim.x * kHeavyThreads) {
    const bool live = h0 + lane < nh;
    const uint32_t s = heavy[live ? h0 + lane : nh - 1u];
    const float4 p = pos[s];
    const uint32_t i = __float_as_uint(p.w);
    int32_t c[3];
    cell_of(a, p.x, p.y, p.z, c);
    // ascending; unused = +inf
    double bd[KMAX];
    uint32_t bj[KMAX];
#pragma unroll
    for (int m = 0; m < KMAX; ++m) {
      bd[m] = INFINITY;
      bj[m] = 0xffffffffu;
    }
    int waiting = 0;
#pragma unroll 1
    for (int r = 0; r <= kRuns; ++r) {   // (after the runs: those still waiting)
      uint32_t t = 0u, hi = 0u;
      if (r < kRuns) run_of(a, c, r, start, n_pos, t, hi);
      if (!live) hi = t;
#pragma unroll 1
      for (bool more = true; more;) {
        more = __builtin_amdgcn_ballot_w64(t < hi) != 0ull;
        if (more) {
          float4 v[kAhead];
#pragma unroll
          for (uint32_t q = 0; q < kAhead; ++q)   // (past the run's end: the Gaussian itself)
            v[q] = pos[t < hi && t + q < hi ? min(t + q, t + q - n_pos) : s];
          if (t < hi) t += kAhead;
#pragma unroll
          for (int q = 0; q < kAhead; ++q) {
            const double d2 = dist2(p, v[q]);
            const uint32_t j = __float_as_uint(v[q].w);
            if (j != i && d2 < a.tau2) {
              wait_d[waiting][lane] = d2;
              wait_j[waiting][lane] = j;
              ++waiting;
            }
          }
        }
        if (r < kRuns && __builtin_amdgcn_ballot_w64(waiting > kHeavyRoom - (int)kAhead) == 0ull) continue;
#pragma unroll 1
        for (int q = 0; __builtin_amdgcn_ballot_w64(q < waiting) != 0ull; ++q) {
          // carry the candidate down, swapping it with every entry it precedes
          // (static indices: registers; a lane without one carries the end's mark)
          const bool has = q < waiting;
          double cd = has ? wait_d[q][lane] : INFINITY;
          uint32_t cj = has ? wait_j[q][lane] : 0xffffffffu;
          const bool in = cd < bd[KMAX - 1] || (cd == bd[KMAX - 1] && cj < bj[KMAX - 1]);
          if (__builtin_amdgcn_ballot_w64(in) == 0ull) continue;
#pragma unroll
          for (int m = 0; m < KMAX; ++m) {
            const bool before = cd < bd[m] || (cd == bd[m] && cj < bj[m]);
            const double td = bd[m];
            const uint32_t tj = bj[m];
            bd[m] = before ? cd : td;
            bj[m] = before ? cj : tj;
            cd = before ? td : cd;
            cj = before ? tj : cj;
          }
        }
        waiting = 0;
      }
    }
    static_assert(KMAX <= kHeavyRoom, "the list fits");
#pragma unroll
    for (int m = 0; m < KMAX; ++m) wait_j[m][lane] = bj[m];
#pragma unroll 1
    for (int m = 0; m < a.k; ++m) {
      const uint32_t j = wait_j[m][lane];
      if (j == 0xffffffffu) break;
      mark_if_redundant(a, rec, i, j, sem);
    }
  }
}
#pragma clang fp contract(on)

// mask = semantic | geometric << 1, and the three counts (integer sums:
// the result does not depend on the order of the atomics); a thread takes four
// Gaussians (their bytes as one word where the mask's address allows it).  The
// mask stays as it was when a mean was out of range.
__global__ void __launch_bounds__(256) k_prune_final(int64_t n, int vec, const uint8_t* __restrict__ sem,
                                                     const uint8_t* __restrict__ geo, uint8_t* __restrict__ mask,
                                                     PruneCounters* __restrict__ pc) {
  __shared__ uint32_t sh[4][3];
  if (pc->range_err) return;
  uint32_t c[3] = {0u, 0u, 0u};
  for (int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i0 < n; i0 += (int64_t)gridDim.x * 1024) {
    uint32_t sv = 0u, gv = 0u;
    if (i0 + 4 <= n) {
      sv = *(const uint32_t*)(sem + i0);
      gv = *(const uint32_t*)(geo + i0);
    } else {
      for (int k = 0; i0 + k < n; ++k) {
        sv |= (uint32_t)sem[i0 + k] << (8 * k);
        gv |= (uint32_t)geo[i0 + k] << (8 * k);
      }
    }
    const uint32_t mv = sv | (gv << 1);
    if (vec && i0 + 4 <= n) {
      *(uint32_t*)(mask + i0) = mv;
    } else {
      for (int k = 0; k < 4 && i0 + k < n; ++k) mask[i0 + k] = (uint8_t)(mv >> (8 * k));
    }
    c[0] += (uint32_t)__popc(sv);
    c[1] += (uint32_t)__popc(gv);
    c[2] += (uint32_t)__popc(sv | gv);
  }
  for (int o = 32; o > 0; o >>= 1)
    for (int k = 0; k < 3; ++k) c[k] += (uint32_t)__shfl_xor((int)c[k], o);
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 3; ++k) sh[threadIdx.x >> 6][k] = c[k];
  __syncthreads();
  if (threadIdx.x < 3) {
    const int k = threadIdx.x;
    const uint32_t s = (sh[0][k] + sh[1][k]) + (sh[2][k] + sh[3][k]);
    if (s) atomicAdd(&pc->counts[k], (unsigned long long)s);
  }
}

unsigned blocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

template <bool BF16>
void launch_t(const PruneArgs& a, const PruneWork& w, hipStream_t s) {
  Rec<BF16>* rec = (Rec<BF16>*)w.rec;
  ZeroRanges z;
  z.p[0] = w.count;
  z.n[0] = a.buckets;
  z.p[1] = (uint32_t*)w.pc;
  z.n[1] = sizeof(PruneCounters) / 4;
  launch_zero(z, s);
  hipLaunchKernelGGL(k_prune_pack<BF16>, dim3(blocks(a.n, 256)), dim3(256), 0, s, a, rec, w.geo, w.sem, w.count,
                     w.list, w.pc);
  launch_scan(SCAN_VALUE, w.count, w.start, w.start + a.buckets, a.buckets, w.temp, s);
  hipLaunchKernelGGL(k_prune_fill, dim3(blocks(a.n, 256)), dim3(256), 0, s, a, (const uint32_t*)w.start,
                     (const uint32_t*)w.list, w.pos);
  // from here on w.list holds the Gaussians with more than k neighbours
  const size_t lds = (size_t)(kRunWords + a.k) * kPairThreads * sizeof(uint32_t) + (size_t)kPairThreads * a.k;
  hipLaunchKernelGGL(k_prune_pairs<BF16>, dim3(blocks(a.n, kPairThreads)), dim3(kPairThreads), lds, s, a,
                     (const uint32_t*)w.start, (const float4*)w.pos, (const Rec<BF16>*)rec, w.sem, w.list, w.pc);
  hipLaunchKernelGGL((a.k <= kPruneKMax / 2 ? k_prune_heavy<BF16, kPruneKMax / 2> : k_prune_heavy<BF16, kPruneKMax>),
                     dim3(std::min(blocks(a.n, kHeavyThreads), 8192u)), dim3(kHeavyThreads), 0, s, a,
                     (const uint32_t*)w.start, (const float4*)w.pos, (const Rec<BF16>*)rec, w.sem,
                     (const uint32_t*)w.list, (const PruneCounters*)w.pc);
}

}  // namespace

int prune_k_max() { return kPruneKMax; }

size_t prune_rec_bytes(int bf16) { return bf16 ? sizeof(Rec<true>) : sizeof(Rec<false>); }

// At least two buckets per Gaussian, so that folded cells add few candidates.
uint32_t prune_buckets(int64_t n) {
  uint32_t m = kMinBuckets;
  while ((int64_t)m < 2 * n) m *= 2u;
  return m;
}

void launch_prune(const PruneArgs& a, const PruneWork& w, uint8_t* mask, hipStream_t s) {
  if (a.feat_bf16) launch_t<true>(a, w, s);
  else launch_t<false>(a, w, s);
  const int vec = ((uintptr_t)mask & 3u) == 0;
  hipLaunchKernelGGL(k_prune_final, dim3(std::min(blocks(a.n, 1024), 256u)), dim3(256), 0, s, a.n, vec,
                     (const uint8_t*)w.sem, (const uint8_t*)w.geo, mask, w.pc);
}

}  // namespace lgs
