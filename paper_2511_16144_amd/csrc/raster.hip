// Per-pixel compositing of RGB + depth + 16-d feature (forward) and its
// reverse-order backward, plus the per-Gaussian segmented reduction of the
// backward's partial sums.
//
// Paper: Sec. III-B.1 renders the image and the feature map with the usual
// 3D Gaussian Splatting rasterizer; Eq. (1) uses the rendered depth; Sec. III-B.3
// optimises the Gaussians through this renderer.  Per pixel, front to back
// over the Gaussians of its tile in (depth, index) order:
//   alpha = min(alpha_max, o exp(-m2/2)), skipped unless m2 <= cutoff2 and
//   alpha >= alpha_min; T' = T (1 - alpha); stop before T' < T_eps;
//   Y += alpha T [r, g, b, z, f0..f15]; T = T'.
//
// Execution.  One wave64 renders one 8x8 pixel block (one pixel per lane)
// and walks the list of the binning tile that holds the block, 64 entries at
// a time: each lane loads one entry's geometry record with a vector load and
// tests whether the entry's ellipse can reach the block at all (cull_hit); a
// ballot gives the mask of entries to evaluate.  The wave then visits those
// entries in list order.  What an entry carries is wave-uniform: its geometry
// comes to SGPRs by a scalar load, requested one entry ahead, and is used
// directly as VALU operands, its appearance goes to the matrix cores, so no
// LDS staging of records is needed.  The wave leaves the list as soon as a ballot
// shows every lane finished.  Waves pop blocks from per-XCD work queues
// (persistent grid).
//
// Backward.  Each wave restarts from the last entry that any of its pixels can
// have taken (the list's end unless they all terminated before it) and walks the
// list backwards, recovering T before each entry as T / (1 - alpha)
// and the weighted sum of what lies behind as a single running scalar.  The
// sums over the wave's pixels, 6 geometric (the moments of dL/dalpha alpha up to
// the second in the Gaussian's frame) and 20 colour / depth / feature partials, sum_p w_p
// g_p, are products on the matrix cores over batches of 16 entries.  Both go
// to the entry's own (Gaussian, block) slot; a segmented
// reduction over each Gaussian's slots then forms its gradient.  No atomics:
// results are deterministic run to run.
#include "lgs_internal.h"

#include <algorithm>
#include <type_traits>

namespace lgs {
namespace {

// The forward and the backward evaluate an entry with this one function so
// that their discrete decisions agree bit for bit.
struct Eval {
  float m2, G, araw, alpha;
  bool pass;
};

__device__ __forceinline__ Eval eval_entry(float dx, float dy, float qa, float qb2, float qc, float o,
                                           float cutoff2, float alpha_max, float alpha_min) {
#pragma clang fp contract(off)
  Eval e;
  const float t1 = qc * dy;
  const float t2 = t1 * dy;
  const float t3 = qb2 * dx;
  const float t4 = __builtin_fmaf(t3, dy, t2);
  const float t5 = qa * dx;
  e.m2 = __builtin_fmaf(t5, dx, t4);
  e.G = __builtin_amdgcn_exp2f(e.m2 * -0.72134752044448170f);   // exp(-m2/2)
  e.araw = o * e.G;
  // min(araw, alpha_max) as a single v_min_f32 (equal to fminf here: araw
  // is a product, never a signalling NaN); fminf would first canonicalise
  // the setting with an instruction of its own at every entry
  asm("v_min_f32 %0, %1, %2" : "=v"(e.alpha) : "s"(alpha_max), "v"(e.araw));
  e.pass = (e.m2 <= cutoff2) && (e.alpha >= alpha_min);
  return e;
}

__device__ __forceinline__ bool block_in_bbox(uint32_t bb, uint32_t bx, uint32_t by) {
  return bx >= (bb & 255u) && bx <= ((bb >> 8) & 255u) && by >= ((bb >> 16) & 255u) && by <= (bb >> 24);
}

// Can the entry's ellipse reach the 8x8 block (bx, by) at all?  The minimum
// of the quadratic form over the block's pixel rectangle is 0 when the
// rectangle holds the centre, else the smallest of the four edge minima (a
// clamped 1-D minimiser per edge).  The entry is skipped only when that
// minimum exceeds the per-pixel cut min(cutoff2, 2 ln(o / alpha_min)) by a
// margin that covers the FP32 rounding of both this test and the per-pixel
// evaluation (whose error grows with (qa + qc) |d|^2), so the test never
// drops an entry that eval_entry would accept at some pixel of the block.
// The edge minimisers use the hardware reciprocal (about 1 ulp): a minimiser
// off by that much raises the edge minimum by a second-order amount, far
// inside the margin.
__device__ __forceinline__ bool cull_hit(const GeomRec& g, uint32_t bx, uint32_t by, float cutoff2,
                                         float log2_alpha_min) {
  const int bx0 = (int)(g.bbox & 255u), by0 = (int)((g.bbox >> 16) & 255u);
  const float x0 = (float)(8 * ((int)bx - bx0)) - g.mx, x1 = x0 + 7.f;
  const float y0 = (float)(8 * ((int)by - by0)) - g.my, y1 = y0 + 7.f;
  float m = 0.f;
  if (!(x0 <= 0.f && x1 >= 0.f && y0 <= 0.f && y1 >= 0.f)) {
    const float ia = -g.qb2 * __builtin_amdgcn_rcpf(2.f * g.qa), ic = -g.qb2 * __builtin_amdgcn_rcpf(2.f * g.qc);
    auto qf = [&](float dx, float dy) { return g.qa * dx * dx + g.qb2 * dx * dy + g.qc * dy * dy; };
    // clamps as one v_med3_f32 each (finite operands: no NaN handling)
    const float e0 = qf(x0, __builtin_amdgcn_fmed3f(ic * x0, y0, y1));
    const float e1 = qf(x1, __builtin_amdgcn_fmed3f(ic * x1, y0, y1));
    const float e2 = qf(__builtin_amdgcn_fmed3f(ia * y0, x0, x1), y0);
    const float e3 = qf(__builtin_amdgcn_fmed3f(ia * y1, x0, x1), y1);
    m = __builtin_fminf(__builtin_fminf(e0, e1), __builtin_fminf(e2, e3));
  }
  const float r2 = fminf(cutoff2, 1.3862943611198906f * (__builtin_amdgcn_logf(g.o) - log2_alpha_min));
  const float d2 = fmaxf(x0 * x0, x1 * x1) + fmaxf(y0 * y0, y1 * y1);
  return m <= r2 * 1.0001f + 1e-3f + 4e-6f * (g.qa + g.qc) * d2;
}

// A list entry's whole record for the cull test, requested as one: its
// fields are used at once, so the compiler cannot defer those the box test
// does not need below that test's branch (a further dependent round trip
// per chunk).
__device__ __forceinline__ GeomRec load_rec_whole(const GeomRec* __restrict__ p) {
  const GeomRec g = *p;
  asm volatile("" ::"v"(g.mx), "v"(g.my), "v"(g.qa), "v"(g.qb2), "v"(g.qc), "v"(g.o), "v"(g.z), "v"(g.bbox));
  return g;
}

// The lowest set bit of a wave mask (~0 if none: as a lane index, 63) and a
// mask without bit j (an empty mask stays empty): one scalar instruction each,
// in loops where the scalar unit is nearly as busy as the vector unit.
__device__ __forceinline__ uint32_t first_lane(uint64_t m) {
  uint32_t j;
  asm("s_ff1_i32_b64 %0, %1" : "=s"(j) : "s"(m));
  return j;
}
__device__ __forceinline__ uint64_t without_lane(uint64_t m, uint32_t j) {
  asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(j));
  return m;
}

// Record of list entry j's Gaussian (rid in lane j) by a scalar load whose
// offset is a 32-bit register (records sit below 2^32 bytes): one shift of
// the index instead of 64-bit address arithmetic per entry.
__device__ __forceinline__ GeomRec rec_of_lane(const GeomRec* __restrict__ geom, uint32_t rid_l, uint32_t j) {
  const uint32_t off = (uint32_t)__builtin_amdgcn_readlane((int)rid_l, (int)j) << 5;
  return *(const GeomRec*)((const char*)geom + off);
}

// Pop one work item for the whole wave.  Every active lane executes the
// atomic (no lane-dependent branch around it): the first active lane adds 1,
// the others 0, and the first active lane's return value is broadcast.  A
// "lane 0 only" branch here let the compiler merge it with the other
// lane-0 branches of the loop and drop lane 0 from EXEC at the back edge,
// after which readfirstlane read another lane's stale value.
__device__ __forceinline__ uint32_t pop_item(uint32_t* counter) {
  const uint64_t exec = __builtin_amdgcn_read_exec();
  const uint32_t lane = __lane_id();
  const bool leader = lane == (uint32_t)(__builtin_ctzll(exec));
  const uint32_t old = atomicAdd(counter, leader ? 1u : 0u);
  return __builtin_amdgcn_readfirstlane(old);
}

// Next work item of the calling wave from the queue of its XCD (workgroup
// index mod kQueues), or n_items once that queue is empty.  Wave-uniform.
// (Taking items from other queues once the own queue is empty was measured
// slower: the longest-first order already leaves a short tail.)
__device__ __forceinline__ uint32_t next_item(uint32_t* ctr, const uint32_t* __restrict__ qoff, uint32_t q,
                                              uint32_t n_items) {
  const uint32_t k = pop_item(&ctr[q * kLineWords]);
  const uint32_t b = qoff[q], e = qoff[q + 1];
  return k < e - b ? b + k : n_items;
}

// The image planes' addresses come from tables in memory: said to be global
// memory, their accesses are global ones and not flat ones (which wait on the
// LDS counter too).
typedef __attribute__((address_space(1))) float* gfloat_ptr;
typedef __attribute__((address_space(3))) float* lds_ptr;
__device__ __forceinline__ float gload(const float* p) { return *(gfloat_ptr)p; }
__device__ __forceinline__ void gstore(float* p, float x) { *(gfloat_ptr)p = x; }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// Forward accumulation on the matrix cores.
//
// FP32 appearance: an entry adds w[p] y[s] to the 20 sums of every pixel p, an
// outer product, which v_mfma_f32_4x4x1_16b_f32 forms for 4 channels and all
// 64 pixels at once.  Its 16 blocks are 4 x 4 x 1 products: with one block's
// A broadcast to all of them (cbsz 4, abid j), the A operand is channels
// 4 j .. 4 j + 3 (lane c of a register holding the entry's channel c, so one
// load per entry brings all 20), the B operand is each lane's own weight, and
// the result lands in the pixel's own lane (register i of block j: slot
// 4 j + i).  Each step is an FP32 fused multiply-add, bit for bit that of
// v_fmac_f32: five instructions of the matrix pipe in place of 20 of the VALU.
//
// BF16 appearance: the 20 sums acc[p][s] = sum_e w[p][e] y[e][s] of a batch
// of 8 entries form one v_mfma_f32_16x16x32_bf16 per group of 4 channel slots
// s and per term of the weights: the K index runs over (pixel group g' =
// lane / 16, entry e), the weights w (the B operand) are each lane's own, and
// the A operand is block diagonal (the appearance y in the rows of the lane's
// own pixel group, zero elsewhere), so the result lands in the lane of its
// pixel: lane l holds acc[l][4 j + i] in register i of block j.  The weights
// are split exactly into three BF16 terms (8 significant bits each) and the
// BF16 appearance is exact, so every product is exact and only the FP32
// accumulation rounds.
//
// The depth slot is accumulated separately in FP32 in both.
// LDS of one wave (BF16): the batch's weights [8 entries][64 pixels] (FP32, so
// that an entry's store is one conflict-free word per lane; they are split
// when the batch is full), its appearance [20 slots][8 entries] (BF16; the
// lanes past the 20 slots store slot 19's value to its place too, so the
// store needs no lane mask) and a zero block [20][8].
constexpr int kFwdY = 20 * 8;
constexpr int kFwdW = 8 * 64;
constexpr int kFwdWaveLds = kFwdW * 4 + 2 * kFwdY * 2;
constexpr int kAppAll = 4;   // cbsz of the FP32 form: one of the 16 blocks broadcast to all

// Lane c's channel slot of Gaussian g's appearance (c < 20; the lanes past
// them repeat the last one, which no product reads); slot 3 is 0.  A buffer
// load takes the record's offset as a scalar and the lane's offset in it as a
// fixed register, so it needs no address arithmetic on the vector side and no
// registers for it.  (The records stay below 2^32 bytes.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t app_buffer(const void* app) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)app, 0, -1, 0x00020000);
}
template <bool BF16>
__device__ __forceinline__ uint32_t load_app_lane(__amdgpu_buffer_rsrc_t app, uint32_t g, uint32_t ylane) {
  if (BF16) return __builtin_amdgcn_raw_buffer_load_b16(app, 2u * ylane, g * 40u, 0);
  return __builtin_amdgcn_raw_buffer_load_b32(app, 4u * ylane, g * 80u, 0);
}

// px - 8 bx0 for a pixel coordinate px and a record's first block bx0, both
// offset by 2^23, where the FP32 spacing is 1: integer arithmetic on the
// scalar side, one exact subtraction per lane.
constexpr float kPixBias = 8388608.f;
__device__ __forceinline__ float block_px_bias(uint32_t b0) { return __uint_as_float(0x4b000000u + (b0 << 3)); }

// FP32 appearance: eight waves per SIMD (64 VGPRs).  BF16 appearance: seven
// (72 VGPRs), so that a batch's weight operands stay in registers across its
// five channel blocks (faster than eight waves that re-read them).
//
// What bounds it: instruction issue, the vector and the scalar unit together
// (per visited entry 38 vector and 26 scalar instructions, of which 5 and few
// are the 64-entry cull's), and in calls with few blocks the latency of one
// wave's loop.  300k Gaussians, 640 x 480, FP32: 158 -> 103 us (products in
// place of 20 multiply-adds; the records of the next entry in flight while one
// is worked on, without the copies and branches that cost: 158 -> 120; scalar
// mask arithmetic by single instructions: -> 103).  500k Gaussians, 8 views,
// BF16: 690 -> 609 us.
// NC: per-pixel contributor counts are written (a caller asked for them);
// without them the entry loop keeps no count.
template <bool BF16, bool CNT, bool NC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(BF16 ? 7 : 8, BF16 ? 7 : 8))) k_raster_fwd(
    Settings st, Groups gr, const ViewDesc* __restrict__ views, const ViewImages* __restrict__ out,
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ vals,
    const GeomRec* __restrict__ geom, const void* __restrict__ app, uint32_t npad_mask,
    const uint32_t* __restrict__ items, const uint32_t* __restrict__ qoff, uint32_t n_items,
    Counters* __restrict__ cnt, uint32_t* __restrict__ work_q, int32_t* __restrict__ last_idx,
    float* __restrict__ T_state) {
  const int lane = threadIdx.x & 63;
  if (cnt->overflow) return;
  if (gr.total > 1) {   // (groups of one pixel write the same last entry and T)
    out += (size_t)blockIdx.y * gr.n_views;
    app = (const char*)app + blockIdx.y * gr.app_stride;
    work_q += blockIdx.y * kQueueWords;
  }
  extern __shared__ __attribute__((aligned(16))) float lds_f[];
  float* ws = lds_f + (threadIdx.x >> 6) * (kFwdWaveLds / 4);
  unsigned short* ys = (unsigned short*)(ws + kFwdW);
  unsigned short* yz = ys + kFwdY;
  // A-operand rows: lane l reads slot 4 j + (l & 3) when its row group
  // (l & 15) / 4 equals its k-block l / 16, else the zero block
  const unsigned short* abase = (((lane & 15) >> 2) == (lane >> 4) ? ys : yz) + (lane & 3) * 8;
  const uint32_t ylane = lane < 20 ? (uint32_t)lane : 19u;
  const __amdgpu_buffer_rsrc_t app_b = app_buffer(app);
  if (BF16) {
    // the zero block, and the weights: a partial batch leaves the weights of
    // its unused entries as they were (their appearance is zeroed instead),
    // so they must never hold a NaN or infinity from whatever LDS held before
    ((uint32_t*)yz)[lane] = 0u;
    if (lane < kFwdY / 2 - 64) ((uint32_t*)yz)[64 + lane] = 0u;
#pragma unroll
    for (int e = 0; e < 8; ++e) ws[e * 64 + lane] = 0.f;
  }
  // this wave's work (CNT: the profiling variant), added to the 64-bit
  // counters once at the end (a wave's own count stays far below 2^32); the
  // timed variant carries none of this bookkeeping in its entry loop
  uint32_t n_eval = 0, n_con = 0, n_ent = 0;
  const uint32_t q = blockIdx.x % (uint32_t)kQueues;
  for (;;) {
    const uint32_t it = next_item(work_q, qoff, q, n_items);
    if (it >= n_items) break;
    const uint32_t item = items[it];
    const uint32_t bx = item & 255u, by = (item >> 8) & 255u, v = item >> 16;
    const ViewDesc* V = views + v;
    const int W = V->W, H = V->H;
    const int px = (int)bx * kBlock + (lane & 7), py = (int)by * kBlock + (lane >> 3);
    const bool inside = px < W && py < H;
    const float pxb = kPixBias + (float)px, pyb = kPixBias + (float)py;
    const uint32_t tile = (uint32_t)V->tile_off + (by >> st.tile_shift) * (uint32_t)V->tiles_x +
                          (bx >> st.tile_shift);
    const uint2 r = ranges[tile];
    float T = 1.f;
    f32x4 D[5];      // slots 4 j .. 4 j + 3 of this lane's pixel
#pragma unroll
    for (int jb = 0; jb < 5; ++jb) D[jb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float accz = 0.f;
    int nb = 0;
    auto flush = [&]() {
      if (nb < 8 && lane < 20)
        for (int e = nb; e < 8; ++e) ys[lane * 8 + e] = 0;
      // the weights (the B operand, the same for the five channel blocks):
      // w = hi + mid + lo exactly, each term the top 8 significant bits of
      // what is left (truncation), so each is a BF16 value: the high halves
      // of two entries' words are packed by one byte permutation
      uint32_t tw[3][4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        uint32_t u[2][3];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float w = ws[(e + i) * 64 + lane];
          const float r1 = w - __uint_as_float(__float_as_uint(w) & 0xffff0000u);
          const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
          u[i][0] = __float_as_uint(w);
          u[i][1] = __float_as_uint(r1);
          u[i][2] = __float_as_uint(r2);
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) tw[t][e / 2] = __builtin_amdgcn_perm(u[1][t], u[0][t], 0x07060302u);
      }
      bf16x8_t bw[3];
#pragma unroll
      for (int t = 0; t < 3; ++t)
        bw[t] = __builtin_bit_cast(bf16x8_t, make_uint4(tw[t][0], tw[t][1], tw[t][2], tw[t][3]));
      // two channel blocks at a time, so that a product does not wait for the
      // one before it
#pragma unroll
      for (int jb = 0; jb < 5; jb += 2) {
        const bf16x8_t a0 = *(const bf16x8_t*)(abase + 32 * jb);
        const bf16x8_t a1 = *(const bf16x8_t*)(abase + 32 * (jb < 4 ? jb + 1 : jb));
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          D[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bw[t], D[jb], 0, 0, 0);
          if (jb < 4) D[jb + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bw[t], D[jb + 1], 0, 0, 0);
        }
      }
      nb = 0;
    };
    // the last list entry a pixel can have taken: the one before that which
    // would have ended it, else the list's last (set where a pixel ends, not at
    // every contribution: what lies between its last contributor and this
    // entry fails the same tests again in the backward)
    int32_t last = (int32_t)r.y - 1, ncon = 0;
    // the lanes still compositing, as a wave mask in SGPRs: per-lane tests
    // enter it through ballots of single comparisons and leave it through
    // inverse ballots, so the bookkeeping costs scalar instructions only
    uint64_t live = __builtin_amdgcn_ballot_w64(inside);
    // the list entries of the next chunk are requested a chunk ahead
    uint32_t rid_n = 0;
    if (r.x + (uint32_t)lane < r.y) rid_n = vals[r.x + (uint32_t)lane];
    for (uint32_t base = r.x; base < r.y && live != 0ull; base += 64) {
      // lane l takes entry base + l and decides whether the wave visits it
      const uint32_t kl = base + (uint32_t)lane;
      const uint32_t rid_l = rid_n;
      bool hit = false;
      if (kl < r.y) {
        const GeomRec g_l = load_rec_whole(geom + rid_l);
        hit = block_in_bbox(g_l.bbox, bx, by) && cull_hit(g_l, bx, by, st.cutoff2, st.log2_alpha_min);
      }
      if (kl + 64u < r.y) rid_n = vals[kl + 64u];
      uint64_t hm = __builtin_amdgcn_ballot_w64(hit);
      if (hm == 0ull) continue;
      int left = __builtin_popcountll(hm);   // the entries to visit
      // An entry's records (geometry by a scalar load, appearance by one lane
      // load) are requested while the entry before it is worked on.  The loop
      // takes two entries a turn, so that each of the two sets of registers
      // is loaded in place (a copy from one to the other would wait for the
      // load).  After the chunk's last entry the request repeats lane 63's
      // records (a list entry's, or record 0 past the end), which nothing
      // uses: no branch around it.
      auto request = [&](uint32_t& j, GeomRec& gr, uint32_t& yw) {
        j = first_lane(hm);
        hm = without_lane(hm, j);
        gr = rec_of_lane(geom, rid_l, j);
        yw = load_app_lane<BF16>(app_b, __builtin_amdgcn_readlane(rid_l, j) & npad_mask, ylane);
        // the requests stay here: the loads are not moved to their uses
        asm volatile("" ::: "memory");
      };
      // the record has arrived (scalar loads return in any order, so this
      // waits for all: the next request comes after it)
      auto arrived = [&](const GeomRec& gr) {
        asm volatile("" ::"s"(gr.mx), "s"(gr.my), "s"(gr.qa), "s"(gr.qb2), "s"(gr.qc), "s"(gr.o), "s"(gr.z),
                     "s"(gr.bbox));
      };
      auto work = [&](uint32_t j, const GeomRec& gr, uint32_t yw) {
        const uint32_t bb = gr.bbox;
        if (CNT) {
          n_eval += (uint32_t)__popcll(live);
          ++n_ent;
        }
        const float dx = (pxb - block_px_bias(bb & 255u)) - gr.mx;
        const float dy = (pyb - block_px_bias((bb >> 16) & 255u)) - gr.my;
        const Eval e = eval_entry(dx, dy, gr.qa, gr.qb2, gr.qc, gr.o, st.cutoff2, st.alpha_max, st.alpha_min);
        const float Tn = T * (1.f - e.alpha);
        // e.pass, as a mask
        const uint64_t pm = live & __builtin_amdgcn_ballot_w64(e.m2 <= st.cutoff2) &
                            __builtin_amdgcn_ballot_w64(e.alpha >= st.alpha_min);
        const uint64_t tm = pm & __builtin_amdgcn_ballot_w64(Tn < st.T_eps);   // terminates here
        if (tm != 0ull) {
          live &= ~tm;
          if (live == 0ull) left = 1;   // nothing after this entry
          last = __builtin_amdgcn_inverse_ballot_w64(tm) ? (int32_t)(base + j) - 1 : last;
        }
        const uint64_t cmask = pm & ~tm;
        if (cmask != 0ull) {
          const bool con = __builtin_amdgcn_inverse_ballot_w64(cmask);
          if (CNT) n_con += (uint32_t)__popcll(cmask);
          const float w = con ? e.alpha * T : 0.f;
          accz = __builtin_fmaf(w, gr.z, accz);
          T = con ? Tn : T;
          if (NC) ncon += con ? 1 : 0;
          if (BF16) {
            ws[nb * 64 + lane] = w;
            ys[ylane * 8 + nb] = (unsigned short)yw;
            if (++nb == 8) flush();
          } else {
            const float y = __uint_as_float(yw);
            D[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(y, w, D[0], kAppAll, 0, 0);
            D[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(y, w, D[1], kAppAll, 1, 0);
            D[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(y, w, D[2], kAppAll, 2, 0);
            D[3] = __builtin_amdgcn_mfma_f32_4x4x1f32(y, w, D[3], kAppAll, 3, 0);
            D[4] = __builtin_amdgcn_mfma_f32_4x4x1f32(y, w, D[4], kAppAll, 4, 0);
          }
        }
      };
      uint32_t j0, j1, y0, y1;
      GeomRec g0, g1;
      request(j0, g0, y0);
      for (;;) {
        arrived(g0);
        request(j1, g1, y1);
        work(j0, g0, y0);
        if (--left == 0) break;
        arrived(g1);
        request(j0, g0, y0);
        work(j1, g1, y1);
        if (--left == 0) break;
      }
    }
    if (BF16 && nb > 0) flush();
    if (inside) {
      const ViewImages o = out[v];
      const size_t HW = (size_t)W * H, p = (size_t)py * W + px;
#pragma unroll
      for (int c = 0; c < 3; ++c) gstore(o.rgb + c * HW + p, D[0][c]);
      gstore(o.depth + p, accz);
#pragma unroll
      for (int c = 0; c < 16; ++c)
        if (c < st.nfeat) gstore(o.feat + c * HW + p, D[1 + c / 4][c & 3]);
      gstore(o.T + p, T);
      if (NC && o.n_contrib) o.n_contrib[p] = ncon;
      last_idx[(size_t)V->pix_off + p] = last;
      T_state[(size_t)V->pix_off + p] = T;
    }
  }
  if (CNT && lane == 0) {
    atomicAdd(&cnt->fwd_evals, (unsigned long long)n_eval);
    atomicAdd(&cnt->fwd_contrib, (unsigned long long)n_con);
    atomicAdd(&cnt->fwd_entries, (unsigned long long)n_ent);
  }
}

__device__ __forceinline__ int wave_max_i32(int x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = max(x, __shfl_xor(x, off, 64));
  return x;
}

// Backward compositing.  What bounds it: VALU issue when every SIMD holds
// several waves (large calls), and the latency of one wave's entry loop when
// a call has few blocks (a single view has about as many blocks as the chip
// has wave slots).  So what is a contraction goes to the matrix cores, whose
// pipe is idle otherwise, and what an entry reads is requested an entry (its
// geometry) or a group of four entries (their appearance) ahead.
//   - gy[p] = sum_c g[p][c] y[c], per pixel and entry: for four entries at
//     once by the 16-block 4 x 4 products (block b: the four lanes 4 b ..
//     4 b + 3, its columns their pixels, its rows the four entries; the A
//     block of 4 channels broadcast to all blocks by cbsz / abid).  The
//     appearance is the A operand as it is loaded: lane 4 q + i brings
//     channels 4 q .. 4 q + 3 of entry i.  With BF16 appearance and the sign
//     upstream, v_mfma_f32_4x4x4_16b_bf16 takes 4 channels an instruction
//     (exact products); else v_mfma_f32_4x4x1_16b_f32 takes one (FP32 fused
//     multiply-adds).
//   - the six geometric sums sum_p u[p] {1, X, Y, X^2, X Y, Y^2}, u =
//     dL/dalpha alpha, X, Y the pixel's position from the block's centre:
//     (6 x pixels) x (pixels x entries) in FP64 (v_mfma_f64_4x4x4_4b_f64, its
//     four blocks four entries each), once per batch of 16 entries; then they
//     are moved to the entry's mean.  The move cancels, the more the smaller the
//     Gaussian is against its distance from the centre.  (Scale and
//     rotation gradients of Gaussians of up to 1.2 px alone on their pixels are
//     3e-7 to 6e-7 of their norm off with FP32 sums about the centres of 4 x 4
//     quarters, 1.0e-7 to 1.3e-7 with FP32 sums about the mean, 0.8e-7 to 1.1e-7
//     so.)  A row of pixels and its mirror image in the block's middle have the
//     same {1, X, X^2, Y^2} and opposite {Y, X Y}, so products of the rows' sums
//     and differences are half as many: 16 of 16 cycles for a batch, where the
//     quarters' were 16 of 32.  Still in FP64 the sums go to the entry's own frame
//     (frame_shear), in which they are rounded (eight views of 500k: 1085 ->
//     1092 us).
//   - the 20 colour partials sum_p g[p][c] w[p]: (channels x pixels) x (pixels
//     x entries) on BF16 terms whose sums are exact, once per batch; a lane
//     then holds four consecutive channels of one entry and stores them as
//     they are.
// The vector and the matrix pipe of a SIMD hardly overlap here (their busy
// cycles add up to nearly all of the kernel's), so a product is worth its place
// only where it takes fewer cycles than the vector instructions it replaces.
// Per visited entry 59 vector instructions (88 with the sums by lane exchanges
// and dot products and a batch of 8), 3 of them products, and 30 scalar ones.
// On one card, 500k Gaussians, 8 views, BF16, fused L1: 1385 -> 1100 us; 300k,
// 640 x 480, FP32: 139 -> 107 us; 2k, 128 x 96: 47 -> 30 us (there the records
// in flight an entry ahead and a block's planes requested at once count).
// Batches of 8 took 12 % longer; five waves per SIMD in place of four changed
// nothing.
constexpr int kBatch = 16;                 // entries per batch
constexpr int kZRow = 72;                  // bf16 per upstream row (64 pixels + pad; 144 B, 16-B aligned)
constexpr int kWRow = 68;                  // floats per weight / u row (64 pixels + pad; 272 B, 16-B aligned)
constexpr int kBatchBytes = 2 * kBatch * kWRow * 4;
// LDS bytes of one backward wave: the batch's weight rows and u rows (FP32),
// and the upstream rows of channels 16-19 (BF16, hi, and lo with a given
// upstream).  The block's other upstream rows (hi 0-15, then lo) pass through
// the batch's rows on their way into registers.
__host__ __device__ constexpr int bwd_wave_lds(int up_mode) {
  return kBatchBytes + (up_mode == UP_EXPLICIT ? 8 : 4) * kZRow * 2;
}
static_assert(32 * kZRow * 2 <= kBatchBytes, "the upstream rows fit");
// ... and of the work-group: the moments' basis over a row's 8 pixels, FP64:
// 1, X, X^2, then of each row distance k + 1/2 from the block's middle Y^2, Y and
// X Y (4 rows each)
constexpr int kBasisOne = 0, kBasisYY = 3, kBasisY = 7, kBasisXY = 11, kBasisRows = 15;
constexpr int kBasisBytes = kBasisRows * 8 * 8;
// FP32 -> BF16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ unsigned short bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf16_to_f(unsigned short h) { return __uint_as_float((uint32_t)h << 16); }

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ int amdgcn_writelane(int val, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// A value of each row of 16 lanes brought to every lane's column: rows 0 and 1,
// the same of rows 2 and 3 in the upper half (even, odd); then the halves.
__device__ __forceinline__ void exchange_rows(double x, double& even, double& odd) {
  const u32x2_t w = __builtin_bit_cast(u32x2_t, x);
  const auto a = __builtin_amdgcn_permlane16_swap(w[0], w[0], false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(w[1], w[1], false, false);
  even = __builtin_bit_cast(double, (u32x2_t){(uint32_t)a[0], (uint32_t)b[0]});
  odd = __builtin_bit_cast(double, (u32x2_t){(uint32_t)a[1], (uint32_t)b[1]});
}
__device__ __forceinline__ void exchange_halves(double x, double& lower, double& upper) {
  const u32x2_t w = __builtin_bit_cast(u32x2_t, x);
  const auto a = __builtin_amdgcn_permlane32_swap(w[0], w[0], false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(w[1], w[1], false, false);
  lower = __builtin_bit_cast(double, (u32x2_t){(uint32_t)a[0], (uint32_t)b[0]});
  upper = __builtin_bit_cast(double, (u32x2_t){(uint32_t)a[1], (uint32_t)b[1]});
}

// Four waves per SIMD (128 VGPRs; what the LDS allows too).
template <bool BF16, int UPM, bool CNT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) k_raster_bwd(
    Settings st, Groups gr, const ViewDesc* __restrict__ views, const ViewImages* __restrict__ upstream,
    const ViewImages* __restrict__ fwd_out, const ViewImages* __restrict__ targets,
    const float* __restrict__ loss_w, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ vals, const GeomRec* __restrict__ geom,
    const void* __restrict__ app, uint32_t npad_mask, const uint32_t* __restrict__ items,
    const uint32_t* __restrict__ qoff, uint32_t n_items, Counters* __restrict__ cnt,
    uint32_t* __restrict__ work_q, const int32_t* __restrict__ last_idx,
    const float* __restrict__ T_state, const uint32_t* __restrict__ slot_base,
    float* __restrict__ partials, uint8_t* __restrict__ mask) {
  const int lane = threadIdx.x & 63;
  extern __shared__ __attribute__((aligned(16))) float lds_z[];
  // upstream per channel: the sign of the L1 residual (formed here from the
  // forward's images and the targets; exact in BF16, the per-channel scale is
  // applied after the product) or a given FP32 value (split hi + lo)
  constexpr bool kSignRGB = UPM == UP_L1;
  constexpr bool kSignDF = UPM != UP_EXPLICIT;
  // gy's feature part (and RGB with the sign upstream) on BF16 products
  constexpr bool kDotGy = BF16 && kSignDF;
  double* tab = (double*)lds_z;                      // [kBasisRows][8], the same from every wave
  float* ws = lds_z + kBasisBytes / 4 + (threadIdx.x >> 6) * (bwd_wave_lds(UPM) / 4);   // weight rows
  float* us = ws + kBatch * kWRow;                                                      // u rows
  lds_ptr wl = (lds_ptr)(ws + lane);                 // this lane's place in a row
  asm volatile("" : "+v"(wl));   // (one addition of a scalar per entry)
  unsigned short* wz = (unsigned short*)ws;          // upstream rows, before the first batch
  unsigned short* gz = wz + kBatchBytes / 2;         // upstream rows of channels 16-19 (hi, lo)
  const int grp = lane >> 4, col = lane & 15;
  if (cnt->overflow) return;
  if (gr.total > 1) {
    const uint32_t j = blockIdx.y, gi = ((uint32_t)gr.first + j) % (uint32_t)gr.total;
    const size_t tab_off = (size_t)gi * gr.n_views;
    if (UPM != UP_L1) upstream += tab_off;
    if (UPM != UP_EXPLICIT) {
      fwd_out += tab_off;
      targets += tab_off;
      loss_w += 4 * gi;
    }
    app = (const char*)app + gi * gr.app_stride;
    work_q += gi * kQueueWords;
    partials += j * gr.slots * kSlotFloats;
    mask += j * gr.mask_stride;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h, row = i >> 3, k = row < kBasisYY ? 0 : (row - kBasisYY) & 3;
    const double X = (double)(i & 7) - 3.5, Y = (double)k + 0.5;
    const double b = row == kBasisOne ? 1.0 : row == 1 ? X : row == 2 ? X * X : row < kBasisY ? Y * Y : row < kBasisXY ? Y : X * Y;
    if (row < kBasisRows) tab[i] = b;
  }
  asm volatile("" ::: "memory");
  // appearance of a group of four entries: lane 4 q + i loads channels 4 q ..
  // 4 q + 3 of entry i (q < 5; the lanes past them repeat the last channels)
  const __amdgpu_buffer_rsrc_t app_b = app_buffer(app);
  const uint32_t yoff = (uint32_t)min(lane >> 2, 4) * (BF16 ? 8u : 16u), yent = 8u * ((uint32_t)lane & 3u);
  // this wave's work (CNT: the profiling variant), added to the 64-bit
  // counters once at the end (a wave's own count stays far below 2^32)
  uint32_t n_eval = 0, n_con = 0, n_ent = 0, n_wr = 0;
  const uint32_t q = blockIdx.x % (uint32_t)kQueues;
  for (;;) {
    const uint32_t it = next_item(work_q, qoff, q, n_items);
    if (it >= n_items) break;
    const uint32_t item = items[it];
    const uint32_t bx = item & 255u, by = (item >> 8) & 255u, v = item >> 16;
    const ViewDesc* V = views + v;
    const int W = V->W, H = V->H;
    const int px = (int)bx * kBlock + (lane & 7), py = (int)by * kBlock + (lane >> 3);
    const bool inside = px < W && py < H;
    const size_t HW = (size_t)W * H, p = (size_t)py * W + px;
    int32_t last = -1;
    float Tfin = 1.f, gT = 0.f;
    float g[20];
#pragma unroll
    for (int c = 0; c < 20; ++c) g[c] = 0.f;
    if (inside) {
      // every plane requested before any value is used (planes past nfeat read
      // the first feature plane, which is there, and drop it): a load under a
      // test of its own would be waited for alone, one round trip per channel
      float a[20], b[20];
      auto feat_at = [&](const float* f, int c) { return gload(f + (c < st.nfeat ? c : 0) * HW + p); };
      if (kSignDF) {
        const ViewImages Y = fwd_out[v], Yt = targets[v];
        const float* __restrict__ Urgb = kSignRGB ? nullptr : upstream[v].rgb;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          a[c] = kSignRGB ? gload(Y.rgb + c * HW + p) : gload(Urgb + c * HW + p);
          b[c] = kSignRGB ? gload(Yt.rgb + c * HW + p) : 0.f;
        }
        a[3] = gload(Y.depth + p);
        b[3] = gload(Yt.depth + p);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          a[4 + c] = feat_at(Y.feat, c);
          b[4 + c] = feat_at(Yt.feat, c);
        }
      } else {
        const ViewImages U = upstream[v];
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = gload(U.rgb + c * HW + p);
        a[3] = gload(U.depth + p);
#pragma unroll
        for (int c = 0; c < 16; ++c) a[4 + c] = feat_at(U.feat, c);
        if (U.T) gT = gload(U.T + p);
      }
      last = last_idx[(size_t)V->pix_off + p];
      Tfin = T_state[(size_t)V->pix_off + p];
      asm volatile("" ::: "memory");
      if (kSignDF) {
        const float s_rgb = loss_w[0] / (3.f * (float)HW), s_d = loss_w[1] / (float)HW;
        const float s_f = loss_w[2] / (16.f * (float)HW);
#pragma unroll
        for (int c = 0; c < 20; ++c) {
          const float sc = c < 3 ? s_rgb : (c == 3 ? s_d : s_f), d = a[c] - b[c];
          g[c] = c < 3 && !kSignRGB ? a[c] : (d > 0.f ? sc : (d < 0.f ? -sc : 0.f));
          if (c >= 4 && c - 4 >= st.nfeat) g[c] = 0.f;
        }
      } else {
#pragma unroll
        for (int c = 0; c < 20; ++c) g[c] = c < 4 || c - 4 < st.nfeat ? a[c] : 0.f;
      }
    }
    // every lane holds the same maximum; readfirstlane makes that visible to
    // the compiler, so the entry loop below stays on the scalar unit
    const int kmax = __builtin_amdgcn_readfirstlane(wave_max_i32(last));
    const uint32_t tile = (uint32_t)V->tile_off + (by >> st.tile_shift) * (uint32_t)V->tiles_x +
                          (bx >> st.tile_shift);
    const uint32_t kbeg = ranges[tile].x;
    if (kmax < (int)kbeg) continue;
    const float pxb = kPixBias + (float)px, pyb = kPixBias + (float)py;
    const float gTT = gT * Tfin;
    float Tc = Tfin, sB = 0.f;
    // upstream rows: for the fused L1 gradient the sign (exact in BF16; the
    // per-channel scale is applied to the MFMA result), else hi + lo BF16.
    // The colour partials of a batch of entries, dY[e][c] = sum_p w[p][e] g[p][c],
    // are a (entries x pixels) x (pixels x channels) product: v_mfma_f32_16x16x32_bf16
    // on the exact terms of w (and hi + lo of a general upstream), FP32
    // accumulation.  The rows are written once per block and read back
    // transposed as the products' B operands, which stay in registers.
    float gscale[3] = {1.f, 1.f, 1.f};
    if (kSignDF) {
      const float HWf = (float)HW;
      // (the rows hold g's sign, which is the weight's times the residual's)
      gscale[0] = kSignRGB ? fabsf(loss_w[0]) / (3.f * HWf) : 1.f;
      gscale[1] = fabsf(loss_w[1]) / HWf;
      gscale[2] = fabsf(loss_w[2]) / (16.f * HWf);
    }
    asm volatile("" ::: "memory");   // (the last block's record reads come before)
#pragma unroll
    for (int c = 0; c < 20; ++c) {
      unsigned short* row = c < 16 ? wz + c * kZRow : gz + (c - 16) * kZRow;
      if (c < 3 ? kSignRGB : kSignDF) {
        const float sgn = g[c] > 0.f ? 1.f : (g[c] < 0.f ? -1.f : 0.f);
        row[lane] = bf16_rne(sgn);
      } else {
        const unsigned short hi = bf16_rne(g[c]);
        row[lane] = hi;
        row[(c < 16 ? 16 : 4) * kZRow + lane] = bf16_rne(g[c] - bf16_to_f(hi));
      }
    }
    asm volatile("" ::: "memory");
    bf16x8_t bh0[2], bl0[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int off = 32 * ks + 8 * grp;
      bh0[ks] = *(const bf16x8_t*)(wz + col * kZRow + off);
      if (UPM == UP_EXPLICIT) {
        bl0[ks] = *(const bf16x8_t*)(wz + (16 + col) * kZRow + off);
      } else if (UPM == UP_RGB) {   // lo rows exist for the three colour channels only
        bl0[ks] = *(const bf16x8_t*)(wz + (16 + (col < 3 ? col : 0)) * kZRow + off);
        if (col >= 3) bl0[ks] = (bf16x8_t){};
      }
    }
    asm volatile("" ::: "memory");
    // B operands of gy with the sign upstream and BF16 appearance: the signs
    // of channels 4 k .. 4 k + 3 (slot 3, the depth, apart)
    s16x4_t sg[5];
    if (kDotGy) {
#pragma unroll
      for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = g[4 * k + i];
          sg[k][i] = k == 0 && i == 3 ? (short)0 : (a > 0.f ? (short)0x3f80 : (a < 0.f ? (short)0xbf80 : (short)0));
        }
    }
    int nb = 0;
    uint32_t ridv = 0;   // lane e: the record id of the batch's entry e
    // Write the batch's nb partial records: the colour partials, sum_p g_p
    // w_p (each weight term against the same upstream, so with a sign upstream
    // every product is exact and only the FP32 accumulation rounds), and the
    // moments of u.  Lane (grp, col) gets channels 4 grp .. 4 grp + 3 of entry
    // col, channels 16 .. 19 in group 0, and of the moments 1, X, X^2, Y^2 and
    // Y, X Y, Y, X Y one each in the four groups.
    auto flush = [&]() {
      // (its lane constants are worked out here: the registers that they would
      // hold across the entry loop are short)
      int fl = lane;
      asm volatile("" : "+v"(fl));
      const int grp = fl >> 4, col = fl & 15;
      // the entries' geometry and slot bases again (used after the products)
      const uint32_t re = (uint32_t)__builtin_amdgcn_ds_bpermute(col * 4, (int)ridv);
      const GeomRec* __restrict__ ge = geom + re;
      const float emx = ge->mx, emy = ge->my, eqa = ge->qa, eqb = ge->qb2;
      const uint32_t ebb = ge->bbox, esb = slot_base[re];
      asm volatile("" ::: "memory");
      f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
      // K index: row distance grp; lane's row of A: col & 3
      double me = 0.0, mo = 0.0;   // of the sums and of the differences of mirrored rows
      {
        const int row = col & 3;
        const double* te = tab + 8 * (row < 3 ? row : kBasisYY + grp);
        const double* to = tab + 8 * ((row & 1 ? kBasisXY : kBasisY) + grp);
        const float *ua = us + col * kWRow + 8 * (4 + grp), *ub = us + col * kWRow + 8 * (3 - grp);
#pragma unroll
        for (int x = 0; x < 8; x += 4) {
          const f32x4 a = *(const f32x4*)(ua + x), b = *(const f32x4*)(ub + x);
#pragma unroll
          for (int i = 0; i < 4; i += 2) {
            const f64x2 e = *(const f64x2*)(te + x + i), o = *(const f64x2*)(to + x + i);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const double p = (double)a[i + h], q = (double)b[i + h];
              me = __builtin_amdgcn_mfma_f64_4x4x4f64(e[h], p + q, me, 0, 0, 0);
              mo = __builtin_amdgcn_mfma_f64_4x4x4f64(o[h], p - q, mo, 0, 0, 0);
            }
          }
          asm volatile("" ::: "memory");   // (half a row's operands at a time: no spills)
        }
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int off = 32 * ks + 8 * grp;
        // w = hi + mid + lo exactly: each term keeps the top 8 significant bits
        // of what is left (truncation), so each is a BF16 value: the high
        // halves of two pixels' words are packed by one byte permutation
        uint32_t tw[3][4];
        {
#pragma clang fp contract(off)
          const f32x4 w0 = *(const f32x4*)(ws + col * kWRow + off), w1 = *(const f32x4*)(ws + col * kWRow + off + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            uint32_t t3[2][3];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const float w = e < 2 ? w0[2 * e + i] : w1[2 * e - 4 + i];
              const float r1 = w - __uint_as_float(__float_as_uint(w) & 0xffff0000u);
              const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
              t3[i][0] = __float_as_uint(w);
              t3[i][1] = __float_as_uint(r1);
              t3[i][2] = __float_as_uint(r2);
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) tw[t][e] = __builtin_amdgcn_perm(t3[1][t], t3[0][t], 0x07060302u);
          }
        }
        bf16x8_t aw[3];
#pragma unroll
        for (int t = 0; t < 3; ++t)
          aw[t] = __builtin_bit_cast(bf16x8_t, make_uint4(tw[t][0], tw[t][1], tw[t][2], tw[t][3]));
        // (rows 4-15 of the second product repeat rows 0-3 and are not used)
        const bf16x8_t bh1 = *(const bf16x8_t*)(gz + (col & 3) * kZRow + off);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh0[ks], aw[t], c0, 0, 0, 0);
          c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh1, aw[t], c1, 0, 0, 0);
        }
        if (UPM == UP_EXPLICIT) {
          // the given upstream's lo term (relative 2^-8 of hi) against the two
          // leading weight terms: the dropped products are below 2^-24
          const bf16x8_t bl1 = *(const bf16x8_t*)(gz + (4 + (col & 3)) * kZRow + off);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl0[ks], aw[t], c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl1, aw[t], c1, 0, 0, 0);
          }
        } else if (UPM == UP_RGB) {
#pragma unroll
          for (int t = 0; t < 2; ++t) c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl0[ks], aw[t], c0, 0, 0, 0);
        }
      }
      // (the reads above precede the next batch's writes: the LDS operations
      // of a wave run in order; this keeps the compiler's order too)
      asm volatile("" ::: "memory");
      const uint32_t ebx = ebb & 255u, eby = (ebb >> 16) & 255u;
      const uint32_t sl = esb + (by - eby) * (((ebb >> 8) & 255u) - ebx + 1u) + (bx - ebx);
      // dx = X + x0, dy = Y + y0
      const double x0 = (double)(8 * ((int)bx - (int)ebx)) - (double)emx + 3.5;
      const double y0 = (double)(8 * ((int)by - (int)eby)) - (double)emy + 3.5;
      double e02, e13, m0, mx, mxx, myy, my, mxy;
      exchange_rows(me, e02, e13);
      exchange_halves(e02, m0, mxx);
      exchange_halves(e13, mx, myy);
      exchange_rows(mo, my, mxy);
      const double fx = __builtin_fma(x0, m0, mx), fy = __builtin_fma(y0, m0, my);
      const double gxx = __builtin_fma(x0, mx + fx, mxx), gyy = __builtin_fma(y0, my + fy, myy);
      const double gxy = __builtin_fma(x0, fy, __builtin_fma(y0, mx, mxy));
      // in the entry's frame
      const double kq = (double)frame_shear(eqa, eqb);
      const double fp = __builtin_fma(kq, fy, fx), gpy = __builtin_fma(kq, gyy, gxy);
      const double gpp = __builtin_fma(kq, gxy + gpy, gxx);
      const float s0 = grp == 0 ? gscale[0] : gscale[2], s3 = grp == 0 ? gscale[1] : gscale[2];
      float* rec = partials + (size_t)sl * kSlotFloats;
      if (col < nb) {
        *(float4*)(rec + 4 * grp) = make_float4(c0[0] * s0, c0[1] * s0, c0[2] * s0, c0[3] * s3);
        if (grp < 2) {
          float4 v4;
          v4.x = grp == 0 ? c1[0] * gscale[2] : (float)fp;   // Sp
          v4.y = grp == 0 ? c1[1] * gscale[2] : (float)fy;   // Sy
          v4.z = grp == 0 ? c1[2] * gscale[2] : (float)gpp;  // Spp
          v4.w = grp == 0 ? c1[3] * gscale[2] : (float)m0;   // S0
          *(float4*)(rec + 16 + 4 * grp) = v4;
        } else {
          rec[22 + grp] = (float)(grp == 2 ? gpy : gyy);     // Spy, Syy
        }
        if (grp == 0) mask[sl] = 1;
      }
      static_assert(kPartGeo == 20 && kPartials == 26, "the record's layout");
      nb = 0;
    };
    // the list entries of the next chunk are requested a chunk ahead
    uint32_t rid_n = 0;
    if (kmax - lane >= (int)kbeg) rid_n = vals[kmax - lane];
    for (int top = kmax; top >= (int)kbeg; top -= 64) {
      // lane l takes entry top - l (the list backwards) and decides whether
      // the wave visits it
      const int kl = top - lane;
      const uint32_t rid_l = rid_n;
      bool hit = false;
      if (kl >= (int)kbeg) {
        const GeomRec g_l = load_rec_whole(geom + rid_l);
        hit = block_in_bbox(g_l.bbox, bx, by) && cull_hit(g_l, bx, by, st.cutoff2, st.log2_alpha_min);
      }
      if (kl - 64 >= (int)kbeg) rid_n = vals[kl - 64];
      uint64_t hm = __builtin_amdgcn_ballot_w64(hit);
      if (hm == 0ull) continue;
      // The chunk's entries in groups of four.  take: the next group's lanes
      // (63 past the last) and its appearance, requested while the group
      // before it is worked on.
      uint32_t jn[4];
      u32x4_t yn;
      auto take = [&]() {
        uint32_t jp = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          jn[i] = first_lane(hm);
          hm = without_lane(hm, jn[i]);
          jp |= (jn[i] & 63u) << (8 * i + 2);
        }
        const uint32_t ge = (uint32_t)__builtin_amdgcn_ds_bpermute((int)__builtin_amdgcn_ubfe(jp, yent, 8),
                                                                   (int)rid_l) & npad_mask;
        if (BF16) {
          const u32x2_t t = __builtin_amdgcn_raw_buffer_load_b64(app_b, (ge * 5u << 3) + yoff, 0, 0);
          yn[0] = t[0];
          yn[1] = t[1];
        } else {
          yn = __builtin_amdgcn_raw_buffer_load_b128(app_b, (ge * 5u << 4) + yoff, 0, 0);
        }
        asm volatile("" ::: "memory");   // the request stays here
      };
      // an entry's record id and geometry, requested one entry ahead into the
      // other of two register sets (a copy would wait for the load)
      auto request = [&](uint32_t j, uint32_t& rid, GeomRec& gr) {
        rid = __builtin_amdgcn_readlane(rid_l, j);
        gr = *(const GeomRec*)((const char*)geom + (rid << 5));
        asm volatile("" ::: "memory");
      };
      // the geometry has arrived (scalar loads return in any order, so this
      // waits for all: the next request comes after it)
      auto arrived = [&](const GeomRec& gr) {
        asm volatile("" ::"s"(gr.mx), "s"(gr.my), "s"(gr.qa), "s"(gr.qb2), "s"(gr.qc), "s"(gr.o), "s"(gr.z),
                     "s"(gr.bbox));
      };
      auto work = [&](uint32_t j, uint32_t rid, const GeomRec& gr, float gyf, float gyc) {
        const int k = top - (int)j;
        const uint64_t lm = __builtin_amdgcn_ballot_w64(k <= last);   // lanes this entry can reach
        if (CNT) {
          n_eval += (uint32_t)__popcll(lm);
          ++n_ent;
        }
        const float dx = (pxb - block_px_bias(gr.bbox & 255u)) - gr.mx;
        const float dy = (pyb - block_px_bias((gr.bbox >> 16) & 255u)) - gr.my;
        const Eval e = eval_entry(dx, dy, gr.qa, gr.qb2, gr.qc, gr.o, st.cutoff2, st.alpha_max, st.alpha_min);
        // (k <= last) && e.pass, as a mask of single-comparison ballots and
        // back as a lane predicate (no VALU spent on the conversion)
        const uint64_t cmask = lm & __builtin_amdgcn_ballot_w64(e.m2 <= st.cutoff2) &
                               __builtin_amdgcn_ballot_w64(e.alpha >= st.alpha_min);
        if (cmask == 0ull) return;
        const bool con = __builtin_amdgcn_inverse_ballot_w64(cmask);
        if (CNT) {
          n_con += (uint32_t)__popcll(cmask);
          ++n_wr;
        }
        // a lane the entry does not reach: alpha 0, so T stays as it is (the
        // reciprocal of 1 is 1) and its weight is 0
        const float al = con ? e.alpha : 0.f;
        const float rinv = __builtin_amdgcn_rcpf(1.f - al);
        const float Tp = Tc * rinv;
        const float w = al * Tp;
        const float gy = kDotGy ? __builtin_fmaf(g[3], gr.z, __builtin_fmaf(gscale[2], gyf, kSignRGB ? gscale[0] * gyc : gyc))
                                : __builtin_fmaf(g[3], gr.z, gyf);
        const float dal = Tp * gy - (UPM == UP_EXPLICIT ? sB + gTT : sB) * rinv;   // gT = 0 otherwise
        sB = con ? __builtin_fmaf(w, gy, sB) : sB;
        Tc = Tp;
        // dL/dm2 per pixel is -1/2 u; the slot keeps the moments of u over the
        // pixel offsets (the factor -1/2 and the conic's entries are per
        // Gaussian, so they are applied once to the summed moments in the
        // projection backward), and their zeroth, from which the opacity's
        // gradient follows (below the clamp alpha is o G)
        const bool free_al = __builtin_amdgcn_inverse_ballot_w64(cmask & ~__builtin_amdgcn_ballot_w64(e.araw > st.alpha_max));
        const float u = free_al ? dal * al : 0.f;
        const lds_ptr row = wl + nb * kWRow;
        row[0] = w;
        row[kBatch * kWRow] = u;
        ridv = (uint32_t)amdgcn_writelane((int)rid, nb, (int)ridv);
        if (++nb == kBatch) flush();
      };
      int left = __builtin_popcountll(hm);
      uint32_t r0, r1;
      GeomRec g0, g1;
      take();
      request(jn[0], r0, g0);
      for (;;) {
        // gy of the group's four entries: entry i in register i
        f32x4 gf = {0.f, 0.f, 0.f, 0.f}, gc = {0.f, 0.f, 0.f, 0.f};
        if (kDotGy) {
          const s16x4_t ya = __builtin_bit_cast(s16x4_t, (u32x2_t){yn[0], yn[1]});
          gf = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ya, sg[1], gf, 4, 1, 0);
          gf = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ya, sg[2], gf, 4, 2, 0);
          gf = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ya, sg[3], gf, 4, 3, 0);
          gf = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ya, sg[4], gf, 4, 4, 0);
          if (kSignRGB) {
            gc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ya, sg[0], gc, 4, 0, 0);
          } else {
            gc = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(yn[0] << 16), g[0], gc, 4, 0, 0);
            gc = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(yn[0] & 0xffff0000u), g[1], gc, 4, 0, 0);
            gc = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(yn[1] << 16), g[2], gc, 4, 0, 0);
          }
        } else {
          float y4[4];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            y4[i] = __uint_as_float(!BF16 ? yn[i] : (i & 1) ? yn[i >> 1] & 0xffff0000u : yn[i >> 1] << 16);
#define LGS_GY(Q, I) gf = __builtin_amdgcn_mfma_f32_4x4x1f32(y4[I], g[4 * Q + I], gf, 4, Q, 0);
#define LGS_GY4(Q) LGS_GY(Q, 0) LGS_GY(Q, 1) LGS_GY(Q, 2) LGS_GY(Q, 3)
          LGS_GY(0, 0) LGS_GY(0, 1) LGS_GY(0, 2)
          LGS_GY4(1) LGS_GY4(2) LGS_GY4(3) LGS_GY4(4)
#undef LGS_GY4
#undef LGS_GY
        }
        const uint32_t j0 = jn[0], j1 = jn[1], j2 = jn[2], j3 = jn[3];
        take();
        arrived(g0);
        request(j1, r1, g1);
        work(j0, r0, g0, gf[0], gc[0]);
        if (left == 1) break;
        arrived(g1);
        request(j2, r0, g0);
        work(j1, r1, g1, gf[1], gc[1]);
        if (left == 2) break;
        arrived(g0);
        request(j3, r1, g1);
        work(j2, r0, g0, gf[2], gc[2]);
        if (left == 3) break;
        arrived(g1);
        request(jn[0], r0, g0);
        work(j3, r1, g1, gf[3], gc[3]);
        left -= 4;
        if (left == 0) break;
      }
    }
    if (nb > 0) flush();
  }
  if (CNT && lane == 0) {
    atomicAdd(&cnt->bwd_evals, (unsigned long long)n_eval);
    atomicAdd(&cnt->bwd_contrib, (unsigned long long)n_con);
    atomicAdd(&cnt->bwd_entries, (unsigned long long)n_ent);
    atomicAdd(&cnt->bwd_written, (unsigned long long)n_wr);
  }
}

// Per-Gaussian sum of the backward's partials.  Visible (view, Gaussian) c
// owns the slot range [slot_off[c], slot_off[c + 1]) (the last one ends at
// n_slots); a slot holds a partial only where the backward set its mask byte.
// Each half of a wave takes one c (waves loop over pairs of c, grid-stride,
// persistent grid).  Lane l of a half sums value l of every written slot, in
// slot order, so a half reads each slot as one contiguous 128-byte access
// and needs no exchange between lanes: per window of 32 slots, lane l tests
// slot l's mask byte, a ballot gives the half its written slots, and the
// half walks them lowest first in batches (2 kSegBatch while that many are
// left, else kSegBatch), each batch's loads requested before the first is
// added.  A fixed order, so results are deterministic.
//
// An id with more than kLongSlots slots (a near Gaussian that covers much of
// the frame: up to 12750 of them at 1200 x 680) would keep one half busy long
// after the others have run out.  A work-group takes it, in windows of 64 slots
// dealt to its four waves in turn: a wave adds its window's records to the sum
// that it finds in LDS, leaves the sum there for the next wave, and requests
// its next window's records, which have the three other waves' turns to
// arrive.  The order of the additions, and so the result, is that of one half.
// These ids (listed by the scan of the block counts) come first.
// 1 M Gaussians, 1200 x 680, 15.3 M slots of which 2.56 M are written (0.33 GB,
// 64 us at the rate of a large copy): 201 -> 115 us; 300k at 640 x 480, 0.68 M
// written: 36 -> 29; eight views of 640 x 480, 25 slots to an id (1.0 GB,
// 200 us, which the records' lines bound): 260 -> 257.  The line at 512: 256
// gives 139 and 26 us for the first two, 1024 gives 118 and 32.  (Adding an
// eighth of the range per half and then the eight sums is as fast, but another
// order of the additions moves gradients with much cancellation by 1e-3.)
constexpr int kSegBatch = 8;
constexpr int kSegWaves = 4;
__global__ void __launch_bounds__(256, 8) k_seg_reduce(Groups gr, const uint32_t* __restrict__ slot_off,
                                                    const float* __restrict__ partials,
                                                    uint8_t* __restrict__ mask,
                                                    const uint32_t* __restrict__ long_ids,
                                                    const Counters* __restrict__ cnt,
                                                    float* __restrict__ grad2d, int64_t stride) {
  partials += blockIdx.y * gr.slots * kSlotFloats;
  mask += blockIdx.y * gr.mask_stride;
  grad2d += blockIdx.y * stride;
  __shared__ float sum[32];
  const int lane = threadIdx.x & 63;
  if (cnt->overflow) return;
  const uint32_t nv = cnt->n_visible, ns = cnt->n_slots;
  const uint32_t n_waves = (gridDim.x * blockDim.x) >> 6;
  const uint32_t w0 = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint32_t half = (uint32_t)lane >> 5, hl = (uint32_t)lane & 31u;
  // The slot range of the pair two ahead and the first mask byte of the
  // next pair are requested before the current pair is summed, so a pair
  // waits on one memory round trip (its records) instead of three (range,
  // mask, records).  The requests are unconditional, at clamped indices, and
  // their words are combined only when the pair comes up, so nothing waits
  // on them early.
  if (nv == 0u) return;
  const uint32_t n_long = cnt->n_long;
  for (uint32_t e = blockIdx.x; e < n_long; e += gridDim.x) {
    const uint32_t c = long_ids[e];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t beg = slot_off[c], end = c + 1u < nv ? slot_off[c + 1u] : ns;
    const uint32_t n_win = (end - beg + 63u) / 64u;
    auto byte_of = [&](uint32_t win) { return mask[min(beg + 64u * win + (uint32_t)lane, end - 1u)]; };
    // record 2 j of the window in the lower half of t[j], 2 j + 1 in the upper
    constexpr int kPairs = 32;
    float t[kPairs];
    uint32_t n_rec = 0u;
    auto request = [&](uint32_t win, uint32_t m) {
      const uint32_t sl = beg + 64u * win + (uint32_t)lane;
      const bool written = sl < end && m != 0u;
      if (written) mask[sl] = 0;   // cleared for the next backward over these slots
      uint64_t left = __builtin_amdgcn_ballot_w64(written);
      n_rec = (uint32_t)__builtin_popcountll(left);
      const float* rec = partials + (size_t)(beg + 64u * win) * kSlotFloats + hl;
#pragma unroll
      for (int q = 0; q < kPairs; q += 8)
        if (n_rec > 2u * q) {
#pragma unroll
          for (int j = q; j < q + 8; ++j) {
            // past the last record: the window's first slot, dropped below
            const uint32_t i0 = left ? (uint32_t)__builtin_ctzll(left) : 0u;
            left &= left - 1ull;
            const uint32_t i1 = left ? (uint32_t)__builtin_ctzll(left) : 0u;
            left &= left - 1ull;
            t[j] = rec[(half ? i1 : i0) * kSlotFloats];
          }
        }
    };
    uint32_t m = byte_of(wave);
    const uint32_t m1 = byte_of(wave + kSegWaves);
    request(wave, m);
    m = m1;
    for (uint32_t win = 0; win < n_win; ++win) {
      if (win % kSegWaves == wave) {
        float acc = win ? sum[hl] : 0.f;
#pragma unroll
        for (int q = 0; q < kPairs; q += 8)
          if (n_rec > 2u * q) {
#pragma unroll
            for (int j = q; j < q + 8; ++j) {
              // (the upper half's value in the lower half; the upper half's own sum is not used)
              const uint32_t x = __float_as_uint(t[j]);
              const float up = __uint_as_float(__builtin_amdgcn_permlane32_swap(x, x, false, false)[1]);
              acc += 2u * j < n_rec ? t[j] : 0.f;
              acc += 2u * j + 1u < n_rec ? up : 0.f;
            }
          }
        if (half == 0u) sum[hl] = acc;
        if (win + 1u == n_win && lane < kPartials) grad2d[(size_t)c * kPartials + lane] = acc;
      }
      // the sum has to be there, the requested records not: no wait for them
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (win % kSegWaves == wave) {
        request(win + kSegWaves, m);
        m = byte_of(win + 2 * kSegWaves);
      }
    }
  }
  const uint32_t step = 2 * n_waves;
  auto req = [&](uint32_t cc, uint32_t& b, uint32_t& e) {   // raw words of pair member cc
    const uint32_t ci = min(cc, nv - 1u);
    b = slot_off[ci];
    e = slot_off[min(ci + 1u, nv - 1u)];
  };
  auto range = [&](uint32_t cc, uint32_t braw, uint32_t eraw, uint32_t& b, uint32_t& l) {
    const bool valid = cc < nv;
    b = valid ? braw : 0u;
    l = valid ? (cc + 1u < nv ? eraw : ns) - braw : 0u;
  };
  auto req_mask = [&](uint32_t b, uint32_t l) {   // the byte of this lane's first slot (or slot 0)
    return mask[l > 0u ? b + min(hl, l - 1u) : 0u];
  };
  uint32_t rb0, re0, rb1, re1;
  req(2 * w0 + half, rb0, re0);
  req(2 * w0 + step + half, rb1, re1);
  uint32_t b0, l0;
  range(2 * w0 + half, rb0, re0, b0, l0);
  uint32_t mraw0 = req_mask(b0, l0);
  for (uint32_t c0 = 2 * w0; c0 < nv; c0 += step) {
    const uint32_t c = c0 + half;
    uint32_t rb2, re2;
    req(c0 + 2 * step + half, rb2, re2);
    uint32_t b1, l1;
    range(c0 + step + half, rb1, re1, b1, l1);
    const uint32_t mraw1 = req_mask(b1, l1);
    // the requests above stay ahead of the summing below (no memory operation
    // moves across this point)
    asm volatile("" ::: "memory");
    const bool done = l0 > kLongSlots;   // (summed above)
    const uint32_t base = b0, len = done ? 0u : l0;
    const uint32_t maxlen = __builtin_amdgcn_readfirstlane(max(len, (uint32_t)__shfl_xor((int)len, 32, 64)));
    // the slot a lane with nothing to add reads: the half's last one read
    // (already in cache), slot 0 before the first (read by every wave)
    uint32_t last = 0u;
    float acc = 0.f;
    uint32_t mraw = mraw0;
    for (uint32_t o = 0; o < maxlen; o += 32) {
      const uint32_t sl = base + o + hl;
      // the first window's bytes were requested a pair ago, the others' a
      // window ago
      const bool written = o + hl < len && mraw != 0u;
      mraw = mask[len > 0u ? base + min(o + 32u + hl, len - 1u) : 0u];   // the next window's
      asm volatile("" ::: "memory");
      if (written) mask[sl] = 0;   // cleared for the next backward over these slots
      const uint64_t bal = __builtin_amdgcn_ballot_w64(written);
      const uint32_t lo = (uint32_t)bal, hi = (uint32_t)(bal >> 32);
      uint32_t mine = half ? hi : lo;
      const uint32_t nmax = max((uint32_t)__builtin_popcount(lo), (uint32_t)__builtin_popcount(hi));
      const uint32_t sb = base + o;
      auto batch = [&](auto nb_tag) {
        constexpr int NB = decltype(nb_tag)::value;
        float t[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          // the lowest written slot left (once none is, the last slot read,
          // whose value is dropped)
          const bool v = mine != 0u;
          last = v ? sb + (uint32_t)__builtin_ctz(mine) : last;
          mine &= mine - 1u;
          const float x = partials[(size_t)last * kSlotFloats + hl];
          t[j] = v ? x : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) acc += t[j];
      };
      // long runs (a view where a Gaussian covers many blocks) in batches of
      // 2 kSegBatch, the rest in batches of kSegBatch
      uint32_t k = 0;
      for (; k + 2 * kSegBatch <= nmax; k += 2 * kSegBatch) batch(std::integral_constant<int, 2 * kSegBatch>());
      for (; k < nmax; k += kSegBatch) batch(std::integral_constant<int, kSegBatch>());
    }
    if (c < nv && !done && hl < (uint32_t)kPartials) grad2d[(size_t)c * kPartials + hl] = acc;
    b0 = b1;
    l0 = l1;
    mraw0 = mraw1;
    rb1 = rb2;
    re1 = re2;
  }
}

// Waves of a compositing work-group: settings.chunk, at most the four that the
// kernels are compiled for (256 threads).  The waves take blocks from the queues
// one by one, so the results and the blocks do not depend on it.
constexpr int kMaxWaves = 4;
int group_threads(int chunk) { return 64 * std::min(chunk, kMaxWaves); }

}  // namespace

template <bool BF16, bool CNT, bool NC>
static void launch_fwd_t(const Settings& st, const Groups& gr, const ViewDesc* views, const ViewImages* out, const uint2* ranges,
                         const uint32_t* vals, const GeomRec* geom, const void* app, uint32_t npad_mask,
                         const uint32_t* items, const uint32_t* qoff, int64_t n_items, Counters* cnt,
                         uint32_t* work_q, int chunk, int32_t* last_idx, float* T_state, hipStream_t s) {
  const int threads = group_threads(chunk), waves = threads / 64;
  const size_t lds = BF16 ? (size_t)waves * kFwdWaveLds : 0;
  static Residency known;
  int64_t grid = resident_groups(known, k_raster_fwd<BF16, CNT, NC>, threads, lds);
  const int64_t need = (n_items + waves - 1) / waves;
  if (grid > need) grid = need;
  if (grid < kQueues) grid = kQueues;   // every queue needs a workgroup (index mod kQueues) to drain it
  hipLaunchKernelGGL((k_raster_fwd<BF16, CNT, NC>), dim3((unsigned)grid, gr.count), dim3(threads), lds, s, st, gr, views, out,
                     ranges, vals, geom, app, npad_mask, items, qoff, (uint32_t)n_items, cnt, work_q, last_idx,
                     T_state);
}

void launch_raster_fwd(const Settings& st, const Groups& gr, const ViewDesc* views, const ViewImages* out, const uint2* ranges,
                       const uint32_t* vals, const GeomRec* geom, const void* app, int app_bf16,
                       uint32_t npad_mask, const uint32_t* items, const uint32_t* qoff, int64_t n_items,
                       Counters* cnt, uint32_t* work_q, int chunk, int32_t* last_idx, float* T_state, int n_contrib,
                       hipStream_t s) {
  if (n_items <= 0) return;
#define LGS_FWD(B, K, N)                                                                                     \
  launch_fwd_t<B, K, N>(st, gr, views, out, ranges, vals, geom, app, npad_mask, items, qoff, n_items, cnt,   \
                        work_q, chunk, last_idx, T_state, s)
#define LGS_FWD_N(B, K)        \
  if (n_contrib) LGS_FWD(B, K, true); \
  else LGS_FWD(B, K, false)
  if (app_bf16) {
    if (st.count) LGS_FWD_N(true, true);
    else LGS_FWD_N(true, false);
  } else {
    if (st.count) LGS_FWD_N(false, true);
    else LGS_FWD_N(false, false);
  }
#undef LGS_FWD_N
#undef LGS_FWD
}

template <bool BF16, int UPM, bool CNT>
static void launch_bwd_t(const Settings& st, const Groups& gr, const ViewDesc* views, const ViewImages* upstream,
                         const ViewImages* fwd_out, const ViewImages* targets, const float* loss_w,
                         const uint2* ranges, const uint32_t* vals, const GeomRec* geom, const void* app,
                         uint32_t npad_mask, const uint32_t* items, const uint32_t* qoff, int64_t n_items,
                         Counters* cnt, uint32_t* work_q, int chunk, const int32_t* last_idx, const float* T_state,
                         const uint32_t* slot_base, float* partials, uint8_t* mask, hipStream_t s) {
  const int threads = group_threads(chunk), waves = threads / 64;
  const size_t lds = kBasisBytes + (size_t)waves * bwd_wave_lds(UPM);
  static Residency known;
  int64_t grid = resident_groups(known, k_raster_bwd<BF16, UPM, CNT>, threads, lds);
  const int64_t need = (n_items + waves - 1) / waves;
  if (grid > need) grid = need;
  if (grid < kQueues) grid = kQueues;   // every queue needs a workgroup (index mod kQueues) to drain it
  hipLaunchKernelGGL((k_raster_bwd<BF16, UPM, CNT>), dim3((unsigned)grid, gr.count), dim3(threads), lds, s, st, gr, views,
                     upstream, fwd_out, targets, loss_w, ranges, vals, geom, app, npad_mask, items, qoff,
                     (uint32_t)n_items, cnt, work_q, last_idx, T_state, slot_base, partials, mask);
}

void launch_raster_bwd(int up_mode, const Settings& st, const Groups& gr, const ViewDesc* views, const ViewImages* upstream,
                       const ViewImages* fwd_out, const ViewImages* targets, const float* loss_w,
                       const uint2* ranges, const uint32_t* vals, const GeomRec* geom, const void* app,
                       int app_bf16, uint32_t npad_mask, const uint32_t* items, const uint32_t* qoff,
                       int64_t n_items, Counters* cnt, uint32_t* work_q, int chunk, const int32_t* last_idx,
                       const float* T_state, const uint32_t* slot_base, float* partials, uint8_t* mask,
                       hipStream_t s) {
  if (n_items <= 0) return;
#define LGS_BWD(B, M)                                                                                     \
  (st.count ? launch_bwd_t<B, M, true>(st, gr, views, upstream, fwd_out, targets, loss_w, ranges, vals, geom, app,  \
                                       npad_mask, items, qoff, n_items, cnt, work_q, chunk, last_idx,      \
                                       T_state, slot_base, partials, mask, s)                                 \
            : launch_bwd_t<B, M, false>(st, gr, views, upstream, fwd_out, targets, loss_w, ranges, vals, geom,  \
                                        app, npad_mask, items, qoff, n_items, cnt, work_q, chunk, last_idx, \
                                        T_state, slot_base, partials, mask, s))
  if (app_bf16) {
    if (up_mode == UP_L1) LGS_BWD(true, UP_L1);
    else if (up_mode == UP_RGB) LGS_BWD(true, UP_RGB);
    else LGS_BWD(true, UP_EXPLICIT);
  } else {
    if (up_mode == UP_L1) LGS_BWD(false, UP_L1);
    else if (up_mode == UP_RGB) LGS_BWD(false, UP_RGB);
    else LGS_BWD(false, UP_EXPLICIT);
  }
#undef LGS_BWD
}

void launch_seg_reduce(const Groups& gr, const uint32_t* slot_off, const float* partials, uint8_t* mask,
                       const uint32_t* long_ids, const Counters* cnt, int64_t n_max, float* grad2d, int64_t stride,
                       hipStream_t s) {
  if (n_max <= 0) return;
  static Residency known;
  int64_t grid = resident_groups(known, k_seg_reduce, 256, 0);
  const int64_t need = (n_max + 7) / 8;   // two visible ids per wave
  if (grid > need) grid = need;
  hipLaunchKernelGGL(k_seg_reduce, dim3((unsigned)grid, gr.count), dim3(256), 0, s, gr, slot_off, partials, mask, long_ids, cnt,
                     grad2d, stride);
}

}  // namespace lgs
