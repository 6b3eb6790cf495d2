// Internal declarations shared by the HIP translation units of the
// rasterizer: device-side records, per-view descriptors, launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <atomic>

namespace lgs {

// Pixel blocks are 8x8: one wave64 renders one block, one pixel per lane.
constexpr int kBlock = 8;
constexpr int kMaxSide = 2048;          // 8-bit block coordinates in records
constexpr int kChannels = 20;           // RGB 3 + depth 1 + feature 16
constexpr int kPartials = 26;           // y 20, then the geometric sums Sp, Sy, Spp, S0, Spy, Syy (frame_shear)
constexpr int kPartGeo = 20;            // the first of the geometric sums
constexpr uint32_t kLongSlots = 512;   // a longer slot range is summed by a whole work-group
constexpr int kSlotFloats = 32;         // a backward slot record: the kPartials floats padded to 128 bytes

// Per-view constants, shared by every stage (device array of n_views).
struct ViewDesc {
  double fx, fy, cx, cy;
  double R[9], t[3];
  double limx, limy;          // Jacobian clamp limits on x/z, y/z
  int32_t W, H;
  int32_t blocks_x, blocks_y; // 8x8 blocks
  int32_t tiles_x, tiles_y;   // binning tiles
  int32_t tile_off;           // first global tile id of this view
  int32_t item_off;           // first work item (8x8 block) of this view
  int32_t pix_off;            // first pixel of this view in packed state
  int32_t pad;
};

// Output / upstream image pointers of one view.
struct ViewImages {
  float *rgb, *depth, *feat, *T;
  int32_t *n_contrib;
};

// One view of the mapping loss (rendered and observed images, gradient
// planes, FP32 [C][H][W]) and its scale factors:
//   s_l1 = w_rgb (1 - lam) / (3HW), s_ssim = w_rgb lam / (3HW),
//   s_d = w_depth / (HW), s_f = w_feat / (D HW).
// Colour work-groups of the view: [blk_off, blk_off + n_blk), three per
// 32 x 32 tile (one per channel); depth + feature work-groups: [df_off,
// df_off + n_df), one per run of kLossDfPixels pixels; vec4: the depth and
// feature planes allow 16-byte accesses.
struct LossView {
  const float *x, *xt, *d, *dt, *f, *ft;
  float *gx, *gd, *gf;
  int32_t W, H, tiles_x, blk_off, n_blk, df_off, n_df, vec4, nf, pad;   // nf: feature planes D
  float s_l1, s_ssim, s_d, s_f;
};
constexpr int kLossDfPixels = 2048;
constexpr int kSsimRadius = 5;   // 11 x 11 SSIM window
struct LossConsts {
  float w[2 * kSsimRadius + 1];  // normalised 1-D window weights
  float c1, c2;
  int32_t ssim;                  // 0: lam = 0, the SSIM stencil is skipped
  int32_t n_views;
};

// Screen-space record of one visible (view, Gaussian), 32 bytes, read by the
// compositing kernels through scalar loads (wave-uniform).
//   mx, my : mean' relative to the pixel origin (8 bx0, 8 by0) of its bbox
//   qa, qb2, qc : conic (Q_xx, 2 Q_xy, Q_yy)
//   o      : opacity
//   z      : camera depth (the depth channel value)
//   bbox   : block rectangle bx0 | bx1 << 8 | by0 << 16 | by1 << 24 (inclusive)
struct __attribute__((aligned(32))) GeomRec {
  float mx, my, qa, qb2, qc, o, z;
  uint32_t bbox;
};

// The geometric sums are kept in FP32 in the Gaussian's own frame: of p = dx +
// k dy, y = dy, k = Q_xy / Q_xx, in which the conic has no mixed term.  The
// gradient of a thin Gaussian is what its short axis leaves of them, and in the
// image's axes that is a difference of sums as much larger as the square of the
// axes' ratio, each rounded on its own (up to 22 px long and 0.6 across, alone
// on their pixels: 1e-6 to 4e-6 of the gradients' norm, here at most 3.7e-7;
// rotations in rooms of near Gaussians: a quarter less).  The writer of the sums has the conic's
// FP32 words from the record, their reader rounds its own FP64 conic: a k that
// differs in its last bit costs what one of the sums' roundings would in the
// image's axes.  (A gather of the records cost the reader 16 of 67 us on eight
// views of 500k.)  A conic so flat that k is past FP64's reach keeps the axes.
__device__ __forceinline__ float frame_shear(float qa, float qb2) {
  const float k = 0.5f * qb2 * __builtin_amdgcn_rcpf(qa);
  return fabsf(k) < 65536.f ? k : 0.f;
}

// The language features of dimension D are processed in groups of 16
// channels (the last group of D = 8 has 8): the compositing kernels carry
// RGB + depth + one group; further groups re-run them with that group's
// appearance records (blend weights do not depend on the features).
constexpr int kFeatGroup = 16;
struct Settings {
  float z_near, eps2d, fov_clamp, alpha_max, alpha_min, T_eps, cutoff2;
  int32_t tile, tile_shift;   // tile side and log2(tile / 8)
  int32_t feat_dim;           // D: feature planes of the inputs
  int32_t nfeat;              // feature channels of the group being processed (8 or 16)
  int32_t count;              // 1: the compositing kernels' profiling variants, which count their work
  float log2_alpha_min;       // log2(alpha_min), for the compositing kernels' block cull
};

// Device-resident counters of one forward (written by kernels, read by
// kernels; the host reads n_pairs in eager mode).
// Work items of the compositing kernels are split into kQueues queues, one
// per XCD (the GPU dispatches workgroup i to XCD i mod 8): all blocks of a
// binning tile go to the same queue, so the tile's list is fetched into one
// XCD's L2 and reused there by the blocks that walk it.
#ifndef LGS_XCD_QUEUES
#define LGS_XCD_QUEUES 1
#endif
constexpr int kQueues = 8;

constexpr int kLineWords = 32;   // one 128-byte line per queue counter

// Work-groups of a kernel that the current device holds at once: asked of the
// runtime once per device and work-group size (one slot of the kernel's own
// table each; the answer never changes).
struct Residency {
  static constexpr int kDevices = 16, kSizes = 5;   // 64 << size threads
  std::atomic<int> groups[kDevices][kSizes] = {};
};
template <class F>
int64_t resident_groups(Residency& known, F kernel, int threads, size_t lds) {
  int dev = 0, size = 0;
  (void)hipGetDevice(&dev);
  while ((64 << size) < threads) ++size;
  const bool keep = dev >= 0 && dev < Residency::kDevices && size < Residency::kSizes && (64 << size) == threads;
  if (keep)
    if (const int n = known.groups[dev][size].load(std::memory_order_relaxed)) return n;
  int cus = 256, occ = 1;
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, threads, lds);
  const int n = cus * (occ > 0 ? occ : 1);
  if (keep) known.groups[dev][size].store(n, std::memory_order_relaxed);
  return n;
}

struct __attribute__((aligned(128))) Counters {
  uint32_t n_visible;   // M
  uint32_t n_pairs;     // P
  uint32_t n_slots;     // S
  uint32_t overflow;    // set when P exceeds the pair capacity
  uint32_t n_pairs_eff; // n_pairs, or 0 after an overflow
  uint32_t n_long;      // visible ids with more than kLongSlots slots
  uint32_t pad1[2];
  // work actually done by the compositing kernels (one atomic per wave):
  // (pixel, entry) evaluations and contributions, the list entries a wave
  // visited (its records were loaded), forward and backward, and the
  // backward's partial records written
  unsigned long long fwd_evals, fwd_contrib, fwd_entries;
  unsigned long long bwd_evals, bwd_contrib, bwd_entries, bwd_written;
  uint32_t pad2[10];
};
static_assert(sizeof(Counters) % 128 == 0, "whole lines");

// Work counters of one feature group's compositing, queue q at word
// q * kLineWords, each on its own line so that the queues' atomics do not
// serialise on one address
constexpr int kQueueWords = kQueues * kLineWords;

// Queue of the items of binning tile t (global tile index) in the raster
// and list-length orders (settings.order 0 and 1): neighbouring tiles go to
// different XCDs.
__host__ __device__ inline uint32_t tile_queue(uint32_t t) { return LGS_XCD_QUEUES ? (t % kQueues) : 0u; }
// Spatial order (settings.order 2): the views are cut into super-tiles of
// kSuperPx x kSuperPx pixels and each super-tile goes to one queue (a
// lattice over (super-tile x, y, view), so that neighbouring super-tiles go
// to different XCDs); inside a queue items run in descending tile-list
// length as in order 1.  The tiles of one region then share their XCD's L2
// for the records of the Gaussians they have in common.
constexpr int kSuperPx = 128;
__host__ __device__ inline uint32_t super_queue(uint32_t v, uint32_t bx, uint32_t by) {
  constexpr uint32_t sh = 4;   // log2(kSuperPx / 8): 8x8 blocks per super-tile side
  static_assert((8u << sh) == (uint32_t)kSuperPx, "super-tile side");
  return LGS_XCD_QUEUES ? (((bx >> sh) + 3u * (by >> sh) + 5u * v) % (uint32_t)kQueues) : 0u;
}

// ---------------------------------------------------------------------------
// launchers (each defined next to its kernels)
// ---------------------------------------------------------------------------
// projection (K1)
void launch_project(const Settings& st, const ViewDesc* views, int n_views,
                    const float* means, const float* log_scales, const float* quats,
                    const float* logits, const void* rgb, const void* feat, int app_bf16,
                    int64_t n, uint32_t npad_shift,
                    GeomRec* geom, uint32_t* cnt_t, uint32_t* cnt_b, uint32_t* dkey,
                    void* app, Counters* cnt, hipStream_t s);   // also zeroes *cnt (the step's first kernel)

// scans
size_t scan_temp_bytes(int64_t n);
enum ScanInput { SCAN_FLAG_NONZERO = 0, SCAN_VALUE = 1, SCAN_GATHER = 2 };
// out[i] = exclusive prefix of in(i); total written to *total.
// in(i) = (src[i] != 0) / src[i] / src[idx[i]] by mode.
// Compaction (flag scans only, ent == nullptr for none): for every flagged item i, with c = out[i]: ent[c] =
// ent_copy[c] = i and keys[c] = key_src[i].
struct Compact {
  const uint32_t* key_src = nullptr;
  uint32_t* ent = nullptr;
  uint32_t* ent_copy = nullptr;
  uint32_t* keys = nullptr;
  // value and gather scans: the items i whose value exceeds big_min, in any order
  uint32_t* big = nullptr;
  uint32_t* n_big = nullptr;   // their number (added to)
  uint32_t big_min = 0;
};
void launch_scan(int mode, const uint32_t* src, uint32_t* out, uint32_t* total, int64_t n, void* temp, hipStream_t s,
                 Compact cp = Compact());
// Two gather scans of the same count (*n_dev, at most n_max).  out_at_idx (or
// NULL): each value also written at its source index, out_at_idx[idx[i]] =
// out[i].  out also holds the gathered values between the two passes, so it
// must not overlap src or idx.
struct GatherScan {
  const uint32_t *src, *idx;
  uint32_t *out, *total, *out_at_idx;
  Compact cp;
};
void launch_gather_scans(const GatherScan& a, const GatherScan& b, const uint32_t* n_dev, int64_t n_max, void* temp,
                         hipStream_t s);

// pair emission (load-balanced over pairs), tile ranges
// (also sets the step's overflow flag and effective counts and zeroes
// zero[0 .. n_zero))
void launch_emit(const GeomRec* geom, const ViewDesc* views, const uint32_t* srid,
                 const uint32_t* off_t, Counters* cnt, int64_t cap_pairs, int64_t cap_slots, int npad_shift,
                 int tile_shift, uint32_t* keys, uint32_t* vals, uint32_t* zero, int64_t n_zero, hipStream_t s);
void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s);
// ranges of words zeroed by one launch
struct ZeroRanges {
  static constexpr int kMax = 4;
  uint32_t* p[kMax] = {nullptr, nullptr, nullptr, nullptr};
  int64_t n[kMax] = {0, 0, 0, 0};
};
void launch_zero(const ZeroRanges& r, hipStream_t s);
void launch_tile_ranges(const uint32_t* keys, const Counters* cnt, int64_t grid_max,
                        uint2* ranges, hipStream_t s);
// Stable LSD radix sort.  n_max bounds the count (read from *n_dev when
// n_dev != nullptr); up to small_max it is sorted with the fewest launches.  That
// form is the fastest for up to some 300k keys and as fast as the next one at
// 2^19 (71 and 70 us), so ids, of which only the visible ones are sorted, take it
// up to a bound of 2^19; pairs, whose bound is the count or a capacity near it,
// up to 2^17 (200k pairs of 14 bits: 26 us, in the next form 22).
constexpr int64_t kSmallPairs = 1ll << 17, kSmallIds = 1ll << 19;
size_t radix_temp_bytes(int64_t n_max, int64_t small_max);
void radix_sort_u32(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                    const uint32_t* n_dev, int64_t n_max, int64_t small_max, int begin_bit, int end_bit,
                    void* temp, hipStream_t s, bool* result_in_alt);

// The lists between projection and pair emission, of n_rid <= kSmallFront
// (view, Gaussian) ids, by one work-group: what the flag scan with compaction,
// the depth sort and the two gather scans give, with the same contents.
constexpr int64_t kSmallFront = 4096;
struct FrontLists {
  const uint32_t *cnt_t, *cnt_b, *dkey;             // [n_rid]
  uint32_t *cidx, *ent;                             // prefix of the visibility flags; visible ids, index order
  uint32_t *srid, *off_t;                           // visible ids, depth order; their pair offsets
  uint32_t *slot_off, *slot_base;                   // slot offsets, visible order and by id
  uint32_t* long_ids;                               // visible ids (their place) with more than kLongSlots slots
};
void launch_small_front(const FrontLists& f, int64_t n_rid, Counters* cnt, hipStream_t s);

// work queue ordering (blocks by descending tile-list length): each queue's
// tiles re-sorted by the length of their list (counting sort on coarse
// length buckets, one work-group per queue), a tile's blocks kept together;
// qoff: the queues' item offsets, tiles: the queue-major tile table, tq: its
// queues' tile offsets (kQueues + 1); returns out
struct TileItems {
  uint32_t first;   // index of the tile's first item in the static table
  uint32_t count;   // its blocks (items)
  uint32_t tile;    // global tile id
  uint32_t queue;
};
uint32_t* launch_order_items(const uint2* ranges, const uint32_t* items, const uint32_t* qoff, const TileItems* tiles,
                             const uint32_t* tq, int64_t n_tiles, uint32_t* out, hipStream_t s);

// compositing
// Feature groups in one launch (blockIdx.y = j): group (first + j) mod total;
// its image tables start n_views after the group's before it, its appearance
// app_stride bytes, its work counters kQueueWords words; the backward's partial
// records and marks of j start j * slots records and mask_stride bytes in.
struct Groups {
  int32_t first = 0, count = 1, total = 1, n_views = 0;
  int64_t app_stride = 0, slots = 0, mask_stride = 0;
};
void launch_raster_fwd(const Settings& st, const Groups& gr, const ViewDesc* views, const ViewImages* out,
                       const uint2* ranges, const uint32_t* vals, const GeomRec* geom,
                       const void* app, int app_bf16, uint32_t npad_mask,
                       const uint32_t* items, const uint32_t* qoff, int64_t n_items, Counters* cnt,
                       uint32_t* work_q, int chunk, int32_t* last_idx, float* T_state, int n_contrib,
                       hipStream_t s);   // n_contrib: some view's out table asks for contributor counts
// Upstream of the backward compositing kernel: dL/dY given per channel
// (upstream), the L1 loss gradient formed from the forward's images and the
// targets (loss_w), or the colour channels given and depth + features from
// the L1 residual (the D-SSIM loss, whose colour gradient a kernel writes).
enum UpMode { UP_EXPLICIT = 0, UP_L1 = 1, UP_RGB = 2 };
void launch_raster_bwd(int up_mode, const Settings& st, const Groups& gr, const ViewDesc* views, const ViewImages* upstream,
                       const ViewImages* fwd_out, const ViewImages* targets, const float* loss_w,
                       const uint2* ranges, const uint32_t* vals, const GeomRec* geom,
                       const void* app, int app_bf16, uint32_t npad_mask,
                       const uint32_t* items, const uint32_t* qoff, int64_t n_items, Counters* cnt, uint32_t* work_q,
                       int chunk, const int32_t* last_idx, const float* T_state,
                       const uint32_t* slot_base, float* partials, uint8_t* mask, hipStream_t s);

// mapping loss (L1 + D-SSIM) and its gradient: the colour channels (L1 and
// SSIM stencil), the depth and feature channels (L1), and the per-view terms
// {mean|I-I*|, 1 - SSIM (0 when ssim = 0), mean|D-D*|, mean|F-F*|} from the
// work-groups' partial sums
int64_t loss_blocks(int W, int H);
int64_t loss_df_blocks(int W, int H);
int loss_tiles_x(int W);
void launch_loss_rgb(const LossView* views, const LossConsts& k, int64_t n_blocks, float2* partials,
                     hipStream_t s);
// colour, depth and features in one launch
void launch_loss(const LossView* views, const LossConsts& k, int feat_dim, int64_t n_rgb, int64_t n_df,
                 float2* part_rgb, float2* part_df, hipStream_t s);
void launch_loss_terms(const LossView* views, int n_views, int ssim, const float2* part_rgb,
                       const float2* part_df, float* terms, hipStream_t s);

// feature decoder (1x1 convolution 16 -> C) and its L1 distillation loss
// over one or more views (each view's loss normalised by its own C H W, the
// views' losses summed): dL/dF per view, dL/dW, dL/db and the loss.  Every
// work-group works on one view's chunks; part holds grid x part_stride
// floats of per-work-group partial sums (dW [C][16], db [C], loss), already
// times the view's scale
constexpr int kDecMaxViews = 16;
struct DecView {
  const float* feat;                   // F [16][n]
  const void* target;                  // F* [C][n], BF16 or FP32
  float* grad_feat;                    // dL/dF [16][n]
  int64_t n;                           // pixels
  float scale;                         // w_feat / (C n)
  int32_t g0, groups;                  // its work-groups g0 .. g0 + groups - 1 (decoder_assign)
};
struct DecArgs {
  const float *weight, *bias;          // W [C][16], b [C]
  float *grad_weight, *grad_bias, *loss;
  int64_t part_stride;                 // >= 17 C + 1
  int32_t C;                           // 256 or 512
  int32_t n_views;                     // 1 .. kDecMaxViews
  DecView v[kDecMaxViews];
};
bool decoder_dim_ok(int C);
// shares out the work-groups of the launch among the views (at most one per
// CU and at most `cap` in all, unless there are more views; at least one per
// view, at most one per 32-pixel chunk) and returns the grid
int decoder_assign(DecArgs& a, int cap);
void launch_decoder(const DecArgs& a, int target_bf16, float* part, int grid, hipStream_t s);

// language-guided pruning (K nearest neighbours in a uniform grid of cell
// side tau_dist) and the geometric criteria
struct PruneArgs {
  const float *means, *logits, *log_scales;   // [3][n], [n], [3][n]
  const void* feat;                           // [planes][n], FP32 or BF16
  int32_t feat_bf16, planes, k;               // planes: 8 or 16; k <= prune_k_max()
  uint32_t buckets;                           // prune_buckets(n)
  int64_t n;
  double tau2, inv_cell, tau_sim;             // tau_dist^2, 1 / tau_dist, tau_sim
  double logit_min, log_scale_max;            // log(o / (1 - o)) of min_opacity, log(max_scale)
  float tau2_above;                           // above any FP32 |p_i - p_j|^2 whose FP64 value is below tau2
};
struct PruneCounters {
  unsigned long long counts[3];   // redundant, geometric, pruned
  uint32_t n_heavy;               // Gaussians with more than k neighbours within tau_dist
  uint32_t range_err;             // a finite mean lies outside the grid's range
};
struct PruneWork {
  void* rec;                      // n x prune_rec_bytes
  float4* pos;                    // n
  uint32_t *count, *start;        // buckets, buckets + 1
  uint32_t* list;                 // n
  uint8_t *geo, *sem;             // n each
  void* temp;                     // scan_temp_bytes(buckets)
  PruneCounters* pc;
};
int prune_k_max();
size_t prune_rec_bytes(int bf16);
uint32_t prune_buckets(int64_t n);
// the whole pass (n > 0); leaves the mask alone when w.pc->range_err
void launch_prune(const PruneArgs& a, const PruneWork& w, uint8_t* mask, hipStream_t s);

// feature groups beyond the first (feat: the first group's planes): appearance
// records (RGB 0, the group's features), app_stride bytes from one to the next
void launch_pack_app_groups(const void* feat, int app_bf16, int64_t n, int n_groups, void* app, int64_t app_stride,
                            hipStream_t s);
// geo_acc[c][0 .. 5] (= | +=) the geometric sums of `count` groups' reductions,
// one after the other (stride floats apart)
void launch_group_geo_acc(const float* grad2d, int64_t stride, int count, const Counters* cnt, int64_t n_max,
                          float* geo_acc, int first, hipStream_t s);
// the feature gradients of those of the groups that are not the first
void launch_group_feat_grad(const Groups& gr, int64_t n, uint32_t npad_shift, const Counters* cnt,
                            const uint32_t* cnt_t, const uint32_t* cidx, const float* grad2d, int64_t stride,
                            float* g_feat, hipStream_t s);

// gradient reduction and projection backward
void launch_seg_reduce(const Groups& gr, const uint32_t* slot_off, const float* partials, uint8_t* mask,
                       const uint32_t* long_ids, const Counters* cnt, int64_t n_max, float* grad2d, int64_t stride,
                       hipStream_t s);
// Geometric sums of the feature groups besides the first, added to its own:
// those summed before (or NULL), then n reductions, stride floats apart.
struct GroupGeo {
  const float *acc = nullptr, *grad2d = nullptr;
  int64_t stride = 0;
  int32_t n = 0;
};
// workspace of launch_project_bwd for at most n_rid visible (view, Gaussian)
size_t project_bwd_temp_bytes(int64_t n_rid, int n_views);
// the projection backward: per visible (view, Gaussian) c the view's chain
// rule (ent: c's record id, in (view, Gaussian) order), then per Gaussian
// the views summed in order and the activation's chain rule
void launch_project_bwd(const Settings& st, const ViewDesc* views, int n_views, const float* means,
                        const float* log_scales, const float* quats, const float* logits, int64_t n,
                        uint32_t npad_shift, int64_t n_rid, const Counters* cnt, const uint32_t* cnt_t,
                        const uint32_t* cidx, const uint32_t* ent, const GroupGeo& geo, const float* grad2d, float* g_means,
                        float* g_ls, float* g_q, float* g_logit, float* g_rgb, float* g_feat, float* twist,
                        void* temp, hipStream_t s);

}  // namespace lgs
