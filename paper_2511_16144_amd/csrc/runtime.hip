// Host runtime behind the C ABI of include/lego_raster.h: argument checks,
// a caching device allocator per context, the launch sequences of the eager
// forward / backward, the captured whole-step hipGraph, and the autotuner.
#include "lgs_internal.h"
#include "../../include/lego_raster.h"

#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <cstddef>
#include <type_traits>
#include <vector>

using namespace lgs;

// ---------------------------------------------------------------------------
// context, allocator
// ---------------------------------------------------------------------------
// A cached device block and the event after which its last user's work on
// that user's stream is done (null: free now).  Blocks are handed out again
// in stream order: the new user's stream waits for the event on the device,
// the host never blocks.  Host staging kept for in-flight copies is freed the
// same way, once its event has completed.
using SharedEvent = std::shared_ptr<std::remove_pointer<hipEvent_t>::type>;
struct FreeBlock {
  void* p;
  SharedEvent ready;
};
struct DeferredHost {
  SharedEvent ready;
  std::deque<std::vector<char>> host;
};

struct lgs_context {
  int device = 0;
  std::string err;
  std::multimap<size_t, FreeBlock> free_blocks;   // size -> block (cached)
  std::map<void*, size_t> live;                    // ptr -> size
  std::vector<DeferredHost> deferred;              // host tables of released work, until their event
  // items tables per (views signature, tile) cached on the device
  std::map<std::string, std::pair<uint32_t*, int64_t>> items_cache;
  // lgs_loss workspace: view table (pinned staging + device copy, the copy
  // marked by an event so that the staging is rewritten only after it), and
  // the work-groups' partial sums
  LossView* loss_host = nullptr;
  LossView* loss_tab = nullptr;
  int loss_tab_cap = 0;
  float2* loss_part = nullptr;
  int64_t loss_part_cap = 0;
  hipEvent_t loss_copied = nullptr;
  // lgs_decoder_l1 workspace: per-work-group partial sums
  float* dec_part = nullptr;
  int64_t dec_part_cap = 0;
  // pinned staging of the readbacks: a step's counters, lgs_prune's
  lgs::Counters* counts_host = nullptr;
  lgs::PruneCounters* prune_host = nullptr;
  // device address of this GPU's copy of the fixed scratch array used by
  // lgs_decoder_l1_noalloc
  float* scratch = nullptr;
};

// Partial sums of lgs_decoder_l1_noalloc: a fixed device array instead of an
// allocation, sized for kScratchGroups work-groups of the widest decoder
// (C = 512: 17 C + 1 floats rounded up to 64, 8768 floats = 35 KB each),
// 8.98 MB in all.  Every GPU the library runs on holds its own copy until
// the process ends; host code reaches it only through the address that
// hipGetSymbolAddress returns for the current device (scratch_address).
constexpr int kScratchGroups = 256;
constexpr int64_t kScratchStride = ((17 * 512 + 1 + 63) / 64) * 64;
constexpr int64_t kScratchFloats = (int64_t)kScratchGroups * kScratchStride;
static __device__ __align__(256) float scratch[kScratchFloats];

namespace {

lgs_status fail(lgs_context* ctx, lgs_status s, const std::string& msg) {
  if (ctx) ctx->err = msg;
  return s;
}

#define HIP_TRY(ctx, expr)                                                              \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      return fail(ctx, LGS_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

SharedEvent make_event() {
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return SharedEvent();
  return SharedEvent(e, [](hipEvent_t x) { hipEventDestroy(x); });
}

// Drop the host staging whose copies have completed.
void sweep_deferred(lgs_context* ctx) {
  auto& d = ctx->deferred;
  d.erase(std::remove_if(d.begin(), d.end(),
                         [](const DeferredHost& x) { return !x.ready || hipEventQuery(x.ready.get()) == hipSuccess; }),
          d.end());
}

// hipMalloc that leaves no error behind when it fails (the caller tries
// something else, and a launch check after it would report the old error)
bool device_alloc(void** p, size_t bytes) {
  if (hipMalloc(p, bytes) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

// A device block of at least `bytes` for work enqueued on `stream`: a cached
// block (the stream first waits, on the device, for the block's previous
// user) or a new allocation.
void* pool_alloc(lgs_context* ctx, size_t bytes, hipStream_t stream) {
  bytes = ((bytes + 255) / 256) * 256;
  if (bytes == 0) bytes = 256;
  auto it = ctx->free_blocks.lower_bound(bytes);
  if (it != ctx->free_blocks.end() && it->first <= 2 * bytes + (64u << 20)) {
    void* p = it->second.p;
    if (it->second.ready && hipStreamWaitEvent(stream, it->second.ready.get(), 0) != hipSuccess)
      hipEventSynchronize(it->second.ready.get());
    ctx->live[p] = it->first;
    ctx->free_blocks.erase(it);
    return p;
  }
  // a new block between 4 and 17 MB takes hipMalloc 140 to 270 us, one of 17 MB
  // and more 30
  const size_t asked = bytes;
  if (bytes > (4u << 20) && bytes < (17u << 20)) bytes = 17u << 20;
  void* p = nullptr;
  if (!device_alloc(&p, bytes)) {
    // drop the cache and retry, at last with no more than was asked for
    for (auto& kv : ctx->free_blocks) {
      if (kv.second.ready) hipEventSynchronize(kv.second.ready.get());
      hipFree(kv.second.p);
    }
    ctx->free_blocks.clear();
    if (!device_alloc(&p, bytes) && (bytes == asked || !device_alloc(&p, bytes = asked))) return nullptr;
  }
  ctx->live[p] = bytes;
  return p;
}

// Return a block to the cache; `ready` (may be null) marks the end of the
// work that still uses it.
void pool_free(lgs_context* ctx, void* p, const SharedEvent& ready) {
  if (!p) return;
  auto it = ctx->live.find(p);
  if (it == ctx->live.end()) return;
  ctx->free_blocks.emplace(it->second, FreeBlock{p, ready});
  ctx->live.erase(it);
}

uint32_t ceil_log2(uint64_t x) {
  uint32_t b = 0;
  while ((1ull << b) < x) ++b;
  return b;
}

lgs_status check_settings(lgs_context* ctx, const lgs_settings* st) {
  if (!st) return fail(ctx, LGS_ERR_INVALID_ARG, "settings is NULL");
  if (st->tile != 8 && st->tile != 16 && st->tile != 32)
    return fail(ctx, LGS_ERR_INVALID_ARG, "tile must be 8, 16 or 32");
  if (st->chunk != 1 && st->chunk != 2 && st->chunk != 4 && st->chunk != 8)
    return fail(ctx, LGS_ERR_INVALID_ARG, "chunk must be 1, 2, 4 or 8");
  if (st->order < 0 || st->order > 2) return fail(ctx, LGS_ERR_INVALID_ARG, "order must be 0, 1 or 2");
  if (st->profile & ~(LGS_PROFILE_EVENTS | LGS_PROFILE_COUNTS))
    return fail(ctx, LGS_ERR_INVALID_ARG, "profile takes the bits LGS_PROFILE_EVENTS | LGS_PROFILE_COUNTS");
  if (!(st->z_near > 0.f) || !(st->eps2d >= 0.f) || !(st->fov_clamp > 0.f) ||
      !(st->alpha_max > 0.f && st->alpha_max < 1.f) || !(st->alpha_min > 0.f) ||
      !(st->T_eps > 0.f && st->T_eps < 1.f) || !(st->cutoff2 > 0.f))
    return fail(ctx, LGS_ERR_INVALID_ARG, "settings constants out of range");
  return LGS_OK;
}

bool aligned4(const void* p) { return ((uintptr_t)p & 3u) == 0; }

lgs_status check_gaussians(lgs_context* ctx, const lgs_gaussians* g) {
  if (!g) return fail(ctx, LGS_ERR_INVALID_ARG, "gaussians is NULL");
  if (g->n < 0) return fail(ctx, LGS_ERR_INVALID_ARG, "n < 0");
  if (g->n > (int64_t)1 << 30) return fail(ctx, LGS_ERR_UNSUPPORTED, "n > 2^30");
  if (g->appearance_dtype != LGS_F32 && g->appearance_dtype != LGS_BF16)
    return fail(ctx, LGS_ERR_INVALID_ARG, "unknown appearance dtype");
  if (!(g->feat_dim == 0 || g->feat_dim == 8 || (g->feat_dim % kFeatGroup == 0 && g->feat_dim >= 16 &&
                                                  g->feat_dim <= 128)))
    return fail(ctx, LGS_ERR_INVALID_ARG, "feat_dim must be 8 or a multiple of 16 up to 128 (0: 16)");
  if (g->n > 0) {
    const void* ps[6] = {g->means, g->log_scales, g->quats, g->opacity_logits, g->rgb, g->feat};
    for (int i = 0; i < 6; ++i) {
      if (!ps[i]) return fail(ctx, LGS_ERR_INVALID_ARG, "NULL Gaussian array");
      if (!aligned4(ps[i]) && !(i >= 4 && g->appearance_dtype == LGS_BF16 && ((uintptr_t)ps[i] & 1u) == 0))
        return fail(ctx, LGS_ERR_INVALID_ARG, "misaligned Gaussian array");
    }
  }
  return LGS_OK;
}

lgs_status check_cams(lgs_context* ctx, int32_t n_views, const lgs_camera* cams) {
  if (n_views < 1 || n_views > 1024) return fail(ctx, LGS_ERR_INVALID_ARG, "n_views must be in [1, 1024]");
  if (!cams) return fail(ctx, LGS_ERR_INVALID_ARG, "cams is NULL");
  for (int v = 0; v < n_views; ++v) {
    const lgs_camera& c = cams[v];
    if (c.width < 1 || c.height < 1 || c.width > kMaxSide || c.height > kMaxSide)
      return fail(ctx, LGS_ERR_INVALID_ARG, "image sides must be in [1, 2048]");
    if (!(c.fx > 0.f) || !(c.fy > 0.f) || !isfinite(c.cx) || !isfinite(c.cy))
      return fail(ctx, LGS_ERR_INVALID_ARG, "bad intrinsics");
    for (int k = 0; k < 9; ++k)
      if (!isfinite(c.R_cw[k])) return fail(ctx, LGS_ERR_INVALID_ARG, "non-finite pose");
    for (int k = 0; k < 3; ++k)
      if (!isfinite(c.t_cw[k])) return fail(ctx, LGS_ERR_INVALID_ARG, "non-finite pose");
  }
  return LGS_OK;
}

lgs_status check_images(lgs_context* ctx, int32_t n_views, const lgs_images* im, bool need_T,
                        const char* what) {
  if (!im) return fail(ctx, LGS_ERR_INVALID_ARG, std::string(what) + " is NULL");
  for (int v = 0; v < n_views; ++v) {
    if (!im[v].rgb || !im[v].depth || !im[v].feat || (need_T && !im[v].final_T))
      return fail(ctx, LGS_ERR_INVALID_ARG, std::string(what) + ": NULL image plane");
    if (!aligned4(im[v].rgb) || !aligned4(im[v].depth) || !aligned4(im[v].feat) ||
        (im[v].final_T && !aligned4(im[v].final_T)) || (im[v].n_contrib && !aligned4(im[v].n_contrib)))
      return fail(ctx, LGS_ERR_INVALID_ARG, std::string(what) + ": misaligned image plane");
  }
  return LGS_OK;
}

// Per-call geometry of the batch: view descriptors and work sizes.
struct Plan {
  std::vector<ViewDesc> views;
  int64_t n_tiles = 0, n_items = 0, n_pix = 0;
  int tile_shift = 1;
  std::string sig;
};

Plan make_plan(const lgs_settings* st, int32_t n_views, const lgs_camera* cams) {
  Plan P;
  P.tile_shift = st->tile == 8 ? 0 : (st->tile == 16 ? 1 : 2);
  char buf[128];
  snprintf(buf, sizeof buf, "t%d:", st->tile);
  P.sig = buf;
  for (int v = 0; v < n_views; ++v) {
    const lgs_camera& c = cams[v];
    ViewDesc d;
    memset(&d, 0, sizeof d);
    d.fx = c.fx; d.fy = c.fy; d.cx = c.cx; d.cy = c.cy;
    for (int k = 0; k < 9; ++k) d.R[k] = c.R_cw[k];
    for (int k = 0; k < 3; ++k) d.t[k] = c.t_cw[k];
    // view-angle clamp of the Jacobian (reading: fov_clamp x the half-extent
    // of the image seen from the principal point)
    d.limx = (double)st->fov_clamp * fmax((double)c.cx + 0.5, (double)c.width - 0.5 - (double)c.cx) / (double)c.fx;
    d.limy = (double)st->fov_clamp * fmax((double)c.cy + 0.5, (double)c.height - 0.5 - (double)c.cy) / (double)c.fy;
    d.W = c.width; d.H = c.height;
    d.blocks_x = (c.width + kBlock - 1) / kBlock;
    d.blocks_y = (c.height + kBlock - 1) / kBlock;
    d.tiles_x = (c.width + st->tile - 1) / st->tile;
    d.tiles_y = (c.height + st->tile - 1) / st->tile;
    d.tile_off = (int32_t)P.n_tiles;
    d.item_off = (int32_t)P.n_items;
    d.pix_off = (int32_t)P.n_pix;
    P.n_tiles += (int64_t)d.tiles_x * d.tiles_y;
    P.n_items += (int64_t)d.blocks_x * d.blocks_y;
    P.n_pix += (int64_t)c.width * c.height;
    P.views.push_back(d);
    snprintf(buf, sizeof buf, "%dx%d,", c.width, c.height);
    P.sig += buf;
  }
  return P;
}

// Work items (8x8 blocks) grouped by queue, tile by tile inside a queue,
// raster order inside a tile.  A tile's queue: tile_queue of its global
// index (orders 0 and 1) or super_queue of its region (order 2).  Layout of
// the table: the n_items items, the kQueues + 1 queue offsets, then one
// TileItems record per tile in the same order (its first item, block count,
// global tile id and queue), then the kQueues + 1 offsets of each queue's
// tiles among those records; from these k_order_items re-sorts each queue
// by list length, tile by tile (orders 1 and 2), keeping the queue sizes.
std::vector<uint32_t> make_items(const Plan& P, int tile, bool spatial) {
  std::vector<std::vector<uint32_t>> qs(kQueues);
  std::vector<std::vector<TileItems>> qt(kQueues);
  const int bpt = tile / kBlock;
  for (size_t v = 0; v < P.views.size(); ++v) {
    const ViewDesc& d = P.views[v];
    for (int ty = 0; ty < d.tiles_y; ++ty)
      for (int tx = 0; tx < d.tiles_x; ++tx) {
        const uint32_t t = (uint32_t)(d.tile_off + ty * d.tiles_x + tx);
        const uint32_t q = spatial ? super_queue((uint32_t)v, (uint32_t)(tx * bpt), (uint32_t)(ty * bpt))
                                   : tile_queue(t);
        TileItems ti{(uint32_t)qs[q].size(), 0u, t, q};
        for (int j = 0; j < bpt; ++j)
          for (int i = 0; i < bpt; ++i) {
            const int bx = tx * bpt + i, by = ty * bpt + j;
            if (bx < d.blocks_x && by < d.blocks_y) {
              qs[q].push_back((uint32_t)bx | ((uint32_t)by << 8) | ((uint32_t)v << 16));
              ++ti.count;
            }
          }
        qt[q].push_back(ti);
      }
  }
  // layout: the items queue by queue, the queues' item offsets (kQueues +
  // 1), the tile table queue by queue (4 words a tile), the queues' tile
  // offsets in it (kQueues + 1)
  std::vector<uint32_t> items;
  items.reserve(P.n_items + kQueues + 1 + 4 * P.n_tiles + kQueues + 1);
  std::vector<uint32_t> off(kQueues + 1, 0u);
  for (int q = 0; q < kQueues; ++q) {
    off[q] = (uint32_t)items.size();
    items.insert(items.end(), qs[q].begin(), qs[q].end());
  }
  off[kQueues] = (uint32_t)items.size();
  items.insert(items.end(), off.begin(), off.end());
  uint32_t nt = 0;
  for (int q = 0; q < kQueues; ++q)
    for (const TileItems& ti : qt[q]) {
      items.push_back(off[q] + ti.first);
      items.push_back(ti.count);
      items.push_back(ti.tile);
      items.push_back(ti.queue);
    }
  for (int q = 0; q < kQueues; ++q) {
    items.push_back(nt);
    nt += (uint32_t)qt[q].size();
  }
  items.push_back(nt);
  return items;
}

// the kernels' settings for features of D channels (a dimension above 16 is a
// multiple of 16: every group of channels is whole)
Settings dev_settings(const lgs_settings* st, int tile_shift, int D) {
  Settings s;
  s.z_near = st->z_near; s.eps2d = st->eps2d; s.fov_clamp = st->fov_clamp;
  s.alpha_max = st->alpha_max; s.alpha_min = st->alpha_min; s.T_eps = st->T_eps;
  s.cutoff2 = st->cutoff2; s.tile = st->tile; s.tile_shift = tile_shift;
  s.feat_dim = D;
  s.nfeat = std::min(D, kFeatGroup);
  s.count = (st->profile & LGS_PROFILE_COUNTS) != 0;
  s.log2_alpha_min = log2f(st->alpha_min);
  return s;
}

int feat_dim_of(const lgs_gaussians* g) { return g->feat_dim == 0 ? kFeatGroup : g->feat_dim; }

// Loss constants: the normalised 1-D SSIM window (sigma 1.5, computed in
// double, rounded once), C1 = 0.01^2, C2 = 0.03^2 (dynamic range 1).
LossConsts loss_consts(float ssim_lambda, int n_views) {
  LossConsts k;
  double w[2 * kSsimRadius + 1], sum = 0.0;
  for (int i = -kSsimRadius; i <= kSsimRadius; ++i) sum += (w[i + kSsimRadius] = exp(-(double)(i * i) / 4.5));
  for (int i = 0; i < 2 * kSsimRadius + 1; ++i) k.w[i] = (float)(w[i] / sum);
  k.c1 = 1e-4f;
  k.c2 = 9e-4f;
  k.ssim = ssim_lambda != 0.f;
  k.n_views = n_views;
  return k;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Loss view table; returns the number of colour work-groups and, in *n_df,
// the number of depth + feature work-groups (their partial sums follow the
// colour ones).
int64_t make_loss_views(int32_t n_views, const lgs_camera* cams, int feat_dim, const lgs_images* out,
                        const lgs_images* tgt, const lgs_images* grad, const float loss_w[3], float lam, LossView* dst,
                        int64_t* n_df) {
  int64_t nb = 0, nd = 0;
  for (int v = 0; v < n_views; ++v) {
    LossView L;
    memset(&L, 0, sizeof L);
    L.x = out[v].rgb; L.xt = tgt[v].rgb;
    L.d = out[v].depth; L.dt = tgt[v].depth;
    L.f = out[v].feat; L.ft = tgt[v].feat;
    L.gx = grad[v].rgb; L.gd = grad[v].depth; L.gf = grad[v].feat;
    L.W = cams[v].width; L.H = cams[v].height;
    L.tiles_x = loss_tiles_x(L.W);
    L.blk_off = (int32_t)nb;
    L.n_blk = (int32_t)loss_blocks(L.W, L.H);
    L.df_off = (int32_t)nd;
    L.n_df = (int32_t)loss_df_blocks(L.W, L.H);
    const int64_t hw = (int64_t)L.W * L.H;
    L.vec4 = hw % 4 == 0 && aligned16(L.d) && aligned16(L.dt) && aligned16(L.f) && aligned16(L.ft) &&
             aligned16(L.gd) && aligned16(L.gf);
    const double n = (double)L.W * (double)L.H;
    L.s_l1 = (float)((double)loss_w[0] * (1.0 - (double)lam) / (3.0 * n));
    L.s_ssim = (float)((double)loss_w[0] * (double)lam / (3.0 * n));
    L.s_d = (float)((double)loss_w[1] / n);
    L.s_f = (float)((double)loss_w[2] / ((double)feat_dim * n));
    L.nf = feat_dim;
    dst[v] = L;
    nb += L.n_blk;
    nd += L.n_df;
  }
  *n_df = nd;
  return nb;
}

lgs_status check_loss_args(lgs_context* ctx, const float loss_w[3], float lam) {
  if (!loss_w) return fail(ctx, LGS_ERR_INVALID_ARG, "loss_w is NULL");
  for (int i = 0; i < 3; ++i)
    if (!isfinite(loss_w[i])) return fail(ctx, LGS_ERR_INVALID_ARG, "non-finite loss weight");
  if (!(lam >= 0.f && lam <= 1.f)) return fail(ctx, LGS_ERR_INVALID_ARG, "ssim_lambda must be in [0, 1]");
  return LGS_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// device buffers of one forward(+backward): an eager state or a graph
// ---------------------------------------------------------------------------
struct Work {
  lgs_context* ctx = nullptr;
  std::vector<void*> bufs;
  // host tables whose asynchronous copies may still be in flight, and the
  // stream the work was last enqueued on (release is ordered after it)
  std::deque<std::vector<char>> host_keep;
  hipStream_t stream = nullptr;
  lgs_settings st{};
  Plan plan;
  int64_t n = 0, n_rid = 0;
  int npad_shift = 0, app_bf16 = 0;
  int64_t cap_pairs = 0, cap_slots = 0;
  lgs_counts counts{};
  ViewDesc* d_views = nullptr;
  // per-view image tables, one set of n_views per feature group: forward
  // outputs (d_out), upstream (d_up), the forward's images read by the fused
  // loss gradient (d_fo), targets (d_tgt); loss weights (4 per group)
  ViewImages *d_out = nullptr, *d_up = nullptr, *d_fo = nullptr, *d_tgt = nullptr;
  float* d_lossw = nullptr;
  int want_ncon = 0;                         // some view of the forward's outputs asks for contributor counts
  int D = kFeatGroup, G = 1;                 // feature dimension and groups
  float* scratch_img = nullptr;              // groups 1 ..: their RGB / depth / T outputs (discarded)
  float* zero_img = nullptr;                 // groups 1 ..: zero RGB / depth upstream
  int gb = 1;                                // groups at once in the backward
  int64_t app_stride = 0;                    // bytes from one group's appearance records to the next
  int64_t grad2d_stride = 0, mask_stride = 0;
  float* geo_acc = nullptr;
  uint32_t *work_q = nullptr, *work_qb = nullptr;   // [group][kQueueWords]
  GeomRec* geom = nullptr;
  uint32_t *cnt_t = nullptr, *cnt_b = nullptr, *cidx = nullptr, *slot_base = nullptr;
  uint32_t *ent = nullptr, *ent_a = nullptr, *ent_b = nullptr, *srid = nullptr;
  uint32_t *off_t = nullptr, *slot_off = nullptr, *long_ids = nullptr;
  uint32_t *dkey = nullptr, *dk0 = nullptr, *dk1 = nullptr;
  void* app = nullptr;
  Counters* counters = nullptr;
  int32_t* last_idx = nullptr;
  float* T_state = nullptr;
  void *scan_tmp = nullptr, *radix_small = nullptr, *radix_big = nullptr;
  uint32_t *k0 = nullptr, *v0 = nullptr, *k1 = nullptr, *v1 = nullptr, *pkeys = nullptr, *pvals = nullptr;
  uint2* ranges = nullptr;
  int64_t range_words = 0;    // to be cleared from there on
  const uint32_t* items_static = nullptr;
  uint32_t* ii_a = nullptr;   // work items in scheduling order
  const uint32_t* items = nullptr;
  float* partials = nullptr;
  uint8_t* mask = nullptr;
  int64_t mask_words = 0;     // still to be zeroed
  float* grad2d = nullptr;
  void* ttmp = nullptr;
  bool bwd_alloc = false;
  // graph with the D-SSIM loss: upstream planes [20][H][W] per view, the
  // loss view table and partial sums
  float* up_buf = nullptr;
  LossView* loss_tab = nullptr;
  float2* loss_part = nullptr;
  int64_t loss_blocks = 0;
  LossConsts loss_k{};
  // settings.profile: events on the caller's stream around each stage
  // (0 forward start, 1 front end, 2 pairs start, 3 raster start, 4 raster
  // end, 5 backward raster start, 6 backward raster end, 7 backward end)
  hipEvent_t ev[8] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
};

namespace {

void* w_alloc(Work* W, size_t bytes, bool& ok) {
  void* p = pool_alloc(W->ctx, bytes, W->stream);
  if (!p) ok = false;
  else W->bufs.push_back(p);
  return p;
}

// Give the buffers from number `from` on back to the context without waiting:
// they become reusable once the work enqueued so far on the Work's stream has
// run (the returned event; null: it has).
SharedEvent w_give_back(Work* W, size_t from) {
  SharedEvent ev = make_event();
  if (ev && hipEventRecord(ev.get(), W->stream) != hipSuccess) ev.reset();
  if (!ev) hipStreamSynchronize(W->stream);
  for (size_t i = from; i < W->bufs.size(); ++i) pool_free(W->ctx, W->bufs[i], ev);
  W->bufs.resize(from);
  return ev;
}

// All of them, and the host tables.
void w_release(Work* W) {
  const SharedEvent ev = w_give_back(W, 0);
  if (!W->host_keep.empty()) {
    W->ctx->deferred.push_back(DeferredHost{ev, std::move(W->host_keep)});
    W->host_keep.clear();
  }
  sweep_deferred(W->ctx);
  for (int i = 0; i < 8; ++i)
    if (W->ev[i]) {
      hipEventDestroy(W->ev[i]);
      W->ev[i] = nullptr;
    }
}

// Buffers of a Work that share one block of the pool, each on a 256-byte line;
// where no block holds them all, they get blocks of their own (those added as
// `joined` stay behind the one before them).
class Carve {
 public:
  template <class T>
  void add(T*& p, size_t bytes, bool joined = false) {
    parts_.push_back({(void*)&p, total_, joined});
    total_ += (bytes + 255) / 256 * 256;
  }
  // all of the buffers, or none (and all pointers null)
  bool get(Work* W) {
    const size_t held = W->bufs.size();
    if (take(W, 0, parts_.size())) return true;
    bool ok = true;
    for (size_t i = 0, j; ok && i < parts_.size(); i = j) {
      for (j = i + 1; j < parts_.size() && parts_[j].joined;) ++j;
      ok = take(W, i, j);
    }
    if (ok) return true;
    for (const Part& x : parts_) set(x, nullptr);
    w_give_back(W, held);
    return false;
  }

 private:
  struct Part {
    void* p;   // the pointer to set
    size_t off;
    bool joined;
  };
  static void set(const Part& x, char* at) { memcpy(x.p, &at, sizeof at); }
  bool take(Work* W, size_t i, size_t j) {
    bool ok = true;
    const size_t off = i < j ? parts_[i].off : 0, end = j < parts_.size() ? parts_[j].off : total_;
    char* base = (char*)w_alloc(W, end - off, ok);
    for (; ok && i < j; ++i) set(parts_[i], base + (parts_[i].off - off));
    return ok;
  }
  std::vector<Part> parts_;
  size_t total_ = 0;
};

// Asynchronous copy of host tables to device buffers that follow one another
// in one block, as one copy; the host copy is kept with the Work (then with
// the context until the copy has surely run).
struct Table {
  void* dst;
  const void* src;
  size_t bytes;
};
hipError_t upload_tables(Work* W, std::initializer_list<Table> tables, hipStream_t s) {
  char* const base = (char*)tables.begin()->dst;
  const Table& last = *(tables.end() - 1);
  std::vector<char> host((char*)last.dst + last.bytes - base);
  for (const Table& t : tables)
    if (t.bytes) memcpy(host.data() + ((char*)t.dst - base), t.src, t.bytes);
  if (host.empty()) return hipSuccess;
  W->host_keep.push_back(std::move(host));
  const std::vector<char>& b = W->host_keep.back();
  return hipMemcpyAsync(base, b.data(), b.size(), hipMemcpyHostToDevice, s);
}
template <class T>
Table table(void* dst, const std::vector<T>& v) {
  return Table{dst, v.data(), v.size() * sizeof(T)};
}

void w_mark(Work* W, int i, hipStream_t s) {
  if (W->ev[i]) hipEventRecord(W->ev[i], s);
}

uint32_t* get_items(lgs_context* ctx, const Plan& P, int tile, bool spatial) {
  const std::string key = P.sig + (spatial ? "s" : "r");
  auto it = ctx->items_cache.find(key);
  if (it != ctx->items_cache.end()) return it->second.first;
  std::vector<uint32_t> items = make_items(P, tile, spatial);
  uint32_t* d = nullptr;
  if (hipMalloc(&d, std::max<size_t>(4, items.size() * 4)) != hipSuccess) return nullptr;
  if (!items.empty() && hipMemcpy(d, items.data(), items.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
    hipFree(d);
    return nullptr;
  }
  ctx->items_cache[key] = {d, (int64_t)items.size()};
  return d;
}

lgs_status w_init(Work* W, lgs_context* ctx, const lgs_settings* st, const lgs_gaussians* g, int32_t n_views,
                  const lgs_camera* cams, hipStream_t stream) {
  W->ctx = ctx;
  W->stream = stream;
  W->st = *st;
  W->plan = make_plan(st, n_views, cams);
  W->n = g->n;
  W->app_bf16 = g->appearance_dtype == LGS_BF16;
  W->D = feat_dim_of(g);
  W->G = (W->D + kFeatGroup - 1) / kFeatGroup;
  W->npad_shift = (int)ceil_log2((uint64_t)std::max<int64_t>(g->n, 1));
  W->n_rid = (int64_t)n_views << W->npad_shift;
  // the compositing kernels address the per-(view, Gaussian) records (32
  // bytes) and the per-Gaussian appearance records (40 bytes BF16, 80 FP32)
  // by 32-bit byte offsets
  if (W->n_rid > ((int64_t)1 << 27)) return fail(ctx, LGS_ERR_UNSUPPORTED, "n_views * 2^ceil(log2 n) exceeds 2^27");
  if (((int64_t)(W->app_bf16 ? 40 : 80) << W->npad_shift) > ((int64_t)1 << 32))
    return fail(ctx, LGS_ERR_UNSUPPORTED, "2^ceil(log2 n) exceeds 2^26 (BF16 appearance) or 2^25 (FP32)");
  if (W->plan.n_items > ((int64_t)1 << 31)) return fail(ctx, LGS_ERR_UNSUPPORTED, "too many pixels");
  return LGS_OK;
}

// buffers whose size does not depend on the pair count
lgs_status w_alloc_front(Work* W) {
  Carve block;
  const int V = (int)W->plan.views.size();
  const int64_t n_rid = W->n_rid, npix = std::max<int64_t>(W->plan.n_pix, 1);
  // (uploaded together: views and out; fo, tgt and lossw)
  block.add(W->d_views, sizeof(ViewDesc) * V);
  const int G = W->G;
  block.add(W->d_out, sizeof(ViewImages) * V * G, true);
  block.add(W->d_up, sizeof(ViewImages) * V * G);
  block.add(W->d_fo, sizeof(ViewImages) * V * G);
  block.add(W->d_tgt, sizeof(ViewImages) * V * G, true);
  block.add(W->d_lossw, 16 * G, true);
  if (G > 1) block.add(W->scratch_img, sizeof(float) * 5 * npix);
  block.add(W->geom, sizeof(GeomRec) * n_rid);
  block.add(W->cnt_t, 4 * n_rid);
  block.add(W->cnt_b, 4 * n_rid);
  block.add(W->cidx, 4 * n_rid);
  block.add(W->slot_base, 4 * n_rid);
  block.add(W->ent, 4 * n_rid);
  block.add(W->ent_a, 4 * n_rid);
  block.add(W->ent_b, 4 * n_rid);
  block.add(W->off_t, 4 * n_rid);
  block.add(W->slot_off, 4 * n_rid);
  block.add(W->long_ids, 4 * n_rid);
  block.add(W->dkey, 4 * n_rid);
  block.add(W->dk0, 4 * n_rid);
  block.add(W->dk1, 4 * n_rid);
  W->app_stride = (std::max<int64_t>(W->n, 1) * (W->app_bf16 ? 40 : 80) + 255) / 256 * 256;
  block.add(W->app, (size_t)W->app_stride * G);
  block.add(W->counters, sizeof(Counters));
  block.add(W->last_idx, 4 * npix);
  block.add(W->T_state, 4 * npix);
  block.add(W->scan_tmp, scan_temp_bytes(n_rid));
  block.add(W->radix_small, radix_temp_bytes(n_rid, kSmallIds));
  // the tile ranges and the forward's work counters, cleared together
  W->range_words = (2 * W->plan.n_tiles + kLineWords - 1) / kLineWords * kLineWords + (int64_t)G * kQueueWords;
  block.add(W->ranges, 4 * W->range_words);
  block.add(W->work_qb, 4 * (size_t)G * kQueueWords);
  const int64_t ni = std::max<int64_t>(W->plan.n_items, 1);
  block.add(W->ii_a, 4 * ni);
  W->items_static = get_items(W->ctx, W->plan, W->st.tile, W->st.order == 2);
  if (!block.get(W) || !W->items_static) return fail(W->ctx, LGS_ERR_HIP, "device allocation failed");
  W->work_q = (uint32_t*)W->ranges + (W->range_words - (int64_t)G * kQueueWords);
  return LGS_OK;
}

lgs_status w_alloc_pairs(Work* W, int64_t cap_pairs, int64_t cap_slots) {
  Carve block;
  W->cap_pairs = cap_pairs;
  W->cap_slots = cap_slots;
  const int64_t pa = std::max<int64_t>(cap_pairs, 1);
  block.add(W->k0, 4 * pa);
  block.add(W->v0, 4 * pa);
  block.add(W->k1, 4 * pa);
  block.add(W->v1, 4 * pa);
  block.add(W->radix_big, radix_temp_bytes(pa, kSmallPairs));
  if (!block.get(W)) return fail(W->ctx, LGS_ERR_HIP, "device allocation failed (pairs)");
  return LGS_OK;
}

constexpr int64_t kGroupBytes = 1ll << 31;

lgs_status w_alloc_bwd(Work* W) {
  if (W->bwd_alloc) return LGS_OK;
  const int64_t S = std::max<int64_t>(W->cap_slots, 1), R = std::max<int64_t>(W->n_rid, 1);
  // as many feature groups at once as keep their records within 2 GB (a frame
  // large enough to pass that fills the chip with one), fewer where memory for
  // so many is not to be had
  W->gb = (int)std::min<int64_t>(W->G, std::max<int64_t>(1, kGroupBytes / (4 * (S * kSlotFloats + R * kPartials))));
  W->grad2d_stride = R * kPartials;
  W->mask_stride = (S + 8 + 255) / 256 * 256;
  for (;; W->gb /= 2) {
    Carve block;
    block.add(W->partials, sizeof(float) * kSlotFloats * S * W->gb);
    block.add(W->mask, W->mask_stride * W->gb);
    block.add(W->grad2d, sizeof(float) * W->grad2d_stride * W->gb);
    block.add(W->ttmp, project_bwd_temp_bytes(W->n_rid, (int)W->plan.views.size()));
    if (W->gb < W->G) block.add(W->geo_acc, sizeof(float) * 6 * R);
    if (block.get(W)) break;
    if (W->gb == 1) return fail(W->ctx, LGS_ERR_HIP, "device allocation failed (backward)");
  }
  // the slot mask starts at zero (the first backward clears it, together with
  // its counters); every reduction leaves it at zero again
  W->mask_words = W->mask_stride * W->gb / 4;
  W->bwd_alloc = true;
  return LGS_OK;
}

int64_t view_plane(const Work* W, int v) { return (int64_t)W->plan.views[v].W * W->plan.views[v].H; }

// zero RGB / depth upstream of the groups beyond the first, where a backward
// is given its upstream
lgs_status w_zero_img(Work* W) {
  if (W->G == 1 || W->zero_img) return LGS_OK;
  bool ok = true;
  const size_t n = 4 * (size_t)std::max<int64_t>(W->plan.n_pix, 1);
  W->zero_img = (float*)w_alloc(W, sizeof(float) * n, ok);
  if (!ok) return fail(W->ctx, LGS_ERR_HIP, "device allocation failed (backward)");
  launch_fill_u32((uint32_t*)W->zero_img, 0u, (int64_t)n, W->stream);
  return LGS_OK;
}

// Per-group tables, [group][view], from the callers' images: group g reads or
// writes feature planes 16 g ... of each view's feature image.
enum TableKind { TAB_OUT, TAB_UP, TAB_FO, TAB_TGT, TAB_UP_RGB };
std::vector<ViewImages> group_tables(const Work* W, const lgs_images* im, TableKind kind) {
  const int V = (int)W->plan.views.size();
  std::vector<ViewImages> t((size_t)V * W->G);
  for (int gi = 0; gi < W->G; ++gi)
    for (int v = 0; v < V; ++v) {
      const int64_t hw = view_plane(W, v), po = W->plan.views[v].pix_off;
      float* feat = im && im[v].feat ? im[v].feat + (int64_t)kFeatGroup * gi * hw : nullptr;
      ViewImages x{nullptr, nullptr, feat, nullptr, nullptr};
      if (gi == 0) {
        x = ViewImages{im[v].rgb, im[v].depth, im[v].feat, kind == TAB_TGT ? nullptr : im[v].final_T,
                       kind == TAB_OUT ? im[v].n_contrib : nullptr};
        if (kind == TAB_UP_RGB) x = ViewImages{im[v].rgb, nullptr, nullptr, nullptr, nullptr};
      } else if (kind == TAB_OUT) {
        float* sc = W->scratch_img + 5 * po;     // RGB, depth, T of this group go nowhere
        x = ViewImages{sc, sc + 3 * hw, feat, sc + 4 * hw, nullptr};
      } else if (kind == TAB_UP || kind == TAB_UP_RGB) {
        float* z = W->zero_img + 4 * po;          // no colour or depth upstream in this group
        x = ViewImages{z, z + 3 * hw, kind == TAB_UP ? feat : nullptr, nullptr, nullptr};
      } else {                                    // TAB_FO, TAB_TGT: the residual's images
        x = ViewImages{im[v].rgb, im[v].depth, feat, nullptr, nullptr};
      }
      t[(size_t)gi * V + v] = x;
    }
  return t;
}

// loss weights per group: colour and depth terms in group 0 only; the
// feature term's 1/(16 HW) scale in the kernel becomes 1/(D HW)
std::vector<float> group_lossw(const Work* W, const float loss_w[3]) {
  std::vector<float> lw(4 * (size_t)W->G, 0.f);
  const float wf = loss_w[2] * ((float)kFeatGroup / (float)W->D);
  for (int gi = 0; gi < W->G; ++gi) {
    lw[4 * gi + 0] = gi == 0 ? loss_w[0] : 0.f;
    lw[4 * gi + 1] = gi == 0 ? loss_w[1] : 0.f;
    lw[4 * gi + 2] = wf;
  }
  return lw;
}

lgs_status w_upload(Work* W, const lgs_images* out, hipStream_t stream) {
  const int V = (int)W->plan.views.size();
  const std::vector<ViewImages> himg = group_tables(W, out, TAB_OUT);
  W->want_ncon = 0;
  for (int v = 0; v < V; ++v) W->want_ncon |= out[v].n_contrib != nullptr;
  HIP_TRY(W->ctx, upload_tables(W, {table(W->d_views, W->plan.views), table(W->d_out, himg)}, stream));
  return LGS_OK;
}

// projection .. slot bases: everything up to the pair / slot counts
void enqueue_front(Work* W, const lgs_gaussians* g, hipStream_t s) {
  const Settings ds = dev_settings(&W->st, W->plan.tile_shift, W->D);
  const int V = (int)W->plan.views.size();
  const int64_t n_rid = W->n_rid;
  launch_project(ds, W->d_views, V, g->means, g->log_scales, g->quats, g->opacity_logits, g->rgb, g->feat,
                 W->app_bf16, W->n, W->npad_shift, W->geom, W->cnt_t, W->cnt_b, W->dkey, W->app, W->counters, s);
  if (n_rid <= kSmallFront) {
    W->srid = W->ent_a;
    launch_small_front(FrontLists{W->cnt_t, W->cnt_b, W->dkey, W->cidx, W->ent, W->srid, W->off_t, W->slot_off,
                                  W->slot_base, W->long_ids},
                       n_rid, W->counters, s);
  } else {
    // the visibility scan also compacts: ent (kept, index order), a copy that
    // the depth sort permutes, and the depth keys in the same order
    Compact cp;
    cp.key_src = W->dkey;
    cp.ent = W->ent;
    cp.ent_copy = W->ent_a;
    cp.keys = W->dk0;
    launch_scan(SCAN_FLAG_NONZERO, W->cnt_t, W->cidx, &W->counters->n_visible, n_rid, W->scan_tmp, s, cp);
    bool alt = false;
    radix_sort_u32(W->dk0, W->ent_a, W->dk1, W->ent_b, &W->counters->n_visible, n_rid, kSmallIds, 0, 32,
                   W->radix_small, s, &alt);
    W->srid = alt ? W->ent_b : W->ent_a;
    // pair offsets in depth order; slot offsets in visible order, and the same
    // as each record's slot base
    const GatherScan pairs{W->cnt_t, W->srid, W->off_t, &W->counters->n_pairs, nullptr, Compact()};
    GatherScan slots{W->cnt_b, W->ent, W->slot_off, &W->counters->n_slots, W->slot_base, Compact()};
    slots.cp.big = W->long_ids;
    slots.cp.n_big = &W->counters->n_long;
    slots.cp.big_min = kLongSlots;
    launch_gather_scans(pairs, slots, &W->counters->n_visible, n_rid, W->scan_tmp, s);
  }
  launch_pack_app_groups(g->feat, W->app_bf16, W->n, W->G, W->app, W->app_stride, s);
}

// emission, tile sort, tile ranges, work order (capacity-bounded)
void enqueue_pairs(Work* W, hipStream_t s) {
  const Plan& P = W->plan;
  launch_emit(W->geom, W->d_views, W->srid, W->off_t, W->counters, W->cap_pairs, W->cap_slots, W->npad_shift,
              P.tile_shift, W->k0, W->v0, (uint32_t*)W->ranges, W->range_words, s);
  const int tile_bits = std::max<int>(1, (int)ceil_log2((uint64_t)P.n_tiles));
  bool alt = false;
  radix_sort_u32(W->k0, W->v0, W->k1, W->v1, &W->counters->n_pairs_eff, std::max<int64_t>(W->cap_pairs, 1),
                 kSmallPairs, 0, tile_bits, W->radix_big, s, &alt);
  W->pkeys = alt ? W->k1 : W->k0;
  W->pvals = alt ? W->v1 : W->v0;
  launch_tile_ranges(W->pkeys, W->counters, W->cap_pairs, W->ranges, s);
  if (W->st.order != 0)
    W->items = launch_order_items(W->ranges, W->items_static, W->items_static + P.n_items,
                                  (const TileItems*)(W->items_static + P.n_items + kQueues + 1),
                                  W->items_static + P.n_items + kQueues + 1 + 4 * P.n_tiles, P.n_tiles, W->ii_a, s);
  else
    W->items = W->items_static;
}

Groups groups_of(const Work* W) {
  Groups gr;
  gr.count = gr.total = W->G;
  gr.n_views = (int)W->plan.views.size();
  gr.app_stride = W->app_stride;
  gr.slots = std::max<int64_t>(W->cap_slots, 1);
  gr.mask_stride = W->mask_stride;
  return gr;
}

// every feature group over the same lists, at once: group 0 (RGB, depth,
// features 0..15) and the further ones (their RGB / depth / T outputs go to
// scratch).  A small frame has fewer blocks than the chip has wave slots: four
// groups of 320 x 240 took 4 x 58 us one after the other, 84 at once, and their
// backwards 4 x 73 and 139.
void enqueue_raster_fwd(Work* W, hipStream_t s) {
  const Settings ds = dev_settings(&W->st, W->plan.tile_shift, W->D);
  launch_raster_fwd(ds, groups_of(W), W->d_views, W->d_out, W->ranges, W->pvals, W->geom, W->app, W->app_bf16,
                    (uint32_t)((1ull << W->npad_shift) - 1), W->items, W->items_static + W->plan.n_items,
                    W->plan.n_items, W->counters, W->work_q, W->st.chunk, W->last_idx, W->T_state, W->want_ncon, s);
}

// Backward compositing: the feature groups in the order 1 .., 0, W->gb at a
// time; upstream by mode (UpMode): d_up; dL1/dY from (d_fo, d_tgt, d_lossw); or
// colour channels from d_up and depth + features from the L1 residual.  Each
// batch of groups but the last is reduced per Gaussian, its feature gradients
// written and its geometric sums accumulated here; the last one's reduction and
// the projection backward follow in enqueue_backward_reduce.
// The slot mask is cleared by the first backward over it; from then on the
// reduction clears each byte it reads.
Groups backward_groups(const Work* W, int at) {
  Groups gr = groups_of(W);
  gr.first = (1 + at) % W->G;
  gr.count = std::min(W->gb, W->G - at);
  return gr;
}

void enqueue_group_reduce(Work* W, const Groups& gr, const lgs_grads* out, hipStream_t s) {
  launch_seg_reduce(gr, W->slot_off, W->partials, W->mask, W->long_ids, W->counters, W->n_rid, W->grad2d,
                    W->grad2d_stride, s);
  if (W->G > 1)
    launch_group_feat_grad(gr, W->n, (uint32_t)W->npad_shift, W->counters, W->cnt_t, W->cidx, W->grad2d,
                           W->grad2d_stride, out->feat, s);
}

void enqueue_backward_raster(Work* W, const lgs_grads* out, int mode, hipStream_t s) {
  const Settings ds = dev_settings(&W->st, W->plan.tile_shift, W->D);
  const bool sign = mode != UP_EXPLICIT;
  if (W->G > 1) w_mark(W, 5, s);
  ZeroRanges z;
  z.p[0] = W->work_qb;
  z.n[0] = (int64_t)W->G * kQueueWords;
  z.p[1] = (uint32_t*)&W->counters->bwd_evals;   // bwd_evals, _contrib, _entries, _written
  z.n[1] = 8;
  z.p[2] = (uint32_t*)W->mask;
  z.n[2] = W->mask_words;
  W->mask_words = 0;
  launch_zero(z, s);
  if (W->G == 1) w_mark(W, 5, s);   // one group: the stage is the kernel alone
  for (int at = 0; at < W->G; at += W->gb) {
    const Groups gr = backward_groups(W, at);
    launch_raster_bwd(mode, ds, gr, W->d_views, W->d_up, sign ? W->d_fo : nullptr, sign ? W->d_tgt : nullptr,
                      sign ? W->d_lossw : nullptr, W->ranges, W->pvals, W->geom, W->app, W->app_bf16,
                      (uint32_t)((1ull << W->npad_shift) - 1), W->items, W->items_static + W->plan.n_items,
                      W->plan.n_items, W->counters, W->work_qb, W->st.chunk, W->last_idx, W->T_state, W->slot_base,
                      W->partials, W->mask, s);
    if (at + gr.count == W->G) break;
    enqueue_group_reduce(W, gr, out, s);
    launch_group_geo_acc(W->grad2d, W->grad2d_stride, gr.count, W->counters, W->n_rid, W->geo_acc, at == 0, s);
  }
  w_mark(W, 6, s);
}

void enqueue_backward_reduce(Work* W, const lgs_gaussians* g, const lgs_grads* gr, hipStream_t s) {
  const Settings ds = dev_settings(&W->st, W->plan.tile_shift, W->D);
  const int V = (int)W->plan.views.size();
  const int last = (W->G - 1) / W->gb * W->gb;
  const Groups lg = backward_groups(W, last);
  enqueue_group_reduce(W, lg, gr, s);
  GroupGeo geo;   // group 0 is the batch's last
  geo.acc = last > 0 ? W->geo_acc : nullptr;
  geo.grad2d = W->grad2d;
  geo.stride = W->grad2d_stride;
  geo.n = lg.count - 1;
  launch_project_bwd(ds, W->d_views, V, g->means, g->log_scales, g->quats, g->opacity_logits, W->n,
                     W->npad_shift, W->n_rid, W->counters, W->cnt_t, W->cidx, W->ent, geo,
                     W->grad2d + (lg.count - 1) * W->grad2d_stride, gr->means,
                     gr->log_scales, gr->quats, gr->opacity_logits, gr->rgb, gr->feat, gr->twist, W->ttmp, s);
  w_mark(W, 7, s);
}

void enqueue_backward(Work* W, const lgs_gaussians* g, const lgs_grads* gr, int mode, hipStream_t s) {
  enqueue_backward_raster(W, gr, mode, s);
  enqueue_backward_reduce(W, g, gr, s);
}

lgs_status read_counts(Work* W, hipStream_t s, Counters* hc) {
  lgs_context* ctx = W->ctx;
  if (!ctx->counts_host)
    HIP_TRY(ctx, hipHostMalloc((void**)&ctx->counts_host, sizeof(Counters), hipHostMallocDefault));
  HIP_TRY(ctx, hipMemcpyAsync(ctx->counts_host, W->counters, offsetof(Counters, pad2), hipMemcpyDeviceToHost, s));
  HIP_TRY(ctx, hipStreamSynchronize(s));
  *hc = *ctx->counts_host;
  W->counts.n_visible = hc->n_visible;
  W->counts.n_pairs = hc->n_pairs;
  W->counts.n_slots = hc->n_slots;
  W->counts.n_tiles = W->plan.n_tiles;
  W->counts.n_items = W->plan.n_items;
  W->counts.fwd_evals = (int64_t)hc->fwd_evals;
  W->counts.fwd_contrib = (int64_t)hc->fwd_contrib;
  W->counts.bwd_evals = (int64_t)hc->bwd_evals;
  W->counts.bwd_contrib = (int64_t)hc->bwd_contrib;
  W->counts.fwd_entries = (int64_t)hc->fwd_entries;
  W->counts.bwd_entries = (int64_t)hc->bwd_entries;
  W->counts.bwd_written = (int64_t)hc->bwd_written;
  return LGS_OK;
}

lgs_status check_grads(lgs_context* ctx, const lgs_gaussians* g, const lgs_grads* grads) {
  if (!grads) return fail(ctx, LGS_ERR_INVALID_ARG, "grads is NULL");
  if (g->n > 0 && (!grads->means || !grads->log_scales || !grads->quats || !grads->opacity_logits ||
                   !grads->rgb || !grads->feat))
    return fail(ctx, LGS_ERR_INVALID_ARG, "NULL gradient plane");
  return LGS_OK;
}

}  // namespace

struct lgs_fwd_state {
  Work W;
};

static constexpr bool kGraphEnabled = true;

struct lgs_graph {
  Work W;
  hipGraph_t graph = nullptr;        // the whole step (settings.profile = 0)
  hipGraphExec_t exec = nullptr;
  // settings.profile = 1: the five stages captured as five graphs, launched
  // back to back with events recorded between them on the launching stream
  // (events recorded inside a captured graph cannot be timed)
  hipGraph_t sgraph[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  hipGraphExec_t sexec[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  hipStream_t cap_stream = nullptr;
  hipStream_t last_stream = nullptr;
  lgs_gaussians g{};
  lgs_grads grads{};
  hipEvent_t ev[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  bool profile = false;
};

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

const char* lgs_status_string(lgs_status s) {
  switch (s) {
    case LGS_OK: return "LGS_OK";
    case LGS_ERR_INVALID_ARG: return "LGS_ERR_INVALID_ARG";
    case LGS_ERR_HIP: return "LGS_ERR_HIP";
    case LGS_ERR_CAPACITY: return "LGS_ERR_CAPACITY";
    case LGS_ERR_UNSUPPORTED: return "LGS_ERR_UNSUPPORTED";
    case LGS_ERR_STATE: return "LGS_ERR_STATE";
    default: break;
  }
  return "LGS_ERR_UNKNOWN";
}

const char* lgs_last_error(const lgs_context* ctx) { return ctx ? ctx->err.c_str() : "NULL context"; }

lgs_settings lgs_default_settings(void) {
  lgs_settings s;
  s.z_near = 0.2f; s.eps2d = 0.3f; s.fov_clamp = 1.3f; s.alpha_max = 0.99f;
  s.alpha_min = 1.0f / 255.0f; s.T_eps = 1e-4f; s.cutoff2 = 9.0f;
  s.tile = 16; s.chunk = 4; s.order = 0; s.profile = 0;
  return s;
}

// Device address of the scratch array on `device` (which must be current),
// looked up once per device and kept for the life of the process; null when
// the lookup fails.
static float* scratch_address(int device) {
  static std::mutex mu;
  static std::map<int, float*> table;
  std::lock_guard<std::mutex> lock(mu);
  auto it = table.find(device);
  if (it != table.end()) return it->second;
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
  table[device] = (float*)p;
  return (float*)p;
}

lgs_status lgs_context_create(int hip_device, lgs_context** out) {
  if (!out) return LGS_ERR_INVALID_ARG;
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) return LGS_ERR_HIP;
  if (hip_device < 0 || hip_device >= count) return LGS_ERR_INVALID_ARG;
  if (hipSetDevice(hip_device) != hipSuccess) return LGS_ERR_HIP;
  float* sp = scratch_address(hip_device);
  if (!sp) return LGS_ERR_HIP;
  lgs_context* c = new lgs_context();
  c->device = hip_device;
  c->scratch = sp;
  *out = c;
  return LGS_OK;
}

void lgs_context_destroy(lgs_context* ctx) {
  if (!ctx) return;
  hipSetDevice(ctx->device);
  hipDeviceSynchronize();
  for (auto& kv : ctx->free_blocks) hipFree(kv.second.p);
  ctx->free_blocks.clear();   // drops the blocks' events before the context goes
  ctx->deferred.clear();
  for (auto& kv : ctx->live) hipFree(kv.first);
  for (auto& kv : ctx->items_cache) hipFree(kv.second.first);
  if (ctx->loss_host) hipHostFree(ctx->loss_host);
  if (ctx->loss_tab) hipFree(ctx->loss_tab);
  if (ctx->loss_part) hipFree(ctx->loss_part);
  if (ctx->loss_copied) hipEventDestroy(ctx->loss_copied);
  if (ctx->dec_part) hipFree(ctx->dec_part);
  if (ctx->counts_host) hipHostFree(ctx->counts_host);
  if (ctx->prune_host) hipHostFree(ctx->prune_host);
  delete ctx;
}

lgs_status lgs_state_counts(const lgs_fwd_state* s, lgs_counts* out) {
  if (!s || !out) return LGS_ERR_INVALID_ARG;
  lgs_fwd_state* S = const_cast<lgs_fwd_state*>(s);
  hipSetDevice(S->W.ctx->device);
  hipDeviceSynchronize();
  Counters hc;
  lgs_status rc = read_counts(&S->W, nullptr, &hc);
  if (rc != LGS_OK) return rc;
  *out = S->W.counts;
  return LGS_OK;
}

lgs_status lgs_state_stage_ms(const lgs_fwd_state* s, float ms[5]) {
  if (!s || !ms) return LGS_ERR_INVALID_ARG;
  const Work* W = &s->W;
  if (!W->ev[0]) return fail(W->ctx, LGS_ERR_STATE, "forward was run without settings.profile");
  HIP_TRY(W->ctx, hipEventSynchronize(W->ev[7]));
  const int a[5] = {0, 2, 3, 5, 6}, b[5] = {1, 3, 4, 6, 7};
  for (int i = 0; i < 5; ++i) HIP_TRY(W->ctx, hipEventElapsedTime(&ms[i], W->ev[a[i]], W->ev[b[i]]));
  return LGS_OK;
}

lgs_status lgs_state_release(lgs_context* ctx, lgs_fwd_state* s) {
  if (!ctx || !s) return LGS_ERR_INVALID_ARG;
  if (s->W.ctx != ctx) return fail(ctx, LGS_ERR_STATE, "state belongs to another context");
  hipSetDevice(ctx->device);
  w_release(&s->W);   // stream-ordered: queued work keeps its buffers until it has run
  delete s;
  return LGS_OK;
}

lgs_status lgs_forward(lgs_context* ctx, const lgs_settings* st, const lgs_gaussians* g, int32_t n_views,
                       const lgs_camera* cams, const lgs_images* out, lgs_fwd_state** state_out,
                       hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  if (!state_out) return fail(ctx, LGS_ERR_INVALID_ARG, "state_out is NULL");
  *state_out = nullptr;
  lgs_status rc;
  if ((rc = check_settings(ctx, st)) != LGS_OK) return rc;
  if ((rc = check_gaussians(ctx, g)) != LGS_OK) return rc;
  if ((rc = check_cams(ctx, n_views, cams)) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, out, true, "out")) != LGS_OK) return rc;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  lgs_fwd_state* S = new lgs_fwd_state();
  Work* W = &S->W;
  auto bail = [&](lgs_status e) {
    w_release(W);
    delete S;
    return e;
  };
  if ((rc = w_init(W, ctx, st, g, n_views, cams, stream)) != LGS_OK) return bail(rc);
  if ((rc = w_alloc_front(W)) != LGS_OK) return bail(rc);
  if ((rc = w_upload(W, out, stream)) != LGS_OK) return bail(rc);
  if (st->profile & LGS_PROFILE_EVENTS)
    for (int i = 0; i < 8; ++i)
      if (hipEventCreate(&W->ev[i]) != hipSuccess) return bail(fail(ctx, LGS_ERR_HIP, "event creation failed"));
  w_mark(W, 0, stream);
  enqueue_front(W, g, stream);
  w_mark(W, 1, stream);
  if (hipGetLastError() != hipSuccess) return bail(fail(ctx, LGS_ERR_HIP, "kernel launch failed"));
  Counters hc;
  if ((rc = read_counts(W, stream, &hc)) != LGS_OK) return bail(rc);
  if ((rc = w_alloc_pairs(W, hc.n_pairs, hc.n_slots)) != LGS_OK) return bail(rc);
  w_mark(W, 2, stream);
  enqueue_pairs(W, stream);
  w_mark(W, 3, stream);
  enqueue_raster_fwd(W, stream);
  w_mark(W, 4, stream);
  if (hipGetLastError() != hipSuccess) return bail(fail(ctx, LGS_ERR_HIP, "kernel launch failed"));
  *state_out = S;
  return LGS_OK;
}

lgs_status lgs_backward(lgs_context* ctx, const lgs_fwd_state* Sc, const lgs_gaussians* g,
                        const lgs_images* grad_out, lgs_grads* grads, hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  if (!Sc) return fail(ctx, LGS_ERR_INVALID_ARG, "state is NULL");
  lgs_fwd_state* S = const_cast<lgs_fwd_state*>(Sc);
  Work* W = &S->W;
  if (W->ctx != ctx) return fail(ctx, LGS_ERR_STATE, "state belongs to another context");
  lgs_status rc;
  if ((rc = check_gaussians(ctx, g)) != LGS_OK) return rc;
  if (g->n != W->n) return fail(ctx, LGS_ERR_INVALID_ARG, "n differs from the forward's");
  if (feat_dim_of(g) != W->D) return fail(ctx, LGS_ERR_INVALID_ARG, "feat_dim differs from the forward's");
  const int V = (int)W->plan.views.size();
  if ((rc = check_images(ctx, V, grad_out, false, "grad_out")) != LGS_OK) return rc;
  if ((rc = check_grads(ctx, g, grads)) != LGS_OK) return rc;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  W->stream = stream;
  if ((rc = w_alloc_bwd(W)) != LGS_OK) return rc;
  if ((rc = w_zero_img(W)) != LGS_OK) return rc;
  const std::vector<ViewImages> hup = group_tables(W, grad_out, TAB_UP);
  HIP_TRY(ctx, upload_tables(W, {table(W->d_up, hup)}, stream));
  enqueue_backward(W, g, grads, UP_EXPLICIT, stream);
  HIP_TRY(ctx, hipGetLastError());
  return LGS_OK;
}

lgs_status lgs_backward_l1(lgs_context* ctx, const lgs_fwd_state* Sc, const lgs_gaussians* g,
                           const lgs_images* out, const lgs_images* targets, const float loss_w[3],
                           lgs_grads* grads, hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  if (!Sc) return fail(ctx, LGS_ERR_INVALID_ARG, "state is NULL");
  lgs_fwd_state* S = const_cast<lgs_fwd_state*>(Sc);
  Work* W = &S->W;
  if (W->ctx != ctx) return fail(ctx, LGS_ERR_STATE, "state belongs to another context");
  lgs_status rc;
  if ((rc = check_gaussians(ctx, g)) != LGS_OK) return rc;
  if (g->n != W->n) return fail(ctx, LGS_ERR_INVALID_ARG, "n differs from the forward's");
  if (feat_dim_of(g) != W->D) return fail(ctx, LGS_ERR_INVALID_ARG, "feat_dim differs from the forward's");
  const int V = (int)W->plan.views.size();
  if ((rc = check_images(ctx, V, out, true, "out")) != LGS_OK) return rc;
  if ((rc = check_images(ctx, V, targets, false, "targets")) != LGS_OK) return rc;
  if (!loss_w) return fail(ctx, LGS_ERR_INVALID_ARG, "loss_w is NULL");
  if ((rc = check_grads(ctx, g, grads)) != LGS_OK) return rc;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  W->stream = stream;
  if ((rc = w_alloc_bwd(W)) != LGS_OK) return rc;
  const std::vector<ViewImages> ho = group_tables(W, out, TAB_FO), ht = group_tables(W, targets, TAB_TGT);
  const std::vector<float> lw = group_lossw(W, loss_w);
  HIP_TRY(ctx, upload_tables(W, {table(W->d_fo, ho), table(W->d_tgt, ht), table(W->d_lossw, lw)}, stream));
  enqueue_backward(W, g, grads, UP_L1, stream);
  HIP_TRY(ctx, hipGetLastError());
  return LGS_OK;
}

lgs_status lgs_loss(lgs_context* ctx, int32_t n_views, const lgs_camera* cams, int32_t feat_dim,
                    const lgs_images* out, const lgs_images* targets, const float loss_w[3], float ssim_lambda,
                    const lgs_images* grad, float* terms, hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  lgs_status rc;
  if ((rc = check_cams(ctx, n_views, cams)) != LGS_OK) return rc;
  if (feat_dim == 0) feat_dim = kFeatGroup;
  if (!(feat_dim == 8 || (feat_dim % kFeatGroup == 0 && feat_dim >= 16 && feat_dim <= 128)))
    return fail(ctx, LGS_ERR_INVALID_ARG, "feat_dim must be 8 or a multiple of 16 up to 128 (0: 16)");
  if ((rc = check_images(ctx, n_views, out, false, "out")) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, targets, false, "targets")) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, grad, false, "grad")) != LGS_OK) return rc;
  if ((rc = check_loss_args(ctx, loss_w, ssim_lambda)) != LGS_OK) return rc;
  if (terms && !aligned4(terms)) return fail(ctx, LGS_ERR_INVALID_ARG, "misaligned terms");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  if (!ctx->loss_copied) HIP_TRY(ctx, hipEventCreateWithFlags(&ctx->loss_copied, hipEventDisableTiming));
  HIP_TRY(ctx, hipEventSynchronize(ctx->loss_copied));   // the staging's previous copy is done
  int64_t nb = 0, nd = 0;
  for (int v = 0; v < n_views; ++v) {
    nb += loss_blocks(cams[v].width, cams[v].height);
    nd += loss_df_blocks(cams[v].width, cams[v].height);
  }
  const int64_t np = nb + nd;
  if (n_views > ctx->loss_tab_cap || np > ctx->loss_part_cap) {
    HIP_TRY(ctx, hipDeviceSynchronize());   // earlier calls may still read the old buffers
    if (n_views > ctx->loss_tab_cap) {
      if (ctx->loss_host) hipHostFree(ctx->loss_host);
      if (ctx->loss_tab) hipFree(ctx->loss_tab);
      ctx->loss_host = nullptr;
      ctx->loss_tab = nullptr;
      ctx->loss_tab_cap = 0;
      HIP_TRY(ctx, hipHostMalloc((void**)&ctx->loss_host, sizeof(LossView) * n_views, hipHostMallocDefault));
      HIP_TRY(ctx, hipMalloc((void**)&ctx->loss_tab, sizeof(LossView) * n_views));
      ctx->loss_tab_cap = n_views;
    }
    if (np > ctx->loss_part_cap) {
      if (ctx->loss_part) hipFree(ctx->loss_part);
      ctx->loss_part = nullptr;
      ctx->loss_part_cap = 0;
      HIP_TRY(ctx, hipMalloc((void**)&ctx->loss_part, sizeof(float2) * np));
      ctx->loss_part_cap = np;
    }
  }
  make_loss_views(n_views, cams, feat_dim, out, targets, grad, loss_w, ssim_lambda, ctx->loss_host, &nd);
  HIP_TRY(ctx, hipMemcpyAsync(ctx->loss_tab, ctx->loss_host, sizeof(LossView) * n_views, hipMemcpyHostToDevice,
                              stream));
  HIP_TRY(ctx, hipEventRecord(ctx->loss_copied, stream));
  const LossConsts k = loss_consts(ssim_lambda, n_views);
  launch_loss(ctx->loss_tab, k, feat_dim, nb, nd, ctx->loss_part, ctx->loss_part + nb, stream);
  if (terms) launch_loss_terms(ctx->loss_tab, n_views, k.ssim, ctx->loss_part, ctx->loss_part + nb, terms, stream);
  HIP_TRY(ctx, hipGetLastError());
  return LGS_OK;
}

// Validation and launch arguments shared by the decoder entry points: views
// v < n_views of width[v] x height[v] pixels, with their planes feat[v],
// target[v], grad_feat[v].
static lgs_status decoder_args(lgs_context* ctx, int32_t n_views, const int32_t* width, const int32_t* height,
                               int32_t out_dim, const float* const* feat, const float* weight, const float* bias,
                               const void* const* target, lgs_dtype target_dtype, float w_feat,
                               float* const* grad_feat, float* grad_weight, float* grad_bias, float* loss,
                               DecArgs* a) {
  if (n_views < 1 || n_views > kDecMaxViews)
    return fail(ctx, n_views < 1 ? LGS_ERR_INVALID_ARG : LGS_ERR_UNSUPPORTED,
                "n_views must be 1 .. " + std::to_string(kDecMaxViews));
  if (!width || !height || !feat || !target || !grad_feat) return fail(ctx, LGS_ERR_INVALID_ARG, "NULL view array");
  if (!decoder_dim_ok(out_dim)) return fail(ctx, LGS_ERR_UNSUPPORTED, "out_dim must be 256 or 512");
  if (target_dtype != LGS_F32 && target_dtype != LGS_BF16)
    return fail(ctx, LGS_ERR_INVALID_ARG, "unknown target dtype");
  if (!isfinite(w_feat)) return fail(ctx, LGS_ERR_INVALID_ARG, "non-finite w_feat");
  if (!weight || !bias || !grad_weight || !grad_bias) return fail(ctx, LGS_ERR_INVALID_ARG, "NULL array");
  if (!aligned4(weight) || !aligned4(bias) || !aligned4(grad_weight) || !aligned4(grad_bias) ||
      (loss && !aligned4(loss)))
    return fail(ctx, LGS_ERR_INVALID_ARG, "misaligned array");
  memset(a, 0, sizeof *a);
  a->weight = weight; a->bias = bias;
  a->grad_weight = grad_weight; a->grad_bias = grad_bias; a->loss = loss;
  a->part_stride = ((17 * (int64_t)out_dim + 1 + 63) / 64) * 64;
  a->C = out_dim;
  a->n_views = n_views;
  for (int v = 0; v < n_views; ++v) {
    if (width[v] < 1 || height[v] < 1) return fail(ctx, LGS_ERR_INVALID_ARG, "width and height must be >= 1");
    const int64_t n = (int64_t)width[v] * height[v];
    if (n > ((int64_t)1 << 31)) return fail(ctx, LGS_ERR_UNSUPPORTED, "more than 2^31 pixels");
    if (!feat[v] || !target[v] || !grad_feat[v]) return fail(ctx, LGS_ERR_INVALID_ARG, "NULL array");
    if (!aligned4(feat[v]) || !aligned4(grad_feat[v]) ||
        ((uintptr_t)target[v] & (target_dtype == LGS_BF16 ? 1u : 3u)) != 0)
      return fail(ctx, LGS_ERR_INVALID_ARG, "misaligned array");
    DecView& d = a->v[v];
    d.feat = feat[v];
    d.target = target[v];
    d.grad_feat = grad_feat[v];
    d.n = n;
    d.scale = (float)((double)w_feat / ((double)out_dim * (double)n));
  }
  return LGS_OK;
}

// The allocating entry points: partial sums in the context's buffer, grown
// when a call needs more.
static lgs_status decoder_run(lgs_context* ctx, DecArgs& a, lgs_dtype target_dtype, hipStream_t stream) {
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  const int grid = decoder_assign(a, INT32_MAX);
  const int64_t need = (int64_t)grid * a.part_stride;
  if (need > ctx->dec_part_cap) {
    HIP_TRY(ctx, hipDeviceSynchronize());   // earlier calls may still use the old buffer
    if (ctx->dec_part) hipFree(ctx->dec_part);
    ctx->dec_part = nullptr;
    ctx->dec_part_cap = 0;
    HIP_TRY(ctx, hipMalloc((void**)&ctx->dec_part, sizeof(float) * need));
    ctx->dec_part_cap = need;
  }
  launch_decoder(a, target_dtype == LGS_BF16, ctx->dec_part, grid, stream);
  HIP_TRY(ctx, hipGetLastError());
  return LGS_OK;
}

lgs_status lgs_decoder_l1(lgs_context* ctx, int32_t width, int32_t height, int32_t out_dim, const float* feat,
                          const float* weight, const float* bias, const void* target, lgs_dtype target_dtype,
                          float w_feat, float* grad_feat, float* grad_weight, float* grad_bias, float* loss,
                          hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  DecArgs a;
  lgs_status rc = decoder_args(ctx, 1, &width, &height, out_dim, &feat, weight, bias, &target, target_dtype,
                               w_feat, &grad_feat, grad_weight, grad_bias, loss, &a);
  if (rc != LGS_OK) return rc;
  return decoder_run(ctx, a, target_dtype, stream);
}

lgs_status lgs_decoder_l1_views(lgs_context* ctx, int32_t n_views, const int32_t* width, const int32_t* height,
                                int32_t out_dim, const float* const* feat, const float* weight, const float* bias,
                                const void* const* target, lgs_dtype target_dtype, float w_feat,
                                float* const* grad_feat, float* grad_weight, float* grad_bias, float* loss,
                                hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  DecArgs a;
  lgs_status rc = decoder_args(ctx, n_views, width, height, out_dim, feat, weight, bias, target, target_dtype,
                               w_feat, grad_feat, grad_weight, grad_bias, loss, &a);
  if (rc != LGS_OK) return rc;
  return decoder_run(ctx, a, target_dtype, stream);
}

lgs_status lgs_decoder_l1_noalloc(lgs_context* ctx, int32_t width, int32_t height, int32_t out_dim,
                                  const float* feat, const float* weight, const float* bias, const void* target,
                                  lgs_dtype target_dtype, float w_feat, float* grad_feat, float* grad_weight,
                                  float* grad_bias, float* loss, hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  DecArgs a;
  lgs_status rc = decoder_args(ctx, 1, &width, &height, out_dim, &feat, weight, bias, &target, target_dtype,
                               w_feat, &grad_feat, grad_weight, grad_bias, loss, &a);
  if (rc != LGS_OK) return rc;
  if (!ctx->scratch) return fail(ctx, LGS_ERR_STATE, "no scratch address for this context's device");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  const int grid = decoder_assign(a, kScratchGroups);   // one view: at most kScratchGroups
  const int64_t need = (int64_t)grid * a.part_stride;
  if (need > kScratchFloats)
    return fail(ctx, LGS_ERR_CAPACITY, "decoder partial sums need " + std::to_string(need) +
                                           " floats, more than the fixed scratch array's " +
                                           std::to_string(kScratchFloats));
  // every work-group writes its whole partial row before the reduction
  // reads it, so nothing left by an earlier call needs clearing
  launch_decoder(a, target_dtype == LGS_BF16, ctx->scratch, grid, stream);
  HIP_TRY(ctx, hipGetLastError());
  return LGS_OK;
}

lgs_prune_params lgs_default_prune_params(void) {
  lgs_prune_params p;
  p.k = 16;
  p.tau_dist = 0.02f;
  p.tau_sim = 0.9f;
  p.min_opacity = 0.005f;
  p.max_scale = 0.3f;
  return p;
}

lgs_status lgs_prune(lgs_context* ctx, const lgs_gaussians* g, const lgs_prune_params* prm, uint8_t* mask,
                     int64_t counts[3], hipStream_t stream) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  lgs_status rc;
  if ((rc = check_gaussians(ctx, g)) != LGS_OK) return rc;
  if (!prm) return fail(ctx, LGS_ERR_INVALID_ARG, "params is NULL");
  if (prm->k < 1 || prm->k > prune_k_max()) return fail(ctx, LGS_ERR_INVALID_ARG, "k must be in [1, 32]");
  if (!(prm->tau_dist > 0.f) || !isfinite(prm->tau_dist) || !isfinite(prm->tau_sim) ||
      !(prm->min_opacity > 0.f && prm->min_opacity < 1.f) || !(prm->max_scale > 0.f))
    return fail(ctx, LGS_ERR_INVALID_ARG, "pruning thresholds out of range");
  if (g->n > 0 && !mask) return fail(ctx, LGS_ERR_INVALID_ARG, "mask is NULL");
  if (counts) counts[0] = counts[1] = counts[2] = 0;
  if (g->n == 0) return LGS_OK;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  const int64_t n = g->n;
  std::vector<void*> held;
  auto take = [&](size_t bytes) {
    void* p = pool_alloc(ctx, bytes, stream);
    if (p) held.push_back(p);
    return p;
  };
  auto release = [&]() {
    for (void* p : held) pool_free(ctx, p, SharedEvent());   // the call has synchronised
  };
  const int bf16 = g->appearance_dtype == LGS_BF16;
  const uint32_t buckets = prune_buckets(n);
  PruneWork w;
  w.rec = take(prune_rec_bytes(bf16) * n);
  w.pos = (float4*)take(sizeof(float4) * n);
  w.count = (uint32_t*)take(4 * (size_t)buckets);
  w.start = (uint32_t*)take(4 * ((size_t)buckets + 1));
  w.list = (uint32_t*)take(4 * n);
  w.geo = (uint8_t*)take(n);
  w.sem = (uint8_t*)take(n);
  w.temp = take(scan_temp_bytes(buckets));
  w.pc = (PruneCounters*)take(sizeof(PruneCounters));
  if (held.size() != 9) {
    release();
    return fail(ctx, LGS_ERR_HIP, "device allocation failed (pruning)");
  }
  PruneArgs a;
  a.means = g->means; a.logits = g->opacity_logits; a.log_scales = g->log_scales; a.feat = g->feat;
  a.feat_bf16 = bf16;
  a.planes = g->feat_dim == 8 ? 8 : 16;
  a.k = prm->k;
  a.buckets = buckets;
  a.n = n;
  const double tau = (double)prm->tau_dist;
  a.tau2 = tau * tau;
  // FP32: the differences and the three squares' sum round by less than 2^-20
  // of the result, or by a few of the least denormals
  a.tau2_above = a.tau2 < 1e38 ? (float)(a.tau2 * (1.0 + 1.0 / (1 << 20)) + 1e-37) : INFINITY;
  a.inv_cell = 1.0 / tau;
  a.tau_sim = (double)prm->tau_sim;
  a.logit_min = log((double)prm->min_opacity / (1.0 - (double)prm->min_opacity));
  a.log_scale_max = log((double)prm->max_scale);
  auto run = [&]() -> lgs_status {
    if (!ctx->prune_host)
      HIP_TRY(ctx, hipHostMalloc((void**)&ctx->prune_host, sizeof(PruneCounters), hipHostMallocDefault));
    launch_prune(a, w, mask, stream);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipMemcpyAsync(ctx->prune_host, w.pc, sizeof(PruneCounters), hipMemcpyDeviceToHost, stream));
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    const PruneCounters hc = *ctx->prune_host;
    if (hc.range_err)
      return fail(ctx, LGS_ERR_UNSUPPORTED, "a mean lies more than 2^20 cells of tau_dist from the origin");
    if (counts)
      for (int i = 0; i < 3; ++i) counts[i] = (int64_t)hc.counts[i];
    return LGS_OK;
  };
  rc = run();
  if (rc != LGS_OK) hipStreamSynchronize(stream);   // queued work may still use the buffers
  release();
  return rc;
}

// ---------------------------------------------------------------------------
// whole-step graph
// ---------------------------------------------------------------------------
lgs_status lgs_graph_create(lgs_context* ctx, const lgs_settings* st, const lgs_gaussians* g, int32_t n_views,
                            const lgs_camera* cams, const lgs_images* targets, const float loss_w[3],
                            float ssim_lambda, const lgs_images* out, const lgs_grads* grads,
                            int64_t pair_capacity, hipStream_t stream, lgs_graph** graph_out) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  if (!graph_out) return fail(ctx, LGS_ERR_INVALID_ARG, "graph_out is NULL");
  *graph_out = nullptr;
  lgs_status rc;
  if ((rc = check_settings(ctx, st)) != LGS_OK) return rc;
  if ((rc = check_gaussians(ctx, g)) != LGS_OK) return rc;
  if ((rc = check_cams(ctx, n_views, cams)) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, out, true, "out")) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, targets, false, "targets")) != LGS_OK) return rc;
  if ((rc = check_loss_args(ctx, loss_w, ssim_lambda)) != LGS_OK) return rc;
  if ((rc = check_grads(ctx, g, grads)) != LGS_OK) return rc;
  if (pair_capacity < 0) return fail(ctx, LGS_ERR_INVALID_ARG, "pair_capacity < 0");
  if (!kGraphEnabled) return fail(ctx, LGS_ERR_UNSUPPORTED, "graph mode is switched off in this build");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  // measure the workload once (eager) to size the pair and slot buffers
  lgs_fwd_state* probe = nullptr;
  if ((rc = lgs_forward(ctx, st, g, n_views, cams, out, &probe, stream)) != LGS_OK) return rc;
  const lgs_counts pc = probe->W.counts;
  lgs_state_release(ctx, probe);
  int64_t capP, capS;
  const double sp = pc.n_pairs > 0 ? (double)pc.n_slots / (double)pc.n_pairs : 1.0;
  if (pair_capacity > 0) {
    capP = pair_capacity;
    capS = (int64_t)ceil((double)pair_capacity * std::max(1.0, sp) * 1.25) + 4096;
  } else {
    capP = (int64_t)ceil(1.5 * (double)pc.n_pairs) + 4096;
    capS = (int64_t)ceil(1.5 * (double)pc.n_slots) + 4096;
  }
  if (capP > 0xFFFFFFFFll || capS > 0xFFFFFFFFll) return fail(ctx, LGS_ERR_UNSUPPORTED, "capacity exceeds 2^32");
  lgs_graph* G = new lgs_graph();
  Work* W = &G->W;
  G->g = *g;
  G->grads = *grads;
  auto bail = [&](lgs_status e) {
    if (G->exec) hipGraphExecDestroy(G->exec);
    if (G->graph) hipGraphDestroy(G->graph);
    for (int i = 0; i < 5; ++i) {
      if (G->sexec[i]) hipGraphExecDestroy(G->sexec[i]);
      if (G->sgraph[i]) hipGraphDestroy(G->sgraph[i]);
    }
    if (G->cap_stream) hipStreamDestroy(G->cap_stream);
    for (int i = 0; i < 6; ++i)
      if (G->ev[i]) hipEventDestroy(G->ev[i]);
    w_release(W);
    delete G;
    return e;
  };
  if ((rc = w_init(W, ctx, st, g, n_views, cams, stream)) != LGS_OK) return bail(rc);
  if ((rc = w_alloc_front(W)) != LGS_OK) return bail(rc);
  if ((rc = w_alloc_pairs(W, capP, capS)) != LGS_OK) return bail(rc);
  if ((rc = w_alloc_bwd(W)) != LGS_OK) return bail(rc);
  // (cleared now: the captured step must not clear it on each launch)
  launch_fill_u32((uint32_t*)W->mask, 0u, W->mask_words, stream);
  W->mask_words = 0;
  if ((rc = w_upload(W, out, stream)) != LGS_OK) return bail(rc);
  {
    const std::vector<ViewImages> ho = group_tables(W, out, TAB_FO), ht = group_tables(W, targets, TAB_TGT);
    const std::vector<float> lw = group_lossw(W, loss_w);
    if (upload_tables(W, {table(W->d_fo, ho), table(W->d_tgt, ht), table(W->d_lossw, lw)}, stream) != hipSuccess)
      return bail(fail(ctx, LGS_ERR_HIP, "upload failed"));
  }
  if (ssim_lambda != 0.f) {
    // the loss kernel writes the colour part of dL/dY (L1 + D-SSIM) into
    // graph-owned planes [3][H][W] per view; the backward reads them and
    // forms the depth and feature L1 gradients itself
    bool ok = true;
    W->up_buf = (float*)w_alloc(W, sizeof(float) * 3 * std::max<int64_t>(W->plan.n_pix, 1), ok);
    W->loss_tab = (LossView*)w_alloc(W, sizeof(LossView) * n_views, ok);
    std::vector<lgs_images> gi(n_views);
    for (int v = 0; v < n_views; ++v) {
      float* base = W->up_buf + 3 * (int64_t)W->plan.views[v].pix_off;
      gi[v] = lgs_images{base, nullptr, nullptr, nullptr, nullptr};
    }
    if ((rc = w_zero_img(W)) != LGS_OK) return bail(rc);
    const std::vector<ViewImages> hu = group_tables(W, gi.data(), TAB_UP_RGB);
    std::vector<LossView> lv(n_views);
    int64_t n_df = 0;
    W->loss_blocks = make_loss_views(n_views, cams, W->D, out, targets, gi.data(), loss_w, ssim_lambda,
                                     lv.data(), &n_df);
    W->loss_part = (float2*)w_alloc(W, sizeof(float2) * std::max<int64_t>(W->loss_blocks, 1), ok);
    W->loss_k = loss_consts(ssim_lambda, n_views);
    if (!ok) return bail(fail(ctx, LGS_ERR_HIP, "device allocation failed (loss)"));
    if (upload_tables(W, {table(W->loss_tab, lv)}, stream) != hipSuccess ||
        upload_tables(W, {table(W->d_up, hu)}, stream) != hipSuccess)
      return bail(fail(ctx, LGS_ERR_HIP, "upload failed"));
  }
  if (hipStreamCreateWithFlags(&G->cap_stream, hipStreamNonBlocking) != hipSuccess)
    return bail(fail(ctx, LGS_ERR_HIP, "stream creation failed"));
  G->profile = (st->profile & LGS_PROFILE_EVENTS) != 0;
  if (G->profile)
    for (int i = 0; i < 6; ++i)
      if (hipEventCreate(&G->ev[i]) != hipSuccess) return bail(fail(ctx, LGS_ERR_HIP, "event creation failed"));
  auto stage = [&](int i) {
    switch (i) {
      case 0: enqueue_front(W, &G->g, G->cap_stream); break;
      case 1: enqueue_pairs(W, G->cap_stream); break;
      case 2: enqueue_raster_fwd(W, G->cap_stream); break;
      case 3:
        if (W->loss_tab) {
          // the colour gradient (L1 + D-SSIM) into up_buf; depth and feature
          // L1 gradients are formed inside the backward
          launch_loss_rgb(W->loss_tab, W->loss_k, W->loss_blocks, W->loss_part, G->cap_stream);
          enqueue_backward_raster(W, &G->grads, UP_RGB, G->cap_stream);
        } else {
          enqueue_backward_raster(W, &G->grads, UP_L1, G->cap_stream);
        }
        break;
      default: enqueue_backward_reduce(W, &G->g, &G->grads, G->cap_stream); break;
    }
  };
  auto capture = [&](int first, int last, hipGraph_t* gr, hipGraphExec_t* ex) -> lgs_status {
    if (hipStreamBeginCapture(G->cap_stream, hipStreamCaptureModeRelaxed) != hipSuccess)
      return fail(ctx, LGS_ERR_HIP, "hipStreamBeginCapture failed");
    for (int i = first; i <= last; ++i) stage(i);
    hipError_t e = hipStreamEndCapture(G->cap_stream, gr);
    if (e != hipSuccess) return fail(ctx, LGS_ERR_HIP, std::string("capture failed: ") + hipGetErrorString(e));
    e = hipGraphInstantiate(ex, *gr, nullptr, nullptr, 0);
    if (e != hipSuccess) return fail(ctx, LGS_ERR_HIP, std::string("instantiate failed: ") + hipGetErrorString(e));
    return LGS_OK;
  };
  if (G->profile) {
    for (int i = 0; i < 5; ++i)
      if ((rc = capture(i, i, &G->sgraph[i], &G->sexec[i])) != LGS_OK) return bail(rc);
  } else if ((rc = capture(0, 4, &G->graph, &G->exec)) != LGS_OK) {
    return bail(rc);
  }
  // the table uploads and the waits for reused blocks were enqueued on
  // `stream`; the graph may later be launched on any stream, so creation
  // ends once they have run
  if (hipStreamSynchronize(stream) != hipSuccess) return bail(fail(ctx, LGS_ERR_HIP, "stream synchronisation failed"));
  W->counts = pc;
  *graph_out = G;
  return LGS_OK;
}

lgs_status lgs_graph_launch(lgs_graph* G, hipStream_t stream) {
  if (!G) return LGS_ERR_INVALID_ARG;
  HIP_TRY(G->W.ctx, hipSetDevice(G->W.ctx->device));
  if (G->profile) {
    for (int i = 0; i < 5; ++i) {
      HIP_TRY(G->W.ctx, hipEventRecord(G->ev[i], stream));
      HIP_TRY(G->W.ctx, hipGraphLaunch(G->sexec[i], stream));
    }
    HIP_TRY(G->W.ctx, hipEventRecord(G->ev[5], stream));
  } else {
    HIP_TRY(G->W.ctx, hipGraphLaunch(G->exec, stream));
  }
  G->last_stream = stream;
  return LGS_OK;
}

lgs_status lgs_graph_status(lgs_graph* G) {
  if (!G) return LGS_ERR_INVALID_ARG;
  HIP_TRY(G->W.ctx, hipSetDevice(G->W.ctx->device));
  Counters hc;
  lgs_status rc = read_counts(&G->W, G->last_stream, &hc);
  if (rc != LGS_OK) return rc;
  if (hc.overflow) return fail(G->W.ctx, LGS_ERR_CAPACITY, "pair or slot capacity exceeded; re-create the graph");
  return LGS_OK;
}

lgs_status lgs_graph_counts(lgs_graph* G, lgs_counts* out) {
  if (!G || !out) return LGS_ERR_INVALID_ARG;
  HIP_TRY(G->W.ctx, hipSetDevice(G->W.ctx->device));
  Counters hc;
  lgs_status rc = read_counts(&G->W, G->last_stream, &hc);
  if (rc != LGS_OK) return rc;
  *out = G->W.counts;
  return LGS_OK;
}

lgs_status lgs_graph_stage_ms(lgs_graph* G, float ms[5]) {
  if (!G || !ms) return LGS_ERR_INVALID_ARG;
  if (!G->profile) return fail(G->W.ctx, LGS_ERR_STATE, "graph was created without settings.profile");
  HIP_TRY(G->W.ctx, hipSetDevice(G->W.ctx->device));
  HIP_TRY(G->W.ctx, hipEventSynchronize(G->ev[5]));
  for (int i = 0; i < 5; ++i) HIP_TRY(G->W.ctx, hipEventElapsedTime(&ms[i], G->ev[i], G->ev[i + 1]));
  return LGS_OK;
}

void lgs_graph_destroy(lgs_graph* G) {
  if (!G) return;
  hipSetDevice(G->W.ctx->device);
  hipDeviceSynchronize();
  if (G->exec) hipGraphExecDestroy(G->exec);
  if (G->graph) hipGraphDestroy(G->graph);
  for (int i = 0; i < 5; ++i) {
    if (G->sexec[i]) hipGraphExecDestroy(G->sexec[i]);
    if (G->sgraph[i]) hipGraphDestroy(G->sgraph[i]);
  }
  if (G->cap_stream) hipStreamDestroy(G->cap_stream);
  for (int i = 0; i < 6; ++i)
    if (G->ev[i]) hipEventDestroy(G->ev[i]);
  w_release(&G->W);
  delete G;
}

// ---------------------------------------------------------------------------
// autotuner
// ---------------------------------------------------------------------------
// Cache key: everything that changes which setting is fastest (Gaussian
// count, appearance storage, feature dimension, the step's loss form, the
// views' sizes).
static std::string tune_key(const lgs_gaussians* g, int32_t n_views, const lgs_camera* cams) {
  char buf[128];
  snprintf(buf, sizeof buf, "n%lld_%s_d%d_l1_v%d", (long long)g->n,
           g->appearance_dtype == LGS_BF16 ? "bf16" : "f32", feat_dim_of(g), n_views);
  std::string k = buf;
  for (int v = 0; v < n_views; ++v) {
    snprintf(buf, sizeof buf, "_%dx%d", cams[v].width, cams[v].height);
    k += buf;
  }
  return k;
}

static bool tune_cache_read(const char* path, const std::string& key, lgs_settings* s) {
  FILE* f = fopen(path, "r");
  if (!f) return false;
  char line[1024];
  bool found = false;
  while (fgets(line, sizeof line, f)) {
    char k[900];
    int tile, chunk, order;
    if (sscanf(line, " \"%899[^\"]\": {\"tile\": %d, \"chunk\": %d, \"order\": %d}", k, &tile, &chunk, &order) == 4 &&
        key == k) {
      s->tile = tile; s->chunk = chunk; s->order = order;
      found = true;
    }
  }
  fclose(f);
  return found;
}

static void tune_cache_write(const char* path, const std::string& key, const lgs_settings& s) {
  std::vector<std::string> lines;
  if (FILE* f = fopen(path, "r")) {
    char line[1024];
    while (fgets(line, sizeof line, f)) {
      char k[900];
      std::string L(line);
      if (sscanf(line, " \"%899[^\"]\":", k) == 1 && key != k) {
        while (!L.empty() && (L.back() == '\n' || L.back() == ',')) L.pop_back();
        lines.push_back(L);
      }
    }
    fclose(f);
  }
  char buf[1024];
  snprintf(buf, sizeof buf, "  \"%s\": {\"tile\": %d, \"chunk\": %d, \"order\": %d}", key.c_str(), s.tile,
           s.chunk, s.order);
  lines.push_back(buf);
  FILE* f = fopen(path, "w");
  if (!f) return;
  fprintf(f, "{\n");
  for (size_t i = 0; i < lines.size(); ++i) fprintf(f, "%s%s\n", lines[i].c_str(), i + 1 < lines.size() ? "," : "");
  fprintf(f, "}\n");
  fclose(f);
}

lgs_status lgs_autotune(lgs_context* ctx, const lgs_settings* st, const lgs_gaussians* g, int32_t n_views,
                        const lgs_camera* cams, const lgs_images* targets, const float loss_w[3],
                        const lgs_images* out, const lgs_grads* grads, int64_t pair_capacity, hipStream_t stream,
                        const char* cache_path, lgs_settings* best_out) {
  if (!ctx) return LGS_ERR_INVALID_ARG;
  ctx->err.clear();
  if (!best_out) return fail(ctx, LGS_ERR_INVALID_ARG, "best_out is NULL");
  lgs_status rc;
  if ((rc = check_settings(ctx, st)) != LGS_OK) return rc;
  if ((rc = check_gaussians(ctx, g)) != LGS_OK) return rc;
  if ((rc = check_cams(ctx, n_views, cams)) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, out, true, "out")) != LGS_OK) return rc;
  if ((rc = check_images(ctx, n_views, targets, false, "targets")) != LGS_OK) return rc;
  if ((rc = check_grads(ctx, g, grads)) != LGS_OK) return rc;
  if (!loss_w) return fail(ctx, LGS_ERR_INVALID_ARG, "loss_w is NULL");
  const std::string key = tune_key(g, n_views, cams);
  *best_out = *st;
  if (cache_path && tune_cache_read(cache_path, key, best_out)) return LGS_OK;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  (void)hipGetLastError();   // launch checks below see only this call's errors
  // Each candidate is timed as it will run: the whole step captured as one
  // graph (lgs_graph_create), two warm-up launches, then the median of 7
  // launches measured by HIP events on the stream (device time only: no
  // allocation, readback or host work inside).  Candidates are visited in a
  // fixed order, and a later one replaces the best only when it is faster
  // by more than 1 %, so that settings within run-to-run noise of each other
  // resolve to the same choice.
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIP_TRY(ctx, hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) {
    hipEventDestroy(e0);
    return fail(ctx, LGS_ERR_HIP, "event creation failed");
  }
  double best_ms = 1e30;
  const int tiles[3] = {32, 16, 8}, orders[3] = {2, 1, 0}, chunks[3] = {4, 2, 1};
  for (int ti = 0; ti < 3; ++ti)
    for (int oi = 0; oi < 3; ++oi)
      for (int ci = 0; ci < 3; ++ci) {
        lgs_settings s = *st;
        s.tile = tiles[ti]; s.chunk = chunks[ci]; s.order = orders[oi]; s.profile = 0;
        lgs_graph* G = nullptr;
        if (lgs_graph_create(ctx, &s, g, n_views, cams, targets, loss_w, 0.f, out, grads, pair_capacity, stream,
                             &G) != LGS_OK)
          continue;
        std::vector<float> t;
        bool ok = true;
        for (int r = 0; r < 9 && ok; ++r) {
          ok = hipEventRecord(e0, stream) == hipSuccess && lgs_graph_launch(G, stream) == LGS_OK &&
               hipEventRecord(e1, stream) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
          float ms = 0.f;
          if (ok && r >= 2) ok = hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
          if (ok && r >= 2) t.push_back(ms);
        }
        if (ok) ok = lgs_graph_status(G) == LGS_OK;
        lgs_graph_destroy(G);
        if (!ok) continue;
        std::sort(t.begin(), t.end());
        const double ms = t[t.size() / 2];
        if (ms < best_ms * 0.99) {
          best_ms = ms;
          *best_out = s;
        }
      }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  ctx->err.clear();
  if (best_ms >= 1e29) return fail(ctx, LGS_ERR_HIP, "no setting ran");
  best_out->profile = st->profile;
  if (cache_path) tune_cache_write(cache_path, key, *best_out);
  return LGS_OK;
}

}  // extern "C"
