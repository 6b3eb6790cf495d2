// Host-side test of the workspace pool where device memory is short: this
// translation unit includes the runtime source with the allocation, event and
// stream calls replaced by a model of a card (so much memory, and blocks of at
// most so much), and exports one entry point that the CPU test calls through
// ctypes.  No HIP runtime call is made.
#include <hip/hip_runtime.h>

#include <stdlib.h>

#include <map>

namespace card {
size_t free_bytes = 0, largest = 0, used = 0;
std::map<void*, size_t> blocks;
hipError_t last = hipSuccess;
void set(size_t bytes, size_t block = ~(size_t)0) { free_bytes = bytes, largest = block; }
hipError_t alloc(void** p, size_t n) {
  if (n > free_bytes || n > largest) return last = hipErrorOutOfMemory;
  // (addresses only: nothing is read or written behind them)
  static uintptr_t at = (uintptr_t)1 << 40;
  *p = (void*)at;
  at += (n + 4095) / 4096 * 4096;
  blocks[*p] = n;
  free_bytes -= n;
  used += n;
  return hipSuccess;
}
hipError_t release(void* p) {
  auto it = blocks.find(p);
  if (it == blocks.end()) return last = hipErrorInvalidValue;
  free_bytes += it->second;
  used -= it->second;
  blocks.erase(it);
  return hipSuccess;
}
hipError_t take_last() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t event(hipEvent_t* e) {
  static uintptr_t at = 1;
  *e = (hipEvent_t)at++;
  return hipSuccess;
}
}  // namespace card

#define hipMalloc(p, n) card::alloc((void**)(p), n)
#define hipFree(p) card::release(p)
#define hipMemcpy(d, s, n, k) hipSuccess
#define hipGetLastError() card::take_last()
#define hipEventCreateWithFlags(e, f) card::event(e)
#define hipEventDestroy(e) hipSuccess
#define hipEventRecord(e, s) hipSuccess
#define hipEventSynchronize(e) hipSuccess
#define hipEventQuery(e) hipSuccess
#define hipStreamWaitEvent(s, e, f) hipSuccess
#define hipStreamSynchronize(s) hipSuccess
#include "../../paper_2511_16144_amd/csrc/runtime.hip"

namespace {

int g_fail = 0;
#define CHECK(cond)                                                              \
  do {                                                                           \
    if (!(cond)) {                                                               \
      fprintf(stderr, "pool_host_test: %s:%d: %s\n", __FILE__, __LINE__, #cond); \
      ++g_fail;                                                                  \
    }                                                                            \
  } while (0)

constexpr size_t MB = 1u << 20;

void drop(lgs_context* ctx) {   // as lgs_context_destroy, for the next scenario
  for (auto& kv : ctx->free_blocks) hipFree(kv.second.p);
  for (auto& kv : ctx->live) hipFree(kv.first);
  for (auto& kv : ctx->items_cache) hipFree(kv.second.first);
  CHECK(card::used == 0);
}

// a block that fits as asked for, but not rounded up
void unrounded() {
  lgs_context ctx;
  card::set(6 * MB);
  void* p = pool_alloc(&ctx, 5 * MB, nullptr);
  CHECK(p && card::used >= 5 * MB && ctx.live[p] == card::used);
  CHECK(hipGetLastError() == hipSuccess);
  CHECK(!pool_alloc(&ctx, 5 * MB, nullptr));
  drop(&ctx);
  card::set(100 * MB);   // (with room to spare it is rounded)
  lgs_context roomy;
  CHECK(pool_alloc(&roomy, 5 * MB, nullptr) && card::used == 17 * MB);
  drop(&roomy);
}

// a request that fits once the cache is dropped leaves no error behind
void after_the_cache() {
  lgs_context ctx;
  card::set(100 * MB);
  void* p = pool_alloc(&ctx, 60 * MB, nullptr);
  pool_free(&ctx, p, SharedEvent());
  CHECK(pool_alloc(&ctx, 90 * MB, nullptr) != nullptr);
  CHECK(hipGetLastError() == hipSuccess);
  drop(&ctx);
}

lgs_status init(Work* W, lgs_context* ctx, int64_t n, int D) {
  lgs_camera c;
  memset(&c, 0, sizeof c);
  c.width = 320, c.height = 240;
  c.fx = c.fy = 300.f;
  c.R_cw[0] = c.R_cw[4] = c.R_cw[8] = 1.f;
  const std::vector<lgs_camera> cams(3, c);
  lgs_gaussians g;
  memset(&g, 0, sizeof g);
  g.n = n;
  g.feat_dim = D;
  const lgs_settings st = lgs_default_settings();
  return w_init(W, ctx, &st, &g, 3, cams.data(), nullptr);
}

// the stage's buffers where no block holds them all: blocks of their own, the
// tables that are uploaded together still behind one another
void in_parts() {
  for (size_t largest : {~(size_t)0, 7 * MB}) {
    lgs_context ctx;
    Work W;
    card::set(200 * MB);
    CHECK(init(&W, &ctx, 20000, 64) == LGS_OK);
    card::set(200 * MB, largest);
    CHECK(w_alloc_front(&W) == LGS_OK);
    CHECK(W.geom && W.cnt_t && W.app && W.ranges && W.counters && W.ii_a && W.work_q);
    CHECK((char*)W.d_out == (char*)W.d_views + (sizeof(ViewDesc) * 3 + 255) / 256 * 256);
    const size_t im = (sizeof(ViewImages) * 3 * 4 + 255) / 256 * 256;
    CHECK((char*)W.d_tgt == (char*)W.d_fo + im && (char*)W.d_lossw == (char*)W.d_tgt + im);
    CHECK((W.bufs.size() > 1) == (largest != ~(size_t)0));
    CHECK(hipGetLastError() == hipSuccess);
    w_release(&W);
    drop(&ctx);
  }
  // and where the parts do not fit either: an error, and every block back in the cache
  lgs_context ctx;
  Work W;
  card::set(200 * MB);
  CHECK(init(&W, &ctx, 20000, 16) == LGS_OK);
  card::set(4 * MB);
  CHECK(w_alloc_front(&W) != LGS_OK);
  CHECK(!W.geom && W.bufs.empty() && ctx.live.empty());
  drop(&ctx);
}

// feature groups side by side only as far as memory goes
void fewer_groups() {
  size_t one = 0;
  for (int left : {4, 2, 1, 0}) {
    lgs_context ctx;
    Work W;
    card::set(4000 * MB);
    CHECK(init(&W, &ctx, 20000, 64) == LGS_OK);
    CHECK(w_alloc_front(&W) == LGS_OK);
    CHECK(w_alloc_pairs(&W, 100000, 400000) == LGS_OK);
    const int64_t per = 4 * (400000ll * kSlotFloats + W.n_rid * kPartials);
    if (left < 4) card::set((size_t)(per * left + (left ? per / 2 + (int64_t)one : 0)));
    const size_t before = card::used;
    const lgs_status rc = w_alloc_bwd(&W);
    if (left == 4) one = (card::used - before) - (size_t)(per * 4);   // what does not depend on the groups
    CHECK((rc == LGS_OK) == (left > 0));
    if (left > 0) {
      CHECK(W.gb == left && W.bwd_alloc && W.partials && W.mask && W.grad2d && W.ttmp);
      CHECK((W.geo_acc != nullptr) == (left < 4));
      CHECK(W.mask_words == W.mask_stride * left / 4);
      CHECK(hipGetLastError() == hipSuccess);
    } else {
      CHECK(!W.bwd_alloc && !W.partials && !W.ttmp);
    }
    w_release(&W);
    drop(&ctx);
  }
}

}  // namespace

extern "C" int lgs_pool_selftest() {
  g_fail = 0;
  unrounded();
  after_the_cache();
  in_parts();
  fewer_groups();
  return g_fail;
}
