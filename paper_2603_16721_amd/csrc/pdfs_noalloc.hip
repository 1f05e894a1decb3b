// Allocation-free variant of pdfs_best_combo (one argmax round, Alg. 1 step 4
// done as Alg. 2) for callers that cannot allocate device memory: code under
// HIP graph capture, tight serving loops, harnesses that forbid hipMalloc.
//
// Every per-round buffer the round's kernels use (uncovered-sample list,
// active list, re-packed rows, unpacked bytes for the pair table, pair and
// work lists, work items, argmax slots, counter rows, round state, round
// record) is carved from one file-scope device array, `scratch`, instead of
// the context's own lazily allocated workspace.  The cohort itself (sorted
// rows, permutation, uncovered mask) is the context's, made by pdfs_create.
//
// The array's device address is taken once per device with
// hipGetSymbolAddress when a context is first created there (the device is
// current then), and only that address is passed to kernels and fill
// launches.  Every call on a device shares that device's array and leaves its
// contents behind; a call clears what must start at zero (round state, slots,
// counter rows) itself.  Calls that overlap on one device race.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>

#include "../../include/pdfs.h"
#include "pdfs_dev.h"
#include "pdfs_host.h"

namespace pdfs {

namespace {

// Size of the static scratch array: held on every device the library sets up
// a context on, until the process ends.
#ifndef PDFS_NOALLOC_SCRATCH_MIB
#define PDFS_NOALLOC_SCRATCH_MIB 64
#endif
constexpr size_t kScratchBytes = (size_t)PDFS_NOALLOC_SCRATCH_MIB << 20;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};
hipError_t g_scratch_rc[kMaxDevices] = {};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The lazy round's small buffers, each on a 256-byte boundary.
size_t lazy_small(LazyWork& W, unsigned char* at, int n_tumor) {
  size_t o = 0;
  auto put = [&](auto** p, size_t n) {
    *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(at + o);
    o = align256(o + n * sizeof(**p));
  };
  put(&W.Uc, kMaxW64);
  put(&W.cursor, kMaxCount + 1);
  put(&W.pool, kLazyWaves);
  put(&W.wins, 3 * (kLazyWaves / 4));
  put(&W.n_win, 3 * 64);
  put(&W.inc, 2 * kCursorStride);
  put(&W.S, 2);
  put(&W.U2, 2 * kMaxW64);
  put(&W.tcov, 64 * kMaxW64);
  put(&W.uncs, (size_t)n_tumor + 2);
  put(&W.shard, 2 * kIncShards * kCursorStride);
  return o;
}

const size_t kLazyBytes = [] {
  LazyWork W;
  return lazy_small(W, reinterpret_cast<unsigned char*>((uintptr_t)256), 64 * kMaxW64);
}();

// Byte offsets of the round workspace inside the scratch array.
struct Layout {
  size_t st, recs, slots, tallies, zero_end;   // [st, zero_end) is cleared per call
  size_t cols, act, flags, TA, NA, A8, N8, hist, cursors, seed, pairs, work, items;
  size_t B, bits, list, cmax, lazy;   // lazy round
  int nw = 0, seg = 0, gw = 0;
  size_t total;
  unsigned long long pair_cap = 0, item_cap = 0;
};

// Every pair of nA rows.
unsigned long long all_pairs(int nA) {
  return (unsigned long long)nA * (nA > 0 ? nA - 1 : 0) / 2;
}

// Plans the workspace of one round at row width w64max.  The fixed part is
// sized exactly; the pair list and a lazy round's shares, or its bound-mode
// copy and the item list, take what is left, up to every pair.  Returns false
// (with the bytes the fixed part needs) when it does not fit.
bool plan(const pdfs_ctx* c, int h, bool lazy, Layout& L, size_t* need) {
  L = Layout();
  const int nA = c->prune_mode == PDFS_PRUNE_NONE ? c->G : c->nA_max;
  const size_t rows = (size_t)((nA + 127) / 128 * 128 + 128);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = align256(o + bytes);
    return at;
  };
  L.st = take(sizeof(RoundState));
  L.recs = take(sizeof(RoundRecord));
  // (a lazy round has the pair table's counter rows only, and no slots)
  const bool bound = c->prune_mode == PDFS_PRUNE_BOUND;
  L.tallies = take((size_t)(lazy ? 1 : kSlotPhases) * kPersistBlocks * kTallyN * 8);
  L.zero_end = o;
  L.slots = take(lazy ? 0 : (size_t)kSlotPhases * kSlotsPerPhase * sizeof(Slot));
  L.cols = take((size_t)c->n_tumor * 4);
  L.act = take((size_t)c->G * 4);
  L.flags = take((size_t)c->G);
  L.TA = take(rows * 2 * (size_t)c->w64_max * 4);
  L.NA = take(rows * (size_t)kMaxWN32 * 4);
  L.A8 = take(rows * (size_t)unpacked_row_bytes(c->w64_max));
  L.N8 = take(h == 2 ? rows * (size_t)unpacked_row_bytes(c->wn) : 0);
  L.hist = take((size_t)(kMaxCount + 1) * 4);
  L.cursors = take((size_t)kSubQueues * kCursorStride * 8);
  L.seed = take((size_t)kSeedCap * 8);
  size_t nw_max = 0;
  if (lazy) {
    // The transposed rows (8 w64 bytes a gene) and the general walk's bitmaps
    // (nw / 8) lie over the unpacked rows (128 ceil(w64 / 2) a gene), which the
    // pair table is done with: 1024 waves fit from w64 = 3 on, 768 always.
    L.gw = (nA + 63) / 64 > 0 ? (nA + 63) / 64 : 1;
    const size_t nb = align256((size_t)64 * c->w64_max * L.gw * 8);
    const size_t per_wave = (size_t)lazy_levels(h) * L.gw * 8;
    const size_t room = rows * (size_t)unpacked_row_bytes(c->w64_max);
    nw_max = nb + kLazyWaves * per_wave <= room ? kLazyWaves : kLazyWaves / 4 * 3;
    L.B = L.A8;
    L.bits = L.B + nb;
    if (nb + nw_max * per_wave > room) return false;   // (cannot happen, by the sizes above)
    L.lazy = take(kLazyBytes);
  }
  *need = o;
  if (o >= kScratchBytes) return false;
  L.pairs = L.work = L.items = o;
  if (h >= 3) {
    // The rest holds the pair list and, for a lazy round, its waves' shares (8
    // bytes a pair, and a bound per 64); otherwise the bound mode's work copy and
    // the item list: two 16-byte items per 64-pair batch and 2048 spare items.
    const size_t fixed = lazy ? 4 * 256 + (size_t)kLazyWaves * (8 + 4)   // the shares' round-up
                              : (size_t)2048 * sizeof(Item) + 3 * 256;
    const size_t avail = kScratchBytes - o;
    if (avail <= fixed + 64 * 17) return false;
    const double per_pair = lazy ? 16.0 + 4.0 / kWave
                                 : (bound ? 16.0 : 8.0) + 2.0 * sizeof(Item) / kPairBatch;
    unsigned long long cap = (unsigned long long)((double)(avail - fixed) / per_pair);
    cap = std::min(cap, all_pairs(nA));
    if (cap < 64) cap = 64;
    L.pair_cap = cap;
    L.pairs = take(cap * 8);
    if (lazy) {
      L.nw = std::min(lazy_waves(cap), (int)nw_max);
      L.seg = (int)((cap + L.nw - 1) / L.nw);
      const size_t chunks = (size_t)L.nw * ((L.seg + kWave - 1) / kWave);
      L.list = take((size_t)L.nw * L.seg * 8);
      L.cmax = take(chunks * 4);
      L.total = o;
      *need = o;
      return o <= kScratchBytes;
    }
    L.work = bound ? take(cap * 8) : L.pairs;
    L.item_cap = 2 * ((cap + kPairBatch - 1) / kPairBatch) + 2048;
    L.items = take(L.item_cap * sizeof(Item));
  }
  L.total = o;
  *need = o;
  return o <= kScratchBytes;
}

int32_t nfail(pdfs_ctx* c, int32_t code, const std::string& msg) {
  return ctx_fail(c, code, msg);
}

#define NCK(expr)                                                                         \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return nfail(c, PDFS_ERR_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

}  // namespace

void scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (g_scratch_done[device]) return;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  g_scratch_rc[device] = e;
  g_scratch_ptr[device] = e == hipSuccess ? p : nullptr;
  g_scratch_done[device] = true;
}

}  // namespace pdfs

using namespace pdfs;

extern "C" {

int32_t pdfs_best_combo_noalloc(pdfs_ctx* c, int32_t h, uint32_t p, uint32_t q,
                                const uint64_t* uncovered, pdfs_combo* out, pdfs_stats* stats) {
  int32_t rc = check_call(c, h, p, q);
  if (rc != PDFS_OK) return rc;
  if (!out) return nfail(c, PDFS_ERR_INVALID_ARG, "out is NULL");
  if (h > 4) return nfail(c, PDFS_ERR_UNSUPPORTED, "the allocation-free round takes h <= 4");
  unsigned char* base = nullptr;
  {
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (c->device >= 0 && c->device < kMaxDevices && g_scratch_done[c->device]) {
      if (!g_scratch_ptr[c->device])
        return nfail(c, PDFS_ERR_DEVICE,
                     std::string("static scratch address: ") +
                         hipGetErrorString(g_scratch_rc[c->device]));
      base = static_cast<unsigned char*>(g_scratch_ptr[c->device]);
    }
  }
  if (!base) return nfail(c, PDFS_ERR_DEVICE, "static scratch not set up on this device");
  // A bound-pruned round goes out lazily where that is the faster way, and where
  // the walk's lists could not hold every pair beside its work copy.
  Layout L;
  size_t need = 0;
  bool lazy = h >= 3 && c->prune_mode == PDFS_PRUNE_BOUND;
  if (lazy) {
    int n = c->n_tumor;
    if (uncovered) {
      n = 0;
      for (int k = 0; k < c->wt; ++k) n += __builtin_popcountll(uncovered[k]);
    }
    lazy = lazy_pays({c->nA_max, c->n_tumor, n, c->tumor_bits, c->tn_literal}, h, c->prune_mode, 1,
                     false) ||
           !plan(c, h, false, L, &need) || L.pair_cap < all_pairs(c->nA_max);
  }
  if (!plan(c, h, lazy, L, &need))
    return nfail(c, PDFS_ERR_UNSUPPORTED,
                 "round workspace of " + std::to_string(need) + " bytes exceeds the " +
                     std::to_string(kScratchBytes) + "-byte static scratch");
  const auto t0 = std::chrono::steady_clock::now();
  begin_stats(c, stats);
  memset(out, 0, sizeof(*out));
  const int32_t n_unc = set_uncovered(c, uncovered);
  if (n_unc < 0) return n_unc;
  if (n_unc == 0) return PDFS_NO_COMBO;
  const int w64 = dfs_row_words((n_unc + 63) / 64);
  if (w64 < 0 || w64 > c->w64_max) return nfail(c, PDFS_ERR_UNSUPPORTED, "row too wide");

  const Problem P = make_problem(c, h, p, q);
  Work w = make_work(c, w64, c->n_tumor + 1);
  w.st = reinterpret_cast<RoundState*>(base + L.st);
  w.recs = reinterpret_cast<RoundRecord*>(base + L.recs);
  w.rec_cap = 1;
  w.tallies = reinterpret_cast<unsigned long long*>(base + L.tallies);
  w.slots = reinterpret_cast<Slot*>(base + L.slots);
  w.cols = reinterpret_cast<int32_t*>(base + L.cols);
  w.act = reinterpret_cast<int32_t*>(base + L.act);
  w.flags = base + L.flags;
  w.TA = reinterpret_cast<uint32_t*>(base + L.TA);
  w.NA = reinterpret_cast<uint32_t*>(base + L.NA);
  w.A8 = reinterpret_cast<int8_t*>(base + L.A8);
  w.N8 = reinterpret_cast<int8_t*>(base + L.N8);
  w.hist = reinterpret_cast<uint32_t*>(base + L.hist);
  w.cursors = reinterpret_cast<unsigned long long*>(base + L.cursors);
  w.seed_pairs = reinterpret_cast<unsigned long long*>(base + L.seed);
  w.pairs = reinterpret_cast<unsigned long long*>(base + L.pairs);
  w.work_pairs = reinterpret_cast<unsigned long long*>(base + L.work);
  w.items = reinterpret_cast<Item*>(base + L.items);
  w.pair_cap = L.pair_cap;
  w.item_cap = L.item_cap;
  // single-kernel depth 4 (no prefix lists), no deep-walk rings
  w.tri = w.tri_s = nullptr;
  w.tri_rank = nullptr;
  w.c_hist = nullptr;
  w.tri_cap = 0;
  w.deepq = nullptr;

  hipStream_t s = c->stream;
  // what a round expects to start from zero; the rest is written before use
  NCK(launch_zero_u32(base + L.st, (L.zero_end - L.st) / 4, s));
  if (!lazy) NCK(launch_clear_slots(w.slots, kSlotPhases * kSlotsPerPhase, s));
  const int slot = c->next_slot;
  if (lazy) {
    // as the rounds of a bound-pruned run (14 launches 183 us, so 115 us
    // at G = 3067)
    LazyWork W = {};
    lazy_small(W, base + L.lazy, c->n_tumor);
    W.B = reinterpret_cast<uint64_t*>(base + L.B);
    W.bits = reinterpret_cast<uint64_t*>(base + L.bits);
    W.list = reinterpret_cast<unsigned long long*>(base + L.list);
    W.cmax = reinterpret_cast<int32_t*>(base + L.cmax);
    W.gw = L.gw;
    W.nw = L.nw;
    W.seg = L.seg;
    W.levels = lazy_levels(h);
    W.tally = stats ? w.tallies : nullptr;   // (the pair table is done with them)
    hipEvent_t* ev = c->ev[slot][0];
    rc = enqueue_lists(c, P, w, W, 1, ev);
    if (rc != PDFS_OK) return rc;
    if (c->time_kernels) NCK(hipEventRecord(ev[2], s));
    NCK(launch_lazy_round(P, w, W, 0, true, s));
    if (c->time_kernels) NCK(hipEventRecord(ev[3], s));
    NCK(launch_lazy_round(P, w, W, 1, false, s));
  } else {
    rc = enqueue_round(c, P, w, c->ev[slot][0], false, 1);
    if (rc != PDFS_OK) return rc;
  }
  RoundState* hs = &c->h_slots[slot];
  NCK(hipMemcpyAsync(hs, w.st, sizeof(RoundState), hipMemcpyDeviceToHost, s));
  NCK(hipMemcpyAsync(c->h_rec, w.recs, sizeof(RoundRecord), hipMemcpyDeviceToHost, s));
  NCK(hipStreamSynchronize(s));
  c->h_st = hs;
  if (c->time_kernels && hs->executed > 0) {
    hipEvent_t* ev = c->ev[slot][0];
    float ms = 0.f;
    if (h >= 2) {
      NCK(hipEventElapsedTime(&ms, ev[0], ev[1]));
      c->kernel_ns[0] += (int64_t)(ms * 1e6);
      c->kernel_launches[0] += 1;
    }
    if (h >= 3) {
      NCK(hipEventElapsedTime(&ms, ev[2], ev[3]));
      c->kernel_ns[1] += (int64_t)(ms * 1e6);
      c->kernel_launches[1] += 1;
    }
  }
  if (hs->overflow & 2) return nfail(c, PDFS_ERR_DEVICE, "corrupt per-wave result slot");
  if (hs->overflow)
    return nfail(c, PDFS_ERR_OUT_OF_MEMORY,
                 "the round's " + std::to_string(hs->n_pairs) +
                     " pairs exceed the static scratch's pair list of " +
                     std::to_string(L.pair_cap));
  end_stats(c, stats, t0);
  if (hs->rounds < 1 || !c->h_rec->found) return PDFS_NO_COMBO;
  if (lazy)   // recorded by sorted index only
    for (int k = 0; k < h; ++k) c->h_rec->genes[k] = c->h_perm[c->h_rec->sorted_idx[k]];
  fill_combo(out, *c->h_rec, h);
  return PDFS_OK;
}

}  // extern "C"
