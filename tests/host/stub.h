// The HIP calls and kernel launches that pdfs_api.cpp makes, on host memory: an
// allocation can be made to fail, and a launch checks that the buffers handed
// to it are held and long enough.  The rounds themselves are not computed: a
// run covers one sample a round for stub::rounds rounds.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "pdfs.h"
#include "pdfs_dev.h"
#include "pdfs_host.h"

namespace stub {

inline std::map<char*, size_t> held;
inline size_t bytes_held = 0;
inline size_t limit = ~(size_t)0;    // bytes that may be held at once
inline long fail_at = -1;            // the allocation (counted from 0) that fails
inline long allocs = 0;
inline hipError_t last = hipSuccess;
inline unsigned long long emit = 100;   // pairs a listing emits
inline int rounds = 3;
inline long lazy_launches = 0, walked_rounds = 0, counted = 0;

[[noreturn]] inline void die(const char* what) {
  std::printf("FAILED: %s\n", what);
  std::fflush(stdout);
  std::exit(1);
}

inline void need(const void* p, size_t bytes, const char* what) {
  if (!p) die(what);
  auto it = held.upper_bound((char*)p);
  if (it == held.begin()) die(what);
  --it;
  if ((char*)p + bytes > it->first + it->second) die(what);
}

inline hipError_t alloc(void** p, size_t n) {
  if (allocs++ == fail_at || bytes_held + n > limit) return last = hipErrorOutOfMemory;
  char* q = (char*)std::calloc(1, n);
  held[q] = n;
  bytes_held += n;
  *p = q;
  return hipSuccess;
}

inline hipError_t release(void* p) {
  if (!p) return hipSuccess;
  auto it = held.find((char*)p);
  if (it == held.end()) die("free of memory that is not held");
  bytes_held -= it->second;
  std::free(it->first);
  held.erase(it);
  return hipSuccess;
}

inline hipError_t take_last() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}

// One round ends: a sample is covered.
inline void commit(const pdfs::Problem& P, const pdfs::Work& w, int h) {
  pdfs::RoundState* st = w.st;
  if (st->done) return;
  pdfs::RoundRecord r = {};
  r.h = h;
  r.found = 1;
  r.tp = 1;
  for (int i = 0; i < h; ++i) r.sorted_idx[i] = r.genes[i] = i;
  need(w.recs, (size_t)w.rec_cap * sizeof(r), "records");
  if (st->rounds < w.rec_cap) w.recs[st->rounds] = r;
  st->rounds += 1;
  st->executed += 1;
  st->covered += 1;
  st->n_unc -= 1;
  st->done = st->n_unc <= 0 || st->rounds >= rounds || st->covered >= w.target ||
             (st->max_rounds > 0 && st->rounds >= st->max_rounds);
}

}  // namespace stub

// ---------------------------------------------------------------- HIP runtime
extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return stub::alloc(p, n); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return stub::alloc(p, n); }
hipError_t hipMallocFromPoolAsync(void** p, size_t n, hipMemPool_t, hipStream_t) {
  return stub::alloc(p, n);
}
hipError_t hipFree(void* p) { return stub::release(p); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return stub::release(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = (size_t)1 << 38;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 4;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipGetLastError() { return stub::take_last(); }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
}

// ------------------------------------------------------------------- launches
namespace pdfs {

using stub::need;

int dfs_row_words(int w) {
  if (w < 1 || w > kMaxW64) return -1;
  return w <= 8 ? w : (w + 1) / 2 * 2;
}
size_t sort_tmp_words(int G, int) { return (size_t)G; }
hipError_t sort_genes(const uint32_t*, int G, int, uint32_t*, int32_t* perm, hipStream_t) {
  for (int i = 0; i < G; ++i) perm[i] = i;
  return stub::take_last();
}
hipError_t launch_gene_counts(const uint64_t*, int64_t, const uint64_t*, int64_t, int, int, int,
                              uint32_t*, hipStream_t) {
  return stub::take_last();
}
hipError_t launch_gather_sorted(const uint64_t* T, int64_t ts, const uint64_t*, int64_t,
                                const int32_t*, int G, int wt, int, uint64_t* Ts, uint64_t*,
                                hipStream_t) {
  for (int g = 0; g < G; ++g) std::memcpy(Ts + (size_t)g * wt, T + g * ts, 8 * (size_t)wt);
  return stub::take_last();
}
hipError_t launch_normal_counts(const uint64_t*, int, int, int32_t*, hipStream_t) {
  return stub::take_last();
}
hipError_t launch_total_bits(const uint64_t* Ts, size_t words, RoundState* st, hipStream_t) {
  for (size_t i = 0; i < words; ++i) st->tumor_bits += (unsigned)__builtin_popcountll(Ts[i]);
  return stub::take_last();
}
hipError_t launch_check_pad(const uint64_t*, int64_t, int, int, int*, hipStream_t) {
  return stub::take_last();
}
hipError_t launch_front(const Problem& P, const Work& w, int run_rounds, bool full, bool rows,
                        bool unpack_tumor, bool unpack_normal, hipStream_t) {
  RoundState* st = w.st;
  if (full)
    for (int i = 0; i < P.n_tumor; ++i) w.U[i >> 6] |= 1ull << (i & 63);
  if (run_rounds >= 0) {
    int c = 0;
    for (int k = 0; k < P.wt; ++k) c += __builtin_popcountll(w.U[k]);
    st->n_unc = c;
    st->covered = P.n_tumor - c;
    st->rounds = st->executed = st->overflow = 0;
    st->max_rounds = run_rounds;
    st->done = c == 0 || st->covered >= w.target;
  }
  st->nA = P.G;
  if (rows) {
    const size_t n = (size_t)P.G;
    need(w.TA, n * 8 * (size_t)w.w64, "rows");
    need(w.NA, n * 4 * kMaxWN32, "normal rows");
    if (unpack_tumor) need(w.A8, n * (size_t)unpacked_row_bytes(w.w64), "unpacked rows");
    if (unpack_normal) need(w.N8, n * (size_t)unpacked_row_bytes(P.wn), "unpacked normals");
  }
  return stub::take_last();
}
hipError_t launch_h1(const Problem&, const Work&, hipStream_t) { return stub::take_last(); }

static hipError_t list(const Work& w) {
  need(w.pairs, (size_t)w.pair_cap * 8, "pair list");
  w.st->n_pairs = stub::emit;
  return stub::take_last();
}
hipError_t launch_pairs(const Problem& P, const Work& w, hipStream_t) {
  return P.h == 2 ? stub::take_last() : list(w);
}
hipError_t launch_pair_list(const Problem&, const Work& w, hipStream_t) { return list(w); }
hipError_t launch_list_pairs(const Work& w, const LazyWork&, int, hipStream_t) { return list(w); }
hipError_t launch_pair_hist(const Work&, hipStream_t) { return stub::take_last(); }
hipError_t launch_seed_select(const Problem&, const Work& w, hipStream_t) {
  need(w.seed_pairs, kSeedCap * 8, "seed list");
  return stub::take_last();
}
hipError_t launch_make_items(const Problem&, const Work& w, bool, hipStream_t) {
  need(w.items, (size_t)w.item_cap * sizeof(Item), "items");
  if (w.st->n_pairs > w.pair_cap) w.st->overflow |= kOverflowPairs;
  return stub::take_last();
}
hipError_t launch_filter_pairs(const Problem&, const Work& w, hipStream_t) {
  need(w.work_pairs, (size_t)w.pair_cap * 8, "work list");
  return stub::take_last();
}
hipError_t launch_use_all_pairs(const Work&, hipStream_t) { return stub::take_last(); }
hipError_t launch_dfs(const Problem&, const Work& w, int, hipStream_t) {
  need(w.work_pairs, (size_t)w.pair_cap * 8, "work list");
  return stub::take_last();
}
hipError_t launch_dfs_deep(const Problem&, const Work& w, int, hipStream_t) {
  need(w.deepq, deep_ring_words(w.w64, 4) * 4, "prefix rings");
  return stub::take_last();
}
hipError_t launch_tri_begin(const Work&, hipStream_t) { return stub::take_last(); }
hipError_t launch_count_long(const Problem&, const Work& w, hipStream_t) {
  w.st->n_tri = 50;
  return stub::take_last();
}
hipError_t launch_sort_triples(const Work& w, hipStream_t) {
  need(w.tri, (size_t)w.tri_cap * 8, "prefix list");
  need(w.tri_s, (size_t)w.tri_cap * 8, "sorted prefix list");
  need(w.tri_rank, (size_t)w.tri_cap * 4, "prefix ranks");
  return stub::take_last();
}
hipError_t launch_dfs4_tiles(const Problem&, const Work&, hipStream_t) { return stub::take_last(); }
hipError_t launch_finish_round(const Problem& P, const Work& w, int, int, hipStream_t) {
  if (w.st->overflow) w.st->done = 1;
  if (!w.st->done) stub::walked_rounds += 1;
  stub::commit(P, w, P.h);
  return stub::take_last();
}
hipError_t launch_run_resume(const Work& w, hipStream_t) {
  w.st->overflow = 0;
  w.st->done = 0;
  return stub::take_last();
}
size_t deep_ring_words(int w64_max, int n_cu) { return (size_t)w64_max * (size_t)n_cu * 1000; }
void scratch_init(int) {}

int lazy_levels(int h) { return h <= 4 ? 1 : h - 3; }

static void check_lists(const Problem& P, const Work& w, const LazyWork& L) {
  if (L.nw < 4 || L.nw % 4 || L.nw > kLazyWaves) stub::die("waves");
  if ((size_t)L.nw * L.seg < w.pair_cap) stub::die("shares below the pair capacity");
  need(L.list, (size_t)L.nw * L.seg * 8, "shares");
  need(L.cmax, (size_t)L.nw * ((L.seg + kWave - 1) / kWave) * 4, "shares' bounds");
  need(L.B, (size_t)64 * w.w64 * L.gw * 8, "transposed rows");
  need(L.pool, (size_t)L.nw * sizeof(Slot), "pool");
  need(L.uncs, ((size_t)P.n_tumor + 2) * 4, "uncovered counts");
  if (P.h >= 4) need(L.bits, (size_t)L.nw * L.levels * L.gw * 8, "bitmaps");
}
hipError_t launch_lazy_begin(const Problem&, const Work& w, const LazyWork& L, hipStream_t) {
  need(L.B, (size_t)64 * w.w64 * L.gw * 8, "transposed rows");
  L.S[1].done = 0;
  return stub::take_last();
}
hipError_t launch_lazy_deal(const Problem& P, const Work& w, const LazyWork& L, hipStream_t) {
  check_lists(P, w, L);
  if (w.st->n_pairs > w.pair_cap) {
    w.st->overflow |= kOverflowPairs;
    L.S[1].done = 1;
  }
  return stub::take_last();
}
hipError_t launch_lazy_round(const Problem& P, const Work& w, const LazyWork& L, int n, bool,
                             hipStream_t) {
  check_lists(P, w, L);
  stub::lazy_launches += 1;
  if (n > 0 && !L.S[1].done) stub::commit(P, w, P.h);
  return stub::take_last();
}
int count_segments(int nA) { return (nA + 511) / 512 > 0 ? (nA + 511) / 512 : 1; }
size_t count_table_rows(int nA) { return (size_t)count_segments(nA) * 64 + 1; }
hipError_t launch_count(const Problem& P, const Work& w, const LazyWork& L, const CountWork& C,
                        int nA_max, hipStream_t) {
  const size_t R1 = (size_t)w.st->executed + 1;
  stub::counted += 1;
  need(C.order, 64 * kMaxW64 * 4, "sample order");
  need(C.pref, (size_t)64 * w.w64 * L.gw * 2, "list places");
  need(C.tg, (size_t)count_segments(nA_max) * 512 * 2, "gene rounds");
  if (P.h >= 4) need(C.q, (size_t)(P.h - 3) * C.q_n * 8, "list sums");
  if (P.h == 4) need(C.sw, C.q_n * 8, "list sums of words");
  if (P.h == 3 || P.h == 4) {
    const size_t seg = (size_t)count_segments(nA_max) * R1 * 4;
    const size_t tab = count_table_rows(nA_max) * R1 * 4;
    need(C.seg_v, seg, "segments");
    need(C.seg_w, seg, "segments of words");
    need(C.tab_v, tab, "table");
    need(C.tab_w, tab, "table of words");
  }
  if (P.h >= 4) need(C.bits, (size_t)C.waves * L.levels * L.gw * 8, "counters' bitmaps");
  return stub::take_last();
}
hipError_t launch_clear_slots(Slot*, int, hipStream_t) { return stub::take_last(); }

}  // namespace pdfs
