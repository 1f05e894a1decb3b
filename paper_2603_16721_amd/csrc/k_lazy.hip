// Rounds of a greedy run under score-bound pruning, as a lazy best-first
// search over the pairs of the run's first round (h = 2..9).
//
// A combination's score S = p*TP + q*TN can only fall while the cover grows
// (TP counts uncovered samples, TN does not change), so an upper bound on the
// scores below a pair stays one for the rest of the run.  The non-empty pairs
// of the starting mask are listed once, each with such a bound (p*C_T + q*N_n
// to begin with), and a round only opens the pairs whose bound still reaches
// the best combination found so far; an opened pair leaves a tighter bound
// behind (the best leaf scored or the largest bound pruned below it).  What a
// round costs is then the pairs whose bounds have come into reach, not the
// cohort: one launch, no re-packing, no pair table, no work lists.
//
// Everything lives in the run's own index space: the genes and samples that
// are active / uncovered at its start (rows TA, re-packed once), plus the
// transposed bit matrix B (one row of genes per sample).  Below a pair the
// candidates are counted 64 genes per lane at a time: the B rows of the
// prefix's samples are added up in bit slices, and one comparison of the
// slices with the least useful TP keeps the candidates that can matter.  A
// short list of those (their samples compressed to one 64-bit mask) is then
// searched from LDS.
//
// Pairs are dealt to the waves in order of their first counts, one each in
// turn; a wave owns its share for the whole run (no queue, no atomics), 64
// pairs to a chunk with the chunk's largest bound beside it.  Each round a
// wave re-evaluates the best leaf it knows, publishes it, and then opens its
// pairs from the largest bounds down.  The leaves that no incumbent beat are
// left in a short list, and the next launch begins by taking their argmax and
// updating the cover (every block for itself, the first one for the record):
// no block waits for another.  Taking it in the last block to finish instead
// costs its chain of loads (7 us) and the count of finished blocks (3 us) at
// the end of every round.
#include <type_traits>

#include "dfs_core.h"
#include "lazy_core.h"
#include "pdfs_dev.h"
#include "slot_reduce.h"

namespace pdfs {

namespace {

// |Ta & Tb & U| of one pair per lane, u in LDS; loads of four words in flight.
__device__ __forceinline__ int pair_count(const uint64_t* __restrict__ ra,
                                          const uint64_t* __restrict__ rb, const uint64_t* u,
                                          int w64) {
  int ct = 0, k = 0;
  for (; k + 4 <= w64; k += 4) {
    uint64_t x[4], y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = ra[k + i];
      y[i] = rb[k + i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) ct += popc64(x[i] & y[i] & u[k + i]);
  }
  for (; k < w64; ++k) ct += popc64(ra[k] & rb[k] & u[k]);
  return ct;
}

// ------------------------------------------------------------- run start
// One wave per 64 genes x 64 samples: the rows' word transposed by ballots.
// The first block also starts the run's control words.
__global__ __launch_bounds__(256) void k_lazy_begin(Problem P, Work w, LazyWork L) {
  RoundState* st = w.st;
  if (st->done) {   // nothing to cover: the round launches do nothing either
    if (blockIdx.x == 0 && threadIdx.x == 0) L.S[1].done = 1;
    return;
  }
  const int lane = threadIdx.x & 63;
  const int nA = st->nA;
  if (blockIdx.x == 0) {
    const int n_unc = st->n_unc;
    for (int k = threadIdx.x; k < kMaxW64; k += 256) {
      const int lo = 64 * k;
      L.U2[kMaxW64 + k] = n_unc - lo >= 64 ? ~0ull : (n_unc > lo ? (1ull << (n_unc - lo)) - 1ull : 0ull);
    }
    if (threadIdx.x == 0) L.uncs[0] = n_unc;
    for (int v = threadIdx.x; v <= kMaxCount; v += 256) L.cursor[v] = 0u;
    if (threadIdx.x < 3) L.n_win[64 * threadIdx.x] = 0u;
    if (threadIdx.x < 2) L.inc[threadIdx.x * kCursorStride] = 0ull;
    if (threadIdx.x < 2 * kIncShards) L.shard[threadIdx.x * kCursorStride] = 0ull;
    if (threadIdx.x == 0) {
      const LazyState z = {n_unc, 0, 0, 0, 0};
      L.S[1] = z;
    }
  }
  const uint64_t* T = reinterpret_cast<const uint64_t*>(w.TA);
  const int tiles = L.gw * w.w64;
  const int waves = gridDim.x * (kBlock / kWave);
  for (int t = blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6); t < tiles; t += waves) {
    const int gq = t / w.w64, sw = t % w.w64;
    const int g = gq * 64 + lane;
    const uint64_t x = g < nA ? T[(size_t)g * w.w64 + sw] : 0ull;
    uint64_t mine = 0;
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      const unsigned long long col = __ballot((x >> j) & 1ull);
      mine = lane == j ? col : mine;
    }
    L.B[(size_t)(sw * 64 + lane) * L.gw + gq] = mine;
  }
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < L.nw; i += gridDim.x * kBlock)
    L.pool[i].s = -1;
  if (L.tally)
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < kWorkRows * kLazyFields;
         i += gridDim.x * kBlock)
      L.tally[i] = 0ull;
}

// The pair list in order of falling count, dealt one by one to the waves: the
// pair of rank r is entry r / nw of wave r % nw.  A block takes kDeal pairs,
// counts them in LDS, reserves its stretch of every bin with one atomic and
// places them (the order inside a bin is of no consequence).
constexpr int kDeal = 4096;

__global__ __launch_bounds__(256) void k_lazy_deal(Problem P, Work w, LazyWork L) {
  __shared__ uint32_t cnt[kMaxCount + 1];
  __shared__ uint32_t base[kMaxCount + 1];
  __shared__ uint32_t part[kBlock];
  RoundState* st = w.st;
  if (L.S[1].done) return;
  const unsigned long long np = st->n_pairs;
  const int tid = threadIdx.x;
  if (np > w.pair_cap) {
    // n_pairs keeps the count emitted; the run stops before its first round
    if (blockIdx.x == 0 && tid == 0) {
      st->overflow |= kOverflowPairs;
      L.S[1].done = 1;
    }
    return;
  }
  constexpr int kPer = (kMaxCount + kBlock) / kBlock;   // bins per thread, from the top
  uint32_t sum = 0;
  for (int k = 0; k < kPer; ++k) {
    const int v = kMaxCount - tid * kPer - k;
    if (v >= 0) sum += w.hist[v];
  }
  part[tid] = sum;
  __syncthreads();
  for (int o = 1; o < kBlock; o <<= 1) {
    const uint32_t add = tid >= o ? part[tid - o] : 0u;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  uint32_t run = part[tid] - sum;
  for (int k = 0; k < kPer; ++k) {
    const int v = kMaxCount - tid * kPer - k;
    if (v >= 0) {
      base[v] = run;
      run += w.hist[v];
    }
  }
  const int chunks = (L.seg + kWave - 1) / kWave;
  for (unsigned long long i0 = (unsigned long long)blockIdx.x * kDeal; i0 < np;
       i0 += (unsigned long long)gridDim.x * kDeal) {
    __syncthreads();
    for (int v = tid; v <= kMaxCount; v += kBlock) cnt[v] = 0u;
    __syncthreads();
    unsigned long long e[kDeal / kBlock];
    uint32_t rk[kDeal / kBlock];
#pragma unroll
    for (int u = 0; u < kDeal / kBlock; ++u) {
      const unsigned long long i = i0 + (unsigned long long)u * kBlock + tid;
      e[u] = i < np ? w.pairs[i] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < kDeal / kBlock; ++u)
      rk[u] = e[u] ? atomicAdd(&cnt[(e[u] >> 32) & 0xffff], 1u) : 0u;
    __syncthreads();
    for (int v = tid; v <= kMaxCount; v += kBlock) {
      const uint32_t n = cnt[v];
      cnt[v] = n ? base[v] + atomicAdd(&L.cursor[v], n) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kDeal / kBlock; ++u) {
      if (!e[u]) continue;
      const int ct = (int)((e[u] >> 32) & 0xffff);
      const uint32_t r = cnt[ct] + rk[u];
      const uint32_t wv = r % (uint32_t)L.nw, slot = r / (uint32_t)L.nw;
      if (slot >= (uint32_t)L.seg) continue;   // r < pair_cap <= nw * seg
      const uint32_t sb = (uint32_t)(P.p * ct + P.q * P.n_normal);
      L.list[(size_t)wv * L.seg + slot] = (e[u] & 0xffffffffull) | ((unsigned long long)sb << 32);
      // ranks fall in count, so a chunk's first entry holds its largest bound
      if (slot % kWave == 0) L.cmax[(size_t)wv * chunks + slot / kWave] = (int32_t)sb;
    }
  }
}

// ------------------------------------------------------------- one round
// A wave's share of LDS: level lists (candidates with their samples as a mask
// over the pair's at most 64 samples), the prefix's sample ids, intersections
// per depth of the general walk, the prefix and the best leaf's tuple.
struct WaveLds {
  uint64_t* mask;    // [levels][cap]
  uint64_t* y;       // [kMaxH][kMaxW64]
  uint16_t* idx;     // [levels][cap]
  uint16_t* smp;     // [kMaxCount]
  uint16_t* pre;     // [kMaxH + 1] prefix (active indices, ascending)
  uint16_t* tup;     // [kMaxH + 1] best leaf's tuple
};

constexpr int kLazyCap(int h) { return h <= 5 ? 256 : 128; }
constexpr int kListSamples = 256;   // samples of a pair whose candidates are listed, at most
constexpr int kLazyLevels(int h) { return h <= 4 ? 1 : h - 3; }

size_t lazy_wave_bytes(int h) {
  const size_t lv = (size_t)kLazyLevels(h), cap = (size_t)kLazyCap(h);
  size_t b = lv * cap * 8 + (size_t)kMaxH * kMaxW64 * 8 + lv * cap * 2 + kMaxCount * 2 +
             2 * (kMaxH + 1) * 2;
  return (b + 15) / 16 * 16;
}

__device__ __forceinline__ WaveLds wave_lds(char* p, int h) {
  const int lv = h <= 4 ? 1 : h - 3, cap = h <= 5 ? 256 : 128;
  WaveLds s;
  s.mask = reinterpret_cast<uint64_t*>(p);
  s.y = s.mask + lv * cap;
  s.idx = reinterpret_cast<uint16_t*>(s.y + kMaxH * kMaxW64);
  s.smp = s.idx + lv * cap;
  s.pre = s.smp + kMaxCount;
  s.tup = s.pre + kMaxH + 1;
  return s;
}

// Bit-sliced count: slice k of s holds bit k of, for each of the 64 genes of
// word wd, the number of listed samples that carry it.
template <int NB>
__device__ __forceinline__ void slice_count(const uint64_t* __restrict__ B, int gw,
                                            const uint16_t* smp, int m, int wd, bool on,
                                            uint64_t (&s)[NB]) {
#pragma unroll
  for (int k = 0; k < NB; ++k) s[k] = 0;
  auto add = [&](uint64_t x) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const uint64_t c = s[k] & x;
      s[k] ^= x;
      x = c;
    }
  };
  int j = 0;
  auto rows = [&](auto n) {   // n rows in flight
    uint64_t x[decltype(n)::value];
#pragma unroll
    for (int u = 0; u < n; ++u) {
      const uint64_t* row = B + (size_t)uniform(smp[j + u]) * gw;
      x[u] = on ? row[wd] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < n; ++u) add(x[u]);
    j += n;
  };
  while (j + 8 <= m) rows(std::integral_constant<int, 8>());
  if (j + 4 <= m) rows(std::integral_constant<int, 4>());
  while (j < m) rows(std::integral_constant<int, 1>());
}

// Genes of the word whose count is at least `need` (wave-uniform, >= 1).
template <int NB>
__device__ __forceinline__ uint64_t slices_ge(const uint64_t (&s)[NB], int need) {
  if (need >> NB) return 0ull;
  uint64_t ge = ~0ull;
#pragma unroll
  for (int k = 0; k < NB; ++k) ge = ((need >> k) & 1) ? (s[k] & ge) : (s[k] | ge);
  return ge;
}

template <int NB>
__device__ __forceinline__ int slice_at(const uint64_t (&s)[NB], int bit) {
  int c = 0;
#pragma unroll
  for (int k = 0; k < NB; ++k) c |= (int)((s[k] >> bit) & 1ull) << k;
  return c;
}

// The pair list straight from the rows: a wave takes a gene, adds up the
// transposed rows of the gene's samples in bit slices (64 later genes per lane),
// and every later gene with a count is a pair.  The work is one word per sample
// of the gene and 64 later genes, so it follows the mutations there are, where
// the matrix cores' table follows the genes squared times the samples.  Genes in
// many samples come last in the order: with few genes behind them their rows are
// and-ed instead, a later gene per lane.  Bound by each gene's chain (row, sample
// rows, records), so many waves with few genes each.  Records are staged per wave
// and a block reserves its stretch of the list once (an atomic per gene would
// queue on the count's one address).
// G = 20000 at 66 mutations a sample: 38 us, the table 181 us; without the rows
// of the common genes 75 us, with 16 waves to a block 76 us.
constexpr int kListWaves = 8;    // waves of a block
constexpr int kListBuf = 384;    // records a wave stages

// The lanes' next n records (n per lane, as next() gives them) to the wave's
// stage, or with the staged ones to the list where the stage would overflow.
template <class F>
__device__ __forceinline__ void put_records(const Work& w, int n, unsigned long long* buf,
                                            int& have, int lane, F next) {
  const int before = wave_before(n, lane);
  const int tot = uniform(__shfl(before + n, 63, 64));
  if (!tot) return;
  if (have + tot <= kListBuf) {
    for (int i = have + before, e = i + n; i < e; ++i) buf[i] = next();
    have += tot;
    return;
  }
  unsigned long long base = 0;
  if (lane == 0) base = atomicAdd(&w.st->n_pairs, (unsigned long long)(have + tot));
  base = readlane64(base, 0);
  wave_lds_sync();
  for (int i = lane; i < have; i += kWave)
    if (base + i < w.pair_cap) w.pairs[base + i] = buf[i];
  wave_lds_sync();
  unsigned long long pos = base + have + before;
  for (int i = 0; i < n; ++i, ++pos) {
    const unsigned long long r = next();
    if (pos < w.pair_cap) w.pairs[pos] = r;
  }
  have = 0;
}

__device__ __forceinline__ unsigned long long pair_record(int a, int b, int ct) {
  return (unsigned long long)a | ((unsigned long long)b << 16) | ((unsigned long long)ct << 32);
}

template <int NB>
__device__ __forceinline__ void list_by_slices(const Work& w, const LazyWork& L, int a, int hi,
                                               int m, const uint16_t* smp,
                                               unsigned long long* buf, int& have, int lane) {
  const int w_hi = (hi + 63) >> 6;
  for (int w0 = (a + 1) >> 6; w0 < w_hi; w0 += kWave) {
    const int wd = w0 + lane;
    uint64_t s[NB];
    slice_count<NB>(L.B, L.gw, smp, m, wd, wd < w_hi, s);
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < NB; ++k) any |= s[k];
    any &= range_bits(wd, a + 1, hi);
    put_records(w, popc64(any), buf, have, lane, [&]() {
      const int bit = __builtin_ctzll(any);
      any &= any - 1;
      return pair_record(a, wd * 64 + bit, slice_at<NB>(s, bit));
    });
  }
}

__device__ __forceinline__ void list_by_rows(const Work& w, const uint64_t* __restrict__ T, int a,
                                             int hi, unsigned long long* buf, int& have, int lane) {
  const int w64 = w.w64;
  const uint64_t* ra = T + (size_t)a * w64;
  for (int b0 = a + 1; b0 < hi; b0 += kWave) {
    const int b = b0 + lane;
    const uint64_t* rb = T + (size_t)(b < hi ? b : a) * w64;
    int ct = 0, k = 0;
    for (; k + 4 <= w64; k += 4) {
      uint64_t x[4], y[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = ra[k + i];
        y[i] = rb[k + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) ct += popc64(x[i] & y[i]);
    }
    for (; k < w64; ++k) ct += popc64(ra[k] & rb[k]);
    put_records(w, b < hi && ct > 0 ? 1 : 0, buf, have, lane,
                [&]() { return pair_record(a, b, ct); });
  }
}

__global__ __launch_bounds__(kListWaves * 64) void k_list_pairs(Work w, LazyWork L) {
  __shared__ unsigned long long s_buf[kListWaves][kListBuf];
  __shared__ uint16_t s_smp[kListWaves][kMaxCount];
  __shared__ int s_n[kListWaves];
  __shared__ unsigned long long s_base;
  RoundState* st = w.st;
  if (st->done) return;
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const int nA = st->nA;
  const int a_hi = min(nA, st->amax[1]), hi = min(nA, st->amax[2]);   // Alg. 2's loop bounds
  const uint64_t* T = reinterpret_cast<const uint64_t*>(w.TA);
  unsigned long long* buf = s_buf[wave];
  uint16_t* smp = s_smp[wave];
  int have = 0;
  for (int a = (int)blockIdx.x * kListWaves + wave; a < a_hi; a += (int)gridDim.x * kListWaves) {
    const int m = list_samples(lane < w.w64 ? T[(size_t)a * w.w64 + lane] : 0ull, smp, lane);
    // batches of dependent loads: 8 sample rows per 64 words, 4 row words per 64 genes
    const int rest = hi - a - 1;
    if ((m + 7) / 8 * ((rest >> 12) + 1) > ((rest + 63) >> 6) * ((w.w64 + 3) >> 2))
      list_by_rows(w, T, a, hi, buf, have, lane);
    else if (m <= 3) list_by_slices<2>(w, L, a, hi, m, smp, buf, have, lane);
    else if (m <= 15) list_by_slices<4>(w, L, a, hi, m, smp, buf, have, lane);
    else if (m <= 127) list_by_slices<7>(w, L, a, hi, m, smp, buf, have, lane);
    else list_by_slices<11>(w, L, a, hi, m, smp, buf, have, lane);
  }
  if (lane == 0) s_n[wave] = have;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int k = 0; k < kListWaves; ++k) tot += s_n[k];
    s_base = tot ? atomicAdd(&st->n_pairs, (unsigned long long)tot) : 0ull;
  }
  __syncthreads();
  unsigned long long pos = s_base;
  for (int k = 0; k < wave; ++k) pos += (unsigned long long)s_n[k];
  for (int i = lane; i < have; i += kWave)
    if (pos + i < w.pair_cap) w.pairs[pos + i] = buf[i];
}

// Largest count over the genes `in` of all lanes; in is cut to the genes that
// reach it.
template <int NB>
__device__ __forceinline__ int slices_max(const uint64_t (&s)[NB], uint64_t& in) {
  int v = 0;
#pragma unroll
  for (int k = NB - 1; k >= 0; --k) {
    const uint64_t t = in & s[k];
    if (__any(t != 0)) {
      in = t;
      v |= 1 << k;
    }
  }
  return v;
}

// The state of one wave in one round.
struct Wave {
  const Problem& P;
  const Work& w;
  const LazyWork& L;
  WaveLds s;
  const uint64_t* T;
  int lane, nA, w64, h;
  uint64_t u;                   // lane k < w64: word k of the uncovered mask
  unsigned long long* incp;     // the launch's incumbent and its shards
  unsigned long long* shard;
  unsigned long long inc;       // newest incumbent seen
  int bs, btp, bfp;             // best leaf (tuple in s.tup)
  // the pair being opened
  bool own;                     // the wave's best leaf lies below this pair
  int tie_s;                    // a score this pair has reached: its later tuples lose the tie
  int a, b, need, sub, lmax;    // best score below it; per lane: largest TP pruned
  // Work counted: lane f holds field f (LazyField), so that a depth known only at
  // run time needs no indexed registers and the round's end one store: 0.6 us of a
  // round of 21 at h = 5 (1.4 us with a register per depth, whose selects at the
  // end are cold code); h = 2 and 3 covers 2 % longer than uncounted, h = 4 no
  // longer, h = 5 3 %.
  long long work;
  uint32_t ne3;                 // h = 3, per lane: non-empty leaves of the slices
};

__device__ __forceinline__ int count_lanes(bool on) { return __popcll(__ballot(on)); }

// Nodes of one depth: formed, non-empty, pruned (depth 2: pairs opened).
__device__ __forceinline__ void count_nodes(Wave& v, int depth, int vis, int ne, int bp) {
  const int x = v.lane < kLfNe ? vis : (v.lane < kLfBp ? ne : bp);
  v.work += v.lane < kLfFp && (v.lane & 7) == depth - 2 ? x : 0;
}

__device__ __forceinline__ unsigned long long load_inc(const Wave& v) {
  return __hip_atomic_load(v.incp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void refresh_need(Wave& v) {
  if (v.inc == 0) {
    v.need = 1;
    return;
  }
  const int s = (int)(v.inc >> 32) - 1;
  const int g1 = 0xffff - (int)((v.inc >> 16) & 0xffff);
  const int g2 = 0xffff - (int)(v.inc & 0xffff);
  const bool tie = s != v.tie_s && (v.a < g1 || (v.a == g1 && v.b <= g2));
  v.need = min_tp_for(v.P, s, tie);
}

// Both walks below a pair go in tuple order.  Once the prefix s.pre[0, np) has
// passed the wave's own best leaf, no later leaf of the pair wins its tie.
__device__ __forceinline__ void pass_own_best(Wave& v, int np) {
  if (!v.own) return;
  for (int i = 2; i < np; ++i) {
    const int x = uniform(v.s.pre[i]), y = uniform(v.s.tup[i]);
    if (x < y) return;
    if (x > y) {
      v.own = false;
      v.tie_s = v.bs;
      refresh_need(v);
      return;
    }
  }
}

__device__ __forceinline__ void publish_key(Wave& v, unsigned long long key) {
  if (key > v.inc) {
    unsigned long long best = key;
    if (v.lane == 0) {
      unsigned long long old =
          atomicMax(&v.shard[(blockIdx.x % kIncShards) * kCursorStride], key);
      if (old < key) {
        old = load_inc(v);
        if (old < key) old = atomicMax(v.incp, key);
      }
      best = old > key ? old : key;
    }
    v.inc = __shfl(best, 0, 64);
  }
}

__device__ __forceinline__ void publish(Wave& v, int s, int a, int b) {
  publish_key(v, leaf_key(s, a, b));
}

// Takes the leaf (first np genes of s.pre, then d) if it beats the wave's best.
__device__ __forceinline__ bool take_leaf(Wave& v, int sc, int tp, int fp, int np, int d) {
  bool better = sc > v.bs;
  if (sc == v.bs) {
    wave_lds_sync();
    bool decided = false;
    for (int i = 0; i <= np && !decided; ++i) {
      const int x = i < np ? (int)v.s.pre[i] : d;
      const int y = (int)v.s.tup[i];
      if (x != y) {
        better = x < y;
        decided = true;
      }
    }
    better = uniform(better ? 1 : 0) != 0;
  }
  if (!better) return false;
  v.bs = sc;
  v.btp = tp;
  v.bfp = fp;
  wave_lds_sync();
  if (v.lane <= np) v.s.tup[v.lane] = v.lane < np ? v.s.pre[v.lane] : (uint16_t)d;
  wave_lds_sync();
  return true;
}

// Leaves: the prefix s.pre[0, np) with each hit lane's candidate d (TP tp).
// True when one of them became the wave's best.
__device__ __forceinline__ bool score_leaves(Wave& v, int np, bool hit, int d, int tp) {
  if (!__any(hit)) return false;
  wave_lds_sync();
  const bool lit = v.P.tn_literal != 0;
  const uint32_t* NA = v.w.NA;
  uint32_t z = 0;
  if (v.lane < kMaxWN32) {
    z = NA[(size_t)v.s.pre[0] * kMaxWN32 + v.lane];
    for (int i = 1; i < np; ++i) z = nrm_join(z, NA[(size_t)v.s.pre[i] * kMaxWN32 + v.lane], lit);
  }
  // normal words that can hold a false positive
  unsigned long long zm = __ballot(lit ? v.lane < v.w.wn32 : (v.lane < kMaxWN32 && z != 0));
  if (zm) {
    const int n = count_lanes(hit);
    v.work += v.lane == kLfFp ? n : 0;
  }
  int fp = 0;
  while (zm) {
    const int k = __builtin_ctzll(zm);
    zm &= zm - 1;
    const uint32_t zk = (uint32_t)__builtin_amdgcn_readlane((int)z, k);
    if (hit) fp += __popc(nrm_join(zk, NA[(size_t)d * kMaxWN32 + k], lit));
  }
  const int sc = hit ? v.P.p * tp + v.P.q * (v.P.n_normal - fp) : -1;
  const int smax = wave_max(sc);
  v.sub = max(v.sub, smax);
  if (smax < v.bs) return false;
  const int dmin = wave_min(sc == smax ? d : 0x7fffffff);
  const unsigned long long at = __ballot(sc == smax && d == dmin);
  const int src = __builtin_ctzll(at);
  const int btp = __builtin_amdgcn_readlane(tp, src), bfp = __builtin_amdgcn_readlane(fp, src);
  const bool took = take_leaf(v, smax, btp, bfp, np, dmin);
  // genes 0 and 1 of the tuple (np >= 1)
  const int g0 = uniform(v.s.pre[0]);
  const int g1 = np >= 2 ? uniform(v.s.pre[1]) : dmin;
  publish(v, smax, g0, g1);
  return took;
}

// Two ways to count the candidates [lo, nA) of a prefix with m samples: adding
// up its samples' rows of B (64 genes per lane, m loads deep) or and-ing each
// candidate's own row with the prefix (a gene per lane, w64 loads deep).  The
// rows win where few genes are left, as below the most frequent genes, which
// come last: with 140 samples and 3 candidates 59 us by slices, 13 us by
// rows.
__device__ __forceinline__ bool count_by_rows(const Wave& v, int m, int lo) {
  const int words = ((v.nA + 63) >> 6) - (lo >> 6);
  return words * v.w64 < m * ((words + 63) >> 6);
}

// |y & T_d| of one candidate per lane, y in LDS.
__device__ __forceinline__ int row_count(const Wave& v, const uint64_t* y, int d, bool on) {
  return on ? pair_count(v.T + (size_t)d * v.w64, v.T + (size_t)d * v.w64, y, v.w64) : 0;
}

// Candidates [lo, nA) below the prefix s.pre[0, np) with intersection y, as
// leaves; `in` (may be null) limits them to a bitmap.
__device__ __forceinline__ void leaves_by_rows(Wave& v, const uint64_t* y, int np, int lo,
                                               const uint64_t* in) {
  int vis = 0, ne = 0;
  for (int d0 = lo & ~63; d0 < v.nA; d0 += kWave) {
    const int d = d0 + v.lane;
    bool on = d >= lo && d < v.nA;
    if (in) on = on && ((in[d0 >> 6] >> v.lane) & 1ull);
    const int tp = row_count(v, y, d, on);
    const bool hit = on && tp >= v.need;
    v.lmax = max(v.lmax, hit ? 0 : tp);
    if (in) vis += count_lanes(on);
    ne += count_lanes(tp > 0);
    score_leaves(v, np, hit, d, tp);
    refresh_need(v);
  }
  count_nodes(v, np + 1, in ? vis : v.nA - lo, ne, 0);
}

// The candidates that keep at least `need` of y's samples as a list (false:
// they do not fit), or as a bitmap.
__device__ __forceinline__ bool list_by_rows(Wave& v, const uint64_t* y, int lo, int cap, int& n) {
  n = 0;
  int ne = 0;
  for (int d0 = lo; d0 < v.nA; d0 += kWave) {
    const int d = d0 + v.lane;
    const int tp = row_count(v, y, d, d < v.nA);
    const bool hit = d < v.nA && tp >= v.need;
    v.lmax = max(v.lmax, hit ? 0 : tp);
    const unsigned long long hm = __ballot(hit);
    if (n + __popcll(hm) > cap) return false;
    if (hit) v.s.idx[rank_below(hm, n)] = (uint16_t)d;
    n += __popcll(hm);
    ne += count_lanes(tp > 0);
  }
  count_nodes(v, 3, v.nA - lo, ne, ne - n);
  wave_lds_sync();
  return true;
}

__device__ __forceinline__ void bits_by_rows(Wave& v, const uint64_t* y, int depth, int lo,
                                             const uint64_t* in, uint64_t* out) {
  int vis = 0, ne = 0, keep = 0;
  for (int d0 = lo & ~63; d0 < v.nA; d0 += kWave) {
    const int d = d0 + v.lane;
    bool on = d >= lo && d < v.nA;
    if (in) on = on && ((in[d0 >> 6] >> v.lane) & 1ull);
    const int tp = row_count(v, y, d, on);
    const bool hit = on && tp >= v.need;
    v.lmax = max(v.lmax, hit ? 0 : tp);
    const unsigned long long hm = __ballot(hit);
    if (v.lane == 0) out[d0 >> 6] = hm;
    vis += count_lanes(on);
    ne += count_lanes(tp > 0);
    keep += __popcll(hm);
  }
  count_nodes(v, depth, vis, ne, ne - keep);
}

// Genes of `in` that some listed sample carries.
template <int NB>
__device__ __forceinline__ uint64_t slices_any(const uint64_t (&s)[NB], uint64_t in) {
  uint64_t x = 0;
#pragma unroll
  for (int k = 0; k < NB; ++k) x |= s[k];
  return x & in;
}

// All candidates in [lo, nA) against the m listed samples, as leaves below the
// prefix s.pre[0, np); `in` (may be null) limits them to a bitmap.
template <int NB>
__device__ __forceinline__ void leaves_by_slices(Wave& v, int m, int np, int lo, const uint64_t* in) {
  const int w_hi = (v.nA + 63) >> 6;
  int vis = 0, ne = 0;
  for (int w0 = lo >> 6; w0 < w_hi; w0 += 64) {
    const int wd = w0 + v.lane;
    uint64_t s[NB];
    slice_count<NB>(v.L.B, v.L.gw, v.s.smp, m, wd, wd < w_hi, s);
    uint64_t r = wd < w_hi ? range_bits(wd, lo, v.nA) : 0ull;
    if (in && r) r &= in[wd];
    ne += popc64(slices_any<NB>(s, r));
    if (in) vis += popc64(r);
    uint64_t ge = slices_ge<NB>(s, v.need) & r;
    uint64_t rest = r & ~ge;
    v.lmax = max(v.lmax, slices_max<NB>(s, rest));
    while (__any(ge != 0)) {
      const bool has = ge != 0;
      const int bit = has ? __builtin_ctzll(ge) : 0;
      ge &= ge - 1;
      const int tp = has ? slice_at<NB>(s, bit) : 0;
      const bool hit = tp >= v.need && has;
      v.lmax = max(v.lmax, has && !hit ? tp : 0);
      score_leaves(v, np, hit, wd * 64 + bit, tp);
      refresh_need(v);
    }
  }
  if (in) {
    count_nodes(v, np + 1, wave_sum(vis), wave_sum(ne), 0);
  } else {   // below the pair itself
    count_nodes(v, 3, v.nA - lo, 0, 0);
    v.ne3 += (uint32_t)ne;
  }
}

// Candidates in [lo, nA) with a count of at least `need` into the level-0
// list (ascending); false when they do not fit.
template <int NB>
__device__ __forceinline__ bool list_by_slices(Wave& v, int m, int lo, int cap, int& n) {
  const int w_hi = (v.nA + 63) >> 6;
  n = 0;
  int ne = 0;
  for (int w0 = lo >> 6; w0 < w_hi; w0 += 64) {
    const int wd = w0 + v.lane;
    uint64_t s[NB];
    slice_count<NB>(v.L.B, v.L.gw, v.s.smp, m, wd, wd < w_hi, s);
    const uint64_t r = wd < w_hi ? range_bits(wd, lo, v.nA) : 0ull;
    uint64_t ge = slices_ge<NB>(s, v.need) & r;
    uint64_t rest = r & ~ge;
    v.lmax = max(v.lmax, slices_max<NB>(s, rest));
    // (the non-empty ones in the upper half: at most 4096 of either)
    const int c = popc64(ge) | popc64(slices_any<NB>(s, r)) << 16;
    int pos = wave_before(c, v.lane);
    const int both = uniform(__shfl(pos + c, 63, 64)), tot = both & 0xffff;
    if (n + tot > cap) return false;
    ne += both >> 16;
    pos = (pos & 0xffff) + n;
    while (ge) {
      v.s.idx[pos++] = (uint16_t)(wd * 64 + __builtin_ctzll(ge));
      ge &= ge - 1;
    }
    n += tot;
  }
  count_nodes(v, 3, v.nA - lo, ne, ne - n);
  wave_lds_sync();
  return true;
}

// Candidate bitmap of one level of the general walk: genes of [lo, nA) (and
// of `in`) with a count of at least `need`.
template <int NB>
__device__ __forceinline__ void bits_by_slices(Wave& v, int m, int depth, int lo, const uint64_t* in,
                                               uint64_t* out) {
  const int w_hi = (v.nA + 63) >> 6;
  int vis = 0, ne = 0, keep = 0;
  for (int w0 = lo >> 6; w0 < w_hi; w0 += 64) {
    const int wd = w0 + v.lane;
    uint64_t s[NB];
    slice_count<NB>(v.L.B, v.L.gw, v.s.smp, m, wd, wd < w_hi, s);
    uint64_t r = wd < w_hi ? range_bits(wd, lo, v.nA) : 0ull;
    if (in && r) r &= in[wd];
    const uint64_t ge = slices_ge<NB>(s, v.need) & r;
    uint64_t rest = r & ~ge;
    v.lmax = max(v.lmax, slices_max<NB>(s, rest));
    if (wd < w_hi) out[wd] = ge;
    vis += popc64(r);
    ne += popc64(slices_any<NB>(s, r));
    keep += popc64(ge);
  }
  ne = wave_sum(ne);
  count_nodes(v, depth, wave_sum(vis), ne, ne - wave_sum(keep));
}

// The slice count that holds m.
#define PDFS_BY_SLICES(m, call)                         \
  do {                                                  \
    if ((m) < 4) { constexpr int NB = 2; call; }        \
    else if ((m) < 16) { constexpr int NB = 4; call; }  \
    else if ((m) < 128) { constexpr int NB = 7; call; } \
    else { constexpr int NB = 11; call; }               \
  } while (0)

// The general walk below the pair (any number of samples and candidates):
// depth first, every level's candidates as a bitmap in the wave's scratch.
__device__ __forceinline__ void open_general(Wave& v, uint64_t y2, uint64_t* bits) {
  const int h = v.h, lane = v.lane;
  // level l (0-based) holds the candidates of depth l + 3 below prefix
  // (s.pre[0, l + 2)), whose intersection is s.y[l]
  int l = 0;
  // (s.y[0] holds y2)
  const int m2 = wave_sum(popc64(y2));
  if (count_by_rows(v, m2, v.b + 1)) {
    bits_by_rows(v, v.s.y, 3, v.b + 1, nullptr, bits);
  } else {
    list_samples(y2, v.s.smp, lane);
    PDFS_BY_SLICES(m2, (bits_by_slices<NB>(v, m2, 3, v.b + 1, nullptr, bits)));
  }
  __threadfence_block();
  int at = v.b + 1;
  for (;;) {
    const uint64_t* bm = bits + (size_t)l * v.L.gw;
    const int c = next_bit(bm, at, v.nA, lane);
    if (c < 0) {
      if (l == 0) break;
      --l;
      at = uniform(v.s.pre[l + 2]) + 1;   // past the gene whose subtree is done
      continue;
    }
    // prefix of l + 3 genes
    wave_lds_sync();
    if (lane == 0) v.s.pre[l + 2] = (uint16_t)c;
    uint64_t y = 0;
    if (lane < v.w64) y = v.s.y[l * kMaxW64 + lane] & v.T[(size_t)c * v.w64 + lane];
    const int cnt = wave_sum(popc64(y));
    v.inc = max(v.inc, load_inc(v));
    refresh_need(v);
    wave_lds_sync();
    pass_own_best(v, l + 3);
    at = c + 1;
    if (cnt < v.need) {
      v.lmax = max(v.lmax, cnt);
      count_nodes(v, l + 3, 0, 0, 1);
      continue;
    }
    const bool by_rows = count_by_rows(v, cnt, c + 1);
    const uint64_t* yl = v.s.y + (l + 1) * kMaxW64;
    if (lane < v.w64) v.s.y[(l + 1) * kMaxW64 + lane] = y;
    wave_lds_sync();
    if (!by_rows) list_samples(y, v.s.smp, lane);
    if (l + 4 == h) {
      if (by_rows) leaves_by_rows(v, yl, h - 1, c + 1, bm);
      else PDFS_BY_SLICES(cnt, (leaves_by_slices<NB>(v, cnt, h - 1, c + 1, bm)));
      continue;
    }
    uint64_t* nx = bits + (size_t)(l + 1) * v.L.gw;
    if (by_rows) bits_by_rows(v, yl, l + 4, c + 1, bm, nx);
    else PDFS_BY_SLICES(cnt, (bits_by_slices<NB>(v, cnt, l + 4, c + 1, bm, nx)));
    __threadfence_block();
    ++l;
  }
}

// The walk over the level lists (the pair's samples fit one mask word): level
// l's entries are candidates of depth l + 3 with their samples; entry i's
// children are the later entries of its list.
__device__ __forceinline__ void open_lists(Wave& v, int n0) {
  const int h = v.h, lane = v.lane;
  const int cap = h <= 5 ? 256 : 128;
  int l = 0;
  int n = n0, i = 0;
  // resume points of the suspended levels, one per lane
  int keep_n = 0, keep_i = 0;
  for (;;) {
    uint64_t* mk = v.s.mask + l * cap;
    uint16_t* ix = v.s.idx + l * cap;
    if (i + 1 >= n) {
      if (l == 0) break;
      --l;
      n = __builtin_amdgcn_readlane(keep_n, l);
      i = __builtin_amdgcn_readlane(keep_i, l) + 1;
      continue;
    }
    if (l == 0 && (i & 15) == 0) {
      v.inc = max(v.inc, load_inc(v));
      refresh_need(v);
    }
    const uint64_t mi = mk[i];
    const int ci = uniform(popc64(mi));
    if (ci < v.need) {
      v.lmax = max(v.lmax, ci);
      count_nodes(v, l + 3, 0, 0, 1);
      ++i;
      continue;
    }
    wave_lds_sync();
    if (lane == 0) v.s.pre[l + 2] = ix[i];
    wave_lds_sync();
    if (v.own) {
      pass_own_best(v, l + 3);
      if (ci < v.need) {
        v.lmax = max(v.lmax, ci);
        count_nodes(v, l + 3, 0, 0, 1);
        ++i;
        continue;
      }
    }
    int ne = 0;
    if (l + 4 == h) {
      for (int j0 = i + 1; j0 < n; j0 += kWave) {
        const int j = j0 + lane;
        const int tp = j < n ? popc64(mi & mk[j]) : 0;
        const bool hit = tp >= v.need;
        v.lmax = max(v.lmax, hit ? 0 : tp);
        ne += count_lanes(tp > 0);
        if (__any(hit)) {
          // the lists are walked in tuple order: a leaf found here precedes
          // every later one of the pair with its score
          if (score_leaves(v, h - 1, hit, j < n ? (int)ix[j] : 0, tp)) v.tie_s = v.bs;
          refresh_need(v);
        }
      }
      count_nodes(v, l + 4, n - i - 1, ne, 0);
      ++i;
      continue;
    }
    // the next level's list
    uint64_t* mo = mk + cap;
    uint16_t* io = ix + cap;
    int k = 0;
    for (int j0 = i + 1; j0 < n; j0 += kWave) {
      const int j = j0 + lane;
      const uint64_t mj = j < n ? (mi & mk[j]) : 0ull;
      const int tp = popc64(mj);
      const bool hit = tp >= v.need;
      v.lmax = max(v.lmax, hit ? 0 : tp);
      const unsigned long long hm = __ballot(hit);
      if (hit) {
        const int pos = rank_below(hm, k);
        mo[pos] = mj;
        io[pos] = ix[j];
      }
      k += __popcll(hm);
      ne += count_lanes(tp > 0);
    }
    count_nodes(v, l + 4, n - i - 1, ne, ne - k);
    wave_lds_sync();
    keep_n = lane == l ? n : keep_n;
    keep_i = lane == l ? i : keep_i;
    ++l;
    n = k;
    i = 0;
  }
}

// A candidate's samples as a mask over the pair's m <= 64 * MW.
template <int MW>
struct Mask {
  uint64_t w[MW];
};

template <int MW>
__device__ __forceinline__ int mask_count(const Mask<MW>& m) {
  int c = 0;
#pragma unroll
  for (int k = 0; k < MW; ++k) c += popc64(m.w[k]);
  return c;
}

// Every lane's candidate row cut to the samples of y2 (lane k: word k).
template <int MW>
__device__ __forceinline__ Mask<MW> sample_mask(const Wave& v, uint64_t y2, int ix, bool on) {
  Mask<MW> m;
#pragma unroll
  for (int k = 0; k < MW; ++k) m.w[k] = 0;
  const uint64_t* row = v.T + (size_t)(on ? ix : 0) * v.w64;
  int pos = 0;
  for (int k = 0; k < v.w64; ++k) {
    uint64_t yk = readlane64(y2, k);
    if (!yk) continue;
    const uint64_t r = on ? row[k] : 0ull;
    while (yk) {
      const uint64_t bit = ((r >> __builtin_ctzll(yk)) & 1ull) << (pos & 63);
      yk &= yk - 1;
#pragma unroll
      for (int i = 0; i < MW; ++i) m.w[i] |= i == (pos >> 6) ? bit : 0ull;
      ++pos;
    }
  }
  return m;
}

// The same walk over a list of at most 64 candidates held one per lane (gene
// ix, samples mk; `set`: the lanes of this level): an entry's children are the
// later lanes that share enough of its samples.  No LDS round trip per entry:
// 20 candidates at h = 5 take 13 us from the LDS lists, 7 us here; and masks
// of several words cost little more, where the general walk takes about 6 us a
// candidate (a pair with 100 samples and 49 candidates: 300 us).
template <int LV, int MW>
__device__ __forceinline__ void open_lanes(Wave& v, const Mask<MW>& mk, int ix,
                                           unsigned long long set) {
  const int lane = v.lane, h = v.h;
  int n = 0;
  while (set & (set - 1)) {   // the last entry has no later one
    const int i = __builtin_ctzll(set);
    set &= set - 1;
    if (LV == 0 && (++n & 15) == 0) {
      v.inc = max(v.inc, load_inc(v));
      refresh_need(v);
    }
    Mask<MW> mj;
    int ci = 0;
#pragma unroll
    for (int k = 0; k < MW; ++k) {
      const uint64_t mi = readlane64(mk.w[k], i);
      ci += __popcll(mi);
      mj.w[k] = mi & mk.w[k];
    }
    if (lane == 0) v.s.pre[LV + 2] = (uint16_t)__builtin_amdgcn_readlane(ix, i);
    if (v.own) {
      wave_lds_sync();
      pass_own_best(v, LV + 3);
    }
    if (ci < v.need) {
      v.lmax = max(v.lmax, ci);
      count_nodes(v, LV + 3, 0, 0, 1);
      continue;
    }
    const bool in = __builtin_amdgcn_inverse_ballot_w64(set);
    const int tp = in ? mask_count(mj) : 0;
    const bool hit = in && tp >= v.need;
    v.lmax = max(v.lmax, hit ? 0 : tp);
    const unsigned long long hm = __ballot(hit);
    const int ne = count_lanes(tp > 0);
    count_nodes(v, LV + 4, __popcll(set), ne, LV + 4 == h ? 0 : ne - __popcll(hm));
    if (!hm) continue;
    if (LV + 4 == h) {
      // in tuple order: a leaf found here precedes every later one of the
      // pair with its score
      if (score_leaves(v, h - 1, hit, ix, tp)) v.tie_s = v.bs;
      refresh_need(v);
    } else {
      if constexpr (LV + 4 < kMaxH) open_lanes<LV + 1, MW>(v, mj, ix, hm);
    }
  }
}

// (few samples: their words are fetched four at a time, in flight together)
template <int MW>
__device__ __forceinline__ void open_few(Wave& v, uint64_t y2, int m, int n) {
  const bool on = v.lane < n;
  const int ix = on ? (int)v.s.idx[v.lane] : 0;
  Mask<MW> mk;
  if (MW == 1 && m <= 24) {
    const uint64_t* row = v.T + (size_t)ix * v.w64;
    uint64_t x = 0;
    if (on) {
#pragma unroll 4
      for (int j = 0; j < m; ++j) {
        const int sid = v.s.smp[j];
        x |= ((row[sid >> 6] >> (sid & 63)) & 1ull) << j;
      }
    }
    mk.w[0] = x;
  } else {
    mk = sample_mask<MW>(v, y2, ix, on);
  }
  open_lanes<0, MW>(v, mk, ix, n < 64 ? (1ull << n) - 1ull : ~0ull);
}

// Opens the pair (a, b): every leaf below it that can beat (or tie with a
// smaller tuple) the incumbent is scored.  Returns an upper bound on the
// scores below the pair under the current mask (-1: none is non-empty).
__device__ __forceinline__ int open_pair(Wave& v, int a, int b, uint64_t* bits) {
  const int lane = v.lane;
  v.a = a;
  v.b = b;
  v.own = v.bs >= 0 && uniform(v.s.tup[0]) == a && uniform(v.s.tup[1]) == b;
  v.tie_s = -1;
  v.sub = -1;
  v.lmax = 0;
  const unsigned long long newest = load_inc(v);   // in flight with the rows
  uint64_t y2 = 0;
  if (lane < v.w64)
    y2 = v.T[(size_t)a * v.w64 + lane] & v.T[(size_t)b * v.w64 + lane] & v.u;
  const int m = wave_sum(popc64(y2));
  if (m == 0) return -1;
  v.inc = max(v.inc, newest);
  refresh_need(v);
  const int ub = v.P.p * m + v.P.q * v.P.n_normal;
  if (m < v.need) return ub;
  count_nodes(v, 2, 0, 0, 1);
  const bool by_rows = count_by_rows(v, m, b + 1);
  wave_lds_sync();
  if (lane == 0) {
    v.s.pre[0] = (uint16_t)a;
    v.s.pre[1] = (uint16_t)b;
  }
  if (lane < v.w64) v.s.y[lane] = y2;
  wave_lds_sync();
  if (m <= 64 || !by_rows) list_samples(y2, v.s.smp, lane);
  if (v.h == 3) {
    if (by_rows) leaves_by_rows(v, v.s.y, 2, b + 1, nullptr);
    else PDFS_BY_SLICES(m, (leaves_by_slices<NB>(v, m, 2, b + 1, nullptr)));
  } else {
    // more than 64 samples: a list only where one candidate per lane holds it
    int n = 0;
    bool listed = false;
    if (m <= kListSamples) {
      const int cap = m > 64 ? kWave : (v.h <= 5 ? 256 : 128);
      if (by_rows) listed = list_by_rows(v, v.s.y, b + 1, cap, n);
      else PDFS_BY_SLICES(m, listed = list_by_slices<NB>(v, m, b + 1, cap, n));
    }
    if (listed && n <= kWave) {
      if (m <= 64) open_few<1>(v, y2, m, n);
      else if (m <= 128) open_few<2>(v, y2, m, n);
      else open_few<4>(v, y2, m, n);
    } else if (listed) {
      // the candidates' samples as masks over the pair's
      for (int i0 = 0; i0 < n; i0 += kWave) {
        const int i = i0 + lane;
        if (i < n) {
          const uint64_t* row = v.T + (size_t)v.s.idx[i] * v.w64;
          uint64_t mk = 0;
#pragma unroll 4
          for (int j = 0; j < m; ++j) {
            const int sid = v.s.smp[j];
            mk |= ((row[sid >> 6] >> (sid & 63)) & 1ull) << j;
          }
          v.s.mask[i] = mk;
        }
      }
      wave_lds_sync();
      open_lists(v, n);
    } else {
      open_general(v, y2, bits);
    }
  }
  const int lm = wave_max(v.lmax);
  const int pr = lm > 0 ? v.P.p * lm + v.P.q * v.P.n_normal : -1;
  return min(ub, max(v.sub, pr));
}

// A first leaf below the pair (a, b): at every depth the candidate that keeps
// most samples.
__device__ __forceinline__ void dive(Wave& v, int a, int b) {
  const int lane = v.lane, h = v.h;
  v.a = a;
  v.b = b;
  v.own = false;
  v.tie_s = -1;
  v.need = 1;
  uint64_t y = 0;
  if (lane < v.w64) y = v.T[(size_t)a * v.w64 + lane] & v.T[(size_t)b * v.w64 + lane] & v.u;
  wave_lds_sync();
  if (lane == 0) {
    v.s.pre[0] = (uint16_t)a;
    v.s.pre[1] = (uint16_t)b;
  }
  wave_lds_sync();
  int last = b;
  for (int depth = 3; depth <= h; ++depth) {
    const int m = wave_sum(popc64(y));
    if (m == 0) return;
    const int hi = v.w.st->amax[depth];
    int best = 0, gene = -1;
    const bool by_rows = count_by_rows(v, m, last + 1);
    if (by_rows) {
      wave_lds_sync();
      if (lane < v.w64) v.s.y[lane] = y;
      wave_lds_sync();
      for (int d0 = last + 1; d0 < hi; d0 += kWave) {
        const int d = d0 + lane;
        const int tp = row_count(v, v.s.y, d, d < hi);
        const int c = wave_max(tp);
        if (c > best) {
          best = c;
          gene = wave_min(tp == c && d < hi ? d : 0x7fffffff);
        }
      }
    } else {
      list_samples(y, v.s.smp, lane);
    }
    const int w_hi = by_rows ? 0 : (hi + 63) >> 6;
    for (int w0 = (last + 1) >> 6; w0 < w_hi; w0 += 64) {
      const int wd = w0 + lane;
      uint64_t in = wd < w_hi ? range_bits(wd, last + 1, hi) : 0ull;
      int c = 0;
      PDFS_BY_SLICES(m, {
        uint64_t s[NB];
        slice_count<NB>(v.L.B, v.L.gw, v.s.smp, m, wd, wd < w_hi, s);
        c = slices_max<NB>(s, in);
      });
      if (c > best) {
        best = c;
        gene = wave_min(in ? wd * 64 + __builtin_ctzll(in) : 0x7fffffff);
      }
    }
    if (gene < 0) return;
    if (depth == h) {
      score_leaves(v, h - 1, lane == 0, gene, best);
      return;
    }
    wave_lds_sync();
    if (lane == 0) v.s.pre[depth - 1] = (uint16_t)gene;
    wave_lds_sync();
    if (lane < v.w64) y &= v.T[(size_t)gene * v.w64 + lane];
    last = gene;
  }
}

// h = 2: the chunk's pairs are the leaves.  Every lane whose pair can still
// win takes its exact score, which stays its bound.
__device__ __forceinline__ void chunk_h2(Wave& v, unsigned long long& e, bool nd, int ct,
                                         bool& changed) {
  const int a = (int)(e & 0xffff), b = (int)((e >> 16) & 0xffff);
  int fp = 0, sc = -1;
  if (nd && ct > 0) {
    const uint32_t* NA = v.w.NA;
    const bool lit = v.P.tn_literal != 0;
    const uint4* na = reinterpret_cast<const uint4*>(NA + (size_t)a * kMaxWN32);
    const uint4* nb = reinterpret_cast<const uint4*>(NA + (size_t)b * kMaxWN32);
#pragma unroll
    for (int k = 0; k < kMaxWN32 / 4; ++k) {   // rows are zero past the last normal
      const uint4 x = na[k], y = nb[k];
      fp += __popc(nrm_join(x.x, y.x, lit)) + __popc(nrm_join(x.y, y.y, lit)) +
            __popc(nrm_join(x.z, y.z, lit)) + __popc(nrm_join(x.w, y.w, lit));
    }
    sc = v.P.p * ct + v.P.q * (v.P.n_normal - fp);
    e = (e & 0xffffffffull) | ((unsigned long long)(uint32_t)sc << 32);
    changed = true;
  }
  const int smax = wave_max(sc);
  if (smax < 0 || smax < v.bs) return;
  // smallest (a, b) of the best score
  const int key = sc == smax ? (a << 15 | b >> 1) : 0x7fffffff;   // 31 bits of a << 16 | b
  const int kmin = wave_min(key);
  const int lowb = wave_min(key == kmin && sc == smax ? (b & 1) : 2);
  const unsigned long long at = __ballot(sc == smax && key == kmin && (b & 1) == lowb);
  const int src = __builtin_ctzll(at);
  const int ba = __builtin_amdgcn_readlane(a, src), bb = __builtin_amdgcn_readlane(b, src);
  wave_lds_sync();
  if (v.lane == 0) v.s.pre[0] = (uint16_t)ba;
  wave_lds_sync();
  take_leaf(v, smax, __builtin_amdgcn_readlane(ct, src), __builtin_amdgcn_readlane(fp, src), 1, bb);
  publish(v, smax, ba, bb);
}

// The answer of the launch before this one, for every wave of the block: the
// argmax of the leaves it left, in best (s = -1: none).
__device__ __forceinline__ void last_answer(const LazyWork& L, int n, int nA, int h, Slot* best) {
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x, ring = (n + 2) % 3;
    const Slot* wins = L.wins + (size_t)ring * (kLazyWaves / 4);
    const int n_win = (int)L.n_win[64 * ring];
    Slot b = empty_slot();
    for (int i = lane; i < n_win; i += kWave) {
      const Slot c = wins[i];
      slot_take_if(b, c, slot_better(c, b));
    }
    if (n_win > 1) b = wave_best(b);
    if (lane == 0) *best = b;
  }
  __syncthreads();
}

// The rows of work, summed in parts by the waves behind the first, which is busy
// with the answer.
constexpr int kWorkParts = (kBlock - kWave) / kLazyFields;

__device__ __forceinline__ unsigned long long rows_of_work(const LazyWork& L) {
  unsigned long long x = 0;
  if (threadIdx.x >= kWave) {
    const int f = threadIdx.x % kLazyFields, r0 = (threadIdx.x - kWave) / kLazyFields;
#pragma unroll
    for (int r = r0; r < kWorkRows; r += kWorkParts) x += L.tally[r * kLazyFields + f];
  }
  return x;
}

// The work that a finished run's launches counted, into the run's totals (the
// first block).  A pair's node is formed when it is listed, and again in a later
// round that counts it.  Under empty-intersection pruning the counters follow
// from an enumeration; only the leaves whose false positives were counted are
// taken from here.
__device__ __forceinline__ void total_work(const Problem& P, const Work& w, const LazyWork& L,
                                           int h, unsigned long long x) {
  __shared__ unsigned long long part[kWorkParts][kLazyFields];
  RoundState* st = w.st;
  const int tid = threadIdx.x, f = tid % kLazyFields;
  if (tid >= kWave) part[(tid - kWave) / kLazyFields][f] = x;
  __syncthreads();
  if (tid >= kLazyFields) return;
  x = 0;
#pragma unroll
  for (int r = 0; r < kWorkParts; ++r) x += part[r][f];
  if (f == kLfFp && h <= 4) st->tx_fp_leaves = x;
  if (P.mode != kPruneBound) return;
  const int d = 2 + f % 8;
  if (f < kLfFp && d <= h) {
    const unsigned long long listed = st->n_pairs;
    if (f < kLfNe) {
      st->tot.visited[d] = x + (d == 2 ? st->cnt.visited[2] : 0ull);
      if (d == 3 && h <= 4) st->tx_vis3 = x;
      if (d == 4 && h == 4) st->tx_vis4 = x;
    } else if (f < kLfBp) {
      st->tot.nonempty[d] = x + (d == 2 ? listed : 0ull);
      if (d == h && h >= 3 && h <= 4) st->tx_leaves = x;
    } else if (d < h) {
      // bp[2] holds the pairs opened: the others formed were pruned
      unsigned long long formed = listed;
      for (int r = 0; r < kWorkParts; ++r) formed += part[r][kLfNe];
      st->tot.bound_pruned[d] = d == 2 ? formed - x : x;
    }
  }
  if (f == kLfWords3 && h <= 4) st->tx_vis_words3 = x;
  if (f == kLfWords4 && h == 4) st->tx_vis_words4 = x;
  if (f == kLfFp) {
    st->tot.visited[1] = st->cnt.visited[1];
    st->tot.nonempty[1] = st->cnt.nonempty[1];
    const unsigned long long a1 = (unsigned long long)st->amax[1];
    const unsigned long long a2 = (unsigned long long)st->amax[2];
    st->tx_pair_macs = (a1 ? a1 * a2 - a1 * (a1 + 1) / 2 : 0) * (unsigned long long)L.uncs[0];
  }
}

// Commits it (the first block): the round's record, the state and the masks.
__device__ __forceinline__ void commit_answer(const Problem& P, const Work& w, const LazyWork& L,
                                              int h, const LazyState& z, const LazyState& nz,
                                              const Slot& best, bool found, uint64_t* un,
                                              bool early, unsigned long long work) {
  RoundState* st = w.st;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint64_t* T = reinterpret_cast<const uint64_t*>(w.TA);
  const uint64_t* uo = un == L.U2 ? L.U2 + kMaxW64 : L.U2;
  for (int k = tid >> 6; k < w.w64; k += kBlock / kWave) {
    const uint64_t u = uo[k];
    uint64_t cov = found ? u : 0ull;
    for (int i = 0; i < h && found; ++i) cov &= T[(size_t)best.idx[i] * w.w64 + k];
    const uint64_t left = u & ~cov;
    // a covered sample was uncovered in every round so far
    if ((cov >> lane) & 1ull) L.tcov[k * 64 + lane] = nz.executed;
    if (lane == 0) un[k] = left;
    if (nz.done) {   // the cohort's own mask follows when the run stops
      const int smp = k * 64 + lane;
      if (lane == 0) L.Uc[k] = left;
      if (smp < L.uncs[0] && !((left >> lane) & 1ull)) {
        const int c = w.cols[smp];
        atomicAnd(reinterpret_cast<unsigned long long*>(&w.U[c >> 6]), ~(1ull << (c & 63)));
      }
    }
  }
  // (the genes' caller ids are looked up where the record is read)
  RoundRecord* rec = found && z.rounds < w.rec_cap ? w.recs + z.rounds : nullptr;
  if (rec && tid >= 64 && tid < 64 + kMaxH) {
    const int i = tid - 64;
    rec->sorted_idx[i] = i < h ? w.act[best.idx[i]] : -1;
    rec->genes[i] = -1;
  }
  if (tid == 0) {
    if (rec) {
      rec->h = h;
      rec->found = 1;
      rec->tp = best.tp;
      rec->fp = best.fp;
      rec->tn = P.n_normal - best.fp;
      rec->uncovered_before = z.n_unc;
      rec->score_num = (int64_t)P.p * best.tp + (int64_t)P.q * (P.n_normal - best.fp);
      rec->score_den = (int64_t)P.q * (int64_t)(z.n_unc + P.n_normal);
    }
    st->found = found;
    if (nz.executed < P.n_tumor + 2) L.uncs[nz.executed] = nz.n_unc;
    st->covered = P.n_tumor - nz.n_unc;
    st->n_unc = nz.n_unc;
    st->rounds = nz.rounds;
    st->executed = nz.executed;
    st->done = nz.done;
  }
  if (nz.done && L.tally) total_work(P, w, L, h, early ? work : rows_of_work(L));
}

// H: the combination size, or 0 for 5..9 (taken from P).
template <int H>
__global__ __launch_bounds__(256) void k_lazy_round(Problem P, Work w, LazyWork L, int n,
                                                    int search) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ Slot wave_slot[kBlock / kWave];
  __shared__ unsigned long long wave_key[kBlock / kWave];
  __shared__ Slot s_best;
  __shared__ unsigned long long wave_work[kBlock / kWave][kLazyFields];
  RoundState* st = w.st;
  const int lane = threadIdx.x & 63;
  const int wib = uniform(threadIdx.x >> 6);
  const int wv = blockIdx.x * (kBlock / kWave) + wib;
  const int h = H > 0 ? H : P.h;
  const uint64_t* T = reinterpret_cast<const uint64_t*>(w.TA);
  const int cur = n & 1;
  const LazyState z = L.S[cur ^ 1];
  if (z.done) {   // launches queued past the stop hand the state on
    if (blockIdx.x == 0 && threadIdx.x == 0) L.S[cur] = z;
    return;
  }
  const int nA = uniform(st->nA);
  uint64_t u = lane < w.w64 ? L.U2[(cur ^ 1) * kMaxW64 + lane] : 0ull;
  // the best leaf this wave knows from earlier rounds: its rows are on their
  // way while the last round's answer is taken
  const Slot pool = L.pool[wv];
  uint64_t py = ~0ull;
  if (uniform(pool.s) >= 0) {
#pragma unroll
    for (int i = 0; i < kMaxH; ++i)
      if (i < h && lane < w.w64) py &= T[(size_t)pool.idx[i] * w.w64 + lane];
  }
  LazyState nz = z;
  // (a launch that only commits may end the run: its rows of work, meanwhile)
  const bool early = !search && L.tally;
  const unsigned long long work = early ? rows_of_work(L) : 0ull;
  if (z.searched) {
    last_answer(L, n, nA, h, &s_best);
    const Slot& best = s_best;
    bool found = best.s >= 0;
    if (found) {
      bool ok = best.tp > 0;
      for (int i = 0; i < h; ++i)
        ok = ok && best.idx[i] >= 0 && best.idx[i] < nA && (i == 0 || best.idx[i] > best.idx[i - 1]);
      if (!ok) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->overflow |= 2;
        found = false;
      }
    }
    const int tp = found ? best.tp : 0;
    const int max_rounds = st->max_rounds;
    nz.n_unc = z.n_unc - tp;
    nz.executed = z.executed + 1;
    nz.rounds = z.rounds + (found ? 1 : 0);
    const int cov = P.n_tumor - nz.n_unc;
    nz.done = !found || cov >= w.target || cov >= P.n_tumor ||
              (max_rounds > 0 && nz.rounds >= max_rounds);
    if (found && lane < w.w64) {
      uint64_t c = u;
      for (int i = 0; i < h; ++i) c &= T[(size_t)best.idx[i] * w.w64 + lane];
      u &= ~c;
    }
    if (blockIdx.x == 0)
      commit_answer(P, w, L, h, z, nz, best, found, L.U2 + cur * kMaxW64,
                    early, work);
  } else if (blockIdx.x == 0 && threadIdx.x < w.w64) {
    L.U2[cur * kMaxW64 + lane] = u;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      nz.searched = search;
      L.S[cur] = nz;
      // cleared for the next launch; last used by the one before this
      L.n_win[64 * ((n + 1) % 3)] = 0u;
      L.inc[(cur ^ 1) * kCursorStride] = 0ull;
    }
    if (threadIdx.x < kIncShards)
      L.shard[((cur ^ 1) * kIncShards + threadIdx.x) * kCursorStride] = 0ull;
  }
  if (nz.done || !search) return;

  Wave v{P, w, L, wave_lds(lds + (size_t)wib * L.wave_bytes, h), T};
  v.lane = lane;
  v.nA = nA;
  v.w64 = w.w64;
  v.h = h;
  v.u = u;
  v.incp = L.inc + cur * kCursorStride;
  v.shard = L.shard + cur * kIncShards * kCursorStride;
  v.inc = 0;
  v.bs = -1;
  v.btp = v.bfp = 0;
  v.a = v.b = 0;
  v.own = false;
  v.tie_s = -1;
  v.need = 1;
  v.sub = -1;
  v.lmax = 0;
  v.work = 0;
  v.ne3 = 0u;
  wave_lds_sync();
  if (lane < w.w64) v.s.y[(kMaxH - 1) * kMaxW64 + lane] = v.u;   // the mask, for lane-wise counts
  const uint64_t* um = v.s.y + (kMaxH - 1) * kMaxW64;
  wave_lds_sync();

  // the wave's known leaf under the new mask
  if (uniform(pool.s) >= 0) {
    const int tp = wave_sum(popc64(py & v.u));
    if (tp > 0) {
      v.bfp = uniform(pool.fp);
      v.btp = tp;
      v.bs = P.p * tp + P.q * (P.n_normal - v.bfp);
#pragma unroll
      for (int i = 0; i < kMaxH; ++i)
        if (i < h && lane == i) v.s.tup[i] = (uint16_t)pool.idx[i];
      wave_lds_sync();
    }
  }
  // published once per block
  {
    const unsigned long long key = v.bs >= 0 ? leaf_key(v.bs, v.s.tup[0], v.s.tup[1]) : 0ull;
    if (lane == 0) wave_key[wib] = key;
    __syncthreads();
    unsigned long long top = wave_key[0];
    for (int i = 1; i < kBlock / kWave; ++i) top = max(top, wave_key[i]);
    if (wib == 0 && top > 0) publish_key(v, top);
    v.inc = max(v.inc, top);
  }

  const unsigned long long E = st->n_pairs < w.pair_cap ? st->n_pairs : w.pair_cap;
  const int n_mine = (unsigned long long)wv < E
                         ? (int)((E - (unsigned long long)wv + (unsigned long long)L.nw - 1ull) /
                                 (unsigned long long)L.nw)
                         : 0;
  const int n_chunk = (n_mine + kWave - 1) / kWave;
  unsigned long long* list = L.list + (size_t)wv * L.seg;
  int32_t* cmax = L.cmax + (size_t)wv * ((L.seg + kWave - 1) / kWave);
  uint64_t* bits = L.bits + (size_t)wv * L.levels * L.gw;

  // No incumbent yet (a run's first round): a greedy leaf below the wave's
  // best pair first, so that the pairs are opened against something.
  if (h >= 3 && n_mine > 0 && v.inc == 0) {
    const unsigned long long e = list[0];
    dive(v, uniform((int)(e & 0xffff)), uniform((int)((e >> 16) & 0xffff)));
    v.work = 0;   // (a leaf that is met again below its pair)
  }

  for (int k0 = 0; k0 < n_chunk; k0 += kWave) {
    const int cm = k0 + lane < n_chunk ? cmax[k0 + lane] : -1;
    v.inc = max(v.inc, load_inc(v));
    unsigned long long todo = __ballot(cm >= 0 && cm >= (int)(v.inc >> 32) - 1);
    while (todo) {
      const int kc = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int i = (k0 + kc) * kWave + lane;
      unsigned long long e = i < n_mine ? list[i] : (0xffffffffull << 32);
      const int a = (int)(e & 0xffff), b = (int)((e >> 16) & 0xffff);
      bool changed = false;
      int sb = (int)(e >> 32);
      bool nd = sb >= 0 && !dominated(sb, a, b, v.inc);
      int ct = 0;
      if (__any(nd)) {
        // today's count of the pairs in reach, one per lane
        if (nd) {
          ct = pair_count(v.T + (size_t)a * w.w64, v.T + (size_t)b * w.w64, um, w.w64);
          const int ub = ct > 0 ? P.p * ct + P.q * P.n_normal : -1;
          if (ub < sb) {
            sb = ub;
            changed = true;
          }
        }
        // (the first round's are counted as they are listed)
        if (nz.executed > 0) count_nodes(v, 2, count_lanes(nd), count_lanes(ct > 0), 0);
        nd = nd && sb >= 0 && !dominated(sb, a, b, v.inc);
        if (h == 2) {
          e = (e & 0xffffffffull) | ((unsigned long long)(uint32_t)sb << 32);
          chunk_h2(v, e, nd, ct, changed);
          sb = (int)(e >> 32);
        } else {
          for (;;) {
            // the largest bound in reach first
            nd = nd && !dominated(sb, a, b, v.inc);
            const int top = wave_max(nd ? sb : -1);
            if (top < 0) break;
            const int src = __builtin_ctzll(__ballot(nd && sb == top));
            const int pa = __builtin_amdgcn_readlane(a, src);
            const int pb = __builtin_amdgcn_readlane(b, src);
            const int nb = open_pair(v, pa, pb, bits);
            if (lane == src) {
              if (nb < sb) {
                sb = nb;
                changed = true;
              }
              nd = false;
            }
          }
        }
      }
      if (__any(changed)) {
        if (i < n_mine)
          list[i] = (e & 0xffffffffull) | ((unsigned long long)(uint32_t)sb << 32);
        const int mx = wave_max(i < n_mine ? sb : -1);
        if (lane == 0) cmax[k0 + kc] = mx;
      }
    }
  }

  // the wave's best leaf stays its pool leaf
  Slot sl = empty_slot();
  wave_lds_sync();
  if (v.bs >= 0) {
    sl.s = v.bs;
    sl.tp = v.btp;
    sl.fp = v.bfp;
#pragma unroll
    for (int i = 0; i < kMaxH; ++i) sl.idx[i] = i < h ? (int)v.s.tup[i] : 0;
  }
  if (lane == 0) {
    L.pool[wv] = sl;
    wave_slot[wib] = sl;
  }
  if (L.tally) {
    unsigned long long x = (unsigned long long)v.work;
    if (h == 3) {
      const int ne3 = wave_sum((int)v.ne3);
      if (lane == kLfNe + 1) x += (unsigned long long)ne3;
    }
    if (h == 3 || h == 4) {
      const unsigned long long words = (unsigned long long)((nz.n_unc + 63) / 64);
      const unsigned long long x3 = readlane64(x, 1), x4 = readlane64(x, 2);
      if (lane == kLfWords3) x = x3 * words;
      if (lane == kLfWords4) x = x4 * words;
    }
    if (lane < kLazyFields) wave_work[wib][lane] = x;
  }
  __syncthreads();
  if (L.tally && wib == kBlock / kWave - 1 && lane < kLazyFields) {   // (the first one is busy)
    unsigned long long x = 0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) x += wave_work[i][lane];
    if (x) atomicAdd(&L.tally[(blockIdx.x % kWorkRows) * kLazyFields + lane], x);
  }
  if (threadIdx.x == 0) {
    Slot r = wave_slot[0];
    for (int i = 1; i < kBlock / kWave; ++i)
      slot_take_if(r, wave_slot[i], slot_better(wave_slot[i], r));
    // only a leaf that the incumbent does not beat can be the answer
    const unsigned long long inc = load_inc(v);
    if (r.s >= 0 && leaf_key(r.s, r.idx[0], r.idx[1]) >= inc) {
      const uint32_t pos = atomicAdd(&L.n_win[64 * (n % 3)], 1u);
      L.wins[(size_t)(n % 3) * (kLazyWaves / 4) + pos] = r;   // one per block at most
    }
  }
}

}  // namespace

int lazy_levels(int h) { return kLazyLevels(h); }

hipError_t launch_lazy_begin(const Problem& P, const Work& w, const LazyWork& L, hipStream_t s) {
  const int tiles = L.gw * w.w64;
  int blocks = (tiles + 3) / 4;
  if (blocks > 2048) blocks = 2048;
  k_lazy_begin<<<blocks, kBlock, 0, s>>>(P, w, L);
  return hipGetLastError();
}

hipError_t launch_list_pairs(const Work& w, const LazyWork& L, int nA_max, hipStream_t s) {
  int blocks = (nA_max + kListWaves - 1) / kListWaves;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  k_list_pairs<<<blocks, kListWaves * 64, 0, s>>>(w, L);
  return hipGetLastError();
}

hipError_t launch_lazy_deal(const Problem& P, const Work& w, const LazyWork& L, hipStream_t s) {
  unsigned long long blocks = (w.pair_cap + kDeal - 1) / kDeal;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  k_lazy_deal<<<(int)blocks, kBlock, 0, s>>>(P, w, L);
  return hipGetLastError();
}

hipError_t launch_lazy_round(const Problem& P, const Work& w, const LazyWork& L0, int n,
                             bool search, hipStream_t s) {
  LazyWork L = L0;
  L.wave_bytes = (int)lazy_wave_bytes(P.h);
  const size_t lds = (size_t)L.wave_bytes * (kBlock / kWave);
  const int blocks = search ? L.nw / (kBlock / kWave) : 1;
  const int sr = search ? 1 : 0;
  switch (P.h) {
    case 2: k_lazy_round<2><<<blocks, kBlock, lds, s>>>(P, w, L, n, sr); break;
    case 3: k_lazy_round<3><<<blocks, kBlock, lds, s>>>(P, w, L, n, sr); break;
    case 4: k_lazy_round<4><<<blocks, kBlock, lds, s>>>(P, w, L, n, sr); break;
    default: k_lazy_round<0><<<blocks, kBlock, lds, s>>>(P, w, L, n, sr); break;
  }
  return hipGetLastError();
}

}  // namespace pdfs
