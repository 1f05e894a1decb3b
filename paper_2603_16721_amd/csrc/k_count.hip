// The counters of an empty-intersection run (Alg. 2's visited and non-empty
// nodes, summed over its rounds), from one enumeration after the last round.
//
// A node is non-empty in every round that starts with one of its samples
// uncovered, so over a whole run it counts t = max t_s times, t_s being the
// number of rounds that found sample s uncovered.  With the samples in order
// of falling t that is the t of the node's first sample, and the run's
// counters are sums over the nodes of its first round: every non-empty node
// once, weighted, instead of once a round.
//
//  - A pair (or deeper prefix) left with a single sample has the rest of that
//    sample's gene list below it and nothing else: binomials, and suffix sums
//    along the list for the visited counts (one lane per pair; most pairs of
//    a sparse cohort).
//  - A pair with more samples lists the genes that meet it (the union of its
//    samples' rows of B) with their samples compressed to a 64-bit mask, and
//    its subtree is enumerated over that list, down to single-sample
//    prefixes; one wave per pair.
//  - Pairs with more than 64 samples, or more candidates than the list holds,
//    are walked depth first with candidate bitmaps.
//
// The counts of candidates over active genes (dfs_visits) need, for a prefix
// that lives t rounds and ends in gene b, the sum over later genes c of
// min(t, t_c): a table over t and every eighth gene, finished from the t_c of
// the genes in between.
#include "dfs_core.h"
#include "lazy_core.h"
#include "pdfs_dev.h"
#include "slot_reduce.h"

namespace pdfs {

namespace {

// Counter row of a block (kTallyN fields).
enum CountField {
  kCNe2 = 0,
  kCVis3 = 1,
  kCNe3 = 2,     // nonempty[3..9]: fields 2..8
  kCVis4 = 9,    // visited[4..9]: fields 9..14
  // h <= 4 (visited[5..] do not exist there)
  kCXv3 = 10,
  kCXw3 = 11,
  kCXv4 = 12,
  kCXw4 = 13
};

constexpr int kTabGenes = 8;      // genes per table row
constexpr int kTabSeg = 512;      // genes per block of the table kernels

// ------------------------------------------------------------- sample order
// One block: rounds per sample, the samples in order of falling rounds, and
// the row words of the first k rounds (wc[k]).
__global__ __launch_bounds__(1024) void k_count_order(Work w, LazyWork L, CountWork C) {
  __shared__ uint32_t hist[kCountMaxT + 2];
  __shared__ uint32_t part[1024];
  const int tid = threadIdx.x;
  const int n0 = L.uncs[0], R = min(w.st->executed, kCountMaxT);
  for (int i = tid; i < kCountMaxT + 2; i += 1024) hist[i] = 0u;
  __syncthreads();
  int t[2] = {0, 0};
  for (int u = 0; u < 2; ++u) {
    const int s = tid + 1024 * u;
    if (s >= n0) continue;
    t[u] = (L.Uc[s >> 6] >> (s & 63)) & 1ull ? R : min(L.tcov[s], R);
    atomicAdd(&hist[t[u]], 1u);
  }
  __syncthreads();
  // two scans over the rounds, two entries per thread: samples with more
  // rounds, and row words of earlier rounds
  auto scan = [&](uint32_t x, uint32_t y, uint32_t& before) {
    part[tid] = x + y;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const uint32_t add = tid >= o ? part[tid - o] : 0u;
      __syncthreads();
      part[tid] += add;
      __syncthreads();
    }
    before = part[tid] - x - y;
    __syncthreads();
  };
  {
    const int v0 = R - 2 * tid, v1 = v0 - 1;
    const uint32_t x = v0 >= 0 ? hist[v0] : 0u, y = v1 >= 0 ? hist[v1] : 0u;
    uint32_t run;
    scan(x, y, run);
    if (v0 >= 0) hist[v0] = run;
    if (v1 >= 0) hist[v1] = run + x;
    const int r0 = 2 * tid, r1 = r0 + 1;
    const uint32_t a = r0 < R ? (uint32_t)((L.uncs[r0] + 63) / 64) : 0u;
    const uint32_t b = r1 < R ? (uint32_t)((L.uncs[r1] + 63) / 64) : 0u;
    scan(a, b, run);
    if (tid == 0) C.wc[0] = 0;
    if (r0 < R) C.wc[r0 + 1] = run + a;
    if (r1 < R) C.wc[r1 + 1] = run + a + b;
  }
  __syncthreads();
  for (int u = 0; u < 2; ++u) {
    const int s = tid + 1024 * u;
    if (s >= n0) continue;
    const uint32_t p = atomicAdd(&hist[t[u]], 1u);
    C.order[p] = s;
    C.tt[p] = t[u];
  }
  for (int p = n0 + tid; p < 64 * kMaxW64; p += 1024) {
    C.order[p] = 0;
    C.tt[p] = 0;
  }
}

// Rows over the reordered samples (written over the run's rows), and each
// sample's gene count before every word of its row.
__global__ __launch_bounds__(256) void k_count_rows(Work w, LazyWork L, CountWork C) {
  const int lane = threadIdx.x & 63;
  const int wv = blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
  const int waves = gridDim.x * (kBlock / kWave);
  const int n0 = L.uncs[0], nA = w.st->nA;
  uint64_t* T = reinterpret_cast<uint64_t*>(w.TA);
  const int tiles = L.gw * w.w64;
  for (int t = wv; t < tiles; t += waves) {
    const int gq = t / w.w64, sw = t % w.w64;
    const int p = sw * 64 + lane;
    const uint64_t x = p < n0 ? L.B[(size_t)C.order[p] * L.gw + gq] : 0ull;
    uint64_t mine = 0;
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      const unsigned long long row = __ballot((x >> j) & 1ull);
      mine = lane == j ? row : mine;
    }
    const int g = gq * 64 + lane;
    if (g < nA) T[(size_t)g * w.w64 + sw] = mine;
  }
  for (int p = wv; p < n0; p += waves) {
    const uint64_t* row = L.B + (size_t)C.order[p] * L.gw;
    int base = 0;
    for (int w0 = 0; w0 < L.gw; w0 += 64) {
      const int wd = w0 + lane;
      const int c = wd < L.gw ? popc64(row[wd]) : 0;
      const int before = wave_before(c, lane);
      if (wd < L.gw) C.pref[(size_t)p * L.gw + wd] = (uint16_t)(base + before);
      base += uniform(__shfl(before + c, 63, 64));
    }
    if (lane == 0) C.kc[p] = base;
  }
}

// Rounds per gene (its first sample's), and per segment of genes the sums of
// min(t, t_g) and wc[min(t, t_g)] for every t.
__global__ __launch_bounds__(256) void k_count_genes(Work w, LazyWork L, CountWork C, int tables) {
  __shared__ uint16_t tg[kTabSeg];
  const int nA = w.st->nA, R = min(w.st->executed, kCountMaxT);
  const int g0 = blockIdx.x * kTabSeg;
  const uint64_t* T = reinterpret_cast<const uint64_t*>(w.TA);
  for (int i = threadIdx.x; i < kTabSeg; i += kBlock) {
    const int g = g0 + i;
    int t = 0;
    if (g < nA) {
      for (int k = 0; k < w.w64; ++k) {
        const uint64_t x = T[(size_t)g * w.w64 + k];
        if (x) {
          t = C.tt[k * 64 + __builtin_ctzll(x)];
          break;
        }
      }
    }
    tg[i] = (uint16_t)t;
    C.tg[g] = (uint16_t)t;   // [whole segments]
  }
  __syncthreads();
  if (!tables) return;
  for (int t = threadIdx.x; t <= R; t += kBlock) {
    uint32_t a = 0, b = 0;
    for (int i = 0; i < kTabSeg; ++i) {
      const int m = min(t, (int)tg[i]);
      a += (uint32_t)m;
      b += C.wc[m];
    }
    C.seg_v[(size_t)blockIdx.x * (R + 1) + t] = a;
    C.seg_w[(size_t)blockIdx.x * (R + 1) + t] = b;
  }
}

// The tables: row k, entry t = the sums over the genes from kTabGenes * k on.
__global__ __launch_bounds__(256) void k_count_tables(Work w, LazyWork L, CountWork C, int segs) {
  __shared__ uint16_t tg[kTabSeg];
  const int R = min(w.st->executed, kCountMaxT);
  const int sg = blockIdx.x;
  for (int i = threadIdx.x; i < kTabSeg; i += kBlock) tg[i] = C.tg[sg * kTabSeg + i];
  __syncthreads();
  for (int t = threadIdx.x; t <= R; t += kBlock) {
    uint32_t a = 0, b = 0;
    for (int s = sg + 1; s < segs; ++s) {
      a += C.seg_v[(size_t)s * (R + 1) + t];
      b += C.seg_w[(size_t)s * (R + 1) + t];
    }
    const size_t row0 = (size_t)sg * (kTabSeg / kTabGenes);
    if (sg == segs - 1) {
      C.tab_v[(row0 + kTabSeg / kTabGenes) * (R + 1) + t] = 0;
      C.tab_w[(row0 + kTabSeg / kTabGenes) * (R + 1) + t] = 0;
    }
    for (int k = kTabSeg / kTabGenes - 1; k >= 0; --k) {
#pragma unroll
      for (int i = kTabGenes - 1; i >= 0; --i) {
        const int m = min(t, (int)tg[k * kTabGenes + i]);
        a += (uint32_t)m;
        b += C.wc[m];
      }
      C.tab_v[(row0 + k) * (R + 1) + t] = a;
      C.tab_w[(row0 + k) * (R + 1) + t] = b;
    }
  }
}

// Sum over the genes c > b of min(t, t_c) and of wc[min(t, t_c)].
__device__ __forceinline__ void later_visits(const CountWork& C, int R, int b, int t,
                                             unsigned long long& v, unsigned long long& wv) {
  const int k = b / kTabGenes;
  const uint4 q = *reinterpret_cast<const uint4*>(C.tg + (size_t)k * kTabGenes);
  uint32_t a = C.tab_v[(size_t)(k + 1) * (R + 1) + t];
  uint32_t x = C.tab_w[(size_t)(k + 1) * (R + 1) + t];
  const uint32_t pk[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 1; i < kTabGenes; ++i) {
    if (i > b % kTabGenes) {
      const int m = min(t, (int)((pk[i >> 1] >> (16 * (i & 1))) & 0xffff));
      a += (uint32_t)m;
      x += C.wc[m];
    }
  }
  v = a;
  wv = x;
}

// One block: where each sample's list starts.
__global__ __launch_bounds__(1024) void k_count_offsets(LazyWork L, CountWork C) {
  __shared__ uint32_t part[1024];
  const int tid = threadIdx.x, n0 = L.uncs[0];
  const uint32_t a = 2 * tid < n0 ? (uint32_t)C.kc[2 * tid] : 0u;
  const uint32_t b = 2 * tid + 1 < n0 ? (uint32_t)C.kc[2 * tid + 1] : 0u;
  part[tid] = a + b;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const uint32_t add = tid >= o ? part[tid - o] : 0u;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  const uint32_t base = part[tid] - a - b;
  if (2 * tid < n0) C.off[2 * tid] = base;
  if (2 * tid + 1 < n0) C.off[2 * tid + 1] = base + a;
}

__device__ __forceinline__ unsigned long long shfl64(unsigned long long v, int src) {
  return (unsigned long long)__shfl((long long)v, src, 64);
}

// Sum of v over the lanes above this one; total in `all`.
__device__ __forceinline__ unsigned long long wave_after(unsigned long long v, int lane,
                                                         unsigned long long& all) {
  unsigned long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long x = (unsigned long long)__shfl_down((long long)incl, o, 64);
    if (lane + o < 64) incl += x;
  }
  all = shfl64(incl, 0);
  return incl - v;
}

// One wave per sample: its genes in order, and along the list
//   q[i - 1][pos] = sum over the i-subsets of the later genes of the largest
//                   one's sorted index (i = 1 .. h - 3),
//   and for h = 4 the later genes' later_visits sums.
__global__ __launch_bounds__(256) void k_count_lists(Problem P, Work w, LazyWork L, CountWork C) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
  if (p >= L.uncs[0]) return;
  const int R = min(w.st->executed, kCountMaxT), h = P.h;
  const uint64_t* row = L.B + (size_t)C.order[p] * L.gw;
  const size_t off = C.off[p];
  const int n = C.kc[p], t = C.tt[p];
  for (int wd = lane; wd < L.gw; wd += kWave) {
    uint64_t x = row[wd];
    size_t pos = off + C.pref[(size_t)p * L.gw + wd];
    while (x) {
      C.genes[pos++] = (uint16_t)(wd * 64 + __builtin_ctzll(x));
      x &= x - 1;
    }
  }
  __threadfence_block();
  // genes above the depth-L loop bound G - 1 - (h - L), by h - L
  if (lane >= 1 && lane < kMaxH) {
    int e = 0;
    for (int i = n - 1; i >= 0 && i >= n - lane; --i)
      e += w.act[C.genes[off + i]] > P.G - 1 - lane ? 1 : 0;
    C.ecnt[(size_t)p * 16 + lane] = (uint8_t)e;
  }
  if (lane == 0) C.ecnt[(size_t)p * 16] = 0;
  const int nq = h - 3;
  unsigned long long carry[kMaxH - 3] = {0};
  unsigned long long cv = 0, cw = 0;
  for (int hi = n; hi > 0; hi -= kWave) {
    const int i = hi - kWave + lane;
    const bool ok = i >= 0;
    const int g = ok ? (int)C.genes[off + i] : 0;
    unsigned long long v = ok ? (unsigned long long)w.act[g] : 0ull, all;
#pragma unroll
    for (int k = 0; k < kMaxH - 3; ++k) {
      if (k < nq) {
        const unsigned long long q = carry[k] + wave_after(v, lane, all);
        carry[k] += all;
        if (ok) C.q[(size_t)k * C.q_n + off + i] = q;
        v = ok ? q : 0ull;
      }
    }
    if (h == 4) {
      unsigned long long a = 0, b = 0;
      if (ok) later_visits(C, R, g, t, a, b);
      const unsigned long long sv = cv + wave_after(a, lane, all);
      cv += all;
      const unsigned long long sw = cw + wave_after(b, lane, all);
      cw += all;
      if (ok) {
        C.sv[off + i] = sv;
        C.sw[off + i] = sw;
      }
    }
  }
}

// ------------------------------------------------------------- enumeration
constexpr int count_cap(int h) { return h <= 4 ? 384 : (h == 5 ? 256 : 192); }
constexpr int count_levels(int h) { return h <= 4 ? 1 : h - 3; }

// A wave's share of LDS.
struct CountLds {
  uint64_t* mask;            // [levels][cap]
  uint64_t* y;               // [levels + 1][kMaxW64]
  uint32_t* ts;              // [kWave] rounds of the pair's samples
  uint16_t* idx;             // [levels][cap]
  uint16_t* smp;             // [kMaxCount]
};

size_t count_wave_bytes(int h) {
  const size_t lv = (size_t)count_levels(h), cap = (size_t)count_cap(h);
  const size_t b = lv * cap * 8 + (lv + 1) * kMaxW64 * 8 + kWave * 4 + lv * cap * 2 + kMaxCount * 2;
  return (b + 15) / 16 * 16;
}

__device__ __forceinline__ CountLds count_lds(char* p, int h) {
  const int lv = count_levels(h), cap = count_cap(h);
  CountLds s;
  s.mask = reinterpret_cast<uint64_t*>(p);
  s.y = s.mask + lv * cap;
  s.ts = reinterpret_cast<uint32_t*>(s.y + (lv + 1) * kMaxW64);
  s.idx = reinterpret_cast<uint16_t*>(s.ts + kWave);
  s.smp = s.idx + lv * cap;
  return s;
}

// Depths are template arguments throughout, so that the per-lane sums of every
// depth stay in registers.
template <int H>
struct Count {
  const Problem& P;
  const Work& w;
  const LazyWork& L;
  const CountWork& C;
  CountLds s;
  const uint64_t* T;
  const uint16_t* order;   // LDS: [kMaxCount] samples by falling rounds
  const uint16_t* tt;      // LDS: their rounds
  int lane, nA, w64, h, R;
  unsigned long long ne2, vis3, xv3, xw3, xv4, xw4;
  unsigned long long ne[kMaxH + 1], vis[kMaxH + 1];   // depths 3.., 4..

  // 0-based loop bound of depth l
  __device__ __forceinline__ int lim(int l) const { return P.G - h + l - 1; }

  __device__ __forceinline__ const uint64_t* brow(int p) const {
    return L.B + (size_t)order[p] * L.gw;
  }

  // Position of gene g in the list of sample p (which carries it).
  __device__ __forceinline__ int pos_in(int p, int g) const {
    const int wd = g >> 6;
    return (int)C.pref[(size_t)p * L.gw + wd] +
           popc64(brow(p)[wd] & ((1ull << (g & 63)) - 1ull));
  }

  // Everything below a depth-l prefix whose only sample is p and whose last
  // gene is at `pos` of the sample's list.
  template <int l>
  __device__ __forceinline__ void below_single(int p, int pos, unsigned long long t) {
    const int n = C.kc[p];
    const size_t off = C.off[p];
    constexpr int top = H > 0 ? H : kMaxH;
#pragma unroll
    for (int i = 1; l + i <= top; ++i) {
      const int d = l + i;   // depth counted
      if (d > h) continue;
      const int e = C.ecnt[(size_t)p * 16 + (h - d)];
      const int r = n - 1 - pos - e;
      unsigned long long c = 1;
#pragma unroll
      for (int k = 1; k <= i; ++k)
        c = c * (unsigned long long)(r - k + 1 > 0 ? r - k + 1 : 0) / (unsigned long long)k;
      ne[d] += t * c;
      if (d + 1 > h) continue;
      // visits below them: sum of lim(d + 1) - largest index
      unsigned long long q = C.q[(size_t)(i - 1) * C.q_n + off + pos];
      for (int x = 0; x < e; ++x) {   // subsets ending above the bound do not count
        const int at = n - 1 - x;
        const int u = at - pos;       // 1-based among the later genes
        unsigned long long b = 1;
#pragma unroll
        for (int k = 1; k <= i - 1; ++k)
          b = b * (unsigned long long)(u - k > 0 ? u - k : 0) / (unsigned long long)k;
        q -= b * (unsigned long long)w.act[C.genes[off + at]];
      }
      if (d + 1 <= kMaxH) vis[d + 1 <= kMaxH ? d + 1 : kMaxH] += t * ((unsigned long long)lim(d + 1) * c - q);
    }
    if (H == 4 && l == 2) {
      xv4 += C.sv[off + pos];
      xw4 += C.sw[off + pos];
    }
  }

  // One depth-l prefix ending in gene c, living t rounds; false past the loop
  // bound (nothing below it counts either).
  template <int l>
  __device__ __forceinline__ bool node(int c, unsigned long long t) {
    const int ai = w.act[c];
    if (ai > lim(l)) return false;
    ne[l] += t;
    if (l < kMaxH && l + 1 <= h)
      vis[l < kMaxH ? l + 1 : l] += t * (unsigned long long)(lim(l + 1) - ai);
    if (H == 4 && l == 3) {
      unsigned long long a, b;
      later_visits(C, R, c, (int)t, a, b);
      xv4 += a;
      xw4 += b;
    }
    return true;
  }

  // Leaves below a prefix with the m listed samples and last gene lo - 1,
  // counted at their first sample.
  __device__ __forceinline__ unsigned long long leaves(int m, int lo) {
    const int w_hi = (nA + 63) >> 6;
    unsigned long long sum = 0;
    for (int w0 = lo >> 6; w0 < w_hi; w0 += kWave) {
      const int wd = w0 + lane;
      const uint64_t r = wd < w_hi ? range_bits(wd, lo, nA) : 0ull;
      uint64_t acc = ~r;
#pragma unroll 4
      for (int j = 0; j < m; ++j) {
        const int p = s.smp[j];
        const uint64_t x = wd < w_hi ? brow(p)[wd] : 0ull;
        sum += (unsigned long long)tt[p] * (unsigned long long)popc64(x & ~acc);
        acc |= x;
      }
    }
    return sum;
  }

  // Union of the m listed samples' genes in [lo, nA).
  __device__ __forceinline__ uint64_t union_word(int m, int wd, int w_hi, int lo) {
    uint64_t x = 0;
    if (wd < w_hi) {
#pragma unroll 4
      for (int j = 0; j < m; ++j) x |= brow(s.smp[j])[wd];
      x &= range_bits(wd, lo, nA);
    }
    return x;
  }

  // The general walk (any number of samples and candidates): level LV, the
  // candidates of depth LV + 3 as a bitmap, below the prefix with samples
  // s.y[LV] (listed, m of them) and last gene lo - 1.
  template <int LV>
  __device__ __forceinline__ void general(int m, int lo, uint64_t* bits) {
    uint64_t* bm = bits + (size_t)LV * L.gw;
    const int w_hi = (nA + 63) >> 6;
    for (int w0 = lo >> 6; w0 < w_hi; w0 += kWave) {
      const uint64_t x = union_word(m, w0 + lane, w_hi, lo);
      if (w0 + lane < w_hi) bm[w0 + lane] = x;
    }
    __threadfence_block();
    for (int c = next_bit(bm, lo, nA, lane); c >= 0; c = next_bit(bm, c + 1, nA, lane)) {
      uint64_t y = 0;
      if (lane < w64) y = s.y[LV * kMaxW64 + lane] & T[(size_t)c * w64 + lane];
      const int mc = list_samples(y, s.smp, lane);
      const int p = uniform(s.smp[0]);
      const unsigned long long t = (unsigned long long)tt[p];
      if (w.act[c] > lim(LV + 3)) continue;
      if (lane == 0) {
        node<LV + 3>(c, t);
        if (mc == 1) below_single<LV + 3>(p, pos_in(p, c), t);
      }
      if (mc == 1) continue;
      if (LV + 4 == h) {
        ne[LV + 4] += leaves(mc, c + 1);
        continue;
      }
      if constexpr (LV + 4 < (H > 0 ? H : kMaxH)) {
        wave_lds_sync();
        if (lane < w64) s.y[(LV + 1) * kMaxW64 + lane] = y;
        wave_lds_sync();
        general<LV + 1>(mc, c + 1, bits);
      }
    }
  }

  // One depth-(LV + 3) candidate per lane (samples mk, gene ix): its node, and
  // all below it where one sample is left.
  template <int LV>
  __device__ __forceinline__ void candidate(uint64_t mk, int ix) {
    const int f = __builtin_ctzll(mk);
    const unsigned long long t = s.ts[f];
    if (!node<LV + 3>(ix, t)) return;
    if ((mk & (mk - 1)) == 0 && LV + 3 < h) {
      const int p = s.smp[f];
      below_single<LV + 3>(p, pos_in(p, ix), t);
    }
  }

  // The subtree over at most 64 candidates held one per lane (`set`): below an
  // entry with several samples lie the later lanes that share one.
  template <int LV>
  __device__ __forceinline__ void lanes(uint64_t mk, int ix, unsigned long long set) {
    const bool on = __builtin_amdgcn_inverse_ballot_w64(set);
    if (on) candidate<LV>(mk, ix);
    unsigned long long many = __ballot(on && (mk & (mk - 1)) != 0);
    while (many) {
      const int i = __builtin_ctzll(many);
      many &= many - 1;
      const unsigned long long later = set & ~((2ull << i) - 1ull);
      if (!later) break;
      const uint64_t mi = readlane64(mk, i) & mk;
      const unsigned long long kids =
          __ballot(__builtin_amdgcn_inverse_ballot_w64(later) && mi != 0);
      if (!kids) continue;
      if (LV + 4 == h) {
        if (__builtin_amdgcn_inverse_ballot_w64(kids))
          ne[LV + 4] += (unsigned long long)s.ts[__builtin_ctzll(mi)];
      } else {
        if constexpr (LV + 4 < (H > 0 ? H : kMaxH)) lanes<LV + 1>(mi, ix, kids);
      }
    }
  }

  // The same over a longer list in LDS.
  template <int LV>
  __device__ __forceinline__ void lists(int n) {
    const int cap = count_cap(h);
    const uint64_t* mk = s.mask + LV * cap;
    const uint16_t* ix = s.idx + LV * cap;
    for (int i = lane; i < n; i += kWave) candidate<LV>(mk[i], ix[i]);
    for (int i = 0; i + 1 < n; ++i) {
      const uint64_t mi = readlane64(mk[i], 0);
      if ((mi & (mi - 1)) == 0) continue;   // a single sample: counted above
      if (LV + 4 == h) {
        for (int j = i + 1 + lane; j < n; j += kWave) {
          const uint64_t x = mi & mk[j];
          if (x) ne[LV + 4] += (unsigned long long)s.ts[__builtin_ctzll(x)];
        }
        continue;
      }
      if constexpr (LV + 4 < (H > 0 ? H : kMaxH)) {
        uint64_t* mo = s.mask + (LV + 1) * cap;
        uint16_t* io = s.idx + (LV + 1) * cap;
        int k = 0;
        for (int j0 = i + 1; j0 < n; j0 += kWave) {
          const int j = j0 + lane;
          const uint64_t x = j < n ? (mi & mk[j]) : 0ull;
          const unsigned long long hm = __ballot(x != 0);
          if (x) {
            const int pos = rank_below(hm, k);
            mo[pos] = x;
            io[pos] = ix[j];
          }
          k += __popcll(hm);
        }
        wave_lds_sync();
        if (k > kWave) {
          lists<LV + 1>(k);
        } else if (k > 0) {
          const uint64_t x = lane < k ? mo[lane] : 0ull;
          const int g = lane < k ? (int)io[lane] : 0;
          wave_lds_sync();
          lanes<LV + 1>(x, g, k < 64 ? (1ull << k) - 1ull : ~0ull);
        }
      }
    }
  }

  // A pair with several samples, by the whole wave.
  __device__ __forceinline__ void pair(int a, int b, uint64_t* bits) {
    uint64_t y2 = 0;
    if (lane < w64) y2 = T[(size_t)a * w64 + lane] & T[(size_t)b * w64 + lane];
    const int m = list_samples(y2, s.smp, lane);
    if (h == 3) {
      ne[3] += leaves(m, b + 1);
      return;
    }
    if constexpr (H != 2 && H != 3) {
      const int cap = count_cap(h);
      bool listed = m <= 64;
      int n = 0;
      if (listed) {
        const int w_hi = (nA + 63) >> 6;
        for (int w0 = (b + 1) >> 6; w0 < w_hi && listed; w0 += kWave) {
          const int wd = w0 + lane;
          uint64_t x = union_word(m, wd, w_hi, b + 1);
          const int c = popc64(x);
          int pos = wave_before(c, lane);
          const int tot = uniform(__shfl(pos + c, 63, 64));
          if (n + tot > cap) {
            listed = false;
            break;
          }
          pos += n;
          while (x) {
            s.idx[pos++] = (uint16_t)(wd * 64 + __builtin_ctzll(x));
            x &= x - 1;
          }
          n += tot;
        }
      }
      if (!listed) {
        wave_lds_sync();
        if (lane < w64) s.y[lane] = y2;
        wave_lds_sync();
        general<0>(m, b + 1, bits);
        return;
      }
      if (lane < m) s.ts[lane] = (uint32_t)tt[s.smp[lane]];
      wave_lds_sync();
      auto mask_of = [&](int g) {
        const uint64_t* row = T + (size_t)g * w64;
        uint64_t mk = 0;
#pragma unroll 4
        for (int j = 0; j < m; ++j) {
          const int p = s.smp[j];
          mk |= ((row[p >> 6] >> (p & 63)) & 1ull) << j;
        }
        return mk;
      };
      if (n <= kWave) {
        const int ix = lane < n ? (int)s.idx[lane] : 0;
        const uint64_t mk = lane < n ? mask_of(ix) : 0ull;
        lanes<0>(mk, ix, n < 64 ? (1ull << n) - 1ull : ~0ull);
        return;
      }
      for (int i = lane; i < n; i += kWave) s.mask[i] = mask_of(s.idx[i]);
      wave_lds_sync();
      lists<0>(n);
    }
  }
};

// One lane per pair: pairs with a single sample in closed form, the others by
// the wave in turn.  Wave q takes every nsub-th pair of share q % nw, so that
// the pairs with most samples (first in every share) spread over all waves.
// Bound by chains of dependent loads: the sample order sits in LDS, the lists
// of most pairs in lanes, and 25 KB of LDS a block keep six blocks on a compute
// unit (48 KB, lists in LDS and the order in memory: G = 20000, h = 4 1251 us,
// 954 us now; one round of G = 5000, h = 5 837 us, 314 us now).
template <int H>
__global__ __launch_bounds__(256) void k_count_pairs(Problem P, Work w, LazyWork L, CountWork C) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ uint16_t s_order[kMaxCount], s_tt[kMaxCount];
  RoundState* st = w.st;
  const int lane = threadIdx.x & 63;
  const int wib = uniform(threadIdx.x >> 6);
  const int q = blockIdx.x * (kBlock / kWave) + wib;
  const int h = H > 0 ? H : P.h;
  const int n0 = L.uncs[0];
  for (int i = threadIdx.x; i < n0; i += kBlock) {
    s_order[i] = (uint16_t)C.order[i];
    s_tt[i] = (uint16_t)C.tt[i];
  }
  __syncthreads();
  Count<H> v{P, w, L, C, count_lds(lds + (size_t)wib * C.wave_bytes, h),
             reinterpret_cast<const uint64_t*>(w.TA), s_order, s_tt};
  v.lane = lane;
  v.nA = uniform(st->nA);
  v.w64 = w.w64;
  v.h = h;
  v.R = min(uniform(st->executed), kCountMaxT);
  v.ne2 = v.vis3 = v.xv3 = v.xw3 = v.xv4 = v.xw4 = 0;
#pragma unroll
  for (int d = 0; d <= kMaxH; ++d) v.ne[d] = v.vis[d] = 0;
  const int nsub = gridDim.x * (kBlock / kWave) / L.nw;
  const int seg = q % L.nw, sub = q / L.nw;
  const unsigned long long E = st->n_pairs < w.pair_cap ? st->n_pairs : w.pair_cap;
  const int n_mine = sub < nsub && (unsigned long long)seg < E
                         ? (int)((E - (unsigned long long)seg + (unsigned long long)L.nw - 1ull) /
                                 (unsigned long long)L.nw)
                         : 0;
  const unsigned long long* list = L.list + (size_t)seg * L.seg;
  uint64_t* bits = C.bits + (size_t)q * L.levels * L.gw;
  const bool last_out = st->amax[3] < v.nA;   // h >= 4: the last gene is past depth 3's bound
  for (int s0 = sub; s0 < n_mine; s0 += nsub * kWave) {
    const int slot = s0 + nsub * lane;
    const bool on = slot < n_mine;
    const unsigned long long e = on ? list[slot] : 0ull;
    const int a = (int)(e & 0xffff), b = (int)((e >> 16) & 0xffff);
    int m = 0, p = 0;
    if (on) {
      const uint64_t* ra = v.T + (size_t)a * w.w64;
      const uint64_t* rb = v.T + (size_t)b * w.w64;
#pragma unroll 4
      for (int k = 0; k < w.w64; ++k) {
        const uint64_t x = ra[k] & rb[k];
        if (m == 0 && x) p = k * 64 + __builtin_ctzll(x);
        m += popc64(x);
      }
    }
    if (m > 0) {
      const unsigned long long t = (unsigned long long)s_tt[p];
      v.ne2 += t;
      if (h >= 3) {
        v.vis3 += t * (unsigned long long)(v.lim(3) - w.act[b]);
        if (H == 3 || H == 4) {
          unsigned long long x, y;
          later_visits(C, v.R, b, (int)t, x, y);
          if (H == 4 && last_out) {
            const int tl = min((int)t, (int)C.tg[v.nA - 1]);
            x -= (unsigned long long)tl;
            y -= (unsigned long long)C.wc[tl];
          }
          v.xv3 += x;
          v.xw3 += y;
        }
        if (m == 1) v.template below_single<2>(p, v.pos_in(p, b), t);
      }
    }
    if (h >= 3) {
      unsigned long long many = __ballot(m > 1);
      while (many) {
        const int src = __builtin_ctzll(many);
        many &= many - 1;
        v.pair(__builtin_amdgcn_readlane(a, src), __builtin_amdgcn_readlane(b, src), bits);
      }
    }
  }
  unsigned long long row[kTallyN] = {0};
  row[kCNe2] = v.ne2;
  row[kCVis3] = v.vis3;
#pragma unroll
  for (int d = 3; d <= kMaxH; ++d) row[kCNe3 + d - 3] = v.ne[d];
#pragma unroll
  for (int d = 4; d <= kMaxH; ++d) row[kCVis4 + d - 4] = v.vis[d];
  if (H == 3 || H == 4) {
    row[kCXv3] = v.xv3;
    row[kCXw3] = v.xw3;
    row[kCXv4] = v.xv4;
    row[kCXw4] = v.xw4;
  }
  block_tally_to(w.tallies + (size_t)blockIdx.x * kTallyN, row);
}

// One block: the depth-1 and depth-2 counts from the genes' rounds, and the
// blocks' rows summed into the run's totals.
__global__ __launch_bounds__(1024) void k_count_finish(Problem P, Work w, LazyWork L, CountWork C,
                                                       int rows) {
  __shared__ unsigned long long tsum[16][kTallyN];
  __shared__ unsigned long long gsum[16][2], msum[16];
  __shared__ uint32_t h1[kCountMaxT + 2], h2[kCountMaxT + 2];
  RoundState* st = w.st;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int h = P.h, nA = st->nA, R = min(st->executed, kCountMaxT);
  for (int i = tid; i < kCountMaxT + 2; i += 1024) h1[i] = h2[i] = 0u;
  __syncthreads();
  unsigned long long ne1 = 0, vis2 = 0;
  for (int g = tid; g < nA; g += 1024) {
    const int s = w.act[g], t = C.tg[g];
    if (s <= P.G - h) {
      ne1 += (unsigned long long)t;
      vis2 += (unsigned long long)t * (unsigned long long)(P.G - h + 1 - s);
      atomicAdd(&h1[t], 1u);
    }
    if (s <= P.G - h + 1) atomicAdd(&h2[t], 1u);
  }
  unsigned long long v = 0;
  for (int i = tid; i < rows * kTallyN; i += 1024) v += w.tallies[i];
  v += __shfl_xor((long long)v, 16, 64);
  v += __shfl_xor((long long)v, 32, 64);
  for (int o = 32; o > 0; o >>= 1) {
    ne1 += (unsigned long long)__shfl_xor((long long)ne1, o, 64);
    vis2 += (unsigned long long)__shfl_xor((long long)vis2, o, 64);
  }
  __syncthreads();   // the histograms are whole
  // genes active in round r: those with at least r rounds
  for (int o = 1; o < 2048; o <<= 1) {
    uint32_t x[2][2] = {{0, 0}, {0, 0}};
    for (int u = 0; u < 2; ++u) {
      const int r = tid + 1024 * u;
      if (r + o < kCountMaxT + 2) {
        x[u][0] = h1[r + o];
        x[u][1] = h2[r + o];
      }
    }
    __syncthreads();
    for (int u = 0; u < 2; ++u) {
      const int r = tid + 1024 * u;
      if (r < kCountMaxT + 2) {
        h1[r] += x[u][0];
        h2[r] += x[u][1];
      }
    }
    __syncthreads();
  }
  // round r: every active pair inside the depth-1/2 bounds, times |U|
  unsigned long long macs = 0;
  for (int r = tid + 1; r <= R; r += 1024) {
    const unsigned long long a1 = h1[r], a2 = h2[r];
    macs += (a1 ? a1 * a2 - a1 * (a1 + 1) / 2 : 0) * (unsigned long long)L.uncs[r - 1];
  }
  for (int o = 32; o > 0; o >>= 1)
    macs += (unsigned long long)__shfl_xor((long long)macs, o, 64);
  if (lane == 0) msum[wid] = macs;
  if (lane < kTallyN) tsum[wid][lane] = v;
  if (lane == 0) {
    gsum[wid][0] = ne1;
    gsum[wid][1] = vis2;
  }
  __syncthreads();
  if (tid >= 64 && tid < 64 + kTallyN) {
    const int f = tid - 64;
    unsigned long long x = 0;
    for (int i = 0; i < 16; ++i) x += tsum[i][f];
    if (f == kCNe2 && h >= 2) st->tot.nonempty[2] = x;
    if (f == kCVis3 && h >= 3) st->tot.visited[3] = x;
    if (f >= kCNe3 && f < kCNe3 + 7 && f - kCNe3 + 3 <= h) {
      st->tot.nonempty[f - kCNe3 + 3] = x;
      if (f - kCNe3 + 3 == h && h <= 4) st->tx_leaves = x;
    }
    if (f >= kCVis4 && f < kCVis4 + 6 && f - kCVis4 + 4 <= h) st->tot.visited[f - kCVis4 + 4] = x;
    if (h == 3 || h == 4) {
      if (f == kCXv3) st->tx_vis3 = x;
      if (f == kCXw3) st->tx_vis_words3 = x;
    }
    if (h == 4) {
      if (f == kCXv4) st->tx_vis4 = x;
      if (f == kCXw4) st->tx_vis_words4 = x;
    }
  }
  if (tid == 0) {
    unsigned long long n1 = 0, v2 = 0;
    macs = 0;
    for (int i = 0; i < 16; ++i) {
      n1 += gsum[i][0];
      v2 += gsum[i][1];
    }
    st->tot.visited[1] = (unsigned long long)R * (unsigned long long)(P.G - h + 1);
    st->tot.nonempty[1] = n1;
    st->tot.visited[2] = v2;
    for (int i = 0; i < 16; ++i) macs += msum[i];
    st->tx_pair_macs = macs;
  }
}

}  // namespace

size_t count_table_rows(int nA) {
  return (size_t)count_segments(nA) * (kTabSeg / kTabGenes) + 1;
}

int count_segments(int nA) { return (nA + kTabSeg - 1) / kTabSeg > 0 ? (nA + kTabSeg - 1) / kTabSeg : 1; }

hipError_t launch_count(const Problem& P, const Work& w, const LazyWork& L, const CountWork& C0,
                        int nA_max, hipStream_t s) {
  CountWork C = C0;
  C.wave_bytes = (int)count_wave_bytes(P.h);
  const int segs = count_segments(nA_max);
  const bool tables = P.h == 3 || P.h == 4;
  k_count_order<<<1, 1024, 0, s>>>(w, L, C);
  int blocks = (L.gw * w.w64 + 3) / 4;
  if (blocks > 1024) blocks = 1024;
  k_count_rows<<<blocks, kBlock, 0, s>>>(w, L, C);
  k_count_genes<<<segs, kBlock, 0, s>>>(w, L, C, tables ? 1 : 0);
  if (tables) k_count_tables<<<segs, kBlock, 0, s>>>(w, L, C, segs);
  if (P.h >= 3) {
    k_count_offsets<<<1, 1024, 0, s>>>(L, C);
    k_count_lists<<<(64 * w.w64 + 3) / 4, kBlock, 0, s>>>(P, w, L, C);
  }
  const size_t lds = (size_t)C.wave_bytes * (kBlock / kWave);
  const int grid = C.waves / (kBlock / kWave);
  switch (P.h) {
    case 2: k_count_pairs<2><<<grid, kBlock, lds, s>>>(P, w, L, C); break;
    case 3: k_count_pairs<3><<<grid, kBlock, lds, s>>>(P, w, L, C); break;
    case 4: k_count_pairs<4><<<grid, kBlock, lds, s>>>(P, w, L, C); break;
    case 5: k_count_pairs<5><<<grid, kBlock, lds, s>>>(P, w, L, C); break;
    case 6: k_count_pairs<6><<<grid, kBlock, lds, s>>>(P, w, L, C); break;
    default: k_count_pairs<0><<<grid, kBlock, lds, s>>>(P, w, L, C); break;
  }
  k_count_finish<<<1, 1024, 0, s>>>(P, w, L, C, grid);
  return hipGetLastError();
}

}  // namespace pdfs
