// Every allocation of a call in turn fails: the call says so (a lazy run goes out
// as walked rounds), and the context's next calls work on buffers that are held
// and long enough.
#include "stub.h"

#include <vector>

static std::vector<uint64_t> rows(int G, int wt, int n) {
  std::vector<uint64_t> m((size_t)G * wt, 0);
  for (int g = 0; g < G; ++g)
    for (int k = 0; k < 3; ++k) {
      const int s = (g * 7 + k * 31) % n;
      m[(size_t)g * wt + (s >> 6)] |= 1ull << (s & 63);
    }
  return m;
}

struct Step {
  int mode, h, rounds;
  unsigned long long emit;
};

static int32_t call(pdfs_ctx* c, const Step& s) {
  pdfs_combo out[8];
  pdfs_stats st;
  int32_t n = 0;
  stub::emit = s.emit;
  stub::rounds = s.rounds;
  pdfs_set_prune_mode(c, s.mode);
  const int32_t rc = pdfs_wsc_run(c, s.h, 1, 10, 0, 0, nullptr, out, 8, &n, nullptr, &st);
  if (rc == PDFS_OK && n != s.rounds) stub::die("rounds");
  return rc;
}

int main() {
  const int G = 300, nt = 200, wt = 4;
  const std::vector<uint64_t> T = rows(G, wt, nt), N = rows(G, 1, 60);
  const pdfs_matrix m = {G, nt, 60, 0, T.data(), N.data(), wt, 1};
  // what runs with a failure, and what runs before and after it
  const Step steps[] = {
      {PDFS_PRUNE_BOUND, 2, 3, 100}, {PDFS_PRUNE_BOUND, 3, 3, 30000}, {PDFS_PRUNE_BOUND, 4, 3, 100},
      {PDFS_PRUNE_BOUND, 6, 2, 40000}, {PDFS_PRUNE_EMPTY, 3, 5, 100}, {PDFS_PRUNE_EMPTY, 4, 6, 30000},
      {PDFS_PRUNE_EMPTY, 5, 2, 100}, {PDFS_PRUNE_NONE, 3, 2, 30000}, {PDFS_PRUNE_NONE, 5, 2, 100},
  };
  long tried = 0;
  const int n_steps = (int)(sizeof(steps) / sizeof(steps[0]));
  for (int f = -1; f < n_steps; ++f)   // -1: the failure meets a context that has run nothing
    for (const Step& hit : steps)
      for (long k = 0;; ++k) {
        pdfs_options o = {PDFS_PRUNE_BOUND, 0, nullptr, 0, 64};
        pdfs_ctx* c = nullptr;
        stub::fail_at = -1;
        if (pdfs_create(&m, &o, &c) != PDFS_OK) stub::die("create");
        if (f >= 0 && call(c, steps[f]) != PDFS_OK) stub::die("first call");
        stub::allocs = 0;
        stub::fail_at = k;
        const int32_t rc = call(c, hit);
        const bool failed = stub::allocs > k;
        stub::fail_at = -1;
        if (rc != PDFS_OK && rc != PDFS_ERR_OUT_OF_MEMORY) stub::die("status");
        if (!failed && rc != PDFS_OK) stub::die("a call without a failure");
        if (hit.mode != PDFS_PRUNE_NONE && rc != PDFS_OK) stub::die("walked rounds would have fit");
        // a shorter need, the same call, then everything else
        if (call(c, {hit.mode, hit.h, 1, 64}) != PDFS_OK) stub::die("the next call");
        if (call(c, hit) != PDFS_OK) stub::die("the same call again");
        for (const Step& s : steps)
          if (call(c, s) != PDFS_OK) stub::die("later calls");
        pdfs_destroy(c);
        if (stub::bytes_held) stub::die("memory left behind");
        ++tried;
        if (!failed) break;
      }
  std::printf("ok %ld\n", tried);
  return 0;
}
