// What a run does without: counters that nobody asked for, and lists that do not
// fit in device memory.
#include "stub.h"

#include <vector>

static const int G = 300, nt = 200, wt = 4;
static std::vector<uint64_t> T((size_t)G * wt, 0), N((size_t)G, 0);

static pdfs_ctx* make(int mode) {
  const pdfs_matrix m = {G, nt, 60, 0, T.data(), N.data(), wt, 1};
  const pdfs_options o = {mode, 0, nullptr, 0, 64};
  pdfs_ctx* c = nullptr;
  if (pdfs_create(&m, &o, &c) != PDFS_OK) stub::die("create");
  return c;
}

static int32_t cover(pdfs_ctx* c, int h, bool stats, int* n_out, pdfs_combo* out, uint64_t* left) {
  pdfs_stats st;
  return pdfs_wsc_run(c, h, 1, 10, 0, 0, nullptr, out, 8, n_out, left, stats ? &st : nullptr);
}

int main() {
  for (int g = 0; g < G; ++g)
    for (int k = 0; k < 3; ++k) {
      const int s = (g * 7 + k * 31) % nt;
      T[(size_t)g * wt + (s >> 6)] |= 1ull << (s & 63);
    }
  pdfs_combo out[8];
  uint64_t left[4];
  int32_t n = 0;
  for (int h : {2, 3, 4, 5, 7}) {
    // counters are made, and their memory taken, where they are asked for
    pdfs_ctx* c = make(PDFS_PRUNE_EMPTY);
    stub::emit = 30000;
    stub::counted = 0;
    if (cover(c, h, false, &n, out, left) != PDFS_OK || n != 3) stub::die("cover");
    if (stub::counted) stub::die("counters that nobody asked for");
    const size_t without = stub::bytes_held;
    pdfs_combo one;
    if (pdfs_best_combo(c, 4, 1, 10, nullptr, &one, nullptr) != PDFS_OK) stub::die("round");
    if (stub::counted) stub::die("counters of a round that nobody asked for");
    if (cover(c, h, true, &n, out, left) != PDFS_OK || n != 3) stub::die("counted cover");
    if (stub::counted != 1 || stub::bytes_held <= without) stub::die("counters asked for");
    pdfs_destroy(c);

    // every limit on what may be held: the run goes out as lazy rounds, or walked
    // ones, or is refused before it has run; h = 2 needs no list
    for (int mode : {PDFS_PRUNE_EMPTY, PDFS_PRUNE_BOUND}) {
      stub::lazy_launches = stub::walked_rounds = 0;
      c = make(mode);
      const size_t base = stub::bytes_held;
      if (cover(c, h, true, &n, out, left) != PDFS_OK || !stub::lazy_launches) stub::die("lazy cover");
      const size_t full = stub::bytes_held;
      pdfs_destroy(c);
      int walked = 0, refused = 0;
      for (size_t room = full; room > base; room -= (full - base) / 64 + 1) {
        c = make(mode);
        stub::limit = room;
        stub::walked_rounds = 0;
        const int32_t rc = cover(c, h, true, &n, out, left);
        stub::limit = ~(size_t)0;
        if (rc == PDFS_OK && n != 3) stub::die("rounds under a limit");
        if (rc != PDFS_OK && (rc != PDFS_ERR_OUT_OF_MEMORY || n != 0)) stub::die("status under a limit");
        walked += stub::walked_rounds > 0;
        refused += rc != PDFS_OK;
        if (cover(c, h, true, &n, out, left) != PDFS_OK || n != 3) stub::die("after the limit");
        pdfs_destroy(c);
      }
      if (h == 2 && !walked) stub::die("no cover of h = 2 was walked");
    }
  }
  if (stub::bytes_held) stub::die("memory left behind");
  std::printf("ok\n");
  return 0;
}
