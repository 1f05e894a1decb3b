// Lazy or walked rounds: the choice at measured rounds and covers nearest to where
// the faster way changes (each at least 1.7 times as fast as the other), and its
// edges.
#include "stub.h"

constexpr int kEmpty = PDFS_PRUNE_EMPTY, kBound = PDFS_PRUNE_BOUND;

static const struct {
  int h, mode, max_rounds, nA, n_tumor;
  unsigned long long bits;
  double lazy_ms, walked_ms;
} kMeasured[] = {
    {2, kBound, 0, 10000, 200, 399975, 5.06, 2.87},
    {2, kBound, 0, 5000, 500, 749865, 3.52, 1.78},
    {2, kBound, 0, 10000, 200, 200074, 2.62, 4.62},
    {2, kBound, 0, 1000, 200, 89943, 0.31, 0.56},
    {2, kEmpty, 0, 2500, 1200, 1349142, 2.19, 1.29},
    {2, kEmpty, 0, 150, 200, 13492, 0.36, 0.62},
    {2, kEmpty, 0, 1000, 60, 11982, 0.36, 0.62},
    {3, kBound, 0, 16, 700, 60, 0.14, 0.24},
    {3, kBound, 0, 150, 700, 47115, 2.23, 3.88},
    {3, kBound, 1, 400, 700, 55902, 0.63, 0.36},
    {3, kBound, 1, 150, 1200, 53974, 0.47, 0.26},
    {3, kBound, 1, 150, 200, 6073, 0.14, 0.24},
    {3, kBound, 1, 150, 700, 15832, 0.13, 0.23},
    {3, kEmpty, 0, 1000, 1200, 539620, 27.98, 15.91},
    {3, kEmpty, 0, 60, 60, 1626, 0.52, 0.92},
    {3, kEmpty, 0, 150, 700, 31438, 2.61, 4.78},
    {3, kEmpty, 1, 60, 1200, 3717, 0.28, 0.17},
    {3, kEmpty, 1, 18, 400, 35, 0.18, 0.10},
    {3, kEmpty, 1, 1000, 200, 15988, 0.26, 0.44},
    {3, kEmpty, 1, 1000, 400, 48086, 0.52, 0.90},
    {4, kBound, 0, 150, 400, 26971, 9.68, 5.52},
    {4, kBound, 0, 60, 1200, 32309, 23.09, 12.86},
    {4, kBound, 0, 18, 400, 35, 0.13, 0.22},
    {4, kBound, 0, 32, 60, 37, 0.13, 0.23},
    {4, kBound, 1, 400, 200, 35889, 0.76, 0.42},
    {4, kBound, 1, 150, 400, 11976, 0.53, 0.28},
    {4, kBound, 1, 60, 200, 946, 0.12, 0.21},
    {4, kBound, 1, 20, 700, 291, 0.09, 0.16},
    {4, kBound, 3, 150, 1200, 35889, 2.07, 1.20},
    {4, kBound, 3, 30, 1200, 9097, 1.55, 0.90},
    {4, kEmpty, 0, 400, 400, 71939, 34.61, 19.22},
    {4, kEmpty, 0, 60, 700, 18909, 14.56, 7.60},
    {4, kEmpty, 0, 20, 200, 216, 0.34, 0.59},
    {4, kEmpty, 0, 400, 60, 10792, 2.37, 4.23},
    {4, kEmpty, 1, 20, 1200, 4851, 0.50, 0.29},
    {4, kEmpty, 1, 150, 700, 20879, 0.99, 0.57},
    {4, kEmpty, 1, 400, 60, 2915, 0.22, 0.37},
    {4, kEmpty, 1, 400, 700, 5592, 0.21, 0.36},
    {5, kBound, 0, 150, 1200, 53974, 313.67, 154.73},
    {5, kBound, 0, 150, 400, 26971, 64.35, 20.75},
    {5, kBound, 0, 20, 400, 404, 0.23, 0.40},
    {5, kBound, 0, 150, 700, 31438, 37.36, 66.36},
    {5, kBound, 1, 60, 700, 12675, 1.48, 0.87},
    {5, kBound, 1, 150, 700, 20879, 1.41, 0.80},
    {5, kBound, 1, 20, 1200, 111, 0.08, 0.13},
    {5, kBound, 1, 60, 1200, 372, 0.09, 0.15},
    {5, kBound, 3, 250, 500, 37501, 7.17, 4.21},
    {5, kBound, 3, 100, 500, 17469, 5.38, 3.10},
    {5, kEmpty, 0, 9, 200, 23, 0.23, 0.13},
    {5, kEmpty, 0, 18, 400, 35, 0.26, 0.15},
    {5, kEmpty, 0, 20, 1200, 1255, 0.59, 1.03},
    {5, kEmpty, 0, 150, 1200, 866, 0.32, 0.57},
    {5, kEmpty, 1, 6, 60, 8, 0.12, 0.07},
    {5, kEmpty, 1, 20, 1200, 1255, 0.30, 0.17},
    {5, kEmpty, 1, 60, 700, 8441, 1.06, 1.82},
    {5, kEmpty, 1, 150, 200, 1583, 0.19, 0.33},
    {6, kBound, 0, 60, 700, 924, 0.25, 0.43},
    {6, kBound, 0, 6, 60, 8, 0.11, 0.20},
    {6, kBound, 1, 20, 700, 6298, 1.01, 0.58},
    {6, kBound, 1, 60, 200, 5384, 1.95, 1.02},
    {6, kBound, 1, 20, 400, 172, 0.07, 0.13},
    {6, kBound, 1, 57, 400, 469, 0.08, 0.13},
    {6, kBound, 3, 100, 1200, 30008, 30.83, 11.73},
    {6, kBound, 3, 150, 500, 26081, 41.86, 14.14},
    {6, kEmpty, 0, 20, 200, 344, 0.29, 0.17},
    {6, kEmpty, 0, 20, 1200, 463, 0.28, 0.16},
    {6, kEmpty, 0, 185, 400, 775, 0.31, 0.60},
    {6, kEmpty, 0, 45, 60, 224, 0.46, 0.91},
    {6, kEmpty, 1, 31, 60, 62, 0.14, 0.08},
    {6, kEmpty, 1, 13, 60, 29, 0.13, 0.08},
    {6, kEmpty, 1, 60, 200, 1439, 0.35, 0.60},
    {6, kEmpty, 1, 355, 400, 3143, 0.19, 0.35},
    {8, kBound, 0, 6, 60, 8, 0.11, 0.19},
    {8, kBound, 0, 14, 60, 17, 0.11, 0.19},
    {8, kBound, 1, 60, 700, 18909, 58.94, 30.33},
    {8, kBound, 1, 60, 1200, 32309, 339.01, 91.97},
    {8, kBound, 1, 20, 700, 291, 0.08, 0.13},
    {8, kBound, 1, 150, 1200, 14356, 0.80, 1.38},
    {8, kEmpty, 0, 39, 60, 81, 0.24, 0.14},
    {8, kEmpty, 0, 20, 200, 216, 0.26, 0.16},
    {8, kEmpty, 0, 60, 700, 2219, 0.90, 1.58},
    {8, kEmpty, 0, 60, 200, 603, 0.45, 0.82},
    {8, kEmpty, 1, 39, 60, 81, 0.15, 0.09},
    {8, kEmpty, 1, 64, 60, 139, 0.16, 0.09},
    {8, kEmpty, 1, 381, 700, 1343, 0.18, 0.32},
    {8, kEmpty, 1, 440, 400, 1974, 0.19, 0.34},
};

int main() {
  int n = 0;
  for (const auto& m : kMeasured) {
    const pdfs::RunShape s = {m.nA, m.n_tumor, m.n_tumor, m.bits};
    const bool lazy = pdfs::lazy_pays(s, m.h, m.mode, m.max_rounds, true);
    if (lazy != (m.lazy_ms < m.walked_ms)) {
      std::printf("FAILED: h %d mode %d rounds %d nA %d n %d\n", m.h, m.mode, m.max_rounds, m.nA,
                  m.n_tumor);
      return 1;
    }
    ++n;
  }
  // the literal reading of T-: a single round's opens are not pruned
  for (int h = 3; h <= 5; ++h) {
    const pdfs::RunShape lit = {1500, 300, 300, 22500, true}, plain = {1500, 300, 300, 22500};
    if (pdfs::lazy_pays(lit, h, kBound, 1, false) || !pdfs::lazy_pays(plain, h, kBound, 1, false) ||
        !pdfs::lazy_pays(lit, h, kBound, 0, false))
      stub::die("literal reading");
  }
  for (int h = 1; h <= PDFS_MAX_H; ++h)
    for (int rounds = 0; rounds < 6; ++rounds) {
      // no gene, no uncovered sample, the largest cohort
      for (int mode : {PDFS_PRUNE_NONE, kEmpty, kBound}) {
        for (int counters = 0; counters < 2; ++counters) {
          (void)pdfs::lazy_pays({0, 1, 0, 1}, h, mode, rounds, counters);
          const bool lazy = pdfs::lazy_pays({65535, 1280, 1280, 65535ull * 1280}, h, mode, rounds, counters);
          if (lazy && (h < 2 || mode == PDFS_PRUNE_NONE)) stub::die("lazy where no lazy round is");
        }
      }
      if (h == 2 && rounds == 1 && pdfs::lazy_pays({5000, 1000, 1000, 25000}, h, kBound, rounds, true))
        stub::die("a single round of h = 2 is the table's");
    }
  std::printf("ok %d\n", n);
  return 0;
}
