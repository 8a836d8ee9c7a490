// Random batches through the host's cutting of a row-lane launch (cut.h): every
// read lies in one pack on lanes of its own, the segments cover the reference,
// waves, halos and scratch are numbered without gaps or overlaps, and the cut
// keeps to its scratch.  Prints "ok <cases>" or the first that fails.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>
#include <random>

#include "../../paper_2211_07340_amd/csrc/cut.h"

using namespace sdtw;

static int g_case = 0;
static long g_allocations = 0;
void* operator new(size_t n) {
  ++g_allocations;
  void* p = malloc(n);
  if (!p) abort();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      printf("case %d, line %d: %s\n", g_case, __LINE__, #cond);           \
      exit(1);                                                             \
    }                                                                      \
  } while (0)

using Reads = std::vector<std::pair<int32_t, int32_t>>;

static void check_layout(const RowLayout& lay, const Reads& reads, int max_reads) {
  std::vector<int> seen(reads.size(), 0);
  int32_t pack = 0, last = 33;
  for (int k = 0; k < lay.nclasses; ++k) {
    const RowClass& c = lay.classes[k];
    CHECK(c.rows_per_lane < last);
    last = c.rows_per_lane;
    CHECK(c.first_pack == pack && c.npacks >= 1);
    for (int32_t i = 0; i < c.npacks; ++i, ++pack) {
      const RowPack& p = lay.packs[(size_t)pack];
      CHECK(p.nreads >= 1 && p.nreads <= max_reads && p.lane0[0] == 0);
      for (int j = 0; j < p.nreads; ++j) {
        const int32_t m = reads[(size_t)p.item[j]].second;
        ++seen[(size_t)p.item[j]];
        CHECK(p.lane0[j + 1] - p.lane0[j] == rows_lanes(m, c.rows_per_lane));
        CHECK(p.lane0[j + 1] <= kLanes && p.lane0[j + 1] > p.lane0[j]);
        CHECK(m <= p.max_m && p.max_m <= c.max_m);
        CHECK(p.lane0[j + 1] - p.lane0[j] <= p.max_lanes && p.max_lanes <= c.max_lanes);
      }
      for (int j = p.nreads; j < kRowsReads; ++j) CHECK(p.lane0[j + 1] == p.lane0[p.nreads]);
    }
  }
  CHECK(pack == (int32_t)lay.packs.size());
  for (int s : seen) CHECK(s == 1);
}

static void check_cut(const RowsArgs& a, const RowLayout& lay, int64_t n, bool stream,
                      int64_t words) {
  CHECK(a.nclasses == lay.nclasses);
  int64_t waves = 0, halos = 0, bound = 0, results = 0;
  for (int k = 0; k < a.nclasses; ++k) {
    const RowClass& c = a.cls[k];
    CHECK(c.segcols % 64 == 0 && c.segcols >= 64);
    CHECK((int64_t)c.nseg * c.segcols >= n && (int64_t)(c.nseg - 1) * c.segcols < n);
    CHECK(c.first_wave == waves && c.first_halo == halos);
    waves += (int64_t)c.nseg * c.npacks;
    halos += (int64_t)(c.nseg - 1) * c.npacks;
    if (c.nseg > 1) {
      CHECK(c.bound_at == bound && c.result_at == results);
      bound += (int64_t)(c.nseg - 1) * c.npacks * rows_bound_words(c.rows_per_lane);
      results += (int64_t)c.npacks * (stream ? kRowsStreamReads : kRowsReads) *
                 (rows_groups(c.nseg) + 1);
    }
  }
  CHECK(a.nwaves == waves && a.nhalo == halos && a.nresults == results);
  if (!halos) return;
  RowsArgs b = a;
  rows_scratch(b, (uint64_t*)4096);
  CHECK((char*)b.done == (char*)b.keys + 8 * results);
  CHECK((char*)b.fail >= (char*)b.done + 4 * results);
  CHECK((char*)b.bound >= (char*)b.fail + 4 * waves && (uintptr_t)b.bound % 8 == 0);
  CHECK((char*)b.bound + 4 * bound <= (char*)b.keys + 8 * words);
}

int main() {
  std::mt19937_64 g(7);
  auto log_uniform = [&](double lo, double hi) {
    const double u = std::uniform_real_distribution<double>(log(lo), log(hi + 0.999))(g);
    return (int64_t)exp(u);
  };
  for (g_case = 0; g_case < 1500; ++g_case) {
    const bool stream = g() % 2, f32 = g() % 2;
    const int max_reads = stream ? kRowsStreamReads : kRowsReads;
    const int32_t nq = (int32_t)log_uniform(1, 3000);
    const int32_t lo = (int32_t)log_uniform(1, kRowsMaxM);
    const int32_t hi = std::min<int32_t>(kRowsMaxM, (int32_t)log_uniform(lo, 8.0 * lo));
    Reads reads;
    for (int32_t i = 0; i < nq; ++i)
      reads.emplace_back(i, lo + (int32_t)(g() % (uint64_t)(std::max(hi, lo) - lo + 1)));
    std::sort(reads.begin(), reads.end(), [](const auto& a, const auto& b) {
      return a.second > b.second;
    });
    for (int32_t i = 0; i < nq; ++i) reads[(size_t)i].first = i;
    const int cus = g() % 4 ? 256 : 1 + (int)(g() % 304);
    for (int alone = 0; alone < 2; ++alone) {
      RowLayout lay = rows_layout(reads, alone, max_reads);
      lay.max_held = stream ? (int32_t)log_uniform(1, 32767) : 0;
      check_layout(lay, reads, max_reads);
      for (int k = 0; k < 3; ++k) {
        const int64_t n = k == 2 ? (int64_t)INT32_MAX - 2 * kPadUnit : log_uniform(1, 2e8);
        const int64_t most = g() % 2 ? INT64_MAX : log_uniform(1e3, 1e7);
        RowsArgs a{};
        a.cus = cus;
        int64_t words = 0;
        const double t = rows_best_cut(a, lay, alone, n, f32, stream, most, &words);
        CHECK(t > 0.0 && words <= most);
        check_cut(a, lay, n, stream, words);
        // one segment per pack is always to be had, and none better is passed over
        RowsArgs b{};
        b.cus = cus;
        const double uncut = rows_best_cut(b, lay, alone, n, f32, stream, 0, &words);
        CHECK(b.nhalo == 0 && words == 0 && b.nwaves == (int32_t)lay.packs.size());
        check_cut(b, lay, n, stream, 0);
        CHECK(t <= uncut);
        // a plan's scratch holds the cuts that are tried, or is at its bound
        const int64_t plan_words = rows_most_words(lay, cus);
        CHECK(plan_words <= kMostPlanWords);
        if (!stream && plan_words < kMostPlanWords) {
          RowsArgs c{};
          c.cus = cus;
          CHECK(rows_best_cut(c, lay, alone, n, f32, false, INT64_MAX, &words) ==
                rows_best_cut(c, lay, alone, n, f32, false, plan_words, &words));
        }
      }
    }
  }
  // one read alone: the layout of a batch of one, without an allocation
  for (int32_t m = 1; m <= kRowsMaxM; ++m) {
    const RowLayout batch = rows_layout({{0, m}}, true, 1);
    g_allocations = 0;
    RowPack pack;
    const RowLayout one = one_layout(m, &pack);
    RowsArgs a{};
    a.cus = 256;
    int64_t words = 0;
    (void)rows_best_cut(a, one, true, 1000 * (int64_t)m, false, false, INT64_MAX, &words);
    CHECK(g_allocations == 0);
    CHECK(one.nclasses == 1 && batch.nclasses == 1);
    CHECK(memcmp(&one.classes[0], &batch.classes[0], sizeof(RowClass)) == 0);
    CHECK(memcmp(&pack, &batch.packs[0], sizeof pack) == 0);
  }
  // scratch does not grow with reads that fill the device by themselves
  for (int32_t m : {250, 2000}) {
    Reads one(1, {0, m}), many;
    for (int32_t i = 0; i < 65536; ++i) many.emplace_back(i, m);
    const RowLayout few = rows_layout(one, true, kRowsReads);
    const RowLayout all = rows_layout(many, false, kRowsReads);
    CHECK(rows_most_words(few, 256) <= (m == 250 ? 1 << 20 : 5 << 20));
    CHECK(rows_most_words(all, 256) == 0);
    CHECK(!alone_pays(all, 256));
  }
  printf("ok %d\n", g_case);
  return 0;
}
