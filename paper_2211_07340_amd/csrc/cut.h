// How the host cuts a row-lane launch (kernels in rows.h): reads packed into
// waves, the reference into column segments, by a model of the launch's time.
#pragma once
#include <math.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "common.h"

namespace sdtw {

// Reads on the lanes of waves: packs class by class (rows per lane), most
// rows per lane first.
struct RowLayout {
  std::vector<RowPack> packs;
  int32_t nclasses = 0;
  RowClass classes[kRowsClasses];
  int32_t max_held = 0;  // most rows that a chunk's resident row holds already
};

// Rows per lane of a read that shares waves with reads like it: those that
// leave the smallest share of the lanes' work to idle lanes and to what a
// step does besides cells (about 1.5 instructions a column against 2 R).
static int rows_to_share(int32_t m, int max_reads) {
  int best = 0;
  double most = 0.0;
  for (int R : kRowsPerLane) {
    const int32_t lanes = rows_lanes(m, R);
    if (!lanes) continue;
    const int32_t reads = std::min<int32_t>(max_reads, kLanes / lanes);
    const double part = (double)reads * m / (kLanes * (R + 0.2));
    if (part > most) {
      most = part;
      best = R;
    }
  }
  return best;
}
// Rows per lane of a read alone in its wave: the fewest (the shortest steps).
static int rows_alone(int32_t m) {
  for (int R : {2, 4, 8, 16, 32})
    if (rows_lanes(m, R)) return R;
  return 0;
}

// Packs of the reads (item, rows), longest first.  `alone`: a read per pack;
// else reads of the same rows per lane share a wave while their lanes fit,
// each pack filled with the longest that still fit.
static RowLayout rows_layout(const std::vector<std::pair<int32_t, int32_t>>& reads, bool alone,
                             int max_reads) {
  RowLayout out;
  // the reads class by class, longest first: so in a class those of a number of
  // lanes follow one another, most lanes first
  std::vector<uint8_t> kind(reads.size());
  std::vector<int32_t> of(reads.size());
  int32_t count[kRowsClasses + 1] = {};
  int32_t m = 0;
  int at = 0;
  for (size_t i = 0; i < reads.size(); ++i) {
    if (reads[i].second != m) {
      m = reads[i].second;
      const int R = alone ? rows_alone(m) : rows_to_share(m, max_reads);
      at = (int)(std::find(kRowsPerLane, kRowsPerLane + kRowsClasses, R) - kRowsPerLane);
    }
    kind[i] = (uint8_t)at;
    ++count[at + 1];
  }
  for (int k = 0; k < kRowsClasses; ++k) count[k + 1] += count[k];
  int32_t next[kRowsClasses];
  std::copy(count, count + kRowsClasses, next);
  for (size_t i = 0; i < reads.size(); ++i) of[(size_t)next[kind[i]]++] = (int32_t)i;
  if (alone) max_reads = 1;
  if (alone) out.packs.reserve(reads.size());
  for (int k = kRowsClasses - 1; k >= 0; --k) {
    if (count[k] == count[k + 1]) continue;
    const int R = kRowsPerLane[k];
    int32_t head[kLanes + 1] = {}, end[kLanes + 1] = {};  // the reads of l lanes: of[head, end)
    for (int32_t i = count[k]; i < count[k + 1]; ++i) {
      const int32_t l = rows_lanes(reads[(size_t)of[(size_t)i]].second, R);
      if (end[l] == 0) head[l] = i;
      end[l] = i + 1;
    }
    RowClass c{};
    c.rows_per_lane = R;
    c.first_pack = (int32_t)out.packs.size();
    for (int top = kLanes; top >= 1;) {
      if (head[top] == end[top]) {
        --top;
        continue;
      }
      RowPack p{};
      int32_t room = kLanes;
      while (p.nreads < max_reads && room > 0) {
        int l = std::min(room, top);
        while (l >= 1 && head[l] == end[l]) --l;
        if (l < 1) break;
        const auto& rd = reads[(size_t)of[(size_t)head[l]++]];
        p.item[p.nreads] = rd.first;
        p.lane0[p.nreads] = kLanes - room;
        ++p.nreads;
        room -= l;
        p.max_lanes = std::max(p.max_lanes, (int32_t)l);
        p.max_m = std::max(p.max_m, rd.second);
      }
      for (int j = p.nreads; j <= kRowsReads; ++j) p.lane0[j] = kLanes - room;
      c.max_m = std::max(c.max_m, p.max_m);
      c.max_lanes = std::max(c.max_lanes, p.max_lanes);
      out.packs.push_back(p);
    }
    c.npacks = (int32_t)out.packs.size() - c.first_pack;
    out.classes[out.nclasses++] = c;
  }
  return out;
}
// One read of m rows, alone in its wave: the pack goes to *pack, and nothing is
// allocated.
static RowLayout one_layout(int32_t m, RowPack* pack) {
  RowLayout out;
  RowClass& c = out.classes[out.nclasses++];
  c = RowClass{};
  c.rows_per_lane = rows_alone(m);
  c.npacks = 1;
  c.max_m = m;
  c.max_lanes = rows_lanes(m, c.rows_per_lane);
  *pack = RowPack{};
  pack->nreads = 1;
  pack->max_lanes = c.max_lanes;
  pack->max_m = m;
  for (int j = 1; j <= kRowsReads; ++j) pack->lane0[j] = c.max_lanes;
  return out;
}

// The time of a launch in cycles, by a model of the sweep and the halo
// kernel: a wave's share of its SIMD for a step at R rows per lane, with
// `waves` on the SIMD, is cells[] for each row and over[] besides (LDS, rows
// handed on, latency that nothing hides).  Fitted to the sweep's times at 2 to
// 32 rows per lane x 1, 2, 3, 4 and 8 waves (29,892 columns, both types and
// both ways to hand rows on; within 7% from 4 rows per lane up).  The float32
// cells do best with two or four waves: 16 rows per lane x 59,796 columns
// reach 18.0 TCUPS with two, 16.0 with three and 17.4 with four, the int16
// cells 15.7, 16.4 and 16.5.  Resident rows cost a step about 170, 110 and 90
// cycles more (86 packs at 20 rows per lane x 59,796 columns).
struct RowCost {
  bool dpp, f32, stream;
  double step(int R, double waves) const {
    struct Fit { double over[4], cells[4]; };
    static const Fit kLds[] = {{{230, 105, 80, 72}, {33.6, 35.2, 34.8, 34.8}},
                               {{205, 115, 75, 92}, {51.5, 31.6, 36.6, 32.2}}};
    static const Fit kDpp[] = {{{165, 95, 85, 85}, {33.6, 33.1, 32.5, 32.5}},
                               {{150, 113, 82, 80}, {51.7, 39.2, 37.4, 36.2}}};
    const Fit& f = (dpp ? kDpp : kLds)[f32];
    const int w = (int)std::min(std::max(waves, 1.0), 4.0) - 1;
    static const double kResident[4] = {170, 110, 90, 90};
    return f.over[w] + f.cells[w] * R + (stream ? kResident[w] : 0.0);
  }
};
// What a step costs besides its cells, in rows: waves of different rows per
// lane end together when columns are dealt out by rows and this.
constexpr double kRowsStepOver = 2.2;

// Waves of a SIMD that a launch is cut into, one after another or at once.  0: one
// segment per pack, without halo and scratch, where the reads' rows make up much
// of the reference (512 reads of 2,000 rows x 4,000 columns: 877 us in two
// segments, 578 in one).
constexpr int kRowsRounds[] = {0, 1, 2, 3, 4, 6, 8, 12, 16};
// More than four pay where the packs' last, shorter segments are a good part of
// the waves; few packs have equal waves already (22 packs are cut in 4 rounds, 86
// in 6, 300 in 16), and their scratch stays small.
static bool rounds_pay(int rounds, const RowLayout& lay) {
  return rounds <= 4 || (int64_t)lay.packs.size() >= 12 * (int64_t)rounds;
}

// Cuts the reference of n columns into segments for every class so that each
// SIMD gets `rounds` waves of about equal work (or as many as there are
// packs for); fills a's counts.  Returns the modelled cycles; *words: the
// scratch (64-bit words) needed.
static double rows_cut(RowsArgs& a, const RowLayout& lay, int64_t n, double rounds, RowCost cost,
                       bool stream, int64_t* words) {
  const int64_t room = (int64_t)(a.cus * 4 * rounds);
  auto columns = [&](const RowClass& c, double tau) {  // a segment's, for waves of tau row steps
    const double cols = 4.0 * (tau / (c.rows_per_lane + kRowsStepOver) - c.max_lanes);
    const int64_t least = std::max<int64_t>(64, c.max_m / 4);
    const int64_t whole = (n + 63) & ~(int64_t)63;
    return std::min(whole, (std::max(least, (int64_t)std::min(cols, (double)whole)) + 63) &
                               ~(int64_t)63);
  };
  auto count = [&](double tau) {
    int64_t w = 0;
    for (int k = 0; k < lay.nclasses; ++k) {
      const RowClass& c = lay.classes[k];
      const int64_t cols = columns(c, tau);
      w += c.npacks * ((n + cols - 1) / cols);
    }
    return w;
  };
  // the shortest waves that the SIMDs have room for
  double lo = 0.0, hi = (0.25 * (double)n + 2 * kLanes) * (32.0 + kRowsStepOver);
  for (int i = 0; i < 40 && count(lo) > room && hi - lo > 4e-3 * hi; ++i) {
    const double mid = 0.5 * (lo + hi);
    (count(mid) > room ? lo : hi) = mid;
  }
  const double tau = count(lo) > room ? hi : lo;
  a.nclasses = lay.nclasses;
  a.nwaves = a.nhalo = 0;
  int64_t bound = 0, results = 0;
  for (int k = 0; k < a.nclasses; ++k) {
    RowClass c = lay.classes[k];
    const int64_t cols = columns(c, tau), s = (n + cols - 1) / cols;
    c.nseg = (int32_t)s;
    c.segcols = (int32_t)cols;
    c.first_wave = a.nwaves;
    c.first_halo = a.nhalo;
    c.bound_at = bound;
    c.result_at = results;
    a.nwaves += (int32_t)(s * c.npacks);
    a.nhalo += (int32_t)((s - 1) * c.npacks);
    if (s > 1) {
      bound += (s - 1) * c.npacks * rows_bound_words(c.rows_per_lane);
      results += (int64_t)c.npacks * (stream ? kRowsStreamReads : kRowsReads) *
                 (rows_groups((int32_t)s) + 1);
    }
    a.cls[k] = c;
  }
  a.nresults = results;
  *words = a.nhalo ? results + (results + 1) / 2 + ((int64_t)a.nwaves + 1) / 2 + (bound + 1) / 2
                   : 0;
  // The sweep: up to four waves of a SIMD (chunks: fewer, see rows_side_by_side) run
  // side by side and the fullest SIMD ends last; more follow one another, and what
  // is left at the end is about how far the longest wave exceeds the mean, or the
  // last round's gap.
  // Each pack's last segment is shorter than the others, so many rounds of
  // short waves fill the SIMDs better than one (1,024 reads of 250 to 500
  // rows x 10 M columns: 248 ms with 4, 231 with 8, 224 with 16).  A launch
  // takes about 8 us besides its steps.
  const double simds = 4.0 * a.cus, per = a.nwaves / simds;
  const double side = rows_side_by_side(stream, cost.f32, a.cls[0].rows_per_lane);
  double work = 0.0, longest = 0.0, halo = 0.0;
  for (int k = 0; k < a.nclasses; ++k) {
    const RowClass& c = a.cls[k];
    const double steps = c.segcols / 4.0 + c.max_lanes;
    const double wave = steps * cost.step(c.rows_per_lane, std::min(std::ceil(per), side));
    work += wave * (double)c.nseg * c.npacks / simds;
    longest = std::max(longest, wave);
    if (c.nseg > 1) {
      // (a climb of 0.3 of the rows held: 0.05 for a read that fits nowhere,
      // 0.35 to 0.65 for an on-target read)
      const double h = (1.125 * c.max_m + 64.0 + 0.3 * lay.max_held) / 4.0 + c.max_lanes;
      halo += h * (double)(c.nseg - 1) * c.npacks / a.nhalo *
              (RowCost{cost.dpp, cost.f32, false}.step(c.rows_per_lane, 4.0) +
               (cost.dpp ? 0.0 : 20.0));
    }
  }
  const double mean = work / per;
  const double sweep = per > side ? work + std::max(longest - mean, 0.5 * (std::ceil(per) - per) * mean)
                                 : std::max(work, longest * std::ceil(per));
  // A halo is two waves, and the launch takes about one more (1.0 to 1.3 at 2
  // to 30 rows per lane x 1 to 7 waves per SIMD): it ends with those that try
  // again and with the fullest SIMDs.  (With rows handed on in registers, long halos
  // few enough for SIMDs of their own take little more than one: 7 of 2,000 rows 466
  // us a call, 421 modelled, 707 with a wave more.)
  const double waves = 2.0 * a.nhalo / simds;
  const double more = cost.dpp ? std::min(halo, std::max(halo * waves, 8000.0)) : 1.3 * halo;
  halo = halo * std::max(waves, 1.0) + more;
  return sweep + halo + (a.nhalo ? 35000.0 : 20000.0);
}

// The best of the cuts with scratch of at most most_words words (one segment per
// pack needs none), its modelled cycles, and whether to hand rows on in registers
// (packs of one read, `alone`).
static double rows_best_cut(RowsArgs& a, const RowLayout& lay, bool alone, int64_t n, bool f32,
                            bool stream, int64_t most_words, int64_t* words) {
  double best = -1.0;
  RowsArgs at = a;
  for (int dpp = 0; dpp <= (alone ? 1 : 0); ++dpp) {
    for (int rounds : kRowsRounds) {
      if (!rounds_pay(rounds, lay)) continue;
      int64_t w = 0;
      const double t = rows_cut(at, lay, n, rounds, RowCost{dpp != 0, f32, stream}, stream, &w);
      if (w > most_words && at.nhalo) continue;
      if (best < 0.0 || t < best) {
        best = t;
        a.nclasses = at.nclasses;
        a.nwaves = at.nwaves;
        a.nhalo = at.nhalo;
        a.nresults = at.nresults;
        std::copy(at.cls, at.cls + kRowsClasses, a.cls);
        a.dpp = dpp;
        *words = w;
      }
    }
  }
  return best;
}
// The scratch (64-bit words) for the cuts of a batch that are tried on references
// of any length, at most kMostPlanWords (1,024 reads of 250 to 500 rows x 10 M
// columns in 16 rounds take 11.9 M, and 224 ms; in 12 rounds 227).
constexpr int64_t kMostPlanWords = 12 << 20;
static int64_t rows_most_words(const RowLayout& lay, int cus) {
  int64_t most = 0;
  for (int rounds : kRowsRounds) {
    if (!rounds_pay(rounds, lay)) continue;
    RowsArgs a{};
    a.cus = cus;
    int64_t w = 0;
    (void)rows_cut(a, lay, INT32_MAX - 2 * kPadUnit, rounds, RowCost{}, false, &w);
    most = std::max(most, w);
  }
  // (on some shorter references rounding gives a class a few segments more)
  return std::min(most + most / 8, kMostPlanWords);
}
// Whether reads alone in their waves are worth a layout: not with four waves of
// shared ones for every SIMD.
static bool alone_pays(const RowLayout& shared, int cus) {
  return (int64_t)shared.packs.size() < 16 * (int64_t)cus;
}
// Whether reads of up to kRowsMaxM rows run on the row-lane kernel beside longer
// ones, which run before them on the column-lane kernels: not if few long reads
// leave more of the device idle meanwhile than the row-lane kernel saves on the
// others.  In rows, all against the same columns: the device takes about 600
// rows of a batch in the time of one of the longest read (21 ns a column and read
// at 2 waves, 12.6e12 cells a second), and the row-lane kernel saves about 0.19 of
// theirs (15.5e12).  One read of 4,096 rows and 2,000 of 500 x 59,796 columns: 16.1
// ms apart, 12.1 together, tuned 10.1 and 7.2; 1,000 of 2,500 and 1,000 of 1,800:
// 18.2 and 18.5.  (Reads of up to 64 rows have a launch of their own there too.)
static bool split_pays(int32_t max_m, int32_t next_m, double long_rows, double short_rows,
                       int cus) {
  return next_m < skew_min_m(1) ||
         600.0 / 256.0 * cus * max_m - long_rows < 0.19 * short_rows;
}
// The parts of the scratch of a cut launch.
static void rows_scratch(RowsArgs& a, uint64_t* s) {
  if (!a.nhalo) return;
  a.keys = s;
  a.done = (uint32_t*)(s + a.nresults);
  a.fail = (uint32_t*)(s + a.nresults + (a.nresults + 1) / 2);
  a.bound = a.fail + (((int64_t)a.nwaves + 1) & ~(int64_t)1);
}

}  // namespace sdtw
