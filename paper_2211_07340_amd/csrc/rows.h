// Row-lane alignment: lanes own rows of the query, the reference streams by.
//
// Lane l of a wave owns R (or R - 1) consecutive rows of a read, their query
// values and the previous column's costs in registers; the wave walks the
// reference four columns at a time, lane l one step (four columns) behind
// lane l - 1.  A step is 4 R cells: for the four new columns a lane takes
// the row above its own from the lane to its left (through LDS, written a
// step earlier) and the four reference values from LDS.  There is no tile to
// switch and no row to hand from tile to tile, so a step is almost nothing
// but cells: 8 R VALU instructions on int16 (v_min3_u32 + v_sad_u32) and 12 R on
// float32 (v_sub + v_min3 + v_add; 8 cycles per 64 cells either way) and about
// one more.  Reads of 64 R rows or fewer share a wave, each on its own lanes.
//
// Uneven rows.  A read of M rows takes L lanes, the first a = M - L (R - 1)
// of them with R rows and the others with R - 1, which leaves no row of the
// read unowned and no padded row in any result.  Every lane publishes its
// two last register rows at per-lane LDS addresses, of which one is a dump
// slot, so which row is a lane's last costs no instruction.  In the same
// way a read's first lane takes the row above from a slot of zeros (the
// free start) or from a copy of the resident row, and its last lane
// publishes into the output slots that the wave folds every 64 steps into
// the running (cost, first column) minimum (and, extending a resident row,
// writes back).
//
// Column segments.  The reference is cut into segments of `segcols` columns
// that waves work on at once, so the parallelism does not hang on the number
// of reads.  A segment needs the column left of it, gamma(., c0 - 1).  The
// halo kernel computes it without waiting for the segment to the left: it
// starts `H` columns earlier and runs two recurrences side by side, one with
// +inf and one with a lower bound of every cost (0, or the minimum of the
// resident row: a chunk's row never costs less than the cheapest cell of the
// row it extends) as the column before its first.  Eq. 1 is monotone in its
// inputs, in float32 as in integers (min, |x - y| + v and rounding are), so
// the true column lies between the two; where they are equal in every row,
// that is the true column, and what follows from it is exact.  Paths that
// start in the halo beat paths that cross all of it after about as many
// columns as the read has rows, or when a row is extended as it takes to
// climb from the row's minimum to its other costs (halo_body has the figures); a
// segment whose column does not settle in three attempts, each twice as far
// left (a stretch without variation; more attempts for chunks), is left to
// the wave of the segment to its left, which goes on into it: its own state at
// the border is exact.
//
// What bounds it, and what it measured (MI355X, against the column-lane
// kernels of align.hip and the row scan of wide.hip that ran before).  The
// sweep is bound by VALU issue: on int16 2.02 to 2.05 instructions per 64 cells from
// 16 rows per lane up, of which 2 are the cells' (float32: 3.02 and 3), at 4.3 to
// 4.5 cycles each with three or four waves on a SIMD (bare v_min3_u32 and v_sad_u32
// reach 4.5), the rest being clock (2.2-2.35 of the 2.4 GHz, 2.0 on float32) and idle
// lanes.  1,024 reads of 250-500 rows x 9,999,990 columns 306 -> 224 ms, 4,096 of
// 250 x 59,796 in float32 4.2 -> 3.4 ms, 8,192 of 100-2,000 x 59,796 34.3 -> 32.4
// ms, 48 of 20-300 x 59,796 2.88 -> 0.14 ms, one of 250 x 9,999,990 2.09 -> 0.29 ms
// and x 59,796 0.53 -> 0.06 ms, two 400-row chunks on 256 resident rows x 9,999,990
// 340 -> 129 ms, on 4 one by one 26.8 -> 4.3 ms.
#pragma once
#include <limits.h>

#include <algorithm>

#include "cells.h"
#include "device.h"

namespace sdtw {
namespace {

constexpr int kMainWaves = 4;  // waves of a sweep workgroup: one per SIMD, each on its own work
constexpr int kHaloWaves = 2;  // of a halo workgroup: the two recurrences of a segment

// LDS of a wave, in bytes: 128 groups of four reference values (the window
// of the 64 steps of a block over 64 lanes), then four planes, one per step
// modulo 4, each with a 16-byte slot per lane, a slot of zeros, a dump slot (STREAM:
// the last lane's, which none reads), and per read of the wave 8 output slots and
// (STREAM) 8 slots of the resident row.  Four workgroups of four waves fit on a
// CU, and one of either kind beside three of STREAM that are held apart
// (share_lds).
template <bool STREAM>
struct Lds {
  static constexpr int kReads = STREAM ? kRowsStreamReads : kRowsReads;
  static constexpr int kPairs = (kReads + 1) / 2;
  static constexpr int kY = 2048;  // bytes before the planes
  static constexpr int kZero = 1024, kDump = STREAM ? 16 * 63 : 1040;
  static constexpr int kOut = STREAM ? 1040 : 1056;
  static constexpr int kAcc = kOut + 128 * kReads;
  static constexpr int kPlane = kAcc + (STREAM ? 128 * kReads : 0);
  static constexpr int kBytes = kY + 4 * kPlane;
  static_assert(kMainWaves * kBytes <= (128 - 3 * 33) * 1280);
};

__device__ __forceinline__ uint4 lds_get(const char* lds, uint32_t at) {
  return *(const uint4*)(lds + at);
}
__device__ __forceinline__ void lds_put(char* lds, uint32_t at, uint4 v) {
  *(uint4*)(lds + at) = v;
}
// Orders the wave's LDS operations for the compiler (the hardware executes a
// wave's LDS operations in order).
__device__ __forceinline__ void lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// v of the lane to the left; in lane 0 `first`, or 0
__device__ __forceinline__ uint32_t left_lane(uint32_t v, uint32_t first) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t left_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);
}

// Four columns of a lane's R rows: v[r][c] from the rows above s[c], the
// diagonal sd left of s[0] and the previous column h[r].  Cells are written
// out by anti-diagonals, whose cells are independent.  Returns the last two
// rows.
template <class F, int R>
__device__ __forceinline__ void cells4(const uint32_t (&x)[R], uint32_t (&h)[R], uint32_t& sd,
                                       const uint4& s4, const uint4& y4, uint4& last,
                                       uint4& before) {
  const uint32_t s[4] = {s4.x, s4.y, s4.z, s4.w}, y[4] = {y4.x, y4.y, y4.z, y4.w};
  uint32_t v[R][4];
  static_for<0, R + 3>([&](auto dc) {
    static_for<0, 4>([&](auto cc) {
      constexpr int c = decltype(cc)::value, r = decltype(dc)::value - c;
      if constexpr (r >= 0 && r < R) {
        const uint32_t up = r ? v[r ? r - 1 : 0][c] : s[c];
        const uint32_t dg = c ? (r ? v[r ? r - 1 : 0][c ? c - 1 : 0] : s[c ? c - 1 : 0])
                              : (r ? h[r ? r - 1 : 0] : sd);
        const uint32_t lf = c ? v[r][c ? c - 1 : 0] : h[r];
        v[r][c] = F::cell(x[r], y[c], min3u(up, dg, lf));
      }
    });
  });
#pragma unroll
  for (int r = 0; r < R; ++r) h[r] = v[r][3];
  sd = s[3];
  last = make_uint4(v[R - 1][0], v[R - 1][1], v[R - 1][2], v[R - 1][3]);
  before = make_uint4(v[R - 2][0], v[R - 2][1], v[R - 2][2], v[R - 2][3]);
}

// A call of one read brings its pack and work item along as arguments.
__device__ __forceinline__ RowPack get_pack(const RowsArgs& a, int32_t i) {
  return a.packs ? a.packs[i] : a.pack;
}
__device__ __forceinline__ StreamItem get_item(const RowsCall& a, int32_t i) {
  return a.items ? a.items[i] : a.item;
}

// What a lane of a pack works on.
struct LaneRows {
  int32_t item;    // work item (read of the batch, or entry of the stream items)
  int32_t j;       // the read's place in the pack
  int32_t lag;     // the lane's place among the read's lanes: steps it trails the first
  int32_t nr;      // rows of this lane (0: idle)
  bool first, last, full;
  int64_t q0;      // query index of the lane's first row
  uint32_t* acc;   // STREAM: the resident row
  bool resident;   // STREAM: it holds rows already,
  int32_t held;    // so many
};

template <int R, bool STREAM>
__device__ __forceinline__ LaneRows lane_rows(const RowsCall& a, const RowPack& pk, int lane) {
  LaneRows w{};
  int32_t lane0 = 0, lane1 = pk.lane0[1];
  w.item = pk.item[0];
#pragma unroll
  for (int k = 1; k < Lds<STREAM>::kReads; ++k) {
    if (k < pk.nreads && lane >= pk.lane0[k]) {
      w.j = k;
      w.item = pk.item[k];
      lane0 = pk.lane0[k];
      lane1 = pk.lane0[k + 1];
    }
  }
  const int32_t lanes = lane1 - lane0, l = lane - lane0;
  int64_t q0;
  int32_t m;
  if constexpr (STREAM) {
    const StreamItem it = get_item(a, w.item);
    q0 = it.q0;
    m = it.m;
    w.acc = it.acc;
    w.resident = it.m_old > 0;
    w.held = it.m_old;
  } else {
    q0 = a.offs ? a.offs[w.item] : 0;
    m = a.offs ? (int32_t)(a.offs[w.item + 1] - q0) : a.single_m;
  }
  const int32_t nfull = m - lanes * (R - 1);  // lanes with R rows, the first ones
  w.full = l < nfull;
  w.nr = l >= lanes ? 0 : (w.full ? R : R - 1);
  w.lag = l < lanes ? l : 0;
  w.first = l == 0;
  w.last = l == lanes - 1;
  w.q0 = q0 + (w.full ? l * R : l * (R - 1) + nfull);
  return w;
}

template <class F, int R>
__device__ __forceinline__ void load_rows(const RowsCall& a, const LaneRows& w,
                                          uint32_t (&x)[R]) {
  const typename F::qin* q = (const typename F::qin*)a.q;
#pragma unroll
  for (int r = 0; r < R; ++r) x[r] = r < w.nr ? (uint32_t)F::to_lds(q[w.q0 + r]) : 0u;
}

// Columns [c0, c0 + 4 ngroups) of a pack, from the column left of them (h,
// and sd above each lane's first row) to its last.  MAIN: folds the reads' last
// rows in columns below c1 into best, bestj (and writes them back, STREAM);
// otherwise every lane stops behind its last column.  DPP (one read in the
// wave): the row above comes from the lane to the left by a register move
// instead of through LDS, which costs eight instructions a step more and
// saves the LDS round trip, the better bargain where a SIMD has one wave.
template <class F, int R, bool STREAM, bool DPP, bool MAIN>
__device__ __forceinline__ void sweep(const RowsCall& a, const RowPack& pk, const LaneRows& w,
                                      char* lds, int32_t c0, int32_t ngroups, int32_t c1,
                                      const uint32_t (&x)[R], uint32_t (&h)[R], uint32_t& sd,
                                      uint32_t (&best)[Lds<STREAM>::kPairs],
                                      int32_t (&bestj)[Lds<STREAM>::kPairs]) {
  using D = Lds<STREAM>;
  constexpr int P = D::kPlane, NP = D::kPairs;
  const int lane = (int)threadIdx.x & 63, half = lane >> 5, i32 = lane & 31;
  // where the lane's last row goes: to the lane on its right, or out
  const uint32_t slot = D::kY + 16u * lane, dump = D::kY + D::kDump;
  const bool out = w.last && w.nr > 0;
  const uint32_t mine = out ? D::kY + D::kOut + 128u * w.j : (DPP ? dump : slot);
  const uint32_t wa0 = w.nr > 0 && (DPP || w.full) ? mine : dump;
  const uint32_t wb0 = w.nr > 0 && !w.full ? mine : dump;
  const uint32_t wai = out && (DPP || w.full) ? 16u : 0u, wbi = out && !w.full ? 16u : 0u;
  // where the row above its first comes from: the lane on its left, zeros,
  // or the resident row
  const bool from_acc = STREAM && w.first && w.nr > 0 && w.resident;
  uint32_t ra0 = w.first || w.nr == 0 ? D::kY + D::kZero : slot - 16u, rai = 0u;
  if (STREAM && from_acc) {
    ra0 = D::kY + D::kAcc + 128u * w.j;
    rai = 16u;
  }
  [[maybe_unused]] const bool lane0_acc =
      STREAM && __builtin_amdgcn_readfirstlane(from_acc ? 1 : 0) != 0;
  if constexpr (DPP && STREAM) {
    // every lane reads lane 0's slots (only lane 0 keeps the value)
    if (lane0_acc) {
      ra0 = D::kY + D::kAcc;
      rai = 16u;
    } else {
      ra0 = D::kY + D::kZero;
    }
  }
  if (lane < 4) lds_put(lds, D::kY + lane * P + D::kZero, make_uint4(0, 0, 0, 0));

  // Per pair of reads: lanes 0 .. 31 serve the first, lanes 32 .. 63 the
  // second, 32 steps at a time.
  int32_t lag[NP];                            // steps by which the read's last lane trails
  [[maybe_unused]] uint32_t* acc[NP];         // STREAM: its resident row,
  [[maybe_unused]] bool res[NP];              // whether it holds rows,
  [[maybe_unused]] uint4 an[NP];              // and its next 32 groups
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const bool second = half && 2 * k + 1 < D::kReads;
    lag[k] = (second ? pk.lane0[2 * k + 2 < D::kReads ? 2 * k + 2 : D::kReads] -
                           pk.lane0[2 * k + 1]
                     : pk.lane0[2 * k + 1] - pk.lane0[2 * k]) - 1;
    if constexpr (STREAM) {
      acc[k] = nullptr;
      res[k] = false;
      an[k] = make_uint4(0, 0, 0, 0);
      if (2 * k + half < pk.nreads) {
        const StreamItem it = get_item(a, half ? pk.item[2 * k + 1 < kRowsReads ? 2 * k + 1 : 0]
                                               : pk.item[2 * k]);
        acc[k] = it.acc;
        res[k] = it.m_old > 0;
      }
    }
  }
  auto fetch_acc = [&](int32_t hb) {  // half-block hb's groups
    if constexpr (STREAM) {
#pragma unroll
      for (int k = 0; k < NP; ++k)
        if (res[k]) an[k] = *(const uint4*)(acc[k] + c0 + 4 * (int64_t)(32 * hb + i32));
    }
  };

  const uint4* const yg = (const uint4*)(a.ref + c0);
  uint4 yn = yg[lane];
  fetch_acc(0);
  uint4 o4 = make_uint4(0, 0, 0, 0);  // DPP: the lane's last row of the previous step
  const int32_t steps = ngroups + pk.max_lanes - 1;
  for (int32_t b = 0; b * 64 < steps; ++b) {
    // the block's window of reference values: the last 64 groups and the next
    lds_put(lds, 16u * lane, lds_get(lds, 1024u + 16u * lane));
    lds_put(lds, 1024u + 16u * lane, yn);
    yn = yg[64 * (b + 1) + lane];
    lds_fence();
    uint32_t ya = (64u - w.lag) * 16u;
    uint4 y4 = lds_get(lds, ya);
    for (int32_t hb = 0; hb < 2; ++hb) {
      const int32_t s0 = 64 * b + 32 * hb, left = steps - s0;
      const int32_t n4 = left < 32 ? (left + 3) / 4 : 8;
      if (n4 <= 0) break;
      if constexpr (STREAM) {
#pragma unroll
        for (int k = 0; k < NP; ++k)
          if (res[k])
            lds_put(lds, D::kY + ((lane + 3) & 3) * P + D::kAcc + 128 * (2 * k + half) +
                             (i32 >> 2) * 16, an[k]);
        fetch_acc(2 * b + hb + 1);
        lds_fence();
      }
      uint32_t ra = ra0, wa = wa0, wb = wb0;
      // Step u (modulo 4) of the half-block, `s` of the sweep.  Guarded: the
      // lanes start one step apart and, in the halo, stop so.
      auto step = [&](auto u, auto guarded, int32_t s) {
        uint4 s4;
        if constexpr (DPP) {
          if constexpr (STREAM) {
            const uint4 in = lds_get(lds, ra + ((u + 3) & 3) * P);
            s4 = make_uint4(left_lane(o4.x, in.x), left_lane(o4.y, in.y), left_lane(o4.z, in.z),
                            left_lane(o4.w, in.w));
          } else {
            s4 = make_uint4(left_lane(o4.x), left_lane(o4.y), left_lane(o4.z), left_lane(o4.w));
          }
        } else {
          s4 = lds_get(lds, ra + ((u + 3) & 3) * P);
        }
        const uint4 yc = y4;
        y4 = lds_get(lds, ya + 16u * (u + 1));
        // the next step's values are asked for here, a step ahead of their use
        // (left to itself the compiler asks just before it and waits)
        __builtin_amdgcn_sched_barrier(0);
        const int32_t g = s - w.lag;
        if (!decltype(guarded)::value || (g >= 0 && (MAIN || g < ngroups))) {
          uint4 last, before;
          cells4<F, R>(x, h, sd, s4, yc, last, before);
          if constexpr (DPP) {
            o4.x = w.full ? last.x : before.x;
            o4.y = w.full ? last.y : before.y;
            o4.z = w.full ? last.z : before.z;
            o4.w = w.full ? last.w : before.w;
            if constexpr (MAIN) lds_put(lds, wa + u * P, o4);
          } else {
            lds_put(lds, wa + u * P, last);
            lds_put(lds, wb + u * P, before);
          }
        }
        if constexpr (!DPP) lds_fence();
      };
      auto advance = [&] {
        ya += 64u;
        ra += rai;
        wa += wai;
        wb += wbi;
      };
      const int32_t lead = pk.max_lanes - 1 - s0;  // steps until every lane has started
      int32_t s4 = 0;
      for (; s4 < n4 && (!MAIN || 4 * s4 < lead); ++s4) {
        // (not unrolled: few steps of a long sweep; a halo that unrolls the steps
        // between is no faster where halos count: 250 rows x 59,796 columns 62.5 us
        // a call against 61.9)
        for (int32_t u = 0; u < 4; ++u) step(u, std::true_type{}, s0 + 4 * s4 + u);
        advance();
      }
      if constexpr (MAIN) {
        for (; s4 < n4; ++s4) {
          static_for<0, 4>([&](auto uc) { step(uc, std::false_type{}, 0); });
          advance();
        }
        // the last rows of these steps' columns
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          if (2 * k < pk.nreads) {
            const uint4 o = lds_get(lds, D::kY + (lane & 3) * P + D::kOut +
                                             128 * (2 * k + half < D::kReads ? 2 * k + half : 0) +
                                             (i32 >> 2) * 16);
            const int32_t g = s0 + i32 - lag[k];
            if ((uint32_t)g < (uint32_t)ngroups && 2 * k + half < pk.nreads) {
              const int32_t col = c0 + 4 * g;
              if (min(min3u(o.x, o.y, o.z), o.w) < best[k]) {
                const uint32_t v[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  if (col + c < c1 && v[c] < best[k]) {
                    best[k] = v[c];
                    bestj[k] = col + c;
                  }
                }
              }
              if constexpr (STREAM) *(uint4*)(acc[k] + col) = o;
            }
          }
        }
        lds_fence();
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The columns left of the segments: a workgroup of two waves per segment,
// wave 0 with the lower bound as the column before the halo, wave 1 with +inf
// ---------------------------------------------------------------------------

template <class F, int R, bool STREAM, bool DPP>
__device__ __forceinline__ void halo_body(const RowsCall& a, const RowClass& cl,
                                          const RowPack& pk, int32_t pack, int32_t seg,
                                          int32_t wave, char* smem) {
  using D = Lds<STREAM>;
  char* const lds = smem + wave * D::kBytes;
  const int lane = (int)threadIdx.x & 63;
  const LaneRows w = lane_rows<R, STREAM>(a, pk, lane);
  uint32_t x[R], h[R], sd = 0u;
  load_rows<F, R>(a, w, x);
  const int32_t c1 = seg * cl.segcols;  // the column wanted is c1 - 1
  uint32_t bound = 0u;
  if constexpr (STREAM) {
    if (w.resident) bound = w.acc[a.row_min_at];
  }
  // Columns until the two recurrences meet, measured on simulated reads: 0.8
  // to 1.1 M, and for a chunk as many columns again as a path needs to climb
  // from the resident row's minimum to the row's costs hereabouts, 0.55 to 0.65
  // held (1 - minimum / cost): nothing for a read that fits nowhere, 700 to 1,300
  // columns for an on-target read with 2,000 rows held, whatever the chunk.  (On
  // 59,796 columns in 233 segments every one of 36 chunks of 40, 270 and 400
  // rows on 400, 2,000 and 3,600 settles at once, at noise of 0.1 to 0.3 sd; with
  // 0.64 for 0.68 up to 4% try twice, which holds up the sweep.  16 reads with
  // 2,000 rows held, by 40: 1.77 ms when 1.33 M + 64 columns, doubled twice, left
  // 98% of the segments to their left neighbours, 0.17 so.)
  float climb = 0.0f;
  if constexpr (STREAM) {
    if (w.resident) {
      float cost = 0.0f;  // (a segment has at least 64 columns)
#pragma unroll
      for (int k = 0; k < 4; ++k) cost += 0.25f * F::value(w.acc[c1 - 1 - 16 * k]);
      climb = 0.68f * (float)w.held * (1.0f - F::value(bound) / cost);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) climb = fmaxf(climb, __shfl_xor(climb, off));
    climb = climb > 0.0f ? fminf(climb, 1e9f) : 0.0f;  // (0 of a row without costs)
  }
  int32_t H = pk.max_m + pk.max_m / 8 + 32 +
              __builtin_amdgcn_readfirstlane((int32_t)climb);
  H = (H + 3) & ~3;
  uint32_t* const sw = (uint32_t*)smem;  // the exchange: (R + 1) words per lane
  bool ok = false;
  // (three times: reads that repeat the reference to the value settle within
  // 1.6 M, at the second; and for a chunk on a reference without runs of equal values as
  // long as the halo is shorter than the segment that the wave to the left would
  // walk instead; where such runs are, tries in vain would take 16 chunks of 400 on
  // 9,999,990 columns, a fiftieth of them equal, from 24 to 40 ms)
  for (int attempt = 0; !ok && (attempt < 3 || (STREAM && a.far && H < cl.segcols));
       ++attempt) {
    const int32_t c0 = c1 > H ? c1 - H : 0;  // (c1 is a multiple of 4)
    const bool edge = c0 == 0;               // the left edge: +inf is the true column
    const uint32_t before = edge || wave == 1 ? F::kInf : bound;
#pragma unroll
    for (int r = 0; r < R; ++r) h[r] = before;
    sd = before;
    if (w.first) {
      sd = 0u;
      if constexpr (STREAM) {
        if (w.resident) sd = edge ? F::kInf : w.acc[c0 - 1];
      }
    }
    uint32_t best[D::kPairs];
    int32_t bestj[D::kPairs];
    sweep<F, R, STREAM, DPP, false>(a, pk, w, lds, c0, (c1 - c0) / 4, c1, x, h, sd, best, bestj);
    __syncthreads();  // both waves are done with their LDS
    if (wave == 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) sw[r * 64 + lane] = h[r];
    }
    __syncthreads();
    uint32_t differ = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r)
      differ |= r < w.nr && sw[r * 64 + lane] != h[r] ? 1u : 0u;
    ok = __syncthreads_or((int)differ) == 0 || edge;
    H = H < c1 / 2 ? 2 * H : c1;  // (c1: the left edge)
  }
  if (wave == 1) {
    uint32_t* const out = a.bound + cl.bound_at +
                          ((int64_t)(pack - cl.first_pack) * (cl.nseg - 1) + (seg - 1)) *
                              rows_bound_words(R);
#pragma unroll
    for (int r = 0; r < R; ++r) out[r * 64 + lane] = h[r];
    out[R * 64 + lane] = sd;
    if (lane == 0)
      a.fail[cl.first_wave + (pack - cl.first_pack) * cl.nseg + seg] = ok ? 0u : 1u;
    // the reads' result words, for the sweep that follows
    if (seg == 1) {
      if (lane == 0) a.fail[cl.first_wave + (pack - cl.first_pack) * cl.nseg] = 0u;
      const int32_t per = rows_groups(cl.nseg) + 1;
      const int64_t at = cl.result_at + (int64_t)(pack - cl.first_pack) * D::kReads * per;
      for (int32_t i = lane; i < D::kReads * per; i += 64) {
        a.keys[at + i] = ~0ull;
        a.done[at + i] = 0u;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The segments
// ---------------------------------------------------------------------------

// One result of `of` that meet in word `at`: true for the last to come, with
// the smallest key of all.  Atomics alone carry it, so order among them is
// enough: the minimum has come back before the count goes out.
__device__ __forceinline__ bool meet(const RowsCall& a, int64_t at, uint32_t of, uint64_t& key) {
  const uint64_t old = __hip_atomic_fetch_min(&a.keys[at], key, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::"v"((uint32_t)old), "v"((uint32_t)(old >> 32)) : "memory");
  if (__hip_atomic_fetch_add(&a.done[at], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 != of)
    return false;
  key = __hip_atomic_load(&a.keys[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// Columns [c0, c1) of a pack.
template <class F, int R, bool STREAM, bool DPP>
__device__ __forceinline__ void main_body(const RowsCall& a, const RowClass& cl,
                                          const RowPack& pk, int32_t pack, int32_t seg, int32_t c0,
                                          int32_t c1, char* lds,
                                          uint32_t (&best)[Lds<STREAM>::kPairs],
                                          int32_t (&bestj)[Lds<STREAM>::kPairs]) {
  const int lane = (int)threadIdx.x & 63;
  const LaneRows w = lane_rows<R, STREAM>(a, pk, lane);
  uint32_t x[R], h[R], sd;
  load_rows<F, R>(a, w, x);
  if (c0 > 0) {
    const uint32_t* b = a.bound + cl.bound_at +
                        ((int64_t)(pack - cl.first_pack) * (cl.nseg - 1) + (seg - 1)) *
                            rows_bound_words(R);
#pragma unroll
    for (int r = 0; r < R; ++r) h[r] = b[r * 64 + lane];
    sd = b[R * 64 + lane];
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) h[r] = F::kInf;
    sd = w.first && !(STREAM && w.resident) ? 0u : F::kInf;
  }
  sweep<F, R, STREAM, DPP, true>(a, pk, w, lds, c0, (c1 - c0 + 3) / 4, c1, x, h, sd, best, bestj);
}

// f(integral_constant<int, R>) for the class's rows per lane.  DPP: the
// powers of two alone.
template <bool DPP, class Fn>
__device__ __forceinline__ void for_rows(int32_t rows, Fn&& f) {
#define SDTW_ROWS(R) \
  case R: f(std::integral_constant<int, R>{}); break;
  if constexpr (DPP) {
    switch (rows) { SDTW_ROWS(2) SDTW_ROWS(4) SDTW_ROWS(8) SDTW_ROWS(16) SDTW_ROWS(32) }
  } else {
    switch (rows) {
      SDTW_ROWS(2) SDTW_ROWS(4) SDTW_ROWS(6) SDTW_ROWS(8) SDTW_ROWS(10) SDTW_ROWS(12)
      SDTW_ROWS(14) SDTW_ROWS(16) SDTW_ROWS(18) SDTW_ROWS(20) SDTW_ROWS(22) SDTW_ROWS(24)
      SDTW_ROWS(26) SDTW_ROWS(28) SDTW_ROWS(30) SDTW_ROWS(32)
    }
  }
#undef SDTW_ROWS
}

// (with few classes the arguments are read where they are)
template <bool DPP>
using Call = std::conditional_t<DPP, const RowsCall&, const RowsCall>;

template <class F, bool STREAM, bool DPP>
__global__ __launch_bounds__(64 * kHaloWaves, 4) void k_rows_halo(RowsArgs a) {
  extern __shared__ __align__(16) char smem[];
  const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
  const int32_t at = (int32_t)blockIdx.x;
  int c = 0;
  for (int k = 1; k < a.nclasses; ++k)
    if (at >= a.cls[k].first_halo) c = k;
  const RowClass cl = a.cls[c];
  issue_first_if_short(cl.segcols);
  const int32_t in = at - cl.first_halo;
  const int32_t pack = cl.first_pack + in / (cl.nseg - 1), seg = 1 + in % (cl.nseg - 1);
  Call<DPP> call = a;
  const RowPack pk = get_pack(a, pack);
  for_rows<DPP>(cl.rows_per_lane, [&](auto rc) {
    halo_body<F, decltype(rc)::value, STREAM, DPP>(call, cl, pk, pack, seg, wave, smem);
  });
}

// A workgroup's waves take consecutive items, mostly segments of one pack,
// and so end together.
template <class F, bool STREAM, bool DPP>
__global__ __launch_bounds__(64 * kMainWaves, 4) void k_rows_main(RowsArgs a) {
  using D = Lds<STREAM>;
  extern __shared__ __align__(16) char smem[];
  const int lane = (int)threadIdx.x & 63, half = lane >> 5;
  const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
  const int32_t at = (int32_t)blockIdx.x * kMainWaves + wave;
  if (at >= a.nwaves) return;
  if (a.skip && *a.skip) return;
  int c = 0;
  for (int k = 1; k < a.nclasses; ++k)
    if (at >= a.cls[k].first_wave) c = k;
  const RowClass cl = a.cls[c];
  issue_first_if_short(cl.segcols);
  const int32_t in = at - cl.first_wave;
  const int32_t pack = cl.first_pack + in / cl.nseg, seg = in % cl.nseg;
  Call<DPP> call = a;
  const RowPack pk = get_pack(a, pack);
  int32_t nsegs = 1;  // segments this wave covers
  if (cl.nseg > 1) {
    const uint32_t* f = call.fail + at - seg;
    if (seg > 0 && f[seg])
      nsegs = 0;  // the wave to the left comes here
    else
      while (seg + nsegs < cl.nseg && f[seg + nsegs]) ++nsegs;
  }
  uint32_t best[D::kPairs];
  int32_t bestj[D::kPairs];
#pragma unroll
  for (int k = 0; k < D::kPairs; ++k) {
    best[k] = 0xFFFFFFFFu;
    bestj[k] = INT_MAX;
  }
  if (nsegs > 0) {
    const int32_t c0 = seg * cl.segcols;
    const int32_t c1 =
        seg + nsegs == cl.nseg ? (int32_t)call.n : (seg + nsegs) * cl.segcols;
    for_rows<DPP>(cl.rows_per_lane, [&](auto rc) {
      main_body<F, decltype(rc)::value, STREAM, DPP>(call, cl, pk, pack, seg, c0, c1,
                                                     smem + wave * D::kBytes, best, bestj);
    });
  }
#pragma unroll
  for (int k = 0; k < D::kReads; ++k) {
    if (k >= pk.nreads) continue;
    uint32_t bv = half == (k & 1) ? best[k / 2] : 0xFFFFFFFFu;
    int32_t bj = half == (k & 1) ? bestj[k / 2] : INT_MAX;
    wave_argmin(bv, bj);
    if (lane == 0) {
      uint64_t key = ((uint64_t)bv << 32) | (uint32_t)bj;
      bool write = true;
      if (cl.nseg > 1) {
        // the last of the read's waves to come here writes its result
        const int32_t groups = rows_groups(cl.nseg);
        const int64_t res = cl.result_at +
                            ((int64_t)(pack - cl.first_pack) * D::kReads + k) * (groups + 1);
        if (groups) {
          const int32_t g = seg / kRowsGroup, left = cl.nseg - g * kRowsGroup;
          write = meet(call, res + 1 + g, left < kRowsGroup ? left : kRowsGroup, key);
        }
        write = write && meet(call, res, groups ? groups : cl.nseg, key);
      }
      if (write) {
        const int32_t item = pk.item[k];
        int32_t out = item;
        if constexpr (STREAM) {
          const StreamItem it = get_item(call, item);
          out = it.out;
          it.acc[call.row_min_at] = (uint32_t)(key >> 32);
        }
        F::store_cost(call.cost, out, (uint32_t)(key >> 32));
        call.end[out] = (int32_t)(uint32_t)key;
      }
    }
  }
}

// The least LDS of a workgroup (which needs `need` bytes) that lets no more than
// `share` of them onto a CU (160 KB, allocated by 1,280 bytes).
inline size_t share_lds(size_t need, int64_t share) {
  return std::max(need, (size_t)(128 / (share + 1) + 1) * 1280);
}

template <class F, bool STREAM, bool DPP>
hipError_t launch_t(const RowsArgs& a, hipStream_t st, int parts) {
  if (a.nhalo > 0 && (parts & kRowsHalo)) {
    const size_t lds = kHaloWaves * Lds<STREAM>::kBytes;
    hipLaunchKernelGGL((k_rows_halo<F, STREAM, DPP>), dim3((uint32_t)a.nhalo),
                       dim3(64 * kHaloWaves), lds, st, a);
  }
  if (!(parts & kRowsSweep)) return hipGetLastError();
  const int64_t blocks = (a.nwaves + kMainWaves - 1) / kMainWaves;
  // Long launches: an even share of the workgroups for every CU (the dispatcher
  // would fill some and leave others empty: 64 chunks of 400 rows x 10 M columns 18.0
  // ms with three on each, 18.6 as they come), and of chunk launches no more than
  // leaves short calls on other HIP streams a wave per SIMD and 37,120 bytes: 16
  // chunks x 59,796 columns beside 256 x 10 M columns waited 38 ms for a place when
  // those took four waves per SIMD.  Short launches reserve nothing, to find room
  // there; alone they take the same time either way.
  const size_t need = kMainWaves * Lds<STREAM>::kBytes;
  const int64_t even = std::max<int64_t>((blocks + a.cus - 1) / std::max(a.cus, 1), 1);
  const int64_t most =
      rows_side_by_side(STREAM, std::is_same_v<F, FmtF32>, a.cls[0].rows_per_lane);
  const size_t lds = rows_short(a) ? need : share_lds(need, std::min(even, most));
  hipError_t e = hipFuncSetAttribute((const void*)k_rows_main<F, STREAM, DPP>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_rows_main<F, STREAM, DPP>), dim3((uint32_t)blocks), dim3(64 * kMainWaves),
                     lds, st, a);
  return hipGetLastError();
}

template <class F, bool STREAM>
hipError_t launch_rows(const RowsArgs& a, hipStream_t st, int parts) {
  return a.dpp ? launch_t<F, STREAM, true>(a, st, parts)
               : launch_t<F, STREAM, false>(a, st, parts);
}

}  // namespace
}  // namespace sdtw
