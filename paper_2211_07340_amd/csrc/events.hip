// Event detection on the device: raw samples of each read -> the event values
// the alignment uses as its query (section 4.1 segments raw samples into
// events before normalisation; section 5.2 takes its R9.4 parameters from the
// two-window t-test detector of f5c and nanopolish).
//
// The detector, as this library reads it:
//  1. t statistic at each boundary position i (between samples i-1 and i),
//     window length w: means m1, m2 and population variances v1, v2 of the w
//     samples before and the w samples from i;
//         t_w(i) = |m2 - m1| / max(sqrt((v1 + v2) / w), 1e-30),
//     0 outside w <= i <= L - w.  float64, sums in index order.
//  2. Short (w = 3, threshold 1.4) and long (w = 6, threshold 9.0) peak
//     detectors with peak height 0.2 scan the positions in order (short
//     first).  Without a candidate a detector follows the running minimum of
//     t and opens a candidate once t rises more than the peak height above
//     it; with one it moves the candidate to any higher t, the short
//     detector's candidate above its threshold masks the long detector up to
//     candidate + 6 (dropping its candidate), a candidate above threshold
//     becomes valid once t falls more than the peak height below it, and a
//     valid candidate is emitted as a boundary once the position is more
//     than w / 2 past it; the detector restarts from the current t.
//  3. Events are the segments between consecutive distinct boundaries (0 and
//     L the outer ends); an event's value is the float32 rounding of the
//     float64 mean of its samples, summed in index order.
//  4. The first `trim` events (adaptor) are dropped, the next `keep` kept.
//
// The detectors are a sequential state machine, about 20 dependent operations
// a position.  But its state soon forgets where it came from (an emitted
// boundary restarts the short detector, a strong short candidate the long one):
// started blank 16 positions early it agrees with the true state, bit for
// bit, after 4 positions in the median and 13 at most (1,538 starts in simulated
// reads).  So one wave scans a read in blocks of 1,024 positions: all lanes
// compute the t statistics, 16 positions each, into LDS; lane l runs the
// machine over its 16 positions from a blank state 16 positions before; then
// every lane compares the state it started from with the one its left
// neighbour ended in, and those that differ run again from that one, until none
// does.  Lane 0 starts from the true state, so at the end all did, whatever
// the signal: the outcome is the sequential machine's.
//
// Measured on MI355X: 4,096 reads of about 3,150 samples 790 us with a lane per
// read (the machine's 2,700 positions at 700 cycles each), 130 us so (9,600
// VALU instructions a wave, half of them the float64 of the t statistics; two
// waves on a SIMD, by the 17 KB of statistics in LDS); the next 2,400 samples
// of 512 reads 660 -> 75 us (a wave on every other SIMD: its own latency).
//
// Boundaries go into a bitmap of the last 2,048 positions (they can be emitted
// out of order while a candidate of the other detector stays open), which is
// moved to a sorted list block by block; an older candidate's is inserted
// there.  The list is final below the smallest open candidate; the scan stops
// as soon as its first trim + keep boundaries are final, which is the first few
// thousand samples of a read in Read Until.  Then every lane sums one event at
// a time.
#include <float.h>
#include <limits.h>
#include <math.h>

#include "device.h"

namespace sdtw {
namespace {

constexpr int kEvPer = 16;              // positions per lane and block
constexpr int kEvBlock = 64 * kEvPer;  // positions per block
constexpr int kWShort = 3, kWLong = 6;
constexpr double kTShort = 1.4, kTLong = 9.0, kPeakHeight = 0.2, kDenFloor = 1e-30;

template <int W>
__device__ __forceinline__ double tstat(const float* __restrict__ x, int64_t L, int64_t i) {
  if (i < W || i > L - W) return 0.0;
  double s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    s1 += (double)x[i - W + k];
    s2 += (double)x[i + k];
  }
  const double m1 = s1 / (double)W, m2 = s2 / (double)W;
  double q1 = 0.0, q2 = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const double d1 = (double)x[i - W + k] - m1;
    const double d2 = (double)x[i + k] - m2;
    q1 += d1 * d1;
    q2 += d2 * d2;
  }
  const double v1 = q1 / (double)W, v2 = q2 / (double)W;
  const double den = fmax(sqrt((v1 + v2) / (double)W), kDenFloor);
  return fabs(m2 - m1) / den;
}

// a / W, correctly rounded: with r = RN(1 / W) the product is within an ulp,
// the remainder is exact, and one fused step rounds the quotient (Markstein),
// for the magnitudes that finite float32 samples lead to: 0 or 1e-122 .. 1e80.
template <int W>
__device__ __forceinline__ double div_const(double a) {
  constexpr double r = 1.0 / (double)W;
  const double q = a * r;
  return fma(fma(-q, (double)W, a), r, q);
}

// A window's mean and population variance, as tstat() sums them.
template <int W>
__device__ __forceinline__ void window(const double* x, double& mean, double& var) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) s += x[k];
  mean = div_const<W>(s);
  double q = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const double d = x[k] - mean;
    q += d * d;
  }
  var = div_const<W>(q);
}
template <int W>
__device__ __forceinline__ double tstat_of(double m1, double v1, double m2, double v2) {
  const double den = fmax(sqrt(div_const<W>(v1 + v2)), kDenFloor);
  return fabs(m2 - m1) / den;
}

// The state of both detectors; positions relative to the block's first.
constexpr int32_t kNone = INT_MIN;         // no candidate; no mask
constexpr int32_t kOld = -(1 << 30);       // a candidate from before the bitmap's window
struct Detectors {
  int32_t sp, lp;  // candidates
  int32_t lm;      // the long detector is masked up to here
  double sv, lv;   // a candidate's t, or the running minimum
  bool sok, lok;   // the candidate has become valid
};
__device__ __forceinline__ Detectors blank_detectors() {
  return Detectors{kNone, kNone, kNone, INFINITY, INFINITY, false, false};
}

// One position.  emit(p, k): detector k (0 short, 1 long) emits boundary p.
// Written with selects: the lanes of a wave are at different places of the
// machine, so branches would take every side anyway and their masks on top.
template <class Emit>
__device__ __forceinline__ void step(Detectors& d, int32_t i, double ts, double tl, Emit&& emit) {
  {
    const bool cand = d.sp != kNone;
    const bool open = !cand && ts - d.sv > kPeakHeight;  // (never with ts < sv)
    const bool higher = cand && ts > d.sv;
    d.sp = open || higher ? i : d.sp;
    d.sv = open || higher || (!cand && ts < d.sv) ? ts : d.sv;
    const bool strong = cand && d.sv > kTShort;  // the short detector masks the long one
    d.lm = strong ? d.sp + kWLong : d.lm;
    d.lp = strong ? kNone : d.lp;
    d.lv = strong ? INFINITY : d.lv;
    d.lok = d.lok && !strong;
    d.sok = d.sok || (strong && d.sv - ts > kPeakHeight);
    const bool out = cand && d.sok && i - d.sp > kWShort / 2;
    if (out) emit(d.sp, 0);
    d.sp = out ? kNone : d.sp;
    d.sv = out ? ts : d.sv;
    d.sok = d.sok && !out;
  }
  {
    const bool on = d.lm < i, cand = d.lp != kNone;
    const bool open = !cand && tl - d.lv > kPeakHeight;
    const bool higher = cand && tl > d.lv;
    const bool move = on && (open || higher);
    d.lv = move || (on && !cand && tl < d.lv) ? tl : d.lv;
    d.lp = move ? i : d.lp;
    d.lok = d.lok || (on && cand && d.lv > kTLong && d.lv - tl > kPeakHeight);
    const bool out = on && cand && d.lok && i - d.lp > kWLong / 2;
    if (out) emit(d.lp, 1);
    d.lp = out ? kNone : d.lp;
    d.lv = out ? tl : d.lv;
    d.lok = d.lok && !out;
  }
}

__device__ __forceinline__ double shfl_double(double v, int lane) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __shfl((int)(uint32_t)b, lane), hi = __shfl((int)(b >> 32), lane);
  return __longlong_as_double((int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo));
}
__device__ __forceinline__ Detectors from_lane(const Detectors& d, int lane) {
  Detectors r;
  r.sp = __shfl(d.sp, lane);
  r.lp = __shfl(d.lp, lane);
  r.lm = __shfl(d.lm, lane);
  r.sv = shfl_double(d.sv, lane);
  r.lv = shfl_double(d.lv, lane);
  const int f = __shfl((d.sok ? 1 : 0) | (d.lok ? 2 : 0), lane);
  r.sok = f & 1;
  r.lok = f & 2;
  return r;
}
// The same from position i on (a mask that has ended is none).
__device__ __forceinline__ bool same_from(const Detectors& a, const Detectors& b, int32_t i) {
  return a.sp == b.sp && a.lp == b.lp && (a.lm < i ? kNone : a.lm) == (b.lm < i ? kNone : b.lm) &&
         __double_as_longlong(a.sv) == __double_as_longlong(b.sv) &&
         __double_as_longlong(a.lv) == __double_as_longlong(b.lv) && a.sok == b.sok &&
         a.lok == b.lok;
}

// Insert b into the sorted distinct list bs[0..n) of at most cap entries;
// true if an entry had to go (the largest) or b did not fit.
__device__ __forceinline__ bool insert_bound(int64_t* bs, int32_t& n, int32_t cap, int64_t b) {
  if (n == cap && b > bs[n - 1]) return true;
  int32_t k = n;
  while (k > 0 && bs[k - 1] > b) --k;
  if (k > 0 && bs[k - 1] == b) return false;
  const bool full = n == cap;
  for (int32_t j = full ? cap - 1 : n; j > k; --j) bs[j] = bs[j - 1];
  bs[k] = b;
  if (!full) ++n;
  return full;
}

// A wave's scan of one read: the detectors over samples x[0 .. L), positions
// in order, and the boundaries they emit.
struct Scan {
  struct Shared {
    // t statistics of a block (16 positions of a lane 17 doubles apart: no
    // bank conflicts); before them, in the same place, its samples, likewise
    double ts[64 * (kEvPer + 1)], tl[64 * (kEvPer + 1)];
    uint32_t bits[64];
    int64_t old[2];  // boundaries of candidates older than the window, or -1
    int32_t n;       // list entries after an insertion
    int32_t lost;
  };
  Shared* sh;
  const float* x;
  int64_t L;
  Detectors d;         // uniform over the wave, as the rest
  int64_t old_s, old_l;  // positions of candidates marked kOld
  int64_t* list;       // sorted distinct boundaries from before the window
  int32_t n, cap;
  bool lost;           // a boundary did not fit
  int64_t b0;          // the block's first position
  uint32_t word;       // this lane's 32 positions from b0 - 1024 + 32 lane on

  __device__ __forceinline__ void statistics(int64_t nblk) {
    const int lane = (int)threadIdx.x;
    float* const xs = (float*)sh->ts;
    __syncthreads();
    for (int q = lane; q < kEvBlock + 12; q += 64) {
      const int64_t i = b0 - 6 + q;
      xs[q + (q >> 4)] = i >= 0 && i < L ? x[i] : 0.0f;
    }
    __syncthreads();
    const int64_t from = b0 + kEvPer * lane;
    double* const ts = sh->ts + (kEvPer + 1) * lane;
    double* const tl = sh->tl + (kEvPer + 1) * lane;
    float xf[kEvPer + 11];
    bool odd = false;
#pragma unroll
    for (int k = 0; k < kEvPer + 11; ++k) {
      xf[k] = xs[17 * lane + k + (k >> 4)];  // x[from - 6 + k]
      odd = odd || !(fabsf(xf[k]) < INFINITY);
    }
    __syncthreads();
    if (__ballot(odd)) {
      // infinities and NaN: as written (the fast quotients are for finite values)
      for (int j = 0; j < kEvPer; ++j) {
        if (kEvPer * lane + j >= nblk) break;
        ts[j] = tstat<kWShort>(x, L, from + j);
        tl[j] = tstat<kWLong>(x, L, from + j);
      }
    } else {
      double xd[kEvPer + 11], m3[kEvPer + 6], v3[kEvPer + 6], m6[kEvPer + 6], v6[kEvPer + 6];
#pragma unroll
      for (int k = 0; k < kEvPer + 11; ++k) xd[k] = (double)xf[k];
#pragma unroll
      for (int k = 0; k < kEvPer + 6; ++k) {  // windows that start at from - 6 + k
        window<6>(xd + k, m6[k], v6[k]);
        if (k >= 3) window<3>(xd + k, m3[k], v3[k]);
        if (k >= 6) {
          const int64_t i = from + k - 6;
          ts[k - 6] = i < kWShort || i > L - kWShort
                          ? 0.0
                          : tstat_of<3>(m3[k - 3], v3[k - 3], m3[k], v3[k]);
          tl[k - 6] = i < kWLong || i > L - kWLong
                          ? 0.0
                          : tstat_of<6>(m6[k - 6], v6[k - 6], m6[k], v6[k]);
        }
      }
    }
    __syncthreads();
  }

  // Positions [b0, b0 + nblk).
  __device__ __forceinline__ void block(int32_t nblk) {
    const int lane = (int)threadIdx.x;
    statistics(nblk);
    const int32_t first = kEvPer * lane;
    const bool in = first < nblk;
    // boundaries: bit p - first + 48 for p >= first - 48, one older per detector
    uint64_t mask = 0;
    int32_t far_s = kNone, far_l = kNone;
    auto emit = [&](int32_t p, int k) {
      if (p >= first - 48)
        mask |= 1ull << (p - first + 48);
      else if (k == 0)
        far_s = p;
      else
        far_l = p;
    };
    // (the next position's statistics are asked for before the step)
    auto run = [&](Detectors& m, int32_t lane_of, int32_t n, auto&& to) {
      const double* const ts = sh->ts + (kEvPer + 1) * lane_of;
      const double* const tl = sh->tl + (kEvPer + 1) * lane_of;
      double a = ts[0], b = tl[0];
      for (int32_t j = 0; j < n; ++j) {
        const double a1 = ts[j + 1], b1 = tl[j + 1];
        step(m, kEvPer * lane_of + j, a, b, to);
        a = a1;
        b = b1;
      }
    };
    const int32_t own = nblk - first < kEvPer ? nblk - first : kEvPer;
    Detectors mine = lane == 0 ? d : blank_detectors();
    if (lane > 0 && in) run(mine, lane - 1, kEvPer, [](int32_t, int) {});
    Detectors start = mine;
    run(mine, lane, own, emit);
    while (true) {
      const Detectors left = from_lane(mine, lane > 0 ? lane - 1 : 0);
      const bool wrong = lane > 0 && in && !same_from(start, left, first);
      if (!__ballot(wrong)) break;
      if (wrong) {
        start = mine = left;
        mask = 0;
        far_s = far_l = kNone;
        run(mine, lane, own, emit);
      }
    }
    d = from_lane(mine, (nblk - 1) / kEvPer);
    // the block's boundaries into the bitmap
    sh->bits[lane] = word;
    if (lane == 0) sh->old[0] = sh->old[1] = -1;
    __syncthreads();
    if (mask) {
      const int32_t at = first - 48 + kEvBlock;  // of bit 0
      const int w = at >> 5, o = at & 31;
      const uint32_t lo = (uint32_t)(mask << o), mid = (uint32_t)(mask >> (32 - o));
      const uint32_t hi = o ? (uint32_t)(mask >> (64 - o)) : 0u;
      if (lo) atomicOr(&sh->bits[w], lo);
      if (mid) atomicOr(&sh->bits[w + 1], mid);
      if (hi) atomicOr(&sh->bits[w + 2], hi);
    }
    for (int k = 0; k < 2; ++k) {
      const int32_t p = k ? far_l : far_s;
      if (p == kNone) continue;
      if (p == kOld)
        sh->old[k] = k ? old_l : old_s;
      else
        atomicOr(&sh->bits[(p + kEvBlock) >> 5], 1u << ((p + kEvBlock) & 31));
    }
    __syncthreads();
    word = sh->bits[lane];
    for (int k = 0; k < 2; ++k) {
      if (sh->old[k] >= 0) {
        if (lane == 0) {
          int32_t m = n;
          sh->lost = insert_bound(list, m, cap, sh->old[k]) ? 1 : 0;
          sh->n = m;
        }
        __syncthreads();
        n = sh->n;
        lost = lost || sh->lost;
        __syncthreads();
      }
    }
  }

  // Moves the boundaries of the lanes below `lanes` to the list.
  __device__ __forceinline__ void commit(int lanes) {
    const int lane = (int)threadIdx.x;
    uint32_t w = lane < lanes ? word : 0u;
    int32_t upto = __popc(w);
    const int32_t own = upto;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t v = __shfl_up(upto, off);
      if (lane >= off) upto += v;
    }
    int32_t at = n + upto - own;
    const int64_t base = b0 - kEvBlock + 32 * lane;
    while (w) {
      const int k = __ffs(w) - 1;
      if (at < cap) list[at] = base + k;
      ++at;
      w &= w - 1;
    }
    const int32_t all = n + __shfl(upto, 63);
    lost = lost || all > cap;
    n = all < cap ? all : cap;
    __syncthreads();
  }

  // The next block follows: this block's half of the bitmap moves up.
  __device__ __forceinline__ void advance() {
    const int lane = (int)threadIdx.x;
    commit(32);
    const uint32_t up = (uint32_t)__shfl((int)word, (lane + 32) & 63);
    word = lane < 32 ? up : 0u;
    auto back = [&](int32_t& p, int64_t& old) {
      if (p == kNone || p == kOld) return;
      if (p - kEvBlock < -kEvBlock) {
        old = b0 + p;
        p = kOld;
      } else {
        p -= kEvBlock;
      }
    };
    back(d.sp, old_s);
    back(d.lp, old_l);
    d.lm = d.lm < kEvBlock ? kNone : d.lm - kEvBlock;
    b0 += kEvBlock;
  }

  // Below this position no boundary can still appear (scanned: the positions
  // scanned so far).
  __device__ __forceinline__ int64_t cut(int64_t scanned) const {
    int64_t c = scanned;
    if (d.sp != kNone) c = min(c, d.sp == kOld ? old_s : b0 + d.sp);
    if (d.lp != kNone) c = min(c, d.lp == kOld ? old_l : b0 + d.lp);
    return c;
  }
  // Boundaries of the list below c, by all lanes.
  __device__ __forceinline__ int32_t below(int64_t c) const {
    int32_t k = 0;
    for (int32_t i = (int32_t)threadIdx.x; i < n; i += 64) k += list[i] < c ? 1 : 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) k += __shfl_xor(k, off);
    return k;
  }
  // Whether the first `want` boundaries are final, below c (not asked while a
  // candidate older than the window is open).
  __device__ __forceinline__ bool enough(int64_t c, int32_t want) const {
    if (d.sp == kOld || d.lp == kOld) return false;
    const int64_t rel = c - (b0 - kEvBlock + 32 * (int64_t)threadIdx.x);  // in this lane's word
    const uint32_t w = rel >= 32 ? word : (rel <= 0 ? 0u : word & ((1u << rel) - 1u));
    int32_t k = __popc(w);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) k += __shfl_xor(k, off);
    return n + k >= want;
  }
};

// The value of an event, samples [lo, up): their float64 mean in index order.
__device__ __forceinline__ float event_value(const float* __restrict__ x, int64_t lo, int64_t up) {
  double sum = 0.0;
  int64_t q = lo;
  for (; q + 4 <= up; q += 4) {
    const float a = x[q], b = x[q + 1], c = x[q + 2], e = x[q + 3];
    sum += (double)a;
    sum += (double)b;
    sum += (double)c;
    sum += (double)e;
  }
  for (; q < up; ++q) sum += (double)x[q];
  return (float)(sum / (double)(up - lo));
}

// One wave per read.  Read r is raw[offs[stride r] .. offs[stride r + 1])
// (stride 1: CSR offsets; stride 2: start/end pairs).  Its events trim_r ..
// trim_r + keep - 1 are wanted, trim_r = trims[r] (or `trim` without trims;
// trim_r <= trim).  With `prefix` the samples are only the beginning of a
// longer read: the scan stops where the t statistics still depend on samples
// not yet received (position L - 5), and only events whose end boundary is
// final are written.
__global__ __launch_bounds__(64) void k_detect_events(const float* __restrict__ raw,
                                                      const int64_t* __restrict__ offs,
                                                      int32_t stride,
                                                      const int32_t* __restrict__ trims,
                                                      int32_t trim, int32_t keep, int32_t prefix,
                                                      float* __restrict__ out,
                                                      int32_t* __restrict__ counts) {
  issue_first();
  __shared__ Scan::Shared sh;
  extern __shared__ int64_t ev_list[];  // [trim + keep]
  const int lane = (int)threadIdx.x;
  const int32_t r = (int32_t)blockIdx.x;
  const int64_t a = offs[(int64_t)stride * r];
  const int64_t L = offs[(int64_t)stride * r + 1] - a;
  // a first event outside [0, trim] marks the read as bad (count -1)
  const int32_t tr0 = trims ? trims[r] : trim;
  const bool bad = tr0 < 0 || tr0 > trim;
  const int32_t tr = bad ? 0 : tr0, cap = tr + keep;
  // positions whose t statistics are final (all of them for a whole read)
  const int64_t scanL = prefix ? (L > kWLong - 1 ? L - (kWLong - 1) : 0) : L;
  Scan s{&sh, raw + a, L, blank_detectors(), -1, -1, ev_list, 0, cap, false, 0, 0u};
  int32_t closed = 0;  // events whose end is known (no samples, no event)
  if (scanL > 0 && !bad) {
    while (true) {
      const int32_t nblk = (int32_t)min(scanL - s.b0, (int64_t)kEvBlock);
      s.block(nblk);
      const int64_t scanned = s.b0 + nblk, c = s.cut(scanned);
      if (s.enough(c, cap)) {
        s.commit(64);
        closed = cap;  // stopped early: events 0 .. cap-1 are closed
        break;
      }
      if (scanned >= scanL) {
        s.commit(64);
        closed = prefix ? s.below(c) : s.n + 1;  // (the last event of a whole read ends at L)
        break;
      }
      s.advance();
    }
  }
  // events: cut_0 = 0, cut_j = list[j-1], and L after the last
  const int32_t hi = closed < cap ? closed : cap;
  const int32_t n_out = hi > tr ? hi - tr : 0;
  for (int32_t e = lane; e < keep; e += 64) {
    float v = 0.0f;
    if (e < n_out) {
      const int32_t j = tr + e;
      v = event_value(s.x, j == 0 ? 0 : ev_list[j - 1], j < s.n ? ev_list[j] : L);
    }
    out[(int64_t)r * keep + e] = v;
  }
  if (lane == 0) counts[r] = bad ? -1 : n_out;
}

// ---- reads received chunk by chunk: the detectors' state kept between calls

constexpr int kPending = 32;  // emitted boundaries not yet delivered, per read

struct EventState {
  int64_t pos;           // next position to scan (from the read's first sample)
  int64_t last;          // start of the next undelivered event
  int64_t s_masked, s_peak, l_masked, l_peak;
  double s_val, l_val;
  int32_t s_valid, l_valid;
  int32_t index;         // index of the next undelivered event in the read
  int32_t npend;
  int64_t pend[kPending];
};

__global__ void k_event_state_init(EventState* __restrict__ states,
                                   const int32_t* __restrict__ slots, int32_t n) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= n) return;
  EventState& e = states[slots[i]];
  e.pos = 0;
  e.last = 0;
  e.s_masked = e.l_masked = -1;
  e.s_peak = e.l_peak = -1;
  e.s_val = e.l_val = INFINITY;
  e.s_valid = e.l_valid = 0;
  e.index = 0;
  e.npend = 0;
}

// One wave per read.  Read r's samples so far are raw[ranges[2r] ..
// ranges[2r+1]) (the start fixed across calls); its state is
// states[slots[r]].  Positions pos .. L-6 are scanned (those whose t
// statistics are final) and emitted boundaries join the pending list (in
// LDS, room for keep + 32); then the final ones (below every open
// candidate) are delivered in order as events last .. boundary, events
// below `trim` consumed without being written, at most keep written; at most
// 32 undelivered boundaries may carry over to the next call.
__global__ __launch_bounds__(64) void k_events_continue(
    const float* __restrict__ raw, const int64_t* __restrict__ ranges,
    const int32_t* __restrict__ slots, EventState* __restrict__ states, int32_t trim,
    int32_t keep, float* __restrict__ out, int32_t* __restrict__ counts) {
  issue_first();
  __shared__ Scan::Shared sh;
  extern __shared__ int64_t pend[];  // [keep + kPending]
  const int32_t r = (int32_t)blockIdx.x;
  const int lane = (int)threadIdx.x;
  const int64_t a = ranges[2 * (int64_t)r];
  const int64_t L = ranges[2 * (int64_t)r + 1] - a;
  EventState* __restrict__ st = states + slots[r];
  const int64_t scanL = L > kWLong - 1 ? L - (kWLong - 1) : 0;
  const int64_t pos0 = st->pos;
  Scan s{&sh, raw + a, L, blank_detectors(), -1, -1, pend, 0, keep + kPending, false, pos0, 0u};
  // the state, positions relative to the first block
  auto place = [&](int64_t p, int64_t& old) -> int32_t {
    if (p < 0) return kNone;
    if (p - pos0 < -kEvBlock) {
      old = p;
      return kOld;
    }
    return (int32_t)(p - pos0);
  };
  s.d.sp = place(st->s_peak, s.old_s);
  s.d.lp = place(st->l_peak, s.old_l);
  s.d.lm = st->l_masked < pos0 ? kNone : (int32_t)(st->l_masked - pos0);
  s.d.sv = st->s_val;
  s.d.lv = st->l_val;
  s.d.sok = st->s_valid != 0;
  s.d.lok = st->l_valid != 0;
  // pending boundaries: the recent ones into the bitmap
  const int32_t np = st->npend;
  const int64_t mine = lane < np ? st->pend[lane] : LLONG_MAX;
  const uint64_t before = __ballot(mine < pos0 - kEvBlock);
  s.n = __popcll(before);
  sh.bits[lane] = 0u;
  __syncthreads();
  if (lane < s.n)
    pend[lane] = mine;
  else if (lane < np)
    atomicOr(&sh.bits[(mine - pos0 + kEvBlock) >> 5], 1u << ((mine - pos0 + kEvBlock) & 31));
  __syncthreads();
  s.word = sh.bits[lane];
  __syncthreads();
  int64_t scanned = pos0;
  while (scanned < scanL) {
    if (scanned > pos0) s.advance();
    const int32_t nblk = (int32_t)min(scanL - s.b0, (int64_t)kEvBlock);
    s.block(nblk);
    scanned = s.b0 + nblk;
  }
  s.commit(64);
  const int32_t final = s.below(s.cut(scanned));
  const int32_t index = st->index, skipped = trim > index ? trim - index : 0;
  const int32_t skip = skipped < final ? skipped : final;
  const int32_t nout = final - skip < keep ? final - skip : keep;
  const int32_t used = skip + nout;
  const int64_t start = skip > 0 ? pend[skip - 1] : st->last;
  const bool over = s.lost || s.n - used > kPending;
  // the delivered events: start .. pend[skip], pend[skip] .. pend[skip+1], ...
  for (int32_t e = lane; e < keep; e += 64) {
    out[(int64_t)r * keep + e] =
        e < nout ? event_value(s.x, e == 0 ? start : pend[skip + e - 1], pend[skip + e]) : 0.0f;
  }
  __syncthreads();
  const int32_t left = s.n - used < kPending ? s.n - used : kPending;
  if (lane < left) st->pend[lane] = pend[used + lane];
  if (lane == 0) {
    auto at = [&](int32_t p, int64_t old) -> int64_t {
      return p == kNone ? -1 : (p == kOld ? old : s.b0 + p);
    };
    st->pos = scanned;
    st->last = used > 0 ? pend[used - 1] : st->last;
    st->index = index + used;
    st->s_masked = -1;
    st->s_peak = at(s.d.sp, s.old_s);
    st->s_val = s.d.sv;
    st->s_valid = s.d.sok;
    st->l_masked = s.d.lm == kNone ? -1 : s.b0 + s.d.lm;
    st->l_peak = at(s.d.lp, s.old_l);
    st->l_val = s.d.lv;
    st->l_valid = s.d.lok;
    st->npend = left;
    counts[r] = over ? -1 : nout;
  }
}

}  // namespace

size_t event_state_bytes() { return sizeof(EventState); }

hipError_t launch_event_state_init(void* states, const int32_t* slots, int32_t n,
                                   hipStream_t st) {
  hipLaunchKernelGGL(k_event_state_init, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     (EventState*)states, slots, n);
  return hipGetLastError();
}

hipError_t launch_events_continue(const float* raw, const int64_t* ranges, const int32_t* slots,
                                  void* states, int32_t nreads, int32_t trim, int32_t keep,
                                  float* out, int32_t* counts, hipStream_t st) {
  const size_t lds = sizeof(int64_t) * (size_t)(keep + kPending);
  hipLaunchKernelGGL(k_events_continue, dim3((unsigned)nreads), dim3(64), lds, st, raw, ranges,
                     slots, (EventState*)states, trim, keep, out, counts);
  return hipGetLastError();
}

hipError_t launch_detect_events(const float* raw, const int64_t* offs, int32_t stride,
                                const int32_t* trims, int32_t nreads, int32_t trim,
                                int32_t keep, int32_t prefix, float* out, int32_t* counts,
                                hipStream_t st) {
  const size_t lds = sizeof(int64_t) * (size_t)(trim + keep);
  const hipError_t e = hipFuncSetAttribute(
      (const void*)k_detect_events, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_detect_events, dim3((unsigned)nreads), dim3(64), lds, st, raw, offs, stride,
                     trims, trim, keep, prefix, out, counts);
  return hipGetLastError();
}

}  // namespace sdtw
