// Reference and query preparation (section 4.1; section 2.2 k-mer model).
//
// Reference: k-mer model lookup of both strands (one thread per output
// sample), then a joint z-score over the concatenation whose mean and
// population sd equal, bit for bit, those of a plain loop that accumulates in
// double in index order (see "Sums in index order" below), then fixed-point
// codes.
//
// Queries: one wave per read; lane 0 walks the read's events in index order
// for the mean and for the sum of squared deviations, so each read's
// statistics come from exactly the same sequence of IEEE double operations as
// a plain sequential loop (no contraction: the library is built with
// -ffp-contract=off).
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "device.h"

namespace sdtw {
namespace {

constexpr int kPrepThreads = 256;

__device__ __forceinline__ int16_t to_code(float z, double scale, unsigned long long* nsat_local) {
  double r = rint((double)z * scale);  // round half to even
  if (r > 32767.0) { r = 32767.0; ++*nsat_local; }
  if (r < -32768.0) { r = -32768.0; ++*nsat_local; }
  return (int16_t)r;
}

// Expected current of k-mer p of the forward strand (p < nk) or of k-mer
// p - nk of the reverse-complement strand read 5'->3'.
__global__ void k_kmer(const uint8_t* __restrict__ g, int64_t L, int k,
                       const float* __restrict__ table, float* __restrict__ sig) {
  const int64_t nk = L - k + 1;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= 2 * nk) return;
  uint32_t idx = 0;
  if (p < nk) {
    for (int m = 0; m < k; ++m) idx = idx * 4u + (g[p + m] & 3u);
  } else {
    const int64_t q = p - nk;  // position in revcomp(g)
    for (int m = 0; m < k; ++m) idx = idx * 4u + (3u - (g[L - 1 - (q + m)] & 3u));
  }
  sig[p] = table[idx];
}

// x and z may be the same array (normalised in place): each thread reads its
// element before writing it, so neither pointer is declared restrict.
__global__ void k_normalize(const float* x, int64_t n, const double* __restrict__ stats,
                            double scale, float* z, int16_t* __restrict__ codes,
                            int64_t* __restrict__ nsat) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long sat = 0;
  if (i < n) {
    const double mean = stats[0], sd = stats[1];
    const float zi = sd > 0.0 ? (float)(((double)x[i] - mean) / sd) : 0.0f;
    z[i] = zi;
    if (codes) codes[i] = to_code(zi, scale, &sat);
  }
  if (nsat && sat) atomicAdd((unsigned long long*)nsat, sat);
}

__global__ void k_zero_i64(int64_t* p) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0;
}

// One wave per read.  Events are staged through LDS in coalesced chunks and
// lane 0 accumulates the sum and then the sum of squared deviations in index
// order, so the statistics come from the same sequence of double operations
// as a plain sequential loop; all lanes then normalise and quantise.  The
// next chunk's loads are issued before lane 0 sums the current one (two LDS
// buffers), so memory latency hides behind the sequential sum.
constexpr int kQChunk = 512;
constexpr int kQPer = kQChunk / 64;

__device__ __forceinline__ double wave_seq_sum(const float* __restrict__ raw, int64_t a, int64_t b,
                                               double mean, bool squares, float* buf) {
  const int lane = (int)threadIdx.x;
  double acc = 0.0;
  float pre[kQPer];
  auto fetch = [&](int64_t base) {
#pragma unroll
    for (int j = 0; j < kQPer; ++j) {
      const int64_t i = base + lane + 64 * j;
      pre[j] = i < b ? raw[i] : 0.0f;
    }
  };
  fetch(a);
  int cur = 0;
  for (int64_t base = a; base < b; base += kQChunk) {
    const int n = (int)min<int64_t>(kQChunk, b - base);
    float* const cb = buf + cur * kQChunk;
#pragma unroll
    for (int j = 0; j < kQPer; ++j) cb[lane + 64 * j] = pre[j];
    // one barrier per chunk: the other buffer, written next, was last read
    // by lane 0 before it reached this barrier
    __syncthreads();
    if (base + kQChunk < b) fetch(base + kQChunk);
    if (lane == 0) {
      for (int k = 0; k < n; ++k) {
        const double v = (double)cb[k];
        if (squares) {
          const double d = v - mean;
          acc += d * d;
        } else {
          acc += v;
        }
      }
    }
    cur ^= 1;
  }
  __syncthreads();  // lane 0 is done with both buffers before they are reused
  return __shfl(acc, 0);
}

// ---------------------------------------------------------------------------
// Sums in index order, in parallel
//
// The sum of a plain loop, s_k = fl(s_{k-1} + t_k), rounds at every step, so
// another order of additions gives another last bit.  But while the running
// sum stays within one binade [2^e, 2^(e+1)) it is S u for an integer S and
// u = 2^(e-52), and a step adds an integer: with q = t / u (a scaling by a
// power of two, exact),
//     S' = S + floor(q) + (1 if the fraction of q exceeds 1/2, or equals it
//          and S + floor(q) is odd: round half to even).
// So a step maps S to S + d[S mod 2] for two integers, such maps compose to
// maps of the same kind, and a run of terms is one map, found in any order of
// composition.  The wave that applies the maps checks, with the exact S it
// has, that S starts and ends in the binade (terms are >= 0, so every sum in
// between is in it too); where that fails (a binade is crossed, about once per
// doubling of the sum) it looks at shorter runs and, at the crossing itself,
// at 16 terms one by one.  The exponent a tile's map is made for is only a
// guess, from sums in another order.  Runs with a negative or non-finite term
// are added up term by term, as the plain loop does it.
//
// A sum of values that are all multiples of 2^q and together below 2^(53 + q)
// needs no rounding at all, so any order gives it: the first sum, of currents
// with 24-bit significands, ends there (8.6e8 pA in steps of 2^-18).
//
// Measured on MI355X, the whole preparation of 9,999,990 values: 233 ms with one
// lane adding them up, whose additions follow each other at about 30 cycles;
// 0.45 ms so, 0.2 of them the walk over the second sum's binade crossings (a
// chain of one wave's look-ups, about 10 us a crossing), the rest passes over
// memory.  59,796 values: 1.4 -> 0.15 ms.
// ---------------------------------------------------------------------------

constexpr int kSumTile = 1024;           // terms per map
constexpr int kSumPer = kSumTile / 64;   // per lane of the wave that makes it
constexpr int32_t kNoBinade = INT32_MIN;  // no map

struct SumMap {
  int64_t d[2];  // S -> S + d[S mod 2]
};
__device__ __forceinline__ SumMap then(const SumMap& f, const SumMap& g) {  // f, then g
  SumMap h;
  h.d[0] = f.d[0] + ((f.d[0] & 1) ? g.d[1] : g.d[0]);
  h.d[1] = f.d[1] + (((f.d[1] + 1) & 1) ? g.d[1] : g.d[0]);
  return h;
}
__device__ __forceinline__ int64_t shfl_up64(int64_t v, int off) {
  const int lo = __shfl_up((int)(uint32_t)v, off), hi = __shfl_up((int)(v >> 32), off);
  return (int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}
__device__ __forceinline__ int64_t shfl64(int64_t v, int lane) {
  const int lo = __shfl((int)(uint32_t)v, lane), hi = __shfl((int)(v >> 32), lane);
  return (int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}
// Inclusive composition over the wave's lanes, lane 0's map first.
__device__ __forceinline__ SumMap scan_sum_maps(SumMap m) {
  const int lane = (int)threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    SumMap o;
    o.d[0] = shfl_up64(m.d[0], off);
    o.d[1] = shfl_up64(m.d[1], off);
    if (lane >= off) m = then(o, m);
  }
  return m;
}

// A sum's binade, or kNoBinade (zero, negative, subnormal, non-finite, or so
// far out that a scaling by 2^(52 - e) would not be exact).
__device__ __forceinline__ int32_t binade(double s) {
  const int64_t bits = __double_as_longlong(s);
  const int32_t e = (int32_t)(bits >> 52) - 1023;
  return e >= -900 && e <= 900 ? e : kNoBinade;
}
__device__ __forceinline__ int64_t significand(double s) {
  return (__double_as_longlong(s) & ((int64_t(1) << 52) - 1)) | int64_t(1) << 52;
}
__device__ __forceinline__ double power_of_two(int32_t e) {
  return __longlong_as_double((int64_t)(e + 1023) << 52);
}

template <bool SQUARES>
__device__ __forceinline__ double term(float x, double mean) {
  const double v = (double)x;
  if constexpr (SQUARES) {
    const double d = v - mean;
    return d * d;
  } else {
    return v;
  }
}

// Appends term t to the map m of binade e (scale = 2^(52 - e)); false if
// there is no such map.
__device__ __forceinline__ bool append(SumMap& m, double t, double scale) {
  const double q = t * scale;
  if (!(q >= 0.0 && q < 9007199254740992.0)) return false;  // negative, NaN, or past the binade
  const double fl = floor(q), fr = q - fl;
  const int64_t f = (int64_t)fl;
  SumMap g;
  g.d[0] = f + (fr > 0.5 || (fr == 0.5 && (f & 1)) ? 1 : 0);
  g.d[1] = f + (fr > 0.5 || (fr == 0.5 && !(f & 1)) ? 1 : 0);
  m = then(m, g);
  return true;
}

// How many of the lanes' runs the sum s can take in one go: the leading lanes
// with a map (`ok`), up to the last that ends in s's binade.  s becomes the
// sum behind them.
__device__ __forceinline__ int take_runs(double& s, int32_t e, bool ok, SumMap m) {
  const SumMap all = scan_sum_maps(m);
  const int64_t S = significand(s);
  const int64_t end = S + ((S & 1) ? all.d[1] : all.d[0]);
  const uint64_t bad = __ballot(!ok || end >= (int64_t(1) << 53) || end < S);
  const int runs = bad ? __builtin_ctzll(bad) : 64;
  if (runs > 0) s = (double)shfl64(end, runs - 1) * power_of_two(e - 52);
  return runs;
}

// buf[0 .. n) added to s one by one: the chain of additions, with the next 16
// values on their way from LDS.
__device__ __forceinline__ double add_all(const float4& v, double s) {
  s += (double)v.x;
  s += (double)v.y;
  s += (double)v.z;
  return s + (double)v.w;
}
__device__ __forceinline__ double add_all(const double2& v, double s) {
  s += v.x;
  return s + v.y;
}
template <class T>
__device__ __forceinline__ double add_plain(const T* buf, int n, double s) {
  using V = std::conditional_t<sizeof(T) == 4, float4, double2>;
  constexpr int kVecs = (int)(16 * sizeof(T) / sizeof(V));
  V next[kVecs];
  auto fetch = [&](int at) {
    const V* const from = (const V*)(buf + (at < kSumTile - 16 ? at : kSumTile - 16));
#pragma unroll
    for (int k = 0; k < kVecs; ++k) next[k] = from[k];
  };
  fetch(0);
  int at = 0;
  for (; at + 16 <= n; at += 16) {
    V now[kVecs];
#pragma unroll
    for (int k = 0; k < kVecs; ++k) now[k] = next[k];
    fetch(at + 16);
#pragma unroll
    for (int k = 0; k < kVecs; ++k) s = add_all(now[k], s);
  }
  for (; at < n; ++at) s += (double)buf[at];
  return s;
}

// One wave adds terms [a, b) (at most kSumTile) to s, staged in buf.  A tile with
// no maps for more than a few of its runs (kPlainRuns: a try at the maps costs as
// much as about 300 additions) is added up term by term: on a table of signed
// levels 9,999,990 values took 470 ms when every run of 16 was tried first, the
// plain loop of one lane 229.
constexpr int kPlainRuns = 3;
template <bool SQUARES>
__device__ __forceinline__ double add_tile(const float* __restrict__ x, int64_t a, int64_t b,
                                           double mean, double s, float* buf) {
  const int lane = (int)threadIdx.x & 63;
  const int n = (int)(b - a);
  __syncthreads();
  for (int i = lane; i < n; i += 64) buf[i] = x[a + i];
  __syncthreads();
  if constexpr (!SQUARES) {
    bool mapped = true;
#pragma unroll
    for (int k = 0; k < kSumPer; ++k) {
      const int i = lane * kSumPer + k;
      mapped = mapped && (i >= n || buf[i] >= 0.0f);
    }
    if (__popcll(__ballot(!mapped)) > kPlainRuns) return add_plain(buf, n, s);
  }
  for (int at = 0; at < n;) {
    const int32_t e = binade(s);
    if (e != kNoBinade) {
      const double scale = power_of_two(52 - e);
      SumMap m{{0, 0}};
      bool ok = true;
      const int first = at + lane * kSumPer;
#pragma unroll
      for (int k = 0; k < kSumPer; ++k)
        if (first + k < n) ok = ok && append(m, term<SQUARES>(buf[first + k], mean), scale);
      at += take_runs(s, e, ok, m) * kSumPer;
      if (at >= n) break;
    }
    const int to = at + kSumPer < n ? at + kSumPer : n;
    for (; at < to; ++at) s += term<SQUARES>(buf[at], mean);
  }
  return s;
}

// The largest q such that x is a multiple of 2^q (INT_MAX for 0); INT_MIN for
// a negative or non-finite x.
__device__ __forceinline__ int32_t lowest_bit(float x) {
  const uint32_t bits = __float_as_uint(x), exp = bits >> 23, frac = bits & 0x7FFFFFu;
  if (bits == 0u) return INT_MAX;
  if (exp >= 255u) return INT_MIN;  // (with the sign bit: also every negative value)
  return exp ? (int32_t)exp - 150 + __builtin_ctz(frac | 0x800000u) : -149 + __builtin_ctz(frac);
}

// Tile sums in any order, for the guess, and without SQUARES the smallest
// lowest_bit: one wave per tile.
template <bool SQUARES>
__global__ __launch_bounds__(256) void k_sum_guess(const float* __restrict__ x, int64_t n,
                                                   const double* __restrict__ stats,
                                                   double* __restrict__ sums,
                                                   int32_t* __restrict__ low, int32_t ntiles) {
  const int lane = (int)threadIdx.x & 63;
  const int32_t tile = (int32_t)blockIdx.x * 4 + ((int32_t)threadIdx.x >> 6);
  if (tile >= ntiles) return;
  const double mean = SQUARES ? stats[0] : 0.0;
  double s = 0.0;
  int32_t q = INT_MAX;
#pragma unroll
  for (int k = 0; k < kSumPer; ++k) {
    const int64_t i = (int64_t)tile * kSumTile + lane + 64 * k;
    if (i < n) {
      const float v = x[i];
      s += term<SQUARES>(v, mean);
      if constexpr (!SQUARES) q = min(q, lowest_bit(v));
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    s += __shfl_xor(s, off);
    if constexpr (!SQUARES) q = min(q, __shfl_xor(q, off));
  }
  if (lane == 0) {
    sums[tile] = s;
    if constexpr (!SQUARES) low[tile] = q;
  }
}

// The binade that each tile's sums lie in by the guess, or none: one workgroup.
// Without SQUARES: if no sum rounds, stats[0] becomes the mean and *exact 1,
// else 0.
template <bool SQUARES>
__global__ __launch_bounds__(1024) void k_sum_binades(const double* __restrict__ sums,
                                                      const int32_t* __restrict__ low, int64_t n,
                                                      int32_t ntiles, int32_t* __restrict__ e,
                                                      double* __restrict__ stats,
                                                      int32_t* __restrict__ exact) {
  __shared__ double part[1024];
  __shared__ int32_t bits[1024];
  const int t = (int)threadIdx.x;
  const int32_t per = (ntiles + 1023) / 1024;
  const int32_t a = t * per < ntiles ? t * per : ntiles;
  const int32_t b = a + per < ntiles ? a + per : ntiles;
  double s = 0.0;
  int32_t q = INT_MAX;
  for (int32_t i = a; i < b; ++i) {
    s += sums[i];
    if constexpr (!SQUARES) q = min(q, low[i]);
  }
  part[t] = s;
  bits[t] = q;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const double v = t >= off ? part[t - off] : 0.0;
    const int32_t w = t >= off ? bits[t - off] : INT_MAX;
    __syncthreads();
    part[t] += v;
    bits[t] = min(bits[t], w);
    __syncthreads();
  }
  if constexpr (!SQUARES) {
    if (t == 1023) {
      // (a sum of non-negative values: no partial sum is larger; 0 of zeros)
      const bool is = bits[t] > INT_MIN &&
                      (bits[t] == INT_MAX || part[t] < ldexp(1.0, 52 + bits[t]));
      *exact = is ? 1 : 0;
      if (is) stats[0] = part[t] / (double)n;
    }
  }
  s = t > 0 ? part[t - 1] : 0.0;
  for (int32_t i = a; i < b; ++i) {
    const double next = s + sums[i];
    const int32_t lo = binade(s), hi = binade(next);
    e[i] = lo == hi ? lo : kNoBinade;
    s = next;
  }
}

// The tiles' maps for those binades: one wave per tile.  Clears e[tile] where
// there is none.
template <bool SQUARES>
__global__ __launch_bounds__(256) void k_sum_maps(const float* __restrict__ x, int64_t n,
                                                  const double* __restrict__ stats,
                                                  int32_t* __restrict__ e,
                                                  int64_t* __restrict__ maps, int32_t ntiles,
                                                  const int32_t* __restrict__ exact) {
  if (!SQUARES && *exact) return;
  __shared__ float stage[4][kSumTile];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int32_t tile = (int32_t)blockIdx.x * 4 + wave;
  const int64_t base = (int64_t)tile * kSumTile;
  float* const buf = stage[wave];
  if (tile < ntiles) {
    for (int i = lane; i < kSumTile; i += 64) buf[i] = base + i < n ? x[base + i] : 0.0f;
  }
  __syncthreads();
  if (tile >= ntiles) return;
  const int32_t et = e[tile];
  if (et == kNoBinade) return;
  const double mean = SQUARES ? stats[0] : 0.0, scale = power_of_two(52 - et);
  SumMap m{{0, 0}};
  bool ok = true;
#pragma unroll
  for (int k = 0; k < kSumPer; ++k) {
    const int i = lane * kSumPer + k;
    if (base + i < n) ok = ok && append(m, term<SQUARES>(buf[i], mean), scale);
  }
  m = scan_sum_maps(m);
  const bool all = __ballot(!ok) == 0ull;
  if (lane == 63) {
    if (all) {
      maps[2 * (int64_t)tile] = m.d[0];
      maps[2 * (int64_t)tile + 1] = m.d[1];
    } else {
      e[tile] = kNoBinade;
    }
  }
}

// The maps of kSuper tiles together, where they have one: one wave each.
constexpr int kSuper = 64;
__global__ __launch_bounds__(64) void k_sum_supers(const int32_t* __restrict__ e,
                                                   const int64_t* __restrict__ maps,
                                                   int32_t ntiles, int32_t* __restrict__ super_e,
                                                   int64_t* __restrict__ super_maps) {
  const int lane = (int)threadIdx.x;
  const int32_t super = (int32_t)blockIdx.x, mine = super * kSuper + lane;
  const bool in = mine < ntiles;
  const int32_t et = in ? e[mine] : kNoBinade;
  const int32_t e0 = __shfl(et, 0);
  SumMap m{{0, 0}};
  if (in && et != kNoBinade) {
    m.d[0] = maps[2 * (int64_t)mine];
    m.d[1] = maps[2 * (int64_t)mine + 1];
  }
  m = scan_sum_maps(m);
  const bool all = __ballot(in && et != e0) == 0ull;
  if (lane == 63) {
    super_e[super] = all ? e0 : kNoBinade;
    super_maps[2 * (int64_t)super] = m.d[0];
    super_maps[2 * (int64_t)super + 1] = m.d[1];
  }
}

// The leading ones of the up to 64 maps from `at` that s can take in one go;
// s becomes the sum behind them.  (The first sum of signed values has no maps:
// asked first there.)
template <bool SQUARES>
__device__ __forceinline__ int take_maps(double& s, int32_t es, const int32_t* __restrict__ e,
                                         const int64_t* __restrict__ maps, int32_t at,
                                         int32_t n) {
  const int32_t mine = at + ((int32_t)threadIdx.x & 63);
  const bool ok = mine < n && e[mine] == es;
  if (!SQUARES && !__builtin_amdgcn_readfirstlane(ok ? 1 : 0)) return 0;
  SumMap m{{0, 0}};
  if (ok) {
    m.d[0] = maps[2 * (int64_t)mine];
    m.d[1] = maps[2 * (int64_t)mine + 1];
  }
  return take_runs(s, es, ok, m);
}

// The sum, by one wave: 64 maps of kSuper tiles at a time, or of tiles, or a
// tile's terms.  Without SQUARES stats[0] becomes the mean, with it stats[1] the
// population sd (and nsat, if given, 0).
template <bool SQUARES>
__global__ __launch_bounds__(64) void k_sum_walk(const float* __restrict__ x, int64_t n,
                                                 const int32_t* __restrict__ e,
                                                 const int64_t* __restrict__ maps,
                                                 const int32_t* __restrict__ super_e,
                                                 const int64_t* __restrict__ super_maps,
                                                 int32_t ntiles, double* __restrict__ stats,
                                                 int64_t* __restrict__ nsat,
                                                 const int32_t* __restrict__ exact) {
  if (!SQUARES && *exact) return;
  __shared__ __align__(16) float buf[kSumTile];
  const double mean = SQUARES ? stats[0] : 0.0;
  const int32_t nsupers = (ntiles + kSuper - 1) / kSuper;
  double s = 0.0;
  for (int32_t tile = 0; tile < ntiles;) {
    const int32_t es = binade(s);
    if (es != kNoBinade) {
      if (tile % kSuper == 0) {
        const int runs = take_maps<SQUARES>(s, es, super_e, super_maps, tile / kSuper, nsupers);
        tile += runs * kSuper;
        if (runs == 64 || tile >= ntiles) continue;
      }
      const int32_t end = (tile / kSuper + 1) * kSuper;  // of this super
      const int runs = take_maps<SQUARES>(s, es, e, maps, tile, end < ntiles ? end : ntiles);
      tile += runs;
      if (tile >= ntiles || tile == end) continue;
    }
    const int64_t a = (int64_t)tile * kSumTile;
    s = add_tile<SQUARES>(x, a, a + kSumTile < n ? a + kSumTile : n, mean, s, buf);
    ++tile;
  }
  if (threadIdx.x == 0) {
    if constexpr (SQUARES) {
      stats[1] = sqrt(s / (double)n);
      if (nsat) *nsat = 0;
    } else {
      stats[0] = s / (double)n;
    }
  }
}

// Both sums by one wave, term by term: a few thousand values do not pay for the
// ten launches of the parallel sums, and so close to zero the sums cross a
// binade every few runs (preparing 2,000 bases: 77 us term by term, 98 in
// parallel; 1,000: 44 and 84; 500: 33 to 42 and 76).
constexpr int64_t kSmallSum = 5 * kSumTile;
__global__ __launch_bounds__(64) void k_sum_small(const float* __restrict__ x, int32_t n,
                                                  double* __restrict__ stats,
                                                  int64_t* __restrict__ nsat) {
  __shared__ __align__(16) double buf[kSumTile];
  auto sum = [&](auto&& term_of) {
    double s = 0.0;
    for (int32_t a = 0; a < n; a += kSumTile) {
      const int32_t len = a + kSumTile < n ? kSumTile : n - a;
      __syncthreads();
      for (int32_t i = (int32_t)threadIdx.x; i < len; i += 64) buf[i] = term_of(x[a + i]);
      __syncthreads();
      s = add_plain(buf, len, s);
    }
    return s;
  };
  const double mean = sum([](float v) { return term<false>(v, 0.0); }) / (double)n;
  const double squares = sum([&](float v) { return term<true>(v, mean); });
  if (threadIdx.x == 0) {
    stats[0] = mean;
    stats[1] = sqrt(squares / (double)n);
    if (nsat) *nsat = 0;
  }
}

template <bool SQUARES>
void launch_sum(const float* x, int64_t n, double* scratch, int64_t* nsat, hipStream_t st) {
  const int32_t ntiles = (int32_t)((n + kSumTile - 1) / kSumTile);
  double* const stats = scratch;
  double* const sums = scratch + 2;
  int64_t* const maps = (int64_t*)(sums + ntiles);
  const int32_t nsupers = (ntiles + kSuper - 1) / kSuper;
  int64_t* const super_maps = maps + 2 * (int64_t)ntiles;
  int32_t* const e = (int32_t*)(super_maps + 2 * (int64_t)nsupers);
  int32_t* const super_e = e + ntiles;
  int32_t* const low = super_e + nsupers;
  int32_t* const exact = low + ntiles;
  const dim3 grid((unsigned)((ntiles + 3) / 4));
  hipLaunchKernelGGL(k_sum_guess<SQUARES>, grid, dim3(256), 0, st, x, n, stats, sums, low, ntiles);
  hipLaunchKernelGGL(k_sum_binades<SQUARES>, dim3(1), dim3(1024), 0, st, sums, low, n, ntiles, e,
                     stats, exact);
  hipLaunchKernelGGL(k_sum_maps<SQUARES>, grid, dim3(256), 0, st, x, n, stats, e, maps, ntiles,
                     exact);
  hipLaunchKernelGGL(k_sum_supers, dim3((unsigned)nsupers), dim3(64), 0, st, e, maps, ntiles,
                     super_e, super_maps);
  hipLaunchKernelGGL(k_sum_walk<SQUARES>, dim3(1), dim3(64), 0, st, x, n, e, maps, super_e,
                     super_maps, ntiles, stats, nsat, exact);
}

// stats_in (optional): per-read (mean, sd) to apply instead of the read's
// own statistics; stats_out (optional): the (mean, sd) applied.
__global__ __launch_bounds__(64) void k_prep_queries(const float* __restrict__ raw,
                                                     const int64_t* __restrict__ offs, int32_t nq,
                                                     double scale,
                                                     const double* __restrict__ stats_in,
                                                     double* __restrict__ stats_out,
                                                     float* __restrict__ z,
                                                     int16_t* __restrict__ codes,
                                                     int64_t* __restrict__ nsat) {
  issue_first();
  __shared__ float buf[2 * kQChunk];
  const int32_t r = (int32_t)blockIdx.x;
  if (r >= nq) return;
  const int64_t a = offs[r], b = offs[r + 1];
  if (b <= a) return;
  double mean, sd;
  if (stats_in) {
    mean = stats_in[2 * r];
    sd = stats_in[2 * r + 1];
  } else {
    const double n = (double)(b - a);
    mean = wave_seq_sum(raw, a, b, 0.0, false, buf) / n;
    sd = sqrt(wave_seq_sum(raw, a, b, mean, true, buf) / n);
  }
  if (stats_out && threadIdx.x == 0) {
    stats_out[2 * r] = mean;
    stats_out[2 * r + 1] = sd;
  }
  unsigned long long sat = 0;
  for (int64_t i = a + threadIdx.x; i < b; i += 64) {
    const float zi = sd > 0.0 ? (float)(((double)raw[i] - mean) / sd) : 0.0f;
    z[i] = zi;
    if (codes) codes[i] = to_code(zi, scale, &sat);
  }
  if (nsat && sat) atomicAdd((unsigned long long*)nsat, sat);
}

// Device layout of a reference: int16 -> u32 with +32768 bias, float -> bits;
// zero padding up to n_pad (a multiple of the workgroup).  Counted: non-finite
// float values, and the waves whose 64 values are equal.
__global__ void k_layout(const void* __restrict__ src, int64_t n, int dtype,
                         uint32_t* __restrict__ dst, int64_t n_pad, int32_t* __restrict__ found) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t v = 0;
  if (i < n) {
    if (dtype == SDTW_I16) {
      v = (uint32_t)((int32_t)((const int16_t*)src)[i] + (int32_t)kI16Bias);
    } else {
      const float f = ((const float*)src)[i];
      if (!isfinite(f)) atomicAdd(&found[0], 1);
      v = __float_as_uint(f);
    }
  }
  dst[i] = v;
  const uint32_t v0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  const bool equal = __ballot(i < n && v == v0) == ~0ull;
  // (several words: a constant reference's waves would queue at one)
  if (equal && (threadIdx.x & 63) == 0) atomicAdd(&found[1 + blockIdx.x % kFlatCounts], 1);
}

inline unsigned grid_for(int64_t n, int threads) {
  return (unsigned)((n + threads - 1) / threads);
}

}  // namespace

hipError_t launch_prepare_reference(const uint8_t* g, int64_t L, const float* table, int k,
                                    double scale, float* z, int16_t* codes, int64_t* nsat,
                                    double* scratch, hipStream_t st) {
  const int64_t n = 2 * (L - k + 1);
  // the raw signal is produced in z and normalised in place
  hipLaunchKernelGGL(k_kmer, dim3(grid_for(n, kPrepThreads)), dim3(kPrepThreads), 0, st,
                     g, L, k, table, z);
  double* stats = scratch;
  if (n <= kSmallSum) {
    hipLaunchKernelGGL(k_sum_small, dim3(1), dim3(64), 0, st, z, (int32_t)n, stats,
                       nsat);
  } else {
    launch_sum<false>(z, n, scratch, nullptr, st);
    launch_sum<true>(z, n, scratch, nsat, st);
  }
  hipLaunchKernelGGL(k_normalize, dim3(grid_for(n, kPrepThreads)), dim3(kPrepThreads), 0, st,
                     z, n, stats, scale, z, codes, nsat);
  return hipGetLastError();
}

int64_t ref_scratch_doubles(int64_t n) {
  const int64_t tiles = (n + kSumTile - 1) / kSumTile;
  const int64_t supers = (tiles + kSuper - 1) / kSuper;
  return 2 + tiles + 2 * (tiles + supers) + (2 * tiles + supers + 2) / 2;
}

hipError_t launch_prepare_queries(const float* raw, const int64_t* offs, int32_t nq,
                                  double scale, const double* stats_in, double* stats_out,
                                  float* z, int16_t* codes, int64_t* nsat, hipStream_t st) {
  if (nsat) hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(64), 0, st, nsat);
  hipLaunchKernelGGL(k_prep_queries, dim3(nq), dim3(64), 0, st, raw, offs, nq, scale, stats_in,
                     stats_out, z, codes, nsat);
  return hipGetLastError();
}

hipError_t launch_layout_reference(const void* src, int64_t n, int dtype, uint32_t* dst,
                                   int64_t n_pad, int32_t* found, hipStream_t st) {
  hipLaunchKernelGGL(k_layout, dim3(grid_for(n_pad, kPrepThreads)), dim3(kPrepThreads), 0, st,
                     src, n, dtype, dst, n_pad, found);
  return hipGetLastError();
}

}  // namespace sdtw
