// C ABI of the sDTW library: validation, object lifetimes, scheduling.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <numeric>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "common.h"
#include "cut.h"

struct sdtw_ref_s {
  int device;
  int dtype;
  int64_t n;       // true length
  int64_t n_pad;   // device layout length
  uint32_t* data;  // u32 biased int16 or float bits
  int64_t flat;    // columns in runs of at least 64 equal values
  std::atomic<int> open_streams;
  std::atomic<int> stream_strip{0};  // sdtw_stream_set_config for this reference (0: automatic)
  std::atomic<int> stream_bands{0};
};

namespace sdtw {
// Completion of one sdtw_stream_extend call (one event per call, shared by
// the streams it extended); the event returns to a pool when released.
struct CallToken {
  hipEvent_t ev = nullptr;
  ~CallToken();
};
}  // namespace sdtw

struct sdtw_stream_s {
  int device;
  sdtw_ref ref;
  uint32_t* row;        // resident row gamma(rows, .), n_pad entries
  size_t bytes;
  int32_t rows;         // query rows folded in so far
  std::shared_ptr<sdtw::CallToken> last;  // last extend that used the row
};

struct sdtw_plan_s {
  int device;
  int dtype;
  int32_t nq;
  int32_t max_m;
  std::vector<int32_t> sorted_m;  // read lengths, longest first (order_dev's order)
  int64_t* offs_dev;              // [nq+1]
  int32_t* order_dev;             // [nq]: read indices, longest first
  uint32_t* sched_dev;            // [kSchedWords]: pull and placement state of a launch
  int strip;                      // columns per lane
  int chains;                     // most chains per lane (K) the long reads use
  int bands;                      // waves per read (row bands) of the skew kernel
  int32_t band_rows;              // target rows per band (0: as many bands as fit)
  int waves_per_cu;               // persistent grid density (bands x workgroups per CU)
  int cus;                        // compute units of the device
  // Row-lane kernel (rows.h), for the reads of up to kRowsMaxM rows: order[nlong ..),
  // or none (nlong == nq) beside few longer ones (split_pays)
  bool rows;                      // use it (a launch shape set by the caller: the skew kernel)
  int32_t nlong;                  // reads that it does not take
  sdtw::RowLayout* lay[2];        // reads sharing waves; reads alone in theirs
  sdtw::RowPack* packs_dev[2];
  int64_t scratch_words;
  uint64_t* scratch;
  int64_t cut_n;                  // reference length that `cut` is for (0: none yet)
  int cut_lay;
  double cut_cycles;              // modelled
  double short_rows;              // rows of order[nlong ..) in all
  sdtw::RowsArgs cut;             // how it is cut
};

namespace sdtw {

static thread_local char g_err[512] = "";

int set_error(int status, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return status;
}

int check_hip(hipError_t e, const char* what) {
  if (e == hipSuccess) return SDTW_OK;
  if (e == hipErrorOutOfMemory)
    return set_error(SDTW_ENOMEM, "%s: %s", what, hipGetErrorString(e));
  return set_error(SDTW_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

int max_lds_bytes() {
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 65536;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    return 65536;
  return v;
}

static int current_device() {
  int d = -1;
  if (hipGetDevice(&d) != hipSuccess) return -1;
  return d;
}

// Kernels run on the current device; objects of another device would be
// reached through peer addresses, so every call that launches checks.
static int require_device(int dev, const char* who) {
  const int cur = current_device();
  if (cur != dev)
    return set_error(SDTW_EINVAL, "%s: objects live on device %d, current device is %d", who, dev,
                     cur);
  return SDTW_OK;
}

static int cu_count() {
  int dev = current_device(), v = 0;
  if (dev < 0 || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return v;
}

// Whether reads or chunks of `rows` rows in all leave the row-lane kernel, cut
// as in `a` (of `cycles` modelled cycles), for the column-lane kernels on n
// columns of this reference.  Equal values cost a path that stays on a row of about the same
// value next to nothing, so the column segments that they fill do not settle, and
// one wave per pack walks them: 48 reads of 250 rows against 1,000,000 equal
// values 73.7 ms, 22.5 on the column-lane kernels, and with a tenth of the values
// equal 8.6 and 22.5.  A walked step takes up to 1.4 times the model's; the
// column-lane kernels take a read's tiles one after another at 50 cycles a column
// (40 for chunks on long references) or, with many reads, 4,500 cells a cycle.
static bool walked_longer(sdtw_ref ref, int64_t n, const RowsArgs& a, double cycles, double rows,
                          bool stream) {
  if (ref->flat == 0) return false;
  double step = 0.0;
  for (int k = 0; k < a.nclasses; ++k)
    step = std::max(step, RowCost{a.dpp != 0, ref->dtype == SDTW_F32, stream}.step(
                              a.cls[k].rows_per_lane, 1.0));
  const double walk = 1.4 / 4.0 * step * (double)ref->flat * (double)n / (double)ref->n;
  const double tiles = (double)n * (stream && n >= (int64_t(1) << 20) ? 40.0 : 50.0);
  return cycles + walk > std::max(tiles, rows * (double)n / (4500.0 / 256.0 * a.cus));
}

static bool valid_strip(int s) { return s == 8 || s == 16 || s == 32; }

}  // namespace sdtw

namespace sdtw {

// ---- events recycled across extend calls -----------------------------------
static std::mutex g_ev_mu;
static std::vector<hipEvent_t> g_ev_free;

static hipEvent_t event_get() {
  {
    std::lock_guard<std::mutex> g(g_ev_mu);
    if (!g_ev_free.empty()) {
      hipEvent_t e = g_ev_free.back();
      g_ev_free.pop_back();
      return e;
    }
  }
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return nullptr;
  return e;
}

CallToken::~CallToken() {
  if (!ev) return;
  std::lock_guard<std::mutex> g(g_ev_mu);
  g_ev_free.push_back(ev);
}

// ---- resident-row pool: a byte budget per device, rows cached by size ----
struct RowPool {
  std::mutex mu;
  int64_t budget = int64_t(16) << 30;
  int64_t in_use = 0;
  int64_t cached = 0;
  std::map<size_t, std::vector<void*>> free_rows;
};
constexpr int kMaxDevices = 64;
static RowPool g_pool[kMaxDevices];

static RowPool* pool_for(int dev) {
  return (dev >= 0 && dev < kMaxDevices) ? &g_pool[dev] : nullptr;
}

// ---- pinned descriptor slots for stream_extend -----------------------------
struct DescSlot {
  StreamItem* host = nullptr;
  StreamItem* dev = nullptr;  // room for cap items and packs, then one int32 work counter
  int32_t cap = 0;
  // (on the host likewise; a call's packs follow its n items, so that one copy
  // takes just those)
  static constexpr size_t kPer = sizeof(StreamItem) + sizeof(RowPack);
  RowPack* host_packs(int32_t n) { return (RowPack*)(host + n); }
  RowPack* dev_packs(int32_t n) { return (RowPack*)(dev + n); }
  int32_t* counter() { return (int32_t*)((char*)dev + kPer * (size_t)cap); }
  uint64_t* part = nullptr;  // scratch of the call: per-segment minima (sdtw_stream_best_two),
                             // boundary columns and results, flags of a row scan
  int64_t part_cap = 0;
  std::shared_ptr<CallToken> last;
};
// A call takes a slot whose previous call has completed, adding slots (up to
// kMaxDescSlots) while every slot is still in use, so that a long call on
// one HIP stream never holds back calls on other streams.
constexpr int kMaxDescSlots = 64;
struct DescRing {
  std::mutex mu;
  std::vector<std::unique_ptr<DescSlot>> slot;
  int next = 0;  // round-robin victim when all kMaxDescSlots are busy
  // long-reference stream extensions enqueued and perhaps still running, with
  // their workgroup counts
  std::vector<std::pair<std::shared_ptr<CallToken>, int>> long_inflight;
};
static DescRing g_ring[kMaxDevices];
static std::atomic<int> g_stream_bands{0};  // sdtw_stream_set_config (0: automatic)
static std::atomic<int> g_stream_strip{0};

static int ensure_slot(DescSlot& sl, int32_t n) {
  if (sl.cap >= n) return SDTW_OK;
  int32_t cap = std::max<int32_t>(n, std::max<int32_t>(2 * sl.cap, 1024));
  if (sl.host) (void)hipHostFree(sl.host);
  if (sl.dev) (void)hipFree(sl.dev);
  sl.host = nullptr;
  sl.dev = nullptr;
  sl.cap = 0;
  int rc = check_hip(hipHostMalloc((void**)&sl.host, DescSlot::kPer * (size_t)cap),
                     "sdtw_stream_extend: pinned descriptors");
  if (!rc)
    rc = check_hip(hipMalloc((void**)&sl.dev, DescSlot::kPer * (size_t)cap + 64),
                   "sdtw_stream_extend: device descriptors");
  if (rc) return rc;
  sl.cap = cap;
  return SDTW_OK;
}

// A slot's scratch.  The first allocation already holds 2^23 words (64 MiB), and
// sdtw_stream_extend cuts its launches to fit, so that serving loops do not regrow
// it: hipFree of the old buffer would wait for all work on the device, including
// long launches on other HIP streams.  (256 chunks of 400 rows x 10 M columns take
// 32 MB, 1,024 of them 63; segment minima 8 MB for 1,024 rows of 16 M columns.)
constexpr int64_t kPartWords = int64_t(1) << 23;
static int ensure_part(DescSlot& sl, int64_t n) {
  if (sl.part_cap >= n) return SDTW_OK;
  const int64_t cap = std::max<int64_t>(std::max<int64_t>(n, 2 * sl.part_cap), kPartWords);
  if (sl.part) (void)hipFree(sl.part);
  sl.part = nullptr;
  sl.part_cap = 0;
  int rc = check_hip(hipMalloc((void**)&sl.part, sizeof(uint64_t) * (size_t)cap),
                     "scratch of a call");
  if (rc) return rc;
  sl.part_cap = cap;
  return SDTW_OK;
}

// A descriptor slot for a call of n items: one whose previous call has
// completed, else a new one (up to kMaxDescSlots), else the round-robin
// victim after its call completes.  The caller holds ring.mu.
static int acquire_slot(DescRing& ring, int32_t n, DescSlot** out, const char* who) {
  DescSlot* pick = nullptr;
  for (auto& c : ring.slot) {
    if (!c->last || !c->last->ev || hipEventQuery(c->last->ev) == hipSuccess) {
      pick = c.get();
      break;
    }
  }
  if (!pick && (int)ring.slot.size() < kMaxDescSlots) {
    ring.slot.push_back(std::make_unique<DescSlot>());
    pick = ring.slot.back().get();
  }
  if (!pick) {
    pick = ring.slot[(size_t)ring.next].get();
    ring.next = (ring.next + 1) % kMaxDescSlots;
    int rc = check_hip(hipEventSynchronize(pick->last->ev), who);
    if (rc) return rc;
  }
  int rc = ensure_slot(*pick, n);
  if (rc) return rc;
  *out = pick;
  return SDTW_OK;
}

}  // namespace sdtw

using namespace sdtw;

#define SDTW_REQUIRE(cond, ...) \
  do {                          \
    if (!(cond)) return set_error(SDTW_EINVAL, __VA_ARGS__); \
  } while (0)

// The end of an entry point whose body allocates on the host: nothing is thrown
// through the C ABI.
#define SDTW_NO_MEMORY(who)                                      \
  catch (const std::bad_alloc&) {                                \
    return set_error(SDTW_ENOMEM, "%s: host allocation", who);   \
  }

extern "C" {

const char* sdtw_last_error(void) { return g_err; }

int sdtw_version(void) { return 1; }

// ---------------------------------------------------------------------------
// preparation
// ---------------------------------------------------------------------------

int sdtw_prepare_reference(const uint8_t* genome_dev, int64_t L, const float* table_dev, int k,
                           double scale, float* z_dev, int16_t* codes_dev, int64_t* nsat_dev,
                           void* stream) {
  SDTW_REQUIRE(genome_dev && table_dev && z_dev, "sdtw_prepare_reference: null pointer");
  SDTW_REQUIRE(k >= 1 && k <= 12, "sdtw_prepare_reference: k=%d outside [1, 12]", k);
  SDTW_REQUIRE(L >= k, "sdtw_prepare_reference: genome length %lld < k=%d", (long long)L, k);
  SDTW_REQUIRE(L - k + 1 <= (int64_t)INT32_MAX / 2,
               "sdtw_prepare_reference: genome too long (%lld bases)", (long long)L);
  SDTW_REQUIRE(isfinite(scale) && scale > 0.0, "sdtw_prepare_reference: scale must be > 0");
  hipStream_t st = (hipStream_t)stream;
  double* scratch = nullptr;
  int rc = check_hip(hipMallocAsync((void**)&scratch,
                                    ref_scratch_doubles(2 * (L - k + 1)) * sizeof(double), st),
                     "sdtw_prepare_reference: scratch");
  if (rc) return rc;
  rc = check_hip(launch_prepare_reference(genome_dev, L, table_dev, k, scale, z_dev, codes_dev,
                                          nsat_dev, scratch, st),
                 "sdtw_prepare_reference: launch");
  hipError_t e = hipFreeAsync(scratch, st);
  if (rc) return rc;
  return check_hip(e, "sdtw_prepare_reference: free");
}

int sdtw_prepare_queries(const float* raw_dev, const int64_t* offsets_dev, int32_t nq,
                         double scale, float* z_dev, int16_t* codes_dev, int64_t* nsat_dev,
                         void* stream) {
  SDTW_REQUIRE(raw_dev && offsets_dev && z_dev, "sdtw_prepare_queries: null pointer");
  SDTW_REQUIRE(nq >= 1, "sdtw_prepare_queries: nq=%d < 1", nq);
  SDTW_REQUIRE(isfinite(scale) && scale > 0.0, "sdtw_prepare_queries: scale must be > 0");
  return check_hip(launch_prepare_queries(raw_dev, offsets_dev, nq, scale, nullptr, nullptr,
                                          z_dev, codes_dev, nsat_dev, (hipStream_t)stream),
                   "sdtw_prepare_queries: launch");
}

int sdtw_prepare_queries_ex(const float* raw_dev, const int64_t* offsets_dev, int32_t nq,
                            double scale, const double* stats_in_dev, double* stats_out_dev,
                            float* z_dev, int16_t* codes_dev, int64_t* nsat_dev, void* stream) {
  SDTW_REQUIRE(raw_dev && offsets_dev && z_dev, "sdtw_prepare_queries_ex: null pointer");
  SDTW_REQUIRE(nq >= 1, "sdtw_prepare_queries_ex: nq=%d < 1", nq);
  SDTW_REQUIRE(isfinite(scale) && scale > 0.0, "sdtw_prepare_queries_ex: scale must be > 0");
  return check_hip(launch_prepare_queries(raw_dev, offsets_dev, nq, scale, stats_in_dev,
                                          stats_out_dev, z_dev, codes_dev, nsat_dev,
                                          (hipStream_t)stream),
                   "sdtw_prepare_queries_ex: launch");
}

int sdtw_detect_events(const float* raw_dev, const int64_t* offsets_dev, int32_t nreads,
                       int32_t trim, int32_t keep, float* events_dev, int32_t* counts_dev,
                       void* stream) {
  SDTW_REQUIRE(raw_dev && offsets_dev && events_dev && counts_dev,
               "sdtw_detect_events: null pointer");
  SDTW_REQUIRE(nreads >= 1, "sdtw_detect_events: nreads=%d < 1", nreads);
  SDTW_REQUIRE(trim >= 0 && keep >= 1 && keep <= SDTW_MAX_QUERY &&
                   (int64_t)trim + keep <= kMaxEventList,
               "sdtw_detect_events: trim=%d keep=%d outside trim >= 0, 1 <= keep <= %d, "
               "trim + keep <= %d", trim, keep, SDTW_MAX_QUERY, kMaxEventList);
  return check_hip(launch_detect_events(raw_dev, offsets_dev, 1, nullptr, nreads, trim, keep, 0,
                                        events_dev, counts_dev, (hipStream_t)stream),
                   "sdtw_detect_events: launch");
}

int sdtw_detect_events_prefix(const float* raw_dev, const int64_t* ranges_dev,
                              const int32_t* firsts_dev, int32_t nreads, int32_t max_first,
                              int32_t keep, float* events_dev, int32_t* counts_dev,
                              void* stream) {
  SDTW_REQUIRE(raw_dev && ranges_dev && firsts_dev && events_dev && counts_dev,
               "sdtw_detect_events_prefix: null pointer");
  SDTW_REQUIRE(nreads >= 1, "sdtw_detect_events_prefix: nreads=%d < 1", nreads);
  SDTW_REQUIRE(max_first >= 0 && keep >= 1 && keep <= SDTW_MAX_QUERY &&
                   (int64_t)max_first + keep <= kMaxEventList,
               "sdtw_detect_events_prefix: max_first=%d keep=%d outside max_first >= 0, "
               "1 <= keep <= %d, max_first + keep <= %d", max_first, keep, SDTW_MAX_QUERY,
               kMaxEventList);
  return check_hip(launch_detect_events(raw_dev, ranges_dev, 2, firsts_dev, nreads, max_first,
                                        keep, 1, events_dev, counts_dev, (hipStream_t)stream),
                   "sdtw_detect_events_prefix: launch");
}

int64_t sdtw_event_state_bytes(void) { return (int64_t)event_state_bytes(); }

int sdtw_event_state_init(void* states_dev, const int32_t* slots_dev, int32_t n, void* stream) {
  SDTW_REQUIRE(states_dev && slots_dev, "sdtw_event_state_init: null pointer");
  SDTW_REQUIRE(n >= 1, "sdtw_event_state_init: n=%d < 1", n);
  return check_hip(launch_event_state_init(states_dev, slots_dev, n, (hipStream_t)stream),
                   "sdtw_event_state_init: launch");
}

int sdtw_detect_events_continue(const float* raw_dev, const int64_t* ranges_dev,
                                const int32_t* slots_dev, void* states_dev, int32_t nreads,
                                int32_t trim, int32_t keep, float* events_dev,
                                int32_t* counts_dev, void* stream) {
  SDTW_REQUIRE(raw_dev && ranges_dev && slots_dev && states_dev && events_dev && counts_dev,
               "sdtw_detect_events_continue: null pointer");
  SDTW_REQUIRE(nreads >= 1, "sdtw_detect_events_continue: nreads=%d < 1", nreads);
  SDTW_REQUIRE(trim >= 0 && keep >= 1 && keep <= SDTW_MAX_QUERY,
               "sdtw_detect_events_continue: trim=%d keep=%d outside trim >= 0, "
               "1 <= keep <= %d", trim, keep, SDTW_MAX_QUERY);
  return check_hip(launch_events_continue(raw_dev, ranges_dev, slots_dev, states_dev, nreads,
                                          trim, keep, events_dev, counts_dev,
                                          (hipStream_t)stream),
                   "sdtw_detect_events_continue: launch");
}

// ---------------------------------------------------------------------------
// reference
// ---------------------------------------------------------------------------

int sdtw_load_reference(const void* ref, int64_t n, int dtype, int ref_is_device, void* stream,
                        sdtw_ref* out) {
  SDTW_REQUIRE(ref && out, "sdtw_load_reference: null pointer");
  SDTW_REQUIRE(dtype == SDTW_F32 || dtype == SDTW_I16, "sdtw_load_reference: bad dtype %d", dtype);
  SDTW_REQUIRE(n >= 1 && n <= (int64_t)INT32_MAX - 2 * kPadUnit,
               "sdtw_load_reference: length %lld outside [1, 2^31)", (long long)n);
  hipStream_t st = (hipStream_t)stream;
  const size_t esz = dtype == SDTW_I16 ? 2 : 4;
  const int64_t n_pad = padded_length(n);
  uint32_t* data = nullptr;
  void* tmp = nullptr;
  int32_t* found = nullptr;
  int32_t host_found[1 + kFlatCounts] = {};  // non-finite values, runs of 64 equal ones
  int rc = check_hip(hipMalloc((void**)&data, (size_t)n_pad * 4), "sdtw_load_reference: alloc");
  if (!rc) rc = check_hip(hipMalloc((void**)&found, sizeof host_found), "sdtw_load_reference: alloc");
  if (!rc) rc = check_hip(hipMemcpyAsync(found, host_found, sizeof host_found,
                                         hipMemcpyHostToDevice, st), "sdtw_load_reference: copy");
  const void* src = ref;
  if (!rc && !ref_is_device) {
    rc = check_hip(hipMalloc(&tmp, (size_t)n * esz), "sdtw_load_reference: alloc");
    if (!rc) rc = check_hip(hipMemcpyAsync(tmp, ref, (size_t)n * esz, hipMemcpyHostToDevice, st),
                            "sdtw_load_reference: copy");
    src = tmp;
  }
  if (!rc) rc = check_hip(launch_layout_reference(src, n, dtype, data, n_pad, found, st),
                          "sdtw_load_reference: layout");
  if (!rc) rc = check_hip(hipMemcpyAsync(host_found, found, sizeof host_found,
                                         hipMemcpyDeviceToHost, st), "sdtw_load_reference: copy");
  if (!rc) rc = check_hip(hipStreamSynchronize(st), "sdtw_load_reference: sync");
  if (tmp) (void)hipFree(tmp);
  if (found) (void)hipFree(found);
  if (!rc && host_found[0])
    rc = set_error(SDTW_EINVAL, "sdtw_load_reference: %d non-finite values", host_found[0]);
  if (rc) {
    if (data) (void)hipFree(data);
    return rc;
  }
  sdtw_ref_s* r = new (std::nothrow) sdtw_ref_s;
  if (!r) {
    (void)hipFree(data);
    return set_error(SDTW_ENOMEM, "sdtw_load_reference: host allocation");
  }
  r->device = current_device();
  r->dtype = dtype;
  r->n = n;
  r->n_pad = n_pad;
  r->data = data;
  r->flat = 0;
  for (int k = 0; k < kFlatCounts; ++k) r->flat += 64 * (int64_t)host_found[1 + k];
  r->open_streams = 0;
  *out = r;
  return SDTW_OK;
}

int sdtw_reference_info(sdtw_ref ref, int64_t* n, int* dtype) {
  SDTW_REQUIRE(ref, "sdtw_reference_info: null reference");
  if (n) *n = ref->n;
  if (dtype) *dtype = ref->dtype;
  return SDTW_OK;
}

int sdtw_free_reference(sdtw_ref ref) {
  SDTW_REQUIRE(ref, "sdtw_free_reference: null reference");
  if (ref->open_streams > 0)
    return set_error(SDTW_ESTATE, "sdtw_free_reference: %d streams still open",
                     ref->open_streams.load());
  int rc = check_hip(hipFree(ref->data), "sdtw_free_reference");
  delete ref;
  return rc;
}

// ---------------------------------------------------------------------------
// plans
// ---------------------------------------------------------------------------

// One launch of the batch: reads order[first, first + count), longest first,
// run by the skew kernel with `chains` chains per lane and `bands` waves per
// read (chains == 0: the synchronised single-wave kernel).
struct LaunchGroup {
  int32_t first, count, max_m, chains, bands, max_band, band_target;
};

static std::vector<LaunchGroup> launch_groups(const sdtw_plan_s* p, bool rows) {
  std::vector<LaunchGroup> g;
  int32_t pos = 0;
  const int32_t n = rows ? p->nlong : p->nq;  // the rest: the row-lane kernel
  for (int k = p->chains; k >= 1; k /= 2) {
    if (!valid_strip_chains(p->strip, k)) continue;
    const int bands = valid_skew_config(p->strip, k, p->bands) ? p->bands : 1;
    const int32_t target = bands > 1 ? p->band_rows : 0;
    const int32_t lo = skew_min_m(k);
    const int32_t start = pos;
    int32_t max_band = 0;
    while (pos < n && p->sorted_m[pos] >= lo) {
      max_band = std::max(max_band, skew_band_rows(p->sorted_m[pos], k, bands, target));
      ++pos;
    }
    if (pos > start)
      g.push_back({start, pos - start, p->sorted_m[start], k, bands, max_band, target});
  }
  if (pos < n) g.push_back({pos, n - pos, p->sorted_m[pos], 0, 1, 0, 0});
  return g;
}

// Resident waves per CU for a skew launch: whole workgroups of `bands` waves
// within the CU's 160 KiB of LDS, at most 16 waves (four per SIMD).
static int skew_waves_per_cu(int strip, int chains, int bands, int max_band,
                             bool stream = false) {
  const size_t per = skew_lds_bytes(strip, chains, bands, max_band, stream);
  const int groups = (int)std::min<size_t>(16 / bands, (160 * 1024) / std::max<size_t>(per, 1));
  return std::max(groups, 1) * bands;
}

// LDS to reserve per workgroup so that `blocks` workgroups spread evenly over
// the compute units: when there are fewer than the CUs could hold, reserve a
// 1/ceil(blocks/cus) share of a CU's 160 KiB (whole KiB) so that no CU takes
// more than its share (the dispatcher would otherwise fill some CUs up to
// their limit and leave others with less work).  `min_share` > 1 leaves room
// for that many launches at once on every CU.
static int32_t spread_lds(size_t need, int blocks, int groups_per_cu, int cus,
                          int min_share = 1) {
  constexpr size_t kCuLds = 160 * 1024;
  if ((int64_t)blocks >= (int64_t)groups_per_cu * cus) return 0;
  const int share = std::max((blocks + cus - 1) / cus, min_share);
  // 1 KiB less than the share leaves room for the kernel's static LDS (a
  // share-sized reservation would let only share - 1 workgroups in)
  const size_t cap = (size_t)max_lds_bytes() - 1024;
  const size_t want = (std::min(kCuLds / (size_t)share, cap + 1024) - 1024) & ~(size_t)1023;
  return want > need ? (int32_t)want : 0;
}

// Default launch shape.  A wave issues about one VALU instruction per 10
// cycles when its instructions depend on each other and no faster than one
// per 5 cycles however independent they are (measured on gfx950), while a
// SIMD issues one per about 4.3 cycles from two or more waves.  So every SIMD
// needs two or more waves: with four or more reads per SIMD one wave per
// read and one chain per lane; with fewer, each read is cut into two row
// bands when its rows allow (measured on 1,024 reads of 250-500 rows x 10 M
// columns: 1.73x one band, 1.23x four bands, whose 64 tile-switch steps per
// band of ~94 rows cost more than the extra waves bring), else two chains.
static void choose_config(sdtw_plan_s* p) {
  p->strip = 16;
  const int64_t simds = (int64_t)p->cus * 4;
  const int32_t median_m = p->sorted_m[(size_t)p->nq / 2];
  if (p->nq >= 4 * simds) {
    p->chains = 1;
    p->bands = 1;
  } else if (median_m >= 2 * skew_min_m(1)) {
    p->chains = 1;
    p->bands = 2;
  } else {
    p->chains = 2;
    p->bands = 1;
  }
  p->band_rows = 0;
  p->waves_per_cu = skew_waves_per_cu(p->strip, p->chains, p->bands,
                                      std::max(skew_band_rows(p->max_m, p->chains, p->bands),
                                               skew_min_m(p->chains)));
}

// Frees a plan and what it holds; the first error.
static hipError_t plan_free(sdtw_plan_s* p) {
  hipError_t first = hipSuccess;
  for (void* d : {(void*)p->offs_dev, (void*)p->order_dev, (void*)p->sched_dev,
                  (void*)p->packs_dev[0], (void*)p->packs_dev[1], (void*)p->scratch}) {
    const hipError_t e = hipFree(d);
    if (first == hipSuccess) first = e;
  }
  delete p->lay[0];
  delete p->lay[1];
  delete p;
  return first;
}

int sdtw_plan_create(const int64_t* offsets_host, int32_t nq, int dtype, sdtw_plan* out) try {
  SDTW_REQUIRE(offsets_host && out, "sdtw_plan_create: null pointer");
  SDTW_REQUIRE(nq >= 1, "sdtw_plan_create: nq=%d < 1", nq);
  SDTW_REQUIRE(dtype == SDTW_F32 || dtype == SDTW_I16, "sdtw_plan_create: bad dtype %d", dtype);
  SDTW_REQUIRE(offsets_host[0] >= 0, "sdtw_plan_create: negative offset");
  std::vector<int32_t> order((size_t)nq);
  int32_t max_m = 0;
  for (int32_t r = 0; r < nq; ++r) {
    const int64_t m = offsets_host[r + 1] - offsets_host[r];
    SDTW_REQUIRE(m >= 1 && m <= SDTW_MAX_QUERY,
                 "sdtw_plan_create: read %d has length %lld outside [1, %d]", r, (long long)m,
                 SDTW_MAX_QUERY);
    order[(size_t)r] = r;
    max_m = std::max<int32_t>(max_m, (int32_t)m);
  }
  auto len = [&](int32_t r) { return offsets_host[r + 1] - offsets_host[r]; };
  std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
    return len(a) != len(b) ? len(a) > len(b) : a < b;
  });

  struct Free {
    void operator()(sdtw_plan_s* plan) const { (void)plan_free(plan); }
  };
  std::unique_ptr<sdtw_plan_s, Free> own(new sdtw_plan_s());
  sdtw_plan_s* const p = own.get();
  p->device = current_device();
  p->dtype = dtype;
  p->nq = nq;
  p->max_m = max_m;
  p->sorted_m.resize((size_t)nq);
  for (int32_t i = 0; i < nq; ++i) p->sorted_m[(size_t)i] = (int32_t)len(order[(size_t)i]);
  p->cus = cu_count();
  if (p->cus <= 0) p->cus = 256;
  choose_config(p);
  p->rows = true;
  double long_rows = 0.0;
  for (int32_t i = 0; i < nq; ++i) {
    const int32_t m = p->sorted_m[(size_t)i];
    (m > kRowsMaxM ? long_rows : p->short_rows) += m;
    if (m > kRowsMaxM) ++p->nlong;
  }
  if (p->nlong && p->nlong < nq &&
      !split_pays(max_m, p->sorted_m[(size_t)p->nlong], long_rows, p->short_rows, p->cus))
    p->nlong = nq;
  std::vector<std::pair<int32_t, int32_t>> reads;
  for (int32_t i = p->nlong; i < nq; ++i)
    reads.emplace_back(order[(size_t)i], p->sorted_m[(size_t)i]);
  for (int i = 0; i < 2; ++i) {
    if (i == 1 && !alone_pays(*p->lay[0], p->cus)) break;
    p->lay[i] = new RowLayout(rows_layout(reads, i == 1, kRowsReads));
    p->scratch_words = std::max(p->scratch_words, rows_most_words(*p->lay[i], p->cus));
  }
  int rc = check_hip(hipMalloc((void**)&p->offs_dev, sizeof(int64_t) * (size_t)(nq + 1)),
                     "sdtw_plan_create: alloc");
  if (!rc) rc = check_hip(hipMalloc((void**)&p->order_dev, sizeof(int32_t) * (size_t)nq),
                          "sdtw_plan_create: alloc");
  if (!rc) rc = check_hip(hipMalloc((void**)&p->sched_dev, sizeof(uint32_t) * kSchedWords),
                          "sdtw_plan_create: alloc");
  if (!rc) rc = check_hip(hipMemcpy(p->offs_dev, offsets_host, sizeof(int64_t) * (size_t)(nq + 1),
                                    hipMemcpyHostToDevice), "sdtw_plan_create: copy");
  if (!rc) rc = check_hip(hipMemcpy(p->order_dev, order.data(), sizeof(int32_t) * (size_t)nq,
                                    hipMemcpyHostToDevice), "sdtw_plan_create: copy");
  for (int i = 0; i < 2 && !rc && !reads.empty() && p->lay[i]; ++i) {
    const size_t bytes = sizeof(RowPack) * p->lay[i]->packs.size();
    rc = check_hip(hipMalloc((void**)&p->packs_dev[i], bytes), "sdtw_plan_create: alloc");
    if (!rc)
      rc = check_hip(hipMemcpy(p->packs_dev[i], p->lay[i]->packs.data(), bytes,
                               hipMemcpyHostToDevice), "sdtw_plan_create: copy");
  }
  if (!rc && p->scratch_words &&
      hipMalloc((void**)&p->scratch, sizeof(uint64_t) * (size_t)p->scratch_words) != hipSuccess) {
    (void)hipGetLastError();
    p->scratch = nullptr;
    p->scratch_words = 0;  // one segment per pack
  }
  if (rc) return rc;
  *out = own.release();
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_plan_create")

int sdtw_plan_info(sdtw_plan plan, int32_t* nq, int* dtype, int32_t* max_m) {
  SDTW_REQUIRE(plan, "sdtw_plan_info: null plan");
  if (nq) *nq = plan->nq;
  if (dtype) *dtype = plan->dtype;
  if (max_m) *max_m = plan->max_m;
  return SDTW_OK;
}

int sdtw_plan_set_config(sdtw_plan plan, int strip, int chains, int bands, int waves_per_cu,
                         int32_t band_rows) {
  SDTW_REQUIRE(plan, "sdtw_plan_set_config: null plan");
  SDTW_REQUIRE(band_rows == -1 || band_rows == 0 || band_rows >= skew_min_m(1),
               "sdtw_plan_set_config: band_rows %d is not -1, 0 or >= %d", band_rows,
               skew_min_m(1));
  SDTW_REQUIRE(strip == 0 || valid_strip(strip), "sdtw_plan_set_config: strip %d not in {8,16,32}",
               strip);
  SDTW_REQUIRE(chains == 0 || chains == 1 || chains == 2 || chains == 4,
               "sdtw_plan_set_config: chains %d not in {1,2,4}", chains);
  SDTW_REQUIRE(bands >= 0 && bands <= 4, "sdtw_plan_set_config: bands %d not in {1,2,3,4}",
               bands);
  SDTW_REQUIRE(waves_per_cu >= 0 && waves_per_cu <= 32,
               "sdtw_plan_set_config: waves_per_cu %d outside [0, 32]", waves_per_cu);
  const int s2 = strip ? strip : plan->strip;
  const int k2 = chains ? chains : plan->chains;
  const int w2 = waves_per_cu ? waves_per_cu : plan->waves_per_cu;
  SDTW_REQUIRE(valid_strip_chains(s2, k2),
               "sdtw_plan_set_config: strip %d with %d chains (strip/chains must be a multiple "
               "of 4)", s2, k2);
  int b2 = bands;
  if (b2 == 0) {  // keep the plan's bands where they fit the rest, else one wave per read
    b2 = plan->bands;
    if (!valid_skew_config(s2, k2, b2) || w2 % b2 != 0) b2 = 1;
  }
  SDTW_REQUIRE(valid_skew_config(s2, k2, b2),
               "sdtw_plan_set_config: strip %d with %d chains and %d bands is not built "
               "(bands > 1: strip 16 with at most 2 chains, strip 32 with 1 chain, or strip "
               "32 with 2 chains and 2 bands)", s2, k2, b2);
  SDTW_REQUIRE(w2 % b2 == 0, "sdtw_plan_set_config: waves_per_cu %d is not a multiple of %d bands",
               w2, b2);
  plan->strip = s2;
  plan->chains = k2;
  plan->bands = b2;
  plan->waves_per_cu = w2;
  if (band_rows >= 0) plan->band_rows = band_rows;
  if (strip || chains || bands || waves_per_cu || band_rows >= 0) plan->rows = false;
  return SDTW_OK;
}

int sdtw_plan_get_config(sdtw_plan plan, int* strip, int* chains, int* bands, int* waves_per_cu,
                         int32_t* band_rows) {
  SDTW_REQUIRE(plan, "sdtw_plan_get_config: null plan");
  if (strip) *strip = plan->strip;
  if (chains) *chains = plan->chains;
  if (bands) *bands = plan->bands;
  if (waves_per_cu) *waves_per_cu = plan->waves_per_cu;
  if (band_rows) *band_rows = plan->band_rows;
  return SDTW_OK;
}

int sdtw_plan_destroy(sdtw_plan plan) {
  SDTW_REQUIRE(plan, "sdtw_plan_destroy: null plan");
  return check_hip(plan_free(plan), "sdtw_plan_destroy");
}

// ---------------------------------------------------------------------------
// alignment
// ---------------------------------------------------------------------------

// Enqueue the batch's launches; `n` reference columns (the autotuner times a
// prefix of the reference).
static int align_batch_impl(sdtw_ref ref, sdtw_plan plan, const void* q_dev, void* cost_dev,
                            int32_t* end_dev, hipStream_t st, int64_t n);

int sdtw_align_batch(sdtw_ref ref, sdtw_plan plan, const void* q_dev, void* cost_dev,
                     int32_t* end_dev, void* stream) try {
  SDTW_REQUIRE(ref && plan, "sdtw_align_batch: null reference or plan");
  SDTW_REQUIRE(q_dev && cost_dev && end_dev, "sdtw_align_batch: null device pointer");
  SDTW_REQUIRE(ref->dtype == plan->dtype, "sdtw_align_batch: reference dtype %d != plan dtype %d",
               ref->dtype, plan->dtype);
  SDTW_REQUIRE(ref->device == plan->device, "sdtw_align_batch: reference and plan on devices %d, %d",
               ref->device, plan->device);
  if (int rc = require_device(ref->device, "sdtw_align_batch")) return rc;
  return align_batch_impl(ref, plan, q_dev, cost_dev, end_dev, (hipStream_t)stream, ref->n);
} SDTW_NO_MEMORY("sdtw_align_batch")

// Cuts the plan's reads of up to kRowsMaxM rows for n columns of ref; false if
// they are better off on the column-lane kernels there.
static bool plan_cut(sdtw_ref ref, sdtw_plan plan, int64_t n) {
  if (plan->nlong == plan->nq) return true;
  if (plan->cut_n != n) {
    const bool f32 = plan->dtype == SDTW_F32;
    RowsArgs ra{}, rb{};
    ra.cus = rb.cus = plan->cus;
    int64_t words = 0;
    const double shared = rows_best_cut(ra, *plan->lay[0], false, n, f32, false,
                                        plan->scratch_words, &words);
    const double alone = plan->lay[1] ? rows_best_cut(rb, *plan->lay[1], true, n, f32, false,
                                                      plan->scratch_words, &words)
                                      : INFINITY;
    plan->cut_lay = alone < shared;
    plan->cut = plan->cut_lay ? rb : ra;
    plan->cut_cycles = plan->cut_lay ? alone : shared;
    plan->cut_n = n;
  }
  return !walked_longer(ref, n, plan->cut, plan->cut_cycles, plan->short_rows, false);
}

static int align_batch_impl(sdtw_ref ref, sdtw_plan plan, const void* q_dev, void* cost_dev,
                            int32_t* end_dev, hipStream_t st, int64_t n) {
  SDTW_REQUIRE(valid_strip(plan->strip), "sdtw_align_batch: bad strip");
  const bool rows = plan->rows && plan_cut(ref, plan, n);
  const std::vector<LaunchGroup> groups = launch_groups(plan, rows);
  const size_t lds_max = (size_t)max_lds_bytes();
  for (const LaunchGroup& g : groups) {
    const size_t lds = g.chains ? skew_lds_bytes(plan->strip, g.chains, g.bands, g.max_band)
                                : plain_lds_bytes(plan->dtype, plan->strip, g.max_m);
    SDTW_REQUIRE(lds <= lds_max, "sdtw_align_batch: %zu bytes of LDS needed, %zu available", lds,
                 lds_max);
  }
  AlignArgs a{};
  a.ref = ref->data;
  a.n = n;
  a.q = q_dev;
  a.offs = plan->offs_dev;
  a.sched = plan->sched_dev;
  a.cost = cost_dev;
  a.end = end_dev;
  for (const LaunchGroup& g : groups) {
    a.order = plan->order_dev + g.first;
    a.nwork = g.count;
    a.max_m = g.max_m;
    a.max_band = g.max_band;
    a.band_target = g.band_target;
    int rc;
    if (g.chains) {
      const int groups_per_cu = std::max(plan->waves_per_cu / g.bands, 1);
      const int blocks = (int)std::min<int64_t>((int64_t)plan->cus * groups_per_cu, g.count);
      a.lds_bytes = spread_lds(skew_lds_bytes(plan->strip, g.chains, g.bands, g.max_band),
                               blocks, groups_per_cu, plan->cus);
      rc = check_hip(launch_align_skew(plan->dtype, plan->strip, g.chains, g.bands, blocks, a, st),
                     "sdtw_align_batch: launch");
    } else {
      rc = check_hip(launch_align_plain(plan->dtype, plan->strip, a, st),
                     "sdtw_align_batch: launch");
    }
    if (rc) return rc;
  }
  if (rows && plan->nlong < plan->nq) {
    RowsArgs ra = plan->cut;
    ra.ref = ref->data;
    ra.n = n;
    ra.q = q_dev;
    ra.offs = plan->offs_dev;
    ra.packs = plan->packs_dev[plan->cut_lay];
    rows_scratch(ra, plan->scratch);
    ra.cost = cost_dev;
    ra.end = end_dev;
    return check_hip(launch_align_rows(plan->dtype, ra, st, false), "sdtw_align_batch: launch");
  }
  return SDTW_OK;
}

int sdtw_align_one(sdtw_ref ref, const void* q_dev, int32_t M, void* cost_dev, int32_t* end_dev,
                   void* stream) {
  SDTW_REQUIRE(ref, "sdtw_align_one: null reference");
  SDTW_REQUIRE(q_dev && cost_dev && end_dev, "sdtw_align_one: null device pointer");
  SDTW_REQUIRE(M >= 1 && M <= SDTW_MAX_QUERY, "sdtw_align_one: M=%d outside [1, %d]", M,
               SDTW_MAX_QUERY);
  if (int rc = require_device(ref->device, "sdtw_align_one")) return rc;
  AlignArgs a{};
  a.ref = ref->data;
  a.n = ref->n;
  a.q = q_dev;
  a.offs = nullptr;
  a.order = nullptr;
  a.nwork = 1;
  a.max_m = M;
  a.single_m = M;
  a.cost = cost_dev;
  a.end = end_dev;
  return check_hip(launch_align_plain(ref->dtype, 16, a, (hipStream_t)stream),
                   "sdtw_align_one: launch");
}

// One read of m <= kRowsMaxM rows, or a chunk of them that extends `row`,
// spread over the device: the row-lane kernel with one read to a wave, unless
// the reference has so many columns without variation that the wave that walks
// them takes longer than the row scan.  250 rows against equal values: 1.74 ms
// walked and 0.54 scanned on 59,796 columns, 25.7 and 0.75 on 1,000,000; a
// fiftieth of 1,000,000 equal: 0.69 and 0.75.  Behind it on long references
// stands the row scan for segments that stay unsettled for another reason; its
// kernels end at once otherwise (about 8 us, too much for a call on a shorter
// reference).
struct OneRead {
  bool fits = false;  // the row scan is not faster
  RowsArgs rows{};
  int cols = 0;       // of the row scan, 0: none
  int64_t words = 0;  // scratch of the row-lane kernel (the row scan's follows)
};
constexpr int64_t kScanBehind = int64_t(1) << 20;  // columns
// Segments left to their neighbours: a wave that walks 16 of 250 rows x 9,999,990
// columns takes as long as the row scan, 2.5 and 2.1 ms.
constexpr int32_t kMostUnsettled = 16;

static int64_t one_words(const OneRead& o, int64_t n, int32_t m) {
  return o.words + (o.cols ? wide_scratch_words(n, m, o.cols) : 0) + 1;
}
static OneRead one_read(sdtw_ref ref, const void* q, int32_t m, bool stream, int64_t max_words,
                        void* cost, int32_t* end, int32_t held = 0) {
  OneRead o;
  RowsArgs& a = o.rows;
  a.ref = ref->data;
  a.n = ref->n;
  a.q = q;
  a.cus = std::max(cu_count(), 1);
  a.single_m = m;
  RowLayout lay = one_layout(m, &a.pack);
  lay.max_held = held;
  if (ref->n >= kScanBehind) {
    o.cols = wide_pick_cols(ref->n, ref->device);
    max_words -= wide_scratch_words(ref->n, m, o.cols) + 1;
  }
  // cycles: a step of one wave on a SIMD per four columns, and the row scan
  // (fitted to 59,796 to 9,999,990 columns x 40 to 400 rows, within a quarter)
  const double walk = 0.25 * (double)ref->flat *
                      RowCost{true, false, stream}.step(lay.classes[0].rows_per_lane, 1.0);
  const double scan = 60000.0 + m * (5000.0 + 0.0015 * (double)ref->n);
  // (a cut of three times the scan's time: the scratch allows too few segments)
  o.fits = rows_best_cut(a, lay, true, ref->n, false, stream, max_words, &o.words) <= 3.0 * scan &&
           walk <= scan;
  if (!a.nhalo) o.cols = 0;
  a.cost = cost;
  a.end = end;
  a.row_min_at = ref->n_pad - 1;
  a.far = ref->flat == 0;
  return o;
}
static hipError_t launch_one(sdtw_ref ref, OneRead& o, uint64_t* scratch, hipStream_t st,
                             uint32_t* row = nullptr, int32_t rows_in = 0) {
  RowsArgs& a = o.rows;
  rows_scratch(a, scratch);
  a.item.acc = row;
  a.item.m = a.single_m;
  a.item.m_old = rows_in;
  const bool stream = row != nullptr;
  if (!o.cols) return launch_align_rows(SDTW_I16, a, st, stream);
  uint64_t* const scan = scratch + o.words;
  uint32_t* const gate = (uint32_t*)(scan + wide_scratch_words(ref->n, a.single_m, o.cols));
  a.skip = gate;
  hipError_t e = launch_align_rows(SDTW_I16, a, st, stream, kRowsHalo);
  if (e == hipSuccess)
    e = launch_wide_gate(a.fail, a.nwaves, kMostUnsettled, gate, ref->n, a.single_m, o.cols, scan,
                         st, rows_in > 0 ? row : nullptr);
  if (e == hipSuccess) e = launch_align_rows(SDTW_I16, a, st, stream, kRowsSweep);
  if (e == hipSuccess)
    e = launch_align_wide(ref->data, ref->n, (const int16_t*)a.q, a.single_m, o.cols, scan,
                          (int32_t*)a.cost, a.end, st, row, rows_in > 0, a.row_min_at, gate);
  return e;
}

int sdtw_align_one_wide(sdtw_ref ref, const void* q_dev, int32_t M, int cols, void* cost_dev,
                        int32_t* end_dev, void* stream) try {
  SDTW_REQUIRE(ref, "sdtw_align_one_wide: null reference");
  SDTW_REQUIRE(q_dev && cost_dev && end_dev, "sdtw_align_one_wide: null device pointer");
  SDTW_REQUIRE(ref->dtype == SDTW_I16, "sdtw_align_one_wide: int16 references only");
  SDTW_REQUIRE(M >= 1 && M <= SDTW_MAX_QUERY, "sdtw_align_one_wide: M=%d outside [1, %d]", M,
               SDTW_MAX_QUERY);
  SDTW_REQUIRE(cols == 0 || cols == 8 || cols == 16 || cols == 32 || cols == 64,
               "sdtw_align_one_wide: cols=%d not in {0, 8, 16, 32, 64}", cols);
  if (int rc = require_device(ref->device, "sdtw_align_one_wide")) return rc;
  const bool may_rows = cols == 0 && M <= kRowsMaxM;
  if (cols == 0) cols = wide_pick_cols(ref->n, ref->device);
  SDTW_REQUIRE(wide_tiles(ref->n, cols) <= (int64_t)INT32_MAX,
               "sdtw_align_one_wide: reference too long for %d columns per thread", cols);
  const int dev = ref->device;
  DescRing& ring = g_ring[dev >= 0 && dev < kMaxDevices ? dev : 0];
  std::lock_guard<std::mutex> g(ring.mu);
  DescSlot* pick = nullptr;
  int rc = acquire_slot(ring, 1, &pick, "sdtw_align_one_wide");
  if (rc) return rc;
  DescSlot& sl = *pick;
  OneRead one;
  if (may_rows) one = one_read(ref, q_dev, M, false, INT64_MAX, cost_dev, end_dev);
  const bool rows = one.fits;
  rc = ensure_part(sl, rows ? one_words(one, ref->n, M) : wide_scratch_words(ref->n, M, cols));
  if (rc) return rc;
  auto tok = std::make_shared<CallToken>();
  tok->ev = event_get();
  if (!tok->ev) return set_error(SDTW_EDEVICE, "sdtw_align_one_wide: event creation failed");
  hipStream_t st = (hipStream_t)stream;
  if (rows) {
    rc = check_hip(launch_one(ref, one, sl.part, st), "sdtw_align_one_wide: launch");
  } else {
    rc = check_hip(launch_align_wide(ref->data, ref->n, (const int16_t*)q_dev, M, cols, sl.part,
                                     (int32_t*)cost_dev, end_dev, st),
                   "sdtw_align_one_wide: launch");
  }
  const int rc_ev = check_hip(hipEventRecord(tok->ev, st), "sdtw_align_one_wide: record");
  if (!rc_ev) sl.last = tok;
  return rc ? rc : rc_ev;
} SDTW_NO_MEMORY("sdtw_align_one_wide")

int sdtw_align_one_wide_noalloc(sdtw_ref ref, const void* q_dev, int32_t M, int cols,
                                void* cost_dev, int32_t* end_dev, void* stream) {
  SDTW_REQUIRE(ref, "sdtw_align_one_wide_noalloc: null reference");
  SDTW_REQUIRE(q_dev && cost_dev && end_dev, "sdtw_align_one_wide_noalloc: null device pointer");
  SDTW_REQUIRE(ref->dtype == SDTW_I16, "sdtw_align_one_wide_noalloc: int16 references only");
  SDTW_REQUIRE(M >= 1 && M <= SDTW_MAX_QUERY, "sdtw_align_one_wide_noalloc: M=%d outside [1, %d]",
               M, SDTW_MAX_QUERY);
  SDTW_REQUIRE(cols == 0 || cols == 8 || cols == 16 || cols == 32 || cols == 64,
               "sdtw_align_one_wide_noalloc: cols=%d not in {0, 8, 16, 32, 64}", cols);
  if (int rc = require_device(ref->device, "sdtw_align_one_wide_noalloc")) return rc;
  const bool rows = cols == 0 && M <= kRowsMaxM;
  if (cols == 0) cols = wide_pick_cols(ref->n, ref->device);
  SDTW_REQUIRE(wide_tiles(ref->n, cols) <= (int64_t)INT32_MAX,
               "sdtw_align_one_wide_noalloc: reference too long for %d columns per thread", cols);
  const int64_t need = wide_scratch_words(ref->n, M, cols);
  SDTW_REQUIRE(need <= wide_noalloc_words(),
               "sdtw_align_one_wide_noalloc: %d rows x %lld columns at %d columns per thread "
               "need %lld words of scratch, the fixed array holds %lld", M, (long long)ref->n,
               cols, (long long)need, (long long)wide_noalloc_words());
  uint64_t* scratch = nullptr;
  int rc = check_hip(wide_noalloc_scratch(ref->device, &scratch),
                     "sdtw_align_one_wide_noalloc: scratch address");
  if (rc) return rc;
  if (rows) {
    OneRead one = one_read(ref, q_dev, M, false, wide_noalloc_words(), cost_dev, end_dev);
    if (one.fits)
      return check_hip(launch_one(ref, one, scratch, (hipStream_t)stream),
                       "sdtw_align_one_wide_noalloc: launch");
  }
  return check_hip(launch_align_wide(ref->data, ref->n, (const int16_t*)q_dev, M, cols, scratch,
                                     (int32_t*)cost_dev, end_dev, (hipStream_t)stream),
                   "sdtw_align_one_wide_noalloc: launch");
}

// ---------------------------------------------------------------------------
// autotuning
// ---------------------------------------------------------------------------

}  // extern "C"

namespace {
// Tuned launch shapes are remembered per (architecture and compute units,
// dtype, reference length, batch shape class); the batch shape class puts
// the number of reads, the median and the longest read length each into
// quarter-octave buckets, so batches of about the same shape (a serving
// loop's ragged batches, a workload drawn again) share a tuned shape.
struct TuneKey {
  std::string arch;
  int cus, dtype;
  int64_t n;
  int nq_b, med_b, max_b;
  bool operator<(const TuneKey& o) const {
    return std::tie(arch, cus, dtype, n, nq_b, med_b, max_b) <
           std::tie(o.arch, o.cus, o.dtype, o.n, o.nq_b, o.med_b, o.max_b);
  }
};
struct TuneVal {
  int strip, chains, bands, waves_per_cu;
  int32_t band_rows;
};

std::mutex g_tune_mu;
std::map<TuneKey, TuneVal> g_tuned;  // best configuration per key
bool g_tune_file_read = false;

int quarter_octave(int64_t v) { return (int)lround(4.0 * log2((double)std::max<int64_t>(v, 1))); }

std::string device_arch(int device) {
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return "unknown";
  std::string a = prop.gcnArchName;
  for (char& c : a)
    if (c == ' ') c = '_';
  return a;
}

// (a plan without reads over kRowsMaxM rows keeps to the buckets below that of
// kRowsMaxM, so that it shares none with plans whose long reads were timed)
TuneKey tune_key(const sdtw_plan_s* p, int64_t n) {
  int max_b = quarter_octave(p->max_m);
  if (p->nlong == 0) max_b = std::min(max_b, quarter_octave(kRowsMaxM) - 1);
  return {device_arch(p->device), p->cus, p->dtype, n, quarter_octave(p->nq),
          quarter_octave(p->sorted_m[p->sorted_m.size() / 2]), max_b};
}

// Optional persistence: SDTW_TUNE_CACHE names a text file with one tuned
// shape per line ("arch cus dtype n nq_b med_b max_b strip chains bands
// waves_per_cu band_rows"), read once per process and rewritten after every
// autotune.  Unset or empty: the cache lives in this process only.
const char* tune_file() {
  const char* f = getenv("SDTW_TUNE_CACHE");
  return (f && *f) ? f : nullptr;
}

void tune_file_read_locked() {
  if (g_tune_file_read) return;
  g_tune_file_read = true;
  const char* path = tune_file();
  if (!path) return;
  FILE* f = fopen(path, "r");
  if (!f) return;
  char arch[256];
  TuneKey k;
  TuneVal v;
  long long n;
  while (fscanf(f, "%255s %d %d %lld %d %d %d %d %d %d %d %d", arch, &k.cus, &k.dtype, &n,
                &k.nq_b, &k.med_b, &k.max_b, &v.strip, &v.chains, &v.bands, &v.waves_per_cu,
                &v.band_rows) == 12) {
    k.arch = arch;
    k.n = n;
    if (valid_skew_config(v.strip, v.chains, v.bands) && v.waves_per_cu >= v.bands &&
        v.waves_per_cu <= 32 && v.waves_per_cu % v.bands == 0)
      g_tuned[k] = v;
  }
  fclose(f);
}

void tune_file_write_locked() {
  const char* path = tune_file();
  if (!path) return;
  const std::string tmp = std::string(path) + ".tmp";
  FILE* f = fopen(tmp.c_str(), "w");
  if (!f) return;
  for (const auto& kv : g_tuned) {
    const TuneKey& k = kv.first;
    const TuneVal& v = kv.second;
    fprintf(f, "%s %d %d %lld %d %d %d %d %d %d %d %d\n", k.arch.c_str(), k.cus, k.dtype,
            (long long)k.n, k.nq_b, k.med_b, k.max_b, v.strip, v.chains, v.bands,
            v.waves_per_cu, (int)v.band_rows);
  }
  if (fclose(f) == 0) rename(tmp.c_str(), path);
}
}  // namespace

extern "C" {

int sdtw_plan_autotune(sdtw_ref ref, sdtw_plan plan, const void* q_dev, void* cost_dev,
                       int32_t* end_dev, int64_t max_columns, void* stream) try {
  SDTW_REQUIRE(ref && plan, "sdtw_plan_autotune: null reference or plan");
  SDTW_REQUIRE(q_dev && cost_dev && end_dev, "sdtw_plan_autotune: null device pointer");
  SDTW_REQUIRE(ref->dtype == plan->dtype,
               "sdtw_plan_autotune: reference dtype %d != plan dtype %d", ref->dtype,
               plan->dtype);
  SDTW_REQUIRE(max_columns >= 0, "sdtw_plan_autotune: negative max_columns");
  SDTW_REQUIRE(ref->device == plan->device,
               "sdtw_plan_autotune: reference and plan on devices %d, %d", ref->device,
               plan->device);
  if (int rc = require_device(ref->device, "sdtw_plan_autotune")) return rc;
  hipStream_t st = (hipStream_t)stream;
  const int64_t n = max_columns ? std::min<int64_t>(ref->n, max_columns) : ref->n;
  // candidates: every strip / chains / bands the kernel is built for with
  // strip >= 16 and at most 2 chains, each at the resident waves per CU its
  // LDS allows and at half that
  // and, with 3 or 4 bands, targets of a half and a third of the median read
  // (equal band heights for reads of different lengths)
  // (the row-lane kernel takes reads of up to kRowsMaxM rows and has no shape to
  // tune: without longer reads there is nothing to time)
  plan->rows = true;
  const bool nothing = plan->nlong == 0 && plan_cut(ref, plan, n);
  std::vector<TuneVal> cand;
  const int32_t median_m = plan->sorted_m[plan->sorted_m.size() / 2];
  for (int strip : {16, 32})
    for (int chains : {1, 2})
      for (int bands : {1, 2, 3, 4}) {
        if (nothing) continue;
        if (!valid_skew_config(strip, chains, bands)) continue;
        if (bands > 1 && plan->max_m < bands * skew_min_m(chains)) continue;
        std::vector<int32_t> targets = {0};
        if (bands > 2)
          for (int32_t t : {(median_m + 1) / 2, (median_m + 2) / 3})
            if (t >= skew_min_m(chains)) targets.push_back(t);
        for (int32_t target : targets) {
          const int band_rows = std::max(skew_band_rows(plan->max_m, chains, bands, target),
                                         skew_min_m(chains));
          const int w = skew_waves_per_cu(strip, chains, bands, band_rows);
          cand.push_back({strip, chains, bands, w, target});
          if (w / 2 >= bands && (w / 2) % bands == 0)
            cand.push_back({strip, chains, bands, w / 2, target});
        }
      }
  std::vector<float> cand_ms(cand.size(), 0.f);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return set_error(SDTW_EDEVICE, "sdtw_plan_autotune: event creation failed");
  }
  const TuneVal keep = {plan->strip, plan->chains, plan->bands, plan->waves_per_cu,
                        plan->band_rows};
  TuneVal best = keep;
  int rc = SDTW_OK;
  // two passes over the candidates, the second in reverse order, each
  // candidate timed once per pass after a warm-up launch, keeping its faster
  // time: the first pass also brings the clock up (the first launches of a
  // cold device run slower), a single timing can misorder shapes a few
  // percent apart, and a clock that drifts during the passes favours no
  // position in the list
  for (int pass = 0; pass < 2 && !rc; ++pass) {
    for (size_t j = 0; j < cand.size(); ++j) {
      const size_t i = pass == 0 ? j : cand.size() - 1 - j;
      const TuneVal& c = cand[i];
      plan->strip = c.strip;
      plan->chains = c.chains;
      plan->bands = c.bands;
      plan->waves_per_cu = c.waves_per_cu;
      plan->band_rows = c.band_rows;
      rc = align_batch_impl(ref, plan, q_dev, cost_dev, end_dev, st, n);  // warm-up
      if (!rc) rc = check_hip(hipEventRecord(e0, st), "sdtw_plan_autotune: record");
      if (!rc) rc = align_batch_impl(ref, plan, q_dev, cost_dev, end_dev, st, n);
      if (!rc) rc = check_hip(hipEventRecord(e1, st), "sdtw_plan_autotune: record");
      if (!rc) rc = check_hip(hipEventSynchronize(e1), "sdtw_plan_autotune: wait");
      float ms = 0.f;
      if (!rc) rc = check_hip(hipEventElapsedTime(&ms, e0, e1), "sdtw_plan_autotune: time");
      if (rc) break;
      if (cand_ms[i] == 0.f || ms < cand_ms[i]) cand_ms[i] = ms;
    }
  }
  float best_ms = 0.f;
  for (size_t i = 0; i < cand.size() && !rc; ++i) {
    if (best_ms == 0.f || cand_ms[i] < best_ms) {
      best_ms = cand_ms[i];
      best = cand[i];
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  plan->strip = best.strip;
  plan->chains = best.chains;
  plan->bands = best.bands;
  plan->waves_per_cu = best.waves_per_cu;
  plan->band_rows = best.band_rows;
  if (rc) return rc;
  const TuneKey key = tune_key(plan, ref->n);
  std::lock_guard<std::mutex> g(g_tune_mu);
  tune_file_read_locked();
  // what was not timed replaces nothing
  if (!cand.empty())
    g_tuned[key] = best;
  else if (!g_tuned.emplace(key, best).second)
    return SDTW_OK;
  tune_file_write_locked();
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_plan_autotune")

int sdtw_plan_use_tuned(sdtw_ref ref, sdtw_plan plan, int* found) try {
  SDTW_REQUIRE(ref && plan, "sdtw_plan_use_tuned: null reference or plan");
  const TuneKey key = tune_key(plan, ref->n);
  std::lock_guard<std::mutex> g(g_tune_mu);
  tune_file_read_locked();
  auto it = g_tuned.find(key);
  if (found) *found = it != g_tuned.end();
  if (it != g_tuned.end()) {
    plan->strip = it->second.strip;
    plan->chains = it->second.chains;
    plan->bands = it->second.bands;
    plan->waves_per_cu = it->second.waves_per_cu;
    plan->band_rows = it->second.band_rows;
    plan->rows = true;
  }
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_plan_use_tuned")

// ---------------------------------------------------------------------------
// streaming extension
// ---------------------------------------------------------------------------

int sdtw_set_row_budget(int64_t bytes) {
  SDTW_REQUIRE(bytes >= 0, "sdtw_set_row_budget: negative budget");
  RowPool* pl = pool_for(current_device());
  SDTW_REQUIRE(pl, "sdtw_set_row_budget: no current device");
  std::lock_guard<std::mutex> g(pl->mu);
  pl->budget = bytes;
  return SDTW_OK;
}

int sdtw_row_pool_trim(void) {
  const int dev = current_device();
  RowPool* pl = pool_for(dev);
  SDTW_REQUIRE(pl, "sdtw_row_pool_trim: no current device");
  std::lock_guard<std::mutex> g(pl->mu);
  hipError_t first = hipSuccess;
  for (auto& kv : pl->free_rows) {
    for (void* row : kv.second) {
      const hipError_t e = hipFree(row);
      if (first == hipSuccess) first = e;
      pl->cached -= (int64_t)kv.first;
    }
  }
  pl->free_rows.clear();
  return check_hip(first, "sdtw_row_pool_trim");
}

int sdtw_row_budget_info(int64_t* budget, int64_t* in_use, int64_t* cached) {
  RowPool* pl = pool_for(current_device());
  SDTW_REQUIRE(pl, "sdtw_row_budget_info: no current device");
  std::lock_guard<std::mutex> g(pl->mu);
  if (budget) *budget = pl->budget;
  if (in_use) *in_use = pl->in_use;
  if (cached) *cached = pl->cached;
  return SDTW_OK;
}

int sdtw_stream_open(sdtw_ref ref, sdtw_stream* out) try {
  SDTW_REQUIRE(ref && out, "sdtw_stream_open: null pointer");
  if (int rc = require_device(ref->device, "sdtw_stream_open")) return rc;
  RowPool* pl = pool_for(ref->device);
  SDTW_REQUIRE(pl, "sdtw_stream_open: bad device");
  const size_t bytes = sizeof(uint32_t) * (size_t)ref->n_pad;
  void* row = nullptr;
  {
    std::lock_guard<std::mutex> g(pl->mu);
    if (pl->in_use + (int64_t)bytes > pl->budget)
      return set_error(SDTW_EBUDGET, "sdtw_stream_open: %zu more bytes exceed the row budget "
                       "(%lld in use of %lld)", bytes, (long long)pl->in_use,
                       (long long)pl->budget);
    auto it = pl->free_rows.find(bytes);
    if (it != pl->free_rows.end() && !it->second.empty()) {
      row = it->second.back();
      it->second.pop_back();
      pl->cached -= (int64_t)bytes;
    } else {
      // make room in the budget by releasing cached rows of other sizes
      for (auto& kv : pl->free_rows) {
        while (pl->in_use + pl->cached + (int64_t)bytes > pl->budget && !kv.second.empty()) {
          (void)hipFree(kv.second.back());
          kv.second.pop_back();
          pl->cached -= (int64_t)kv.first;
        }
      }
      if (hipMalloc(&row, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(SDTW_ENOMEM, "sdtw_stream_open: device allocation of %zu bytes", bytes);
      }
    }
    pl->in_use += (int64_t)bytes;
  }
  sdtw_stream_s* s = new (std::nothrow) sdtw_stream_s();
  if (!s) {
    std::lock_guard<std::mutex> g(pl->mu);
    pl->free_rows[bytes].push_back(row);
    pl->in_use -= (int64_t)bytes;
    pl->cached += (int64_t)bytes;
    return set_error(SDTW_ENOMEM, "sdtw_stream_open: host allocation");
  }
  s->device = ref->device;
  s->ref = ref;
  s->row = (uint32_t*)row;
  s->bytes = bytes;
  s->rows = 0;
  ref->open_streams++;
  *out = s;
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_stream_open")

int sdtw_stream_info(sdtw_stream s, int32_t* rows, int64_t* n) {
  SDTW_REQUIRE(s, "sdtw_stream_info: null stream");
  if (rows) *rows = s->rows;
  if (n) *n = s->ref->n;
  return SDTW_OK;
}

int sdtw_stream_close(sdtw_stream s) try {
  SDTW_REQUIRE(s, "sdtw_stream_close: null stream");
  // the row may still be read or written by enqueued work
  if (s->last && s->last->ev) {
    int rc = check_hip(hipEventSynchronize(s->last->ev), "sdtw_stream_close: wait");
    if (rc) return rc;
  }
  RowPool* pl = pool_for(s->device);
  {
    std::lock_guard<std::mutex> g(pl->mu);
    pl->free_rows[s->bytes].push_back(s->row);
    pl->in_use -= (int64_t)s->bytes;
    pl->cached += (int64_t)s->bytes;
  }
  s->ref->open_streams--;
  delete s;
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_stream_close")

int sdtw_stream_copy_row(sdtw_stream s, void* dst_dev, void* stream) {
  SDTW_REQUIRE(s && dst_dev, "sdtw_stream_copy_row: null pointer");
  if (int rc = require_device(s->device, "sdtw_stream_copy_row")) return rc;
  if (s->rows == 0)
    return set_error(SDTW_ESTATE, "sdtw_stream_copy_row: the stream has no rows yet");
  return check_hip(hipMemcpyAsync(dst_dev, s->row, sizeof(uint32_t) * (size_t)s->ref->n,
                                  hipMemcpyDeviceToDevice, (hipStream_t)stream),
                   "sdtw_stream_copy_row");
}

int sdtw_stream_set_config(sdtw_ref ref, int strip, int bands) {
  SDTW_REQUIRE(strip == 0 || strip == 16 || strip == 32,
               "sdtw_stream_set_config: strip %d not in {0,16,32}", strip);
  SDTW_REQUIRE(bands >= 0 && bands <= 4, "sdtw_stream_set_config: bands %d not in {0,1,2,3,4}",
               bands);
  if (ref) {
    ref->stream_strip.store(strip);
    ref->stream_bands.store(bands);
  } else {
    g_stream_strip.store(strip);
    g_stream_bands.store(bands);
  }
  return SDTW_OK;
}

int sdtw_stream_extend(const sdtw_stream* streams, int32_t ns, const void* chunk_dev,
                       const int64_t* chunk_offsets_host, void* cost_dev, int32_t* end_dev,
                       void* stream) try {
  SDTW_REQUIRE(streams && chunk_dev && chunk_offsets_host && cost_dev && end_dev,
               "sdtw_stream_extend: null pointer");
  SDTW_REQUIRE(ns >= 1, "sdtw_stream_extend: ns=%d < 1", ns);
  SDTW_REQUIRE(streams[0], "sdtw_stream_extend: stream 0 is null");
  const sdtw_ref ref = streams[0]->ref;
  const int dtype = ref->dtype;
  if (int rc = require_device(ref->device, "sdtw_stream_extend")) return rc;
  const int32_t row_cap = dtype == SDTW_I16 ? 32767 : INT32_MAX;
  std::set<const sdtw_stream_s*> seen;
  std::vector<int32_t> order((size_t)ns);
  int32_t max_m = 0;
  for (int32_t i = 0; i < ns; ++i) {
    const sdtw_stream s = streams[i];
    SDTW_REQUIRE(s, "sdtw_stream_extend: stream %d is null", i);
    SDTW_REQUIRE(s->ref == ref, "sdtw_stream_extend: stream %d uses another reference", i);
    SDTW_REQUIRE(seen.insert(s).second, "sdtw_stream_extend: stream %d appears twice", i);
    const int64_t m = chunk_offsets_host[i + 1] - chunk_offsets_host[i];
    SDTW_REQUIRE(chunk_offsets_host[i] >= 0 && m >= 1 && m <= SDTW_MAX_QUERY,
                 "sdtw_stream_extend: chunk %d has length %lld outside [1, %d]", i,
                 (long long)m, SDTW_MAX_QUERY);
    SDTW_REQUIRE((int64_t)s->rows + m <= row_cap,
                 "sdtw_stream_extend: stream %d would exceed %d rows", i, row_cap);
    order[(size_t)i] = i;
    max_m = std::max<int32_t>(max_m, (int32_t)m);
  }
  auto len = [&](int32_t i) { return chunk_offsets_host[i + 1] - chunk_offsets_host[i]; };
  std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
    return len(a) != len(b) ? len(a) > len(b) : a < b;
  });
  // One chain per lane.  Automatic shape: more waves per chunk the fewer
  // chunks there are (a chunk's latency shrinks with its bands while the
  // device is not full): four bands up to two chunks per compute unit (two
  // workgroups of four bands fit on a CU, two waves per SIMD), two up to
  // four, then one; strip 32 for references of 2^20 columns and more (half
  // the tiles per chunk), else 16, whose workgroups need a third of strip
  // 32's LDS, so that short-reference calls find room beside long-reference
  // ones.
  constexpr int kChains = 1;
  const int cus = std::max(cu_count(), 1);
  int bands = ref->stream_bands.load();
  if (bands == 0) bands = g_stream_bands.load();
  if (bands == 0) bands = ns <= 2 * cus ? 4 : (ns <= 4 * cus ? 2 : 1);
  int kStrip = ref->stream_strip.load();
  if (kStrip == 0) kStrip = g_stream_strip.load();
  if (kStrip == 0) kStrip = ref->n >= (int64_t(1) << 20) ? 32 : 16;
  // The row-lane kernel takes chunks of up to kRowsMaxM rows, unless a launch
  // shape was set or it does not suit the reference; order[nskew ..) are its chunks.
  const bool shaped = ref->stream_bands.load() || g_stream_bands.load() ||
                      ref->stream_strip.load() || g_stream_strip.load();
  int32_t nskew = ns;
  if (!shaped)
    for (nskew = 0; nskew < ns && len(order[(size_t)nskew]) > kRowsMaxM;) ++nskew;
  if (nskew > 0 && nskew < ns) {
    double long_rows = 0.0, short_rows = 0.0;
    for (int32_t t = 0; t < ns; ++t)
      (t < nskew ? long_rows : short_rows) += (double)len(order[(size_t)t]);
    const int32_t next = (int32_t)len(order[(size_t)nskew]);
    if (!split_pays(max_m, next, long_rows, short_rows, cus)) nskew = ns;
  }
  RowsArgs ra{};
  RowLayout lay;
  int64_t words = 0;
  if (nskew < ns) {
    std::vector<std::pair<int32_t, int32_t>> chunks;
    double rows = 0.0;
    int32_t held = 0;
    for (int32_t t = nskew; t < ns; ++t) {
      chunks.emplace_back(t, (int32_t)len(order[(size_t)t]));
      rows += (double)chunks.back().second;
      held = std::max(held, streams[order[(size_t)t]]->rows);
    }
    ra.cus = cus;
    RowsArgs rb = ra;
    lay = rows_layout(chunks, false, kRowsStreamReads);
    RowLayout lay1 = rows_layout(chunks, true, kRowsStreamReads);
    lay.max_held = lay1.max_held = held;
    int64_t words1 = 0;
    double cycles = rows_best_cut(ra, lay, false, ref->n, dtype == SDTW_F32, true, kPartWords,
                                  &words);
    const double alone = rows_best_cut(rb, lay1, true, ref->n, dtype == SDTW_F32, true, kPartWords,
                                       &words1);
    if (alone < cycles) {
      lay = std::move(lay1);
      ra = rb;
      words = words1;
      cycles = alone;
    }
    if (walked_longer(ref, ref->n, ra, cycles, rows, true)) {
      nskew = ns;
      lay = RowLayout{};
    }
  }
  int32_t nbig = 0, max_band = 0;
  while (nbig < nskew && len(order[(size_t)nbig]) >= skew_min_m(kChains)) {
    max_band = std::max(max_band, skew_band_rows((int32_t)len(order[(size_t)nbig]), kChains, bands));
    ++nbig;
  }
  const size_t lds_max = (size_t)max_lds_bytes();
  SDTW_REQUIRE(nskew == 0 || (skew_lds_bytes(kStrip, kChains, bands, max_band, true) <= lds_max &&
                              plain_lds_bytes(dtype, kStrip, max_m) <= lds_max),
               "sdtw_stream_extend: chunk of %d rows needs more LDS than available", max_m);

  const int dev = ref->device;
  DescRing& ring = g_ring[dev >= 0 && dev < kMaxDevices ? dev : 0];
  std::lock_guard<std::mutex> g(ring.mu);
  DescSlot* pick = nullptr;
  int rc = acquire_slot(ring, ns, &pick, "sdtw_stream_extend");
  if (rc) return rc;
  DescSlot& sl = *pick;
  for (int32_t t = 0; t < ns; ++t) {
    const int32_t i = order[(size_t)t];
    StreamItem& it = sl.host[t];
    it.acc = streams[i]->row;
    it.q0 = chunk_offsets_host[i];
    it.m = (int32_t)len(i);
    it.m_old = streams[i]->rows;
    it.out = i;
    it.pad = 0;
  }
  const size_t npacks = lay.packs.size();
  if (npacks) {
    if (words && ensure_part(sl, words)) {  // no memory for it: one segment per pack
      (void)hipGetLastError();
      rows_best_cut(ra, lay, false, ref->n, dtype == SDTW_F32, true, 0, &words);
    }
    rows_scratch(ra, sl.part);
    std::copy(lay.packs.begin(), lay.packs.end(), sl.host_packs(ns));
    ra.ref = ref->data;
    ra.n = ref->n;
    ra.q = chunk_dev;
    ra.items = sl.dev;
    ra.packs = sl.dev_packs(ns);
    ra.cost = cost_dev;
    ra.end = end_dev;
    ra.row_min_at = ref->n_pad - 1;
    ra.far = ref->flat == 0;
  }
  auto tok = std::make_shared<CallToken>();
  tok->ev = event_get();
  if (!tok->ev) return set_error(SDTW_EDEVICE, "sdtw_stream_extend: event creation failed");
  hipStream_t st = (hipStream_t)stream;
  rc = check_hip(hipMemcpyAsync(sl.dev, sl.host,
                                sizeof(StreamItem) * (size_t)ns + sizeof(RowPack) * npacks,
                                hipMemcpyHostToDevice, st),
                 "sdtw_stream_extend: descriptors");
  AlignArgs a{};
  a.ref = ref->data;
  a.n = ref->n;
  a.q = chunk_dev;
  a.counter = sl.counter();
  a.cost = cost_dev;
  a.end = end_dev;
  a.row_min_at = ref->n_pad - 1;
  int long_blocks = 0;
  if (!rc && nbig) {
    a.items = sl.dev;
    a.nwork = nbig;
    a.max_m = (int32_t)len(order[0]);
    a.max_band = max_band;
    // No LDS reservation (spread_lds): calls in flight on other HIP streams
    // (other targets, the next batch) must find room on every CU.  Except
    // for long references while this launch and the long-reference launches
    // still running have at most one workgroup per CU between them: two
    // long-reference workgroups fit on a CU (two waves per SIMD), which pays
    // once the device is full, but with CUs idle the dispatcher would also
    // put the next batch's workgroups beside this one's, each then slower
    // than alone on a CU of its own.  Such a launch reserves enough LDS that
    // no second long-reference workgroup joins one of its CUs (short-
    // reference ones, a third of the size, still do).
    const int wpc = skew_waves_per_cu(kStrip, kChains, bands, max_band, true);
    const int blocks = (int)std::min<int64_t>((int64_t)cus * (wpc / bands), nbig);
    int64_t running = 0;
    if (kStrip == 32) {
      auto& v = ring.long_inflight;
      v.erase(std::remove_if(v.begin(), v.end(),
                             [](const std::pair<std::shared_ptr<CallToken>, int>& e) {
                               if (!e.first->ev) return true;
                               if (hipEventQuery(e.first->ev) != hipErrorNotReady) return true;
                               (void)hipGetLastError();  // "not ready" is no error here
                               return false;
                             }),
              v.end());
      for (const auto& e : v) running += e.second;
    }
    a.lds_bytes = 0;
    if (kStrip == 32 && 2 * (blocks + running) <= cus) {
      const size_t need = skew_lds_bytes(kStrip, kChains, bands, max_band, true);
      const size_t alone = ((160 * 1024 - need + 1024 + 1023) & ~(size_t)1023);
      if (alone > need && alone <= lds_max) a.lds_bytes = (int32_t)alone;
    }
    rc = check_hip(launch_align_skew(dtype, kStrip, kChains, bands, blocks, a, st, true),
                   "sdtw_stream_extend: launch");
    if (kStrip == 32) long_blocks = blocks;
  }
  if (!rc && nbig < nskew) {
    a.items = sl.dev + nbig;
    a.nwork = nskew - nbig;
    a.max_m = (int32_t)len(order[(size_t)nbig]);
    rc = check_hip(launch_align_plain(dtype, kStrip, a, st, true), "sdtw_stream_extend: launch");
  }
  if (!rc && npacks)
    rc = check_hip(launch_align_rows(dtype, ra, st, true), "sdtw_stream_extend: launch");
  // the slot is busy until this point of the stream, whatever was enqueued
  const int rc_ev = check_hip(hipEventRecord(tok->ev, st), "sdtw_stream_extend: record");
  if (!rc_ev) sl.last = tok;
  if (!rc) rc = rc_ev;
  if (rc) return rc;
  if (long_blocks) ring.long_inflight.emplace_back(tok, long_blocks);
  for (int32_t i = 0; i < ns; ++i) {
    streams[i]->rows += (int32_t)len(i);
    streams[i]->last = tok;
  }
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_stream_extend")

int sdtw_stream_extend_wide(sdtw_stream s, const void* chunk_dev, int32_t M, int cols,
                            void* cost_dev, int32_t* end_dev, void* stream) try {
  SDTW_REQUIRE(s && chunk_dev && cost_dev && end_dev, "sdtw_stream_extend_wide: null pointer");
  const sdtw_ref ref = s->ref;
  SDTW_REQUIRE(ref->dtype == SDTW_I16, "sdtw_stream_extend_wide: int16 references only");
  SDTW_REQUIRE(M >= 1 && (int64_t)s->rows + M <= SDTW_MAX_QUERY,
               "sdtw_stream_extend_wide: %d rows folded in plus a chunk of %d exceed %d", s->rows,
               M, SDTW_MAX_QUERY);
  SDTW_REQUIRE(cols == 0 || cols == 8 || cols == 16 || cols == 32 || cols == 64,
               "sdtw_stream_extend_wide: cols=%d not in {0, 8, 16, 32, 64}", cols);
  if (int rc = require_device(ref->device, "sdtw_stream_extend_wide")) return rc;
  const bool may_rows = cols == 0 && M <= kRowsMaxM;
  if (cols == 0) cols = wide_pick_cols(ref->n, ref->device);
  SDTW_REQUIRE(wide_tiles(ref->n, cols) <= (int64_t)INT32_MAX,
               "sdtw_stream_extend_wide: reference too long for %d columns per thread", cols);
  const int dev = ref->device;
  DescRing& ring = g_ring[dev >= 0 && dev < kMaxDevices ? dev : 0];
  std::lock_guard<std::mutex> g(ring.mu);
  DescSlot* pick = nullptr;
  int rc = acquire_slot(ring, 1, &pick, "sdtw_stream_extend_wide");
  if (rc) return rc;
  DescSlot& sl = *pick;
  OneRead one;
  if (may_rows) one = one_read(ref, chunk_dev, M, true, INT64_MAX, cost_dev, end_dev, s->rows);
  const bool rows = one.fits;
  rc = ensure_part(sl, rows ? one_words(one, ref->n, M) : wide_scratch_words(ref->n, M, cols));
  if (rc) return rc;
  auto tok = std::make_shared<CallToken>();
  tok->ev = event_get();
  if (!tok->ev) return set_error(SDTW_EDEVICE, "sdtw_stream_extend_wide: event creation failed");
  hipStream_t st = (hipStream_t)stream;
  if (rows) {
    rc = check_hip(launch_one(ref, one, sl.part, st, s->row, s->rows),
                   "sdtw_stream_extend_wide: launch");
  } else {
    rc = check_hip(launch_align_wide(ref->data, ref->n, (const int16_t*)chunk_dev, M, cols,
                                     sl.part, (int32_t*)cost_dev, end_dev, st, s->row,
                                     s->rows > 0, ref->n_pad - 1),
                   "sdtw_stream_extend_wide: launch");
  }
  const int rc_ev = check_hip(hipEventRecord(tok->ev, st), "sdtw_stream_extend_wide: record");
  if (!rc_ev) sl.last = tok;
  if (!rc) rc = rc_ev;
  if (rc) return rc;
  s->rows += M;
  s->last = tok;
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_stream_extend_wide")

int sdtw_stream_best_two(const sdtw_stream* streams, int32_t ns, int32_t window,
                         void* best_cost_dev, int32_t* best_end_dev, void* second_cost_dev,
                         int32_t* second_end_dev, void* stream) try {
  SDTW_REQUIRE(streams && best_cost_dev && best_end_dev && second_cost_dev && second_end_dev,
               "sdtw_stream_best_two: null pointer");
  SDTW_REQUIRE(ns >= 1, "sdtw_stream_best_two: ns=%d < 1", ns);
  SDTW_REQUIRE(window >= 0, "sdtw_stream_best_two: negative window");
  SDTW_REQUIRE(streams[0], "sdtw_stream_best_two: stream 0 is null");
  const sdtw_ref ref = streams[0]->ref;
  if (int rc = require_device(ref->device, "sdtw_stream_best_two")) return rc;
  for (int32_t i = 0; i < ns; ++i) {
    SDTW_REQUIRE(streams[i], "sdtw_stream_best_two: stream %d is null", i);
    SDTW_REQUIRE(streams[i]->ref == ref, "sdtw_stream_best_two: stream %d uses another reference",
                 i);
    if (streams[i]->rows == 0)
      return set_error(SDTW_ESTATE, "sdtw_stream_best_two: stream %d has no rows yet", i);
  }
  const int dev = ref->device;
  DescRing& ring = g_ring[dev >= 0 && dev < kMaxDevices ? dev : 0];
  std::lock_guard<std::mutex> g(ring.mu);
  DescSlot* pick = nullptr;
  int rc = acquire_slot(ring, ns, &pick, "sdtw_stream_best_two");
  if (rc) return rc;
  DescSlot& sl = *pick;
  const int64_t nseg = best_two_segments(ref->n);
  SDTW_REQUIRE((int64_t)ns * nseg <= (int64_t)INT32_MAX,
               "sdtw_stream_best_two: %d rows of %lld columns exceed one launch", ns,
               (long long)ref->n);
  rc = ensure_part(sl, (int64_t)ns * nseg);
  if (rc) return rc;
  for (int32_t i = 0; i < ns; ++i) {
    StreamItem& it = sl.host[i];
    it = StreamItem{};
    it.acc = streams[i]->row;
    it.out = i;
  }
  auto tok = std::make_shared<CallToken>();
  tok->ev = event_get();
  if (!tok->ev) return set_error(SDTW_EDEVICE, "sdtw_stream_best_two: event creation failed");
  hipStream_t st = (hipStream_t)stream;
  rc = check_hip(hipMemcpyAsync(sl.dev, sl.host, sizeof(StreamItem) * (size_t)ns,
                                hipMemcpyHostToDevice, st),
                 "sdtw_stream_best_two: descriptors");
  if (!rc)
    rc = check_hip(launch_best_two(ref->dtype, sl.dev, ns, ref->n, window, sl.part, best_cost_dev,
                                   best_end_dev, second_cost_dev, second_end_dev, st),
                   "sdtw_stream_best_two: launch");
  const int rc_ev = check_hip(hipEventRecord(tok->ev, st), "sdtw_stream_best_two: record");
  if (!rc_ev) sl.last = tok;
  if (!rc) rc = rc_ev;
  if (rc) return rc;
  for (int32_t i = 0; i < ns; ++i) streams[i]->last = tok;  // close waits for the read
  return SDTW_OK;
} SDTW_NO_MEMORY("sdtw_stream_best_two")

}  // extern "C"

