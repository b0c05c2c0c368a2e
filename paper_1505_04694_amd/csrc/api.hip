// C ABI and host-side phase drivers: round loops, colour-class sequencing,
// commit points, compaction and store growth.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <initializer_list>
#include <cstdio>
#include <cstring>
#include <map>
#include <unordered_map>
#include <mutex>
#include <new>
#include <thread>
#include <string>
#include <vector>

#include "../../include/pm.h"
#include "kern.hpp"
#include "blocks.hpp"

using namespace pm;

namespace {

template <class T>
struct DBuf {
  T* p = nullptr;
  size_t n = 0;
};

}  // namespace

// per-kernel HIP-event timing
struct Prof {
  uint32_t mask = 0;
  struct Rec {
    int k;
    hipEvent_t a, b;
    int64_t units;
  };
  std::vector<hipEvent_t> pool;
  std::vector<Rec> open;
  double ms[PM_K_COUNT] = {};
  int64_t launches[PM_K_COUNT] = {};
  int64_t units[PM_K_COUNT] = {};
};

struct pm_mesh {
  hipStream_t s = nullptr;
  hipStream_t cap_s = nullptr;  // private stream that graph captures are recorded on
  // device-driven rounds: instantiated graphs, by the bytes of their launch arguments
  std::vector<std::pair<std::string, hipGraphExec_t>> dr_graphs;
  int dev = 0;                // device current at creation
  double* scratch = nullptr;  // that device's copy of the no-allocation scratch array
  Prof prof;
  Store st;
  uint64_t seed = 0;
  double slack = 2.0;
  std::string err;
  int* ctr = nullptr;   // device counters
  int* hctr = nullptr;  // pinned mirror
  double* hq = nullptr; // pinned doubles
  int* haux = nullptr;   // pinned ints for small read-backs (upper half: staged uploads)
  Mail mail;             // the pinned block's
  hipEvent_t up_ev = nullptr;  // the last staged upload's copy
  // scratch
  DBuf<int> listA, listB, jpU0, jpU1, cls, vt0, vt1, vt2, tt0, tt1, tt2, partial, mid;
  DBuf<uint8_t> nxt, u8tmp;
  DBuf<Met> emet;   // smoothing: per-element mean tensors
  DBuf<VRec> vr;    // coarsening and swapping: vertex records
  DBuf<int> sflag, ctab, ctabs, spart;  // ordered selection and stable class lists
  DBuf<int> stage;       // commit: fallback staging
  DBuf<int> touch, seen; // small rounds: rows rebuilt, selection stamps
  DBuf<int> jpB;         // JP: the neighbour each waiting vertex waits for
  int sel_mark = 0;      // selection stamp, one per small round
  DBuf<int4> ops;        // commit: operation records
  DBuf<uint64_t> own;    // commit: row owner keys
  DBuf<int> dirty;       // commit in vertex order: the epoch that claimed a row last
  DBuf<int> cnt;         // commit: hand-overs counted per row
  DBuf<int4> tgt;        // commit: collapse-target records
  int epoch = 0;         // commit epoch, one per class
  DBuf<JpRec> jprec;  // small colourings: predecessor records
  DBuf<double> qpart;
  DBuf<double2> upx;  // pm_mesh_update: where new coordinates and metrics are checked
  DBuf<Met> upm;
  DBuf<uint64_t> rw;  // round words (priority, active, colour) per vertex
  // mesh ranges (host mirror of Store::vbase/vused/tbase/tused)
  std::vector<int> vbase, vused, tbase, tused;
  int* ranges = nullptr;  // device: vbase[B+1], vused[B], tbase[B+1], tused[B]
  int* mdone = nullptr;   // device: per-mesh "refinement finished" flags
  DBuf<int> rtmp;         // per-mesh scratch (sums, new bases)
  pm_tuning tune{};      // kernel shapes of the current call (zeros: defaults)
  double headroom = 3.0;  // pool and staging room, a multiple of the live entries
  double stage_scale = 1.0;  // grows when the staging area ran out
  int recoveries = 0;     // row rebuilds after running out of room, in the current phase
  bool rows_ok = false;   // the rows are those of the element list (false: their last build failed)
  // Algorithm 1's loop state (pm_adapt): outer iteration, next phase, whether
  // the iteration has changed the mesh
  int ad_iter = 0, ad_phase = 1, ad_changed = 0;
  int64_t peak_bytes = 0, cur_bytes = 0;
  // caller's device memory provider (pm_options.allocator at creation), and
  // the byte count of each block it handed out
  pm_allocator va{};
  std::unordered_map<void*, size_t> va_live;
  int jp_last = 8;    // JP iterations the last colouring took
  int class_seq = 0;  // class-list calls so far (the wide-colour flag's value)
  // elements change only in coarsening, refinement and swapping: each call
  // starts a new topology version; the per-element tensors are kept for one
  uint64_t topo = 1, emet_topo = 0;
};

namespace {

// message of the last failed pm_mesh_create on this thread (no handle survives it)
thread_local std::string g_create_err;

pm_status fail(pm_mesh* m, pm_status st, const std::string& msg) {
  if (m) m->err = msg;
  return st;
}

#define HIPCHK(x)                                                                         \
  do {                                                                                    \
    hipError_t e_ = (x);                                                                  \
    if (e_ != hipSuccess)                                                                 \
      return fail(m, PM_E_DEVICE, std::string(#x) + ": " + hipGetErrorString(e_));        \
  } while (0)

#define TRY(x)                      \
  do {                              \
    pm_status r_ = (x);             \
    if (r_ != PM_OK) return r_;     \
  } while (0)

// Device blocks are recycled through a process-wide cache keyed by device,
// stream and size. A block freed on a stream is handed out again only on the
// same stream, whose order makes the reuse safe without a wait, so handles
// and phase scratch that come and go skip the driver's allocation and free
// (each a synchronising call of tens of microseconds or more). Blocks up to
// twice the request are reused; past kCacheMax cached bytes a freed block is
// returned to the driver, and a failed allocation first empties the cache.
struct CacheKey {
  int dev;
  uintptr_t stream;
  size_t bytes;
  bool operator<(const CacheKey& o) const {
    if (dev != o.dev) return dev < o.dev;
    if (stream != o.stream) return stream < o.stream;
    return bytes < o.bytes;
  }
};
constexpr size_t kCacheMax = 32ull << 30;
std::mutex g_cache_mu;
std::multimap<CacheKey, void*> g_cache_free;
std::map<void*, CacheKey> g_cache_live;
size_t g_cache_bytes = 0;

void cache_drop_all() {
  std::lock_guard<std::mutex> lk(g_cache_mu);
  for (auto& kv : g_cache_free) (void)hipFree(kv.second);
  g_cache_free.clear();
  g_cache_bytes = 0;
}

// *got: the size of the block handed out (a reused block may be larger)
hipError_t cache_get(hipStream_t s, void** p, size_t bytes, size_t* got) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  CacheKey want{dev, (uintptr_t)s, bytes};
  *got = bytes;
  {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto it = g_cache_free.lower_bound(want);
    if (it != g_cache_free.end() && it->first.dev == dev && it->first.stream == want.stream &&
        it->first.bytes <= 2 * bytes) {
      *p = it->second;
      *got = it->first.bytes;
      g_cache_bytes -= it->first.bytes;
      g_cache_live[*p] = it->first;
      g_cache_free.erase(it);
      return hipSuccess;
    }
  }
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    cache_drop_all();
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) return e;
  }
  std::lock_guard<std::mutex> lk(g_cache_mu);
  g_cache_live[*p] = want;
  return hipSuccess;
}

// returns the block's size (0 if it is not a cache block)
size_t cache_put(void* p) {
  std::unique_lock<std::mutex> lk(g_cache_mu);
  auto it = g_cache_live.find(p);
  if (it == g_cache_live.end()) return 0;
  CacheKey k = it->second;
  g_cache_live.erase(it);
  if (g_cache_bytes + k.bytes > kCacheMax) {
    lk.unlock();
    (void)hipFree(p);
    return k.bytes;
  }
  g_cache_free.insert({k, p});
  g_cache_bytes += k.bytes;
  return k.bytes;
}

template <class T>
pm_status dalloc(pm_mesh* m, T** p, size_t n) {
  *p = nullptr;
  if (n == 0) n = 1;
  if (m->va.alloc) {
    void* q = m->va.alloc(n * sizeof(T), (void*)m->s, m->va.user);
    if (!q) return fail(m, PM_E_NOMEM, "the caller's allocator refused " + std::to_string(n * sizeof(T)) + " bytes");
    m->va_live[q] = n * sizeof(T);
    *p = (T*)q;
  } else {
    size_t got = 0;
    hipError_t e = cache_get(m->s, (void**)p, n * sizeof(T), &got);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(m, PM_E_NOMEM, "device allocation of " + std::to_string(n * sizeof(T)) + " bytes failed");
    }
    m->cur_bytes += (int64_t)got;
    m->peak_bytes = std::max(m->peak_bytes, m->cur_bytes);
    return PM_OK;
  }
  m->cur_bytes += (int64_t)(n * sizeof(T));
  m->peak_bytes = std::max(m->peak_bytes, m->cur_bytes);
  return PM_OK;
}
template <class T>
void dfree(pm_mesh* m, T*& p, size_t n);
// arrays of n entries each (null before the call): all of them, or none
template <class... T>
pm_status dalloc_all(pm_mesh* m, size_t n, T*&... p) {
  pm_status r = PM_OK;
  ((r = r == PM_OK ? dalloc(m, &p, n) : r), ...);
  if (r != PM_OK) (dfree(m, p, n), ...);
  return r;
}
// the handle's pinned block: the counter mirror, 64 doubles, and kAuxInts ints
constexpr int kAuxInts = 16384;
static_assert(C_COUNT * sizeof(int) + 64 * sizeof(double) + kAuxInts * sizeof(int) < kPinnedBytes, "pinned block");
bool pinned_get(pm_mesh* m) {
  void* p = pinned_take();
  if (!p) return false;
  m->hctr = (int*)p;
  m->hq = (double*)((char*)p + C_COUNT * sizeof(int));
  m->haux = (int*)((char*)p + C_COUNT * sizeof(int) + 64 * sizeof(double));
  m->mail = mail_of(p);
  return true;
}
void pinned_put(pm_mesh* m) {
  if (!m->hctr) return;
  pinned_give(m->hctr);
  m->hctr = nullptr;
  m->hq = nullptr;
  m->haux = nullptr;
}

template <class T>
void dfree(pm_mesh* m, T*& p, size_t n) {
  if (p && m->va.release) {
    auto it = m->va_live.find((void*)p);
    if (it != m->va_live.end()) {
      m->va.release((void*)p, it->second, (void*)m->s, m->va.user);
      m->cur_bytes -= (int64_t)it->second;
      m->va_live.erase(it);
    }
  } else if (p) {
    m->cur_bytes -= (int64_t)cache_put(p);  // the block's real size
  }
  p = nullptr;
}

// grow-only scratch; contents are not preserved; zero = clear new memory.
// Freed blocks go back to the cache of this stream, where only later work of
// the same stream can take them, so a first allocation needs no wait; a
// replaced block is still waited for.
template <class T>
pm_status ensure(pm_mesh* m, DBuf<T>& b, size_t n, bool zero = false) {
  if (b.n >= n && b.p) return PM_OK;
  if (b.p) HIPCHK(hipStreamSynchronize(m->s));
  dfree(m, b.p, b.n);
  b.n = 0;
  size_t want = std::max<size_t>(n + n / 4, 64);
  TRY(dalloc(m, &b.p, want));
  b.n = want;
  if (zero) HIPCHK(hipMemsetAsync(b.p, 0, want * sizeof(T), m->s));
  return PM_OK;
}

pm_status sync(pm_mesh* m) {
  HIPCHK(hipStreamSynchronize(m->s));
  return PM_OK;
}

hipEvent_t prof_event(pm_mesh* m) {
  if (m->prof.pool.empty()) {
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  hipEvent_t e = m->prof.pool.back();
  m->prof.pool.pop_back();
  return e;
}

// time one launch (or launch sequence) of kernel k when its bit is enabled
template <class F>
void timed(pm_mesh* m, int k, int64_t units, F&& launch) {
  if (!(m->prof.mask & (1u << k))) {
    launch();
    return;
  }
  hipEvent_t a = prof_event(m), b = prof_event(m);
  if (a) (void)hipEventRecord(a, m->s);
  launch();
  if (b) (void)hipEventRecord(b, m->s);
  if (a && b) m->prof.open.push_back({k, a, b, units});
}

// fold finished event pairs into the totals (call after a stream sync)
void prof_flush(pm_mesh* m) {
  for (auto& r : m->prof.open) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, r.a, r.b) == hipSuccess) {
      m->prof.ms[r.k] += t;
      m->prof.launches[r.k] += 1;
      m->prof.units[r.k] += r.units;
    }
    m->prof.pool.push_back(r.a);
    m->prof.pool.push_back(r.b);
  }
  m->prof.open.clear();
}

// the counters a round reads back: pool tops, error bits, list length and the
// epoch of a commit that ran out of room
constexpr int kRoundCtrs = C_FAILEP + 1;

// device counters [lo, lo+n) into the pinned mirror; waits for them (and so
// for all work issued before). Timed launches need the stream synchronised.
pm_status read_ctr(pm_mesh* m, int lo, int n) {
  mail_send(m->mail, m->ctr + lo, n, m->hctr + lo, m->s);
  HIPCHK(mail_wait(m->mail, m->s));
  if (m->prof.mask) HIPCHK(hipStreamSynchronize(m->s));
  return PM_OK;
}

// fresh: the host copy of the counters was read after the last kernel
pm_status check_err(pm_mesh* m, bool fresh = false) {
  if (!fresh) TRY(read_ctr(m, C_ERR, 1));
  int e = m->hctr[C_ERR];
  if (!e) return PM_OK;
  std::string msg = "device error bits " + std::to_string(e) + ":";
  if (e & E_MESH_ID) msg += " element id out of range or repeated;";
  if (e & E_MESH_ORIENT) msg += " element not counter-clockwise (area <= 0);";
  if (e & E_MESH_MANIFOLD) msg += " non-manifold edge/vertex or inconsistent orientation;";
  if (e & E_MESH_METRIC) msg += " metric not SPD or non-finite coordinates;";
  if (e & (E_NN_POOL | E_NE_POOL)) msg += " adjacency pool exhausted;";
  if (e & E_STAGE) msg += " commit staging exhausted;";
  if (e & E_COLOURS) msg += " more than 254 colours;";
  set_int(m->ctr + C_ERR, 0, m->s);
  pm_status st = (e & (E_MESH_ID | E_MESH_ORIENT | E_MESH_MANIFOLD | E_MESH_METRIC)) ? PM_E_MESH : PM_E_NOMEM;
  if (e & E_COLOURS) st = PM_E_MESH;
  return fail(m, st, msg);
}

// Records the launches f(stream) issues into an executable graph: captured on
// the handle's private stream (a graph cannot be captured from the null
// stream, which a caller's stream may be) and later launched on the handle's
// stream, in its order. Only kernel launches are recorded (no memsets).
template <class F>
pm_status capture(pm_mesh* m, F&& f, hipGraphExec_t* out) {
  *out = nullptr;
  if (!m->cap_s) HIPCHK(hipStreamCreateWithFlags(&m->cap_s, hipStreamNonBlocking));
  HIPCHK(hipStreamBeginCapture(m->cap_s, hipStreamCaptureModeThreadLocal));
  f(m->cap_s);
  hipGraph_t g = nullptr;
  HIPCHK(hipStreamEndCapture(m->cap_s, &g));
  hipError_t e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return fail(m, PM_E_DEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
  return PM_OK;
}

// ---- store allocation -----------------------------------------------------------------------
pm_status grow_vertices(pm_mesh* m, int need) {
  Store& s = m->st;
  if (need <= s.Vcap) return PM_OK;
  int nc = std::max(need, s.Vcap + s.Vcap / 2);
  double2* xy = nullptr;
  Met* met = nullptr;
  uint8_t *tag = nullptr, *va = nullptr;
  Hdr* hdr = nullptr;
  int2* cap = nullptr;
  TRY(dalloc_all(m, nc, xy, met, tag, va, hdr, cap));
  // one launch; the old blocks go back to this stream's cache, where only later
  // work can take them
  Store to = s;
  to.xy = xy;
  to.met = met;
  to.tag = tag;
  to.valive = va;
  to.hdr = hdr;
  to.cap = cap;
  copy_vertices(s, to, nc, m->s);
  dfree(m, s.xy, s.Vcap);
  dfree(m, s.met, s.Vcap);
  dfree(m, s.tag, s.Vcap);
  dfree(m, s.valive, s.Vcap);
  dfree(m, s.hdr, s.Vcap);
  dfree(m, s.cap, s.Vcap);
  s.xy = xy;
  s.met = met;
  s.tag = tag;
  s.valive = va;
  s.hdr = hdr;
  s.cap = cap;
  s.Vcap = nc;
  return PM_OK;
}

pm_status grow_elements(pm_mesh* m, int need) {
  Store& s = m->st;
  if (need <= s.Tcap) return PM_OK;
  int nc = std::max(need, s.Tcap + s.Tcap / 2);
  Elem* tri;
  TRY(dalloc(m, &tri, nc));
  copy_elements(s, tri, nc, m->s);
  dfree(m, s.tri, s.Tcap);
  s.tri = tri;
  s.Tcap = nc;
  return PM_OK;
}

// copy the host range arrays to the device and point the store at them
pm_status upload_ranges(pm_mesh* m) {
  Store& st = m->st;
  int B = st.B;
  std::vector<int> all;
  all.insert(all.end(), m->vbase.begin(), m->vbase.end());
  all.insert(all.end(), m->vused.begin(), m->vused.end());
  all.insert(all.end(), m->tbase.begin(), m->tbase.end());
  all.insert(all.end(), m->tused.begin(), m->tused.end());
  if (!m->ranges) TRY(dalloc(m, &m->ranges, all.size()));
  if (B == 1) {
    // written by the row build that follows
  } else if (all.size() <= (size_t)kAuxInts / 2) {
    // staged in the upper half of the pinned ints and copied in stream
    // order; the previous upload's copy has finished before the stage is
    // rewritten
    int* stage = m->haux + kAuxInts / 2;
    if (!m->up_ev) HIPCHK(hipEventCreateWithFlags(&m->up_ev, hipEventDisableTiming));
    else HIPCHK(hipEventSynchronize(m->up_ev));
    std::copy(all.begin(), all.end(), stage);
    HIPCHK(hipMemcpyAsync(m->ranges, stage, sizeof(int) * all.size(), hipMemcpyHostToDevice, m->s));
    HIPCHK(hipEventRecord(m->up_ev, m->s));
  } else {
    HIPCHK(hipStreamSynchronize(m->s));
    HIPCHK(hipMemcpy(m->ranges, all.data(), sizeof(int) * all.size(), hipMemcpyHostToDevice));
  }
  st.vbase = m->ranges;
  st.vused = st.vbase + B + 1;
  st.tbase = st.vused + B;
  st.tused = st.tbase + B + 1;
  return PM_OK;
}

// ranges of a single mesh: everything in use
pm_status single_ranges(pm_mesh* m) {
  m->vbase = {0, m->st.V};
  m->vused = {m->st.V};
  m->tbase = {0, m->st.T};
  m->tused = {m->st.T};
  return upload_ranges(m);
}

// Pools of up to so many entries (64 MB each) are sized by a bound on the rows,
// without a read-back of what they need: 3-5 % of an adaptation of some thousand
// elements, nothing at half a million.
constexpr int64_t kSmallPool = 1 << 24;

// (Re)build every adjacency row from the element list into fresh pools.
// check: read the error bits back at the end (else they stay set for the
// caller's next read-back)
pm_status build_rows(pm_mesh* m, bool check = true) {
  Store& st = m->st;
  int V = st.V;
  m->rows_ok = false;
  TRY(ensure(m, m->vt0, V));
  TRY(ensure(m, m->partial, scan_partials_needed(V)));
  // room for rows that outgrow their slot before the next rebuild: the
  // headroom (3 by default) times the used entries. Slot capacities are at
  // most c(1+slack) + slack + 7 for a vertex in c elements, and the c sum to
  // 3T, which bounds both totals; when the pools hold the headroom times that
  // bound they are large enough without a read-back. Small pools are simply
  // sized by it (about twice what the rows need), which saves the read-back too.
  double bound = 3.0 * st.T * (1.0 + m->slack) + (double)V * (m->slack + 7.0);
  double extra = m->headroom >= 3.0 ? 4096.0 : 64.0;
  double room = m->headroom * bound + extra;
  bool fits = room <= (double)INT32_MAX && (double)st.nn_pool >= room && (double)st.ne_pool >= room;
  bool small = m->headroom >= 3.0 && room <= (double)kSmallPool;
  int* place = nullptr;
  auto pools = [&](int64_t nn_used, int64_t ne_used) -> pm_status {
    int64_t nn_need = (int64_t)(m->headroom * (double)nn_used + extra);
    int64_t ne_need = (int64_t)(m->headroom * (double)ne_used + extra);
    if (nn_need > INT32_MAX || ne_need > INT32_MAX)
      return fail(m, PM_E_NOMEM, "adjacency pool beyond 2^31 entries");
    if (st.nn_pool < nn_need || st.ne_pool < ne_need) {
      dfree(m, st.nn, st.nn_pool);
      dfree(m, st.ne, st.ne_pool);
      st.nn_pool = st.ne_pool = 0;
      place = nullptr;
      TRY(dalloc(m, &st.nn, nn_need));
      TRY(dalloc(m, &st.ne, ne_need));
      st.nn_pool = nn_need;
      st.ne_pool = ne_need;
    }
    return PM_OK;
  };
  if (!fits && small) {
    pm_status r = pools((int64_t)bound, (int64_t)bound);
    if (r != PM_OK && r != PM_E_NOMEM) return r;
    small = r == PM_OK;  // (no memory for the bound: by the entries)
  }
  // the incidences' places lie in the NN pool, which the row finish writes last
  int64_t places = 3 * (int64_t)st.T;
  place = st.nn_pool >= places ? st.nn : nullptr;
  build_start(m->vt0.p, st.B == 1 ? m->ranges : nullptr, m->vused[0], m->tused[0], V, st.T, m->s);
  build_count(st, m->vt0.p, place, m->s);
  build_headers(st, m->vt0.p, m->slack, m->ctr, (int2*)m->partial.p, m->s);
  if (!fits && !small) {
    TRY(read_ctr(m, C_NN_TOP, 2));
    TRY(pools(m->hctr[C_NN_TOP], m->hctr[C_NE_TOP]));
  }
  // (the pool was not there yet, was replaced, or is short of a place for every
  // element slot: counted again)
  int* own = nullptr;
  if (!place) {
    if (st.nn_pool < places) TRY(dalloc(m, &own, places));
    place = own ? own : st.nn;
    zero_ints(m->vt0.p, V, m->s);
    build_count(st, m->vt0.p, place, m->s);
  }
  build_fill(st, place, m->s);
  dfree(m, own, places);
  build_finish(st, m->ctr, m->s);
  m->rows_ok = true;
  return check ? check_err(m) : PM_OK;
}
// Before a call reads rows: a build that found no memory left them short of the
// element list, or in blocks that are gone; built now, or the call fails too.
pm_status rows_ready(pm_mesh* m) { return m->rows_ok ? PM_OK : build_rows(m); }

// free pool space check between rounds: rebuild (repack) when a round could
// plausibly exhaust it
// from the host copy of the pool tops
bool needs_repack(const pm_mesh* m) {
  int64_t nn_top = m->hctr[C_NN_TOP], ne_top = m->hctr[C_NE_TOP];
  return nn_top * 3 > m->st.nn_pool * 2 || ne_top * 3 > m->st.ne_pool * 2;
}
pm_status maybe_repack(pm_mesh* m, bool fresh = false) {
  if (!fresh) TRY(read_ctr(m, C_NN_TOP, 2));
  if (needs_repack(m)) return build_rows(m);
  return PM_OK;
}

pm_status ensure_phase_scratch(pm_mesh* m) {
  int V = std::max(m->st.V, 1), T = std::max(m->st.T, 1);
  TRY(ensure(m, m->listA, V));
  TRY(ensure(m, m->listB, V));
  TRY(ensure(m, m->jpU0, ((size_t)V + kJpChunk - 1) / kJpChunk * kJpChunk));
  TRY(ensure(m, m->jpB, ((size_t)V + kJpChunk - 1) / kJpChunk * kJpChunk));
  TRY(ensure(m, m->jpU1, (size_t)V / kBlock + 1));  // chunk counts of the chunked JP
  TRY(ensure(m, m->cls, V));
  TRY(ensure(m, m->jprec, (size_t)std::min(V, kSmallColour)));
  TRY(ensure(m, m->rw, V, true));
  TRY(ensure(m, m->nxt, V, true));
  TRY(ensure(m, m->ops, V, true));
  TRY(ensure(m, m->touch, std::max(V, 65536)));
  TRY(ensure(m, m->seen, V, true));
  TRY(ensure(m, m->own, V, true));
  TRY(ensure(m, m->dirty, V, true));
  TRY(ensure(m, m->cnt, V, true));
  TRY(ensure(m, m->tgt, V, true));
  TRY(ensure(m, m->sflag, V));
  TRY(ensure(m, m->spart, scan_partials_needed(V) + 2));
  // staging for the rows past the wavefront path (more than 64 candidates):
  // 4 ids per candidate; a round that runs out is redone from a row rebuild
  // with twice the staging
  size_t stage = (size_t)(m->stage_scale * m->headroom / 3.0 * (4.0 * T + 4.0 * V)) +
                 (m->headroom >= 3.0 ? 65536 : 64);
  TRY(ensure(m, m->stage, stage));
  return PM_OK;
}

Commit commit_of(pm_mesh* m) {
  Commit c;
  c.epoch = m->epoch;
  c.ops = m->ops.p;
  c.touched = nullptr;
  c.touched_cap = (int)std::min<size_t>(m->touch.n, INT32_MAX);
  c.own = m->own.p;
  c.by_member = 1;
  c.dirty = m->dirty.p;
  c.cnt = m->cnt.p;
  c.tgt = m->tgt.p;
  c.stage = m->stage.p;
  c.stage_cap = (int64_t)m->stage.n;
  c.nxt = m->nxt.p;
  return c;
}

// A phase that stops early, with status r, may leave vertices selected for its
// next round, or coloured for it: no other phase sees them.
pm_status round_left(pm_mesh* m, pm_status r) {
  if (m->nxt.p) HIPCHK(hipMemsetAsync(m->nxt.p, 0, m->nxt.n, m->s));
  if (m->rw.p) HIPCHK(hipMemsetAsync(m->rw.p, 0, sizeof(uint64_t) * m->rw.n, m->s));
  return r;
}

struct Classes {
  int ncol = 0;
  std::vector<int> size, off;
  int jp_iters = 0;
};

// Jones-Plassmann on list A (n entries): round words in rd.rw (the caller
// clears them), class lists in m->cls. Iterations run on a chunked copy of A
// and are launched in batches between read-backs of the count still waiting;
// a launch past the end of the work finds only empty chunks.
constexpr int kJpBatch = 4;
constexpr int kFinish = 2048;

// the classes of a one-block colouring, from the host copy of the counters
void small_classes(pm_mesh* m, Classes& out) {
  out.jp_iters = m->hctr[C_TOTAL];
  out.ncol = std::max(m->hctr[C_NCOL], 0);
  out.size.assign(m->hctr + C_HIST, m->hctr + C_HIST + out.ncol);
  out.off.assign(m->hctr + C_OFF, m->hctr + C_OFF + out.ncol);
}

pm_status colour_list(pm_mesh* m, const int* A, int n, Round rd, Classes& out) {
  out = Classes();
  if (n == 0) return PM_OK;
  if (n <= kSmallColour && !m->tune.small_work) {
    timed(m, PM_K_JP, 0,
          [&] { colour_small(m->st, A, n, nullptr, n, rd, m->jprec.p, m->cls.p, m->ctr, m->s); });
    TRY(read_ctr(m, 0, C_NCOL + 1));
    TRY(check_err(m, true));
    small_classes(m, out);
    return PM_OK;
  }
  int nb = (n + kBlock - 1) / kBlock;
  TRY(ensure(m, m->ctab, 256 * (size_t)nb + 256));
  TRY(ensure(m, m->ctabs, 256 * (size_t)nb + 256));
  TRY(ensure(m, m->spart, scan_partials_needed(256 * nb) + 2));
  jp_init(m->st, A, n, rd, m->ctr, m->s);
  bool finish = !m->tune.small_work;
  int it = 0;
  for (;;) {
    // first batch: as many iterations as the last colouring needed, so that
    // most colourings need one read-back; the class lists are cut before
    // that read-back, which then also returns them (cut again if the
    // colouring was not finished)
    // (with the one-block finish: until few enough wait for it)
    int batch = it == 0 ? std::min(std::max(m->jp_last, finish ? 1 : kJpBatch), 64) : kJpBatch;
    for (int b = 0; b < batch; ++b, ++it)
      timed(m, PM_K_JP, 0,
            [&] { jp_chunk(m->st, A, n, m->jpU0.p, m->jpB.p, m->jpU1.p, it == 0, rd, m->ctr, it, m->s); });
    if (finish) {
      // what every iteration of the last eight left (C_JPL), then the rest
      timed(m, PM_K_JP, 0, [&] {
        jp_finish(m->st, n, m->jpU0.p, m->jpU1.p, rd, m->jprec.p, m->cls.p, m->ctr, it - 1, m->s);
      });
    }
    else stripe_sum(m->ctr, S_JPL + ((it - 1) & 7), 1, C_JP, m->s);
    m->class_seq = m->class_seq >= 0x3FFFFFFF ? 1 : m->class_seq + 1;
    class_lists(A, n, rd.rw, m->ctr, m->cls.p, m->ctab.p, m->ctabs.p, m->spart.p,
                m->tune.class_colours ? m->tune.class_colours : kClassNarrow, m->class_seq, m->s);
    TRY(read_ctr(m, 0, C_NCOL + 1));
    int left = m->hctr[C_JP];
    if (left == 0) break;
    if (it > 4096) return fail(m, PM_E_DEVICE, "colouring did not finish");
  }
  if (m->hctr[C_NCOL] == -2 && m->tune.class_colours != 256) {
    // a colour past the narrow table: the full table
    class_lists(A, n, rd.rw, m->ctr, m->cls.p, m->ctab.p, m->ctabs.p, m->spart.p, 256, 0, m->s);
    TRY(read_ctr(m, 0, C_NCOL + 1));
  }
  out.jp_iters = it + (finish ? m->hctr[C_JPIT] : 0);
  // the iterations to run before the finish next time: until no more than
  // kFinish wait (the counts of the last seven are there; a further iteration
  // takes 7 us, solving 8,000 vertices 60 and 2,000 vertices 15); without the
  // finish, all
  m->jp_last = it;
  if (finish)
    while (m->jp_last > 1 && it - m->jp_last < 6 && m->hctr[C_JPL + ((m->jp_last - 2) & 7)] <= kFinish) --m->jp_last;
  if (finish && m->jp_last == it && m->hctr[C_JPL + ((it - 1) & 7)] > kFinish) ++m->jp_last;
  TRY(check_err(m, true));
  out.ncol = std::max(m->hctr[C_NCOL], 0);
  out.size.assign(m->hctr + C_HIST, m->hctr + C_HIST + out.ncol);
  out.off.assign(m->hctr + C_OFF, m->hctr + C_OFF + out.ncol);
  return PM_OK;
}

void stats_zero(pm_mesh* m) { phase_start(m->ctr, m->s); }

pm_status stats_read(pm_mesh* m, pm_stats* st) {
  // summed straight into the pinned mirror
  mail_next(m->mail);
  stripe_mail(m->ctr, S_EVAL, 6, m->hctr + C_EVAL, m->mail, m->s);
  HIPCHK(mail_wait(m->mail, m->s));
  if (m->prof.mask) HIPCHK(hipStreamSynchronize(m->s));
  prof_flush(m);
  if (st) {
    st->v[2] += m->hctr[C_EVAL];
    st->v[3] += m->hctr[C_DEFER];
    st->v[4] += m->hctr[C_COMMIT];
    st->v[11] += m->hctr[C_RELOC];
    st->v[10] += m->hctr[C_ROWS];
    st->v[6] += m->hctr[C_EDGES];
  }
  return PM_OK;
}

// headroom a batched mesh keeps after its used slots (refinement grows into it)
int headroom(int used) { return std::max(used / 2, 64); }

// A single mesh: the scans in vt1 and tt1 are the new ids, their totals the new
// sizes. When every slot is live the renumbering is the identity, and the rows
// stay.
pm_status compact_one(pm_mesh* m) {
  Store& st = m->st;
  TRY(read_ctr(m, 0, C_TOTAL2 + 1));
  int nV = m->hctr[C_TOTAL], nT = m->hctr[C_TOTAL2];
  if (nV == st.V && nT == st.T) return check_err(m, true);
  Store to = st;
  to.xy = nullptr;
  to.met = nullptr;
  to.tag = to.valive = nullptr;
  to.tri = nullptr;
  TRY(dalloc(m, &to.tri, st.Tcap));
  pm_status r = dalloc_all(m, st.Vcap, to.xy, to.met, to.tag, to.valive);
  if (r != PM_OK) {
    dfree(m, to.tri, st.Tcap);
    return r;
  }
  compact_vertices(st, m->vt1.p, to.xy, to.met, to.tag, to.valive, m->s);
  compact_elements(st, m->vt1.p, m->tt1.p, to.tri, m->s);
  clear_tail(to, nV, nT, m->s);
  dfree(m, st.xy, st.Vcap);
  dfree(m, st.met, st.Vcap);
  dfree(m, st.tag, st.Vcap);
  dfree(m, st.valive, st.Vcap);
  dfree(m, st.tri, st.Tcap);
  st = to;
  st.V = nV;
  st.T = nT;
  m->vbase = {0, nV};
  m->vused = {nV};
  m->tbase = {0, nT};
  m->tused = {nT};
  TRY(upload_ranges(m));
  return build_rows(m);
}

// Stable renumbering of live vertices and elements. A single mesh is packed
// densely; the meshes of a batch are packed into consecutive ranges with
// headroom (extra_v / extra_t: further slots a mesh is known to need).
pm_status compact(pm_mesh* m, const std::vector<int>* extra_v = nullptr, const std::vector<int>* extra_t = nullptr) {
  Store& st = m->st;
  int V = st.V, T = st.T, B = st.B;
  TRY(ensure(m, m->vt0, V));
  TRY(ensure(m, m->vt1, V));
  TRY(ensure(m, m->vt2, V));
  TRY(ensure(m, m->tt0, T));
  TRY(ensure(m, m->tt1, T));
  TRY(ensure(m, m->tt2, T));
  TRY(ensure(m, m->rtmp, 4 * (size_t)B + 4));
  TRY(ensure(m, m->partial, scan_partials_needed(V) + scan_partials_needed(T)));
  scan_live(st, m->vt0.p, m->vt1.p, m->ctr + C_TOTAL, m->tt0.p, m->tt1.p, m->ctr + C_TOTAL2, m->partial.p, m->s);
  if (B == 1) return compact_one(m);
  range_sums(m->vt1.p, m->vt0.p, st.vbase, st.vused, B, m->rtmp.p, m->s);
  range_sums(m->tt1.p, m->tt0.p, st.tbase, st.tused, B, m->rtmp.p + B, m->s);
  std::vector<int> live(2 * B);
  HIPCHK(hipMemcpyAsync(live.data(), m->rtmp.p, sizeof(int) * 2 * B, hipMemcpyDeviceToHost, m->s));
  TRY(sync(m));
  std::vector<int> nvb(B + 1, 0), ntb(B + 1, 0);
  for (int i = 0; i < B; ++i) {
    int lv = live[i], lt = live[B + i];
    int ev = extra_v ? (*extra_v)[i] : 0, et = extra_t ? (*extra_t)[i] : 0;
    int cv = lv + ev + headroom(lv + ev);
    int ct = lt + et + headroom(lt + et);
    if ((int64_t)nvb[i] + cv > (1ll << 30) || (int64_t)ntb[i] + ct > (1ll << 30))
      return fail(m, PM_E_NOMEM, "store beyond 2^30 slots");
    nvb[i + 1] = nvb[i] + cv;
    ntb[i + 1] = ntb[i] + ct;
  }
  int nV = nvb[B], nT = ntb[B];
  HIPCHK(hipMemcpyAsync(m->rtmp.p, nvb.data(), sizeof(int) * (B + 1), hipMemcpyHostToDevice, m->s));
  HIPCHK(hipMemcpyAsync(m->rtmp.p + B + 1, ntb.data(), sizeof(int) * (B + 1), hipMemcpyHostToDevice, m->s));
  mesh_maps(m->vt0.p, m->vt1.p, st.vmesh, st.vbase, m->rtmp.p, V, m->vt2.p, m->s);
  mesh_maps(m->tt0.p, m->tt1.p, st.tmesh, st.tbase, m->rtmp.p + B + 1, T, m->tt2.p, m->s);
  int vcap = std::max(nV, 1), tcap = std::max(nT, 1);
  double2* xy2 = nullptr;
  Met* met2 = nullptr;
  uint8_t *tag2 = nullptr, *va2 = nullptr;
  Elem* tri2 = nullptr;
  int *vmesh2 = nullptr, *tmesh2 = nullptr;
  Hdr* hdr2 = nullptr;
  int2* cap2 = nullptr;
  TRY(dalloc_all(m, vcap, xy2, met2, tag2, va2, vmesh2, hdr2, cap2));
  pm_status r = dalloc_all(m, tcap, tri2, tmesh2);
  if (r != PM_OK) {
    dfree(m, xy2, vcap);
    dfree(m, met2, vcap);
    dfree(m, tag2, vcap);
    dfree(m, va2, vcap);
    dfree(m, vmesh2, vcap);
    dfree(m, hdr2, vcap);
    dfree(m, cap2, vcap);
    return r;
  }
  HIPCHK(hipMemsetAsync(va2, 0, vcap, m->s));
  HIPCHK(hipMemsetAsync(tri2, 0, sizeof(Elem) * (size_t)tcap, m->s));
  compact_vertices(st, m->vt2.p, xy2, met2, tag2, va2, m->s);
  compact_elements(st, m->vt2.p, m->tt2.p, tri2, m->s);
  fill_mesh_ids(m->rtmp.p, B, nV, vmesh2, m->s);
  fill_mesh_ids(m->rtmp.p + B + 1, B, nT, tmesh2, m->s);
  // headers and capacities follow the new slot count
  HIPCHK(hipMemsetAsync(hdr2, 0, sizeof(Hdr) * (size_t)vcap, m->s));
  HIPCHK(hipMemsetAsync(cap2, 0, sizeof(int2) * (size_t)vcap, m->s));
  HIPCHK(hipStreamSynchronize(m->s));
  dfree(m, st.hdr, st.Vcap);
  dfree(m, st.cap, st.Vcap);
  st.hdr = hdr2;
  st.cap = cap2;
  dfree(m, st.vmesh, st.Vcap);
  dfree(m, st.tmesh, st.Tcap);
  st.vmesh = vmesh2;
  st.tmesh = tmesh2;
  dfree(m, st.xy, st.Vcap);
  dfree(m, st.met, st.Vcap);
  dfree(m, st.tag, st.Vcap);
  dfree(m, st.valive, st.Vcap);
  dfree(m, st.tri, st.Tcap);
  st.xy = xy2;
  st.met = met2;
  st.tag = tag2;
  st.valive = va2;
  st.tri = tri2;
  st.Vcap = vcap;
  st.Tcap = tcap;
  st.V = nV;
  st.T = nT;
  m->vbase = nvb;
  m->tbase = ntb;
  for (int i = 0; i < B; ++i) {
    m->vused[i] = live[i];
    m->tused[i] = live[B + i];
  }
  TRY(upload_ranges(m));
  return build_rows(m);
}

bool bad_tuning(const pm_tuning& t) {
  auto in = [](int v, std::initializer_list<int> ok) {
    for (int x : ok)
      if (v == x) return true;
    return false;
  };
  return !in(t.op_lanes, {0, 1, 8, 16}) || !in(t.smooth_lanes, {0, 1, 8}) ||
         !in(t.commit_chunk, {0, 16, 32, 64, 128}) || !in(t.small_work, {0, 1}) ||
         !in(t.class_colours, {0, 4, 8, 16, 32, 64, 128, 256}) || !in(t.commit_order, {0, 1, 2}) ||
         !in(t.host_rounds, {0, 1, 2}) || t.reserved != 0;
}

bool bad_opts(const pm_options* o) {
  return !(o->L_low2 > 0.0) || !(o->L_up2 > 0.0) || !(o->q_min >= 0.0) || o->coarsen_rounds < 0 ||
         o->swap_rounds < 0 || o->refine_passes < 0 || o->smooth_sweeps < 0 || o->sweep < 0 || o->sweep > 4095 ||
         (o->smooth_kind != PM_SMOOTH_LAPLACE && o->smooth_kind != PM_SMOOTH_GRADIENT &&
          o->smooth_kind != PM_SMOOTH_MINMAX) || !(o->slack >= 1.0) ||
         !(o->pool_headroom == 0.0 || (o->pool_headroom >= 1.0 && o->pool_headroom <= 64.0)) ||
         o->max_iterations < 0 || o->max_iterations > 4095 || o->max_phases < 0 || bad_tuning(o->tune) ||
         (o->quality != PM_QUALITY_MEAN_RATIO && o->quality != PM_QUALITY_VASILEVSKII) || o->reserved != 0 ||
         (o->allocator && (!o->allocator->alloc || !o->allocator->release));
}

// Collapse runs on groups of lanes per member by default: each lane loads
// one neighbour and one element of the member's 1-ring side by side and
// keeps it in registers, so a member costs a few dependent loads and no
// re-reads (one thread per member walks the ring serially and, with tens of
// thousands of members in flight per XCD, re-fetches it from HBM). 16 lanes
// by default; 8, or one thread per member, by tuning.
int op_lanes(const pm_mesh* m) { return m->tune.op_lanes ? m->tune.op_lanes : 16; }
int smooth_lanes(const pm_mesh* m) { return m->tune.smooth_lanes ? m->tune.smooth_lanes : 8; }

pm_status run_rounds_in(pm_mesh* m, const pm_options* o, pm_stats* st, int kind);

// rounds of colour -> classes -> op + commit (coarsen: kind 0, swap: kind 1);
// vertices stay fixed through the rounds, so their records are built once
pm_status run_rounds(pm_mesh* m, const pm_options* o, pm_stats* st, int kind) {
  TRY(rows_ready(m));
  TRY(ensure(m, m->vr, (size_t)std::max(m->st.V, 1)));
  vertex_records(m->st, m->vr.p, m->s);
  m->st.vr = m->vr.p;
  pm_status r = run_rounds_in(m, o, st, kind);
  m->st.vr = nullptr;
  return r == PM_OK ? r : round_left(m, r);
}

// One class of a round: the operation over its members, then the commit of
// the rows they changed (one launch for a small class)
void run_class(pm_mesh* m, int kind, const Classes& cl, int c, const OpArgs& a, Commit cm) {
  const int* list = m->cls.p + cl.off[c];
  int n = cl.size[c];
  if (n <= kSmallClass && !m->tune.small_work) {
    timed(m, kind == 0 ? PM_K_COLLAPSE : PM_K_FLIP, n, [&] { class_small(m->st, list, n, a, cm, kind, m->ctr, m->s); });
    return;
  }
  bool sweep = m->tune.commit_order == 2 || (m->tune.commit_order == 0 && (int64_t)n * 64 >= m->st.V);
  cm.by_member = sweep ? 0 : 1;
  if (kind == 0)
    timed(m, PM_K_COLLAPSE, n, [&] { collapse_class(m->st, list, n, a, cm, m->ctr, op_lanes(m), m->s); });
  else
    timed(m, PM_K_FLIP, n, [&] {
      if (op_lanes(m) == 1) flip_class(m->st, list, n, a, cm, m->ctr, m->s);
      else flip_class_g(m->st, list, n, a, cm, m->ctr, m->s);
    });
  if (sweep) {
    timed(m, PM_K_COMMIT, 0, [&] { commit_sweep(m->st, cm, kind != 0, m->ctr, m->s); });
  } else {
    timed(m, PM_K_COMMIT, 0,
          [&] { commit_rows(m->st, list, n, cm, kind != 0, m->tune.commit_chunk, m->ctr, m->s); });
  }
}

// A commit ran out of pool or staging room in this round (the host copy of
// the counters says so): rebuild every row from the element list with twice
// the room, then run the classes after the one that ran out. Their kernels
// exited at once; the failing class's operations are all in the element list.
// class_epoch[c]: the epoch class c ran with (-1: not run).
pm_status recover_round(pm_mesh* m, int kind, const Classes& cl, std::vector<int>& class_epoch, Round rd,
                        const pm_options* o, int listA_n) {
  double qmin2 = o->q_min * o->q_min;
  for (;;) {
    int err = m->hctr[C_ERR], fe = m->hctr[C_FAILEP];
    if (!(err & kRoomErr)) return PM_OK;
    int cf = -1;
    for (int c = 0; c < cl.ncol; ++c)
      if (class_epoch[c] == fe) cf = c;
    if (cf < 0) return fail(m, PM_E_DEVICE, "room error of an unknown class");
    ++m->recoveries;
    if (err & (E_NN_POOL | E_NE_POOL)) m->headroom *= 2.0;
    if (err & E_STAGE) m->stage_scale *= 2.0;
    set_int(m->ctr + C_ERR, err & ~kRoomErr, m->s);
    set_int(m->ctr + C_FAILEP, INT_MAX, m->s);
    // every row again from the element list, packed, with the larger room
    TRY(build_rows(m, false));
    TRY(ensure_phase_scratch(m));
    // the round words were cleared with the round: set them again from the
    // class lists, run the remaining classes, clear them again
    std::vector<int> offs(cl.off.begin(), cl.off.end());
    TRY(ensure(m, m->rtmp, (size_t)std::max(cl.ncol, 1)));
    HIPCHK(hipMemcpyAsync(m->rtmp.p, offs.data(), sizeof(int) * cl.ncol, hipMemcpyHostToDevice, m->s));
    restore_round(m->st, m->cls.p, listA_n, m->rtmp.p, cl.ncol, rd, m->s);
    Commit cm = commit_of(m);
    cm.touched = nullptr;
    std::vector<int> ep = class_epoch;
    for (int c = cf + 1; c < cl.ncol; ++c) {
      if (cl.size[c] == 0) continue;
      cm.epoch = ++m->epoch;
      ep[c] = cm.epoch;
      OpArgs a{m->rw.p, c, rd, o->L_low2, qmin2};
      run_class(m, kind, cl, c, a, cm);
    }
    HIPCHK(hipStreamSynchronize(m->s));  // the offsets' host copy is a local vector
    clear_round(m->cls.p, listA_n, m->rw.p, nullptr, m->s);
    TRY(read_ctr(m, 0, kRoundCtrs));
    class_epoch = ep;
  }
}

// Rounds r, r + 1, ... of a phase whose lists fit one work-group, driven by
// the device: one launch runs them one after another, with one read-back
// (host_rounds 2: the launch replayed from a graph). Round r's
// classes must be coloured (counters and class lists set). Returns with the
// round counter, list and length of where the chain stopped: the list empty,
// the round cap, a list too long for one work-group (r_out's list, not
// coloured), or a selection that declined (declined: round r_out ran, its
// next list is not selected; the host selects over every slot, after
// rebuilding the rows if a commit ran out of room).
constexpr int kDevRounds = 64;  // rounds of one launch (then a read-back, and the next)
pm_status device_rounds(pm_mesh* m, const pm_options* o, pm_stats* st, int kind, int phase, int max_rounds, int r,
                        int* r_out, int* n_out, bool* declined) {
  int mode = kind == 0 ? 1 : 2;
  double qmin2 = o->q_min * o->q_min;
  int* L[2] = {m->listA.p, m->listB.p};
  Round rd{0, m->rw.p};
  OpArgs a{m->rw.p, 0, rd, o->L_low2, qmin2};
  Commit cm = commit_of(m);
  cm.touched = m->touch.p;
  DevRounds dr{L[0], L[1], m->cls.p, m->seen.p, m->rw.p, m->seed,
               o->sweep, phase, r & 1, max_rounds, kDevRounds, mode, 1, r, m->epoch + 1, m->sel_mark};
  if (m->tune.host_rounds == 2) {
    // a launch that is replayed starts from the counters
    dev_rounds_start(m->ctr, r, m->epoch + 1, m->sel_mark, r >= max_rounds ? 1 : 0, m->s);
    dr.start = dr.round = dr.epoch = dr.mark = 0;
    cm.epoch = 0;
  }
  auto rounds = [&](hipStream_t q) { rounds_dev(m->st, dr, a, cm, kind, m->ctr, q); };
  // the graph is kept while its launch arguments stay the same
  // (the same store layout, buffers and parameters)
  hipGraphExec_t ge = nullptr;
  if (m->tune.host_rounds == 2) {
    std::string key;
    auto add = [&](const void* p, size_t n) { key.append((const char*)p, n); };
    add(&m->st, sizeof(Store));
    add(&a, sizeof(a));
    add(&cm, sizeof(cm));
    add(&dr, sizeof(dr));
    add(&kind, sizeof(kind));
    add(&m->ctr, sizeof(m->ctr));
    for (auto& g : m->dr_graphs)
      if (g.first == key) ge = g.second;
    if (!ge) {
      TRY(capture(m, rounds, &ge));
      if (m->dr_graphs.size() >= 4) {
        (void)hipGraphExecDestroy(m->dr_graphs.front().second);
        m->dr_graphs.erase(m->dr_graphs.begin());
      }
      m->dr_graphs.push_back({key, ge});
    }
  }
  pm_status res = PM_OK;
  for (;;) {
    hipError_t e = hipSuccess;
    timed(m, kind == 0 ? PM_K_COLLAPSE : PM_K_FLIP, 0, [&] {
      if (ge) e = hipGraphLaunch(ge, m->s);
      else rounds(m->s);
    });
    dr.start = 0;
    if (e != hipSuccess) {
      res = fail(m, PM_E_DEVICE, std::string("hipGraphLaunch: ") + hipGetErrorString(e));
      break;
    }
    res = read_ctr(m, 0, C_NCOL + 1);
    if (res != PM_OK || m->hctr[C_DSTOP]) break;
  }
  TRY(res);
  int rr = m->hctr[C_DROUND];
  st->v[1] += m->hctr[C_ACC_COL];
  st->v[5] += m->hctr[C_ACC_NCOL];
  st->v[12] += m->hctr[C_ACC_IT];
  m->epoch = m->hctr[C_DEPOCH] - 1;
  m->sel_mark = m->hctr[C_DMARK];
  // the list of round rr is L[(rr - r) & 1]
  int cur = (rr - r) & 1;
  m->listA.p = L[cur];
  m->listB.p = L[cur ^ 1];
  *r_out = rr;
  *n_out = m->hctr[C_LIST_B];
  *declined = m->hctr[C_LIST_B] < 0;
  return PM_OK;
}

pm_status run_rounds_in(pm_mesh* m, const pm_options* o, pm_stats* st, int kind) {
  TRY(ensure_phase_scratch(m));
  m->tune = o->tune;
  m->recoveries = 0;
  int mode = kind == 0 ? 1 : 2;
  int max_rounds = kind == 0 ? o->coarsen_rounds : o->swap_rounds;
  int phase = kind == 0 ? PH_COARSEN : PH_SWAP;
  double qmin2 = o->q_min * o->q_min;
  stats_zero(m);
  timed(m, PM_K_SELECT, m->st.V,
        [&] { select_vertices(m->st, mode, o->L_low2, nullptr, nullptr, m->listA.p, m->ctr, m->sflag.p, m->spart.p, m->s); });
  TRY(read_ctr(m, 0, kRoundCtrs));  // pool tops, error bits and the list length at once
  TRY(check_err(m, true));
  int nA = m->hctr[C_LIST_B];
  int r = 0;
  // a small round colours the next round's list as soon as it is selected,
  // before the read-back that returns its length: one read-back for both
  bool ahead = false;
  Classes next;
  while (nA > 0 && r < max_rounds) {
    // after a repack (all rows rebuilt) the list is coloured again rather
    // than keep classes found before it
    bool repacked = needs_repack(m);
    TRY(maybe_repack(m, true));
    Round rd{stream_seed(m->seed, make_ctx(o->sweep, phase, r)), m->rw.p};
    Classes cl;
    if (ahead && !repacked) {
      cl = next;
    } else {
      TRY(colour_list(m, m->listA.p, nA, rd, cl));
    }
    ahead = false;
    Commit cm = commit_of(m);
    // a small round (coloured by one block) records the rows it rebuilds, so
    // the next round's list comes from its own lists, not from every slot
    bool small = nA <= kSmallColour && !m->tune.small_work;
    cm.touched = small ? m->touch.p : nullptr;
    st->v[1] += nA;
    st->v[5] += cl.ncol;
    st->v[12] += cl.jp_iters;
    bool fits = cl.ncol > 0;
    for (int c = 0; c < cl.ncol && fits; ++c) fits = cl.size[c] <= kSmallClass;
    if (small && m->tune.host_rounds != 1 && fits) {
      int rr = r, nl = 0;
      bool declined = false;
      TRY(device_rounds(m, o, st, kind, phase, max_rounds, r, &rr, &nl, &declined));
      if (!declined) {
        // the next round's list is coloured when it fits one work-group (the
        // counters hold its classes; a class too large for the chain stopped
        // it), else the host colours it
        nA = nl;
        r = rr;
        ahead = m->hctr[C_NCOL] >= 0 && nl > 0;
        if (ahead) small_classes(m, next);
        continue;
      }
      // round rr ran, its selection declined: the classes from the counters
      if (m->hctr[C_NCOL] < 0 || m->hctr[C_NCOL] > kMaxColours)
        return fail(m, PM_E_DEVICE, "device-driven round left no class counters");
      Classes dc;
      small_classes(m, dc);
      std::vector<int> dep(dc.ncol);
      for (int c = 0; c < dc.ncol; ++c) dep[c] = m->hctr[C_DEPOCH0] + c;
      int n_rr = 0;
      for (int c = 0; c < dc.ncol; ++c) n_rr += dc.size[c];
      if (m->hctr[C_ERR] & kRoomErr) {
        Round rdd{stream_seed(m->seed, make_ctx(o->sweep, phase, rr)), m->rw.p};
        TRY(recover_round(m, kind, dc, dep, rdd, o, n_rr));
      }
      timed(m, PM_K_SELECT, m->st.V, [&] {
        select_vertices(m->st, mode, o->L_low2, nullptr, m->nxt.p, m->listB.p, m->ctr, m->sflag.p, m->spart.p, m->s);
      });
      TRY(read_ctr(m, 0, kRoundCtrs));
      TRY(check_err(m, true));
      nA = m->hctr[C_LIST_B];
      std::swap(m->listA, m->listB);
      r = rr + 1;
      ahead = false;
      continue;
    }
    std::vector<int> class_epoch(cl.ncol, -1);
    // a small round whose classes are all small: every class in one block,
    // one launch
    bool all_small = small && cl.ncol > 1;
    for (int c = 0; c < cl.ncol && all_small; ++c) all_small = cl.size[c] <= kSmallClass;
    if (all_small) {
      cm.epoch = m->epoch + 1;
      for (int c = 0; c < cl.ncol; ++c) class_epoch[c] = cm.epoch + c;
      m->epoch += cl.ncol;
      OpArgs a{m->rw.p, 0, rd, o->L_low2, qmin2};
      timed(m, kind == 0 ? PM_K_COLLAPSE : PM_K_FLIP, nA,
            [&] { round_small(m->st, m->cls.p, cl.ncol, a, cm, kind, m->ctr, m->s); });
    }
    for (int c = 0; c < cl.ncol && !all_small; ++c) {
      if (cl.size[c] == 0) continue;
      cm.epoch = ++m->epoch;
      class_epoch[c] = cm.epoch;
      OpArgs a{m->rw.p, c, rd, o->L_low2, qmin2};
      run_class(m, kind, cl, c, a, cm);
    }
    clear_round(m->listA.p, nA, m->rw.p, m->ctr + C_LIST_B, m->s);
    bool listed = false;
    if (small) {
      timed(m, PM_K_SELECT, nA, [&] {
        select_list(m->st, mode, o->L_low2, m->listA.p, nA, m->touch.p, cm.touched_cap, m->nxt.p, m->seen.p,
                    ++m->sel_mark, m->listB.p, m->ctr, m->s);
      });
      bool launch = r + 1 < max_rounds;
      if (launch) {
        Round rn{stream_seed(m->seed, make_ctx(o->sweep, phase, r + 1)), m->rw.p};
        timed(m, PM_K_JP, 0, [&] {
          colour_small(m->st, m->listB.p, 0, m->ctr + C_LIST_B, nA, rn, m->jprec.p, m->cls.p, m->ctr, m->s);
        });
      }
      TRY(read_ctr(m, 0, launch ? C_NCOL + 1 : kRoundCtrs));
      listed = m->hctr[C_LIST_B] >= 0;
      if (launch && listed && m->hctr[C_NCOL] >= 0) {
        ahead = true;
        small_classes(m, next);
      }
    }
    auto select_all = [&]() -> pm_status {
      timed(m, PM_K_SELECT, m->st.V, [&] {
        select_vertices(m->st, mode, o->L_low2, nullptr, m->nxt.p, m->listB.p, m->ctr, m->sflag.p, m->spart.p, m->s);
      });
      return read_ctr(m, 0, kRoundCtrs);
    };
    if (!listed) TRY(select_all());
    if (m->hctr[C_ERR] & kRoomErr) {
      // the selections and the next colouring declined (they saw the error):
      // rebuild, finish the round, then select over every slot
      TRY(recover_round(m, kind, cl, class_epoch, rd, o, nA));
      ahead = false;
      TRY(select_all());
    }
    TRY(check_err(m, true));
    nA = m->hctr[C_LIST_B];
    std::swap(m->listA, m->listB);
    ++r;
  }
  TRY(stats_read(m, st));
  st->v[0] = r;
  st->v[7] = nA == 0 ? 1 : 0;
  st->v[13] = m->recoveries;
  return PM_OK;
}

// partial sums of the quality reduction: one per 256 element slots, at most
// kQualityParts (the same shape for pm_quality and pm_quality_noalloc)
constexpr int kQualityParts = 2048;
int quality_parts(const pm_mesh* m) { return std::min(std::max((m->st.T + 255) / 256, 1), kQualityParts); }

// Device memory that pm_quality_noalloc works in instead of allocating: the
// quality reduction's partial sums and minima and its two results. Each
// device that runs the library holds its own copy until the process ends.
// Host code never uses this name as an address: the device address of each
// device's copy comes from hipGetSymbolAddress, taken once per device with
// that device current (at the first handle created on it).
constexpr int kScratchDoubles = 2 * kQualityParts + 2;
static __device__ __align__(256) double scratch[kScratchDoubles];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_at[kMaxDevices] = {};

// the current device's copy of the scratch array, for handle m
pm_status scratch_setup(pm_mesh* m) {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(m, PM_E_DEVICE, "device index past the scratch table");
  m->dev = dev;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_at[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return fail(m, PM_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    }
    g_scratch_at[dev] = (double*)p;
  }
  m->scratch = g_scratch_at[dev];
  return PM_OK;
}

void fill_defaults(pm_options* o) {
  o->L_low2 = 0.5;
  o->L_up2 = 2.0;
  o->q_min = 0.1;
  o->seed = 0;
  o->sweep = 0;
  o->coarsen_rounds = 200;
  o->swap_rounds = 100;
  o->refine_passes = 32;
  o->smooth_kind = PM_SMOOTH_LAPLACE;
  o->smooth_sweeps = 1;
  o->slack = 2.0;
  o->pool_headroom = 3.0;
  o->max_iterations = 8;
  o->max_phases = 0;
  o->tune = pm_tuning{};
  o->quality = PM_QUALITY_MEAN_RATIO;
  o->reserved = 0;
  o->allocator = nullptr;
}

}  // namespace

namespace pm {
hipError_t block_alloc(hipStream_t s, void** p, size_t bytes) {
  size_t got = 0;
  return cache_get(s, p, bytes, &got);
}
void block_free(void* p) {
  if (p && cache_put(p) == 0) (void)hipFree(p);
}

static std::mutex g_pinned_mu;
static std::vector<void*> g_pinned_free;
void* pinned_take() {
  void* p = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    if (!g_pinned_free.empty()) {
      p = g_pinned_free.back();
      g_pinned_free.pop_back();
      return p;
    }
  }
  // coherent: the host sees a kernel's stores while later work still runs
  if (hipHostMalloc(&p, kPinnedBytes, hipHostMallocCoherent | hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  memset(p, 0, kPinnedBytes);
  return p;
}
void pinned_give(void* p) {
  if (!p) return;
  std::lock_guard<std::mutex> lk(g_pinned_mu);
  g_pinned_free.push_back(p);
}

static std::vector<void*> g_stage_free;
constexpr size_t kStageKept = 4;
void* stage_take() {
  void* p = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    if (!g_stage_free.empty()) {
      p = g_stage_free.back();
      g_stage_free.pop_back();
      return p;
    }
  }
  if (hipHostMalloc(&p, kStageBytes, hipHostMallocCoherent | hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return p;
}
void stage_give(void* p) {
  if (!p) return;
  {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    if (g_stage_free.size() < kStageKept) {
      g_stage_free.push_back(p);
      return;
    }
  }
  (void)hipHostFree(p);
}

Mail mail_of(void* block) {
  Mail b;
  b.at = (volatile int*)((char*)block + kPinnedBytes - sizeof(int));
  b.no = *b.at;
  return b;
}
static __global__ void k_mail(const int* __restrict__ src, int n, int* dst, int* at, int no) {
  for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) dst[i] = src[i];
  mail_post(at, no);
}
void mail_next(Mail& b) { b.no = b.no == INT_MAX ? 1 : b.no + 1; }
void mail_send(Mail& b, const int* src, int n, int* dst, hipStream_t s) {
  mail_next(b);
  k_mail<<<1, kBlock, 0, s>>>(src, n, dst, (int*)b.at, b.no);
}
// (like the runtime's own wait for a stream, this polls on a core for as long as the
// work takes)
hipError_t mail_wait(const Mail& b, hipStream_t s) {
  hipError_t launch = hipPeekAtLastError();
  for (int64_t k = 1;; ++k) {
    if (__atomic_load_n(b.at, __ATOMIC_ACQUIRE) == b.no) return hipSuccess;
    __builtin_ia32_pause();
    if (k % 16384 == 0) {  // a fraction of a millisecond: has the stream failed?
      hipError_t e = hipStreamQuery(s);
      if (e == hipSuccess) {
        if (__atomic_load_n(b.at, __ATOMIC_ACQUIRE) == b.no) return hipSuccess;
        return launch != hipSuccess ? launch : hipErrorUnknown;  // the letter was not launched
      }
      if (e != hipErrorNotReady) return e;
      (void)hipGetLastError();
      if (k > (1 << 20)) std::this_thread::yield();
    }
  }
}
}  // namespace pm

extern "C" {

const char* pm_version(void) { return "pmesh 0.1 gfx950"; }

pm_status pm_default_options(pm_options* o) {
  if (!o) return PM_E_ARG;
  fill_defaults(o);
  return PM_OK;
}

const char* pm_last_error(const pm_mesh* m) {
  if (!m) return g_create_err.empty() ? "null handle" : g_create_err.c_str();
  return m->err.c_str();
}

pm_status pm_mesh_destroy(pm_mesh* m) {
  if (!m) return PM_OK;
  (void)hipStreamSynchronize(m->s);
  Store& s = m->st;
  dfree(m, s.xy, s.Vcap);
  dfree(m, s.met, s.Vcap);
  dfree(m, s.tag, s.Vcap);
  dfree(m, s.valive, s.Vcap);
  dfree(m, s.hdr, s.Vcap);
  dfree(m, s.cap, s.Vcap);
  dfree(m, s.tri, s.Tcap);
  dfree(m, s.nn, s.nn_pool);
  dfree(m, s.ne, s.ne_pool);
  dfree(m, s.vmesh, s.Vcap);
  dfree(m, s.tmesh, s.Tcap);
  dfree(m, m->ranges, 1);
  dfree(m, m->mdone, 1);
  DBuf<int>* ib[] = {&m->listA, &m->listB, &m->jpU0, &m->jpU1, &m->cls, &m->vt0, &m->vt1, &m->vt2,
                     &m->tt0, &m->tt1, &m->tt2, &m->partial, &m->mid, &m->stage, &m->touch, &m->seen, &m->jpB, &m->rtmp,
                     &m->sflag, &m->ctab, &m->ctabs, &m->spart};
  for (auto* b : ib) dfree(m, b->p, b->n);
  DBuf<uint8_t>* ub[] = {&m->nxt, &m->u8tmp};
  dfree(m, m->emet.p, m->emet.n);
  dfree(m, m->vr.p, m->vr.n);
  for (auto* b : ub) dfree(m, b->p, b->n);
  dfree(m, m->jprec.p, m->jprec.n);
  dfree(m, m->qpart.p, m->qpart.n);
  dfree(m, m->upx.p, m->upx.n);
  dfree(m, m->upm.p, m->upm.n);
  dfree(m, m->rw.p, m->rw.n);
  dfree(m, m->own.p, m->own.n);
  dfree(m, m->dirty.p, m->dirty.n);
  dfree(m, m->cnt.p, m->cnt.n);
  dfree(m, m->tgt.p, m->tgt.n);
  dfree(m, m->ops.p, m->ops.n);
  prof_flush(m);
  for (hipEvent_t e : m->prof.pool) (void)hipEventDestroy(e);
  if (m->up_ev) {
    (void)hipEventSynchronize(m->up_ev);
    (void)hipEventDestroy(m->up_ev);
  }
  dfree(m, m->ctr, C_COUNT);
  pinned_put(m);
  for (auto& g : m->dr_graphs) (void)hipGraphExecDestroy(g.second);
  if (m->cap_s) (void)hipStreamDestroy(m->cap_s);
  delete m;
  return PM_OK;
}

pm_status pm_mesh_create(const pm_mesh_desc* d, const pm_options* o, void* stream, pm_mesh** out) {
  if (!out) return PM_E_ARG;
  *out = nullptr;
  if (!d || !d->xy || !d->tri || !d->metric) return PM_E_ARG;
  if (d->V < 3 || d->T < 1 || d->V > (1ll << 30) || d->T > (1ll << 30)) return PM_E_ARG;
  if (d->mem_kind != PM_MEM_HOST && d->mem_kind != PM_MEM_DEVICE) return PM_E_ARG;
  pm_options def;
  fill_defaults(&def);
  if (!o) o = &def;
  if (bad_opts(o)) return PM_E_ARG;
  pm_mesh* m = new (std::nothrow) pm_mesh();
  if (!m) return PM_E_NOMEM;
  m->s = (hipStream_t)stream;
  m->seed = o->seed;
  m->slack = o->slack;
  m->headroom = o->pool_headroom > 0.0 ? o->pool_headroom : 3.0;
  m->st.qk = o->quality;
  if (o->allocator) m->va = *o->allocator;
  g_create_err.clear();
  auto bail = [&](pm_status st) {
    g_create_err = m->err.empty() ? std::string("pm_mesh_create failed") : m->err;
    pm_mesh_destroy(m);
    return st;
  };
  if (dalloc(m, &m->ctr, C_COUNT) != PM_OK || !pinned_get(m)) return bail(PM_E_NOMEM);
  if (scratch_setup(m) != PM_OK) return bail(PM_E_DEVICE);
  zero_ints(m->ctr, C_COUNT, m->s);
  set_int(m->ctr + C_FAILEP, INT_MAX, m->s);
  int V = (int)d->V, T = (int)d->T;
  if (grow_vertices(m, V) != PM_OK || grow_elements(m, T) != PM_OK) return bail(PM_E_NOMEM);
  Store& st = m->st;
  st.V = V;
  st.T = T;
  hipMemcpyKind kind = d->mem_kind == PM_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
  int* tri3 = nullptr;
  double* xyraw = nullptr;
  if (dalloc(m, &tri3, 3 * (size_t)T) != PM_OK || dalloc(m, &xyraw, 2 * (size_t)V) != PM_OK) {
    dfree(m, tri3, 3 * (size_t)T);
    return bail(PM_E_NOMEM);
  }
  bool ok = hipMemcpyAsync(tri3, d->tri, sizeof(int) * 3 * (size_t)T, kind, m->s) == hipSuccess &&
            hipMemcpyAsync(xyraw, d->xy, sizeof(double) * 2 * (size_t)V, kind, m->s) == hipSuccess &&
            hipMemcpyAsync(st.met, d->metric, sizeof(double) * 3 * (size_t)V, kind, m->s) == hipSuccess;
  if (ok && d->tags) ok = hipMemcpyAsync(st.tag, d->tags, (size_t)V, kind, m->s) == hipSuccess;
  if (!ok) {
    dfree(m, tri3, 3 * (size_t)T);
    dfree(m, xyraw, 2 * (size_t)V);
    return bail(PM_E_DEVICE);
  }
  xy_in(xyraw, V, st.xy, m->s);
  if (!d->tags) tags_from_xy(st.xy, V, st.tag, m->s);
  tri_in(tri3, T, st.tri, m->s);
  fill_u8(st.valive, V, 1, m->s);
  // the staging blocks return to this stream's cache: later work on the
  // stream is ordered after the conversions that read them
  dfree(m, tri3, 3 * (size_t)T);
  dfree(m, xyraw, 2 * (size_t)V);
  pm_status r = single_ranges(m);
  if (r != PM_OK) return bail(r);
  k_validate(st, m->ctr, m->s);
  r = check_err(m);
  if (r != PM_OK) return bail(r);
  r = build_rows(m);
  if (r != PM_OK) return bail(r);
  *out = m;
  return PM_OK;
}

pm_status pm_mesh_sizes(const pm_mesh* m, int64_t* V, int64_t* T) {
  if (!m) return PM_E_ARG;
  if (V) *V = m->st.V;
  if (T) *T = m->st.T;
  return PM_OK;
}

pm_status pm_mesh_memory(const pm_mesh* m, int64_t* current_bytes, int64_t* peak_bytes) {
  if (!m) return PM_E_ARG;
  if (current_bytes) *current_bytes = m->cur_bytes;
  if (peak_bytes) *peak_bytes = m->peak_bytes;
  return PM_OK;
}

pm_status pm_mesh_export(pm_mesh* m, double* xy, int32_t* tri, double* metric, uint8_t* tags, uint8_t* valive,
                         uint8_t* talive, int32_t mem_kind) {
  if (!m) return PM_E_ARG;
  if (mem_kind != PM_MEM_HOST && mem_kind != PM_MEM_DEVICE) return fail(m, PM_E_ARG, "bad mem_kind");
  Store& st = m->st;
  hipMemcpyKind k = mem_kind == PM_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
  if (xy) HIPCHK(hipMemcpyAsync(xy, st.xy, sizeof(double2) * st.V, k, m->s));
  if (metric) HIPCHK(hipMemcpyAsync(metric, st.met, sizeof(Met) * st.V, k, m->s));
  if (tags) HIPCHK(hipMemcpyAsync(tags, st.tag, st.V, k, m->s));
  if (valive) HIPCHK(hipMemcpyAsync(valive, st.valive, st.V, k, m->s));
  if (tri || talive) {
    TRY(ensure(m, m->tt0, 3 * (size_t)st.T));
    TRY(ensure(m, m->u8tmp, (size_t)std::max(st.T, 1)));
    export_tri(st, m->tt0.p, m->u8tmp.p, m->s);
    if (tri) HIPCHK(hipMemcpyAsync(tri, m->tt0.p, sizeof(int) * 3 * (size_t)st.T, k, m->s));
    if (talive) HIPCHK(hipMemcpyAsync(talive, m->u8tmp.p, st.T, k, m->s));
  }
  return sync(m);
}

pm_status pm_mesh_rows(pm_mesh* m, int64_t* nn_total, int64_t* ne_total, int64_t* nn_off, int32_t* nn,
                       int64_t* ne_off, int32_t* ne) {
  if (!m || !nn_total || !ne_total) return PM_E_ARG;
  TRY(rows_ready(m));
  Store& st = m->st;
  std::vector<Hdr> hdr(st.V);
  std::vector<int2> cap(st.V);
  HIPCHK(hipMemcpyAsync(hdr.data(), st.hdr, sizeof(Hdr) * st.V, hipMemcpyDeviceToHost, m->s));
  HIPCHK(hipMemcpyAsync(cap.data(), st.cap, sizeof(int2) * st.V, hipMemcpyDeviceToHost, m->s));
  TRY(sync(m));
  int64_t a = 0, b = 0;
  for (int v = 0; v < st.V; ++v) {
    a += hdr[v].y;
    b += hdr[v].w;
    // the row layout the kernels rely on: slots start at multiples of four
    // entries, hold a multiple of four, and hold their row
    const Hdr& h = hdr[v];
    const int2& c = cap[v];
    bool ok = h.x % 4 == 0 && h.z % 4 == 0 && c.x % 4 == 0 && c.y % 4 == 0 && h.y <= c.x && h.w <= c.y &&
              (int64_t)h.x + c.x <= st.nn_pool && (int64_t)h.z + c.y <= st.ne_pool;
    if (!ok) return fail(m, PM_E_DEVICE, "row slot of vertex " + std::to_string(v) + " breaks the layout");
  }
  *nn_total = a;
  *ne_total = b;
  if (!nn_off || !nn || !ne_off || !ne) return PM_OK;
  std::vector<int> pnn(st.nn_pool), pne(st.ne_pool);
  HIPCHK(hipMemcpyAsync(pnn.data(), st.nn, sizeof(int) * st.nn_pool, hipMemcpyDeviceToHost, m->s));
  HIPCHK(hipMemcpyAsync(pne.data(), st.ne, sizeof(int) * st.ne_pool, hipMemcpyDeviceToHost, m->s));
  TRY(sync(m));
  a = b = 0;
  for (int v = 0; v < st.V; ++v) {
    nn_off[v] = a;
    ne_off[v] = b;
    for (int k = 0; k < hdr[v].y; ++k) nn[a++] = pnn[hdr[v].x + k];
    for (int k = 0; k < hdr[v].w; ++k) ne[b++] = pne[hdr[v].z + k];
  }
  nn_off[st.V] = a;
  ne_off[st.V] = b;
  return PM_OK;
}

pm_status pm_colour(pm_mesh* m, const uint8_t* active, uint32_t ctx, int32_t* colour_out, int32_t* ncolours,
                    int32_t mem_kind) {
  if (!m) return PM_E_ARG;
  if (mem_kind != PM_MEM_HOST && mem_kind != PM_MEM_DEVICE) return fail(m, PM_E_ARG, "bad mem_kind");
  TRY(rows_ready(m));
  TRY(ensure_phase_scratch(m));
  Store& st = m->st;
  const uint8_t* act_in = nullptr;
  if (active) {
    TRY(ensure(m, m->u8tmp, st.V));
    HIPCHK(hipMemcpyAsync(m->u8tmp.p, active, st.V,
                          mem_kind == PM_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice, m->s));
    act_in = m->u8tmp.p;
  }
  select_vertices(st, 0, 0.0, act_in, nullptr, m->listA.p, m->ctr, m->sflag.p, m->spart.p,
                  m->s);
  TRY(read_ctr(m, C_LIST_B, 1));
  int n = m->hctr[C_LIST_B];
  Classes cl;
  pm_status r = colour_list(m, m->listA.p, n, Round{stream_seed(m->seed, ctx), m->rw.p}, cl);
  if (r != PM_OK) return round_left(m, r);
  if (ncolours) *ncolours = cl.ncol;
  if (colour_out) {
    TRY(ensure(m, m->vt0, st.V));
    pm::colour_out(st, m->rw.p, m->vt0.p, m->s);
    HIPCHK(hipMemcpyAsync(colour_out, m->vt0.p, sizeof(int) * st.V,
                          mem_kind == PM_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice, m->s));
  }
  clear_round(m->listA.p, n, m->rw.p, nullptr, m->s);
  return sync(m);
}

pm_status pm_coarsen(pm_mesh* m, const pm_options* o, pm_stats* st) {
  if (!m || !o) return PM_E_ARG;
  if (bad_opts(o)) return fail(m, PM_E_ARG, "bad options");
  ++m->topo;
  pm_stats local;
  if (!st) st = &local;
  memset(st, 0, sizeof(*st));
  TRY(run_rounds(m, o, st, 0));
  TRY(compact(m));
  return st->v[7] ? PM_OK : PM_W_NOT_CONVERGED;
}

pm_status pm_swap(pm_mesh* m, const pm_options* o, pm_stats* st) {
  if (!m || !o) return PM_E_ARG;
  if (bad_opts(o)) return fail(m, PM_E_ARG, "bad options");
  ++m->topo;
  pm_stats local;
  if (!st) st = &local;
  memset(st, 0, sizeof(*st));
  TRY(run_rounds(m, o, st, 1));
  return st->v[7] ? PM_OK : PM_W_NOT_CONVERGED;
}

pm_status pm_smooth(pm_mesh* m, const pm_options* o, pm_stats* st) {
  if (!m || !o) return PM_E_ARG;
  if (bad_opts(o)) return fail(m, PM_E_ARG, "bad options");
  pm_stats local;
  if (!st) st = &local;
  memset(st, 0, sizeof(*st));
  TRY(rows_ready(m));
  TRY(ensure_phase_scratch(m));
  m->tune = o->tune;
  stats_zero(m);
  select_vertices(m->st, 3, 0.0, nullptr, nullptr, m->listA.p, m->ctr, m->sflag.p, m->spart.p, m->s);
  TRY(read_ctr(m, C_LIST_B, 1));
  int n = m->hctr[C_LIST_B];
  // (before the colouring, whose round words are cleared at the end)
  if (m->emet.n < (size_t)std::max(m->st.T, 1)) {
    m->emet_topo = 0;
    TRY(ensure(m, m->emet, (size_t)std::max(m->st.T, 1)));
  }
  Classes cl;
  pm_status rc = colour_list(m, m->listA.p, n, Round{stream_seed(m->seed, make_ctx(o->sweep, PH_SMOOTH, 0)), m->rw.p}, cl);
  if (rc != PM_OK) return round_left(m, rc);
  st->v[1] = n;
  st->v[5] = cl.ncol;
  st->v[12] = cl.jp_iters;
  // topology and metrics stay fixed while smoothing: element tensors once,
  // and kept while the topology does not change
  if (m->emet_topo != m->topo) {
    element_metrics(m->st, m->emet.p, m->s);
    m->emet_topo = m->topo;
  }
  m->st.emet = m->emet.p;
  auto sweep_on = [&](hipStream_t q) {
    for (int c = 0; c < cl.ncol; ++c)
      smooth_class(m->st, m->cls.p + cl.off[c], cl.size[c], o->smooth_kind, m->ctr, smooth_lanes(m), q);
  };
  int64_t members = 0;
  for (int c = 0; c < cl.ncol; ++c) members += cl.size[c];
  if (o->smooth_sweeps > 1) {
    // the classes' launches of one sweep, captured once as a graph and
    // replayed for every sweep (they read only the class lists and the store)
    hipGraphExec_t ge = nullptr;
    TRY(capture(m, sweep_on, &ge));
    pm_status r = PM_OK;
    for (int s = 0; s < o->smooth_sweeps && r == PM_OK; ++s) {
      hipError_t e = hipSuccess;
      timed(m, PM_K_SMOOTH, members, [&] { e = hipGraphLaunch(ge, m->s); });
      if (e != hipSuccess) r = fail(m, PM_E_DEVICE, std::string("hipGraphLaunch: ") + hipGetErrorString(e));
    }
    (void)hipGraphExecDestroy(ge);
    TRY(r);
  } else {
    for (int c = 0; c < cl.ncol; ++c)
      timed(m, PM_K_SMOOTH, cl.size[c], [&] {
        smooth_class(m->st, m->cls.p + cl.off[c], cl.size[c], o->smooth_kind, m->ctr, smooth_lanes(m), m->s);
      });
  }
  m->st.emet = nullptr;
  clear_round(m->listA.p, n, m->rw.p, nullptr, m->s);
  TRY(stats_read(m, st));
  st->v[0] = o->smooth_sweeps;
  st->v[7] = 1;
  return PM_OK;
}

pm_status pm_refine(pm_mesh* m, const pm_options* o, pm_stats* st) {
  if (!m || !o) return PM_E_ARG;
  if (bad_opts(o)) return fail(m, PM_E_ARG, "bad options");
  ++m->topo;
  pm_stats local;
  if (!st) st = &local;
  memset(st, 0, sizeof(*st));
  TRY(rows_ready(m));
  stats_zero(m);
  Store& s = m->st;
  int B = s.B;
  int p = 0;
  bool done = false;
  int relayouts = 0;
  // per-mesh flags: a mesh whose pass found nothing to split is finished
  std::vector<int> mdone(B, 0);
  if (B > 1) {
    if (!m->mdone) TRY(dalloc(m, &m->mdone, B));
    HIPCHK(hipMemcpyAsync(m->mdone, mdone.data(), sizeof(int) * B, hipMemcpyHostToDevice, m->s));
    HIPCHK(hipStreamSynchronize(m->s));
    s.mdone = m->mdone;
  }
  while (p < o->refine_passes) {
    int V0 = s.V, T0 = s.T;
    TRY(ensure(m, m->vt0, V0));
    TRY(ensure(m, m->vt1, V0));
    TRY(ensure(m, m->tt0, T0));
    TRY(ensure(m, m->tt1, T0));
    TRY(ensure(m, m->rtmp, 4 * (size_t)B + 4));
    TRY(ensure(m, m->partial, scan_partials_needed(V0) + scan_partials_needed(T0)));
    refine_scan(s, o->L_up2, m->vt0.p, m->vt1.p, m->ctr + C_TOTAL, m->tt0.p, m->tt1.p, m->ctr + C_TOTAL2, m->ctr,
                m->partial.p, m->s);
    std::vector<int> need(2 * B);
    bool aux = 2 * B <= kAuxInts;
    if (B > 1) {
      // per-mesh needs come back with the totals
      range_sums(m->vt1.p, m->vt0.p, s.vbase, s.vused, B, m->rtmp.p, m->s);
      range_sums(m->tt1.p, m->tt0.p, s.tbase, s.tused, B, m->rtmp.p + B, m->s);
      HIPCHK(hipMemcpyAsync(aux ? m->haux : need.data(), m->rtmp.p, sizeof(int) * 2 * B, hipMemcpyDeviceToHost, m->s));
    }
    mail_next(m->mail);
    mail_sum(m->ctr, C_JP, S_EDGES, C_EDGES, m->hctr, m->mail, m->s);
    HIPCHK(mail_wait(m->mail, m->s));
    if (m->prof.mask) TRY(sync(m));
    if (B > 1) TRY(sync(m));
    TRY(check_err(m, true));  // also the last row build's
    int nv = m->hctr[C_TOTAL], nt = m->hctr[C_TOTAL2];
    if (B == 1) need = {nv, nt};
    else if (aux) std::copy(m->haux, m->haux + 2 * B, need.begin());
    int edges = m->hctr[C_EDGES];
    if (nv == 0) {
      st->v[6] += edges;
      done = true;
      break;
    }

    if (B == 1) {
      if ((int64_t)V0 + nv > (1ll << 30) || (int64_t)T0 + nt > (1ll << 30))
        return fail(m, PM_E_NOMEM, "refinement beyond 2^30 vertices or elements");
      TRY(grow_vertices(m, V0 + nv));
      TRY(grow_elements(m, T0 + nt));
    } else {
      bool fits = true;
      for (int i = 0; i < B; ++i)
        fits &= m->vused[i] + need[i] <= m->vbase[i + 1] - m->vbase[i] &&
                m->tused[i] + need[B + i] <= m->tbase[i + 1] - m->tbase[i];
      if (!fits) {
        // a mesh outgrows its range: re-lay the batch out with room, then redo the pass
        if (++relayouts > 1) return fail(m, PM_E_NOMEM, "refinement could not be given room");
        std::vector<int> ev(need.begin(), need.begin() + B), et(need.begin() + B, need.end());
        TRY(compact(m, &ev, &et));
        continue;
      }
    }
    st->v[6] += edges;
    relayouts = 0;
    // meshes whose pass found nothing to split are finished (checked after any relayout)
    bool newly_done = false;
    for (int i = 0; i < B && B > 1; ++i)
      if (!mdone[i] && need[i] == 0) mdone[i] = 1, newly_done = true;
    if (newly_done) {
      HIPCHK(hipMemcpyAsync(m->mdone, mdone.data(), sizeof(int) * B, hipMemcpyHostToDevice, m->s));
      HIPCHK(hipStreamSynchronize(m->s));
    }
    TRY(ensure(m, m->mid, (size_t)s.nn_pool));
    if (B == 1) {
      m->vused[0] = s.V;  // unchanged until the new slots are counted below
      m->tused[0] = s.T;
    }
    refine_mint(s, o->L_up2, m->vt1.p, m->mid.p, m->s);
    refine_split(s, o->L_up2, m->mid.p, m->tt1.p, m->s);
    for (int i = 0; i < B; ++i) {
      m->vused[i] += need[i];
      m->tused[i] += need[B + i];
    }
    if (B == 1) {
      s.V = V0 + nv;
      s.T = T0 + nt;
      m->vbase[1] = s.V;
      m->tbase[1] = s.T;
    }
    TRY(upload_ranges(m));
    st->v[4] += nv;
    st->v[8] += nv;
    st->v[9] += nt;
    ++p;
    // the next pass's read-back checks this build's error bits
    TRY(build_rows(m, p >= o->refine_passes));
  }
  s.mdone = nullptr;
  // the counts above come from the passes' read-backs; the last of those
  // also left the stream drained
  prof_flush(m);
  st->v[0] = p;
  st->v[7] = done ? 1 : 0;
  return done ? PM_OK : PM_W_NOT_CONVERGED;
}

pm_status pm_quality(pm_mesh* m, double* Q, double* qmin, double* dQdx, double* dQdM) {
  if (!m) return PM_E_ARG;
  if (dQdx || dQdM) TRY(rows_ready(m));
  int nparts = quality_parts(m);
  TRY(ensure(m, m->qpart, 2 * (size_t)nparts + 2));
  if (Q || qmin) {
    timed(m, PM_K_QUALITY, m->st.T,
          [&] { mail_next(m->mail); quality_sum(m->st, m->qpart.p, m->qpart.p + nparts, nparts, m->hq, m->mail, m->s); });
  }
  if (dQdx || dQdM) timed(m, PM_K_ADJOINT, m->st.V, [&] { quality_adjoint(m->st, dQdx, dQdM, m->s); });
  // scalars alone come by mail; gradients are complete when the call returns,
  // for any stream
  if (dQdx || dQdM || m->prof.mask || !(Q || qmin)) TRY(sync(m));
  else HIPCHK(mail_wait(m->mail, m->s));
  prof_flush(m);
  if (Q) *Q = m->hq[0];
  if (qmin) *qmin = m->hq[1];
  return PM_OK;
}

pm_status pm_adapt(pm_mesh* m, const pm_options* o, pm_stats* st) {
  if (!m || !o) return PM_E_ARG;
  if (bad_opts(o)) return fail(m, PM_E_ARG, "bad options");
  pm_stats local;
  if (!st) st = &local;
  memset(st, 0, sizeof(*st));
  int run = 0;
  for (;;) {
    if (m->ad_phase == PM_PHASE_COARSEN && m->ad_iter >= o->max_iterations) m->ad_phase = PM_PHASE_SMOOTH;
    if (m->ad_phase == PM_PHASE_DONE) return PM_OK;
    if (o->max_phases > 0 && run == o->max_phases) return PM_W_PAUSED;
    pm_options po = *o;
    po.sweep = m->ad_phase == PM_PHASE_SMOOTH ? 0 : m->ad_iter;
    pm_stats ph;
    pm_status r;
    int phase = m->ad_phase;
    if (phase == PM_PHASE_COARSEN) r = pm_coarsen(m, &po, &ph);
    else if (phase == PM_PHASE_SWAP) r = pm_swap(m, &po, &ph);
    else if (phase == PM_PHASE_REFINE) r = pm_refine(m, &po, &ph);
    else r = pm_smooth(m, &po, &ph);
    if (r != PM_OK && r != PM_W_NOT_CONVERGED) return r;
    for (int k = 1; k < 16; ++k)
      if (k != 7) st->v[k] += ph.v[k];
    if (phase != PM_PHASE_SMOOTH && ph.v[4] > 0) m->ad_changed = 1;
    if (phase == PM_PHASE_COARSEN) {
      m->ad_phase = PM_PHASE_SWAP;
    } else if (phase == PM_PHASE_SWAP) {
      m->ad_phase = PM_PHASE_REFINE;
    } else if (phase == PM_PHASE_REFINE) {
      ++m->ad_iter;
      st->v[0] += 1;
      if (!m->ad_changed) st->v[7] = 1;
      m->ad_phase = m->ad_changed ? PM_PHASE_COARSEN : PM_PHASE_SMOOTH;
      m->ad_changed = 0;
    } else {
      m->ad_phase = PM_PHASE_DONE;
    }
    ++run;
  }
}

pm_status pm_get_context(const pm_mesh* m, pm_context* c) {
  if (!m || !c) return PM_E_ARG;
  c->seed = m->seed;
  c->iteration = m->ad_iter;
  c->phase = m->ad_phase;
  c->changed = m->ad_changed;
  c->reserved = 0;
  return PM_OK;
}

pm_status pm_set_context(pm_mesh* m, const pm_context* c) {
  if (!m || !c) return PM_E_ARG;
  if (c->iteration < 0 || c->iteration > 4095 || c->phase < PM_PHASE_COARSEN || c->phase > PM_PHASE_DONE ||
      (c->changed != 0 && c->changed != 1) || c->reserved != 0)
    return fail(m, PM_E_ARG, "bad context");
  m->seed = c->seed;
  m->ad_iter = c->iteration;
  m->ad_phase = c->phase;
  m->ad_changed = c->changed;
  return PM_OK;
}

pm_status pm_mesh_update(pm_mesh* m, const double* xy, const double* metric, int32_t mem_kind) {
  if (!m) return PM_E_ARG;
  if (mem_kind != PM_MEM_HOST && mem_kind != PM_MEM_DEVICE) return fail(m, PM_E_ARG, "bad mem_kind");
  if (m->st.B != 1) return fail(m, PM_E_ARG, "pm_mesh_update takes a single mesh");
  if (!xy && !metric) return PM_OK;
  Store& st = m->st;
  size_t V = (size_t)st.V;
  hipMemcpyKind k = mem_kind == PM_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
  // the new values are checked in blocks of their own, which then take the
  // place of the old ones; a refused update leaves the mesh untouched
  Store nst = st;
  if (xy) {
    TRY(ensure(m, m->upx, (size_t)st.Vcap));
    nst.xy = m->upx.p;
    HIPCHK(hipMemcpyAsync(nst.xy, xy, sizeof(double2) * V, k, m->s));
  }
  if (metric) {
    TRY(ensure(m, m->upm, (size_t)st.Vcap));
    nst.met = m->upm.p;
    HIPCHK(hipMemcpyAsync(nst.met, metric, sizeof(Met) * V, k, m->s));
  }
  k_validate(nst, m->ctr, m->s);
  TRY(check_err(m));
  if (xy) {
    std::swap(st.xy, m->upx.p);
    m->upx.n = (size_t)st.Vcap;
  }
  if (metric) {
    std::swap(st.met, m->upm.p);
    m->upm.n = (size_t)st.Vcap;
  }
  ++m->topo;  // the per-element tensors smoothing keeps follow the metric
  return PM_OK;
}

pm_status pm_quality_noalloc(pm_mesh* m, double* Q, double* qmin, double* dQdx, double* dQdM) {
  if (!m) return PM_E_ARG;
  int nparts = quality_parts(m);
  if (nparts > kQualityParts)  // cannot happen for a handle this library made (T < 2^30)
    return fail(m, PM_E_ARG, "pm_quality_noalloc: more than " + std::to_string(kQualityParts) + " partial sums");
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (!m->scratch || dev != m->dev)
    return fail(m, PM_E_ARG, "pm_quality_noalloc: call it with the handle's device current");
  if ((dQdx || dQdM) && !m->rows_ok)
    return fail(m, PM_E_NOMEM, "pm_quality_noalloc: the rows' last build found no memory (pm_quality builds them)");
  double* ps = m->scratch;
  if (Q || qmin) {
    mail_next(m->mail);
    quality_sum(m->st, ps, ps + nparts, nparts, m->hq, m->mail, m->s);
  }
  if (dQdx || dQdM) quality_adjoint(m->st, dQdx, dQdM, m->s);
  HIPCHK(hipStreamSynchronize(m->s));
  if (Q) *Q = m->hq[0];
  if (qmin) *qmin = m->hq[1];
  return PM_OK;
}

namespace {
// host arrays to consecutive places on the device (each padded to 16 bytes),
// through two pinned blocks in turn
struct Upload {
  char* dst;
  hipStream_t s;
  char* block[2] = {nullptr, nullptr};
  hipEvent_t ev[2] = {nullptr, nullptr};
  bool busy[2] = {false, false};
  int cur = 0;
  size_t at = 0;
  Upload(char* d, hipStream_t stream) : dst(d), s(stream) {}
  Upload(const Upload&) = delete;
  ~Upload() { done(); }
  bool flush() {
    if (at == 0) return true;
    if (hipMemcpyAsync(dst, block[cur], at, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipEventRecord(ev[cur], s) != hipSuccess)
      return false;
    busy[cur] = true;
    dst += at;
    at = 0;
    cur ^= 1;
    return true;
  }
  bool put(const void* src, size_t n) {
    const char* from = (const char*)src;
    size_t pad = (16 - n % 16) % 16;
    while (n + pad > 0) {
      if (at == 0) {
        if (!block[cur]) {
          block[cur] = (char*)pm::stage_take();
          if (!block[cur]) {  // no pinned memory: straight from the caller's, which outlives the copy
            bool ok = n == 0 || hipMemcpyAsync(dst, from, n, hipMemcpyHostToDevice, s) == hipSuccess;
            dst += n + pad;
            return ok;
          }
          if (hipEventCreateWithFlags(&ev[cur], hipEventDisableTiming) != hipSuccess) return false;
        }
        if (busy[cur] && hipEventSynchronize(ev[cur]) != hipSuccess) return false;
        busy[cur] = false;
      }
      size_t k = std::min(n, pm::kStageBytes - at);
      memcpy(block[cur] + at, from, k);
      from += k;
      n -= k;
      at += k;
      if (n == 0) {
        k = std::min(pad, pm::kStageBytes - at);
        memset(block[cur] + at, 0, k);
        pad -= k;
        at += k;
      }
      if (at == pm::kStageBytes && !flush()) return false;
    }
    return true;
  }
  // once the stream is past the copies
  void done() {
    for (int k = 0; k < 2; ++k) {
      if (busy[k]) (void)hipEventSynchronize(ev[k]);
      busy[k] = false;
      if (ev[k]) (void)hipEventDestroy(ev[k]);
      ev[k] = nullptr;
      pm::stage_give(block[k]);
      block[k] = nullptr;
    }
  }
};
}  // namespace

pm_status pm_batch_create(const pm_mesh_desc* meshes, int32_t count, const pm_options* o, void* stream,
                          pm_mesh** out) {
  if (!out) return PM_E_ARG;
  *out = nullptr;
  if (!meshes || count < 1) return PM_E_ARG;
  pm_options def;
  fill_defaults(&def);
  if (!o) o = &def;
  if (bad_opts(o)) return PM_E_ARG;
  std::vector<int> vb(count + 1, 0), tb(count + 1, 0), vu(count), tu(count);
  for (int i = 0; i < count; ++i) {
    const pm_mesh_desc& d = meshes[i];
    if (!d.xy || !d.tri || !d.metric || d.mem_kind != PM_MEM_HOST || d.V < 3 || d.T < 1) return PM_E_ARG;
    // (one mesh is packed and grown like any single one)
    int64_t cv = d.V + (count > 1 ? headroom((int)std::min<int64_t>(d.V, 1 << 29)) : 0);
    int64_t ct = d.T + (count > 1 ? headroom((int)std::min<int64_t>(d.T, 1 << 29)) : 0);
    if (vb[i] + cv > (1ll << 30) || tb[i] + ct > (1ll << 30)) return PM_E_ARG;
    vu[i] = (int)d.V;
    tu[i] = (int)d.T;
    vb[i + 1] = vb[i] + (int)cv;
    tb[i + 1] = tb[i] + (int)ct;
  }
  int nV = vb[count], nT = tb[count];
  // the caller's arrays go up as they are, one mesh behind the other, a table of
  // their places first
  std::vector<BatchIn> in(count);
  int64_t bytes = 0;
  auto take = [&](int64_t n) {
    int64_t at = bytes;
    bytes += (n + 15) / 16 * 16;
    return at;
  };
  take(sizeof(BatchIn) * count);
  for (int i = 0; i < count; ++i) {
    const pm_mesh_desc& d = meshes[i];
    in[i].xy = take(sizeof(double) * 2 * d.V);
    in[i].met = take(sizeof(double) * 3 * d.V);
    in[i].tri = take(sizeof(int) * 3 * d.T);
    in[i].tag = d.tags ? take(d.V) : -1;
  }
  g_create_err.clear();
  pm_mesh* m = new (std::nothrow) pm_mesh();
  if (!m) return PM_E_NOMEM;
  m->s = (hipStream_t)stream;
  m->seed = o->seed;
  m->slack = o->slack;
  m->headroom = o->pool_headroom > 0.0 ? o->pool_headroom : 3.0;
  m->st.qk = o->quality;
  if (o->allocator) m->va = *o->allocator;
  auto bail = [&](pm_status st) {
    g_create_err = m->err.empty() ? std::string("pm_batch_create failed") : m->err;
    pm_mesh_destroy(m);
    return st;
  };
  if (dalloc(m, &m->ctr, C_COUNT) != PM_OK || !pinned_get(m)) return bail(PM_E_NOMEM);
  if (scratch_setup(m) != PM_OK) return bail(PM_E_DEVICE);
  zero_ints(m->ctr, C_COUNT, m->s);
  set_int(m->ctr + C_FAILEP, INT_MAX, m->s);
  Store& st = m->st;
  st.B = count;
  if (grow_vertices(m, nV) != PM_OK || grow_elements(m, nT) != PM_OK) return bail(PM_E_NOMEM);
  st.V = nV;
  st.T = nT;
  if (count > 1 && (dalloc(m, &st.vmesh, nV) != PM_OK || dalloc(m, &st.tmesh, nT) != PM_OK)) return bail(PM_E_NOMEM);
  m->vbase = vb;
  m->tbase = tb;
  m->vused = vu;
  m->tused = tu;
  pm_status r = upload_ranges(m);
  if (r != PM_OK) return bail(r);
  if (count == 1) build_start(nullptr, m->ranges, vu[0], tu[0], nV, nT, m->s);
  char* raw = nullptr;
  if (dalloc(m, &raw, bytes) != PM_OK) return bail(PM_E_NOMEM);
  Upload up(raw, m->s);
  bool ok = up.put(in.data(), sizeof(BatchIn) * count);
  for (int i = 0; i < count && ok; ++i) {
    const pm_mesh_desc& d = meshes[i];
    ok = up.put(d.xy, sizeof(double) * 2 * d.V) && up.put(d.metric, sizeof(double) * 3 * d.V) &&
         up.put(d.tri, sizeof(int) * 3 * d.T) && (!d.tags || up.put(d.tags, d.V));
  }
  ok = ok && up.flush();
  if (ok) {
    batch_in(raw, count, st, m->ctr, m->s);
    k_validate(st, m->ctr, m->s);
  }
  // (the copies have left the staging blocks)
  r = ok ? read_ctr(m, 0, kRoundCtrs) : fail(m, PM_E_DEVICE, "upload of the batch");
  if (r != PM_OK) (void)hipStreamSynchronize(m->s);
  up.done();
  dfree(m, raw, bytes);
  if (r != PM_OK) return bail(r);
  if (m->hctr[C_FAILEP] != INT_MAX) {
    m->err = "mesh " + std::to_string(m->hctr[C_FAILEP]) + ": element id out of range";
    return bail(PM_E_MESH);
  }
  r = check_err(m, true);
  if (r != PM_OK) return bail(r);
  r = build_rows(m);
  if (r != PM_OK) return bail(r);
  *out = m;
  return PM_OK;
}

pm_status pm_batch_count(const pm_mesh* m, int32_t* count) {
  if (!m || !count) return PM_E_ARG;
  *count = m->st.B;
  return PM_OK;
}

pm_status pm_batch_sizes(const pm_mesh* m, int32_t i, int64_t* V, int64_t* T) {
  if (!m || i < 0 || i >= m->st.B) return PM_E_ARG;
  if (V) *V = m->vused[i];
  if (T) *T = m->tused[i];
  return PM_OK;
}

pm_status pm_batch_export(pm_mesh* m, int32_t i, double* xy, int32_t* tri, double* metric, uint8_t* tags,
                          uint8_t* valive, uint8_t* talive) {
  if (!m || i < 0 || i >= m->st.B) return PM_E_ARG;
  Store& st = m->st;
  int v0 = m->vbase[i], nv = m->vused[i], t0 = m->tbase[i], nt = m->tused[i];
  // one launch that writes what is asked for into pinned memory, local ids and
  // all, where a block of it holds the mesh: five copies to pageable memory and a
  // pass over the elements took 94 us a mesh of 250 KB, this takes 33
  BatchOut bo{};
  int64_t bytes = 0;
  auto take = [&](bool on, int64_t n) {
    if (!on) return (int64_t)-1;
    int64_t at = bytes;
    bytes += (n + 15) / 16 * 16;
    return at;
  };
  bo.xy = take(xy, sizeof(double2) * (int64_t)nv);
  bo.met = take(metric, sizeof(Met) * (int64_t)nv);
  bo.tri = take(tri, sizeof(int) * 3 * (int64_t)nt);
  bo.tag = take(tags, nv);
  bo.valive = take(valive, nv);
  bo.talive = take(talive, nt);
  char* b = bytes <= (int64_t)kStageBytes ? (char*)stage_take() : nullptr;
  if (b) {
    batch_out(st, v0, nv, t0, nt, bo, b, m->s);
    mail_send(m->mail, m->ctr, 0, m->hctr, m->s);
    hipError_t e = mail_wait(m->mail, m->s);
    if (e != hipSuccess) (void)hipStreamSynchronize(m->s);
    if (e == hipSuccess) {
      if (xy) memcpy(xy, b + bo.xy, sizeof(double2) * nv);
      if (metric) memcpy(metric, b + bo.met, sizeof(Met) * nv);
      if (tri) memcpy(tri, b + bo.tri, sizeof(int) * 3 * nt);
      if (tags) memcpy(tags, b + bo.tag, nv);
      if (valive) memcpy(valive, b + bo.valive, nv);
      if (talive) memcpy(talive, b + bo.talive, nt);
    }
    stage_give(b);
    HIPCHK(e);
    if (m->prof.mask) TRY(sync(m));
    return PM_OK;
  }
  if (xy) HIPCHK(hipMemcpyAsync(xy, st.xy + v0, sizeof(double2) * nv, hipMemcpyDeviceToHost, m->s));
  if (metric) HIPCHK(hipMemcpyAsync(metric, st.met + v0, sizeof(Met) * nv, hipMemcpyDeviceToHost, m->s));
  if (tags) HIPCHK(hipMemcpyAsync(tags, st.tag + v0, nv, hipMemcpyDeviceToHost, m->s));
  if (valive) HIPCHK(hipMemcpyAsync(valive, st.valive + v0, nv, hipMemcpyDeviceToHost, m->s));
  std::vector<Elem> e(nt);
  HIPCHK(hipMemcpyAsync(e.data(), st.tri + t0, sizeof(Elem) * nt, hipMemcpyDeviceToHost, m->s));
  TRY(sync(m));
  for (int t = 0; t < nt; ++t) {
    if (tri) {
      tri[3 * t] = e[t].w ? e[t].x - v0 : e[t].x;
      tri[3 * t + 1] = e[t].w ? e[t].y - v0 : e[t].y;
      tri[3 * t + 2] = e[t].w ? e[t].z - v0 : e[t].z;
    }
    if (talive) talive[t] = e[t].w ? 1 : 0;
  }
  return PM_OK;
}

pm_status pm_batch_quality(pm_mesh* m, double* Q, double* qmin) {
  if (!m) return PM_E_ARG;
  int B = m->st.B;
  TRY(ensure(m, m->qpart, 2 * (size_t)B + 2));
  quality_per_mesh(m->st, m->qpart.p, m->s);
  std::vector<double> h(2 * (size_t)B);
  HIPCHK(hipMemcpyAsync(h.data(), m->qpart.p, sizeof(double) * 2 * B, hipMemcpyDeviceToHost, m->s));
  TRY(sync(m));
  for (int i = 0; i < B; ++i) {
    if (Q) Q[i] = h[2 * i];
    if (qmin) qmin[i] = h[2 * i + 1];
  }
  return PM_OK;
}

pm_status pm_profile(pm_mesh* m, uint32_t mask) {
  if (!m) return PM_E_ARG;
  TRY(sync(m));
  prof_flush(m);
  m->prof.mask = mask;
  for (int k = 0; k < PM_K_COUNT; ++k) {
    m->prof.ms[k] = 0.0;
    m->prof.launches[k] = m->prof.units[k] = 0;
  }
  stripe_zero(m->ctr, S_PJP, 2, m->s);
  stripe_zero(m->ctr, S_POPS, 1, m->s);
  return sync(m);
}

pm_status pm_profile_read(pm_mesh* m, int32_t id, double* ms, int64_t* launches, int64_t* units) {
  if (!m || id < 0 || id > PM_K_COMMIT_OPS) return PM_E_ARG;
  TRY(sync(m));
  prof_flush(m);
  stripe_sum(m->ctr, S_PJP, 2, C_PROF_JP, m->s);
  stripe_sum(m->ctr, S_POPS, 1, C_PROF_OPS, m->s);
  TRY(read_ctr(m, C_PROF_JP, 3));
  int k = id == PM_K_COMMIT_OPS ? PM_K_COMMIT : id;
  if (ms) *ms = m->prof.ms[k];
  if (launches) *launches = m->prof.launches[k];
  if (units) {
    *units = m->prof.units[k];
    if (id == PM_K_JP) *units = m->hctr[C_PROF_JP];
    if (id == PM_K_COMMIT) *units = m->hctr[C_PROF_ROWS];
    if (id == PM_K_COMMIT_OPS) *units = m->hctr[C_PROF_OPS];
  }
  return PM_OK;
}

pm_status pm_fp64_selfcheck(const double* a, const double* b, int64_t n, double* quot, double* root) {
  if (!a || !b || !quot || !root || n < 0 || n > (1ll << 28)) return PM_E_ARG;
  if (n == 0) return PM_OK;
  double* d = nullptr;
  size_t bytes = sizeof(double) * (size_t)n;
  if (hipMalloc((void**)&d, 4 * bytes) != hipSuccess) return PM_E_NOMEM;
  bool ok = hipMemcpy(d, a, bytes, hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(d + n, b, bytes, hipMemcpyHostToDevice) == hipSuccess;
  if (ok) {
    fp64_probe(d, d + n, (int)n, d + 2 * n, d + 3 * n, nullptr);
    ok = hipDeviceSynchronize() == hipSuccess &&
         hipMemcpy(quot, d + 2 * n, bytes, hipMemcpyDeviceToHost) == hipSuccess &&
         hipMemcpy(root, d + 3 * n, bytes, hipMemcpyDeviceToHost) == hipSuccess;
  }
  (void)hipFree(d);
  return ok ? PM_OK : PM_E_DEVICE;
}

}  // extern "C"
