// Adaptation kernels: Jones-Plassmann colouring, colour-class lists, the four
// operations (collapse, flip, smoothing; refinement lives in store.hip), the
// deferred-update commit and the quality functional with its adjoint.
//
// Round structure (Sec. 3.2-3.4): the active vertices are coloured once per
// round; the colour classes run one kernel after another. A class kernel
// re-validates each member against same-class neighbours in the current
// graph, evaluates its operation from the state left by the previous class,
// rewrites only elements the member owns, marks the adjacency rows it touches
// dirty and queues the additions those rows need. The commit then lets the
// owner of each dirty row rebuild it, so no two threads ever write one row.
#include <algorithm>
#include <atomic>

#include "kern.hpp"
#include "scan.hpp"

namespace pm {

constexpr int kG = 8;    // lanes per vertex in the lane-group kernels
constexpr int kGC = 16;  // lanes per vertex in the lane-group collapse

__device__ __forceinline__ uint64_t key_of(const Store& st, const Round& rd, int v) {
  return vkey(rd.sseed, (uint32_t)local_id(st, v));
}
__device__ __forceinline__ void rw_put(uint64_t* rw, int v, uint64_t x) { ((volatile uint64_t*)rw)[v] = x; }

__global__ void k_clear_round(const int* __restrict__ list, int n, uint64_t* __restrict__ rw, int* zero) {
  if (zero && blockIdx.x == 0 && threadIdx.x == 0) *zero = 0;
  for (int i = gtid(); i < n; i += gstride()) rw[list[i]] = 0;
}
void clear_round(const int* list, int n, uint64_t* rw, int* zero, hipStream_t s) {
  if (n > 0) k_clear_round<<<grid_for(n), kBlock, 0, s>>>(list, n, rw, zero);
}
// ---- lists -----------------------------------------------------------------------------
__device__ bool has_candidate(const Store& st, int v, double L_low2) {
  Hdr h = st.hdr[v];
  double2 pv = st.xy[v];
  Met mv = st.met[v];
  uint8_t tv = st.tag[v];
  for (int j = 0; j < h.y; ++j) {
    int u = st.nn[h.x + j];
    if (tv & ~st.tag[u]) continue;
    if (len2(pv, mv, st.xy[u], st.met[u]) < L_low2) return true;
  }
  return false;
}

// mode: 0 colour (active flags or all live), 1 coarsen (has a short edge),
// 2 swap (all live), 3 smooth (live interior)
__device__ __forceinline__ bool want(const Store& st, int v, int mode, double L_low2, const uint8_t* active) {
  if (!st.valive[v]) return false;
  switch (mode) {
    case 0: return active ? active[v] != 0 : true;
    case 1: return has_candidate(st, v, L_low2);
    case 2: return true;
    default: return st.tag[v] == 0;
  }
}

// Every vertex v with (nxt == null or nxt[v]) and want(v); clears nxt.
// After a commit that ran out of room (the rows are being rebuilt) it selects
// nothing and leaves the flags for the selection that follows the rebuild.
// The selected vertices in ascending id order (an ordered compaction), so that
// lists and the colour classes cut from them follow the mesh's layout.
void select_vertices(const Store& store, int mode, double L_low2, const uint8_t* active, uint8_t* nxt, int* out,
                     int* ctr, int* flag, int* partial, hipStream_t s) {
  Store st = store;
  scan_fused<int, 1>(
      [=] __device__(int v, bool on) {
        if (!on) return 0;
        int f = 0;
        if (!nxt || !room_failed(ctr)) {
          bool sel = nxt ? nxt[v] != 0 : true;
          if (nxt && sel) nxt[v] = 0;
          f = sel && want(st, v, mode, L_low2, active) ? 1 : 0;
        }
        flag[v] = f;
        return f;
      },
      [=] __device__(int v) { return flag[v]; },
      [=] __device__(int v, int at, int f) {
        if (f) out[at] = v;
      },
      [=] __device__(int t) { ctr[C_LIST_B] = t; }, st.V, partial, s);
}

// ---- Jones-Plassmann colouring (Sec. 3.2) ------------------------------------------------
__global__ void k_jp_init(Store st, const int* __restrict__ A, int n, Round rd, int* ctr) {
  if (blockIdx.x == 0 && threadIdx.x < kStripes)
    for (int k = 0; k < 8; ++k) ctr[C_STRIPE + threadIdx.x * kStripeW + S_JPL + k] = 0;
  for (int i = gtid(); i < n; i += gstride()) {
    int v = A[i];
    uint64_t prio = key_of(st, rd, v) >> 32;
    rd.rw[v] = (prio << 32) | kRwAct | 0xFFull;
  }
}
void jp_init(const Store& st, const int* A, int n, Round rd, int* ctr, hipStream_t s) {
  if (n > 0) k_jp_init<<<grid_for(n), kBlock, 0, s>>>(st, A, n, rd, ctr);
}

// start of device-driven rounds: round r, next epoch, last stamp; the
// accumulated statistics cleared
__global__ void k_dev_rounds_start(int* ctr, int r, int epoch, int mark, int stop) {
  if (threadIdx.x == 0) {
    ctr[C_DROUND] = r;
    ctr[C_DEPOCH] = epoch;
    ctr[C_DEPOCH0] = epoch;
    ctr[C_DMARK] = mark;
    ctr[C_DSTOP] = stop;
    ctr[C_ACC_COL] = 0;
    ctr[C_ACC_NCOL] = 0;
    ctr[C_ACC_IT] = 0;
  }
}
void dev_rounds_start(int* ctr, int r, int epoch, int mark, int stop, hipStream_t s) {
  k_dev_rounds_start<<<1, 64, 0, s>>>(ctr, r, epoch, mark, stop);
}

// round words of a coloured list again, from its class lists (the list is
// the classes' union, class c holds the vertices of colour c)
__global__ void k_restore_round(Store st, const int* __restrict__ cls, int n, const int* __restrict__ off, int ncol,
                                Round rd) {
  for (int i = gtid(); i < n; i += gstride()) {
    int c = 0;
    while (c + 1 < ncol && off[c + 1] <= i) ++c;
    int v = cls[i];
    uint64_t prio = key_of(st, rd, v) >> 32;
    rd.rw[v] = (prio << 32) | kRwAct | (uint64_t)c;
  }
}
void restore_round(const Store& st, const int* cls, int n, const int* off, int ncol, Round rd, hipStream_t s) {
  if (n > 0) k_restore_round<<<grid_for(n), kBlock, 0, s>>>(st, cls, n, off, ncol, rd);
}

// A vertex is ready once every active neighbour of larger key has a colour;
// it then takes the smallest colour none of them has. Colours read while a
// neighbour is being written are either unset (not ready yet) or final, so
// the result does not depend on timing. Returns false while v must wait.
// blocker: in, a neighbour that kept v waiting before (or -1); out, the
// neighbour that keeps it waiting now. While that neighbour has no colour, v
// cannot be ready, and one load settles the visit.
// The round words are read through the caches. At a launch's start
// every colour set before it is visible; a colour set during the launch may
// read as unset, which only makes v wait (priorities and active bits do not
// change during the colouring), and the vertex of largest key still waiting
// is ready at every launch, so each chunked launch makes progress.
// LIVE: round words change under the loop that calls this (solve_items), so
// they are read as atomics of the work-group.
template <bool LIVE>
__device__ __forceinline__ uint64_t rw_get(const uint64_t* rw, int v) {
  if constexpr (LIVE) return __hip_atomic_load(rw + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return rw[v];
}
template <bool LIVE = false>
__device__ bool jp_try(const Store& st, int v, const Round& rd, int* ctr, int& blocker) {
  constexpr int B = 8;  // neighbours fetched side by side
  const uint64_t* rw = rd.rw;
  if (!LIVE && blocker >= 0 && (rw[blocker] & 0xFF) == 0xFF) return false;
  uint64_t rv = rw[v];
  Hdr h = st.hdr[v];
  uint64_t used = 0;
  bool big = false;
  for (int j0 = 0; j0 < h.y; j0 += B) {
    int w[B];
    uint64_t x[B];
    row8(st.nn, h.x + j0, h.y - j0, w);
#pragma unroll
    for (int q = 0; q < B; ++q) x[q] = w[q] >= 0 ? rw_get<LIVE>(rw, w[q]) : 0ull;
    int wait = -1;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      if (!(x[q] & kRwAct) || !rw_beats(x[q], w[q], rv, v)) continue;
      int c = (int)(x[q] & 0xFF);
      if (c == 0xFF) wait = wait < 0 ? w[q] : wait;
      else if (c < 64) used |= 1ull << c;
      else big = true;
    }
    if (wait >= 0) {
      blocker = wait;
      return false;
    }
  }
  int c;
  if (~used != 0ull && !big) {
    c = __ffsll((unsigned long long)~used) - 1;
  } else {
    // slow path: colours beyond 63 among the neighbours
    c = 0;
    for (;;) {
      bool taken = false;
      for (int j = 0; j < h.y && !taken; ++j) {
        int w = st.nn[h.x + j];
        uint64_t x = rw_get<LIVE>(rw, w);
        if (!(x & kRwAct) || !rw_beats(x, w, rv, v)) continue;
        taken = (int)(x & 0xFF) == c;
      }
      if (!taken) break;
      ++c;
    }
  }
  if (c >= kMaxColours) {
    atomicOr(&ctr[C_ERR], E_COLOURS);
    c = kMaxColours - 1;
  }
  rw_put(rd.rw, v, (rv & ~0xFFull) | (uint64_t)c);
  return true;
}

// One block per chunk; each thread takes R entries (item r of thread
// t is entry r * kBlock + t). The waiting vertices are packed to the front of
// the chunk in their old order: every read happens before the block barrier,
// every write after it, so the compaction can run in place. One atomic per
// chunk (on a stripe) counts what is left.
constexpr int kJpLocal = 3;  // passes per launch over a chunk that makes progress
template <int R>
__global__ void __launch_bounds__(256) k_jp_chunk(Store st, const int* __restrict__ A, int n, int* W, int* WB,
                                                  int* __restrict__ cnt, int first, Round rd, int* ctr, int slot,
                                                  int next_slot) {
  constexpr int kChunk = R * kBlock;
  __shared__ int wtot[R][kBlock / kWave];
  int kb = xcd_block();
  if (blockIdx.x == 0 && threadIdx.x < kStripes) ctr[C_STRIPE + threadIdx.x * kStripeW + next_slot] = 0;
  int m = first ? min(kChunk, n - kb * kChunk) : cnt[kb];
  if (m <= 0) {
    if (first && threadIdx.x == 0) cnt[kb] = 0;
    return;
  }
  const int* in = (first ? A : W) + (size_t)kb * kChunk;
  const int* inb = WB + (size_t)kb * kChunk;
  int vv[R], bl[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int i = r * kBlock + (int)threadIdx.x;
    vv[r] = i < m ? in[i] : -1;
    bl[r] = (i < m && !first) ? inb[i] : -1;
  }
  bool keep[R];
  int tries = 0;  // this thread's vertex visits, for the profile's unit count
  bool moved = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    keep[r] = vv[r] >= 0 && !jp_try(st, vv[r], rd, ctr, bl[r]);
    moved |= vv[r] >= 0 && !keep[r];
    tries += vv[r] >= 0 ? 1 : 0;
  }
  // more passes over the chunk's waiting vertices while the chunk makes
  // progress: chains of neighbours inside the chunk resolve in one launch
  for (int pass = 1; pass < kJpLocal; ++pass) {
    bool waiting = false;
#pragma unroll
    for (int r = 0; r < R; ++r) waiting |= keep[r];
    if (!__syncthreads_or(moved && waiting)) break;
    moved = false;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (keep[r]) {
        ++tries;
        keep[r] = !jp_try(st, vv[r], rd, ctr, bl[r]);
        moved |= !keep[r];
      }
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) tries += __shfl_xor(tries, d);
  int lane = __lane_id(), wv = (int)threadIdx.x / kWave;
  uint64_t bal[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    bal[r] = __ballot(keep[r]);
    if (lane == 0) wtot[r][wv] = __popcll(bal[r]);
  }
  __syncthreads();
  int base = 0, pos[R];
  uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int before = 0, row = 0;
#pragma unroll
    for (int q = 0; q < kBlock / kWave; ++q) {
      int c = wtot[r][q];
      row += c;
      if (q < wv) before += c;
    }
    pos[r] = base + before + __popcll(bal[r] & below);
    base += row;
  }
  int* out = W + (size_t)kb * kChunk;
  int* outb = WB + (size_t)kb * kChunk;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (keep[r]) {
      out[pos[r]] = vv[r];
      outb[pos[r]] = bl[r];
    }
  if (threadIdx.x == 0) {
    cnt[kb] = base;
    int* sp = ctr + C_STRIPE + (kb & (kStripes - 1)) * kStripeW;
    if (base) atomicAdd(sp + slot, base);
  }
  if (lane == 0 && tries) atomicAdd(stripe_ptr(ctr, S_PJP), tries);
}

// Entries per chunk: 512 for long lists (a chunk resolves chains of neighbours
// inside it, and the launch is bound by the rows' line look-ups on full CUs),
// 256 for lists whose blocks are then all resident at once (66,000 vertices are
// 130 blocks of 512 on 256 CUs, each CU bound by its own look-ups).
int jp_chunk_of(int n) { return n <= kJpShort ? kBlock : 2 * kBlock; }

void jp_chunk(const Store& st, const int* A, int n, int* W, int* WB, int* cnt, bool first, Round rd, int* ctr,
              int it, hipStream_t s) {
  int chunk = jp_chunk_of(n), nch = (n + chunk - 1) / chunk;
  if (nch <= 0) return;
  auto k = chunk == kBlock ? k_jp_chunk<1> : k_jp_chunk<2>;
  k<<<nch, kBlock, 0, s>>>(st, A, n, W, WB, cnt, first ? 1 : 0, rd, ctr, S_JPL + (it & 7), S_JPL + ((it + 1) & 7));
}

// ---- striped counters --------------------------------------------------------------------------
__global__ void k_stripe_zero(int* ctr, int slot, int nslots) {
  int w = (int)threadIdx.x;
  for (int k = 0; k < nslots; ++k) ctr[C_STRIPE + w * kStripeW + slot + k] = 0;
}
void stripe_zero(int* ctr, int slot, int nslots, hipStream_t s) {
  k_stripe_zero<<<1, kStripes, 0, s>>>(ctr, slot, nslots);
}
__global__ void k_stripe_sum(int* ctr, int slot, int nslots, int dst) {
  int w = (int)threadIdx.x;
  for (int k = 0; k < nslots; ++k) {
    int x = ctr[C_STRIPE + w * kStripeW + slot + k];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
    if (w == 0) ctr[dst + k] = x;
  }
}
__global__ void k_phase_start(int* ctr) {
  for (int k = 0; k < 6; ++k) ctr[C_STRIPE + threadIdx.x * kStripeW + S_EVAL + k] = 0;
  if (threadIdx.x == 0) ctr[C_FAILEP] = INT_MAX;
}
void phase_start(int* ctr, hipStream_t s) { k_phase_start<<<1, kStripes, 0, s>>>(ctr); }
__global__ void k_stripe_mail(const int* ctr, int slot, int nslots, int* dst, int* at, int no) {
  for (int k = 0; k < nslots; ++k) {
    int x = ctr[C_STRIPE + threadIdx.x * kStripeW + slot + k];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
    if (threadIdx.x == 0) dst[k] = x;
  }
  mail_post(at, no);
}
void stripe_mail(const int* ctr, int slot, int nslots, int* dst, const Mail& b, hipStream_t s) {
  k_stripe_mail<<<1, kStripes, 0, s>>>(ctr, slot, nslots, dst, (int*)b.at, b.no);
}
// the first n counters to the host, with a striped count's sum in the place of
// ctr[where]; the stripes start again at zero
__global__ void k_mail_sum(int* ctr, int n, int slot, int where, int* dst, int* at, int no) {
  for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x)
    if (i != where) dst[i] = ctr[i];
  int* mine = &ctr[C_STRIPE + threadIdx.x * kStripeW + slot];
  int x = *mine;
  *mine = 0;
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
  if (threadIdx.x == 0) dst[where] = x;
  mail_post(at, no);
}
void mail_sum(int* ctr, int n, int slot, int where, int* dst, const Mail& b, hipStream_t s) {
  k_mail_sum<<<1, kStripes, 0, s>>>(ctr, n, slot, where, dst, (int*)b.at, b.no);
}
void stripe_sum(int* ctr, int slot, int nslots, int dst, hipStream_t s) {
  static_assert(kStripes == kWave, "one lane per stripe");
  k_stripe_sum<<<1, kStripes, 0, s>>>(ctr, slot, nslots, dst);
}

// Class lists by a stable counting sort on the colour: per block (256 list
// entries) the number of each colour, an exclusive scan over (colour, block),
// then every entry goes to its colour's range at the position of its rank
// among equal colours in the block. Class lists keep the order of A.
// Class lists for colours below CM: per block a colour histogram in LDS,
// the (colour, block) table scanned in colour-major order, then each vertex
// placed at its colour's block offset plus its rank in the block. A block
// that meets a colour of CM or more stores seq to ctr[C_CWIDE] (only while it
// does not hold seq yet); the lists then report -2 colours, and the caller
// cuts them again with CM = 256. With CM = 32 the scanned table is an eighth
// of the full one.
template <int CM>
__global__ void k_class_count(const int* __restrict__ A, int n, const uint64_t* __restrict__ rw, int nb,
                              int* __restrict__ tab, int* ctr, int seq) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) atomicAdd(&h[(int)(rw[A[i]] & 0xFF)], 1);
  __syncthreads();
  if ((int)threadIdx.x < CM) tab[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
  if (CM < 256) {
    bool wide = (int)threadIdx.x >= CM && h[threadIdx.x] > 0;
    if (__ballot(wide) && __lane_id() == 0 && ((volatile int*)ctr)[C_CWIDE] != seq) ctr[C_CWIDE] = seq;
  }
}

// rank of each lane among the lanes of its block holding the same colour, in lane order
__device__ int block_rank(int c, bool valid, int* wcnt /* 4 waves x 256 */) {
  int lane = __lane_id(), w = threadIdx.x / kWave;
  uint64_t lt = (1ull << lane) - 1ull;
  int rank = 0;
  uint64_t left = __ballot(valid);
  while (left) {
    int lead = __ffsll((unsigned long long)left) - 1;
    int cc = __shfl(c, lead);
    uint64_t mask = __ballot(valid && c == cc);
    if (valid && c == cc) rank = __popcll(mask & lt);
    if (lane == lead) wcnt[w * 256 + cc] = __popcll(mask);
    left &= ~mask;
  }
  __syncthreads();
  if (valid)
    for (int k = 0; k < w; ++k) rank += wcnt[k * 256 + c];
  return rank;
}

template <int CM>
__global__ void k_class_place(const int* __restrict__ A, int n, const uint64_t* __restrict__ rw, int nb,
                              const int* __restrict__ tabscan, int* __restrict__ out) {
  __shared__ int wcnt[4 * 256];
  for (int k = threadIdx.x; k < 4 * 256; k += blockDim.x) wcnt[k] = 0;
  __syncthreads();
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  bool valid = i < n;
  int v = valid ? A[i] : -1;
  int c = valid ? (int)(rw[v] & 0xFF) : 0;
  int r = block_rank(c, valid, wcnt);
  if (valid && c < CM) out[tabscan[(int64_t)c * nb + blockIdx.x] + r] = v;
}

template <int CM>
__global__ void k_class_sizes(const int* __restrict__ tabscan, int nb, int n, int* ctr, int seq) {
  int c = threadIdx.x;
  int lo = tabscan[(int64_t)c * nb];
  int hi = c < CM - 1 ? tabscan[(int64_t)(c + 1) * nb] : n;
  ctr[C_HIST + c] = hi - lo;
  ctr[C_OFF + c] = lo;
  __syncthreads();
  if (c == 0) {
    int ncol = 0;
    for (int k = 0; k < CM; ++k)
      if (ctr[C_HIST + k]) ncol = k + 1;
    if (CM < 256 && ctr[C_CWIDE] == seq) ncol = -2;
    ctr[C_NCOL] = ncol;
  }
}

template <int CM>
static void class_lists_cm(const int* A, int n, const uint64_t* rw, int* ctr, int* out, int* tab, int* tabscan,
                           int* partial, int nb, int seq, hipStream_t s) {
  k_class_count<CM><<<nb, kBlock, 0, s>>>(A, n, rw, nb, tab, ctr, seq);
  scan_excl(tab, tabscan, CM * nb, ctr + C_TOTAL, partial, s);
  k_class_place<CM><<<nb, kBlock, 0, s>>>(A, n, rw, nb, tabscan, out);
  k_class_sizes<CM><<<1, CM, 0, s>>>(tabscan, nb, n, ctr, seq);
}

void class_lists(const int* A, int n, const uint64_t* rw, int* ctr, int* out, int* tab, int* tabscan, int* partial,
                 int cm, int seq, hipStream_t s) {
  static_assert(kBlock == 256, "class kernels use one LDS slot per colour and thread");
  int nb = (n + kBlock - 1) / kBlock;
  if (nb < 1) nb = 1;
  switch (cm) {
    case 4: class_lists_cm<4>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
    case 8: class_lists_cm<8>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
    case 16: class_lists_cm<16>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
    case 32: class_lists_cm<32>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
    case 64: class_lists_cm<64>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
    case 128: class_lists_cm<128>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
    default: class_lists_cm<256>(A, n, rw, ctr, out, tab, tabscan, partial, nb, seq, s); break;
  }
}

// A list of at most kSmallColour vertices is coloured and cut into classes by one
// block. Classes come out in no particular order; the members of a class are an
// independent set, so their order does not change any result.
// The colours lie in LDS. The round words carry each vertex's place in the list
// (bits 9 ..), one scan of a vertex's row then gives its record: the colours of the
// neighbours before it that are coloured already, and the places of up to eight
// that are not. From there on a vertex only follows its predecessors' colours,
// bytes in LDS, without barriers.
// Scanning rows is eleven line look-ups a vertex, which one CU does at about
// one a clock: re-scanning every waiting row per iteration took 31 us for 1,500
// vertices, this 22 (19 scanned by many blocks). Lists of more than kOneBlock are
// scanned by as many blocks as they fill (k_jp_pred, into JpRec records), so that
// only the solving is one block's.
constexpr int kSmallThreads = 1024;
constexpr int kPlaceBit = 9;
static_assert(kSmallColour <= 1 << 16, "places are 16-bit");
struct Preds {
  uint64_t lo, hi;  // places, 16 bits each, in row order
  uint64_t used;    // colours taken, below 64
  int cnt;          // places; -1: more than eight, or a colour past 63 (then jp_try)
};
__device__ __forceinline__ Preds preds_of(const Store& st, int v, const Round& rd) {
  constexpr int B = 8;
  uint64_t rv = rd.rw[v];
  Hdr h = st.hdr[v];
  Preds p{0, 0, 0, 0};
  bool big = false;
  for (int j0 = 0; j0 < h.y; j0 += B) {
    int w[B];
    uint64_t x[B];
    row8(st.nn, h.x + j0, h.y - j0, w);
#pragma unroll
    for (int q = 0; q < B; ++q) x[q] = w[q] >= 0 ? rd.rw[w[q]] : 0ull;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      if (!(x[q] & kRwAct) || !rw_beats(x[q], w[q], rv, v)) continue;
      int c = (int)(x[q] & 0xFF);
      if (c == 0xFF) {
        if (p.cnt >= 8) big = true;
        uint64_t at = (x[q] >> kPlaceBit) & 0xFFFF;
        if (p.cnt < 4) p.lo |= at << (16 * p.cnt);
        else p.hi |= at << (16 * (p.cnt & 3));
        ++p.cnt;
      } else if (c < 64) {
        p.used |= 1ull << c;
      } else {
        big = true;
      }
    }
  }
  if (big) p.cnt = -1;
  return p;
}

// Colours the list A (n <= K * NT vertices) from its predecessor records, each
// thread K of them (recs: their records, else one scan each). col: a byte per
// place, 0xFF at the start. No barriers: every thread goes round its own
// vertices until all have a colour; the waiting one of largest key is always
// ready, so the passes end (they are bounded all the same). What bounds it: the
// longest chain of waiting vertices, an LDS round trip per link. Adds the
// visits to *visits, raises *its to the passes of a thread.
constexpr int kMaxPasses = 1 << 20;
template <int NT, int K>
__device__ __forceinline__ void solve_items(const Store& st, const int* A, int n, const JpRec* recs, const Round& rd,
                                            volatile uint8_t* col, int* ctr, int* its, int* visits) {
  int tid = (int)threadIdx.x;
  Preds p[K];
  uint32_t todo = 0, far = 0;  // far: the vertices that jp_try colours
#pragma unroll
  for (int k = 0; k < K; ++k) {
    int i = tid + k * NT;
    p[k] = Preds{0, 0, 0, 0};
    if (i >= n) continue;
    todo |= 1u << k;
    if (recs) {
      JpRec r = recs[i];
      p[k] = Preds{r.lo, r.hi, r.used, r.cnt};
    } else {
      p[k] = preds_of(st, A[i], rd);
    }
    if (p[k].cnt < 0) far |= 1u << k;
  }
  if (!recs) __syncthreads();  // every row is scanned before a colour is stored
  int pass = 0, mine = __popc(todo);
  for (; todo && pass < kMaxPasses; ++pass) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!((todo & ~far) >> k & 1)) continue;
      Preds& q = p[k];
      while (q.cnt > 0) {
        int y = col[q.lo & 0xFFFF];
        if (y == 0xFF) break;
        if (y < 64) q.used |= 1ull << y;
        else far |= 1u << k;
        q.lo = q.lo >> 16 | q.hi << 48;
        q.hi >>= 16;
        --q.cnt;
      }
      if (q.cnt > 0) continue;
      if (!~q.used) far |= 1u << k;
      if (far >> k & 1) continue;
      int c = __ffsll((unsigned long long)~q.used) - 1, i = tid + k * NT;
      col[i] = (uint8_t)c;
      // the low half of the round word: the priority stays
      ((volatile uint32_t*)rd.rw)[2 * (int64_t)A[i]] = (uint32_t)kRwAct | (uint32_t)c;
      todo &= ~(1u << k);
    }
    uint32_t slow = todo & far;
    while (slow) {
      int k = __ffs((int)slow) - 1, i = tid + k * NT, b = -1;
      slow &= slow - 1;
      if (!jp_try<true>(st, A[i], rd, ctr, b)) continue;
      col[i] = (uint8_t)(rw_get<true>(rd.rw, A[i]) & 0xFF);
      todo &= ~(1u << k);
    }
  }
  if (pass) {
    atomicMax(its, pass);
    atomicAdd(visits, mine);
  }
  if (todo) atomicOr(&ctr[C_ERR], E_COLOURS);  // cannot happen
}

struct ColourLds {
  int big, ncol, its, visits;
  int hist[256], cur[256];
  int wsum[4];
  uint8_t col[kSmallColour];
};
// The n <= K * NT vertices of A, by the NT threads of the block; recs: their
// records, with the round words set, or null (both made here). Returns the
// size of the largest class; L.its: the most passes of a thread.
// The class offsets are a scan by 256 threads: one thread adding them up one
// after another took 8 us, half of the colouring of some hundred vertices.
template <int NT, int K>
__device__ __forceinline__ int colour_body(const Store& st, const int* A, int n, const JpRec* recs, const Round& rd,
                                           int* out, int* ctr, ColourLds& L) {
  int tid = (int)threadIdx.x;
  for (int i = tid; i < n; i += NT) {
    if (!recs) {
      int v = A[i];
      uint64_t prio = key_of(st, rd, v) >> 32;
      rd.rw[v] = (prio << 32) | ((uint64_t)i << kPlaceBit) | kRwAct | 0xFFull;
    }
    L.col[i] = 0xFF;
  }
  if (tid < 256) L.hist[tid] = 0;
  if (tid == 0) L.ncol = L.its = L.visits = L.big = 0;
  __syncthreads();
  solve_items<NT, K>(st, A, n, recs, rd, L.col, ctr, &L.its, &L.visits);
  __syncthreads();
  for (int i = tid; i < n; i += NT) atomicAdd(&L.hist[L.col[i]], 1);
  __syncthreads();
  int h = tid < 256 ? L.hist[tid] : 0, incl = h, lane = __lane_id();
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (tid < 256 && lane == kWave - 1) L.wsum[tid / kWave] = incl;
  if (h) atomicMax(&L.ncol, tid + 1);
  int big = h;
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) big = max(big, __shfl_xor(big, d));
  __syncthreads();
  if (tid < 256) {
    int o = incl - h;
    for (int w = 0; w < tid / kWave; ++w) o += L.wsum[w];
    L.cur[tid] = o;
    ctr[C_OFF + tid] = o;
    ctr[C_HIST + tid] = h;
  }
  if (tid == 0) {
    ctr[C_NCOL] = L.ncol;
    ctr[C_JP] = 0;
    ctr[C_TOUCH] = 0;
    ctr[C_TOTAL] = L.its;
    atomicAdd(ctr + C_STRIPE + S_PJP, L.visits);
  }
  __syncthreads();
  if (tid < 256 && lane == 0) atomicMax(&L.big, big);
  for (int i = tid; i < n; i += NT) out[atomicAdd(&L.cur[L.col[i]], 1)] = A[i];
  __syncthreads();
  return L.big;
}

// the list length, or -1 for one that the small colouring does not take
__device__ __forceinline__ int small_length(int n, const int* n_dev) {
  if (n_dev) n = *n_dev;
  return n < 0 || n > kSmallColour ? -1 : n;
}
__global__ void k_jp_place(Store st, const int* __restrict__ A, int n, const int* n_dev, Round rd) {
  n = small_length(n, n_dev);
  for (int i = gtid(); i < n; i += gstride()) {
    int v = A[i];
    uint64_t prio = key_of(st, rd, v) >> 32;
    rd.rw[v] = (prio << 32) | ((uint64_t)i << kPlaceBit) | kRwAct | 0xFFull;
  }
}
__global__ void k_jp_pred(Store st, const int* __restrict__ A, int n, const int* n_dev, Round rd,
                          JpRec* __restrict__ recs) {
  n = small_length(n, n_dev);
  for (int i = gtid(); i < n; i += gstride()) {
    Preds p = preds_of(st, A[i], rd);
    recs[i] = JpRec{p.lo, p.hi, p.used, p.cnt, 0};
  }
}
__global__ void __launch_bounds__(kSmallThreads) k_colour_small(Store st, const int* A, int n, const int* n_dev, Round rd,
                                                              const JpRec* recs, int* out, int* ctr) {
  __shared__ ColourLds L;
  // the list length may come from the device (a colouring launched ahead of
  // the read-back); a list this kernel does not take is reported as -1 colours
  n = small_length(n, n_dev);
  if (n < 0) {
    if (threadIdx.x == 0) ctr[C_NCOL] = -1;
    return;
  }
  if (n <= 2 * kSmallThreads) (void)colour_body<kSmallThreads, 2>(st, A, n, recs, rd, out, ctr, L);
  else (void)colour_body<kSmallThreads, kSmallColour / kSmallThreads>(st, A, n, recs, rd, out, ctr, L);
}
void colour_small(const Store& st, const int* A, int n, const int* n_dev, int n_about, Round rd, JpRec* recs, int* out,
                  int* ctr, hipStream_t s) {
  bool one = n_about <= kOneBlock;
  if (!one) {
    int nb = grid_for(n_dev ? kSmallColour : n);
    k_jp_place<<<nb, kBlock, 0, s>>>(st, A, n, n_dev, rd);
    k_jp_pred<<<nb, kBlock, 0, s>>>(st, A, n, n_dev, rd, recs);
  }
  k_colour_small<<<1, kSmallThreads, 0, s>>>(st, A, n, n_dev, rd, one ? nullptr : recs, out, ctr);
}

// The rest of a chunked colouring, when the launch that counted its waiting
// vertices in `slot` left no more than kSmallColour (else nothing happens and
// *nleft is -1): gathered into `list` with their places, then scanned by many
// blocks and solved by one. A launch of the chunked form takes 7 us however few
// wait, and the last five to ten of a colouring have a tenth of the list.
__global__ void __launch_bounds__(kSmallThreads) k_jp_gather(const int* __restrict__ W, const int* __restrict__ cnt, int nch,
                                                           int chunk, Round rd, int* list, int* ctr, int slot, int* nleft) {
  constexpr int NT = kSmallThreads;
  __shared__ int offs[NT], wsum[NT / kWave], left;
  int tid = (int)threadIdx.x, lane = __lane_id(), wv = tid / kWave;
  if (tid == 0) ctr[C_JPIT] = 0;
  // wavefront w adds up what the iterations w modulo 8 left
  if (wv < 8) {
    int x = ctr[C_STRIPE + lane * kStripeW + S_JPL + wv];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
    if (lane == 0) ctr[C_JPL + wv] = x;
    if (S_JPL + wv == slot && lane == 0) {
      left = x;
      *nleft = x <= kSmallColour ? x : -1;
      ctr[C_JP] = x <= kSmallColour ? 0 : x;
    }
  }
  __syncthreads();
  int n = left;
  if (n == 0 || n > kSmallColour) return;
  // thread t's chunks are [t * per, (t + 1) * per); offs: the entries before them
  int per = (nch + NT - 1) / NT, sum = 0;
  for (int c = tid * per; c < min(nch, (tid + 1) * per); ++c) sum += cnt[c];
  int incl = sum;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == kWave - 1) wsum[wv] = incl;
  __syncthreads();
  int before = incl - sum;
  for (int w = 0; w < wv; ++w) before += wsum[w];
  offs[tid] = before;
  __syncthreads();
  for (int i = tid; i < n; i += NT) {
    int t = 0;  // the last thread whose entries start at or before i
#pragma unroll
    for (int b = NT / 2; b > 0; b >>= 1)
      if (offs[t + b] <= i) t += b;
    int k = i - offs[t], c = t * per;
    while (k >= cnt[c]) k -= cnt[c++];
    int v = W[(size_t)c * chunk + k];
    list[i] = v;
    rw_put(rd.rw, v, rd.rw[v] | ((uint64_t)i << kPlaceBit));
  }
}
__global__ void __launch_bounds__(kSmallThreads) k_jp_solve(Store st, const int* A, const int* nleft, Round rd,
                                                          const JpRec* recs, int* ctr) {
  __shared__ uint8_t col[kSmallColour];
  __shared__ int its, visits;
  int n = *nleft;
  if (n <= 0) return;
  for (int i = (int)threadIdx.x; i < n; i += kSmallThreads) col[i] = 0xFF;
  if (threadIdx.x == 0) its = visits = 0;
  __syncthreads();
  if (n <= 2 * kSmallThreads) solve_items<kSmallThreads, 2>(st, A, n, recs, rd, col, ctr, &its, &visits);
  else solve_items<kSmallThreads, kSmallColour / kSmallThreads>(st, A, n, recs, rd, col, ctr, &its, &visits);
  __syncthreads();
  if (threadIdx.x == 0) {
    ctr[C_JPIT] = its;
    atomicAdd(ctr + C_STRIPE + S_PJP, visits);
  }
}
void jp_finish(const Store& st, int n, const int* W, const int* cnt, Round rd, JpRec* recs, int* list, int* ctr, int it,
               hipStream_t s) {
  int chunk = jp_chunk_of(n), nch = (n + chunk - 1) / chunk;
  if (nch <= 0) return;
  int* nleft = ctr + C_JPN;
  k_jp_gather<<<1, kSmallThreads, 0, s>>>(W, cnt, nch, chunk, rd, list, ctr, S_JPL + (it & 7), nleft);
  k_jp_pred<<<grid_for(kSmallColour), kBlock, 0, s>>>(st, list, 0, nleft, rd, recs);
  k_jp_solve<<<1, kSmallThreads, 0, s>>>(st, list, nleft, rd, recs, ctr);
}

// The vertices to act on next, from the members A and the rows rebuilt, each
// once; returns their number (every thread of the block makes this call).
template <int NT>
__device__ __forceinline__ int select_body(const Store& st, int mode, double L_low2, const int* A, int nA,
                                           const int* touched, int nt, uint8_t* nxt, int* seen, int mark, int* out,
                                           int* cnt) {
  if (threadIdx.x == 0) *cnt = 0;
  __syncthreads();
  for (int i = (int)threadIdx.x; i < nA + nt; i += NT) {
    int x = i < nA ? A[i] : touched[i - nA];
    if (!nxt[x] || atomicMax(&seen[x], mark) >= mark) continue;
    nxt[x] = 0;
    if (want(st, x, mode, L_low2, nullptr)) out[atomicAdd(cnt, 1)] = x;
  }
  __syncthreads();
  int n = *cnt;
  __syncthreads();
  return n;
}

// The same on a grid: a list of some thousand vertices took one block up to
// 60 us. ctr[C_LIST_B] is 0 at the start (clear_round), or -1 at the end when
// the host has to select over every slot (and rebuild the rows first after a
// commit that ran out of room).
__global__ void k_select_list(Store st, int mode, double L_low2, const int* __restrict__ A, int nA,
                              const int* __restrict__ touched, int cap, uint8_t* __restrict__ nxt,
                              int* __restrict__ seen, int mark, int* __restrict__ out, int* ctr) {
  int nt = ctr[C_TOUCH];
  if (nt > cap || room_failed(ctr)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctr[C_LIST_B] = -1;
    return;
  }
  for (int i = gtid(); i < nA + nt; i += gstride()) {
    int x = i < nA ? A[i] : touched[i - nA];
    if (!nxt[x] || atomicMax(&seen[x], mark) >= mark) continue;
    nxt[x] = 0;
    if (want(st, x, mode, L_low2, nullptr)) out[wave_append_slot(&ctr[C_LIST_B])] = x;
  }
}
void select_list(const Store& st, int mode, double L_low2, const int* A, int nA, const int* touched, int cap,
                 uint8_t* nxt, int* seen, int mark, int* out, int* ctr, hipStream_t s) {
  // the rows rebuilt are about five times the members
  k_select_list<<<grid_for(6 * (int64_t)nA, 256), kBlock, 0, s>>>(st, mode, L_low2, A, nA, touched, cap, nxt, seen, mark,
                                                                  out, ctr);
}

__global__ void k_colour_out(int V, const uint64_t* __restrict__ rw, int* __restrict__ out) {
  for (int v = gtid(); v < V; v += gstride()) out[v] = (rw[v] & kRwAct) ? (int)(rw[v] & 0xFF) : -1;
}
void colour_out(const Store& st, const uint64_t* rw, int* out, hipStream_t s) {
  k_colour_out<<<grid_for(st.V), kBlock, 0, s>>>(st.V, rw, out);
}

// ---- deferred update: stamps and claims (Sec. 3.3) -------------------------------------------
// A committed member stamps its operation and claims every row it changes.
// Where the commit starts from the members, the claim with the largest key
// (the smallest member id) wins the row: an atomic per row. Where it walks the
// rows in vertex order, it needs no owner, only the mark: a plain store (the
// largest collapse launch of the 2049 x 2049 step 560 -> 546 us with one
// 32-bit atomic a member instead of eight 64-bit ones).
__device__ __forceinline__ void claim_row(const Commit& cm, int x, int v) {
  if (cm.by_member)
    atomicMax((unsigned long long*)&cm.own[x], (unsigned long long)own_key(cm.epoch, v));
  else
    cm.dirty[x] = cm.epoch;
}
__device__ __forceinline__ void stamp(const Commit& cm, int v, int a, int b, int c) {
  cm.ops[v] = make_int4(cm.epoch, a, b, c);
}
// a record (a, b) for row u in this epoch. A member v collapsing onto u hands
// over its NE row: (ne_off, ne_cnt). A flip of the edge (v, w) with far
// vertices a and b gives rows a and b its two elements (lo, hi); rows v and w
// only lose elements. After a commit out of room the count at the last
// rebuild may lag behind: the row then goes to its neighbours' own records
// (two or more) or, without a record of this epoch, takes none.
__device__ __forceinline__ void mark_target(const Commit& cm, int u, int a, int b) {
  *(int3*)&cm.tgt[u] = make_int3(a, b, cm.epoch);
  atomicAdd(&cm.cnt[u], 1);
}

// a member is deferred when a same-class active neighbour has a larger key
__device__ __forceinline__ bool same_class_beats(const OpArgs& a, int w, uint64_t rv, int v) {
  uint64_t x = a.rw[w];
  return (x & kRwAct) && (int)(x & 0xFF) == a.cls && rw_beats(x, w, rv, v);
}
__device__ __forceinline__ bool beaten(const Store& st, int v, const OpArgs& a) {
  uint64_t rv = a.rw[v];
  Hdr h = st.hdr[v];
  for (int j = 0; j < h.y; ++j)
    if (same_class_beats(a, st.nn[h.x + j], rv, v)) return true;
  return false;
}

__device__ __forceinline__ Geo geo_of(const Store& st, int3 t) {
  return make_geo(st.xy[t.x], st.xy[t.y], st.xy[t.z], st.met[t.x], st.met[t.y], st.met[t.z]);
}
__device__ __forceinline__ Geo geo_of(const Store& st, const Elem& e) {
  return make_geo(st.xy[e.x], st.xy[e.y], st.xy[e.z], st.met[e.x], st.met[e.y], st.met[e.z]);
}

// per-wave stats: evaluated / deferred / committed; pops: also count the
// committed operations as the unit of the separate commit kernel that follows
// (grid-wide class kernels)
__device__ __forceinline__ void count_status(int status, int* ctr, bool pops = false) {
  // status: -1 idle lane, 0 deferred, 1 evaluated, 2 evaluated + committed
  uint64_t d = __ballot(status == 0);
  uint64_t e = __ballot(status >= 1);
  uint64_t c = __ballot(status == 2);
  if (__lane_id() == 0) {
    int* sp = stripe_ptr(ctr, 0);
    if (d) atomicAdd(sp + S_DEFER, __popcll(d));
    if (e) atomicAdd(sp + S_EVAL, __popcll(e));
    if (c) atomicAdd(sp + S_COMMIT, __popcll(c));
    if (c && pops) atomicAdd(sp + S_POPS, __popcll(c));
  }
}

// ---- coarsening (Sec. 2.4.1) --------------------------------------------------------------
// Candidates u: neighbours on every boundary side v lies on, with L^2 < L_low2,
// tried in ascending (L^2, u); the first whose re-pointed elements all keep
// area > 0 and q^2 >= q_min^2 is taken.
__device__ __forceinline__ int collapse_one(const Store& st, int v, const OpArgs& a, const Commit& cm, int* ctr) {
  Hdr h = st.hdr[v];
  double2 pv = st.xy[v];
  Met mv = st.met[v];
  uint8_t tv = st.tag[v];
  uint64_t rv = a.rw[v];
  // one pass over the 1-ring: re-validation and the first candidate together
  double bL = INFINITY;
  int bU = -1;
  for (int j = 0; j < h.y; ++j) {
    int w = st.nn[h.x + j];
    if (same_class_beats(a, w, rv, v)) {
      cm.nxt[v] = 1;
      return 0;
    }
    if (tv & ~st.tag[w]) continue;
    double L = len2(pv, mv, st.xy[w], st.met[w]);
    if (!(L < a.L_low2)) continue;
    if (bU < 0 || L < bL || (L == bL && w < bU)) {
      bL = L;
      bU = w;
    }
  }
  double lastL = -INFINITY;
  int lastU = -1;
  int u = -1;
  for (bool first = true;; first = false) {
    if (!first) {
      bL = INFINITY;
      bU = -1;
      for (int j = 0; j < h.y; ++j) {
      int w = st.nn[h.x + j];
      if (tv & ~st.tag[w]) continue;
      double L = len2(pv, mv, st.xy[w], st.met[w]);
      if (!(L < a.L_low2)) continue;
      bool after = L > lastL || (L == lastL && w > lastU);
      bool better = bU < 0 || L < bL || (L == bL && w < bU);
      if (after && better) {
        bL = L;
        bU = w;
      }
      }
    }
    if (bU < 0) break;
    bool ok = true;
    for (int i = 0; i < h.w && ok; ++i) {
      Elem e = st.tri[st.ne[h.z + i]];
      if (holds(e, bU)) continue;
      int k = slot_of(e, v);
      int3 r = rot_min(k == 0 ? bU : e.x, k == 1 ? bU : e.y, k == 2 ? bU : e.z);
      Geo g = geo_of(st, r);
      if (!(area2(g) > 0.0) || !(qd2(g, st.qk) >= a.qmin2)) ok = false;
    }
    if (ok) {
      u = bU;
      break;
    }
    lastL = bL;
    lastU = bU;
  }
  if (u < 0) return 1;
  // apply: v's elements are owned by v within this independent set
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    Elem e = st.tri[t];
    if (holds(e, u)) {
      e.w = 0;
    } else {
      int k = slot_of(e, v);
      int3 r = rot_min(k == 0 ? u : e.x, k == 1 ? u : e.y, k == 2 ? u : e.z);
      e = make_int4(r.x, r.y, r.z, 1);
    }
    st.tri[t] = e;
  }
  st.valive[v] = 0;
  stamp(cm, v, -(u + 1), h.z, h.w);
  mark_target(cm, u, h.z, h.w);
  for (int j = 0; j < h.y; ++j) claim_row(cm, st.nn[h.x + j], v);
  return 2;
}

template <int QK>
__global__ void k_collapse(Store st, const int* __restrict__ list, int n, OpArgs a, Commit cm, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  if (room_failed(ctr)) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctr[C_STAGE] = 0;  // the commit's fallback staging
  int i = xtid();
  int status = -1;
  if (i < n) status = collapse_one(st, list[i], a, cm, ctr);
  count_status(status, ctr, true);
}
template <int G, int QK>
__global__ void __launch_bounds__(256, 5) k_collapse_g(Store st, const int* __restrict__ list, int n, OpArgs a,
                                                    Commit cm, int* ctr);
void collapse_class(const Store& st, const int* list, int n, OpArgs a, Commit cm, int* ctr, int lanes,
                    hipStream_t s) {
  if (n <= 0) return;
  if (lanes == 16)
    (st.qk ? k_collapse_g<16, 1> : k_collapse_g<16, 0>)<<<(int)(((int64_t)n * 16 + kBlock - 1) / kBlock), kBlock, 0, s>>>(
        st, list, n, a, cm, ctr);
  else if (lanes == 8)
    (st.qk ? k_collapse_g<8, 1> : k_collapse_g<8, 0>)<<<(int)(((int64_t)n * 8 + kBlock - 1) / kBlock), kBlock, 0, s>>>(
        st, list, n, a, cm, ctr);
  else
    (st.qk ? k_collapse<1> : k_collapse<0>)<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(st, list, n, a, cm, ctr);
}

// ---- swapping (Sec. 2.4.3) ------------------------------------------------------------------
// For every interior edge (v, w): (v,w,a) and (w,v,b) become (v,b,a) and (w,a,b)
// when both areas stay positive and the smaller q^2 rises strictly; the best
// new minimum wins, ties to the smaller w; the element holding v keeps the
// smaller id.
__device__ __forceinline__ int flip_one(const Store& st, int v, const OpArgs& a, const Commit& cm, int* ctr) {
  if (beaten(st, v, a)) {
    cm.nxt[v] = 1;
    return 0;
  }
  Hdr h = st.hdr[v];
  double best = 0.0;
  int bw = -1, bT1 = -1, bT2 = -1, ba = -1, bb = -1;
  for (int i = 0; i < h.w; ++i) {
    int T1 = st.ne[h.z + i];
    Elem e1 = st.tri[T1];
    int k1 = slot_of(e1, v);
    int w = at(e1, k1 == 2 ? 0 : k1 + 1);
    int av = at(e1, k1 == 0 ? 2 : k1 - 1);
    int T2 = -1, bv = -1;
    Elem e2;
    for (int j = 0; j < h.w; ++j) {
      int t = st.ne[h.z + j];
      Elem e = st.tri[t];
      int k = slot_of(e, v);
      if (at(e, k == 0 ? 2 : k - 1) == w) {
        T2 = t;
        e2 = e;
        bv = at(e, k == 2 ? 0 : k + 1);
        break;
      }
    }
    if (T2 < 0) continue;
    Geo gv = geo_of(st, rot_min(v, bv, av));
    Geo gw = geo_of(st, rot_min(w, av, bv));
    if (!(area2(gv) > 0.0) || !(area2(gw) > 0.0)) continue;
    double qv = qd2(gv, st.qk), qw = qd2(gw, st.qk);
    double q1 = qd2(geo_of(st, e1), st.qk), q2 = qd2(geo_of(st, e2), st.qk);
    double nmin = qw < qv ? qw : qv;
    double omin = q2 < q1 ? q2 : q1;
    if (!(nmin > omin)) continue;
    if (bw < 0 || nmin > best || (nmin == best && w < bw)) {
      best = nmin;
      bw = w;
      bT1 = T1;
      bT2 = T2;
      ba = av;
      bb = bv;
    }
  }
  if (bw < 0) return 1;
  int lo = min(bT1, bT2), hi = max(bT1, bT2);
  int3 tv = rot_min(v, bb, ba), tw = rot_min(bw, ba, bb);
  st.tri[lo] = make_int4(tv.x, tv.y, tv.z, 1);
  st.tri[hi] = make_int4(tw.x, tw.y, tw.z, 1);
  stamp(cm, v, lo, hi, 0);
  mark_target(cm, ba, lo, hi);
  mark_target(cm, bb, lo, hi);
  claim_row(cm, v, v);
  claim_row(cm, bw, v);
  claim_row(cm, ba, v);
  claim_row(cm, bb, v);
  return 2;
}

template <int QK>
__global__ void k_flip(Store st, const int* __restrict__ list, int n, OpArgs a, Commit cm, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  if (room_failed(ctr)) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctr[C_STAGE] = 0;  // the commit's fallback staging
  int i = xtid();
  int status = -1;
  if (i < n) status = flip_one(st, list[i], a, cm, ctr);
  count_status(status, ctr, true);
}
void flip_class(const Store& st, const int* list, int n, OpArgs a, Commit cm, int* ctr, hipStream_t s) {
  if (n > 0) (st.qk ? k_flip<1> : k_flip<0>)<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(st, list, n, a, cm, ctr);
}

// ---- deferred update: commit ------------------------------------------------------------------
// Each claimed row is rebuilt once, by its owner's lane group, from its candidate
// elements: the old NE(x), all of NE(w) for a neighbour w collapsed onto x,
// and the two elements of every committed flip around x. NE(x) becomes the
// sorted candidates that are live and hold x (the canonical order); NN(x) is
// then the set of the other vertices of those elements.

// the candidates of row x that are live and hold x (possibly repeated),
// written to dst[k] when dst is given; returns how many there are. A class
// holds one kind of operation: F, flips (records (epoch, t1, t2, 0)), else
// collapses (records (epoch, -(u+1), ne_off, ne_cnt), the member's NE row).
// Only the general path takes this loop, one entry after another, so that the
// commit kernels keep their registers for the lane groups.
__device__ __forceinline__ bool keeps(const Elem& e, int x) { return e.w && holds(e, x); }

template <bool F>
__device__ __forceinline__ int row_candidates(const Store& st, const Commit& cm, int x, Hdr h, int* dst) {
  int n = 0;
  auto put = [&](int t) {
    if (keeps(st.tri[t], x)) {
      if (dst) dst[n] = t;
      ++n;
    }
  };
  // NE(x) (j < 0), then what each neighbour's record of this epoch hands over
#pragma unroll 1
  for (int j = -1; j < h.y; ++j) {
    int o = h.z, c = h.w;
    if (j >= 0) {
      int4 r = cm.ops[st.nn[h.x + j]];
      bool from = r.x == cm.epoch && (F ? r.y >= 0 : r.y == -x - 1);
      if (F && from) {
        put(r.y);
        put(r.z);
      }
      o = r.z;
      c = from && !F ? r.w : 0;
    }
#pragma unroll 1
    for (int k = 0; k < c; ++k) put(st.ne[o + k]);
  }
  return n;
}

__device__ void sort_unique(int* a, int& n) {
  for (int i = 1; i < n; ++i) {
    int x = a[i];
    int j = i - 1;
    while (j >= 0 && a[j] > x) {
      a[j + 1] = a[j];
      --j;
    }
    a[j + 1] = x;
  }
  int m = 0;
  for (int i = 0; i < n; ++i)
    if (m == 0 || a[i] != a[m - 1]) a[m++] = a[i];
  n = m;
}

__device__ __forceinline__ int grown_cap(int n) { return max(8, (2 * n + 3) & ~3); }

// write a sorted row, in place when it fits, else in fresh pool space; on
// pool exhaustion the row keeps its slot and is cut to its capacity, so no
// later read leaves the pool, and the error bit has the host rebuild every
// row before the round goes on
__device__ int put_row(int* pool, int64_t pool_cap, int* top, int& off, int& cap, const int* src, int n, int err,
                       int epoch, int* ctr) {
  if (n > cap) {
    int nc = grown_cap(n);
    int o = atomicAdd(top, nc);
    if ((int64_t)o + nc > pool_cap) {
      room_fail(ctr, err, epoch);
      n = cap;
    } else {
      off = o;
      cap = nc;
      atomicAdd(stripe_ptr(ctr, S_RELOC), 1);
    }
  }
  for (int k = 0; k < n; ++k) pool[off + k] = src[k];
  return n;
}

// general path: candidates in a private staging range, insertion sorts there
template <bool F>
__device__ __forceinline__ void rebuild_staged(const Store& st, const Commit& cm, int x, int* ctr) {
  Hdr h = st.hdr[x];
  int2 cp = st.cap[x];
  int tot = row_candidates<F>(st, cm, x, h, nullptr);
  int64_t need = 4 * (int64_t)tot + 4;
  int base = atomicAdd(&ctr[C_STAGE], (int)need);
  if ((int64_t)base + need > cm.stage_cap) {
    room_fail(ctr, E_STAGE, cm.epoch);
    return;
  }
  int* s = cm.stage + base;
  row_candidates<F>(st, cm, x, h, s);
  int m = tot;
  sort_unique(s, m);
  int* q = s + tot;
  int nq = 0;
  for (int k = 0; k < m; ++k) {
    Elem e = st.tri[s[k]];
    if (e.x != x) q[nq++] = e.x;
    if (e.y != x) q[nq++] = e.y;
    if (e.z != x) q[nq++] = e.z;
  }
  sort_unique(q, nq);
  int ne_off = h.z, ne_cap = cp.y, nn_off = h.x, nn_cap = cp.x;
  m = put_row(st.ne, st.ne_pool, &ctr[C_NE_TOP], ne_off, ne_cap, s, m, E_NE_POOL, cm.epoch, ctr);
  nq = put_row(st.nn, st.nn_pool, &ctr[C_NN_TOP], nn_off, nn_cap, q, nq, E_NN_POOL, cm.epoch, ctr);
  st.hdr[x] = make_int4(nn_off, nq, ne_off, m);
  st.cap[x] = make_int2(nn_cap, ne_cap);
}

// lane l's value of another lane of its 16-lane row, rotated by K (1 .. 15)
template <int K>
__device__ __forceinline__ int ror16(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + K, 0xF, 0xF, false);
}
// f(o) with the value v of every other lane of this lane's group of G lanes
// holding an item (lanes 0 .. n - 1; the others are passed or not, and hold a
// value that f ignores). G = 16: rotations inside the row of lanes, one move
// each; G = 64: one lane read per item, n the same for the whole wavefront.
template <int G, int K = 1, class Fn>
__device__ __forceinline__ void each_other(int v, int n, Fn&& f) {
  if constexpr (G == 16) {
    if constexpr (K < 16) {
      f(ror16<K>(v));
      each_other<G, K + 1>(v, n, f);
    }
  } else {
    n = __builtin_amdgcn_readfirstlane(n);
    for (int k = 0; k < n; ++k) f(__builtin_amdgcn_readlane(v, k));
  }
}

// Rebuild row x on a group of G lanes (16, or a whole wavefront for the rows
// that do not fit 16): x is the group's, negative for an idle group. Lane l
// takes the l-th entry of the old NE(x) and of the row x absorbs, then those
// two elements; the candidates that are live and hold x are packed to the
// group's LDS slots (3 G ints: id, next vertex, previous vertex), one per
// lane, and each lane counts the smaller ones for its place in the sorted
// row. NE(x) = those ids; NN(x) = their "next" vertices plus the one
// "previous" vertex that is no next (x on the boundary). An element reaches
// a row twice only in a flip (once from NE(x), once from the record): the
// record's is dropped.
// A row that holds more than G of anything goes to the block's queue bq (G =
// 16, each queued row then takes a wavefront), or to the general path; so do
// rows whose elements form no disk or half-disk around x.
// What bounds it: a chain of four dependent gathers (header and records;
// row entries; elements; stores), about 19 cache lines a row.
// One thread per row read the elements twice and wrote the rows entry by
// entry, 36 lines a row, and sorted in registers (96 of them): the commits of
// a 33 x 33 adaptation took 1.72 ms so and take 0.77, the member-driven ones
// of the 2049 x 2049 step 34 us a launch and 17. The largest vertex-order
// launches (1.3 million collapses) take 550 us either way.
template <bool F, int G>
__device__ __forceinline__ void rebuild_group(const Store& st, const Commit& cm, int x, int* slots, int* ctr, int* bq,
                                              int* bqn, int& rows) {
  int lane = __lane_id(), l = lane & (G - 1), gb = lane & ~(G - 1);
  uint64_t gm = G == 64 ? ~0ull : (1ull << G) - 1ull;
  uint64_t below = (1ull << l) - 1ull;
  auto gballot = [&](bool p) { return (__ballot(p) >> gb) & gm; };
  bool act = x >= 0;
  int xs = max(x, 0);
  Hdr h = st.hdr[xs];
  int2 cp = st.cap[xs];
  int4 tg = cm.tgt[xs];
  int ct = cm.cnt[xs];
  // members that hand something over to x in this epoch
  int nt = tg.z == cm.epoch ? ct - tg.w : 0;
  bool fits = act && h.w <= G && (nt <= 1 || h.y <= G) && (F || nt != 1 || tg.y <= G);
  int t0 = -1, t1 = -1;
  if (fits && l < h.w) t0 = st.ne[h.z + l];
  if (fits && nt == 1) {
    if (F) t1 = l == 0 ? tg.x : (l == 1 ? tg.y : -1);
    else if (l < tg.y) t1 = st.ne[tg.x + l];
  }
  Elem e0 = st.tri[max(t0, 0)], e1 = st.tri[max(t1, 0)];
  int n = 0;
  auto add = [&](bool k, int t, const Elem& e) {
    uint64_t b = gballot(k);
    int pos = n + __popcll(b & below);
    if (k && pos < G) {
      int sl = slot_of(e, x);
      slots[pos] = t;
      slots[G + pos] = at(e, sl == 2 ? 0 : sl + 1);
      slots[2 * G + pos] = at(e, sl == 0 ? 2 : sl - 1);
    }
    n += __popcll(b);
  };
  // a flip's element t (in lanes 0 and 1) that NE(x) holds already (every
  // lane of the group makes this call: it votes)
  auto known = [&](int t) {
    int a = __shfl(t, gb), b = __shfl(t, gb + 1);
    uint64_t ka = gballot(t0 >= 0 && t0 == a), kb = gballot(t0 >= 0 && t0 == b);
    return l == 0 ? ka != 0 : kb != 0;
  };
  add(t0 >= 0 && keeps(e0, x), t0, e0);
  if (nt == 1) {
    bool old = F ? known(t1) : false;
    add(t1 >= 0 && !old && keeps(e1, x), t1, e1);
  } else if (nt > 1 && fits) {
    // several members: from the neighbours' own records
    int4 r = make_int4(0, 0, 0, 0);
    if (l < h.y) r = cm.ops[st.nn[h.x + l]];
    uint64_t from = gballot(l < h.y && r.x == cm.epoch && (F ? r.y >= 0 : r.y == -x - 1));
    while (from) {
      int q = gb + __ffsll((unsigned long long)from) - 1;
      from &= from - 1;
      int ry = __shfl(r.y, q), rz = __shfl(r.z, q), rw = __shfl(r.w, q);
      int t = -1;
      if (F) {
        t = l == 0 ? ry : (l == 1 ? rz : -1);
      } else if (rw > G) {
        fits = false;
        break;
      } else if (l < rw) {
        t = st.ne[rz + l];
      }
      Elem e = st.tri[max(t, 0)];
      bool old = F ? known(t) : false;
      add(t >= 0 && !old && keeps(e, x), t, e);
    }
  }
  fits = fits && n <= G;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  bool own = fits && l < n;
  int id = own ? slots[l] : INT_MAX, nx = own ? slots[G + l] : INT_MAX, pv = own ? slots[2 * G + l] : -1;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  int nn_ = fits ? n : 0, rid = 0, rnx = 0, same = 0;
  bool found = false;
  each_other<G>(id, nn_, [&](int o) { rid += o < id ? 1 : 0; });
  each_other<G>(nx, nn_, [&](int o) {
    rnx += o < nx ? 1 : 0;
    same += o == nx ? 1 : 0;
    found |= o == pv;
  });
  // a next vertex that comes twice (a wavefront's lanes also meet themselves): two
  // lanes with one place. Counted in the loop, 1 us of the 234 of a vertex-order
  // launch at 2049 x 2049; as the missing rest of the places' sum it cost fewer
  // registers, but the loads came apart and the launch took 283.
  bool twice = gballot(own && same > (G == 64 ? 1 : 0)) != 0;
  uint64_t lone = gballot(own && !found);
  int nextra = __popcll(lone);
  int ex = nextra ? __shfl(pv, gb + __ffsll((unsigned long long)lone) - 1) : INT_MAX;
  int exat = __popcll(gballot(own && nx < ex));
  bool reg = fits && nextra <= 1 && !twice;
  int nq = n + nextra;
  if (own && ex < nx) ++rnx;
  // slots: in place when the row fits, else fresh pool space
  int ne_off = h.z, ne_cap = cp.y, nn_off = h.x, nn_cap = cp.x, lim_ne = n, lim_nn = nq;
  int ne_need = reg && n > ne_cap ? grown_cap(n) : 0;
  int nn_need = reg && nq > nn_cap ? grown_cap(nq) : 0;
  if (ne_need | nn_need) {
    int o0 = 0, o1 = 0;
    if (l == 0) {
      if (ne_need) o0 = atomicAdd(&ctr[C_NE_TOP], ne_need);
      if (nn_need) o1 = atomicAdd(&ctr[C_NN_TOP], nn_need);
      atomicAdd(stripe_ptr(ctr, S_RELOC), (ne_need ? 1 : 0) + (nn_need ? 1 : 0));
    }
    o0 = __shfl(o0, gb);
    o1 = __shfl(o1, gb);
    // a pool that is used up: the row keeps its slot and is cut to it (the
    // host rebuilds every row before the round goes on)
    if (ne_need) {
      if ((int64_t)o0 + ne_need > st.ne_pool) {
        if (l == 0) room_fail(ctr, E_NE_POOL, cm.epoch);
        lim_ne = min(n, ne_cap);
      } else {
        ne_off = o0;
        ne_cap = ne_need;
      }
    }
    if (nn_need) {
      if ((int64_t)o1 + nn_need > st.nn_pool) {
        if (l == 0) room_fail(ctr, E_NN_POOL, cm.epoch);
        lim_nn = min(nq, nn_cap);
      } else {
        nn_off = o1;
        nn_cap = nn_need;
      }
    }
  }
  if (reg) {
    if (own && rid < lim_ne) st.ne[ne_off + rid] = id;
    if (own && rnx < lim_nn) st.nn[nn_off + rnx] = nx;
    if (l == 0) {
      if (nextra && exat < lim_nn) st.nn[nn_off + exat] = ex;
      st.hdr[x] = make_int4(nn_off, lim_nn, ne_off, lim_ne);
      if (ne_need | nn_need) st.cap[x] = make_int2(nn_cap, ne_cap);
      if (ct != tg.w) cm.tgt[x].w = ct;
      ++rows;
    }
  } else if (act && l == 0) {
    int slot = G == 16 && !fits ? atomicAdd(bqn, 1) : kBlock;
    if (slot < kBlock) {
      bq[slot] = x;
    } else {
      rebuild_staged<F>(st, cm, x, ctr);
      cm.tgt[x].w = ct;
      ++rows;
    }
  }
  if (G == 16 && act && l == 0) cm.nxt[x] = 1;  // a row's first visit flags it for the next round
}

// LDS of a block's row rebuilds (NT threads)
template <int NT>
struct RowLds {
  int slots[3 * NT];      // 3 per lane: the candidates of the rows in flight
  int bq[kBlock];         // rows of more than 16 of anything
  int bqn;
};
// Rebuild the n rows row(0 .. n - 1) with the NT threads of the block, 16
// lanes each (every thread makes this call; bqn is zero). In small rounds the
// rows are listed for the next selection.
template <bool F, int NT, class Row>
__device__ __forceinline__ void rebuild_rows(const Store& st, const Commit& cm, int n, Row&& row, RowLds<NT>& L,
                                             int* ctr, int& rows) {
  constexpr int G = 16;
  int tid = (int)threadIdx.x, g = tid / G;
  if (cm.touched && n > 0) {
    __shared__ int tb;
    if (tid == 0) tb = atomicAdd(&ctr[C_TOUCH], n);
    __syncthreads();
    for (int i = tid; i < n; i += NT)
      if (tb + i < cm.touched_cap) cm.touched[tb + i] = row(i);
    __syncthreads();
  }
  for (int r0 = 0; r0 < n; r0 += NT / G)
    rebuild_group<F, G>(st, cm, r0 + g < n ? row(r0 + g) : -1, L.slots + 3 * G * g, ctr, L.bq, &L.bqn, rows);
}
// the queued rows, one per wavefront
template <bool F, int NT>
__device__ __forceinline__ void rebuild_queued(const Store& st, const Commit& cm, RowLds<NT>& L, int* ctr, int& rows) {
  __syncthreads();
  int nbig = min(L.bqn, kBlock), wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  for (int b = wv; b < nbig; b += NT / kWave)
    rebuild_group<F, kWave>(st, cm, L.bq[b], L.slots + 3 * kWave * wv, ctr, nullptr, nullptr, rows);
}
// the rows rebuilt by this wavefront, into the counters
__device__ __forceinline__ void count_rows(int rows, int* ctr) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) rows += __shfl_xor(rows, d);
  if (__lane_id() == 0 && rows) {
    int* sp = stripe_ptr(ctr, 0);
    atomicAdd(sp + S_ROWS, rows);
    atomicAdd(sp + S_PROWS, rows);
  }
}

// block-wide exclusive scan of one int per thread; returns the block total
template <int NT>
__device__ __forceinline__ int block_scan(int x, int& excl, int* wsum) {
  int lane = __lane_id(), wv = (int)threadIdx.x / kWave;
  int incl = x;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == kWave - 1) wsum[wv] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int q = 0; q < NT / kWave; ++q) {
    int c = wsum[q];
    total += c;
    if (q < wv) before += c;
  }
  excl = before + incl - x;
  return total;
}

// LDS of one commit block
constexpr int kPairB = 8;  // neighbours per member taken per pair round (two 16-byte loads)
template <int NT>
struct CommitLds {
  RowLds<NT> rows;
  int q[kPairB * NT];       // rows queued in a pair round
  int wsum[NT / kWave];
};

// Rebuild the rows claimed by the committed members list[base .. base + cnt)
// (cnt <= NT), with all NT threads of the block. Each member has tpm
// threads (a power of two: as many as fit, so a block of few members spreads
// each member's neighbours over its threads); a thread takes kPairB of its
// member's neighbours per pair round (row entries, then owner keys, loaded
// side by side). The rows a member owns are queued in LDS in block order and
// rebuilt, 16 lanes each. For flips one more round queues the members' own
// rows, after the rounds that read the members' rows.
template <bool F, int NT>
__device__ __forceinline__ void commit_chunk(const Store& st, const int* __restrict__ list, int base, int cnt,
                                             const Commit& cm, int* ctr, CommitLds<NT>& L) {
  int tid = (int)threadIdx.x;
  int lg = 0;
  while ((cnt << (lg + 1)) <= NT) ++lg;
  int mi = tid >> lg, sl = tid & ((1 << lg) - 1);
  int v = -1, deg = 0, off = 0;
  bool com = false;
  if (mi < cnt) {
    v = list[base + mi];
    int ep = cm.ops[v].x;
    Hdr h = st.hdr[v];
    com = ep == cm.epoch;
    if (com) {
      deg = h.y;
      off = h.x;
    }
  }
  uint64_t key = own_key(cm.epoch, v);
  int rows = 0;
  if (tid == 0) L.rows.bqn = 0;
  bool own_round = F;
  for (int j0 = sl * kPairB;; j0 += kPairB << lg) {
    bool pairs = __syncthreads_or(j0 < deg);
    if (!pairs && !own_round) break;
    int y[kPairB];
    uint64_t k[kPairB];
    if (pairs) {
      row8(st.nn, off + j0, deg - j0, y);
#pragma unroll
      for (int q = 0; q < kPairB; ++q) k[q] = y[q] >= 0 ? cm.own[y[q]] : 0ull;
    } else {
      own_round = false;
      bool mine_row = com && sl == 0;
#pragma unroll
      for (int q = 0; q < kPairB; ++q) y[q] = -1;
      if (mine_row) y[0] = v;
      k[0] = mine_row ? cm.own[v] : 0ull;
#pragma unroll
      for (int q = 1; q < kPairB; ++q) k[q] = 0ull;
    }
    int mine = 0;
#pragma unroll
    for (int q = 0; q < kPairB; ++q) mine += (y[q] >= 0 && k[q] == key) ? 1 : 0;
    int at;
    int tot = block_scan<NT>(mine, at, L.wsum);
#pragma unroll
    for (int q = 0; q < kPairB; ++q)
      if (y[q] >= 0 && k[q] == key) L.q[at++] = y[q];
    __syncthreads();
    rebuild_rows<F, NT>(st, cm, tot, [&](int i) { return L.q[i]; }, L.rows, ctr, rows);
  }
  rebuild_queued<F, NT>(st, cm, L.rows, ctr, rows);
  count_rows(rows, ctr);
  __syncthreads();  // the LDS is reused by the next chunk
}

// One block per mpb class members (commit_rows chooses mpb), in XCD-aware
// block order; one kernel per kind of operation.
template <bool F>
__global__ void __launch_bounds__(256, 5) k_commit(Store st, const int* __restrict__ list, int n, int mpb, Commit cm,
                                                int* ctr) {
  __shared__ CommitLds<kBlock> L;
  if (room_failed_block(ctr)) return;  // other blocks may set it meanwhile: one answer per block
  int base = xcd_block() * mpb;
  commit_chunk<F, kBlock>(st, list, base, min(mpb, n - base), cm, ctr, L);
}

// The same rebuild in vertex order, for classes whose claimed rows cover a
// good part of the mesh: a work-group scans `chunk` consecutive vertex slots
// (at most kSweepMax), queues the rows claimed in this epoch in LDS in slot
// order (a block-wide ordered compaction, so every lane group of a rebuild pass
// has a row), and rebuilds them. Consecutive rows then read
// nearby headers, capacities, owner keys and target records, and walk rows
// and elements in the order they are laid out, where the member-driven form
// above touches them in its members' neighbour order. Every row is still
// rebuilt once, from the same candidates, so the rows are the same.
constexpr int kSweepStep = kPairB * kBlock;  // slots scanned per block-wide pass
constexpr int kSweepMax = 2 * kSweepStep;    // most slots per work-group (16-bit offsets in LDS)
struct SweepLds {
  RowLds<kBlock> rows;
  uint16_t q[kSweepMax];
  int wsum[kBlock / kWave];
};
static_assert(kSweepMax <= 65536, "slot offsets are 16-bit");

template <bool F>
__global__ void __launch_bounds__(256, 5) k_commit_sweep(Store st, Commit cm, int chunk, int* ctr) {
  __shared__ SweepLds L;
  if (room_failed_block(ctr)) return;
  int tid = (int)threadIdx.x;
  int base = xcd_block() * chunk;
  int end = min(st.V, base + chunk);
  // each pass: thread tid reads the marks of kPairB consecutive slots,
  // all in flight together, and one block-wide scan places the claimed rows
  // in slot order
  int qn = 0;
  for (int s0 = base; s0 < end; s0 += kSweepStep) {
    int first = s0 + tid * kPairB;
    bool dirty[kPairB];
    int mine = 0;
    {
      int k[kPairB];
#pragma unroll
      for (int q = 0; q < kPairB; ++q) k[q] = first + q < end ? cm.dirty[first + q] : -1;
#pragma unroll
      for (int q = 0; q < kPairB; ++q) {
        dirty[q] = first + q < end && k[q] == cm.epoch;
        mine += dirty[q] ? 1 : 0;
      }
    }
    int at;
    int tot = block_scan<kBlock>(mine, at, L.wsum);
    at += qn;
#pragma unroll
    for (int q = 0; q < kPairB; ++q)
      if (dirty[q]) L.q[at++] = (uint16_t)(first + q - base);
    qn += tot;
    __syncthreads();  // wsum is reused by the next scan
  }
  if (tid == 0) L.rows.bqn = 0;
  __syncthreads();
  int rows = 0;
  rebuild_rows<F, kBlock>(st, cm, qn, [&](int i) { return base + (int)L.q[i]; }, L.rows, ctr, rows);
  rebuild_queued<F, kBlock>(st, cm, L.rows, ctr, rows);
  count_rows(rows, ctr);
}

// Work-groups of `fn` (kBlock threads) resident on the current device at
// once: work-groups per CU from the occupancy calculator times the CUs,
// kept per device. The commits size their grids by it, so that a grid runs
// as one generation of resident work-groups: a grid slightly larger than
// that runs a second, short generation that leaves most of the chip idle.
constexpr int kMaxDevices = 64;
int resident_blocks(const void* fn, int which) {
  static std::atomic<int> cache[4][kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = -1;
  if (dev >= 0) {
    int r = cache[which][dev].load(std::memory_order_relaxed);
    if (r > 0) return r;
  }
  int per = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kBlock, 0) != hipSuccess || per <= 0) per = 4;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev < 0 ? 0 : dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  int r = per * cus;
  if (dev >= 0) cache[which][dev].store(r, std::memory_order_relaxed);
  return r;
}

void commit_sweep(const Store& st, Commit cm, bool flips, int* ctr, hipStream_t s) {
  if (st.V <= 0) return;
  int res = flips ? resident_blocks((const void*)&k_commit_sweep<true>, 0)
                  : resident_blocks((const void*)&k_commit_sweep<false>, 1);
  // slots per work-group: a multiple of 32, at most kSweepMax (on a mesh of
  // 1,500 vertices 256 slots left a work-group 12 passes one after another,
  // 15 us a launch; 32 slots: two, 7 us)
  int64_t per = ((int64_t)st.V + res - 1) / res;
  int chunk = (int)std::min<int64_t>(kSweepMax, std::max<int64_t>(32, (per + 31) / 32 * 32));
  int nb = (st.V + chunk - 1) / chunk;
  if (flips)
    k_commit_sweep<true><<<nb, kBlock, 0, s>>>(st, cm, chunk, ctr);
  else
    k_commit_sweep<false><<<nb, kBlock, 0, s>>>(st, cm, chunk, ctr);
}

void commit_rows(const Store& st, const int* list, int n, Commit cm, bool flips, int chunk, int* ctr, hipStream_t s) {
  if (n <= 0) return;
  int mpb = chunk;
  if (mpb <= 0) {
    // members per work-group: at least 4 (a small class then spreads over
    // more work-groups, each with several threads per member), more when
    // that keeps the grid within one generation of resident work-groups
    int res = flips ? resident_blocks((const void*)&k_commit<true>, 2)
                    : resident_blocks((const void*)&k_commit<false>, 3);
    mpb = std::min(kBlock, std::max(4, (n + res - 1) / res));
  }
  int nb = (n + mpb - 1) / mpb;
  if (flips)
    k_commit<true><<<nb, kBlock, 0, s>>>(st, list, n, mpb, cm, ctr);
  else
    k_commit<false><<<nb, kBlock, 0, s>>>(st, list, n, mpb, cm, ctr);
}


// ---- smoothing (Sec. 2.4.4) ---------------------------------------------------------------------
__global__ void k_elem_metric(Store st, Met* __restrict__ out) {
  for (int t = gtid(); t < st.T; t += gstride()) {
    Elem e = st.tri[t];
    if (!e.w) continue;
    Met m0 = st.met[e.x], m1 = st.met[e.y], m2 = st.met[e.z];
    Met r;
    r.a = third((m0.a + m1.a) + m2.a);
    r.b = third((m0.b + m1.b) + m2.b);
    r.c = third((m0.c + m1.c) + m2.c);
    out[t] = r;
  }
}
void element_metrics(const Store& st, Met* out, hipStream_t s) {
  k_elem_metric<<<grid_for(st.T), kBlock, 0, s>>>(st, out);
}

__global__ void k_vertex_records(Store st, VRec* __restrict__ out) {
  for (int v = gtid(); v < st.V; v += gstride()) {
    double2 p = st.xy[v];
    Met m = st.met[v];
    VRec r;
    r.x = p.x;
    r.y = p.y;
    r.a = m.a;
    r.b = m.b;
    r.c = m.c;
    r.tag = st.tag[v];
    r.pad0 = 0;
    r.pad1 = 0.0;
    r.pad2 = 0.0;
    out[v] = r;
  }
}
void vertex_records(const Store& st, VRec* out, hipStream_t s) {
  if (st.V > 0) k_vertex_records<<<grid_for(st.V), kBlock, 0, s>>>(st, out);
}

// element t's geometry with vertex v at p; the mean tensor comes from the
// per-element array when present (the same value, computed once)
__device__ __forceinline__ Geo patch_elem_geo(const Store& st, int t, const Elem& e, int v, double2 p) {
  double2 p0 = e.x == v ? p : st.xy[e.x];
  double2 p1 = e.y == v ? p : st.xy[e.y];
  double2 p2 = e.z == v ? p : st.xy[e.z];
  if (st.emet) {
    Geo g;
    g.x[0] = p0.x; g.y[0] = p0.y;
    g.x[1] = p1.x; g.y[1] = p1.y;
    g.x[2] = p2.x; g.y[2] = p2.y;
    Met m = st.emet[t];
    g.a = m.a;
    g.b = m.b;
    g.c = m.c;
    return g;
  }
  return make_geo(p0, p1, p2, st.met[e.x], st.met[e.y], st.met[e.z]);
}

// smallest q^2 over v's elements with v placed at p; valid = all areas positive
__device__ double patch_min_q2(const Store& st, int v, Hdr h, double2 p, bool& valid) {
  valid = true;
  double mn = 0.0;
  bool first = true;
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    Elem e = st.tri[t];
    Geo g = patch_elem_geo(st, t, e, v, p);
    if (!(area2(g) > 0.0)) valid = false;
    double q2 = qd2(g, st.qk);
    if (first || q2 < mn) mn = q2;
    first = false;
  }
  return mn;
}

__device__ double patch_q(const Store& st, int v, Hdr h, double2 p) {
  double s = 0.0;
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    Elem e = st.tri[t];
    s = s + qval(patch_elem_geo(st, t, e, v, p), st.qk);
  }
  return s;
}

// "first or smaller" running minimum, as in a serial loop over the row
__device__ __forceinline__ void run_min(double q, bool first, double& mn) {
  if (first || q < mn) mn = q;
}

__device__ bool smooth_laplace(Store st, int v) {
  Hdr h = st.hdr[v];
  double2 pv = st.xy[v];
  Met mv = st.met[v];
  double Ga = 0.0, Gb = 0.0, Gc = 0.0, rx = 0.0, ry = 0.0;
  for (int j = 0; j < h.y; ++j) {
    int w = st.nn[h.x + j];
    Met mw = st.met[w];
    double2 pw = st.xy[w];
    double ea = (mv.a + mw.a) * 0.5;
    double eb = (mv.b + mw.b) * 0.5;
    double ec = (mv.c + mw.c) * 0.5;
    double dx = pw.x - pv.x, dy = pw.y - pv.y;
    Ga = Ga + ea;
    Gb = Gb + eb;
    Gc = Gc + ec;
    rx = rx + (ea * dx + eb * dy);
    ry = ry + (eb * dx + ec * dy);
  }
  double det = Ga * Gc - Gb * Gb;
  double2 p = make_double2(pv.x + (Gc * rx - Gb * ry) / det, pv.y + (Ga * ry - Gb * rx) / det);
  // one pass over the patch: minimum q^2 at the old and at the new position
  double oldmin = 0.0, newmin = 0.0;
  bool vn = true;
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    Elem e = st.tri[t];
    Geo go = patch_elem_geo(st, t, e, v, pv);
    Geo gn = go;
    int k = slot_of(e, v);
    gn.x[0] = k == 0 ? p.x : go.x[0];
    gn.y[0] = k == 0 ? p.y : go.y[0];
    gn.x[1] = k == 1 ? p.x : go.x[1];
    gn.y[1] = k == 1 ? p.y : go.y[1];
    gn.x[2] = k == 2 ? p.x : go.x[2];
    gn.y[2] = k == 2 ? p.y : go.y[2];
    run_min(qd2(go, st.qk), i == 0, oldmin);
    if (!(area2(gn) > 0.0)) vn = false;
    run_min(qd2(gn, st.qk), i == 0, newmin);
  }
  if (vn && newmin >= oldmin) {
    st.xy[v] = p;
    return true;
  }
  return false;
}

// geometry with slot k moved to p
__device__ __forceinline__ Geo moved(const Geo& g, int k, double2 p) {
  Geo r = g;
  r.x[0] = k == 0 ? p.x : g.x[0];
  r.y[0] = k == 0 ? p.y : g.y[0];
  r.x[1] = k == 1 ? p.x : g.x[1];
  r.y[1] = k == 1 ? p.y : g.y[1];
  r.x[2] = k == 2 ? p.x : g.x[2];
  r.y[2] = k == 2 ? p.y : g.y[2];
  return r;
}

__device__ bool smooth_gradient(Store st, int v) {
  Hdr h = st.hdr[v];
  double2 pv = st.xy[v];
  // pass 1: gradient of Q_v, Q_v and the minimum q^2 at the current position
  double gx = 0.0, gy = 0.0, Qold = 0.0, oldmin = 0.0;
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    Elem e = st.tri[t];
    Geo g = patch_elem_geo(st, t, e, v, pv);
    double ex, ey;
    qgrad_x(g, slot_of(e, v), st.qk, ex, ey);
    gx = gx + ex;
    gy = gy + ey;
    Qold = Qold + qval(g, st.qk);
    run_min(qd2(g, st.qk), i == 0, oldmin);
  }
  if (gx == 0.0 && gy == 0.0) return false;
  double ax = fabs(gx), ay = fabs(gy);
  double nrm = ax < ay ? ay : ax;
  double dx = gx / nrm, dy = gy / nrm;
  double hh = 0.0;
  for (int j = 0; j < h.y; ++j) {
    double2 pw = st.xy[st.nn[h.x + j]];
    double hx = fabs(pw.x - pv.x), hy = fabs(pw.y - pv.y);
    double hj = hx < hy ? hy : hx;
    if (j == 0 || hj < hh) hh = hj;
  }
  // pass 2: the four trial steps h/2 .. h/16 together; the first acceptable wins
  double2 p[4];
  double step = hh;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    step = step * 0.5;
    p[k] = make_double2(pv.x + step * dx, pv.y + step * dy);
  }
  double mn[4] = {0.0, 0.0, 0.0, 0.0}, Q[4] = {0.0, 0.0, 0.0, 0.0};
  bool ok[4] = {true, true, true, true};
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    Elem e = st.tri[t];
    Geo g = patch_elem_geo(st, t, e, v, pv);
    int sl = slot_of(e, v);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Geo gk = moved(g, sl, p[k]);
      if (!(area2(gk) > 0.0)) ok[k] = false;
      run_min(qd2(gk, st.qk), i == 0, mn[k]);
      Q[k] = Q[k] + qval(gk, st.qk);
    }
  }
  int pick = -1;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (pick < 0 && ok[k] && mn[k] >= oldmin && Q[k] > Qold) pick = k;
  if (pick < 0) return false;
  // recompute the chosen point rather than index the trial array
  double sp = hh;
  for (int k = 0; k <= pick; ++k) sp = sp * 0.5;
  st.xy[v] = make_double2(pv.x + sp * dx, pv.y + sp * dy);
  return true;
}

// Min-max: ascent on the patch's smallest quality. The worst element (the
// smallest q, ties to the first in NE(v)) gives the direction, its gradient
// in x_v; when the second worst is within 1% (q2 <= 1.01 q1), the point
// nearest the origin on the segment between the two gradients. Normalised in
// the max-norm; steps h/2 .. h/16 as in the gradient step; the first step
// that keeps every area positive and raises the patch minimum of q^2
// strictly is taken.
__device__ bool smooth_minmax(Store st, int v) {
  Hdr h = st.hdr[v];
  double2 pv = st.xy[v];
  int i1 = -1, i2 = -1;
  double q1 = 0.0, q2 = 0.0;
  for (int i = 0; i < h.w; ++i) {
    int t = st.ne[h.z + i];
    double q = qval(patch_elem_geo(st, t, st.tri[t], v, pv), st.qk);
    if (i1 < 0 || q < q1) {
      i2 = i1;
      q2 = q1;
      i1 = i;
      q1 = q;
    } else if (i2 < 0 || q < q2) {
      i2 = i;
      q2 = q;
    }
  }
  if (i1 < 0) return false;
  int t1 = st.ne[h.z + i1];
  Elem e1 = st.tri[t1];
  double ax, ay;
  qgrad_x(patch_elem_geo(st, t1, e1, v, pv), slot_of(e1, v), st.qk, ax, ay);
  double gx = ax, gy = ay;
  if (i2 >= 0 && q2 <= q1 * 1.01) {
    int t2 = st.ne[h.z + i2];
    Elem e2 = st.tri[t2];
    double bx, by;
    qgrad_x(patch_elem_geo(st, t2, e2, v, pv), slot_of(e2, v), st.qk, bx, by);
    double ex = bx - ax, ey = by - ay;
    double den = ex * ex + ey * ey;
    if (den > 0.0) {
      double lam = -(ax * ex + ay * ey) / den;
      lam = lam < 0.0 ? 0.0 : (lam > 1.0 ? 1.0 : lam);
      gx = ax + lam * ex;
      gy = ay + lam * ey;
    }
  }
  if (gx == 0.0 && gy == 0.0) return false;
  double nx = fabs(gx), ny = fabs(gy);
  double nrm = nx < ny ? ny : nx;
  double dx = gx / nrm, dy = gy / nrm;
  double hh = 0.0;
  for (int j = 0; j < h.y; ++j) {
    double2 pw = st.xy[st.nn[h.x + j]];
    double hx = fabs(pw.x - pv.x), hy = fabs(pw.y - pv.y);
    double hj = hx < hy ? hy : hx;
    if (j == 0 || hj < hh) hh = hj;
  }
  bool vo;
  double oldmin = patch_min_q2(st, v, h, pv, vo);
  double step = hh;
  for (int k = 0; k < 4; ++k) {
    step = step * 0.5;
    double2 p = make_double2(pv.x + step * dx, pv.y + step * dy);
    bool vn;
    double newmin = patch_min_q2(st, v, h, p, vn);
    if (!vn || !(newmin > oldmin)) continue;
    st.xy[v] = p;
    return true;
  }
  return false;
}

template <int QK>
__global__ void k_smooth(Store st, const int* __restrict__ list, int n, int kind, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  int i = xtid();
  int status = -1;
  if (i < n) {
    int v = list[i];
    bool moved = kind == 0 ? smooth_laplace(st, v) : (kind == 1 ? smooth_gradient(st, v) : smooth_minmax(st, v));
    status = moved ? 2 : 1;
  }
  count_status(status, ctr);
}
template <int K, int QK>
__global__ void __launch_bounds__(256, 4) k_smooth_g(Store st, const int* __restrict__ list, int n, int* ctr);
void smooth_class(const Store& st, const int* list, int n, int kind, int* ctr, int lanes, hipStream_t s) {
  if (n <= 0) return;
  int nb = (int)(((int64_t)n * kG + kBlock - 1) / kBlock);
  if (lanes == kG && kind == 2)
    (st.qk ? k_smooth_g<2, 1> : k_smooth_g<2, 0>)<<<nb, kBlock, 0, s>>>(st, list, n, ctr);
  else if (lanes == kG && kind == 0)
    (st.qk ? k_smooth_g<0, 1> : k_smooth_g<0, 0>)<<<nb, kBlock, 0, s>>>(st, list, n, ctr);
  else if (lanes == kG)
    (st.qk ? k_smooth_g<1, 1> : k_smooth_g<1, 0>)<<<nb, kBlock, 0, s>>>(st, list, n, ctr);
  else
    (st.qk ? k_smooth<1> : k_smooth<0>)<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(st, list, n, kind, ctr);
}

// ---- lane groups: 8 lanes per vertex ----------------------------------------------------------
// A vertex's 1-ring is spread over a group of kG lanes: lane j owns the j-th
// neighbour and the j-th element of the vertex's sorted rows, loads them in
// parallel and keeps its element's geometry in registers. Sums run over the
// lanes in row order (one shuffle per term), so every FP64 sum has the same
// rounding sequence as a serial loop over the row. Vertices with more than
// kG neighbours or elements take the one-thread path on the group's lane 0.
struct Grp {
  int j;     // index in the group
  int base;  // first lane of the group in the wavefront
};
__device__ __forceinline__ Grp grp() {
  int l = __lane_id();
  return Grp{l & (kG - 1), l & ~(kG - 1)};
}
__device__ __forceinline__ double gget(double v, int k, const Grp& g) { return __shfl(v, g.base + k); }
__device__ __forceinline__ int gget(int v, int k, const Grp& g) { return __shfl(v, g.base + k); }
// Sums over a group's lanes in row order, acc = ((0 + v_0) + v_1) + ..., go
// through LDS: every lane stores its terms (0 in a lane without one: adding it
// changes nothing), then reads the group's terms of a sum back, 16 bytes at a
// time. A shuffle of a double is two LDS instructions per term and lane.
constexpr int kSumW = kWave + 2;  // stride of one sum's terms (offsets the banks of the sums)
__device__ __forceinline__ void wave_lds() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// the group's terms at t (16-byte aligned), summed
__device__ __forceinline__ double sum8(const double* t) {
  const double2* p = (const double2*)t;
  double2 a = p[0], b = p[1], c = p[2], d = p[3];
  return (((((((0.0 + a.x) + a.y) + b.x) + b.y) + c.x) + c.y) + d.x) + d.y;
}
// one sum, in every lane of the group
__device__ __forceinline__ double gsum(double v, const Grp& g, double* lds) {
  lds[g.base + g.j] = v;
  wave_lds();
  double s = sum8(lds + g.base);
  wave_lds();
  return s;
}
// N sums side by side: lane c < N adds up the c-th (its return value)
template <int N>
__device__ __forceinline__ double gsum_lane(const double (&v)[N], const Grp& g, double* lds) {
#pragma unroll
  for (int c = 0; c < N; ++c) lds[c * kSumW + g.base + g.j] = v[c];
  wave_lds();
  double s = sum8(lds + (g.j < N ? g.j : 0) * kSumW + g.base);
  wave_lds();
  return s;
}
// N sums, every one in every lane of the group
template <int N>
__device__ __forceinline__ void gsums(double (&v)[N], const Grp& g, double* lds) {
  double s = gsum_lane<N>(v, g, lds);
  lds[g.base + g.j] = s;
  wave_lds();
#pragma unroll
  for (int c = 0; c < N; ++c) v[c] = lds[g.base + c];
  wave_lds();
}
// a double moved inside each row of 16 lanes by a DPP control
template <int C>
__device__ __forceinline__ double dpp64(double v) {
  int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), C, 0xF, 0xF, false);
  int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), C, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
// serial "first or smaller" minimum over lanes 0..n-1: three exchanges across
// the eight lanes. The serial loop starts from lane 0 and takes no value that
// is no number after it, so such a value counts as infinite, and as the result
// in lane 0.
__device__ __forceinline__ double gmin(double v, int n, const Grp& g) {
  double m = g.j < n && v == v ? v : INFINITY;
  double o = dpp64<0xB1>(m);   // lanes 1 0 3 2
  m = o < m ? o : m;
  o = dpp64<0x4E>(m);          // lanes 2 3 0 1
  m = o < m ? o : m;
  o = dpp64<0x141>(m);         // lanes 7 6 5 4 3 2 1 0
  m = o < m ? o : m;
  uint64_t bad = __ballot(!(v == v));
  if (bad) {
    double f = __shfl(v, g.base);
    if (!(f == f)) m = f;
  }
  return n > 0 ? m : 0.0;
}
__device__ __forceinline__ bool gany(bool p, const Grp& g) {
  uint64_t b = __ballot(p);
  return ((b >> g.base) & 0xFFull) != 0;
}
__device__ __forceinline__ uint64_t gor64(uint64_t v, const Grp& g) {
#pragma unroll
  for (int d = 1; d < kG; d <<= 1) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    lo |= (uint32_t)__shfl_xor((int)lo, d);
    hi |= (uint32_t)__shfl_xor((int)hi, d);
    v = ((uint64_t)hi << 32) | lo;
  }
  return v;
}

// one element of a vertex's patch, in stored order; slot k holds the vertex
struct PatchElem {
  double x0, y0, x1, y1, x2, y2;
  double a, b, c;  // mean tensor (stored order)
  int k;
};

// element t = e of v's patch; the mean tensor from the per-element array
// when present (the same value, computed once per phase), else from the
// three vertices
__device__ __forceinline__ PatchElem load_patch_elem(const Store& st, int t, const Elem& e, int v) {
  PatchElem pe;
  double2 p0 = st.xy[e.x], p1 = st.xy[e.y], p2 = st.xy[e.z];
  pe.x0 = p0.x; pe.y0 = p0.y;
  pe.x1 = p1.x; pe.y1 = p1.y;
  pe.x2 = p2.x; pe.y2 = p2.y;
  if (st.emet) {
    Met m = st.emet[t];
    pe.a = m.a;
    pe.b = m.b;
    pe.c = m.c;
  } else {
    Met m0 = st.met[e.x], m1 = st.met[e.y], m2 = st.met[e.z];
    pe.a = third((m0.a + m1.a) + m2.a);
    pe.b = third((m0.b + m1.b) + m2.b);
    pe.c = third((m0.c + m1.c) + m2.c);
  }
  pe.k = slot_of(e, v);
  return pe;
}

// the element's geometry with the patch vertex placed at p
__device__ __forceinline__ Geo patch_geo(const PatchElem& pe, double2 p) {
  Geo g;
  g.x[0] = pe.k == 0 ? p.x : pe.x0;
  g.y[0] = pe.k == 0 ? p.y : pe.y0;
  g.x[1] = pe.k == 1 ? p.x : pe.x1;
  g.y[1] = pe.k == 1 ? p.y : pe.y1;
  g.x[2] = pe.k == 2 ? p.x : pe.x2;
  g.y[2] = pe.k == 2 ? p.y : pe.y2;
  g.a = pe.a;
  g.b = pe.b;
  g.c = pe.c;
  return g;
}

// patch minimum of q^2 and validity with the vertex at p (lanes j < nw own elements)
__device__ __forceinline__ double gpatch_min(const PatchElem& pe, bool own, double2 p, int nw, const Grp& g,
                                             int qk, bool& valid) {
  double q2 = 0.0;
  bool bad = false;
  if (own) {
    Geo gg = patch_geo(pe, p);
    bad = !(area2(gg) > 0.0);
    q2 = qd2(gg, qk);
  }
  valid = !gany(bad, g);
  return gmin(q2, nw, g);
}

__device__ __forceinline__ double gpatch_q(const PatchElem& pe, bool own, double2 p, const Grp& g, int qk, double* lds) {
  return gsum(own ? qval(patch_geo(pe, p), qk) : 0.0, g, lds);
}

// sums a smoothing step takes side by side
constexpr int kSmoothSums = 5;
__device__ __forceinline__ bool smooth_group(Store& st, int v, Hdr h, int kind, const Grp& g, double* lds) {
  double2 pv = st.xy[v];
  Met mv = st.met[v];
  bool ownn = g.j < h.y, owne = g.j < h.w;
  // row entries, then neighbour data and elements, then the elements'
  // vertex data, each level issued together (index 0 for an empty lane)
  int w = ownn ? st.nn[h.x + g.j] : -1;
  int t = owne ? st.ne[h.z + g.j] : -1;
  double2 pw = st.xy[max(w, 0)];
  Met mw = st.met[max(w, 0)];
  Elem e = st.tri[max(t, 0)];
  if (!ownn) {
    pw = make_double2(0.0, 0.0);
    mw = Met{0.0, 0.0, 0.0};
  }
  PatchElem pe = load_patch_elem(st, max(t, 0), e, v);
  if (!owne) pe = PatchElem{};
  double2 p;
  if (kind == 0) {
    double ea = (mv.a + mw.a) * 0.5;
    double eb = (mv.b + mw.b) * 0.5;
    double ec = (mv.c + mw.c) * 0.5;
    double dx = pw.x - pv.x, dy = pw.y - pv.y;
    double t[5] = {ownn ? ea : 0.0, ownn ? eb : 0.0, ownn ? ec : 0.0, ownn ? ea * dx + eb * dy : 0.0,
                   ownn ? eb * dx + ec * dy : 0.0};
    gsums(t, g, lds);
    double Ga = t[0], Gb = t[1], Gc = t[2], rx = t[3], ry = t[4];
    double det = Ga * Gc - Gb * Gb;
    p = make_double2(pv.x + (Gc * rx - Gb * ry) / det, pv.y + (Ga * ry - Gb * rx) / det);
    bool vo, vn;
    double oldmin = gpatch_min(pe, owne, pv, h.w, g, st.qk, vo);
    double newmin = gpatch_min(pe, owne, p, h.w, g, st.qk, vn);
    if (!(vn && newmin >= oldmin)) return false;
  } else if (kind == 1) {
    double ex = 0.0, ey = 0.0;
    if (owne) qgrad_x(patch_geo(pe, pv), pe.k, st.qk, ex, ey);
    double t[3] = {ex, ey, owne ? qval(patch_geo(pe, pv), st.qk) : 0.0};
    gsums(t, g, lds);
    double gx = t[0], gy = t[1], Qold = t[2];
    if (gx == 0.0 && gy == 0.0) return false;
    double ax = fabs(gx), ay = fabs(gy);
    double nrm = ax < ay ? ay : ax;
    double dx = gx / nrm, dy = gy / nrm;
    double hx = fabs(pw.x - pv.x), hy = fabs(pw.y - pv.y);
    double hh = gmin(hx < hy ? hy : hx, h.y, g);
    bool vo;
    double oldmin = gpatch_min(pe, owne, pv, h.w, g, st.qk, vo);
    double step = hh;
    bool ok = false;
    for (int k = 1; k <= 4 && !ok; ++k) {
      step = step * 0.5;
      p = make_double2(pv.x + step * dx, pv.y + step * dy);
      bool vn;
      double newmin = gpatch_min(pe, owne, p, h.w, g, st.qk, vn);
      if (!vn || !(newmin >= oldmin)) continue;
      if (!(gpatch_q(pe, owne, p, g, st.qk, lds) > Qold)) continue;
      ok = true;
    }
    if (!ok) return false;
  } else {
    // min-max: the worst element (smallest q, ties to the first in NE(v)) and
    // the second worst, taken in row order as a serial loop takes them
    double q = owne ? qval(patch_geo(pe, pv), st.qk) : 0.0;
    int i1 = -1, i2 = -1;
    double q1 = 0.0, q2 = 0.0;
#pragma unroll
    for (int k = 0; k < kG; ++k) {
      double t = gget(q, k, g);
      if (k < h.w) {
        if (i1 < 0 || t < q1) {
          i2 = i1;
          q2 = q1;
          i1 = k;
          q1 = t;
        } else if (i2 < 0 || t < q2) {
          i2 = k;
          q2 = t;
        }
      }
    }
    if (i1 < 0) return false;
    double ex = 0.0, ey = 0.0;
    if (owne) qgrad_x(patch_geo(pe, pv), pe.k, st.qk, ex, ey);
    double ax = gget(ex, i1, g), ay = gget(ey, i1, g);
    double bx = gget(ex, max(i2, 0), g), by = gget(ey, max(i2, 0), g);
    double gx = ax, gy = ay;
    if (i2 >= 0 && q2 <= q1 * 1.01) {
      double fx = bx - ax, fy = by - ay;
      double den = fx * fx + fy * fy;
      if (den > 0.0) {
        double lam = -(ax * fx + ay * fy) / den;
        lam = lam < 0.0 ? 0.0 : (lam > 1.0 ? 1.0 : lam);
        gx = ax + lam * fx;
        gy = ay + lam * fy;
      }
    }
    if (gx == 0.0 && gy == 0.0) return false;
    double nx = fabs(gx), ny = fabs(gy);
    double nrm = nx < ny ? ny : nx;
    double dx = gx / nrm, dy = gy / nrm;
    double hx = fabs(pw.x - pv.x), hy = fabs(pw.y - pv.y);
    double hh = gmin(hx < hy ? hy : hx, h.y, g);
    bool vo;
    double oldmin = gpatch_min(pe, owne, pv, h.w, g, st.qk, vo);
    double step = hh;
    bool ok = false;
    for (int k = 0; k < 4 && !ok; ++k) {
      step = step * 0.5;
      p = make_double2(pv.x + step * dx, pv.y + step * dy);
      bool vn;
      double newmin = gpatch_min(pe, owne, p, h.w, g, st.qk, vn);
      if (!vn || !(newmin > oldmin)) continue;
      ok = true;
    }
    if (!ok) return false;
  }
  if (g.j == 0) st.xy[v] = p;
  return true;
}

// one kernel per smoothing kind (K = 0 plain, 1 gradient), each with its own
// register allocation
template <int K, int QK>
__global__ void __launch_bounds__(256, 4) k_smooth_g(Store st, const int* __restrict__ list, int n, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  __shared__ __align__(16) double terms[kBlock / kWave][kSmoothSums * kSumW];
  double* lds = terms[threadIdx.x / kWave];
  Grp g = grp();
  int gid = (int)(((int64_t)xcd_block() * blockDim.x + threadIdx.x) / kG);
  int status = -1;
  if (gid < n) {
    int v = list[gid];
    Hdr h = st.hdr[v];
    if (h.y > kG || h.w > kG) {
      if (g.j == 0)
        status = (K == 0 ? smooth_laplace(st, v) : (K == 1 ? smooth_gradient(st, v) : smooth_minmax(st, v))) ? 2 : 1;
    } else {
      bool moved = smooth_group(st, v, h, K, g, lds);
      if (g.j == 0) status = moved ? 2 : 1;
    }
  }
  count_status(status, ctr);
}
template __global__ void k_smooth_g<0, 0>(Store, const int*, int, int*);
template __global__ void k_smooth_g<0, 1>(Store, const int*, int, int*);
template __global__ void k_smooth_g<1, 0>(Store, const int*, int, int*);
template __global__ void k_smooth_g<2, 0>(Store, const int*, int, int*);
template __global__ void k_smooth_g<2, 1>(Store, const int*, int, int*);
template __global__ void k_smooth_g<1, 1>(Store, const int*, int, int*);

// ---- collapse with lane groups -----------------------------------------------------------------
// G lanes per member (G = kGC): small classes are made of the vertices that
// earlier rounds left, often of high degree, so the groups are wider here.
template <int G>
__device__ __forceinline__ Grp grp_of() {
  int l = __lane_id();
  return Grp{l & (G - 1), l & ~(G - 1)};
}
template <int G>
__device__ __forceinline__ bool gany_of(bool p, const Grp& g) {
  uint64_t b = __ballot(p);
  return ((b >> g.base) & ((1ull << G) - 1ull)) != 0;
}
template <int G>
__device__ __forceinline__ int collapse_group(const Store& st, int v, Hdr h, const OpArgs& a, const Commit& cm, int* ctr, const Grp& g) {
  bool ownn = g.j < h.y, owne = g.j < h.w;
  // loads by dependency level, each level issued together (index 0 stands
  // in for a lane with no neighbour or element): the member's own data and
  // its rows' entries; then each neighbour's round word and data and each
  // element; the deferral test comes after them
  uint64_t rv = a.rw[v];
  VRec rcv = st.vr[v];
  double2 pv = make_double2(rcv.x, rcv.y);
  Met mv{rcv.a, rcv.b, rcv.c};
  int tv = rcv.tag;
  int w = ownn ? st.nn[h.x + g.j] : -1;
  int t = owne ? st.ne[h.z + g.j] : -1;
  int ws = max(w, 0);
  uint64_t xw = a.rw[ws];
  VRec rcw = st.vr[ws];
  double2 pw = make_double2(rcw.x, rcw.y);
  Met mw{rcw.a, rcw.b, rcw.c};
  int tw = rcw.tag;
  Elem e = st.tri[max(t, 0)];
  bool beat = ownn && (xw & kRwAct) && (int)(xw & 0xFF) == a.cls && rw_beats(xw, w, rv, v);
  if (gany_of<G>(beat, g)) {
    if (g.j == 0) cm.nxt[v] = 1;
    return 0;
  }
  double L = INFINITY;
  bool cand = false;
  if (ownn) {
    if (!(tv & ~tw)) {
      L = len2(pv, mv, pw, mw);
      cand = L < a.L_low2;
    }
  } else {
    pw = make_double2(0.0, 0.0);
    mw = Met{0.0, 0.0, 0.0};
  }
  // element lane: ids and data of the element's other two vertices
  double2 q0 = make_double2(0.0, 0.0), q1 = q0;
  Met n0{0.0, 0.0, 0.0}, n1 = n0;
  int o0 = -1, o1 = -1, k = 0;
  if (!owne) e = make_int4(0, 0, 0, 0);
  if (owne) {
    k = slot_of(e, v);
    o0 = at(e, k == 2 ? 0 : k + 1);  // next after v
    o1 = at(e, k == 0 ? 2 : k - 1);  // before v
    VRec r0 = st.vr[o0], r1 = st.vr[o1];
    q0 = make_double2(r0.x, r0.y);
    q1 = make_double2(r1.x, r1.y);
    n0 = Met{r0.a, r0.b, r0.c};
    n1 = Met{r1.a, r1.b, r1.c};
  }
  double lastL = -INFINITY;
  int lastU = -1, u = -1;
  for (;;) {
    // group minimum of (L, w) over candidates after (lastL, lastU)
    bool after = cand && (L > lastL || (L == lastL && w > lastU));
    double bL = after ? L : INFINITY;
    int bU = after ? w : INT_MAX;
    int bj = after ? g.j : -1;
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
      double oL = __shfl_xor(bL, d);
      int oU = __shfl_xor(bU, d);
      int oj = __shfl_xor(bj, d);
      if (oL < bL || (oL == bL && oU < bU)) {
        bL = oL;
        bU = oU;
        bj = oj;
      }
    }
    if (bj < 0) break;
    // the candidate's data from the lane that owns it
    double2 pu = make_double2(gget(pw.x, bj, g), gget(pw.y, bj, g));
    Met mu{gget(mw.a, bj, g), gget(mw.b, bj, g), gget(mw.c, bj, g)};
    bool bad = false;
    if (owne && o0 != bU && o1 != bU) {
      // element (u, o0, o1) in cyclic order, rotated smallest id first
      int r;  // rotation: which of (u, o0, o1) comes first
      if (bU < o0 && bU < o1) r = 0;
      else if (o0 < bU && o0 < o1) r = 1;
      else r = 2;
      double2 c0 = r == 0 ? pu : (r == 1 ? q0 : q1);
      double2 c1 = r == 0 ? q0 : (r == 1 ? q1 : pu);
      double2 c2 = r == 0 ? q1 : (r == 1 ? pu : q0);
      Met d0 = r == 0 ? mu : (r == 1 ? n0 : n1);
      Met d1 = r == 0 ? n0 : (r == 1 ? n1 : mu);
      Met d2 = r == 0 ? n1 : (r == 1 ? mu : n0);
      Geo gg = make_geo(c0, c1, c2, d0, d1, d2);
      bad = !(area2(gg) > 0.0) || !(qd2(gg, st.qk) >= a.qmin2);
    }
    if (!gany_of<G>(bad, g)) {
      u = bU;
      break;
    }
    lastL = bL;
    lastU = bU;
  }
  if (u < 0) return 1;
  if (owne) {
    Elem ne;
    if (o0 == u || o1 == u) {
      ne = e;
      ne.w = 0;
    } else {
      int3 r3 = rot_min(u, o0, o1);
      ne = make_int4(r3.x, r3.y, r3.z, 1);
    }
    st.tri[t] = ne;
  }
  if (ownn) claim_row(cm, w, v);
  if (g.j == 0) {
    st.valive[v] = 0;
    stamp(cm, v, -(u + 1), h.z, h.w);
    mark_target(cm, u, h.z, h.w);
  }
  return 2;
}

template <int G, int QK>
__global__ void __launch_bounds__(256, 5) k_collapse_g(Store st, const int* __restrict__ list, int n, OpArgs a,
                                                    Commit cm, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  if (room_failed(ctr)) return;
  Grp g = grp_of<G>();
  if (blockIdx.x == 0 && threadIdx.x == 0) ctr[C_STAGE] = 0;  // the commit's fallback staging
  int gid = (int)(((int64_t)xcd_block() * blockDim.x + threadIdx.x) / G);
  int status = -1;
  if (gid < n) {
    int v = list[gid];
    Hdr h = st.hdr[v];
    if (h.y > G || h.w > G) {
      if (g.j == 0) status = collapse_one(st, v, a, cm, ctr);
    } else {
      int r = collapse_group<G>(st, v, h, a, cm, ctr, g);
      if (g.j == 0) status = r;
    }
  }
  count_status(status, ctr, true);
}
template __global__ void k_collapse_g<8, 0>(Store, const int*, int, OpArgs, Commit, int*);
template __global__ void k_collapse_g<8, 1>(Store, const int*, int, OpArgs, Commit, int*);
template __global__ void k_collapse_g<16, 0>(Store, const int*, int, OpArgs, Commit, int*);
template __global__ void k_collapse_g<16, 1>(Store, const int*, int, OpArgs, Commit, int*);

// ---- flips with lane groups -----------------------------------------------------------------------
// Lane j owns the member's j-th element T1 = (v, w, a) (cyclic from v): the
// edge (v, w) and its data. The element across that edge, T2, is the one
// whose vertex before v is w; the lane holding it hands over its id, its
// other vertex b and its quality. Each lane then evaluates the flip of its
// edge; the group keeps the largest new minimum quality, ties to the smaller
// w, as the one-thread scan does.
template <int G>
__device__ __forceinline__ int flip_group(const Store& st, int v, Hdr h, const OpArgs& a, const Commit& cm,
                                          const Grp& g) {
  bool ownn = g.j < h.y, owne = g.j < h.w;
  // loads by dependency level, each level issued together: the member's
  // data and its rows' entries, then the neighbours' round words and the
  // elements; the deferral test comes after them
  uint64_t rv = a.rw[v];
  VRec rcv = st.vr[v];
  double2 pv = make_double2(rcv.x, rcv.y);
  Met mv{rcv.a, rcv.b, rcv.c};
  int y = ownn ? st.nn[h.x + g.j] : -1;
  int T1 = owne ? st.ne[h.z + g.j] : -1;
  uint64_t ry = a.rw[max(y, 0)];
  Elem e1 = st.tri[max(T1, 0)];
  bool beat = ownn && (ry & kRwAct) && (int)(ry & 0xFF) == a.cls && rw_beats(ry, y, rv, v);
  if (gany_of<G>(beat, g)) {
    if (g.j == 0) cm.nxt[v] = 1;
    return 0;
  }
  int k1 = 0, w = -1, av = -1;
  double2 pw = make_double2(0.0, 0.0), pa = pw;
  Met mw{0.0, 0.0, 0.0}, ma = mw;
  if (owne) {
    k1 = slot_of(e1, v);
    w = at(e1, k1 == 2 ? 0 : k1 + 1);
    av = at(e1, k1 == 0 ? 2 : k1 - 1);
    VRec rcw = st.vr[w], rca = st.vr[av];
    pw = make_double2(rcw.x, rcw.y);
    mw = Met{rcw.a, rcw.b, rcw.c};
    pa = make_double2(rca.x, rca.y);
    ma = Met{rca.a, rca.b, rca.c};
  }
  // quality of T1 in its stored order (slot k1 holds v, then w, then a)
  double q1 = 0.0;
  if (owne) {
    double2 s0 = k1 == 0 ? pv : (k1 == 1 ? pa : pw);
    double2 s1 = k1 == 1 ? pv : (k1 == 2 ? pa : pw);
    double2 s2 = k1 == 2 ? pv : (k1 == 0 ? pa : pw);
    Met n0 = k1 == 0 ? mv : (k1 == 1 ? ma : mw);
    Met n1 = k1 == 1 ? mv : (k1 == 2 ? ma : mw);
    Met n2 = k1 == 2 ? mv : (k1 == 0 ? ma : mw);
    q1 = qd2(make_geo(s0, s1, s2, n0, n1, n2), st.qk);
  }
  // the lane whose element has w before v holds T2
  int j2 = -1;
#pragma unroll
  for (int q = 0; q < G; ++q) {
    int pq = gget(av, q, g);
    if (j2 < 0 && owne && q < h.w && pq == w) j2 = q;
  }
  int src = g.base + (j2 >= 0 ? j2 : 0);
  int T2 = __shfl(T1, src);
  int bv = __shfl(w, src);
  double2 pb = make_double2(__shfl(pw.x, src), __shfl(pw.y, src));
  Met mb{__shfl(mw.a, src), __shfl(mw.b, src), __shfl(mw.c, src)};
  double q2 = __shfl(q1, src);
  bool cand = owne && j2 >= 0;
  double nmin = 0.0;
  if (cand) {
    // (v, b, a) and (w, a, b), each rotated smallest id first
    int r1 = (v < bv && v < av) ? 0 : ((bv < v && bv < av) ? 1 : 2);
    double2 c0 = r1 == 0 ? pv : (r1 == 1 ? pb : pa);
    double2 c1 = r1 == 0 ? pb : (r1 == 1 ? pa : pv);
    double2 c2 = r1 == 0 ? pa : (r1 == 1 ? pv : pb);
    Met d0 = r1 == 0 ? mv : (r1 == 1 ? mb : ma);
    Met d1 = r1 == 0 ? mb : (r1 == 1 ? ma : mv);
    Met d2 = r1 == 0 ? ma : (r1 == 1 ? mv : mb);
    Geo gv = make_geo(c0, c1, c2, d0, d1, d2);
    int r2 = (w < av && w < bv) ? 0 : ((av < w && av < bv) ? 1 : 2);
    double2 e0 = r2 == 0 ? pw : (r2 == 1 ? pa : pb);
    double2 e1p = r2 == 0 ? pa : (r2 == 1 ? pb : pw);
    double2 e2 = r2 == 0 ? pb : (r2 == 1 ? pw : pa);
    Met f0 = r2 == 0 ? mw : (r2 == 1 ? ma : mb);
    Met f1 = r2 == 0 ? ma : (r2 == 1 ? mb : mw);
    Met f2 = r2 == 0 ? mb : (r2 == 1 ? mw : ma);
    Geo gw = make_geo(e0, e1p, e2, f0, f1, f2);
    if (!(area2(gv) > 0.0) || !(area2(gw) > 0.0)) {
      cand = false;
    } else {
      double qv = qd2(gv, st.qk), qw = qd2(gw, st.qk);
      nmin = qw < qv ? qw : qv;
      double omin = q2 < q1 ? q2 : q1;
      cand = nmin > omin;
    }
  }
  // the best candidate: largest new minimum, ties to the smaller w
  double bq = cand ? nmin : -INFINITY;
  int bw = cand ? w : INT_MAX;
  int bj = cand ? g.j : -1;
#pragma unroll
  for (int d = 1; d < G; d <<= 1) {
    double oq = __shfl_xor(bq, d);
    int ow = __shfl_xor(bw, d);
    int oj = __shfl_xor(bj, d);
    if (oj >= 0 && (bj < 0 || oq > bq || (oq == bq && ow < bw))) {
      bq = oq;
      bw = ow;
      bj = oj;
    }
  }
  if (bj < 0) return 1;
  if (g.j == bj) {
    int lo = min(T1, T2), hi = max(T1, T2);
    int3 tv = rot_min(v, bv, av), tw = rot_min(w, av, bv);
    st.tri[lo] = make_int4(tv.x, tv.y, tv.z, 1);
    st.tri[hi] = make_int4(tw.x, tw.y, tw.z, 1);
    stamp(cm, v, lo, hi, 0);
    mark_target(cm, av, lo, hi);
    mark_target(cm, bv, lo, hi);
    claim_row(cm, v, v);
    claim_row(cm, w, v);
    claim_row(cm, av, v);
    claim_row(cm, bv, v);
  }
  return 2;
}

template <int G, int QK>
__global__ void __launch_bounds__(256) k_flip_g(Store st, const int* __restrict__ list, int n, OpArgs a, Commit cm,
                                                int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  if (room_failed(ctr)) return;
  Grp g = grp_of<G>();
  if (blockIdx.x == 0 && threadIdx.x == 0) ctr[C_STAGE] = 0;  // the commit's fallback staging
  int gid = (int)(((int64_t)xcd_block() * blockDim.x + threadIdx.x) / G);
  int status = -1;
  if (gid < n) {
    int v = list[gid];
    Hdr h = st.hdr[v];
    if (h.y > G || h.w > G) {
      if (g.j == 0) status = flip_one(st, v, a, cm, ctr);
    } else {
      int r = flip_group<G>(st, v, h, a, cm, g);
      if (g.j == 0) status = r;
    }
  }
  count_status(status, ctr, true);
}
void flip_class_g(const Store& st, const int* list, int n, OpArgs a, Commit cm, int* ctr, hipStream_t s) {
  if (n > 0) (st.qk ? k_flip_g<16, 1> : k_flip_g<16, 0>)<<<(int)(((int64_t)n * 16 + kBlock - 1) / kBlock), kBlock, 0, s>>>(
      st, list, n, a, cm, ctr);
}

// A small class in one block: the operation (collapse or flips on groups of
// kGC lanes per member), a block barrier, then the commit of the same
// members. Every thread reaches every barrier.
constexpr int kClassThreads = 512;
template <bool F>
__device__ __forceinline__ void class_body(const Store& st, const int* list, int n, const OpArgs& a,
                                           const Commit& cm, int* ctr, CommitLds<kClassThreads>& L) {
  constexpr int NT = kClassThreads;
  int tid = (int)threadIdx.x;
  if (tid == 0) ctr[C_STAGE] = 0;  // the commit's fallback staging
  Grp g = grp_of<kGC>();
  for (int p0 = 0; p0 < n; p0 += NT / kGC) {
    int gid = p0 + tid / kGC;
    int status = -1;
    if (gid < n) {
      int v = list[gid];
      Hdr h = st.hdr[v];
      if (h.y > kGC || h.w > kGC) {
        if (g.j == 0) status = F ? flip_one(st, v, a, cm, ctr) : collapse_one(st, v, a, cm, ctr);
      } else {
        int r = F ? flip_group<kGC>(st, v, h, a, cm, g) : collapse_group<kGC>(st, v, h, a, cm, ctr, g);
        if (g.j == 0) status = r;
      }
    }
    count_status(status, ctr);
  }
  __syncthreads();
  for (int base = 0; base < n; base += NT) commit_chunk<F, NT>(st, list, base, min(NT, n - base), cm, ctr, L);
}

// one small class, one launch instead of two
template <bool F, int QK>
__global__ void __launch_bounds__(kClassThreads) k_class_small(Store st, const int* __restrict__ list, int n, OpArgs a,
                                                               Commit cm, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  __shared__ CommitLds<kClassThreads> L;
  if (room_failed_block(ctr)) return;
  class_body<F>(st, list, n, a, cm, ctr, L);
}
void class_small(const Store& st, const int* list, int n, OpArgs a, Commit cm, int kind, int* ctr, hipStream_t s) {
  if (n <= 0) return;
  auto k = kind ? (st.qk ? k_class_small<true, 1> : k_class_small<true, 0>)
                : (st.qk ? k_class_small<false, 1> : k_class_small<false, 0>);
  k<<<1, kClassThreads, 0, s>>>(st, list, n, a, cm, ctr);
}

// Every class of a round in one block, one after the other (a round whose
// classes are all small): class c takes epoch epoch0 + c and its size and
// offset from the colouring's counters. Returns false when a commit ran out
// of room: the host rebuilds the rows and runs the remaining classes.
template <bool F>
__device__ __forceinline__ bool round_body(const Store& st, const int* cls, int ncol, int epoch0,
                                           const OpArgs& a, const Commit& cm, int* ctr, CommitLds<kClassThreads>& L) {
  for (int c = 0; c < ncol; ++c) {
    if (room_failed_block(ctr)) return false;
    int n = ctr[C_HIST + c], off = ctr[C_OFF + c];
    if (n == 0) continue;
    Commit cc = cm;
    cc.epoch = epoch0 + c;
    OpArgs ac = a;
    ac.cls = c;
    class_body<F>(st, cls + off, n, ac, cc, ctr, L);
  }
  return !room_failed_block(ctr);
}

// One launch per round instead of one per class, and the block's caches stay
// warm from class to class.
template <bool F, int QK>
__global__ void __launch_bounds__(kClassThreads) k_round_small(Store st, const int* __restrict__ cls, int ncol, OpArgs a,
                                                               Commit cm, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  __shared__ CommitLds<kClassThreads> L;
  round_body<F>(st, cls, ncol, cm.epoch, a, cm, ctr, L);
}
void round_small(const Store& st, const int* cls, int ncol, OpArgs a, Commit cm, int kind, int* ctr, hipStream_t s) {
  if (ncol == 0) return;
  auto k = kind ? (st.qk ? k_round_small<true, 1> : k_round_small<true, 0>)
                : (st.qk ? k_round_small<false, 1> : k_round_small<false, 0>);
  k<<<1, kClassThreads, 0, s>>>(st, cls, ncol, a, cm, ctr);
}

// Rounds driven by the device: from the coloured round ctr[C_DROUND] on, one
// block runs a round's classes, clears its round words, selects the next
// list (from list A into list B, then the other way round) and colours it,
// and goes on until the list is empty, the round cap or the launch's budget of
// rounds is reached, a selection declines (C_LIST_B = -1), or a list or class
// is too large for one block (the list is then uncoloured, C_NCOL = -1, or
// coloured and left to the host). With four launches a round (classes, round
// words, selection, colouring) the 64 such rounds of a 33 x 33 adaptation took
// 256 launches and 1.2 ms of kernels; in 16 launches they take 0.59 ms. 512
// threads: 32 members or rows at a time, against 16 with 256 (the flips' 165
// registers leave no room for 1024).
// LDS: the classes' and the colouring's are never in use together.
constexpr int kDevItems = 2;  // vertices a thread colours, at most
template <bool F, int QK>
__global__ void __launch_bounds__(kClassThreads) k_rounds_dev(Store st, DevRounds d, OpArgs a, Commit cm, int* ctr) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  constexpr int NT = kClassThreads;
  __shared__ union {
    CommitLds<NT> commit;
    ColourLds colour;
  } L;
  __shared__ int cnt;
  int tid = (int)threadIdx.x;
  int r = ctr[C_DROUND], stop = ctr[C_DSTOP], epoch = ctr[C_DEPOCH], epoch0 = ctr[C_DEPOCH0], mark = ctr[C_DMARK];
  int n = ctr[C_LIST_B], ncol = ctr[C_NCOL];
  int acc_col = ctr[C_ACC_COL], acc_ncol = ctr[C_ACC_NCOL], acc_it = ctr[C_ACC_IT];
  if (d.start) {
    r = d.round;
    epoch = epoch0 = d.epoch;
    mark = d.mark;
    stop = r >= d.max_rounds ? 1 : 0;
    acc_col = acc_ncol = acc_it = 0;
  }
  __syncthreads();  // every thread has read the counters before they change
  for (int k = 0; k < d.budget && !stop; ++k) {
    const int* A = (r ^ d.par) & 1 ? d.L1 : d.L0;
    int* B = (r ^ d.par) & 1 ? d.L0 : d.L1;
    epoch0 = epoch;
    epoch += ncol;
    bool room = round_body<F>(st, d.cls, ncol, epoch0, a, cm, ctr, L.commit);
    for (int i = tid; i < n; i += NT) d.rw[A[i]] = 0;
    int nt = __hip_atomic_load(&ctr[C_TOUCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!room || nt > cm.touched_cap) {
      n = -1;
      stop = 1;
      break;
    }
    n = select_body<NT>(st, d.mode, a.L_low2, A, n, cm.touched, nt, cm.nxt, d.seen, ++mark, B, &cnt);
    ++r;
    if (n == 0 || r >= d.max_rounds) {
      ncol = 0;
      stop = 1;
      break;
    }
    if (n > kDevItems * NT) {
      ncol = -1;
      stop = 1;
      break;
    }
    Round rd{stream_seed(d.seed, make_ctx(d.sweep, d.phase, r)), d.rw};
    int big = colour_body<NT, kDevItems>(st, B, n, nullptr, rd, d.cls, ctr, L.colour);
    ncol = L.colour.ncol;
    int its = L.colour.its;
    __syncthreads();
    if (big > kSmallClass) {
      // the host runs this round, coloured as it is (and counts it)
      stop = 1;
      break;
    }
    acc_col += n;
    acc_ncol += ncol;
    acc_it += its;
  }
  __syncthreads();
  if (tid == 0) {
    ctr[C_DROUND] = r;
    ctr[C_DEPOCH] = epoch;
    ctr[C_DEPOCH0] = epoch0;
    ctr[C_DMARK] = mark;
    ctr[C_DSTOP] = stop;
    ctr[C_LIST_B] = n;
    ctr[C_NCOL] = ncol;
    ctr[C_ACC_COL] = acc_col;
    ctr[C_ACC_NCOL] = acc_ncol;
    ctr[C_ACC_IT] = acc_it;
  }
}
void rounds_dev(const Store& st, const DevRounds& d, OpArgs a, Commit cm, int kind, int* ctr, hipStream_t s) {
  auto k = kind ? (st.qk ? k_rounds_dev<true, 1> : k_rounds_dev<true, 0>)
                : (st.qk ? k_rounds_dev<false, 1> : k_rounds_dev<false, 0>);
  k<<<1, kClassThreads, 0, s>>>(st, d, a, cm, ctr);
}

// ---- adjoint with lane groups ---------------------------------------------------------------------
template <int QK>
__global__ void __launch_bounds__(256) k_adjoint_g(Store st, double* __restrict__ dQdx, double* __restrict__ dQdM) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  __shared__ __align__(16) double terms[kBlock / kWave][5 * kSumW];
  double* lds = terms[threadIdx.x / kWave];
  Grp g = grp();
  int v = (int)(((int64_t)xcd_block() * blockDim.x + threadIdx.x) / kG);
  if (v >= st.V) return;
  Hdr h = st.hdr[v];
  double sum = 0.0;  // lane 0, 1: dQ/dx; 2, 3, 4: dQ/dM
  for (int c0 = 0; c0 < h.w; c0 += kG) {
    double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (c0 + g.j < h.w) {
      Elem e = st.tri[st.ne[h.z + c0 + g.j]];
      Geo gg = geo_of(st, e);
      qgrad_x(gg, slot_of(e, v), st.qk, t[0], t[1]);
      qgrad_m(gg, st.qk, t[2], t[3], t[4]);
      t[2] = third(t[2]);
      t[3] = third(t[3]);
      t[4] = third(t[4]);
    }
    // terms past a row's first eight go on from its sum so far
    if (c0 == 0) {
      sum = gsum_lane<5>(t, g, lds);
    } else {
#pragma unroll
      for (int c = 0; c < 5; ++c) lds[c * kSumW + g.base + g.j] = t[c];
      wave_lds();
      for (int k = 0; k < kG; ++k) sum = sum + lds[(g.j < 5 ? g.j : 0) * kSumW + g.base + k];
      wave_lds();
    }
  }
  if (g.j < 2) {
    if (dQdx) dQdx[2 * (int64_t)v + g.j] = sum;
  } else if (g.j < 5) {
    if (dQdM) dQdM[3 * (int64_t)v + g.j - 2] = sum;
  }
}

// ---- quality functional and adjoint (Sec. 2.2) --------------------------------------------------
constexpr int QB = 256;

template <int QK>
__global__ void k_quality(Store st, double* __restrict__ psum, double* __restrict__ pmin) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  __shared__ double ls[QB], lm[QB];
  double s = 0.0, mn = INFINITY;
  for (int t = gtid(); t < st.T; t += gstride()) {
    Elem e = st.tri[t];
    if (!e.w) continue;
    double q = qval(geo_of(st, e), st.qk);
    s = s + q;
    mn = q < mn ? q : mn;
  }
  ls[threadIdx.x] = s;
  lm[threadIdx.x] = mn;
  __syncthreads();
  for (int d = QB / 2; d > 0; d >>= 1) {
    if ((int)threadIdx.x < d) {
      ls[threadIdx.x] = ls[threadIdx.x] + ls[threadIdx.x + d];
      double o = lm[threadIdx.x + d];
      lm[threadIdx.x] = o < lm[threadIdx.x] ? o : lm[threadIdx.x];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    psum[blockIdx.x] = ls[0];
    pmin[blockIdx.x] = lm[0];
  }
}
__global__ void k_quality_final(const double* __restrict__ psum, const double* __restrict__ pmin, int np,
                                double* __restrict__ out, int* at, int no) {
  __shared__ double ls[QB], lm[QB];
  double s = 0.0, mn = INFINITY;
  for (int i = threadIdx.x; i < np; i += QB) {
    s = s + psum[i];
    mn = pmin[i] < mn ? pmin[i] : mn;
  }
  ls[threadIdx.x] = s;
  lm[threadIdx.x] = mn;
  __syncthreads();
  for (int d = QB / 2; d > 0; d >>= 1) {
    if ((int)threadIdx.x < d) {
      ls[threadIdx.x] = ls[threadIdx.x] + ls[threadIdx.x + d];
      double o = lm[threadIdx.x + d];
      lm[threadIdx.x] = o < lm[threadIdx.x] ? o : lm[threadIdx.x];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = ls[0];
    out[1] = lm[0];
  }
  mail_post(at, no);
}
// one block per mesh of a batch: Q and qmin of each mesh's element range
template <int QK>
__global__ void k_quality_mesh(Store st, double* __restrict__ out) {
  st.qk = QK;  // the functional as a constant: one instantiation per kind
  __shared__ double ls[QB], lm[QB];
  int i = blockIdx.x;
  int lo = st.tbase[i], hi = st.tbase[i] + st.tused[i];
  double s = 0.0, mn = INFINITY;
  for (int t = lo + (int)threadIdx.x; t < hi; t += QB) {
    Elem e = st.tri[t];
    if (!e.w) continue;
    double q = qval(geo_of(st, e), st.qk);
    s = s + q;
    mn = q < mn ? q : mn;
  }
  ls[threadIdx.x] = s;
  lm[threadIdx.x] = mn;
  __syncthreads();
  for (int d = QB / 2; d > 0; d >>= 1) {
    if ((int)threadIdx.x < d) {
      ls[threadIdx.x] = ls[threadIdx.x] + ls[threadIdx.x + d];
      double o = lm[threadIdx.x + d];
      lm[threadIdx.x] = o < lm[threadIdx.x] ? o : lm[threadIdx.x];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * i] = ls[0];
    out[2 * i + 1] = lm[0];
  }
}
void quality_per_mesh(const Store& st, double* out, hipStream_t s) {
  (st.qk ? k_quality_mesh<1> : k_quality_mesh<0>)<<<st.B, QB, 0, s>>>(st, out);
}

void quality_sum(const Store& st, double* psum, double* pmin, int nparts, double* out2, const Mail& b, hipStream_t s) {
  (st.qk ? k_quality<1> : k_quality<0>)<<<nparts, QB, 0, s>>>(st, psum, pmin);
  k_quality_final<<<1, QB, 0, s>>>(psum, pmin, nparts, out2, (int*)b.at, b.no);
}

void quality_adjoint(const Store& st, double* dQdx, double* dQdM, hipStream_t s) {
  (st.qk ? k_adjoint_g<1> : k_adjoint_g<0>)<<<(int)(((int64_t)st.V * kG + kBlock - 1) / kBlock), kBlock, 0, s>>>(
      st, dQdx, dQdM);
}

__global__ void k_fp64_probe(const double* __restrict__ a, const double* __restrict__ b, int n,
                             double* __restrict__ q, double* __restrict__ r) {
  for (int i = gtid(); i < n; i += gstride()) {
    q[i] = a[i] / b[i];
    r[i] = sqrt(a[i]);
  }
}
void fp64_probe(const double* a, const double* b, int n, double* q, double* r, hipStream_t s) {
  k_fp64_probe<<<grid_for(n), kBlock, 0, s>>>(a, b, n, q, r);
}

}  // namespace pm
