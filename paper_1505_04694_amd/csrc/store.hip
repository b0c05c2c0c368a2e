// Device mesh store: ordered scan, input validation, slack-padded CSR rows
// built from the element list, stable compaction, and template refinement.
//
// Rows: NE(v) = live elements holding v, NN(v) = the other vertices of those
// elements (Sec. 3.1: per-vertex adjacency lists). Every row is a sorted id
// set stored in a slack-padded slot of its pool, so the commit can grow it in
// place; a row that outgrows its slot moves to the pool's bump region.
#include <algorithm>

#include "kern.hpp"
#include "scan.hpp"

namespace pm {

// ---- ordered exclusive scan --------------------------------------------------------
// room for the chunk sums of the finest split
int scan_partials_needed(int n) { return n / kBlock + 4; }

// short arrays: one block of 1024 threads, each scanning a contiguous piece
// of at most eight entries (its loads are serial, two passes: longer pieces
// made a 65536-entry scan take 100 us, against a few for the three-kernel
// form)
constexpr int kScanSingle = 8192;
__global__ void __launch_bounds__(1024) k_scan_single(const int* __restrict__ in, int* __restrict__ out, int n,
                                                      int* __restrict__ total) {
  __shared__ int lds[1024 / kWave];
  int per = (n + 1023) / 1024;
  int lo = (int)threadIdx.x * per;
  int hi = min(n, lo + per);
  int s = 0;
  for (int i = lo; i < hi; ++i) s += in[i];
  int tot;
  int acc = block_excl(s, lds, tot);
  for (int i = lo; i < hi; ++i) {
    int t = in[i];
    out[i] = acc;
    acc += t;
  }
  if (threadIdx.x == 0) *total = tot;
}

void scan_excl(const int* in, int* out, int n, int* total, int* partial, hipStream_t s) {
  if (n <= kScanSingle) {
    k_scan_single<<<1, 1024, 0, s>>>(in, out, n, total);
    return;
  }
  scan_fused<int, 8>([=] __device__(int i, bool on) { return on ? in[i] : 0; }, [=] __device__(int i) { return in[i]; },
                     [=] __device__(int i, int at, int) { out[i] = at; }, [=] __device__(int t) { *total = t; }, n,
                     partial, s);
}

// ---- validation ---------------------------------------------------------------------
// elements arrive already rotated (smallest id first) by the creation kernel
__global__ void k_validate_elems(const Elem* __restrict__ tri, int T, int V, const double2* __restrict__ xy,
                                 int* ctr) {
  for (int t = gtid(); t < T; t += gstride()) {
    Elem e = tri[t];
    if (!e.w) continue;  // unused slot of a mesh's range
    if (e.x < 0 || e.y < 0 || e.z < 0 || e.x >= V || e.y >= V || e.z >= V || e.x == e.y || e.y == e.z ||
        e.x == e.z) {
      atomicOr(&ctr[C_ERR], E_MESH_ID);
      continue;
    }
    double2 p0 = xy[e.x], p1 = xy[e.y], p2 = xy[e.z];
    double D = (p1.x - p0.x) * (p2.y - p0.y) - (p2.x - p0.x) * (p1.y - p0.y);
    if (!(D > 0.0)) atomicOr(&ctr[C_ERR], E_MESH_ORIENT);
  }
}

__global__ void k_validate_verts(const double2* __restrict__ xy, const Met* __restrict__ met,
                                 const uint8_t* __restrict__ valive, int V, int* ctr) {
  for (int v = gtid(); v < V; v += gstride()) {
    if (!valive[v]) continue;
    Met m = met[v];
    double2 p = xy[v];
    bool ok = (m.a > 0.0) && (m.a * m.c - m.b * m.b > 0.0) && isfinite(m.a) && isfinite(m.b) &&
              isfinite(m.c) && isfinite(p.x) && isfinite(p.y);
    if (!ok) atomicOr(&ctr[C_ERR], E_MESH_METRIC);
  }
}

void k_validate(const Store& st, int* ctr, hipStream_t s) {
  k_validate_elems<<<grid_for(st.T), kBlock, 0, s>>>(st.tri, st.T, st.V, st.xy, ctr);
  k_validate_verts<<<grid_for(st.V), kBlock, 0, s>>>(st.xy, st.met, st.valive, st.V, ctr);
}

// ---- row build ----------------------------------------------------------------------
// Element-to-vertex incidence counts, and the place of each incidence in its
// vertex's NE row (rows are sorted by the row finish, so any order does). A block
// takes a contiguous chunk of kIncChunk elements; when the chunk's vertices span
// at most kIncSpan ids (meshes numbered with locality), it counts in LDS, where an
// incidence takes its rank among the chunk's, and makes one global atomic per
// vertex it touches instead of one per incidence, which reserves the chunk's
// places. The places go to the fill, which needs no atomics and no chunks:
// reserving again there, beside loads of the same headers, took 103 us on the 201^2
// planar-front mesh (670 thousand elements), the stores alone take 28. Counting
// there takes 50, the rate of global atomics: its chunks are wide and touch most
// vertices once, so a hash table in LDS in place of the window did not help (60).
constexpr int kIncPer = 4;
constexpr int kIncChunk = kBlock * kIncPer;
constexpr int kIncSpan = 4096;
struct Place3 {
  int x, y, z;
};
__device__ __forceinline__ void chunk_span(const Elem (&e)[kIncPer], int& vmin, int& vmax, int* red) {
  int lo = INT_MAX, hi = -1;
#pragma unroll
  for (int r = 0; r < kIncPer; ++r) {
    if (!e[r].w) continue;
    lo = min(lo, min(e[r].x, min(e[r].y, e[r].z)));
    hi = max(hi, max(e[r].x, max(e[r].y, e[r].z)));
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    lo = min(lo, __shfl_xor(lo, d));
    hi = max(hi, __shfl_xor(hi, d));
  }
  int wv = (int)threadIdx.x / kWave;
  if (__lane_id() == 0) {
    red[2 * wv] = lo;
    red[2 * wv + 1] = hi;
  }
  __syncthreads();
  vmin = INT_MAX;
  vmax = -1;
#pragma unroll
  for (int q = 0; q < kBlock / kWave; ++q) {
    vmin = min(vmin, red[2 * q]);
    vmax = max(vmax, red[2 * q + 1]);
  }
  __syncthreads();
}

__global__ void __launch_bounds__(256) k_ne_count(const Elem* __restrict__ tri, int T, int* __restrict__ cnt,
                                                 Place3* __restrict__ place) {
  __shared__ int loc[kIncSpan];
  __shared__ int red[2 * kBlock / kWave];
  int t0 = blockIdx.x * kIncChunk + (int)threadIdx.x;
  Elem e[kIncPer];
#pragma unroll
  for (int r = 0; r < kIncPer; ++r) e[r] = t0 + r * kBlock < T ? tri[t0 + r * kBlock] : make_int4(0, 0, 0, 0);
  int vmin, vmax;
  chunk_span(e, vmin, vmax, red);
  if (vmax < 0) return;
  int span = vmax - vmin + 1;
  if (span > kIncSpan) {
    Place3 k[kIncPer];
#pragma unroll
    for (int r = 0; r < kIncPer; ++r)
      if (e[r].w) k[r] = Place3{atomicAdd(&cnt[e[r].x], 1), atomicAdd(&cnt[e[r].y], 1), atomicAdd(&cnt[e[r].z], 1)};
#pragma unroll
    for (int r = 0; r < kIncPer; ++r)
      if (e[r].w && place) place[t0 + r * kBlock] = k[r];
    return;
  }
  for (int i = (int)threadIdx.x; i < span; i += kBlock) loc[i] = 0;
  __syncthreads();
  Place3 k[kIncPer];
#pragma unroll
  for (int r = 0; r < kIncPer; ++r)
    if (e[r].w)
      k[r] = Place3{atomicAdd(&loc[e[r].x - vmin], 1), atomicAdd(&loc[e[r].y - vmin], 1),
                    atomicAdd(&loc[e[r].z - vmin], 1)};
  __syncthreads();
  // loc[i] becomes the chunk's first place in row vmin + i; a thread's
  // reservations are all in flight before it uses one
  constexpr int R = kIncSpan / kBlock;
  int at[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    int i = q * kBlock + (int)threadIdx.x;
    int c = i < span ? loc[i] : 0;
    at[q] = c ? atomicAdd(&cnt[vmin + i], c) : 0;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    int i = q * kBlock + (int)threadIdx.x;
    if (i < span) loc[i] = at[q];
  }
  if (!place) return;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kIncPer; ++r)
    if (e[r].w)
      place[t0 + r * kBlock] =
          Place3{loc[e[r].x - vmin] + k[r].x, loc[e[r].y - vmin] + k[r].y, loc[e[r].z - vmin] + k[r].z};
}

void build_count(const Store& st, int* ne_cnt, int* place, hipStream_t s) {
  int nb = (st.T + kIncChunk - 1) / kIncChunk;
  if (nb > 0) k_ne_count<<<nb, kBlock, 0, s>>>(st.tri, st.T, ne_cnt, (Place3*)place);
}

__device__ __forceinline__ int round4(int x) { return (x + 3) & ~3; }

// a row's slots (NN, NE) for c elements
__device__ __forceinline__ int2 caps_of(int c, double slack) {
  if (c == 0) return make_int2(0, 0);
  int a = (int)ceil((double)c * slack);
  int b = (int)ceil((double)(c + 1) * slack);
  return make_int2(round4(max(c + 3, b)), round4(max(c + 2, a)));
}

// every row's header and slots, one behind the other in the pools, whose bump
// pointers the totals become
void build_headers(const Store& st, const int* ne_cnt, double slack, int* ctr, int2* partial, hipStream_t s) {
  Hdr* hdr = st.hdr;
  int2* cap = st.cap;
  scan_fused<int2, 8>([=] __device__(int v, bool on) { return on ? caps_of(ne_cnt[v], slack) : make_int2(0, 0); },
                      [=] __device__(int v) { return caps_of(ne_cnt[v], slack); },
                      [=] __device__(int v, int2 at, int2 c) {
                        hdr[v] = make_int4(at.x, 0, at.y, ne_cnt[v]);
                        cap[v] = c;
                      },
                      [=] __device__(int2 t) {
                        ctr[C_NN_TOP] = t.x;
                        ctr[C_NE_TOP] = t.y;
                      },
                      st.V, partial, s);
}

__global__ void __launch_bounds__(256) k_ne_fill(const Elem* __restrict__ tri, int T, const Hdr* __restrict__ hdr,
                                                const Place3* __restrict__ place, int* __restrict__ ne) {
  for (int t = gtid(); t < T; t += gstride()) {
    Elem e = tri[t];
    if (!e.w) continue;
    Place3 k = place[t];
    ne[hdr[e.x].z + k.x] = t;
    ne[hdr[e.y].z + k.y] = t;
    ne[hdr[e.z].z + k.z] = t;
  }
}

void build_fill(const Store& st, const int* place, hipStream_t s) {
  if (st.T > 0) k_ne_fill<<<grid_for(st.T), kBlock, 0, s>>>(st.tri, st.T, st.hdr, (const Place3*)place, st.ne);
}

__device__ void isort(int* a, int n) {
  for (int i = 1; i < n; ++i) {
    int x = a[i];
    int j = i - 1;
    while (j >= 0 && a[j] > x) {
      a[j + 1] = a[j];
      --j;
    }
    a[j + 1] = x;
  }
}

// sort NE(v); NN(v) = sorted "next" vertices of v's elements, plus the one
// "previous" vertex that is not a next (boundary vertices). A repeated next
// means a directed edge is used twice: inconsistent orientation or a
// non-manifold edge; more than one unmatched previous is a pinched vertex.
// Rows of up to 16 elements are finished in registers: sorting networks,
// and every previous looked up among all nexts (8-wide when a wavefront's
// rows all fit, 16-wide otherwise).
constexpr int kFinishReg = 16;
template <int N>
__device__ __forceinline__ void row_finish_reg(const Elem* __restrict__ tri, Hdr* __restrict__ hdr, int ncap,
                                               int* __restrict__ nn, int* __restrict__ ne, int v, Hdr h,
                                               int* ctr) {
  int c = h.w;
  int r[N];
  if constexpr (N == 8) {
    row8(ne, h.z, c, r);
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (k >= c) r[k] = INT_MAX;
  } else {
#pragma unroll
    for (int k = 0; k < N; ++k) r[k] = k < c ? ne[h.z + k] : INT_MAX;
  }
  bitonic<N>(r);
  // the elements' loads go out together (an empty slot loads the first
  // element again rather than branch around its load)
  int nx[N], pv[N];
  if constexpr (N == 8) {
    // the sorted row, four entries per store (the slot holds a multiple of four)
    *(int4*)(ne + h.z) = make_int4(r[0], r[1], r[2], r[3]);
    if (c > 4) *(int4*)(ne + h.z + 4) = make_int4(r[4], r[5], r[6], r[7]);
  }
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (N != 8 && k < c) ne[h.z + k] = r[k];
    Elem e = tri[k < c ? r[k] : r[0]];
    int s = slot_of(e, v);
    nx[k] = k < c ? at(e, s == 2 ? 0 : s + 1) : INT_MAX;
    pv[k] = k < c ? at(e, s == 0 ? 2 : s - 1) : INT_MAX;
  }
  bitonic<N>(nx);
  bool bad = false;
#pragma unroll
  for (int k = 1; k < N; ++k) bad |= nx[k] != INT_MAX && nx[k] == nx[k - 1];
  int extra = INT_MAX, nextra = 0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (pv[k] == INT_MAX) continue;
    bool found = false;
#pragma unroll
    for (int q = 0; q < N; ++q) found |= nx[q] == pv[k];
    if (!found) {
      extra = pv[k];
      ++nextra;
    }
  }
  int n = c + nextra;
  if (nextra > 1 || n > ncap) bad = true;
  if (bad) {
    atomicOr(&ctr[C_ERR], E_MESH_MANIFOLD);
    n = c;
    nextra = 0;
  }
  int w = 0;
  bool put = nextra == 0;
  int* out = nn + h.x;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    int x = nx[k];
    if (x == INT_MAX) continue;
    if (!put && extra < x) {
      out[w++] = extra;
      put = true;
    }
    out[w++] = x;
  }
  if (!put) out[w++] = extra;
  reinterpret_cast<int*>(&hdr[v])[1] = n;
}

// a longer row by one thread
__device__ void row_finish_serial(const Elem* __restrict__ tri, Hdr* __restrict__ hdr, int ncap, int* __restrict__ nn,
                                  int* __restrict__ ne, int v, Hdr h, int* ctr) {
  int c = h.w;
  int* row = ne + h.z;
  isort(row, c);
  int* out = nn + h.x;
  for (int i = 0; i < c; ++i) {
    Elem e = tri[row[i]];
    int k = slot_of(e, v);
    out[i] = at(e, k == 2 ? 0 : k + 1);
  }
  isort(out, c);
  bool bad = false;
  for (int i = 1; i < c; ++i)
    if (out[i] == out[i - 1]) bad = true;
  int n = c, extra = 0;
  for (int i = 0; i < c && !bad; ++i) {
    Elem e = tri[row[i]];
    int k = slot_of(e, v);
    int p = at(e, k == 0 ? 2 : k - 1);
    // binary search in the current sorted row out[0..n)
    int lo = 0, hi = n;
    while (lo < hi) {
      int mid = (lo + hi) >> 1;
      if (out[mid] < p) lo = mid + 1;
      else hi = mid;
    }
    if (lo < n && out[lo] == p) continue;
    if (++extra > 1 || n + 1 > ncap) {
      bad = true;
      break;
    }
    // insert p into out[0..n)
    int j = n - 1;
    while (j >= 0 && out[j] > p) {
      out[j + 1] = out[j];
      --j;
    }
    out[j + 1] = p;
    ++n;
  }
  if (bad) atomicOr(&ctr[C_ERR], E_MESH_MANIFOLD);
  reinterpret_cast<int*>(&hdr[v])[1] = n;
}
// a row of at most kWave elements by a wavefront, an element a lane: places are
// numbers of smaller ones
__device__ __forceinline__ void row_finish_wave(const Elem* __restrict__ tri, Hdr* __restrict__ hdr, int ncap,
                                                int* __restrict__ nn, int* __restrict__ ne, int v, Hdr h, int* ctr) {
  int lane = __lane_id(), c = h.w;
  bool has = lane < c;
  int t = has ? ne[h.z + lane] : INT_MAX;
  Elem e = tri[has ? t : 0];
  int s = slot_of(e, v);
  int nx = has ? at(e, s == 2 ? 0 : s + 1) : INT_MAX, pv = has ? at(e, s == 0 ? 2 : s - 1) : -1;
  int rid = 0, rnx = 0;
  bool found = false, twice = false;
  for (int k = 0; k < c; ++k) {
    int ot = __builtin_amdgcn_readlane(t, k), on = __builtin_amdgcn_readlane(nx, k);
    rid += ot < t ? 1 : 0;
    rnx += on < nx || (on == nx && k < lane) ? 1 : 0;
    found |= on == pv;
    twice |= on == nx && k != lane;
  }
  uint64_t lone = __ballot(has && !found);
  int nextra = __popcll(lone), n = c + nextra;
  int ex = nextra ? __shfl(pv, __ffsll((unsigned long long)lone) - 1) : INT_MAX;
  bool bad = __ballot(has && twice) != 0 || nextra > 1 || n > ncap;
  if (bad) {
    if (lane == 0) atomicOr(&ctr[C_ERR], E_MESH_MANIFOLD);
    n = c;
    ex = INT_MAX;
  }
  int exat = __popcll(__ballot(has && nx < ex));
  if (has) {
    ne[h.z + rid] = t;
    nn[h.x + rnx + (ex < nx ? 1 : 0)] = nx;
  }
  if (lane == 0) {
    if (n > c) nn[h.x + exat] = ex;
    reinterpret_cast<int*>(&hdr[v])[1] = n;
  }
}

// Rows past the registers' are gathered and take a wavefront each: one thread
// sorting such a row in memory held up the whole launch, 70 us on a batch of 64
// meshes with a few rows of 17 and more elements; the mean over its builds went from
// 52 to 28 us.
__global__ void __launch_bounds__(kBlock) k_row_finish(const Elem* __restrict__ tri, Hdr* __restrict__ hdr,
                                                     const int2* __restrict__ cap, int* __restrict__ nn,
                                                     int* __restrict__ ne, int V, int* ctr) {
  __shared__ int q[kBlock], qn;
  for (int v0 = (int)blockIdx.x * kBlock; v0 < V; v0 += gstride()) {
    int v = v0 + (int)threadIdx.x;
    Hdr h = v < V ? hdr[v] : make_int4(0, 0, 0, 0);
    int c = h.w;
    if (threadIdx.x == 0) qn = 0;
    bool any = __syncthreads_or(c > kFinishReg);
    if (c > kFinishReg) q[atomicAdd(&qn, 1)] = v;
    if (c > 0 && c <= kFinishReg) {
      if (__all(c <= 8)) row_finish_reg<8>(tri, hdr, cap[v].x, nn, ne, v, h, ctr);
      else row_finish_reg<kFinishReg>(tri, hdr, cap[v].x, nn, ne, v, h, ctr);
    }
    if (!any) continue;
    __syncthreads();
    for (int i = (int)threadIdx.x / kWave; i < qn; i += kBlock / kWave) {
      int w = __builtin_amdgcn_readfirstlane(q[i]);
      Hdr g = hdr[w];
      g.w = __builtin_amdgcn_readfirstlane(g.w);
      int nc = cap[w].x;
      if (g.w <= kWave) row_finish_wave(tri, hdr, nc, nn, ne, w, g, ctr);
      else if (__lane_id() == 0) row_finish_serial(tri, hdr, nc, nn, ne, w, g, ctr);
    }
    __syncthreads();
  }
}

void build_finish(const Store& st, int* ctr, hipStream_t s) {
  k_row_finish<<<grid_for(st.V), kBlock, 0, s>>>(st.tri, st.hdr, st.cap, st.nn, st.ne, st.V, ctr);
}

// ---- compaction --------------------------------------------------------------------------
// live flags of vertices and elements, their scans and totals
void scan_live(const Store& st, int* vflag, int* vpos, int* vtotal, int* tflag, int* tpos, int* ttotal, int* partial,
               hipStream_t s) {
  const uint8_t* valive = st.valive;
  const Elem* tri = st.tri;
  auto put = [] __device__(int* flag, int i, bool on, int x) {
    if (on) flag[i] = x;
    return x;
  };
  scan_fused2<int, 8>([=] __device__(int v, bool on) { return put(vflag, v, on, on && valive[v] ? 1 : 0); },
                      [=] __device__(int v) { return vflag[v]; },
                      [=] __device__(int v, int at, int) { vpos[v] = at; }, [=] __device__(int t) { *vtotal = t; },
                      st.V, [=] __device__(int t, bool on) { return put(tflag, t, on, on && tri[t].w ? 1 : 0); },
                      [=] __device__(int t) { return tflag[t]; },
                      [=] __device__(int t, int at, int) { tpos[t] = at; }, [=] __device__(int t) { *ttotal = t; },
                      st.T, partial, s);
}

__global__ void k_compact_v(const double2* __restrict__ xy, const Met* __restrict__ met,
                            const uint8_t* __restrict__ tag, const uint8_t* __restrict__ valive, int V,
                            const int* __restrict__ vmap, double2* __restrict__ xy2, Met* __restrict__ met2,
                            uint8_t* __restrict__ tag2, uint8_t* __restrict__ va2) {
  for (int v = gtid(); v < V; v += gstride()) {
    if (!valive[v]) continue;
    int n = vmap[v];
    xy2[n] = xy[v];
    met2[n] = met[v];
    tag2[n] = tag[v];
    va2[n] = 1;
  }
}
void compact_vertices(const Store& st, const int* vmap, double2* xy2, Met* met2, uint8_t* tag2, uint8_t* va2,
                      hipStream_t s) {
  k_compact_v<<<grid_for(st.V), kBlock, 0, s>>>(st.xy, st.met, st.tag, st.valive, st.V, vmap, xy2, met2, tag2, va2);
}

__global__ void k_range_sums(const int* __restrict__ scan, const int* __restrict__ src, const int* __restrict__ base,
                             const int* __restrict__ used, int B, int* __restrict__ out) {
  for (int i = gtid(); i < B; i += gstride()) {
    int lo = base[i], hi = base[i] + used[i];
    // inclusive value at hi - 1 minus exclusive value at lo
    out[i] = hi > lo ? scan[hi - 1] + src[hi - 1] - scan[lo] : 0;
  }
}
void range_sums(const int* scan, const int* src, const int* base, const int* used, int B, int* out, hipStream_t s) {
  k_range_sums<<<grid_for(B), kBlock, 0, s>>>(scan, src, base, used, B, out);
}

__global__ void k_mesh_maps(const int* __restrict__ flag, const int* __restrict__ scan, const int* __restrict__ mesh,
                            const int* __restrict__ base, const int* __restrict__ nbase, int n, int* __restrict__ map) {
  for (int x = gtid(); x < n; x += gstride()) {
    if (!flag[x]) continue;
    int i = mesh ? mesh[x] : 0;
    map[x] = nbase[i] + scan[x] - scan[base[i]];
  }
}
void mesh_maps(const int* flag, const int* scan, const int* mesh, const int* base, const int* nbase, int n, int* map,
               hipStream_t s) {
  k_mesh_maps<<<grid_for(n), kBlock, 0, s>>>(flag, scan, mesh, base, nbase, n, map);
}

__global__ void k_fill_mesh_ids(const int* __restrict__ base, int B, int n, int* __restrict__ mesh) {
  for (int x = gtid(); x < n; x += gstride()) {
    int lo = 0, hi = B;  // last i with base[i] <= x
    while (hi - lo > 1) {
      int mid = (lo + hi) >> 1;
      if (base[mid] <= x) lo = mid;
      else hi = mid;
    }
    mesh[x] = lo;
  }
}
void fill_mesh_ids(const int* base, int B, int n, int* mesh, hipStream_t s) {
  k_fill_mesh_ids<<<grid_for(n), kBlock, 0, s>>>(base, B, n, mesh);
}

__global__ void k_compact_t(const Elem* __restrict__ tri, int T, const int* __restrict__ vmap,
                            const int* __restrict__ tmap, Elem* __restrict__ tri2) {
  for (int t = gtid(); t < T; t += gstride()) {
    Elem e = tri[t];
    if (!e.w) continue;
    // the renumbering is monotone, so the smallest id stays first
    tri2[tmap[t]] = make_int4(vmap[e.x], vmap[e.y], vmap[e.z], 1);
  }
}
void compact_elements(const Store& st, const int* vmap, const int* tmap, Elem* tri2, hipStream_t s) {
  k_compact_t<<<grid_for(st.T), kBlock, 0, s>>>(st.tri, st.T, vmap, tmap, tri2);
}

// ---- refinement (Sec. 2.4.2) ------------------------------------------------------------
__device__ __forceinline__ double elen2(const double2* xy, const Met* met, int i, int j) {
  return len2(xy[i], met[i], xy[j], met[j]);
}

// count long edges (a, b > a) per vertex; also counts tested edges. Meshes of
// a batch that have finished refining are skipped.
// (called by full wavefronts)
__device__ __forceinline__ int refine_mark(const Store& st, double L_up2, int* cnt, int* ctr, int a, bool on) {
  int tested = 0, c = 0;
  if (on) {
    bool skip = st.mdone && st.mdone[st.vmesh ? st.vmesh[a] : 0];
    if (st.valive[a] && !skip) {
      Hdr h = st.hdr[a];
      for (int j = 0; j < h.y; ++j) {
        int b = st.nn[h.x + j];
        if (b <= a) continue;
        ++tested;
        if (elen2(st.xy, st.met, a, b) > L_up2) ++c;
      }
    }
    cnt[a] = c;
  }
  wave_add_full(stripe_ptr(ctr, S_EDGES), tested);
  return c;
}
__device__ __forceinline__ int refine_count(const Store& st, double L_up2, int* ecnt, int t, bool on) {
  if (!on) return 0;
  Elem e = st.tri[t];
  int c = 0;
  if (e.w) {
    c += elen2(st.xy, st.met, e.x, e.y) > L_up2;
    c += elen2(st.xy, st.met, e.y, e.z) > L_up2;
    c += elen2(st.xy, st.met, e.z, e.x) > L_up2;
  }
  ecnt[t] = c;
  return c;
}

// new vertex ids inside the vertex's mesh range: base + used + (long edges of
// the mesh before a, in (a, b) order) + rank in a's row
__global__ void k_refine_mint(Store st, double L_up2, const int* __restrict__ vscan, int* __restrict__ mid) {
  for (int a = gtid(); a < st.V; a += gstride()) {
    if (!st.valive[a]) continue;
    int i = st.vmesh ? st.vmesh[a] : 0;
    if (a >= st.vbase[i] + st.vused[i]) continue;  // minted in this pass
    Hdr h = st.hdr[a];
    int first = st.vbase[i] + st.vused[i] + vscan[a] - vscan[st.vbase[i]];
    int k = 0;
    for (int j = 0; j < h.y; ++j) {
      int b = st.nn[h.x + j];
      if (b <= a) continue;
      if (!(elen2(st.xy, st.met, a, b) > L_up2)) continue;
      int id = first + k++;
      mid[h.x + j] = id;
      double2 pa = st.xy[a], pb = st.xy[b];
      Met ma = st.met[a], mb = st.met[b];
      st.xy[id] = make_double2((pa.x + pb.x) * 0.5, (pa.y + pb.y) * 0.5);
      Met mm;
      mm.a = (ma.a + mb.a) * 0.5;
      mm.b = (ma.b + mb.b) * 0.5;
      mm.c = (ma.c + mb.c) * 0.5;
      st.met[id] = mm;
      st.tag[id] = st.tag[a] & st.tag[b];
      st.valive[id] = 1;
    }
  }
}
void refine_mint(const Store& st, double L_up2, const int* vscan, int* mid, hipStream_t s) {
  k_refine_mint<<<grid_for(st.V), kBlock, 0, s>>>(st, L_up2, vscan, mid);
}

// per vertex the edges to split that it owns (the smaller end), per element its
// edges to split: counts, scans and totals
void refine_scan(const Store& store, double L_up2, int* vcnt, int* vscan, int* vtotal, int* ecnt, int* escan,
                 int* etotal, int* ctr, int* partial, hipStream_t s) {
  Store st = store;
  scan_fused2<int, 1>([=] __device__(int a, bool on) { return refine_mark(st, L_up2, vcnt, ctr, a, on); },
                      [=] __device__(int a) { return vcnt[a]; },
                      [=] __device__(int a, int at, int) { vscan[a] = at; }, [=] __device__(int t) { *vtotal = t; },
                      st.V, [=] __device__(int t, bool on) { return refine_count(st, L_up2, ecnt, t, on); },
                      [=] __device__(int t) { return ecnt[t]; },
                      [=] __device__(int t, int at, int) { escan[t] = at; }, [=] __device__(int t) { *etotal = t; },
                      st.T, partial, s);
}

__device__ int midpoint_of(const Hdr* hdr, const int* nn, const int* mid, int p, int q) {
  int a = min(p, q), b = max(p, q);
  Hdr h = hdr[a];
  int lo = 0, hi = h.y;
  while (lo < hi) {
    int m = (lo + hi) >> 1;
    if (nn[h.x + m] < b) lo = m + 1;
    else hi = m;
  }
  return mid[h.x + lo];
}

__device__ __forceinline__ Elem mk(int a, int b, int c) {
  int3 r = rot_min(a, b, c);
  return make_int4(r.x, r.y, r.z, 1);
}

// children by template; the first keeps the parent id, the others take ids
// inside the element's mesh range: base + used + (new children of the mesh
// before t) + (child index - 1)
__global__ void k_refine_split(Store st, double L_up2, const int* __restrict__ mid, const int* __restrict__ escan) {
  const double2* xy = st.xy;
  const Met* met = st.met;
  Elem* tri = st.tri;
  const Hdr* hdr = st.hdr;
  const int* nn = st.nn;
  int T = st.T;
  for (int t = gtid(); t < T; t += gstride()) {
    Elem e = tri[t];
    if (!e.w) continue;
    int i = st.tmesh ? st.tmesh[t] : 0;
    if (t >= st.tbase[i] + st.tused[i]) continue;  // a child written in this pass
    int m0 = elen2(xy, met, e.x, e.y) > L_up2 ? midpoint_of(hdr, nn, mid, e.x, e.y) : -1;
    int m1 = elen2(xy, met, e.y, e.z) > L_up2 ? midpoint_of(hdr, nn, mid, e.y, e.z) : -1;
    int m2 = elen2(xy, met, e.z, e.x) > L_up2 ? midpoint_of(hdr, nn, mid, e.z, e.x) : -1;
    int ns = (m0 >= 0) + (m1 >= 0) + (m2 >= 0);
    if (ns == 0) continue;
    Elem ch[4];
    if (ns == 1) {
      // the split edge k runs P -> Q with mid-point M, R opposite
      int k = m0 >= 0 ? 0 : (m1 >= 0 ? 1 : 2);
      int P = at(e, k), Q = at(e, k == 2 ? 0 : k + 1), R = at(e, k == 0 ? 2 : k - 1);
      int M = k == 0 ? m0 : (k == 1 ? m1 : m2);
      ch[0] = mk(P, M, R);
      ch[1] = mk(M, Q, R);
    } else if (ns == 2) {
      // the unsplit edge k runs P -> Q; M1 on Q-R, M2 on R-P
      int k = m0 < 0 ? 0 : (m1 < 0 ? 1 : 2);
      int P = at(e, k), Q = at(e, k == 2 ? 0 : k + 1), R = at(e, k == 0 ? 2 : k - 1);
      int M1 = k == 0 ? m1 : (k == 1 ? m2 : m0);
      int M2 = k == 0 ? m2 : (k == 1 ? m0 : m1);
      ch[0] = mk(M1, R, M2);
      double dP = elen2(xy, met, P, M1), dQ = elen2(xy, met, Q, M2);
      if (dP <= dQ) {
        ch[1] = mk(P, Q, M1);
        ch[2] = mk(P, M1, M2);
      } else {
        ch[1] = mk(P, Q, M2);
        ch[2] = mk(Q, M1, M2);
      }
    } else {
      ch[0] = mk(e.x, m0, m2);
      ch[1] = mk(m0, e.y, m1);
      ch[2] = mk(m2, m1, e.z);
      ch[3] = mk(m0, m1, m2);
    }
    tri[t] = ch[0];
    int base = st.tbase[i] + st.tused[i] + escan[t] - escan[st.tbase[i]];
    tri[base] = ch[1];
    if (ns >= 2) tri[base + 1] = ch[2];
    if (ns == 3) tri[base + 2] = ch[3];
  }
}
void refine_split(const Store& st, double L_up2, const int* mid, const int* escan, hipStream_t s) {
  k_refine_split<<<grid_for(st.T), kBlock, 0, s>>>(st, L_up2, mid, escan);
}

// ---- small utilities ---------------------------------------------------------------------------
// (plain kernels rather than memset nodes, so the sequences stay graph-safe)
__global__ void k_zero(int* __restrict__ p, int n) {
  for (int i = gtid(); i < n; i += gstride()) p[i] = 0;
}
void zero_ints(int* p, int n, hipStream_t s) {
  if (n > 0) k_zero<<<grid_for(n, 1024), kBlock, 0, s>>>(p, n);
}
__global__ void k_fill_u8(uint8_t* __restrict__ p, int n, uint8_t v) {
  for (int i = gtid(); i < n; i += gstride()) p[i] = v;
}
void fill_u8(uint8_t* p, int n, uint8_t v, hipStream_t s) {
  if (n > 0) k_fill_u8<<<grid_for(n, 1024), kBlock, 0, s>>>(p, n, v);
}
__global__ void k_set_int(int* p, int v) { *p = v; }
void set_int(int* p, int v, hipStream_t s) { k_set_int<<<1, 1, 0, s>>>(p, v); }

__global__ void k_copy_vertices(Store a, Store b, int n) {
  for (int v = gtid(); v < n; v += gstride()) {
    bool old = v < a.V;
    if (old) {
      b.xy[v] = a.xy[v];
      b.met[v] = a.met[v];
      b.tag[v] = a.tag[v];
    }
    b.valive[v] = old ? a.valive[v] : 0;
    b.hdr[v] = old ? a.hdr[v] : make_int4(0, 0, 0, 0);
    b.cap[v] = old ? a.cap[v] : make_int2(0, 0);
  }
}
void copy_vertices(const Store& from, const Store& to, int n, hipStream_t s) {
  k_copy_vertices<<<grid_for(n), kBlock, 0, s>>>(from, to, n);
}
__global__ void k_copy_elements(const Elem* __restrict__ a, int T, Elem* __restrict__ b, int n) {
  for (int t = gtid(); t < n; t += gstride()) b[t] = t < T ? a[t] : make_int4(0, 0, 0, 0);
}
void copy_elements(const Store& from, Elem* to, int n, hipStream_t s) {
  k_copy_elements<<<grid_for(n), kBlock, 0, s>>>(from.tri, from.T, to, n);
}
__global__ void k_clear_tail(Store st, int V, int T) {
  for (int v = V + gtid(); v < st.Vcap; v += gstride()) st.valive[v] = 0;
  for (int t = T + gtid(); t < st.Tcap; t += gstride()) st.tri[t] = make_int4(0, 0, 0, 0);
}
void clear_tail(const Store& st, int V, int T, hipStream_t s) {
  k_clear_tail<<<grid_for(std::max(st.Vcap - V, st.Tcap - T)), kBlock, 0, s>>>(st, V, T);
}
__global__ void k_build_start(int* __restrict__ cnt, int* r, int vused, int tused, int V, int T) {
  for (int i = gtid(); cnt && i < V; i += gstride()) cnt[i] = 0;
  if (!r || gtid() != 0) return;
  r[0] = 0;
  r[1] = V;
  r[2] = vused;
  r[3] = 0;
  r[4] = T;
  r[5] = tused;
}
void build_start(int* cnt, int* ranges, int vused, int tused, int V, int T, hipStream_t s) {
  k_build_start<<<grid_for(V, 1024), kBlock, 0, s>>>(cnt, ranges, vused, tused, V, T);
}

// A batch's slots from the callers' arrays: mesh numbers, offset and rotated ids,
// tags from the coordinates where none are given; unused slots are dead, with the
// identity metric. The host built all this and sent it, headroom and all, in 9 ms
// for 64 meshes of 16 MB in all; copying the arrays and this launch take 1.3 ms.
__device__ __forceinline__ int mesh_of(const int* base, int B, int i) {
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (base[mid] <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
__global__ void k_batch_in(const char* __restrict__ raw, int B, Store st, int* ctr) {
  const BatchIn* in = (const BatchIn*)raw;
  for (int i = gtid(); i < max(st.V, st.T); i += gstride()) {
    if (i < st.V) {
      int b = mesh_of(st.vbase, B, i), v = i - st.vbase[b];
      double2 p = make_double2(0.0, 0.0);
      Met m{1.0, 0.0, 1.0};
      uint8_t tag = 0, live = 0;
      if (v < st.vused[b]) {
        p = ((const double2*)(raw + in[b].xy))[v];
        const double* q = (const double*)(raw + in[b].met) + 3 * (int64_t)v;
        m = Met{q[0], q[1], q[2]};
        live = 1;
        if (in[b].tag >= 0) tag = ((const uint8_t*)(raw + in[b].tag))[v];
        else tag = (p.x == 0.0 ? 1 : 0) | (p.x == 1.0 ? 2 : 0) | (p.y == 0.0 ? 4 : 0) | (p.y == 1.0 ? 8 : 0);
      }
      if (st.vmesh) st.vmesh[i] = b;
      st.xy[i] = p;
      st.met[i] = m;
      st.tag[i] = tag;
      st.valive[i] = live;
    }
    if (i < st.T) {
      int b = mesh_of(st.tbase, B, i), t = i - st.tbase[b];
      Elem e = make_int4(0, 0, 0, 0);
      if (t < st.tused[b]) {
        const int* q = (const int*)(raw + in[b].tri) + 3 * (int64_t)t;
        int x = q[0], y = q[1], z = q[2], n = st.vused[b], v0 = st.vbase[b];
        if (x < 0 || y < 0 || z < 0 || x >= n || y >= n || z >= n) {
          atomicMin(&ctr[C_FAILEP], b);
        } else {
          x += v0;
          y += v0;
          z += v0;
          if (x < y && x < z) e = make_int4(x, y, z, 1);
          else if (y < x && y < z) e = make_int4(y, z, x, 1);
          else e = make_int4(z, x, y, 1);
        }
      }
      if (st.tmesh) st.tmesh[i] = b;
      st.tri[i] = e;
    }
  }
}
void batch_in(const char* raw, int B, const Store& st, int* ctr, hipStream_t s) {
  k_batch_in<<<grid_for(std::max(st.V, st.T)), kBlock, 0, s>>>(raw, B, st, ctr);
}

// a mesh's slots to host memory, with local ids
__global__ void k_batch_out(Store st, int v0, int nv, int t0, int nt, BatchOut o, char* dst) {
  for (int i = gtid(); i < max(nv, nt); i += gstride()) {
    if (i < nv) {
      if (o.xy >= 0) ((double2*)(dst + o.xy))[i] = st.xy[v0 + i];
      if (o.met >= 0) ((Met*)(dst + o.met))[i] = st.met[v0 + i];
      if (o.tag >= 0) ((uint8_t*)(dst + o.tag))[i] = st.tag[v0 + i];
      if (o.valive >= 0) ((uint8_t*)(dst + o.valive))[i] = st.valive[v0 + i];
    }
    if (i < nt) {
      Elem e = st.tri[t0 + i];
      if (o.tri >= 0) {
        int d = e.w ? v0 : 0;
        int* q = (int*)(dst + o.tri) + 3 * (int64_t)i;
        q[0] = e.x - d;
        q[1] = e.y - d;
        q[2] = e.z - d;
      }
      if (o.talive >= 0) ((uint8_t*)(dst + o.talive))[i] = e.w ? 1 : 0;
    }
  }
}
void batch_out(const Store& st, int v0, int nv, int t0, int nt, const BatchOut& o, char* dst, hipStream_t s) {
  k_batch_out<<<grid_for(std::max(nv, nt)), kBlock, 0, s>>>(st, v0, nv, t0, nt, o, dst);
}

// input triangles (T x 3) to stored elements: rotated smallest-id first, live
__global__ void k_tri_in(const int* __restrict__ tri3, int T, Elem* __restrict__ tri) {
  for (int t = gtid(); t < T; t += gstride()) {
    int a = tri3[3 * t], b = tri3[3 * t + 1], c = tri3[3 * t + 2];
    int3 r = rot_min(a, b, c);
    tri[t] = make_int4(r.x, r.y, r.z, 1);
  }
}
void tri_in(const int* tri3, int T, Elem* tri, hipStream_t s) {
  k_tri_in<<<grid_for(T), kBlock, 0, s>>>(tri3, T, tri);
}
__global__ void k_xy_in(const double* __restrict__ xy, int V, double2* __restrict__ out) {
  for (int v = gtid(); v < V; v += gstride()) out[v] = make_double2(xy[2 * v], xy[2 * v + 1]);
}
void xy_in(const double* xy, int V, double2* out, hipStream_t s) {
  k_xy_in<<<grid_for(V), kBlock, 0, s>>>(xy, V, out);
}
// unit-square side tags from exact coordinates
__global__ void k_tags(const double2* __restrict__ xy, int V, uint8_t* __restrict__ tag) {
  for (int v = gtid(); v < V; v += gstride()) {
    double2 p = xy[v];
    uint8_t t = 0;
    if (p.x == 0.0) t |= 1;
    if (p.x == 1.0) t |= 2;
    if (p.y == 0.0) t |= 4;
    if (p.y == 1.0) t |= 8;
    tag[v] = t;
  }
}
void tags_from_xy(const double2* xy, int V, uint8_t* tag, hipStream_t s) {
  k_tags<<<grid_for(V), kBlock, 0, s>>>(xy, V, tag);
}

// ---- export --------------------------------------------------------------------------------
__global__ void k_export_tri(const Elem* __restrict__ tri, int T, int* __restrict__ tri3, uint8_t* talive) {
  for (int t = gtid(); t < T; t += gstride()) {
    Elem e = tri[t];
    if (tri3) {
      tri3[3 * t] = e.x;
      tri3[3 * t + 1] = e.y;
      tri3[3 * t + 2] = e.z;
    }
    if (talive) talive[t] = e.w ? 1 : 0;
  }
}
void export_tri(const Store& st, int* tri3, uint8_t* talive, hipStream_t s) {
  k_export_tri<<<grid_for(st.T), kBlock, 0, s>>>(st.tri, st.T, tri3, talive);
}

}  // namespace pm
