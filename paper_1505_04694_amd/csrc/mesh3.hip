// Tetrahedral meshes of the unit cube (Sec. 4's extrusion of the method to
// three dimensions): coarsening, refinement and Laplacian smoothing in the
// metric over Jones-Plassmann colour classes, as independent sets; no swaps.
//
// Layout: per vertex xyz (double4, w unused), the six metric entries, tag and
// live bytes, a row header int4 (nn_off, nn_cnt, ne_off, ne_cnt); per element
// an int4 of vertex ids and a live byte. After every class that changes the
// topology the rows it touched are rebuilt from their old entries and those of
// the members collapsed onto them; creation, refinement and renumbering build all
// rows (count, scan, fill, finish per vertex). A class's members are pairwise
// non-adjacent, so the class kernel writes only its members' own elements, and
// the next class reads the current graph. Every floating-point expression is
// written in one fixed order and compiled without contraction, so decisions are
// the ones a serial IEEE-754 program makes from the same inputs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/pm3.h"
#include "common.hpp"
#include "kern.hpp"
#include "blocks.hpp"
#include "scan.hpp"

namespace pm3 {

using pm::gstride;
using pm::gtid;
using pm::make_ctx;
using pm::stream_seed;
using pm::vkey;
using pm::kWave;

constexpr int kB = 256;
constexpr int kMaxColours = 256;
enum { PH3_COARSEN = 1, PH3_SMOOTH = 3 };

// device counters
enum {
  K_ERR = 0,        // error bits
  K_COLOURED = 1,   // vertices coloured in a JP iteration
  K_NCOL = 2,       // colours used (max + 1)
  K_EVAL = 3,       // members evaluated
  K_DEFER = 4,      // members deferred by re-validation
  K_COMMIT = 5,     // collapses / accepted moves
  K_EDGES = 6,      // edges tested by refinement
  K_TOTAL = 7,      // scan total
  K_ROOM = 8,       // a row commit ran out of room (pool stripe full, or a row past the wavefront form)
  K_ROOMEP = 9,     // the epoch of the class whose commit ran out of room
  K_WAIT = 10,      // vertices left to the one-block end of a colouring
  // by the parity of a class's epoch (its commit clears the other's):
  K_CCOMMIT = 11,   // 11, 12: 1: the class collapsed something (gates its row commit)
  K_NROWS = 13,     // 13, 14: rows stamped by the class (the length of its row list)
  K_LIST = 15,      // length of the list selected last
  K_TOTAL2 = 16,    // the second total of two scans at once
  K_COUNT = 32,
  K_CLASS = K_COUNT,                    // class sizes, cursors and offsets, kMaxColours each
  K_STRIPE = K_CLASS + 3 * kMaxColours, // kStripes lines of striped counts
  K_ALL = K_STRIPE + 64 * 32
};
// Counts that every wavefront adds to are striped over 64 lines and summed by
// the read-back: adds to one line take about 10 ns each, one after another (the
// four counts of the largest collapse launches, 58,000 wavefronts, took most of
// their 1.5 ms).
constexpr int kStripes = 64, kStripeW = 32;
enum { S_COLOURED, S_EVAL, S_DEFER, S_COMMIT, S_EDGES, S_SLOTS };
__device__ __forceinline__ int counter_of(int slot) {
  return slot == S_COLOURED ? K_COLOURED : slot == S_EVAL ? K_EVAL : slot == S_DEFER ? K_DEFER : slot == S_COMMIT ? K_COMMIT : K_EDGES;
}
enum { E_MESH = 1, E_METRIC = 2, E_COLOURS = 4, E_LEAVES = 8 };

struct Met6 {
  double a00, a01, a02, a11, a12, a22;
};

struct Store3 {
  int V = 0, T = 0;
  double4* xyz = nullptr;
  Met6* met = nullptr;
  uint8_t* tag = nullptr;
  uint8_t* valive = nullptr;
  int4* tet = nullptr;
  uint8_t* talive = nullptr;
  int4* hdr = nullptr;  // (nn_off, nn_cnt, ne_off, ne_cnt); NN's slot is 3 x NE's
  int* cap = nullptr;   // NE slot capacity of each row (NN's: 3 x)
  int* nn = nullptr;
  int* ne = nullptr;
};

// ---- canonical geometry --------------------------------------------------------------

__device__ __forceinline__ Met6 edge_met(const Met6& p, const Met6& q) {
  return Met6{(p.a00 + q.a00) * 0.5, (p.a01 + q.a01) * 0.5, (p.a02 + q.a02) * 0.5,
              (p.a11 + q.a11) * 0.5, (p.a12 + q.a12) * 0.5, (p.a22 + q.a22) * 0.5};
}

// e^T M e, bitwise the same for -e
__device__ __forceinline__ double qform(const Met6& e, double dx, double dy, double dz) {
  return (((e.a00 * dx) * dx + ((2.0 * e.a01) * dx) * dy) + ((2.0 * e.a02) * dx) * dz) +
         (((e.a11 * dy) * dy + ((2.0 * e.a12) * dy) * dz) + (e.a22 * dz) * dz);
}

__device__ __forceinline__ double len2(const Store3& st, int i, int j) {
  double4 pi = st.xyz[i], pj = st.xyz[j];
  return qform(edge_met(st.met[i], st.met[j]), pj.x - pi.x, pj.y - pi.y, pj.z - pi.z);
}

__device__ __forceinline__ double det3(const Met6& g) {
  return (g.a00 * (g.a11 * g.a22 - g.a12 * g.a12) - g.a01 * (g.a01 * g.a22 - g.a12 * g.a02)) +
         g.a02 * (g.a01 * g.a12 - g.a11 * g.a02);
}

struct Geo3 {
  double4 p[4];
  Met6 m;
};

__device__ __forceinline__ int at4(const int4& t, int k) { return k == 0 ? t.x : (k == 1 ? t.y : (k == 2 ? t.z : t.w)); }
__device__ __forceinline__ bool has4(const int4& t, int v) { return t.x == v || t.y == v || t.z == v || t.w == v; }
__device__ __forceinline__ int4 replace4(int4 t, int v, int u) {
  if (t.x == v) t.x = u;
  else if (t.y == v) t.y = u;
  else if (t.z == v) t.z = u;
  else if (t.w == v) t.w = u;
  return t;
}

// orientation-preserving canonical order: the smallest id first (one of the
// four even permutations that bring a vertex to the front), then the other
// three rotated so that the smallest of them comes second
__device__ __forceinline__ int4 canon4(int4 t) {
  int k = 0, mn = t.x;
  if (t.y < mn) { k = 1; mn = t.y; }
  if (t.z < mn) { k = 2; mn = t.z; }
  if (t.w < mn) { k = 3; }
  int4 r;
  if (k == 0) r = t;
  else if (k == 1) r = make_int4(t.y, t.x, t.w, t.z);
  else if (k == 2) r = make_int4(t.z, t.w, t.x, t.y);
  else r = make_int4(t.w, t.z, t.y, t.x);
  int j = 1;
  int mj = r.y;
  if (r.z < mj) { j = 2; mj = r.z; }
  if (r.w < mj) { j = 3; }
  if (j == 2) r = make_int4(r.x, r.z, r.w, r.y);
  else if (j == 3) r = make_int4(r.x, r.w, r.y, r.z);
  return r;
}

// element t's geometry
__device__ __forceinline__ Geo3 geo(const Store3& st, int4 t) {
  Geo3 g;
  g.p[0] = st.xyz[t.x];
  g.p[1] = st.xyz[t.y];
  g.p[2] = st.xyz[t.z];
  g.p[3] = st.xyz[t.w];
  Met6 a = st.met[t.x], b = st.met[t.y], c = st.met[t.z], d = st.met[t.w];
  g.m = Met6{(((a.a00 + b.a00) + c.a00) + d.a00) / 4.0, (((a.a01 + b.a01) + c.a01) + d.a01) / 4.0,
             (((a.a02 + b.a02) + c.a02) + d.a02) / 4.0, (((a.a11 + b.a11) + c.a11) + d.a11) / 4.0,
             (((a.a12 + b.a12) + c.a12) + d.a12) / 4.0, (((a.a22 + b.a22) + c.a22) + d.a22) / 4.0};
  return g;
}

__device__ __forceinline__ double vol6(const Geo3& g) {
  double ax = g.p[1].x - g.p[0].x, ay = g.p[1].y - g.p[0].y, az = g.p[1].z - g.p[0].z;
  double bx = g.p[2].x - g.p[0].x, by = g.p[2].y - g.p[0].y, bz = g.p[2].z - g.p[0].z;
  double cx = g.p[3].x - g.p[0].x, cy = g.p[3].y - g.p[0].y, cz = g.p[3].z - g.p[0].z;
  return (ax * (by * cz - bz * cy) - ay * (bx * cz - bz * cx)) + az * (bx * cy - by * cx);
}

// sum of the six squared metric edge lengths, edges (01, 02, 03, 12, 13, 23)
__device__ __forceinline__ double edge_sum(const Geo3& g) {
  const int E0[6] = {0, 0, 0, 1, 1, 2}, E1[6] = {1, 2, 3, 2, 3, 3};
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double4 a = g.p[E0[k]], b = g.p[E1[k]];
    s = s + qform(g.m, b.x - a.x, b.y - a.y, b.z - a.z);
  }
  return s;
}

// q^3 = 432 det(M) D^2 / S^3 (decisions)
__device__ __forceinline__ double qual3(const Geo3& g) {
  double D = vol6(g), S = edge_sum(g), det = det3(g.m);
  return (((432.0 * det) * D) * D) / ((S * S) * S);
}

// q = 12 (3 |K|_M)^(2/3) / S (reported)
__device__ __forceinline__ double qual(const Geo3& g) {
  double D = vol6(g), S = edge_sum(g), det = det3(g.m);
  return (12.0 * cbrt(((det * D) * D) * 0.25)) / S;
}

__device__ __forceinline__ bool tag_ok(const Store3& st, int v, int u) { return (st.tag[v] & ~st.tag[u]) == 0; }

// the sum of x over the wavefront (every lane calls it) to a striped count
__device__ __forceinline__ void count_add(int* ctr, int slot, int x) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
  int w = (int)((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) & (kStripes - 1));
  if (__lane_id() == 0 && x) atomicAdd(&ctr[K_STRIPE + w * kStripeW + slot], x);
}
// counters zero, and no stripe holds anything
__global__ void k_zero_ctr(int* ctr) {
  if (threadIdx.x < K_COUNT) ctr[threadIdx.x] = 0;
  if (threadIdx.x < kStripes)
    for (int k = 0; k < S_SLOTS; ++k) ctr[K_STRIPE + threadIdx.x * kStripeW + k] = 0;
}
// a colouring's counts zero
__device__ __forceinline__ void zero_colouring(int* ctr) {
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0) ctr[K_ERR] = ctr[K_NCOL] = ctr[K_WAIT] = 0;
  if (threadIdx.x < kStripes) ctr[K_STRIPE + threadIdx.x * kStripeW + S_COLOURED] = 0;
}
// the counters (and `more` class sizes behind them) to the host, striped counts
// summed (256 threads); the next selection counts its list from zero
__global__ void k_mail3(int* ctr, int more, int* dst, int* at, int no) {
  int tid = (int)threadIdx.x;
  for (int i = tid; i < K_COUNT + more; i += (int)blockDim.x) {
    bool striped = i == K_COLOURED || i == K_EVAL || i == K_DEFER || i == K_COMMIT || i == K_EDGES;
    if (!striped) dst[i] = ctr[i];
    if (i == K_LIST) ctr[i] = 0;
  }
  for (int k = tid / kWave; k < S_SLOTS; k += (int)blockDim.x / kWave) {
    int x = ctr[K_STRIPE + (tid & (kWave - 1)) * kStripeW + k];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d);
    if ((tid & (kWave - 1)) == 0) dst[counter_of(k)] = x;
  }
  pm::mail_post(at, no);
}

// ---- input, validation ------------------------------------------------------------------

__global__ void k_in(const double* __restrict__ xyz, const int* __restrict__ tet, const double* __restrict__ met,
                     Store3 st, int* ctr) {
  for (int v = gtid(); v < st.V; v += gstride()) {
    st.xyz[v] = make_double4(xyz[3 * v], xyz[3 * v + 1], xyz[3 * v + 2], 0.0);
    const double* p = met + 6 * v;
    Met6 g{p[0], p[1], p[2], p[3], p[4], p[5]};
    st.met[v] = g;
    st.valive[v] = 1;
    if (!(g.a00 > 0.0) || !(g.a00 * g.a11 - g.a01 * g.a01 > 0.0) || !(det3(g) > 0.0)) atomicOr(&ctr[K_ERR], E_METRIC);
  }
  for (int t = gtid(); t < st.T; t += gstride()) {
    int4 e = make_int4(tet[4 * t], tet[4 * t + 1], tet[4 * t + 2], tet[4 * t + 3]);
    bool bad = e.x < 0 || e.y < 0 || e.z < 0 || e.w < 0 || e.x >= st.V || e.y >= st.V || e.z >= st.V ||
               e.w >= st.V || e.x == e.y || e.x == e.z || e.x == e.w || e.y == e.z || e.y == e.w || e.z == e.w;
    if (bad) {
      atomicOr(&ctr[K_ERR], E_MESH);
      e = make_int4(0, 1, 2, 3);
    }
    st.tet[t] = canon4(e);
    st.talive[t] = 1;
  }
}

__global__ void k_tags(Store3 st) {
  for (int v = gtid(); v < st.V; v += gstride()) {
    double4 p = st.xyz[v];
    uint8_t t = 0;
    if (p.x == 0.0) t |= 1;
    if (p.x == 1.0) t |= 2;
    if (p.y == 0.0) t |= 4;
    if (p.y == 1.0) t |= 8;
    if (p.z == 0.0) t |= 16;
    if (p.z == 1.0) t |= 32;
    st.tag[v] = t;
  }
}

__global__ void k_orient(Store3 st, int* ctr) {
  for (int t = gtid(); t < st.T; t += gstride()) {
    int4 e = st.tet[t];
    if (!(vol6(geo(st, e)) > 0.0)) atomicOr(&ctr[K_ERR], E_MESH);
  }
}

// ---- rows from the element list ----------------------------------------------------------

// how many elements a vertex has, and every element's places in its vertices' rows
// (in any order: the rows are sorted afterwards), for the filling. A work-group
// counts its elements' vertices in a hash table in LDS and reserves their places
// with one add per vertex: the rate of global atomics bounds this. With one per
// incidence, on average over the builds of the 29^3 planar-front adaptation (up to
// 3.4 million elements), it took 197 us and takes 58; the filling took 206 us
// with adds of its own and takes 31.
constexpr int kCountPer = 2, kCountSlots = 4096;
__global__ void __launch_bounds__(256) k_ne_count(Store3 st, int* cnt, int4* __restrict__ rank) {
  __shared__ __align__(16) int key[kCountSlots], num[kCountSlots];
  int tid = (int)threadIdx.x, t0 = (int)blockIdx.x * kB * kCountPer + tid;
  for (int i = tid; i < kCountSlots / 4; i += kB) {
    ((int4*)key)[i] = make_int4(-1, -1, -1, -1);
    ((int4*)num)[i] = make_int4(0, 0, 0, 0);
  }
  int4 e[kCountPer];
  bool on[kCountPer];
#pragma unroll
  for (int r = 0; r < kCountPer; ++r) {
    int t = max(0, min(t0 + r * kB, st.T - 1));
    on[r] = t0 + r * kB < st.T && st.talive[t];
    e[r] = st.tet[t];
  }
  __syncthreads();
  // (at most 4 kB kCountPer = half the table)
  int at[kCountPer][4], k[kCountPer][4];
#pragma unroll
  for (int r = 0; r < kCountPer; ++r) {
    if (!on[r]) continue;
    int v[4] = {e[r].x, e[r].y, e[r].z, e[r].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int a = (int)(((uint32_t)v[q] * 2654435761u) >> 20);
      for (;;) {
        int old = atomicCAS(&key[a], -1, v[q]);
        if (old == -1 || old == v[q]) break;
        a = (a + 1) & (kCountSlots - 1);
      }
      at[r][q] = a;
      k[r][q] = atomicAdd(&num[a], 1);
    }
  }
  __syncthreads();
  constexpr int R = kCountSlots / kB;
  int base[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    int c = num[q * kB + tid];
    base[q] = c ? atomicAdd(&cnt[key[q * kB + tid]], c) : 0;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) num[q * kB + tid] = base[q];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kCountPer; ++r)
    if (on[r])
      rank[t0 + r * kB] =
          make_int4(num[at[r][0]] + k[r][0], num[at[r][1]] + k[r][1], num[at[r][2]] + k[r][2], num[at[r][3]] + k[r][3]);
}
__global__ void __launch_bounds__(256) k_ne_fill(Store3 st, const int* __restrict__ off, const int4* __restrict__ rank) {
  for (int t = gtid(); t < st.T; t += gstride()) {
    if (!st.talive[t]) continue;
    int4 e = st.tet[t], k = rank[t];
    st.ne[off[e.x] + k.x] = t;
    st.ne[off[e.y] + k.y] = t;
    st.ne[off[e.z] + k.z] = t;
    st.ne[off[e.w] + k.w] = t;
  }
}

__device__ void isort(int* a, int n) {
  for (int i = 1; i < n; ++i) {
    int x = a[i], j = i - 1;
    while (j >= 0 && a[j] > x) {
      a[j + 1] = a[j];
      --j;
    }
    a[j + 1] = x;
  }
}

// Serial form for rows longer than a wavefront: sort NE(v) in place; NN(v) =
// the sorted distinct other vertices of NE(v)'s elements, inserted one at a
// time into a slot of three entries per NE entry (a binary search finds and
// skips repeats).
__device__ void rows_finish_serial(const Store3& st, int v, int o, int n) {
  int* row = st.ne + o;
  isort(row, n);
  int* nb = st.nn + 3 * o;
  int u = 0;
  for (int i = 0; i < n; ++i) {
    int4 e = st.tet[row[i]];
    int id[4] = {e.x, e.y, e.z, e.w};
    for (int j = 0; j < 4; ++j) {
      int x = id[j];
      if (x == v) continue;
      int lo = 0, hi = u;
      while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (nb[mid] < x) lo = mid + 1;
        else hi = mid;
      }
      if (lo < u && nb[lo] == x) continue;
      for (int q = u; q > lo; --q) nb[q] = nb[q - 1];
      nb[lo] = x;
      ++u;
    }
  }
  st.hdr[v] = make_int4(3 * o, u, o, n);
  st.cap[v] = n;
}

// ---- row commit after a collapse class ---------------------------------------------------------
// The collapse kernel stamps every row its members change with the class
// epoch (own) and records each committed member's target (rec). One
// wavefront per stamped row x rebuilds it: the candidates are NE(x) and the
// NE rows of the members collapsed onto x (neighbours of x whose record
// names x); NE(x) = the sorted distinct candidates that are live and hold x,
// NN(x) = the sorted distinct other vertices of those elements. The row is
// written in place when it fits its slot, else in fresh space from one of
// kTopStripes bump pointers (a stripe per row id modulo the count, each with
// its own range of the pool). A row of more than kRowMax elements and a full
// stripe set the room counter instead; the later classes of the round then
// stand down and the host rebuilds every row before it runs them again.
constexpr int kTopStripes = 64;
constexpr int kTopStride = 16;  // ints between two stripes' bump pointers

__device__ __forceinline__ void room3(int* ctr, int epoch) {
  ctr[K_ROOMEP] = epoch;
  atomicOr(&ctr[K_ROOM], 1);
}

// The two rows of a vertex are made by one wavefront. With at most kWave
// elements and neighbours (24 and 14 on average) lane l < m holds the l-th
// element id and its other three vertices. A lane's place in NE is the number of
// smaller ids, one lane read and compare per element, or its lane where the ids
// come sorted; the other vertices go through a hash table in LDS, which leaves
// each once, and are placed the same way. Longer rows, to kRowMax elements, do
// the same with everything in LDS. What bounds the kernels now is a row's chain of
// loads and the memory behind it: two rows side by side on the halves of a
// wavefront took as long (103 against 101 us a class). Before, it was the rate of
// vector instructions: sorting networks over the 64 lanes with four and eight slots each took
// some 700 exchanges a row, whatever its length, and kept for the long rows alone
// they still cost the others their registers and some 200 spilled scalars. Over
// the 53 large classes of the 29^3 planar-front coarsening a commit took 135 us
// on average with them and takes 101 us without; a build of all rows 341 and 230.
constexpr int kRowMax = 4 * kWave;
struct StarLds {
  int hash[256];
  int list[kWave];
  int4 kept[kWave];
};
union RowLds {
  StarLds s;
  struct {
    int hash[1024];
    int list[3 * kRowMax];
    int id[kRowMax];
  } w;
};
__device__ __forceinline__ void star_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// whether x was not in the table yet; at most 3/4 of it come in, so a slot is free
template <int BITS>
__device__ __forceinline__ bool hash_in(int* hash, int x) {
  uint32_t at = ((uint32_t)x * 2654435761u) >> (32 - BITS);
  for (;;) {
    int old = atomicCAS(&hash[at], -1, x);
    if (old == -1) return true;
    if (old == x) return false;
    at = (at + 1) & ((1u << BITS) - 1u);
  }
}
// False (nothing decided) when an id comes twice or there are more neighbours.
__device__ __forceinline__ bool star_rows(int m, int id, const int (&oth)[3], bool sorted, StarLds& L, int& rid, int& u,
                                          int& val, int& rnn) {
  int lane = __lane_id();
  bool has = lane < m;
  m = __builtin_amdgcn_readfirstlane(m);
  rid = lane;
  bool twice = false;
  if (!sorted) {
    rid = 0;
    int same = 0;
    for (int k = 0; k < m; k += 4) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // lanes from m on hold INT_MAX
        int o = __builtin_amdgcn_readlane(id, k + q);
        rid += o < id ? 1 : 0;
        same += o == id ? 1 : 0;
      }
    }
    twice = same > 1;
  }
  *(int4*)(L.hash + 4 * lane) = make_int4(-1, -1, -1, -1);
  star_sync();
  u = 0;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    bool fresh = has && hash_in<8>(L.hash, oth[q]);
    uint64_t b = __ballot(fresh);
    int pos = u + __popcll(b & ((1ull << lane) - 1ull));
    if (fresh && pos < kWave) L.list[pos] = oth[q];
    u += __popcll(b);
  }
  if (__ballot(has && twice) || u > kWave) return false;
  star_sync();
  u = __builtin_amdgcn_readfirstlane(u);
  val = lane < u ? L.list[lane] : INT_MAX;
  rnn = 0;
  for (int k = 0; k < u; k += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) rnn += __builtin_amdgcn_readlane(val, k + q) < val ? 1 : 0;
  }
  star_sync();
  return true;
}
__device__ __forceinline__ void others_of(const int4& e, int x, int (&o)[3]) {
  o[0] = e.x == x ? e.y : e.x;
  o[1] = e.x == x || e.y == x ? e.z : e.y;
  o[2] = e.w == x ? e.z : e.w;
}

// Row x's slot for m entries: its own (o, room for cap), else fresh space from
// one of the stripes. False when that is full.
__device__ __forceinline__ bool row_slot(int x, int m, int& o, int& cap, int* tops, int64_t base, int64_t per) {
  if (m <= cap) return true;
  int need = 2 * m;
  int sidx = x % kTopStripes;
  int got = 0;
  if (__lane_id() == 0) got = atomicAdd(&tops[sidx * kTopStride], need);
  got = __builtin_amdgcn_readfirstlane(got);
  if ((int64_t)got + need > base + (int64_t)(sidx + 1) * per) return false;
  o = got;
  cap = need;
  return true;
}

// Row x from the m <= kRowMax element ids in L.w.id, in any order, repeats
// dropped. False, with nothing written, when its stripe is full.
__device__ __forceinline__ bool wide_put(const Store3& st, int x, int m, int o, int cap, int* tops, int64_t base,
                                         int64_t per, RowLds& L) {
  constexpr int K = kRowMax / kWave;
  int lane = __lane_id();
  m = __builtin_amdgcn_readfirstlane(m);
  star_sync();
  int a[K], at[K];
#pragma unroll
  for (int r = 0; r < K; ++r) {
    a[r] = r * kWave + lane < m ? L.w.id[r * kWave + lane] : INT_MAX;
    at[r] = 0;
  }
  for (int k = 0; k < m; ++k) {
    int q = L.w.id[k];
#pragma unroll
    for (int r = 0; r < K; ++r) at[r] |= q == a[r] && k < r * kWave + lane ? 1 : 0;
  }
  star_sync();
  int kept = 0;
#pragma unroll
  for (int r = 0; r < K; ++r) {
    if (a[r] != INT_MAX && at[r]) {
      a[r] = INT_MAX;
      L.w.id[r * kWave + lane] = INT_MAX;
    }
    at[r] = 0;
    kept += __popcll(__ballot(a[r] != INT_MAX));
  }
  star_sync();
  for (int k = 0; k < m; ++k) {
    int q = L.w.id[k];
#pragma unroll
    for (int r = 0; r < K; ++r) at[r] += q < a[r] ? 1 : 0;
  }
  m = kept;
  if (!row_slot(x, m, o, cap, tops, base, per)) return false;
  for (int i = lane; i < 1024; i += kWave) L.w.hash[i] = -1;
  star_sync();
  int u = 0;
#pragma unroll
  for (int r = 0; r < K; ++r) {
    bool has = a[r] != INT_MAX;
    if (has) st.ne[o + at[r]] = a[r];
    int oth[3];
    others_of(st.tet[has ? a[r] : 0], x, oth);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      bool fresh = has && hash_in<10>(L.w.hash, oth[q]);
      uint64_t b = __ballot(fresh);
      if (fresh) L.w.list[u + __popcll(b & ((1ull << lane) - 1ull))] = oth[q];
      u += __popcll(b);
    }
  }
  star_sync();
  u = __builtin_amdgcn_readfirstlane(u);
  for (int c = lane; c < u; c += kWave) {
    int val = L.w.list[c], rnn = 0;
    for (int k = 0; k < u; ++k) rnn += L.w.list[k] < val ? 1 : 0;
    st.nn[3 * (int64_t)o + rnn] = val;
  }
  if (lane == 0) {
    st.hdr[x] = make_int4(3 * o, u, o, m);
    st.cap[x] = cap;
  }
  star_sync();
  return true;
}

// one stamped row (every lane of the wavefront); false: left to a full rebuild
__device__ __forceinline__ bool commit_row3(const Store3& st, int x, int epoch, const int2* __restrict__ rec, int* tops,
                                            int64_t base, int64_t per, RowLds& L) {
  int lane = __lane_id();
  uint64_t below = (1ull << lane) - 1ull;
  int4 h = st.hdr[x];
  int cap = __builtin_amdgcn_readfirstlane(st.cap[x]);
  int nnb = __builtin_amdgcn_readfirstlane(h.x), nn = __builtin_amdgcn_readfirstlane(h.y);
  int neb = __builtin_amdgcn_readfirstlane(h.z), ne = __builtin_amdgcn_readfirstlane(h.w);
  if (nn <= kWave && ne <= kWave) {
    int w = lane < nn ? st.nn[nnb + lane] : -1, t = lane < ne ? st.ne[neb + lane] : -1;
    int2 rc = rec[max(w, 0)];
    int4 e = st.tet[max(t, 0)];
    bool al = st.talive[max(t, 0)] != 0;
    // members collapsed onto x: neighbours whose record names x
    uint64_t ab = __ballot(w >= 0 && rc.x == epoch && rc.y == x);
    bool sorted = ab == 0, fits = true;
    int m = 0;
    auto keep = [&]() {
      bool k = t >= 0 && al && has4(e, x);
      uint64_t b = __ballot(k);
      int pos = m + __popcll(b & below);
      if (k && pos < kWave) {
        int q[3];
        others_of(e, x, q);
        L.s.kept[pos] = make_int4(t, q[0], q[1], q[2]);
      }
      m += __popcll(b);
    };
    keep();
    for (; ab; ab &= ab - 1) {
      int4 hz = st.hdr[__builtin_amdgcn_readlane(w, __ffsll((unsigned long long)ab) - 1)];
      if (hz.w > kWave) {
        fits = false;
        break;
      }
      t = lane < hz.w ? st.ne[hz.z + lane] : -1;
      e = st.tet[max(t, 0)];
      al = st.talive[max(t, 0)] != 0;
      keep();
    }
    if (fits && m <= kWave) {
      star_sync();
      int4 mine = lane < m ? L.s.kept[lane] : make_int4(INT_MAX, -1, -1, -1);
      int oth[3] = {mine.y, mine.z, mine.w};
      int rid, u, val, rnn;
      if (star_rows(m, mine.x, oth, sorted, L.s, rid, u, val, rnn)) {
        if (!row_slot(x, m, neb, cap, tops, base, per)) return false;
        if (lane < m) st.ne[neb + rid] = mine.x;
        if (lane < u) st.nn[3 * (int64_t)neb + rnn] = val;
        if (lane == 0) {
          st.hdr[x] = make_int4(3 * neb, u, neb, m);
          st.cap[x] = cap;
        }
        return true;
      }
    }
    star_sync();
  }
  int m = 0;
  auto gather = [&](int o, int n) {
    for (int jb = 0; jb < n; jb += kWave) {
      int t = jb + lane < n ? st.ne[o + jb + lane] : -1;
      bool k = t >= 0 && st.talive[max(t, 0)] != 0 && has4(st.tet[max(t, 0)], x);
      uint64_t b = __ballot(k);
      int pos = m + __popcll(b & below);
      if (k && pos < kRowMax) L.w.id[pos] = t;
      m += __popcll(b);
    }
  };
  gather(neb, ne);
  for (int jb = 0; jb < nn; jb += kWave) {
    int w = jb + lane < nn ? st.nn[nnb + jb + lane] : -1;
    int2 rc = rec[max(w, 0)];
    for (uint64_t ab = __ballot(w >= 0 && rc.x == epoch && rc.y == x); ab; ab &= ab - 1) {
      int4 hz = st.hdr[__builtin_amdgcn_readlane(w, __ffsll((unsigned long long)ab) - 1)];
      gather(hz.z, hz.w);
    }
  }
  return m <= kRowMax && wide_put(st, x, m, neb, cap, tops, base, per, L);
}

// whether the class has rows to commit; the next class's counts start at zero
__device__ __forceinline__ bool class_committed(int* ctr, int epoch) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctr[K_CCOMMIT + (~epoch & 1)] = 0;
    ctr[K_NROWS + (~epoch & 1)] = 0;
  }
  int committed = ctr[K_CCOMMIT + (epoch & 1)], room = ctr[K_ROOM];
  return committed != 0 && room == 0;
}

// Two launch shapes rebuild the same rows, each once. Vertex order (large
// classes): each wavefront takes a range of vertex slots, reads their stamps
// a wavefront at a time and rebuilds the stamped rows in turn, so
// consecutive wavefronts read nearby rows. Row list (small classes): each
// wavefront takes rows of the class's row list in a wavefront-strided loop,
// and the grid is sized by the class rather than by the mesh.
__global__ void __launch_bounds__(256) k_commit3(Store3 st, int epoch, const int* __restrict__ own,
                                                 const int2* __restrict__ rec, int* tops, int64_t base,
                                                 int64_t per, int* ctr) {
  if (!class_committed(ctr, epoch)) return;
  __shared__ __align__(16) RowLds L[kB / kWave];
  int lane = __lane_id();
  int wid = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave));
  int nw = (int)((int64_t)gridDim.x * blockDim.x / kWave);
  int per_wave = (st.V + nw - 1) / nw;
  int x0 = (int)min((int64_t)wid * per_wave, (int64_t)st.V), x1 = min(st.V, x0 + per_wave);
  for (int c0 = x0; c0 < x1; c0 += kWave) {
    int xi = c0 + lane;
    uint64_t dm = __ballot(xi < x1 && own[xi] == epoch);
    while (dm) {
      int l = __ffsll((unsigned long long)dm) - 1;
      dm &= dm - 1;
      if (!commit_row3(st, c0 + l, epoch, rec, tops, base, per, L[threadIdx.x / kWave]) && lane == 0) room3(ctr, epoch);
    }
  }
}

__global__ void __launch_bounds__(256) k_commit3_list(Store3 st, int epoch, const int* __restrict__ rows,
                                                      const int2* __restrict__ rec, int* tops, int64_t base,
                                                      int64_t per, int* ctr) {
  __shared__ __align__(16) RowLds L[kB / kWave];
  int wid = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave));
  int nw = (int)((int64_t)gridDim.x * blockDim.x / kWave);
  // counts and the first row side by side (the list has a slot for every vertex)
  int n = ctr[K_NROWS + (epoch & 1)];
  int x = __builtin_amdgcn_readfirstlane(rows[min(wid, st.V - 1)]);
  if (!class_committed(ctr, epoch)) return;
  for (int i = wid; i < n; i += nw) {
    if (i != wid) x = __builtin_amdgcn_readfirstlane(rows[i]);
    if (!commit_row3(st, x, epoch, rec, tops, base, per, L[threadIdx.x / kWave]) && __lane_id() == 0) room3(ctr, epoch);
  }
}

// Sorted rows from the element lists gathered in build order: NE(v) sorted;
// NN(v) = the sorted distinct other vertices of NE(v)'s elements, in a slot
// of three entries per NE entry. One wavefront per vertex; rows of more than
// kRowMax elements take the serial form on its first lane.
__global__ void __launch_bounds__(256) k_rows_finish(Store3 st, const int* __restrict__ off, const int* __restrict__ cnt) {
  __shared__ __align__(16) RowLds L[kB / kWave];
  RowLds& mine = L[threadIdx.x / kWave];
  int lane = __lane_id();
  int wid = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave));
  int nw = (int)((int64_t)gridDim.x * blockDim.x / kWave);
  for (int v = wid; v < st.V; v += nw) {
    int o = __builtin_amdgcn_readfirstlane(off[v]), n = __builtin_amdgcn_readfirstlane(cnt[v]);
    if (n <= kWave) {
      bool has = lane < n;
      int t = has ? st.ne[o + lane] : INT_MAX;
      int oth[3], rid, u, val, rnn;
      others_of(st.tet[has ? t : 0], v, oth);
      if (star_rows(n, t, oth, false, mine.s, rid, u, val, rnn)) {
        if (has) st.ne[o + rid] = t;
        if (lane < u) st.nn[3 * (int64_t)o + rnn] = val;
        if (lane == 0) {
          st.hdr[v] = make_int4(3 * o, u, o, n);
          st.cap[v] = n;
        }
        continue;
      }
    }
    if (n > kRowMax) {
      if (lane == 0) rows_finish_serial(st, v, o, n);
      continue;
    }
    star_sync();
    for (int j = lane; j < n; j += kWave) mine.w.id[j] = st.ne[o + j];
    wide_put(st, v, n, o, n, nullptr, 0, 0, mine);
  }
}

// the stripes' bump pointers after a full row build: stripe s owns
// [base + s per, base + (s + 1) per). No commit is out of room.
__global__ void k_tops_init(int* tops, int64_t base, int64_t per, int* ctr) {
  int s = (int)threadIdx.x;
  if (s < kTopStripes) tops[s * kTopStride] = (int)(base + (int64_t)s * per);
  if (s < 2) ctr[K_ROOM + s] = 0;
}

// ---- colouring (Sec. 3.2) -----------------------------------------------------------------
// A vertex takes the first colour free among the active neighbours of larger
// key, once all of those have one: the greedy first-fit colouring in descending
// key order, whatever the order in which threads run. One scan of its row gives
// a vertex's record, the neighbours it waits for; from there on it follows their
// colours one after another. Re-reading the row of every waiting vertex in every
// iteration (14 neighbours, each two look-ups and a hash) took 78 us an iteration
// for the long lists of a mesh of 250,000 vertices.

// Lists of at most kSolve vertices, and what is left of a longer one once no
// more than that wait, are coloured by one work-group in LDS, without barriers:
// a record then holds places in the list (blk), 16 bits each (one work-group
// iterating over the rows took 80 us for some hundred vertices).
constexpr int kSolve = 2048, kSolveThreads = 1024, kPreds = 32;
struct Rec3 {
  uint64_t places[kPreds / 4];  // 16 bits each
  uint64_t used;                // colours taken, below 64
  int cnt;                      // places; -1: more than kPreds, or a colour past 63
  int pad;
};
// of a long list: the neighbours themselves, and how many have been followed
struct RecL {
  int ids[kPreds];
  uint64_t used;
  int cnt, pos;  // cnt: as above (pos: the neighbour it waits for, or -1); -2: the vertex has its colour
};

// no colours, no active vertices
__global__ void k_colour_start(int* col, uint8_t* act, int V, int* ctr) {
  zero_colouring(ctr);
  for (int v = gtid(); v < V; v += gstride()) {
    col[v] = -1;
    act[v] = 0;
  }
}

// a list's length: given, or (colouring ahead of the read-back) the device's,
// 0 when it is too long for one block
__device__ __forceinline__ int list_length(int n, const int* n_dev) {
  if (!n_dev) return n;
  n = *n_dev;
  return n > kSolve ? 0 : n;
}

// the list's vertices active, each with its place
__global__ void k_place(const int* __restrict__ A, int n, uint8_t* act, int* blk) {
  for (int i = gtid(); i < n; i += gstride()) {
    act[A[i]] = 1;
    blk[A[i]] = i;
  }
}
// the vertices of A without a colour: their list, their places, their number
__global__ void k_waiting(const int* __restrict__ A, int n, const int* __restrict__ col, int* out, int* blk, int* ctr) {
  for (int i = gtid(); i < n; i += gstride()) {
    int v = A[i];
    if (col[v] >= 0) continue;
    int k = pm::wave_append_slot(&ctr[K_WAIT]);
    if (k < kSolve) {  // the host has counted them
      out[k] = v;
      blk[v] = k;
    }
  }
}
// eight lanes a vertex, each every eighth entry of its row; a lane's places go
// behind the lower lanes' (their order does not matter)
template <class R>
__global__ void k_pred(Store3 st, const int* __restrict__ A, int n, const int* n_dev, const uint8_t* __restrict__ act,
                       const int* __restrict__ col, const int* __restrict__ blk, uint64_t sseed, R* recs) {
  n = list_length(n, n_dev);
  constexpr bool kLong = std::is_same<R, RecL>::value;
  constexpr int G = 8;
  int lane = __lane_id(), l = lane & (G - 1), gb = lane & ~(G - 1);
  for (int i = gtid() / G; i < n; i += gstride() / G) {
    int v = A[i];
    uint64_t kv = vkey(sseed, (uint32_t)v), used = 0;
    int4 h = st.hdr[v];
    int cnt = 0;
    bool big = false;
    for (int j0 = 0; j0 < h.y; j0 += G) {
      int j = j0 + l, place = -1;
      if (j < h.y) {
        int w = st.nn[h.x + j], cw = col[w];
        if (act[w] && vkey(sseed, (uint32_t)w) > kv) {
          if (cw < 0) place = kLong ? w : blk[w];
          else if ((cw & 0xFF) < 64) used |= 1ull << (cw & 0xFF);
          else big = true;
        }
      }
      uint32_t has = (uint32_t)(__ballot(place >= 0) >> gb) & 0xFFu;
      int at = cnt + __popc(has & ((1u << l) - 1u));
      if (place >= 0 && at < kPreds) {
        if constexpr (kLong) recs[i].ids[at] = place;
        else ((uint16_t*)recs[i].places)[at] = (uint16_t)place;
      }
      cnt += __popc(has);
    }
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
      uint32_t lo = (uint32_t)used, hi = (uint32_t)(used >> 32);
      lo |= (uint32_t)__shfl_xor((int)lo, d);
      hi |= (uint32_t)__shfl_xor((int)hi, d);
      used = (uint64_t)hi << 32 | lo;
    }
    big = ((__ballot(big) >> gb) & 0xFFu) != 0;
    if (l == 0) {
      recs[i].used = used;
      recs[i].cnt = big || cnt > kPreds ? -1 : cnt;
      if constexpr (kLong) recs[i].pos = big || cnt > kPreds ? -1 : 0;
    }
  }
}

__device__ __forceinline__ int colour_of(const int* col, int w) {
  return __hip_atomic_load(col + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// the visit of a vertex whose record did not hold everything: its colour, or -1
// while a neighbour before it has none (blocker: that neighbour, asked first the
// next time). Eight neighbours at a time, their loads in flight together.
__device__ __forceinline__ int far_visit(const Store3& st, int v, const uint8_t* act, const int* col, uint64_t sseed,
                                         int& blocker, int* ctr) {
  if (blocker >= 0 && colour_of(col, blocker) < 0) return -1;
  uint64_t kv = vkey(sseed, (uint32_t)v), used[kMaxColours / 64] = {0, 0, 0, 0};
  int4 h = st.hdr[v];
  constexpr int B = 8;
  for (int j0 = 0; j0 < h.y; j0 += B) {
    int w[B], cw[B];
    uint8_t aw[B];
#pragma unroll
    for (int q = 0; q < B; ++q) w[q] = j0 + q < h.y ? st.nn[h.x + j0 + q] : -1;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      cw[q] = w[q] >= 0 ? colour_of(col, w[q]) : -1;
      aw[q] = w[q] >= 0 ? act[w[q]] : 0;
    }
#pragma unroll
    for (int q = 0; q < B; ++q) {
      if (!aw[q] || vkey(sseed, (uint32_t)w[q]) < kv) continue;
      if (cw[q] < 0) {
        blocker = w[q];
        return -1;
      }
#pragma unroll
      for (int u = 0; u < kMaxColours / 64; ++u)
        if (cw[q] >> 6 == u) used[u] |= 1ull << (cw[q] & 63);
    }
  }
  int c = -1;
#pragma unroll
  for (int q = 0; q < kMaxColours / 64; ++q)
    if (c < 0 && ~used[q]) c = q * 64 + __ffsll((long long)~used[q]) - 1;
  if (c < 0) {
    atomicOr(&ctr[K_ERR], E_COLOURS);
    c = kMaxColours - 1;
  }
  return c;
}

// One iteration over a long list: every waiting vertex follows the neighbours it
// waits for as far as they have colours, kLocal times over (colours stored by
// the work-group itself are seen at once, others at the next launch). Counts go
// to the counters once per wavefront.
constexpr int kLocal = 3;
__global__ void __launch_bounds__(256) k_follow(Store3 st, const int* __restrict__ A, int n, const uint8_t* act, int* col,
                                               uint64_t sseed, RecL* recs, int* ctr) {
  int coloured = 0, ncol = 0;
  for (int i = gtid(); i < n; i += gstride()) {
    RecL& r = recs[i];
    int cnt = r.cnt, pos = r.pos, was = pos;
    if (cnt == -2) continue;
    uint64_t used = r.used;
    int v = A[i], c = -1;
    for (int p = 0; p < kLocal && c < 0; ++p) {
      while (pos < cnt) {
        int y = colour_of(col, r.ids[pos]);
        if (y < 0) break;
        if (y >= 64) {
          cnt = pos = -1;
          break;
        }
        used |= 1ull << y;
        ++pos;
      }
      if (cnt >= 0 && pos == cnt) {
        if (~used) c = __ffsll((long long)~used) - 1;
        else cnt = pos = -1;
      }
      // (its blocker in pos)
      if (cnt < 0) c = far_visit(st, v, act, col, sseed, pos, ctr);
    }
    if (c >= 0) {
      ((volatile int*)col)[v] = c;
      r.cnt = -2;
      ++coloured;
      ncol = max(ncol, c + 1);
    } else {
      if (cnt < 0) r.cnt = cnt;
      if (pos != was) {
        r.used = used;
        r.pos = pos;
      }
    }
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) ncol = max(ncol, __shfl_xor(ncol, d));
  count_add(ctr, S_COLOURED, coloured);
  // (a stale count only costs the add)
  if (__lane_id() == 0 && ncol > ctr[K_NCOL]) atomicMax(&ctr[K_NCOL], ncol);
}

// Colours the list A (n <= K * kSolveThreads) from its records, K vertices a
// thread, each thread going round its own until all have a colour. The waiting
// vertex of largest key is always ready, so the passes end (they are bounded
// all the same). The places are held in registers: what bounds it is the longest
// chain of waiting vertices, an LDS round trip per link.
constexpr int kMaxPasses = 1 << 20;
template <int K>
__device__ __forceinline__ void solve3(const Store3& st, const int* A, int n, const Rec3* recs, const uint8_t* act,
                                       int* col, uint64_t sseed, volatile uint16_t* cl, int* ctr) {
  constexpr int NT = kSolveThreads, W = kPreds / 4;
  int tid = (int)threadIdx.x;
  uint64_t cur[K][W], used[K];
  int pos[K], cnt[K];
  uint32_t todo = 0, far = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    int i = tid + k * NT;
    used[k] = 0;
    pos[k] = cnt[k] = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) cur[k][q] = 0;
    if (i >= n) continue;
    todo |= 1u << k;
    const Rec3& r = recs[i];
    cnt[k] = r.cnt;
    used[k] = r.used;
#pragma unroll
    for (int q = 0; q < W; ++q) cur[k][q] = r.places[q];
    if (r.cnt < 0) far |= 1u << k;
  }
  for (int p = 0; todo && p < kMaxPasses; ++p) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!((todo & ~far) >> k & 1)) continue;
      int i = tid + k * NT;
      while (pos[k] < cnt[k]) {
        int y = cl[cur[k][0] & 0xFFFF];
        if (y == 0xFFFF) break;
        if (y < 64) used[k] |= 1ull << y;
        else far |= 1u << k;
        ++pos[k];
        cur[k][0] >>= 16;
        if ((pos[k] & 3) == 0) {
#pragma unroll
          for (int q = 0; q + 1 < W; ++q) cur[k][q] = cur[k][q + 1];
        }
      }
      if (pos[k] < cnt[k]) continue;
      if (!~used[k]) far |= 1u << k;
      if (far >> k & 1) continue;
      int c = __ffsll((long long)~used[k]) - 1;
      cl[i] = (uint16_t)c;
      ((volatile int*)col)[A[i]] = c;
      todo &= ~(1u << k);
    }
    uint32_t slow = todo & far;
    while (slow) {
      int k = __ffs((int)slow) - 1, i = tid + k * NT;
      slow &= slow - 1;
      int b = -1, c = far_visit(st, A[i], act, col, sseed, b, ctr);
      if (c < 0) continue;
      cl[i] = (uint16_t)c;
      ((volatile int*)col)[A[i]] = c;
      todo &= ~(1u << k);
    }
  }
  if (todo) atomicOr(&ctr[K_ERR], E_COLOURS);  // cannot happen
}

// cnt, off, cls: also the class sizes, offsets and lists (a list coloured here
// as a whole), or null
__global__ void __launch_bounds__(kSolveThreads) k_solve(Store3 st, const int* A, int n, const int* n_dev,
                                                       const Rec3* recs, const uint8_t* act, int* col, uint64_t sseed, int* ctr, int* cnt,
                                                       int* off, int* cls) {
  __shared__ uint16_t cl[kSolve];
  __shared__ int hist[kMaxColours], cur[kMaxColours], wsum[4], ncol;
  int tid = (int)threadIdx.x;
  n = list_length(n, n_dev);
  if (n <= 0) return;
  for (int i = tid; i < n; i += kSolveThreads) cl[i] = 0xFFFF;
  if (tid < kMaxColours) hist[tid] = 0;
  if (tid == 0) ncol = 0;
  __syncthreads();
  if (n <= kSolveThreads) solve3<1>(st, A, n, recs, act, col, sseed, cl, ctr);
  else solve3<kSolve / kSolveThreads>(st, A, n, recs, act, col, sseed, cl, ctr);
  __syncthreads();
  // (a place without a colour, 0xFFFF, is an error that the host sees)
  for (int i = tid; i < n; i += kSolveThreads)
    if (cl[i] < kMaxColours) atomicAdd(&hist[cl[i]], 1);
  __syncthreads();
  int h = tid < kMaxColours ? hist[tid] : 0, incl = h, lane = __lane_id();
  if (h) atomicMax(&ncol, tid + 1);
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (tid < kMaxColours && lane == kWave - 1) wsum[tid / kWave] = incl;
  __syncthreads();
  if (tid == 0) {
    atomicAdd(&ctr[K_STRIPE + S_COLOURED], n);
    atomicMax(&ctr[K_NCOL], ncol);
  }
  if (!cls) return;
  if (tid < kMaxColours) {
    int o = incl - h;
    for (int w = 0; w < tid / kWave; ++w) o += wsum[w];
    cur[tid] = o;
    off[tid] = o;
    cnt[tid] = h;
  }
  __syncthreads();
  for (int i = tid; i < n; i += kSolveThreads)
    if (cl[i] < kMaxColours) cls[atomicAdd(&cur[cl[i]], 1)] = A[i];
}

__global__ void k_fill_int(int* p, int n, int x) {
  for (int i = gtid(); i < n; i += gstride()) p[i] = x;
}

// Class sizes: a histogram of the block's list entries in LDS, then one
// global add per colour and block.
__global__ void k_class_count(const int* __restrict__ A, int n, const int* __restrict__ col, int ncol, int* cnt) {
  __shared__ int h[kMaxColours];
  for (int c = threadIdx.x; c < ncol; c += blockDim.x) h[c] = 0;
  __syncthreads();
  for (int i = gtid(); i < n; i += gstride()) atomicAdd(&h[col[A[i]]], 1);
  __syncthreads();
  for (int c = threadIdx.x; c < ncol; c += blockDim.x)
    if (h[c]) atomicAdd(&cnt[c], h[c]);
}

// Class lists: each block ranks its entries per colour in LDS, reserves one
// range per colour with a global add, and writes the entries there. The
// order inside a class is not fixed; the members of a class are pairwise
// non-adjacent and their decisions do not depend on it.
// the classes' first slots: the exclusive prefix sums of the class sizes
// (one work-group of kMaxColours threads)
__global__ void k_class_offsets(const int* __restrict__ cnt, int ncol, int* off) {
  __shared__ int s[kMaxColours];
  int c = (int)threadIdx.x;
  int own = c < ncol ? cnt[c] : 0;
  s[c] = own;
  __syncthreads();
  for (int d = 1; d < kMaxColours; d <<= 1) {
    int t = c >= d ? s[c - d] : 0;
    __syncthreads();
    s[c] += t;
    __syncthreads();
  }
  if (c < ncol) off[c] = s[c] - own;
}

__global__ void k_class_place(const int* __restrict__ A, int n, const int* __restrict__ col, int ncol,
                              const int* __restrict__ off, int* cur, int* out) {
  __shared__ int h[kMaxColours], base[kMaxColours];
  for (int c = threadIdx.x; c < ncol; c += blockDim.x) h[c] = 0;
  __syncthreads();
  int i = (int)((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  int c = -1, r = 0, v = 0;
  if (i < n) {
    v = A[i];
    c = col[v];
    r = atomicAdd(&h[c], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < ncol; k += blockDim.x)
    if (h[k]) base[k] = off[k] + atomicAdd(&cur[k], h[k]);
  __syncthreads();
  if (c >= 0) out[base[c] + r] = v;
}

// ---- selection of active vertices ------------------------------------------------------------

// whether v (held by the 16 lanes of a group, -1: none) has a short edge it may
// collapse along; lane l takes every 16th neighbour
constexpr int kVL = 16;
__device__ __forceinline__ bool has_candidate(const Store3& st, int v, double L_low2) {
  int lane = __lane_id(), l = lane & (kVL - 1), gb = lane & ~(kVL - 1);
  bool any = false;
  if (v >= 0) {
    int4 h = st.hdr[v];
    for (int j = l; j < h.y && !any; j += kVL) {
      int u = st.nn[h.x + j];
      any = tag_ok(st, v, u) && len2(st, v, u) < L_low2;
    }
  }
  return (__ballot(any) >> gb & 0xFFFFull) != 0;
}

// mode 0: live vertices with a candidate; 1: flagged ones (flags cleared);
// 2: live interior vertices. Their list and its length (ctr[K_LIST], 0 at the
// start): every pass of a work-group over 256 vertices appends what it selects
// with one add. Mode 1 also ends a round: the old list's vertices lose colour
// and activity, and the new ones become active, each with its place (in launches
// of their own over the two lists that took 5 us of a round's 40 besides its
// classes). After a commit that ran out of room mode 1 does nothing and leaves
// the flags for the selection that follows the rebuild.
__global__ void __launch_bounds__(256) k_select(Store3 st, int mode, double L_low2, uint8_t* nxt, int* out, int* col,
                                              uint8_t* act, int* blk, int* ctr) {
  __shared__ int wsum[kB / kWave], base, q[kB];
  if (mode == 1) {
    if (ctr[K_ROOM]) return;
    zero_colouring(ctr);
  }
  int tid = (int)threadIdx.x, lane = __lane_id(), wv = tid / kWave;
  uint64_t below = (1ull << lane) - 1ull;
  // the place of a thread that is `on` among those of the work-group
  auto place = [&](bool on, int& total) {
    uint64_t b = __ballot(on);
    if (lane == 0) wsum[wv] = __popcll(b);
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < kB / kWave; ++k) {
      if (k < wv) before += wsum[k];
      total += wsum[k];
    }
    __syncthreads();
    return before + __popcll(b & below);
  };
  for (int v0 = (int)blockIdx.x * kB; v0 < st.V; v0 += (int)gridDim.x * kB) {
    int v = v0 + tid, total;
    bool on = v < st.V && st.valive[v] != 0;
    if (mode == 1 && v < st.V) {
      on = on && nxt[v];
      nxt[v] = 0;
      if (act[v]) {
        act[v] = 0;
        col[v] = -1;
      }
    }
    if (mode == 2) on = on && st.tag[v] == 0;
    int at = place(on, total);
    if (mode != 2) {
      // those come first that are to be tested, 16 lanes each (one thread went
      // along a row of 14 neighbours load after load: 20 us for a few vertices;
      // the launch now takes 9 us)
      if (on) q[at] = v;
      __syncthreads();
      for (int i0 = 0; i0 < total; i0 += kB / kVL) {
        int i = i0 + tid / kVL, x = i < total ? q[i] : -1;
        bool c = has_candidate(st, x, L_low2);
        if ((tid & (kVL - 1)) == 0 && i < total && !c) q[i] = -1;
      }
      __syncthreads();
      v = tid < total ? q[tid] : -1;
      on = v >= 0;
      at = place(on, total);
    }
    if (tid == 0) base = total ? atomicAdd(&ctr[K_LIST], total) : 0;
    __syncthreads();
    if (on) {
      out[base + at] = v;
      if (mode == 1) {
        act[v] = 1;
        blk[v] = base + at;
      }
    }
    __syncthreads();
  }
}

__global__ void k_compact_list(const int* __restrict__ flag, const int* __restrict__ scan, int n, int* out) {
  for (int v = gtid(); v < n; v += gstride())
    if (flag[v]) out[scan[v]] = v;
}

// ---- coarsening (Sec. 2.4.1) -------------------------------------------------------------------


// a vertex's position and metric, held by a lane
struct Vtx {
  double x, y, z;
  Met6 m;
};
__device__ __forceinline__ Vtx vtx(const Store3& st, int v) {
  double4 p = st.xyz[v];
  return Vtx{p.x, p.y, p.z, st.met[v]};
}
__device__ __forceinline__ double lane_of(double v, int k) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k), __builtin_amdgcn_readlane(__double2loint(v), k));
}
__device__ __forceinline__ Vtx lane_of(const Vtx& v, int k) {
  return Vtx{lane_of(v.x, k), lane_of(v.y, k), lane_of(v.z, k),
             Met6{lane_of(v.m.a00, k), lane_of(v.m.a01, k), lane_of(v.m.a02, k), lane_of(v.m.a11, k),
                  lane_of(v.m.a12, k), lane_of(v.m.a22, k)}};
}
__device__ __forceinline__ Vtx pick(bool c, const Vtx& a, const Vtx& b) {
  return Vtx{c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z,
             Met6{c ? a.m.a00 : b.m.a00, c ? a.m.a01 : b.m.a01, c ? a.m.a02 : b.m.a02, c ? a.m.a11 : b.m.a11,
                  c ? a.m.a12 : b.m.a12, c ? a.m.a22 : b.m.a22}};
}
// The geometry of the element (u, o0, o1, o2) in canonical order, o0 the
// smallest of the three: u first if it is smaller still; else o0, then the
// smallest of the other three, which the orientation has in the cycle (u, o2, o1).
__device__ __forceinline__ Geo3 star_geo(int u, const Vtx& pu, const int (&o)[3], const Vtx (&p)[3]) {
  bool A = u < o[0], B = !A && u < o[1] && u < o[2], C = !A && !B && o[1] < o[2];
  // A: u o0 o1 o2   B: o0 u o2 o1   C: o0 o1 u o2   D: o0 o2 o1 u
  Vtx q0 = pick(A, pu, p[0]);
  Vtx q1 = pick(A, p[0], pick(B, pu, pick(C, p[1], p[2])));
  Vtx q2 = pick(B, p[2], pick(C, pu, p[1]));
  Vtx q3 = pick(B, p[1], pick(A || C, p[2], pu));
  Geo3 g;
  g.p[0] = make_double4(q0.x, q0.y, q0.z, 0.0);
  g.p[1] = make_double4(q1.x, q1.y, q1.z, 0.0);
  g.p[2] = make_double4(q2.x, q2.y, q2.z, 0.0);
  g.p[3] = make_double4(q3.x, q3.y, q3.z, 0.0);
  g.m = Met6{(((q0.m.a00 + q1.m.a00) + q2.m.a00) + q3.m.a00) / 4.0, (((q0.m.a01 + q1.m.a01) + q2.m.a01) + q3.m.a01) / 4.0,
             (((q0.m.a02 + q1.m.a02) + q2.m.a02) + q3.m.a02) / 4.0, (((q0.m.a11 + q1.m.a11) + q2.m.a11) + q3.m.a11) / 4.0,
             (((q0.m.a12 + q1.m.a12) + q2.m.a12) + q3.m.a12) / 4.0, (((q0.m.a22 + q1.m.a22) + q2.m.a22) + q3.m.a22) / 4.0};
  return g;
}
// element e's other vertices, in an order with v before them that keeps its
// orientation, the smallest first
__device__ __forceinline__ void star_others(const int4& e, int v, int (&o)[3]) {
  int a, b, c;
  if (e.x == v) { a = e.y; b = e.z; c = e.w; }
  else if (e.y == v) { a = e.x; b = e.w; c = e.z; }
  else if (e.z == v) { a = e.w; b = e.x; c = e.y; }
  else { a = e.z; b = e.y; c = e.x; }
  bool bf = b < a && b < c, cf = c < a && c < b;
  o[0] = bf ? b : (cf ? c : a);
  o[1] = bf ? c : (cf ? a : b);
  o[2] = bf ? a : (cf ? b : c);
}

// One class: re-validation against the current graph, then each kept
// member's collapse, evaluated and applied (members are pairwise
// non-adjacent, so no member reads what another writes). A member runs on a
// wavefront: lane l holds its l-th neighbour and its l-th element with the
// positions and metrics of that element's other vertices, all gathered once.
// The candidates (neighbours by a short legal edge) are ordered by (L^2, u) by
// counting, and each is tried on registers alone: its data goes from its lane
// to all, and every lane evaluates its re-pointed element. Rows longer than the
// wavefront go on with further loads.
// With 32 lanes a member and the elements' four vertices gathered again for
// every candidate (21 loads a lane), a class of some hundred members took 30 us,
// most of it in candidates that fail: late rounds try every short edge of
// vertices that the quality bound keeps. Where half the lanes hold the elements
// (at most 32), the halves try two candidates side by side: the first classes of
// the 29^3 planar-front coarsening (65 to 116 thousand members) went from 469 to
// 393 us on average, those of up to four members from 7.9 to 7.2 us.
__global__ void __launch_bounds__(256) k_collapse(Store3 st, const int* __restrict__ list, int n,
                                                  const int* __restrict__ col, int c, uint64_t sseed, double L_low2,
                                                  double qmin3, uint8_t* nxt, int epoch, int* own, int* rows,
                                                  int2* rec, int* ctr) {
  // an earlier class's row commit ran out of room: the host rebuilds the
  // rows and runs this class again
  // (its flag and the member are loaded side by side)
  int room = ctr[K_ROOM];
  int lane = __lane_id();
  int gid = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave));
  int v = __builtin_amdgcn_readfirstlane(list[min(gid, n - 1)]);
  if (room || gid >= n) return;
  int4 h = st.hdr[v];
  int nn = __builtin_amdgcn_readfirstlane(h.y), ne = __builtin_amdgcn_readfirstlane(h.w);
  uint64_t kv = vkey(sseed, (uint32_t)v);
  // level by level: row entries; neighbours and elements; the elements' vertices
  // (two candidates side by side where half the lanes hold the elements)
  bool longer = nn > kWave;  // some candidates are not held by lanes
  bool pair = ne <= kWave / 2 && !longer, upper = pair && lane >= kWave / 2;
  int le = upper ? lane - kWave / 2 : lane;
  int w = lane < nn ? st.nn[h.x + lane] : -1, t = le < ne ? st.ne[h.z + le] : -1;
  int ws = max(w, 0);
  Vtx pv = vtx(st, v), pw = vtx(st, ws);
  int cw = col[ws], tv = st.tag[v], tw = st.tag[ws];
  int4 e = st.tet[max(t, 0)];
  bool beat = w >= 0 && cw == c && vkey(sseed, (uint32_t)w) > kv;
  for (int j = kWave + lane; j < nn; j += kWave) {
    int y = st.nn[h.x + j];
    beat = beat || (col[y] == c && vkey(sseed, (uint32_t)y) > kv);
  }
  if (__ballot(beat)) {
    if (lane == 0) {
      nxt[v] = 1;
      atomicAdd(&ctr[K_STRIPE + (gid & (kStripes - 1)) * kStripeW + S_DEFER], 1);
    }
    return;
  }
  auto length = [&](const Vtx& p) {
    return qform(edge_met(pv.m, p.m), p.x - pv.x, p.y - pv.y, p.z - pv.z);
  };
  double L = INFINITY;
  if (w >= 0 && (tv & ~tw) == 0) {
    double l = length(pw);
    if (l < L_low2) L = l;
  }
  bool cand = L < L_low2;
  // a held candidate's place in the order
  int rank = 0;
  uint64_t cb = __ballot(cand);
  int nc = __popcll(cb);
  for (uint64_t b = cb; b; b &= b - 1) {
    int k = __ffsll((unsigned long long)b) - 1;
    double Lk = lane_of(L, k);
    int wk = __builtin_amdgcn_readlane(w, k);
    rank += Lk < L || (Lk == L && wk < w) ? 1 : 0;
  }
  int o[3] = {-1, -1, -1};
  Vtx p[3];
  if (nc > 0 || longer) {
    if (t >= 0) star_others(e, v, o);
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = vtx(st, max(o[q], 0));
  }
  int target = -1, next = 0;
  double pL = -1.0;
  int pu = -1;
  for (;;) {
    // the next candidate: from the lanes, or past pL, pu among all
    Vtx du = pw;
    int u = -1, u2 = -1;
    if (!longer) {
      if (next >= nc) break;
      int k = __ffsll((unsigned long long)__ballot(cand && rank == next)) - 1;
      ++next;
      u = __builtin_amdgcn_readlane(w, k);
      du = lane_of(pw, k);
      if (pair && next < nc) {
        k = __ffsll((unsigned long long)__ballot(cand && rank == next)) - 1;
        ++next;
        u2 = __builtin_amdgcn_readlane(w, k);
        Vtx d2 = lane_of(pw, k);
        if (upper) {
          u = u2;
          du = d2;
        }
      }
    } else {
      double bL = 0.0;
      int bu = -1;
      for (int j = lane; j < nn; j += kWave) {
        int y = st.nn[h.x + j];
        if (!tag_ok(st, v, y)) continue;
        double l = length(vtx(st, y));
        if (!(l < L_low2)) continue;
        bool after = l > pL || (l == pL && y > pu);
        bool before = bu < 0 || l < bL || (l == bL && y < bu);
        if (after && before) {
          bL = l;
          bu = y;
        }
      }
#pragma unroll
      for (int d = kWave / 2; d > 0; d >>= 1) {
        double oL = __shfl_xor(bL, d);
        int ou = __shfl_xor(bu, d);
        if (ou >= 0 && (bu < 0 || oL < bL || (oL == bL && ou < bu))) {
          bL = oL;
          bu = ou;
        }
      }
      u = __builtin_amdgcn_readfirstlane(bu);
      if (u < 0) break;
      pL = bL;
      pu = u;
      du = vtx(st, u);
    }
    bool bad = false;
    if (t >= 0 && o[0] != u && o[1] != u && o[2] != u) {
      Geo3 g = star_geo(u, du, o, p);
      bad = !(vol6(g) > 0.0) || !(qual3(g) >= qmin3);
    }
    uint64_t bb = __ballot(bad);
    if (pair) {
      if ((uint32_t)bb == 0) {
        target = __builtin_amdgcn_readfirstlane(u);
        break;
      }
      if (u2 >= 0 && bb >> 32 == 0) {
        target = u2;
        break;
      }
      continue;
    }
    if (bb) continue;
    for (int k = kWave + lane; k < ne; k += kWave) {
      int4 f = st.tet[st.ne[h.z + k]];
      if (has4(f, u)) continue;
      Geo3 g = geo(st, canon4(replace4(f, v, u)));
      bad = bad || !(vol6(g) > 0.0) || !(qual3(g) >= qmin3);
    }
    if (!__ballot(bad)) {
      target = u;
      break;
    }
  }
  int stripe = K_STRIPE + (gid & (kStripes - 1)) * kStripeW;
  if (lane == 0) {
    atomicAdd(&ctr[stripe + S_EVAL], 1);
    if (target >= 0) {
      atomicAdd(&ctr[stripe + S_COMMIT], 1);
      ctr[K_CCOMMIT + (epoch & 1)] = 1;
      st.valive[v] = 0;
      rec[v] = make_int2(epoch, target);
    }
  }
  if (target < 0) return;
  for (int k = lane; k < ne; k += kWave) {
    int tk = st.ne[h.z + k];
    int4 f = st.tet[tk];
    if (has4(f, target))
      st.talive[tk] = 0;
    else
      st.tet[tk] = canon4(replace4(f, v, target));
  }
  // the changed rows (every neighbour's, the target's among them) for the
  // row commit, stamped with the class epoch; with a row list (rows given)
  // the first stamp of a row in this class also appends it to the list
  // (one add per wavefront)
  for (int jb = 0; jb < nn; jb += kWave) {
    int j = jb + lane;
    int y = -1;
    bool fresh = false;
    if (j < nn) {
      y = st.nn[h.x + j];
      nxt[y] = 1;
      if (rows)
        fresh = atomicExch(&own[y], epoch) != epoch;
      else
        own[y] = epoch;
    }
    if (rows) {
      uint64_t fb = __ballot(fresh);
      int at = 0;
      if (lane == 0 && fb) at = atomicAdd(&ctr[K_NROWS + (epoch & 1)], __popcll(fb));
      at = __builtin_amdgcn_readfirstlane(at);
      if (fresh) rows[at + __popcll(fb & ((1ull << lane) - 1ull))] = y;
    }
  }
}

// Arrays moved to larger blocks, and the new slots of some set to -1 (src null),
// a row of the grid each: a copy of its own for each of the 20 arrays took 1.8 us
// and a gap, 71 times in a cycle of the 11^3 mesh. The blocks start on 256 bytes.
struct Moves {
  struct {
    const void* src;
    void* dst;
    int64_t bytes;
  } e[24];
  int n;
};
__global__ void k_move(Moves mv) {
  auto e = mv.e[blockIdx.y];
  int64_t i0 = gtid(), step = (int64_t)gridDim.x * blockDim.x;
  if (!e.src) {
    for (int64_t i = i0; i < e.bytes / 4; i += step) ((int*)e.dst)[i] = -1;
    return;
  }
  int64_t full = e.bytes / 16;
  for (int64_t i = i0; i < full; i += step) ((int4*)e.dst)[i] = ((const int4*)e.src)[i];
  for (int64_t i = full * 16 + i0; i < e.bytes; i += step) ((uint8_t*)e.dst)[i] = ((const uint8_t*)e.src)[i];
}

// stable renumbering of live vertices and elements (a monotone map keeps the
// elements' canonical order)
__global__ void k_flags(const uint8_t* __restrict__ a, int n, int* f) {
  for (int i = gtid(); i < n; i += gstride()) f[i] = a[i] ? 1 : 0;
}

// the live flags of vertices and elements as counts
__global__ void k_live(Store3 st, int* vf, int* tf) {
  for (int i = gtid(); i < max(st.V, st.T); i += gstride()) {
    if (i < st.V) vf[i] = st.valive[i] ? 1 : 0;
    if (i < st.T) tf[i] = st.talive[i] ? 1 : 0;
  }
}

// (after a renumbering) every slot is live and no vertex selected
__global__ void k_all_live(Store3 st, uint8_t* nxt) {
  for (int i = gtid(); i < max(st.V, st.T); i += gstride()) {
    if (i < st.V) {
      st.valive[i] = 1;
      nxt[i] = 0;
    }
    if (i < st.T) st.talive[i] = 1;
  }
}

__global__ void k_compact_v(Store3 st, const int* __restrict__ vmap, double4* xyz, Met6* met, uint8_t* tag) {
  for (int v = gtid(); v < st.V; v += gstride()) {
    if (!st.valive[v]) continue;
    int o = vmap[v];
    xyz[o] = st.xyz[v];
    met[o] = st.met[v];
    tag[o] = st.tag[v];
  }
}

__global__ void k_compact_t(Store3 st, const int* __restrict__ vmap, const int* __restrict__ tmap, int4* tet) {
  for (int t = gtid(); t < st.T; t += gstride()) {
    if (!st.talive[t]) continue;
    int4 e = st.tet[t];
    tet[tmap[t]] = make_int4(vmap[e.x], vmap[e.y], vmap[e.z], vmap[e.w]);
  }
}

__global__ void k_fill_u8(uint8_t* p, int n, uint8_t x) {
  for (int i = gtid(); i < n; i += gstride()) p[i] = x;
}

// ---- refinement (Sec. 2.4.2) ---------------------------------------------------------------------

// marks the long edges (v, w), w > v, per NN entry; counts them per vertex
// kVL lanes a vertex, lane l every kVL-th neighbour: one thread along a row
// took 41 us on a mesh of 5,600 vertices, however few it had; this takes 6 us
__global__ void k_mark(Store3 st, double L_up2, int* mark, int* cnt, int* ctr) {
  int lane = __lane_id(), l = lane & (kVL - 1), gb = lane & ~(kVL - 1);
  int edges = 0;
  for (int v = gtid() / kVL; v < st.V; v += gstride() / kVL) {
    int4 h = st.hdr[v];
    int c = 0;
    for (int j0 = 0; j0 < h.y; j0 += kVL) {
      int j = j0 + l;
      bool m = false;
      if (j < h.y) {
        int w = st.nn[h.x + j];
        if (w > v) {
          ++edges;
          m = len2(st, v, w) > L_up2;
        }
        mark[h.x + j] = m ? 1 : 0;
      }
      c += __popcll(__ballot(m) >> gb & 0xFFFFull);
    }
    if (l == 0) cnt[v] = c;
  }
  count_add(ctr, S_EDGES, edges);
}
// new vertices on the marked edges (a, b > a), in (a, b) order; the mark
// becomes the new vertex's id
__global__ void k_mint(Store3 st, int V0, const int* __restrict__ vscan, int* mark) {
  int lane = __lane_id(), l = lane & (kVL - 1), gb = lane & ~(kVL - 1);
  for (int v = gtid() / kVL; v < V0; v += gstride() / kVL) {
    int4 h = st.hdr[v];
    int first = V0 + vscan[v];
    for (int j0 = 0; j0 < h.y; j0 += kVL) {
      int j = j0 + l;
      bool m = j < h.y && mark[h.x + j] != 0;
      uint64_t b = __ballot(m) >> gb & 0xFFFFull;
      int id = first + __popcll(b & ((1ull << l) - 1ull));
      first += __popcll(b);
      if (j < h.y) mark[h.x + j] = m ? id : -1;
      if (!m) continue;
      int w = st.nn[h.x + j];
      double4 a = st.xyz[v], p = st.xyz[w];
      st.xyz[id] = make_double4((a.x + p.x) * 0.5, (a.y + p.y) * 0.5, (a.z + p.z) * 0.5, 0.0);
      st.met[id] = edge_met(st.met[v], st.met[w]);
      st.tag[id] = st.tag[v] & st.tag[w];
      st.valive[id] = 1;
    }
  }
}

struct Split {
  int a, b, mid;
  double L2;
};

__device__ __forceinline__ bool split_before(const Split& p, const Split& q) {
  if (p.L2 != q.L2) return p.L2 > q.L2;
  return p.a != q.a ? p.a < q.a : p.b < q.b;
}

// the midpoint id of edge (a, b) (a < b): b's position in NN(a)
__device__ __forceinline__ int mid_of(const Store3& st, const int* mark, int a, int b) {
  int4 h = st.hdr[a];
  int lo = 0, hi = h.y - 1;
  while (lo <= hi) {
    int m = (lo + hi) >> 1;
    int w = st.nn[h.x + m];
    if (w == b) return mark[h.x + m];
    if (w < b) lo = m + 1;
    else hi = m - 1;
  }
  return -1;
}

// The element's split edges in the global order, in s (a column of the work-
// group's LDS). An edge is split when its length says so, the same test that
// marked it; only those are looked up in a row, and only where their midpoints
// are wanted (mark).
constexpr int kSplitThreads = 64;
struct SplitLds {
  Split s[6][kSplitThreads];
  int4 piece[8][kSplitThreads];
  int from[8][kSplitThreads];
};
__device__ __forceinline__ int own_splits(const Store3& st, const int* mark, int4 e, double L_up2, SplitLds& S) {
  int c = (int)threadIdx.x, n = 0;
  int id[4] = {e.x, e.y, e.z, e.w};
  double4 p[4];
  Met6 m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = st.xyz[id[i]];
    m[i] = st.met[id[i]];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = i + 1; j < 4; ++j) {
      double L = qform(edge_met(m[i], m[j]), p[j].x - p[i].x, p[j].y - p[i].y, p[j].z - p[i].z);
      if (!(L > L_up2)) continue;
      int a = min(id[i], id[j]), b = max(id[i], id[j]);
      Split x{a, b, mark ? mid_of(st, mark, a, b) : 0, L};
      int k = n++;
      while (k > 0 && split_before(x, S.s[k - 1][c])) {
        S.s[k][c] = S.s[k - 1][c];
        --k;
      }
      S.s[k][c] = x;
    }
  return n;
}

// Bisection along the first split edge (in the global order) each piece
// holds, children depth first (the child keeping the edge's smaller id
// first). A piece needs only the splits after the one that made it, since it
// lies inside its parent. count_only: returns the number of leaves; else
// writes them (the first into slot t, the rest from base).
constexpr int kMaxLeaves = 64;
__device__ __forceinline__ int bisect(const Store3& st, int ns, int4 e, bool count_only, int t, int base, SplitLds& S) {
  int col = (int)threadIdx.x;
  int top = 0;
  S.piece[0][col] = e;
  S.from[0][col] = 0;
  int leaves = 0;
  while (top >= 0) {
    int4 x = S.piece[top][col];
    int k = S.from[top][col];
    --top;
    while (k < ns && !(has4(x, S.s[k][col].a) && has4(x, S.s[k][col].b))) ++k;
    if (k == ns) {
      if (!count_only) {
        int slot = leaves == 0 ? t : base + leaves - 1;
        st.tet[slot] = canon4(x);
        st.talive[slot] = 1;
      }
      ++leaves;
      continue;
    }
    // (when counting, a number no vertex has stands for the midpoint: it is in
    // no other split edge)
    Split sp = S.s[k][col];
    int mid = count_only ? -1 - k : sp.mid;
    int4 ca = replace4(x, sp.b, mid);  // keeps a
    int4 cb = replace4(x, sp.a, mid);  // keeps b
    // depth first, child a first: push b, then a
    ++top;
    S.piece[top][col] = cb;
    S.from[top][col] = k + 1;
    ++top;
    S.piece[top][col] = ca;
    S.from[top][col] = k + 1;
  }
  return leaves;
}

__global__ void __launch_bounds__(kSplitThreads) k_split_count(Store3 st, int T0, double L_up2, int* tcnt, int* ctr) {
  __shared__ SplitLds S;
  for (int t = gtid(); t < T0; t += gstride()) {
    int c = 0;
    if (st.talive[t]) {
      int4 e = st.tet[t];
      int ns = own_splits(st, nullptr, e, L_up2, S);
      if (ns > 0) {
        int l = bisect(st, ns, e, true, t, 0, S);
        if (l > kMaxLeaves) atomicOr(&ctr[K_ERR], E_LEAVES);
        c = l - 1;
      }
    }
    tcnt[t] = c;
  }
}
__global__ void __launch_bounds__(kSplitThreads) k_split_write(Store3 st, int T0, double L_up2, const int* __restrict__ mark,
                                                             const int* __restrict__ tscan) {
  __shared__ SplitLds S;
  for (int t = gtid(); t < T0; t += gstride()) {
    if (!st.talive[t]) continue;
    int4 e = st.tet[t];
    int ns = own_splits(st, mark, e, L_up2, S);
    if (ns > 0) bisect(st, ns, e, false, t, T0 + tscan[t], S);
  }
}

// ---- smoothing (Sec. 2.4.4) -------------------------------------------------------------------------

// One class of Laplacian moves, a wavefront per member: a lane per neighbour for
// the terms of the sums, then a lane per element for its old and its moved
// quality. The terms lie in LDS and nine lanes add one sum each in row order, so
// each is the serial loop's; the minima fold as the serial loop folds them.
// What bounds a class is one member's chain of loads (header, row, vertices,
// element, its vertices), so the width goes into a member: with 8 lanes each,
// going along a row in steps of 8, a class of the 11^3 mesh took 47 us; this
// takes 9 us (and 47 us in place of 77 us on the 29^3 one, with thousands of
// members).

// the serial loop's minimum over the wavefront (lane 0 holds the first value, a
// lane without any infinity): a value that is no number counts only as the first
__device__ __forceinline__ double wave_min(double v) {
  double m = v == v ? v : INFINITY;
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    double o = __shfl_xor(m, d);
    m = o < m ? o : m;
  }
  double f = lane_of(v, 0);
  return f == f ? m : f;
}

__device__ __forceinline__ double4 pick(bool c, double4 a, double4 b) {
  return make_double4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, 0.0);
}

__global__ void __launch_bounds__(256) k_smooth(Store3 st, const int* __restrict__ list, int n, int* ctr) {
  __shared__ double terms[kB / kWave][9][kWave + 2];
  auto& T = terms[threadIdx.x / kWave];
  int lane = __lane_id();
  int nw = (int)(gridDim.x * (blockDim.x / kWave));
  int ev = 0, cm = 0;
  for (int i = (int)(blockIdx.x * (blockDim.x / kWave)) + (int)threadIdx.x / kWave; i < n; i += nw) {
    int v = __builtin_amdgcn_readfirstlane(list[i]);
    int4 h = st.hdr[v];
    int nn = __builtin_amdgcn_readfirstlane(h.y), ne = __builtin_amdgcn_readfirstlane(h.w);
    double4 pv = st.xyz[v];
    Met6 mv = st.met[v];
    // the neighbours' terms, and this lane's element, side by side
    int t = lane < ne ? st.ne[h.z + lane] : -1;
    int4 t4 = st.tet[max(t, 0)];
    // lane c < 9 adds up the c-th sum in row order
    double sum = 0.0;
    for (int jb = 0; jb < nn; jb += kWave) {
      int j = jb + lane;
      Met6 e{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      double tx = 0.0, ty = 0.0, tz = 0.0;
      if (j < nn) {
        int w = st.nn[h.x + j];
        e = edge_met(mv, st.met[w]);
        double4 pw = st.xyz[w];
        double dx = pw.x - pv.x, dy = pw.y - pv.y, dz = pw.z - pv.z;
        tx = (e.a00 * dx + e.a01 * dy) + e.a02 * dz;
        ty = (e.a01 * dx + e.a11 * dy) + e.a12 * dz;
        tz = (e.a02 * dx + e.a12 * dy) + e.a22 * dz;
      }
      T[0][lane] = e.a00;
      T[1][lane] = e.a01;
      T[2][lane] = e.a02;
      T[3][lane] = e.a11;
      T[4][lane] = e.a12;
      T[5][lane] = e.a22;
      T[6][lane] = tx;
      T[7][lane] = ty;
      T[8][lane] = tz;
      star_sync();
      const double* mine = T[lane < 9 ? lane : 0];
      int cnt = min(kWave, nn - jb);
      for (int q = 0; q < cnt; ++q) sum = sum + mine[q];
      star_sync();
    }
    Met6 G{lane_of(sum, 0), lane_of(sum, 1), lane_of(sum, 2), lane_of(sum, 3), lane_of(sum, 4), lane_of(sum, 5)};
    double rx = lane_of(sum, 6), ry = lane_of(sum, 7), rz = lane_of(sum, 8);
    double det = det3(G);
    double c00 = G.a11 * G.a22 - G.a12 * G.a12, c01 = G.a02 * G.a12 - G.a01 * G.a22,
           c02 = G.a01 * G.a12 - G.a02 * G.a11, c11 = G.a00 * G.a22 - G.a02 * G.a02,
           c12 = G.a01 * G.a02 - G.a00 * G.a12, c22 = G.a00 * G.a11 - G.a01 * G.a01;
    double4 p = make_double4(pv.x + ((c00 * rx + c01 * ry) + c02 * rz) / det,
                             pv.y + ((c01 * rx + c11 * ry) + c12 * rz) / det,
                             pv.z + ((c02 * rx + c12 * ry) + c22 * rz) / det, 0.0);
    if (lane == 0) ++ev;
    bool bad = false;
    double mo = INFINITY, mn = INFINITY;
    for (int k = lane; k < ne; k += kWave) {
      if (k != lane) t4 = st.tet[st.ne[h.z + k]];
      Geo3 go = geo(st, t4);
      Geo3 gn = go;
      gn.p[0] = pick(t4.x == v, p, go.p[0]);
      gn.p[1] = pick(t4.y == v, p, go.p[1]);
      gn.p[2] = pick(t4.z == v, p, go.p[2]);
      gn.p[3] = pick(t4.w == v, p, go.p[3]);
      if (!(vol6(gn) > 0.0)) bad = true;
      double qo = qual3(go), qn = qual3(gn);
      if (k == 0 || qo < mo) mo = qo;
      if (k == 0 || qn < mn) mn = qn;
    }
    double oldmin = wave_min(mo), newmin = wave_min(mn);
    if (__ballot(bad) || !(newmin >= oldmin)) continue;
    if (lane == 0) {
      st.xyz[v] = p;
      ++cm;
    }
  }
  count_add(ctr, S_EVAL, ev);
  count_add(ctr, S_COMMIT, cm);
}

// ---- quality ----------------------------------------------------------------------------------------

constexpr int QB = 256;
__global__ void k_quality(Store3 st, double* psum, double* pmin) {
  __shared__ double ls[QB], lm[QB];
  double s = 0.0, mn = INFINITY;
  for (int t = gtid(); t < st.T; t += gstride()) {
    if (!st.talive[t]) continue;
    double q = qual(geo(st, st.tet[t]));
    s = s + q;
    mn = fmin(mn, q);
  }
  ls[threadIdx.x] = s;
  lm[threadIdx.x] = mn;
  __syncthreads();
  for (int k = QB / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) {
      ls[threadIdx.x] = ls[threadIdx.x] + ls[threadIdx.x + k];
      lm[threadIdx.x] = fmin(lm[threadIdx.x], lm[threadIdx.x + k]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    psum[blockIdx.x] = ls[0];
    pmin[blockIdx.x] = lm[0];
  }
}

// (one thread adding up the 1,024 sums took 73 us)
__global__ void k_quality_final(const double* __restrict__ psum, const double* __restrict__ pmin, int n, double* out,
                                int* at, int no) {
  __shared__ double ls[QB], lm[QB];
  int tid = (int)threadIdx.x;
  double s = 0.0, mn = INFINITY;
  for (int i = tid; i < n; i += QB) {
    s = s + psum[i];
    mn = fmin(mn, pmin[i]);
  }
  ls[tid] = s;
  lm[tid] = mn;
  __syncthreads();
  for (int k = QB / 2; k > 0; k >>= 1) {
    if (tid < k) {
      ls[tid] = ls[tid] + ls[tid + k];
      lm[tid] = fmin(lm[tid], lm[tid + k]);
    }
    __syncthreads();
  }
  if (tid == 0) {
    out[0] = ls[0];
    out[1] = lm[0];
  }
  pm::mail_post(at, no);
}

__global__ void k_export(Store3 st, double* xyz, int* tet, double* met) {
  for (int v = gtid(); v < st.V; v += gstride()) {
    double4 p = st.xyz[v];
    if (xyz) {
      xyz[3 * v] = p.x;
      xyz[3 * v + 1] = p.y;
      xyz[3 * v + 2] = p.z;
    }
    if (met) {
      Met6 g = st.met[v];
      double* q = met + 6 * v;
      q[0] = g.a00;
      q[1] = g.a01;
      q[2] = g.a02;
      q[3] = g.a11;
      q[4] = g.a12;
      q[5] = g.a22;
    }
  }
  if (tet)
    for (int t = gtid(); t < st.T; t += gstride()) {
      int4 e = st.tet[t];
      tet[4 * t] = e.x;
      tet[4 * t + 1] = e.y;
      tet[4 * t + 2] = e.z;
      tet[4 * t + 3] = e.w;
    }
}

inline int grid(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + kB - 1) / kB, 16384)); }

}  // namespace pm3

using namespace pm3;

// ---- host side ------------------------------------------------------------------------------------------

struct pm3_mesh {
  hipStream_t s = nullptr;
  uint64_t seed = 0;
  std::string err;
  Store3 st;
  int Vcap = 0, Tcap = 0;
  int64_t nncap = 0, necap = 0;
  int* ctr = nullptr;   // device counters, then class sizes, cursors and offsets (kMaxColours each)
  int* hctr = nullptr;  // pinned mirror
  pm::Mail mail;        // its block's
  // scratch
  int *cnt = nullptr, *off = nullptr, *flag = nullptr, *scan = nullptr, *partial = nullptr;
  int *A = nullptr, *B = nullptr, *cls = nullptr, *col = nullptr, *blk = nullptr, *mark = nullptr,
      *tcnt = nullptr, *tscan = nullptr;
  Rec3* recs = nullptr;  // one-block colourings: predecessor records
  RecL* recl = nullptr;  // long colourings', lcap of them
  int lcap = 0;
  uint8_t *act = nullptr, *nxt = nullptr;
  double* qbuf = nullptr;
  int scap = 0, tscap = 0, pcap = 0;
  int64_t mcap = 0;
  // row commit: per-vertex class stamps and member records, the stripes'
  // bump pointers, the epoch of the last class, and the pool range above
  // the last full build that the stripes share
  int* own = nullptr;
  int* rows = nullptr;  // the rows stamped by the class in progress, each once
  int2* rec = nullptr;
  int* tops = nullptr;
  int epoch = 0;
  int64_t top_base = 0, top_per = 0;
  double headroom = 3.0;  // pool_headroom of the creation options
  bool rows_ok = false;   // the rows are those of the element list (false: their last build failed)
};

namespace {

thread_local std::string g3_create_err;

pm_status fail3(pm3_mesh* m, pm_status st, const std::string& msg) {
  if (m) m->err = msg;
  return st;
}

#define H3(call)                                                                    \
  do {                                                                              \
    hipError_t e_ = (call);                                                         \
    if (e_ != hipSuccess) return fail3(m, PM_E_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)
#define T3(call)                     \
  do {                               \
    pm_status s_ = (call);           \
    if (s_ != PM_OK) return s_;      \
  } while (0)

// Device blocks come from the library's stream-ordered block cache: a block
// freed on the handle's stream is reused only by later work on that stream,
// so growing an array needs no wait before the old block is released.
template <class T>
pm_status dgrow(pm3_mesh* m, T** p, int64_t old_n, int64_t n, bool keep) {
  if (n <= old_n && *p) return PM_OK;
  T* q = nullptr;
  if (pm::block_alloc(m->s, (void**)&q, sizeof(T) * (size_t)std::max<int64_t>(n, 1)) != hipSuccess) {
    (void)hipGetLastError();
    return fail3(m, PM_E_NOMEM, "device allocation failed");
  }
  if (keep && *p && old_n > 0) H3(hipMemcpyAsync(q, *p, sizeof(T) * (size_t)old_n, hipMemcpyDeviceToDevice, m->s));
  if (*p) pm::block_free(*p);
  *p = q;
  return PM_OK;
}

template <class T>
void dfree3(T*& p) {
  if (p) pm::block_free(p);
  p = nullptr;
}

// the counters, and `more` class sizes behind them
pm_status read_ctr(pm3_mesh* m, int more = 0) {
  pm::mail_next(m->mail);
  k_mail3<<<1, kB, 0, m->s>>>(m->ctr, more, m->hctr, (int*)m->mail.at, m->mail.no);
  H3(hipGetLastError());
  H3(pm::mail_wait(m->mail, m->s));
  return PM_OK;
}

pm_status zero_ctr(pm3_mesh* m) {
  k_zero_ctr<<<1, kB, 0, m->s>>>(m->ctr);
  H3(hipGetLastError());
  return PM_OK;
}

// capacity for V vertices and T elements (kept contents)
pm_status reserve(pm3_mesh* m, int V, int T) {
  Store3& st = m->st;
  Moves mv{};
  int64_t most = 0;
  void* old[24];
  auto grow = [&](auto** p, int64_t n0, int64_t n1, bool keep) -> pm_status {
    using E = std::remove_reference_t<decltype(**p)>;
    E* q = nullptr;
    T3(dgrow(m, &q, 0, n1, false));
    if (*p && keep && n0 > 0) {
      old[mv.n] = *p;
      mv.e[mv.n++] = {*p, q, (int64_t)sizeof(E) * n0};
      most = std::max(most, (int64_t)sizeof(E) * n0);
    } else if (*p) {
      pm::block_free(*p);
    }
    *p = q;
    return PM_OK;
  };
  // new vertex slots carry no class stamp or record
  auto unset = [&](void* from, int64_t bytes) {
    old[mv.n] = nullptr;
    mv.e[mv.n++] = {nullptr, from, bytes};
    most = std::max(most, bytes);
  };
  pm_status rc = PM_OK;
  auto all = [&]() -> pm_status {
    if (V > m->Vcap) {
      int64_t c = m->Vcap, nc = std::max(V, m->Vcap + m->Vcap / 2);
      T3(grow(&st.xyz, c, nc, true));
      T3(grow(&st.met, c, nc, true));
      T3(grow(&st.tag, c, nc, true));
      T3(grow(&st.valive, c, nc, true));
      // growth happens in the middle of a refinement pass, whose rows, vertex
      // scan and element scan must survive it: every array keeps its contents
      T3(grow(&st.hdr, c, nc, true));
      T3(grow(&m->cnt, c + 1, nc + 1, true));
      T3(grow(&m->off, c + 1, nc + 1, true));
      T3(grow(&m->flag, c + 1, nc + 1, true));
      T3(grow(&m->scan, c + 1, nc + 1, true));
      T3(grow(&m->A, c, nc, true));
      T3(grow(&m->B, c, nc, false));
      T3(grow(&m->cls, c, nc, true));
      T3(grow(&m->col, c, nc, true));
      T3(grow(&m->blk, c, nc, true));
      T3(grow(&m->act, c, nc, true));
      T3(grow(&m->nxt, c, nc, true));
      T3(grow(&st.cap, c, nc, true));
      T3(grow(&m->own, c, nc, true));
      T3(grow(&m->rec, c, nc, true));
      T3(grow(&m->rows, c, nc, false));
      unset(m->own + c, sizeof(int) * (nc - c));
      unset(m->rec + c, sizeof(int2) * (nc - c));
      m->Vcap = (int)nc;
    }
    if (T > m->Tcap) {
      int64_t c = m->Tcap, nc = std::max(T, m->Tcap + m->Tcap / 2);
      T3(grow(&st.tet, c, nc, true));
      T3(grow(&st.talive, c, nc, true));
      T3(grow(&m->tcnt, c + 1, nc + 1, true));
      T3(grow(&m->tscan, c + 1, nc + 1, true));
      m->Tcap = (int)nc;
    }
    return PM_OK;
  };
  rc = all();
  // (also what was grown before an allocation failed)
  if (mv.n) {
    k_move<<<dim3(std::min(grid(most / 16 + 1), 2048), mv.n), kB, 0, m->s>>>(mv);
    hipError_t e = hipGetLastError();
    for (int k = 0; k < mv.n; ++k)
      if (old[k]) pm::block_free(old[k]);
    if (rc == PM_OK) H3(e);
  }
  T3(rc);
  int need = pm::scan_partials_needed(m->Vcap) + pm::scan_partials_needed(m->Tcap);
  if (need > m->pcap) {
    T3(dgrow(m, &m->partial, m->pcap, need, false));
    m->pcap = need;
  }
  return PM_OK;
}

// a vertex array's and an element array's exclusive scans with one read-back, of
// their totals and every counter
pm_status scan_both(pm3_mesh* m, const int* v, int* vout, int V, int* nv, const int* t, int* tout, int T, int* nt) {
  int* ctr = m->ctr;
  auto load = [](const int* a) { return [=] __device__(int i, bool on) { return on ? a[i] : 0; }; };
  auto at = [](const int* a) { return [=] __device__(int i) { return a[i]; }; };
  auto put = [](int* a) { return [=] __device__(int i, int before, int) { a[i] = before; }; };
  auto total = [](int* a) { return [=] __device__(int x) { *a = x; }; };
  pm::scan_fused2<int, 8>(load(v), at(v), put(vout), total(ctr + K_TOTAL), V, load(t), at(t), put(tout),
                          total(ctr + K_TOTAL2), T, m->partial, m->s);
  T3(read_ctr(m));
  *nv = m->hctr[K_TOTAL];
  *nt = m->hctr[K_TOTAL2];
  return PM_OK;
}
// the exclusive scan of n ints and its total, likewise
pm_status scan_total(pm3_mesh* m, const int* in, int* out, int n, int* total) {
  pm::scan_excl(in, out, n, m->ctr + K_TOTAL, m->partial, m->s);
  T3(read_ctr(m));
  *total = m->hctr[K_TOTAL];
  return PM_OK;
}

// Every row from the element list, packed and sorted; the pools keep the
// headroom times the packed size free above it for the row commits of a
// coarsening phase (a row that outgrows its slot moves, with twice the room,
// and its old slot stays unused until the next full build), split into the
// stripes' ranges. Clears the room counters.
// (all_live: no element slot is dead, so the rows' total is known without a
// read-back)
pm_status build_rows(pm3_mesh* m, bool all_live) {
  Store3& st = m->st;
  int V = st.V;
  m->rows_ok = false;
  k_fill_int<<<grid(V + 1), kB, 0, m->s>>>(m->cnt, V + 1, 0);
  struct Temp {
    int4* p = nullptr;
    ~Temp() { dfree3(p); }
  } rank;
  T3(dgrow(m, &rank.p, 0, st.T, false));
  k_ne_count<<<std::max(1, (st.T + kB * kCountPer - 1) / (kB * kCountPer)), kB, 0, m->s>>>(st, m->cnt, rank.p);
  int total = 0;
  if (all_live) {
    if (4 * (int64_t)st.T > INT32_MAX) return fail3(m, PM_E_NOMEM, "adjacency pool beyond 2^31 entries");
    total = 4 * st.T;
    pm::scan_excl(m->cnt, m->off, V, m->ctr + K_TOTAL, m->partial, m->s);
  } else {
    T3(scan_total(m, m->cnt, m->off, V, &total));
  }
  int64_t want = total + (int64_t)(m->headroom * (double)total) + kTopStripes * 64;
  if (want > m->necap) {
    int64_t nc = std::max<int64_t>(want, m->necap + m->necap / 2);
    if (3 * nc > INT32_MAX) return fail3(m, PM_E_NOMEM, "adjacency pool beyond 2^31 entries");
    T3(dgrow(m, &st.ne, m->necap, nc, false));
    T3(dgrow(m, &st.nn, m->nncap, 3 * nc, false));
    m->necap = nc;
    m->nncap = 3 * nc;
  }
  // refinement marks NN entries of packed rows only
  if (3 * (int64_t)total + 3 > m->mcap) {
    int64_t nc = std::max<int64_t>(3 * (int64_t)total + 3, m->mcap + m->mcap / 2);
    T3(dgrow(m, &m->mark, m->mcap, nc, false));
    m->mcap = nc;
  }
  if (!m->tops) T3(dgrow(m, &m->tops, 0, kTopStripes * kTopStride, false));
  k_ne_fill<<<grid(st.T), kB, 0, m->s>>>(st, m->off, rank.p);
  k_rows_finish<<<grid((int64_t)V * kWave), kB, 0, m->s>>>(st, m->off, m->cnt);
  m->top_base = total;
  m->top_per = (m->necap - total) / kTopStripes;
  k_tops_init<<<1, kTopStripes, 0, m->s>>>(m->tops, m->top_base, m->top_per, m->ctr);
  H3(hipGetLastError());
  m->rows_ok = true;
  return PM_OK;
}
// Before a call reads rows: after a build that found no memory they are not those
// of the element list; built now, or the call fails too.
pm_status rows_ready(pm3_mesh* m) { return m->rows_ok ? PM_OK : build_rows(m, false); }

// list of the vertices selected by mode, in m->A; returns its length
pm_status select_list(pm3_mesh* m, int mode, double L_low2, int* n) {
  k_select<<<grid(m->st.V), kB, 0, m->s>>>(m->st, mode, L_low2, m->nxt, m->A, m->col, m->act, m->blk, m->ctr);
  T3(read_ctr(m));
  *n = m->hctr[K_LIST];
  return PM_OK;
}

// A list of at most kSolve vertices coloured and cut into classes (n_dev: its
// length from the device; n is then the most it can be)
pm_status solve_list(pm3_mesh* m, const int* A, int n, const int* n_dev, uint64_t sseed, bool whole) {
  int* cnt = m->ctr + K_CLASS;
  k_pred<<<grid(8 * (int64_t)n), kB, 0, m->s>>>(m->st, A, n, n_dev, m->act, m->col, m->blk, sseed, m->recs);
  k_solve<<<1, kSolveThreads, 0, m->s>>>(m->st, A, n, n_dev, m->recs, m->act, m->col, sseed, m->ctr, cnt,
                                       cnt + kMaxColours, whole ? m->cls : nullptr);
  H3(hipGetLastError());
  return PM_OK;
}

// Jones-Plassmann colouring of the list A[0, n); col holds the colours
// (-1 elsewhere); returns the colour count. A short list comes with its class
// lists (*listed: m->cls, and the sizes in the counters' mirror). clean: no
// vertex has a colour or is active, the colouring's counts are zero
pm_status colour_list(pm3_mesh* m, int n, uint32_t ctx, bool clean, int* ncol, bool* listed) {
  Store3& st = m->st;
  uint64_t sseed = stream_seed(m->seed, ctx);
  *listed = false;
  *ncol = 0;
  if (!m->recs) T3(dgrow(m, &m->recs, 0, kSolve, false));
  if (!clean) k_colour_start<<<grid(st.V), kB, 0, m->s>>>(m->col, m->act, st.V, m->ctr);
  if (n == 0) return PM_OK;
  int done = 0;
  if (!clean) k_place<<<grid(n), kB, 0, m->s>>>(m->A, n, m->act, m->blk);
  if (n <= kSolve) {
    T3(solve_list(m, m->A, n, nullptr, sseed, true));
    T3(read_ctr(m, kMaxColours));
    *listed = true;
    done = m->hctr[K_COLOURED];
  } else {
    if (n > m->lcap) {
      T3(dgrow(m, &m->recl, m->lcap, m->Vcap, false));
      m->lcap = m->Vcap;
    }
    k_pred<<<grid(8 * (int64_t)n), kB, 0, m->s>>>(st, m->A, n, nullptr, m->act, m->col, m->blk, sseed, m->recl);
  }
  // iterations in batches of kJpBatch between read-backs, until few enough
  // vertices wait for the one-block end
  constexpr int kJpBatch = 4;
  for (int it = 0; done < n;) {
    if (*listed || it > n + 8) return fail3(m, PM_E_DEVICE, "colouring made no progress");
    for (int b = 0; b < kJpBatch; ++b, ++it)
      k_follow<<<grid(n), kB, 0, m->s>>>(st, m->A, n, m->act, m->col, sseed, m->recl, m->ctr);
    H3(hipGetLastError());
    T3(read_ctr(m));
    if (m->hctr[K_ERR] & E_COLOURS) return fail3(m, PM_E_DEVICE, "more than 256 colours");
    done = m->hctr[K_COLOURED];
    if (done < n && n - done <= kSolve) {
      k_waiting<<<grid(n), kB, 0, m->s>>>(m->A, n, m->col, m->cls, m->blk, m->ctr);
      T3(solve_list(m, m->cls, n - done, nullptr, sseed, false));
      T3(read_ctr(m));
      done = m->hctr[K_COLOURED];
      if (done < n) return fail3(m, PM_E_DEVICE, "colouring made no progress");
    }
  }
  if (m->hctr[K_ERR] & E_COLOURS) return fail3(m, PM_E_DEVICE, "more than 256 colours");
  *ncol = m->hctr[K_NCOL];
  return PM_OK;
}

// class lists of the coloured list: m->cls, offsets and sizes on the host
pm_status class_lists(pm3_mesh* m, int n, int ncol, bool listed, std::vector<int>& off, std::vector<int>& size) {
  // sizes, offsets and placement on the device; one read-back of the sizes
  // (the host computes the same offsets from them)
  int *cnt = m->ctr + K_CLASS, *place = cnt + kMaxColours, *coff = place + kMaxColours;
  if (!listed && n > 0) {
    k_fill_int<<<1, 2 * kMaxColours, 0, m->s>>>(cnt, 2 * kMaxColours, 0);
    k_class_count<<<grid(n), kB, 0, m->s>>>(m->A, n, m->col, ncol, cnt);
    k_class_offsets<<<1, kMaxColours, 0, m->s>>>(cnt, ncol, coff);
    k_class_place<<<std::max(1, (n + kB - 1) / kB), kB, 0, m->s>>>(m->A, n, m->col, ncol, coff, place, m->cls);
    H3(hipGetLastError());
    T3(read_ctr(m, kMaxColours));
  }
  size.assign(ncol, 0);
  off.assign(ncol + 1, 0);
  for (int c = 0; c < ncol; ++c) {
    size[c] = m->hctr[K_COUNT + c];
    off[c + 1] = off[c] + size[c];
  }
  return PM_OK;
}

pm_status compact(pm3_mesh* m) {
  Store3& st = m->st;
  int V = st.V, T = st.T;
  int nv = 0, nt = 0;
  k_live<<<grid(std::max(V, T)), kB, 0, m->s>>>(st, m->flag, m->tcnt);
  T3(scan_both(m, m->flag, m->scan, V, &nv, m->tcnt, m->tscan, T, &nt));
  double4* xyz = nullptr;
  Met6* met = nullptr;
  uint8_t* tag = nullptr;
  int4* tet = nullptr;
  T3(dgrow(m, &xyz, 0, m->Vcap, false));
  T3(dgrow(m, &met, 0, m->Vcap, false));
  T3(dgrow(m, &tag, 0, m->Vcap, false));
  T3(dgrow(m, &tet, 0, m->Tcap, false));
  k_compact_v<<<grid(V), kB, 0, m->s>>>(st, m->scan, xyz, met, tag);
  k_compact_t<<<grid(T), kB, 0, m->s>>>(st, m->scan, m->tscan, tet);
  H3(hipGetLastError());
  dfree3(st.xyz);
  dfree3(st.met);
  dfree3(st.tag);
  dfree3(st.tet);
  st.xyz = xyz;
  st.met = met;
  st.tag = tag;
  st.tet = tet;
  st.V = nv;
  st.T = nt;
  k_all_live<<<grid(std::max(nv, nt)), kB, 0, m->s>>>(st, m->nxt);
  H3(hipGetLastError());
  return build_rows(m, true);
}

void put_stats(pm_stats* out, const int64_t* v) {
  if (!out) return;
  for (int i = 0; i < 16; ++i) out->v[i] = v[i];
}

}  // namespace

extern "C" {

pm_status pm3_mesh_create(const pm3_mesh_desc* d, const pm_options* o, void* stream, pm3_mesh** out) {
  if (!out) return PM_E_ARG;
  *out = nullptr;
  if (!d || !d->xyz || !d->tet || !d->metric) return PM_E_ARG;
  if (d->V < 4 || d->T < 1 || d->V > (1ll << 29) || d->T > (1ll << 29)) return PM_E_ARG;
  if (d->mem_kind != PM_MEM_HOST && d->mem_kind != PM_MEM_DEVICE) return PM_E_ARG;
  pm_options def;
  if (!o) {
    pm_default_options(&def);
    o = &def;
  }
  pm3_mesh* m = new (std::nothrow) pm3_mesh();
  if (!m) return PM_E_NOMEM;
  m->s = (hipStream_t)stream;
  m->seed = o->seed;
  if (!(o->pool_headroom == 0.0 || (o->pool_headroom >= 1.0 && o->pool_headroom <= 64.0))) {
    delete m;
    g3_create_err = "pool_headroom: 0 (the default) or within [1, 64]";
    return PM_E_ARG;
  }
  m->headroom = o->pool_headroom > 0.0 ? o->pool_headroom : 3.0;
  auto bail = [&](pm_status s) {
    g3_create_err = m->err.empty() ? std::string("pm3_mesh_create failed") : m->err;
    pm3_mesh_destroy(m);
    return s;
  };
  int V = (int)d->V, T = (int)d->T;
  if (pm::block_alloc(m->s, (void**)&m->ctr, sizeof(int) * K_ALL) != hipSuccess ||
      !(m->hctr = (int*)pm::pinned_take())) {
    (void)hipGetLastError();
    return bail(PM_E_NOMEM);
  }
  m->mail = pm::mail_of(m->hctr);
  if (reserve(m, V, T) != PM_OK) return bail(PM_E_NOMEM);
  Store3& st = m->st;
  st.V = V;
  st.T = T;
  double *xyz = nullptr, *met = nullptr;
  int* tet = nullptr;
  uint8_t* tags = nullptr;
  hipMemcpyKind kind = d->mem_kind == PM_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
  if (dgrow(m, &xyz, 0, 3 * (int64_t)V, false) != PM_OK || dgrow(m, &met, 0, 6 * (int64_t)V, false) != PM_OK ||
      dgrow(m, &tet, 0, 4 * (int64_t)T, false) != PM_OK)
    return bail(PM_E_NOMEM);
  bool ok = hipMemcpyAsync(xyz, d->xyz, sizeof(double) * 3 * V, kind, m->s) == hipSuccess &&
            hipMemcpyAsync(met, d->metric, sizeof(double) * 6 * V, kind, m->s) == hipSuccess &&
            hipMemcpyAsync(tet, d->tet, sizeof(int) * 4 * T, kind, m->s) == hipSuccess;
  if (ok && d->tags) ok = hipMemcpyAsync(st.tag, d->tags, (size_t)V, kind, m->s) == hipSuccess;
  if (!ok) return bail(PM_E_DEVICE);
  if (zero_ctr(m) != PM_OK) return bail(PM_E_DEVICE);
  k_in<<<grid(std::max(V, T)), kB, 0, m->s>>>(xyz, tet, met, st, m->ctr);
  if (!d->tags) k_tags<<<grid(V), kB, 0, m->s>>>(st);
  k_orient<<<grid(T), kB, 0, m->s>>>(st, m->ctr);
  if (read_ctr(m) != PM_OK) return bail(PM_E_DEVICE);
  dfree3(xyz);
  dfree3(met);
  dfree3(tet);
  if (m->hctr[K_ERR]) {
    m->err = "invalid mesh: ids, orientation or metric";
    return bail(PM_E_MESH);
  }
  k_fill_u8<<<grid(V), kB, 0, m->s>>>(m->nxt, V, 0);
  if (build_rows(m, true) != PM_OK) return bail(PM_E_DEVICE);
  if (hipStreamSynchronize(m->s) != hipSuccess) return bail(PM_E_DEVICE);
  *out = m;
  return PM_OK;
}

pm_status pm3_mesh_destroy(pm3_mesh* m) {
  if (!m) return PM_OK;
  (void)hipStreamSynchronize(m->s);
  Store3& st = m->st;
  dfree3(st.xyz);
  dfree3(st.met);
  dfree3(st.tag);
  dfree3(st.valive);
  dfree3(st.tet);
  dfree3(st.talive);
  dfree3(st.hdr);
  dfree3(st.nn);
  dfree3(st.ne);
  for (int** p : {&m->cnt, &m->off, &m->flag, &m->scan, &m->partial, &m->A, &m->B, &m->cls, &m->col,
                  &m->blk, &m->mark, &m->tcnt, &m->tscan, &m->ctr})
    dfree3(*p);
  dfree3(m->recs);
  dfree3(m->recl);
  dfree3(m->act);
  dfree3(m->nxt);
  dfree3(m->qbuf);
  dfree3(st.cap);
  dfree3(m->own);
  dfree3(m->rows);
  dfree3(m->rec);
  dfree3(m->tops);
  pm::pinned_give(m->hctr);
  delete m;
  return PM_OK;
}

pm_status pm3_mesh_sizes(const pm3_mesh* m, int64_t* V, int64_t* T) {
  if (!m) return PM_E_ARG;
  if (V) *V = m->st.V;
  if (T) *T = m->st.T;
  return PM_OK;
}

pm_status pm3_mesh_export(pm3_mesh* m, double* xyz, int32_t* tet, double* metric, uint8_t* tags, uint8_t* valive,
                          uint8_t* talive, int32_t mem_kind) {
  if (!m) return PM_E_ARG;
  if (mem_kind != PM_MEM_HOST && mem_kind != PM_MEM_DEVICE) return fail3(m, PM_E_ARG, "bad mem_kind");
  Store3& st = m->st;
  int V = st.V, T = st.T;
  bool host = mem_kind == PM_MEM_HOST;
  double *dx = nullptr, *dm = nullptr;
  int* dt = nullptr;
  if (host) {
    if (xyz) T3(dgrow(m, &dx, 0, 3 * (int64_t)V, false));
    if (metric) T3(dgrow(m, &dm, 0, 6 * (int64_t)V, false));
    if (tet) T3(dgrow(m, &dt, 0, 4 * (int64_t)T, false));
  } else {
    dx = xyz;
    dm = metric;
    dt = tet;
  }
  k_export<<<grid(std::max(V, T)), kB, 0, m->s>>>(st, dx, dt, dm);
  H3(hipGetLastError());
  hipMemcpyKind k = host ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
  if (host) {
    if (xyz) H3(hipMemcpyAsync(xyz, dx, sizeof(double) * 3 * V, k, m->s));
    if (metric) H3(hipMemcpyAsync(metric, dm, sizeof(double) * 6 * V, k, m->s));
    if (tet) H3(hipMemcpyAsync(tet, dt, sizeof(int) * 4 * T, k, m->s));
  }
  if (tags) H3(hipMemcpyAsync(tags, st.tag, (size_t)V, k, m->s));
  if (valive) H3(hipMemcpyAsync(valive, st.valive, (size_t)V, k, m->s));
  if (talive) H3(hipMemcpyAsync(talive, st.talive, (size_t)T, k, m->s));
  H3(hipStreamSynchronize(m->s));
  if (host) {  // staging blocks (for device exports they are the caller's arrays)
    dfree3(dx);
    dfree3(dm);
    dfree3(dt);
  }
  return PM_OK;
}

pm_status pm3_mesh_rows(pm3_mesh* m, int64_t* nn_total, int64_t* ne_total, int64_t* nn_off, int32_t* nn,
                        int64_t* ne_off, int32_t* ne) {
  if (!m) return PM_E_ARG;
  T3(rows_ready(m));
  Store3& st = m->st;
  int V = st.V;
  std::vector<int4> hdr(V);
  H3(hipMemcpyAsync(hdr.data(), st.hdr, sizeof(int4) * V, hipMemcpyDeviceToHost, m->s));
  H3(hipStreamSynchronize(m->s));
  int64_t a = 0, b = 0;
  for (int v = 0; v < V; ++v) {
    a += hdr[v].y;
    b += hdr[v].w;
  }
  if (nn_total) *nn_total = a;
  if (ne_total) *ne_total = b;
  if (!nn_off || !nn || !ne_off || !ne) return PM_OK;
  std::vector<int> hnn(m->nncap > 0 ? (size_t)std::min<int64_t>(m->nncap, 3 * b + 3) : 1),
      hne((size_t)std::max<int64_t>(b, 1));
  if (b > 0) {
    H3(hipMemcpyAsync(hnn.data(), st.nn, sizeof(int) * (size_t)(3 * b), hipMemcpyDeviceToHost, m->s));
    H3(hipMemcpyAsync(hne.data(), st.ne, sizeof(int) * (size_t)b, hipMemcpyDeviceToHost, m->s));
    H3(hipStreamSynchronize(m->s));
  }
  int64_t pa = 0, pb = 0;
  for (int v = 0; v < V; ++v) {
    nn_off[v] = pa;
    ne_off[v] = pb;
    for (int j = 0; j < hdr[v].y; ++j) nn[pa++] = hnn[hdr[v].x + j];
    for (int j = 0; j < hdr[v].w; ++j) ne[pb++] = hne[hdr[v].z + j];
  }
  nn_off[V] = pa;
  ne_off[V] = pb;
  return PM_OK;
}

pm_status pm3_colour(pm3_mesh* m, const uint8_t* active, uint32_t ctx, int32_t* colour_out, int32_t* ncolours) {
  if (!m) return PM_E_ARG;
  T3(rows_ready(m));
  Store3& st = m->st;
  int n = 0;
  if (active) {
    std::vector<int> f(st.V);
    std::vector<uint8_t> va(st.V);
    H3(hipMemcpyAsync(va.data(), st.valive, (size_t)st.V, hipMemcpyDeviceToHost, m->s));
    H3(hipStreamSynchronize(m->s));
    for (int v = 0; v < st.V; ++v) f[v] = (active[v] && va[v]) ? 1 : 0;
    H3(hipMemcpyAsync(m->flag, f.data(), sizeof(int) * st.V, hipMemcpyHostToDevice, m->s));
    int total = 0;
    T3(scan_total(m, m->flag, m->scan, st.V, &total));
    k_compact_list<<<grid(st.V), kB, 0, m->s>>>(m->flag, m->scan, st.V, m->A);
    n = total;
  } else {
    k_flags<<<grid(st.V), kB, 0, m->s>>>(st.valive, st.V, m->flag);
    int total = 0;
    T3(scan_total(m, m->flag, m->scan, st.V, &total));
    k_compact_list<<<grid(st.V), kB, 0, m->s>>>(m->flag, m->scan, st.V, m->A);
    n = total;
  }
  int ncol = 0;
  bool listed;
  T3(colour_list(m, n, ctx, false, &ncol, &listed));
  if (ncolours) *ncolours = ncol;
  if (colour_out) {
    H3(hipMemcpyAsync(colour_out, m->col, sizeof(int) * st.V, hipMemcpyDeviceToHost, m->s));
    H3(hipStreamSynchronize(m->s));
  }
  return PM_OK;
}

pm_status pm3_coarsen(pm3_mesh* m, const pm_options* o, pm_stats* out) {
  if (!m || !o) return PM_E_ARG;
  if (!(o->L_low2 > 0.0) || !(o->q_min >= 0.0) || o->coarsen_rounds < 0) return fail3(m, PM_E_ARG, "bad options");
  Store3& st = m->st;
  int64_t sv[16] = {};
  double qmin3 = (o->q_min * o->q_min) * o->q_min;
  int n = 0, ncol = 0;
  bool lists = false;
  T3(rows_ready(m));
  T3(zero_ctr(m));
  T3(select_list(m, 0, o->L_low2, &n));
  k_fill_u8<<<grid(st.V), kB, 0, m->s>>>(m->nxt, st.V, 0);
  int r = 0;
  auto ctx_of = [&](int round) { return make_ctx(o->sweep, PH3_COARSEN, round); };
  if (n > 0 && r < o->coarsen_rounds) T3(colour_list(m, n, ctx_of(0), false, &ncol, &lists));
  std::vector<int> off, size;
  while (n > 0 && r < o->coarsen_rounds) {
    uint64_t sseed = stream_seed(m->seed, ctx_of(r));
    sv[PM_S_COLOURED] += n;
    sv[PM_S_COLOURS] += ncol;
    T3(class_lists(m, n, ncol, lists, off, size));
    // The phase's stats accumulate on the device. Each class: the
    // collapses, then the commit of the rows they changed. A commit that runs
    // out of room makes the round's later classes stand down; the host then
    // rebuilds every row from the elements and runs those classes again.
    // The next list is selected, and coloured if one block takes it, before the
    // round's one read-back.
    std::vector<int> class_epoch(ncol, -1);
    int c0 = 0;
    for (;;) {
      for (int c = c0; c < ncol; ++c) {
        if (size[c] == 0) continue;
        int ep = ++m->epoch;
        class_epoch[c] = ep;
        // the row list while the class can stamp at most about an eighth of
        // the rows (a wavefront for about every row a member's neighbours
        // give, at most one grid's worth), else vertex order
        int64_t reach = (int64_t)size[c] * 16;
        bool listed = reach * 8 <= st.V;
        int nb = (int)(((int64_t)size[c] * kWave + kB - 1) / kB);
        k_collapse<<<nb, kB, 0, m->s>>>(st, m->cls + off[c], size[c], m->col, c, sseed, o->L_low2, qmin3,
                                         m->nxt, ep, m->own, listed ? m->rows : nullptr, m->rec, m->ctr);
        if (listed)
          k_commit3_list<<<grid(reach * kWave), kB, 0, m->s>>>(st, ep, m->rows, m->rec, m->tops, m->top_base,
                                                              m->top_per, m->ctr);
        else
          k_commit3<<<grid((int64_t)st.V * kWave), kB, 0, m->s>>>(st, ep, m->own, m->rec, m->tops, m->top_base,
                                                                   m->top_per, m->ctr);
        H3(hipGetLastError());
      }
      k_select<<<grid(st.V), kB, 0, m->s>>>(st, 1, o->L_low2, m->nxt, m->B, m->col, m->act, m->blk, m->ctr);
      if (r + 1 < o->coarsen_rounds) {
        const int* len = m->ctr + K_LIST;
        T3(solve_list(m, m->B, kSolve, len, stream_seed(m->seed, ctx_of(r + 1)), true));
      }
      T3(read_ctr(m, kMaxColours));
      if (m->hctr[K_ERR] & E_COLOURS) return fail3(m, PM_E_DEVICE, "more than 256 colours");
      if (!m->hctr[K_ROOM]) break;
      // (nothing was selected: the classes and their lists are as they were)
      int failed = -1;
      for (int c = 0; c < ncol; ++c)
        if (class_epoch[c] == m->hctr[K_ROOMEP]) failed = c;
      if (failed < c0) return fail3(m, PM_E_DEVICE, "row commit: room counter names no class of this round");
      T3(build_rows(m, false));
      ++sv[13];
      c0 = failed + 1;
      k_fill_int<<<1, kWave, 0, m->s>>>(m->ctr + K_CCOMMIT, 4, 0);
    }
    std::swap(m->A, m->B);
    n = m->hctr[K_LIST];
    ++r;
    lists = n <= kSolve;
    ncol = m->hctr[K_NCOL];
    sv[PM_S_EVALUATED] = m->hctr[K_EVAL];
    sv[PM_S_DEFERRED] = m->hctr[K_DEFER];
    sv[PM_S_COMMITTED] = m->hctr[K_COMMIT];
    if (lists && r < o->coarsen_rounds && m->hctr[K_COLOURED] != n)
      return fail3(m, PM_E_DEVICE, "colouring made no progress");
    if (!lists && r < o->coarsen_rounds) T3(colour_list(m, n, ctx_of(r), true, &ncol, &lists));
  }
  sv[PM_S_ROUNDS] = r;
  sv[PM_S_CONVERGED] = n == 0 ? 1 : 0;
  T3(compact(m));
  H3(hipStreamSynchronize(m->s));
  put_stats(out, sv);
  return n == 0 ? PM_OK : PM_W_NOT_CONVERGED;
}

pm_status pm3_refine(pm3_mesh* m, const pm_options* o, pm_stats* out) {
  if (!m || !o) return PM_E_ARG;
  if (!(o->L_up2 > 0.0) || o->refine_passes < 0) return fail3(m, PM_E_ARG, "bad options");
  Store3& st = m->st;
  int64_t sv[16] = {};
  int p = 0;
  bool done = false;
  T3(rows_ready(m));
  for (; p < o->refine_passes; ++p) {
    int V0 = st.V, T0 = st.T;
    T3(zero_ctr(m));
    k_mark<<<grid(kVL * (int64_t)V0), kB, 0, m->s>>>(st, o->L_up2, m->mark, m->cnt, m->ctr);
    k_split_count<<<std::max(1, (T0 + kSplitThreads - 1) / kSplitThreads), kSplitThreads, 0, m->s>>>(st, T0, o->L_up2, m->tcnt, m->ctr);
    int nv = 0, nt = 0;
    T3(scan_both(m, m->cnt, m->scan, V0, &nv, m->tcnt, m->tscan, T0, &nt));
    sv[PM_S_EDGES] += m->hctr[K_EDGES];
    if (nv == 0) {
      done = true;
      break;
    }
    if (m->hctr[K_ERR] & E_LEAVES) return fail3(m, PM_E_DEVICE, "an element split into too many pieces");
    T3(reserve(m, V0 + nv, T0 + nt));
    k_mint<<<grid(kVL * (int64_t)V0), kB, 0, m->s>>>(st, V0, m->scan, m->mark);
    st.V = V0 + nv;
    k_split_write<<<std::max(1, (T0 + kSplitThreads - 1) / kSplitThreads), kSplitThreads, 0, m->s>>>(st, T0, o->L_up2, m->mark, m->tscan);
    st.T = T0 + nt;
    H3(hipGetLastError());
    sv[PM_S_NEWV] += nv;
    sv[PM_S_NEWT] += nt;
    sv[PM_S_COMMITTED] += nv;
    T3(build_rows(m, true));
  }
  H3(hipStreamSynchronize(m->s));
  sv[PM_S_ROUNDS] = p;
  sv[PM_S_CONVERGED] = done ? 1 : 0;
  put_stats(out, sv);
  return done ? PM_OK : PM_W_NOT_CONVERGED;
}

pm_status pm3_smooth(pm3_mesh* m, const pm_options* o, pm_stats* out) {
  if (!m || !o) return PM_E_ARG;
  if (o->smooth_sweeps < 0) return fail3(m, PM_E_ARG, "bad options");
  Store3& st = m->st;
  int64_t sv[16] = {};
  int n = 0;
  T3(rows_ready(m));
  T3(select_list(m, 2, 0.0, &n));
  int ncol = 0;
  bool lists;
  T3(colour_list(m, n, make_ctx(o->sweep, PH3_SMOOTH, 0), false, &ncol, &lists));
  sv[PM_S_COLOURED] += n;
  sv[PM_S_COLOURS] += ncol;
  std::vector<int> off, size;
  T3(class_lists(m, n, ncol, lists, off, size));
  T3(zero_ctr(m));
  for (int s = 0; s < o->smooth_sweeps; ++s)
    for (int c = 0; c < ncol; ++c)
      if (size[c] > 0) k_smooth<<<grid((int64_t)size[c] * kWave), kB, 0, m->s>>>(st, m->cls + off[c], size[c], m->ctr);
  H3(hipGetLastError());
  T3(read_ctr(m));
  sv[PM_S_EVALUATED] = m->hctr[K_EVAL];
  sv[PM_S_COMMITTED] = m->hctr[K_COMMIT];
  sv[PM_S_ROUNDS] = o->smooth_sweeps;
  sv[PM_S_CONVERGED] = 1;
  put_stats(out, sv);
  return PM_OK;
}

pm_status pm3_quality(pm3_mesh* m, double* Q, double* qmin) {
  if (!m) return PM_E_ARG;
  constexpr int NB = 1024;
  if (!m->qbuf) T3(dgrow(m, &m->qbuf, 0, 2 * NB, false));
  k_quality<<<NB, QB, 0, m->s>>>(m->st, m->qbuf, m->qbuf + NB);
  double* h = (double*)(m->hctr + 1024);  // in the pinned block, past the counters and class sizes
  static_assert(K_COUNT + kMaxColours <= 1024, "the counters' mirror");
  pm::mail_next(m->mail);
  k_quality_final<<<1, QB, 0, m->s>>>(m->qbuf, m->qbuf + NB, NB, h, (int*)m->mail.at, m->mail.no);
  H3(hipGetLastError());
  H3(pm::mail_wait(m->mail, m->s));
  if (Q) *Q = h[0];
  if (qmin) *qmin = h[1];
  return PM_OK;
}

const char* pm3_last_error(const pm3_mesh* m) { return m ? m->err.c_str() : g3_create_err.c_str(); }

}  // extern "C"
