// Ordered exclusive scans in two launches. The first visits every index once,
// with whatever the caller computes there, and leaves a sum per chunk; in the
// second every work-group adds up the sums before its own range, scans the range
// and hands each index its value and the sum before it. What produces the values
// and what uses the positions thus needs no launches and passes of its own: a
// launch costs some 5 us however small it is, and the selection of a round took
// five of them (flags, three of the scan, scatter), a row build eight of its
// twelve: these scans alone took the 257^2 Vasilevskii adaptation from 1922
// launches to 1535 (13.0 to 12.0 ms).
#pragma once
#include <algorithm>

#include "kern.hpp"

namespace pm {

__device__ __forceinline__ int sum_of(int a, int b) { return a + b; }
__device__ __forceinline__ int2 sum_of(int2 a, int2 b) { return make_int2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ int diff_of(int a, int b) { return a - b; }
__device__ __forceinline__ int2 diff_of(int2 a, int2 b) { return make_int2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ int lane_up(int a, int d) { return __shfl_up(a, d); }
__device__ __forceinline__ int2 lane_up(int2 a, int d) { return make_int2(__shfl_up(a.x, d), __shfl_up(a.y, d)); }

// exclusive scan over the work-group; returns the thread's prefix, sets tot
template <class T>
__device__ __forceinline__ T block_excl(T v, T* lds, T& tot) {
  int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave, nw = blockDim.x / kWave;
  T incl = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T o = lane_up(incl, d);
    if (lane >= d) incl = sum_of(incl, o);
  }
  if (lane == kWave - 1) lds[wid] = incl;
  __syncthreads();
  T before{};
  tot = T{};
  for (int w = 0; w < nw; ++w) {
    if (w == wid) before = tot;
    tot = sum_of(tot, lds[w]);
  }
  __syncthreads();
  return sum_of(before, diff_of(incl, v));
}

constexpr int kScanOut = 8 * kBlock;       // indices a work-group of the second launch takes
constexpr int kScanMany = 8192;            // sums that the second launch's work-groups add up by themselves
constexpr int kScanFine = 1 << 21;         // indices from which on NI = 1 becomes 4

// f(i, i < n) is called once for every i < n, by full wavefronts
template <class T, int NI, class F>
__device__ __forceinline__ void scan_sums(F f, int n, T* part, int chunk) {
  __shared__ T lds[kBlock / kWave];
  T s{};
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    int64_t i = ((int64_t)chunk * NI + k) * kBlock + threadIdx.x;
    T x = f((int)(i < n ? i : 0), i < n);
    if (i < n) s = sum_of(s, x);
  }
  T tot;
  block_excl(s, lds, tot);
  if (threadIdx.x == 0) part[chunk] = tot;
}
template <class T, int NI, class F>
__global__ void __launch_bounds__(kBlock) k_scan_sums(F f, int n, T* part) {
  scan_sums<T, NI>(f, n, part, xcd_block());
}
// two arrays side by side, the second's sums behind the first's nf
template <class T, int NI, class F, class G>
__global__ void __launch_bounds__(kBlock) k_scan_sums2(F f, int n, int nf, G g, int m, T* part) {
  int b = (int)blockIdx.x;
  if (b < nf) scan_sums<T, NI>(f, n, part, b);
  else scan_sums<T, NI>(g, m, part + nf, b - nf);
}

// the sums themselves, where they are many
template <class T>
__global__ void __launch_bounds__(1024) k_scan_many(T* part, int nb) {
  __shared__ T lds[1024 / kWave];
  int per = (nb + 1023) / 1024, lo = min(nb, (int)threadIdx.x * per), hi = min(nb, lo + per);
  T s{}, tot;
  for (int i = lo; i < hi; ++i) s = sum_of(s, part[i]);
  T acc = block_excl(s, lds, tot);
  for (int i = lo; i < hi; ++i) {
    T t = part[i];
    part[i] = acc;
    acc = sum_of(acc, t);
  }
}

// in(i): the value; out(i, sum before, value); total(sum of all)
template <class T, class I, class O, class S>
__device__ __forceinline__ void scan_out(I in, O out, S total, int n, const T* part, int per, bool many, int b,
                                         bool last) {
  __shared__ T lds[kBlock / kWave];
  int tid = (int)threadIdx.x;
  int64_t i0 = (int64_t)b * kScanOut + (int64_t)tid * 8;
  T v[8], s{};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v[k] = i0 + k < n ? in((int)(i0 + k)) : T{};
    s = sum_of(s, v[k]);
  }
  T before{};
  if (many) {
    before = part[(int64_t)b * per];
  } else {
    T x{};
    for (int k = tid; k < b * per; k += kBlock) x = sum_of(x, part[k]);
    block_excl(x, lds, before);
  }
  T tot;
  T acc = sum_of(before, block_excl(s, lds, tot));
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (i0 + k < n) out((int)(i0 + k), acc, v[k]);
    acc = sum_of(acc, v[k]);
  }
  if (last && tid == 0) total(sum_of(before, tot));
}
template <class T, class I, class O, class S>
__global__ void __launch_bounds__(kBlock) k_scan_out(I in, O out, S total, int n, const T* part, int per, bool many) {
  scan_out(in, out, total, n, part, per, many, (int)blockIdx.x, blockIdx.x == gridDim.x - 1);
}
template <class T, class I, class O, class S, class I2, class O2, class S2>
__global__ void __launch_bounds__(kBlock) k_scan_out2(I in, O out, S total, int n, int nf, int nbn, I2 in2, O2 out2,
                                                    S2 total2, int m, const T* part, int per, bool many) {
  int b = (int)blockIdx.x;
  if (b < nbn) scan_out(in, out, total, n, part, per, many, b, b == nbn - 1);
  else scan_out(in2, out2, total2, m, part + nf, per, many, b - nbn, b == (int)gridDim.x - 1);
}

inline int scan_blocks(int n, int chunk) { return std::max(1, (int)(((int64_t)n + chunk - 1) / chunk)); }

// NI: indices a thread takes in the first launch, 8 where f is a load or two. 1
// asks for as many wavefronts as there are (f follows a row); beyond kScanFine
// indices it becomes 4, which leaves the second launch few enough sums (with 4 for
// a million indices already, three sweeps of the 1025^2 mesh went from 7.98 to
// 8.33 ms against 8.06 and 8.29 before).
template <class T, int NI, class F, class I, class O, class S>
void scan_fused(F f, I in, O out, S total, int n, T* part, hipStream_t s) {
  if constexpr (NI == 1) {
    if (n > kScanFine) return scan_fused<T, 4>(f, in, out, total, n, part, s);
  }
  int nb = scan_blocks(n, NI * kBlock);
  bool many = nb > kScanMany;
  k_scan_sums<T, NI><<<nb, kBlock, 0, s>>>(f, n, part);
  if (many) k_scan_many<<<1, 1024, 0, s>>>(part, nb);
  k_scan_out<<<scan_blocks(n, kScanOut), kBlock, 0, s>>>(in, out, total, n, part, 8 / NI, many);
}
// two arrays of one kind at once, in the launches of one
template <class T, int NI, class F, class I, class O, class S, class F2, class I2, class O2, class S2>
void scan_fused2(F f, I in, O out, S total, int n, F2 f2, I2 in2, O2 out2, S2 total2, int m, T* part, hipStream_t s) {
  if constexpr (NI == 1) {
    if (std::max(n, m) > kScanFine) return scan_fused2<T, 4>(f, in, out, total, n, f2, in2, out2, total2, m, part, s);
  }
  int nf = scan_blocks(n, NI * kBlock), ng = scan_blocks(m, NI * kBlock);
  bool many = std::max(nf, ng) > kScanMany;
  k_scan_sums2<T, NI><<<nf + ng, kBlock, 0, s>>>(f, n, nf, f2, m, part);
  if (many) {
    k_scan_many<<<1, 1024, 0, s>>>(part, nf);
    k_scan_many<<<1, 1024, 0, s>>>(part + nf, ng);
  }
  int nbn = scan_blocks(n, kScanOut);
  k_scan_out2<<<nbn + scan_blocks(m, kScanOut), kBlock, 0, s>>>(in, out, total, n, nf, nbn, in2, out2, total2, m, part,
                                                               8 / NI, many);
}

}  // namespace pm
