// The part of an append that follows the nearest-cluster search (Algorithm 1, decode block; UpdateVar of
// Section 4.2), by one wavefront with no workgroup barrier: shared by the stand-alone append kernel, the
// retrieval kernel that finds the nearest cluster during its own pass over the centroid table, and the extension.
// Lane l owns the coordinates 2 l and 2 l + 1.  Bound by latency: the cluster's record and centroid are one trip to memory
// (everything else was requested when the kernel began), the rest a chain of float64 arithmetic.  (By a workgroup, with a
// barrier and a trip to LDS or memory per step, an append took 13 500 cycles of a unit, 5.6 us of a step; by one wavefront about 5000 cycles.)
#pragma once
#include "common.hpp"

namespace dynakv {

// The bits of a key's and a value's coordinates 2 lane and 2 lane + 1 (16-bit types: one word).
struct EntryBits {
  uint2 k, v;
};
template <int DT>
__device__ __forceinline__ void store_pair(void* row, int lane, uint2 x) {
  if constexpr (DT == DYNAKV_F32) ((uint2*)row)[lane] = x;
  else ((uint32_t*)row)[lane] = x.x;
}
template <int DT>
__device__ __forceinline__ float2 pair_value(uint2 x) {
  if constexpr (DT == DYNAKV_F32) return float2{__uint_as_float(x.x), __uint_as_float(x.y)};
  else return float2{bits_value(x.x & 0xFFFFu, DT), bits_value(x.x >> 16, DT)};
}
// The rows of tensors of a caller need not be aligned beyond their elements.
template <int DT>
__device__ __forceinline__ EntryBits load_entry(const void* kin, const void* vin, size_t row, int lane) {
  EntryBits e;
  if constexpr (DT == DYNAKV_F32) {
    const uint32_t* k = (const uint32_t*)kin + row * kHeadDim + 2 * lane;
    const uint32_t* x = (const uint32_t*)vin + row * kHeadDim + 2 * lane;
    e.k = uint2{k[0], k[1]}; e.v = uint2{x[0], x[1]};
  } else {
    const uint16_t* k = (const uint16_t*)kin + row * kHeadDim + 2 * lane;
    const uint16_t* x = (const uint16_t*)vin + row * kHeadDim + 2 * lane;
    e.k = uint2{(uint32_t)k[0] | ((uint32_t)k[1] << 16), 0}; e.v = uint2{(uint32_t)x[0] | ((uint32_t)x[1] << 16), 0};
  }
  return e;
}
// Coordinates 2 lane and 2 lane + 1 of centroid j: the float32 master and, for 16-bit storage, the search copy, whose bits are returned.
template <int DT>
__device__ __forceinline__ uint32_t store_centroid_pair(const View& v, int u, int j, int lane, float2 x) {
  // (the search copy rounds the float32 value: left to itself the compiler turns float64 -> float32 -> 16 bits into one rounding)
  asm("" : "+v"(x.x), "+v"(x.y));
  *(float2*)(unit_R(v, u) + r_index(j, 2 * lane)) = x;
  if constexpr (DT == DYNAKV_F32) return 0;
  const uint32_t w = (uint32_t)round_bits16(x.x, DT) | ((uint32_t)round_bits16(x.y, DT) << 16);
  *(uint32_t*)(unit_Rq(v, u) + rq_index(j, 2 * lane)) = w;
  return w;
}

__device__ __forceinline__ double readlane_f64(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}
// Sum of a float64 over the 64 lanes (DPP butterfly inside the rows, row broadcasts across them); every lane gets it.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xF, false);
  return __hiloint2double(hi, lo);           // a lane that the step does not reach gets +0.0
}
__device__ __forceinline__ double wave_sum_f64(double x) {
  x += dpp_f64<kDppXor1, 0xF>(x);
  x += dpp_f64<kDppXor2, 0xF>(x);
  x += dpp_f64<kDppHalfMirror, 0xF>(x);
  x += dpp_f64<kDppMirror, 0xF>(x);
  x += dpp_f64<kDppBcast15, 0xA>(x);
  x += dpp_f64<kDppBcast31, 0xC>(x);
  return readlane_f64(x, 63);
}
// 1 / n for a count n, and x / n from it, rounded as a division rounds: the remainder of the first quotient, exact in one fused
// multiply-add, corrects it (Markstein).  Three instructions instead of the thirty of a float64 division.
struct CountInverse {
  double n, r;
};
__device__ __forceinline__ CountInverse count_inverse(int n) {
  CountInverse c{(double)n, 0.0};
  c.r = __builtin_amdgcn_rcp(c.n);
  c.r = fma(fma(-c.n, c.r, 1.0), c.r, c.r);
  c.r = fma(fma(-c.n, c.r, 1.0), c.r, c.r);
  return c;
}
__device__ __forceinline__ double over_count(double x, const CountInverse& c) {
  const double q = x * c.r;
  const double d = fma(fma(-c.n, q, x), c.r, q);
  return fabs(q) < __builtin_inf() ? d : q;      // (an infinity has no remainder)
}

// The unit's counters before an append; requested as early as possible.
struct UnitState {
  int M, N, nflag, top, bump;
  double tau;
};
__device__ __forceinline__ UnitState load_unit(const View& v, int u) {
  return UnitState{v.M[u], v.N[u], v.nflag[u], v.free_top[u], v.bump[u], v.tau[u]};
}
// A cluster as an append finds it: lane l its coordinates 2 l and 2 l + 1, the rest the same in every lane.  free_page: the top
// of the unit's stack of free pages.
struct ClusterState {
  float2 r;
  int cn, cb, ctail, cflag, free_page;
  double m2;
};
// One load: lanes 0 .. 6 fetch a word of the record each (see cluster_state).
struct ClusterFetch {
  float2 r;
  int w;
};
__device__ __forceinline__ ClusterFetch fetch_cluster(const View& v, int u, int j, int top, int lane) {
  const size_t cj = (size_t)u * v.Mcap + j;
  ClusterFetch f;
  const int* p = v.cn + cj;
  p = lane == 1 ? v.cb + cj : p;
  p = lane == 2 ? v.ctail + cj : p;
  p = lane == 3 ? v.cflag + cj : p;
  p = lane == 4 ? (const int*)(v.cM2 + cj) : p;
  p = lane == 5 ? (const int*)(v.cM2 + cj) + 1 : p;
  p = lane == 6 && top > 0 ? v.freelist + (size_t)u * v.Pcap + top - 1 : p;
  f.w = lane < 7 ? *p : 0;
  f.r = *(const float2*)(unit_R(v, u) + r_index(j, 2 * lane));
  return f;
}
__device__ __forceinline__ ClusterState cluster_state(const ClusterFetch& f, int top) {
  ClusterState c;
  c.r = f.r;
  c.cn = __builtin_amdgcn_readlane(f.w, 0); c.cb = __builtin_amdgcn_readlane(f.w, 1); c.ctail = __builtin_amdgcn_readlane(f.w, 2);
  c.cflag = __builtin_amdgcn_readlane(f.w, 3);
  c.m2 = __hiloint2double(__builtin_amdgcn_readlane(f.w, 5), __builtin_amdgcn_readlane(f.w, 4));
  c.free_page = top > 0 ? __builtin_amdgcn_readlane(f.w, 6) : -1;
  return c;
}

// What an append does to its cluster and its unit (the same in every lane).
struct AppendResult {
  int ok, commit, page, slot;      // carried out; the statistics were updated (else: buffered); the entry's place
  int nflag, top, bump;            // the unit's counters afterwards
  float2 r;                        // the centroid afterwards (lane l: coordinates 2 l, 2 l + 1)
  uint32_t rq;                     // and its search copy's bits (16-bit types)
  double m2;
};
// Cluster j receives entry s.N of unit u, by one wavefront.  Stores are left in flight.
template <int DT>
__device__ __forceinline__ AppendResult append_wave(const View& v, int u, int j, const UnitState& s, const ClusterState& c,
                                                    const EntryBits& e, int lane) {
  const size_t cj = (size_t)u * v.Mcap + j, up = (size_t)u * v.Pcap;
  AppendResult a{1, 0, c.ctail, 0, s.nflag, s.top, s.bump, c.r, 0, c.m2};
  // UpdateVar: delta_d = k_d - r_d, r'_d = r_d + delta_d / n', M2' = M2 + sum_d delta_d (k_d - r'_d)
  const int n1 = c.cn + 1, sz = c.cn + c.cb;
  const CountInverse inv = count_inverse(n1);
  const float2 kf = pair_value<DT>(e.k);
  const double k0 = (double)kf.x, k1 = (double)kf.y;
  const double d0 = k0 - (double)c.r.x, d1 = k1 - (double)c.r.y;
  const double r0 = (double)c.r.x + over_count(d0, inv), r1 = (double)c.r.y + over_count(d1, inv);
  const double M2 = c.m2 + wave_sum_f64(fma(d0, k0 - r0, d1 * (k1 - r1)));
  // the decisions, by every lane alike (all operands are wavefront-uniform); lane 0 writes
  a.slot = sz % kPageTokens;
  if (a.slot == 0) {                      // no page yet, or the tail page is full: from the free stack, else from the
    int np = -1;                          // untouched tail of the pool
    if (s.top > 0) { np = c.free_page; a.top = s.top - 1; }
    else if (s.bump < v.Pcap) { np = s.bump; a.bump = s.bump + 1; }
    if (np < 0) {
      a.ok = 0;
      if (lane == 0) v.err[u] |= DYNAKV_ERR_TOKENS;
      return a;
    }
    if (lane == 0) {
      v.free_top[u] = a.top; v.bump[u] = a.bump;
      v.pnext[up + np] = -1;
      if (sz != 0) v.pnext[up + a.page] = np;
      if (sz / kPageTokens < kInlinePages) v.cpg[cj * kInlinePages + sz / kPageTokens] = np;
      v.ctail[cj] = np;
    }
    a.page = np;
  }
  char* pg = page_ptr(v, u, a.page);
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
  store_pair<DT>(pg + (size_t)k_index(DT, a.slot, 0) * kEs, lane, e.k);
  store_pair<DT>(pg + (size_t)v_index(DT, a.slot, 0) * kEs, lane, e.v);
  bool trig = false;
  if (!c.cflag && n1 >= 2 && !v.static_update) {
    if (v.var_alpha > 0.f && over_count(M2, inv) > s.tau) trig = true;
    if (v.size_factor > 0.f && (double)n1 * (double)s.M > (double)v.size_factor * (double)(s.N + 1)) trig = true;
  }
  a.commit = !c.cflag && !trig;
  if (!c.cflag && trig) a.nflag = s.nflag + 1;
  if (a.commit) {
    a.r = float2{(float)r0, (float)r1};
    a.rq = store_centroid_pair<DT>(v, u, j, lane, a.r);
    a.m2 = M2;
  }
  if (lane == 0) {
    v.csz[cj] = sz + 1;
    if (a.commit) {
      v.cn[cj] = n1;
      v.cM2[cj] = M2;
    } else {                              // goes to the buffer of a flagged cluster (which this entry has flagged, if trig)
      v.cb[cj] = c.cb + 1;
      if (trig) { v.cflag[cj] = 1; v.flist[(size_t)u * v.Mcap + s.nflag] = j; v.nflag[u] = a.nflag; }
    }
    v.last_assign[u] = j;
    v.N[u] = s.N + 1;
    v.ppos[(up + a.page) * kPageTokens + a.slot] = s.N;
  }
  return a;
}
// Arg-min over (value, index) pairs, one per lane (index < 0: none); equal values go to the lowest index.  Every lane gets it.
template <int CTRL, int ROWS>
__device__ __forceinline__ double min_step(double x) {             // a lane that the step does not reach sees its own value
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(x), __double2loint(x), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(x), __double2hiint(x), CTRL, ROWS, 0xF, false);
  return fmin(x, __hiloint2double(hi, lo));
}
__device__ __forceinline__ void wave_argmin(double& val, int& idx) {
  double m = idx >= 0 ? val : __builtin_inf();
  m = min_step<kDppXor1, 0xF>(m);
  m = min_step<kDppXor2, 0xF>(m);
  m = min_step<kDppHalfMirror, 0xF>(m);
  m = min_step<kDppMirror, 0xF>(m);
  m = min_step<kDppBcast15, 0xA>(m);
  m = min_step<kDppBcast31, 0xC>(m);
  m = readlane_f64(m, 63);
  unsigned long long who = __ballot(idx >= 0 && val == m);
  if (who == 0) who = __ballot(idx >= 0);                          // (nothing but numbers that are none)
  const bool mine = (who >> (threadIdx.x & 63)) & 1ull;
  idx = who ? wave_min(mine ? idx : 0x7FFFFFFE) : -1;
  val = m;
}
// The same over a workgroup of NT threads.  NT / 64 <= 16 wavefronts; sv / si need 16 entries.  Every thread gets the winning index.
template <int NT>
__device__ inline int block_argmin(double val, int idx, double* sv, int* si) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  wave_argmin(val, idx);
  lds_barrier();
  if (lane == 0) { sv[w] = val; si[w] = idx; }
  lds_barrier();
  val = sv[0]; idx = si[0];
#pragma unroll
  for (int k = 1; k < NT / 64; ++k) {
    const double ov = sv[k];
    const int oi = si[k];
    if (oi >= 0 && (idx < 0 || ov < val || (ov == val && oi < idx))) { val = ov; idx = oi; }
  }
  return idx;
}

}  // namespace dynakv
