// Cluster splitting of a decode step (Algorithm 1, decode block; Section 4.2): shared by the stand-alone split
// kernel and by the kernel that runs a whole decode step per unit.
#pragma once
#include <type_traits>

#include "score.hpp"

namespace dynakv {

namespace {

// ------------------------------------------------------------------------------------------- split
constexpr int kStageRow16 = kHeadDim + 8, kStageRow32 = kHeadDim + 4;      // staged keys: rows padded over the banks

struct SplitSmem {
  int chain[kMaxSplitMembers / kPageTokens];      // pages of the cluster being split
  int newpg[kMaxSplitMembers / kPageTokens + 2];  // pages of the two children
  unsigned char side[kMaxSplitMembers];
  unsigned short perm[kMaxSplitMembers];           // members of the staying child in order, then of the moved one
  double cA[kHeadDim], cB[kHeadDim];
  alignas(16) float rA[kHeadDim], rB[kHeadDim];
  double tpart[4];                                 // per-wavefront parts of a sum over the coordinates, two rounds' worth
  double mu2[2];                                   // |mean of the members|^2, in two parts
  int nchg[2];                                     // members that changed side in a round (two rounds' worth)
  unsigned short chg[2][kMaxSplitMembers];         // who they are: member | what happens to the sums of side A << 12
  double sv[16];
  int si[16];
  int scan[64];
  int nchain;
  int did_split;                                   // thread 0 only: the last split_cluster call split its cluster
  int M, nflag, a_top, a_bump;                     // the unit's counters, held here for the whole kernel
  double m2[2];
};

// Access to the keys of the members in their pages, by member index: 8 consecutive coordinates at a time, or one.
template <int DT>
struct Keys {
  const char* pool; const int* chain;
  __device__ const char* row(int i) const {
    constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
    return pool + ((size_t)chain[i >> 4] * kPageElems + (size_t)(DT == DYNAKV_F32 ? k_index32(i & 15, 0) : k_index16(i & 15, 0))) * kEs;
  }
  __device__ void get8(int i, int d8, float (&x)[8]) const { load8(row(i), d8 * 8, DT, x); }
  __device__ float get(int i, int d) const { return load_elem(row(i), d, DT); }
};

constexpr int kSplitThreads = 256;

// Arg-max over (value, index) pairs held one per thread of the whole block; ties go to the lowest index; index < 0 means "no
// candidate".  Result in sv[0], si[0].
__device__ __forceinline__ void block_argmax(double val, int idx, double* sv, int* si) {
  const int j = block_argmin<kSplitThreads>(-val, idx, sv, si);
  __syncthreads();
  if (j == idx && j >= 0) { sv[0] = val; si[0] = j; }
  else if (j < 0 && threadIdx.x == 0) { sv[0] = -1.0; si[0] = -1; }
  __syncthreads();
}

// Squared distances of member i to one or two centres (C = double or float) in the fixed summation order.
// Called by the four lanes of a quad at once: lane q accumulates blocks 4q..4q+3 (coordinates 32q..32q+31),
// the block sums are then added left to right across the quad; every lane returns the totals.
template <class K, class C>
__device__ inline void quad_sqdist(const K& ks, int i, int q, const C* cA, const C* cB, double& dA, double& dB) {
  double sa[4], sb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    // every operand of the block is requested before the first use, so the LDS latency is paid once per block
    float x[8];
    C ca[8], cb[8];
    ks.get8(i, q * 4 + k, x);
#pragma unroll
    for (int e = 0; e < 8; ++e) { ca[e] = cA[(q * 4 + k) * 8 + e]; cb[e] = cB ? cB[(q * 4 + k) * 8 + e] : C(0); }
    asm volatile("" ::: "memory");
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double xd = (double)x[e];
      const double ta = xd - (double)ca[e];
      a = fma(ta, ta, a);
      if (cB) {
        const double tb = xd - (double)cb[e];
        b = fma(tb, tb, b);
      }
    }
    sa[k] = a; sb[k] = b;
  }
  dA = blocked16_quad(sa);
  dB = cB ? blocked16_quad(sb) : 0.0;
}

// Side of member i in a round of the 2-means: A (0) if |x - cA|^2 <= |x - cB|^2, which is <x, w> <= t with
// w = cB - cA and t = (|cB|^2 - |cA|^2) / 2 (ties to A).  Called by the four lanes of a quad at once (lane q takes
// coordinates 32 q .. 32 q + 31); every lane gets the side.  The inner product is first taken in float32 against wf
// (= w rounded to float32); only if it lies within eps of t, the bound on what float32 can have changed, it is
// retaken in float64 against wd.
template <class K>
__device__ inline unsigned char quad_side(const K& ks, int i, int q, const float* wf, const double* wd, double t, float eps) {
  float x[4][8];
#pragma unroll
  for (int k = 0; k < 4; ++k) ks.get8(i, q * 4 + k, x[k]);
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f4 a = *(const f4*)(wf + (q * 4 + k) * 8), b = *(const f4*)(wf + (q * 4 + k) * 8 + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { s = fmaf(x[k][e], a[e], s); s = fmaf(x[k][4 + e], b[e], s); }
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  const float tf = (float)t;
  if (fabsf(s - tf) > eps) return s <= tf ? 0 : 1;            // uniform over the quad
  double sd = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) sd = fma((double)x[k][e], wd[(q * 4 + k) * 8 + e], sd);
  sd += __shfl_xor(sd, 1);
  sd += __shfl_xor(sd, 2);
  return sd <= t ? 0 : 1;
}
// Bound for quad_side: float32 accumulation of 128 products (128 * 2^-24 |x| |w|, doubled for the rounding of w and
// of the products' partial sums across the quad) plus the rounding of t.  xmax >= every member's norm, wmax >= |w|.
__device__ inline float side_eps(float xmax, float wmax, double t) {
  return 1.53e-5f * xmax * wmax + 2.4e-7f * fabsf((float)t) + 1e-30f;
}

// Sum of key(r) over r = r0, r0 + step, .. < n: sixteen operands are requested at a time (clamped, so that the loads do not wait
// for a test); an out-of-range term adds +0.0.
template <class Key>
__device__ __forceinline__ double batched_sum(int r0, int n, int step, Key&& key) {
  double sum = 0.0;
#pragma unroll 1
  for (; r0 < n; r0 += 16 * step) {
    float x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = key(min(r0 + k * step, n - 1));
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += r0 + k * step < n ? (double)x[k] : 0.0;
  }
  return sum;
}

// Exact statistics of both children at once: members perm[0 .. nS) form cluster idS, perm[nS .. m) cluster idM
// (idM < 0: there is no second child).  Threads 0..127 own the coordinates of the first, 128..255 of the
// second.  float32 means go to rA / rB (LDS) and to the centroid table, M2 about those means to s.m2[].
template <class K>
__device__ __forceinline__ void children_stats(const View& v, int u, SplitSmem& s, const K& ks, int nS, int m, int idS, int idM) {
  const int tid = threadIdx.x, d = tid & (kHeadDim - 1), c = (tid >> 7) & 1;
  const int q0 = c ? nS : 0, q1 = c ? m : nS, id = c ? idM : idS;
  float* r = c ? s.rB : s.rA;
  const double sum = batched_sum(q0, q1, 1, [&](int q) { return ks.get(s.perm[q], d); });
  r[d] = q1 > q0 ? (float)(sum / (double)(q1 - q0)) : 0.f;
  if (id >= 0) store_centroid(v, u, id, d, r[d]);
  __syncthreads();
  double acc[2] = {0.0, 0.0};
#pragma unroll 1
  for (int base = 0; base < m; base += kSplitThreads / 4) {
    const int q = base + (tid >> 2), qc = min(q, m - 1);
    double da, db;
    quad_sqdist<K, float>(ks, s.perm[qc], tid & 3, qc < nS ? s.rA : s.rB, nullptr, da, db);
    if ((tid & 3) == 0 && q < m) acc[q >= nS] += da;
  }
  const double a = wave_sum_f64(acc[0]), b = wave_sum_f64(acc[1]);
  if ((tid & 63) == 0) { s.sv[tid >> 6] = a; s.sv[4 + (tid >> 6)] = b; }
  __syncthreads();
  if (tid < 2) s.m2[tid] = ((s.sv[4 * tid] + s.sv[4 * tid + 1]) + s.sv[4 * tid + 2]) + s.sv[4 * tid + 3];
  __syncthreads();
}

// Splits cluster j of unit u (2-means; Algorithm 1 SplitCluster).  Whole block; all branches uniform.  For what the wavefronts'
// path below cannot take: clusters beyond its staging rows, more than 64 flagged clusters, a unit near its capacity.
// The keys are read from their pages in every pass.
template <int DT>
__device__ __forceinline__ void split_cluster_impl(const View& v, int u, int j, int pos, int m, SplitSmem& s) {
  constexpr int NT = kSplitThreads;
  const int tid = threadIdx.x, grp = tid >> 2, kb = tid & 3;
  const size_t cbase = (size_t)u * v.Mcap;
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
  constexpr int kChunks = kHeadDim * kEs / 16;                      // 16-byte chunks per key
  char* const pool = v.pages + (size_t)u * v.Pcap * ((size_t)kPageElems * kEs);
  const Keys<DT> ks{pool, s.chain};
  // byte offset of 16-byte chunk c of the key in `slot` inside its page
  auto kchunk = [](int slot, int c) -> size_t {
    return (size_t)(DT == DYNAKV_F32 ? k_index32(slot, 4 * c) : k_index16(slot, 8 * c)) * kEs;
  };
  bool can_split = m >= 2;
  if (can_split) {
    // seeds: A = member farthest from the mean of all members, B = member farthest from A
    double total_d = batched_sum(tid >> 7, m, 2, [&](int i) { return ks.get(i, tid & (kHeadDim - 1)); });
    if (tid >= kHeadDim) s.cB[tid - kHeadDim] = total_d;
    __syncthreads();
    if (tid < kHeadDim) {                 // thread d < 128: sum of coordinate d over all members
      total_d += s.cB[tid];
      const double mu = total_d / (double)m;
      s.cA[tid] = mu;
      double mu2 = mu * mu;
      for (int o = 32; o > 0; o >>= 1) mu2 += __shfl_xor(mu2, o);
      if ((tid & 63) == 0) s.mu2[tid >> 6] = mu2;                    // |mean|^2, for the rounding bound of the rounds
    }
    int a = 0, b = 0;
    double far_a = 0.0, far_b = 0.0;
#pragma unroll 1
    for (int seed = 0; seed < 2; ++seed) {
      __syncthreads();
      if (seed && tid < kHeadDim) s.cA[tid] = (double)ks.get(a, tid);
      __syncthreads();
      double bv = -1.0;
      int bi = -1;
#pragma unroll 1
      for (int base = 0; base < m; base += NT / 4) {
        const int i = base + grp;
        double t, dummy;
        quad_sqdist<decltype(ks), double>(ks, min(i, m - 1), kb, s.cA, nullptr, t, dummy);
        if (kb == 0 && i < m && t > bv) { bv = t; bi = i; }          // ascending: the first maximum stays
      }
      block_argmax(bv, bi, s.sv, s.si);
      if (seed) { b = max(s.si[0], 0); far_b = s.sv[0]; }
      else { a = max(s.si[0], 0); far_a = s.sv[0]; }
    }
    const float spread = (float)sqrt(far_a) * 1.0001f;                   // every member lies this close to the mean
    const float xmax = spread + (float)sqrt(s.mu2[0] + s.mu2[1]) * 1.0001f;
    __syncthreads();
    can_split = far_b > 0.0;              // false: all members identical
    if (can_split) {
      // Lloyd rounds.  Thread d < 128 owns coordinate d: both centres and the sum of side A (registers); side B is
      // what is left of the total.  A round's side test is one inner product with w = cB - cA per member
      // (quad_side): w goes to s.cA (float64) and s.rA (float32).  Members that change side are listed, and the
      // sums follow the list instead of being formed anew (float64 sums of 16-bit values: exact, or very nearly).
      // Every member and every centre lies within sqrt(far_a) of the mean.  Two barriers per round.
      double ca = 0.0, cb = 0.0, sa = 0.0;
      if (tid < kHeadDim) { ca = s.cA[tid]; cb = (double)ks.get(b, tid); }
      for (int i = tid; i < m; i += NT) s.side[i] = 2;
      if (tid == 0) { s.nchg[0] = 0; s.nchg[1] = 0; }
      int nA = 0;
#pragma unroll 1
      for (int it = 0; it < 16; ++it) {
        const int p = it & 1;
        if (tid < kHeadDim) {             // w and t of the round
          const double w = cb - ca;
          s.cA[tid] = w; s.rA[tid] = (float)w;
          double tp = 0.5 * (cb * cb - ca * ca);
          for (int o = 32; o > 0; o >>= 1) tp += __shfl_xor(tp, o);
          if ((tid & 63) == 0) s.tpart[p * 2 + (tid >> 6)] = tp;
        }
        __syncthreads();
        const double t = s.tpart[p * 2] + s.tpart[p * 2 + 1];
        const float eps = side_eps(xmax, 2.f * spread, t);
#pragma unroll 1
        for (int base = 0; base < m; base += NT / 4) {
          const int i = base + grp;
          const unsigned char ns = quad_side(ks, min(i, m - 1), kb, s.rA, s.cA, t, eps);
          if (kb == 0 && i < m) {
            const unsigned char old = s.side[i];
            if (ns != old) {     // 0: joins side A; 1: leaves nothing (first round, side B); 2: leaves side A
              s.side[i] = ns;
              const int code = ns == 0 ? 0 : old == 2 ? 1 : 2;
              s.chg[p][atomicAdd(&s.nchg[p], 1)] = (unsigned short)(i | (code << 12));
            }
          }
        }
        __syncthreads();
        const int nc = s.nchg[p];
        if (nc == 0) break;                                  // no member moved
        for (int e = 0; e < nc; ++e) {
          const int code = s.chg[p][e] >> 12;
          nA += code == 0 ? 1 : code == 2 ? -1 : 0;
        }
        if (nA == 0 || nA == m) { can_split = false; break; }
        if (tid < kHeadDim) {
          sa += batched_sum(0, nc, 1, [&](int e) {
            const int en = s.chg[p][e], code = en >> 12;
            const float x = ks.get(en & 0xFFF, tid);
            return code == 0 ? x : code == 2 ? -x : 0.f;
          });
          ca = sa / (double)nA;
          cb = (total_d - sa) / (double)(m - nA);
        }
        if (tid == 0) s.nchg[p ^ 1] = 0;
      }
    }
  }
  // stable partition: the child that holds the earliest entry keeps id j (one that cannot be split keeps all)
  if (!can_split) {
    for (int i = tid; i < m; i += NT) s.side[i] = 0;
    __syncthreads();
  }
  const int M = s.M;
  if (can_split && M >= v.Mcap) {
    if (tid == 0) v.err[u] |= DYNAKV_ERR_CLUSTERS;
    return;
  }
  const unsigned char keep = s.side[0];
  const int chunk = (m + NT - 1) / NT;
  const int lo = min(m, tid * chunk), hi = min(m, lo + chunk);
  int mine = 0;
  for (int i = lo; i < hi; ++i) mine += s.side[i] == keep;
  int nS;
  int rs = block_excl_scan(mine, s.scan, nS, kSplitThreads / 64);
  int rm = nS + lo - rs;
  for (int i = lo; i < hi; ++i) s.perm[s.side[i] == keep ? rs++ : rm++] = (unsigned short)i;
  const int nM = m - nS;
  const int pS = (nS + kPageTokens - 1) / kPageTokens, pM = (nM + kPageTokens - 1) / kPageTokens;
  const int need = pS + pM, top = s.a_top, bump = s.a_bump;
  if (can_split && top + (v.Pcap - bump) < need) {
    if (tid == 0) v.err[u] |= DYNAKV_ERR_TOKENS;
    return;
  }
  // fresh pages for both children (recycled pages first); the parent's pages are recycled afterwards
  const int from_free = min(need, top);
  if (can_split)
    for (int k = tid; k < need; k += NT)
      s.newpg[k] = k < from_free ? v.freelist[(size_t)u * v.Pcap + top - 1 - k] : bump + (k - from_free);
  __syncthreads();
  if (can_split) {
    for (int k = tid; k < need; k += NT) {
      const bool last = k == pS - 1 || k == need - 1;
      v.pnext[(size_t)u * v.Pcap + s.newpg[k]] = last ? -1 : s.newpg[k + 1];
    }
    // keys and values in 16-byte chunks of their rows (the V row of a slot lies one K region after its K row)
    constexpr size_t kVRegion = (size_t)kPageTokens * kHeadDim * kEs;
#pragma unroll 2
    for (int t = tid; t < m * kChunks; t += NT) {
      const int q = t / kChunks, c = t % kChunks;
      const int i = s.perm[q];
      const int r = q < nS ? q : q - nS;
      const int dpage = s.newpg[(q < nS ? 0 : pS) + (r >> 4)];
      const char* src = pool + (size_t)s.chain[i >> 4] * (kPageElems * kEs) + kchunk(i & 15, c);
      char* dst = pool + (size_t)dpage * (kPageElems * kEs) + kchunk(r & 15, c);
      const uint4 w = *(const uint4*)src, x = *(const uint4*)(src + kVRegion);
      *(uint4*)dst = w;
      *(uint4*)(dst + kVRegion) = x;
      if (c == 0)
        v.ppos[((size_t)u * v.Pcap + dpage) * kPageTokens + (r & 15)] =
            v.ppos[((size_t)u * v.Pcap + s.chain[i >> 4]) * kPageTokens + (i & 15)];
    }
  }
  children_stats(v, u, s, ks, nS, m, j, can_split ? M : -1);
  if (can_split) {
    for (int k = tid; k < s.nchain; k += NT) v.freelist[(size_t)u * v.Pcap + (top - from_free) + k] = s.chain[k];
    if (tid < kInlinePages) {
      v.cpg[(cbase + j) * kInlinePages + tid] = tid < pS ? s.newpg[tid] : -1;
      v.cpg[(cbase + M) * kInlinePages + tid] = tid < pM ? s.newpg[pS + tid] : -1;
    }
  }
  if (tid == 0) {
    v.cn[cbase + j] = nS; v.csz[cbase + j] = nS; v.cb[cbase + j] = 0; v.cflag[cbase + j] = 0; v.cM2[cbase + j] = s.m2[0];
    if (can_split) {
      v.ctail[cbase + j] = s.newpg[pS - 1];
      v.cn[cbase + M] = nM; v.csz[cbase + M] = nM; v.cb[cbase + M] = 0; v.cflag[cbase + M] = 0; v.cM2[cbase + M] = s.m2[1];
      v.ctail[cbase + M] = s.newpg[pS + pM - 1];
      v.in_req[cbase + M] = 0;
      s.M = M + 1;
      s.a_top = top - from_free + s.nchain;
      s.a_bump = bump + (need - from_free);
    }
    s.nflag -= 1;
    s.did_split = can_split ? 1 : 0;
    v.flist[cbase + pos] = v.flist[cbase + s.nflag];     // the last flagged id takes the freed place
    count(v, u, can_split ? 0 : 1, 1);
  }
  __syncthreads();
}

template <int DT>
__device__ __forceinline__ void split_cluster(const View& v, int u, int j, int pos, SplitSmem& s) {
  const int tid = threadIdx.x;
  const size_t cbase = (size_t)u * v.Mcap;
  const int m = v.cn[cbase + j] + v.cb[cbase + j];
  if (tid == 0) s.did_split = 0;
  if (m > kMaxSplitMembers) {
    if (tid == 0) v.err[u] |= DYNAKV_ERR_SPLIT_SIZE;
    return;
  }
  __syncthreads();
  const int npg = (m + kPageTokens - 1) / kPageTokens;
  if (tid < kInlinePages && tid < npg) s.chain[tid] = v.cpg[(cbase + j) * kInlinePages + tid];
  __syncthreads();
  if (tid == 0) {
    for (int k = kInlinePages; k < npg; ++k) s.chain[k] = v.pnext[(size_t)u * v.Pcap + s.chain[k - 1]];
    s.nchain = npg;
  }
  __syncthreads();
  split_cluster_impl<DT>(v, u, j, pos, m, s);
}

// ---- small clusters: one wavefront per split, or one split by four wavefronts together --------------------
// Most clusters that get split hold a few dozen entries at most.  Up to four flagged clusters of a unit (64 entries of a
// 16-bit type, 32 of float32 each; two if one has up to twice that) are split side by side, one wavefront each, with no
// workgroup barrier inside the 2-means.  A cluster that is split alone has all four wavefronts and the staging rows of all
// contexts (256 entries of a 16-bit type, 160 of float32): staging, sums over the members, statistics and copies are dealt
// to them, the 2-means itself stays with the first.  (One wavefront alone: 47 us of a launch of 256 units for 64
// entries each, 90 for 128; beyond, the workgroup path below took 514 us for 200.)
// Two entries split into one each without a 2-means: 18 -> 12 us of a launch, 15 before their matrix products, which always ended in a tie.
// Same 2-means as split_cluster_impl (seeds, side test with its float64 re-check, rounds, stable partition, exact
// statistics); sums over members are float64 sums, of 16-bit values in no particular order.
// What depends on the order of the splits (new cluster ids, page allocation) is done by one thread between the
// two phases.
constexpr int kWaveSplits = kSplitThreads / 64;
constexpr int kWaveStage = 64 * kStageRow16 * 2;                 // 64 rows of a 16-bit type, 32 of float32
static_assert(32 * kStageRow32 * 4 <= kWaveStage, "float32 rows must fit");
template <int DT>
constexpr int kSmallRows = DT == DYNAKV_F32 ? 32 : 64;           // one context's rows; two contexts': a wide plan
template <int DT>
constexpr int kLoneRows = DT == DYNAKV_F32 ? 160 : 256;          // members of the largest cluster that is split alone
constexpr int kWaveRows = 256;
constexpr int kWavePages = kWaveRows / kPageTokens;
template <int DT>
constexpr int kRowBytes = (DT == DYNAKV_F32 ? kStageRow32 * 4 : kStageRow16 * 2);
template <int DT>
constexpr int kKeyChunks = kHeadDim * (DT == DYNAKV_F32 ? 4 : 2) / 16;                // 16-byte chunks per key
// Values of the first members (16-byte chunk t = 64 (k W + w) + lane of the member-major array of V rows, for wavefront w of
// the W that decide the split, k < kVAhead: 16 W members of a 16-bit type, 8 W of float32) are requested together with the
// keys and wait in registers until the children's pages are known.
constexpr int kVAhead = 4;

struct WaveCtx {
  double cA[kHeadDim], cB[kHeadDim];             // cB: partial sums before and after the 2-means, nrm / R / side during it
  alignas(16) float rA[kHeadDim], rB[kHeadDim];  // the children's means in the end, Rall during the rounds
  float d32[kWaveRows];                          // the members' squared distances in a seed search
  double m2[2];
  alignas(4) unsigned char perm[kWaveRows], inv[kWaveRows];     // inv[member] = its place in perm
  int chain[kWavePages], newpg[kWavePages + 2];
  int pos[kWaveRows];                            // sequence positions of the members
  int j, m, ok, nS, idM;
  int stage_off;                                 // the staged keys start this many bytes past the context itself
  // 16-bit types: the members' squared norms until the seeds are found; then sums of inner products with side A and with all members
  __device__ float* nrm() { return (float*)cB; }
  __device__ float* R() { return (float*)cB; }
  __device__ float* Rall() { return rA; }
  __device__ unsigned short* moved() { return (unsigned short*)perm; }   // members that change side in a round
  __device__ unsigned char* side() { return (unsigned char*)cB; }    // float32: the sides of a round
};
static_assert(sizeof(double) * kHeadDim >= sizeof(float) * kWaveRows && 2 * kHeadDim >= kWaveRows, "norms and sums take the places of WaveCtx::cB, rA and rB");
static_assert(sizeof(WaveCtx) % 16 == 0, "the staging rows behind the contexts are 16-byte aligned");
// The contexts lie at the front of the split's LDS, the staging rows of all of them behind: context x of a plan
// of small clusters has rows 64x .. 64x + 63, context x = 2, 3 of a wide plan rows 128(x - 2) .. 128(x - 2) + 127, a
// cluster split alone all of them.
__device__ __forceinline__ void wave_place_stage(WaveCtx* wc, int x, bool wide, bool lone) {
  const int row0 = lone ? 0 : wide ? 128 * (x - 2) : 64 * x;
  wc[x].stage_off = (int)((kWaveSplits - x) * sizeof(WaveCtx)) + row0 * (kWaveStage / 64);
}
__device__ __forceinline__ unsigned char* wave_stage(WaveCtx& c) { return (unsigned char*)&c + c.stage_off; }

__device__ __forceinline__ void wave_sync() {   // LDS written by some lanes of this wavefront, read by others
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}
// The same for the W wavefronts that work on one split (W = 1 or the whole workgroup).
__device__ __forceinline__ void split_sync(int W) {
  if (W == 1) wave_sync();
  else lds_barrier();
}

template <int DT>
__device__ __forceinline__ void wkey8(const unsigned char* stage, int i, int d8, float (&x)[8]) {
  if constexpr (DT == DYNAKV_F32) {
    const f4* p = (const f4*)((const float*)stage + i * kStageRow32 + d8 * 8);
    const f4 a = p[0], b = p[1];
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[e] = a[e]; x[4 + e] = b[e]; }
  } else {
    const uint4 w = *(const uint4*)((const uint16_t*)stage + i * kStageRow16 + d8 * 8);
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint16_t h = (uint16_t)(ww[e >> 1] >> ((e & 1) * 16));
      x[e] = DT == DYNAKV_F16 ? f16_to_float(h) : bf16_to_float(h);
    }
  }
}

// Key access in the form quad_sqdist expects.
template <int DT>
struct WaveKeys {
  const unsigned char* stage;
  __device__ void get8(int i, int d8, float (&x)[8]) const { wkey8<DT>(stage, i, d8, x); }
};

// A set of members: bit b of the word that lane k < kSetWords holds = member 64 k + b; the other lanes hold nothing.  (Kept across
// lanes rather than in scalar registers so that loops over the words need not be unrolled: this code runs a few times per
// launch at most, and every line of it that is fetched for the first time is a trip to memory.)
typedef unsigned long long MemberSet;
constexpr int kSetWords = kWaveRows / 64;
__device__ __forceinline__ MemberSet set_word(MemberSet s, int k) {             // k wavefront-uniform
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)s, k), hi = __builtin_amdgcn_readlane((int)(unsigned)(s >> 32), k);
  return (MemberSet)hi << 32 | lo;
}
__device__ __forceinline__ int set_count(MemberSet s) {
  int n = __popcll(s);                                                       // lanes 0 .. 3
  n += dpp_or_zero<kDppXor1>(n);
  n += dpp_or_zero<kDppXor2>(n);
  return __builtin_amdgcn_readlane(n, 0);
}
static_assert(kSetWords == 4, "a set is one quad of lanes");
__device__ __forceinline__ MemberSet first_members(int m, int lane) {
  const int k = m - 64 * lane;
  return lane >= kSetWords || k <= 0 ? 0ull : k >= 64 ? ~0ull : (1ull << k) - 1ull;
}

// Coordinates 2 lane and 2 lane + 1 of staged member i: one LDS load.
template <int DT>
__device__ __forceinline__ void wpair(const unsigned char* stage, int i, int lane, float& a, float& b) {
  if constexpr (DT == DYNAKV_F32) {
    const float2 x = ((const float2*)((const float*)stage + i * kStageRow32))[lane];
    a = x.x; b = x.y;
  } else {
    const uint32_t w = ((const uint32_t*)((const uint16_t*)stage + i * kStageRow16))[lane];
    a = DT == DYNAKV_F16 ? f16_to_float((uint16_t)w) : bf16_to_float((uint16_t)w);
    b = DT == DYNAKV_F16 ? f16_to_float((uint16_t)(w >> 16)) : bf16_to_float((uint16_t)(w >> 16));
  }
}

// ---- float64 sums of staged keys -----------------------------------------------------------------------
// A 16-bit value is a float64 after a shift: sign to the top, exponent and mantissa to the fields of the same
// name.  That is the value times 2^(15 - 1023) (float16; 2^(127 - 1023) for bfloat16), subnormal ones and zeros included, so
// sums may stay in that scale (exact: its smallest step lies far above float64's) and are scaled once at the end.  Two to three
// integer instructions per value instead of two conversions, one of them at a quarter of the rate: the sum of 64 members
// 5300 -> 2900 cycles.  An infinity or a NaN would become a finite value: `finite` false takes the conversions.
template <int DT>
constexpr int kKeyShift = DT == DYNAKV_F16 ? 6 : 3;
template <int DT>
constexpr int kKeyMask = DT == DYNAKV_F16 ? (int)0x81FFFC00u : (int)0x8FFFE000u;
template <int DT>
__device__ __forceinline__ double key_scale() {                    // what a sum is multiplied by in the end
  return DT == DYNAKV_F32 ? 1.0 : __hiloint2double((1023 + (DT == DYNAKV_F16 ? 1008 : 896)) << 20, 0);
}
template <int DT>
__device__ __forceinline__ double key_unscale() {                  // its inverse
  return DT == DYNAKV_F32 ? 1.0 : __hiloint2double((1023 - (DT == DYNAKV_F16 ? 1008 : 896)) << 20, 0);
}
template <int DT>
__device__ __forceinline__ double scaled_lo(uint32_t w) { return __hiloint2double(((int)(w << 16) >> kKeyShift<DT>) & kKeyMask<DT>, 0); }
template <int DT>
__device__ __forceinline__ double scaled_hi(uint32_t w) { return __hiloint2double(((int)w >> kKeyShift<DT>) & kKeyMask<DT>, 0); }

// Sums of coordinates 2 lane and 2 lane + 1 over the members of `set` (all keys finite), those in `less` with a minus sign.
// Eight loads per round trip to LDS; the set is walked with scalar instructions.
template <int DT>
__device__ __forceinline__ void wave_set_sums(const unsigned char* stage, MemberSet set, MemberSet less, int m, int lane, double& s0,
                                              double& s1) {
  s0 = 0.0; s1 = 0.0;
#pragma unroll 1
  for (int g = 0; 64 * g < m; ++g) {
    MemberSet mk = set_word(set, g);
    const MemberSet ls = set_word(less, g);
#pragma unroll 1
    while (mk) {
      uint32_t w[8];
      float2 f[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool in = mk != 0;
        const int b = in ? (int)__builtin_ctzll(mk) : 0, i = in ? 64 * g + b : 0;     // member 0 always exists
        mk &= mk - 1;
        const bool neg = ((ls >> b) & 1ull) != 0;
        if constexpr (DT == DYNAKV_F32) {
          f[k] = ((const float2*)((const float*)stage + i * kStageRow32))[lane];
          if (neg) { f[k].x = -f[k].x; f[k].y = -f[k].y; }
          if (!in) f[k] = float2{0.f, 0.f};
        } else {
          w[k] = ((const uint32_t*)((const uint16_t*)stage + i * kStageRow16))[lane];
          w[k] = in ? w[k] ^ (neg ? 0x80008000u : 0u) : 0u;
        }
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if constexpr (DT == DYNAKV_F32) { s0 += (double)f[k].x; s1 += (double)f[k].y; }
        else { s0 += scaled_lo<DT>(w[k]); s1 += scaled_hi<DT>(w[k]); }
      }
    }
  }
  s0 *= key_scale<DT>(); s1 *= key_scale<DT>();
}
// Sum over all m members by the W wavefronts of a split: their 4 W rows of 16 lanes take every (4 W)-th member each, a lane
// adding up the eight coordinates of its 16-byte chunk; the rows' parts are then added and handed to the lanes that own the
// coordinates (2 lane, 2 lane + 1 of every wavefront) through `part` (128 W float64).
template <int DT>
__device__ __forceinline__ void wave_total(const unsigned char* stage, int m, int w, int W, int lane, double* part, double& s0,
                                           double& s1) {
  const int r = 4 * w + (lane >> 4), ch = lane & 15;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  if constexpr (DT == DYNAKV_F32) {
#pragma unroll 2
    for (int i = r; i < m; i += 4 * W) {
      float x[8];
      wkey8<DT>(stage, i, ch, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (double)x[e];
    }
  } else {
    unsigned odd = 0;                                    // bit 15 or 31: an exponent of all ones
    constexpr unsigned kExp = DT == DYNAKV_F16 ? 0x04000400u : 0x00800080u;
#pragma unroll 2
    for (int i = r; i < m; i += 4 * W) {
      const uint4 q = *(const uint4*)((const uint16_t*)stage + i * kStageRow16 + ch * 8);
      const uint32_t ww[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        odd |= (ww[e] & 0x7FFF7FFFu) + kExp;
        acc[2 * e] += scaled_lo<DT>(ww[e]); acc[2 * e + 1] += scaled_hi<DT>(ww[e]);
      }
    }
    if (__ballot((odd & 0x80008000u) != 0)) {            // rare: once more with conversions
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll 1
      for (int i = r; i < m; i += 4 * W) {
        float x[8];
        wkey8<DT>(stage, i, ch, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += (double)x[e] * key_unscale<DT>();
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    acc[e] += __shfl_xor(acc[e], 16);
    acc[e] += __shfl_xor(acc[e], 32);
  }
  if ((lane >> 4) == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[w * kHeadDim + 8 * ch + e] = acc[e];
  }
  split_sync(W);
  s0 = 0.0; s1 = 0.0;
#pragma unroll 1
  for (int k = 0; k < W; ++k) {
    const double2 p = *(const double2*)(part + k * kHeadDim + 2 * lane);
    s0 += p.x; s1 += p.y;
  }
  s0 *= key_scale<DT>(); s1 *= key_scale<DT>();
  split_sync(W);
}

// Squared distance of member i to a centre whose coordinates 32 q .. 32 q + 31 are in cr, by the four lanes of a
// quad; every lane gets the total.  Differences, squares and sums in float32: a difference is off by 2^-24 of itself,
// the total by less than 2^-18 of itself.
template <class K>
__device__ __forceinline__ float quad_sqdist32(const K& ks, int i, int q, const float (&cr)[32]) {
  float acc[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float x[8];
    ks.get8(i, q * 4 + k, x);
    float a = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = x[e] - cr[k * 8 + e];
      a = fmaf(t, t, a);
    }
    acc[k] = a;
  }
  float s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), kDppXor1, 0xF, 0xF, false));
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), kDppXor2, 0xF, 0xF, false));
  return s;
}
// This lane's 32 coordinates (32 q ..) of a float32 vector in LDS.
__device__ __forceinline__ void load_quarter(const float* r, int q, float (&fr)[32]) {
#pragma unroll
  for (int e = 0; e < 32; e += 4) {
    const f4 x = *(const f4*)(r + q * 32 + e);
    fr[e] = x[0]; fr[e + 1] = x[1]; fr[e + 2] = x[2]; fr[e + 3] = x[3];
  }
}

// Distances d32[0 .. m) of all members to a centre whose coordinates are in r (float32, LDS), in float32.
template <int DT>
__device__ __forceinline__ void wave_distances(const WaveKeys<DT>& ks, const float* r, float* d32, int m, int lane) {
  const int grp = lane >> 2, kb = lane & 3;
  float cr[32];
  load_quarter(r, kb, cr);
#pragma unroll 1
  for (int base = 0; base < m; base += 16) {
    const int i = base + grp;
    const float d = quad_sqdist32(ks, min(i, m - 1), kb, cr);
    if (kb == 0 && i < m) d32[i] = d;
  }
  wave_sync();
}
// The member farthest from the centre (c0, c1: its coordinates 2 lane and 2 lane + 1), the lowest index among equals, from
// the squared distances d32[0 .. m), each within eps + rel * sqrt(largest) + 3.1e-5 * largest * (rel >= 0) of the true one: the
// members within twice that of the largest are compared in float64 if there are several (at most `most`; more, or matrix-core distances
// (rel < 0) beyond float32: -1).  dub: an upper bound of the largest squared distance (the exact value after a comparison).
template <int DT>
__device__ __forceinline__ int wave_farthest(const unsigned char* stage, const float* d32, int m, int lane, float eps, float rel, int most,
                                             double c0, double c1, double& dub) {
  float fm = -1.f;
#pragma unroll 1
  for (int i = lane; i < m; i += 64) fm = fmaxf(fm, d32[i]);
  const float top = __int_as_float(wave_max(__float_as_int(fm)));       // (ordered like their bits; a NaN is passed over)
  if (rel >= 0.f) eps = rel * sqrtf(top) + 3.1e-5f * top;
  const bool bound = eps < __builtin_inff();            // otherwise the squares leave float32: every member is compared
  const float thr = bound ? top - 2.f * eps : -__builtin_inff();
  int n = 0, best = -1;
#pragma unroll 1
  for (int g = 0; g < m; g += 64) {
    const MemberSet mk = __ballot(g + lane < m && d32[min(g + lane, m - 1)] >= thr);
    if (mk && best < 0) best = g + (int)__builtin_ctzll(mk);
    n += __popcll(mk);
  }
  if (n == 1 && bound) {
    dub = (double)(top + eps);
    return best;
  }
  if (n == 0 || n > most || (!bound && rel < 0.f)) { dub = -1.0; return -1; }
  best = -1;
  double bv = -1.0;
#pragma unroll 1
  for (int g = 0; g < m; g += 64)
#pragma unroll 1
    for (MemberSet mk = __ballot(g + lane < m && d32[min(g + lane, m - 1)] >= thr); mk; mk &= mk - 1) {
      const int i = g + (int)__builtin_ctzll(mk);
      float a, b;
      wpair<DT>(stage, i, lane, a, b);
      const double d0 = (double)a - c0, d1 = (double)b - c1;
      const double di = wave_sum_f64(fma(d0, d0, d1 * d1));
      if (di > bv) { bv = di; best = i; }
    }
  dub = bv;
  return best;
}

// ---- inner products of every member with one vector, on the matrix cores (16-bit types) -------------------
// The 2-means asks for the inner product of every member with a vector three to twenty times: the mean, a seed, the
// difference of the two centres in each round.  One v_mfma_f32_16x16x32 chain per 16 members does it: columns = the members as
// they are staged, rows 4g .. 4g + 2 (g = 0 .. 3, the same in each) = the vector as a sum of three 16-bit terms, so that the
// lanes of every row of 16 end up with the whole product of member lane % 16 and four tiles give each lane one member.
// Products are exact, accumulation is float32: |error| <= 2^-17 |member| |vector| plus what the terms leave (float16:
// scaled to the middle of its range, 2^-33; bfloat16: 2^-24), which the callers' bounds cover twice.
// Bound by latency: one trip to LDS, a chain of four matrix instructions per tile, four tiles at a time.
constexpr int kTermRow = kHeadDim + 8;           // 16-bit elements from one term to the next: the rows hit different banks
static_assert(3 * kTermRow * 2 <= (int)sizeof(double) * kHeadDim, "the terms take the place of WaveCtx::cA");
// Power of two that brings the largest coordinate of a vector (coordinates a, b of each lane) to 2^13 .. 2^14 (float16).
template <int DT>
__device__ __forceinline__ float wave_scale(float a, float b, float& inverse) {
  if constexpr (DT != DYNAKV_F16) { inverse = 1.f; return 1.f; }
  const int e = wave_max(__float_as_int(fmaxf(fabsf(a), fabsf(b)))) >> 23;
  const int f = min(max(267 - e, 1), 253);
  inverse = __int_as_float((254 - f) << 23);
  return __int_as_float(f << 23);
}
// A operand of the vector whose coordinates 2 lane and 2 lane + 1 are w0 and w1 (scaled).
template <int DT>
__device__ __forceinline__ void wave_terms(WaveCtx& c, float w0, float w1, int lane, uint4 (&a)[4]) {
  uint32_t* t = (uint32_t*)c.cA;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint16_t b0, b1;
    if constexpr (DT == DYNAKV_BF16) {
      const __bf16 h0 = (__bf16)w0, h1 = (__bf16)w1;
      b0 = __builtin_bit_cast(uint16_t, h0); b1 = __builtin_bit_cast(uint16_t, h1);
      w0 -= (float)h0; w1 -= (float)h1;
    } else {
      const _Float16 h0 = (_Float16)w0, h1 = (_Float16)w1;
      b0 = __builtin_bit_cast(uint16_t, h0); b1 = __builtin_bit_cast(uint16_t, h1);
      w0 -= (float)h0; w1 -= (float)h1;
    }
    t[k * (kTermRow / 2) + lane] = (uint32_t)b0 | ((uint32_t)b1 << 16);
  }
  wave_sync();
  const uint16_t* p = (const uint16_t*)c.cA + min(lane & 3, 2) * kTermRow + 8 * (lane >> 4);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint4 x = *(const uint4*)(p + 32 * s);
    a[s] = (lane & 3) == 3 ? uint4{0, 0, 0, 0} : x;
  }
  wave_sync();
}
__device__ __forceinline__ float wave_sum_f32(float x) {
  x += __int_as_float(dpp_or_zero<kDppXor1>(__float_as_int(x)));
  x += __int_as_float(dpp_or_zero<kDppXor2>(__float_as_int(x)));
  x += __int_as_float(dpp_or_zero<kDppHalfMirror>(__float_as_int(x)));
  x += __int_as_float(dpp_or_zero<kDppMirror>(__float_as_int(x)));
  return rows_sum(x);
}
// Staged members first .. first + 16 NT - 1 as matrix operands (lane l: chunk l / 16 of member first + 16 T + l % 16).
template <int NT>
__device__ __forceinline__ void load_tiles(const unsigned char* stage, int first, int lane, uint4 (&b)[NT][4]) {
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    const uint16_t* p = (const uint16_t*)stage + (first + 16 * T + (lane & 15)) * kStageRow16 + 8 * (lane >> 4);
#pragma unroll
    for (int s = 0; s < 4; ++s) b[T][s] = *(const uint4*)(p + 32 * s);
  }
}
// The tile's Gram matrix has |member|^2 on its diagonal: member c's in register c % 4 of lane c + 16 (c / 4); every lane gets its own.
__device__ __forceinline__ float gram_diagonal(const f4& g, int lane) {
  const int c = lane & 15;
  return __shfl(sel4(g, c & 3), c + 16 * (c >> 2));
}
enum { kDotNorm, kDotVector, kDotRows };
// NT tiles of 16 members from member `first` on, one value per lane for member first + lane: its |member|^2 (kDotNorm), its inner
// product with the vector whose terms are in a (kDotVector), the sum of its inner products with the sixteen rows in a (kDotRows).
// Lanes past the last member get the product with whatever its staging row holds: nobody may look at it.
template <int DT, int WHAT, int NT>
__device__ __forceinline__ float dot_tiles(const unsigned char* stage, int first, int lane, const uint4 (&a)[4]) {
  constexpr bool BF = DT == DYNAKV_BF16;
  uint4 b[NT][4];
  load_tiles<NT>(stage, first, lane, b);
  f4 acc[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T) acc[T] = f4{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int T = 0; T < NT; ++T) acc[T] = mfma_k32<BF>(WHAT == kDotNorm ? b[T][s] : a[s], b[T][s], acc[T]);
  float res = 0.f;
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    const float d = WHAT == kDotNorm ? gram_diagonal(acc[T], lane) : WHAT == kDotVector ? (acc[T][0] + acc[T][1]) + acc[T][2]
                                     : rows_sum((acc[T][0] + acc[T][1]) + (acc[T][2] + acc[T][3]));
    res = T == 0 || (lane >> 4) == T ? d : res;
  }
  return res;
}
template <int DT, int WHAT>
__device__ __forceinline__ float wave_dots(const unsigned char* stage, int first, int m, int lane, const uint4 (&a)[4]) {
  if (m - first <= 16) return dot_tiles<DT, WHAT, 1>(stage, first, lane, a);       // wavefront-uniform
  return dot_tiles<DT, WHAT, 4>(stage, first, lane, a);
}

// The 2-means of up to 16 members of a 16-bit type from their Gram matrix alone, by one wavefront: the sides of every round follow
// from sums of inner products,  <x, c_A> = sum_{j in A} <x, x_j> / n_A,  |c_A|^2 = sum_{i in A} <x_i, c_A> / n_A, a handful of
// vector instructions a round.  Every inner product is off by 2^-17 x2 at most (x2 >= every |member|^2), and so is a mean of
// them; B's are what A's leave of the totals, so theirs is off by m / n_B times that: eps below is the sum of what enters a
// comparison, rounded up.  A seed's distance takes in 4 such units (|x|^2, twice a product or mean, |centre|^2); the float32 sums behind
// it (five additions for a mean, doubled, eleven for the mean's norm, the roundings of 1 / m, products and differences) come to less
// than 40 * 2^-24 x2, 0.32 of a unit: 4.5.  Returns 1 (split: side holds A), 0 (one side ran empty) or -1: a decision fell within eps; wave_two_means takes it.
template <int DT>
__device__ __forceinline__ int gram_two_means(const unsigned char* stage, int m, int lane, unsigned& side) {
  constexpr bool BF = DT == DYNAKV_BF16;
  const int lg = lane >> 4, cl = lane & 15;
  uint4 b[1][4];
  load_tiles<1>(stage, 0, lane, b);
  f4 G = {0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 4; ++s) G = mfma_k32<BF>(b[0][s], b[0][s], G);       // G[i] = <member 4 lg + i, member cl>
  const float nrm = gram_diagonal(G, lane);
  const bool in = cl < m;                                       // every row of lanes holds all members
  const unsigned all = (1u << m) - 1u;
  const float x2 = __int_as_float(wave_max(in ? __float_as_int(nrm) & 0x7fffffff : 0)) * 1.0001f, unit = 7.7e-6f * x2;      // 1.01 * 2^-17 x2
  if (!(x2 < 1e30f)) return -1;
  // sum over the members of a set of their inner products with this lane's member
  auto with = [&](unsigned set) __attribute__((always_inline)) {
    float r = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) r += (set >> (4 * lg + i)) & 1u ? G[i] : 0.f;
    return rows_sum(r);
  };
  // the set's only member within 2 eps of the largest d; -1: there are several
  auto farthest = [&](float d, float eps) __attribute__((always_inline)) {
    d = in ? fmaxf(d, 0.f) : -1.f;
    const float top = __int_as_float(wave_max(__float_as_int(d)));
    const unsigned cand = (unsigned)__ballot(in && d >= top - 2.f * eps) & 0xFFFFu;
    return __popc(cand) == 1 && top > 2.f * eps ? (int)__builtin_ctz(cand) : -1;
  };
  const float Rall = with(all), im = 1.f / (float)m;
  const int a = farthest(nrm - 2.f * Rall * im + wave_sum_f32(lane < m ? Rall : 0.f) * im * im, 4.5f * unit);
  if (a < 0) return -1;
  const float na = __shfl(nrm, a), Ga = with(1u << a);
  const int bb = farthest(nrm - 2.f * Ga + na, 4.5f * unit);
  if (bb < 0) return -1;
  float s = with(1u << bb) - Ga, t = 0.5f * (__shfl(nrm, bb) - na), eps = 4.f * unit;
  unsigned A = all;
#pragma unroll 1
  for (int it = 0; it < 16; ++it) {
    if (__ballot(in && !(fabsf(s - t) > eps))) return -1;
    const unsigned nw = (unsigned)__ballot(in && s <= t) & 0xFFFFu;
    if (it > 0 && nw == A) break;
    const int nA = __popc(nw), nB = m - nA;
    if (nA == 0 || nB == 0) return 0;
    A = nw;
    const float ia = 1.f / (float)nA, ib = 1.f / (float)nB;
    const float RA = with(A), RB = Rall - RA;
    const float QA = wave_sum_f32(lane < m && ((A >> cl) & 1u) ? RA : 0.f), QB = wave_sum_f32(lane < m && !((A >> cl) & 1u) ? RB : 0.f);
    s = RB * ib - RA * ia;
    t = 0.5f * (QB * ib * ib - QA * ia * ia);
    eps = unit * (2.f + 2.f * (float)(m + nA) * ib);
  }
  side = A;
  return 1;
}

// quad_side with the float32 weights of coordinates 32 q .. 32 q + 31 already in registers (wr).
template <class K>
__device__ __forceinline__ unsigned char quad_side_reg(const K& ks, int i, int q, const float (&wr)[32], const double* wd,
                                                       double t, float eps) {
  float x[4][8];
#pragma unroll
  for (int k = 0; k < 4; ++k) ks.get8(i, q * 4 + k, x[k]);
  float part[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float a = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) a = fmaf(x[k][e], wr[k * 8 + e], a);
    part[k] = a;
  }
  float s = (part[0] + part[1]) + (part[2] + part[3]);
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), kDppXor1, 0xF, 0xF, false));
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), kDppXor2, 0xF, 0xF, false));
  const float tf = (float)t;
  if (fabsf(s - tf) > eps) return s <= tf ? 0 : 1;            // uniform over the quad
  double sd = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) sd = fma((double)x[k][e], wd[(q * 4 + k) * 8 + e], sd);
  sd += dpp_f64<kDppXor1, 0xF>(sd);
  sd += dpp_f64<kDppXor2, 0xF>(sd);
  return sd <= t ? 0 : 1;
}

// Members within the rounding bound of the border of a round, one at a time in float64: `side` with their bits put right.
// g: member of the word's bit 0; w, t: the border, <x, w> <= t on side A.
template <int DT>
__device__ __forceinline__ MemberSet retake_sides(const unsigned char* stage, MemberSet side, MemberSet unsure, int g, int lane, double w0,
                                                  double w1, double t) {
#pragma unroll 1
  for (; unsure; unsure &= unsure - 1) {
    const int i = (int)__builtin_ctzll(unsure);
    float x0, x1;
    wpair<DT>(stage, g + i, lane, x0, x1);
    const bool isA = wave_sum_f64(fma((double)x0, w0, (double)x1 * w1)) <= t;
    side = isA ? side | (1ull << i) : side & ~(1ull << i);
  }
  return side;
}

// Seeds of a staged cluster's 2-means by one wavefront: A = the member farthest from the mean (w0, w1: its coordinates 2 lane
// and 2 lane + 1; mn2 >= its squared norm), B = the member farthest from A.  spread >= every member's distance from the mean.
// False: all members are identical (or not finite).  For 16-bit types c.nrm holds the members' squared norms, x2 the largest.
// The matrix cores' distances |x|^2 - 2 <x, w> + |w|^2 are off by 2^-17 of |x|^2 + 2 |x| |w| (twice that below); where that
// leaves many members, and for float32 keys, they are taken from the differences, whose rounding is relative to them (and
// rounding the mean moves a difference by 2^-24 |mean|, a distance by 2^-23 |mean| sqrt(distance)).
template <int DT>
__device__ __forceinline__ bool find_seeds(WaveCtx& c, const unsigned char* stage, int m, int lane, double w0, double w1, double mn2,
                                           float x2, float& spread, int& seed_a, int& seed_b) {
  const WaveKeys<DT> ks{stage};
  const float mn = (float)sqrt(mn2) * 1.0001f;
  float na = (float)mn2;
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    bool direct = DT == DYNAKV_F32;
    if constexpr (DT != DYNAKV_F32) {
      float inv;
      const float scale = wave_scale<DT>((float)w0, (float)w1, inv);
      uint4 op[4];
      wave_terms<DT>(c, (float)w0 * scale, (float)w1 * scale, lane, op);
#pragma unroll 1
      for (int g = 0; g < m; g += 64) {
        const float dot = inv * wave_dots<DT, kDotVector>(stage, g, m, lane, op);
        if (pass == 0) c.Rall()[g + lane] = dot * (float)m;
        c.d32[g + lane] = fmaxf(c.nrm()[g + lane] - 2.f * dot + na, 0.f);
      }
      wave_sync();
    }
    double dub = -1.0;
    int far = -1;
    const float reach = __builtin_sqrtf(x2) + (pass == 0 ? mn : __builtin_sqrtf(x2));
#pragma unroll 1
    while (true) {
      if (direct) {
        float* const r = (float*)c.cA;                 // (the terms are dead)
        r[2 * lane] = (float)w0; r[2 * lane + 1] = (float)w1;
        wave_sync();
        wave_distances<DT>(ks, r, c.d32, m, lane);
      }
      far = wave_farthest<DT>(stage, c.d32, m, lane, 1.53e-5f * reach * reach + 1e-30f,
                              !direct ? -1.f : pass == 0 ? 2.4e-7f * mn : 0.f, direct ? kWaveRows : 12, w0, w1, dub);
      if (far >= 0 || direct) break;
      direct = true;
    }
    far = max(far, 0);                       // (keys that are not finite: no member is farthest)
    if (pass == 0) {
      seed_a = far;
      spread = (float)sqrt(fmax(dub, 0.0)) * 1.0001f;
      float f0, f1;
      wpair<DT>(stage, far, lane, f0, f1);
      w0 = (double)f0; w1 = (double)f1;
      if constexpr (DT != DYNAKV_F32) na = c.nrm()[far];
    } else {
      seed_b = far;
      return dub > 0.0;
    }
  }
  return false;
}

// The 2-means of a staged cluster by one wavefront: seeds, rounds, stable partition (c.ok, c.nS, c.perm, c.inv) and the float32
// means of the children (c.rA, c.rB; of the whole cluster in c.rA if it cannot be split).  tot0, tot1: the sum of all
// members, coordinates 2 lane and 2 lane + 1.  The sides of a round are sets of bits.
// 16-bit types: what a round asks of a member is its inner products with the two centres, sums over the sides of inner
// products of members: R = sum over side A (c.R) starts from the first round's side as one vector and then follows the members
// that changed side, sixteen at a time as rows of a matrix product against all members.  float32 keys: the sum of side A follows the
// members that moved, and each round takes the inner products with cB - cA anew.
template <int DT>
__device__ inline void wave_two_means(WaveCtx& c, const unsigned char* stage, int m, double tot0, double tot1) {
  const int lane = threadIdx.x & 63;
  const MemberSet all = first_members(m, lane);
  double sa0 = tot0, sa1 = tot1;                 // sum of side A (16-bit types: as the first round left it, first_A)
  MemberSet A = all, first_A = all;
  bool can = m >= 2;
  int quick = -1;
  if (m == 2) {                                            // each is its own centre, whichever is taken first, unless they are equal
    float a0, a1, b0, b1;
    wpair<DT>(stage, 0, lane, a0, a1);
    wpair<DT>(stage, 1, lane, b0, b1);
    const double d0 = (double)a0 - (double)b0, d1 = (double)a1 - (double)b1, apart = wave_sum_f64(fma(d0, d0, d1 * d1));
    quick = apart > 0.0 && apart < __builtin_inf();
    can = quick == 1;
    if (can) { A = lane == 0 ? 1ull : 0ull; sa0 = (double)a0; sa1 = (double)a1; }
  }
  if constexpr (DT != DYNAKV_F32)
    if (m > 2 && m <= 16) {
      unsigned side = 0;
      quick = gram_two_means<DT>(stage, m, lane, side);
      if (quick == 1) A = lane == 0 ? (MemberSet)side : 0ull;
      if (quick == 0) can = false;
    }
  if (can && quick < 0) {
    const CountInverse im = count_inverse(m);
    const double mu0 = over_count(tot0, im), mu1 = over_count(tot1, im), mn2 = wave_sum_f64(mu0 * mu0 + mu1 * mu1);
    float x2 = 0.f, spread = 0.f;
    if constexpr (DT != DYNAKV_F32) {                              // |member|^2, and the largest of them
      int nmax = 0;
#pragma unroll 1
      for (int g = 0; g < m; g += 64) {
        const uint4 unused[4] = {};
        const float n = wave_dots<DT, kDotNorm>(stage, g, m, lane, unused);
        c.nrm()[g + lane] = n;
        // (an infinity or a NaN is larger than everything)
        nmax = max(nmax, g + lane < m ? __float_as_int(n) & 0x7fffffff : 0);
      }
      x2 = __int_as_float(wave_max(nmax)) * 1.0001f;
      wave_sync();
    }
    int a, b;
    can = find_seeds<DT>(c, stage, m, lane, mu0, mu1, mn2, x2, spread, a, b);
    if (can) {
      float fa0, fa1, fb0, fb1;
      wpair<DT>(stage, a, lane, fa0, fa1);
      wpair<DT>(stage, b, lane, fb0, fb1);
      double ca0 = (double)fa0, ca1 = (double)fa1, cb0 = (double)fb0, cb1 = (double)fb1;       // centres
      const float mn = (float)sqrt(mn2) * 1.0001f;
      float err_r = 0.f;                                           // bound of |error| of R
      const float unit = 7.7e-6f * x2;                             // 1.01 * 2^-17 x2
#pragma unroll 1
      for (int it = 0; it < 16; ++it) {
        // w = cB - cA, t = (|cB|^2 - |cA|^2) / 2: a member is on side A if <x, w> <= t
        MemberSet nw = 0;
        if (DT == DYNAKV_F32 || it == 0) {
          const double w0 = cb0 - ca0, w1 = cb1 - ca1;
          const double t = wave_sum_f64(0.5 * ((cb0 * cb0 - ca0 * ca0) + (cb1 * cb1 - ca1 * ca1)));
          const float eps = side_eps(spread + mn, 2.f * spread, t), tf = (float)t;      // every member and centre lies within `spread` of the mean
          if constexpr (DT != DYNAKV_F32) {
            float inv;
            const float scale = wave_scale<DT>((float)w0, (float)w1, inv);
            uint4 op[4];
            wave_terms<DT>(c, (float)w0 * scale, (float)w1 * scale, lane, op);
#pragma unroll 1
            for (int g = 0; g < m; g += 64) {
              const float s = wave_dots<DT, kDotVector>(stage, g, m, lane, op) * inv;
              const MemberSet side = retake_sides<DT>(stage, __ballot(g + lane < m && s <= tf),
                                                      __ballot(g + lane < m && !(fabsf(s - tf) > eps)), g, lane, w0, w1, t);
              nw = lane == (g >> 6) ? side : nw;
            }
          } else {
            const int grp = lane >> 2, kb = lane & 3;              // four lanes per member
            c.cA[2 * lane] = w0; c.cA[2 * lane + 1] = w1;
            c.rA[2 * lane] = (float)w0; c.rA[2 * lane + 1] = (float)w1;
            wave_sync();
            float wr[32];
            load_quarter(c.rA, kb, wr);
            const WaveKeys<DT> ks{stage};
#pragma unroll 1
            for (int base = 0; base < m; base += 16) {
              const int i = base + grp;
              const unsigned char ns = quad_side_reg(ks, min(i, m - 1), kb, wr, c.cA, t, eps);
              if (kb == 0 && i < m) c.side()[i] = ns;
            }
            wave_sync();
#pragma unroll 1
            for (int g = 0; g < m; g += 64) {
              const MemberSet side = __ballot(g + lane < m && c.side()[min(g + lane, m - 1)] == 0);
              nw = lane == (g >> 6) ? side : nw;
            }
          }
        } else {
          // from R: <x, cB> - <x, cA> = (Rall - R) / nB - R / nA, and the squared norms as means of those over the sides
          const int nA = set_count(A);
          const float ia = 1.f / (float)nA, ib = 1.f / (float)(m - nA);
          float qa = 0.f, qb = 0.f;
#pragma unroll 1
          for (int g = 0; g < m; g += 64) {
            const bool inA = (set_word(A, g >> 6) >> lane) & 1ull;
            const float ra = c.R()[g + lane], rb = c.Rall()[g + lane] - ra;
            qa += inA ? ra : 0.f;
            qb += !inA && g + lane < m ? rb : 0.f;
          }
          const float t = 0.5f * (wave_sum_f32(qb) * ib * ib - wave_sum_f32(qa) * ia * ia);
          // R / nA, (Rall - R) / nB, half of the same again in t, and the roundings of this block
          const float eps = 1.6f * (err_r * ia + (1.1f * (float)m * unit + err_r) * ib) + 2.f * unit;
          MemberSet unsure = 0;
#pragma unroll 1
          for (int g = 0; g < m; g += 64) {
            const float ra = c.R()[g + lane], s = (c.Rall()[g + lane] - ra) * ib - ra * ia;
            const float gap = fabsf(s - t);              // (not finite: a sum has left float32, which no bound covers)
            const MemberSet side = __ballot(g + lane < m && s <= t), un = __ballot(g + lane < m && !(gap > eps && gap < __builtin_inff()));
            nw = lane == (g >> 6) ? side : nw;
            unsure = lane == (g >> 6) ? un : unsure;
          }
          if (__ballot(unsure != 0)) {                             // float64 centres for those
            double w0, w1, d0, d1;
            wave_set_sums<DT>(stage, A ^ first_A, first_A & ~A, m, lane, d0, d1);
            const CountInverse na = count_inverse(nA), nb = count_inverse(m - nA);       // (rounded as a division: exact ties stay)
            ca0 = over_count(sa0 + d0, na); ca1 = over_count(sa1 + d1, na);
            cb0 = over_count(tot0 - (sa0 + d0), nb); cb1 = over_count(tot1 - (sa1 + d1), nb);
            w0 = cb0 - ca0; w1 = cb1 - ca1;
            const double tt = wave_sum_f64(0.5 * ((cb0 * cb0 - ca0 * ca0) + (cb1 * cb1 - ca1 * ca1)));
#pragma unroll 1
            for (int g = 0; g < m; g += 64) {
              const MemberSet side = retake_sides<DT>(stage, set_word(nw, g >> 6), set_word(unsure, g >> 6), g, lane, w0, w1, tt);
              nw = lane == (g >> 6) ? side : nw;
            }
          }
        }
        const MemberSet joins = nw & ~A, leaves = A & ~nw, moved = joins | leaves;
        const bool first = it == 0;
        if (!first && __ballot(moved != 0) == 0) break;           // no member moved
        const int nA = set_count(nw);
        if (nA == 0 || nA == m) { can = false; break; }
        A = nw;
        if constexpr (DT == DYNAKV_F32) {
          // the sum of side A: formed from the smaller side in the first round (A was everything before), then corrected by the
          // members that moved; side B is what is left of the total
          const bool anew = first && 2 * nA <= m;
          double d0, d1;
          wave_set_sums<DT>(stage, anew ? nw : moved, anew ? 0ull : leaves, m, lane, d0, d1);
          sa0 = anew ? d0 : sa0 + d0; sa1 = anew ? d1 : sa1 + d1;
          const CountInverse ia = count_inverse(nA), ib = count_inverse(m - nA);
          ca0 = over_count(sa0, ia); ca1 = over_count(sa1, ia);
          cb0 = over_count(tot0 - sa0, ib); cb1 = over_count(tot1 - sa1, ib);
        } else if (first) {                                        // R of the smaller side, as one vector (Rall: from the seeds' search)
          const bool isA = 2 * nA <= m;
          double d0, d1;
          wave_set_sums<DT>(stage, isA ? nw : leaves, 0ull, m, lane, d0, d1);
          first_A = nw;
          sa0 = isA ? d0 : tot0 - d0; sa1 = isA ? d1 : tot1 - d1;
          float inv;
          const float scale = wave_scale<DT>((float)d0, (float)d1, inv);
          uint4 op[4];
          wave_terms<DT>(c, (float)d0 * scale, (float)d1 * scale, lane, op);
#pragma unroll 1
          for (int g = 0; g < m; g += 64) {
            const float r = wave_dots<DT, kDotVector>(stage, g, m, lane, op) * inv;
            c.R()[g + lane] = isA ? r : c.Rall()[g + lane] - r;
          }
          err_r = 1.1f * unit * (float)(isA ? nA : 2 * m - nA);
        } else {
          // the members that moved, sixteen at a time as rows (those that leave side A with their signs changed)
          unsigned short* const list = c.moved();
          int n = 0;
#pragma unroll 1
          for (int g = 0; g < m; g += 64) {
            const MemberSet mv = set_word(moved, g >> 6), lv = set_word(leaves, g >> 6);
            if ((mv >> lane) & 1ull)
              list[n + __popcll(mv & ((1ull << lane) - 1ull))] = (unsigned short)(g + lane | ((lv >> lane) & 1ull ? 0x8000 : 0));
            n += __popcll(mv);
          }
          wave_sync();
#pragma unroll 1
          for (int k = 0; k < n; k += 16) {
            const bool have = k + (lane & 15) < n;
            const int e = list[min(k + (lane & 15), n - 1)];
            const uint32_t flip = e & 0x8000 ? 0x80008000u : 0u;
            const uint16_t* p = (const uint16_t*)stage + (e & 0x7FFF) * kStageRow16 + 8 * (lane >> 4);
            uint4 op[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint4 x = *(const uint4*)(p + 32 * q);
              op[q] = have ? uint4{x.x ^ flip, x.y ^ flip, x.z ^ flip, x.w ^ flip} : uint4{0, 0, 0, 0};
            }
#pragma unroll 1
            for (int g = 0; g < m; g += 64) c.R()[g + lane] += wave_dots<DT, kDotRows>(stage, g, m, lane, op);
            err_r += unit * (float)(min(16, n - k) + 1) + 4.8e-7f * (float)m * x2;      // (eight roundings of numbers up to m x2)
          }
          wave_sync();
        }
      }
    }
  }
  // stable partition: the child that holds the earliest entry comes first and keeps the id
  const bool a_first = (__builtin_amdgcn_readlane((int)(unsigned)A, 0) & 1) != 0;
  const MemberSet S = !can ? all : a_first ? A : all & ~A;
  const int nS = set_count(S), nM = m - nS;
  int before = 0;                                            // members of the staying child in the groups before
#pragma unroll 1
  for (int g = 0; g < m; g += 64) {
    const MemberSet sw = set_word(S, g >> 6);
    const int i = g + lane;
    if (i < m) {
      const int b = before + __popcll(sw & ((1ull << lane) - 1ull));
      const int q = (sw >> lane) & 1ull ? b : nS + i - b;
      c.perm[q] = (unsigned char)i;
      c.inv[i] = (unsigned char)q;
    }
    before += __popcll(sw);
  }
  if (lane == 0) { c.ok = can ? 1 : 0; c.nS = nS; }
  double sS0 = tot0, sS1 = tot1;
  if (can) {
    if constexpr (DT == DYNAKV_F32) { sS0 = a_first ? sa0 : tot0 - sa0; sS1 = a_first ? sa1 : tot1 - sa1; }
    else {                                                   // from the first round's, by the members that have moved since
      const bool fewer = quick == 1 && 2 * nS > m;           // (none: from all members, by the smaller side)
      const MemberSet base = quick == 1 ? (fewer ? all : 0ull) : a_first ? first_A : all & ~first_A;
      double b0 = fewer ? tot0 : 0.0, b1 = fewer ? tot1 : 0.0, d0, d1;
      if (quick != 1) { b0 = a_first ? sa0 : tot0 - sa0; b1 = a_first ? sa1 : tot1 - sa1; }
      wave_set_sums<DT>(stage, S ^ base, base & ~S, m, lane, d0, d1);
      sS0 = b0 + d0; sS1 = b1 + d1;
    }
  }
  const CountInverse iS = count_inverse(nS), iM = count_inverse(max(nM, 1));
  c.rA[2 * lane] = (float)over_count(sS0, iS); c.rA[2 * lane + 1] = (float)over_count(sS1, iS);
  if (can) { c.rB[2 * lane] = (float)over_count(tot0 - sS0, iM); c.rB[2 * lane + 1] = (float)over_count(tot1 - sS1, iM); }
}

// Decides one split, by one wavefront (W = 1; w = 0) or by the W wavefronts of the workgroup together (wavefront w of them):
// stages the keys (c.chain lists their pages), 2-means, stable partition, exact statistics of the children (of the unsplit
// cluster if the 2-means finds nothing to split).  Sets c.ok, c.nS, c.perm, c.inv, c.pos, the float32 means c.rA / c.rB and
// the M2 about them, c.m2.  part: 128 W float64 of LDS.  f64: SplitPlan::f64.
template <int DT>
__device__ __forceinline__ void wave_split_decide(const View& v, int u, WaveCtx& c, int w, int W, bool f64, double* part,
                                                  uint4 (&vahead)[kVAhead]) {
  const int lane = threadIdx.x & 63;
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
  constexpr int kChunks = kKeyChunks<DT>;
  const char* const pool = v.pages + (size_t)u * v.Pcap * ((size_t)kPageElems * kEs);
  const int m = c.m;
  unsigned char* const stage = wave_stage(c);
  const int total = m * kChunks;
  // the values requested ahead and the positions ride along
#pragma unroll
  for (int k = 0; k < kVAhead; ++k) {
    const int t = (k * W + w) * 64 + lane, i = t / kChunks, ch = t % kChunks;
    vahead[k] = uint4{0, 0, 0, 0};
    if (i < m) {
      const size_t off = (size_t)(DT == DYNAKV_F32 ? v_index32(i & 15, 4 * ch) : v_index16(i & 15, 8 * ch)) * kEs;
      vahead[k] = *(const uint4*)(pool + (size_t)c.chain[i >> 4] * (kPageElems * kEs) + off);
    }
  }
  auto fetch = [&](int t0, auto ahead) __attribute__((always_inline)) {
    constexpr int kAhead = decltype(ahead)::value;         // key loads in flight per lane
    f4 x[kAhead];                                          // (a plain vector type: these stay in registers)
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int t = min(t0 + (k * W + w) * 64 + lane, total - 1);
      const int i = t / kChunks, ch = t % kChunks;
      const size_t off = (size_t)(DT == DYNAKV_F32 ? k_index32(i & 15, 4 * ch) : k_index16(i & 15, 8 * ch)) * kEs;
      x[k] = *(const f4*)(pool + (size_t)c.chain[i >> 4] * (kPageElems * kEs) + off);
    }
    if (t0 == 0)
      for (int i = w * 64 + lane; i < m; i += 64 * W) c.pos[i] = v.ppos[((size_t)u * v.Pcap + c.chain[i >> 4]) * kPageTokens + (i & 15)];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int t = t0 + (k * W + w) * 64 + lane;
      if (t < total) *(f4*)(stage + (size_t)(t / kChunks) * kRowBytes<DT> + (t % kChunks) * 16) = x[k];
    }
  };
  if (total <= 4 * 64 * W) fetch(0, std::integral_constant<int, 4>{});
  else
#pragma unroll 1
    for (int t0 = 0; t0 < total; t0 += 16 * 64 * W) fetch(t0, std::integral_constant<int, 16>{});
  split_sync(W);
  double tot0, tot1;
  wave_total<DT>(stage, m, w, W, lane, part, tot0, tot1);
  if (w == 0) wave_two_means<DT>(c, stage, m, tot0, tot1);
  split_sync(W);
  // M2 of the children about their means (differences in float32, off by 2^-24 of themselves; sums of 32 squares in
  // float32, the rest in float64; all of it in float64 in a plan with a cluster that only four wavefronts together take, as the
  // workgroup path has it)
  const WaveKeys<DT> ks{stage};
  const int grp = lane >> 2, kb = lane & 3, nS = c.nS;
  double acc[2] = {0.0, 0.0};
#pragma unroll 1
  for (int base = 16 * w; base < m; base += 16 * W) {
    const int q = base + grp;
    double d;
    if (f64) {                                            // the same in every wavefront
      double none;
      quad_sqdist<WaveKeys<DT>, float>(ks, c.perm[min(q, m - 1)], kb, q < nS ? c.rA : c.rB, nullptr, d, none);
    } else {
      float fr[32];
      load_quarter(q < nS ? c.rA : c.rB, kb, fr);
      d = (double)quad_sqdist32(ks, c.perm[min(q, m - 1)], kb, fr);
    }
    const double dv = kb == 0 && q < m ? d : 0.0;
    acc[0] += q < nS ? dv : 0.0;
    acc[1] += q < nS ? 0.0 : dv;
  }
  acc[0] = wave_sum_f64(acc[0]); acc[1] = wave_sum_f64(acc[1]);
  if (lane == 0) { part[2 * w] = acc[0]; part[2 * w + 1] = acc[1]; }
  split_sync(W);
  if (w == 0 && lane < 2) {
    double sum = 0.0;
#pragma unroll 1
    for (int k = 0; k < W; ++k) sum += part[2 * k + lane];
    c.m2[lane] = sum;
  }
  split_sync(W);
}

// Last phase, once the children's id and pages are assigned: pages, centroids and records, by the W wavefronts that call it
// (any number; wavefront w of them).  With c.ok == 0 the cluster is only unflagged, with exact statistics.
// wave_split_decide has run on c, by WD wavefronts; what each of them requested ahead is written by wave_split_commit_ahead.
template <int DT>
__device__ __forceinline__ char* split_vdest(char* pool, const WaveCtx& c, int i, int ch) {
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
  const int q = c.inv[i], r = q < c.nS ? q : q - c.nS, pS = (c.nS + kPageTokens - 1) / kPageTokens;
  return pool + (size_t)c.newpg[(q < c.nS ? 0 : pS) + (r >> 4)] * ((size_t)kPageElems * kEs) +
         (size_t)(DT == DYNAKV_F32 ? v_index32(r & 15, 4 * ch) : v_index16(r & 15, 8 * ch)) * kEs;
}
template <int DT>
__device__ __forceinline__ void wave_split_commit_ahead(const View& v, int u, const WaveCtx& c, int w, int WD, const uint4 (&vahead)[kVAhead]) {
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
  char* const pool = v.pages + (size_t)u * v.Pcap * ((size_t)kPageElems * kEs);
  if (!c.ok) return;
#pragma unroll
  for (int k = 0; k < kVAhead; ++k) {
    const int t = (k * WD + w) * 64 + (threadIdx.x & 63), i = t / kKeyChunks<DT>;
    if (i < c.m) *(uint4*)split_vdest<DT>(pool, c, i, t % kKeyChunks<DT>) = vahead[k];
  }
}
template <int DT>
__device__ __forceinline__ void wave_split_commit(const View& v, int u, WaveCtx& c, int WD, int w, int W) {
  const int lane = threadIdx.x & 63, t_own = w * 64 + lane, step = W * 64;
  const size_t cbase = (size_t)u * v.Mcap;
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
  constexpr int kChunks = kKeyChunks<DT>;
  constexpr size_t kPageBytes = (size_t)kPageElems * kEs;
  char* const pool = v.pages + (size_t)u * v.Pcap * kPageBytes;
  const int m = c.m, j = c.j, nS = c.nS, nM = m - nS, idM = c.ok ? c.idM : -1;
  const int pS = (nS + kPageTokens - 1) / kPageTokens, pM = (nM + kPageTokens - 1) / kPageTokens, need = pS + pM;
  const unsigned char* const stage = wave_stage(c);
  if (c.ok) {
    // values past those requested ahead, straight from their old pages, eight loads in flight per lane; keys from LDS
    constexpr int kVFlight = 8;
    for (int t0 = kVAhead * 64 * WD; t0 < m * kChunks; t0 += kVFlight * step) {
      f4 x[kVFlight];
#pragma unroll
      for (int k = 0; k < kVFlight; ++k) {
        const int t = min(t0 + k * step + t_own, m * kChunks - 1), i = t / kChunks, ch = t % kChunks;
        x[k] = *(const f4*)(pool + (size_t)c.chain[i >> 4] * kPageBytes +
                            (size_t)(DT == DYNAKV_F32 ? v_index32(i & 15, 4 * ch) : v_index16(i & 15, 8 * ch)) * kEs);
      }
#pragma unroll
      for (int k = 0; k < kVFlight; ++k) {
        const int t = t0 + k * step + t_own;
        if (t < m * kChunks) *(f4*)split_vdest<DT>(pool, c, t / kChunks, t % kChunks) = x[k];
      }
    }
    for (int t = t_own; t < m * kChunks; t += step) {
      const int q = t / kChunks, ch = t % kChunks;
      const int i = c.perm[q];
      const int r = q < nS ? q : q - nS;
      const int dpage = c.newpg[(q < nS ? 0 : pS) + (r >> 4)];
      const size_t off = (size_t)(DT == DYNAKV_F32 ? k_index32(r & 15, 4 * ch) : k_index16(r & 15, 8 * ch)) * kEs;
      *(uint4*)(pool + (size_t)dpage * kPageBytes + off) = *(const uint4*)(stage + (size_t)i * kRowBytes<DT> + ch * 16);
    }
    if (t_own < need) v.pnext[(size_t)u * v.Pcap + c.newpg[t_own]] = (t_own == pS - 1 || t_own == need - 1) ? -1 : c.newpg[t_own + 1];
    for (int i = t_own; i < m; i += step) {
      const int q = c.inv[i];
      const int r = q < nS ? q : q - nS;
      const int dpage = c.newpg[(q < nS ? 0 : pS) + (r >> 4)];
      v.ppos[((size_t)u * v.Pcap + dpage) * kPageTokens + (r & 15)] = c.pos[i];
    }
  }
  for (int d = t_own; d < kHeadDim; d += step) {
    store_centroid(v, u, j, d, c.rA[d]);
    if (idM >= 0) store_centroid(v, u, idM, d, c.rB[d]);
  }
  if (w != 0) return;
  if (c.ok && lane < kInlinePages) {
    v.cpg[(cbase + j) * kInlinePages + lane] = lane < pS ? c.newpg[lane] : -1;
    v.cpg[(cbase + idM) * kInlinePages + lane] = lane < pM ? c.newpg[pS + lane] : -1;
  }
  if (lane == 0) {
    v.cn[cbase + j] = nS; v.csz[cbase + j] = nS; v.cb[cbase + j] = 0; v.cflag[cbase + j] = 0; v.cM2[cbase + j] = c.m2[0];
    if (c.ok) {
      v.ctail[cbase + j] = c.newpg[pS - 1];
      v.cn[cbase + idM] = nM; v.csz[cbase + idM] = nM; v.cb[cbase + idM] = 0; v.cflag[cbase + idM] = 0; v.cM2[cbase + idM] = c.m2[1];
      v.ctail[cbase + idM] = c.newpg[pS + pM - 1];
      v.in_req[cbase + idM] = 0;
    }
  }
}

// Plan of one unit's splits, made from the list of its flagged clusters (at most 64 of them).
constexpr int kFreeAhead = 24;
struct SplitPlan {
  int id[64], req[64], cb[64], m[64];   // the flagged clusters
  alignas(16) int pg[64][kInlinePages]; // their first pages
  int cand[64];                          // positions in the list, in the order of the splits
  int n_cand, forced, fast;
  int f64;                               // a cluster is larger than two contexts' rows: the statistics of all are float64 sums of float64 squares
  int M, top, bump;                      // the unit's counters while the plan is carried out
  int fl[kFreeAhead], fl_base;           // top of the free-page stack, read ahead: fl[k] = entry fl_base - 1 - k
};

// LDS of one unit's splits: `raw` holds either the workgroup-wide split or the wavefronts' contexts and staged keys.
template <int DT>
constexpr size_t kWaveRaw = kWaveSplits * sizeof(WaveCtx) + (size_t)kLoneRows<DT> * kRowBytes<DT>;
static_assert(kWaveSplits * kWaveStage <= kLoneRows<DYNAKV_F16> * kRowBytes<DYNAKV_F16> && kWaveSplits * kWaveStage <= kLoneRows<DYNAKV_F32> * kRowBytes<DYNAKV_F32>, "rows of four contexts");
template <int DT>
constexpr size_t kSplitRaw = sizeof(SplitSmem) > kWaveRaw<DT> ? sizeof(SplitSmem) : kWaveRaw<DT>;
static_assert((kWaveSplits - 1) * sizeof(WaveCtx) >= kWaveSplits * kHeadDim * sizeof(double), "a cluster split alone keeps its partial sums in the contexts it does not use");
struct SplitWork {
  SplitPlan pl;
  long long s_tot;
  int s_min;
  int nf0, M0, npre;                     // left by plan_finish: flagged clusters, clusters, splits decided ahead ...
  int wide;                              // ... and whether they are wide
  int ready;                             // set (release) once the plan is in place, for wavefronts that do not share a
                                         // barrier with the one that made it
  int flagged0[64];                      // for plan_fetch_early: the flagged list before the append
};
// Candidate k of a round of wavefront splits is handled by wavefront k and held in context ctx_of(k): the
// contexts of the first candidates lie at the far end of `raw`, clear of what a caller of split_predecide may
// still be using at the front.
__device__ __forceinline__ int ctx_of(int k) { return kWaveSplits - 1 - k; }

// What the plan needs about one flagged cluster; id < 0: no cluster.
struct PlanEntry {
  int id, req, cb, m;
};
// Fetches it for flagged cluster `c` (slot i of the plan), into the plan and for the calling lane.
__device__ __forceinline__ PlanEntry plan_fetch(const View& v, size_t cbase, SplitPlan& pl, int i, int c) {
  const int b = v.cb[cbase + c];
  const int4 pg = *(const int4*)&v.cpg[(cbase + c) * kInlinePages];
  const int4 pg2 = *(const int4*)&v.cpg[(cbase + c) * kInlinePages + 4];
  const PlanEntry e{c, v.in_req[cbase + c], b, v.cn[cbase + c] + b};
  pl.id[i] = e.id; pl.req[i] = e.req; pl.cb[i] = e.cb; pl.m[i] = e.m;
  *(int4*)&pl.pg[i][0] = pg; *(int4*)&pl.pg[i][4] = pg2;
  return e;
}
// Everything the page allocation will need, requested in the same round trip: entry k of the read-ahead.
__device__ __forceinline__ void plan_fetch_pages(const View& v, int u, SplitPlan& pl, int k, int top, int M0) {
  if (k < top) pl.fl[k] = v.freelist[(size_t)u * v.Pcap + top - 1 - k];
  if (k == 0) { pl.M = M0; pl.top = top; pl.bump = v.bump[u]; pl.fl_base = top; }
}

// The order of the unit's splits, by one whole wavefront: lane i < nf0 <= 64 brings flagged cluster i (e.id < 0 in
// the other lanes); pl.M, pl.top and pl.bump are in place.  Delayed splits first: flagged clusters of the active
// set (all flagged ones if nothing is buffered) in ascending id; then, if the remaining buffers hold B_max
// entries, the fullest of them (lowest id among equals).
template <int DT>
__device__ inline void plan_splits(const View& v, SplitPlan& pl, const PlanEntry& e) {
  const int lane = threadIdx.x & 63;
  const bool have = e.id >= 0;
  const bool delayed = have && (v.Bmax == 0 || e.req != 0);
  const unsigned long long dmask = __ballot(delayed);
  int rank = 0;
  for (unsigned long long mm = dmask; mm; mm &= mm - 1) {          // ids are distinct: rank = smaller ids
    const int other = __builtin_amdgcn_readlane(e.id, __ffsll((long long)mm) - 1);
    rank += other < e.id ? 1 : 0;
  }
  if (delayed) pl.cand[rank] = lane;
  int nc = __popcll(dmask), forced = 0, fl = -1;
  if (v.Bmax > 0) {
    const bool rest = have && !delayed;
    const int total = wave_sum(rest ? e.cb : 0);
    const int bcb = wave_max(rest ? e.cb : -1);                                  // the fullest buffer ...
    const int bid = wave_min(rest && e.cb == bcb ? e.id : 0x7ffffffe);           // ... of the lowest id among equals
    const unsigned long long who = __ballot(rest && e.cb == bcb && e.id == bid);
    const int bl = who ? __ffsll((long long)who) - 1 : 0;
    if (bcb >= 0 && total >= v.Bmax) {
      if (lane == 0) pl.cand[nc] = bl;
      fl = bl; ++nc; forced = 1;
    }
  }
  // the wavefronts take the plan if every cluster fits the staging rows (those that need more than one wavefront's are split
  // alone, see split_run) and no capacity limit can be hit
  const bool isc = delayed || lane == fl;
  const int largest = wave_max(isc ? e.m : 0);
  const int pages = wave_sum(isc ? (e.m + kPageTokens - 1) / kPageTokens + 1 : 0);
  if (lane == 0) {
    pl.n_cand = nc; pl.forced = forced;
    pl.f64 = largest > 2 * kSmallRows<DT>;
    pl.fast = largest <= kLoneRows<DT> && pl.M + nc <= v.Mcap && pages <= pl.top + (v.Pcap - pl.bump);
  }
}
// How many of the plan's splits base, base + 1, .. < nc are carried out side by side: up to kWaveSplits clusters of one
// context's rows each, up to half as many if one of them needs two contexts' (wide), a larger one alone.
template <int DT>
__device__ __forceinline__ int split_run(const SplitPlan& pl, int base, int nc, bool& wide) {
  wide = false;
  int n = 0;
#pragma unroll 1
  for (; n < kWaveSplits && base + n < nc; ++n) {
    const int m = pl.m[pl.cand[base + n]];
    if (m > 2 * kSmallRows<DT>) return n == 0 ? 1 : n;
    const bool w = wide || m > kSmallRows<DT>;
    if (w && n >= kWaveSplits / 2) break;
    wide = w;
  }
  return n;
}

// Hands candidate `at` of the plan to context x (one wavefront).  lone: it has all the staging rows.
__device__ __forceinline__ void wave_take(const View& v, int u, const SplitPlan& pl, int at, WaveCtx* wc, int x, bool wide, bool lone,
                                          int lane) {
  WaveCtx& c = wc[x];
  const int m = pl.m[at];
  if (lane == 0) { c.j = pl.id[at]; c.m = m; wave_place_stage(wc, x, wide, lone); }
  if (lane < kInlinePages) c.chain[lane] = pl.pg[at][lane];
  wave_sync();
  if (m > kInlinePages * kPageTokens && lane == 0)         // pages past the inline table (only a cluster split alone has any)
    for (int k = kInlinePages; k * kPageTokens < m; ++k) c.chain[k] = v.pnext[(size_t)u * v.Pcap + c.chain[k - 1]];
  wave_sync();
}

// ---- head start for split_unit inside a kernel that has just selected the active set and appended a token ----
// The plan's inputs are requested before the append is committed (plan_fetch_early, first wavefront, after the
// selection), corrected for what the append changed and turned into the plan right after it (plan_finish); the
// first splits of the plan can then be decided (split_predecide, one wavefront each) while the rest
// of the workgroup is busy elsewhere: deciding only reads the index.
struct PlanEarly {
  int id, req, cb, cn;     // lane i < nflag: flagged cluster i; lane nflag: the cluster the append may flag
  int fl0;                 // free-page stack entry top - 1 - lane
  int4 pg, pg2;
};
// flagged0: entry `lane` of the flagged list; s: the unit before the append; ja: the cluster the append goes to (< 0: no append).
// selbits: the active set of the selection that has just run, one bit per cluster (LDS); null: the flags in memory say it.
__device__ __forceinline__ PlanEarly plan_fetch_early(const View& v, int u, int flagged0, const UnitState& s, int ja, int lane,
                                                      const unsigned* selbits) {
  const size_t cbase = (size_t)u * v.Mcap;
  PlanEarly e{-1, 0, 0, 0, 0, int4{-1, -1, -1, -1}, int4{-1, -1, -1, -1}};
  const int c = lane < s.nflag ? flagged0 : lane == s.nflag ? ja : -1;
  if (c >= 0 && s.nflag <= 64) {
    e.id = c; e.cb = v.cb[cbase + c]; e.cn = v.cn[cbase + c];
    e.req = selbits ? (int)((selbits[c >> 5] >> (c & 31)) & 1u) : (int)v.in_req[cbase + c];
    e.pg = *(const int4*)&v.cpg[(cbase + c) * kInlinePages];
    e.pg2 = *(const int4*)&v.cpg[(cbase + c) * kInlinePages + 4];
  }
  if (lane <= kFreeAhead && lane < s.top) e.fl0 = v.freelist[(size_t)u * v.Pcap + s.top - 1 - lane];
  return e;
}
// First wavefront, after the append (a: what it did, sz0: entries of cluster ja before it; appended: there was one).  Leaves the
// plan in wk.pl and wk.nf0 / M0 / npre (npre <= max_pre = splits to decide ahead).  True if the plan needs what the append has
// stored (the caller waits for it before anybody reads on).
template <int DT>
__device__ __forceinline__ bool plan_finish(const View& v, SplitWork& wk, PlanEarly e, const UnitState& s, int ja, bool appended,
                                            const AppendResult& a, int sz0, int max_pre) {
  SplitPlan& pl = wk.pl;
  const int lane = threadIdx.x & 63;
  int nf = s.nflag, top = s.top, bump = s.bump;
  if (appended && a.ok) {
    nf = a.nflag; top = a.top; bump = a.bump;
    const bool newflag = nf > s.nflag;
    if (newflag ? lane == s.nflag : (lane < s.nflag && e.id == ja)) {
      e.cb = newflag ? 1 : e.cb + 1;                     // the token went to the buffer of a flagged cluster
      if (a.slot == 0) {                                 // and opened a page
        const int k = sz0 / kPageTokens;
        if (k == 0) e.pg.x = a.page;
        else if (k == 1) e.pg.y = a.page;
        else if (k == 2) e.pg.z = a.page;
        else if (k == 3) e.pg.w = a.page;
        else if (k == 4) e.pg2.x = a.page;
        else if (k == 5) e.pg2.y = a.page;
        else if (k == 6) e.pg2.z = a.page;
        else if (k == 7) e.pg2.w = a.page;
      }
    }
  }
  if (lane >= nf) e.id = -1;
  const int fl = __shfl(e.fl0, min(lane + (s.top - top), 63));    // the append took at most the top page
  if (lane == 0) {
    wk.nf0 = nf; wk.M0 = s.M; wk.npre = 0;
    pl.fast = 0; pl.M = s.M; pl.top = top; pl.bump = bump; pl.fl_base = top;
  }
  if (nf == 0) return false;
  if (nf > 64) return true;
  if (lane < kFreeAhead && lane < top) pl.fl[lane] = fl;
  if (e.id >= 0) {
    pl.id[lane] = e.id; pl.req[lane] = e.req; pl.cb[lane] = e.cb; pl.m[lane] = e.cn + e.cb;
    *(int4*)&pl.pg[lane][0] = e.pg; *(int4*)&pl.pg[lane][4] = e.pg2;
  }
  wave_sync();
  plan_splits<DT>(v, pl, PlanEntry{e.id, e.req, e.cb, e.cn + e.cb});
  wave_sync();
  bool wide = false;
  const int n = pl.fast ? min(split_run<DT>(pl, 0, pl.n_cand, wide), max_pre) : 0;
  if (lane == 0) {
    wk.wide = wide;
    wk.npre = n > 0 && pl.m[pl.cand[0]] <= 2 * kSmallRows<DT> ? n : 0;
  }
  return pl.n_cand > 0 || !pl.fast;
}
// Wavefront k < wk.npre decides split k of the plan and computes the children's statistics, into context
// ctx_of(k) of `raw`; pre_v: the values requested ahead, for the same wavefront to hand to split_unit.
template <int DT>
__device__ inline void split_predecide(const View& v, int u, unsigned char* raw, const SplitWork& wk, int k,
                                       uint4 (&pre_v)[kVAhead]) {
  WaveCtx& c = ((WaveCtx*)raw)[ctx_of(k)];
  // the split is the longest chain of dependent steps of its unit: it goes ahead of the wavefront that streams pages
  // on the same SIMD (the tiles that one does not take meanwhile go to the other wavefronts)
  __builtin_amdgcn_s_setprio(3);
  wave_take(v, u, wk.pl, wk.pl.cand[k], (WaveCtx*)raw, ctx_of(k), wk.wide != 0, false, threadIdx.x & 63);
  wave_split_decide<DT>(v, u, c, 0, 1, wk.pl.f64 != 0, c.cB, pre_v);
  __builtin_amdgcn_s_setprio(0);
}

// First wavefront: ids and pages for the decided splits (contexts ctx_of(0 .. n-1)), in the order of the plan.
__device__ __forceinline__ void split_assign(const View& v, int u, WaveCtx* wc, SplitPlan& pl, int n) {
  const int lane = threadIdx.x & 63;
  int M = pl.M, top = pl.top, bump = pl.bump;
  const int fl_base = pl.fl_base;
#pragma unroll 1
  for (int w = 0; w < n; ++w) {
    WaveCtx& cw = wc[ctx_of(w)];
    if (!cw.ok) continue;
    const int need = (cw.nS + kPageTokens - 1) / kPageTokens + (cw.m - cw.nS + kPageTokens - 1) / kPageTokens;
    const int from_free = min(need, top);
    if (lane < need) {
      const int ra = fl_base - (top - lane);             // pl.fl holds the stack as it was at fl_base
      cw.newpg[lane] = lane >= from_free ? bump + (lane - from_free)
                       : (ra >= 0 && ra < kFreeAhead) ? pl.fl[ra]
                                                       : v.freelist[(size_t)u * v.Pcap + top - 1 - lane];
    }
    if (lane == 0) cw.idM = M;
    M += 1; top -= from_free; bump += need - from_free;
  }
  if (lane == 0) { pl.M = M; pl.top = top; pl.bump = bump; }
}
static_assert(kWavePages + 2 <= 64, "one lane per page of the children");
// First wavefront, once the n splits are committed and nothing reads the parents' pages any more: recycles them.
// base: place of the first of them in the plan (a forced split is the plan's last entry and is counted as forced
// only if it was carried out).
__device__ __forceinline__ void split_recycle(const View& v, int u, const WaveCtx* wc, SplitPlan& pl, int n, int base) {
  const int lane = threadIdx.x & 63;
  int top = pl.top, done = 0, failed = 0, forced = 0;
#pragma unroll 1
  for (int w = 0; w < n; ++w) {
    const WaveCtx& cw = wc[ctx_of(w)];
    if (!cw.ok) { ++failed; continue; }
    ++done;
    if (pl.forced && base + w == pl.n_cand - 1) forced = 1;
    const int npg = (cw.m + kPageTokens - 1) / kPageTokens;
    if (lane < npg) v.freelist[(size_t)u * v.Pcap + top + lane] = cw.chain[lane];
    top += npg;
  }
  if (lane == 0) {
    pl.top = top;
    if (done) { pl.fl_base = -(1 << 30); count(v, u, 0, done); }   // the stack has changed: what was read ahead no longer applies
    if (failed) count(v, u, 1, failed);
    if (forced) count(v, u, 2, 1);
  }
}

// All splits of unit u that are due (Algorithm 1, decode block: delayed splits, then the forced one), by the
// first kSplitThreads threads of the workgroup; no other thread of the workgroup may still be running.
// raw: kSplitRaw<DT> bytes of LDS, 16-byte aligned.  prepared: plan_finish and split_predecide have run and the
// caller has assigned (split_assign) and committed (wave_split_commit) the wk.npre splits decided ahead, with a
// barrier since; their parents' pages are still to be recycled.
template <int DT>
__device__ __forceinline__ void split_unit(const View& v, int u, unsigned char* raw, SplitWork& wk, bool prepared) {
  constexpr int NT = kSplitThreads;
  SplitPlan& pl = wk.pl;
  int& s_min = wk.s_min;
  long long& s_tot = wk.s_tot;
  SplitSmem& s = *(SplitSmem*)raw;
  WaveCtx* const wc = (WaveCtx*)raw;
  const int tid = threadIdx.x;
  const size_t cbase = (size_t)u * v.Mcap;
  int M0, nf0, npre = 0;
  if (prepared) {
    M0 = wk.M0; nf0 = wk.nf0; npre = wk.npre;
    if (nf0 == 0) return;
  } else {
    // requested together with the flag count, so that the plan below starts one round trip earlier
    const int c_ahead = tid < min(64, v.Mcap) ? v.flist[cbase + tid] : 0;
    const int top_ahead = v.free_top[u];
    M0 = v.M[u];
    nf0 = v.nflag[u];
    if (nf0 == 0) return;
    if (nf0 <= 64) {
      PlanEntry e{-1, 0, 0, 0};
      if (tid < nf0) e = plan_fetch(v, cbase, pl, tid, c_ahead);
      if (tid >= 64 && tid < 64 + kFreeAhead) plan_fetch_pages(v, u, pl, tid - 64, top_ahead, M0);
      __syncthreads();
      if (tid < 64) plan_splits<DT>(v, pl, e);
      __syncthreads();
    }
  }

  // ---- the plan's splits, up to four side by side, one per wavefront
  if (nf0 <= 64) {
    if (pl.fast) {
      const int wave = tid >> 6, lane = tid & 63;
      const int nc = pl.n_cand;
      if (npre > 0) {                      // committed by the caller
        if (wave == 0) split_recycle(v, u, wc, pl, npre, 0);
        __syncthreads();
      }
#pragma unroll 1
      for (int base = npre, n; base < nc; base += n) {
        bool wide;
        n = split_run<DT>(pl, base, nc, wide);
        // one split, and not a small one: by all wavefronts together (24 float16 entries: 27 us by one, 25 by four)
        const int W = n == 1 && pl.m[pl.cand[base]] > 16 ? kWaveSplits : 1;
        const int w = W == 1 ? 0 : wave, k = W == 1 ? wave : 0;                           // this wavefront's place and candidate
        const bool mine = k < n;
        uint4 vahead[kVAhead];
        WaveCtx& c = wc[ctx_of(k)];
        if (mine && w == 0) wave_take(v, u, pl, pl.cand[base + k], wc, ctx_of(k), wide, W > 1, lane);
        if (W > 1) lds_barrier();
        if (mine) wave_split_decide<DT>(v, u, c, w, W, pl.f64 != 0, W > 1 ? (double*)raw : c.cB, vahead);
        lds_barrier();
        if (wave == 0) split_assign(v, u, wc, pl, n);            // ids and pages, in the order of the splits
        lds_barrier();
        if (mine) wave_split_commit_ahead<DT>(v, u, c, w, W, vahead);
        for (int i = 0; i < n; ++i) wave_split_commit<DT>(v, u, wc[ctx_of(i)], W, wave, kWaveSplits);
        lds_barrier();                                           // (every read of the parents' pages has its value)
        if (wave == 0) split_recycle(v, u, wc, pl, n, base);     // the parents' pages are recycled only now
        if (base + n < nc) __syncthreads();                      // the next splits read the stack of free pages
      }
      if (wave == 0 && nc > 0) {           // (no split: list and counters are as they were)
        if (lane < nc) pl.id[pl.cand[lane]] = -1;
        wave_sync();
        const int id = lane < nf0 ? pl.id[lane] : -1;
        const unsigned long long keep = __ballot(id >= 0);
        if (id >= 0) v.flist[cbase + __popcll(keep & ((1ull << lane) - 1ull))] = id;
        if (lane == 0) { v.nflag[u] = __popcll(keep); v.M[u] = pl.M; v.free_top[u] = pl.top; v.bump[u] = pl.bump; }
      }
      return;
    }
  }

  // ---- general path: one split at a time by the whole workgroup
  if (tid == 0) { s.M = M0; s.nflag = nf0; s.a_top = v.free_top[u]; s.a_bump = v.bump[u]; }
  // One loop, one call site: first the delayed splits (flagged clusters that the last retrieval selected, in
  // ascending id), then, once, the forced split of the fullest buffer if the buffers hold B_max entries.  Both
  // searches walk the list of flagged clusters, which holds a handful of ids.
  __syncthreads();
  int cursor = 0;
  bool forced_done = false;
  while (true) {
    int j = -1, pos = -1;
    const int nf = s.nflag;
    if (!forced_done) {
      if (tid == 0) s_min = 0x7FFFFFFF;
      __syncthreads();
      for (int i = tid; i < nf; i += NT) {
        const int c = v.flist[cbase + i];
        if (c >= cursor && c < M0 && (v.Bmax == 0 || v.in_req[cbase + c])) atomicMin(&s_min, c);
      }
      __syncthreads();
      if (s_min != 0x7FFFFFFF) j = s_min;
      __syncthreads();
      if (j >= 0) cursor = j + 1;
    }
    if (j < 0) {
      if (forced_done) break;
      forced_done = true;
      if (!(v.Bmax > 0 && nf > 0)) break;
      if (tid == 0) s_tot = 0;
      __syncthreads();
      double bv = -1.0; int bi = -1;
      long long tot = 0;
      for (int i = tid; i < nf; i += NT) {
        const int c = v.flist[cbase + i];
        const int b = v.cb[cbase + c];
        tot += b;
        if ((double)b > bv || ((double)b == bv && c < bi)) { bv = (double)b; bi = c; }
      }
      if (tot) atomicAdd((unsigned long long*)&s_tot, (unsigned long long)tot);
      block_argmax(bv, bi, s.sv, s.si);
      const int arg = s.si[0];
      const long long total = s_tot;
      __syncthreads();
      if (!(arg >= 0 && total >= v.Bmax)) break;
      j = arg;
    }
    // the cluster's place in the list of flagged clusters
    if (tid == 0) s_min = -1;
    __syncthreads();
    for (int i = tid; i < nf; i += NT)
      if (v.flist[cbase + i] == j) s_min = i;
    __syncthreads();
    pos = s_min;
    __syncthreads();
    split_cluster<DT>(v, u, j, pos, s);
    if (forced_done && tid == 0 && s.did_split) count(v, u, 2, 1);     // a forced split counts once carried out
    __syncthreads();
    if (forced_done) break;
  }
  __syncthreads();
  if (tid == 0) { v.M[u] = s.M; v.nflag[u] = s.nflag; v.free_top[u] = s.a_top; v.bump[u] = s.a_bump; }
}

}  // namespace

}  // namespace dynakv
