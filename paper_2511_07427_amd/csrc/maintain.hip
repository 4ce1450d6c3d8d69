// Decode, second half of a step (Algorithm 1, decode block; Section 4.2):
//   append_kernel - nearest cluster (its own scan of the table, or the per-block results the score kernel of a
//                   whole-step call left), UpdateVar, threshold test, AddEntry + UpdateStats or buffer + flag;
//                   in a whole-step call the due splits follow in the same launch
//   split_kernel  - delayed splits of flagged clusters in the active set, then the forced split
//   extend_batch_kernel, extend_kernel - a further chunk of the prompt, entry by entry, with every split done at once
// One workgroup per unit; each unit's record is touched by that workgroup only.  All decisions are
// taken on float64 values, or on float32 ones where their rounding could not change them; ties to the lowest index.
#include "split.hpp"
#include "score.hpp"

namespace dynakv {

namespace {

// ------------------------------------------------------------------------------------------- append
// How the kernel finds the nearest cluster:
//   kScanMean  its own float64 scan of the float32 means
//   kPreMean   the score kernel of the same step has left the nearest cluster of every block of 256 clusters
//              (float64, float32 means)
//   kPreZ      a matrix-core pass (the score kernel of the same step, or a pass of its own launched before this
//              kernel) has left z_j = <k, r~_j> - |r~_j|^2 / 2 of every cluster of the 16-bit search copy: the
//              largest is taken if the runner-up lies beyond the float32 error bound, otherwise the clusters within
//              the bound are compared in float64
// SPLIT: the unit's due splits follow in the same launch (the rest of a decode step on the separate-kernel path).
enum { kScanMean = 0, kPreMean = 1, kPreZ = 2 };
template <int DT, bool ON>
struct SplitLds {
  alignas(16) unsigned char raw[kSplitRaw<DT>];
  SplitWork wk;
};
template <int DT>
struct SplitLds<DT, false> {};
template <int DT, int MODE, bool SPLIT>
__global__ __launch_bounds__(256) void append_kernel(View v, const void* kin, const void* vin) {
  static_assert(kSplitThreads == 256, "split_unit is run by this kernel's whole workgroup");
  __shared__ double kd[kHeadDim];
  __shared__ double sv[16];
  __shared__ int si[16];
  __shared__ float s2[16];
  __shared__ SplitLds<DT, SPLIT> sp;
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const float* R = unit_R(v, u);
  f4 row[8];
  if constexpr (MODE == kScanMean)
    if ((size_t)(tid | 63) * kHeadDim < v.Rstride) load_centroid_head(R, tid, row);     // requested before anything else
  // what the first wavefront will need for the append and for the plan of the splits
  const UnitState us = load_unit(v, u);
  EntryBits entry{uint2{0, 0}, uint2{0, 0}};
  int flagged0 = 0;
  if (tid < 64) {
    entry = load_entry<DT>(kin, vin, u, lane);
    if constexpr (SPLIT) flagged0 = lane < v.Mcap ? v.flist[(size_t)u * v.Mcap + lane] : 0;
  }
  const int M = us.M;
  const bool room = us.N < v.Ncap && M > 0;             // otherwise refused (workgroup-uniform); due splits still run
  int j = -1;
  if (room) {
    float k2 = 0.f;
    if (tid < kHeadDim) {
      const float kf = load_elem(kin, (size_t)u * kHeadDim + tid, DT);
      kd[tid] = (double)kf;
      k2 = kf * kf;
    }
    if constexpr (MODE == kPreZ) {
      // the matrix-core pass has left best / runner-up per 64 clusters
      float zb = -__builtin_inff(), z2 = -__builtin_inff();
      int jb = -1;
      const size_t wbase = (size_t)u * v.NB * 4;
      for (int w = tid; w * 64 < M; w += 256) merge_best2(zb, jb, z2, v.near_zb[wbase + w], v.near_zj[wbase + w], v.near_z2[wbase + w]);
      const float rmax2 = __int_as_float(v.rmax2[u]);
      for (int o = 32; o > 0; o >>= 1) k2 += __shfl_xor(k2, o);
      wave_best2(zb, jb, z2);
      if (lane == 0) { const int w = tid >> 6; sv[w] = (double)zb; si[w] = jb; s2[w] = z2; s2[8 + w] = k2; }
      lds_barrier();
      const float kn = __builtin_sqrtf(s2[8] + s2[9]) * 1.0001f;
      j = nearest_decide<256>(v, u, M, kn, rmax2, v.zdist + (size_t)u * v.Mcap, unit_Rq(v, u), kd, sv, si, s2);
    } else {
      __syncthreads();
      double best = __builtin_inf();
      int arg = -1;
      if constexpr (MODE == kPreMean) {
        for (int b = tid; b * 256 < M; b += 256) {          // blocks past the last cluster hold nothing of this step
          const double d = v.near_d[(size_t)u * v.NB + b];
          const int jj = v.near_j[(size_t)u * v.NB + b];
          if (arg < 0 || d < best || (d == best && jj < arg)) { best = d; arg = jj; }
        }
      } else {
        // nearest centre (squared Euclidean distance); lane = cluster, 16 contiguous bytes per lane and load
        for (int jj = tid; jj < M; jj += 256) {
          double dist[1];
          if (jj != tid) load_centroid_head(R, jj, row);
          centroid_sums<1>(R, jj, row, dist, [&](int d, float rv, double (&acc)[1]) __attribute__((always_inline)) {
            const double t = kd[d] - (double)rv;
            acc[0] = fma(t, t, acc[0]);
          });
          if (dist[0] < best || arg < 0) { best = dist[0]; arg = jj; }
        }
      }
      j = block_argmin<256>(best, arg, sv, si);
    }
  }
  // the append and the plan of the splits, by the first wavefront: what both ask of memory travels together
  if (tid < 64) {
    ClusterFetch cf{float2{0.f, 0.f}, 0};
    PlanEarly pe{};
    if (room) cf = fetch_cluster(v, u, j, us.top, lane);
    if constexpr (SPLIT) pe = plan_fetch_early(v, u, flagged0, us, j, lane, nullptr);
    AppendResult res{};
    int sz0 = 0;
    if (room) {
      const ClusterState cs = cluster_state(cf, us.top);
      res = append_wave<DT>(v, u, j, us, cs, entry, lane);
      sz0 = cs.cn + cs.cb;
    } else if (lane == 0) {
      v.err[u] |= DYNAKV_ERR_TOKENS;
    }
    if constexpr (SPLIT)
      if (plan_finish<DT>(v, sp.wk, pe, us, j, room, res, sz0, 0)) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the entry is in place
  }
  if constexpr (SPLIT) {
    lds_barrier();
    split_unit<DT>(v, u, sp.raw, sp.wk, true);
  }
}

// ------------------------------------------------------------------------------------------- chunked prefill
// Adaptive clustering through a long prefill (Section 7, Discussion 1): one workgroup per unit walks the chunk's n
// entries in order; each entry is assigned to its nearest cluster (matrix cores + float64 where needed for the
// 16-bit search copy, float64 scan for float32 means), appended with UpdateVar and the threshold test, and a
// flagged cluster is split at once (the view's B_max is 0).  K, V: [U][n][128].
// Entry t + 1 depends on what entry t did, so a unit's time is a chain, and what counts is what an entry waits for.
//
// extend_batch_kernel (16-bit search copy): up to sixteen entries are the rows of one pass over the table (z_j = <k, r~_j> -
// |r~_j|^2 / 2 of each entry and cluster, kept in LDS), and the records and centroids of the clusters that they are likely to join are
// fetched together into slots of LDS.  The entries are then taken one after another by the first wavefront with no
// trip to memory: nearest cluster from the entry's row of z (float64 where the runner-up lies within the rounding bound), UpdateVar and
// threshold on the slot, and one matrix product of the new centroid with the entries to come, which corrects their z of that
// cluster.  A cluster outside the slots is fetched when it is met; a flag calls the whole workgroup for the split, after which the
// z of the two clusters that it leaves are put right in the same way (a split of any other cluster ends the batch).  LDS holds z
// of kExtendClusters clusters for two entries, of an eighth of that for sixteen.
// 256 units, 256 clusters, 1024 entries (163 splits a unit): 10.3 -> 4.8 ms, of which an entry takes 2.1 us where nothing is
// flagged (6.6).
//
// extend_kernel (float32 means; more clusters than that; one or two entries): one entry per pass over the table, the table in batches of four
// tiles per wavefront with the next batch in flight.  It is the faster one where a pass serves a single entry: 8 units of 8000 clusters, 64
// entries 2.93 ms against 3.67, of 5000 clusters, two entries a pass, 1.70 in batches against 2.2; a lone entry to one unit of 2000 clusters
// 65 us against 74 with the import before it, two of them 77 against 82, three 91 against 86.
constexpr int kExtendBatch = 16, kExtendSpare = 8, kExtendZ = 10240;      // entries per batch, slots beyond them, floats of z
constexpr int kExtendRoom = kExtendBatch;                                 // clusters that a batch may add
constexpr int kExtendLeast = 3;                                           // entries that warrant a batch
constexpr int kExtendClusters = kExtendZ / 2 - kExtendRoom - 4;
static_assert(kSplitThreads == 2 * kHeadDim, "one coordinate of the key or of the value per thread");

// What the extension holds of a cluster in LDS.
struct ExtendSlot {
  float2 r[64];
  double m2;
  int id, cn, cb, ctail, cflag, pad_;
};

// Best and runner-up of row[0 .. M) (padded to a multiple of four with -inf), by one wavefront; every lane gets them.
__device__ __forceinline__ void row_best2(const float* row, int M, int lane, float& zb, int& jb, float& z2) {
  zb = -__builtin_inff(); z2 = -__builtin_inff(); jb = -1;
#pragma unroll 1
  for (int j0 = 4 * lane; j0 < M; j0 += 256) {
    const f4 z = *(const f4*)(row + j0);
    const float hi01 = fmaxf(z[0], z[1]), lo01 = fminf(z[0], z[1]), hi23 = fmaxf(z[2], z[3]), lo23 = fminf(z[2], z[3]);
    const float hi = fmaxf(hi01, hi23), next = fmaxf(fminf(hi01, hi23), hi01 >= hi23 ? lo01 : lo23);
    const int at = j0 + (hi == z[0] ? 0 : hi == z[1] ? 1 : hi == z[2] ? 2 : 3);
    z2 = fmaxf(fminf(zb, hi), fmaxf(z2, next));
    if (jb < 0 || hi > zb) { zb = hi; jb = min(at, M - 1); }
  }
  wave_best2(zb, jb, z2);
}

template <int DT>
__global__ __launch_bounds__(256) void extend_batch_kernel(View v, const void* K, const void* V, int n) {
  static_assert(DT != DYNAKV_F32, "needs the 16-bit search copy");
  constexpr bool BF = DT == DYNAKV_BF16;
  __shared__ SplitLds<DT, true> sp;
  __shared__ __align__(16) float zs[kExtendZ];
  __shared__ __align__(16) ExtendSlot slot[kExtendBatch + kExtendSpare];
  __shared__ __align__(16) unsigned char rows[kExtendBatch][2][kHeadDim * 2];
  __shared__ __align__(16) uint32_t vec[2][kHeadDim / 2];
  __shared__ int s_rmax2, s_done, s_nflag, s_j, s_at, s_planned;
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, cl = lane & 15;
  const uint4* tiles = (const uint4*)unit_Rq(v, u);
  int t = 0;
#pragma unroll 1
  while (t < n) {
    UnitState us = load_unit(v, u);                    // (a full barrier lies behind the last store)
    const int M = us.M;
    if (us.N >= v.Ncap || M <= 0) {                    // workgroup-uniform
      if (tid == 0) v.err[u] |= DYNAKV_ERR_TOKENS;
      t = n;
      break;
    }
    if (M > kExtendClusters) break;
    int B = kExtendBatch;
    const int stride = (M + kExtendRoom + 3) & ~3;
    while (B > 1 && B * stride > kExtendZ) B >>= 1;
    const int nb = min(min(B, n - t), v.Ncap - us.N);
    // ---- the entries, and z of every cluster
    uint32_t x[kExtendBatch];
#pragma unroll
    for (int i = 0; i < kExtendBatch; ++i)
      x[i] = ((const uint16_t*)(tid < kHeadDim ? K : V))[((size_t)u * n + min(t + i, n - 1)) * kHeadDim + (tid & (kHeadDim - 1))];
    int fl = us.top - 1 - lane >= 0 ? v.freelist[(size_t)u * v.Pcap + us.top - 1 - lane] : -1;      // the top of the free stack
#pragma unroll
    for (int i = 0; i < kExtendBatch; ++i) ((uint16_t*)rows[i][0])[tid] = (uint16_t)x[i];
    if (tid == 0) s_rmax2 = 0;
    if (tid < kExtendSpare) slot[kExtendBatch + tid].id = -1;
    lds_barrier();
    uint4 A[4];                                        // rows = the entries (those past nb repeat others: nobody asks for them)
#pragma unroll
    for (int s = 0; s < 4; ++s) A[s] = *(const uint4*)(rows[cl][0] + 64 * s + 16 * lg);
    float kn = 0.f;                                    // |entry cl|
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint32_t ww[4] = {A[s].x, A[s].y, A[s].z, A[s].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float k = bits_value((ww[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu, DT);
        kn = fmaf(k, k, kn);
      }
    }
    kn = __builtin_sqrtf(rows_sum(kn)) * 1.0001f;
    const int ntile = (M + kTileClusters - 1) / kTileClusters;
    float rmax2 = 0.f;
#pragma unroll 1
    for (int T0 = wave * 4; T0 < ntile; T0 += 16) {
      uint4 b[4][4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) b[k][s] = tiles[((size_t)min(T0 + k, ntile - 1) * 4 + s) * 64 + lane];
      f4 acc[4], gram[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) { acc[k] = f4{0, 0, 0, 0}; gram[k] = f4{0, 0, 0, 0}; }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          acc[k] = mfma_k32<BF>(A[s], b[k][s], acc[k]);
          gram[k] = mfma_k32<BF>(b[k][s], b[k][s], gram[k]);
        }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float nrm2 = gram_diagonal(gram[k], lane);
        const int j = (T0 + k) * kTileClusters + cl;
        if (j >= M) continue;                          // (clusters of a repeated tile lie past M as well)
        rmax2 = fmaxf(rmax2, nrm2);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * lg + i < B) zs[(4 * lg + i) * stride + j] = acc[k][i] - 0.5f * nrm2;
      }
    }
    for (int i = tid; i < B * (kExtendRoom + 4); i += 256) {
      const int j = M + i % (kExtendRoom + 4);
      if (j < stride) zs[i / (kExtendRoom + 4) * stride + j] = -__builtin_inff();
    }
    atomicMax(&s_rmax2, __float_as_int(rmax2));        // (non-negative floats order like their bits)
    lds_barrier();
    // ---- the clusters that the entries would join as things stand: four entries per wavefront, fetched together
    int pj[4];
    ClusterFetch pf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float zb, z2;
      pj[i] = -1;
      if (4 * wave + i < nb) row_best2(zs + (4 * wave + i) * stride, M, lane, zb, pj[i], z2);
      if (pj[i] >= 0) pf[i] = fetch_cluster(v, u, pj[i], 0, lane);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ExtendSlot& sl = slot[4 * wave + i];
      if (pj[i] >= 0) {
        const ClusterState c = cluster_state(pf[i], 0);
        sl.r[lane] = c.r;
        if (lane == 0) { sl.m2 = c.m2; sl.cn = c.cn; sl.cb = c.cb; sl.ctail = c.ctail; sl.cflag = c.cflag; }
      }
      if (lane == 0) sl.id = pj[i];
    }
    lds_barrier();
    // ---- the entries one after another
    int r = 0, spare = kExtendBatch, Mz = M;             // entries done, slots in use, clusters in z (first wavefront)
    float rmax = __builtin_sqrtf(__int_as_float(s_rmax2)) * 1.0001f;
    while (true) {
      if (wave == 0) {
        const int top0 = us.top;
        // z of the clusters whose search copies are in vec: columns of even number the first, of odd number the second
        auto correct = [&](int ja, int jb) __attribute__((always_inline)) {
          uint4 b[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) b[s] = *(const uint4*)((const unsigned char*)vec[lane & 1] + 64 * s + 16 * lg);
          f4 acc = {0, 0, 0, 0}, gram = {0, 0, 0, 0};
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            acc = mfma_k32<BF>(A[s], b[s], acc);
            gram = mfma_k32<BF>(b[s], b[s], gram);       // row and column of the same parity: |r|^2
          }
          const float nrm2 = (cl & 1) ? gram[1] : gram[0];
          const int j = (cl & 1) ? jb : ja, e = 4 * lg + (cl >> 1);
          if (cl < 8 && e < B && j >= 0) zs[e * stride + j] = sel4(acc, cl >> 1) - 0.5f * nrm2;
          // (lanes 0 and 1 hold the two norms: the bound must be the same in every lane)
          const float na = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(nrm2), 0));
          const float nb2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(nrm2), 1));
          rmax = fmaxf(rmax, __builtin_sqrtf(fmaxf(na, nb2)) * 1.0001f);
          wave_sync();
        };
        if (r > 0) {                                     // back from a split: what it has left of cluster s_j and the one it may have added
          const int j = s_j, jn = us.M > Mz ? Mz : -1;
          const ClusterFetch fa = fetch_cluster(v, u, j, 0, lane), fb = fetch_cluster(v, u, max(jn, 0), 0, lane);
          vec[0][lane] = *(const uint32_t*)(unit_Rq(v, u) + rq_index(j, 2 * lane));
          vec[1][lane] = *(const uint32_t*)(unit_Rq(v, u) + rq_index(jn >= 0 ? jn : j, 2 * lane));
          const ClusterState ca = cluster_state(fa, 0), cb = cluster_state(fb, 0);
          ExtendSlot& sa = slot[s_at];
          sa.r[lane] = ca.r;
          if (lane == 0) { sa.m2 = ca.m2; sa.cn = ca.cn; sa.cb = ca.cb; sa.ctail = ca.ctail; sa.cflag = ca.cflag; }
          if (jn >= 0 && spare < kExtendBatch + kExtendSpare) {
            ExtendSlot& sb = slot[spare++];
            sb.r[lane] = cb.r;
            if (lane == 0) { sb.m2 = cb.m2; sb.cn = cb.cn; sb.cb = cb.cb; sb.ctail = cb.ctail; sb.cflag = cb.cflag; sb.id = jn; }
          }
          wave_sync();
          correct(j, jn);
          Mz = us.M;
        }
        bool planned = false;
        int j = -1, at = 0;
#pragma unroll 1
        for (; r < nb; ++r) {
          float* const row = zs + r * stride;
          float zb, z2;
          row_best2(row, Mz, lane, zb, j, z2);
          const EntryBits e{uint2{((const uint32_t*)rows[r][0])[lane], 0}, uint2{((const uint32_t*)rows[r][1])[lane], 0}};
          const float knr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(kn), r));
          const float eps = kAccBound * (knr * rmax + 0.5f * rmax * rmax) * 1.01f;
          if (!(zb - z2 > 2.f * eps)) {                  // several within the bound of the best: float64, the lowest id among equals
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (this batch's centroids are in place)
            const float2 kf = pair_value<DT>(e.k);
            double best = __builtin_inf();
            j = -1;
#pragma unroll 1
            for (int j0 = 0; j0 < Mz; j0 += 64)
#pragma unroll 1
              for (unsigned long long mk = __ballot(j0 + lane < Mz && row[min(j0 + lane, Mz - 1)] >= zb - 2.f * eps); mk; mk &= mk - 1) {
                const int c = j0 + (int)__builtin_ctzll(mk);
                const float2 rf = pair_value<DT>(uint2{*(const uint32_t*)(unit_Rq(v, u) + rq_index(c, 2 * lane)), 0});
                const double d0 = (double)kf.x - (double)rf.x, d1 = (double)kf.y - (double)rf.y;
                const double d = wave_sum_f64(fma(d0, d0, d1 * d1));
                if (d < best || j < 0) { best = d; j = c; }
              }
            j = max(j, 0);                               // (an entry that is not finite is near nothing: as dynakv_append has it)
            if (lane == 0) count(v, u, 7, 1);
          }
          // the cluster's slot: the first that holds it
          const unsigned long long hit = __ballot(lane < kExtendBatch + kExtendSpare && slot[min(lane, kExtendBatch + kExtendSpare - 1)].id == j);
          if (hit) at = (int)__builtin_ctzll(hit);
          else {
            if (spare == kExtendBatch + kExtendSpare) break;       // no slot left: the next batch begins with this entry
            at = spare++;
            const ClusterState c = cluster_state(fetch_cluster(v, u, j, 0, lane), 0);      // (not touched in this batch)
            slot[at].r[lane] = c.r;
            if (lane == 0) { slot[at].m2 = c.m2; slot[at].cn = c.cn; slot[at].cb = c.cb; slot[at].ctail = c.ctail; slot[at].cflag = c.cflag; slot[at].id = j; }
            wave_sync();
          }
          ExtendSlot& sl = slot[at];
          ClusterState c{sl.r[lane], sl.cn, sl.cb, sl.ctail, sl.cflag, -1, sl.m2};
          c.cn = __builtin_amdgcn_readfirstlane(c.cn); c.cb = __builtin_amdgcn_readfirstlane(c.cb);
          c.ctail = __builtin_amdgcn_readfirstlane(c.ctail); c.cflag = __builtin_amdgcn_readfirstlane(c.cflag);
          c.free_page = us.top > 0 ? __builtin_amdgcn_readlane(fl, top0 - us.top) : -1;
          const AppendResult a = append_wave<DT>(v, u, j, us, c, e, lane);
          if (!a.ok) continue;
          if (a.nflag > 0) {                             // its split follows at once
            if (us.nflag == 0) {                         // (the plan, where this flag is the only one)
              PlanEarly pe{-1, 0, 0, 0, __shfl(fl, min(lane + top0 - us.top, 63)), int4{-1, -1, -1, -1}, int4{-1, -1, -1, -1}};
              if (lane == 0) {
                const int4* pg = (const int4*)&v.cpg[((size_t)u * v.Mcap + j) * kInlinePages];
                pe.id = j; pe.cn = c.cn; pe.pg = pg[0]; pe.pg2 = pg[1];
              }
              plan_finish<DT>(v, sp.wk, pe, us, j, true, a, c.cn + c.cb, 0);
              planned = true;
            }
            us.nflag = a.nflag;
            ++r;
            break;
          }
          us.N += 1; us.top = a.top; us.bump = a.bump;
          if (a.commit) {
            sl.r[lane] = a.r;
            vec[0][lane] = a.rq; vec[1][lane] = a.rq;
            if (lane == 0) { sl.m2 = a.m2; sl.cn = c.cn + 1; sl.ctail = a.page; }
            wave_sync();
            correct(j, -1);
          }
        }
        if (lane == 0) { s_done = r; s_nflag = us.nflag; s_j = j; s_at = at; s_planned = planned; }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // what was stored is in place
      }
      __syncthreads();
      r = s_done;
      const bool own = s_planned != 0;                 // the entry's own flag is the unit's only one
      if (s_nflag == 0) break;                         // workgroup-uniform
      split_unit<DT>(v, u, sp.raw, sp.wk, own);
      __syncthreads();
      if (r == nb) break;
      const int M1 = us.M;
      us = load_unit(v, u);
      fl = us.top - 1 - lane >= 0 ? v.freelist[(size_t)u * v.Pcap + us.top - 1 - lane] : -1;
      // clusters that were flagged before the call are split along with the first entry: z and slots of the batch still hold their
      // parents, and the next batch begins
      if (!own || us.nflag != 0 || us.M > M1 + 1) break;
    }
    t += r;
    __syncthreads();                                   // (s_done and the slots are read before the next batch writes them)
  }
  if (tid == 0) v.nflagged[u] = t;                     // how far this kernel came
}

template <int DT, bool MEAN>
__global__ __launch_bounds__(256) void extend_kernel(View v, const void* K, const void* V, int n, int resumes) {
  __shared__ double kd[kHeadDim];
  __shared__ double sv[16];
  __shared__ int si[16];
  __shared__ float s2[16];
  __shared__ int s_rmax2, s_nflag;
  __shared__ SplitLds<DT, true> sp;
  constexpr bool BF = DT == DYNAKV_BF16;
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // kRows entries' keys and values at a time wait in LDS: one trip to memory for all of them
  constexpr int kRows = 16, kEs = DT == DYNAKV_F32 ? 4 : 2;
  __shared__ __align__(16) unsigned char rows[kRows][2][kHeadDim * kEs];
  const int t0 = resumes ? v.nflagged[u] : 0;             // where extend_batch_kernel has stopped
  for (int t = t0; t < n; ++t) {
    const int r = (t - t0) % kRows;
    if (r == 0) {                                       // (a full barrier lies behind the last use of the rows)
      uint32_t x[kRows];
#pragma unroll
      for (int i = 0; i < kRows; ++i)
        x[i] = load_bits(tid < kHeadDim ? K : V, ((size_t)u * n + min(t + i, n - 1)) * kHeadDim + (tid & (kHeadDim - 1)), DT);
#pragma unroll
      for (int i = 0; i < kRows; ++i) store_bits(rows[i][0], tid, x[i], DT);
      lds_barrier();
    }
    constexpr int kBatch = 4;
    const uint4* tiles = MEAN ? nullptr : (const uint4*)unit_Rq(v, u);
    const int table_tiles = (int)(v.Rstride / kTileElems);   // the table's padded end: these rows exist in every state
    uint4 cur[kBatch][4], nxt[kBatch][4];
    auto fetch = [&](uint4 (&dst)[kBatch][4], int T0) __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int T = min(T0 + b * 4, table_tiles - 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) dst[b][s] = tiles[((size_t)T * 4 + s) * 64 + lane];
      }
    };
    ScoreRows<1> A;
    if constexpr (!MEAN) {
      fetch(cur, wave);
      load_score_rows<1>(A, 0, nullptr, rows[r][0], 0, lane);    // row 0 = the entry
    }
    const UnitState us = load_unit(v, u);
    const int M = us.M;
    if (us.N >= v.Ncap || M <= 0) {                    // workgroup-uniform
      if (tid == 0) v.err[u] |= DYNAKV_ERR_TOKENS;
      return;
    }
    float k2 = 0.f;
    if (tid < kHeadDim) {
      const float kf = bits_value(load_bits(rows[r][0], tid, DT), DT);
      kd[tid] = (double)kf;
      k2 = kf * kf;
    }
    if (tid == 0) s_rmax2 = 0;
    lds_barrier();
    int j;
    if constexpr (MEAN) {
      const float* R = unit_R(v, u);
      double best = __builtin_inf();
      int arg = -1;
      for (int jj = tid; jj < M; jj += 256) {
        f4 row[8];
        double dist[1];
        load_centroid_head(R, jj, row);
        centroid_sums<1>(R, jj, row, dist, [&](int d, float rv, double (&acc)[1]) __attribute__((always_inline)) {
          const double x = kd[d] - (double)rv;
          acc[0] = fma(x, x, acc[0]);
        });
        if (dist[0] < best || arg < 0) { best = dist[0]; arg = jj; }
      }
      j = block_argmin<256>(best, arg, sv, si);
    } else {
      for (int o = 32; o > 0; o >>= 1) k2 += __shfl_xor(k2, o);
      if (lane == 0) s2[wave] = k2;
      float* zd = v.zdist + (size_t)u * v.Mcap;
      float zb = -__builtin_inff(), z2 = -__builtin_inff(), rmax2 = 0.f;
      int jb = -1;
      const int ntile = (M + kTileClusters - 1) / kTileClusters;
      for (int T0 = wave; T0 < ntile; T0 += 4 * kBatch) {
        const bool more = T0 + 4 * kBatch < ntile;
        if (more) fetch(nxt, T0 + 4 * kBatch);
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
          const int T = T0 + b * 4;
          if (T >= ntile) break;                         // wavefront-uniform
          float red, kdot, nrm2;
          score_tile<BF, 1, true>(cur[b], A, 0, DYNAKV_GROUP_MAX, lane, red, kdot, nrm2);
          const int jj = T * kTileClusters + lane;
          if (lane < kTileClusters && jj < M) {
            const float z = kdot - 0.5f * nrm2;
            zd[jj] = z;
            rmax2 = fmaxf(rmax2, nrm2);
            if (jb < 0 || z > zb) { z2 = jb < 0 ? z2 : zb; zb = z; jb = jj; }
            else z2 = fmaxf(z2, z);
          }
        }
        if (more) {
#pragma unroll
          for (int b = 0; b < kBatch; ++b)
#pragma unroll
            for (int s = 0; s < 4; ++s) cur[b][s] = nxt[b][s];
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) rmax2 = fmaxf(rmax2, __shfl_xor(rmax2, o));
      if (lane == 0) atomicMax(&s_rmax2, __float_as_int(rmax2));
      lds_barrier();                                    // (nearest_resolve waits for zd itself if it needs it)
      const float kn = __builtin_sqrtf(s2[0] + s2[1]) * 1.0001f;
      j = nearest_resolve<256>(v, u, M, zb, jb, z2, kn, __int_as_float(s_rmax2), zd, unit_Rq(v, u), kd, sv, si, s2);
    }
    if (wave == 0) {
      const ClusterFetch cf = fetch_cluster(v, u, j, us.top, lane);
      EntryBits e;
      if constexpr (DT == DYNAKV_F32) { e.k = ((const uint2*)rows[r][0])[lane]; e.v = ((const uint2*)rows[r][1])[lane]; }
      else { e.k = uint2{((const uint32_t*)rows[r][0])[lane], 0}; e.v = uint2{((const uint32_t*)rows[r][1])[lane], 0}; }
      const AppendResult a = append_wave<DT>(v, u, j, us, cluster_state(cf, us.top), e, lane);
      if (lane == 0) s_nflag = a.nflag;
    }
    __syncthreads();                                    // the append's record is in place for the whole workgroup
    if (s_nflag == 0) continue;                         // workgroup-uniform (and nothing above writes it before a barrier)
    split_unit<DT>(v, u, sp.raw, sp.wk, false);
    __syncthreads();                                    // and the unit's counters for the next entry
  }
}

// Baseline without clustering (Section 8.1): the new entry becomes cluster M of its unit, its own representative.
__global__ __launch_bounds__(256) void append_token_kernel(View v, const void* kin, const void* vin) {
  __shared__ int s_page;
  const int u = blockIdx.x, tid = threadIdx.x;
  const int M = v.M[u], N = v.N[u];
  const size_t cbase = (size_t)u * v.Mcap;
  if (tid == 0) {
    int page = -1;
    if (N >= v.Ncap) v.err[u] |= DYNAKV_ERR_TOKENS;
    else if (M >= v.Mcap) v.err[u] |= DYNAKV_ERR_CLUSTERS;
    else {
      const int top = v.free_top[u], bump = v.bump[u];
      if (top > 0) { page = v.freelist[(size_t)u * v.Pcap + top - 1]; v.free_top[u] = top - 1; }
      else if (bump < v.Pcap) { page = bump; v.bump[u] = bump + 1; }
      else v.err[u] |= DYNAKV_ERR_TOKENS;
    }
    if (page >= 0) {
      v.pnext[(size_t)u * v.Pcap + page] = -1;
      for (int p = 0; p < kInlinePages; ++p) v.cpg[(cbase + M) * kInlinePages + p] = p == 0 ? page : -1;
      v.ctail[cbase + M] = page;
      v.cn[cbase + M] = 1; v.cb[cbase + M] = 0; v.csz[cbase + M] = 1; v.cflag[cbase + M] = 0; v.cM2[cbase + M] = 0.0;
      v.in_req[cbase + M] = 0;
      v.ppos[((size_t)u * v.Pcap + page) * kPageTokens] = N;
      v.last_assign[u] = M;
      v.M[u] = M + 1; v.N[u] = N + 1;
      if (v.local_W > 0) v.lcount[u] += 1;
    }
    s_page = page;
  }
  __syncthreads();
  const int page = s_page;
  if (page < 0) return;
  char* pg = page_ptr(v, u, page);
  if (tid < kHeadDim) {
    store_centroid(v, u, M, tid, load_elem(kin, (size_t)u * kHeadDim + tid, v.dtype));
    copy_elem(pg, k_index(v.dtype, 0, tid), kin, (size_t)u * kHeadDim + tid, v.dtype);
  } else {
    copy_elem(pg, v_index(v.dtype, 0, tid - kHeadDim), vin, (size_t)u * kHeadDim + tid - kHeadDim, v.dtype);
  }
}

// Local update (Section 2.3): the last W clusters of the unit, one entry each, are clustered among themselves by
// Lloyd's k-means into k clusters that take their place.  One workgroup per unit; keys staged in LDS as float32
// (exact for every storage type), float64 distances and sums, centres stored as float32.
__global__ __launch_bounds__(256) void local_recluster_kernel(View v, int iters) {
  __shared__ float x[kLocalWindowMax][kHeadDim + 1];
  __shared__ float r[kLocalClustersMax][kHeadDim];
  __shared__ double dist[kLocalWindowMax], m2[kLocalClustersMax];
  __shared__ int label[kLocalWindowMax], pos[kLocalWindowMax], opage[kLocalWindowMax], rank[kLocalWindowMax];
  __shared__ int cnt[kLocalClustersMax], pgbase[kLocalClustersMax + 1], npage[kLocalClustersMax + kLocalWindowMax / kPageTokens + 1];
  __shared__ int s_ok;
  const int u = blockIdx.x, tid = threadIdx.x, W = v.local_W, k = v.local_k;
  if (v.lcount[u] != W) return;                         // workgroup-uniform: an append of this window was refused
  const int M = v.M[u], base = M - W;
  const size_t cb = (size_t)u * v.Mcap;
  const int es = elem_size(v.dtype);
  if (tid < W) {
    const int pg = v.cpg[(cb + base + tid) * kInlinePages];
    opage[tid] = pg;
    pos[tid] = v.ppos[((size_t)u * v.Pcap + pg) * kPageTokens];
  }
  __syncthreads();
  for (int t = tid; t < W * kHeadDim; t += 256) x[t >> 7][t & 127] = page_key(v, u, opage[t >> 7], 0, t & 127);
  __syncthreads();
  for (int t = tid; t < k * kHeadDim; t += 256) r[t >> 7][t & 127] = x[(t >> 7) * W / k][t & 127];
  __syncthreads();
  for (int it = 0; it < iters; ++it) {
    if (tid < W) {                                      // nearest centre, ties to the lowest
      double best = __builtin_inf();
      int arg = 0;
      for (int j = 0; j < k; ++j) {
        double acc = 0.0;
#pragma unroll 8
        for (int d = 0; d < kHeadDim; ++d) {
          const double t = (double)x[tid][d] - (double)r[j][d];
          acc = fma(t, t, acc);
        }
        if (acc < best) { best = acc; arg = j; }
      }
      label[tid] = arg;
    }
    __syncthreads();
    for (int t = tid; t < k * kHeadDim; t += 256) {     // mean of the members; a centre without members stays
      const int j = t >> 7, d = t & 127;
      double sum = 0.0;
      int n = 0;
      for (int i = 0; i < W; ++i)
        if (label[i] == j) { sum += (double)x[i][d]; ++n; }
      if (n > 0) r[j][d] = (float)(sum / (double)n);
    }
    __syncthreads();
  }
  if (tid < W) {                                        // distance to the stored centre, place inside the cluster
    const int j = label[tid];
    double acc = 0.0;
    for (int d = 0; d < kHeadDim; ++d) {
      const double t = (double)x[tid][d] - (double)r[j][d];
      acc = fma(t, t, acc);
    }
    dist[tid] = acc;
    int rk = 0;
    for (int i = 0; i < tid; ++i) rk += label[i] == j;
    rank[tid] = rk;
  }
  __syncthreads();
  if (tid < k) {
    int n = 0;
    double s = 0.0;
    for (int i = 0; i < W; ++i)
      if (label[i] == tid) { ++n; s += dist[i]; }
    cnt[tid] = n; m2[tid] = s;
  }
  __syncthreads();
  if (tid == 0) {                                       // fresh pages for the k clusters; the W old pages are freed below
    int need = 0;
    for (int j = 0; j < k; ++j) { pgbase[j] = need; need += (cnt[j] + kPageTokens - 1) / kPageTokens; }
    pgbase[k] = need;
    int top = v.free_top[u], bump = v.bump[u];
    s_ok = top + (v.Pcap - bump) >= need;
    if (s_ok) {
      for (int p = 0; p < need; ++p) npage[p] = top > 0 ? v.freelist[(size_t)u * v.Pcap + --top] : bump++;
      v.free_top[u] = top; v.bump[u] = bump;
    } else {
      v.err[u] |= DYNAKV_ERR_TOKENS;
      v.lcount[u] = 0;
    }
  }
  __syncthreads();
  if (!s_ok) return;
  char* pool = v.pages + (size_t)u * v.Pcap * ((size_t)kPageElems * es);
  const int chunks = kHeadDim * es / 16;                // 16-byte chunks per row
  for (int t = tid; t < W * 2 * chunks; t += 256) {     // keys and values, row by row, old page -> new page
    const int i = t / (2 * chunks), c = t % (2 * chunks), kv = c / chunks, ch = c % chunks;
    const int j = label[i], dpage = npage[pgbase[j] + rank[i] / kPageTokens], slot = rank[i] % kPageTokens;
    const size_t so = (size_t)(kv ? v_index(v.dtype, 0, 0) : k_index(v.dtype, 0, 0)) * es + (size_t)ch * 16;
    const size_t dof = (size_t)(kv ? v_index(v.dtype, slot, 0) : k_index(v.dtype, slot, 0)) * es + (size_t)ch * 16;
    *(uint4*)(pool + (size_t)dpage * kPageElems * es + dof) = *(const uint4*)(pool + (size_t)opage[i] * kPageElems * es + so);
  }
  if (tid < W) {
    const int j = label[tid];
    v.ppos[((size_t)u * v.Pcap + npage[pgbase[j] + rank[tid] / kPageTokens]) * kPageTokens + rank[tid] % kPageTokens] = pos[tid];
  }
  for (int t = tid; t < k * kHeadDim; t += 256) store_centroid(v, u, base + (t >> 7), t & 127, r[t >> 7][t & 127]);
  if (tid < k) {
    const size_t cj = cb + base + tid;
    const int np = pgbase[tid + 1] - pgbase[tid];
    v.cn[cj] = cnt[tid]; v.cb[cj] = 0; v.csz[cj] = cnt[tid]; v.cflag[cj] = 0; v.cM2[cj] = m2[tid];
    for (int p = 0; p < kInlinePages; ++p) v.cpg[cj * kInlinePages + p] = p < np ? npage[pgbase[tid] + p] : -1;
    v.ctail[cj] = np ? npage[pgbase[tid] + np - 1] : -1;
    for (int p = 0; p < np; ++p) v.pnext[(size_t)u * v.Pcap + npage[pgbase[tid] + p]] = p + 1 < np ? npage[pgbase[tid] + p + 1] : -1;
  }
  for (int j = base + tid; j < M; j += 256) v.in_req[cb + j] = 0;
  __syncthreads();                                      // every copy has read its old page
  if (tid == 0) {
    int top = v.free_top[u];
    for (int i = 0; i < W; ++i) v.freelist[(size_t)u * v.Pcap + top++] = opage[i];
    v.free_top[u] = top;
    v.M[u] = base + k; v.lcount[u] = 0;
  }
}

// ------------------------------------------------------------------------------------------- split
template <int DT>
__global__ __launch_bounds__(kSplitThreads) void split_kernel(View v) {
  __shared__ __align__(16) unsigned char raw[kSplitRaw<DT>];
  __shared__ SplitWork wk;
  split_unit<DT>(v, blockIdx.x, raw, wk, false);
}

}  // namespace

// prescanned: the score kernel of the same step has already looked at the new key (launch_score_select with kin).
// Otherwise, with the 16-bit search copy, a matrix-core pass of its own comes first.
hipError_t launch_append(const View& v, const void* k, const void* val, bool prescanned, bool split, hipStream_t st) {
  if (v.token_level) {
    append_token_kernel<<<v.U, 256, 0, st>>>(v, k, val);
    return hipGetLastError();
  }
  if (!v.search_mean && !prescanned) {
    const hipError_t e = launch_near(v, k, st);
    if (e != hipSuccess) return e;
  }
  const int mode = !v.search_mean ? kPreZ : prescanned ? kPreMean : kScanMean;
#define DYNAKV_APPEND_M(DT, MODE)                                                         \
  do {                                                                                     \
    if (split) append_kernel<DT, MODE, true><<<v.U, 256, 0, st>>>(v, k, val);              \
    else append_kernel<DT, MODE, false><<<v.U, 256, 0, st>>>(v, k, val);                   \
  } while (0)
#define DYNAKV_APPEND(DT)                                                                  \
  do {                                                                                     \
    if (mode == kPreZ) DYNAKV_APPEND_M(DT, kPreZ);                                         \
    else if (mode == kPreMean) DYNAKV_APPEND_M(DT, kPreMean);                              \
    else DYNAKV_APPEND_M(DT, kScanMean);                                                   \
  } while (0)
  if (v.dtype == DYNAKV_F32) {
    if (prescanned) DYNAKV_APPEND_M(DYNAKV_F32, kPreMean);
    else DYNAKV_APPEND_M(DYNAKV_F32, kScanMean);
  }
  else if (v.dtype == DYNAKV_F16) DYNAKV_APPEND(DYNAKV_F16);
  else DYNAKV_APPEND(DYNAKV_BF16);
#undef DYNAKV_APPEND
#undef DYNAKV_APPEND_M
  return hipGetLastError();
}
hipError_t launch_local_recluster(const View& v, int iters, hipStream_t st) {
  local_recluster_kernel<<<v.U, 256, 0, st>>>(v, iters);
  return hipGetLastError();
}
hipError_t launch_extend(const View& v, const void* K, const void* V, int n, hipStream_t st) {
  const bool batch = n >= kExtendLeast;
  if (v.dtype == DYNAKV_F32) extend_kernel<DYNAKV_F32, true><<<v.U, 256, 0, st>>>(v, K, V, n, false);
  else if (v.dtype == DYNAKV_F16) {
    if (v.search_mean) extend_kernel<DYNAKV_F16, true><<<v.U, 256, 0, st>>>(v, K, V, n, false);
    else {
      if (batch) extend_batch_kernel<DYNAKV_F16><<<v.U, 256, 0, st>>>(v, K, V, n);
      if (!batch || v.Mcap > kExtendClusters) extend_kernel<DYNAKV_F16, false><<<v.U, 256, 0, st>>>(v, K, V, n, batch);
    }
  } else {
    if (v.search_mean) extend_kernel<DYNAKV_BF16, true><<<v.U, 256, 0, st>>>(v, K, V, n, false);
    else {
      if (batch) extend_batch_kernel<DYNAKV_BF16><<<v.U, 256, 0, st>>>(v, K, V, n);
      if (!batch || v.Mcap > kExtendClusters) extend_kernel<DYNAKV_BF16, false><<<v.U, 256, 0, st>>>(v, K, V, n, batch);
    }
  }
  return hipGetLastError();
}
hipError_t launch_split(const View& v, hipStream_t st) {
  if (v.dtype == DYNAKV_F32) split_kernel<DYNAKV_F32><<<v.U, kSplitThreads, 0, st>>>(v);
  else if (v.dtype == DYNAKV_F16) split_kernel<DYNAKV_F16><<<v.U, kSplitThreads, 0, st>>>(v);
  else split_kernel<DYNAKV_BF16><<<v.U, kSplitThreads, 0, st>>>(v);
  return hipGetLastError();
}
}  // namespace dynakv
