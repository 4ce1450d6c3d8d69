// Decode, second half of a step (Algorithm 1, decode block; Section 4.2):
//   append_kernel - nearest cluster (its own scan of the table, or the per-block results the score kernel of a
//                   whole-step call left), UpdateVar, threshold test, AddEntry + UpdateStats or buffer + flag;
//                   in a whole-step call the due splits follow in the same launch
//   split_kernel  - delayed splits of flagged clusters in the active set, then the forced split
// One workgroup per unit; each unit's record is touched by that workgroup only.  All decisions are
// taken on float64 values summed in an order that does not depend on the launch, ties to the lowest index.
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
template <bool ON>
struct SplitLds {
  alignas(16) unsigned char raw[kSplitRaw];
  SplitWork wk;
};
template <>
struct SplitLds<false> {};
template <int DT, int MODE, bool SPLIT>
__global__ __launch_bounds__(256) void append_kernel(View v, const void* kin, const void* vin) {
  static_assert(kSplitThreads == 256, "split_unit is run by this kernel's whole workgroup");
  __shared__ AppendSmem a;
  __shared__ double sv[16];
  __shared__ int si[16];
  __shared__ float s2[16];
  __shared__ SplitLds<SPLIT> sp;
  const int u = blockIdx.x, tid = threadIdx.x;
  const float* R = unit_R(v, u);
  f4 row[8];
  if constexpr (MODE == kScanMean)
    if ((size_t)(tid | 63) * kHeadDim < v.Rstride) load_centroid_head(R, tid, row);     // requested before anything else
  const int M = v.M[u], N = v.N[u];
  if (N >= v.Ncap || M <= 0) {                          // refused (workgroup-uniform); due splits still run
    if (tid == 0) v.err[u] |= DYNAKV_ERR_TOKENS;
    if constexpr (SPLIT) {
      __syncthreads();
      split_unit<DT>(v, u, sp.raw, sp.wk, false);
    }
    return;
  }
  float k2 = 0.f;
  if (tid < kHeadDim) {
    const float kf = load_elem(kin, (size_t)u * kHeadDim + tid, v.dtype);
    a.kd[tid] = (double)kf;
    k2 = kf * kf;
  }
  __syncthreads();
  int j;
  if constexpr (MODE == kPreZ) {
    for (int o = 32; o > 0; o >>= 1) k2 += __shfl_xor(k2, o);
    if ((tid & 63) == 0) s2[tid >> 6] = k2;
    __syncthreads();
    const float kn = __builtin_sqrtf(s2[0] + s2[1]) * 1.0001f;
    const float* zd = v.zdist + (size_t)u * v.Mcap;
    // the matrix-core pass has left best / runner-up per 64 clusters
    float zb = -__builtin_inff(), z2 = -__builtin_inff();
    int jb = -1;
    const size_t wbase = (size_t)u * v.NB * 4;
    for (int w = tid; w * 64 < M; w += 256) merge_best2(zb, jb, z2, v.near_zb[wbase + w], v.near_zj[wbase + w], v.near_z2[wbase + w]);
    j = nearest_resolve<256>(v, u, M, zb, jb, z2, kn, __int_as_float(v.rmax2[u]), zd, unit_Rq(v, u), a.kd, sv, si, s2);
  } else {
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
          const double t = a.kd[d] - (double)rv;
          acc[0] = fma(t, t, acc[0]);
        });
        if (dist[0] < best || arg < 0) { best = dist[0]; arg = jj; }
      }
    }
    j = block_argmin<256>(best, arg, sv, si);
  }
  const AppendFetch f = append_fetch(v, u, j);
  append_commit<256>(v, u, j, M, N, kin, vin, a, f);
  if constexpr (SPLIT) {
    __syncthreads();                                    // the append's record is in place for the whole workgroup
    split_unit<DT>(v, u, sp.raw, sp.wk, false);
  }
}

// ------------------------------------------------------------------------------------------- chunked prefill
// Adaptive clustering through a long prefill (Section 7, Discussion 1): one workgroup per unit walks the chunk's n
// entries in order; each entry is assigned to its nearest cluster (matrix cores + float64 where needed for the
// 16-bit search copy, float64 scan for float32 means), appended with UpdateVar and the threshold test, and a
// flagged cluster is split at once (the view's B_max is 0).  K, V: [U][n][128].
// Entry t + 1 depends on what entry t did, so a unit's time is a chain of round trips to memory and what counts is how many
// of them an entry waits for: the table in batches of four tiles per wavefront with the next batch in flight (read wherever
// they lie in the table's padded range, so that the first does not wait for M), the entries' rows sixteen
// at a time through LDS, the split's look at the flagged list only where the append has left a flag.
// 256 units, 256 clusters, 1024 entries (163 splits a unit): 11.5 -> 10.4 ms.  Per entry: 6.6 us in the static update mode,
// where no cluster is ever flagged (1024 entries behind 2048 as well as 2048 behind 4096); 7.3 and 7.6 us with one and five
// splits per unit on average, because the launch waits for the unit with most of them; 10.1 and 10.5 us with 163 and 334.
template <int DT, bool MEAN>
__global__ __launch_bounds__(256) void extend_kernel(View v, const void* K, const void* V, int n) {
  __shared__ AppendSmem a;
  __shared__ double sv[16];
  __shared__ int si[16];
  __shared__ float s2[16];
  __shared__ int s_rmax2;
  __shared__ SplitLds<true> sp;
  constexpr bool BF = DT == DYNAKV_BF16;
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  static_assert(kSplitThreads == 2 * kHeadDim, "one coordinate of the key or of the value per thread");
  // kRows entries' keys and values at a time wait in LDS: one trip to memory for all of them
  constexpr int kRows = 16, kEs = DT == DYNAKV_F32 ? 4 : 2;
  __shared__ __align__(16) unsigned char rows[kRows][2][kHeadDim * kEs];
  for (int t = 0; t < n; ++t) {
    const int r = t % kRows;
    if (r == 0) {                                       // (a full barrier lies behind the last use of the rows)
      uint32_t x[kRows];
#pragma unroll
      for (int i = 0; i < kRows; ++i)
        x[i] = load_bits(tid < kHeadDim ? K : V, ((size_t)u * n + min(t + i, n - 1)) * kHeadDim + (tid & (kHeadDim - 1)), DT);
#pragma unroll
      for (int i = 0; i < kRows; ++i) store_bits(rows[i][0], tid, x[i], DT);
      lds_barrier();
    }
    const uint32_t held = load_bits(rows[r][0], tid, DT);
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
    const int M = v.M[u], N = v.N[u], top = v.free_top[u];
    if (N >= v.Ncap || M <= 0) {                       // workgroup-uniform
      if (tid == 0) v.err[u] |= DYNAKV_ERR_TOKENS;
      return;
    }
    float k2 = 0.f;
    if (tid < kHeadDim) {
      const float kf = bits_value(held, v.dtype);
      a.kd[tid] = (double)kf;
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
          const double x = a.kd[d] - (double)rv;
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
      j = nearest_resolve<256>(v, u, M, zb, jb, z2, kn, __int_as_float(s_rmax2), zd, unit_Rq(v, u), a.kd, sv, si, s2);
    }
    const AppendFetch f = append_fetch(v, u, j, top);
    append_commit<256, true>(v, u, j, M, N, nullptr, nullptr, a, f, held);
    __syncthreads();                                    // the append's record is in place for the whole workgroup
    if (a.nflag1 == 0) continue;                        // workgroup-uniform (and nothing above writes it before a barrier)
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
  __shared__ __align__(16) unsigned char raw[kSplitRaw];
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
  if (v.dtype == DYNAKV_F32) extend_kernel<DYNAKV_F32, true><<<v.U, 256, 0, st>>>(v, K, V, n);
  else if (v.dtype == DYNAKV_F16) {
    if (v.search_mean) extend_kernel<DYNAKV_F16, true><<<v.U, 256, 0, st>>>(v, K, V, n);
    else extend_kernel<DYNAKV_F16, false><<<v.U, 256, 0, st>>>(v, K, V, n);
  } else {
    if (v.search_mean) extend_kernel<DYNAKV_BF16, true><<<v.U, 256, 0, st>>>(v, K, V, n);
    else extend_kernel<DYNAKV_BF16, false><<<v.U, 256, 0, st>>>(v, K, V, n);
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
