// The index as a whole: its snapshot out (dynakv_export_state) and in (dynakv_import_state), and the page pool laid out
// afresh by co-retrieval (dynakv_place_by_coretrieval; Section 5.1, Eq. 8).
#include "common.hpp"

namespace dynakv {

namespace {

// ------------------------------------------------------------------------------------------- export
// A snapshot is bound by the bytes it moves, so everything but the prefix sum over the clusters' sizes is spread over
// the whole chip.  (With one workgroup per unit for all of it, 8 units of 50 000 clusters took 4.4 ms out and 6.3 ms in;
// now 0.17 and 0.54 ms.  256 units of 12 000 entries in 1900 clusters: 0.32 -> 0.18 and 1.18 -> 0.83 ms, of which 0.64 ms move
// 3.1 GB of keys and values at 4.9 TB/s, the rate of a plain copy.)
constexpr int kScanRun = 8;        // consecutive clusters per thread and round of a unit's prefix sum
constexpr int kStateTile = 64;     // clusters per workgroup of the copies: one tile of the lane-interleaved table

// Where more than kSelectLds clusters are possible, a retrieval lists the selected clusters by id or by score, whichever it can do
// sooner, and a snapshot lists them by descending score (lowest id among equals).
__device__ inline bool lists_by_score(const View& v, int u) {
  return v.Mcap > kSelectLds && v.n_list[u] > 0;       // (an imported selection has no list and stays as it came)
}
// By a workgroup of 1024 threads: the clusters of unit u's list sorted in LDS, their ids, and for each place of the list where its entries
// begin in that order.  Bound by the sort's dependent trips to LDS, most of which (pairs less than 128 apart) stay in a wavefront.
// The price of a retrieval that does not rank what it selects (8 units of 50 000 clusters, 1600 selected: 125 -> 110 us): a snapshot of
// ids and entries takes 76 us instead of 50, with 4000 selected 93 instead of 54.  (By counting the clusters before each in memory, for
// every cluster and again for every list entry: 900 and 1630.)
__device__ __forceinline__ void rank_selection(const View& v, const dynakv_state_t& o, int u, int* sm) {
  __shared__ unsigned long long key[kCountBig];
  const int tid = threadIdx.x, n = min(v.n_sel[u], kCountBig);
  const size_t cb = (size_t)u * v.Mcap;
  const int* off = list_offsets(v, u);
  int P = 64;
  while (P < n) P *= 2;
  static_assert(kMaxClusters <= 1 << 17 && kCountBig <= 1 << 12, "score, id and place in one key");
  for (int i = tid; i < P; i += 1024) {
    const int id = i < n ? v.sel_ids[cb + i] : 0;
    key[i] = i < n ? (unsigned long long)~orderable(v.score[cb + id]) << 32 | (unsigned)id << 12 | (unsigned)i : ~0ull;
  }
  __syncthreads();
  for (int run = 2; run <= P; run *= 2)                 // bitonic sort, ascending
    for (int d = run / 2; d > 0; d /= 2) {
      for (int t = tid; t < P / 2; t += 1024) {
        const int a = 2 * t - (t & (d - 1)), b = a + d;
        const unsigned long long x = key[a], y = key[b];
        if ((x > y) == ((a & run) == 0)) { key[a] = y; key[b] = x; }
      }
      if (d > 64 || d == 1) lds_barrier();              // (pairs t .. t + 63 of a wavefront: keys 2 t .. 2 t + 127)
      else { asm volatile("" ::: "memory"); __builtin_amdgcn_wave_barrier(); asm volatile("" ::: "memory"); }
    }
  constexpr int kRun = kCountBig / 1024;
  int w[kRun], tot = 0, all;
#pragma unroll
  for (int k = 0; k < kRun; ++k) {
    const int r = tid * kRun + k, i = r < n ? (int)(key[r] & 0xFFF) : 0;
    w[k] = r < n ? (i + 1 < v.n_sel[u] ? off[i + 1] : v.t_sel[u]) - off[i] : 0;
    tot += w[k];
  }
  int at = block_excl_scan(tot, sm, all);
#pragma unroll
  for (int k = 0; k < kRun; ++k) {
    const int r = tid * kRun + k;
    if (r < n) {
      score_offsets(v, u)[key[r] & 0xFFF] = at;
      if (o.selected) o.selected[cb + r] = (int)(key[r] >> 12 & (kMaxClusters - 1));
    }
    at += w[k];
  }
}

// One workgroup per unit: the scalars, and where every cluster's members start.
__global__ __launch_bounds__(1024) void export_unit_kernel(View v, dynakv_state_t o) {
  __shared__ int sm[64];
  const int u = blockIdx.x, tid = threadIdx.x, M = v.M[u];
  const size_t cbase = (size_t)u * v.Mcap;
  if (tid == 0) {
    if (o.n_clusters) o.n_clusters[u] = M;
    if (o.n_tokens) o.n_tokens[u] = v.N[u];
    if (o.error) o.error[u] = v.err[u];
    if (o.tau) o.tau[u] = v.tau[u];
    if (o.n_selected) o.n_selected[u] = v.n_sel[u];
    if (o.n_gathered) o.n_gathered[u] = v.t_sel[u];
    if (o.last_assign) o.last_assign[u] = v.last_assign[u];
    if (o.counters) {
      for (int k = 0; k < kCounters; ++k) o.counters[(size_t)u * kCounters + k] = v.counters[(size_t)u * kCounters + k];
      o.counters[(size_t)u * kCounters + 3] = v.bump[u] - v.free_top[u];
    }
  }
  if ((o.selected || o.gathered) && lists_by_score(v, u)) rank_selection(v, o, u, sm);     // workgroup-uniform
  if (!(o.offsets || o.members || o.keys || o.values)) return;
  int before = 0;
  for (int j0 = 0; j0 < M; j0 += 1024 * kScanRun) {
    int w[kScanRun], tot = 0;
#pragma unroll
    for (int k = 0; k < kScanRun; ++k) {
      const int j = j0 + tid * kScanRun + k;
      w[k] = j < M ? v.csz[cbase + j] : 0;
      tot += w[k];
    }
    int total;
    int run = before + block_excl_scan(tot, sm, total);
#pragma unroll
    for (int k = 0; k < kScanRun; ++k) {
      const int j = j0 + tid * kScanRun + k;
      if (j < M) {
        v.tok_off[cbase + j] = run;
        if (o.offsets) o.offsets[(size_t)u * (v.Mcap + 1) + j] = run;
      }
      run += w[k];
    }
    before += total;
  }
  if (o.offsets)
    for (int j = M + tid; j <= v.Mcap; j += 1024) o.offsets[(size_t)u * (v.Mcap + 1) + j] = before;
}

// A tile of 64 centroids between the lane-interleaved table and rows of 128 floats, by a workgroup of 256: a wavefront
// moves four clusters x 64 coordinates at a time, i.e. 64 contiguous bytes on the table's side and 256 on the rows'.
// f(cluster inside the tile, first coordinate of four).
template <class F>
__device__ __forceinline__ void for_each_table_piece(F&& f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll 4
  for (int k = wave; k < 32; k += 4) f((k >> 1) * 4 + (lane & 3), ((k & 1) * 16 + (lane >> 2)) * 4);
}

// Clusters 64 blockIdx.x .. + 63 of unit blockIdx.y: records, centroids, and the members (keys and values too) page by page,
// sixteen lanes per cluster.
__global__ __launch_bounds__(256) void export_clusters_kernel(View v, dynakv_state_t o) {
  const int u = blockIdx.y, tid = threadIdx.x, M = v.M[u], j0 = blockIdx.x * kStateTile;
  const size_t cbase = (size_t)u * v.Mcap;
  const bool by_score = lists_by_score(v, u);           // (the ids are written: rank_selection)
  if (tid < kStateTile && j0 + tid < v.Mcap) {
    const int j = j0 + tid;
    const size_t cj = cbase + j;
    const bool in = j < M;
    if (o.size) o.size[cj] = in ? v.cn[cj] : 0;
    if (o.buffered) o.buffered[cj] = in ? v.cb[cj] : 0;
    if (o.flag) o.flag[cj] = in ? v.cflag[cj] : 0;
    if (o.m2) o.m2[cj] = in ? v.cM2[cj] : 0.0;
    if (o.scores) o.scores[cj] = in ? v.score[cj] : 0.f;
    if (o.selected) {
      const int n = v.n_sel[u];
      if (j >= n) o.selected[cj] = -1;
      else if (!by_score) o.selected[cj] = v.sel_ids[cj];
    }
    if (o.first_page) o.first_page[cj] = in && v.csz[cj] > 0 ? v.cpg[cj * kInlinePages] : -1;
  }
  if (o.centroids) {
    const float* R = unit_R(v, u);
    if (j0 >= M) {                                       // nothing but unused slots: whole lines of zeros
      float* z = o.centroids + (cbase + j0) * kHeadDim;
      const int n = min(kStateTile, v.Mcap - j0) * (kHeadDim / 4);
#pragma unroll 8
      for (int t = tid; t < n; t += 256) *(f4u*)(z + 4 * t) = f4{0, 0, 0, 0};
    } else
    for_each_table_piece([&](int c, int d) __attribute__((always_inline)) {
      const int j = j0 + c;
      if (j < v.Mcap) *(f4u*)(o.centroids + (cbase + j) * kHeadDim + d) = j < M ? *(const f4*)(R + r_index(j, d)) : f4{0, 0, 0, 0};
    });
  }
  if (o.gathered) {
    const int nl = v.n_list[u];
    for (int w = blockIdx.x * 256 + tid; w < nl; w += gridDim.x * 256) {
      const int e = v.plist[(size_t)u * v.Lcap + w];
      int t0 = v.plist_off[(size_t)u * v.Lcap + w];
      if (by_score) {                                    // the cluster that this entry belongs to, and its place by score
        const int* off = list_offsets(v, u);
        int lo = 0, hi = v.n_sel[u] - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (off[mid] <= t0) lo = mid; else hi = mid - 1;
        }
        t0 += score_offsets(v, u)[lo] - off[lo];
      }
      const int page = e >> 4, first = ((e >> 2) & 3) * 4, nv = (e & 3) + 1;
      for (int sl = 0; sl < nv; ++sl)
        if ((unsigned)(t0 + sl) < (unsigned)v.Ncap) o.gathered[(size_t)u * v.Ncap + t0 + sl] = v.ppos[((size_t)u * v.Pcap + page) * kPageTokens + first + sl];
    }
  }
  if (!(o.members || o.keys || o.values)) return;
  const int es = elem_size(v.dtype), c = tid & 15;
  for (int j = j0 + (tid >> 4); j < min(M, j0 + kStateTile); j += 16) {
    int w = v.tok_off[cbase + j], left = v.csz[cbase + j], page = -1;
    for (int k = 0; left > 0; ++k) {
      page = cluster_page(v, u, cbase + j, k, page);
      if (page < 0) break;
      const int nv = min(left, kPageTokens);
      const int pos = c < nv ? v.ppos[((size_t)u * v.Pcap + page) * kPageTokens + c] : 0;
      if (o.members && c < nv) o.members[(size_t)u * v.Ncap + w + c] = pos;
      if (o.keys || o.values) {
        const char* pg = page_ptr(v, u, page);
        for (int sl = 0; sl < nv; ++sl) {
          const size_t row = ((size_t)u * v.Ncap + __shfl(pos, sl, 16)) * kHeadDim * es;
          for (int ch = c; ch < kHeadDim * es / 16; ch += 16) {
            if (o.keys) *(uint4*)((char*)o.keys + row + ch * 16) = *(const uint4*)(pg + (size_t)k_index(v.dtype, sl, 0) * es + ch * 16);
            if (o.values) *(uint4*)((char*)o.values + row + ch * 16) = *(const uint4*)(pg + (size_t)v_index(v.dtype, sl, 0) * es + ch * 16);
          }
        }
      }
      w += nv; left -= nv;
    }
  }
}

// ------------------------------------------------------------------------------------------- import
// One thread: unit u's scalars as they are before its first retrieval, with nothing flagged or selected and no page recycled.
__device__ inline void reset_unit(const View& v, int u, int M, int N, double tau, int pages) {
  v.M[u] = M; v.N[u] = N; v.tau[u] = tau; v.err[u] = 0; v.nflag[u] = 0; v.n_sel[u] = 0; v.t_sel[u] = 0; v.n_list[u] = 0;
  v.ticket[u] = 0; v.ticket[v.U + u] = 0; v.ticket[2 * v.U + u] = 0; v.bump[u] = pages; v.free_top[u] = 0; v.last_assign[u] = -1; v.lcount[u] = 0; v.rmax2[u] = 0;
  for (int k = 0; k < kCounters; ++k) v.counters[(size_t)u * kCounters + k] = 0;
}

// First kernel of an import, one workgroup per unit: checks the snapshot's sizes, deals out the pages cluster by cluster
// (v.pg_off), and writes the unit's scalars, flagged list and active set.
// v.nflagged[u] tells the kernels that follow whether the unit was accepted.  first: the index has never been built, so a
// refused unit has no previous state to keep: it becomes an empty one.
__global__ __launch_bounds__(1024) void import_unit_kernel(View v, dynakv_state_t s, int first) {
  __shared__ int sm[64];
  __shared__ int s_bad, s_nflag;
  const int u = blockIdx.x, tid = threadIdx.x;
  const size_t cbase = (size_t)u * v.Mcap;
  const int M = s.n_clusters[u], N = s.n_tokens[u];
  const int* off = s.offsets + (size_t)u * (v.Mcap + 1);
  const bool sane = M >= 1 && M <= v.Mcap && N >= 0 && N <= v.Ncap;
  if (tid == 0) { s_bad = 0; s_nflag = 0; }
  __syncthreads();
  long long pages = 0;
  if (sane) {
    if (tid == 0 && (off[0] != 0 || off[M] != N)) s_bad = 1;
    for (int j0 = 0; j0 < M; j0 += 1024 * kScanRun) {
      int np[kScanRun], tot = 0;
#pragma unroll
      for (int k = 0; k < kScanRun; ++k) {
        const int j = j0 + tid * kScanRun + k;
        np[k] = 0;
        if (j >= M) continue;
        const int n = s.size[cbase + j], b = s.buffered[cbase + j], m = off[j + 1] - off[j];
        if (n < 0 || b < 0 || m != n + b || m > N || (b != 0 && s.flag[cbase + j] == 0)) s_bad = 1;
        np[k] = (min(max(m, 0), N) + kPageTokens - 1) / kPageTokens;
        tot += np[k];
      }
      int total;
      int run = (int)pages + block_excl_scan(tot, sm, total);
#pragma unroll
      for (int k = 0; k < kScanRun; ++k) {
        const int j = j0 + tid * kScanRun + k;
        if (j < M) v.pg_off[cbase + j] = run;
        run += np[k];
      }
      pages += total;
    }
  }
  __syncthreads();
  if (!sane || s_bad || pages > v.Pcap) {
    if (tid == 0) {
      if (first) reset_unit(v, u, 0, 0, 0.0, 0);
      v.err[u] |= DYNAKV_ERR_IMPORT; v.nflagged[u] = 0;
    }
    return;
  }
  for (int j = tid; j < v.Mcap; j += 1024) {
    v.in_req[cbase + j] = 0;
    if (j < M && s.flag[cbase + j] != 0) v.flist[cbase + atomicAdd(&s_nflag, 1)] = j;
  }
  __syncthreads();
  int nsel = 0;
  if (s.selected) {
    nsel = min(max(s.n_selected[u], 0), M);
    for (int i = tid; i < nsel; i += 1024) {
      const int id = min(max(s.selected[cbase + i], 0), M - 1);
      v.sel_ids[cbase + i] = id; v.in_req[cbase + id] = 1;
    }
  }
  if (tid == 0) {
    reset_unit(v, u, M, N, s.tau[u], (int)pages);
    v.nflag[u] = s_nflag; v.n_sel[u] = nsel; v.nflagged[u] = 1;
  }
}

// Clusters 64 blockIdx.x .. + 63 of unit blockIdx.y: records, centroids, page tables and, for the copy that follows, the
// owner of every page (kept in the free-page stack, which is empty after an import).
__global__ __launch_bounds__(256) void import_clusters_kernel(View v, dynakv_state_t s) {
  const int u = blockIdx.y, tid = threadIdx.x, j0 = blockIdx.x * kStateTile;
  if (!v.nflagged[u]) return;
  const int M = v.M[u];
  const size_t cbase = (size_t)u * v.Mcap;
  const int* off = s.offsets + (size_t)u * (v.Mcap + 1);
  if (tid < kStateTile && j0 + tid < v.Mcap) {
    const int j = j0 + tid;
    const size_t cj = cbase + j;
    const bool in = j < M;
    v.score[cj] = 0.f;
    v.cn[cj] = in ? s.size[cj] : 0; v.cb[cj] = in ? s.buffered[cj] : 0; v.csz[cj] = in ? off[j + 1] - off[j] : 0;
    v.cflag[cj] = in ? s.flag[cj] != 0 : 0; v.cM2[cj] = in ? s.m2[cj] : 0.0;
  }
  for (int t = tid; t < kStateTile * kInlinePages; t += 256) {
    const int j = j0 + t / kInlinePages, p = t % kInlinePages;
    if (j >= v.Mcap) break;
    const int m = j < M ? off[j + 1] - off[j] : 0, np = (m + kPageTokens - 1) / kPageTokens;
    const int base = np ? v.pg_off[cbase + j] : 0;
    v.cpg[(cbase + j) * kInlinePages + p] = p < np ? base + p : -1;
    if (p == 0) v.ctail[cbase + j] = np ? base + np - 1 : -1;
    for (int q = p; q < np; q += kInlinePages) {
      v.pnext[(size_t)u * v.Pcap + base + q] = q + 1 < np ? base + q + 1 : -1;
      v.freelist[(size_t)u * v.Pcap + base + q] = j;
    }
  }
  if (j0 < M) {
    float* R = unit_R(v, u);
    for_each_table_piece([&](int c, int d) __attribute__((always_inline)) {
      const int j = j0 + c;
      if (j >= M) return;
      const f4 x = *(const f4u*)(s.centroids + (cbase + j) * kHeadDim + d);
      *(f4*)(R + r_index(j, d)) = x;
      if (v.dtype != DYNAKV_F32) {
        const uint2 q = {round_bits16(x[0], v.dtype) | ((uint32_t)round_bits16(x[1], v.dtype) << 16),
                         round_bits16(x[2], v.dtype) | ((uint32_t)round_bits16(x[3], v.dtype) << 16)};
        *(uint2*)(unit_Rq(v, u) + rq_index(j, d)) = q;
      }
    });
  }
}

// One page per sixteen lanes: positions, keys and values of its tokens, the rows of a page in flight together.
// Keys and values of the snapshot: [U][Ncap][128].
template <int ES>
__global__ __launch_bounds__(256) void import_pages_kernel(View v, dynakv_state_t s) {
  constexpr int kCh = kHeadDim * ES / 256;             // 16-byte chunks per lane and row
  constexpr int kRows = 16 / kCh;                      // rows in flight
  const int u = blockIdx.y, page = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  if (!v.nflagged[u] || page >= v.bump[u]) return;
  const int j = v.freelist[(size_t)u * v.Pcap + page];
  const int* off = s.offsets + (size_t)u * (v.Mcap + 1);
  const int end = off[j + 1], q0 = off[j] + (page - v.pg_off[(size_t)u * v.Mcap + j]) * kPageTokens, nv = min(kPageTokens, end - q0);
  const int pos = min(max(s.members[(size_t)u * v.Ncap + min(q0 + c, end - 1)], 0), v.Ncap - 1);
  if (c < nv) v.ppos[((size_t)u * v.Pcap + page) * kPageTokens + c] = pos;
  char* pg = page_ptr(v, u, page);
#pragma unroll
  for (int kv = 0; kv < 2; ++kv) {
    const char* src = (const char*)(kv ? s.values : s.keys);
    char* dst = pg + (kv ? (size_t)v_index(v.dtype, 0, 0) * ES : 0);
#pragma unroll
    for (int r0 = 0; r0 < kPageTokens; r0 += kRows) {
      if (r0 >= nv) break;
      f4 w[kRows][kCh];                              // (a plain vector type: these stay in registers)
#pragma unroll
      for (int r = 0; r < kRows; ++r) {                // rows past the last repeat it: their loads hit the same lines
        const int p = __shfl(pos, min(r0 + r, nv - 1), 16);
#pragma unroll
        for (int ch = 0; ch < kCh; ++ch) w[r][ch] = *(const f4*)(src + ((size_t)u * v.Ncap + p) * (kHeadDim * ES) + ch * 256 + c * 16);
      }
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int ch = 0; ch < kCh; ++ch)
          if (r0 + r < nv) *(f4*)(dst + (size_t)(r0 + r) * (kHeadDim * ES) + ch * 256 + c * 16) = w[r][ch];
    }
  }
}

// ------------------------------------------------------------------------------------------- placement
// First kernel of a placement, one workgroup per unit: whether the unit is as a build or an import left it
// (v.nflagged[u], for the kernels that follow), and the storage order of its entries, read from the index's own pages
// because the arrays of the k-means hold nothing after an import: start of every cluster (koff), and for every place its
// position (order) and cluster (labels).  A position beyond the caller's K and V refuses the unit.
__global__ __launch_bounds__(1024) void place_members_kernel(View v, int n_tokens) {
  __shared__ int sm[64];
  __shared__ int s_bad;
  const int u = blockIdx.x, tid = threadIdx.x, c = tid & 15;
  const size_t cbase = (size_t)u * v.Mcap;
  int* koff = v.koff + (size_t)u * (v.Mcap + 1);
  if (v.M[u] != v.M0 || v.N[u] != n_tokens || v.nflag[u] != 0 || v.free_top[u] != 0) {     // workgroup-uniform
    if (tid == 0) v.nflagged[u] = 0;
    return;
  }
  if (tid == 0) s_bad = 0;
  int before = 0;
  for (int j0 = 0; j0 < v.M0; j0 += 1024) {
    int total;
    const int run = before + block_excl_scan(j0 + tid < v.M0 ? v.csz[cbase + j0 + tid] : 0, sm, total);
    if (j0 + tid < v.M0) koff[j0 + tid] = run;
    before += total;
  }
  if (tid == 0) koff[v.M0] = before;
  __syncthreads();
  for (int j = tid >> 4; j < v.M0 && before == n_tokens; j += 64) {
    int w = koff[j], left = v.csz[cbase + j], page = -1;
    for (int k = 0; left > 0; ++k) {
      page = cluster_page(v, u, cbase + j, k, page);
      if (page < 0) break;
      const int nv = min(left, kPageTokens);
      if (c < nv) {
        const int pos = v.ppos[((size_t)u * v.Pcap + page) * kPageTokens + c];
        if (pos < 0 || pos >= n_tokens) s_bad = 1;
        v.order[(size_t)u * v.Ncap + w + c] = pos;
        v.labels[(size_t)u * v.Ncap + w + c] = j;
      }
      w += nv; left -= nv;
    }
    if (left > 0) s_bad = 1;
  }
  __syncthreads();
  if (tid == 0) v.nflagged[u] = before == n_tokens && !s_bad;
}

// 16 consecutive places of the storage order per workgroup, 16 threads per entry: keys and values move by
// position into their cluster's (new) pages as whole 16-byte chunks.  `stride`: tokens per unit in K and V.
__global__ __launch_bounds__(256) void place_copy_kernel(View v, const void* K, const void* V, int stride) {
  const int u = blockIdx.y, q = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  if (!v.nflagged[u] || q >= v.N[u]) return;
  const int pos = v.order[(size_t)u * v.Ncap + q];
  const int j = v.labels[(size_t)u * v.Ncap + q];
  const int rank = q - v.koff[(size_t)u * (v.Mcap + 1) + j];
  const int page = v.pg_off[(size_t)u * v.Mcap + j] + rank / kPageTokens, slot = rank % kPageTokens;
  char* pg = page_ptr(v, u, page);
  const size_t src = ((size_t)u * stride + pos) * kHeadDim + c * 8;
  if (v.dtype == DYNAKV_F32) {
    const f4* ks = (const f4*)((const float*)K + src);
    const f4* vs = (const f4*)((const float*)V + src);
    *(f4*)((float*)pg + k_index32(slot, c * 8)) = ks[0];
    *(f4*)((float*)pg + k_index32(slot, c * 8 + 4)) = ks[1];
    *(f4*)((float*)pg + v_index32(slot, c * 8)) = vs[0];
    *(f4*)((float*)pg + v_index32(slot, c * 8 + 4)) = vs[1];
  } else {
    *(uint4*)((uint16_t*)pg + k_index16(slot, c * 8)) = *(const uint4*)((const uint16_t*)K + src);
    *(uint4*)((uint16_t*)pg + v_index16(slot, c * 8)) = *(const uint4*)((const uint16_t*)V + src);
  }
  if (c == 0) v.ppos[((size_t)u * v.Pcap + page) * kPageTokens + slot] = pos;
}

// Correlation-aware placement (Section 5.1, Eq. 8).  F = P while counting: [U][M0][M0] float32 counts (exact).
__global__ __launch_bounds__(256) void cor_zero_kernel(float* F, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) F[i] = 0.f;
}
// After one reference retrieval: every ordered pair of different selected clusters is counted once.  One
// workgroup per unit; a pair belongs to one thread, and the launches of different queries follow each other.
__global__ __launch_bounds__(256) void cor_count_kernel(View v, float* F) {
  const int u = blockIdx.x, n = v.n_sel[u], M0 = v.M0;
  const int* ids = v.sel_ids + (size_t)u * v.Mcap;
  float* f = F + (size_t)u * M0 * M0;
  for (long long t = threadIdx.x; t < (long long)n * n; t += 256) {
    const int a = ids[t / n], b = ids[t % n];
    if (a != b && a < M0 && b < M0) f[(size_t)a * M0 + b] += 1.f;
  }
}
// One workgroup of 1024 threads per unit: the greedy chain on the counts, Eq. 8's normalisation, and the page
// table of the unit in chain order (pg_off / cpg / ctail / pnext), for the copy kernel that follows.
__global__ __launch_bounds__(1024) void cor_finish_kernel(View v, float* F, int* order_out) {
  __shared__ float rowsum[kMaxInitClusters];
  __shared__ unsigned char placed[kMaxInitClusters];
  __shared__ float rv[16];
  __shared__ int ri[16];
  __shared__ double rt[16];
  __shared__ int s_last;
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, M0 = v.M0;
  const size_t cb = (size_t)u * v.Mcap;
  float* f = F + (size_t)u * M0 * M0;
  int* chain = v.tok_off + cb;
  if (!v.nflagged[u]) {                                    // workgroup-uniform
    if (tid == 0) atomicOr(&v.err[u], DYNAKV_ERR_PLACE);
    return;
  }
  double tot = 0.0;
  for (int i = tid; i < M0; i += 1024) {
    float rs = 0.f;
    for (int j = 0; j < M0; ++j) rs += f[(size_t)i * M0 + j];          // whole numbers below 2^24: exact
    rowsum[i] = rs; placed[i] = 0;
    tot += (double)rs;
  }
  for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o);
  if (lane == 0) rt[w] = tot;
  __syncthreads();
  double total = 0.0;
  for (int k = 0; k < 16; ++k) total += rt[k];
  // arg-max over (value, id) pairs of the workgroup, lowest id among equals; id < 0: none
  auto argmax = [&](float val, int id) {
    for (int o = 32; o > 0; o >>= 1) {
      const float ov = __shfl_xor(val, o);
      const int oi = __shfl_xor(id, o);
      if (oi >= 0 && (id < 0 || ov > val || (ov == val && oi < id))) { val = ov; id = oi; }
    }
    __syncthreads();
    if (lane == 0) { rv[w] = val; ri[w] = id; }
    __syncthreads();
    if (tid == 0) {
      float bv = rv[0]; int bi = ri[0];
      for (int k = 1; k < 16; ++k)
        if (ri[k] >= 0 && (bi < 0 || rv[k] > bv || (rv[k] == bv && ri[k] < bi))) { bv = rv[k]; bi = ri[k]; }
      s_last = bi;
    }
    __syncthreads();
    return s_last;
  };
  int last;
  {
    float bv = -1.f; int bi = -1;
    for (int i = tid; i < M0; i += 1024)
      if (rowsum[i] > bv) { bv = rowsum[i]; bi = i; }                  // ascending i per thread: the first maximum stays
    last = argmax(bv, bi);
  }
  for (int k = 0; k < M0; ++k) {
    if (tid == 0) { chain[k] = last; placed[last] = 1; }
    __syncthreads();
    if (k + 1 == M0) break;
    float bv = -1.f; int bi = -1;
    for (int j = tid; j < M0; j += 1024)
      if (!placed[j] && f[(size_t)last * M0 + j] > bv) { bv = f[(size_t)last * M0 + j]; bi = j; }
    last = argmax(bv, bi);
  }
  // Eq. 8
  const float inv = total > 0.0 ? (float)(1.0 / total) : 0.f;
  for (size_t t = tid; t < (size_t)M0 * M0; t += 1024) f[t] = total > 0.0 ? (float)((double)f[t] / total) : 0.f;
  (void)inv;
  if (order_out)
    for (int k = tid; k < M0; k += 1024) order_out[(size_t)u * M0 + k] = chain[k];
  // pages in chain order
  if (tid == 0) {
    int base = 0;
    for (int k = 0; k < M0; ++k) {
      const int j = chain[k];
      v.pg_off[cb + j] = base;
      base += (v.cn[cb + j] + kPageTokens - 1) / kPageTokens;
    }
  }
  __syncthreads();
  for (int j = tid; j < M0; j += 1024) {
    const int np = (v.cn[cb + j] + kPageTokens - 1) / kPageTokens, base = v.pg_off[cb + j];
    for (int p = 0; p < kInlinePages; ++p) v.cpg[(cb + j) * kInlinePages + p] = p < np ? base + p : -1;
    v.ctail[cb + j] = np ? base + np - 1 : -1;
    for (int p = 0; p < np; ++p) v.pnext[(size_t)u * v.Pcap + base + p] = p + 1 < np ? base + p + 1 : -1;
  }
}
}  // namespace

hipError_t launch_export(const View& v, const dynakv_state_t& dst, hipStream_t st) {
  export_unit_kernel<<<v.U, 1024, 0, st>>>(v, dst);
  export_clusters_kernel<<<dim3((v.Mcap + kStateTile - 1) / kStateTile, v.U), 256, 0, st>>>(v, dst);
  return hipGetLastError();
}
hipError_t launch_place(const View& v, const void* K, const void* V, int n_tokens, const void* Qref, int n_ref, int budget,
                        float* P, int* order, hipStream_t st) {
  const size_t n = (size_t)v.U * v.M0 * v.M0;
  cor_zero_kernel<<<1024, 256, 0, st>>>(P, n);
  const size_t qbytes = (size_t)v.U * v.G * kHeadDim * elem_size(v.dtype);
  for (int r = 0; r < n_ref; ++r) {
    const hipError_t e = launch_score_select(v, (const char*)Qref + (size_t)r * qbytes, budget, nullptr, st);
    if (e != hipSuccess) return e;
    cor_count_kernel<<<v.U, 256, 0, st>>>(v, P);
  }
  place_members_kernel<<<v.U, 1024, 0, st>>>(v, n_tokens);
  cor_finish_kernel<<<v.U, 1024, 0, st>>>(v, P, order);
  place_copy_kernel<<<dim3((n_tokens + 15) / 16, v.U), 256, 0, st>>>(v, K, V, n_tokens);
  return hipGetLastError();
}
hipError_t launch_import(const View& v, const dynakv_state_t& src, bool first, hipStream_t st) {
  import_unit_kernel<<<v.U, 1024, 0, st>>>(v, src, first);
  import_clusters_kernel<<<dim3((v.Mcap + kStateTile - 1) / kStateTile, v.U), 256, 0, st>>>(v, src);
  const dim3 pages((v.Pcap + 15) / 16, v.U);
  if (v.dtype == DYNAKV_F32) import_pages_kernel<4><<<pages, 256, 0, st>>>(v, src);
  else import_pages_kernel<2><<<pages, 256, 0, st>>>(v, src);
  return hipGetLastError();
}

}  // namespace dynakv
