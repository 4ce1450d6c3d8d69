// Prefill: Lloyd's k-means per unit (Section 4.1, Eq. 3-4; Algorithm 1, prefill block; the
// remark of Section 7 that it must cope with empty clusters), cluster statistics, the head-specific
// threshold, and the cluster-contiguous page layout (Section 5.1, intra-cluster placement,
// kept here as the HBM layout).
//
// Every label is the float64 nearest centre (ties to the lowest index): a matrix-core filter in
// float32 settles the clear cases, every point within its error bound is decided in float64.
// Centre sums are float64 sums over the members.
//
// One iteration of a 16-bit type is two launches that matter: the assignment, which reads every key once, and the
// update, which reads the keys of the points that changed their cluster.  256 units x 4096 float16 keys x 256 centres:
// assignment 116 us, update 37 us, where nine launches that formed every sum anew, checked near-ties in a kernel of their
// own and split the centres into two 16-bit terms took 320 us; build and export of the partition 4.12 -> 2.56 ms (128 x 8192 x
// 512: 5.21 -> 3.17 ms; 8 x 16384 x 2048 bfloat16: 3.72 -> 2.16 ms); with the distances in the layout pass, records in whole
// lines and reseeding spread over the chip 2.25, 2.94 and 2.08 ms.  How many points the float64 decisions take depends on the
// keys; what is slower than on the mixture of these figures is given where it is handled (Offset, scan_centres,
// kmeans_changed_kernel, kmeans_slow_kernel).
#include <algorithm>

#include "common.hpp"

namespace dynakv {

namespace {

typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

// Terms that a centre is split into for the filter (see kmeans_assign_kernel): what one float16 leaves of a coordinate
// leaves 2 to 6 % of the points undecided by the filter, of one bfloat16 a third of them.
template <int DT>
constexpr int kTerms = DT == DYNAKV_F16 ? 1 : 2;
template <int DT>
constexpr int kChunkTiles = 2 / kTerms<DT>;          // tiles of 32 centres per LDS buffer of the assignment: 16 KB

// ---- scratch of a build -------------------------------------------------------------------------------------------
// The page pool holds nothing until the layout at the end of a build, so each unit's part of it serves as scratch:
// the offset that the filter takes off the centres (see Offset), float64 centre sums [M0][128], the centres as plain rows [M0][128] (float32; the comparison of two centres reads whole
// rows, which the lane-interleaved table has in 32 places), the list of points that changed their cluster [N0], member
// counts [2][M0].  (1024 + M0 (1024 + 512 + 8) + 8 N0 bytes against at least (M0 + N0 / 16) pages of 8 KB.)
struct Changed {
  int pos;
  unsigned move;                                     // old cluster | new cluster << 16
};
static_assert(kMaxInitClusters <= 65536, "two cluster ids per word");
// What the keys of a unit have in common: a vector c of the keys' type, zero if nothing stands out.  <x, r_j> - |r_j|^2 / 2 and
// <x, r_j - c> - <c, r_j - c> - |r_j - c|^2 / 2 differ by a number that is the same for every centre, but the second leaves a
// 16-bit term of a centre only its distance from c to round.  (256 units x 4096 float16 keys x 256 centres, 16 N(0, 1) added
// per channel: build 20.1 -> 4.0 ms; 64 N(0, 1): 30.2 -> 17.7 ms; without: 2.2 ms either way.  Two terms without the offset,
// as there once were, took 10.4, 55.9 and 3.8 ms.)
struct Offset {
  uint16_t bits[kHeadDim];
  float c[kHeadDim];
  float norm;                                        // |c| or a little more; 0: c is zero
};
static_assert(sizeof(Offset) <= 1024, "room in front of the sums");
__device__ inline Offset* km_offset(const View& v, int u) { return (Offset*)page_ptr(v, u, 0); }
__device__ inline double* km_sums(const View& v, int u) { return (double*)(page_ptr(v, u, 0) + 1024); }
__device__ inline float* km_rows(const View& v, int u) { return (float*)(km_sums(v, u) + (size_t)v.M0 * kHeadDim); }
__device__ inline Changed* km_changed(const View& v, int u) { return (Changed*)(km_rows(v, u) + (size_t)v.M0 * kHeadDim); }
__device__ inline int* km_counts(const View& v, int u, int N0, int which) {
  return (int*)(km_changed(v, u) + N0) + which * v.M0;
}

// Points that changed their cluster in the iterations of parity `slot`.
__device__ inline int& km_changed_count(const View& v, int u, int slot) { return v.xrange[4 * u + 2 + slot]; }

// A-operand order of one 32-cluster tile: [term][k-step of 16][lane][8], lane = (k%16)/8*32 + row.
__device__ inline size_t kmA_index(int nterms, int j, int term, int d) {
  return ((((size_t)(j >> 5) * nterms + term) * 8 + (d >> 4)) * 64 + (((d & 15) >> 3) << 5) + (j & 31)) * 8 + (d & 7);
}

// Sum over the 16 lanes of a row in any order (for bounds); every lane of the row gets it (float64 butterfly on DPP row
// operations).
template <int CTRL>
__device__ __forceinline__ double row_step(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, false);
  return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum_f64(double x) {
  x = row_step<kDppXor1>(x);
  x = row_step<kDppXor2>(x);
  x = row_step<kDppHalfMirror>(x);
  return row_step<kDppMirror>(x);
}

// Sum over the 16 lanes of a row, left to right as common.hpp fixes it for sums over the coordinates (lane c holding the sum of
// block c); lane 15 of the row has it.
__device__ __forceinline__ double row_blocked16(double x) {
  double t = x;
#pragma unroll
  for (int k = 1; k < 16; ++k) {                      // lanes 0 .. k hold their prefixes
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(t), 0x111, 0xF, 0xF, false);     // row_shr:1
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(t), 0x111, 0xF, 0xF, false);
    t = __hiloint2double(hi, lo) + x;
  }
  return t;
}

constexpr float kNoCentre = -3.0e38f;                  // in place of -|r_j|^2 / 2 (finite: the filter writes into its low bits)
// Norms that bound the filter's error, folded over the clusters that a thread has written.
struct CentreNorms {
  float r, rho;                                      // |d_j| = |r_j - offset|, |d_j - its 16-bit terms|
};
// Coordinates 8c .. 8c+7 of the unit's offset, requested at the start of a kernel for the centres that it writes at its end.
struct OffsetPart {
  f4 lo, hi;
};
template <int DT>
__device__ inline OffsetPart load_offset(const View& v, int u, int c) {
  OffsetPart o{{0, 0, 0, 0}, {0, 0, 0, 0}};
  if constexpr (DT != DYNAKV_F32) { const f4* p = (const f4*)(km_offset(v, u)->c + c * 8); o.lo = p[0]; o.hi = p[1]; }
  return o;
}
// Sixteen lanes write centre j (lane c of them coordinates 8c .. 8c+7): the float32 table and, for 16-bit types, the
// filter's terms of d = r_j - offset in A-operand order with -<offset, d> - |d|^2 / 2.
template <int DT>
__device__ inline void write_centre(const View& v, int u, int j, int c, const float (&r)[8], const OffsetPart& off, CentreNorms& cn) {
  float* R = unit_R(v, u);
  *(f4*)(R + r_index(j, c * 8)) = f4{r[0], r[1], r[2], r[3]};
  *(f4*)(R + r_index(j, c * 8 + 4)) = f4{r[4], r[5], r[6], r[7]};
  if constexpr (DT != DYNAKV_F32) {
    float* row = km_rows(v, u) + (size_t)j * kHeadDim + c * 8;
    *(f4*)row = f4{r[0], r[1], r[2], r[3]};
    *(f4*)(row + 4) = f4{r[4], r[5], r[6], r[7]};
    constexpr int NT = kTerms<DT>;
    uint16_t bits[NT][8];
    double nn = 0.0, rr = 0.0, cc = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double ce = (double)(e < 4 ? off.lo[e] : off.hi[e - 4]);
      double rem = (double)r[e] - ce;
      nn = fma(rem, rem, nn);
      cc = fma(ce, rem, cc);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        double part;
        if constexpr (DT == DYNAKV_BF16) { const __bf16 b = (__bf16)(float)rem; part = (double)(float)b; bits[t][e] = __builtin_bit_cast(uint16_t, b); }
        else { const _Float16 hh = (_Float16)(float)rem; part = (double)(float)hh; bits[t][e] = __builtin_bit_cast(uint16_t, hh); }
        rem -= part;
      }
      rr = fma(rem, rem, rr);
    }
    nn = row_sum_f64(nn);
    rr = row_sum_f64(rr);
    cc = row_sum_f64(cc);
    // a centre that is not finite is nearest to no point: it enters the filter as a padding row does
    const bool finite = nn < __builtin_inf();
    uint16_t* A = v.kmA + (size_t)u * v.kmA_stride;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      uint4 w;
      w.x = bits[t][0] | ((uint32_t)bits[t][1] << 16); w.y = bits[t][2] | ((uint32_t)bits[t][3] << 16);
      w.z = bits[t][4] | ((uint32_t)bits[t][5] << 16); w.w = bits[t][6] | ((uint32_t)bits[t][7] << 16);
      *(uint4*)(A + kmA_index(NT, j, t, c * 8)) = finite ? w : uint4{0, 0, 0, 0};
    }
    if (c == 0) v.hn[(size_t)u * km_pad(v.M0) + j] = finite ? (float)(-0.5 * nn - cc) : kNoCentre;
    if (finite) {
      cn.r = fmaxf(cn.r, (float)sqrt(nn) * 1.000001f);
      cn.rho = fmaxf(cn.rho, (float)sqrt(rr) * 1.000001f);
    }
  }
}
// The workgroup's maxima into the unit's (which only ever grow during a build: a bound of an earlier centre stays a
// bound).  Non-negative floats order like their bits.  sm: 2 ints of LDS per wavefront.
__device__ inline void fold_norms(const View& v, int u, CentreNorms cn, int* sm) {
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int r = wave_max(__float_as_int(cn.r)), q = wave_max(__float_as_int(cn.rho));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { sm[2 * w] = r; sm[2 * w + 1] = q; }
  __syncthreads();
  if (threadIdx.x == 0) {
    int mr = sm[0], mq = sm[1];
    for (int k = 1; k < nw; ++k) { mr = max(mr, sm[2 * k]); mq = max(mq, sm[2 * k + 1]); }
    atomicMax((int*)&v.rmax[2 * u], mr);
    atomicMax((int*)&v.rmax[2 * u + 1], mq);
  }
}

// ---- start --------------------------------------------------------------------------------------------------------
// One workgroup per unit, first kernel of a build: clears the unit's error word and the k-means' own counters, then flags
// initial positions that are out of range or given twice (the build still runs, with such a position clamped).  For 16-bit
// types also the unit's offset: the mean of (up to 64 of) the initial centres, if it outweighs their spread about it.
template <int DT>
__global__ __launch_bounds__(256) void kmeans_check_init_kernel(View v, const void* X, int N0, const int* init_idx) {
  __shared__ unsigned seen[kMaxPrefill / 32];
  const int u = blockIdx.x, tid = threadIdx.x;
  for (int i = tid; i < kMaxPrefill / 32; i += 256) seen[i] = 0u;
  if (tid == 0) {
    v.err[u] = 0; v.has_empty[u] = 0; v.rmax[2 * u] = 0.f; v.rmax[2 * u + 1] = 0.f;
    v.xrange[4 * u] = 0x7FFFFFFF; v.xrange[4 * u + 1] = -0x7FFFFFFF; v.xrange[4 * u + 2] = 0; v.xrange[4 * u + 3] = 0;
  }
  __syncthreads();
  bool bad = false;
  for (int j = tid; j < v.M0; j += 256) {
    const int p = init_idx[(size_t)u * v.M0 + j];
    if (p < 0 || p >= N0) bad = true;
    else if (atomicOr(&seen[p >> 5], 1u << (p & 31)) & (1u << (p & 31))) bad = true;
  }
  if (bad) atomicOr(&v.err[u], DYNAKV_ERR_INIT);
  if constexpr (DT != DYNAKV_F32) {
    __shared__ float part[16][kHeadDim];
    __shared__ float s_sq[4], s_m2[2];
    const int n = min(v.M0, 64), c = tid & 15;
    float s[8] = {}, sq = 0.f;
    for (int k = tid >> 4; k < n; k += 16) {
      float x[8];
      const int p = min(max(init_idx[(size_t)u * v.M0 + k], 0), N0 - 1);
      load8(X, ((size_t)u * N0 + p) * kHeadDim + c * 8, DT, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) { s[e] += x[e]; sq = fmaf(x[e], x[e], sq); }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[tid >> 4][c * 8 + e] = s[e];
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
    if ((tid & 63) == 0) s_sq[tid >> 6] = sq;
    __syncthreads();
    float m = 0.f, m2 = 0.f;
    if (tid < kHeadDim) {
#pragma unroll
      for (int k = 0; k < 16; ++k) m += part[k][tid];
      m /= (float)n;
      m2 = m * m;
      for (int o = 32; o > 0; o >>= 1) m2 += __shfl_xor(m2, o);
      if ((tid & 63) == 0) s_m2[tid >> 6] = m2;
    }
    __syncthreads();
    m2 = s_m2[0] + s_m2[1];
    const float mean_sq = (s_sq[0] + s_sq[1] + s_sq[2] + s_sq[3]) / (float)n;
    const bool use = mean_sq < __builtin_inff() && m2 > 0.5f * mean_sq;       // (false for a NaN)
    Offset* o = km_offset(v, u);
    __syncthreads();                                     // every thread has read s_m2
    if (tid < kHeadDim) {
      const uint16_t b = use ? round_bits16(m, DT) : 0;
      const float x = DT == DYNAKV_F16 ? f16_to_float(b) : bf16_to_float(b);
      o->bits[tid] = b;
      o->c[tid] = x;
      float c2 = x * x;
      for (int w = 32; w > 0; w >>= 1) c2 += __shfl_xor(c2, w);
      if ((tid & 63) == 0) s_m2[tid >> 6] = c2;
    }
    __syncthreads();
    if (tid == 0) o->norm = __builtin_sqrtf(s_m2[0] + s_m2[1]) * 1.0001f;
  }
}

// Centre j = key at position init_idx[u][j]; the rows that pad the filter's table to whole chunks lose every comparison.
// grid (ceil(M0 / 16) or ceil(km_pad(M0) / 16), U), sixteen lanes per centre.
template <int DT>
__global__ __launch_bounds__(256) void kmeans_start_kernel(View v, const void* X, int N0, const int* init_idx) {
  __shared__ int sm[8];
  const int u = blockIdx.y, j = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  CentreNorms cn{0.f, 0.f};
  if (j < v.M0) {
    const int p = min(max(init_idx[(size_t)u * v.M0 + j], 0), N0 - 1);
    float r[8];
    load8(X, ((size_t)u * N0 + p) * kHeadDim + c * 8, DT, r);
    write_centre<DT>(v, u, j, c, r, load_offset<DT>(v, u, c), cn);
  } else if (DT != DYNAKV_F32 && j < km_pad(v.M0)) {
    uint16_t* A = v.kmA + (size_t)u * v.kmA_stride;
    for (int t = 0; t < kTerms<DT>; ++t) *(uint4*)(A + kmA_index(kTerms<DT>, j, t, c * 8)) = uint4{0, 0, 0, 0};
    if (c == 0) v.hn[(size_t)u * km_pad(v.M0) + j] = kNoCentre;
  }
  if constexpr (DT != DYNAKV_F32) fold_norms(v, u, cn, sm);
}

// ---- order-free centre sums -----------------------------------------------------------------------------
// The centre of a cluster is the float64 sum of its members, divided by the count.  Every
// key of a 16-bit type is an integer multiple of 2^q, q = (smallest exponent in the unit) - (mantissa bits), and
// smaller than 2^(emax+1); if (emax + 1 + ceil(log2 N0)) - q <= 53, every partial sum of any subset in any order
// is exactly representable.  The sum then does not depend on the order at all and can follow the points that join and
// leave a cluster: an update reads the changed points' keys only, and its result is the sum formed anew, bit for bit.
// (float16 with at most 8192 keys always qualifies: exponents -14 .. 15 on a grid of 2^-24.  A key that is not finite needs no
// exception there: it is at no finite distance from any centre, so every assignment leaves it in cluster 0, whose sums in
// the coordinates concerned are infinite or NaN whichever way they are formed.)  Units whose keys span
// too wide a range, and float32 keys, have their sums formed anew in ascending position in every iteration.
__host__ __device__ inline bool sums_order_free_by_type(int dtype, int N0) { return dtype == DYNAKV_F16 && N0 <= 8192; }
__device__ inline bool sums_order_free(const View& v, int u, int N0) {
  if (v.dtype == DYNAKV_F32) return false;
  if (sums_order_free_by_type(v.dtype, N0)) return true;
  const int lo = v.xrange[4 * u], hi = v.xrange[4 * u + 1];
  const int mbits = v.dtype == DYNAKV_F16 ? 10 : 7;
  if (hi < lo) return true;                           // all keys zero
  int L = 0;
  while ((1 << L) < N0) ++L;
  return hi < 0x3FFFFFFF && (hi + 1 + L) - (lo - mbits) <= 53;
}

// ---- assignment, float32 keys -------------------------------------------------------------------------------------
// Four lanes per point, 32 coordinates each, nearest centre in exact float64, centres staged through LDS in tiles.  (One
// lane per point left a small prompt on a handful of wavefronts: 2048 keys x 32 centres 55 us, now 17 us.)
constexpr int kTileC = 32;
__global__ __launch_bounds__(256) void kmeans_assign_f64_kernel(View v, const void* X, int N0) {
  constexpr int kRow = kHeadDim + 16;                 // quarters 36 floats apart: the four lanes of a point hit different banks
  __shared__ __align__(16) float rs[kTileC][kRow];
  const int u = blockIdx.y, q = threadIdx.x & 3;
  const int i = blockIdx.x * 64 + (threadIdx.x >> 2);
  const bool live = i < N0;
  float x[32];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float t[8];
    load8(X, ((size_t)u * N0 + (live ? i : 0)) * kHeadDim + q * 32 + k * 8, DYNAKV_F32, t);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[k * 8 + e] = t[e];
  }
  double best = __builtin_inf();
  int arg = 0;
  const float* R = unit_R(v, u);
  for (int j0 = 0; j0 < v.M0; j0 += kTileC) {
    const int nt = min(kTileC, v.M0 - j0);
    __syncthreads();
    for (int t = threadIdx.x; t < kTileC * 32; t += 256) {           // 16 bytes per thread, contiguous over the clusters
      const int d4 = t / kTileC, jj = t % kTileC;
      if (jj < nt) *(f4*)&rs[jj][d4 * 4 + (d4 >> 3) * 4] = *(const f4*)(R + r_index(j0 + jj, d4 * 4));
    }
    __syncthreads();
    for (int jj = 0; jj < nt; ++jj) {
      double blk[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f4 a = *(const f4*)&rs[jj][q * 36 + k * 8], b = *(const f4*)&rs[jj][q * 36 + k * 8 + 4];
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double t = (double)x[k * 8 + e] - (double)(e < 4 ? a[e] : b[e - 4]);
          s = fma(t, t, s);
        }
        blk[k] = s;
      }
      const double acc = blocked16_quad(blk);
      if (acc < best) { best = acc; arg = j0 + jj; }
    }
  }
  if (live && q == 0) v.labels[(size_t)u * v.Ncap + i] = arg;
}

// c + the inner product of two pairs of 16-bit values, in float32.
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef __bf16 b2v __attribute__((ext_vector_type(2)));
template <bool BF>
__device__ __forceinline__ float dot2(uint32_t w, uint32_t y, float c) {
  if constexpr (BF) return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2v, w), __builtin_bit_cast(b2v, y), c, false);
  else return __builtin_amdgcn_fdot2(__builtin_bit_cast(h2v, w), __builtin_bit_cast(h2v, y), c, false);
}

// BYTES (4 or 16) from each lane's global address to LDS at base + lane * BYTES, with no detour through registers.  As an
// instruction of its own because the compiler, which cannot tell the two LDS buffers of a pipeline apart, would wait for
// the load before the next read of either; the caller waits (vmcnt) and synchronises before it reads the data.
template <int BYTES>
__device__ __forceinline__ void load_to_lds(const void* src, void* base) {
  const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)base);
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(src) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(at), "v"(src) : "memory", "m0");
}

// ---- assignment through the matrix cores --------------------------------------------------------------
// z_ij = <x_i, d_j> - <c, d_j> - |d_j|^2/2 with d_j = r_j - c, c the unit's offset (see Offset; mostly zero), orders the centres
// like the squared distance.  The filter evaluates it with MFMA on 16-bit operands: x is exact in its storage type, d_j is
// replaced by the sum of its 16-bit terms (one for float16, two for bfloat16), accumulation is float32.
// |error of z| <= eps_i:
//   |x_i| max_j |d_j - terms|               what the terms leave of a centre (its exact norm is known)
//   NT 2^-16 ((|x_i| + |c|) B + B^2 / 2)    accumulation of NT x 128 exact products onto -<c, d_j> - |d_j|^2/2, doubled
//   2^bits 2^-23 |z|                        the running best three carry the centre's number in their low mantissa bits
//   1e-35                                   all of these where float32 has no digits left: products, squares of |x|^2 and
//                                           z itself below 2^-126 (up to 128 of them), the number in a z of zero
// B bounds |d_j| of every centre that can be the nearest: such a centre is no farther from x_i than the best one found,
// whose distance follows from its z and |x_i - c| (and B <= max |d|).
// A point whose best and second-best values are more than 2 eps_i apart has the same nearest centre in exact arithmetic.
// If only the second lies within that distance, the two centres are compared in float64 by 16 lanes; if the third does too
// (about one point in a thousand), the workgroup goes through all centres in float64.  Labels therefore equal the
// float64 definition (sums in the one order of common.hpp whichever way a point is decided; ties to the lowest index).
//
// Shape: 64 points per wavefront as two B operands held in registers; Z^T = R~ X^T in 32x32 tiles, so lane (p, h) ends up
// with 16 values of point p per tile and the running best three need no cross-lane work until the end.  Four vector
// instructions per value (number into the low bits, two medians, one maximum) against 8 NT matrix instructions per 32
// values: with one term the vector pipe is the longer one (busy in 53 % of the cycles, the matrix pipe in 32 %, at 256 x 4096 x
// 256), with two they would change places, which is why the second term of
// float16 was worth dropping for a few per cent of the points to be re-checked.  Centres go through two LDS buffers of 16 KB, the next one filled by direct
// global-to-LDS loads while this one is consumed, one barrier per buffer; four wavefronts share them (eight were slower: one phase
// of latency more in step).  All workgroups of a unit have the same number modulo 8, i.e. share an L2.
// The first iteration (first) labels every point; later ones list the points whose label changed.
constexpr int kAssignWaves = 4;

// Nearest of all centres in float64 for NP points (xd: their coordinates in LDS; n of them count) by one wavefront of the
// `share` that split the centres among them: lane = centre, NC centres per lane at once.  Every coordinate of a centre is
// loaded once for NP points and every coordinate of a point read once for NC centres; the float64 pipe is what is left.
// (One point at a time by the whole workgroup read the centres anew for each: 64 units x 4096 float16 keys of 64 different
// values x 256 centres, where every point has several equal candidates, 25.4 ms, now 16.)
constexpr int kScanPoints = 4, kScanCentres = 2;
// Wavefronts that share the centres of a batch of points; the others take further batches.
__device__ __forceinline__ int scan_share(int M0, int nc) { return M0 <= 64 * nc ? 1 : M0 <= 128 * nc ? 2 : kAssignWaves; }
template <int NP, int NC>
__device__ __forceinline__ void scan_centres(const View& v, int u, const double* xd, int n, int mine, int share,
                                             double (*out_d)[kAssignWaves], int (*out_j)[kAssignWaves]) {
  const int lane = threadIdx.x & 63;
  const float* R = unit_R(v, u);
  double bd[NP];
  int bj[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) { bd[p] = __builtin_inf(); bj[p] = 0x7FFFFFFF; }
  for (int j0 = mine * NC * 64; j0 < v.M0; j0 += share * NC * 64) {
    double acc[NC][NP];
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int p = 0; p < NP; ++p) acc[k][p] = 0.0;
    for (int d8 = 0; d8 < 16; ++d8) {
      f4 r[NC][2];
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const int j = min(j0 + k * 64 + lane, v.M0 - 1);
        r[k][0] = *(const f4*)(R + r_index(j, d8 * 8)); r[k][1] = *(const f4*)(R + r_index(j, d8 * 8 + 4));
      }
      double blk[NC][NP];
#pragma unroll
      for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int p = 0; p < NP; ++p) blk[k][p] = 0.0;
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const double x = xd[p * kHeadDim + d8 * 8 + e];
#pragma unroll
          for (int k = 0; k < NC; ++k) {
            const double t = x - (double)r[k][e >> 2][e & 3];
            blk[k][p] = fma(t, t, blk[k][p]);
          }
          if (p + 1 == NP && (e & 1)) asm volatile("" ::: "memory");      // points' coordinates stay two deep in registers
        }
#pragma unroll
      for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[k][p] += blk[k][p];
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int j = j0 + k * 64 + lane;
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (j < v.M0 && acc[k][p] < bd[p]) { bd[p] = acc[k][p]; bj[p] = j; }      // ascending j per lane: the first minimum stays
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double od = __shfl_xor(bd[p], o);
      const int oj = __shfl_xor(bj[p], o);
      if (od < bd[p] || (od == bd[p] && oj < bj[p])) { bd[p] = od; bj[p] = oj; }
    }
    if (lane == 0 && p < n) { out_d[p][mine] = bd[p]; out_j[p][mine] = bj[p]; }
  }
}

template <int DT>
__global__ __launch_bounds__(kAssignWaves * 64, 4) void kmeans_assign_kernel(View v, const void* X, int N0, int gx, int first, int slot,
                                                                  int code_bits) {
  constexpr bool BF = DT == DYNAKV_BF16;
  constexpr int NT = kTerms<DT>, NW = kAssignWaves;
  constexpr int kTileBytes = NT * 8 * 1024;                // one 32-centre tile of terms
  constexpr int kTiles = kChunkTiles<DT>, kChunkC = 32 * kTiles, kChunkBytes = kTiles * kTileBytes;
  __shared__ __align__(16) unsigned char sA[2][kChunkBytes];
  __shared__ __align__(16) float shn[2][kChunkC];
  __shared__ short s_list[NW * 64];
  __shared__ double s_d[kScanPoints * NW][kAssignWaves];
  __shared__ int s_j[kScanPoints * NW][kAssignWaves], s_n3;
  static_assert(sizeof(sA) >= sizeof(double) * kScanPoints * NW * kHeadDim, "points of a scan, in float64");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // workgroup L: unit 8 (L / 8 / gx) + L % 8, points (L / 8) % gx
  const int u = (blockIdx.x >> 3) / gx * 8 + (blockIdx.x & 7), xb = (blockIdx.x >> 3) % gx;
  if (u >= v.U) return;
  const int p = lane & 31, h = lane >> 5;
  const int nchunk = km_pad(v.M0) / kChunkC;
  const int pbase = (xb * NW + wave) * 64;
  const char* gA = (const char*)(v.kmA + (size_t)u * v.kmA_stride);
  const float* hn = v.hn + (size_t)u * km_pad(v.M0);
  auto fetch = [&](int chunk, int buf) __attribute__((always_inline)) {
    constexpr int kPer = kChunkBytes / 1024 / NW;          // 1 KB pieces per wavefront
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int piece = wave * kPer + k;
      load_to_lds<16>(gA + (size_t)chunk * kChunkBytes + piece * 1024 + lane * 16, sA[buf] + piece * 1024);
    }
    if (wave == NW - 1 && lane < kChunkC) load_to_lds<4>(hn + chunk * kChunkC + lane, shn[buf]);
  };
  fetch(0, 0);
  if (tid == 0) s_n3 = 0;
  if (xb == 0 && tid == 0) km_changed_count(v, u, slot ^ 1) = 0;        // the list of the coming iteration
  uint4 bx[2][8];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int pt = pbase + t * 32 + p;
    const uint16_t* xr = (const uint16_t*)X + ((size_t)u * N0 + (pt < N0 ? pt : N0 - 1)) * kHeadDim + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) bx[t][ks] = *(const uint4*)(xr + ks * 16);
  }
  const float kLow = -3.2e38f;
  float best[2] = {kLow, kLow}, second[2] = {kLow, kLow}, third[2] = {kLow, kLow};
  unsigned keep = ~((1u << code_bits) - 1u);
  asm("" : "+v"(keep));                                    // in a vector register: mask and number go in with one instruction
  int old = 0;
  if (!first) old = v.labels[(size_t)u * v.Ncap + min(pbase + lane, N0 - 1)];
  __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0), in a form that the compiler counts with: no waits for
                                                           // the operands inside the loop
  __syncthreads();
  for (int ch = 0; ch < nchunk; ++ch) {
    const int cur = ch & 1;
    if (ch + 1 < nchunk) fetch(ch + 1, cur ^ 1);
#pragma unroll
    for (int tt = 0; tt < kTiles; ++tt) {
      f16v acc[2];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f4 n4 = *(const f4*)&shn[cur][tt * 32 + 8 * g + 4 * h];
#pragma unroll
        for (int e = 0; e < 4; ++e) { acc[0][4 * g + e] = n4[e]; acc[1][4 * g + e] = n4[e]; }
      }
#pragma unroll
      for (int term = 0; term < NT; ++term)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const uint4 a = *(const uint4*)(sA[cur] + tt * kTileBytes + (term * 8 + ks) * 1024 + lane * 16);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            if constexpr (BF)
              acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8v, a), __builtin_bit_cast(b8v, bx[t][ks]), acc[t], 0, 0, 0);
            else
              acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8v, a), __builtin_bit_cast(h8v, bx[t][ks]), acc[t], 0, 0, 0);
          }
        }
      const int code0 = (ch * kTiles + tt) * 16;                // this lane's values are numbered in the order it sees them
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int code = code0 + i;
        asm("" : "+s"(code));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const float val = __uint_as_float((__float_as_uint(acc[t][i]) & keep) | (unsigned)code);
          third[t] = __builtin_amdgcn_fmed3f(second[t], third[t], val);      // best >= second >= third
          second[t] = __builtin_amdgcn_fmed3f(best[t], second[t], val);
          // (as an instruction of its own: the compiler would canonicalise val first)
          asm("v_max_f32_e32 %0, %1, %2" : "=v"(best[t]) : "v"(best[t]), "v"(val));
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wavefront's part of the next buffer is in place
    __syncthreads();
  }
  float xnorm[2];                                          // |x| of this lane's two points
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    float nn = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint32_t ww[4] = {bx[t][ks].x, bx[t][ks].y, bx[t][ks].z, bx[t][ks].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) nn = dot2<BF>(ww[e], ww[e], nn);
    }
    nn += __shfl_xor(nn, 32);
    xnorm[t] = __builtin_sqrtf(nn + 2e-36f) * 1.0001f;     // (128 squares below 2^-126 may be missing)
  }
  const float cnorm = km_offset(v, u)->norm;
  float xc[2] = {0.f, 0.f};                                // <x, offset> of the two points
  if (cnorm > 0.f) {                                       // workgroup-uniform
    const uint16_t* cb = km_offset(v, u)->bits + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint4 w = *(const uint4*)(cb + ks * 16);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        xc[t] = dot2<BF>(bx[t][ks].w, w.w, dot2<BF>(bx[t][ks].z, w.z, dot2<BF>(bx[t][ks].y, w.y, dot2<BF>(bx[t][ks].x, w.x, xc[t]))));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) xc[t] += __shfl_xor(xc[t], 32);
  }
  if (first && !sums_order_free_by_type(DT, N0)) {         // the exponents of the unit's coordinates, once
    unsigned lo16 = 0xFFFFu, hi16 = 0u;                    // smallest (zeros left out, minus one) and largest magnitude bits
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const uint32_t ww[4] = {bx[t][ks].x, bx[t][ks].y, bx[t][ks].z, bx[t][ks].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned mag = (ww[e >> 1] >> ((e & 1) * 16)) & 0x7FFFu;
          hi16 = max(hi16, mag);
          lo16 = min(lo16, (mag - 1u) & 0xFFFFu);
        }
      }
    const int hiw = wave_max((int)hi16), low = wave_min((int)lo16);
    if (lane == 0 && hiw > 0) {
      constexpr int mbits = BF ? 7 : 10, bias = BF ? 127 : 15, emask = BF ? 255 : 31;
      const int eh = hiw >> mbits, el = (low + 1) >> mbits;
      // subnormals share the grid of the smallest normal exponent; infinities and NaNs make the range unusable
      atomicMax(&v.xrange[4 * u + 1], eh == emask ? 0x3FFFFFFF : max(eh, 1) - bias);
      atomicMin(&v.xrange[4 * u], max(el, 1) - bias);
    }
  }
  // the two halves of every point's centres; afterwards lane l speaks for point pbase + l
  float pb = kLow, ps = kLow, pt3 = kLow, pn = 0.f, pc = 0.f;
  int ib = 0, is = 0;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    auto number = [&](float x, int hh) {
      const unsigned code = __float_as_uint(x) & ~keep;
      return (int)((code >> 4) * 32 + 8 * ((code & 15) >> 2) + 4 * hh + (code & 3));
    };
    const float ob = __shfl_xor(best[t], 32), os = __shfl_xor(second[t], 32), o3 = __shfl_xor(third[t], 32);
    const bool mine = best[t] > ob || (best[t] == ob && h == 0);
    const float u1 = mine ? ob : best[t];                              // the loser of the two bests
    const bool s_mine = second[t] > os || (second[t] == os && h == 0);
    const float u2 = s_mine ? second[t] : os;
    const int n1 = mine ? number(ob, h ^ 1) : number(best[t], h), n2 = s_mine ? number(second[t], h) : number(os, h ^ 1);
    if (t == h) {
      pb = mine ? best[t] : ob;
      ib = mine ? number(best[t], h) : number(ob, h ^ 1);
      ps = fmaxf(u1, u2);
      is = u1 >= u2 ? n1 : n2;
      pt3 = fmaxf(fminf(u1, u2), fmaxf(third[t], o3));
      pn = xnorm[t];
      pc = xc[t];
    }
  }
  const int pt = pbase + lane;
  const bool valid = pt < N0;
  const float rmax = v.rmax[2 * u], rho = v.rmax[2 * u + 1];
  const float code_err = (float)(1 << code_bits) * 1.2e-7f * fabsf(pb);
  // |x - offset|^2, not below: the norms are rounded up, the product errs by 128 * 2^-24 of theirs at most
  const float y2 = fmaxf(pn * pn - 2.f * pc + cnorm * cnorm, 0.f) + 1e-4f * pn * cnorm;
  const float slack = (float)NT / 16384.0f * ((pn + cnorm) * rmax + rmax * rmax) + 4.f * pn * rho + 4.f * code_err;
  const float B = fminf(rmax, __builtin_sqrtf(y2) + __builtin_sqrtf(fmaxf(y2 - 2.f * pb, 0.f) + slack));
  const float eps = pn * rho * 1.0001f + (float)NT / 65536.0f * ((pn + cnorm) * B + 0.5f * B * B) * 1.01f + code_err + 1e-35f;
  const bool near2 = valid && !(pb - ps > 2.f * eps);
  const bool near3 = near2 && !(pb - pt3 > 2.f * eps);
  int label = min(ib, v.M0 - 1);                           // (padding rows win where no value is finite; such a point is near3)
  is = min(is, v.M0 - 1);
  const float* rows = km_rows(v, u);
  int at3 = -1;
  if (near3) { at3 = atomicAdd(&s_n3, 1); s_list[at3] = (short)(wave * 64 + lane); }
  unsigned long long m2 = __ballot(near2 && !near3), swap = 0ull;
  while (m2) {                                             // four points at a time, sixteen lanes each, 8 coordinates per lane
    int owner[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      owner[g] = m2 ? (int)__builtin_ctzll(m2) : g ? owner[g - 1] : 0;
      m2 &= m2 - 1;
    }
    const int g = lane >> 4, c = lane & 15;
    const int o = g == 0 ? owner[0] : g == 1 ? owner[1] : g == 2 ? owner[2] : owner[3];
    const int ja = __shfl(label, o), jb = __shfl(is, o);
    float x[8];
    load8(X, ((size_t)u * N0 + min(pbase + o, N0 - 1)) * kHeadDim + c * 8, DT, x);
    const f4* ra = (const f4*)(rows + (size_t)ja * kHeadDim + c * 8);
    const f4* rb = (const f4*)(rows + (size_t)jb * kHeadDim + c * 8);
    const f4 a0 = ra[0], a1 = ra[1], b0 = rb[0], b1 = rb[1];
    double da = 0.0, db = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double ta = (double)x[e] - (double)(e < 4 ? a0[e] : a1[e - 4]), tb = (double)x[e] - (double)(e < 4 ? b0[e] : b1[e - 4]);
      da = fma(ta, ta, da); db = fma(tb, tb, db);
    }
    da = row_blocked16(da); db = row_blocked16(db);
    const unsigned long long take = __ballot(c == 15 && (db < da || (db == da && jb < ja))) >> 15;
#pragma unroll
    for (int gg = 0; gg < 4; ++gg)
      if ((take >> (16 * gg)) & 1ull) swap |= 1ull << owner[gg];
  }
  if ((swap >> lane) & 1ull) label = is;
  // points with three or more candidates: all centres in float64, lane = centre.  One point alone: its centres are dealt
  // to all wavefronts.  Several: four at a time per wavefront, against two centres per lane.
  __syncthreads();
  const int n3 = s_n3;
  for (int q0 = 0; q0 < n3;) {                             // workgroup-uniform
    const bool alone = n3 - q0 == 1;
    const int share = scan_share(v.M0, alone ? 1 : kScanCentres), mine = wave % share, group = wave / share;
    const int nq = alone ? 1 : min(n3 - q0, kScanPoints * (NW / share));
    double* xd = (double*)sA;                              // the buffers of the filter are dead
    for (int t = tid; t < nq * 16; t += NW * 64) {
      float x[8];
      load8(X, ((size_t)u * N0 + xb * NW * 64 + s_list[q0 + (t >> 4)]) * kHeadDim + (t & 15) * 8, DT, x);
#pragma unroll
      for (int e = 0; e < 8; e += 2) *(double2*)(xd + t * 8 + e) = double2{(double)x[e], (double)x[e + 1]};
    }
    __syncthreads();
    const int p0 = group * kScanPoints;
    if (alone) {
      if (group == 0) scan_centres<1, 1>(v, u, xd, 1, mine, share, s_d, s_j);
    } else if (p0 < nq) {
      scan_centres<kScanPoints, kScanCentres>(v, u, xd + p0 * kHeadDim, min(kScanPoints, nq - p0), mine, share, s_d + p0, s_j + p0);
    }
    __syncthreads();
    if (at3 >= q0 && at3 < q0 + nq) {
      double bd = s_d[at3 - q0][0];
      int bj = s_j[at3 - q0][0];
      for (int w = 1; w < share; ++w) {
        const double od = s_d[at3 - q0][w];
        const int oj = s_j[at3 - q0][w];
        if (od < bd || (od == bd && oj < bj)) { bd = od; bj = oj; }
      }
      label = bj < v.M0 ? bj : 0;                          // (a key that is not finite is at no finite distance from any)
    }
    __syncthreads();
    q0 += nq;
  }
  int* lab = v.labels + (size_t)u * v.Ncap;
  if (first) {
    if (valid) lab[pt] = label;
    return;
  }
  const bool moved = valid && old != label;
  const unsigned long long mv = __ballot(moved);
  if (mv == 0) return;
  int base = 0;
  if (lane == 0) base = atomicAdd(&km_changed_count(v, u, slot), __popcll(mv));
  base = __builtin_amdgcn_readfirstlane(base);
  if (moved) {
    lab[pt] = label;
    km_changed(v, u)[base + __popcll(mv & ((1ull << lane) - 1ull))] = Changed{pt, (unsigned)old | ((unsigned)label << 16)};
  }
}

// ---- members of every cluster -------------------------------------------------------------------------------------
// Stable counting sort of one unit's labels by a workgroup of 1024: members of every cluster in ascending position
// (v.order) and the start of every cluster (v.koff).  Each of the first nw wavefronts counts a contiguous range of
// positions, one prefix sum over (cluster, wavefront) turns the counts into places, and each wavefront hands them out in
// order, 64 positions at a time: the lanes with equal labels find each other by one ballot per bit of the label.
// cnt: kSortCounters ints of LDS; sm: 64.  Returns (to every thread) whether some cluster has no member.  (A bitonic sort of (label, position) in LDS took 53 us for 4096 keys and
// 212 us for 16384; this takes 8 and 25 us.)
constexpr int kSortCounters = 32768;
static_assert(kMaxInitClusters * 4 <= kSortCounters, "at least four wavefronts hold counters");
__device__ inline bool sort_members(const View& v, int u, int N0, int* cnt, int* sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, M0 = v.M0;
  int nw = 16;
  while (nw * M0 > kSortCounters) nw >>= 1;
  const int* lab = v.labels + (size_t)u * v.Ncap;
  int* order = v.order + (size_t)u * v.Ncap;
  int* koff = v.koff + (size_t)u * (v.Mcap + 1);
  for (int i = tid; i < nw * M0; i += 1024) cnt[i] = 0;
  __syncthreads();
  const int per = ((N0 + nw - 1) / nw + 63) & ~63, b = min(N0, wave * per), e = wave < nw ? min(N0, b + per) : b;
  for (int i = b + lane; i < e; i += 64) atomicAdd(&cnt[wave * M0 + lab[i]], 1);
  __syncthreads();
  const int R = (M0 + 1023) / 1024;                   // consecutive clusters per thread
  int tot = 0, empty = 0;
  for (int k = 0; k < R; ++k) {
    const int j = tid * R + k;
    if (j >= M0) break;
    int n = 0;
    for (int w = 0; w < nw; ++w) n += cnt[w * M0 + j];
    tot += n; empty |= n == 0;
  }
  int total;
  int run = block_excl_scan(tot, sm, total);
  for (int k = 0; k < R; ++k) {
    const int j = tid * R + k;
    if (j >= M0) break;
    koff[j] = run;
    for (int w = 0; w < nw; ++w) { const int n = cnt[w * M0 + j]; cnt[w * M0 + j] = run; run += n; }
  }
  if (tid == 0) koff[M0] = N0;
  const bool any_empty = __syncthreads_or(empty);
  int bits = 0;
  while ((1 << bits) < M0) ++bits;
  for (int i0 = b; i0 < e; i0 += 64) {                 // (no barrier inside: ranges differ from wavefront to wavefront)
    const int i = i0 + lane;
    const bool in = i < e;
    const int l = in ? lab[i] : 0;
    unsigned long long same = __ballot(in);
    for (int k = 0; k < bits; ++k) {
      const unsigned long long bal = __ballot((l >> k) & 1);
      same &= ((l >> k) & 1) ? bal : ~bal;
    }
    if (in) {
      const int rank = __popcll(same & ((1ull << lane) - 1ull)), at = cnt[wave * M0 + l];
      order[at + rank] = i;
      asm volatile("" ::: "memory");
      if (rank == __popcll(same) - 1) cnt[wave * M0 + l] = at + rank + 1;       // (lock step: every lane has read the counter)
    }
    asm volatile("" ::: "memory");
  }
  __syncthreads();
  return any_empty;
}
__global__ __launch_bounds__(1024) void kmeans_sort_kernel(View v, int N0, int last) {
  __shared__ int cnt[kSortCounters];
  __shared__ int sm[64];
  const int u = blockIdx.x, tid = threadIdx.x;
  const bool any_empty = sort_members(v, u, N0, cnt, sm);
  if (tid == 0) v.has_empty[u] = any_empty;
  if (!last) return;
  // the labels are final: the first page of every cluster, for the layout
  const int* koff = v.koff + (size_t)u * (v.Mcap + 1);
  const int R = (v.M0 + 1023) / 1024;
  auto pages = [&](int j) { return j < v.M0 ? (koff[j + 1] - koff[j] + kPageTokens - 1) / kPageTokens : 0; };
  int n = 0, total;
  for (int k = 0; k < R; ++k) n += pages(tid * R + k);
  int base = block_excl_scan(n, sm, total);
  for (int k = 0; k < R && tid * R + k < v.M0; ++k) {
    v.pg_off[(size_t)u * v.Mcap + tid * R + k] = base;
    base += pages(tid * R + k);
  }
}

// ---- update ---------------------------------------------------------------------------------------------
// Sixteen lanes, eight coordinates each, form the sum of cluster j's members in the order of v.order (ascending
// position: Eq. 4 in a fixed order) and write centre, sums and count.  The lanes fetch the next 16 member positions with
// one load while the current 16 rows, all in flight at once, are added.  A cluster without members keeps its centre.
// RB: rows in flight per lane.
template <int DT, int RB = 16>
__device__ inline void update_cluster(const View& v, const void* X, int N0, int u, int j, int c, int* counts, const OffsetPart& off,
                                      CentreNorms& cn) {
  const int* koff = v.koff + (size_t)u * (v.Mcap + 1);
  const int* order = v.order + (size_t)u * v.Ncap;
  const int b = koff[j], e = koff[j + 1];
  if (DT != DYNAKV_F32 && c == 0) counts[j] = e - b;
  double s[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) s[k] = 0.0;
  if (e > b) {
    int mine = b + c < e ? order[b + c] : 0;            // lane c holds member c of the current 16
    for (int q0 = b; q0 < e; q0 += 16) {
      const int next = q0 + 16 + c < e ? order[q0 + 16 + c] : 0;
#pragma unroll
      for (int h = 0; h < 16; h += RB) {
        float x[RB][8];
#pragma unroll
        for (int k = 0; k < RB; ++k) {
          const int pos = __shfl(mine, h + k, 16);
          load8(X, ((size_t)u * N0 + pos) * kHeadDim + c * 8, DT, x[k]);
        }
#pragma unroll
        for (int k = 0; k < RB; ++k)
          if (q0 + h + k < e) {
#pragma unroll
            for (int d = 0; d < 8; ++d) s[d] += (double)x[k][d];
          }
      }
      mine = next;
    }
    float r[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) r[d] = (float)(s[d] / (double)(e - b));
    write_centre<DT>(v, u, j, c, r, off, cn);
  }
  if constexpr (DT != DYNAKV_F32) {
    double* S = km_sums(v, u) + (size_t)j * kHeadDim + c * 8;
#pragma unroll
    for (int d = 0; d < 8; d += 2) *(double2*)(S + d) = double2{s[d], s[d + 1]};
  }
}
// All sums formed anew from the sorted members.  A unit with empty clusters is left to kmeans_slow_kernel (it needs the old
// centres), except in the last iteration, where they stay empty.  grid (ceil(M0/16), U).
template <int DT>
__global__ __launch_bounds__(256) void kmeans_update_kernel(View v, const void* X, int N0, int which, int last) {
  __shared__ int sm[8];
  const int u = blockIdx.y, j = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  if (v.has_empty[u] && !last) return;                  // workgroup-uniform
  CentreNorms cn{0.f, 0.f};
  if (j < v.M0) update_cluster<DT>(v, X, N0, u, j, c, km_counts(v, u, N0, which), load_offset<DT>(v, u, c), cn);
  if constexpr (DT != DYNAKV_F32) fold_norms(v, u, cn, sm);
}

// dist[i] = squared distance of point i to the centre of its own cluster for the points first, first + step, .. (sixteen lanes
// each, eight points in flight).
template <int DT>
__device__ __forceinline__ void own_distances(const View& v, const void* X, int N0, int u, int first, int step) {
  const int c = threadIdx.x & 15;
  const int* lab = v.labels + (size_t)u * v.Ncap;
  double* dist = v.dist + (size_t)u * v.Ncap;
  const float* R = unit_R(v, u);
  constexpr int kPts = DT == DYNAKV_F32 ? 4 : 8;
  for (int i0 = first; i0 < N0; i0 += step * kPts) {
    float x[kPts][8];
    f4 ra[kPts], rb[kPts];
#pragma unroll
    for (int k = 0; k < kPts; ++k) {
      const int i = min(i0 + step * k, N0 - 1), j = lab[i];
      load8(X, ((size_t)u * N0 + i) * kHeadDim + c * 8, DT, x[k]);
      if constexpr (DT == DYNAKV_F32) { ra[k] = *(const f4*)(R + r_index(j, c * 8)); rb[k] = *(const f4*)(R + r_index(j, c * 8 + 4)); }
      else { const f4* r = (const f4*)(km_rows(v, u) + (size_t)j * kHeadDim + c * 8); ra[k] = r[0]; rb[k] = r[1]; }
    }
#pragma unroll
    for (int k = 0; k < kPts; ++k) {
      double acc = 0.0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double t = (double)x[k][e] - (double)(e < 4 ? ra[k][e] : rb[k][e - 4]);
        acc = fma(t, t, acc);
      }
      acc = row_blocked16(acc);
      if (c == 15 && i0 + step * k < N0) dist[i0 + step * k] = acc;
    }
  }
}

// The sums follow the points that changed their cluster (16-bit types whose sums are order-free).  A workgroup takes 16
// clusters: it reads the unit's list of changes once, counts every cluster's members (counts are kept twice, the old ones
// are still being read by other workgroups) and queues the changes of its own clusters in LDS; sixteen lanes per cluster then
// add and subtract the rows.  If some cluster of the unit has run empty, the centres are left to kmeans_slow_kernel.  Bound by the dependent round trips list - rows - sums; the list is short after the first iterations.
// A cluster with more changes than its queue holds (hundreds of keys per cluster, or one cluster that most keys share) has its
// sixteen lanes go through the list again, 64 entries at a time.  (One entry at a time: 64 units x 16384 float16 keys x 64
// centres build in 4.5 ms, 8 x 16384 bfloat16 x 128 in 2.4; now 3.1 and 1.7.)
constexpr int kQueue = 96, kLook = 4, kRowsAhead = 8;
template <int DT>
__global__ __launch_bounds__(256) void kmeans_changed_kernel(View v, const void* X, int N0, int slot, int which, int last) {
  extern __shared__ int delta[];                        // [M0]
  __shared__ int queue[16][kQueue], nq[16];
  __shared__ int any_empty, sm[8];
  const int u = blockIdx.y, tid = threadIdx.x, j0 = blockIdx.x * 16;
  if (!sums_order_free(v, u, N0)) return;               // workgroup-uniform
  const int n = km_changed_count(v, u, slot);
  const Changed* chg = km_changed(v, u);
  const int* was = km_counts(v, u, N0, which ^ 1);
  int* now = km_counts(v, u, N0, which);
  const int c = tid & 15;
  const OffsetPart off = load_offset<DT>(v, u, c);
  for (int i = tid; i < v.M0; i += 256) delta[i] = 0;
  if (tid < 16) nq[tid] = 0;
  if (tid == 0) any_empty = 0;
  __syncthreads();
  for (int i = tid; i < n; i += 256) {
    const Changed ch = chg[i];
    const int from = (int)(ch.move & 0xFFFFu), to = (int)(ch.move >> 16);
    atomicAdd(&delta[from], -1);
    atomicAdd(&delta[to], 1);
    if ((unsigned)(from - j0) < 16u) {
      const int at = atomicAdd(&nq[from - j0], 1);
      if (at < kQueue) queue[from - j0][at] = ch.pos << 1 | 1;
    }
    if ((unsigned)(to - j0) < 16u) {
      const int at = atomicAdd(&nq[to - j0], 1);
      if (at < kQueue) queue[to - j0][at] = ch.pos << 1;
    }
  }
  __syncthreads();
  bool centres = true;
  if (!last) {
    for (int i = tid; i < v.M0; i += 256)
      if (was[i] + delta[i] == 0) any_empty = 1;
    __syncthreads();
    if (any_empty) {                                    // the same in every workgroup of the unit
      // the sums follow as ever, but the old centres stay until kmeans_slow_kernel has chosen points for the empty
      // clusters: by their distances to those centres, of which each workgroup takes a share
      centres = false;
      if (blockIdx.x == 0 && tid == 0) v.has_empty[u] = 1;
      own_distances<DT>(v, X, N0, u, blockIdx.x * 16 + (tid >> 4), gridDim.x * 16);
    }
  }
  const int k = tid >> 4, j = j0 + k;
  CentreNorms cn{0.f, 0.f};
  if (j < v.M0) {
    const int m = was[j] + delta[j], q = nq[k];
    if (c == 0) now[j] = m;
    if (q > 0) {
      double* S = km_sums(v, u) + (size_t)j * kHeadDim + c * 8;
      double s[8];
#pragma unroll
      for (int d = 0; d < 8; d += 2) { const double2 w = *(const double2*)(S + d); s[d] = w.x; s[d + 1] = w.y; }
      auto apply = [&](const float (&x)[8], bool out) __attribute__((always_inline)) {
#pragma unroll
        for (int d = 0; d < 8; ++d) s[d] += out ? -(double)x[d] : (double)x[d];
      };
      auto drain = [&](int have) __attribute__((always_inline)) {
        for (int i0 = 0; i0 < have; i0 += kRowsAhead) {  // so many rows in flight
          float x[kRowsAhead][8];
          int e[kRowsAhead];
#pragma unroll
          for (int i = 0; i < kRowsAhead; ++i) {
            e[i] = queue[k][min(i0 + i, have - 1)];
            load8(X, ((size_t)u * N0 + (e[i] >> 1)) * kHeadDim + c * 8, DT, x[i]);
          }
#pragma unroll
          for (int i = 0; i < kRowsAhead; ++i)
            if (i0 + i < have) apply(x[i], e[i] & 1);
        }
      };
      if (q <= kQueue) drain(q);
      else {                                            // more changes than the queue holds: it is filled again and again
        int have = 0;
        for (int i0 = 0; i0 < n; i0 += 16 * kLook) {
          Changed ch[kLook];
#pragma unroll
          for (int l = 0; l < kLook; ++l) ch[l] = chg[min(i0 + l * 16 + c, n - 1)];
#pragma unroll
          for (int l = 0; l < kLook; ++l) {
            const bool out = (int)(ch[l].move & 0xFFFFu) == j;
            const bool hit = i0 + l * 16 + c < n && (out || (int)(ch[l].move >> 16) == j);
            const unsigned hits = (unsigned)(__ballot(hit) >> (tid & 48)) & 0xFFFFu;
            if (hit) queue[k][have + __popc(hits & ((1u << c) - 1u))] = ch[l].pos << 1 | (int)out;
            have += __popc(hits);
          }
          asm volatile("" ::: "memory");                 // (one wavefront: LDS keeps program order, the compiler must too)
          if (have > kQueue - 16 * kLook || i0 + 16 * kLook >= n) { drain(have); have = 0; }
          asm volatile("" ::: "memory");
        }
      }
#pragma unroll
      for (int d = 0; d < 8; d += 2) *(double2*)(S + d) = double2{s[d], s[d + 1]};
      if (m > 0 && centres) {
        float r[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) r[d] = (float)(s[d] / (double)m);
        write_centre<DT>(v, u, j, c, r, off, cn);
      }
    }
  }
  if (centres) fold_norms(v, u, cn, sm);                // (workgroup-uniform)
}

// Largest (value, index) of a wavefront, lowest index among equal values, index < 0: none.  Every lane of the last row gets it
// (ROW: every lane of a row gets its row's).
template <int CTRL, int ROWS>
__device__ __forceinline__ void far_step(double& val, int& idx) {
  const int lo = dpp_or<CTRL, ROWS>(__double2loint(val), __double2loint(val)), hi = dpp_or<CTRL, ROWS>(__double2hiint(val), __double2hiint(val));
  const int oi = dpp_or<CTRL, ROWS>(idx, idx);
  const double ov = __hiloint2double(hi, lo);
  if (oi >= 0 && (idx < 0 || ov > val || (ov == val && oi < idx))) { val = ov; idx = oi; }
}
template <bool ROW>
__device__ __forceinline__ void far_reduce(double& val, int& idx) {
  far_step<kDppXor1, 0xF>(val, idx);
  far_step<kDppXor2, 0xF>(val, idx);
  far_step<kDppHalfMirror, 0xF>(val, idx);
  far_step<kDppMirror, 0xF>(val, idx);
  if constexpr (!ROW) { far_step<kDppBcast15, 0xA>(val, idx); far_step<kDppBcast31, 0xC>(val, idx); }
}

// What the parallel kernels leave, in workgroups of 1024.  Most launches find nothing to do (4.5 us); where the first centres
// leave some cluster empty, one or two iterations do.
//   units with an empty cluster, one workgroup each: every empty cluster, in ascending id, takes the not-yet-taken point that is
//     farthest from its own (old) centre, ties to the lowest position; the others get their centres from their sums, which the
//     changes have followed (256 units x 4096 x 256: 46 us; 160 us while this workgroup took all distances and sums itself)
//   units whose sums are not order-free, in every iteration after the first: all sums formed anew.  Each of the unit's
//     gridDim.y workgroups sorts the labels for itself (all write the same order) and takes its share of the clusters
// The points' distances stay in registers while the empty clusters choose, and their centres are written together afterwards:
// with some 200 empty clusters in each of ten iterations (2 units x 4096 float16 keys of 300 values x 512 centres) a launch
// took 1180 us when every choice wrote its centre and read all distances again, now 610.
// A workgroup has room for 64 clusters at a time; where few units leave the chip idle, each gets as many workgroups as that
// (8 units x 16384 bfloat16 keys x 2048 centres, not order-free: 4 workgroups a unit 100 us, 32 52 us).
// (One workgroup per compute unit at most, for launches that find nothing to do; one per unit where no sums are formed anew.)
constexpr int kSlowShare = 64, kSlowMost = 256;          // clusters per workgroup, workgroups of a launch
inline int slow_workgroups(const View& v, int N0) {
  if (v.dtype == DYNAKV_F32 || sums_order_free_by_type(v.dtype, N0)) return 1;
  const int few = std::min(16, (v.M0 + 511) / 512);      // (many units: one for every 512 clusters)
  return std::max(few, std::min(std::min(32, (v.M0 + kSlowShare - 1) / kSlowShare), kSlowMost / v.U));
}
template <int DT>
__global__ __launch_bounds__(1024) void kmeans_slow_kernel(View v, const void* X, int N0, int which, int first, int last) {
  __shared__ int cnt[kSortCounters];
  __shared__ int sm[64];
  __shared__ double sv[2][16];
  __shared__ int si[2][16];
  const int u = blockIdx.x, tid = threadIdx.x, c = tid & 15;
  const bool sorted = first || DT == DYNAKV_F32;         // this iteration's kmeans_sort_kernel has run
  const bool anew = !sorted && !sums_order_free(v, u, N0);
  if (!anew && (blockIdx.y > 0 || last || !v.has_empty[u])) return;       // workgroup-uniform
  const bool any_empty = sorted || !anew ? true : sort_members(v, u, N0, cnt, sm);
  const bool reseed = any_empty && !last;
  if (reseed && blockIdx.y > 0) return;
  const int* koff = v.koff + (size_t)u * (v.Mcap + 1);
  const double* dist = v.dist + (size_t)u * v.Ncap;
  const bool follows = !sorted && !anew;                 // kmeans_changed_kernel has taken sums, counts and distances
  if (reseed && !follows) {                             // distances to the centres of this assignment, before the update
    own_distances<DT>(v, X, N0, u, tid >> 4, 64);
    __syncthreads();
  }
  CentreNorms cn{0.f, 0.f};
  int* counts = km_counts(v, u, N0, which);
  const int share = reseed ? 1 : gridDim.y, mine = reseed ? 0 : blockIdx.y;
  if (follows) {
    const OffsetPart off = load_offset<DT>(v, u, c);
    for (int j = tid >> 4; j < v.M0; j += 64) {
      const int m = counts[j];
      if (m == 0) continue;
      const double* S = km_sums(v, u) + (size_t)j * kHeadDim + c * 8;
      float r[8];
#pragma unroll
      for (int d = 0; d < 8; d += 2) {
        const double2 w = *(const double2*)(S + d);
        r[d] = (float)(w.x / (double)m); r[d + 1] = (float)(w.y / (double)m);
      }
      write_centre<DT>(v, u, j, c, r, off, cn);
    }
  } else
  for (int j = mine * 64 + (tid >> 4); j < v.M0; j += share * 64)
    update_cluster<DT, DT == DYNAKV_F32 ? 8 : 16>(v, X, N0, u, j, c, counts, load_offset<DT>(v, u, c), cn);
  if (reseed) {
    const int lane = tid & 63, w = tid >> 6;
    int* const ids = cnt;                                // empty clusters, ascending
    int* const pick = cnt + kMaxInitClusters;            // the points they take
    const int R = (v.M0 + 1023) / 1024;
    auto empty = [&](int j) { return j < v.M0 && (follows ? counts[j] == 0 : koff[j + 1] == koff[j]); };
    int mine_empty = 0, n;
    for (int k = 0; k < R; ++k) mine_empty += empty(tid * R + k);
    int at = block_excl_scan(mine_empty, sm, n);
    for (int k = 0; k < R; ++k)
      if (empty(tid * R + k)) ids[at++] = tid * R + k;
    constexpr int kHeld = kMaxPrefill / 1024;
    double d[kHeld];                                     // points tid, tid + 1024, ..
#pragma unroll
    for (int k = 0; k < kHeld; ++k) d[k] = tid + 1024 * k < N0 ? dist[tid + 1024 * k] : -2.0;
    int taken = 0;
    for (; taken < n; ++taken) {
      double bv = -1.0;
      int bi = -1;
#pragma unroll
      for (int k = 0; k < kHeld; ++k)
        if (d[k] > bv) { bv = d[k]; bi = tid + 1024 * k; }          // ascending: the first maximum stays
      far_reduce<false>(bv, bi);
      if (lane == 63) { sv[taken & 1][w] = bv; si[taken & 1][w] = bi; }
      lds_barrier();                                     // (two places in turn: one barrier per choice)
      bv = sv[taken & 1][lane & 15]; bi = si[taken & 1][lane & 15];
      far_reduce<true>(bv, bi);
      if (bi < 0) break;                                 // every point already taken (the same in every thread)
#pragma unroll
      for (int k = 0; k < kHeld; ++k)
        if (bi == tid + 1024 * k) d[k] = -2.0;
      if (tid == 0) pick[taken] = bi;
    }
    __syncthreads();
    for (int e = tid >> 4; e < taken; e += 64) {
      float r[8];
      load8(X, ((size_t)u * N0 + pick[e]) * kHeadDim + c * 8, DT, r);
      write_centre<DT>(v, u, ids[e], c, r, load_offset<DT>(v, u, c), cn);
    }
  }
  if constexpr (DT != DYNAKV_F32) fold_norms(v, u, cn, sm);
  if (blockIdx.y == 0 && tid == 0) v.has_empty[u] = 0;
}

// 16 consecutive entries of the sorted order per workgroup, 16 lanes per entry, 8 coordinates per lane: keys and values move
// as whole 16-byte chunks of their token's rows, and dist[q] = squared distance of entry q of that order to the (updated)
// centre of its own cluster, taken while its key is at hand.  Entries lie in cluster order, so the 16 of a workgroup mostly share one
// centre and its lines of the lane-interleaved table are fetched once.  Bound by memory: 256 units x 4096 float16 entries 0.54 GB
// read and as much written (221 us; a distance pass of its own read the keys once more: 317 us together).
template <int DT>
__global__ __launch_bounds__(256) void layout_copy_kernel(View v, const void* K, const void* V, int N0) {
  const int u = blockIdx.y, q = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  const int pos = v.order[(size_t)u * v.Ncap + min(q, N0 - 1)];
  const int j = v.labels[(size_t)u * v.Ncap + pos];
  const size_t src = ((size_t)u * N0 + pos) * kHeadDim + c * 8;
  float x[8];
  uint4 kb[DT == DYNAKV_F32 ? 2 : 1], vb[DT == DYNAKV_F32 ? 2 : 1];
  constexpr int kEs = DT == DYNAKV_F32 ? 4 : 2;
#pragma unroll
  for (int h = 0; h < kEs / 2; ++h) {
    kb[h] = ((const uint4*)((const char*)K + src * kEs))[h];
    vb[h] = ((const uint4*)((const char*)V + src * kEs))[h];
  }
  const float* R = unit_R(v, u);
  const f4 ra = *(const f4*)(R + r_index(j, c * 8)), rb = *(const f4*)(R + r_index(j, c * 8 + 4));
  const int rank = q - v.koff[(size_t)u * (v.Mcap + 1) + j];
  const int page = v.pg_off[(size_t)u * v.Mcap + j] + rank / kPageTokens, slot = rank % kPageTokens;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint4 w = kb[e / (16 / kEs)];
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
    if constexpr (DT == DYNAKV_F32) x[e] = __uint_as_float(ww[e & 3]);
    else x[e] = bits_value((ww[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu, DT);
  }
  double acc = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double t = (double)x[e] - (double)(e < 4 ? ra[e] : rb[e - 4]);
    acc = fma(t, t, acc);
  }
  acc = row_blocked16(acc);
  if (q >= N0) return;
  char* pg = page_ptr(v, u, page);
#pragma unroll
  for (int h = 0; h < kEs / 2; ++h) {
    ((uint4*)(pg + (size_t)k_index(DT, slot, c * 8) * kEs))[h] = kb[h];
    ((uint4*)(pg + (size_t)v_index(DT, slot, c * 8) * kEs))[h] = vb[h];
  }
  if (c == 0) v.ppos[((size_t)u * v.Pcap + page) * kPageTokens + slot] = pos;
  if (c == 15) v.dist[(size_t)u * v.Ncap + q] = acc;
}

// One workgroup per unit, last kernel of a build: per-cluster n, M2 (members in order), page chains, tau, counters, the search
// copy.  Consecutive threads take consecutive clusters throughout, so that every array is written in whole lines.
__global__ __launch_bounds__(1024) void finalize_kernel(View v, int N0) {
  __shared__ double jsum[16];                   // per-wavefront sums of M2, for the objective that gives tau
  const int u = blockIdx.x, tid = threadIdx.x;
  const int* koff = v.koff + (size_t)u * (v.Mcap + 1);
  const double* dist = v.dist + (size_t)u * v.Ncap;
  const size_t cb = (size_t)u * v.Mcap;
  // M2 of cluster j = sum of its members' distances in storage order: one thread per cluster, eight members requested at a
  // time, added one by one
  double jmine = 0.0;
  for (int j = tid; j < v.Mcap; j += 1024) {
    const bool in = j < v.M0;
    const int b = in ? koff[j] : 0, e = in ? koff[j + 1] : 0, np = (e - b + kPageTokens - 1) / kPageTokens;
    const int base = in ? v.pg_off[cb + j] : 0;
    v.cn[cb + j] = e - b; v.csz[cb + j] = e - b; v.ctail[cb + j] = np ? base + np - 1 : -1;
    v.cb[cb + j] = 0; v.cflag[cb + j] = 0; v.in_req[cb + j] = 0; v.score[cb + j] = 0.f;
    int4* pg = (int4*)&v.cpg[(cb + j) * kInlinePages];
    auto page = [&](int p) { return p < np ? base + p : -1; };
    pg[0] = int4{page(0), page(1), page(2), page(3)};
    pg[1] = int4{page(4), page(5), page(6), page(7)};
    for (int p = 0; p < np; ++p) v.pnext[(size_t)u * v.Pcap + base + p] = p + 1 < np ? base + p + 1 : -1;
    double m2 = 0.0;
    for (int q0 = b; q0 < e; q0 += 8) {
      double x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = dist[min(q0 + k, e - 1)];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (q0 + k < e) m2 += x[k];
    }
    v.cM2[cb + j] = m2;
    jmine += m2;
  }
  for (int o = 32; o > 0; o >>= 1) jmine += __shfl_xor(jmine, o);
  if ((tid & 63) == 0) jsum[tid >> 6] = jmine;
  if (v.dtype != DYNAKV_F32) {               // search copy of the final centroids, eight coordinates (16 bytes) at a time
    const float* R = unit_R(v, u);
    uint16_t* Rq = unit_Rq(v, u);
    for (int t = tid; t < ((v.M0 + 15) & ~15) * (kHeadDim / 8); t += 1024) {      // lane order of the copy's tiles: 16 clusters, then the next chunk
      const int tile = t / (16 * 16), r = t % (16 * 16), j = tile * 16 + (r & 15), d = (r >> 4) * 8;
      if (j >= v.M0) continue;
      const f4 a = *(const f4*)(R + r_index(j, d)), b = *(const f4*)(R + r_index(j, d + 4));
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = e < 2 ? a[2 * e] : b[2 * e - 4], hi = e < 2 ? a[2 * e + 1] : b[2 * e - 3];
        w[e] = (uint32_t)round_bits16(lo, v.dtype) | ((uint32_t)round_bits16(hi, v.dtype) << 16);
      }
      *(uint4*)(Rq + rq_index(j, d)) = uint4{w[0], w[1], w[2], w[3]};
    }
  }
  __syncthreads();
  if (tid == 0) {
    double J = 0.0;
    for (int w = 0; w < 16; ++w) J += jsum[w];
    const int last = v.M0 - 1, total = v.pg_off[cb + last] + (koff[v.M0] - koff[last] + kPageTokens - 1) / kPageTokens;
    v.tau[u] = (double)v.var_alpha * (J / (double)N0);
    v.M[u] = v.M0; v.N[u] = N0; v.nflag[u] = 0; v.n_sel[u] = 0; v.t_sel[u] = 0; v.n_list[u] = 0;
    v.ticket[u] = 0; v.ticket[v.U + u] = 0; v.ticket[2 * v.U + u] = 0; v.bump[u] = total;
    v.free_top[u] = 0; v.last_assign[u] = -1; v.lcount[u] = 0; v.rmax2[u] = 0;
    for (int k = 0; k < kCounters; ++k) v.counters[(size_t)u * kCounters + k] = 0;
  }
}

}  // namespace

template <int DT>
static void launch_kmeans(const View& v, const void* K, int N0, const int* init_idx, int iters, hipStream_t st) {
  const dim3 gcl((v.M0 + 15) / 16, v.U);
  kmeans_check_init_kernel<DT><<<v.U, 256, 0, st>>>(v, K, N0, init_idx);
  kmeans_start_kernel<DT><<<dim3(((DT == DYNAKV_F32 ? v.M0 : km_pad(v.M0)) + 15) / 16, v.U), 256, 0, st>>>(v, K, N0, init_idx);
  for (int it = 0; it < iters; ++it) {
    const int first = it == 0, last = it + 1 == iters, slot = it & 1, which = it & 1;
    if constexpr (DT == DYNAKV_F32) {
      kmeans_assign_f64_kernel<<<dim3((N0 + 63) / 64, v.U), 256, 0, st>>>(v, K, N0);
    } else {
      int code_bits = 4;                                // a lane sees half of the centres: 16 per tile of 32
      while ((1 << code_bits) < km_pad(v.M0) / 2) ++code_bits;
      const int gx = (N0 + 64 * kAssignWaves - 1) / (64 * kAssignWaves);
      kmeans_assign_kernel<DT><<<gx * ((v.U + 7) / 8 * 8), 64 * kAssignWaves, 0, st>>>(v, K, N0, gx, first, slot, code_bits);
    }
    if (first || DT == DYNAKV_F32) {
      kmeans_sort_kernel<<<v.U, 1024, 0, st>>>(v, N0, last);
      kmeans_update_kernel<DT><<<gcl, 256, 0, st>>>(v, K, N0, which, last);
    } else if constexpr (DT != DYNAKV_F32) {
      kmeans_changed_kernel<DT><<<gcl, 256, v.M0 * sizeof(int), st>>>(v, K, N0, slot, which, last);
    }
    const bool sorted = first || DT == DYNAKV_F32;
    if (!last || (!sorted && !sums_order_free_by_type(DT, N0)))
      kmeans_slow_kernel<DT><<<dim3(v.U, slow_workgroups(v, N0)), 1024, 0, st>>>(v, K, N0, which, first, last);
  }
  if (DT != DYNAKV_F32 && iters > 1) kmeans_sort_kernel<<<v.U, 1024, 0, st>>>(v, N0, 1);
}

hipError_t launch_build_index(const View& v, const void* K, const void* V, int N0, const int* init_idx, int iters,
                              void* ws, size_t ws_bytes, hipStream_t st) {
  (void)ws; (void)ws_bytes;
  if (v.dtype == DYNAKV_F32) launch_kmeans<DYNAKV_F32>(v, K, N0, init_idx, iters, st);
  else if (v.dtype == DYNAKV_F16) launch_kmeans<DYNAKV_F16>(v, K, N0, init_idx, iters, st);
  else launch_kmeans<DYNAKV_BF16>(v, K, N0, init_idx, iters, st);
  const dim3 grid((N0 + 15) / 16, v.U);
  if (v.dtype == DYNAKV_F32) layout_copy_kernel<DYNAKV_F32><<<grid, 256, 0, st>>>(v, K, V, N0);
  else if (v.dtype == DYNAKV_F16) layout_copy_kernel<DYNAKV_F16><<<grid, 256, 0, st>>>(v, K, V, N0);
  else layout_copy_kernel<DYNAKV_BF16><<<grid, 256, 0, st>>>(v, K, V, N0);
  finalize_kernel<<<v.U, 1024, 0, st>>>(v, N0);
  return hipGetLastError();
}

}  // namespace dynakv
