// knn.h -- KNN search on the assignment kernel's layout (bf16/fp16 rows,
// D a multiple of 16 up to 256): for every query, the k database rows at the
// smallest squared Euclidean distance, nearest first, ties to the lowest
// index.  The paper lists KNN build and search beside KMeans among the
// dispatcher-backed families of Section 6 (recall 1.0); this is the same fused
// distance contraction with a top-k in place of the arg-min, and the k x N
// distance matrix is never stored.  Instantiated once per storage type in
// knn_bf16.hip and knn_f16.hip.
//
// Queries play the points' role: each wave keeps 32 or 64 queries in registers
// (32-column MFMA tiles).  Database rows play the centroids' role: a first
// pass writes their -|r|^2/2 (the rows are already in the storage type, so
// nothing is rounded; rows whose width is not a multiple of 16 are copied into
// padded ones), and they stream through LDS in the assignment kernel's stages
// (direct L2-to-LDS loads, XOR-swizzled rows, double buffering).  When the
// query blocks do not fill the chip, each takes the rows in several shares
// (blockIdx.z) and knn_merge_kernel merges their lists.  Few queries go to
// knn_scan.h instead.
//
// Top-k.  Lane 32 h + n holds, for query n, the 16 scores of rows
// 8 q + 4 h + r of each 32-row tile, and keeps its own list of the KMAX best
// (score, index) in registers, best first.  Rows reach a lane in increasing
// index order, so a strict compare keeps equal scores in index order.  A tile
// costs one compare per score against the lane's KMAX-th best when no lane of
// the wave improves; otherwise a score enters by a compare-exchange pass down
// the list (branch-free per lane, one wave-uniform branch).  At the end the
// two halves' lists of a query merge by (score, then lower index), and the
// first k entries are written with d = max(0, |q|^2 - 2 s).
#pragma once

#include "assign_pipe.h"

namespace fkm {

// -|r|^2/2 of every database row, read in the stages' layout through LDS (one
// stage per workgroup, whole rows per load), and the rows of the last, partial
// stages copied to `tail` (ASSIGN_KPAD rows per instance from row `ntail0` on;
// zero rows with score -FLT_MAX past N), so that the search streams every
// other stage straight from the caller's array.  Replaces a copy of all rows:
// 275 -> 41 us at 1,048,576 x 128 bf16 (6.5 TB/s).
template <int DT, int CPL>
__global__ __launch_bounds__(256) void knn_norm_kernel(const uint4* __restrict__ R, int N, int Np,
                                                       int ntail0, float* __restrict__ cinit,
                                                       uint4* __restrict__ tail) {
  using L = PipeLayout<CPL>;
  constexpr int LOADS = L::TCS * L::RCP / ASSIGN_THREADS;
  __shared__ __attribute__((aligned(16))) char buf[L::CHUNKS];
  const int b = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, h = lane >> 5;
  R += (size_t)b * N * L::RC;
  PipeOffsets<CPL, LOADS> o;
  pipe_offsets<CPL, LOADS>(o, tid, n, h);
  const int row0 = blockIdx.x * L::TCS;
  pipe_issue_rows<CPL, LOADS>(R, row0, N, tid, buf);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (wave >= L::TILES) return;
  uint4 a[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) a[c] = lds_at<uint4>(buf, o.a[c] + wave * L::TILE, 0);
  float ss = tree_sumsq<DT, CPL>(a);
  ss += __shfl_xor(ss, 32);
  const int row = row0 + wave * 32 + n;
  if (h == 0) cinit[(size_t)b * Np + row] = row < N ? -0.5f * ss : -0x1.fffffep127f;
  if (row >= ntail0) {
    uint4* t = tail + ((size_t)b * ASSIGN_KPAD + (row - ntail0)) * L::RC + h * CPL;
#pragma unroll
    for (int c = 0; c < CPL; ++c) t[c] = row < N ? a[c] : make_uint4(0, 0, 0, 0);
  }
}

// Database rows to the staged layout: row j of each instance to chat (padded to
// Np rows: zero rows with score -FLT_MAX; rows of Din elements widened to D
// with zeros), and its -|r|^2/2.  A lane takes one 16-byte chunk of a row and a
// group of prep_lanes(D) lanes the row; the norm's chunks are added in the order of
// tree_sumsq, as by the kernels that read rows in place and by the scan, so a
// search has the same bits on every route.
__host__ __device__ inline int prep_lanes(int D) {
  int g = 2;
  while (g < D / 8) g *= 2;
  return g;
}
template <int DT>
__global__ __launch_bounds__(256) void knn_prep_kernel(const uint16_t* __restrict__ R, int64_t B,
                                                       int N, int Np, int Din, int D,
                                                       uint16_t* __restrict__ chat,
                                                       float* __restrict__ cinit) {
  const int g = prep_lanes(D), rc = D / 8, half = rc / 2;
  const int lane = threadIdx.x & 63, l = threadIdx.x % g;  // l: the lane's chunk
  const int64_t row = (int64_t)blockIdx.x * (256 / g) + threadIdx.x / g;
  if (row >= B * Np) return;  // whole groups
  const int64_t b = row / Np;
  const int j = (int)(row % Np);
  const bool pad = j >= N;
  uint4 q = make_uint4(0, 0, 0, 0);
  if (!pad && l < rc) {
    const uint16_t* r = R + (b * N + j) * Din;
    if (8 * l + 8 <= Din) {
      __builtin_memcpy(&q, r + 8 * l, 16);  // rows of any Din start at any 2-byte boundary
    } else {
      uint16_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = 8 * l + e < Din ? r[8 * l + e] : (uint16_t)0;
      __builtin_memcpy(&q, h, 16);
    }
  }
  if (l < rc) *reinterpret_cast<uint4*>(chat + row * D + 8 * l) = q;
  float ss = chunk_sumsq<DT>(q, 0.f);
  const int c = l < half ? l : l - half;
  for (int d = 1; d < half; d *= 2) {
    const float v = __shfl(ss, lane + d);
    if (c % (2 * d) == 0 && c + d < half) ss += v;
  }
  const float v = __shfl(ss, lane + half);
  if (l == 0) cinit[row] = pad ? -0x1.fffffep127f : -0.5f * (ss + v);
}

// Insert (s, i) into a best-first list: a compare-exchange pass down the list
// carries the displaced entry along; the last one falls off.
template <int KMAX>
__device__ __forceinline__ void knn_insert(float (&v)[KMAX], int (&ix)[KMAX], float s, int i) {
#pragma unroll
  for (int t = 0; t < KMAX; ++t) {
    const bool up = s > v[t];
    const float vt = v[t];
    const int it = ix[t];
    v[t] = up ? s : vt;
    ix[t] = up ? i : it;
    s = up ? vt : s;
    i = up ? it : i;
  }
}

// The same, ordering equal scores by index (merging two lists).
template <int KMAX>
__device__ __forceinline__ void knn_insert_by_index(float (&v)[KMAX], int (&ix)[KMAX], float s,
                                                    int i) {
#pragma unroll
  for (int t = 0; t < KMAX; ++t) {
    const bool up = s > v[t] || (s == v[t] && i < ix[t]);
    const float vt = v[t];
    const int it = ix[t];
    v[t] = up ? s : vt;
    ix[t] = up ? i : it;
    s = up ? vt : s;
    i = up ? it : i;
  }
}

// The MFMAs of one 32-row tile (tile index at run time) into acc, one
// accumulator per 32-query tile: each row fragment read from LDS feeds NSUB
// MFMAs, and the scores are read once for all of them.
template <int DT, int CPL, int NSUB, int LOADS>
__device__ __forceinline__ void knn_mfma_tile(f32x16 (&acc)[NSUB], const uint4 (&xr)[NSUB][CPL],
                                              char* buf, const PipeOffsets<CPL, LOADS>& o,
                                              int tile) {
  using L = PipeLayout<CPL>;
  f32x16 cin;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = lds_at<f32x4>(buf, o.n_read + (tile * 32 + 8 * q) * 4, 0);
    cin[4 * q + 0] = v[0];
    cin[4 * q + 1] = v[1];
    cin[4 * q + 2] = v[2];
    cin[4 * q + 3] = v[3];
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const uint4 a = lds_at<uint4>(buf, o.a[c] + tile * L::TILE, 0);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT>(a, xr[p][c], c == 0 ? cin : acc[p]);
  }
}

// Score j of the tile (a select chain: j differs per lane).
__device__ __forceinline__ float knn_pick(const f32x16& acc, int j) {
  float s = acc[0];
#pragma unroll
  for (int t = 1; t < 16; ++t) s = j == t ? acc[t] : s;
  return s;
}

// The top-k update of one tile: unless no lane's best score of the tile beats
// its KMAX-th best, the scores that do are marked, and while any lane has a
// mark left, each lane inserts its lowest marked score (so rows still enter
// in index order).
template <int KMAX>
__device__ __forceinline__ void knn_update(const f32x16& acc, int base, float (&v)[KMAX],
                                           int (&ix)[KMAX]) {
  // first the tile's best score (a max3 tree): once the lists have filled, no
  // lane's usually beats its KMAX-th best, and the tile costs 8 instructions
  const float t0 = __builtin_fmaxf(__builtin_fmaxf(acc[0], acc[1]), acc[2]);
  const float t1 = __builtin_fmaxf(__builtin_fmaxf(acc[3], acc[4]), acc[5]);
  const float t2 = __builtin_fmaxf(__builtin_fmaxf(acc[6], acc[7]), acc[8]);
  const float t3 = __builtin_fmaxf(__builtin_fmaxf(acc[9], acc[10]), acc[11]);
  const float t4 = __builtin_fmaxf(__builtin_fmaxf(acc[12], acc[13]), acc[14]);
  const float mx = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(t0, t1), t2),
                                   __builtin_fmaxf(__builtin_fmaxf(t3, t4), acc[15]));
  if (!__ballot(mx > v[KMAX - 1])) return;
  uint32_t mark = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) mark |= (acc[j] > v[KMAX - 1] ? 1u : 0u) << j;
  while (__ballot(mark != 0)) {
    if (mark != 0) {
      const int j = __builtin_ctz(mark);
      mark &= mark - 1;
      const float sc = knn_pick(acc, j);
      // an earlier insertion may have raised the bar
      if (sc > v[KMAX - 1]) knn_insert<KMAX>(v, ix, sc, base + 8 * (j >> 2) + (j & 3));
    }
  }
}

// One stage in `cur`: start the next stage into `nxt` (a different LDS array,
// so no read of `cur` waits for it), then per 32-row tile the MFMAs and the
// top-k update; with 32-entry lists (one wave per SIMD, nothing else to hide
// behind) the MFMAs of the next tile run beside this tile's update (two
// accumulator sets: the matrix pipe and the vector ALU overlap only within a
// wave's own instruction stream).  Store the next stage's scores, wait for
// its loads and sync.
template <int DT, int CPL, int NSUB, int KMAX, int LOADS>
__device__ __forceinline__ void knn_stage(int st, int nst, char* cur, char* nxt,
                                          const PipeOffsets<CPL, LOADS>& o,
                                          const uint4 (&xr)[NSUB][CPL], const u32x4* rows,
                                          const u32x4* tail, int nfull,
                                          const float* cinit, int tid, int h,
                                          float (&v)[NSUB][KMAX], int (&ix)[NSUB][KMAX]) {
  using L = PipeLayout<CPL>;
  const bool more = st + 1 < nst;
  float nn = 0.f;
  if (more) {
    // stages from nfull on come from the padded copy (a scalar select, no branch)
    const u32x4* src = st + 1 < nfull ? rows + (size_t)(st + 1) * (L::TCS * L::RC)
                                      : tail + (size_t)(st + 1 - nfull) * (L::TCS * L::RC);
    pipe_issue_dma<CPL, LOADS>(src, 0, tid, o, nxt);
    nn = pipe_score<CPL>(cinit, st + 1, tid);
  }
  if constexpr (KMAX > 16) {
    static_assert(NSUB == 1, "32-entry lists keep one query tile per wave");
    f32x16 acc[2][1];
    knn_mfma_tile<DT, CPL, 1, LOADS>(acc[0], xr, cur, o, 0);
#pragma unroll
    for (int tile = 0; tile < L::TILES; ++tile) {
      if (tile + 1 < L::TILES)
        knn_mfma_tile<DT, CPL, 1, LOADS>(acc[(tile + 1) & 1], xr, cur, o, tile + 1);
      knn_update<KMAX>(acc[tile & 1][0], (st * L::TILES + tile) * 32 + 4 * h, v[0], ix[0]);
    }
  } else {
    // within 256 registers the second accumulator set costs spills
    for (int tile = 0; tile < L::TILES; ++tile) {
      f32x16 acc[NSUB];
      knn_mfma_tile<DT, CPL, NSUB, LOADS>(acc, xr, cur, o, tile);
#pragma unroll
      for (int p = 0; p < NSUB; ++p)
        knn_update<KMAX>(acc[p], (st * L::TILES + tile) * 32 + 4 * h, v[p], ix[p]);
    }
  }
  if (more) lds_at<float>(nxt, o.n_store, 0) = nn;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}

// Lists of 8 or 16 fit two waves per SIMD (the update's latency then hides
// behind the other wave's MFMAs); 32 entries take the whole register file.
// NSUB 32-query tiles per wave: with two, each row fragment read from LDS
// feeds two MFMAs (with one, the four SIMDs' fragment and score reads ask
// more of the LDS than the matrix pipes take in).
template <int DT, int CPL, int NSUB, int KMAX>
__global__ __launch_bounds__(ASSIGN_THREADS, KMAX <= 16 ? 2 : 1) void knn_kernel(
    const uint4* __restrict__ Q, const uint4* __restrict__ rows, const uint4* __restrict__ tail,
    const float* __restrict__ cinit, int M, int nrows, int nfull, int Np, int per, int k,
    int32_t* __restrict__ nbr_idx, float* __restrict__ nbr_dist) {
  using L = PipeLayout<CPL>;
  constexpr int RC = L::RC;
  constexpr int LOADS = L::TCS * L::RCP / ASSIGN_THREADS;
  static_assert(LOADS >= 1 && LOADS * ASSIGN_THREADS == L::TCS * L::RCP, "stage must split evenly");
  constexpr int QPW = 32 * NSUB, QPB = 4 * QPW;  // queries per wave, per workgroup

  __shared__ __attribute__((aligned(16))) char buf0[L::STAGE];
  __shared__ __attribute__((aligned(16))) char buf1[L::STAGE];

  const int b = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, h = lane >> 5;
  Q += (size_t)b * M * RC;
  const u32x4* rows4 = reinterpret_cast<const u32x4*>(rows) + (size_t)b * nrows * RC;
  const u32x4* tail4 = reinterpret_cast<const u32x4*>(tail) + (size_t)b * ASSIGN_KPAD * RC;
  cinit += (size_t)b * Np;
  // this workgroup's share of the stages (`per` of them; all without a split)
  const int sp = blockIdx.z, st0 = sp * per, nst = min(st0 + per, Np / L::TCS);

  PipeOffsets<CPL, LOADS> o;
  pipe_offsets<CPL, LOADS>(o, tid, n, h);
  pipe_issue_dma<CPL, LOADS>(st0 < nfull ? rows4 + (size_t)st0 * (L::TCS * RC)
                                         : tail4 + (size_t)(st0 - nfull) * (L::TCS * RC),
                             0, tid, o, buf0);
  const float nn = pipe_score<CPL>(cinit, st0, tid);

  const int q0 = blockIdx.x * QPB + wave * QPW + n;  // this lane's query of tile 0
  uint4 xr[NSUB][CPL];
  float ss[NSUB];
#pragma unroll
  for (int p = 0; p < NSUB; ++p) {
    const int qt = q0 + 32 * p;
#pragma unroll
    for (int c = 0; c < CPL; ++c)
      xr[p][c] = qt < M ? Q[(size_t)qt * RC + h * CPL + c] : make_uint4(0, 0, 0, 0);
    const float a = tree_sumsq<DT, CPL>(xr[p]);
    ss[p] = a + __shfl_xor(a, 32);
  }

  float v[NSUB][KMAX];
  int ix[NSUB][KMAX];
#pragma unroll
  for (int p = 0; p < NSUB; ++p)
#pragma unroll
    for (int t = 0; t < KMAX; ++t) {
      v[p][t] = -__builtin_inff();
      ix[p][t] = 0x7fffffff;
    }

  lds_at<float>(buf0, o.n_store, 0) = nn;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  int st = st0;
  for (; st + 2 <= nst; st += 2) {  // two stages per trip: each buffer is a fixed array
    knn_stage<DT, CPL, NSUB, KMAX, LOADS>(st, nst, buf0, buf1, o, xr, rows4, tail4, nfull, cinit,
                                          tid, h, v, ix);
    knn_stage<DT, CPL, NSUB, KMAX, LOADS>(st + 1, nst, buf1, buf0, o, xr, rows4, tail4, nfull,
                                          cinit, tid, h, v, ix);
  }
  if (st < nst)
    knn_stage<DT, CPL, NSUB, KMAX, LOADS>(st, nst, buf0, buf1, o, xr, rows4, tail4, nfull, cinit,
                                          tid, h, v, ix);

#pragma unroll
  for (int p = 0; p < NSUB; ++p) {
    // merge the other half's list (rows 4..7 of each group of 8) into lane h = 0's
#pragma unroll
    for (int t = 0; t < KMAX; ++t) {
      const float so = __shfl_xor(v[p][t], 32);
      const int io = __shfl_xor(ix[p][t], 32);
      if (h == 0) knn_insert_by_index<KMAX>(v[p], ix[p], so, io);
    }
    const int qt = q0 + 32 * p;
    if (h == 0 && qt < M) {
      // with a split: the share's list (its scores as they are) beside the others
      const bool part = gridDim.z > 1;
      const size_t at = (((size_t)b * M + qt) * gridDim.z + sp) * k;
      int32_t* oi = nbr_idx + at;
      float* od = nbr_dist + at;
#pragma unroll
      for (int t = 0; t < KMAX; ++t) {
        if (t < k) {
          oi[t] = ix[p][t];
          od[t] = part ? v[p][t] : __builtin_fmaxf(__builtin_fmaf(-2.f, v[p][t], ss[p]), 0.f);
        }
      }
    }
  }
}

// The lists of a query's `splits` (at most 64) shares into one: one wave per
// query, lane l at the head of list l; k times the best head by (score, then
// lower index) is taken and its lane moves on.
template <int DT, int CPL>
__global__ __launch_bounds__(256) void knn_merge_kernel(const uint4* __restrict__ Q, int64_t MB,
                                                        int splits, int k,
                                                        const int32_t* __restrict__ pidx,
                                                        const float* __restrict__ pv,
                                                        int32_t* __restrict__ nbr_idx,
                                                        float* __restrict__ nbr_dist) {
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (q >= MB) return;
  // |q|^2 as the search sums it, half by half
  const uint4* qr = Q + q * (2 * CPL);
  const float qn = tree_sumsq_of<DT, CPL>([&](int c) { return qr[c]; }) +
                   tree_sumsq_of<DT, CPL>([&](int c) { return qr[CPL + c]; });
  const size_t base = ((size_t)q * splits + lane) * k;
  const bool has = lane < splits;
  int at = 0;
  float v = has ? pv[base] : -__builtin_inff();
  int i = has ? pidx[base] : 0x7fffffff;
  for (int t = 0; t < k; ++t) {
    float m = v;
    int im = i;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const float mo = __shfl_xor(m, d);
      const int io = __shfl_xor(im, d);
      const bool take = mo > m || (mo == m && io < im);
      m = take ? mo : m;
      im = take ? io : im;
    }
    if (lane == 0) {
      nbr_idx[q * k + t] = im;
      nbr_dist[q * k + t] = __builtin_fmaxf(__builtin_fmaf(-2.f, m, qn), 0.f);
    }
    if (has && i == im && v == m) {  // this lane's head was taken (indices are distinct)
      ++at;
      v = at < k ? pv[base + at] : -__builtin_inff();
      i = at < k ? pidx[base + at] : 0x7fffffff;
    }
  }
}

// Two query tiles per wave where the lists leave room for them (16 entries
// and D <= 128, which keeps two waves per SIMD), else one.
template <int CPL, int KMAX>
constexpr int knn_nsub() { return KMAX <= 16 && CPL <= 8 ? 2 : 1; }

template <int DT, int CPL, int KMAX>
hipError_t launch_knn_cpl(const void* Q, const KnnRows& r, int64_t B, int64_t M, int k,
                          const KnnSplit& sp, int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  using L = PipeLayout<CPL>;
  constexpr int NSUB = knn_nsub<CPL, KMAX>();
  constexpr int QPB = 4 * 32 * NSUB;
  const int nst = (int)(r.Np / L::TCS);
  const int per = (int)((nst + sp.splits - 1) / sp.splits);
  const int splits = (nst + per - 1) / per;
  const dim3 grid((unsigned)((M + QPB - 1) / QPB), (unsigned)B, (unsigned)splits);
  const bool part = splits > 1;
  knn_kernel<DT, CPL, NSUB, KMAX><<<grid, dim3(ASSIGN_THREADS), 0, s>>>(
      (const uint4*)Q, (const uint4*)r.rows, (const uint4*)r.tail, r.cinit, (int)M, (int)r.nrows,
      (int)(r.tail ? r.N / L::TCS : nst), (int)r.Np, per, k, part ? sp.idx : nbr_idx,
      part ? sp.v : nbr_dist);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !part) return e;
  knn_merge_kernel<DT, CPL><<<dim3((unsigned)((B * M + 3) / 4)), 256, 0, s>>>(
      (const uint4*)Q, B * M, splits, k, sp.idx, sp.v, nbr_idx, nbr_dist);
  return hipGetLastError();
}

template <int DT, int KMAX>
hipError_t launch_knn_k(const void* Q, const KnnRows& r, int64_t B, int64_t M, int64_t D, int k,
                        const KnnSplit& sp, int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  switch (D / 16) {
#define FKM_KNN_CASE(c) \
  case c: return launch_knn_cpl<DT, c, KMAX>(Q, r, B, M, k, sp, nbr_idx, nbr_dist, s);
    FKM_KNN_CASE(1) FKM_KNN_CASE(2) FKM_KNN_CASE(3) FKM_KNN_CASE(4)
    FKM_KNN_CASE(5) FKM_KNN_CASE(6) FKM_KNN_CASE(7) FKM_KNN_CASE(8)
    FKM_KNN_CASE(9) FKM_KNN_CASE(10) FKM_KNN_CASE(11) FKM_KNN_CASE(12)
    FKM_KNN_CASE(13) FKM_KNN_CASE(14) FKM_KNN_CASE(15) FKM_KNN_CASE(16)
#undef FKM_KNN_CASE
    default: return hipErrorInvalidValue;
  }
}

// The norms of the database rows, read in place, and the tail copy.
template <int DT>
hipError_t launch_knn_norm(const void* R, int64_t B, int64_t N, int64_t Np, int64_t D,
                           float* cinit, void* tail, hipStream_t s) {
  switch (D / 16) {
#define FKM_KNN_CASE(c)                                                                            \
  case c: {                                                                                        \
    using L = PipeLayout<c>;                                                                       \
    knn_norm_kernel<DT, c><<<dim3((unsigned)(Np / L::TCS), (unsigned)B), 256, 0, s>>>(             \
        (const uint4*)R, (int)N, (int)Np, (int)(N / L::TCS * L::TCS), cinit, (uint4*)tail);        \
    break;                                                                                         \
  }
    FKM_KNN_CASE(1) FKM_KNN_CASE(2) FKM_KNN_CASE(3) FKM_KNN_CASE(4)
    FKM_KNN_CASE(5) FKM_KNN_CASE(6) FKM_KNN_CASE(7) FKM_KNN_CASE(8)
    FKM_KNN_CASE(9) FKM_KNN_CASE(10) FKM_KNN_CASE(11) FKM_KNN_CASE(12)
    FKM_KNN_CASE(13) FKM_KNN_CASE(14) FKM_KNN_CASE(15) FKM_KNN_CASE(16)
#undef FKM_KNN_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The padded copy of database rows of Din elements in rows of D (chat), and their scores.
template <int DT>
hipError_t launch_knn_prep(const void* R, int64_t B, int64_t N, int64_t Np, int64_t Din, int64_t D,
                           void* chat, float* cinit, hipStream_t s) {
  const int64_t rows = 256 / prep_lanes((int)D);  // per workgroup
  knn_prep_kernel<DT><<<dim3((unsigned)((B * Np + rows - 1) / rows)), 256, 0, s>>>(
      (const uint16_t*)R, B, (int)N, (int)Np, (int)Din, (int)D, (uint16_t*)chat, cinit);
  return hipGetLastError();
}

// The search for one storage type over prepared rows; k <= KNN_MAX_K, rows of
// D elements, D % 16 == 0, D <= 256.
template <int DT>
hipError_t launch_knn_dt(const void* Q, const KnnRows& r, int64_t B, int64_t M, int64_t D, int k,
                         const KnnSplit& sp, int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  if (D % 16 != 0 || D > 256 || k < 1 || k > KNN_MAX_K || r.Np % ASSIGN_KPAD != 0 ||
      sp.splits < 1 || sp.splits > KNN_MAX_SPLITS)
    return hipErrorInvalidValue;
  if (k <= 8) return launch_knn_k<DT, 8>(Q, r, B, M, D, k, sp, nbr_idx, nbr_dist, s);
  if (k <= 10) return launch_knn_k<DT, 10>(Q, r, B, M, D, k, sp, nbr_idx, nbr_dist, s);
  if (k <= 16) return launch_knn_k<DT, 16>(Q, r, B, M, D, k, sp, nbr_idx, nbr_dist, s);
  return launch_knn_k<DT, KNN_MAX_K>(Q, r, B, M, D, k, sp, nbr_idx, nbr_dist, s);
}

}  // namespace fkm
