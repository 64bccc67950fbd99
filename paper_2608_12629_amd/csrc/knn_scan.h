// knn_scan.h -- KNN search for few queries (bf16/fp16 rows, D a multiple of 16
// up to 256): one streaming pass over the database that keeps only the best
// score of every group of rows, then an exact search of the k best groups of
// each query.  Instantiated once per storage type in knn_scan_bf16.hip and
// knn_scan_f16.hip; knn.h holds the list kernel for many queries.
//
// Why.  With few queries the search is bound by reading the database once, and
// the list kernel's workgroups (128 or 256 queries each) are too few to fill
// the chip: 100 queries were one workgroup on one of 256 CUs.  Here the rows
// are split over the chip instead, and since lists that start empty in every
// split would spend longer filling than the rows take to arrive, the pass
// keeps no lists.
//
// Pass 1 (knn_scan_kernel).  A group is 2^gs consecutive 32-row tiles.  The k
// groups with the largest best score (ties to the lower group) hold the k
// best rows: a row of any other group is beaten by the best row of each of
// them, by score or, at equal scores, by its lower index (groups are ranges of
// the row index in order).  Rows stream through LDS straight from the caller's
// array in the assignment kernel's stages (rows past N - 1 repeat row N - 1);
// each wave sums the squares of one tile's rows from LDS, so no pass over the
// database prepares norms.
//
// Pass 2 (knn_pick_kernel).  One workgroup per query picks the k groups and
// scores their rows again with the same instructions in the same order (the
// same bits as in pass 1); rows that reach the k-th group's best score are
// ranked by (score, then lower index).
//
// Measured (100 queries, 1,000,003 rows, D = 128 bf16, k = 10): the list kernel
// 15,730 us + 268 us of preparation; here 51 us (5.0 TB/s) + 16 us for pass 2.
#pragma once

#include "assign_pipe.h"

namespace fkm {

constexpr int KNN_PICK_THREADS = 512;
constexpr int KNN_PICK_CAND = 2048;  // candidate rows held at a time

// -|r|^2/2 of row n of a tile from the two lanes' fragments (lane h holds the
// row's half h).
template <int DT, int CPL>
__device__ __forceinline__ float knn_half_norm(const uint4 (&a)[CPL]) {
  const float ss = tree_sumsq<DT, CPL>(a);
  return -0.5f * (ss + __shfl_xor(ss, 32));
}

// A barrier that waits for the wave's LDS accesses only: the next stage's
// loads stay in flight across it.
__device__ __forceinline__ void knn_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // vmcnt and expcnt at their maxima, lgkmcnt 0
  asm volatile("s_barrier" ::: "memory");
}

// Grid (splits of the rows, blocks of 128 queries, instances); `per` stages of
// TCS rows per workgroup (a whole number of groups, at most KNN_SCAN_GL).
template <int DT, int CPL>
__global__ __launch_bounds__(ASSIGN_THREADS, 2) void knn_scan_kernel(
    const uint4* __restrict__ Q, const uint4* __restrict__ R, int M, int N, int nrows, int per,
    int gs, int ngroups, float* __restrict__ gmax) {
  using L = PipeLayout<CPL>;
  constexpr int RC = L::RC, TILES = L::TILES;
  constexpr int LOADS = L::TCS * L::RCP / ASSIGN_THREADS;
  __shared__ __attribute__((aligned(16))) char buf0[L::CHUNKS];
  __shared__ __attribute__((aligned(16))) char buf1[L::CHUNKS];
  __shared__ __attribute__((aligned(16))) float lds_n[L::TCS];
  __shared__ float gm[128][KNN_SCAN_GL + 1];
  const int b = blockIdx.z, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, h = lane >> 5;
  Q += (size_t)b * M * RC;
  R += (size_t)b * nrows * RC;
  const int nst = (N + L::TCS - 1) / L::TCS;
  const int st0 = blockIdx.x * per, st1 = min(st0 + per, nst);

  PipeOffsets<CPL, LOADS> o;
  pipe_offsets<CPL, LOADS>(o, tid, n, h);
  pipe_issue_rows<CPL, LOADS>(R, st0 * L::TCS, N, tid, buf0);
  const int q0 = blockIdx.y * 128 + wave * 32;
  const bool live = q0 < M;  // the wave has queries (uniform)
  uint4 xr[1][CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c)
    xr[0][c] = q0 + n < M ? Q[(size_t)(q0 + n) * RC + h * CPL + c] : make_uint4(0, 0, 0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  float run = -__builtin_inff();  // best score of the open group, this lane's rows
  auto stage = [&](int st, char* cur, char* nxt) {
    if (st + 1 < st1) pipe_issue_rows<CPL, LOADS>(R, (st + 1) * L::TCS, N, tid, nxt);
    if (wave < TILES) {  // each wave the norms of one tile
      uint4 a[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) a[c] = lds_at<uint4>(cur, o.a[c] + wave * L::TILE, 0);
      const float nn = knn_half_norm<DT, CPL>(a);
      const int row = st * L::TCS + wave * 32 + n;
      if (h == 0) lds_n[wave * 32 + n] = row < N ? nn : -0x1.fffffep127f;
    }
    knn_lds_sync();
    if (live) {
#pragma unroll
      for (int tile = 0; tile < TILES; ++tile) {
        f32x16 acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(&lds_n[tile * 32 + 8 * q + 4 * h]);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[4 * q + r] = v[r];
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c)
          acc = mfma32_chunk<DT>(lds_at<uint4>(cur, o.a[c] + tile * L::TILE, 0), xr[0][c], acc);
#pragma unroll
        for (int j = 0; j < 16; j += 2) run = __builtin_fmaxf(__builtin_fmaxf(acc[j], acc[j + 1]), run);
        const int t = (st - st0) * TILES + tile + 1;  // tiles done
        if ((t & ((1 << gs) - 1)) == 0 || (st + 1 == st1 && tile + 1 == TILES)) {  // the group ends
          const float other = __shfl_xor(run, 32);
          if (h == 0) gm[wave * 32 + n][(t - 1) >> gs] = __builtin_fmaxf(run, other);
          run = -__builtin_inff();
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };
  int st = st0;
  for (; st + 2 <= st1; st += 2) {  // two stages per trip: each buffer is a fixed array
    stage(st, buf0, buf1);
    stage(st + 1, buf1, buf0);
  }
  if (st < st1) stage(st, buf0, buf1);

  // the workgroup's groups, query by query
  const int g0 = (st0 * TILES) >> gs, ng = min(g0 + ((per * TILES) >> gs), ngroups) - g0;
  const int nq = min(128, M - (int)blockIdx.y * 128);
  for (int i = tid; i < nq * ng; i += ASSIGN_THREADS) {
    const int q = i / ng, g = i - q * ng;
    gmax[((size_t)b * M + blockIdx.y * 128 + q) * ngroups + g0 + g] = gm[q][g];
  }
}

// A (score, index) pair as one key: the larger key has the larger score, or at
// equal scores the lower index.
__device__ __forceinline__ uint64_t knn_key(float v, int i) {
  const uint32_t u = __float_as_uint(v);
  const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)o << 32) | (uint32_t)~i;
}
__device__ __forceinline__ float knn_key_score(uint64_t key) {
  const uint32_t o = (uint32_t)(key >> 32);
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
__device__ __forceinline__ int knn_key_index(uint64_t key) { return (int)~(uint32_t)key; }

// One workgroup per query (grid M x B).  Bound by latency: a chain of a few
// dozen microsecond-sized steps, so each is spread over the workgroup: the k
// best are found by counting, for every candidate, the better ones (taking
// them one after the other was 8 us of 29), and the rows come through LDS as
// whole rows, a tile ahead (a lane's own 16-byte pieces of 32 rows took 13 us).
template <int DT, int CPL>
__global__ __launch_bounds__(KNN_PICK_THREADS) void knn_pick_kernel(
    const uint4* __restrict__ Q, const uint4* __restrict__ R, int M, int N, int nrows, int gs,
    int ngroups, int k, const float* __restrict__ gmax, int32_t* __restrict__ nbr_idx,
    float* __restrict__ nbr_dist) {
  using L = PipeLayout<CPL>;
  constexpr int RC = L::RC;
  constexpr int T = KNN_PICK_THREADS, W = T / 64;
  constexpr int BL = 128;                  // groups i with the same i % BL form a block
  constexpr int VPT = KNN_MAX_GROUPS / T;  // groups per thread
  constexpr int NB = CPL <= 8 ? 2 : 1;     // tile buffers per wave
  constexpr int LW = 32 * L::RCP / 64;     // loads per lane for a tile
  static_assert(T % BL == 0 && BL >= KNN_MAX_K && BL <= KNN_PICK_CAND &&
                KNN_MAX_K * (KNN_MAX_GROUPS / BL) <= KNN_PICK_CAND, "candidate room");
  __shared__ __attribute__((aligned(16))) char tiles[W * NB * L::TILE];
  __shared__ uint64_t cand[KNN_PICK_CAND];
  __shared__ uint64_t best[T];
  __shared__ uint64_t kept[KNN_MAX_K];
  __shared__ int sel[KNN_MAX_K];
  __shared__ int cnt;
  const int q = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const float ninf = -__builtin_inff();
  const float* gq = gmax + ((size_t)b * M + q) * ngroups;
  R += (size_t)b * nrows * RC;

  // the query in every column, and its squared norm
  const uint4* qrow = Q + ((size_t)b * M + q) * RC + h * CPL;
  uint4 x[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) x[c] = qrow[c];
  float qn = tree_sumsq<DT, CPL>(x);
  qn += __shfl_xor(qn, 32);

  // the best `keep` of the first c candidates, in order, into kept (all threads)
  auto rank = [&](int c, int keep) {
    for (int i = tid; i < c; i += T) {
      const uint64_t key = cand[i];
      int r = 0;
#pragma unroll 8
      for (int j = 0; j < c; ++j) r += cand[j] > key ? 1 : 0;
      if (r < keep) kept[r] = key;
    }
    __syncthreads();
  };

  // The k best groups.  They lie in the k blocks whose best group is best (any
  // other block's groups are beaten by those k), and reach the last of these:
  // rank the BL blocks, then the few groups that are left.
  float v[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) v[u] = tid + T * u < ngroups ? gq[tid + T * u] : ninf;
  uint64_t bk = tid < ngroups ? knn_key(v[0], tid) : 0;
#pragma unroll
  for (int u = 1; u < VPT; ++u) {
    const uint64_t key = tid + T * u < ngroups ? knn_key(v[u], tid + T * u) : 0;
    bk = key > bk ? key : bk;
  }
  best[tid] = bk;
  if (tid == 0) cnt = 0;
  __syncthreads();
  if (tid < BL) {
#pragma unroll
    for (int u = 1; u < T / BL; ++u) bk = best[tid + BL * u] > bk ? best[tid + BL * u] : bk;
    cand[tid] = bk;
  }
  __syncthreads();
  const int nsel = min(k, ngroups);
  const int nblk = min(nsel, BL);
  rank(BL, nblk);
  const uint64_t bthr = kept[nblk - 1];
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int g = tid + T * u;
    // at most nblk * (KNN_MAX_GROUPS / BL) groups reach the key: distinct keys,
    // and none outside the nblk blocks does
    if (g < ngroups && knn_key(v[u], g) >= bthr) cand[atomicAdd(&cnt, 1)] = knn_key(v[u], g);
  }
  __syncthreads();
  const int have = cnt;
  rank(have, nsel);
  // with fewer groups than k every row is a candidate
  float thr = nsel == k ? knn_key_score(kept[k - 1]) : ninf;
  if (tid < nsel) sel[tid] = knn_key_index(kept[tid]);
  if (tid == 0) cnt = 0;
  __syncthreads();

  // Their rows, one 32-row tile per wave at a time through the wave's own part
  // of LDS (the assignment's swizzled rows; rows past N - 1 repeat row N - 1).
  const int ntile = nsel << gs;
  auto tile_row = [&](int t) { return ((sel[t >> gs] << gs) + (t & ((1 << gs) - 1))) * 32; };
  auto fetch = [&](int t, char* buf) {
    const int row0 = tile_row(t);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // this wave's reads of the buffer are done (lgkmcnt 0)
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      const int sl = lane + u * 64;
      const int r = sl / L::RCP, c = (sl % L::RCP) ^ (r & L::SWZ);
      lds_dma16(R + (size_t)min(row0 + r, N - 1) * RC + (c < RC ? c : 0), buf + u * 1024);
    }
  };
  auto score = [&](int t, char* buf) {
    const int row0 = tile_row(t);
    uint4 a[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c)
      a[c] = lds_at<uint4>(buf, (n * L::RCP + ((h * CPL + c) ^ (n & L::SWZ))) * 16, 0);
    const float nn = knn_half_norm<DT, CPL>(a);  // of row row0 + n
    f32x16 acc;
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = __shfl(nn, 8 * (j >> 2) + 4 * h + (j & 3));
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc = mfma32_chunk<DT>(a[c], x[c], acc);
    // every column holds the same scores: lane n < 16 of each half takes row j = n
    float s = acc[0];
#pragma unroll
    for (int j = 1; j < 16; ++j) s = n == j ? acc[j] : s;
    const int row = row0 + 8 * (n >> 2) + 4 * h + (n & 3);
    if (n < 16 && row < N && s >= thr) cand[atomicAdd(&cnt, 1)] = knn_key(s, row);
  };
  char* mine = tiles + wave * NB * L::TILE;
  const bool fits = ntile * 32 <= KNN_PICK_CAND;  // every row of every tile could be kept
  if (wave < ntile) fetch(wave, mine);
  for (int t0 = 0, i = 0; t0 < ntile; t0 += W, ++i) {
    const int t = t0 + wave;
    char* cur = mine + (NB == 2 ? (i & 1) * L::TILE : 0);
    if (t < ntile) {
      if (NB == 2 && t + W < ntile) {
        fetch(t + W, mine + (~i & 1) * L::TILE);
        __builtin_amdgcn_s_waitcnt((LW & 15) | ((LW >> 4) << 14) | 0x0F70);  // vmcnt(LW): tile t is here
      } else {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      }
      asm volatile("" ::: "memory");
      score(t, cur);
      if (NB == 1 && t + W < ntile) fetch(t + W, mine);
    }
    if (fits) continue;
    __syncthreads();
    const int c = cnt;
    if (t0 + W < ntile && c > KNN_PICK_CAND - 32 * W) {  // room for the next tiles: keep the best k
      rank(c, k);
      if (tid < k) cand[tid] = kept[tid];
      if (tid == 0) cnt = k;
      thr = knn_key_score(kept[k - 1]);
    }
    __syncthreads();
  }
  __syncthreads();
  rank(cnt, k);
  if (tid < k) {
    const size_t o = ((size_t)b * M + q) * k + tid;
    nbr_idx[o] = knn_key_index(kept[tid]);
    nbr_dist[o] = __builtin_fmaxf(__builtin_fmaf(-2.f, knn_key_score(kept[tid]), qn), 0.f);
  }
}

template <int DT, int CPL>
hipError_t launch_knn_scan_cpl(const void* Q, const void* R, int64_t B, int64_t M, int64_t N,
                               int64_t nrows, int k, const KnnScanPlan& p, float* gmax,
                               int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  using L = PipeLayout<CPL>;
  if (p.tcs != L::TCS || ((p.per * L::TILES) & ((1 << p.gs) - 1)) != 0 ||
      (p.per * L::TILES) >> p.gs > KNN_SCAN_GL || p.ngroups > KNN_MAX_GROUPS)
    return hipErrorInvalidValue;
  knn_scan_kernel<DT, CPL><<<dim3((unsigned)p.splits, (unsigned)((M + 127) / 128), (unsigned)B),
                             ASSIGN_THREADS, 0, s>>>((const uint4*)Q, (const uint4*)R, (int)M,
                                                     (int)N, (int)nrows, (int)p.per, p.gs,
                                                     (int)p.ngroups, gmax);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  knn_pick_kernel<DT, CPL><<<dim3((unsigned)M, (unsigned)B), KNN_PICK_THREADS, 0, s>>>(
      (const uint4*)Q, (const uint4*)R, (int)M, (int)N, (int)nrows, p.gs, (int)p.ngroups, k,
      gmax, nbr_idx, nbr_dist);
  return hipGetLastError();
}

// Q and R: rows of D elements, D % 16 == 0, D <= 256; R has nrows >= N rows per instance.
template <int DT>
hipError_t launch_knn_scan_dt(const void* Q, const void* R, int64_t B, int64_t M, int64_t N,
                              int64_t nrows, int64_t D, int k, const KnnScanPlan& p, float* gmax,
                              int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  if (D % 16 != 0 || k < 1 || k > KNN_MAX_K || k > N) return hipErrorInvalidValue;
  switch (D / 16) {
#define FKM_KNN_CASE(c)                                                                         \
  case c:                                                                                       \
    return launch_knn_scan_cpl<DT, c>(Q, R, B, M, N, nrows, k, p, gmax, nbr_idx, nbr_dist, s);
    FKM_KNN_CASE(1) FKM_KNN_CASE(2) FKM_KNN_CASE(3) FKM_KNN_CASE(4)
    FKM_KNN_CASE(5) FKM_KNN_CASE(6) FKM_KNN_CASE(7) FKM_KNN_CASE(8)
    FKM_KNN_CASE(9) FKM_KNN_CASE(10) FKM_KNN_CASE(11) FKM_KNN_CASE(12)
    FKM_KNN_CASE(13) FKM_KNN_CASE(14) FKM_KNN_CASE(15) FKM_KNN_CASE(16)
#undef FKM_KNN_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fkm
