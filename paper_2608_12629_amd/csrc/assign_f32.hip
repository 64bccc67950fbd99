// assign_f32.hip -- the fp32 assignment (D = 32 .. 256) on the bf16 matrix cores.
//
// Every fp32 value is the sum of three bf16 pieces, v = h + m + l, each the
// rounding of what the ones before leave: |m| <= 2^-9 |v|, |l| <= 2^-18 |v|,
// and what l leaves is below 2^-27 |v|.  <x, c> is the six products
// hh + hm + mh + mm + hl + lh, accumulated in fp32; the three left out (ml,
// lm, ll) are below 2^-26 |x_d c_d| each, a quarter of the rounding of one
// fp32 product.  A bf16 32x32x16 product takes 1/16 of the matrix time of the
// same fp32 one, so six take 3/8 of it.
//
// What bounds it: the matrix cores (the six products at the bf16 rate).
// Layout: the workgroup's points stay in registers as pieces (3 D / 16 16-byte
// fragments a lane and 32-point tile), the centroids stream through LDS in
// stages of TCS rows, double-buffered, L2 to LDS directly.  prep3_kernel writes
// each stage as the image that LDS holds (rows of 6 D bytes at an odd stride
// of 16-byte chunks, so the 16-byte reads of 32 rows meet no bank twice; then
// the scores), so a stage is a linear copy and a lane keeps one offset.  The
// MFMAs of a tile and the arg-max of the tile before share a basic block on
// two accumulator sets, as in assign_pipe.h, whose tile layout this has.
#include "assign_pipe.h"

namespace fkm {

namespace {

template <int CP>
struct X3Layout {
  static constexpr int D = 16 * CP, RC = 6 * CP, RCP = RC + 1;
  static constexpr int TCS = (int)X3_TCS(D), TILES = TCS / 32;
  static constexpr int CHUNKS = TCS * RCP * 16;  // bytes of rows; the scores follow
  static constexpr int NW = (int)x3_stage_bytes(D) / 1024;
  static constexpr int STAGE = NW * 1024;
  static constexpr int TILE = 32 * RCP * 16;
  static_assert(CHUNKS + TCS * 4 <= STAGE, "a stage holds its rows and scores");
};

// Two point tiles of six chunks leave no registers for a second accumulator
// set (it spilled 648 bytes): there a tile's arg-max follows its own MFMAs and
// the other wave of the SIMD fills in.  500,000 x 96, K = 1,024, before the
// products were reordered: 388 us; one point tile a wave with two sets: 431.
constexpr bool x3_piped(int cp, int nsub) { return cp * nsub <= 10 || nsub == 1; }

// Centroid rows (Dc elements, zeros up to D) into the stage images, one wave a row.
__global__ __launch_bounds__(256) void prep3_kernel(const float* __restrict__ C, int64_t rows, int K,
                                                    int Dc, X3Images im) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int64_t b = row / im.Kst;
  const int k = (int)(row % im.Kst);
  prep3_row(C + (b * K + (k < K ? k : 0)) * Dc, k >= K, Dc, im, b, k, lane);
}

// Start a stage image on its way into `buf`: the waves take its 1 KiB pieces in turn.
template <int CP>
__device__ __forceinline__ void x3_issue(const char* img, int st, int wave, int lane, char* buf) {
  using L = X3Layout<CP>;
  const char* src = img + (size_t)st * L::STAGE + lane * 16;
#pragma unroll
  for (int u = 0; u < (L::NW + 3) / 4; ++u) {
    const int i = u * 4 + wave;
    if (u * 4 + 3 < L::NW || i < L::NW) lds_dma16(src + i * 1024, buf + i * 1024);
  }
}

// <x, c> of one tile, the small products of all dimensions first: each add
// of the matrix cores rounds relative to the running sum, which hh then joins
// in D / 16 steps, and the score is added last, by the vector ALU.  With the
// score first and all products in one loop the kernel is 8% faster at D = 96,
// but min_dist was 2e-8 too large on average at D = 256 (4e-9 either way with
// the fp32 instructions) and its rms error 2.4e-7 (1.4e-7 now).
template <int TILE, int CP, int NSUB>
__device__ __forceinline__ void x3_mfma_tile(f32x16 (&acc)[NSUB], f32x16& cin,
                                             const uint4 (&xh)[NSUB][CP], const uint4 (&xm)[NSUB][CP],
                                             const uint4 (&xl)[NSUB][CP], char* buf, int off, int noff) {
  using L = X3Layout<CP>;
#pragma unroll
  for (int p = 0; p < NSUB; ++p)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[p][j] = 0.f;
#pragma unroll
  for (int c = 0; c < CP; ++c) {
    const uint4 ah = lds_at<uint4>(buf, off, TILE * L::TILE + c * 16);
    const uint4 am = lds_at<uint4>(buf, off, TILE * L::TILE + (2 * CP + c) * 16);
    const uint4 al = lds_at<uint4>(buf, off, TILE * L::TILE + (4 * CP + c) * 16);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT_BF16>(al, xh[p][c], acc[p]);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT_BF16>(am, xm[p][c], acc[p]);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT_BF16>(ah, xl[p][c], acc[p]);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT_BF16>(am, xh[p][c], acc[p]);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT_BF16>(ah, xm[p][c], acc[p]);
  }
  // a second offset hides that these are the fragments read above: keeping
  // them would take 4 CP registers
  int off2 = off;
  asm volatile("" : "+v"(off2));
#pragma unroll
  for (int c = 0; c < CP; ++c) {
    const uint4 ah = lds_at<uint4>(buf, off2, TILE * L::TILE + c * 16);
#pragma unroll
    for (int p = 0; p < NSUB; ++p) acc[p] = mfma32_chunk<DT_BF16>(ah, xh[p][c], acc[p]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = lds_at<f32x4>(buf, noff, L::CHUNKS + (TILE * 32 + 8 * q) * 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) cin[4 * q + r] = v[r];
  }
}

// Exact arg-max of a tile's scores: rows ascend with j, and a strict compare
// keeps the lowest of equal ones (a NaN score never wins).
template <int NSUB>
__device__ __forceinline__ void x3_epilogue(const f32x16 (&acc)[NSUB], const f32x16& cin, int tcode,
                                            float (&best)[NSUB], int (&code)[NSUB]) {
#pragma unroll
  for (int j = 0; j < 16; ++j)
#pragma unroll
    for (int p = 0; p < NSUB; ++p) {
      const float v = acc[p][j] + cin[j];
      const bool gt = v > best[p];
      best[p] = gt ? v : best[p];
      code[p] = gt ? tcode + j : code[p];
    }
}

template <int CP, int NSUB>
__device__ __forceinline__ void x3_stage(int st, int nst, const char* img, int wave, int lane,
                                         f32x16 (&accA)[NSUB], f32x16 (&accB)[NSUB],
                                         f32x16& cinA, f32x16& cinB, const uint4 (&xh)[NSUB][CP], const uint4 (&xm)[NSUB][CP],
                                         const uint4 (&xl)[NSUB][CP], char* cur, char* nxt, int off,
                                         int noff, float (&best)[NSUB], int (&code)[NSUB]) {
  using L = X3Layout<CP>;
  x3_issue<CP>(img, min(st + 1, nst - 1), wave, lane, nxt);
  __builtin_amdgcn_sched_barrier(0);
  const int tb = L::TILES * st;  // accA holds tile tb - 1
  if constexpr (!x3_piped(CP, NSUB)) {
    x3_mfma_tile<0, CP, NSUB>(accA, cinA, xh, xm, xl, cur, off, noff);
    x3_epilogue<NSUB>(accA, cinA, tb * 16, best, code);
    x3_mfma_tile<1, CP, NSUB>(accA, cinA, xh, xm, xl, cur, off, noff);
    x3_epilogue<NSUB>(accA, cinA, (tb + 1) * 16, best, code);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    return;
  }
  if constexpr (L::TILES == 2) {
    x3_mfma_tile<0, CP, NSUB>(accB, cinB, xh, xm, xl, cur, off, noff);
    x3_epilogue<NSUB>(accA, cinA, (tb - 1) * 16, best, code);
    x3_mfma_tile<1, CP, NSUB>(accA, cinA, xh, xm, xl, cur, off, noff);
    x3_epilogue<NSUB>(accB, cinB, tb * 16, best, code);
  } else {
    x3_mfma_tile<0, CP, NSUB>(accB, cinB, xh, xm, xl, cur, off, noff);
    x3_epilogue<NSUB>(accA, cinA, (tb - 1) * 16, best, code);
  }
  // a few LDS reads ahead, then two reads to 3 NSUB MFMAs with vector work between
  __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
  for (int i = 0; i < L::TILES * CP * 2; ++i) {
#pragma unroll
    for (int k = 0; k < 3 * NSUB; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
      if (k == 0 || k == 2) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}

// X [B,N,D] fp32; img [B, nst] stage images.
template <int CP, int NSUB>
__global__ __launch_bounds__(ASSIGN_THREADS, 2) void assign_x3_kernel(
    const float* __restrict__ X, const char* __restrict__ img, int N, int nst,
    int32_t* __restrict__ idx, float* __restrict__ min_dist, double* __restrict__ objpart) {
  using L = X3Layout<CP>;
  constexpr int D = L::D;
  __shared__ __attribute__((aligned(16))) char buf0[L::STAGE];
  __shared__ __attribute__((aligned(16))) char buf1[L::STAGE];
  const int b = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  img += (size_t)b * nst * L::STAGE;
  x3_issue<CP>(img, 0, wave, lane, buf0);

  const int pbase = (blockIdx.x * 4 + wave) * 32 * NSUB;
  uint4 xh[NSUB][CP], xm[NSUB][CP], xl[NSUB][CP];
  float xn[NSUB];
#pragma unroll
  for (int p = 0; p < NSUB; ++p) {
    const int pt = min(pbase + p * 32 + n, N - 1);  // points past N repeat the last one
    const uint4* row = reinterpret_cast<const uint4*>(X + ((size_t)b * N + pt) * D + h * (D / 2));
    uint4 q[2 * CP];
#pragma unroll
    for (int c = 0; c < 2 * CP; ++c) q[c] = row[c];
    xn[p] = tree_sumsq<DT_F32, 2 * CP>(q);
    xn[p] += __shfl_xor(xn[p], 32);
#pragma unroll
    for (int c = 0; c < CP; ++c) {
      const float v[8] = {__uint_as_float(q[2 * c].x),     __uint_as_float(q[2 * c].y),
                          __uint_as_float(q[2 * c].z),     __uint_as_float(q[2 * c].w),
                          __uint_as_float(q[2 * c + 1].x), __uint_as_float(q[2 * c + 1].y),
                          __uint_as_float(q[2 * c + 1].z), __uint_as_float(q[2 * c + 1].w)};
      bf16x8 ph, pm, pl;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        __bf16 eh, em, el;
        split3(v[e], eh, em, el);
        ph[e] = eh;
        pm[e] = em;
        pl[e] = el;
      }
      xh[p][c] = __builtin_bit_cast(uint4, ph);
      xm[p][c] = __builtin_bit_cast(uint4, pm);
      xl[p][c] = __builtin_bit_cast(uint4, pl);
    }
    __builtin_amdgcn_sched_barrier(0);  // one tile's fp32 rows in registers at a time
  }
  float best[NSUB];
  int code[NSUB];
  f32x16 accA[NSUB], accB[NSUB], cinA, cinB;
#pragma unroll
  for (int j = 0; j < 16; ++j) cinA[j] = cinB[j] = 0.f;
#pragma unroll
  for (int p = 0; p < NSUB; ++p) {
    best[p] = -__builtin_inff();
    code[p] = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) accA[p][j] = -__builtin_inff();  // no tile before the first
  }
  const int off = (n * L::RCP + h * CP) * 16, noff = 16 * h;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  int st = 0;
  if constexpr (L::TILES == 2) {
    for (; st + 2 <= nst; st += 2) {  // two stages per trip: each buffer is a fixed array
      x3_stage<CP, NSUB>(st, nst, img, wave, lane, accA, accB, cinA, cinB, xh, xm, xl, buf0, buf1, off, noff, best, code);
      x3_stage<CP, NSUB>(st + 1, nst, img, wave, lane, accA, accB, cinA, cinB, xh, xm, xl, buf1, buf0, off, noff, best, code);
    }
    if (st < nst)
      x3_stage<CP, NSUB>(st, nst, img, wave, lane, accA, accB, cinA, cinB, xh, xm, xl, buf0, buf1, off, noff, best, code);
    if constexpr (x3_piped(CP, NSUB)) x3_epilogue<NSUB>(accA, cinA, (L::TILES * nst - 1) * 16, best, code);
  } else {
    // one tile a stage: the accumulator sets alternate with the buffers
    for (; st + 2 <= nst; st += 2) {
      x3_stage<CP, NSUB>(st, nst, img, wave, lane, accA, accB, cinA, cinB, xh, xm, xl, buf0, buf1, off, noff, best, code);
      x3_stage<CP, NSUB>(st + 1, nst, img, wave, lane, accB, accA, cinB, cinA, xh, xm, xl, buf1, buf0, off, noff, best, code);
    }
    if (st < nst) {
      x3_stage<CP, NSUB>(st, nst, img, wave, lane, accA, accB, cinA, cinB, xh, xm, xl, buf0, buf1, off, noff, best, code);
      x3_epilogue<NSUB>(accB, cinB, (nst - 1) * 16, best, code);
    } else {
      x3_epilogue<NSUB>(accA, cinA, (nst - 1) * 16, best, code);
    }
  }

  double obj = 0.0;
#pragma unroll
  for (int p = 0; p < NSUB; ++p) {
    float v = best[p];
    const int j = code[p] & 15;
    int i = (code[p] >> 4) * 32 + 8 * (j >> 2) + 4 * h + (j & 3);
    const float vo = __shfl_xor(v, 32);
    const int io = __shfl_xor(i, 32);
    const bool take = (vo > v) || (vo == v && io < i);
    v = take ? vo : v;
    i = take ? io : i;
    const int pt = pbase + p * 32 + n;
    if (h == 0 && pt < N) {
      // unassigned: a norm that is not finite, or no real centroid's score finite
      const bool asg = xn[p] <= __FLT_MAX__ && v > -__FLT_MAX__;
      const float md = __builtin_fmaxf(__builtin_fmaf(-2.f, v, xn[p]), 0.f);
      idx[(size_t)b * N + pt] = asg ? i : -1;
      min_dist[(size_t)b * N + pt] = asg ? md : __builtin_nanf("");
      obj += asg ? (double)md : 0.0;
    }
  }
#pragma unroll
  for (int msk = 1; msk < 64; msk <<= 1) obj += __shfl_xor(obj, msk);
  double* lds_obj = reinterpret_cast<double*>(buf0);  // free since the last stage's barrier
  if (lane == 0) lds_obj[wave] = obj;
  __syncthreads();
  if (tid == 0)
    objpart[(size_t)b * gridDim.x + blockIdx.x] = ((lds_obj[0] + lds_obj[1]) + lds_obj[2]) + lds_obj[3];
}

template <int CP>
hipError_t launch_x3(const float* X, const Workspace& w, int64_t B, int64_t N, int64_t K,
                     int32_t* idx, float* min_dist, hipStream_t s) {
  const dim3 grid((unsigned)w.n_assign_blocks, (unsigned)B), block(ASSIGN_THREADS);
  const int nst = (int)((K + X3Layout<CP>::TCS - 1) / X3Layout<CP>::TCS);
  if (x3_nsub(16 * CP, B * N) == 1) {
    assign_x3_kernel<CP, 1><<<grid, block, 0, s>>>(X, w.img.p, (int)N, nst, idx, min_dist, w.objpart);
  } else if constexpr (CP <= X3_WIDE_CP) {
    assign_x3_kernel<CP, 2><<<grid, block, 0, s>>>(X, w.img.p, (int)N, nst, idx, min_dist, w.objpart);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prep3(const float* C, const Workspace& w, int64_t B, int64_t K, int64_t Dc,
                        hipStream_t s) {
  const int64_t rows = B * w.img.Kst;
  prep3_kernel<<<dim3((unsigned)((rows + 3) / 4)), 256, 0, s>>>(C, rows, (int)K, (int)Dc, w.img);
  return hipGetLastError();
}

hipError_t launch_assign_f32(const float* X, const Workspace& w, int64_t B, int64_t N, int64_t D,
                             int64_t K, int32_t* idx, float* min_dist, hipStream_t s) {
  if (D % 16 != 0 || D < 32 || D > 256 || !w.x3) return hipErrorInvalidValue;
  switch (D / 16) {
    case 2: return launch_x3<2>(X, w, B, N, K, idx, min_dist, s);
    case 3: return launch_x3<3>(X, w, B, N, K, idx, min_dist, s);
    case 4: return launch_x3<4>(X, w, B, N, K, idx, min_dist, s);
    case 5: return launch_x3<5>(X, w, B, N, K, idx, min_dist, s);
    case 6: return launch_x3<6>(X, w, B, N, K, idx, min_dist, s);
    case 7: return launch_x3<7>(X, w, B, N, K, idx, min_dist, s);
    case 8: return launch_x3<8>(X, w, B, N, K, idx, min_dist, s);
    case 9: return launch_x3<9>(X, w, B, N, K, idx, min_dist, s);
    case 10: return launch_x3<10>(X, w, B, N, K, idx, min_dist, s);
    case 11: return launch_x3<11>(X, w, B, N, K, idx, min_dist, s);
    case 12: return launch_x3<12>(X, w, B, N, K, idx, min_dist, s);
    case 13: return launch_x3<13>(X, w, B, N, K, idx, min_dist, s);
    case 14: return launch_x3<14>(X, w, B, N, K, idx, min_dist, s);
    case 15: return launch_x3<15>(X, w, B, N, K, idx, min_dist, s);
    case 16: return launch_x3<16>(X, w, B, N, K, idx, min_dist, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fkm
