// knn_bf16.hip -- KNN search for bf16 rows: the list kernel and its preparation.
#include "knn.h"

namespace fkm {

hipError_t launch_knn_norm_bf16(const void* R, int64_t B, int64_t N, int64_t Np, int64_t D,
                               float* cinit, void* tail, hipStream_t s) {
  return launch_knn_norm<DT_BF16>(R, B, N, Np, D, cinit, tail, s);
}

hipError_t launch_knn_prep_bf16(const void* R, int64_t B, int64_t N, int64_t Np, int64_t Din,
                               int64_t D, void* chat, float* cinit, hipStream_t s) {
  return launch_knn_prep<DT_BF16>(R, B, N, Np, Din, D, chat, cinit, s);
}

hipError_t launch_knn_bf16(const void* Q, const KnnRows& r, int64_t B, int64_t M, int64_t D, int k,
                          const KnnSplit& sp, int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  return launch_knn_dt<DT_BF16>(Q, r, B, M, D, k, sp, nbr_idx, nbr_dist, s);
}

}  // namespace fkm
