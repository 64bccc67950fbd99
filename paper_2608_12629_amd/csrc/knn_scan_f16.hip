// knn_scan_f16.hip -- KNN search for few queries, f16 rows.
#include "knn_scan.h"

namespace fkm {

hipError_t launch_knn_scan_f16(const void* Q, const void* R, int64_t B, int64_t M, int64_t N,
                               int64_t nrows, int64_t D, int k, const KnnScanPlan& p, float* gmax,
                               int32_t* nbr_idx, float* nbr_dist, hipStream_t s) {
  return launch_knn_scan_dt<DT_F16>(Q, R, B, M, N, nrows, D, k, p, gmax, nbr_idx, nbr_dist, s);
}

}  // namespace fkm
