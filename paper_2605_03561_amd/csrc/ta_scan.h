// ta_scan.h -- declarations shared by the exact outlier scan's kernel files.
#pragma once

#include "ta_internal.h"

namespace ta {

// What the row scores need of a column: z = ((2x - med2) * zc) / zd, and
// zy = 1 / zd rounded to nearest.
struct alignas(32) ColZ {
  int64_t med2;
  double zc, zd, zy;
};

// The robust z of a cell in one division with per-column (zc, zd): when
// mad4 > 0, (2.0, 1.4826 * mad4) -- (2x - med2) * 2 converts to the same double
// as 4x - 2 med2; when only the mean absolute deviation is positive,
// (n, 1.253314 * sumdev); else (0, 1) (every cell is the median, z = 0).
__host__ __device__ inline void z_coefs(int64_t mad4, int64_t sumdev, int64_t n, double &zc, double &zd) {
  if (mad4 > 0) {
    zc = 2.0;
    zd = 1.4826 * (double)mad4;
  } else if (sumdev > 0) {
    zc = (double)n;
    zd = 1.253314 * (double)sumdev;
  } else {
    zc = 0.0;
    zd = 1.0;
  }
}

__device__ inline int nbits64(uint64_t v) { return v ? 64 - __clzll((long long)v) : 0; }

// The robust FULL scan's first stage with columns in registers
// (k_colscan.hip), for at most COL_REG_MAX ranks: m_t[g][r] = mean over rank
// r's iterations of its cells' scores.  st.rc is 0, or col_stat_chunks(R): the
// columns' imbalance partials too, complete when stats_ready (if set) has been
// recorded.  COL_REG_MAX is the longest column with a form here (sixteen waves of
// 48 words a lane; longer ones are not measured): 1,600 columns of 49,152 ranks take
// 656 us this way, of 49,153 by the row-major passes 1,312.  Only columns spread over
// 2^31 and more are slower here, above 32,768 ranks: 6,400 of them of 40,000 ranks
// 3,374 us, by the passes 2,728.
constexpr int64_t COL_REG_MAX = 49152;
int col_stat_chunks(int64_t R);
size_t col_scan_ws_bytes(int64_t R, int IG);
hipError_t launch_col_scan(const int64_t *T, int64_t R, int I, int G, const int32_t *it, ColPartials st,
                           hipEvent_t stats_ready, double *m_t, void *ws, int cus, hipStream_t s);
// m_t from the row-major tensor and the columns' coefficients.
hipError_t launch_score_tensor(const int64_t *T, int64_t R, int I, int G, const int32_t *it,
                               const ColZ *cz, double *m_t, int cus, hipStream_t s);

// Plain z of a cell: (n x - s1) / zd (zy = 1 / zd); (0, 0, 1, 1) where the
// column's deviation is 0.
struct alignas(32) ColMom {
  int64_t n, s1;
  double zd, zy;
};
// m_t from the row-major tensor and the columns' moments.
hipError_t launch_score_plain(const int64_t *T, int64_t R, int I, int G, const int32_t *it,
                              const ColMom *cm, double *m_t, hipStream_t s);

}  // namespace ta
