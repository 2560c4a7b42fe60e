// Constants of the matrix-core nearest-centroid filter (pq_nearest_filter.h; the argument is in pq_encode.hip), in one
// place: the encode and training kernels include this file and the host-side bound tests parse it, so they cannot drift
// apart.  Per token, with X2 = sum x_j^2 (of scaled numbers: pq_filter_scale) and `best` its smallest computed value:
//   off = PQ_FILTER_X2_FACTOR X2 + 3 PQ_FILTER_TAU_ABS, rounded up      (keeps every value positive)
//   tau = PQ_FILTER_TAU_NEAR (X2 + best) + PQ_FILTER_TAU_ABS            (fp32 inputs: PQ_FILTER_TAU_NEAR_F32)
#pragma once

#define PQ_FILTER_X2_FACTOR 0.5025f
#define PQ_FILTER_TAU_ABS 2.4e-07f
#define PQ_FILTER_TAU_NEAR 1.05e-05f
#define PQ_FILTER_TAU_NEAR_F32 2.5e-05f
