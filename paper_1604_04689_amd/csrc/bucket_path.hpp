// What the two units of the vertex-bucket pipeline share on the host.
#pragma once

#include "internal.hpp"

namespace mnb {

constexpr int BK_CUS = 256;            // CUs of the GPU
constexpr int BK_MAX_DEGREE = 40;      // most elements per vertex, on average, of a mesh that takes buckets
constexpr int BK_SMALL_MOST = 1024;    // most small buckets
constexpr int BK_LEAST_RECORDS = 384;  // fewest records a bucket of a small mesh is planned for
constexpr int BK_HIST_BLOCKS = 512;    // blocks of bk_hist aimed at

// Records and vertices a bucket may hold (BkShape).
struct BkSize {
    int cap, vmax;
};
BkSize bk_size(int K, bool large);

hipError_t launch_bucket_rows(const BkPlan& p, int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap,
                              int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, char* w, hipStream_t s);

}  // namespace mnb
