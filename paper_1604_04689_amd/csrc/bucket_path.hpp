// What the two units of the vertex-bucket pipeline share on the host.
#pragma once

#include "internal.hpp"

namespace mnb {

constexpr int BK_CUS = 256;            // CUs of the GPU
constexpr int BK_MAX_DEGREE = 40;      // most elements per vertex, on average, of a mesh that takes buckets
// Most small buckets of a mesh.  More of them run in several rounds, and large
// ones have twice the threads to a bucket: 512 large buckets took 54 / 50 / 61 us
// where 566 / 566 / 850 small ones took 57 / 55 / 71 us (hexahedra 55^3, their
// node relation, 63^3); 512 half-empty large ones lose below (tetrahedra 32^3:
// 54 us against 51 us in 334 small ones).
constexpr int BK_SMALL_MOST = 448;
constexpr int BK_LEAST_RECORDS = 384;  // fewest records a bucket of a small mesh is planned for
// Records of a bucket, percent of what it holds, on average: a bucket with more
// than it holds is finished from memory, and every later one waits for it.  The
// vertices of a mesh of one type differ little; those of a mixed mesh a lot (a
// cell's centre 0 or 6 elements, a corner 17), and 3 of 512 buckets of 4004
// records ran over 4480: 204 instead of 83 us for the rows of a hybrid mesh of
// 2 M ids.
constexpr int BK_FULL = 92, BK_FULL_MIXED = 80;
constexpr int BK_HIST_BLOCKS = 512;    // blocks of bk_hist aimed at

// Records and vertices a bucket may hold (BkShape).
struct BkSize {
    int cap, vmax;
};
BkSize bk_size(int K, bool large);

// The buckets of a mesh, `full` percent full on average, and its records' form,
// for K neighbours a record; false: not for buckets.
bool plan_bucket_map(int64_t n_elem, int64_t n_slots, int32_t n_vert, int K, int full, BkPlan* p);
// Tiles of tile_elems elements of up to most_npe nodes and the workspace; sets p->on.
void plan_bucket_layout(int64_t tile_elems, int most_npe, size_t limit, BkPlan* p);

// Meshes of several element types (both relations).
void plan_mixed_buckets(int64_t n_elem, int64_t n_ids, int32_t n_vert, const Opts& o, size_t limit, BkPlan* p);
hipError_t run_mixed_buckets(const BkPlan& p, const int32_t* conn, const int32_t* elem_off, const uint8_t* etypes,
                             int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap, int32_t* elem_row_ptr,
                             int32_t* elem_cols, int64_t elem_cap, void* ws, hipStream_t s);

hipError_t launch_bucket_rows(const BkPlan& p, int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap,
                              int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, char* w, hipStream_t s);

}  // namespace mnb
