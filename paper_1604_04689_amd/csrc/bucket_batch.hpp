// What the two units of the batch's vertex buckets share on the host.
#pragma once

#include "bucket_path.hpp"

namespace mnb {

// Header words (HDR_*) that hold what the device found the batch to need.
constexpr int HDR_BKB_BUCKETS = 48, HDR_BKB_TILES = 49, HDR_BKB_SCANS = 50;
constexpr int HDR_BKB_SHARED = 51;  // some bucket has shares

// One entry of the batch's bucket table: a mesh, or the vertices between two
// meshes' ranges that no valid record covers (usually none).
struct BkMesh {
    BkMap mp;
    int32_t etype, W;
    uint32_t bucket0, n_tiles, te;  // first bucket; tiles and elements per tile
    uint32_t tile0, scan0;
    int32_t vert_off;
    int64_t n_elem, ids;  // elements, first id in conn
    uint64_t rec0;        // first word of its records
    uint64_t cell0;       // its counts: n_tiles x nb_pad cells
};

struct BkBatchPlan {
    bool on = false;
    bool large = false;      // bucket size (BkShape)
    bool shares = false;     // overfull buckets are shared by several blocks
    int32_t n_mesh = 0, total_vert = 0, max_vert = 0;
    int64_t total_slots = 0, total_pairs = 0;
    int32_t fill[5] = {};    // records a bucket is planned for, by K
    int32_t nb_most = 0;     // most buckets of one mesh
    int32_t tile_slots = 0;  // most slots per tile
    int64_t entries = 0, bucket_most = 0, unit_most = 0, tile_most = 0, scan_most = 0, cell_most = 0, word_most = 0;
    size_t off_mesh = 0, off_tile0 = 0, off_scan0 = 0, off_bmesh = 0, off_tmesh = 0, off_starts = 0,
           off_units = 0, off_rep = 0, off_lb = 0, off_cells = 0, off_rec = 0, off_list = 0;  // (no list: 0)
    size_t total = 0;
};

// Plans the batch's buckets into at most `limit` workspace bytes; p->on says
// whether they apply.  The node relation is wanted, the element one may be.
void plan_batch_buckets(int32_t n_mesh, int64_t total_pairs, int64_t total_slots, int32_t total_vert, int32_t max_vert,
                        const Opts& o, size_t limit, BkBatchPlan* p);
// Element outputs may be null.
hipError_t run_batch_buckets(const BkBatchPlan& p, const int32_t* conn, const mesh_segment* segs,
                             int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap, int32_t* elem_row_ptr,
                             int32_t* elem_cols, int64_t elem_cap, void* ws, hipStream_t s);
hipError_t launch_batch_bucket_rows(const BkBatchPlan& p, int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap,
                                    int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, char* w, hipStream_t s);

}  // namespace mnb
