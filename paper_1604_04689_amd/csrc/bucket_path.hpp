// What the two units of the vertex-bucket pipeline share on the host.
#pragma once

#include "internal.hpp"

namespace mnb {

constexpr int BK_CUS = 256;            // CUs of the GPU
constexpr int BK_MAX_DEGREE = 40;      // most elements per vertex, on average, of a mesh that takes buckets
// Most small buckets of a mesh.  More of them run in several rounds, and large
// ones have twice the threads to a bucket: 512 large buckets took 55 / 52 / 62 us
// where 566 / 566 / 850 small ones took 60 / 56 / 72 us (hexahedra 55^3, their
// node relation, 63^3); 512 half-empty large ones lose below (tetrahedra 32^3:
// 56 us against 52 us in 334 small ones).
constexpr int BK_SMALL_MOST = 448;
constexpr int BK_LEAST_RECORDS = 384;  // fewest records a bucket of a small mesh is planned for
// Records of a bucket, percent of what it holds, on average: a bucket with more
// than it holds is finished from memory, by several blocks (bk_shares), at two to
// four times the cost of its records, and every later one waits for it.  The
// vertices of most meshes of one type differ little.  A pyramid's apex has 6
// elements where a corner of its base has 24, and labels with locality put
// vertices of a kind side by side, so buckets of corners get 24 / 15 of the
// average; in a hybrid mesh they get about twice the average.  These two are the shares of
// cubic lattices; a mesh whose kinds differ more overfills some buckets, one whose
// kinds are well mixed pays for buckets less full than they could be.  (Local
// labels, us: element relation of 90^3 pyramid cells 493 at 92 % and 257 at 56 %;
// hybrid mesh of 4 M ids 353 at 80 % and 181 at 45 %.  Shuffled labels: 90^3 208
// and 209, 60^3 65 and 74, the hybrid mesh 195 and 210.)
constexpr int BK_FULL = 92, BK_FULL_PYRAMID = 56, BK_FULL_MIXED = 45;
constexpr int bk_full(int32_t etype) { return etype == MESH_PYRAMID5 ? BK_FULL_PYRAMID : BK_FULL; }
// Most buckets of a mesh that would fill the GPU with large tiles but has too many
// buckets for their LDS.  Small tiles read and write ten bytes of counts per tile
// and bucket: 165^3 hexahedra and wedges of 180 x 180 x 90 (6649 and 6656 buckets)
// take 1702 and 1359 us, by sorting 1898 and 1534; 170^3 and 190 x 190 x 95 (7670)
// 2052 and 2602, by sorting 2063 and 1787; 176^3 (8191) 3490, by sorting 2277.
constexpr uint32_t BK_SMALL_TILE_MOST = 6656;
constexpr int BK_HIST_BLOCKS = 512;    // blocks of bk_hist aimed at

// Records and vertices a bucket may hold (BkShape).
struct BkSize {
    int cap, vmax;
};
BkSize bk_size(int K, bool large);

// The buckets of a mesh, `full` percent full on average, and its records' form,
// for K neighbours a record; false: not for buckets.
bool plan_bucket_map(int64_t n_elem, int64_t n_slots, int32_t n_vert, int K, int full, BkPlan* p);
// Tiles of tile_elems elements of up to most_npe nodes and the workspace (without what
// shares of overfull buckets need, if it does not fit with it); sets p->on.
void plan_bucket_layout(int64_t tile_elems, int most_npe, size_t limit, BkPlan* p);

// Meshes of several element types (both relations).
void plan_mixed_buckets(int64_t n_elem, int64_t n_ids, int32_t n_vert, const Opts& o, size_t limit, BkPlan* p);
hipError_t run_mixed_buckets(const BkPlan& p, const int32_t* conn, const int32_t* elem_off, const uint8_t* etypes,
                             int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap, int32_t* elem_row_ptr,
                             int32_t* elem_cols, int64_t elem_cap, void* ws, hipStream_t s);

// Records from which on a bucket is shared.
inline uint32_t bk_share_cap(const BkPlan& p) { return p.shares ? (uint32_t)bk_size(p.K, p.large).cap : UINT32_MAX; }

hipError_t launch_bucket_rows(const BkPlan& p, int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap,
                              int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, char* w, hipStream_t s);

}  // namespace mnb
