// Vertex buckets of a batch: every mesh has its own buckets and tiles, and all
// meshes go through each kernel together.  Their sizes stand in the segment
// records in device memory, so the device plans:
//
//   bkb_setup  segment records -> each mesh's buckets, tiles and record form,
//              and where they start among the batch's (one block)
//   bkb_hist   conn -> pairs per bucket and tile
//   bkb_scan   where every tile's records of a bucket go, and
//   bkb_starts where every bucket starts
//   bkb_part   conn -> records in buckets
//   bkb_rows   both CSRs (bucket_batch_rows.hip)
//
// A record must hold only its own mesh's ids and elements, so most meshes take
// the short forms (8 bytes for a triangle's vertex, 12 for a tetrahedron's),
// and a tile's records go to the few buckets of one mesh, in long runs.
#include "bucket_batch.hpp"
#include "buckets.hpp"

namespace mnb {

namespace {

constexpr int BKB_BLOCK = 512;         // bkb_hist, bkb_part
constexpr int BKB_LDS = 78 * 1024;     // of a bkb_part tile: two blocks per CU
constexpr int BKB_NB_MOST = 4096;      // most buckets of one mesh (two words each of that LDS)
// Batches of many tiny meshes go to the sorts: every mesh has a tile and a
// bucket of its own, about 60 ns (16,384 triangle meshes of 54 / 726 / 1350 /
// 3174 slots: 710 / 952 / 1069 / 1341 us against 249 / 826 / 1139 / 2417 us by
// sorting).  Up to 2048 meshes the buckets' fewer launches make up for that
// (2048 meshes of 54 slots: 124 against 185 us).
constexpr int BKB_MESHES = 2048;
constexpr int BKB_MESH_SLOTS = 1400;
constexpr int BKB_TILE_LEAST = 512;    // fewest slots a tile is cut for
constexpr int BKB_SETUP = 1024;
// Most small buckets of a batch: 1.6 M slots in 12 meshes took 80 us in small ones,
// 86 us in large ones (which are not rounded up to whole rounds here), 110,000 in
// 2048 meshes 123 and 141, 1.8 M in 180 meshes 103 and 95.
constexpr int BKB_SMALL_MOST = 1024;

constexpr int bkb_K(int32_t et) { return et == TRI3 || et == QUAD4 ? 2 : et == PYR5 ? 4 : 3; }
static_assert(bkb_K(TRI3) == BkElem<TRI3>::K && bkb_K(QUAD4) == BkElem<QUAD4>::K && bkb_K(TET4) == BkElem<TET4>::K &&
                  bkb_K(HEX8) == BkElem<HEX8>::K && bkb_K(WEDGE6) == BkElem<WEDGE6>::K && bkb_K(PYR5) == BkElem<PYR5>::K,
              "edge-neighbours per type");
// Elements per thread: as many as the LDS takes.
constexpr int bkb_ept(int32_t et) { return et == TRI3 ? 4 : et == QUAD4 ? 3 : et == TET4 ? 2 : 1; }

// Elements per tile of a mesh with nb_pad buckets.
__host__ __device__ inline int32_t bkb_tile_elems(int32_t et, int W, uint32_t nb_pad, int32_t tile_slots) {
    const int npe = nodes_per_elem(et);
    const int fit = (BKB_LDS - 8 * (int)nb_pad) / (npe * (4 * W + 2));
    return tmax(1, tmin(tmin(BKB_BLOCK * bkb_ept(et), fit), tile_slots / npe));
}

// Inclusive scan over the lanes of a wave (DPP: no LDS round trips); 0 is op's
// identity.
template <class Op>
__device__ __forceinline__ uint32_t bkb_wave_scan(uint32_t x, Op op) {
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false));  // row_shr:1
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false));
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false));
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false));
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));  // row_bcast:15
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return x;
}
// Exclusive scans of N values over the block (thread order), each with a
// running carry.
constexpr int BKB_SETUP_WAVES = BKB_SETUP / WAVE;
template <int N, class Op>
__device__ __forceinline__ void bkb_block_scan(uint32_t (&v)[N], uint32_t (&carry)[N],
                                               uint32_t (*s_w)[BKB_SETUP_WAVES], Op op) {
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE;
    __syncthreads();  // s_w free again
#pragma unroll
    for (int q = 0; q < N; ++q) {
        v[q] = bkb_wave_scan(v[q], op);
        if (lane == WAVE - 1) s_w[q][wid] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t w = bkb_wave_scan(lane < BKB_SETUP_WAVES ? s_w[q][lane] : 0u, op);
        const uint32_t waves = wid ? (uint32_t)__builtin_amdgcn_readlane((int)w, wid - 1) : 0u;
        const uint32_t before = op(carry[q], waves);
        const uint32_t left = (uint32_t)__shfl_up((int)v[q], 1, WAVE);
        v[q] = lane == 0 ? before : op(before, left);
        carry[q] = op(carry[q], (uint32_t)__builtin_amdgcn_readlane((int)w, BKB_SETUP_WAVES - 1));
    }
}

struct SetupArgs {
    const mesh_segment* segs;
    int32_t n_mesh, total_vert, max_vert;
    int64_t total_slots, total_pairs;
    int32_t fill[5], vmax[5];
    int32_t nb_most, tile_slots;
    BkMesh* mesh;
    uint32_t* tile0;
    uint32_t* scan0;
    uint32_t* hdr;
};

__device__ __forceinline__ uint32_t ceil_div32(uint32_t a, uint32_t b) { return a / b + (a % b != 0 ? 1u : 0u); }
// Smallest b with 2^b >= n.
__device__ __forceinline__ uint32_t bkb_bits(uint32_t n) { return n <= 1 ? 0u : 32u - (uint32_t)__clz((int)(n - 1)); }

// A table entry but for its offsets.  All 32-bit: a 64-bit division takes a
// hundred instructions, and this runs in one block.
__device__ __forceinline__ BkMesh bkb_entry(const SetupArgs& a, uint32_t nv, uint32_t n_elem, int32_t et,
                                            int32_t vert_off, int64_t ids) {
    BkMesh e{};
    e.etype = et;
    e.vert_off = vert_off;
    e.n_elem = n_elem;
    e.ids = ids;
    e.mp.n_vert = (int32_t)nv;
    const int K = bkb_K(et);
    e.W = K;
    if (nv == 0) return e;
    const uint32_t fill = K == 2 ? a.fill[2] : K == 3 ? a.fill[3] : a.fill[4];
    const uint32_t vmax = K == 2 ? a.vmax[2] : K == 3 ? a.vmax[3] : a.vmax[4];
    const uint32_t by_rec = tmin<uint32_t>(ceil_div32((uint32_t)nodes_per_elem(et) * n_elem, fill), a.nb_most);
    const uint32_t nb = tmax(ceil_div32(nv, vmax - 2), tmax(by_rec, 1u));
    const uint32_t width = tmax(ceil_div32(nv, nb), 2u);
    BkMap& m = e.mp;
    m.mul = 0xffffffffu / width + ((width & (width - 1)) == 0 ? 1u : 0u);  // 2^32 / width
    m.n_bucket = __umulhi(nv - 1, m.mul) + 1;
    m.nb_pad = (m.n_bucket + 1) & ~1u;
    const uint32_t vl_bits = bkb_bits(0xffffffffu / m.mul + 1);
    m.vl_mask = (1u << vl_bits) - 1;
    m.e_bits = tmax(bkb_bits(n_elem), 1u);
    m.id_bits = tmax(bkb_bits(nv), 1u);
    m.e_shift = 2 * m.id_bits + vl_bits;
    if (n_elem == 0) return e;
    e.W = bk_words(K, m.e_bits, m.id_bits, vl_bits);
    e.te = (uint32_t)bkb_tile_elems(et, e.W, m.nb_pad, a.tile_slots);
    e.n_tiles = ceil_div32(n_elem, e.te);
    return e;
}
// Pairs of words its records take.  (An empty last bucket reads one record past
// the others.)
__device__ __forceinline__ uint32_t bkb_word_pairs(const BkMesh& e) {
    return (uint32_t)(((uint64_t)nodes_per_elem(e.etype) * (uint64_t)e.n_elem * (uint32_t)e.W + 8) / 2);
}

// A record is good when it fits the batch's totals and its vertices and slots
// start no earlier than those of the records before it end.  (Where its pairs
// start does not matter here: their number bounds the records' room.)  A record
// that is not is reported and left out, its rows empty.  One block, bound by its instructions and barriers (32-bit
// sums over DPP, the plan keeps every total below 2^32: 12 us for 512 meshes,
// 84 us in 64 bits).
__global__ __launch_bounds__(BKB_SETUP) void bkb_setup_kernel(SetupArgs a) {
    __shared__ uint32_t s_w[5][BKB_SETUP_WAVES];
    const int tid = threadIdx.x;
    if (tid < (int)(HEADER_BYTES / 4)) a.hdr[tid] = 0;
    auto add = [](uint32_t x, uint32_t y) { return x + y; };
    auto most = [](uint32_t x, uint32_t y) { return max(x, y); };
    auto add_up_to = [](uint32_t x, uint32_t y) { return x + y < x ? UINT32_MAX : x + y; };
    uint32_t end[2] = {}, used[1] = {};  // ends so far: vertices and slots of any record; vertices of good ones
    uint32_t pairs[1] = {};              // pairs of any record so far, at most 2^32 - 1
    uint32_t sum[5] = {};                // buckets, tiles, blocks of bkb_scan, cells, word pairs
    uint32_t mine[1] = {};               // slots of this thread's good records
    bool bad = false;
    for (int64_t m0 = 0; m0 <= a.n_mesh; m0 += BKB_SETUP) {
        const int64_t i = m0 + tid;
        const bool in = i < a.n_mesh, tail = i == a.n_mesh;
        mesh_segment sg{};
        if (in) sg = a.segs[i];
        const int npe = nodes_per_elem(sg.etype), ppe = 2 * edges_per_elem(sg.etype);
        bool good = in && (npe > 0 || sg.n_elem == 0) && sg.n_elem >= 0 && sg.n_elem <= INT32_MAX && sg.n_vert >= 0 &&
                    sg.n_vert <= a.max_vert && sg.vert_off >= 0 && (int64_t)sg.vert_off + sg.n_vert <= a.total_vert &&
                    sg.slot_off >= 0 && sg.slot_off <= a.total_slots && sg.slot_off + npe * sg.n_elem <= a.total_slots &&
                    ppe * sg.n_elem <= a.total_pairs;
        const uint32_t vert = good ? (uint32_t)sg.vert_off : 0u, slot = good ? (uint32_t)sg.slot_off : 0u,
                       nv = good ? (uint32_t)sg.n_vert : 0u,
                       ne = good ? (uint32_t)sg.n_elem : 0u;
        uint32_t at[2] = {vert + nv, slot + npe * ne}, before[1] = {(uint32_t)ppe * ne};
        bkb_block_scan(at, end, s_w, most);
        bkb_block_scan(before, pairs, s_w, add_up_to);
        good = good && vert >= at[0] && slot >= at[1] && (int64_t)before[0] + ppe * ne <= a.total_pairs;
        uint32_t from[1] = {good ? vert + nv : 0u};
        bkb_block_scan(from, used, s_w, most);
        if (good) mine[0] += npe * ne;
        bad |= (in && !good) || (good && nv == 0 && ne > 0);
        // the vertices before it that no record covers, and the mesh; after the last one the vertices left
        const uint32_t gap = good ? vert - from[0] : tail ? (uint32_t)a.total_vert - from[0] : 0u;
        BkMesh hole{}, mesh{};
        if (gap) hole = bkb_entry(a, gap, 0, TRI3, (int32_t)from[0], 0);
        // (the type of a mesh without elements may be anything)
        if (good) mesh = bkb_entry(a, nv, nv ? ne : 0u, npe > 0 ? sg.etype : (int32_t)TRI3, sg.vert_off, sg.conn_off);
        const uint32_t scans = ceil_div32(hole.mp.n_bucket, BKS_COLS);
        uint32_t o[5] = {hole.mp.n_bucket + mesh.mp.n_bucket, mesh.n_tiles, scans + ceil_div32(mesh.mp.n_bucket, BKS_COLS),
                         mesh.n_tiles * mesh.mp.nb_pad, bkb_word_pairs(hole) + bkb_word_pairs(mesh)};
        bkb_block_scan(o, sum, s_w, add);
        auto put = [&](int64_t entry, BkMesh& x) {
            x.bucket0 = o[0];
            x.tile0 = o[1];
            x.scan0 = o[2];
            x.cell0 = o[3];
            x.rec0 = 2ull * o[4];
            a.tile0[entry] = x.tile0;
            a.scan0[entry] = x.scan0;
            a.mesh[entry] = x;
        };
        if (in || tail) put(2 * i, hole);
        if (in) {
            o[0] += hole.mp.n_bucket;
            o[2] += scans;
            o[4] += bkb_word_pairs(hole);
            put(2 * i + 1, mesh);
        }
    }
    uint32_t all[1] = {};
    bkb_block_scan(mine, all, s_w, add);
    bad = __syncthreads_or(bad);
    if (tid == 0) {
        a.hdr[HDR_BKB_BUCKETS] = sum[0];
        a.hdr[HDR_BKB_TILES] = sum[1];
        a.hdr[HDR_BKB_SCANS] = sum[2];
        if (bad || all[0] != (uint32_t)a.total_slots) a.hdr[HDR_ERR] = ERR_INDEX_RANGE;
    }
}

// Elements [e0, e0 + count) of a tile counted by bucket into s_h; what was
// found odd.
template <int ET>
__device__ __forceinline__ uint32_t bkb_hist_tile(const int32_t* __restrict__ conn, int64_t e0, int32_t count,
                                                  const BkMap& mp, uint32_t* s_h) {
    constexpr int NPE = Elem<ET>::NPE, EPT = bkb_ept(ET);
    const int tid = threadIdx.x;
    int32_t id[EPT][NPE] = {};
#pragma unroll
    for (int u = 0; u < EPT; ++u)
        if (u * BKB_BLOCK + tid < count) load_elem_ids<ET>(conn, e0 + u * BKB_BLOCK + tid, id[u]);
    for (int i = tid; i < (int)mp.nb_pad; i += BKB_BLOCK) s_h[i] = 0;
    __syncthreads();
    uint32_t found = 0;
    const bool crowded = bk_crowded(bk_bucket((uint32_t)id[0][0], mp.mul));
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const bool in = u * BKB_BLOCK + tid < count;
#pragma unroll
        for (int j = 0; j < NPE; ++j) {
            const uint32_t v = (uint32_t)id[u][j];
            const bool ok = in && v < (uint32_t)mp.n_vert;
            if (in && !ok) found |= BK_BAD_ID;
#pragma unroll
            for (int jj = 0; jj < j; ++jj)
                if (ok && (uint32_t)id[u][jj] == v) found |= BK_HAS_DUP;
            bk_count(s_h, ok ? bk_bucket(v, mp.mul) : 0u, ok, crowded);
        }
    }
    __syncthreads();
    return found;
}

// A block takes every gridDim-th tile.  (Blocks and XCDs go in turn, and the
// grid is a multiple of their number, so a tile's XCD is its number mod 8 here
// and in bkb_part.)
__global__ __launch_bounds__(BKB_BLOCK) void bkb_hist_kernel(const int32_t* __restrict__ conn,
                                                            const BkMesh* __restrict__ mesh,
                                                            const uint32_t* __restrict__ tile0, int entries,
                                                            uint32_t* __restrict__ tmesh, uint32_t* __restrict__ cells,
                                                            uint32_t* hdr) {
    extern __shared__ uint32_t s_h[];
    __shared__ uint32_t s_found;
    const int tid = threadIdx.x;
    if (tid == 0) s_found = 0;
    const uint32_t n_tiles = hdr[HDR_BKB_TILES];
    uint32_t found = 0;
    for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const int k = bk_find(tile0, entries, t);
        const BkMesh& m = mesh[k];
        if (tid == 0) tmesh[t] = (uint32_t)k;
        const uint32_t i = t - m.tile0;
        const int64_t e0 = (int64_t)i * m.te;
        const int32_t count = (int32_t)tmin<int64_t>(m.te, m.n_elem - e0);
        found |= with_type(m.etype, [&](auto et) {
            return bkb_hist_tile<decltype(et)::value>(conn + m.ids, e0, count, m.mp, s_h);
        });
        uint32_t* c = cells + m.cell0 + (uint64_t)i * m.mp.nb_pad;
        for (int b = tid; b < (int)m.mp.n_bucket; b += BKB_BLOCK) c[b] = s_h[b];
        __syncthreads();
    }
    if (found) atomicOr(&s_found, found);
    __syncthreads();
    if (tid == 0 && s_found) {
        atomicOr(&hdr[HDR_BK_ODD], s_found);
        if (s_found & BK_BAD_ID) set_error(hdr + HDR_ERR, ERR_INDEX_RANGE);
    }
}

// cells: the counts of a mesh's tiles become the records of the bucket in the
// tiles before, in the order of the tiles' XCDs; totals[b] the bucket's own,
// more[b] its units less one (bk_shares).  A
// block takes 16 buckets of one mesh, 16 threads each: 41 us for 512 meshes
// (30,000 tiles, 24,000 buckets, 26 MB of cells).
constexpr int BKB_SCAN = 256;
constexpr int BKB_ROWS = BKB_SCAN / BKS_COLS;
constexpr int BKB_AHEAD = 8;  // cells read at once
struct BkbCaps {
    uint32_t K2, K3, K4;  // records a bucket's block holds
};
__global__ __launch_bounds__(BKB_SCAN) void bkb_scan_kernel(const BkMesh* __restrict__ mesh,
                                                           const uint32_t* __restrict__ scan0, int entries,
                                                           uint32_t* __restrict__ cells, uint32_t* __restrict__ totals,
                                                           uint32_t* __restrict__ more, BkbCaps cap,
                                                           uint32_t* __restrict__ bmesh, BkLookback lookback,
                                                           uint32_t* __restrict__ repeats, uint32_t* hdr) {
    __shared__ uint32_t s_sum[BKB_ROWS][BKS_COLS];
    const int tid = threadIdx.x;
    const uint32_t block = blockIdx.x;
    if (block >= hdr[HDR_BKB_SCANS]) return;
    const int k = bk_find(scan0, entries, block);
    const BkMesh& m = mesh[k];
    const int c = tid % BKS_COLS, g = tid / BKS_COLS;
    const uint32_t col = (block - m.scan0) * BKS_COLS + c;
    const uint32_t nb = m.mp.n_bucket, nb_pad = m.mp.nb_pad, n_tiles = m.n_tiles;
    uint32_t* const cell = cells + m.cell0 + tmin(col, nb - 1);
    // tiles in the order x, then y of tile 8 y + x; a run of them per thread
    const uint32_t kk = (n_tiles + BK_XCDS - 1) / BK_XCDS;
    const uint32_t per = (kk * BK_XCDS + BKB_ROWS - 1) / BKB_ROWS;
    const uint32_t q0 = tmin<uint32_t>(g * per, kk * BK_XCDS), q1 = col < nb ? tmin<uint32_t>(q0 + per, kk * BK_XCDS) : 0u;
    auto each = [&](auto f) {  // f(values, their tiles; n_tiles or more: none), some at a time
        if (q0 >= q1) return;
        uint32_t x = q0 / kk, y = q0 % kk;
        for (uint32_t q = q0; q < q1; q += BKB_AHEAD) {
            uint32_t t[BKB_AHEAD], v[BKB_AHEAD];
#pragma unroll
            for (int u = 0; u < BKB_AHEAD; ++u) {
                t[u] = q + u < q1 ? y * BK_XCDS + x : n_tiles;
                v[u] = cell[(uint64_t)tmin(t[u], n_tiles - 1) * nb_pad];
                if (++y == kk) {
                    y = 0;
                    ++x;
                }
            }
#pragma unroll
            for (int u = 0; u < BKB_AHEAD; ++u) v[u] = t[u] < n_tiles ? v[u] : 0u;
            f(v, t);
        }
    };
    uint32_t sum = 0;
    each([&](const uint32_t(&v)[BKB_AHEAD], const uint32_t(&)[BKB_AHEAD]) {
#pragma unroll
        for (int u = 0; u < BKB_AHEAD; ++u) sum += v[u];
    });
    s_sum[g][c] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
#pragma unroll
    for (int r = 0; r < BKB_ROWS; ++r) {
        const uint32_t v = s_sum[r][c];
        run += r < g ? v : 0u;
        tot += v;
    }
    if (g == 0 && col < nb) {
        const uint32_t at = m.bucket0 + col;
        const int K = bkb_K(m.etype);
        const uint32_t shares = bk_shares(tot, K == 2 ? cap.K2 : K == 3 ? cap.K3 : cap.K4);
        totals[at] = tot;
        if (more) more[at] = shares - 1;
        if (shares > 1) atomicOr(&hdr[HDR_BKB_SHARED], 1u);
        bmesh[at] = (uint32_t)k;
        lookback.clear(at);
        repeats[at] = 0;   // counted by bkb_part
    }
    each([&](const uint32_t(&v)[BKB_AHEAD], const uint32_t(&t)[BKB_AHEAD]) {
#pragma unroll
        for (int u = 0; u < BKB_AHEAD; ++u) {
            if (t[u] < n_tiles) cell[(uint64_t)t[u] * nb_pad] = run;
            run += v[u];
        }
    });
}

// The buckets' totals become their starts, in place (one more: the end).  One
// block, eight buckets per thread at a time: 23 us for 24,000 buckets.  (With the
// sums of bkb_scan's blocks handed on in order, by ticket, both took 170 us: the
// tickets of 4500 blocks queue at one address.)
constexpr int BKB_AT_ONCE = 8;
// a[0 .. n) becomes its exclusive sums, plus its places' numbers with `places`;
// a[n] the whole.
__device__ __forceinline__ uint32_t bkb_sums(uint32_t* __restrict__ a, uint32_t n, bool places,
                                             uint32_t (*s_w)[BKB_SETUP_WAVES]) {
    auto add = [](uint32_t x, uint32_t y) { return x + y; };
    uint32_t carry[1] = {};
    for (uint32_t b0 = 0; b0 < n; b0 += BKB_SETUP * BKB_AT_ONCE) {
        const uint32_t b = b0 + threadIdx.x * BKB_AT_ONCE;
        uint32_t v[BKB_AT_ONCE], sum[1] = {};
#pragma unroll
        for (int q = 0; q < BKB_AT_ONCE; ++q) {
            v[q] = b + q < n ? a[b + q] : 0u;
            sum[0] += v[q];
        }
        bkb_block_scan(sum, carry, s_w, add);
#pragma unroll
        for (int q = 0; q < BKB_AT_ONCE; ++q) {
            if (b + q < n) a[b + q] = sum[0] + (places ? b + q : 0u);
            sum[0] += v[q];
        }
    }
    const uint32_t all = carry[0] + (places ? n : 0u);
    if (threadIdx.x == 0) a[n] = all;
    return all;
}
__global__ __launch_bounds__(BKB_SETUP) void bkb_starts_kernel(uint32_t* __restrict__ starts, uint32_t* __restrict__ units,
                                                              BkLookback lookback, uint32_t* hdr) {
    __shared__ uint32_t s_w[1][BKB_SETUP_WAVES];
    const uint32_t n = hdr[HDR_BKB_BUCKETS];
    const bool shared = hdr[HDR_BKB_SHARED] != 0;
    bkb_sums(starts, n, false, s_w);
    uint32_t all = n;
    if (shared) {
        all = bkb_sums(units, n, true, s_w);
        for (uint32_t u = n + threadIdx.x; u < all; u += BKB_SETUP) lookback.clear(u);
    }
    if (threadIdx.x == 0) hdr[HDR_BK_UNITS] = all;
}

// Two tiles per CU at a time.  Bound by the records' way out: the 137 M slots
// of 512 meshes (549 MB in, 1.58 GB out) in 625 us, 3.4 TB/s.
__global__ __launch_bounds__(BKB_BLOCK) void bkb_part_kernel(const int32_t* __restrict__ conn,
                                                            const BkMesh* __restrict__ mesh,
                                                            const uint32_t* __restrict__ tmesh,
                                                            const uint32_t* __restrict__ cells,
                                                            const uint32_t* __restrict__ starts,
                                                            uint32_t* __restrict__ rec, uint32_t* repeats, uint32_t* hdr) {
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_tmp[BKB_BLOCK / WAVE];
    const uint32_t n_tiles = hdr[HDR_BKB_TILES];
    for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const BkMesh& m = mesh[__builtin_amdgcn_readfirstlane((int)tmesh[t])];
        const uint32_t i = t - m.tile0;
        const int64_t e0 = (int64_t)i * m.te;
        const int32_t count = (int32_t)tmin<int64_t>(m.te, m.n_elem - e0);
        const uint32_t* c = cells + m.cell0 + (uint64_t)i * m.mp.nb_pad;
        const uint32_t* st = starts + m.bucket0;
        const uint32_t base = st[0];
        with_type(m.etype, [&](auto et) {
            constexpr int ET = decltype(et)::value, K = BkElem<ET>::K;
            auto part = [&](auto w) {
                bk_part_tile<ET, K, decltype(w)::value, BKB_BLOCK, bkb_ept(ET)>(
                    conn + m.ids, e0, count, m.mp, [&](int b) { return st[b] - base + c[b]; }, rec + m.rec0,
                    Elem<ET>::NPE * m.n_elem, repeats + m.bucket0, hdr, s_dyn, s_tmp);
            };
            if constexpr (K < 4) {
                if (m.W == K) {
                    part(std::integral_constant<int, K>{});
                    return;
                }
            }
            part(std::integral_constant<int, K + 1>{});
        });
        __syncthreads();  // before the LDS is used again
    }
}

}  // namespace

void plan_batch_buckets(int32_t n_mesh, int64_t total_pairs, int64_t total_slots, int32_t total_vert, int32_t max_vert,
                        const Opts& o, size_t limit, BkBatchPlan* p) {
    *p = BkBatchPlan{};
    if (!o.library || n_mesh < 1 || total_slots < 1 || total_vert < 1 || max_vert < 1) return;
    if (total_slots > (int64_t)BK_MAX_DEGREE * total_vert) return;
    if (n_mesh > BKB_MESHES && total_slots < (int64_t)BKB_MESH_SLOTS * n_mesh) return;
    p->n_mesh = n_mesh;
    p->total_vert = total_vert;
    p->max_vert = max_vert;
    p->total_slots = total_slots;
    p->total_pairs = total_pairs;
    p->entries = 2 * (int64_t)n_mesh + 1;
    // (records of a bucket of the fullest kind, which decide the bucket size and the most buckets of a mesh, and the
    // least any is planned for)
    int full_least = INT32_MAX, fill_least = INT32_MAX, vmax_least = INT32_MAX;
    for (int large = 0; large < 2; ++large) {
        p->large = large != 0;
        full_least = fill_least = vmax_least = INT32_MAX;
        for (int K = 2; K <= 4; ++K) {
            const BkSize z = bk_size(K, large != 0);
            // few records still spread over the CUs
            const int64_t spread = large ? z.cap : tmax<int64_t>(BK_LEAST_RECORDS, total_slots / BK_CUS);
            p->fill[K] = (int32_t)tmin<int64_t>(z.cap * (K == 4 ? BK_FULL_PYRAMID : BK_FULL) / 100, spread);
            full_least = tmin(full_least, (int)tmin<int64_t>(z.cap * BK_FULL / 100, spread));
            fill_least = tmin(fill_least, p->fill[K]);
            vmax_least = tmin(vmax_least, z.vmax - 2);
        }
        if (ceil_div(total_slots, (int64_t)full_least) <= BKB_SMALL_MOST) break;
    }
    const int64_t nb_most = tmax<int64_t>(ceil_div(max_vert, (int64_t)vmax_least),
                                          ceil_div((int64_t)max_vert * BK_MAX_DEGREE, (int64_t)full_least)) + 1;
    if (nb_most > BKB_NB_MOST) return;
    p->nb_most = (int32_t)nb_most;
    // few elements still spread over the CUs
    p->tile_slots = (int32_t)tmin<int64_t>(1 << 20, tmax<int64_t>(BKB_TILE_LEAST, total_slots / (2 * BK_CUS)));
    int64_t tile_least = INT32_MAX;
    for (int et = 0; et < N_ELEM_TYPES; ++et)
        tile_least = tmin<int64_t>(tile_least, (int64_t)nodes_per_elem(et) *
                                                   bkb_tile_elems(et, bkb_K(et) + 1, (uint32_t)nb_most + 1, p->tile_slots));
    const int64_t n = p->entries;
    p->bucket_most = ceil_div(total_slots, (int64_t)fill_least) + ceil_div(total_vert, (int64_t)vmax_least) + 3 * n;
    p->tile_most = ceil_div(total_slots, tile_least) + n;
    p->scan_most = ceil_div(p->bucket_most, (int64_t)BKS_COLS) + n;
    p->cell_most = p->tile_most * (nb_most + 1);
    // K + 1 words per slot: a word, and K: the edges' ends (a pyramid has 16 of them for 20 neighbours)
    p->word_most = total_slots + total_pairs + total_pairs / 4 + 16 * n;
    // (without what the shares of overfull buckets need, if it does not fit with it)
    for (int shares = 1; shares >= 0 && !p->on; --shares) {
        p->shares = shares != 0;
        p->unit_most = p->bucket_most;
        for (int K = 2; K <= 4 && p->shares; ++K)
            p->unit_most = tmax(p->unit_most, bk_unit_most(p->bucket_most, total_slots, bk_size(K, p->large).cap));
        size_t off = HEADER_BYTES;
        auto take = [&](size_t* at, size_t bytes) {
            *at = off;
            off += align_up(bytes);
        };
        take(&p->off_mesh, (size_t)n * sizeof(BkMesh));
        take(&p->off_tile0, (size_t)n * 4);
        take(&p->off_scan0, (size_t)n * 4);
        take(&p->off_bmesh, (size_t)p->bucket_most * 4);
        take(&p->off_tmesh, (size_t)p->tile_most * 4);
        take(&p->off_starts, ((size_t)p->bucket_most + 1) * 4);
        if (p->shares) take(&p->off_units, ((size_t)p->bucket_most + 1) * 4);
        take(&p->off_rep, (size_t)p->bucket_most * 4);
        take(&p->off_lb, BkLookback::bytes(p->unit_most, p->shares));
        take(&p->off_rec, (size_t)p->word_most * 4);
        take(&p->off_cells, (size_t)p->cell_most * 4);
        // the lists of shared buckets over the counts, which are done with by then, if they fit
        const size_t with_list = tmax(off, p->off_cells + align_up((size_t)total_slots * 4));
        p->off_list = 0;
        if (p->shares && with_list <= limit) {
            off = with_list;
            p->off_list = p->off_cells;
        }
        p->total = off;
        p->on = off <= limit && p->scan_most <= INT32_MAX && p->entries <= INT32_MAX && p->cell_most <= UINT32_MAX &&
                p->word_most / 2 <= UINT32_MAX;
    }
}

hipError_t run_batch_buckets(const BkBatchPlan& p, const int32_t* conn, const mesh_segment* segs,
                             int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap, int32_t* elem_row_ptr,
                             int32_t* elem_cols, int64_t elem_cap, void* ws, hipStream_t s) {
    char* w = (char*)ws;
    uint32_t* hdr = (uint32_t*)w;
    SetupArgs a{};
    a.segs = segs;
    a.n_mesh = p.n_mesh;
    a.total_vert = p.total_vert;
    a.max_vert = p.max_vert;
    a.total_slots = p.total_slots;
    a.total_pairs = p.total_pairs;
    for (int K = 2; K <= 4; ++K) {
        a.fill[K] = p.fill[K];
        a.vmax[K] = bk_size(K, p.large).vmax;
    }
    a.nb_most = p.nb_most;
    a.tile_slots = p.tile_slots;
    a.mesh = (BkMesh*)(w + p.off_mesh);
    a.tile0 = (uint32_t*)(w + p.off_tile0);
    a.scan0 = (uint32_t*)(w + p.off_scan0);
    a.hdr = hdr;
    const BkMesh* mesh = a.mesh;
    const int entries = (int)p.entries;
    uint32_t* tmesh = (uint32_t*)(w + p.off_tmesh);
    uint32_t* cells = (uint32_t*)(w + p.off_cells);
    uint32_t* starts = (uint32_t*)(w + p.off_starts);
    uint32_t* units = p.shares ? (uint32_t*)(w + p.off_units) : nullptr;
    uint32_t* repeats = (uint32_t*)(w + p.off_rep);
    const BkLookback lookback = BkLookback::at(w + p.off_lb, p.unit_most, p.shares);
    const auto share_cap = [&](int K) { return p.shares ? (uint32_t)bk_size(K, p.large).cap : UINT32_MAX; };
    const BkbCaps caps{share_cap(2), share_cap(3), share_cap(4)};
    const auto grid = [&](int64_t per_cu) {  // a multiple of the XCDs
        return dim3((unsigned)tmin<int64_t>(ceil_div(p.tile_most, (int64_t)BK_XCDS) * BK_XCDS, per_cu * BK_CUS));
    };
    hipError_t e = launch("batch_bucket_setup", bkb_setup_kernel, dim3(1), dim3(BKB_SETUP), s, a);
    if (e == hipSuccess)
        e = launch_shm("batch_bucket_hist", bkb_hist_kernel, grid(4), dim3(BKB_BLOCK), (size_t)(p.nb_most + 1) * 4, s, conn,
                       mesh, (const uint32_t*)a.tile0, entries, tmesh, cells, hdr);
    if (e == hipSuccess)
        e = launch("batch_bucket_scan", bkb_scan_kernel, dim3((unsigned)p.scan_most), dim3(BKB_SCAN), s, mesh,
                   (const uint32_t*)a.scan0, entries, cells, starts, units, caps, (uint32_t*)(w + p.off_bmesh), lookback,
                   repeats, hdr);
    if (e == hipSuccess)
        e = launch("batch_bucket_starts", bkb_starts_kernel, dim3(1), dim3(BKB_SETUP), s, starts, units, lookback, hdr);
    if (e == hipSuccess)
        e = launch_shm("batch_bucket_part", bkb_part_kernel, grid(2), dim3(BKB_BLOCK), (size_t)BKB_LDS, s, conn, mesh,
                       (const uint32_t*)tmesh, (const uint32_t*)cells, (const uint32_t*)starts,
                       (uint32_t*)(w + p.off_rec), repeats, hdr);
    if (e != hipSuccess) return e;
    return launch_batch_bucket_rows(p, node_row_ptr, node_cols, node_cap, elem_row_ptr, elem_cols, elem_cap, w, s);
}

}  // namespace mnb
