// Host side of the vertex-bucket pipeline (buckets.hpp): when it applies, its
// sizes, and its launches up to the rows (bucket_rows.hip).
#include "buckets.hpp"
#include "bucket_path.hpp"

namespace mnb {

namespace {

// Elements per tile and records per tile of a type's tile shapes.
template <int ET>
constexpr int tile_elems(bool large) {
    return large ? BkTile<ET>::BLOCK * BkTile<ET>::EPT : BK_SMALL_BLOCK;
}

int bk_neighbours(int32_t etype) {
    return with_type(etype, [](auto et) { return BkElem<decltype(et)::value>::K; });
}

uint32_t pow2_bits(uint64_t n) {  // smallest b with 2^b >= n
    uint32_t b = 0;
    while (((uint64_t)1 << b) < n) ++b;
    return b;
}

size_t part_lds(int npe, int W, int64_t elems, uint32_t nb_pad) {
    return (size_t)elems * npe * (4 * W + 2) + (size_t)nb_pad * 8 + 256;
}

}  // namespace

bool plan_bucket_map(int64_t n_elem, int64_t n_slots, int32_t n_vert, int K, int full, BkPlan* p) {
    if (n_slots < 1 || n_elem < 1 || n_vert < 1) return false;
    // rows much longer than any mesh's go to the sorts: the networks take 32 values at
    // a time (tetrahedra average 24 elements)
    if (n_slots > (int64_t)BK_MAX_DEGREE * n_vert) return false;
    p->n_elem = n_elem;
    p->n_slots = n_slots;
    p->K = K;
    BkMap& m = p->mp;
    m.n_vert = n_vert;
    m.e_bits = bits_for_count(n_elem);
    m.id_bits = id_bits_for(n_vert);
    // buckets: small ones while a few rounds of them fill the GPU, then large
    // ones (fewer runs in the partition)
    int64_t nb = 0;
    int vmax = 0;
    for (int large = 0; large < 2; ++large) {
        const BkSize z = bk_size(p->K, large != 0);
        nb = tmax<int64_t>(ceil_div(n_slots * 100, (int64_t)z.cap * full), ceil_div(n_vert, z.vmax - 2));
        vmax = z.vmax;
        p->large = large != 0;
        if (nb <= BK_SMALL_MOST) break;
    }
    if (!p->large) {
        // a small mesh still spreads over the CUs
        nb = tmax<int64_t>(nb, tmin<int64_t>(BK_CUS, ceil_div(n_slots, BK_LEAST_RECORDS)));
    } else {
        // two large blocks per CU at a time: whole rounds, of equal buckets
        if (full != BK_FULL_MIXED || nb < 2 * BK_CUS) nb = ceil_div(nb, 2 * BK_CUS) * (2 * BK_CUS);
    }
    const int64_t width = tmax<int64_t>(ceil_div(n_vert, nb), 2);
    m.mul = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)width);
    m.n_bucket = (uint32_t)(((uint64_t)(n_vert - 1) * m.mul) >> 32) + 1;
    m.nb_pad = (m.n_bucket + 1) & ~1u;
    const uint64_t widest = (((uint64_t)1 << 32) + m.mul - 1) / m.mul;
    if ((int64_t)widest > vmax) return false;
    const uint32_t vl_bits = pow2_bits(widest);
    m.vl_mask = (1u << vl_bits) - 1;
    p->W = bk_words(p->K, m.e_bits, m.id_bits, vl_bits);
    m.e_shift = 2 * m.id_bits + vl_bits;
    return p->W != 0;
}

void plan_bucket_layout(int64_t tile_elems, int most_npe, size_t limit, BkPlan* p) {
    const BkMap& m = p->mp;
    p->n_tiles = ceil_div(p->n_elem, tile_elems);
    const int64_t r_most = 65535 / (tile_elems * most_npe);  // 16-bit counts before a tile
    p->R = (int)tmax<int64_t>(1, tmin<int64_t>(ceil_div(p->n_tiles, BK_HIST_BLOCKS), r_most));
    const int64_t blocks = BK_XCDS * ceil_div(p->n_tiles, (int64_t)BK_XCDS * p->R);
    if (blocks > BK_HIST_MOST) return;
    p->hist_blocks = (int)blocks;
    for (int shares = 1; shares >= 0 && !p->on; --shares) {
        p->shares = shares != 0;
        size_t off = HEADER_BYTES;
        auto take = [&](size_t* at, size_t bytes) {
            *at = off;
            off += align_up(bytes);
        };
        take(&p->off_flags, (size_t)p->hist_blocks * sizeof(uint32_t));
        take(&p->off_scan, (size_t)ceil_div(m.n_bucket, BKS_COLS) * sizeof(uint64_t));
        take(&p->off_starts, ((size_t)m.n_bucket + 1) * sizeof(uint32_t));
        if (p->shares) take(&p->off_units, ((size_t)m.n_bucket + 1) * sizeof(uint32_t));
        take(&p->off_rep, (size_t)m.n_bucket * sizeof(uint32_t));
        p->unit_most = p->shares ? bk_unit_most(m.n_bucket, p->n_elem * most_npe, bk_size(p->K, p->large).cap) : m.n_bucket;
        take(&p->off_lb, BkLookback::bytes(p->unit_most, p->shares));
        take(&p->off_rec, ((size_t)p->n_slots + 1) * p->W * sizeof(uint32_t));  // (an empty last bucket reads one past)
        take(&p->off_btot, (size_t)p->hist_blocks * m.nb_pad * sizeof(uint32_t));
        take(&p->off_within, (size_t)p->n_tiles * m.nb_pad * sizeof(uint16_t));
        // the lists of shared buckets over the counts, which are done with by then, if they fit
        const size_t with_list = tmax(off, p->off_btot + align_up((size_t)p->n_slots * sizeof(uint32_t)));
        p->off_list = 0;
        if (p->shares && with_list <= limit) {
            p->off_list = p->off_btot;
            off = with_list;
        }
        p->total = off;
        p->on = off <= limit;
    }
}

void plan_buckets(int64_t n_elem, int32_t etype, int32_t n_vert, const Opts& o, bool node, size_t limit, BkPlan* p) {
    *p = BkPlan{};
    const int npe = nodes_per_elem(etype);
    if (!o.library || !plan_bucket_map(n_elem, (int64_t)npe * n_elem, n_vert, node ? bk_neighbours(etype) : 0, bk_full(etype), p))
        return;
    p->etype = etype;
    // tiles: large ones once they occupy every CU
    const int64_t big = with_type(etype, [](auto et) { return (int64_t)tile_elems<decltype(et)::value>(true); });
    p->large_tile = n_elem >= big * BK_CUS && part_lds(npe, p->W, big, p->mp.nb_pad) <= (size_t)BK_LDS;
    if (!p->large_tile && n_elem >= big * BK_CUS && p->mp.n_bucket > BK_SMALL_TILE_MOST) return;
    const int64_t te = p->large_tile ? big : BK_SMALL_BLOCK;
    if (part_lds(npe, p->W, te, p->mp.nb_pad) > (size_t)BK_LDS) return;
    plan_bucket_layout(te, npe, limit, p);
}

namespace {

template <int ET, int K, int W, bool LT>
hipError_t launch_part(const BkPlan& p, const int32_t* conn, char* w, hipStream_t s) {
    constexpr int BLOCK = LT ? BkTile<ET>::BLOCK : BK_SMALL_BLOCK, EPT = LT ? BkTile<ET>::EPT : 1;
    const size_t shm = part_lds(Elem<ET>::NPE, W, BLOCK * EPT, p.mp.nb_pad) - 256;
    return launch_shm("bucket_part", bk_part_kernel<ET, K, W, BLOCK, EPT>, dim3((unsigned)p.n_tiles), dim3(BLOCK), shm, s,
                      conn, p.n_elem, p.mp, p.R, (const uint16_t*)(w + p.off_within), (const uint32_t*)(w + p.off_btot),
                      (const uint32_t*)(w + p.off_starts), (uint32_t*)(w + p.off_rec), p.n_slots,
                      (uint32_t*)(w + p.off_rep), (uint32_t*)w);
}

template <int ET, bool LT>
hipError_t launch_tiles(const BkPlan& p, const int32_t* conn, char* w, hipStream_t s) {
    constexpr int BLOCK = LT ? BkTile<ET>::BLOCK : BK_SMALL_BLOCK, EPT = LT ? BkTile<ET>::EPT : 1;
    uint32_t* hdr = (uint32_t*)w;
    uint32_t* btot = (uint32_t*)(w + p.off_btot);
    uint32_t* flags = (uint32_t*)(w + p.off_flags);
    hipError_t e = launch_shm("bucket_hist", bk_hist_kernel<ET, BLOCK, EPT>, dim3(p.hist_blocks), dim3(BLOCK),
                              (size_t)p.mp.nb_pad * 4, s, conn, p.n_elem, p.mp, p.n_tiles, p.R,
                              (uint16_t*)(w + p.off_within), btot, flags, (uint64_t*)(w + p.off_scan),
                              (int)ceil_div(p.mp.n_bucket, BKS_COLS), hdr);
    if (e == hipSuccess)
        e = launch("bucket_scan", bk_scan_kernel, dim3((unsigned)ceil_div(p.mp.n_bucket, BKS_COLS)), dim3(BKS_BLOCK), s,
                   btot, p.hist_blocks, p.mp.n_bucket, p.mp.nb_pad, (const uint32_t*)flags,
                   (uint64_t*)(w + p.off_scan), (uint32_t*)(w + p.off_starts), bk_units(p, w),
                   bk_share_cap(p), (uint32_t)p.n_slots, bk_lookback(p, w), (uint32_t*)(w + p.off_rep), hdr);
    if (e != hipSuccess) return e;
    if (p.K == 0)
        return p.W == 1 ? launch_part<ET, 0, 1, LT>(p, conn, w, s) : launch_part<ET, 0, 2, LT>(p, conn, w, s);
    constexpr int K = BkElem<ET>::K;
    if constexpr (K < 4) {
        if (p.W == K) return launch_part<ET, K, K, LT>(p, conn, w, s);
    }
    return launch_part<ET, K, K + 1, LT>(p, conn, w, s);
}

}  // namespace

hipError_t run_buckets(const BkPlan& p, const int32_t* conn, int32_t* node_row_ptr, int32_t* node_cols,
                       int64_t node_cap, int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, void* ws,
                       hipStream_t s) {
    char* w = (char*)ws;
    hipError_t e = with_type(p.etype, [&](auto et) {
        constexpr int ET = decltype(et)::value;
        return p.large_tile ? launch_tiles<ET, true>(p, conn, w, s) : launch_tiles<ET, false>(p, conn, w, s);
    });
    if (e != hipSuccess) return e;
    return launch_bucket_rows(p, node_row_ptr, node_cols, node_cap, elem_row_ptr, elem_cols, elem_cap, w, s);
}

}  // namespace mnb
