// Vertex buckets of a mesh whose elements have their own types: the pipeline of
// buckets.hpp with tiles of elements of any type.  Every record has room for
// four neighbours (a pyramid's apex has them; other positions repeat their
// vertex, which the rows drop).
#include "bucket_path.hpp"
#include "buckets.hpp"

namespace mnb {

namespace {

// Threads, and elements, of a tile: the records (22 bytes each with their
// bucket's number, eight per element) of two small tiles fit a CU's LDS, or of
// one large one, for many buckets (longer runs of records:
// hybrid meshes of 2.0 / 3.25 / 4.0 M ids in 1012 / 1612 / 1982 buckets took 125 /
// 190 / 250 us in small tiles, 124 / 184 / 210 us in large ones).
constexpr int BKX_SMALL = 320, BKX_LARGE = 640;
constexpr uint32_t BKX_SMALL_BUCKETS = 1024;
constexpr int BKX_K = 4, BKX_W = 5;
constexpr int BKX_IDS = MAX_NPE + 1;  // words of an element's ids in the LDS (odd: no bank conflicts)

// The neighbours of every position of every type, four bits each.
struct alignas(16) BkxNbr {
    uint16_t at[MAX_NPE];
};
template <int ET>
constexpr BkxNbr bkx_nbr() {
    using E = BkElem<ET>;
    BkxNbr r{};
    for (int p = 0; p < MAX_NPE; ++p)
        for (int k = 0; k < BKX_K; ++k) {
            const int q = p < E::NPE && k < E::degree(p) ? E::nbr(p, k) : p;
            r.at[p] = (uint16_t)(r.at[p] | (q << (4 * k)));
        }
    return r;
}
static_assert(TRI3 == 0 && TET4 == 1 && HEX8 == 2 && QUAD4 == 3 && WEDGE6 == 4 && PYR5 == 5, "the table's order");
__device__ const BkxNbr BKX_NBR[N_ELEM_TYPES] = {bkx_nbr<TRI3>(),  bkx_nbr<TET4>(),   bkx_nbr<HEX8>(),
                                                 bkx_nbr<QUAD4>(), bkx_nbr<WEDGE6>(), bkx_nbr<PYR5>()};

struct MixedConn {
    const int32_t* conn;
    const int32_t* elem_off;
    const uint8_t* etypes;
    int64_t n_elem, n_ids;
};
// The ids of element e and their number: 0 for none, or an element that is not
// well-formed (*odd).  No id is below n_vert where there is none.
__device__ __forceinline__ int bkx_load(const MixedConn& c, int64_t e, int32_t (&id)[MAX_NPE], uint32_t* type, bool* odd) {
    int npe = 0;
    int64_t a = 0;
    *type = 0;
    if (e < c.n_elem) {
        a = c.elem_off[e];
        const int64_t b = c.elem_off[e + 1];
        *type = c.etypes[e];
        npe = nodes_per_elem((int32_t)*type);
        if (npe == 0 || a < 0 || b - a != npe || b > c.n_ids) {
            *odd = true;
            npe = 0;
        }
    }
#pragma unroll
    for (int j = 0; j < MAX_NPE; ++j) id[j] = j < npe ? c.conn[a + j] : -1;
    return npe;
}

// As bk_hist, a thread per element.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void bkx_hist_kernel(MixedConn c, BkMap mp, int64_t n_tiles, int R,
                                                            uint16_t* __restrict__ within, uint32_t* __restrict__ btot,
                                                            uint32_t* __restrict__ flags, uint64_t* __restrict__ scan_lb,
                                                            int n_scan, uint32_t* __restrict__ hdr) {
    extern __shared__ uint32_t s_h[];  // nb_pad counts
    __shared__ uint32_t s_flags;
    const int tid = threadIdx.x;
    const int nb = (int)mp.nb_pad;
    for (int i = tid; i < nb; i += BLOCK) s_h[i] = 0;
    if (tid == 0) s_flags = 0;
    if (blockIdx.x == 0) {  // what the later kernels need at zero
        if (tid < (int)(HEADER_BYTES / 4)) hdr[tid] = 0;
        for (int i = tid; i < n_scan; i += BLOCK) scan_lb[i] = 0;
    }
    __syncthreads();
    uint32_t found = 0;
    const int64_t x = blockIdx.x % BK_XCDS, k = blockIdx.x / BK_XCDS;
    for (int r = 0; r < R; ++r) {
        const int64_t t = x + BK_XCDS * (R * k + r);
        if (t >= n_tiles) break;
        int32_t id[MAX_NPE];
        uint32_t type;
        bool odd = false;
        const int npe = bkx_load(c, t * BLOCK + tid, id, &type, &odd);
        if (odd) found |= BK_BAD_ID;
        uint32_t* wt = reinterpret_cast<uint32_t*>(within + t * nb);  // two counts per word (nb is even)
        for (int i = tid; i < nb / 2; i += BLOCK) wt[i] = s_h[2 * i] | (s_h[2 * i + 1] << 16);
        __syncthreads();
        const bool crowded = bk_crowded(bk_bucket((uint32_t)id[0], mp.mul));
#pragma unroll
        for (int j = 0; j < MAX_NPE; ++j) {
            const uint32_t v = (uint32_t)id[j];
            const bool ok = v < (uint32_t)mp.n_vert;
            if (j < npe && !ok) found |= BK_BAD_ID;
#pragma unroll
            for (int jj = 0; jj < j; ++jj)
                if (ok && (uint32_t)id[jj] == v) found |= BK_HAS_DUP;
            bk_count(s_h, ok ? bk_bucket(v, mp.mul) : 0u, ok, crowded);
        }
        __syncthreads();
    }
    if (found) atomicOr(&s_flags, found);
    for (int i = tid; i < nb; i += BLOCK) btot[(int64_t)blockIdx.x * nb + i] = s_h[i];
    __syncthreads();
    if (tid == 0) flags[blockIdx.x] = s_flags;
}

size_t bkx_part_lds(int block, uint32_t nb_pad) {
    return (size_t)nb_pad * 8 + (size_t)block * (MAX_NPE * (4 * BKX_W + 2) + 4 * BKX_IDS);
}

// As bk_part, a thread per element: its ids go through the LDS, where a
// position's neighbours are looked up by the element's type.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void bkx_part_kernel(MixedConn c, BkMap mp, int R,
                                                            const uint16_t* __restrict__ within,
                                                            const uint32_t* __restrict__ btot,
                                                            const uint32_t* __restrict__ starts,
                                                            uint32_t* __restrict__ rec, uint32_t* repeats, uint32_t* hdr) {
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_tmp[BLOCK / WAVE];
    const int nb = (int)mp.nb_pad, tid = threadIdx.x;
    uint32_t* const s_cnt = s_dyn;        // counts, then offsets
    uint32_t* const s_glob = s_dyn + nb;  // where the bucket's first record goes, less its offset
    uint32_t* const s_ids = s_glob + nb + tid * BKX_IDS;
    uint32_t* const s_rec = s_glob + nb + BLOCK * BKX_IDS;
    uint16_t* const s_b = reinterpret_cast<uint16_t*>(s_rec + BLOCK * MAX_NPE * BKX_W);
    const uint32_t odd = hdr[HDR_BK_ODD];
    const int64_t t = blockIdx.x, e = t * BLOCK + tid;
    const int64_t h = (t / BK_XCDS / R) * BK_XCDS + t % BK_XCDS;
    int32_t id[MAX_NPE];
    uint32_t type;
    bool ill = false;
    bkx_load(c, e, id, &type, &ill);
    const BkxNbr nbr = BKX_NBR[type < N_ELEM_TYPES ? type : 0];
    for (int i = tid; i < nb; i += BLOCK) {
        s_cnt[i] = 0;
        s_glob[i] = i < (int)mp.n_bucket ? starts[i] + btot[h * nb + i] + within[t * nb + i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < MAX_NPE; ++j) s_ids[j] = (uint32_t)id[j];
    __syncthreads();
    uint32_t place[MAX_NPE / 2] = {};  // two 16-bit places per word
    const bool crowded = bk_crowded(bk_bucket((uint32_t)id[0], mp.mul));
#pragma unroll
    for (int j = 0; j < MAX_NPE; ++j) {
        const uint32_t v = (uint32_t)id[j];
        const bool ok = v < (uint32_t)mp.n_vert;
        place[j / 2] |= bk_count(s_cnt, ok ? bk_bucket(v, mp.mul) : 0u, ok, crowded) << (16 * (j & 1));
    }
    const uint32_t total = bk_tile_offsets<BLOCK>(s_cnt, s_glob, nb, s_tmp);
#pragma unroll
    for (int j = 0; j < MAX_NPE; ++j) {
        const uint32_t v = (uint32_t)id[j];
        if (v >= (uint32_t)mp.n_vert) continue;
        const uint32_t b = bk_bucket(v, mp.mul);
        const uint32_t p = s_cnt[b] + ((place[j / 2] >> (16 * (j & 1))) & 0xffffu);
        if (odd & BK_HAS_DUP) {  // (seldom: some element of the mesh repeats an id)
            bool again = false;
#pragma unroll
            for (int jj = 0; jj < j; ++jj) again |= (uint32_t)id[jj] == v;
            if (again) atomicAdd(&repeats[b], 1u);
        }
        uint32_t n[BKX_K];
#pragma unroll
        for (int k = 0; k < BKX_K; ++k) {
            const uint32_t w = s_ids[(nbr.at[j] >> (4 * k)) & 15];
            n[k] = w < (uint32_t)mp.n_vert ? w : v;
        }
        uint32_t r[BKX_W];
        bk_encode<BKX_K, BKX_W>(mp, (uint32_t)e, v, n, r);
#pragma unroll
        for (int q = 0; q < BKX_W; ++q) s_rec[p * BKX_W + q] = r[q];
        s_b[p] = (uint16_t)b;
    }
    __syncthreads();
    if (!bk_tile_out<BKX_W, BLOCK>(s_rec, s_b, s_glob, total, rec, c.n_ids) && !(odd & BK_BAD_ID))
        set_error(hdr + HDR_ERR, ERR_INTERNAL);
}

}  // namespace

void plan_mixed_buckets(int64_t n_elem, int64_t n_ids, int32_t n_vert, const Opts& o, size_t limit, BkPlan* p) {
    *p = BkPlan{};
    // (32-bit sums of up to eight records per element)
    if (!o.library || n_elem > UINT32_MAX / MAX_NPE || !plan_bucket_map(n_elem, n_ids, n_vert, BKX_K, BK_FULL_MIXED, p)) return;
    if (p->W != BKX_W) return;
    p->large_tile = p->mp.nb_pad > BKX_SMALL_BUCKETS && bkx_part_lds(BKX_LARGE, p->mp.nb_pad) <= (size_t)BK_LDS - 256;
    const int block = p->large_tile ? BKX_LARGE : BKX_SMALL;
    if (bkx_part_lds(block, p->mp.nb_pad) > (size_t)BK_LDS - 256) return;
    plan_bucket_layout(block, MAX_NPE, limit, p);
}

hipError_t run_mixed_buckets(const BkPlan& p, const int32_t* conn, const int32_t* elem_off, const uint8_t* etypes,
                             int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap, int32_t* elem_row_ptr,
                             int32_t* elem_cols, int64_t elem_cap, void* ws, hipStream_t s) {
    char* w = (char*)ws;
    uint32_t* hdr = (uint32_t*)w;
    const MixedConn c{conn, elem_off, etypes, p.n_elem, p.n_slots};
    uint16_t* within = (uint16_t*)(w + p.off_within);
    uint32_t* btot = (uint32_t*)(w + p.off_btot);
    uint32_t* flags = (uint32_t*)(w + p.off_flags);
    uint64_t* scan_lb = (uint64_t*)(w + p.off_scan);
    uint32_t* starts = (uint32_t*)(w + p.off_starts);
    uint32_t* repeats = (uint32_t*)(w + p.off_rep);
    const int n_scan = (int)ceil_div(p.mp.n_bucket, BKS_COLS);
    auto tiles = [&](auto block) {
        constexpr int BLOCK = decltype(block)::value;
        hipError_t e = launch_shm("mixed_bucket_hist", bkx_hist_kernel<BLOCK>, dim3(p.hist_blocks), dim3(BLOCK),
                                  (size_t)p.mp.nb_pad * 4, s, c, p.mp, p.n_tiles, p.R, within, btot, flags, scan_lb, n_scan, hdr);
        if (e == hipSuccess)
            e = launch("bucket_scan", bk_scan_kernel, dim3((unsigned)n_scan), dim3(BKS_BLOCK), s, btot, p.hist_blocks,
                       p.mp.n_bucket, p.mp.nb_pad, (const uint32_t*)flags, scan_lb, starts, bk_units(p, w),
                       bk_share_cap(p), (uint32_t)p.n_slots, bk_lookback(p, w), repeats, hdr);
        if (e == hipSuccess)
            e = launch_shm("mixed_bucket_part", bkx_part_kernel<BLOCK>, dim3((unsigned)p.n_tiles), dim3(BLOCK),
                           bkx_part_lds(BLOCK, p.mp.nb_pad), s, c, p.mp, p.R, (const uint16_t*)within,
                           (const uint32_t*)btot, (const uint32_t*)starts, (uint32_t*)(w + p.off_rec), repeats, hdr);
        return e;
    };
    const hipError_t e = p.large_tile ? tiles(std::integral_constant<int, BKX_LARGE>{}) : tiles(std::integral_constant<int, BKX_SMALL>{});
    if (e != hipSuccess) return e;
    return launch_bucket_rows(p, node_row_ptr, node_cols, node_cap, elem_row_ptr, elem_cols, elem_cap, w, s);
}

}  // namespace mnb
