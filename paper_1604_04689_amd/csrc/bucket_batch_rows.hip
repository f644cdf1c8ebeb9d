// The rows kernel of a batch's vertex buckets: the buckets of meshes of every
// type in one launch, so that one chain of sums gives all node rows their
// places.
#include "bucket_batch.hpp"
#include "bucket_rows.hpp"

namespace mnb {

namespace {

template <bool LARGE>
constexpr int batch_lds_words() {
    const int w2 = BkLds<2, LARGE>::WORDS, w3 = BkLds<3, LARGE>::WORDS, w4 = BkLds<4, LARGE>::WORDS;
    return tmax(w2, tmax(w3, w4));
}

// A block takes units in turn, by ticket, and each by the code for its
// mesh's element type.  (A grid that fills the GPU once: the number of buckets
// is known on the device alone.)
template <bool LARGE>
__global__ __launch_bounds__((BkShape<2, LARGE>::BLOCK)) __attribute__((amdgpu_waves_per_eu(4)))
void bk_batch_rows_kernel(BkRowsArgs all, const BkMesh* __restrict__ mesh, const uint32_t* __restrict__ bmesh) {
    constexpr int BLOCK = BkShape<2, LARGE>::BLOCK;
    static_assert(BkShape<3, LARGE>::BLOCK == BLOCK && BkShape<4, LARGE>::BLOCK == BLOCK, "one block size");
    __shared__ __align__(16) uint32_t s_all[batch_lds_words<LARGE>()];
    __shared__ uint32_t s_tmp[2 * (BLOCK / WAVE)];
    __shared__ uint32_t s_ticket;
    __shared__ uint64_t s_base;
    const uint32_t n_bucket = (uint32_t)__builtin_amdgcn_readfirstlane((int)all.hdr[HDR_BKB_BUCKETS]);
    const uint32_t odd = (uint32_t)__builtin_amdgcn_readfirstlane((int)all.hdr[HDR_BK_ODD]);
    const uint32_t n_unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)all.hdr[HDR_BK_UNITS]);
    while (true) {
        if (threadIdx.x == 0) s_ticket = atomicAdd(&all.hdr[HDR_BK_TICKET], 1u);
        __syncthreads();
        const uint32_t ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_ticket);
        if (ticket >= n_unit) return;
        const BkUnit u = bk_unit_of(ticket, n_unit, n_bucket, all.units);
        const uint32_t bucket = u.bucket;
        const BkMesh& m = mesh[__builtin_amdgcn_readfirstlane((int)bmesh[bucket])];
        BkRowsArgs a = all;
        a.mp = m.mp;
        a.n_elem = m.n_elem;
        a.rec = all.rec + m.rec0;
        a.nrp = all.nrp + m.vert_off;
        if (all.erp) a.erp = all.erp + m.vert_off;
        const uint32_t b = bucket - m.bucket0;
        const uint32_t lo = bk_first_vertex(b, m.mp.mul);
        const uint32_t hi = b + 1 == m.mp.n_bucket ? (uint32_t)m.mp.n_vert : bk_next_first_vertex(lo, b, m.mp.mul);
        const uint32_t r0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)all.starts[bucket]);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)all.starts[bucket + 1]) - r0;
        const uint32_t rec0 = r0 - (uint32_t)__builtin_amdgcn_readfirstlane((int)all.starts[m.bucket0]);
        const int nv = (int)(hi - lo);
        const int form = 8 * (m.etype == TRI3 || m.etype == QUAD4 ? 2 : m.etype == PYR5 ? 4 : 3) + m.W;
        auto rows = [&](auto k, auto w) BK_INLINE {
            bk_unit_rows<decltype(k)::value, decltype(w)::value, LARGE>(a, u, rec0, n, r0, lo, nv, odd, s_all, s_tmp, &s_base);
        };
        using std::integral_constant;
        switch (form) {
            case 8 * 2 + 2: rows(integral_constant<int, 2>{}, integral_constant<int, 2>{}); break;
            case 8 * 2 + 3: rows(integral_constant<int, 2>{}, integral_constant<int, 3>{}); break;
            case 8 * 3 + 3: rows(integral_constant<int, 3>{}, integral_constant<int, 3>{}); break;
            case 8 * 3 + 4: rows(integral_constant<int, 3>{}, integral_constant<int, 4>{}); break;
            default: rows(integral_constant<int, 4>{}, integral_constant<int, 5>{}); break;
        }
        __syncthreads();  // before the LDS is used again
    }
}

}  // namespace

hipError_t launch_batch_bucket_rows(const BkBatchPlan& p, int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap,
                                    int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, char* w, hipStream_t s) {
    const BkRowsArgs a{BkMap{}, (const uint32_t*)(w + p.off_rec), (const uint32_t*)(w + p.off_starts),
                       p.shares ? (const uint32_t*)(w + p.off_units) : nullptr, (const uint32_t*)(w + p.off_rep),
                       BkLookback::at(w + p.off_lb, p.unit_most, p.shares),
                       p.off_list ? (uint32_t*)(w + p.off_list) : nullptr, (uint32_t*)w, node_row_ptr, node_cols,
                       node_cols ? node_cap : 0, elem_row_ptr, elem_cols, elem_cols ? elem_cap : 0, 0};
    const BkMesh* mesh = (const BkMesh*)(w + p.off_mesh);
    const uint32_t* bmesh = (const uint32_t*)(w + p.off_bmesh);
    // two large blocks fit a CU's LDS, four small ones
    if (p.large)
        return launch("batch_bucket_rows", bk_batch_rows_kernel<true>, dim3((unsigned)tmin<int64_t>(p.bucket_most, 2 * BK_CUS)),
                      dim3(BkShape<2, true>::BLOCK), s, a, mesh, bmesh);
    return launch("batch_bucket_rows", bk_batch_rows_kernel<false>, dim3((unsigned)tmin<int64_t>(p.bucket_most, 4 * BK_CUS)),
                  dim3(BkShape<2, false>::BLOCK), s, a, mesh, bmesh);
}

}  // namespace mnb
