// The rows kernel of the vertex-bucket pipeline (bucket_rows.hpp), for every
// number of neighbours and both bucket sizes.
#include "bucket_path.hpp"
#include "bucket_rows.hpp"

namespace mnb {

namespace {

template <class F>
decltype(auto) with_shape(int K, bool large, F&& f) {
    auto pick = [&](auto k) -> decltype(auto) {
        return large ? f(k, std::integral_constant<bool, true>{}) : f(k, std::integral_constant<bool, false>{});
    };
    switch (K) {
        case 2: return pick(std::integral_constant<int, 2>{});
        case 3: return pick(std::integral_constant<int, 3>{});
        case 4: return pick(std::integral_constant<int, 4>{});
        default: return pick(std::integral_constant<int, 0>{});
    }
}

}  // namespace

BkSize bk_size(int K, bool large) {
    return with_shape(K, large, [](auto k, auto l) {
        constexpr int K = decltype(k)::value;
        using S = BkShape<K, decltype(l)::value>;
        static_assert((K > 0 ? K : 1) * S::CAP <= S::POOL && S::POOL < 65536, "a full bucket fits the pool; 16-bit places");
        static_assert(S::POOL % (2 * (S::BLOCK / WAVE)) == 0, "a wave's part of a bit map is whole 64-bit words");
        return BkSize{S::CAP, S::VMAX};
    });
}

hipError_t launch_bucket_rows(const BkPlan& p, int32_t* node_row_ptr, int32_t* node_cols, int64_t node_cap,
                              int32_t* elem_row_ptr, int32_t* elem_cols, int64_t elem_cap, char* w, hipStream_t s) {
    const BkRowsArgs a{p.mp, (const uint32_t*)(w + p.off_rec), (const uint32_t*)(w + p.off_starts),
                       bk_units(p, w), (const uint32_t*)(w + p.off_rep), bk_lookback(p, w),
                       p.off_list ? (uint32_t*)(w + p.off_list) : nullptr, (uint32_t*)w, node_row_ptr, node_cols, node_cols ? node_cap : 0,
                       elem_row_ptr, elem_cols, elem_cols ? elem_cap : 0, p.n_elem};
    return with_shape(p.K, p.large, [&](auto k, auto l) {
        constexpr int K = decltype(k)::value;
        constexpr bool L = decltype(l)::value;
        const dim3 grid(p.mp.n_bucket), block(BkShape<K, L>::BLOCK);
        if constexpr (K == 0) {
            return p.W == 1 ? launch("bucket_rows", bk_rows_kernel<0, 1, L>, grid, block, s, a)
                            : launch("bucket_rows", bk_rows_kernel<0, 2, L>, grid, block, s, a);
        } else {
            if constexpr (K < 4) {
                if (p.W == K) return launch("bucket_rows", bk_rows_kernel<K, K, L>, grid, block, s, a);
            }
            return launch("bucket_rows", bk_rows_kernel<K, K + 1, L>, grid, block, s, a);
        }
    });
}

}  // namespace mnb
