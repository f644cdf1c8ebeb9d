// Vertex buckets, second half: one block turns a bucket's records into the
// rows of its vertices in both CSRs (buckets.hpp has the overview).
//
// The block counts each vertex's records (LDS adds), scans the counts into
// row starts and puts every record's neighbours at its row.  Then a thread
// takes a row: up to 32 of its values are sorted in registers by a Batcher
// network (8, 16, 24 or 32 wide, what the wave's longest row needs), repeats
// drop out, and what is left is sorted with the next values, until the row is
// used up (a tetrahedral row's 72 values, 14 of them distinct, take four
// rounds).  The distinct counts are scanned, and the rows go from the
// registers straight to their place among the bucket's rows, packed, over
// values already read.  The element rows follow in the place the neighbours
// left.  A network needs about a third of an instruction per value and lane
// group where ranking by counting needs ten times that, it has no dependent
// LDS reads and no divergence; hash tables in LDS for the tetrahedral rows
// took three times as long (atomics with return, one dependent probe after
// another).
//
// Where a bucket's element rows start is known beforehand (its records are
// its pairs, less the repeats that bk_part counted).  Where its node rows
// start is the sum of the earlier buckets' distinct neighbours, found by a
// decoupled look-back.  A block announces its sum before it orders and writes
// its element rows, so that the answer is usually there when it asks.
//
// What the registers do not take is done from the records in memory again
// (bk_ranges): a bucket with a row of more than 64 distinct neighbours, and one
// with more records than the LDS holds, which an uneven mesh has.  Several
// blocks share the latter: each has its own place in the look-back and takes a
// run of the bucket's vertices, in ranges that fit the LDS, first to count and
// then to write; a single row longer than the LDS is done in bit maps of a
// window of ids at a time, the windows dealt to the shares that the row spans.
#pragma once

#include <utility>

#include "buckets.hpp"

namespace mnb {

// Lambdas that see register arrays go in before anything else is optimised:
// code shared by two of them would otherwise be merged through memory.
#define BK_INLINE __attribute__((always_inline))

// The thread's number in its block, afresh: what follows from it is not kept
// from one unit of a block for the next, in registers that the rows need.
__device__ __forceinline__ int bk_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ---- sorting -----------------------------------------------------------------
// Batcher's odd-even merge sort of N values, any N: its comparators in order.
template <int N>
struct BkNet {
    static constexpr int count() {
        int c = 0;
        for (int p = 1; p < N; p *= 2)
            for (int k = p; k >= 1; k /= 2)
                for (int j = k % p; j + k < N; j += 2 * k)
                    for (int i = 0; i < k && i + j + k < N; ++i)
                        if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) ++c;
        return c;
    }
    static constexpr int C = count();
    struct List {
        int lo[C], hi[C];
    };
    static constexpr List list() {
        List l{};
        int c = 0;
        for (int p = 1; p < N; p *= 2)
            for (int k = p; k >= 1; k /= 2)
                for (int j = k % p; j + k < N; j += 2 * k)
                    for (int i = 0; i < k && i + j + k < N; ++i)
                        if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                            l.lo[c] = i + j;
                            l.hi[c] = i + j + k;
                            ++c;
                        }
        return l;
    }
    static constexpr List L = list();
};
// f(0) .. f(N - 1), each index a constant (no loop for the compiler to unroll,
// so that arrays indexed by it are registers from the start).
template <class F, int... I>
__device__ __forceinline__ void bk_each(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void bk_each(F&& f) {
    bk_each(std::make_integer_sequence<int, N>{}, f);
}

// The len values at a, sorted (BK_EMPTY after them; reads may run past the
// row, into other rows or the array's padding).
template <int N, int M>
__device__ __forceinline__ void bk_row_load(const uint32_t* a, uint32_t len, uint32_t (&x)[M]) {
    bk_each<N>([&](auto ii) BK_INLINE {
        constexpr int i = decltype(ii)::value;
        x[i] = a[i];
    });
    if (__ballot(len < (uint32_t)N))  // (not in the full windows of long rows)
        bk_each<N>([&](auto ii) BK_INLINE {
            constexpr int i = decltype(ii)::value;
            if ((uint32_t)i >= len) x[i] = BK_EMPTY;
        });
    bk_each<BkNet<N>::C>([&](auto cc) BK_INLINE {
        constexpr int i = BkNet<N>::L.lo[decltype(cc)::value], j = BkNet<N>::L.hi[decltype(cc)::value];
        const uint32_t u = x[i], v = x[j];
        x[i] = min(u, v);
        x[j] = max(u, v);
    });
}
template <int N, int M>
__device__ __forceinline__ uint32_t bk_row_count(const uint32_t (&x)[M]) {
    uint32_t c = x[0] != BK_EMPTY ? 1u : 0u;
    bk_each<N - 1>([&](auto ii) BK_INLINE {
        constexpr int i = decltype(ii)::value + 1;
        c += x[i] != x[i - 1] && x[i] != BK_EMPTY ? 1u : 0u;
    });
    return c;
}
// The distinct values of x to a[0 ..).  No branches: a repeat (and, at the
// end, BK_EMPTY) writes the last kept value to its place again.
template <int N, int M>
__device__ __forceinline__ void bk_row_store(const uint32_t (&x)[M], uint32_t* a) {
    uint32_t last = x[0], c = 0;
    a[0] = last;
    bk_each<N - 1>([&](auto ii) BK_INLINE {
        uint32_t v = x[decltype(ii)::value + 1];
        if (v == BK_EMPTY) v = last;
        c += v != last ? 1u : 0u;
        a[c] = v;
        last = v;
    });
}
// The distinct values of x to the places before `end`, the largest last;
// returns their number.
template <int N, int M>
__device__ __forceinline__ uint32_t bk_row_store_back(const uint32_t (&x)[M], uint32_t* end) {
    uint32_t next = BK_EMPTY, c = 0;
    bk_each<N>([&](auto ii) BK_INLINE {
        const uint32_t v = x[N - 1 - decltype(ii)::value];
        c += v != next ? 1u : 0u;
        *(end - tmax<uint32_t>(c, 1u)) = v;  // (BK_EMPTY, sorted last, is written over)
        next = v;
    });
    return c;
}
// The network that fits the longest row of the wave (at most MAX): f(size).
template <int MAX, class F>
__device__ __forceinline__ void bk_pick_network(uint32_t len, F&& f) {
    if (!__ballot(len > 8)) {
        f(std::integral_constant<int, 8>{});
    } else if (MAX == 16 || !__ballot(len > 16)) {
        f(std::integral_constant<int, 16>{});
    } else if constexpr (MAX > 16) {
        if (!__ballot(len > 24)) f(std::integral_constant<int, 24>{});
        else f(std::integral_constant<int, 32>{});
    }
}
constexpr uint32_t BK_NET_MAX = 32;

// Orders LDS writes before the following reads inside one wave.
__device__ __forceinline__ void bk_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// A wave sorts its 64 E values in registers (bitonic, E values per lane, value
// r * 64 + lane in x[r]).  Steps between lanes go in loops that are not unrolled
// where E is large: unrolled, 2048 values would take 10,000 instructions.
template <int E>
__device__ __forceinline__ void bk_wave_sort(uint32_t (&x)[E]) {
    const int lane = bk_tid() & (WAVE - 1);
    constexpr int UNROLL = E <= 4 ? 6 : 1;
    // (up: which registers' runs ascend; kept out of the loop over them)
    auto between_lanes = [&](int j, bool up_even, bool up_odd, auto odd) BK_INLINE {
        const bool low = (lane & j) == 0, even_low = up_even == low, odd_low = up_odd == low;
        bk_each<E>([&](auto rr) BK_INLINE {
            constexpr int r = decltype(rr)::value;
            const uint32_t y = (uint32_t)__shfl_xor((int)x[r], j, WAVE);
            const uint32_t lo = min(x[r], y), hi = max(x[r], y);
            x[r] = (odd(rr) ? odd_low : even_low) ? lo : hi;
        });
    };
#pragma unroll UNROLL
    for (int k = 2; k <= WAVE; k *= 2)
#pragma unroll UNROLL
        for (int j = k / 2; j > 0; j /= 2)
            between_lanes(j, (lane & k) == 0, k < WAVE && (lane & k) == 0, [](auto rr) BK_INLINE { return (decltype(rr)::value & 1) != 0; });
    auto runs = [&](auto kk) BK_INLINE {  // runs of K registers from runs of K / 2
        constexpr int K = decltype(kk)::value;
#pragma unroll
        for (int j = K / 2; j > 0; j /= 2)
            bk_each<E>([&](auto rr) BK_INLINE {
                constexpr int r = decltype(rr)::value;
                const int q = r ^ j;
                if (q > r) {
                    const uint32_t lo = min(x[r], x[q < E ? q : r]), hi = max(x[r], x[q < E ? q : r]);
                    const bool up = (r & K) == 0;
                    x[r] = up ? lo : hi;
                    x[q < E ? q : r] = up ? hi : lo;
                }
            });
#pragma unroll UNROLL
        for (int j = WAVE / 2; j > 0; j /= 2)
            between_lanes(j, true, false, [](auto rr) BK_INLINE { return (decltype(rr)::value & K) != 0; });
    };
    if constexpr (E >= 2) runs(std::integral_constant<int, 2>{});
    if constexpr (E >= 4) runs(std::integral_constant<int, 4>{});
    if constexpr (E >= 8) runs(std::integral_constant<int, 8>{});
    if constexpr (E >= 16) runs(std::integral_constant<int, 16>{});
    if constexpr (E >= 32) runs(std::integral_constant<int, 32>{});
}
template <int E>
__device__ __forceinline__ void bk_wave_load(const uint32_t* a, uint32_t n, uint32_t (&x)[E]) {
    const uint32_t lane = (uint32_t)(bk_tid() & (WAVE - 1));
    bk_each<E>([&](auto rr) BK_INLINE {
        constexpr int r = decltype(rr)::value;
        x[r] = r * WAVE + lane < n ? a[r * WAVE + lane] : BK_EMPTY;
    });
}
// A wave sorts a[0 .. n), n <= 64 E, and writes the distinct values other than
// BK_EMPTY back to the front; returns their number.  About 1.5 us for 64 values
// where the same in LDS took 10 (a round trip per step).
template <int E>
__device__ __forceinline__ uint32_t bk_wave_sort_unique(uint32_t* a, uint32_t n) {
    const uint32_t lane = (uint32_t)(bk_tid() & (WAVE - 1));
    uint32_t x[E];
    bk_wave_load(a, n, x);
    bk_wave_sort(x);
    uint32_t cnt = 0, prev = BK_EMPTY;
    bk_wave_sync();
    bk_each<E>([&](auto rr) BK_INLINE {
        constexpr int r = decltype(rr)::value;
        uint32_t left = (uint32_t)__shfl_up((int)x[r], 1, WAVE);
        if (lane == 0) left = prev;
        const bool keep = x[r] != BK_EMPTY && x[r] != left;
        const uint64_t m = __ballot(keep);
        prev = (uint32_t)__builtin_amdgcn_readlane((int)x[r], WAVE - 1);
        if (keep) a[cnt + (uint32_t)__popcll(m & ((1ull << lane) - 1))] = x[r];
        cnt += (uint32_t)__popcll(m);
    });
    bk_wave_sync();
    return cnt;
}
constexpr uint32_t BK_WAVE_ROW = 2048;  // values that a wave sorts in registers

// Every 64 E values of a[0 .. n) sorted by a wave in registers.
template <int E, int THREADS>
__device__ __forceinline__ uint32_t bk_sort_pieces(uint32_t* a, uint32_t n) {
    const uint32_t me = (uint32_t)bk_tid();
    for (uint32_t c0 = me / WAVE * (E * WAVE); c0 < n; c0 += THREADS * E) {
        uint32_t x[E];
        bk_wave_load(a + c0, n - c0, x);
        bk_wave_sort(x);
        bk_each<E>([&](auto rr) BK_INLINE {
            constexpr int r = decltype(rr)::value;
            const uint32_t i = c0 + r * WAVE + (me & (WAVE - 1));
            if (i < n) a[i] = x[r];
        });
    }
    __syncthreads();
    return E * WAVE;
}
// The block sorts a[0 .. n) in LDS, any n: pieces by the waves, in registers,
// then the rest of Batcher's network.  The first wave writes the distinct
// values other than BK_EMPTY back to the front; returns their number in its
// lanes.  (The whole network in LDS took 66 steps, about 50 us, for 2000 values.)
template <int THREADS>
__device__ __forceinline__ uint32_t bk_block_sort_unique(uint32_t* a, uint32_t n) {
    const uint32_t me = (uint32_t)bk_tid();
    for (uint32_t p = n <= 4 * THREADS ? bk_sort_pieces<4, THREADS>(a, n) : bk_sort_pieces<16, THREADS>(a, n); p < n; p *= 2) {
        for (uint32_t k = p; k >= 1; k /= 2) {
            const uint32_t j0 = k == p ? 0u : k;
            // comparator c of the step: x and x + k (k is a power of two)
            const uint32_t steps = (((n - 1) >> (__builtin_ctz(k) + 1)) + 1) * k;
            for (uint32_t c = me; c < steps; c += THREADS) {
                const uint32_t x = j0 + 2 * (c & ~(k - 1)) + (c & (k - 1));
                if (x + k < n && (x ^ (x + k)) < 2 * p) {
                    const uint32_t u = a[x], v = a[x + k];
                    if (v < u) {
                        a[x] = v;
                        a[x + k] = u;
                    }
                }
            }
            __syncthreads();
        }
    }
    uint32_t cnt = 0;
    if (bk_tid() < WAVE) {
        const uint32_t lane = (uint32_t)(bk_tid() & (WAVE - 1));
        const uint64_t lt = (1ull << lane) - 1;
        uint32_t prev = BK_EMPTY;
        for (uint32_t c0 = 0; c0 < n; c0 += WAVE) {
            const uint32_t v = c0 + lane < n ? a[c0 + lane] : BK_EMPTY;
            uint32_t left = __shfl_up(v, 1, WAVE);
            if (lane == 0) left = prev;
            const bool keep = v != BK_EMPTY && v != left;
            const uint64_t m = __ballot(keep);
            prev = __shfl(v, WAVE - 1, WAVE);
            bk_wave_sync();
            if (keep) a[cnt + (uint32_t)__popcll(m & lt)] = v;
            bk_wave_sync();
            cnt += (uint32_t)__popcll(m);
        }
    }
    __syncthreads();
    return cnt;
}

// A row of up to MOST values by one wave, sorted without repeats.
template <uint32_t MOST = BK_WAVE_ROW>
__device__ __forceinline__ uint32_t bk_wave_row(uint32_t* a, uint32_t n) {
    n = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
    if (n <= 64) return bk_wave_sort_unique<1>(a, n);
    if (n <= 128) return bk_wave_sort_unique<2>(a, n);
    if (n <= 256) return bk_wave_sort_unique<4>(a, n);
    if (MOST <= 512 || n <= 512) return bk_wave_sort_unique<8>(a, n);
    if constexpr (MOST > 512) return bk_wave_sort_unique<(int)BK_WAVE_ROW / WAVE>(a, n);
}

// Rows that a wave takes for itself: where few of rows [va, vb) have more than
// 512 values, the whole block sorts each of those (2000 values in about 10 us,
// where a wave alone takes 20).
template <int BLOCK, class Len>
__device__ __forceinline__ uint32_t bk_wave_most(int va, int vb, Len&& len) {
    int many = 0;
    for (int v0 = va; v0 < vb; v0 += WAVE) {
        const int v = v0 + (bk_tid() & (WAVE - 1));
        const uint32_t n = v < vb ? len(v) : 0u;
        many += (int)__popcll(__ballot(n > 512 && n <= BK_WAVE_ROW));
    }
    return 2 * many > BLOCK / WAVE ? BK_WAVE_ROW : 512u;
}

// ---- bk_rows -----------------------------------------------------------------
struct BkRowsArgs {
    BkMap mp;
    const uint32_t* rec;
    const uint32_t* starts;
    const uint32_t* units;    // first unit per bucket
    const uint32_t* repeats;  // per bucket: records whose pair an earlier record of the element has
    BkLookback lookback;
    uint32_t* list;  // a word per record for those of shared buckets (null: no room)
    uint32_t* hdr;
    int32_t* nrp;    // node CSR (null: not wanted)
    int32_t* ncols;
    int64_t ncap;
    int32_t* erp;    // element CSR (null: not wanted)
    int32_t* ecols;
    int64_t ecap;
    int64_t n_elem;
};

// Per number of neighbours K: the block, the most records (CAP, what its
// threads hold in registers) and vertices (VMAX) of a bucket, and the words
// its rows share (POOL; two large blocks fit a CU's LDS).  Of the pool
//  - K > 0: K words per record for the neighbours; packed, the node rows
//    take about a word per record, and the elements another;
//  - K = 0: a word per record for the elements.
template <int K, bool LARGE>
struct BkShape;
template <> struct BkShape<0, true> { static constexpr int BLOCK = 512, CAP = 14848, VMAX = 2048, POOL = 14848; };
template <> struct BkShape<2, true> { static constexpr int BLOCK = 512, CAP = 7680, VMAX = 1536, POOL = 15872; };
template <> struct BkShape<3, true> { static constexpr int BLOCK = 512, CAP = 5952, VMAX = 768, POOL = 17920; };
template <> struct BkShape<4, true> { static constexpr int BLOCK = 512, CAP = 4480, VMAX = 768, POOL = 17920; };
template <> struct BkShape<0, false> { static constexpr int BLOCK = 256, CAP = 5120, VMAX = 1024, POOL = 5120; };
template <> struct BkShape<2, false> { static constexpr int BLOCK = 256, CAP = 3072, VMAX = 640, POOL = 6144; };
template <> struct BkShape<3, false> { static constexpr int BLOCK = 256, CAP = 2560, VMAX = 320, POOL = 7680; };
template <> struct BkShape<4, false> { static constexpr int BLOCK = 256, CAP = 2048, VMAX = 320, POOL = 8192; };

constexpr int BK_PAD = 64;  // words a network may read past the last row

template <int K, bool LARGE>
struct BkLds {
    using S = BkShape<K, LARGE>;
    static constexpr int VAL = S::POOL + BK_PAD;
    static constexpr int WORDS = VAL + (S::VMAX + 1) + (S::VMAX + 1) + S::VMAX / 2;
};

// Exclusive sum over the block with one barrier: *turn alternates between the
// two halves of s_tmp (2 x BLOCK / 64 words), so that a call's reads are over
// before its half is written again.
template <int BLOCK>
__device__ __forceinline__ uint32_t bk_block_sum(uint32_t v, uint32_t* s_tmp, int* turn, uint32_t* total) {
    constexpr int WAVES = BLOCK / WAVE;
    const int wid = bk_tid() / WAVE;
    uint32_t* t = s_tmp + *turn * WAVES;
    *turn ^= 1;
    const uint32_t incl = bk_wave_sum(v);
    if ((bk_tid() & (WAVE - 1)) == WAVE - 1) t[wid] = incl;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t x = t[w];
        before += w < wid ? x : 0u;
        sum += x;
    }
    *total = (uint32_t)__builtin_amdgcn_readfirstlane((int)sum);
    return before + incl - v;
}

// Exclusive scan of s[0 .. n) in place, n <= MAXN; s[n] = total, returned.
// Ends with a barrier.
template <int BLOCK, int MAXN>
__device__ __forceinline__ uint32_t bk_scan_lds(uint32_t* s, int n, uint32_t* s_tmp, int* turn) {
    constexpr int PER = (MAXN + BLOCK - 1) / BLOCK;
    uint32_t v[PER], sum = 0;
    const int i0 = bk_tid() * PER;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        v[q] = i0 + q < n ? s[i0 + q] : 0u;
        sum += v[q];
    }
    uint32_t total;
    uint32_t run = bk_block_sum<BLOCK>(sum, s_tmp, turn, &total);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (i0 + q < n) s[i0 + q] = run;
        run += v[q];
    }
    if (bk_tid() == 0) s[n] = total;
    __syncthreads();
    return total;
}

// Barrier and a vote of the block (s_tmp and turn as in bk_block_sum), as a
// scalar: a branch on it is uniform for the compiler too, so what one side keeps
// in registers does not live through the other.
template <int BLOCK>
__device__ __forceinline__ bool bk_any(bool x, uint32_t* s_tmp, int* turn) {
    constexpr int WAVES = BLOCK / WAVE;
    const int tid = bk_tid();
    uint32_t* t = s_tmp + *turn * WAVES;
    *turn ^= 1;
    const bool any = __ballot(x) != 0;
    if ((tid & (WAVE - 1)) == 0) t[tid / WAVE] = any ? 1u : 0u;
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) all |= t[w];
    return __builtin_amdgcn_readfirstlane((int)all) != 0;
}

template <int W>
struct BkWords {
    uint32_t w[W];
};
// Where record i starts, in bytes.
template <int W>
__host__ __device__ constexpr uint64_t bk_record_at(uint64_t i) {
    return i * (uint64_t)(4 * W);
}
static_assert(bk_record_at<5>(1u << 30) == 5ull << 32, "one mesh's records may all be in one bucket, 4 GiB of them and more");
// Record i after rec.  NEAR: one of the first few, by a 32-bit offset.
template <int W, bool NEAR = false>
__device__ __forceinline__ void bk_load(const uint32_t* __restrict__ rec, uint32_t i, uint32_t (&r)[W]) {
    const char* at = reinterpret_cast<const char*>(rec);
    const BkWords<W> x = *reinterpret_cast<const BkWords<W>*>(NEAR ? at + i * (uint32_t)(4 * W) : at + bk_record_at<W>(i));
#pragma unroll
    for (int q = 0; q < W; ++q) r[q] = x.w[q];
}

// What a block does: a bucket, or one of the shares of one.  Its unit is its
// place in the look-back, in the order of the rows.
struct BkUnit {
    uint32_t unit, bucket, share, shares;
    bool last;  // of all
};
// The unit's entries go to its look-back word, the sum of the earlier units'
// comes back (every thread).
__device__ __forceinline__ void bk_publish(uint64_t* lookback, uint32_t unit, uint64_t mine) {
    if (bk_tid() == 0) lb_store(lookback + unit, (unit == 0 ? LB_INC : LB_AGG) | mine);
}
__device__ __forceinline__ uint64_t bk_before(const BkRowsArgs& a, uint64_t* lookback, uint32_t unit, uint64_t mine,
                                              uint64_t* s_base) {
    if (bk_tid() < WAVE) {
        const uint64_t p = wave_lookback_prefix(lookback, unit, mine, a.hdr + HDR_ERR, a.hdr + HDR_BK_PROGRESS);
        if (bk_tid() == 0) *s_base = p;
    }
    __syncthreads();
    return *s_base;
}

// f(record, its place, its number in a turn) for the n records at rec, or for
// those that the n entries of `list` name, over the block, BK_AHEAD of a thread's
// loads on their way at once.  Counts as steps for those that wait.  (A block
// takes some 25 to 50 GB/s of records; 16 loads ahead gained 5 %.)
constexpr int BK_AHEAD = 8;
constexpr uint32_t BK_STEP = 1u << 20;  // records of a step
template <int W, int BLOCK, class F>
__device__ __forceinline__ void bk_each_record(const BkRowsArgs& a, const uint32_t* rec, const uint32_t* list, uint32_t n,
                                               F&& f) {
    for (uint32_t c0 = 0; c0 < n; c0 += BK_STEP) {
        if (bk_tid() == 0) atomicAdd(a.hdr + HDR_BK_PROGRESS, 1u);
        const uint32_t end = c0 + tmin(n - c0, BK_STEP);
        for (uint32_t i0 = c0 + (uint32_t)bk_tid(); i0 < end; i0 += BK_AHEAD * BLOCK) {
            uint32_t at[BK_AHEAD], r[BK_AHEAD][W];
            bk_each<BK_AHEAD>([&](auto uu) BK_INLINE {
                constexpr int u = decltype(uu)::value;
                at[u] = tmin(i0 + u * BLOCK, end - 1);
                if (list) at[u] = list[at[u]];
            });
            bk_each<BK_AHEAD>([&](auto uu) BK_INLINE { bk_load<W>(rec, at[decltype(uu)::value], r[decltype(uu)::value]); });
            bk_each<BK_AHEAD>([&](auto uu) BK_INLINE {
                constexpr int u = decltype(uu)::value;
                if (i0 + u * BLOCK < end) f(r[u], at[u], uu);
            });
        }
    }
}

// Values [src, src + left) of a row, in windows of up to MOST values at a time,
// until the last one is in x (sorted) with c distinct values; src and left
// then describe it.  False for a row that keeps more than 24 distinct values
// in a window, which would use up its other values a few at a time (all of
// them are still in [src, src + left)).  Called by whole waves; a row that is
// done sorts its last window again meanwhile.
template <int MOST>
__device__ __forceinline__ bool bk_row_windows(uint32_t*& src, uint32_t& left, uint32_t (&x)[MOST], uint32_t& c) {
    bool more, fits = true;
    do {
        const uint32_t len = tmin<uint32_t>(left, (uint32_t)MOST);
        bk_pick_network<MOST>(len, [&](auto nn) BK_INLINE {
            constexpr int N = decltype(nn)::value;
            bk_row_load<N>(src, len, x);
            bk_each<MOST - N>([&](auto ii) BK_INLINE { x[N + decltype(ii)::value] = BK_EMPTY; });
        });
        more = MOST > 16 && len != left;
        if (more) {  // the distinct values right before the values to come
            c = bk_row_store_back<MOST>(x, src + len);
            src += len - c;
            left -= len - c;
            fits = c <= 24;
            more = fits;
        }
    } while (__ballot(more));
    c = bk_row_count<MOST>(x);
    return fits;
}

// Rows [va, vb), row v's `per` values per record at s_val + per * (s_start[v]
// - s0): each sorted without repeats, its first value at s_pos[v], its count
// in s_cnt[v].  Rows beyond a window are sorted by a wave or the
// block (bk_wave_most).  All threads; starts and ends with a barrier.
template <int BLOCK>
__device__ __forceinline__ void bk_sort_range(uint32_t* s_val, const uint32_t* s_start, uint32_t s0, int va, int vb,
                                              uint32_t per, uint32_t* s_cnt, uint16_t* s_pos) {
    constexpr uint32_t LONG = 1u << 31, DONE = 1u << 30;
    const int tid = bk_tid(), lane = tid & (WAVE - 1), wid = tid / WAVE;
    __syncthreads();
    for (int v0 = va + wid * WAVE; v0 < vb; v0 += BLOCK) {
        const int v = v0 + lane;
        const uint32_t st = v < vb ? s_start[v] - s0 : 0u;
        uint32_t left = v < vb ? (s_start[v + 1] - s_start[v]) * per : 0u;
        uint32_t* src = s_val + st * per;
        uint32_t x[BK_NET_MAX], c;
        const bool fits = bk_row_windows<(int)BK_NET_MAX>(src, left, x, c);
        if (fits && c) bk_row_store<(int)BK_NET_MAX>(x, src);
        if (v < vb) {
            s_cnt[v] = fits ? c : left | LONG;
            s_pos[v] = (uint16_t)(src - s_val);
        }
    }
    __syncthreads();
    const uint32_t wave_most = bk_wave_most<BLOCK>(va, vb, [&](int v) BK_INLINE { return s_cnt[v] & LONG ? s_cnt[v] & ~LONG : 0u; });
    __syncthreads();  // (before a wave marks one done)
    for (int v0 = va, i = 0; v0 < vb; v0 += WAVE) {  // the waves take the longer rows in turn
        const uint32_t f = v0 + lane < vb ? s_cnt[v0 + lane] : 0u;
        // (a row that another wave has done meanwhile is still marked, so that all count alike)
        const bool wave_row = (f & LONG) && ((f & DONE) || (f & ~LONG) <= wave_most);
        for (uint64_t m = __ballot(wave_row); m; m &= m - 1, ++i) {
            const int l = __builtin_ctzll(m);
            if (i % (BLOCK / WAVE) != wid) continue;
            const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)f, l) & ~LONG;
            const uint32_t c = bk_wave_row(s_val + s_pos[v0 + l], n);
            bk_wave_sync();
            if (lane == 0) s_cnt[v0 + l] = c | LONG | DONE;
        }
    }
    __syncthreads();
    for (int v = va + tid; v < vb; v += BLOCK)
        if (s_cnt[v] & DONE) s_cnt[v] &= ~(LONG | DONE);
    __syncthreads();
    for (int v = va; v < vb; ++v) {
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cnt[v]);
        if (!(n & LONG)) continue;
        __syncthreads();  // (every wave has seen the mark)
        const uint32_t c = bk_block_sort_unique<BLOCK>(s_val + s_pos[v], n & ~LONG);
        if (tid == 0) s_cnt[v] = c;
        __syncthreads();
    }
}

// Windows [wa, wb) of one row (vertex v of the bucket) beyond the LDS, from the
// records that bk_each_record takes, each its ids in a bit map of `words` words at s_map.  With write, they go to cols from
// `at` on (as far as cap lets); with row_start, `at` is where the whole row starts
// (of elements without repeats).  Returns their number.
template <int K, int W, int BLOCK>
__device__ __forceinline__ uint32_t bk_huge_row(const BkRowsArgs& a, const uint32_t* rec, const uint32_t* list,
                                                uint32_t n, uint32_t lo, int v, uint32_t wa, uint32_t wb,
                                                bool elements, bool row_start, uint32_t* s_map, uint32_t words,
                                                uint32_t* s_tmp, int* turn, bool write, int32_t* cols, uint64_t at,
                                                int64_t cap, bool* full) {
    const int tid = bk_tid();
    const uint32_t per = words / (BLOCK / WAVE);  // (even: a static_assert with the shapes)
    uint32_t all = 0;
    for (uint32_t w = wa; w < wb; ++w) {
        const uint32_t w0 = w * 32 * words;  // (below 2^31: an id)
        uint32_t below = 0;
        __syncthreads();
        for (uint32_t i = tid; i < words; i += BLOCK) s_map[i] = 0;
        __syncthreads();
        bk_each_record<W, BLOCK>(a, rec, list, n, [&](const uint32_t (&r)[W], uint32_t, auto) BK_INLINE {
            if (bk_row<K, W>(a.mp, r, lo) != (uint32_t)v) return;
            auto put = [&](uint32_t x) BK_INLINE {
                const uint32_t o = x - w0;
                if (x < w0) ++below;
                else if (o < 32 * words) atomicOr(&s_map[o >> 5], 1u << (o & 31));
            };
            if (elements) {
                put(bk_elem<K, W>(a.mp, r));
            } else if constexpr (K > 0) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const uint32_t x = bk_nbr<K, W>(a.mp, r, k);
                    if (x != lo + (uint32_t)v) put(x);
                }
            }
        });
        __syncthreads();
        // a wave has a run of the map
        const int lane = tid & (WAVE - 1);
        const uint32_t* const map = s_map + (uint32_t)tid / WAVE * per;
        uint32_t c = 0;
        for (uint32_t i = lane; i < per; i += WAVE) c += (uint32_t)__popc(map[i]);
        uint32_t total, skip = 0;
        if (row_start && w == wa && wa > 0) bk_block_sum<BLOCK>(below, s_tmp, turn, &skip);
        at += skip;
        uint32_t place = bk_block_sum<BLOCK>(c, s_tmp, turn, &total);
        place = (uint32_t)__builtin_amdgcn_readfirstlane((int)place);
        for (uint32_t i0 = 0; write && i0 < per; i0 += 2 * WAVE) {  // 64 ids per lane
            const uint32_t i = i0 + 2 * lane, id0 = w0 + 32 * ((uint32_t)tid / WAVE * per + i0);
            uint64_t m = i < per ? (uint64_t)map[i + 1] << 32 | map[i] : 0ull;
            const uint32_t mine = (uint32_t)__popcll(m), upto = bk_wave_sum(mine);
            auto put = [&](uint64_t d, uint32_t id) BK_INLINE {
                if ((int64_t)d < cap) cols[d] = (int32_t)id;
                else *full = true;
            };
            if (!__ballot(mine > 16)) {
                for (uint64_t d = at + all + place + upto - mine; m; m &= m - 1) put(d++, id0 + 64 * lane + __builtin_ctzll(m));
            } else {  // many of them: a lane's go out side by side, by the wave
                const uint32_t hi = (uint32_t)(m >> 32), lo32 = (uint32_t)m;
                uint64_t d = at + all + place;
                for (uint64_t l64 = __ballot(m != 0); l64; l64 &= l64 - 1) {
                    const int l = __builtin_ctzll(l64);
                    const uint32_t h = (uint32_t)__builtin_amdgcn_readlane((int)hi, l), o = (uint32_t)__builtin_amdgcn_readlane((int)lo32, l);
                    const uint64_t q = (uint64_t)h << 32 | o;
                    if (q >> lane & 1) put(d + __builtin_amdgcn_mbcnt_hi(h, __builtin_amdgcn_mbcnt_lo(o, 0u)), id0 + 64 * l + lane);
                    d += (uint32_t)__popcll(q);
                }
            }
            place += (uint32_t)__builtin_amdgcn_readlane((int)upto, WAVE - 1);
        }
        all += total;
    }
    __syncthreads();
    return all;
}

// Records per vertex counted and scanned into s_start (bk_*_ranges).
template <int K, int W, int BLOCK, int VMAX>
__device__ __forceinline__ void bk_count_records(const BkRowsArgs& a, const uint32_t* rec, uint32_t n, uint32_t lo, int nv,
                                                 uint32_t* s_start, uint32_t* s_tmp, int* turn) {
    const int tid = bk_tid();
    __syncthreads();
    for (int v = tid; v < nv; v += BLOCK) s_start[v] = 0;
    __syncthreads();
    bool crowded = false;  // many lanes with one row, which would queue at its counter: one adds for them
    bk_each_record<W, BLOCK>(a, rec, nullptr, n, [&](const uint32_t (&r)[W], uint32_t, auto uu) BK_INLINE {
        const uint32_t v = bk_row<K, W>(a.mp, r, lo);
        if (decltype(uu)::value == 0) crowded = bk_crowded(v);
        uint32_t add = 1;
        if (crowded) {
            const uint32_t v0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
            const uint64_t same = __ballot(v == v0);
            if (v == v0) add = (int)(bk_tid() & (WAVE - 1)) == __builtin_ctzll(same) ? (uint32_t)__popcll(same) : 0u;
        }
        if (v < (uint32_t)nv && add) atomicAdd(&s_start[v], add);
    });
    __syncthreads();
    bk_scan_lds<BLOCK, VMAX>(s_start, nv, s_tmp, turn);
}

// The last vertex end vb > va (vb = va: row va alone is too long) such that the
// records of [va, vb) are at most `most`.
__device__ __forceinline__ int bk_range_end(const uint32_t* s_start, int va, int nv, uint32_t most) {
    int vb = va;
    for (int step = 4096; step >= 1; step >>= 1)
        if (vb + step <= nv && s_start[vb + step] - s_start[va] <= most) vb += step;
    return __builtin_amdgcn_readfirstlane(vb);
}

// The first vertex whose records start at x or beyond (nv: none).
__device__ __forceinline__ int bk_first_from(const uint32_t* s_start, int nv, uint32_t x) {
    int v = 0;
    for (int step = 4096; step >= 1; step >>= 1)
        if (v + step <= nv && s_start[v + step - 1] < x) v += step;
    return __builtin_amdgcn_readfirstlane(v);
}

// One relation of any unit, from its bucket's records in memory: ranges of
// vertices whose records fit the LDS.  elements: the element rows, the bucket's
// starting at `ebase`; else the node rows.  Those, and the element rows of a
// share where the bucket has repeats, are counted first (a unit in one range
// keeps them in the LDS meanwhile).  Share i takes the vertices whose
// records start in the i-th part of the bucket's, and lists them by vertex (at
// `list`, if there is room), so that a range reads only its own.  `again`: the
// unit has done its node rows here, and the counts and the list stand.  Every
// thread of the block calls it.
template <int K, int W, bool LARGE>
__device__ __forceinline__ void bk_ranges(const BkRowsArgs& a, bool elements, bool repeats, const BkUnit& u,
                                          int64_t rec0, uint32_t n, uint32_t lo, int nv, uint64_t ebase, uint32_t* list, bool again,
                                          uint32_t* s_val, uint32_t* s_start, uint32_t* s_cnt, uint16_t* s_pos,
                                          uint32_t* s_tmp, int* turn, uint64_t* s_base) {
    using S = BkShape<K, LARGE>;
    constexpr int BLOCK = S::BLOCK;
    constexpr uint32_t WINDOW = 32u * S::POOL;  // ids of a bit map
    // (nothing of this rarely taken path is computed ahead of it, where it would
    // cost the other path registers)
    const int tid = bk_tid();
    asm volatile("" : "+s"(n), "+s"(lo), "+s"(nv));
    const int lane = tid & (WAVE - 1), wid = tid / WAVE;
    const uint32_t* rec = a.rec + rec0 * W;
    const uint32_t per = elements ? 1u : (uint32_t)(K > 0 ? K : 1);
    const uint32_t most = (uint32_t)S::POOL / per;
    int32_t* const rp = elements ? a.erp : a.nrp;
    int32_t* const cols = elements ? a.ecols : a.ncols;
    const int64_t cap = elements ? a.ecap : a.ncap;
    const uint32_t windows = (uint32_t)(((elements ? (uint64_t)a.n_elem : (uint64_t)a.mp.n_vert) + WINDOW - 1) / WINDOW);
    bool full = false;
    if (!again) bk_count_records<K, W, BLOCK, S::VMAX>(a, rec, n, lo, nv, s_start, s_tmp, turn);
    int v0 = 0, v1 = nv;
    bool head = false;  // the share starts inside the row of vertex v0 - 1, beyond the LDS
    const uint32_t part = (n + u.shares - 1) / u.shares;
    if (u.shares > 1) {
        v0 = u.share == 0 ? 0 : bk_first_from(s_start, nv, u.share * part);
        if (u.share + 1 < u.shares) v1 = bk_first_from(s_start, nv, (u.share + 1) * part);
        head = v0 > 0 && s_start[v0] > u.share * part && s_start[v0] - s_start[v0 - 1] > most;
    }
    // the windows of long row v that share u takes, if it has a few shares: its first one
    // has its records listed
    auto window = [&](int v, bool end) BK_INLINE {
        const uint32_t first = s_start[v] / part, shares = (s_start[v + 1] - 1) / part + 1 - first;
        if (shares < 4) return first != u.share ? windows : end ? windows : 0u;
        return (uint32_t)((uint64_t)windows * (u.share - first + (end ? 1 : 0)) / shares);
    };
    // (the list takes one pass over all records: not for a share of one range, or of a
    // row with most of them)
    const uint32_t mine = s_start[v1] - s_start[v0];
    if (u.shares == 1 || mine <= (again ? (uint32_t)S::POOL / (K > 0 ? K : 1) : most) || mine > 4 * part) list = nullptr;
    if (list && !again) {
        for (int v = v0 + tid; v < v1; v += BLOCK) s_cnt[v] = 0;
        __syncthreads();
        bk_each_record<W, BLOCK>(a, rec, nullptr, n, [&](const uint32_t (&r)[W], uint32_t i, auto) BK_INLINE {
            const uint32_t v = bk_row<K, W>(a.mp, r, lo);
            if (v >= (uint32_t)v0 && v < (uint32_t)v1) list[s_start[v] + atomicAdd(&s_cnt[v], 1u)] = i;
        });
        __syncthreads();
    }
    // what bk_each_record takes for vertices [va, vb) of the share's own
    auto own = [&](int va) BK_INLINE { return list && va >= v0 ? list + s_start[va] : nullptr; };
    auto records = [&](int va, int vb) BK_INLINE { return list && va >= v0 ? s_start[vb] - s_start[va] : n; };
    const bool single = !head && (v0 == v1 || bk_range_end(s_start, v0, v1, most) == v1);
    const bool counted = !elements || (repeats && u.shares > 1);
    uint64_t base = ebase, run = 0;
    if (!counted && u.shares > 1) base += s_start[head ? v0 - 1 : v0];
    for (int phase = counted ? 0 : 1; phase < 2; ++phase) {  // 0: count, 1: write
        run = 0;
        for (int va = head ? v0 - 1 : v0; va < v1;) {
            const int vb = va < v0 ? va : bk_range_end(s_start, va, v1, most);
            const uint64_t at = base + run;
            if (vb == va) {
                if (phase == 1 && va >= v0 && tid == 0) rp[lo + va] = (int32_t)at;
                run += bk_huge_row<K, W, BLOCK>(a, rec, own(va), records(va, va + 1), lo, va, window(va, false),
                                                window(va, true), elements, !counted, s_val, (uint32_t)S::POOL, s_tmp,
                                                turn, phase == 1, cols, at, cap, &full);
                ++va;
                // (where the row ends, if it does in this share; else nothing follows)
                if (!counted && u.shares > 1) run = ebase + s_start[va] - base;
                continue;
            }
            const uint32_t s0 = s_start[va];
            if (phase == 0 || !counted || !single) {
                for (int v = va + tid; v < vb; v += BLOCK) s_cnt[v] = 0;
                __syncthreads();
                bk_each_record<W, BLOCK>(a, rec, own(va), records(va, vb), [&](const uint32_t (&r)[W], uint32_t, auto) BK_INLINE {
                    const uint32_t v = bk_row<K, W>(a.mp, r, lo);
                    if (v < (uint32_t)va || v >= (uint32_t)vb) return;
                    const uint32_t slot = s_start[v] - s0 + atomicAdd(&s_cnt[v], 1u);
                    if (elements) {
                        s_val[slot] = bk_elem<K, W>(a.mp, r);
                    } else if constexpr (K > 0) {
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            const uint32_t x = bk_nbr<K, W>(a.mp, r, k);
                            s_val[slot * K + k] = x == lo + v ? BK_EMPTY : x;
                        }
                    }
                });
                bk_sort_range<BLOCK>(s_val, s_start, s0, va, vb, per, s_cnt, s_pos);
                __syncthreads();
                bk_scan_lds<BLOCK, S::VMAX>(s_cnt + va, vb - va, s_tmp, turn);
            }
            const uint32_t total = s_cnt[vb];
            if (phase == 1) {
                for (int v = va + tid; v < vb; v += BLOCK) rp[lo + v] = (int32_t)(at + s_cnt[v]);
                if ((int64_t)(at + total) > cap) full = true;
                else
                    for (int v = va + wid; v < vb; v += BLOCK / WAVE) {
                        const uint32_t c0 = s_cnt[v], c = s_cnt[v + 1] - c0;
                        const uint32_t* x = s_val + s_pos[v];
                        for (uint32_t i = lane; i < c; i += WAVE) cols[at + c0 + i] = (int32_t)x[i];
                    }
            }
            run += total;
            __syncthreads();
            va = vb;
        }
        if (phase == 0) {
            uint64_t* const lookback = elements ? a.lookback.elems + (u.unit - u.share) : a.lookback.nodes;
            const uint32_t place = elements ? u.share : u.unit;
            bk_publish(lookback, place, run);
            base = bk_before(a, lookback, place, run, s_base);
            if (elements) base += ebase;
            __syncthreads();
        }
    }
    if (u.last && tid == 0) rp[a.mp.n_vert] = (int32_t)(base + run);
    if (full) set_error(a.hdr + HDR_ERR, ERR_CAPACITY);
}

// A bucket of at most CAP records over nv vertices, from registers and LDS.
// Which relations are done: no node rows where one is left to bk_ranges, with
// nothing of them announced or written yet (a row of more than 64 distinct values,
// or a second one of more than 32 among 64 rows), and no element rows where the
// bucket has repeats (of a vertex in an element) and a row beyond the networks.
constexpr int BK_NODE_DONE = 1, BK_ELEM_DONE = 2;
template <int K, int W, bool LARGE>
__device__ __forceinline__ int bk_rows_lds(const BkRowsArgs& a, const BkUnit& u, int64_t rec0, uint32_t n, uint32_t lo,
                                            int nv, uint32_t odd, bool elem, bool repeats, uint64_t ebase, uint32_t* s_val,
                                            uint32_t* s_start,
                                            uint32_t* s_cnt, uint32_t* s_tmp, int* turn, uint64_t* s_base) {
    using S = BkShape<K, LARGE>;
    constexpr int BLOCK = S::BLOCK, CAP = S::CAP, VMAX = S::VMAX;
    constexpr int R = (CAP + BLOCK - 1) / BLOCK;  // records per thread
    constexpr uint32_t NONE = 0xffffffffu, NO_SLOT = 0xffffu;
    static_assert(CAP < (int)NO_SLOT, "16-bit slots");
    const int tid = bk_tid();
    const bool node = K > 0 && a.nrp != nullptr;

    // ---- records into registers; counters and tables cleared meanwhile
    uint32_t r[R][W];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        // (without a branch: past the bucket, its last record again)
        bk_load<W, true>(a.rec + rec0 * W, tmin<uint32_t>(q * BLOCK + tid, n ? n - 1 : 0u), r[q]);
    }
    for (int v = tid; v < nv; v += BLOCK) {
        s_start[v] = 0;
        s_cnt[v] = 0;
    }
    __syncthreads();
    // ---- each record's row and its place there
    uint32_t at[R];  // row << 16 | place
    bool bad = false;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        at[q] = NONE;
        if ((uint32_t)(q * BLOCK + tid) < n) {
            const uint32_t v = bk_row<K, W>(a.mp, r[q], lo);
            if (v < (uint32_t)nv) at[q] = (v << 16) | atomicAdd(&s_start[v], 1u);
            else bad = true;
        }
    }
    __syncthreads();
    bk_scan_lds<BLOCK, VMAX>(s_start, nv, s_tmp, turn);
    auto deg = [&](int v) BK_INLINE { return s_start[v + 1] - s_start[v]; };

    // ---- neighbours to their rows; what stays in registers is each record's
    // element and, two to a word, its slot
    uint32_t ev[R], slots[(R + 1) / 2];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        ev[q] = bk_elem<K, W>(a.mp, r[q]);
        uint32_t slot = NO_SLOT;
        if (at[q] != NONE) {
            const uint32_t v = at[q] >> 16;
            slot = s_start[v] + (at[q] & 0xffffu);
            if constexpr (K == 0) {
                s_val[slot] = ev[q];
            } else {
                // the vertex itself stands for no neighbour: in pyramids, and where ids
                // repeat or are out of range
                uint32_t w[K];
#pragma unroll
                for (int k = 0; k < K; ++k) w[k] = bk_nbr<K, W>(a.mp, r[q], k);
                if (K == 4 || odd) {
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (w[k] == lo + v) w[k] = BK_EMPTY;
                }
#pragma unroll
                for (int k = 0; k < K; ++k) s_val[K * slot + k] = w[k];
            }
        }
        if (q & 1) slots[q / 2] |= slot << 16;
        else slots[q / 2] = slot;
    }
    bool wide = false;  // some node row needs more than the 16-wide network
    if (K > 0 && node) {
        for (int v = tid; v < nv; v += BLOCK) wide |= K * deg(v) > 16;
        wide = bk_any<BLOCK>(wide, s_tmp, turn);
    }
    __syncthreads();

    // ---- node rows
    // (the mark of a row of too many distinct values: more than all rows of a bucket keep,
    // K * CAP being at most POOL, and small enough that the sum of a whole block of marks
    // and of all kept values stays below 2^32)
    constexpr uint32_t STUCK = S::POOL + 1;
    static_assert(K * CAP <= S::POOL && (uint64_t)BLOCK * STUCK + S::POOL <= UINT32_MAX, "marks never cancel out");
    uint32_t total = 0;
    bool stuck = false;
    if (K > 0 && node) {
        constexpr uint32_t MID_ROW = 512;
        auto rows = [&](auto most) BK_INLINE {  // rounds of up to `most` values
            constexpr int MOST = decltype(most)::value;
            for (int v0 = 0; v0 < nv; v0 += BLOCK) {
                const int v = v0 + tid;
                const bool in = v < nv;
                const uint32_t st = in ? s_start[v] : 0u;
                uint32_t left = in ? K * (s_start[v + 1] - st) : 0u;
                uint32_t* src = s_val + K * st;
                uint32_t x[MOST], c;
                const bool fits = bk_row_windows<MOST>(src, left, x, c);
                // the rows the windows leave: by the wave, and back to their lane up to 32
                // distinct values; one row of up to 64 stays spread over the lanes
                int spread = -1;
                uint32_t mine = 0;
                if (MOST > 16 && __popcll(__ballot(!fits)) > 8) {
                    if (!fits) c = STUCK;  // (many such rows: bk_ranges shares them among the waves)
                } else if (MOST > 16 && __ballot(!fits)) {
                    for (uint64_t m = __ballot(!fits); m; m &= m - 1) {
                        const int l = __builtin_ctzll(m);
                        uint32_t* const a0 = s_val + __builtin_amdgcn_readlane((int)(src - s_val), l);
                        const uint32_t n0 = (uint32_t)__builtin_amdgcn_readlane((int)left, l);
                        // (no mesh's row of that many values keeps 64)
                        const uint32_t cl = n0 > MID_ROW ? STUCK : bk_wave_row<MID_ROW>(a0, n0);
                        const bool wide_row = cl > (uint32_t)MOST;
                        if ((tid & (WAVE - 1)) == l) c = wide_row && (cl > 64 || spread >= 0) ? STUCK : cl;
                        if (wide_row && spread < 0) {
                            spread = l;
                            mine = a0[tid & (WAVE - 1)];
                        }
                    }
                    if (!fits) {
                        bk_each<MOST>([&](auto ii) BK_INLINE {
                            constexpr int i = decltype(ii)::value;
                            const uint32_t y = src[i];
                            x[i] = (uint32_t)i < c ? y : BK_EMPTY;
                        });
                    }
                }
                uint32_t sum;
                // (its barrier: every row of this round has been read.  A row goes to or
                // below its own place, so the rows of later rounds are untouched.)
                const uint32_t off = total + bk_block_sum<BLOCK>(c, s_tmp, turn, &sum);
                total += sum;
                if (total >= STUCK) return;  // (before the round stores anything)
                if (c && (tid & (WAVE - 1)) != spread) bk_row_store<MOST>(x, s_val + off);
                if (MOST > 16 && spread >= 0) {
                    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)off, spread);
                    if ((tid & (WAVE - 1)) < __builtin_amdgcn_readlane((int)c, spread)) s_val[o + (tid & (WAVE - 1))] = mine;
                }
                if (in) s_cnt[v] = off;
            }
        };
        if (wide) rows(std::integral_constant<int, (int)BK_NET_MAX>{});
        else rows(std::integral_constant<int, 16>{});
        stuck = total >= STUCK;  // a row beyond the networks
        if (!stuck) bk_publish(a.lookback.nodes, u.unit, total);
    }
    bool full = false;
    auto nodes_out = [&]() BK_INLINE {
        const uint64_t base = bk_before(a, a.lookback.nodes, u.unit, total, s_base);
        for (int v = tid; v < nv; v += BLOCK) a.nrp[lo + v] = (int32_t)(base + s_cnt[v]);
        if (u.last && tid == 0) a.nrp[a.mp.n_vert] = (int32_t)(base + total);
        if ((int64_t)(base + total) > a.ncap) full = true;
        else
            for (uint32_t i = tid; i < total; i += BLOCK) a.ncols[base + i] = (int32_t)s_val[i];
    };
    // rows that share no neighbours leave no room for the elements after them: they go
    // out first (500,000 vertices, 1 M random triangles: 284 us with the rows made again
    // from memory, 171 so)
    const bool crowded = K > 0 && node && elem && !stuck && total + n > (uint32_t)S::POOL;
    if (K > 0 && crowded) {
        nodes_out();
        __syncthreads();
    }

    // ---- element rows, while the look-back word is on its way
    if (elem) {
        uint32_t* const s_elem = K > 0 ? s_val + S::POOL - n : s_val;
        if constexpr (K > 0) {
#pragma unroll
            for (int q = 0; q < R; ++q)
                {
                    const uint32_t slot = (slots[q / 2] >> (16 * (q & 1))) & 0xffffu;
                    if (slot != NO_SLOT) s_elem[slot] = ev[q];
                }
        }
        __syncthreads();
        bool lng = false;
        for (int v0 = 0; v0 < nv; v0 += BLOCK) {
            const int v = v0 + tid;
            const uint32_t d = v < nv ? deg(v) : 0u;
            lng |= d > BK_NET_MAX;
            const uint32_t len = d > BK_NET_MAX ? 0u : d;
            uint32_t* const src = s_elem + (v < nv ? s_start[v] : 0u);
            bk_pick_network<BK_NET_MAX>(len, [&](auto nn) BK_INLINE {
                constexpr int N = decltype(nn)::value;
                uint32_t x[N];
                bk_row_load<N>(src, len, x);
                bk_each<N>([&](auto ii) BK_INLINE {
                    constexpr int i = decltype(ii)::value;
                    if ((uint32_t)i < len) src[i] = x[i];
                });
            });
        }
        lng = bk_any<BLOCK>(lng, s_tmp, turn);
        if (lng && !repeats) {  // longer rows: a wave each, or the block
            const uint32_t wave_most = bk_wave_most<BLOCK>(0, nv, deg);
            for (int v0 = 0; v0 < nv; v0 += WAVE) {
                const int v = v0 + (tid & (WAVE - 1));
                const uint32_t d = v < nv ? deg(v) : 0u;
                uint64_t m = __ballot(d > BK_NET_MAX && d <= wave_most);
                for (int i = 0; m; m &= m - 1, ++i) {
                    const int u = v0 + __builtin_ctzll(m);
                    if (i % (BLOCK / WAVE) == tid / WAVE) bk_wave_row(s_elem + s_start[u], deg(u));
                }
                for (m = __ballot(d > wave_most); m; m &= m - 1) {
                    const int u = v0 + __builtin_ctzll(m);
                    bk_block_sort_unique<BLOCK>(s_elem + s_start[u], deg(u));
                }
            }
            __syncthreads();
        }
        if (repeats && !lng) {  // (seldom) what is left of each row, by its thread
            uint32_t run = 0;
            for (int v0 = 0; v0 < nv; v0 += BLOCK) {
                const int v = v0 + tid;
                const uint32_t d = v < nv ? deg(v) : 0u;
                const uint32_t* const src = s_elem + (v < nv ? s_start[v] : 0u);
                uint32_t c = 0, sum;
                for (uint32_t i = 0; i < d; ++i) c += i == 0 || src[i] != src[i - 1] ? 1u : 0u;
                uint64_t at = ebase + run + bk_block_sum<BLOCK>(c, s_tmp, turn, &sum);
                run += sum;
                if (v < nv) a.erp[lo + v] = (int32_t)at;
                if ((int64_t)(at + c) > a.ecap) full = true;
                else
                    for (uint32_t i = 0; i < d; ++i)
                        if (i == 0 || src[i] != src[i - 1]) a.ecols[at++] = (int32_t)src[i];
            }
            if (u.last && tid == 0) a.erp[a.mp.n_vert] = (int32_t)(ebase + run);
        } else if (!repeats) {
            for (int v = tid; v < nv; v += BLOCK) a.erp[lo + v] = (int32_t)(ebase + s_start[v]);
            if (u.last && tid == 0) a.erp[a.mp.n_vert] = (int32_t)(ebase + n);
            if ((int64_t)(ebase + n) > a.ecap) full = true;
            else
                for (uint32_t i = tid; i < n; i += BLOCK) a.ecols[ebase + i] = (int32_t)s_elem[i];
        }
        elem = !(repeats && lng);
    }

    // ---- node rows out
    if (K > 0 && node && !crowded && !stuck) nodes_out();
    if (full) set_error(a.hdr + HDR_ERR, ERR_CAPACITY);
    // (records beyond the room there is, of an ill-formed mixed mesh, are missing)
    if (bad && !(odd & BK_BAD_ID)) set_error(a.hdr + HDR_ERR, ERR_INTERNAL);
    return (stuck ? 0 : BK_NODE_DONE) | (elem ? BK_ELEM_DONE : 0);
}

// Unit u, of a bucket of n records from rec0 on, the r0-th pair of all: both its
// relations.  Every thread of the block calls it.
template <int K, int W, bool LARGE>
__device__ __forceinline__ void bk_unit_rows(const BkRowsArgs& a, const BkUnit& u, int64_t rec0, uint32_t n, uint32_t r0,
                                             uint32_t lo, int nv, uint32_t odd, uint32_t* s_all, uint32_t* s_tmp,
                                             uint64_t* s_base) {
    using S = BkShape<K, LARGE>;
    using L = BkLds<K, LARGE>;
    uint32_t* const s_val = s_all;
    uint32_t* const s_start = s_val + L::VAL;       // row starts
    uint32_t* const s_cnt = s_start + S::VMAX + 1;  // distinct neighbours, then their offsets
    uint16_t* const s_pos = reinterpret_cast<uint16_t*>(s_cnt + S::VMAX + 1);  // bk_ranges
    const int tid = bk_tid();
    if (nv < 0 || nv > S::VMAX) {  // never: the plan keeps a bucket's vertices below VMAX
        if (tid == 0) set_error(a.hdr + HDR_ERR, ERR_INTERNAL);
        return;
    }
    const bool node = K > 0 && a.nrp != nullptr, elem = a.erp != nullptr;
    int turn = 0;
    // where the element rows start: records less repeats of the earlier buckets
    uint64_t ebase = r0;
    bool repeats = false;
    if (odd & BK_HAS_DUP) {
        uint32_t sum = 0, total;
        for (uint32_t b = tid; b < u.bucket; b += S::BLOCK) sum += a.repeats[b];
        bk_block_sum<S::BLOCK>(sum, s_tmp, &turn, &total);
        ebase -= total;
        repeats = __builtin_amdgcn_readfirstlane((int)a.repeats[u.bucket]) != 0;
    }
    int done = 0;
    if (u.shares == 1 && n <= (uint32_t)S::CAP)
        done = bk_rows_lds<K, W, LARGE>(a, u, rec0, n, lo, nv, odd, elem, repeats, ebase, s_val, s_start, s_cnt, s_tmp, &turn,
                                        s_base);
    const bool node_left = node && !(done & BK_NODE_DONE);
    const bool elem_left = elem && !(done & BK_ELEM_DONE);
#pragma unroll 1
    for (int rel = node_left ? 0 : 1, from = rel; rel < (elem_left ? 2 : 1); ++rel) {
        bk_ranges<K, W, LARGE>(a, rel == 1, repeats, u, rec0, n, lo, nv, ebase, a.list ? a.list + r0 : nullptr, rel != from, s_val,
                               s_start, s_cnt, s_pos, s_tmp, &turn, s_base);
    }
}

// The unit of a ticket: a bucket, where no bucket has shares.
__device__ __forceinline__ BkUnit bk_unit_of(uint32_t ticket, uint32_t n_unit, uint32_t n_bucket,
                                             const uint32_t* __restrict__ units) {
    BkUnit u{ticket, ticket, 0, 1, ticket + 1 == n_unit};
    if (n_unit != n_bucket) {
        u.bucket = (uint32_t)bk_find(units, (int)n_bucket, ticket);
        const uint32_t u0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)units[u.bucket]);
        u.share = ticket - u0;
        u.shares = (uint32_t)__builtin_amdgcn_readfirstlane((int)units[u.bucket + 1]) - u0;
    }
    return u;
}

template <int K, int W, bool LARGE>
__global__ __launch_bounds__((BkShape<K, LARGE>::BLOCK)) __attribute__((amdgpu_waves_per_eu(4)))
void bk_rows_kernel(BkRowsArgs a) {
    using S = BkShape<K, LARGE>;
    __shared__ __align__(16) uint32_t s_all[BkLds<K, LARGE>::WORDS];
    __shared__ uint32_t s_tmp[2 * (S::BLOCK / WAVE)];
    __shared__ uint32_t s_ticket;
    __shared__ uint64_t s_base;
    // the same for every thread: scalar registers
    const uint32_t odd = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.hdr[HDR_BK_ODD]);
    const uint32_t n_unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.hdr[HDR_BK_UNITS]);
    do {
        if (threadIdx.x == 0) s_ticket = atomicAdd(&a.hdr[HDR_BK_TICKET], 1u);  // so that every earlier unit is already running
        __syncthreads();
        const uint32_t ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_ticket);
        if (ticket >= n_unit) return;
        const BkUnit u = bk_unit_of(ticket, n_unit, a.mp.n_bucket, a.units);
        const uint32_t r0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.starts[u.bucket]);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.starts[u.bucket + 1]) - r0;
        uint32_t mul = a.mp.mul;
        asm volatile("" : "+s"(mul));  // (as bk_tid)
        const uint32_t lo = bk_first_vertex(u.bucket, mul);
        const uint32_t hi = u.bucket + 1 == a.mp.n_bucket ? (uint32_t)a.mp.n_vert : bk_next_first_vertex(lo, u.bucket, mul);
        bk_unit_rows<K, W, LARGE>(a, u, r0, n, r0, lo, (int)(hi - lo), odd, s_all, s_tmp, &s_base);
        if (n_unit == a.mp.n_bucket) return;  // (a block per bucket)
        __syncthreads();                      // before the LDS is used again
    } while (true);
}

}  // namespace mnb
