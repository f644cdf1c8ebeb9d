// Vertex buckets: both relations of a mesh from one partition of its
// (vertex, element) pairs, each bucket finished inside one block's LDS.
//
// The pairs of Sec. 2.1.2, each carrying the vertex's edge-neighbours inside
// that element (Sec. 2.1.1), are scattered once into buckets of consecutive
// vertices small enough for the LDS of a CU.  A bucket then holds everything
// its rows need: its block groups the pairs by vertex, orders and
// deduplicates both kinds of rows and writes both CSRs, so there is no sort
// over all pairs, no second look at the connectivity and no staging of rows
// in memory.
//
//   bk_hist   conn -> pairs per bucket, per tile and per block of tiles
//   bk_scan   where every block's pairs of a bucket go; bucket starts
//   bk_part   conn -> records, each tile ordered by bucket in LDS, written at
//             offsets that are known beforehand (no tile waits for another)
//   bk_rows   one block per bucket, or several for one with many records:
//             both CSRs (buckets.hpp's second half)
//
// Tiles are dealt to the XCDs in turn (tile t runs on XCD t mod 8 under the
// usual round-robin dispatch), and a bucket's space is laid out by XCD first:
// the short runs that neighbouring tiles of one XCD write side by side meet in
// that XCD's L2 and leave it as whole lines.  (25.1 M 12-byte records into
// 2048 buckets on MI355X: 154 us this way, 220 us with each block keeping a
// contiguous share of every bucket; the 3582 that 8.4 M triangles get: 168 us.)  The order is only a matter of speed.
#pragma once

#include "common.hpp"
#include "elements.hpp"
#include "internal.hpp"
#include "launch.hpp"

namespace mnb {

constexpr int BK_XCDS = 8;
constexpr uint32_t BK_EMPTY = 0xffffffffu;  // never an id (ids are below 2^31)

// Words of the workspace header this pipeline uses beyond the error word.
constexpr int HDR_BK_SCAN = 34;    // bk_scan's block ticket
constexpr int HDR_BK_ODD = 35;     // what bk_hist found (BK_BAD_ID, BK_HAS_DUP)
constexpr int HDR_BK_TICKET = 36;  // bk_rows' unit ticket
constexpr int HDR_BK_UNITS = 37;   // units of bk_rows: a bucket, or a share of one (bk_shares)
constexpr int HDR_BK_PROGRESS = 38;  // steps of long units, for those that wait
// Per-block findings of bk_hist.
constexpr uint32_t BK_BAD_ID = 1u;   // an id outside [0, n_vert)
constexpr uint32_t BK_HAS_DUP = 2u;  // an element repeats an id: it has more records than pairs

// Edge-neighbours of a node position: K of them (the type's largest count;
// a position with fewer repeats itself, which later drops out).
template <int ET>
struct BkElem {
    static constexpr int NPE = Elem<ET>::NPE;
    static constexpr int degree(int p) {
        int d = 0;
        for (int q = 0; q < NPE; ++q) d += (int)((adjacency_word<ET>() >> (8 * p + q)) & 1ull);
        return d;
    }
    static constexpr int max_degree() {
        int m = 0;
        for (int p = 0; p < NPE; ++p) m = degree(p) > m ? degree(p) : m;
        return m;
    }
    static constexpr int K = max_degree();
    static constexpr int nbr(int p, int k) {
        int d = 0;
        for (int q = 0; q < NPE; ++q)
            if ((adjacency_word<ET>() >> (8 * p + q)) & 1ull) {
                if (d == k) return q;
                ++d;
            }
        return p;
    }
};

// bucket(v) = (v * mul) >> 32: about 2^32 / mul consecutive vertices each.
__host__ __device__ inline uint32_t bk_first_vertex(uint32_t bucket, uint32_t mul) {
    return (uint32_t)((((uint64_t)bucket << 32) + mul - 1) / mul);
}
// The next bucket's, from this one's (lo): one division, and of 32 bits.
__host__ __device__ inline uint32_t bk_next_first_vertex(uint32_t lo, uint32_t bucket, uint32_t mul) {
    const uint32_t width = 0xffffffffu / mul;  // 2^32 / mul, or one less where mul divides it
    const uint64_t next = (uint64_t)(lo + width) * mul, end = (uint64_t)(bucket + 1) << 32;
    return lo + width + (next < end ? 1u : 0u);
}
__device__ __forceinline__ uint32_t bk_bucket(uint32_t v, uint32_t mul) { return __umulhi(v, mul); }

// bk_rows' look-backs, a word per unit each: node entries, and, within a shared
// bucket that has repeats (of a vertex in an element), element entries.
struct BkLookback {
    uint64_t *nodes, *elems;
    __device__ __forceinline__ void clear(uint32_t unit) const {
        nodes[unit] = 0;
        if (elems) elems[unit] = 0;
    }
    // (no element entries where no bucket is shared)
    static size_t bytes(int64_t units, bool shares) { return (size_t)units * (shares ? 2 : 1) * sizeof(uint64_t); }
    static BkLookback at(void* p, int64_t units, bool shares) {
        return {(uint64_t*)p, shares ? (uint64_t*)p + units : nullptr};
    }
};

// Blocks that share a bucket of n records.  Up to cap of them fit one block's
// LDS.  Beyond, every share reads all of the bucket's records (to count them by
// vertex, and to pick its own), so more of them sort more at a time and read more
// in all: 6 M records of 250 vertices took 11.6 / 7.6 / 5.4 / 8.2 / 17.8 ms with up
// to 32 / 64 / 128 / 256 / 512 shares, 600,000 of 250 vertices 1.7 / 1.1 / 0.8 /
// 0.8 / 0.8 ms.
constexpr uint32_t BK_SHARES = 128;
__host__ __device__ inline uint32_t bk_shares(uint32_t n, uint32_t cap) {
    return n <= cap ? 1u : tmin((n - 1) / (cap / 2) + 1, BK_SHARES);
}
// Most units that n_slots records in n_bucket buckets take.
inline int64_t bk_unit_most(int64_t n_bucket, int64_t n_slots, int64_t cap) { return n_bucket + n_slots / (cap / 2) + 1; }

// Inclusive sum over the lanes of a wave (DPP: no LDS round trips).
__device__ __forceinline__ uint32_t bk_wave_sum(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// What a plan with or without shares gives the kernels.
inline uint32_t* bk_units(const BkPlan& p, char* w) { return p.shares ? (uint32_t*)(w + p.off_units) : nullptr; }
inline BkLookback bk_lookback(const BkPlan& p, char* w) { return BkLookback::at(w + p.off_lb, p.unit_most, p.shares); }

// Largest i in [0, n) with off[i] <= x (off ascending from 0), found by a
// whole wave, 64 places at a time.
__device__ __forceinline__ int bk_find(const uint32_t* __restrict__ off, int n, uint32_t x) {
    const int lane = __lane_id();
    int lo = 0, len = n;
    while (len > 1) {
        const int step = (len + WAVE - 1) / WAVE;
        const bool ok = lane * step < len && off[lo + lane * step] <= x;
        const int k = (int)__popcll(__ballot(ok)) - 1;
        lo += k * step;
        len = tmin(step, len - k * step);
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// A record holds the element (e_bits), the low bits of the vertex (vl_bits)
// and its K neighbours (id_bits each) in W words, fewer words where they fit
// (bk_words):
//   W = K + 1        a word per neighbour after the element's; the vertex bits
//                    above the element's and, as far as they do not fit
//                    there, above the first neighbour's
//   K = 3, W = 3     the neighbours in 64 bits, the element and the vertex in 32
//   K = 2, W = 2     all in 64 bits
//   K = 0            element and vertex in one word, or a word each
__host__ __device__ inline int bk_words(int K, uint32_t e_bits, uint32_t id_bits, uint32_t vl_bits) {
    if (K == 0) return e_bits + vl_bits <= 32 ? 1 : 2;
    if (K == 2 && e_bits + vl_bits + 2 * id_bits <= 64) return 2;
    if (K == 3 && 3 * id_bits <= 64 && e_bits + vl_bits <= 32) return 3;
    return (32 - e_bits) + (32 - id_bits) >= vl_bits ? K + 1 : 0;  // 0: not at all
}
template <int K, int W>
__device__ __forceinline__ void bk_encode(const BkMap& m, uint32_t e, uint32_t v, const uint32_t (&nb)[K > 0 ? K : 1],
                                          uint32_t (&r)[W]) {
    const uint32_t vl = v & m.vl_mask;
    if constexpr (K == 0 && W == 2) {
        r[0] = e;
        r[1] = vl;
    } else if constexpr (K == 2 && W == 2) {
        const uint64_t x = (uint64_t)nb[0] | (uint64_t)nb[1] << m.id_bits | (uint64_t)vl << (2 * m.id_bits) |
                           (uint64_t)e << m.e_shift;
        r[0] = (uint32_t)x;
        r[1] = (uint32_t)(x >> 32);
    } else if constexpr (K == 3 && W == 3) {
        const uint64_t x = (uint64_t)nb[0] | (uint64_t)nb[1] << m.id_bits | (uint64_t)nb[2] << (2 * m.id_bits);
        r[0] = e | (vl << m.e_bits);
        r[1] = (uint32_t)x;
        r[2] = (uint32_t)(x >> 32);
    } else {
        r[0] = e | (vl << m.e_bits);
#pragma unroll
        for (int k = 0; k < K; ++k) r[1 + k] = nb[k];
        if constexpr (K > 0) r[1] |= (vl >> (32 - m.e_bits)) << m.id_bits;
    }
}
template <int W>
__device__ __forceinline__ uint64_t bk_pair(const uint32_t (&r)[W], int i) {
    return (uint64_t)r[i] | (uint64_t)r[i + 1] << 32;
}
// The row of a record inside its bucket (first vertex lo).
template <int K, int W>
__device__ __forceinline__ uint32_t bk_row(const BkMap& m, const uint32_t (&r)[W], uint32_t lo) {
    uint32_t vl;
    if constexpr (K == 0 && W == 2) vl = r[1];
    else if constexpr (K == 2 && W == 2) vl = (uint32_t)(bk_pair(r, 0) >> (2 * m.id_bits));
    else if constexpr (K == 0 || W == K) vl = r[0] >> m.e_bits;
    else vl = (r[0] >> m.e_bits) | ((r[1] >> m.id_bits) << (32 - m.e_bits));
    return (vl - lo) & m.vl_mask;
}
template <int K, int W>
__device__ __forceinline__ uint32_t bk_elem(const BkMap& m, const uint32_t (&r)[W]) {
    if constexpr (K == 0 && W == 2) return r[0];
    else if constexpr (K == 2 && W == 2) return (uint32_t)(bk_pair(r, 0) >> m.e_shift);
    else return r[0] & ((1u << m.e_bits) - 1);
}
template <int K, int W>
__device__ __forceinline__ uint32_t bk_nbr(const BkMap& m, const uint32_t (&r)[W], int k) {
    const uint32_t mask = (1u << m.id_bits) - 1;
    if constexpr (K == 2 && W == 2) return (uint32_t)(bk_pair(r, 0) >> (k * m.id_bits)) & mask;
    else if constexpr (K == 3 && W == 3) return (uint32_t)(bk_pair(r, 1) >> (k * m.id_bits)) & mask;
    else return k == 0 ? r[1] & mask : r[1 + k];
}

// Adds one to s[b] for every lane with `valid` and returns each one's old
// value plus its place among the wave's lanes of the same counter.  Every lane
// of the wave calls it.  Lanes that share a counter queue in the LDS, so where
// many do (an element order with locality; bk_crowded tells, once per wave
// and tile), one lane adds for all of them.
__device__ __forceinline__ bool bk_crowded(uint32_t b) {
    return __popcll(__ballot(b == (uint32_t)__builtin_amdgcn_readfirstlane((int)b))) >= 8;
}
__device__ __forceinline__ uint32_t bk_count(uint32_t* s, uint32_t b, bool valid, bool crowded) {
    uint32_t rank = 0;
    if (crowded) {
        uint64_t act = __ballot(valid);
        for (int it = 0; it < 3 && act; ++it) {
            const int lead = __builtin_ctzll(act);
            const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, lead);
            const uint64_t m = __ballot(valid && b == b0);
            uint32_t old = 0;
            if ((int)__lane_id() == lead) old = atomicAdd(&s[b0], (uint32_t)__popcll(m));
            old = (uint32_t)__builtin_amdgcn_readlane((int)old, lead);
            if (valid && b == b0) {
                rank = old + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                valid = false;
            }
            act &= ~m;
        }
    }
    if (valid) rank = atomicAdd(&s[b], 1u);
    return rank;
}

// ---- bk_hist ---------------------------------------------------------------------
// Block h = 8 k + x takes the tiles x + 8 (R k + r), r < R, in order; before
// each it writes down its counts so far (within), at the end all of them
// (btot).  A thread takes whole elements.  Bound by reading conn and by the
// LDS adds: 8.4 M triangles, 3582 buckets in 38 us (100 MB in, 26 MB out);
// 2 M with local labels 26 us, lanes of a wave in the same few counters.
template <int ET, int BLOCK, int EPT>
__global__ __launch_bounds__(BLOCK) void bk_hist_kernel(const int32_t* __restrict__ conn, int64_t n_elem, BkMap mp,
                                                       int64_t n_tiles, int R, uint16_t* __restrict__ within,
                                                       uint32_t* __restrict__ btot, uint32_t* __restrict__ flags,
                                                       uint64_t* __restrict__ scan_lb, int n_scan,
                                                       uint32_t* __restrict__ hdr) {
    constexpr int NPE = Elem<ET>::NPE;
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
        int32_t id[EPT][NPE] = {};
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const int64_t e = t * (BLOCK * EPT) + u * BLOCK + tid;
            if (e < n_elem) load_elem_ids<ET>(conn, e, id[u]);
        }
        uint32_t* wt = reinterpret_cast<uint32_t*>(within + t * nb);  // two counts per word (nb is even)
        for (int i = tid; i < nb / 2; i += BLOCK) wt[i] = s_h[2 * i] | (s_h[2 * i + 1] << 16);
        __syncthreads();
        const bool crowded = bk_crowded(bk_bucket((uint32_t)id[0][0], mp.mul));
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const bool in = t * (BLOCK * EPT) + u * BLOCK + tid < n_elem;
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
    }
    if (found) atomicOr(&s_flags, found);
    for (int i = tid; i < nb; i += BLOCK) btot[(int64_t)blockIdx.x * nb + i] = s_h[i];
    __syncthreads();
    if (tid == 0) flags[blockIdx.x] = s_flags;
}

// ---- bk_scan ---------------------------------------------------------------------
// btot[h][b] becomes the pairs of bucket b in the blocks before h (blocks in
// the order x, then k), starts[b] those of the buckets before b, and units[b]
// the units of the buckets before b (read only where some bucket has shares;
// summed above the pairs in one word): a block
// (by ticket) takes 16 buckets, 64 threads per bucket, each a run of blocks
// held in registers; the blocks' sums meet in a decoupled look-back.  (A last
// block that scanned all totals needed device-wide fences, each a write-back
// of an L2: 68 instead of 9 us on 2560 buckets x 392 blocks; 11 us on 3582 x 456.)  Block 0 sets
// the error word and the repeat flag from what bk_hist found.
constexpr int BKS_BLOCK = 1024;
constexpr int BKS_COLS = 16;
constexpr int BKS_ROWS = BKS_BLOCK / BKS_COLS;
constexpr int BKS_PER = 16;  // most hist blocks per thread
constexpr int BK_HIST_MOST = BKS_ROWS * BKS_PER;
static_assert(BKS_ROWS == WAVE && BKS_COLS == BKS_BLOCK / WAVE, "one wave scans a bucket's runs");

static __global__ __launch_bounds__(BKS_BLOCK) void bk_scan_kernel(uint32_t* __restrict__ btot, int hist_blocks,
                                                                  uint32_t n_bucket, uint32_t nb_pad,
                                                                  const uint32_t* __restrict__ flags,
                                                                  uint64_t* scan_lb, uint32_t* __restrict__ starts,
                                                                  uint32_t* __restrict__ units, uint32_t bucket_cap,
                                                                  uint32_t rec_cap, BkLookback lookback,
                                                                  uint32_t* __restrict__ repeats, uint32_t* hdr) {
    __shared__ uint32_t s_sum[BKS_ROWS][BKS_COLS + 1];
    __shared__ uint32_t s_tot[BKS_COLS];
    __shared__ uint32_t s_block;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid / WAVE;
    if (tid == 0) s_block = atomicAdd(&hdr[HDR_BK_SCAN], 1u);
    __syncthreads();
    const uint32_t block = s_block;
    const int c = tid % BKS_COLS, g = tid / BKS_COLS;
    const uint32_t col = block * BKS_COLS + c;
    const int per = (hist_blocks + BKS_ROWS - 1) / BKS_ROWS;
    const int kk = hist_blocks / BK_XCDS;
    uint32_t* cell[BKS_PER];
    uint32_t v[BKS_PER], sum = 0;
    int x = g * per / kk, k = g * per % kk;
#pragma unroll
    for (int i = 0; i < BKS_PER; ++i) {
        cell[i] = nullptr;
        if (i < per && g * per + i < hist_blocks && col < n_bucket) cell[i] = btot + (int64_t)(k * BK_XCDS + x) * nb_pad + col;
        v[i] = cell[i] ? *cell[i] : 0u;
        if (++k == kk) {
            k = 0;
            ++x;
        }
    }
#pragma unroll
    for (int i = 0; i < BKS_PER; ++i) sum += v[i];
    s_sum[g][c] = sum;
    __syncthreads();
    {  // wave w: the runs of bucket w
        const uint32_t r = s_sum[lane][wid];
        const uint32_t incl = wave_inclusive_sum(r);
        s_sum[lane][wid] = incl - r;
        if (lane == WAVE - 1) s_tot[wid] = incl;
    }
    __syncthreads();
    uint32_t run = s_sum[g][c];
#pragma unroll
    for (int i = 0; i < BKS_PER; ++i) {
        if (cell[i]) *cell[i] = run;
        run += v[i];
    }
    if (wid == 0) {
        const uint32_t b = block * BKS_COLS + lane;
        const bool have = lane < BKS_COLS && b < n_bucket;
        const uint32_t t = have ? s_tot[lane] : 0u;
        uint32_t more = 0, more_incl = 0;
        if (__ballot(t > bucket_cap)) {  // (seldom, and a division)
            more = bk_shares(t, bucket_cap) - 1;
            more_incl = bk_wave_sum(more);
        }
        const uint64_t mine = (uint64_t)more << 32 | t, incl = (uint64_t)more_incl << 32 | bk_wave_sum(t);
        const uint64_t all = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(incl >> 32), WAVE - 1) << 32 |
                             (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
        if (lane == 0) lb_store(scan_lb + block, (block == 0 ? LB_INC : LB_AGG) | all);
        const uint64_t before = wave_lookback_prefix(scan_lb, block, all, hdr + HDR_ERR);
        if (have) {
            // (never more than the records there is room for, which overlapping
            // elements of an ill-formed mixed mesh could ask for)
            const uint64_t to = before + incl, from = to - mine;
            const uint32_t u = b + (uint32_t)(from >> 32);
            starts[b] = tmin((uint32_t)from, rec_cap);
            if (units) units[b] = u;
            for (uint32_t i = 0; i <= more; ++i) lookback.clear(u + i);
            repeats[b] = 0;  // counted by bk_part
            if (b + 1 == n_bucket) {
                starts[n_bucket] = tmin((uint32_t)to, rec_cap);
                if (units) units[n_bucket] = u + more + 1;
                hdr[HDR_BK_UNITS] = u + more + 1;
            }
        }
    }
    if (block != 0) return;
    uint32_t f = 0;
    for (int h = tid; h < hist_blocks; h += BKS_BLOCK) f |= flags[h];
    const bool bad = __syncthreads_or(f & BK_BAD_ID), dup = __syncthreads_or(f & BK_HAS_DUP);
    if (tid == 0) {
        if (bad) set_error(hdr + HDR_ERR, ERR_INDEX_RANGE);
        hdr[HDR_BK_ODD] = (bad ? BK_BAD_ID : 0u) | (dup ? BK_HAS_DUP : 0u);
    }
}

// ---- bk_part ---------------------------------------------------------------------
// A tile's counts become offsets in it, in place, and each bucket's first place
// loses its offset; returns the tile's records.  Starts and ends with a barrier.
template <int BLOCK>
__device__ __forceinline__ uint32_t bk_tile_offsets(uint32_t* s_cnt, uint32_t* s_glob, int nb, uint32_t* s_tmp) {
    const int tid = threadIdx.x;
    __syncthreads();
    const int per = (nb + BLOCK - 1) / BLOCK;  // a thread takes consecutive buckets
    uint32_t sum = 0;
    for (int i = 0; i < per; ++i) {
        const int b = tid * per + i;
        if (b < nb) sum += s_cnt[b];
    }
    uint32_t total;
    uint32_t run = block_exclusive_sum<BLOCK>(sum, s_tmp, &total);
    for (int i = 0; i < per; ++i) {
        const int b = tid * per + i;
        if (b < nb) {
            const uint32_t c = s_cnt[b];
            s_cnt[b] = run;
            s_glob[b] -= run;
            run += c;
        }
    }
    __syncthreads();
    return total;
}
// A tile's records, in bucket order in the LDS, to their places.  False if one
// is beyond the room for records.
template <int W, int BLOCK>
__device__ __forceinline__ bool bk_tile_out(const uint32_t* s_rec, const uint16_t* s_b, const uint32_t* s_glob,
                                            uint32_t total, uint32_t* __restrict__ rec, int64_t rec_cap) {
    struct Words {
        uint32_t w[W];
    };
    bool fits = true;
    for (uint32_t i = threadIdx.x; i < total; i += BLOCK) {
        const uint32_t d = s_glob[s_b[i]] + i;
        Words r;
#pragma unroll
        for (int q = 0; q < W; ++q) r.w[q] = s_rec[i * W + q];
        if ((int64_t)d < rec_cap) reinterpret_cast<Words*>(rec)[d] = r;
        else fits = false;
    }
    return fits;
}

// Elements [e0, e0 + count) of a tile.  Its records' buckets are counted (each
// record keeps its place among the tile's records of that bucket), the counts
// scanned, the records put in bucket order in LDS and written out: consecutive
// lanes write consecutive records, a run per bucket, bucket b's from first(b)
// on.  A slot whose id is out of range has no record; a neighbour that is out
// of range or the vertex itself is stored as the vertex, which its row drops.
// s_dyn: two words per bucket, the records, a 16-bit bucket number each.
template <int ET, int K, int W, int BLOCK, int EPT, class First>
__device__ __forceinline__ void bk_part_tile(const int32_t* __restrict__ conn, int64_t e0, int32_t count,
                                             const BkMap& mp, First&& first, uint32_t* __restrict__ rec,
                                             int64_t rec_cap, uint32_t* repeats, uint32_t* hdr, uint32_t* s_dyn,
                                             uint32_t* s_tmp) {
    using E = BkElem<ET>;
    constexpr int NPE = E::NPE;
    constexpr int T = BLOCK * EPT * NPE;
    static_assert(T <= 65535, "16-bit places");
    const int nb = (int)mp.nb_pad;
    uint32_t* const s_cnt = s_dyn;        // counts, then offsets
    uint32_t* const s_glob = s_dyn + nb;  // where the bucket's first record goes, less its offset
    uint32_t* const s_rec = s_glob + nb;
    uint16_t* const s_b = reinterpret_cast<uint16_t*>(s_rec + count * NPE * W);
    const int tid = threadIdx.x;
    const bool dup = (hdr[HDR_BK_ODD] & BK_HAS_DUP) != 0;
    int32_t id[EPT][NPE] = {};
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const int32_t i = u * BLOCK + tid;
        if (i < count) load_elem_ids<ET>(conn, e0 + i, id[u]);
    }
    for (int i = tid; i < nb; i += BLOCK) {
        s_cnt[i] = 0;
        s_glob[i] = i < (int)mp.n_bucket ? first(i) : 0u;
    }
    __syncthreads();
    uint32_t place[EPT][(NPE + 1) / 2] = {};  // two 16-bit places per word
    const bool crowded = bk_crowded(bk_bucket((uint32_t)id[0][0], mp.mul));
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const bool in = u * BLOCK + tid < count;
#pragma unroll
        for (int j = 0; j < NPE; ++j) {
            const uint32_t v = (uint32_t)id[u][j];
            const bool ok = in && v < (uint32_t)mp.n_vert;
            place[u][j / 2] |= bk_count(s_cnt, ok ? bk_bucket(v, mp.mul) : 0u, ok, crowded) << (16 * (j & 1));
        }
    }
    const uint32_t total = bk_tile_offsets<BLOCK>(s_cnt, s_glob, nb, s_tmp);
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const int32_t i = u * BLOCK + tid;
#pragma unroll
        for (int j = 0; j < NPE; ++j) {
            const uint32_t v = (uint32_t)id[u][j];
            if (i >= count || v >= (uint32_t)mp.n_vert) continue;
            const uint32_t b = bk_bucket(v, mp.mul);
            const uint32_t p = s_cnt[b] + ((place[u][j / 2] >> (16 * (j & 1))) & 0xffffu);
            if (dup) {  // (seldom: some element of the mesh repeats an id)
                bool again = false;
#pragma unroll
                for (int jj = 0; jj < j; ++jj) again |= (uint32_t)id[u][jj] == v;
                if (again) atomicAdd(&repeats[b], 1u);
            }
            uint32_t nbr[K > 0 ? K : 1] = {};
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t w = (uint32_t)id[u][E::nbr(j, k)];
                nbr[k] = w < (uint32_t)mp.n_vert ? w : v;
            }
            uint32_t r[W];
            bk_encode<K, W>(mp, (uint32_t)(e0 + i), v, nbr, r);
#pragma unroll
            for (int q = 0; q < W; ++q) s_rec[p * W + q] = r[q];
            s_b[p] = (uint16_t)b;
        }
    }
    __syncthreads();
    // (beyond it only if conn changed under the call)
    if (!bk_tile_out<W, BLOCK>(s_rec, s_b, s_glob, total, rec, rec_cap)) set_error(hdr + HDR_ERR, ERR_INTERNAL);
}

// Tile t = blockIdx.x.  Bound by the writes' lines: 25.1 M records of 12 bytes
// (100 MB in, 302 MB out), 112 / 154 / 199 us for 1024 / 2048 / 4096 buckets
// (runs of 108 / 54 / 27 bytes).
template <int ET, int K, int W, int BLOCK, int EPT>
__global__ __launch_bounds__(BLOCK) void bk_part_kernel(const int32_t* __restrict__ conn, int64_t n_elem, BkMap mp,
                                                       int R, const uint16_t* __restrict__ within,
                                                       const uint32_t* __restrict__ btot,
                                                       const uint32_t* __restrict__ starts,
                                                       uint32_t* __restrict__ rec, int64_t rec_cap,
                                                       uint32_t* repeats, uint32_t* hdr) {
    constexpr int TE = BLOCK * EPT;
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_tmp[BLOCK / WAVE];
    const int64_t t = blockIdx.x;
    const int64_t h = (t / BK_XCDS / R) * BK_XCDS + t % BK_XCDS;
    const int nb = (int)mp.nb_pad;
    bk_part_tile<ET, K, W, BLOCK, EPT>(
        conn, t * TE, (int32_t)tmin<int64_t>(n_elem - t * TE, TE), mp,
        [&](int b) { return starts[b] + btot[h * nb + b] + within[t * nb + b]; }, rec, rec_cap, repeats, hdr, s_dyn, s_tmp);
}

// The tile shapes: threads x elements per thread.  A large tile fills most of
// a CU's LDS (records and their bucket numbers; what is left, 34 KB for
// triangles' three words and 50 KB for hexahedra's four, holds two words per
// bucket and so bounds their number: 4320 and 6624).  Small tiles spread a small
// mesh's elements over the CUs, and take what has more buckets than that.
template <int ET>
struct BkTile;
template <> struct BkTile<TRI3> { static constexpr int BLOCK = 1024, EPT = 3; };
template <> struct BkTile<QUAD4> { static constexpr int BLOCK = 1024, EPT = 2; };
template <> struct BkTile<TET4> { static constexpr int BLOCK = 768, EPT = 2; };
template <> struct BkTile<HEX8> { static constexpr int BLOCK = 768, EPT = 1; };
template <> struct BkTile<WEDGE6> { static constexpr int BLOCK = 1024, EPT = 1; };
template <> struct BkTile<PYR5> { static constexpr int BLOCK = 1024, EPT = 1; };
constexpr int BK_SMALL_BLOCK = 256;
constexpr int BK_LDS = 160 * 1024;

}  // namespace mnb
