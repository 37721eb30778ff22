// Row analysis: per-row product counts, tier/bin assignment, prefix scans,
// the column-window table of B, and optional input validation.
#pragma once

#include "device_common.hpp"

namespace wsp {

// ---------------------------------------------------------------------------
// Device-wide exclusive scan (int64 output) of a generated sequence: tile sums,
// and tile scans that add up the sums before their tile (up to kScanOwnTiles
// tiles; past them a third launch between the two scans the sums). One tile is
// scanned in one launch, and short sequences by scan_one_block.
// ---------------------------------------------------------------------------
constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanBlock * kScanItems;

// Length of the B row that multiplies A entry i: B.row_ptr[k+1] - B.row_ptr[k]
// with k = A.col_idx[i].
struct BRowLenIn {
    const int32_t *a_col;
    const int32_t *b_rp;
    __device__ __forceinline__ int64_t operator()(int64_t i) const {
        const int32_t k = a_col[i];
        return static_cast<int64_t>(b_rp[k + 1] - b_rp[k]);
    }
};

struct CountIn {
    const int32_t *cnt;
    __device__ __forceinline__ int64_t operator()(int64_t i) const { return cnt[i]; }
};

// Where an input ends that only the device knows (In::end()): past it the
// tiled scan reads nothing and writes nothing (no total at out[n] either); up
// to and with it out is written as ever. Other inputs end at n.
template <typename In>
__device__ __forceinline__ auto scan_end(const In &in, int64_t, int) -> decltype(in.end()) {
    return in.end();
}
template <typename In>
__device__ __forceinline__ int64_t scan_end(const In &, int64_t n, long) {
    return n;
}

template <typename In>
__global__ void __launch_bounds__(kScanBlock) scan_tile_sums(In in, int64_t n, int64_t *partials) {
    __shared__ int64_t red[kScanBlock / kWave];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
    int64_t s = 0;
    if (base >= scan_end(in, n, 0)) {
        if (threadIdx.x == 0) partials[blockIdx.x] = 0;
        return;
    }
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        const int64_t idx = base + static_cast<int64_t>(i) * kScanBlock + threadIdx.x;
        if (idx < n) s += in(idx);
    }
    s = block_sum<kScanBlock>(s, red);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// One block: exclusive scan of partials[0..nb) in place; partials[nb] = total.
__global__ void __launch_bounds__(1024) scan_partials(int64_t *partials, int64_t nb) {
    __shared__ int64_t wsum[16];
    __shared__ int64_t carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    const int ln = lane_id();
    const int w = threadIdx.x / kWave;
    for (int64_t c0 = 0; c0 < nb; c0 += 1024) {
        const int64_t idx = c0 + threadIdx.x;
        const int64_t v = idx < nb ? partials[idx] : 0;
        int64_t incl = v;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int64_t y = __shfl_up(incl, o, kWave);
            if (ln >= o) incl += y;
        }
        if (ln == kWave - 1) wsum[w] = incl;
        __syncthreads();
        int64_t before = carry_s, tot = 0;
        for (int i = 0; i < 16; ++i) {
            before += (i < w) ? wsum[i] : 0;
            tot += wsum[i];
        }
        if (idx < nb) partials[idx] = before + incl - v;
        __syncthreads();
        if (threadIdx.x == 0) carry_s += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[nb] = carry_s;
}

// What a scan's output adds to a checksum of it: the sum of out[i] * (2i + 1)
// for i <= n, modulo 2^64, one atomic per workgroup.
template <int BLOCK>
__device__ __forceinline__ void add_checksum(uint64_t acc, uint64_t *sum, int64_t *scratch) {
    acc = static_cast<uint64_t>(block_sum<BLOCK>(static_cast<int64_t>(acc), scratch));
    if (threadIdx.x == 0)
        atomicAdd(reinterpret_cast<unsigned long long *>(sum), static_cast<unsigned long long>(acc));
}

// out[i] = exclusive prefix for i < n, out[n] = total. OWN: partials holds the
// tile sums themselves, and each workgroup adds up those before its tile (a few
// hundred numbers, in the L2: one launch less). csum (or null) receives out's
// checksum.
constexpr int64_t kScanOwnTiles = 1024;   // tiles a workgroup adds up by itself at most
template <typename In, bool OWN>
__global__ void __launch_bounds__(kScanBlock) scan_tiles(In in, int64_t n, const int64_t *partials,
                                                         int64_t nb, int64_t *out, uint64_t *csum,
                                                         int64_t *host_total) {
    __shared__ int64_t wsum[kScanBlock / kWave];
    int64_t first = 0;
    if (static_cast<int64_t>(blockIdx.x) * kScanTile > scan_end(in, n, 0)) return;
    if constexpr (OWN) {
        for (int64_t i = threadIdx.x; i < blockIdx.x; i += kScanBlock) first += partials[i];
        first = block_sum<kScanBlock>(first, wsum);
    } else {
        first = partials[blockIdx.x];
    }
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        const int64_t idx = base + i;
        v[i] = idx < n ? in(idx) : 0;
        s += v[i];
    }
    const int ln = lane_id();
    const int w = threadIdx.x / kWave;
    int64_t incl = s;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(incl, o, kWave);
        if (ln >= o) incl += y;
    }
    if (ln == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int64_t run = first;
    for (int i = 0; i < kScanBlock / kWave; ++i) run += (i < w) ? wsum[i] : 0;
    run += incl - s;
    uint64_t acc = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        const int64_t idx = base + i;
        if (idx < n) {
            out[idx] = run;
            acc += static_cast<uint64_t>(run) * static_cast<uint64_t>(2 * idx + 1);
        }
        run += v[i];
    }
    // the last item of the last tile: run is the total
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanBlock - 1) {
        out[n] = run;
        if (host_total != nullptr) *host_total = run;
        acc += static_cast<uint64_t>(run) * static_cast<uint64_t>(2 * n + 1);
    }
    if (csum != nullptr) {
        __syncthreads();
        add_checksum<kScanBlock>(acc, csum, wsum);
    }
}

// The same exclusive scan in one workgroup of 1024 threads, for short
// sequences of cheap inputs (one launch instead of two): thread t sums its
// contiguous share, the workgroup scans the shares, and each thread writes its
// share's prefixes. out[n] = total.
template <typename In>
__global__ void __launch_bounds__(1024) scan_one_block(In in, int64_t n, int64_t *out, uint64_t *csum,
                                                       int64_t *host_total) {
    __shared__ int64_t wsum[16];
    const int64_t per = (n + 1023) / 1024;
    const int64_t b = static_cast<int64_t>(threadIdx.x) * per;
    const int64_t e = b + per < n ? b + per : n;
    int64_t s = 0;
    for (int64_t i0 = b; i0 < e; i0 += 8) {   // eight loads in flight at a time
        int64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = i0 + u < e ? in(i0 + u) : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    const int ln = lane_id();
    const int w = threadIdx.x / kWave;
    int64_t incl = s;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(incl, o, kWave);
        if (ln >= o) incl += y;
    }
    if (ln == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int64_t run = 0, tot = 0;
    for (int i = 0; i < 16; ++i) {
        run += i < w ? wsum[i] : 0;
        tot += wsum[i];
    }
    run += incl - s;
    uint64_t acc = 0;
    for (int64_t i0 = b; i0 < e; i0 += 8) {
        int64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = i0 + u < e ? in(i0 + u) : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (i0 + u < e) {
                out[i0 + u] = run;
                acc += static_cast<uint64_t>(run) * static_cast<uint64_t>(2 * (i0 + u) + 1);
            }
            run += v[u];
        }
    }
    if (threadIdx.x == 0) {
        out[n] = tot;
        if (host_total != nullptr) *host_total = tot;
        acc += static_cast<uint64_t>(tot) * static_cast<uint64_t>(2 * n + 1);
    }
    if (csum != nullptr) {
        __syncthreads();
        add_checksum<1024>(acc, csum, wsum);
    }
}

// ---------------------------------------------------------------------------
// Row product counts. One pass over A's entries gathers the lengths of the B
// rows they select: loc[i] is the exclusive prefix of the lengths within entry
// i's tile of kScanTile entries, tile_sum[t] the tile's total. A row's products
// are the difference of its ends' prefixes plus the totals of the tiles between
// (none for nearly every row), so no second pass adds the tiles' offsets in
// (the gather is what a pass costs: 8 M entries 47 us for the sums and 79 us for
// the prefixes before, one pass of 51 us now). The first workgroup also clears the
// control blocks and the stamp it is given, which nothing else touches meanwhile.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kScanBlock) brow_tile_prefix(const int32_t *__restrict__ a_col,
                                                               const int32_t *__restrict__ b_rp, int64_t nnz,
                                                               int64_t *__restrict__ loc,
                                                               int64_t *__restrict__ tile_sum, int32_t *clear0,
                                                               int32_t *clear1, int clear_words, Stamp *stamp) {
    // (a gap after every kScanItems items: threads walk kScanItems consecutive ones each)
    constexpr int ITEM = kScanItems + 1;
    __shared__ int64_t s_len[kScanBlock * ITEM];
    __shared__ int64_t wsum[kScanBlock / kWave];
    const BRowLenIn in{a_col, b_rp};
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
    int64_t v[kScanItems];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        const int64_t idx = base + i * kScanBlock + threadIdx.x;
        v[i] = idx < nnz ? in(idx) : 0;
    }
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < clear_words; i += kScanBlock) {
            if (clear0 != nullptr) clear0[i] = 0;
            if (clear1 != nullptr) clear1[i] = 0;
        }
        if (stamp != nullptr && threadIdx.x == 0) *stamp = Stamp{};
    }
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        const int p = i * kScanBlock + threadIdx.x;
        s_len[p + p / kScanItems] = v[i];
    }
    __syncthreads();
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = s_len[threadIdx.x * ITEM + i];
        s += v[i];
    }
    const int ln = lane_id();
    const int w = threadIdx.x / kWave;
    int64_t incl = s;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(incl, o, kWave);
        if (ln >= o) incl += y;
    }
    if (ln == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int64_t run = incl - s;
    for (int i = 0; i < w; ++i) run += wsum[i];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        s_len[threadIdx.x * ITEM + i] = run;
        run += v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        const int p = i * kScanBlock + threadIdx.x;
        if (base + p <= nnz) loc[base + p] = s_len[p + p / kScanItems];
    }
    if (threadIdx.x == kScanBlock - 1) tile_sum[blockIdx.x] = run;
}

// Products of a row holding A's entries [lo, hi) (0 where this lane has none);
// all lanes of a wave call it. An end at the very end of the entries and of a
// tile has no prefix of its own: its tile begins there. Each lane adds up the
// tiles its row spans, but rows that would keep the wave waiting are added up by
// the whole wave, four loads in flight per lane: those of more than kRowTiles
// tiles for every lane that has so many (a tile costs a lane 76 ns, a row the
// wave about 1 us; one row of 20 M entries, 9766 tiles: the pass 848 us with a
// lane alone, now 119 us; 64 rows of 49 tiles each 60 us, 24 us more by the wave).
constexpr int kRowTiles = 16;
__device__ __forceinline__ int64_t row_products_of(int lo, int hi, int64_t nnz, const int64_t *__restrict__ loc,
                                                   const int64_t *__restrict__ tile_sum) {
    const bool some = lo < hi;
    const int ta = lo / kScanTile, tb = hi / kScanTile;
    int64_t f = 0;
    if (some) f = (hi == nnz && hi % kScanTile == 0 ? 0 : loc[hi]) - loc[lo];
    const int tiles = some ? tb - ta : 0;
    if (ballot(tiles > 0) == 0ull) return f;
    const int many = static_cast<int>(__popcll(ballot(tiles > kRowTiles)));
    const bool by_wave = tiles > kRowTiles * (many > 0 ? many : 1);
    if (!by_wave)
        for (int t = ta; t < ta + tiles; ++t) f += tile_sum[t];
    for (uint64_t left = ballot(by_wave); left != 0ull; left &= left - 1) {
        const int l = __ffsll(static_cast<long long>(left)) - 1;
        const int t1 = __builtin_amdgcn_readlane(tb, l);
        int64_t s[4] = {0, 0, 0, 0};
        for (int t = __builtin_amdgcn_readlane(ta, l) + lane_id(); t < t1; t += 4 * kWave) {
#pragma unroll
            for (int u = 0; u < 4; ++u) s[u] += t + u * kWave < t1 ? tile_sum[t + u * kWave] : 0;
        }
        const int64_t sum = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
        if (lane_id() == l) f += sum;
    }
    return f;
}

// out[i] = products of row i, for every row (the counts the binning uses). The
// first thread ends the workspace's stamp unless it is of this problem and
// layout (`own`), whose kept state has no array in common with these counts.
__global__ void __launch_bounds__(256) row_products_kernel(const int32_t *__restrict__ a_rp, int64_t nnz,
                                                           const int64_t *__restrict__ loc,
                                                           const int64_t *__restrict__ tile_sum, int64_t m,
                                                           int64_t *__restrict__ out, Stamp *stamp, const Stamp own) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i == 0 && !stamp->same_problem(own)) stamp->magic = 0;
    const int64_t f = row_products_of(i < m ? a_rp[i] : 0, i < m ? a_rp[i + 1] : 0, nnz, loc, tile_sum);
    if (i < m) out[i] = f;
}

// ---------------------------------------------------------------------------
// Binning.
// ---------------------------------------------------------------------------
struct BinCfg {
    int64_t ncols;          // columns of B (and C)
    int64_t dense_min_nnz;  // numeric: rows with at least this many entries go dense
    int32_t tiny_max;       // 0 disables the register tier
    int32_t hash_log2_max;  // largest LDS hash table (log2 slots)
    int32_t force_spill;
    int32_t dense_ok;       // the dense tier can take rows of this problem
    int32_t numeric;        // 0: symbolic bins, 1: numeric bins
    int32_t merge_products; // 1: merged rows' products are formed (numeric phase, single pass), 0: counted
    int32_t merge_runs;     // rows of at most this many A entries ...
    int32_t merge_places;   // ... and this many places in LDS are merged (0: none),
    int32_t merge_over_dense;   // rows the dense tier would take up to this many places;
    int32_t merge_long;         // and up to this many products piece by piece (numeric)
};

__device__ __forceinline__ int class_of(int64_t f) {
    // heavier rows get lower class ids (launched first)
    int l = 63 - __clzll(static_cast<unsigned long long>(f > 0 ? f : 1));
    int c = l - 10;
    c = c < 0 ? 0 : (c >= kNumClasses ? kNumClasses - 1 : c);
    return kNumClasses - 1 - c;
}

// Whether a row of f products, which takes `places` places merged, costs less
// there than in an LDS hash table. Merging costs as its kernel's size (the next
// power of two of the places) and a little per pass, hashing as the table's (l by
// the products: columns that repeat make the table smaller but not the inserts
// fewer). Short runs are what hashing is for: their padding makes the kernel
// larger than the table (64 A entries of 2 products each: counted 5.7 ns a row
// merged and 0.93 hashed, formed 6.4 and 2.5).
//
// Formed: equal sizes are merged, up to 512 places from 129 products on (where
// the table's sorted emission takes 5 ns a row) and up to 256 below. At 2048
// places and more the table costs less unless the padding is small (64 entries
// of 16: merged 14.7 ns, hashed 11; 32 of 32: 12.8 and 13.1). C of so many
// columns that the table's rank emission takes more than eight windows makes
// hashing cost twice as much and more, so there the next size is merged too (2 M
// columns, 48 entries of 6: 6.4 and 11.6 ns).
// Counted: the table holds keys alone, so the padding counts for more: at most
// 2.25 places per product, and from 2048 places on only where they are no more
// than the products' power of two or a quarter above the products (48 entries of
// 12: merged 5.9 ns, hashed 3.8; 8 of 128: 3.9 and 5.5).
// Over 2 to 64 A entries of 1 to 256 products each, at 100 K to 2 M columns (1160
// timed pairs), the choice costs 0.7% more than the better of the two on average
// and 24% at most (merging all of them: 30% and 6 times).
__device__ __forceinline__ bool merge_pays(int64_t f, int64_t places, const BinCfg &cfg) {
    int lm = ceil_log2(places);
    if (lm < kMergeLog2Min) lm = kMergeLog2Min;
    if (cfg.merge_products) {
        const int l = ceil_log2(f + (f >> 1));
        const int least = f > 128 ? 9 : 8;
        const int same = l > least ? l : least;
        if (f > 128 && cfg.ncols > (int64_t(512) << l)) return lm <= same + 1;
        return lm <= same && (lm < 11 || 20 * places <= 27 * f);
    }
    const int l = ceil_log2(2 * f);
    return lm <= (l > kMergeLog2Min ? l : kMergeLog2Min) && 4 * places <= 9 * f &&
           (lm < 11 || lm <= ceil_log2(f) || 4 * places <= 5 * f);
}

// f: products of the row; k: its A entries; c: output entries (numeric only);
// bound: out, the hash-table bound when the row spills.
__device__ __forceinline__ int choose_bin(int64_t f, int k, int64_t c, const BinCfg &cfg, int64_t *bound) {
    *bound = 0;
    if (f == 0) return kBinEmpty;
    if (cfg.numeric && c == 0) return kBinEmpty;
    if (f <= cfg.tiny_max) {
        const int s = f <= 8 ? 0 : (f <= 16 ? 1 : (f <= 32 ? 2 : 3));
        return kBinTiny0 + s;
    }
    int64_t need;   // table slots
    if (cfg.numeric) {
        need = c + (c >> 1);                       // load factor <= 2/3
    } else {
        const int64_t b = f < cfg.ncols ? f : cfg.ncols;   // distinct columns <= min(f, n)
        need = 2 * b;                               // load factor <= 1/2
    }
    int l = ceil_log2(need);
    if (l < kHashLog2Min) l = kHashLog2Min;
    // dense preference: numeric rows by their output entries; symbolic rows by their products (a row with c
    // entries has at least c products, so every row the numeric phase will prefer dense goes through the
    // symbolic bitmap kernel and leaves its column set in the structure cache)
    const bool dense_pref = cfg.dense_ok && (cfg.numeric ? c : f) >= cfg.dense_min_nnz;
    const bool hash_fits = !cfg.force_spill && l <= cfg.hash_log2_max && !dense_pref;
    // merge rows, by the places they take in LDS
    const int64_t places = f + int64_t(cfg.merge_products ? kMergePadNum : kMergePadSym) * k;
    if (k <= cfg.merge_runs && places <= (dense_pref ? cfg.merge_over_dense : cfg.merge_places) &&
        (!hash_fits || merge_pays(f, places, cfg))) {
        const int lm = ceil_log2(places);
        return kBinMerge0 + (lm < kMergeLog2Min ? 0 : lm - kMergeLog2Min);
    }
    if (hash_fits) return kBinHash0 + (l - kHashLog2Min);
    if (k <= cfg.merge_runs && f <= cfg.merge_long) return kBinMergeLong;
    if (!cfg.force_spill && cfg.dense_ok) return kBinDense0 + class_of(f);
    *bound = cfg.numeric ? c : (f < cfg.ncols ? f : cfg.ncols);
    return kBinSpill0 + class_of(f);
}

// Binning: at most kBinBlocks workgroups, each over a contiguous share of the
// rows, so that few workgroups add to the shared statistics (with one per 256
// rows the adds to one address took 40 us on a million rows) and rows of a bin
// keep their order across shares. bin_count counts a workgroup's rows of every
// bin into hist[bin][workgroup] and notes each row's bin; bin_scatter turns the
// counts into places.
constexpr int kBinBlocks = 256;
constexpr int kBinBlock = 1024;

// Where a row's product count comes from: the prefixes (kept in row_prod for the
// later phases), or row_prod as an earlier binning left it.
struct RowProducts {
    const int64_t *loc;        // null: row_prod holds the counts
    const int64_t *tile_sum;
    int64_t nnz;
    int64_t *row_prod;
};

// In the symbolic phase (and the single pass) it also writes row_nnz = 0 for
// rows without products; slot_of_row (or null) is set to -1.
__global__ void __launch_bounds__(kBinBlock) bin_count(const int32_t *__restrict__ a_rp, RowProducts rp,
                                                       const int64_t *__restrict__ c_rp, int64_t m, BinCfg cfg,
                                                       Control *ctrl, int32_t *__restrict__ row_nnz,
                                                       int32_t *__restrict__ slot_of_row,
                                                       uint8_t *__restrict__ bin, int32_t *__restrict__ hist) {
    __shared__ int32_t s_cnt[kMaxBins];
    __shared__ unsigned long long s_prod[kMaxBins], s_annz[kMaxBins], s_cnnz[kMaxBins];
    for (int i = threadIdx.x; i < kMaxBins; i += blockDim.x) {
        s_cnt[i] = 0;
        s_prod[i] = s_annz[i] = s_cnnz[i] = 0;
    }
    __syncthreads();
    const int64_t share = (m + gridDim.x - 1) / gridDim.x;
    const int64_t i0 = share * blockIdx.x, i1 = i0 + share < m ? i0 + share : m;
    for (int64_t w0 = i0 + uniform(static_cast<int>(threadIdx.x) / kWave) * kWave; w0 < i1; w0 += kBinBlock) {
        const int64_t i = w0 + lane_id();
        const bool in = i < i1;
        const int32_t a0 = in ? a_rp[i] : 0, a1 = in ? a_rp[i + 1] : 0;
        // (what does not depend on A's row is on its way with it)
        const int64_t c = in && cfg.numeric ? c_rp[i + 1] - c_rp[i] : 0;
        int64_t f = in && rp.loc == nullptr ? rp.row_prod[i] : 0;
        if (rp.loc != nullptr) {
            f = row_products_of(a0, a1, rp.nnz, rp.loc, rp.tile_sum);
            if (in) rp.row_prod[i] = f;
        }
        if (!in) continue;
        int64_t bound;
        const int b = choose_bin(f, a1 - a0, c, cfg, &bound);
        // a whole wave of one bin (usual where rows are alike) adds its sums once instead of lane by lane to one
        // address; sums of 64 numbers below 2^25 fit 32 bits
        const bool small = f < (1 << 25) && a1 - a0 < (1 << 25);   // (c <= f)
        if (ballot(small && b == __builtin_amdgcn_readfirstlane(b)) == ~0ull) {
            const int sf = wave_incl_sum(static_cast<int>(f)), sa = wave_incl_sum(a1 - a0);
            const int sc = wave_incl_sum(static_cast<int>(c));
            if (lane_id() == kWave - 1) {
                atomicAdd(&s_cnt[b], kWave);
                atomicAdd(&s_prod[b], static_cast<unsigned long long>(sf));
                atomicAdd(&s_annz[b], static_cast<unsigned long long>(sa));
                if (cfg.numeric) atomicAdd(&s_cnnz[b], static_cast<unsigned long long>(sc));
            }
        } else {
            atomicAdd(&s_cnt[b], 1);
            atomicAdd(&s_prod[b], static_cast<unsigned long long>(f));
            atomicAdd(&s_annz[b], static_cast<unsigned long long>(a1 - a0));
            if (cfg.numeric) atomicAdd(&s_cnnz[b], static_cast<unsigned long long>(c));
        }
        if (bound > 0) atomicMax(reinterpret_cast<unsigned long long *>(&ctrl->spill_max_bound),
                                 static_cast<unsigned long long>(bound));
        if (!cfg.numeric && b == kBinEmpty) row_nnz[i] = 0;
        if (slot_of_row != nullptr) slot_of_row[i] = -1;
        bin[i] = static_cast<uint8_t>(b);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kNumBins; b += blockDim.x) {
        hist[b * gridDim.x + blockIdx.x] = s_cnt[b];
        if (s_cnt[b]) {
            atomicAdd(&ctrl->bin_count[b], s_cnt[b]);
            atomicAdd(reinterpret_cast<unsigned long long *>(&ctrl->stat_products[b]), s_prod[b]);
            atomicAdd(reinterpret_cast<unsigned long long *>(&ctrl->stat_annz[b]), s_annz[b]);
            atomicAdd(reinterpret_cast<unsigned long long *>(&ctrl->stat_cnnz[b]), s_cnnz[b]);
        }
    }
}

// Writes each non-empty row's id into its bin's range of perm (the grid of
// bin_count); the first workgroup records the bins' offsets, and the stamp when
// it is given one (stamp->rp_sum from the scan that wrote C.row_ptr), and copies
// the control block to host_ctrl (host memory the device can write) when given.
__global__ void __launch_bounds__(kBinBlock) bin_scatter(const uint8_t *__restrict__ bin, int64_t m,
                                                         const int32_t *__restrict__ hist, Control *ctrl,
                                                         int32_t *__restrict__ perm, Stamp *stamp, const Stamp value,
                                                         const Control *sums, int32_t *host_ctrl) {
    __shared__ int32_t s_tot[kMaxBins], s_next[kMaxBins];
    const int wv = threadIdx.x / kWave, ln = lane_id();
    const int nblk = static_cast<int>(gridDim.x), blk = static_cast<int>(blockIdx.x);
    {
        // a wave's bins, all their counts loaded before the first is summed
        constexpr int NW = kBinBlock / kWave, PER = kMaxBins / NW, Q = kBinBlocks / kWave;
        int n[PER][Q];
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int b = wv + i * NW, k = ln + q * kWave;
                n[i][q] = b < kNumBins && k < nblk ? hist[b * nblk + k] : 0;
            }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            int tot = 0, before = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                tot += n[i][q];
                before += ln + q * kWave < blk ? n[i][q] : 0;
            }
            tot = wave_incl_sum(tot);
            before = wave_incl_sum(before);
            if (ln == kWave - 1) {
                s_tot[wv + i * NW] = tot;
                s_next[wv + i * NW] = before;
            }
        }
    }
    __syncthreads();
    if (wv == 0) {
        static_assert(kMaxBins == kWave, "a lane per bin");
        const int first = wave_incl_sum(s_tot[ln]) - s_tot[ln];
        s_next[ln] += first;
        if (blockIdx.x == 0) {
            ctrl->bin_offset[ln] = first;
            if (stamp != nullptr && ln == 0) {
                *stamp = value;
                stamp->rp_sum = sums->rp_sum;
                stamp->magic = kStampMagic;
            }
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && host_ctrl != nullptr) {
        const int32_t *p = reinterpret_cast<const int32_t *>(ctrl);
        for (int i = threadIdx.x; i < static_cast<int>(sizeof(Control) / 4); i += kBinBlock) host_ctrl[i] = p[i];
    }
    const int64_t share = (m + gridDim.x - 1) / gridDim.x;
    const int64_t i0 = share * blockIdx.x, i1 = i0 + share < m ? i0 + share : m;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kBinBlock) {
        const int b = bin[i];
        // one claim for all of a wave's rows of a bin, which keep their order
        uint64_t left = ballot(b != kBinEmpty);
        while (left) {
            const int first = __ffsll(static_cast<long long>(left)) - 1;
            const int b0 = __builtin_amdgcn_readlane(b, first);
            const uint64_t same = ballot(b == b0);
            int at = 0;
            if (ln == first) at = atomicAdd(&s_next[b0], static_cast<int>(__popcll(same)));
            at = __builtin_amdgcn_readlane(at, first);
            if (b == b0) perm[at + __popcll(same & ((1ull << ln) - 1ull))] = static_cast<int32_t>(i);
            left &= ~same;
        }
    }
}

// Words from device memory to host memory the device can write.
__global__ void copy_words(const int32_t *__restrict__ p, int32_t *__restrict__ host, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) host[i] = p[i];
}

// Zero-fill of the control block (a kernel, not a memset, so the sequence can
// be captured in a HIP graph).
__global__ void zero_words(int32_t *p, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ void fill_i64(int64_t *p, int64_t n, int64_t v) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Sharded rows to CSR: entry p of C (row r, c_rp[r] <= p < c_rp[r+1]) comes
// from pool position row_off[r] + p - c_rp[r]. Workgroup w writes entries
// [w*kGatherChunk, (w+1)*kGatherChunk) of C with coalesced stores: one wave
// finds the rows holding the chunk's ends by a 64-ary search of c_rp, the
// chunk's row pointers are staged in LDS, and each thread finds its entry's
// row by binary search there (in c_rp itself when the chunk spans very many,
// mostly empty, rows).
constexpr int kGatherChunk = 4096;
constexpr int kGatherRows = 1024;

// Last row r in [0, nrows) with c_rp[r] <= p (so c_rp[r] <= p < c_rp[r+1]
// for p < c_rp[nrows]). All 64 lanes of one wave take part.
__device__ __forceinline__ int64_t wave_find_row(const int64_t *__restrict__ c_rp, int64_t nrows, int64_t p) {
    int64_t lo = 0, hi = nrows - 1;   // c_rp[lo] <= p holds throughout
    while (hi > lo) {
        const int64_t step = (hi - lo + kWave) / kWave;   // ceil((hi - lo + 1) / 64)
        const int64_t idx = lo + static_cast<int64_t>(lane_id()) * step;
        const bool le = idx <= hi && c_rp[idx] <= p;
        const uint64_t m = ballot(le);
        const int k = 63 - __clzll(m);   // lane 0 always qualifies
        lo = lo + k * step;
        const int64_t h = lo + step - 1;
        hi = h < hi ? h : hi;
    }
    return lo;
}

template <typename V>
__global__ void __launch_bounds__(256) gather_rows(int64_t nrows, const int64_t *__restrict__ row_off,
                                                   const int64_t *__restrict__ c_rp,
                                                   const int32_t *__restrict__ pool_col,
                                                   const V *__restrict__ pool_val, int32_t *__restrict__ c_col,
                                                   V *__restrict__ c_val) {
    __shared__ int64_t s_rp[kGatherRows + 1];
    __shared__ int64_t s_off[kGatherRows];
    __shared__ int64_t s_r[2];
    const int64_t nnz = c_rp[nrows];
    const int64_t p0 = static_cast<int64_t>(blockIdx.x) * kGatherChunk;
    if (p0 >= nnz) return;   // whole workgroup leaves together
    const int64_t p1 = nnz - p0 < kGatherChunk ? nnz : p0 + kGatherChunk;
    if (threadIdx.x < kWave) {
        const int64_t r0 = wave_find_row(c_rp, nrows, p0);
        const int64_t r1 = wave_find_row(c_rp, nrows, p1 - 1);
        if (threadIdx.x == 0) {
            s_r[0] = r0;
            s_r[1] = r1;
        }
    }
    __syncthreads();
    const int64_t r0 = s_r[0], r1 = s_r[1];
    const int64_t nr = r1 - r0 + 1;
    if (nr <= kGatherRows) {
        for (int64_t i = threadIdx.x; i <= nr; i += blockDim.x) s_rp[i] = c_rp[r0 + i];
        for (int64_t i = threadIdx.x; i < nr; i += blockDim.x) s_off[i] = row_off[r0 + i];
        __syncthreads();
        for (int64_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
            int lo = 0, hi = static_cast<int>(nr) - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_rp[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            const int64_t src = s_off[lo] + (p - s_rp[lo]);
            c_col[p] = pool_col[src];
            c_val[p] = pool_val[src];
        }
    } else {
        for (int64_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
            int64_t lo = r0, hi = r1;
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) >> 1;
                if (c_rp[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            const int64_t src = row_off[lo] + (p - c_rp[lo]);
            c_col[p] = pool_col[src];
            c_val[p] = pool_val[src];
        }
    }
}

// Checksum of C.row_ptr[0..m] (the sum of rp[i] * (2i + 1) modulo 2^64) in
// kRpParts parts, one per workgroup, into ctrl->rp_part; the first workgroup
// clears the rest of the control block. With host (host memory the device can
// write), the parts go to the control block's copy there instead, between the
// copies of the stamp and of the kept binning's control block (from ctrl_num),
// laid out as in the workspace from the stamp on.
__global__ void __launch_bounds__(1024) rowptr_checksum(const int64_t *__restrict__ rp, int64_t m, Control *ctrl,
                                                        const Stamp *stamp, const Control *ctrl_num, char *host,
                                                        int64_t host_ctrl, int64_t host_ctrl_num) {
    __shared__ int64_t scratch[1024 / kWave];
    uint64_t acc = 0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i <= m;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        acc += static_cast<uint64_t>(rp[i]) * static_cast<uint64_t>(2 * i + 1);
    acc = static_cast<uint64_t>(block_sum<1024>(static_cast<int64_t>(acc), scratch));
    if (threadIdx.x == 0)
        (host != nullptr ? reinterpret_cast<Control *>(host + host_ctrl) : ctrl)->rp_part[blockIdx.x] = acc;
    if (host != nullptr && blockIdx.x == 1) {
        const int32_t *p = reinterpret_cast<const int32_t *>(stamp), *q = reinterpret_cast<const int32_t *>(ctrl_num);
        for (int i = threadIdx.x; i < static_cast<int>(sizeof(Stamp) / 4); i += blockDim.x)
            reinterpret_cast<int32_t *>(host)[i] = p[i];
        for (int i = threadIdx.x; i < static_cast<int>(sizeof(Control) / 4); i += blockDim.x)
            reinterpret_cast<int32_t *>(host + host_ctrl_num)[i] = q[i];
    }
    if (blockIdx.x == 0) {
        int32_t *p = reinterpret_cast<int32_t *>(ctrl);
        constexpr int lo = offsetof(Control, rp_part) / 4, hi = lo + kRpParts * 2;
        for (int i = threadIdx.x; i < static_cast<int>(sizeof(Control) / 4); i += blockDim.x)
            if (i < lo || i >= hi) p[i] = 0;
    }
}

// The numeric binning the stamp describes is no longer what the workspace
// holds (one thread).
__global__ void drop_kept_bins(Stamp *stamp) {
    if (threadIdx.x == 0 && blockIdx.x == 0) stamp->num_bins = 0;
}

// Flags values that could produce a zero product: exact zeros, and (for
// double) magnitudes below 2^-537, whose products with each other could
// underflow to zero. float products are formed in double and cannot underflow.
template <typename V>
__global__ void __launch_bounds__(256) find_zero_values(const V *__restrict__ val, int64_t n, Control *ctrl) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    bool small = false;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double v = static_cast<double>(val[i]);
        const double a = v < 0 ? -v : v;
        small |= sizeof(V) == 4 ? (a == 0.0) : !(a >= 0x1p-537);
    }
    if (__ballot(small) != 0ull && lane_id() == 0) atomicOr(&ctrl->has_zero_values, 1);
}

// ---------------------------------------------------------------------------
// Column-window table of B: wtab[k*(nwin+1) + w] is the first entry of row k
// with column >= w*wcols (w = nwin gives the row end). With it, the part of a
// row of B inside window w is one slice, found without searching.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) build_window_table(const int32_t *__restrict__ b_rp,
                                                          const int32_t *__restrict__ b_col,
                                                          int64_t nrows_b, int nwin, int wcols,
                                                          int32_t *__restrict__ wtab) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t stride = nwin + 1;
    if (t >= nrows_b * stride) return;
    const int64_t k = t / stride;
    const int w = static_cast<int>(t - k * stride);
    int lo = b_rp[k], hi = b_rp[k + 1];
    if (w < nwin) {
        const int64_t target = static_cast<int64_t>(w) * wcols;
        while (lo < hi) {
            const int mid = lo + ((hi - lo) >> 1);
            if (b_col[mid] < target) lo = mid + 1;
            else hi = mid;
        }
    } else {
        lo = hi;
    }
    wtab[t] = lo;
}

// ---------------------------------------------------------------------------
// Optional validation: one wave per row checks the row_ptr step and that the
// row's columns are in range and strictly increasing.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) validate_csr(const int32_t *__restrict__ rp,
                                                    const int32_t *__restrict__ col, int64_t nrows,
                                                    int64_t ncols, int64_t nnz, Control *ctrl) {
    const int64_t row = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    const int ln = lane_id();
    if (row >= nrows) return;
    bool bad = false;
    const int32_t s = rp[row], e = rp[row + 1];
    if (row == 0 && s != 0) bad = true;
    if (row == nrows - 1 && static_cast<int64_t>(e) != nnz) bad = true;
    if (e < s || s < 0 || static_cast<int64_t>(e) > nnz) {
        bad = true;
    } else {
        for (int32_t p = s + ln; p < e; p += kWave) {
            const int32_t c = col[p];
            if (c < 0 || static_cast<int64_t>(c) >= ncols) bad = true;
            if (p > s && col[p - 1] >= c) bad = true;
        }
    }
    if (bad) atomicOr(&ctrl->error_flags, kErrInvalidMatrix);
}

}  // namespace wsp
