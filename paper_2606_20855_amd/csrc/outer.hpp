// Outer-product SpGEMM, C = A B = sum over k of A[:, k] B[k, :] (paper,
// Section 5.1: the outer-product program of the SpGEMM figure, which runs
// the contraction index k in parallel and guards C with a merge level, a copy
// of C per worker recombined by `coalesce`, Section 4.3).
//
// A comes by its columns (At, the CSR arrays of A's transpose) and B by its
// rows, so the rank-1 update of index k pairs row k of At with row k of B.
// Its |At_k| * |B_k| products, over all k, are numbered flat (q over the
// exclusive prefix pref of the per-k counts):
//   1. claim: every entry of At (row i of A, index k) claims |B_k| places of row
//      i's bucket, the merge level's per-row storage (one atomic per entry, or
//      one for several entries of a row, see op_claim);
//   2. expand: chunks of kOpChunk products are formed and written to their
//      places, so a bucket holds its row's partial entries as whole rows of B
//      scaled, in arbitrary order;
//   3. coalesce: each row's bucket is sorted by column and equal columns summed:
//      in registers up to 256 entries, in LDS up to kOpRowCap, and beyond that as
//      runs of kOpRowCap sorted in LDS then merged pairwise in global memory
//      (merge path, each output tile merged in LDS). Buckets of more than 256
//      entries that are no fewer than C's columns are summed in LDS accumulators
//      instead, past kOpRowCap by pieces (op_by_pieces);
//   4. the compacted rows are scanned into C.row_ptr and gathered into CSR.
// (Sorting and summing each chunk first, as a partial C per workgroup, halved the
// entries the coalesce sees on a mesh but cost more than the rest together: 327
// us of LDS bitonic sort and 101 us of moves for the 6.5 M products of a 512 x
// 512 grid's square, against 83 us for claims and expansion. Where it collapsed
// most products, C of few columns or rows, the accumulators and the claims added
// up in LDS take its place. Whole calls with chunks summed, with neither, and now,
// double: 1 M x 1 by itself 0.39, 177 and 0.17 ms; A^T A of 1 M x 16 with 4
// entries a row 18.6, 161 and 0.30 ms, of 200 K x 4096 with 6 entries a row in
// popular columns 34.3, 74 and 0.47 ms; R-MAT 14, edge factor 16, float 22.7, 14.0
// and 3.4 ms. What is left of it: buckets of one column where C has many, 50 of
// 20 K entries, 0.35, 9.5 and 0.50 ms.)
// Products are formed and summed in double; values are rounded once.
#pragma once

#include "search.hpp"
#include "tiers.hpp"

namespace wsp {

constexpr int kOpChunk = 2048;     // products (expand) or entries of At (claim) per workgroup
constexpr int kOpBlock = 256;      // threads of the claim and expand kernels
constexpr int kOpStage = 2048;     // k indices a chunk stages in LDS
constexpr int kOpSlots = 2048;     // rows whose claims a chunk of At's entries adds up in LDS
constexpr int kOpHot = 6;          // threads that find a row again, of a quarter of the chunk, from which on it does
static_assert(kOpSlots == kOpStage, "the claims' slots take the staged indices' place");
constexpr int kOpMidCap = 256;     // longest row bucket sorted in one wave's registers
constexpr int kOpRowCap = 4096;    // longest row bucket sorted whole in LDS; also the run and merge tile length
constexpr int kOpRowBlock = 256;   // threads per long row in the coalesce
constexpr int kOpHugeBlock = 1024; // threads per row past kOpRowCap
constexpr int kOpPiece = 8192;     // entries of a long bucket summed by one workgroup
constexpr int64_t kOpSumCols = 65536;   // columns of C up to which long buckets are summed by pieces
static_assert(kOpPiece == 2 * kOpRowCap, "a piece's long rows are found from three of its places");

// Products of rank-1 update k: |At_k| * |B_k|.
struct OpProdIn {
    const int32_t *at_rp, *b_rp;
    __device__ __forceinline__ int64_t operator()(int64_t k) const {
        return static_cast<int64_t>(at_rp[k + 1] - at_rp[k]) * static_cast<int64_t>(b_rp[k + 1] - b_rp[k]);
    }
};

// In-place bitonic sort of n (a power of two) key/value pairs in LDS by key,
// ascending, by the threads of the workgroup (all of them call it).
template <typename K>
__device__ void lds_bitonic(K *key, double *val, int n) {
    for (int k = 2; k <= n; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < (n >> 1); t += blockDim.x) {
                const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));   // i has bit j clear
                const int p = i + j;
                const bool up = (i & k) == 0;
                const K a = key[i], b = key[p];
                if ((a > b) == up) {
                    key[i] = b;
                    key[p] = a;
                    const double v = val[i];
                    val[i] = val[p];
                    val[p] = v;
                }
            }
            __syncthreads();
        }
    }
}

// Exclusive workgroup scan of one int per thread; *total gets the sum. All
// threads call it; `scratch` holds one int per wave.
__device__ __forceinline__ int block_excl_scan(int x, int *scratch, int *total) {
    const int nw = blockDim.x / kWave;
    const int w = threadIdx.x / kWave;
    const int incl = wave_incl_sum(x);
    if (lane_id() == kWave - 1) scratch[w] = incl;
    __syncthreads();
    int before = 0, t = 0;
    for (int i = 0; i < nw; ++i) {
        const int s = scratch[i];
        before += i < w ? s : 0;
        t += s;
    }
    __syncthreads();
    *total = t;
    return before + incl - x;
}

// Sums of segments that run on across the threads of a workgroup: given each
// thread's open sum (of its entries from its last segment's start on, or of all
// of them where none starts in it: !any), the sum of the segment that is open
// where the thread begins. s_part holds a double per wave and one before them,
// what was open before the workgroup's entries (read where no segment starts
// before the thread); s_any an int per wave. All threads call it.
__device__ __forceinline__ double block_open_sum(double sum, bool any, double *s_part, int *s_any) {
    const int wv = static_cast<int>(threadIdx.x) / kWave, ln = lane_id();
    int f = any ? 1 : 0;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const double y = __shfl_up(sum, o, kWave);
        const int fy = __shfl_up(f, o, kWave);
        if (ln >= o && f == 0) {
            sum += y;
            f = fy;
        }
    }
    if (ln == kWave - 1) {
        s_part[wv + 1] = sum;
        s_any[wv] = f;
    }
    double before = __shfl_up(sum, 1, kWave);
    int started = __shfl_up(f, 1, kWave);
    if (ln == 0) {
        before = 0.0;
        started = 0;
    }
    __syncthreads();
    if (started == 0) {
        int i = wv;
        do before += s_part[i];
        while (--i >= 0 && s_any[i] == 0);
    }
    return before;
}

// Clears the rows' entry counts, the coalesce's counters and the product
// prefix's first word (0 already, unless At has no rows).
__global__ void __launch_bounds__(256) op_clear(int32_t *__restrict__ row_cnt, int64_t m, int32_t *counters,
                                                int64_t *pref) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < m) row_cnt[i] = 0;
    if (i < 4) counters[i] = 0;
    if (i == 0) pref[0] = 0;
}

// 1. Entry e of At, of index k, claims |B_k| places of its row's bucket:
// place[e] (entries with products only); row_cnt ends at the buckets' sizes.
//
// Bound by the rate of atomics, one per entry (1.2 M entries of 100 K rows 60
// us), unless many are of one row: a counter takes an atomic every 10 ns (1 M of
// one row 10 ms). So a chunk looks at a quarter of its entries, and where kOpHot
// threads or more find a row that another has found, it adds up the claims of
// its rows in LDS first, one atomic a row and one for each entry whose row found
// its slot taken (every chunk doing so: 97 us for the same 1.2 M entries, so 62;
// a 512 x 512 mesh of five points, whose chunks do so, 22 -> 19 us).
__global__ void __launch_bounds__(kOpBlock) op_claim(const int32_t *__restrict__ at_rp,
                                                     const int32_t *__restrict__ at_col,
                                                     const int32_t *__restrict__ b_rp, int K, int64_t nnz,
                                                     int32_t *__restrict__ row_cnt, int32_t *__restrict__ place) {
    __shared__ int32_t s_rp[kOpStage];
    __shared__ int32_t s_cnt[kOpSlots];
    __shared__ int s_t[2];
    constexpr int PER = kOpChunk / kOpBlock;
    const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kOpChunk;
    for (int h = threadIdx.x; h < kOpSlots / 2; h += kOpBlock) s_cnt[h] = -1;
    const int64_t e1 = nnz - e0 < kOpChunk ? nnz : e0 + kOpChunk;
    if (threadIdx.x < 2 * kWave) {
        const int t = wave_last_le([=](int k) { return static_cast<int64_t>(at_rp[k]); }, 0, K - 1,
                                   threadIdx.x < kWave ? e0 : e1 - 1);
        if (lane_id() == 0) s_t[threadIdx.x / kWave] = t;
    }
    __syncthreads();
    const int t0 = s_t[0], nt = s_t[1] - t0 + 1;
    const bool staged = nt <= kOpStage;
    if (staged)
        for (int k = threadIdx.x; k < nt; k += kOpBlock) s_rp[k] = at_rp[t0 + k];
    __syncthreads();
    int row[PER], n[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t e = e0 + threadIdx.x + u * kOpBlock;
        n[u] = 0;
        row[u] = 0;
        if (e < e1) {
            int lo = 0, hi = nt - 1;   // the last index whose entries begin at or before e
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if ((staged ? s_rp[mid] : at_rp[t0 + mid]) <= e) lo = mid;
                else hi = mid - 1;
            }
            row[u] = at_col[e];
            n[u] = b_rp[t0 + lo + 1] - b_rp[t0 + lo];
        }
    }
    // a row's slot
    const auto slot_of = [](int r, int slots) { return (r ^ (r / kOpSlots)) & (slots - 1); };
    bool found = false;
#pragma unroll
    for (int u = 0; u < PER / 4; ++u)
        if (n[u] > 0) found |= atomicCAS(&s_cnt[slot_of(row[u], kOpSlots / 2)], -1, row[u]) == row[u];
    int slot[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) slot[u] = -1;
    if (__syncthreads_count(found) >= kOpHot) {
        // (the staged indices are done with)
        for (int h = threadIdx.x; h < kOpSlots; h += kOpBlock) {
            s_rp[h] = -1;
            s_cnt[h] = 0;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (n[u] <= 0) continue;
            const int h = slot_of(row[u], kOpSlots);
            const int was = atomicCAS(&s_rp[h], -1, row[u]);
            if (was == -1 || was == row[u]) {
                slot[u] = h;
                n[u] = atomicAdd(&s_cnt[h], n[u]);
            }
        }
        __syncthreads();
        for (int h = threadIdx.x; h < kOpSlots; h += kOpBlock)
            if (const int cnt = s_cnt[h]; cnt > 0) s_cnt[h] = atomicAdd(&row_cnt[s_rp[h]], cnt);
        __syncthreads();
    }
    int at[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (slot[u] >= 0) at[u] = s_cnt[slot[u]] + n[u];
        else at[u] = n[u] > 0 ? atomicAdd(&row_cnt[row[u]], n[u]) : -1;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (at[u] >= 0) place[e0 + threadIdx.x + u * kOpBlock] = at[u];
}

// 2. Products [q0, q0 + kOpChunk) formed and written to their places. Bound by the
// latency of its dependent loads (index, At's row and place, bucket): 114 VGPRs in
// double keep 3.6 waves on a SIMD, waiting two thirds of the time (a 512 x 512
// mesh, 6.5 M products: 55 us, 3.0 TB/s, the VALU 40% busy).
template <typename V>
__global__ void __launch_bounds__(kOpBlock) op_expand(const int32_t *__restrict__ at_rp,
                                                      const int32_t *__restrict__ at_col,
                                                      const V *__restrict__ at_val,
                                                      const int32_t *__restrict__ b_rp,
                                                      const int32_t *__restrict__ b_col,
                                                      const V *__restrict__ b_val, int K,
                                                      const int64_t *__restrict__ pref, int64_t P,
                                                      const int32_t *__restrict__ place,
                                                      const int64_t *__restrict__ bucket_off,
                                                      int32_t *__restrict__ bkt_col, double *__restrict__ bkt_val) {
    __shared__ int64_t s_pref[kOpStage];
    __shared__ int s_t[2];
    constexpr int PER = kOpChunk / kOpBlock;
    const int64_t q0 = static_cast<int64_t>(blockIdx.x) * kOpChunk;
    const int64_t q1 = P - q0 < kOpChunk ? P : q0 + kOpChunk;
    if (threadIdx.x < 2 * kWave) {
        const int t = wave_find_entry(pref, K, threadIdx.x < kWave ? q0 : q1 - 1);
        if (lane_id() == 0) s_t[threadIdx.x / kWave] = t;
    }
    __syncthreads();
    const int t0 = s_t[0];
    const int nt = s_t[1] - t0 + 1;
    const bool staged = nt <= kOpStage;
    if (staged)
        for (int k = threadIdx.x; k < nt; k += kOpBlock) s_pref[k] = pref[t0 + k];
    __syncthreads();
    // every thread's products side by side: the loads of one step of all before the next
    int ia[PER], jb[PER], j[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t q = q0 + threadIdx.x + u * kOpBlock < q1 ? q0 + threadIdx.x + u * kOpBlock : q1 - 1;
        const int k = staged ? t0 + lds_find_entry(s_pref, nt, q) : t0 + lds_find_entry(pref + t0, nt, q);
        const uint32_t r = static_cast<uint32_t>(q - (staged ? s_pref[k - t0] : pref[k]));   // (P < 2^31)
        const int b0 = b_rp[k];
        const uint32_t nb = static_cast<uint32_t>(b_rp[k + 1] - b0);   // > 0: index k has products
        const uint32_t ai = r / nb;
        j[u] = static_cast<int>(r - ai * nb);
        ia[u] = at_rp[k] + static_cast<int>(ai);
        jb[u] = b0 + j[u];
    }
    int row[PER], pl[PER], col[PER];
    V av[PER], bv[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        row[u] = at_col[ia[u]];
        pl[u] = place[ia[u]];
        col[u] = b_col[jb[u]];
        av[u] = at_val[ia[u]];
        bv[u] = b_val[jb[u]];
    }
    int64_t at[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) at[u] = bucket_off[row[u]] + pl[u] + j[u];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (q0 + threadIdx.x + u * kOpBlock < q1) {
            bkt_col[at[u]] = col[u];
            bkt_val[at[u]] = to_d(av[u]) * to_d(bv[u]);
        }
    }
}

// 3a. Buckets of at most 32 entries, 32 lanes per row: (column, place) keys
// sorted in registers, equal columns summed, written back compacted from the
// bucket's start (columns in bkt_col, values rounded to V in out_val). Key as in
// tiny_kernel, and bound as it is by VALU issue (busy all the time).
template <typename Key, typename V>
__global__ void __launch_bounds__(256) op_merge_short(const int64_t *__restrict__ bucket_off, int64_t m,
                                                      int32_t *__restrict__ bkt_col,
                                                      const double *__restrict__ bkt_val, V *__restrict__ out_val,
                                                      int32_t *__restrict__ row_nnz) {
    constexpr int S = 32, LOG2S = 5;
    const int64_t row = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) / S;
    const int lane = lane_id(), ln = lane & (S - 1);
    const int64_t lo = row < m ? bucket_off[row] : 0;
    const int64_t len = row < m ? bucket_off[row + 1] - lo : 0;
    const bool mine = row < m && len <= S;
    // a wave without a row of this kernel is done; in the others every lane takes part in the moves
    if (ballot(mine) == 0ull) return;
    const bool live = mine && ln < len;
    const int col = live ? bkt_col[lo + ln] : 0;
    const double v0 = live ? bkt_val[lo + ln] : 0.0;
    Key x[1] = {live ? static_cast<Key>(static_cast<uint32_t>(col)) << LOG2S | static_cast<Key>(ln) : ~Key(0)};
    bitonic_sort<S, 2, 1>(x, ln);
    const uint32_t c = static_cast<uint32_t>(x[0] >> LOG2S);
    const uint32_t prev = static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(c), kDppWaveShr1, 0xf, 0xf, false));
    const bool head = live && (ln == 0 || prev != c);   // (sorted, the keys fill the first len lanes)
    const uint64_t hm = ballot(head) & (0xffffffffull << (lane - ln));
    double sum = __shfl(v0, static_cast<int>(x[0]) & (S - 1), S);
    {
        const uint64_t after = lane < kWave - 1 ? hm >> (lane + 1) : 0ull;
        const int n = after ? __ffsll(static_cast<long long>(after)) : static_cast<int>(len) - ln;
        double t = sum;
        for (int d = 1; ballot(head && d < n) != 0ull; ++d) {
            t = __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(t), 0x130, 0xf, 0xf, false),
                                 __builtin_amdgcn_update_dpp(0, __double2loint(t), 0x130, 0xf, 0xf, false));
            if (head && d < n) sum += t;
        }
    }
    if (head) {
        const int pos = __popcll(hm & ((1ull << lane) - 1ull));
        bkt_col[lo + pos] = static_cast<int32_t>(c);
        out_val[lo + pos] = static_cast<V>(sum);
    }
    if (mine && ln == 0) row_nnz[row] = __popcll(hm);
}

// Bitonic sort of 64 R keys held R per lane (key i in register i / 64 of lane
// i % 64), ascending: distances below 64 across lanes, the others between
// registers.
template <int J, int R>
__device__ __forceinline__ void wave_sort_lanes(uint64_t (&x)[R], int ln, int k) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool up = k >= kWave ? ((r * kWave) & k) == 0 : (ln & k) == 0;
        bitonic_step<J>(x[r], ln, ((ln & J) == 0) == up);
    }
    if constexpr (J > 1) wave_sort_lanes<J / 2, R>(x, ln, k);
}
template <int K, int R>
__device__ __forceinline__ void wave_sort(uint64_t (&x)[R], int ln) {
    if constexpr (K > kWave) {
#pragma unroll
        for (int j = K / 2; j >= kWave; j >>= 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int p = r ^ (j / kWave);
                if (p > r) {
                    const bool swap = ((r * kWave) & K) == 0 ? x[p] < x[r] : x[r] < x[p];
                    const uint64_t a = x[r], b = x[p];
                    x[r] = swap ? b : a;
                    x[p] = swap ? a : b;
                }
            }
        }
        wave_sort_lanes<kWave / 2, R>(x, ln, K);
    } else {
        wave_sort_lanes<K / 2, R>(x, ln, K);
    }
    if constexpr (K < kWave * R) wave_sort<2 * K, R>(x, ln);
}

// One bucket of at most 64 R entries, by one wave: s_val holds 64 R doubles.
template <int R, typename V>
__device__ __forceinline__ void op_merge_wave(int64_t lo, int len, int32_t *__restrict__ bkt_col,
                                              const double *__restrict__ bkt_val, V *__restrict__ out_val,
                                              int32_t *__restrict__ nnz, double *s_val, int ln) {
    uint64_t x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kWave + ln;
        x[r] = i < len ? static_cast<uint64_t>(static_cast<uint32_t>(bkt_col[lo + i])) << 32 | i : ~0ull;
    }
    wave_sort<2, R>(x, ln);
    double v[R];
    uint64_t heads[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kWave + ln;
        v[r] = i < len ? bkt_val[lo + static_cast<int>(x[r] & 0xffffffffu)] : 0.0;
        s_val[i] = v[r];
        const int c = static_cast<int>(x[r] >> 32);
        int prev = __builtin_amdgcn_update_dpp(0, c, kDppWaveShr1, 0xf, 0xf, false);
        if (ln == 0) prev = r > 0 ? __builtin_amdgcn_readlane(static_cast<int>(x[r > 0 ? r - 1 : 0] >> 32), kWave - 1) : -1;
        heads[r] = ballot(i < len && prev != c);
    }
    wave_lds_fence();
    int before = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kWave + ln;
        if ((heads[r] >> ln) & 1ull) {
            // the entries up to the next head
            int end = len;
#pragma unroll
            for (int t = R - 1; t > r; --t)
                if (heads[t]) end = t * kWave + __ffsll(static_cast<long long>(heads[t])) - 1;
            const uint64_t after = ln < kWave - 1 ? heads[r] >> (ln + 1) : 0ull;
            if (after) end = i + __ffsll(static_cast<long long>(after));
            double sum = v[r];
            for (int q = i + 1; q < end; ++q) sum += s_val[q];
            const int pos = before + __popcll(heads[r] & ((1ull << ln) - 1ull));
            bkt_col[lo + pos] = static_cast<int32_t>(x[r] >> 32);
            out_val[lo + pos] = static_cast<V>(sum);
        }
        before += __popcll(heads[r]);
    }
    if (ln == 0) *nnz = before;
    wave_lds_fence();
}

// 3b. Buckets of 33 to kOpMidCap entries, a wave per row; a workgroup looks at
// `per` rows (at most 64, op_mid_rows) and lists the longer ones (one atomic for
// all of them): up to kOpRowCap from the front of long_rows for op_merge_long
// (count in counters[0]), the rest from its back for op_merge_huge (counters[2]).
template <typename V>
__global__ void __launch_bounds__(256) op_merge_mid(const int64_t *__restrict__ bucket_off, int64_t m, int per,
                                                    int32_t *__restrict__ bkt_col,
                                                    const double *__restrict__ bkt_val, V *__restrict__ out_val,
                                                    int32_t *__restrict__ row_nnz, int32_t *__restrict__ long_rows,
                                                    int32_t *counters) {
    __shared__ double s_val[256 / kWave][kOpMidCap];
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int ln = lane_id();
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * per;
    const int64_t row = ln < per ? row0 + ln : m;
    const int64_t lo = row < m ? bucket_off[row] : 0;
    const int64_t len = row < m ? bucket_off[row + 1] - lo : 0;
    if (wv == 0) {
        const uint64_t below = (1ull << ln) - 1ull;
        const uint64_t lng = ballot(len > kOpMidCap && len <= kOpRowCap), huge = ballot(len > kOpRowCap);
        if (lng) {
            int at = 0;
            if (ln == 0) at = atomicAdd(&counters[0], static_cast<int>(__popcll(lng)));
            at = uniform(at);
            if ((lng >> ln) & 1ull) long_rows[at + __popcll(lng & below)] = static_cast<int32_t>(row);
        }
        if (huge) {
            int at = 0;
            if (ln == 0) at = atomicAdd(&counters[2], static_cast<int>(__popcll(huge)));
            at = uniform(at);
            if ((huge >> ln) & 1ull) long_rows[m - 1 - at - __popcll(huge & below)] = static_cast<int32_t>(row);
        }
    }
    uint64_t mid = ballot(len > 32 && len <= kOpMidCap);
    for (int i = 0; mid != 0ull; ++i) {
        const int l = __ffsll(static_cast<long long>(mid)) - 1;
        mid &= mid - 1;
        if ((i & (256 / kWave - 1)) != wv) continue;
        const int64_t rlo = static_cast<int64_t>(
            static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lo >> 32), l))) << 32 |
            static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lo), l)));
        const int n = __builtin_amdgcn_readlane(static_cast<int>(len), l);
        int32_t *nnz = row_nnz + row0 + l;
        if (n <= kWave) op_merge_wave<1, V>(rlo, n, bkt_col, bkt_val, out_val, nnz, s_val[wv], ln);
        else if (n <= 2 * kWave) op_merge_wave<2, V>(rlo, n, bkt_col, bkt_val, out_val, nnz, s_val[wv], ln);
        else op_merge_wave<4, V>(rlo, n, bkt_col, bkt_val, out_val, nnz, s_val[wv], ln);
    }
}

// Whether a bucket is summed in LDS accumulators, by pieces of kOpPiece of the
// buckets' places and then piece by piece, instead of sorted: it is past
// kOpRowCap and C has few columns, no more than the bucket has entries (so a
// window's clearing and reading cost less than its entries) and no more than the
// 16 windows whose passes over a piece's registers still cost less than its sort
// (65536 columns, 100 K x 65536 with popular columns: 1.7 ms, sorted 9.2 ms).
// Sorting kept one workgroup on a bucket: 177 ms for 1 M entries of one column,
// whose sum was one lane's, now 0.17 ms for the whole call.
__device__ __forceinline__ bool op_by_pieces(int64_t len, int64_t ncols) {
    return len > kOpRowCap && ncols <= kOpSumCols && ncols <= len;
}

// The columns [w0, w0 + kOpRowCap) of C, accumulated in acc (bits: those
// stored), into col and val in order; returns how many. pre holds
// kOpRowCap / 32 ints. The whole workgroup calls it, between barriers.
template <typename V>
__device__ __forceinline__ int op_emit_window(int w0, int cols, const uint32_t *bits, const double *acc, int *pre,
                                              int *scan, int32_t *__restrict__ col, V *__restrict__ val) {
    constexpr int WORDS = kOpRowCap / 32;
    const int t = threadIdx.x;
    int total = 0;
    const int before = block_excl_scan(t < WORDS ? static_cast<int>(__popc(bits[t])) : 0, scan, &total);
    if (t < WORDS) pre[t] = before;
    __syncthreads();
    for (int k = t; k < cols; k += blockDim.x) {
        const uint32_t word = bits[k >> 5];
        if (((word >> (k & 31)) & 1u) == 0u) continue;
        const int at = pre[k >> 5] + static_cast<int>(__popc(word & ((1u << (k & 31)) - 1u)));
        col[at] = w0 + k;
        val[at] = static_cast<V>(acc[k]);
    }
    return total;
}
__device__ __forceinline__ void op_add(uint32_t *bits, double *acc, int k, double v) {
    atomicAdd(&acc[k], v);
    const uint32_t bit = 1u << (k & 31);
    if ((bits[k >> 5] & bit) == 0u) atomicOr(&bits[k >> 5], bit);
}

// Piece c of the buckets' places: what it holds of each long bucket, equal
// columns summed and in order, to x_col and x_val at the bucket's places, and
// their number to y_col at the first of them. The rows are those of the piece's
// first, middle and last place (a row of more than half a piece inside it
// covers its middle).
__device__ __forceinline__ void op_sum_piece(int64_t c, const int64_t *__restrict__ bucket_off, int64_t m, int64_t P,
                                             int ncols, const int32_t *__restrict__ bkt_col,
                                             const double *__restrict__ bkt_val, int32_t *__restrict__ x_col,
                                             double *__restrict__ x_val, int32_t *__restrict__ y_col, uint32_t *bits,
                                             double *acc, int *pre, int *scan, int *s_row) {
    constexpr int PER = kOpPiece / kOpRowBlock;
    const int64_t q0 = c * kOpPiece, q1 = P - q0 < kOpPiece ? P : q0 + kOpPiece;
    const int wv = threadIdx.x / kWave;
    if (wv < 3) {
        int64_t q = wv == 0 ? q0 : q0 + kOpRowCap;
        if (wv == 2 || q >= q1) q = q1 - 1;
        const int r = wave_last_le([=](int i) { return bucket_off[i]; }, 0, static_cast<int>(m) - 1, q);
        if (lane_id() == 0) s_row[wv] = r;
    }
    __syncthreads();
    for (int i = 0; i < 3; ++i) {
        const int row = s_row[i];
        if (i > 0 && row == s_row[i - 1]) continue;
        const int64_t lo = bucket_off[row], hi = bucket_off[row + 1];
        if (!op_by_pieces(hi - lo, ncols)) continue;
        const int64_t a = lo > q0 ? lo : q0, b = hi < q1 ? hi : q1;
        int32_t col[PER];
        double v[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t e = a + threadIdx.x + u * kOpRowBlock;
            col[u] = -1;
            v[u] = 0.0;
            if (e < b) {
                col[u] = bkt_col[e];
                v[u] = bkt_val[e];
            }
        }
        int done = 0;
        for (int w0 = 0; w0 < ncols; w0 += kOpRowCap) {
            const int cols = ncols - w0 < kOpRowCap ? ncols - w0 : kOpRowCap;
            for (int k = threadIdx.x; k < cols; k += kOpRowBlock) acc[k] = 0.0;
            if (threadIdx.x < kOpRowCap / 32) bits[threadIdx.x] = 0u;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int k = col[u] - w0;
                if (static_cast<uint32_t>(k) < static_cast<uint32_t>(cols)) op_add(bits, acc, k, v[u]);
            }
            __syncthreads();
            done += op_emit_window(w0, cols, bits, acc, pre, scan, x_col + a + done, x_val + a + done);
            __syncthreads();
        }
        if (threadIdx.x == 0) y_col[a] = done;
    }
}

// 3c. Long buckets (kOpMidCap + 1 .. kOpRowCap entries), a workgroup per row, rows taken
// grid-stride from the list op_merge_mid made: the bucket is sorted in LDS
// and compacted, equal columns summed by a segmented scan over the threads. The workgroups from nlong on sum the
// pieces of longer buckets (op_by_pieces) for op_merge_huge.
template <typename V>
__global__ void __launch_bounds__(kOpRowBlock) op_merge_long(const int64_t *__restrict__ bucket_off, int64_t m,
                                                             int64_t P, int64_t ncols, int nlong,
                                                             int32_t *__restrict__ bkt_col,
                                                             const double *__restrict__ bkt_val,
                                                             V *__restrict__ out_val, int32_t *__restrict__ row_nnz,
                                                             const int32_t *__restrict__ long_rows,
                                                             const int32_t *counters, int32_t *__restrict__ x_col,
                                                             double *__restrict__ x_val,
                                                             int32_t *__restrict__ y_col) {
    __shared__ int32_t s_key[kOpRowCap];
    __shared__ double s_val[kOpRowCap];
    __shared__ int s_scan[kOpRowBlock / kWave];
    __shared__ double s_part[kOpRowBlock / kWave + 1];
    __shared__ int s_any[kOpRowBlock / kWave];
    constexpr int PER = kOpRowCap / kOpRowBlock;
    if (static_cast<int>(blockIdx.x) >= nlong) {
        if (counters[2] == 0) return;
        op_sum_piece(static_cast<int64_t>(blockIdx.x) - nlong, bucket_off, m, P, static_cast<int>(ncols), bkt_col,
                     bkt_val, x_col, x_val, y_col, reinterpret_cast<uint32_t *>(s_key), s_val, s_key + kOpRowCap / 32,
                     s_scan, s_key + kOpRowCap / 16);
        return;
    }
    const int nrows = counters[0];
    for (int idx = blockIdx.x; idx < nrows; idx += nlong) {
        const int row = long_rows[idx];
        const int64_t lo = bucket_off[row];
        const int len = static_cast<int>(bucket_off[row + 1] - lo);
        if (ncols <= len) {
            // C has no more columns than the bucket entries: summed in LDS accumulators
            uint32_t *bits = reinterpret_cast<uint32_t *>(s_key);
            const int cols = static_cast<int>(ncols);
            for (int k = threadIdx.x; k < cols; k += kOpRowBlock) s_val[k] = 0.0;
            if (threadIdx.x < kOpRowCap / 32) bits[threadIdx.x] = 0u;
            __syncthreads();
            for (int e = threadIdx.x; e < len; e += kOpRowBlock) {
                const int k = bkt_col[lo + e];   // (a column that is none of B's stays out of the LDS)
                if (static_cast<uint32_t>(k) < static_cast<uint32_t>(cols)) op_add(bits, s_val, k, bkt_val[lo + e]);
            }
            __syncthreads();
            const int n = op_emit_window(0, cols, bits, s_val, s_key + kOpRowCap / 32, s_scan, bkt_col + lo,
                                         out_val + lo);
            if (threadIdx.x == 0) row_nnz[row] = n;
            __syncthreads();
            continue;
        }
        int np = kWave * 2;
        while (np < len) np <<= 1;
        for (int s = threadIdx.x; s < np; s += blockDim.x) {
            s_key[s] = s < len ? bkt_col[lo + s] : 0x7fffffff;
            s_val[s] = s < len ? bkt_val[lo + s] : 0.0;
        }
        __syncthreads();
        lds_bitonic(s_key, s_val, np);
        // PER consecutive entries per thread: their heads, and the sum of the segment open at their end
        const int s0 = threadIdx.x * PER;
        int heads = 0;
        double open = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int s = s0 + u;
            if (s >= len) continue;
            const bool head = s == 0 || s_key[s - 1] != s_key[s];
            heads += head ? 1 : 0;
            open = head ? s_val[s] : open + s_val[s];
        }
        double sum = block_open_sum(open, heads > 0, s_part, s_any);
        int total = 0;
        int pos = block_excl_scan(heads, s_scan, &total);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int s = s0 + u;
            if (s >= len) continue;
            const int kk = s_key[s];
            const bool head = s == 0 || s_key[s - 1] != kk;
            sum = head ? s_val[s] : sum + s_val[s];
            pos += head ? 1 : 0;
            if (s == len - 1 || s_key[s + 1] != kk) {
                bkt_col[lo + pos - 1] = kk;
                out_val[lo + pos - 1] = static_cast<V>(sum);
            }
        }
        if (threadIdx.x == 0) row_nnz[row] = total;
        __syncthreads();   // LDS is reused by the next row
    }
}

__device__ __forceinline__ int lds_lower_bound(const int32_t *k, int n, int32_t key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (k[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int lds_upper_bound(const int32_t *k, int n, int32_t key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (k[mid] <= key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// 3d. Buckets longer than kOpRowCap, a workgroup per row, rows taken
// grid-stride from the back of long_rows (op_merge_mid lists them there). Those
// summed by pieces (op_by_pieces): their pieces' entries are added up in LDS, a
// wave per piece, window by window of C's columns. The others:
//   runs of kOpRowCap entries are sorted in LDS into buffer X; then runs are
//   merged pairwise, X to Y and back, doubling their length until one is left:
//   each output tile of kOpRowCap entries takes its share of the two runs
//   (merge-path splits at its ends), merges it in LDS by ranks and writes it
//   out coalesced; last, the sorted row is compacted into the bucket's start,
//   equal columns summed by a segmented scan (one lane adding up a run of them:
//   50 rows of 20 K equal columns 9.5 ms, now 0.5). X and Y hold a column array and a value array
//   each, indexed like the bucket; y_val is bkt_val itself (the first step has
//   read the row's bucket before the first merge overwrites it).
template <typename V>
__global__ void __launch_bounds__(kOpHugeBlock) op_merge_huge(const int64_t *__restrict__ bucket_off, int64_t m,
                                                              int64_t ncols, int32_t *bkt_col, double *bkt_val, V *out_val,
                                                              int32_t *__restrict__ row_nnz,
                                                              const int32_t *__restrict__ long_rows,
                                                              const int32_t *counters, int32_t *x_col, double *x_val,
                                                              int32_t *y_col) {
    __shared__ int32_t s_key[kOpRowCap];
    __shared__ double s_val[kOpRowCap];
    __shared__ int32_t o_key[kOpRowCap];
    __shared__ double o_val[kOpRowCap];
    __shared__ int64_t s_split[2];
    __shared__ int s_scan[kOpHugeBlock / kWave];
    __shared__ double s_part[kOpHugeBlock / kWave + 1];
    __shared__ int s_any[kOpHugeBlock / kWave];
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int ln = lane_id();
    const int nrows = counters[2];
    for (int idx = blockIdx.x; idx < nrows; idx += gridDim.x) {
        const int row = long_rows[m - 1 - idx];
        const int64_t lo = bucket_off[row];
        const int64_t len = bucket_off[row + 1] - lo;
        if (op_by_pieces(len, ncols)) {
            uint32_t *bits = reinterpret_cast<uint32_t *>(s_key);
            int done = 0;
            for (int w0 = 0; w0 < static_cast<int>(ncols); w0 += kOpRowCap) {
                const int cols = static_cast<int>(ncols) - w0 < kOpRowCap ? static_cast<int>(ncols) - w0 : kOpRowCap;
                for (int k = threadIdx.x; k < cols; k += kOpHugeBlock) s_val[k] = 0.0;
                if (threadIdx.x < kOpRowCap / 32) bits[threadIdx.x] = 0u;
                __syncthreads();
                for (int64_t c = lo / kOpPiece + wv; c * kOpPiece < lo + len; c += kOpHugeBlock / kWave) {
                    const int64_t a = c * kOpPiece > lo ? c * kOpPiece : lo;
                    const int n = y_col[a];
                    for (int i0 = ln; i0 < n; i0 += 4 * kWave) {
                        int col[4];
                        double v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int i = i0 + u * kWave;
                            col[u] = i < n ? x_col[a + i] : -1;
                            v[u] = i < n ? x_val[a + i] : 0.0;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int k = col[u] - w0;
                            if (static_cast<uint32_t>(k) < static_cast<uint32_t>(cols)) op_add(bits, s_val, k, v[u]);
                        }
                    }
                }
                __syncthreads();
                done += op_emit_window(w0, cols, bits, s_val, s_key + kOpRowCap / 32, s_scan, bkt_col + lo + done,
                                       out_val + lo + done);
                __syncthreads();
            }
            if (threadIdx.x == 0) row_nnz[row] = done;
            continue;
        }
        // runs sorted in LDS, bucket -> X
        for (int64_t r0 = 0; r0 < len; r0 += kOpRowCap) {
            const int n = static_cast<int>(len - r0 < kOpRowCap ? len - r0 : kOpRowCap);
            int np = kWave * 2;
            while (np < n) np <<= 1;
            for (int e = threadIdx.x; e < np; e += blockDim.x) {
                s_key[e] = e < n ? bkt_col[lo + r0 + e] : 0x7fffffff;
                s_val[e] = e < n ? bkt_val[lo + r0 + e] : 0.0;
            }
            __syncthreads();
            lds_bitonic(s_key, s_val, np);
            for (int e = threadIdx.x; e < n; e += blockDim.x) {
                x_col[lo + r0 + e] = s_key[e];
                x_val[lo + r0 + e] = s_val[e];
            }
            __syncthreads();
        }
        // pairwise merges, ping-pong between X and Y
        int32_t *sc = x_col, *dc = y_col;
        double *sv = x_val, *dv = bkt_val;
        for (int64_t w = kOpRowCap; w < len; w <<= 1) {
            for (int64_t s = 0; s < len; s += 2 * w) {
                const int64_t na = len - s < w ? len - s : w;
                const int64_t nb = len - s - na < w ? len - s - na : w;
                const int32_t *ak = sc + lo + s, *bk = ak + na;
                const double *av = sv + lo + s, *bv = av + na;
                for (int64_t d0 = 0; d0 < na + nb; d0 += kOpRowCap) {
                    const int64_t d1 = na + nb - d0 < kOpRowCap ? na + nb : d0 + kOpRowCap;
                    if (threadIdx.x < 2 * kWave) {
                        const int64_t i = wave_merge_split(ak, na, bk, nb, threadIdx.x < kWave ? d0 : d1);
                        if (lane_id() == 0) s_split[threadIdx.x / kWave] = i;
                    }
                    __syncthreads();
                    const int64_t i0 = s_split[0], i1 = s_split[1];
                    const int sa = static_cast<int>(i1 - i0), nt = static_cast<int>(d1 - d0);
                    const int64_t j0 = d0 - i0;
                    for (int e = threadIdx.x; e < nt; e += blockDim.x) {
                        s_key[e] = e < sa ? ak[i0 + e] : bk[j0 + (e - sa)];
                        s_val[e] = e < sa ? av[i0 + e] : bv[j0 + (e - sa)];
                    }
                    __syncthreads();
                    for (int e = threadIdx.x; e < nt; e += blockDim.x) {
                        const int32_t key = s_key[e];
                        const int pos = e < sa ? e + lds_lower_bound(s_key + sa, nt - sa, key)
                                               : (e - sa) + lds_upper_bound(s_key, sa, key);
                        o_key[pos] = key;
                        o_val[pos] = s_val[e];
                    }
                    __syncthreads();
                    for (int e = threadIdx.x; e < nt; e += blockDim.x) {
                        dc[lo + s + d0 + e] = o_key[e];
                        dv[lo + s + d0 + e] = o_val[e];
                    }
                    __syncthreads();   // s_split and the LDS tiles are reused
                }
            }
            int32_t *tc = sc;
            sc = dc;
            dc = tc;
            double *tv = sv;
            sv = dv;
            dv = tv;
        }
        // compaction of the sorted row (sc, sv) into the bucket's start: a segment's last entry writes its sum
        int64_t base = 0;
        for (int64_t e0 = 0; e0 < len; e0 += kOpHugeBlock) {
            const int64_t e = e0 + threadIdx.x;
            const bool live = e < len;
            const int32_t key = live ? sc[lo + e] : 0;
            const bool head = live && (e == 0 || sc[lo + e - 1] != key);
            const bool tail = live && (e == len - 1 || sc[lo + e + 1] != key);
            double sum = live ? sv[lo + e] : 0.0;
            const double open = block_open_sum(sum, head, s_part, s_any);
            if (!head) sum += open;
            int total = 0;
            const int pos = block_excl_scan(head ? 1 : 0, s_scan, &total);
            if (tail) {
                const int64_t at = lo + base + pos + (head ? 1 : 0) - 1;
                bkt_col[at] = key;
                out_val[at] = static_cast<V>(sum);
            }
            if (threadIdx.x == kOpHugeBlock - 1) s_part[0] = sum;
            base += total;
        }
        if (threadIdx.x == 0) row_nnz[row] = static_cast<int32_t>(base);
        __syncthreads();   // LDS is reused by the next row
    }
}

}  // namespace wsp
