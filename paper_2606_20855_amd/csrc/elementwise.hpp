// Elementwise operations on two CSR matrices of one shape (paper, Section 5.2:
// SpAdd, C = A + B, and the Hadamard product, C = A .* B): a row of C is the
// sorted merge of the same rows of A and B, the union of their columns for
// the sum (an entry stored on both sides takes a + b, including an exact
// zero) and the intersection for the product.
//
// A and B are read as one merged sequence: all entries of both in row-major
// (row, column) order, A's entry first where both store a coordinate. The
// sequence is cut into tiles of kEwTile entries by merge-path splits
// (ew_tile_splits: the row holding a boundary found on the summed row
// pointers, then a split of that row's two column lists), a boundary that
// would separate the two entries of a common coordinate taking the B entry
// along. A tile's shares of A and of B are contiguous runs of their entry
// arrays, so a workgroup loads both with coalesced reads into LDS as
// (row, column) keys and matches them there:
//   ew_tile_count: merges the tile: C's entries from it, a two-bit code per
//                  merged entry (which side it is from, whether the other side
//                  stores its coordinate too), and each row's place in the tile;
//   ew_row_ptr:    C's row pointer, from the rows' places and the scan of the
//                  tiles' counts;
//   ew_tile_write: C's entries of a tile from the codes alone (popcounts give
//                  each entry's places in A, B and C), no keys merged again.
// Long and short rows balance by themselves; nothing but the entries, the
// row pointers and C is read or written at the size of the inputs (the codes
// are half a byte per entry).
#pragma once

#include "search.hpp"

namespace wsp {

constexpr int kEwTile = 2048;    // merged entries per tile (one more when a common coordinate straddles)
constexpr int kEwBlock = 256;
constexpr int kEwPer = (kEwTile + 1 + kEwBlock - 1) / kEwBlock;   // consecutive tile positions per thread
enum EwOp { kEwAdd = 0, kEwMul = 1 };
constexpr int64_t kEwEnd = 0x7fffffffffffffffll;   // above every (row, column) key

// Tile boundaries, one wave each: for t in [0, ntiles], d = min(t kEwTile,
// nnz(A) + nnz(B)); split_a[t] and split_b[t] count the A and B entries before
// boundary t and split_r[t] is the row holding it (nrows - 1 at the end).
// nrows >= 1.
__global__ void __launch_bounds__(256) ew_tile_splits(const int32_t *__restrict__ a_rp,
                                                      const int32_t *__restrict__ a_col,
                                                      const int32_t *__restrict__ b_rp,
                                                      const int32_t *__restrict__ b_col, int nrows, int64_t ntiles,
                                                      int64_t *__restrict__ split_a, int64_t *__restrict__ split_b,
                                                      int32_t *__restrict__ split_r) {
    const int64_t t = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
    if (t > ntiles) return;   // whole wave
    const int64_t na_all = a_rp[nrows], nb_all = b_rp[nrows];
    const int64_t total = na_all + nb_all;
    const int64_t d = t * kEwTile < total ? t * kEwTile : total;
    int64_t ia = na_all, ib = nb_all;
    int r = nrows - 1;
    if (d < total) {
        r = wave_last_le([=](int k) { return static_cast<int64_t>(a_rp[k]) + b_rp[k]; }, 0, nrows - 1, d);
        const int64_t ar = a_rp[r], br = b_rp[r];
        const int64_t na = a_rp[r + 1] - ar, nb = b_rp[r + 1] - br;
        const int64_t dd = d - ar - br;   // < na + nb: row r holds position d
        const int64_t i = wave_merge_split(a_col + ar, na, b_col + br, nb, dd);
        int64_t j = dd - i;
        if (i > 0 && j < nb && a_col[ar + i - 1] == b_col[br + j]) ++j;   // keep a common pair together
        ia = ar + i;
        ib = br + j;
    }
    if (lane_id() == 0) {
        split_a[t] = ia;
        split_b[t] = ib;
        split_r[t] = r;
    }
}

// A tile's shares and rows: A entries [ia0, ia0 + na), B entries
// [ib0, ib0 + nb), all in rows [r0, r0 + nr).
struct EwTile {
    int64_t ia0, ib0;
    int na, nb, r0, nr;
};

__device__ __forceinline__ EwTile ew_tile_of(const int64_t *__restrict__ split_a, const int64_t *__restrict__ split_b,
                                             const int32_t *__restrict__ split_r) {
    const int t = blockIdx.x;
    EwTile T;
    T.ia0 = split_a[t];
    T.ib0 = split_b[t];
    T.na = static_cast<int>(split_a[t + 1] - T.ia0);
    T.nb = static_cast<int>(split_b[t + 1] - T.ib0);
    T.r0 = split_r[t];
    T.nr = split_r[t + 1] - T.r0 + 1;
    return T;
}

// A DPP lane move of an unsigned value; lanes with no source read 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROW_MASK, 0xf, false));
}

// Inclusive wave max-scan of unsigned values (identity 0): row shifts within
// 16-lane rows, then row broadcasts of lanes 15 and 31.
__device__ __forceinline__ uint32_t wave_incl_umax(uint32_t v) {
    v = max(v, dpp_u32<kDppRowShr1, 0xf>(v));
    v = max(v, dpp_u32<kDppRowShr2, 0xf>(v));
    v = max(v, dpp_u32<kDppRowShr4, 0xf>(v));
    v = max(v, dpp_u32<kDppRowShr8, 0xf>(v));
    v = max(v, dpp_u32<kDppRowBcast15, 0xa>(v));
    v = max(v, dpp_u32<kDppRowBcast31, 0xc>(v));
    return v;
}

// Exclusive block-wide max-scan of unsigned values (0 for thread 0).
// `scratch` holds BLOCK/64 ints.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_excl_umax(uint32_t x, int *scratch) {
    constexpr int NW = BLOCK / kWave;
    const uint32_t incl = wave_incl_umax(x);
    const int w = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) scratch[w] = static_cast<int>(incl);
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) before = i < w ? max(before, static_cast<uint32_t>(scratch[i])) : before;
    __syncthreads();
    const uint32_t prev = static_cast<uint32_t>(__shfl_up(static_cast<int>(incl), 1, kWave));
    return max(before, lane_id() == 0 ? 0u : prev);
}

// Loads a tile as (row, column) keys in LDS, A's share at [0, na) and B's at
// [na, na + nb): the columns, with coalesced reads, into the keys' low halves, and, at the same time, the row
// pointers of the tile's rows. Then each row that starts inside a share marks
// its first position in the key's high half (row r0 + k as k + 1 in A's
// share, nr + k + 1 in B's, so one max-scan over both shares serves and B's
// marks exceed all of A's), and an exclusive max-scan over the positions,
// kEwPer consecutive ones per thread, replaces the marks by the rows. All
// threads call it.
__device__ __forceinline__ void ew_load_tile(const EwTile &T, const int32_t *__restrict__ a_rp,
                                             const int32_t *__restrict__ a_col, const int32_t *__restrict__ b_rp,
                                             const int32_t *__restrict__ b_col, int64_t *s_key, int *scratch) {
    uint32_t *half = reinterpret_cast<uint32_t *>(s_key);   // [2p] column, [2p + 1] mark, then row
    const int n = T.na + T.nb;
    const uint32_t nr = static_cast<uint32_t>(T.nr);
    // the first kEwBlock rows' pointers, read beside the columns
    const int k0 = threadIdx.x;
    int64_t sa0 = -1, ea0 = -1, sb0 = -1, eb0 = -1;
    if (k0 < T.nr) {
        sa0 = a_rp[T.r0 + k0] - T.ia0;
        ea0 = a_rp[T.r0 + k0 + 1] - T.ia0;
        sb0 = b_rp[T.r0 + k0] - T.ib0;
        eb0 = b_rp[T.r0 + k0 + 1] - T.ib0;
    }
    // position p of the tile (A's share, then B's), kEwPer per thread strided by the block: all loads
    // issued before the first is waited for
    int32_t col[kEwPer];
#pragma unroll
    for (int u = 0; u < kEwPer; ++u) {
        const int p = threadIdx.x + u * kEwBlock;
        col[u] = 0;
        if (p < T.na) col[u] = a_col[T.ia0 + p];
        else if (p < n) col[u] = b_col[T.ib0 + (p - T.na)];
    }
#pragma unroll
    for (int u = 0; u < kEwPer; ++u) {
        const int p = threadIdx.x + u * kEwBlock;
        if (p < n) s_key[p] = static_cast<uint32_t>(col[u]);
    }
    __syncthreads();
    // a non-empty row starting inside a share is the only one to mark that position
    if (k0 < T.nr) {
        if (sa0 >= 0 && sa0 < T.na && ea0 > sa0) half[2 * sa0 + 1] = static_cast<uint32_t>(k0) + 1u;
        if (sb0 >= 0 && sb0 < T.nb && eb0 > sb0) half[2 * (T.na + sb0) + 1] = nr + static_cast<uint32_t>(k0) + 1u;
    }
    for (int k = k0 + blockDim.x; k < T.nr; k += blockDim.x) {   // tiles over many empty rows
        const int64_t sa = a_rp[T.r0 + k] - T.ia0, ea = a_rp[T.r0 + k + 1] - T.ia0;
        if (sa >= 0 && sa < T.na && ea > sa) half[2 * sa + 1] = static_cast<uint32_t>(k) + 1u;
        const int64_t sb = b_rp[T.r0 + k] - T.ib0, eb = b_rp[T.r0 + k + 1] - T.ib0;
        if (sb >= 0 && sb < T.nb && eb > sb) half[2 * (T.na + sb) + 1] = nr + static_cast<uint32_t>(k) + 1u;
    }
    __syncthreads();
    const int p0 = threadIdx.x * kEwPer;
    uint32_t mk[kEwPer];
    uint32_t x = 0;
#pragma unroll
    for (int u = 0; u < kEwPer; ++u) {
        const int p = p0 + u;
        uint32_t v = p < n ? half[2 * p + 1] : 0u;
        if (p == 0 && T.na > 0) v = max(v, 1u);             // A's share starts in row r0
        if (p == T.na && T.nb > 0) v = max(v, nr + 1u);     // and so does B's
        mk[u] = v;
        x = max(x, v);
    }
    uint32_t run = block_excl_umax<kEwBlock>(x, scratch);
#pragma unroll
    for (int u = 0; u < kEwPer; ++u) {
        const int p = p0 + u;
        run = max(run, mk[u]);
        if (p < n) half[2 * p + 1] = static_cast<uint32_t>(T.r0) + (p < T.na ? run - 1u : run - nr - 1u);
    }
    __syncthreads();
}

// Merge-path split inside a tile: the number of A's share among the first d
// entries of the tile's merged order (A first on equal keys).
__device__ __forceinline__ int ew_split(const int64_t *s_key, int na, int nb, int d) {
    int lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s_key[mid] > s_key[na + d - mid - 1]) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// A thread's codes: two bits for each of its kEwPer consecutive merged entries,
// bit 0: the entry is B's, bit 1: its coordinate is common to both sides. (A's
// half of a common coordinate comes first.)
constexpr uint32_t kEwBit = 0x55555555u & ((1u << (2 * kEwPer)) - 1u);
static_assert(2 * kEwPer <= 32, "a thread's codes in one word");
// The low bits of the codes of the first cnt entries.
__device__ __forceinline__ uint32_t ew_valid(int cnt) {
    return cnt >= kEwPer ? kEwBit : (cnt <= 0 ? 0u : kEwBit & ((1u << (2 * cnt)) - 1u));
}
// The entries kept in C, of those in `valid`: for the sum all but the B half of
// a common coordinate, for the product its A half.
__device__ __forceinline__ uint32_t ew_kept(uint32_t codes, uint32_t valid, int op) {
    const uint32_t b = codes & valid, c = (codes >> 1) & valid;
    return op == kEwAdd ? valid & ~(b & c) : c & ~b;
}

// Per tile: tile_cnt[t] = C's entries from the tile, the threads' codes, and for
// every row r that starts in the tile (rows without entries too) row_at[r] = C's
// entries of the tile before the row (rows may be null: the caller has C's row
// pointer). Each thread walks kEwPer positions of the merged order. Bound by VALU
// issue (the sum of R-MAT 20 and its shuffled copy: 71 us, the VALU busy all the
// time, 2.4 TB/s).
__global__ void __launch_bounds__(kEwBlock) ew_tile_count(const int32_t *__restrict__ a_rp,
                                                          const int32_t *__restrict__ a_col,
                                                          const int32_t *__restrict__ b_rp,
                                                          const int32_t *__restrict__ b_col,
                                                          const int64_t *__restrict__ split_a,
                                                          const int64_t *__restrict__ split_b,
                                                          const int32_t *__restrict__ split_r, int op,
                                                          int32_t *__restrict__ tile_cnt,
                                                          uint32_t *__restrict__ codes_out,
                                                          int32_t *__restrict__ row_at) {
    __shared__ int64_t s_key[kEwTile + 1];
    __shared__ uint32_t s_kept[kEwBlock];   // a thread's kept entries, and C's entries before the thread
    __shared__ int32_t s_before[kEwBlock];
    __shared__ int32_t scratch[kEwBlock / kWave];
    const EwTile T = ew_tile_of(split_a, split_b, split_r);
    ew_load_tile(T, a_rp, a_col, b_rp, b_col, s_key, scratch);
    const int n = T.na + T.nb;
    const int d = threadIdx.x * kEwPer;
    uint32_t codes = 0;
    if (d < n) {
        int i = ew_split(s_key, T.na, T.nb, d), j = d - i;
        int64_t ka = i < T.na ? s_key[i] : kEwEnd, kb = j < T.nb ? s_key[T.na + j] : kEwEnd;
        int64_t prev_a = i > 0 ? s_key[i - 1] : -1;
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            if (d + u >= n) continue;
            const bool from_b = ka > kb;
            const bool common = from_b ? prev_a == kb : ka == kb;
            codes |= (static_cast<uint32_t>(from_b) | static_cast<uint32_t>(common) << 1) << (2 * u);
            if (from_b) {
                ++j;
                kb = j < T.nb ? s_key[T.na + j] : kEwEnd;
            } else {
                prev_a = ka;
                ++i;
                ka = i < T.na ? s_key[i] : kEwEnd;
            }
        }
    }
    codes_out[static_cast<int64_t>(blockIdx.x) * kEwBlock + threadIdx.x] = codes;
    const uint32_t kept = ew_kept(codes, ew_valid(n - d), op);
    int total;
    const int before = block_excl_scan<kEwBlock>(static_cast<int>(__popc(kept)), &total, scratch);
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = total;
    if (row_at == nullptr) return;
    s_kept[threadIdx.x] = kept;
    s_before[threadIdx.x] = before;
    __syncthreads();
    for (int k = threadIdx.x; k < T.nr; k += kEwBlock) {
        // the row's first place in the tile; rows of earlier and later tiles are theirs, but for rows that start
        // where the tile ends: the next tile begins at the last of them, and its count before each is 0
        const int64_t p = (a_rp[T.r0 + k] - T.ia0) + (b_rp[T.r0 + k] - T.ib0);
        if (p == n) row_at[T.r0 + k] = 0;
        if (p < 0 || p >= n) continue;
        const int t = static_cast<int>(p) / kEwPer, u = static_cast<int>(p) - t * kEwPer;
        row_at[T.r0 + k] = s_before[t] + static_cast<int>(__popc(s_kept[t] & ((1u << (2 * u)) - 1u)));
    }
}

// C's row pointer: row r starts in the tile its first merged position lies in
// (a boundary that moved past the B half of a common coordinate moved inside a
// row). The last thread also hands the total to the host (host_total may be
// null).
__global__ void __launch_bounds__(256) ew_row_ptr(const int32_t *__restrict__ a_rp, const int32_t *__restrict__ b_rp,
                                                  int64_t nrows, int64_t total_in, int64_t ntiles,
                                                  const int64_t *__restrict__ tile_off,
                                                  const int32_t *__restrict__ row_at, int64_t *__restrict__ c_rp,
                                                  int64_t *host_total) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (r > nrows) return;
    const int64_t p = static_cast<int64_t>(a_rp[r]) + b_rp[r];
    int64_t c = 0;   // rows before the first entry (the first tile begins at the last of them)
    if (p >= total_in) c = tile_off[ntiles];
    else if (p > 0) c = tile_off[p / kEwTile] + row_at[r];
    c_rp[r] = c;
    if (r == nrows && host_total != nullptr) *host_total = c;
}

// The same where a side stores nothing: the other side's rows (sum) or none.
__global__ void __launch_bounds__(256) ew_row_ptr_one_side(const int32_t *__restrict__ a_rp,
                                                           const int32_t *__restrict__ b_rp, int64_t nrows, int op,
                                                           int64_t *__restrict__ c_rp, int64_t *host_total) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (r > nrows) return;
    const int64_t c = op == kEwAdd ? static_cast<int64_t>(a_rp[r]) + b_rp[r] : 0;
    c_rp[r] = c;
    if (r == nrows && host_total != nullptr) *host_total = c;
}

struct EwTileIn {
    const int32_t *cnt;
    __device__ __forceinline__ int64_t operator()(int64_t t) const { return cnt[t]; }
};

// C's entries from a tile, from tile_off[t] on: each thread's codes and one scan
// give its entries' places in A's share, B's share and C; values are formed in
// double and rounded once, and the tile's part of C is staged in LDS and written
// with coalesced stores. The sum needs every entry: both shares are read with
// coalesced loads issued before the codes are looked at, and the codes' owners
// leave each entry's place in C in LDS. The product reads the common entries
// alone, by the threads that own their codes.
//
// Bound by HBM, 5.9 TB/s fetched and written in the sum (the sum of R-MAT 20 and
// its shuffled copy, double: 32 M entries in and out, 780 MB: merging the keys
// again in this kernel 175 us, from the codes 137 us, with each thread reading
// its own entries 228 us; the product of R-MAT 18 with its pattern, float: 46
// us, now 26 us).
template <typename V, int OP>
__global__ void __launch_bounds__(kEwBlock) ew_tile_write(const int32_t *__restrict__ a_col,
                                                          const V *__restrict__ a_val,
                                                          const int32_t *__restrict__ b_col,
                                                          const V *__restrict__ b_val,
                                                          const int64_t *__restrict__ split_a,
                                                          const int64_t *__restrict__ split_b,
                                                          const uint32_t *__restrict__ codes_in,
                                                          const int64_t *__restrict__ tile_off,
                                                          int32_t *__restrict__ c_col, V *__restrict__ c_val) {
    __shared__ V s_oval[kEwTile + 1];
    __shared__ int32_t s_ocol[kEwTile + 1];
    __shared__ int32_t s_place[OP == kEwAdd ? kEwTile + 1 : 1];
    __shared__ int32_t scratch[kEwBlock / kWave];
    const int t = blockIdx.x;
    const int64_t ia0 = split_a[t], ib0 = split_b[t];
    const int na = static_cast<int>(split_a[t + 1] - ia0);
    const int n = na + static_cast<int>(split_b[t + 1] - ib0);
    const int64_t base = tile_off[t];
    const uint32_t codes = codes_in[static_cast<int64_t>(t) * kEwBlock + threadIdx.x];
    // the sum: both shares' entries (A's, then B's), strided by the workgroup
    int32_t col[OP == kEwAdd ? kEwPer : 1];
    V val[OP == kEwAdd ? kEwPer : 1];
    if constexpr (OP == kEwAdd) {
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            const int e = threadIdx.x + u * kEwBlock;
            col[u] = 0;
            val[u] = V(0);
            if (e < na) {
                col[u] = a_col[ia0 + e];
                val[u] = a_val[ia0 + e];
            } else if (e < n) {
                col[u] = b_col[ib0 + (e - na)];
                val[u] = b_val[ib0 + (e - na)];
            }
        }
    }
    const int d = threadIdx.x * kEwPer;
    const uint32_t valid = ew_valid(n - d);
    const uint32_t kept = ew_kept(codes, valid, OP);
    const int from_a = __popc(valid & ~codes);
    // places in A's share and in C: one scan of both counts (at most 2049 each)
    int tot;
    const int at = block_excl_scan<kEwBlock>(static_cast<int>(__popc(kept)) | from_a << 16, &tot, scratch);
    int p = at & 0xffff;
    int i = at >> 16, j = (d < n ? d : n) - i;
    tot &= 0xffff;
    if constexpr (OP == kEwAdd) {
        // every entry's place in C; the B half of a common coordinate: ~(the place of the entry before it, its A half)
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            if (((valid >> (2 * u)) & 1u) == 0u) continue;
            const bool keep = ((kept >> (2 * u)) & 1u) != 0u, from_b = ((codes >> (2 * u)) & 1u) != 0u;
            s_place[from_b ? na + j : i] = keep ? p : ~(p - 1);
            p += keep;
            i += !from_b;
            j += from_b;
        }
        __syncthreads();
        int at_c[kEwPer];
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            const int e = threadIdx.x + u * kEwBlock;
            at_c[u] = e < n ? s_place[e] : -1;
            if (e < n && at_c[u] >= 0) {
                s_ocol[at_c[u]] = col[u];
                s_oval[at_c[u]] = val[u];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            const int e = threadIdx.x + u * kEwBlock;
            if (e < n && at_c[u] < 0)   // (a + b in double, rounded once)
                s_oval[~at_c[u]] = static_cast<V>(to_d(s_oval[~at_c[u]]) + to_d(val[u]));
        }
    } else {
        int32_t oc[kEwPer];
        double av[kEwPer], bv[kEwPer];
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            const uint32_t c = (codes >> (2 * u)) & 3u;
            oc[u] = 0;
            av[u] = 0.0;
            bv[u] = 0.0;
            if (((kept >> (2 * u)) & 1u) != 0u) {
                // A's half of a common coordinate: B's is the next of B's share
                oc[u] = a_col[ia0 + i];
                av[u] = to_d(a_val[ia0 + i]);
                bv[u] = to_d(b_val[ib0 + j]);
            }
            i += (c & 1u) ? 0 : 1;
            j += (c & 1u) ? 1 : 0;
        }
#pragma unroll
        for (int u = 0; u < kEwPer; ++u) {
            if (((kept >> (2 * u)) & 1u) != 0u) {
                s_ocol[p] = oc[u];
                s_oval[p] = static_cast<V>(av[u] * bv[u]);
                ++p;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEwPer; ++u) {
        const int e = threadIdx.x + u * kEwBlock;
        if (e < tot) {
            c_col[base + e] = s_ocol[e];
            c_val[base + e] = s_oval[e];
        }
    }
}

}  // namespace wsp
