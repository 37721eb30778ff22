// Merge rows (part of the hash tier): rows of few A entries. Such a row's
// products are already sorted runs, one per A entry (the selected row of B), so
// they are merged in LDS, pairwise, instead of hashed and sorted again. Equal
// columns are summed in the order of A's entries.
//
// Bound by VALU issue: the work of a product is a merge step per pass, about 13
// instructions, and ceil(log2(runs)) passes (counters on the graphs below: the
// VALU busy all the time where products are only counted, two thirds to nine
// tenths of it where they are formed; the largest size, whose B values are
// gathered at 3.8 to 5.1 TB/s, the least). Measured on rows of R-MAT graphs
// (edge factor 2 and 4, rows of 65 to 8192 products, 1 to 64 runs, mostly 2 to
// 8), against LDS hash tables with their sorted emission: 2.5 M columns, float,
// 435 M products 17.8 ms, here 513 M products (with rows the tables were too
// small for) 4.2 ms; 1 M columns, double, 121 M products 3.48 ms against 0.85
// ms; counting only (symbolic), 513 M products 3.7 ms against 1.85 ms.
#pragma once

#include "tiers.hpp"

namespace wsp {

// One workgroup per row of at most kMergeMaxRuns A entries and CAP places.
template <int CAP, bool NUM>
struct MergeShape {
    // Places per thread: more of them spread a pass's merge-path search over more steps, but in the numeric kernel
    // take the registers that hide the latency (16 places: symbolic 2.3 -> 1.85 ms, numeric 4.7 -> 5.5 ms).
    static constexpr int LOG2VT = CAP <= 256 ? 2 : (CAP <= 512 || NUM ? 3 : 4);
    static constexpr int VT = 1 << LOG2VT;
    static constexpr int BLOCK = CAP / VT;
    static_assert(VT - 1 <= (NUM ? kMergePadNum : kMergePadSym), "the binning allows for every run's padding");
    // wavefronts per SIMD: two workgroups of 1024 threads per CU (their LDS allows it) instead of one (the largest
    // numeric size: 2.4 -> 1.9 ms)
    static constexpr int WAVES = BLOCK >= 1024 ? 8 : 1;
    // Where place p of the row lies in LDS, p in [-1, CAP]: a gap after every VT places keeps threads that read
    // or write VT consecutive places each on separate banks.
    static constexpr int ITEMS = 2 + CAP + CAP / VT + 1;
    __device__ static __forceinline__ int at(int p) { return p + (p >> LOG2VT) + 2; }
};

// A product in LDS: its column and, in the numeric kernel, below it where the
// product comes from (run << 16 | place in the row's product order). The values
// stay in B until the order is known: half the LDS and half its traffic of
// carrying doubles along.
template <bool NUM>
struct MergeItem {
    using type = uint64_t;
    __device__ static __forceinline__ int key(uint64_t t) { return static_cast<int>(t >> 32); }
    __device__ static __forceinline__ uint64_t make(int key, int from) {
        return static_cast<uint64_t>(static_cast<uint32_t>(key)) << 32 | static_cast<uint32_t>(from);
    }
};
template <>
struct MergeItem<false> {
    using type = int32_t;
    __device__ static __forceinline__ int key(int32_t t) { return t; }
    __device__ static __forceinline__ int32_t make(int key, int) { return key; }
};

template <int CAP, bool NUM>
struct MergeLds {
    using S = MergeShape<CAP, NUM>;
    __align__(16) typename MergeItem<NUM>::type item[S::ITEMS];
    uint64_t head[NUM ? CAP / kWave + 1 : 1];   // where runs of equal columns start, a bit per place
    double av[NUM ? kMergeMaxRuns : 1];
    int32_t boff[NUM ? kMergeMaxRuns : 1];
    int32_t pre[kMergeMaxRuns + 1];
    int32_t scratch[S::BLOCK / kWave];
};

// Merges the runs the lanes of every wave hold alike (lane l: B's entries
// [bs, bs + len) times av; together at most CAP places) and returns their
// entries of C. The numeric kernels write them: place(entries) gives where the
// first goes and how many may be written. All threads of the workgroup call it;
// a barrier must come before L is used again.
template <int CAP, bool NUM, typename V, typename Place>
__device__ __forceinline__ int merge_runs(const Mats<V> &M, MergeLds<CAP, NUM> &L, int bs, int len, double av,
                                          Place place, int32_t *__restrict__ c_col, V *__restrict__ c_val) {
    using S = MergeShape<CAP, NUM>;
    using I = MergeItem<NUM>;
    using T = typename I::type;
    constexpr int BLOCK = S::BLOCK;
    constexpr int VT = S::VT;
    constexpr int NW = BLOCK / kWave;
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int ln = lane_id();
    // runs without entries moved behind the others
    const uint64_t full = ballot(len > 0);
    const int nr = __popcll(full);
    {
        const uint64_t below = (1ull << ln) - 1ull;
        const int dst = 4 * (len > 0 ? __popcll(full & below) : nr + __popcll(~full & below));
        bs = __builtin_amdgcn_ds_permute(dst, bs);
        len = __builtin_amdgcn_ds_permute(dst, len);
        if (NUM)
            av = __hiloint2double(__builtin_amdgcn_ds_permute(dst, __double2hiint(av)),
                                  __builtin_amdgcn_ds_permute(dst, __double2loint(av)));
    }
    const int incl = wave_incl_sum(len);
    const int f = __builtin_amdgcn_readlane(incl, kWave - 1);
    int total;   // the runs' entries of C
    if (nr <= 1) {
        // one run: the row of B, scaled
        total = f;
        if (!NUM) return total;
        const longlong2 at = place(total);
        const int64_t cb = at.x, seg = at.y;
        const int lim = total < seg ? total : static_cast<int>(seg);
        const int b0 = __builtin_amdgcn_readlane(bs, 0);
        const double a = readlane_d(av, 0);
        for (int i = threadIdx.x; i < lim; i += BLOCK) {
            __builtin_nontemporal_store(M.b_col[b0 + i], &c_col[cb + i]);
            __builtin_nontemporal_store(static_cast<V>(a * to_d(M.b_val[b0 + i])), &c_val[cb + i]);
        }
        return total;
    }

    const int excl = incl - len;
    const int start = len > 0 ? excl : 0x7fffffff;
    const int boff = bs - excl;
    // every run's place begins at a multiple of VT, its last places holding pads (sorted behind every column)
    const int plen = (len + VT - 1) & ~(VT - 1);
    const int pincl = wave_incl_sum(plen);
    const int first = pincl - plen;
    const int n = __builtin_amdgcn_readlane(pincl, kWave - 1);   // places in use
    // product p of the run goes to place p + shift, in every second run (which descends, see the merge passes)
    // to place shift - p
    const int shift = (ln & 1) ? excl + pincl - 1 : first - excl;
    const T pad = I::make(kPadKey, -1);
    if (wv == 0) {
        L.pre[ln] = first;
        if (ln == 0) L.pre[kMergeMaxRuns] = n;
        if (NUM) {
            L.av[ln] = av;
            L.boff[ln] = boff;
        }
        for (int p = excl + len; p < excl + plen; ++p) L.item[S::at((ln & 1) ? shift - p : shift + p)] = pad;
    }
    // product p of the row (wave w takes [w VT 64, (w + 1) VT 64)): its run, its entry of B and its place
    const int wbase = wv * VT * kWave;
    {
        int32_t c[VT];
        int from[VT], to[VT];
#pragma unroll
        for (int u = 0; u < VT; ++u) {
            const int base = wbase + u * kWave;
            c[u] = 0;
            from[u] = 0;
            to[u] = 0;
            if (base >= f) continue;
            const int p = base + ln;
            const int last = (base + kWave < f ? base + kWave : f) - 1;
            const int ob = 63 - __clzll(ballot(start <= base));
            const int oe = 63 - __clzll(ballot(start <= last));
            int o = ob, bo = __builtin_amdgcn_readlane(boff, ob), sh = __builtin_amdgcn_readlane(shift, ob);
            for (int e = ob + 1; e <= oe; ++e) {
                const int e_boff = __builtin_amdgcn_readlane(boff, e);
                const int e_shift = __builtin_amdgcn_readlane(shift, e);
                if (p >= __builtin_amdgcn_readlane(start, e)) {
                    o = e;
                    bo = e_boff;
                    sh = e_shift;
                }
            }
            from[u] = o << 16 | p;
            to[u] = (o & 1) ? sh - p : sh + p;
            c[u] = M.b_col[bo + (p <= last ? p : last)];
        }
#pragma unroll
        for (int u = 0; u < VT; ++u)
            if (wbase + u * kWave + ln < f) L.item[S::at(to[u])] = I::make(c[u], from[u]);
    }
    __syncthreads();
    // Merge passes: groups of s runs pairwise, in place. A pair's left group ascends and its right group
    // descends, so what is left of the pair lies between the two ends i and j throughout and no end needs a check
    // (once one group is used up, its end walks into the other's largest entries). Each thread produces the VT
    // places from d0 on, which lie in one pair: the merge-path split of d0, then a serial merge. The pairs of the
    // next pass: written ascending and descending in turn.
    const int d0 = static_cast<int>(threadIdx.x) * VT;
    int r0 = 0;   // the run that held place d0
#pragma unroll
    for (int step = kMergeMaxRuns / 2; step >= 1; step >>= 1)
        if (L.pre[r0 + step] <= d0) r0 += step;
    for (int s = 1; s < nr; s <<= 1) {
        T x[VT];
        int to = 0;   // where place d0 goes: d0, or mirrored in its pair
        if (d0 < n) {
            const int g = r0 & ~(2 * s - 1);
            const int lo0 = L.pre[g], mid = L.pre[g + s], end = L.pre[g + 2 * s];
            const int d = d0 - lo0, na = mid - lo0, nb = end - mid;
            int lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
            while (lo < hi) {
                const int m = (lo + hi) >> 1;
                if (I::key(L.item[S::at(lo0 + m)]) <= I::key(L.item[S::at(end - d + m)])) lo = m + 1;
                else hi = m;
            }
            int i = lo0 + lo, j = end - 1 - d + lo;
            to = (g & (2 * s)) ? lo0 + end - 1 - d0 : d0;
            T xl = L.item[S::at(i)], xr = L.item[S::at(j)];
#pragma unroll
            for (int u = 0; u < VT; ++u) {
                const bool left = xl <= xr;   // (equal columns: the earlier run's, whichever end holds it)
                x[u] = left ? xl : xr;
                i += left ? 1 : 0;
                j -= left ? 0 : 1;
                const T nx = L.item[S::at(left ? i : j)];
                xl = left ? nx : xl;
                xr = left ? xr : nx;
            }
        }
        __syncthreads();
        if (d0 < n) {
            // (d0 and a mirrored d0 + 1 are multiples of VT: no gap inside the VT places)
            if (to == d0) {
#pragma unroll
                for (int u = 0; u < VT; ++u) L.item[S::at(d0) + u] = x[u];
            } else {
#pragma unroll
                for (int u = 0; u < VT; ++u) L.item[S::at(to) - u] = x[u];
            }
        }
        __syncthreads();
    }
    // the heads of runs of equal columns are the row's entries
    uint64_t heads[VT];
    T x[VT];
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < VT; ++u) {
        const int p = wbase + u * kWave + ln;
        x[u] = pad;
        bool head = false;
        if (p < f) {
            x[u] = L.item[S::at(p)];
            head = p == 0 || I::key(L.item[S::at(p - 1)]) != I::key(x[u]);
        }
        heads[u] = ballot(head);
        cnt += __popcll(heads[u]);
        if (NUM && ln == 0) L.head[wv * VT + u] = heads[u];
    }
    if (ln == 0) L.scratch[wv] = cnt;
    if constexpr (NUM) {
        // the products, in column order
        double v[VT];
        {
            V b[VT];
#pragma unroll
            for (int u = 0; u < VT; ++u) {
                const int p = wbase + u * kWave + ln;
                const int from = p < f ? static_cast<int>(x[u] & 0xffffffffu) : 0;
                b[u] = M.b_val[L.boff[from >> 16] + (from & 0xffff)];
                v[u] = L.av[from >> 16];
            }
#pragma unroll
            for (int u = 0; u < VT; ++u) v[u] *= to_d(b[u]);
        }
        __syncthreads();   // every item and head is in registers, every count in scratch
        int before = 0;
        total = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int t = L.scratch[i];
            before += i < wv ? t : 0;
            total += t;
        }
        total = uniform(total);
        const longlong2 at = place(total);
        const int64_t cb = at.x, seg = at.y;
        if (total < f) {
            // equal columns: the head adds the products after it (in the order of A's entries), which take the
            // items' place in LDS
            double *s_prod = reinterpret_cast<double *>(L.item);
#pragma unroll
            for (int u = 0; u < VT; ++u) s_prod[S::at(wbase + u * kWave + ln)] = v[u];
            if (threadIdx.x == 0) L.head[CAP / kWave] = 0;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < VT; ++u) {
                const int p = wbase + u * kWave + ln;
                if ((heads[u] >> ln) & 1ull) {
                    // up to kMergeMaxRuns equal columns: the next head is in this word of 64 places or the next
                    const uint64_t here = ln < kWave - 1 ? heads[u] >> (ln + 1) : 0ull;
                    int eq = here ? __ffsll(static_cast<long long>(here)) : 0;
                    if (eq == 0) {
                        const uint64_t next = L.head[wv * VT + u + 1];
                        eq = kWave - ln + (next ? __ffsll(static_cast<long long>(next)) - 1 : kWave);
                    }
                    eq = eq < f - p ? eq : f - p;
                    for (int q = 1; q < eq; ++q) v[u] += s_prod[S::at(p + q)];
                }
            }
        }
        int pos0 = uniform(before);
#pragma unroll
        for (int u = 0; u < VT; ++u) {
            const int pos = pos0 + __popcll(heads[u] & ((1ull << ln) - 1ull));
            if (((heads[u] >> ln) & 1ull) && pos < seg) {
                // streaming stores: C is written once (3% of the tier's time on the same graph)
                __builtin_nontemporal_store(I::key(x[u]), &c_col[cb + pos]);
                __builtin_nontemporal_store(static_cast<V>(v[u]), &c_val[cb + pos]);
            }
            pos0 += __popcll(heads[u]);
        }
    } else {
        __syncthreads();
        total = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) total += L.scratch[i];
        total = uniform(total);
    }
    return total;
}

template <int CAP, typename V, bool NUM>
__global__ void __launch_bounds__((MergeShape<CAP, NUM>::BLOCK), (MergeShape<CAP, NUM>::WAVES)) merge_kernel(
    Mats<V> M, const int32_t *__restrict__ rows, int32_t *__restrict__ row_nnz, RowSink out,
    int32_t *__restrict__ c_col, V *__restrict__ c_val, Control *ctrl) {
    __shared__ MergeLds<CAP, NUM> L;
    __shared__ int64_t s_claim[2];   // pool output: the row's first entry and writable length
    const int ln = lane_id();
    const int row = rows[blockIdx.x];
    const int a_lo = M.a_rp[row], k = M.a_rp[row + 1] - a_lo;
    // lane l: run l, the selected row of B and A's value
    int bs = 0, len = 0;
    double av = 0.0;
    if (ln < k) {
        const int32_t j = M.a_col[a_lo + ln];
        if (NUM) av = to_d(M.a_val[a_lo + ln]);
        bs = M.b_rp[j];
        len = M.b_rp[j + 1] - bs;
    }
    // the row's place: from C.row_ptr, or claimed from the pool by its entry count
    auto place = [&](int total) __attribute__((always_inline)) {
        longlong2 at;
        if (!out.pooled()) {
            at.x = out.c_rp[row];
            at.y = out.c_rp[row + 1] - at.x;
            if (threadIdx.x == 0 && total != at.y) atomicOr(&ctrl->error_flags, kErrRowMismatch);
        } else {
            if (threadIdx.x == 0) s_claim[0] = out.claim(row, total, &s_claim[1]);
            __syncthreads();
            at.x = uniform(s_claim[0]);
            at.y = uniform(s_claim[1]);
        }
        return at;
    };
    const int total = merge_runs<CAP, NUM, V>(M, L, bs, len, av, place, c_col, c_val);
    if (!NUM && threadIdx.x == 0) row_nnz[row] = total;
}

// Longer rows of at most kMergeMaxRuns A entries, CSR output only: merged piece
// by piece, a piece being a range of columns whose part of the row fits the
// places in LDS. The window table gives the row's products before every window
// boundary, and a piece takes as many whole windows as fit; a window that does
// not fit alone is cut at a column found by halving (a column holds at most one
// product per run).
//
// For C of several regions of the rank kernel, where such a row pays the rank
// kernel's fixed work (about 20 K cycles) per region for a few thousand
// entries. Measured on an R-MAT graph of 2.5 M vertices (10 regions; 19.6 K rows
// of 8 K to 20 K products, float): 6.2 ms in the rank kernel, 3.7 ms here; on 1 M
// vertices (4 regions, double) 3.3 ms against 9.5 ms, so there they stay.
constexpr int kMergeLongCap = 1 << kMergeLog2Max;
template <typename V>
__global__ void __launch_bounds__((MergeShape<kMergeLongCap, true>::BLOCK), (MergeShape<kMergeLongCap, true>::WAVES))
merge_long_kernel(Mats<V> M, const int32_t *__restrict__ rows, const int32_t *__restrict__ wtab, int nwin, int wcols,
                  RowSink out, int32_t *__restrict__ c_col, V *__restrict__ c_val, Control *ctrl) {
    constexpr int CAP = kMergeLongCap;
    constexpr int BLOCK = MergeShape<CAP, true>::BLOCK;
    constexpr int VT = MergeShape<CAP, true>::VT;
    constexpr int NW = BLOCK / kWave;
    __shared__ MergeLds<CAP, true> L;
    __shared__ int32_t s_before[2 * kWave + 1];   // the row's products before window w
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int ln = lane_id();
    const int row = rows[blockIdx.x];
    const int a_lo = M.a_rp[row], k = M.a_rp[row + 1] - a_lo;
    // lane l: run l, from entry `cur` of B on, to `stop`
    int cur = 0, stop = 0, j = 0;
    double av = 0.0;
    if (ln < k) {
        j = M.a_col[a_lo + ln];
        av = to_d(M.a_val[a_lo + ln]);
        cur = M.b_rp[j];
        stop = M.b_rp[j + 1];
    }
    const int64_t trow = static_cast<int64_t>(j) * (nwin + 1);
    for (int w = threadIdx.x; w <= nwin; w += BLOCK) s_before[w] = 0;
    __syncthreads();
    for (int r = wv; r < k; r += NW) {
        const int32_t *t = wtab + static_cast<int64_t>(__builtin_amdgcn_readlane(j, r)) * (nwin + 1);
        const int first = __builtin_amdgcn_readlane(cur, r);
        for (int w = ln; w <= nwin; w += kWave) {
            const int n = t[w] - first;
            if (n > 0) atomicAdd(&s_before[w], n);
        }
    }
    __syncthreads();
    const int b0 = ln <= nwin ? s_before[ln] : 0x7fffffff;
    const int b1 = ln + kWave <= nwin ? s_before[ln + kWave] : 0x7fffffff;
    const int b2 = nwin == 2 * kWave ? s_before[nwin] : 0x7fffffff;
    const int f = uniform(s_before[nwin]);
    const int room = CAP - (VT - 1) * k;   // products that fit, every run's end padded
    const int64_t cb = out.c_rp[row];
    const int64_t seg = out.c_rp[row + 1] - cb;
    int taken = 0;        // products of the pieces so far
    int64_t done = 0;     // their entries of C
    int64_t col = 0;      // the next piece's first column
    while (taken < f) {
        // the last window boundary the piece reaches
        const int most = taken + room;
        const int w1 = __popcll(ballot(b0 <= most)) + __popcll(ballot(b1 <= most)) + (b2 <= most ? 1 : 0) - 1;
        const int before1 = w1 < kWave ? __builtin_amdgcn_readlane(b0, w1)
                                       : (w1 < 2 * kWave ? __builtin_amdgcn_readlane(b1, w1 - kWave) : b2);
        int end = cur;
        if (before1 > taken) {
            if (ln < k) end = w1 == nwin ? stop : wtab[trow + w1];
            col = static_cast<int64_t>(w1) * wcols;
        } else {
            int64_t lo = static_cast<int64_t>(w1) * wcols, hi = lo + wcols;
            lo = lo > col ? lo : col;
            const int lim = ln < k ? wtab[trow + w1 + 1] : cur;
            while (hi - lo > 1) {
                const int64_t x = lo + (hi - lo) / 2;
                int p = cur, q = lim;
                while (p < q) {
                    const int m = p + ((q - p) >> 1);
                    if (M.b_col[m] < x) p = m + 1;
                    else q = m;
                }
                const int n = uniform(wave_sum(p - cur));
                end = p;
                col = x;
                if (n > 0 && n <= room) break;
                if (n > 0) hi = x;
                else lo = x;
            }
        }
        const int len = end > cur ? end - cur : 0;
        const int n = uniform(wave_sum(len));
        if (n <= 0 || n > room) {
            // only where B's rows are not sorted
            if (threadIdx.x == 0) atomicOr(&ctrl->error_flags, kErrRowMismatch);
            break;
        }
        auto place = [&](int) __attribute__((always_inline)) {
            longlong2 at;
            at.x = cb + done;
            at.y = seg - done;
            return at;
        };
        done += merge_runs<CAP, true, V>(M, L, cur, len, av, place, c_col, c_val);
        taken += n;
        cur = end > cur ? end : cur;
        __syncthreads();   // L is used again
    }
    if (threadIdx.x == 0 && done != seg) atomicOr(&ctrl->error_flags, kErrRowMismatch);
}

}  // namespace wsp
