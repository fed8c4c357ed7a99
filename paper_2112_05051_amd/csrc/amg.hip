// Aggregation AMG (Section 5.2): parallel pairwise matching, piecewise-
// constant Galerkin products, l1 smoother data, the CSR pieces of the
// V-cycle and the dense coarsest-level solve.
#include "common.hpp"

#include <algorithm>
#include <cstring>

namespace rich {

namespace {

constexpr int TPB = 256;

inline unsigned nblocks(int64_t n, int tpb = TPB) { return (unsigned)((n + tpb - 1) / tpb); }

// --------------------------------------------------------------- matching
// Edge {i,j} (i != j) carries the value a_{lo,hi} of row lo = min(i,j) and
// weight w = 1 - 2 a_{lo,hi} / (a_lolo + a_hihi); edges with a zero value or
// a non-finite weight do not exist.  The strict order is (w desc, lo asc,
// hi asc).  A vertex matches its best free neighbour when that neighbour's
// best free neighbour is the vertex itself (locally dominant edge): repeated
// until no free vertex has a free neighbour, this gives exactly the greedy
// matching that scans all edges in the strict order.

__device__ inline double find_entry(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                    const double *__restrict__ val, int64_t row, int32_t c, bool *found) {
    int64_t lo = rowptr[row], hi = rowptr[row + 1] - 1;
    while (lo <= hi) {
        int64_t mid = (lo + hi) >> 1;
        int32_t cm = col[mid];
        if (cm == c) {
            *found = true;
            return val[mid];
        }
        if (cm < c) lo = mid + 1;
        else hi = mid - 1;
    }
    *found = false;
    return 0.0;
}

// Eight lanes per row: a thread walking its row alone waits for one dependent
// load after another (the weights of a set-up's 18 sweeps at 256^3 10.3 ms, now
// 4.4).  A launch holds fewer than 2^32 threads, so it takes the rows from r0 on,
// at most ROW_SLICE of them.
constexpr int ROW_LANES = 8;
constexpr int64_t ROW_SLICE = (int64_t)1 << 28;
__global__ void k_diag(int64_t r0, int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                       const double *__restrict__ val, double *__restrict__ diag) {
    const int64_t i = r0 + ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / ROW_LANES;
    const int lane = threadIdx.x % ROW_LANES;
    double d = 0.0;
    if (i < n)
        for (int64_t e = rowptr[i] + lane; e < rowptr[i + 1]; e += ROW_LANES)
            if (col[e] == i) d = val[e];
    d = group_sum<ROW_LANES>(d);  // the other lanes hold zeros
    if (i < n && lane == 0) diag[i] = d;
}

// The edge weights of a sweep, once: w[e] = 1 - 2 a_lo,hi / (d_lo + d_hi) for
// the entry e = (i, j), the coupling a read in the lower-numbered row; NaN
// where the entry can never be a candidate (the diagonal, a coupling missing
// from the lower row, a zero coupling).  k_candidates skips every entry
// whose weight is not finite.
__global__ void k_match_weights(int64_t r0, int64_t n, const int64_t *__restrict__ rowptr,
                                const int32_t *__restrict__ col, const double *__restrict__ val,
                                const double *__restrict__ diag, double *__restrict__ w) {
    const int64_t i = r0 + ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / ROW_LANES;
    if (i >= n) return;
    for (int64_t e = rowptr[i] + threadIdx.x % ROW_LANES; e < rowptr[i + 1]; e += ROW_LANES) {
        int32_t j = col[e];
        double we = __builtin_nan("");
        if (j != i) {
            int64_t lo = j < i ? j : i, hi = j < i ? i : j;
            bool found = true;
            double a = lo == i ? val[e] : find_entry(rowptr, col, val, lo, (int32_t)hi, &found);
            if (found && a != 0.0) we = 1.0 - (2.0 * a) / (diag[lo] + diag[hi]);
        }
        w[e] = we;
    }
}

// One matching round: every free row proposes its free neighbour of largest
// weight (ties to the smaller (lo, hi) pair); -1 when there is none.  Rows that
// are no longer free leave their cand as it was: k_commit reads it only for free
// rows.  Four entries' loads are in flight at a time (a set-up's 388 rounds at
// 256^3 18.5 ms, now 10.1).
__global__ void k_candidates(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                             const double *__restrict__ w, const int32_t *__restrict__ mate,
                             int32_t *__restrict__ cand) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || mate[i] != -1) return;
    int32_t best = -1;
    double bw = 0.0;
    int64_t blo = 0, bhi = 0;
    const int64_t e1 = rowptr[i + 1];
    for (int64_t e0 = rowptr[i]; e0 < e1; e0 += 4) {
        int32_t js[4], ms[4];
        double ws[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int64_t e = e0 + u < e1 ? e0 + u : e1 - 1;
            js[u] = col[e];
            ws[u] = w[e];
        }
#pragma unroll
        for (int u = 0; u < 4; u++) ms[u] = mate[js[u]];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int32_t j = js[u];
            const double we = ws[u];
            if (e0 + u >= e1 || j == i || ms[u] != -1 || !isfinite(we)) continue;
            int64_t lo = j < i ? j : i, hi = j < i ? i : j;
            bool better = best < 0 || we > bw || (we == bw && (lo < blo || (lo == blo && hi < bhi)));
            if (better) {
                best = j;
                bw = we;
                blo = lo;
                bhi = hi;
            }
        }
    }
    cand[i] = best;
}

__global__ void k_commit(int64_t n, const int32_t *__restrict__ cand, int32_t *__restrict__ mate,
                         int *__restrict__ still_free) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (mate[i] != -1) return;
    int32_t c = cand[i];
    if (c < 0) {
        mate[i] = -2;  // no free neighbour left: a singleton for good
    } else if (cand[c] == (int32_t)i) {
        mate[i] = c;
    } else {
        *still_free = 1;
    }
}

__global__ void k_leaders(int64_t n, const int32_t *__restrict__ mate, int64_t *__restrict__ flag) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t m = mate[i];
    flag[i] = (m < 0 || i < m) ? 1 : 0;
}

__global__ void k_number(int64_t n, const int32_t *__restrict__ mate, const int64_t *__restrict__ id,
                         int32_t *__restrict__ agg) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t m = mate[i];
    agg[i] = (int32_t)((m < 0 || i < m) ? id[i] : id[m]);
}

// ------------------------------------- decoupled greedy (VMB) aggregation
// DSVMB coarsening (Section 5.2): each block of `block` consecutive rows (a
// "process") aggregates its own rows, ignoring couplings that leave the block,
// so the blocks are independent: one thread per block runs the three greedy
// phases over its rows in index order.  j is strongly coupled to i when
// |a_ij| >= theta sqrt(|a_ii a_jj|).  Phase 1: a free row whose strong
// neighbours are all free starts an aggregate with them; phase 2: a free row
// joins the phase-1 aggregate of its strongest strong neighbour aggregated in
// phase 1 (first in column order on ties); phase 3: a free row starts an
// aggregate with its free strong neighbours.  Ids are block-local here and
// offset by the aggregates of the earlier blocks afterwards.
__global__ void k_row_diag(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                           const double *__restrict__ val, double *__restrict__ diag) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double d = 0.0;
    for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++)
        if (col[e] == i) d = val[e];
    diag[i] = d;
}

__global__ void k_vmb_block(int64_t n, int64_t block, int64_t nblk, const int64_t *__restrict__ rowptr,
                            const int32_t *__restrict__ col, const double *__restrict__ val,
                            const double *__restrict__ diag, double theta, int32_t *__restrict__ agg,
                            int32_t *__restrict__ p1, int64_t *__restrict__ count) {
#pragma clang fp contract(off)
    int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nblk) return;
    const int64_t b0 = b * block, b1 = b0 + block < n ? b0 + block : n;
    auto strong = [&](int64_t i, int64_t e) {
        int64_t j = col[e];
        return j != i && j >= b0 && j < b1 && fabs(val[e]) >= theta * sqrt(fabs(diag[i] * diag[j]));
    };
    int32_t nc = 0;
    for (int64_t i = b0; i < b1; i++) agg[i] = -1;
    for (int64_t i = b0; i < b1; i++) {  // phase 1
        bool ok = agg[i] < 0;
        for (int64_t e = rowptr[i]; ok && e < rowptr[i + 1]; e++)
            if (strong(i, e) && agg[col[e]] >= 0) ok = false;
        if (!ok) continue;
        agg[i] = nc;
        for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++)
            if (strong(i, e)) agg[col[e]] = nc;
        nc++;
    }
    for (int64_t i = b0; i < b1; i++) p1[i] = agg[i];
    for (int64_t i = b0; i < b1; i++) {  // phase 2
        if (agg[i] >= 0) continue;
        double best = -1.0;
        for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++) {
            if (!strong(i, e) || p1[col[e]] < 0) continue;
            double sv = fabs(val[e]) / sqrt(fabs(diag[i] * diag[col[e]]));
            if (sv > best) {
                best = sv;
                agg[i] = p1[col[e]];
            }
        }
    }
    for (int64_t i = b0; i < b1; i++) {  // phase 3
        if (agg[i] >= 0) continue;
        agg[i] = nc;
        for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++)
            if (strong(i, e) && agg[col[e]] < 0) agg[col[e]] = nc;
        nc++;
    }
    count[b] = nc;
}

__global__ void k_vmb_offset(int64_t n, int64_t block, const int64_t *__restrict__ off, int32_t *__restrict__ agg) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    agg[i] += (int32_t)off[i / block];
}

// ---------------------------------------------------------------- Galerkin
__global__ void k_count_members(int64_t n, const int32_t *__restrict__ agg, int64_t *__restrict__ cnt) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    atomicAdd((unsigned long long *)&cnt[agg[i]], 1ull);
}

__global__ void k_place_members(int64_t n, const int32_t *__restrict__ agg, const int64_t *__restrict__ mptr,
                                unsigned int *__restrict__ cursor, int32_t *__restrict__ mem) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t I = agg[i];
    unsigned int pos = atomicAdd(&cursor[I], 1u);
    mem[mptr[I] + pos] = (int32_t)i;
}

// Members were placed in arbitrary order; sort each (small) list ascending.
__global__ void k_sort_members(int64_t nc, const int64_t *__restrict__ mptr, int32_t *__restrict__ mem) {
    int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    int64_t a = mptr[I], b = mptr[I + 1];
    for (int64_t t = a + 1; t < b; t++) {
        int32_t v = mem[t];
        int64_t u = t - 1;
        while (u >= a && mem[u] > v) {
            mem[u + 1] = mem[u];
            u--;
        }
        mem[u + 1] = v;
    }
}

// Symbolic product: the coarse columns J = agg[j] reached from the member
// rows of coarse row I, sorted and unique.  Each coarse row owns a scratch
// segment as long as the sum of its members' row lengths (an upper bound).
__global__ void k_seg_len(int64_t nc, const int64_t *__restrict__ mptr, const int32_t *__restrict__ mem,
                          const int64_t *__restrict__ rowptr, int64_t *__restrict__ seg) {
    int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    int64_t s = 0;
    for (int64_t t = mptr[I]; t < mptr[I + 1]; t++) s += rowptr[mem[t] + 1] - rowptr[mem[t]];
    seg[I] = s;
}

// One thread per coarse row; up to SYM_REG columns are held in LDS (column-major
// over the block's threads, as in k_gal_numeric), longer lists in the segment.
// (Inserting in the segment itself: 23 products of a set-up at 256^3 20.8 ms,
// now 5.0.)
// f(e, i, j, J): entry e = (i, j) of a member row and its coarse column J, in
// order; the loads of four entries are in flight at a time.
template <class F>
__device__ __forceinline__ void member_entries(int64_t m0, int64_t m1, const int32_t *__restrict__ mem,
                                               const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                               const int32_t *__restrict__ agg, F &&f) {
    for (int64_t t = m0; t < m1; t++) {
        const int32_t i = mem[t];
        const int64_t e1 = rowptr[i + 1];
        for (int64_t e0 = rowptr[i]; e0 < e1; e0 += 4) {
            int32_t j[4], J[4];
#pragma unroll
            for (int u = 0; u < 4; u++) j[u] = col[e0 + u < e1 ? e0 + u : e1 - 1];
#pragma unroll
            for (int u = 0; u < 4; u++) J[u] = agg[j[u]];
            f(e0, e1, i, j, J);
        }
    }
}
constexpr int SYM_REG = 32;
__global__ void __launch_bounds__(64) k_sym_collect(int64_t nc, const int64_t *__restrict__ mptr,
                                                    const int32_t *__restrict__ mem, const int64_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ col, const int32_t *__restrict__ agg,
                                                    const int64_t *__restrict__ segptr, int32_t *__restrict__ scratch,
                                                    int64_t *__restrict__ cnt) {
    __shared__ int32_t s_[SYM_REG * 64];
    const int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    int32_t *buf = scratch + segptr[I], *reg = s_ + threadIdx.x;
    int64_t len = 0;
    bool spilled = false;
    // insert J into the sorted unique prefix of a list with stride k
    auto insert = [&](int32_t *b, int k, int32_t J) {
        int64_t lo = 0, hi = len;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (b[mid * k] < J) lo = mid + 1;
            else hi = mid;
        }
        if (lo < len && b[lo * k] == J) return true;
        if (b == reg && len == SYM_REG) return false;
        for (int64_t v = len; v > lo; v--) b[v * k] = b[(v - 1) * k];
        b[lo * k] = J;
        len++;
        return true;
    };
    member_entries(mptr[I], mptr[I + 1], mem, rowptr, col, agg,
                   [&](int64_t e0, int64_t e1, int32_t, const int32_t *, const int32_t *J) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (e0 + u >= e1) continue;
            if (!spilled && insert(reg, 64, J[u])) continue;
            if (!spilled) {
                for (int v = 0; v < SYM_REG; v++) buf[v] = reg[v * 64];
                spilled = true;
            }
            insert(buf, 1, J[u]);
        }
    });
    if (!spilled)
        for (int64_t v = 0; v < len; v++) buf[v] = reg[v * 64];
    cnt[I] = len;
}

__global__ void k_sym_write(int64_t nc, const int64_t *__restrict__ segptr, const int32_t *__restrict__ scratch,
                            const int64_t *__restrict__ crow, int32_t *__restrict__ ccol) {
    int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    const int32_t *buf = scratch + segptr[I];
    int64_t o = crow[I], n = crow[I + 1] - o;
    for (int64_t a = 0; a < n; a++) ccol[o + a] = buf[a];
}

// Numeric product on a fixed pattern: members ascending, each fine row in
// column order, every term added to its coarse entry in that order (the
// oracle's order), starting from zero.  One thread per coarse row; rows of up
// to GAL_REG entries accumulate in LDS (column-major over the block's 64
// threads, so dynamic indexing never spills to scratch memory), longer rows
// directly in the output.
constexpr int GAL_REG = 32;
__global__ void __launch_bounds__(64) k_gal_numeric(int64_t nc, const int64_t *__restrict__ mptr,
                                                    const int32_t *__restrict__ mem, const int64_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ col, const double *__restrict__ val,
                                                    const int32_t *__restrict__ agg, const int64_t *__restrict__ crow,
                                                    const int32_t *__restrict__ ccol, double *__restrict__ cval) {
    __shared__ double acc_s[GAL_REG * 64];
    __shared__ int32_t cj_s[GAL_REG * 64];
    int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    const int t = threadIdx.x;
    int64_t a = crow[I], b = crow[I + 1];
    int len = (int)(b - a);
    if (len <= GAL_REG) {
        for (int e = 0; e < len; e++) {
            cj_s[e * 64 + t] = ccol[a + e];
            acc_s[e * 64 + t] = 0.0;
        }
        member_entries(mptr[I], mptr[I + 1], mem, rowptr, col, agg,
                       [&](int64_t e0, int64_t e1, int32_t, const int32_t *, const int32_t *J) {
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) v[u] = val[e0 + u < e1 ? e0 + u : e1 - 1];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (e0 + u >= e1) continue;
                int lo = 0, hi = len - 1;
                while (lo < hi) {
                    int mid = (lo + hi) >> 1;
                    if (cj_s[mid * 64 + t] < J[u]) lo = mid + 1;
                    else hi = mid;
                }
                acc_s[lo * 64 + t] += v[u];
            }
        });
        for (int e = 0; e < len; e++) cval[a + e] = acc_s[e * 64 + t];
        return;
    }
    for (int64_t e = a; e < b; e++) cval[e] = 0.0;
    for (int64_t q = mptr[I]; q < mptr[I + 1]; q++) {
        int32_t i = mem[q];
        for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++) {
            int32_t J = agg[col[e]];
            int64_t lo = a, hi = b - 1;
            while (lo < hi) {
                int64_t mid = (lo + hi) >> 1;
                if (ccol[mid] < J) lo = mid + 1;
                else hi = mid;
            }
            cval[lo] += val[e];
        }
    }
}

// The numeric product again and again on a fixed pattern (the refreshes): the
// fine values that make up each coarse entry are listed once at set-up, in the
// order of k_gal_numeric, so a refresh is one gather-sum per coarse entry: no
// search, no LDS accumulators (which held k_gal_numeric at six waves a CU), and
// level 0 reads the stencil arrays themselves instead of a CSR copy of them.
// Bound by the list and value reads (12 bytes per fine entry).  A refresh at
// 256^3, five levels: 0.7 ms, against 4.0 with k_gal_numeric and 1.2 for the
// CSR copy of M.
// FILL = false counts the sources of each entry, FILL = true lists them; one
// thread per coarse row, rows of up to GAL_REG entries count in LDS.
struct StencilIndex {  // value index of CSR entry (i, j): e itself, or its place in the M arrays
    int nx, ny, nz;    // nx = 0: CSR
    __device__ uint32_t operator()(int64_t n, int64_t i, int64_t j, int64_t e) const {
        if (nx == 0) return (uint32_t)e;
        if (i == j) return (uint32_t)(M_D * n + i);
        const int64_t lo = i < j ? i : j, d = i < j ? j - i : i - j;
        // an axis of one cell has no coupling; the others differ in their stride
        const int t = nx > 1 && d == 1 ? M_XP : ny > 1 && d == nx ? M_YP : M_ZP;
        return (uint32_t)(t * n + lo);
    }
};
template <bool FILL>
__global__ void __launch_bounds__(64) k_gal_sources(int64_t nc, int64_t n, StencilIndex ix,
                                                    const int64_t *__restrict__ mptr, const int32_t *__restrict__ mem,
                                                    const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                    const int32_t *__restrict__ agg, const int64_t *__restrict__ crow,
                                                    const int32_t *__restrict__ ccol, int64_t *__restrict__ cnt,
                                                    const uint32_t *__restrict__ gptr, uint32_t *__restrict__ gsrc) {
    __shared__ uint32_t cur_s[GAL_REG * 64];
    __shared__ int32_t cj_s[GAL_REG * 64];
    const int64_t I = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    const int t = threadIdx.x;
    const int64_t a = crow[I], b = crow[I + 1];
    const int64_t len = b - a;
    if (len > GAL_REG) {  // counts (and, filling, the next free places) in memory
        for (int64_t q = a; q < b; q++) cnt[q] = 0;
        for (int64_t m = mptr[I]; m < mptr[I + 1]; m++) {
            const int64_t i = mem[m];
            for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++) {
                const int32_t J = agg[col[e]];
                int64_t lo = a, hi = b - 1;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (ccol[mid] < J) lo = mid + 1;
                    else hi = mid;
                }
                if (FILL) gsrc[gptr[lo] + cnt[lo]] = ix(n, i, col[e], e);
                cnt[lo]++;
            }
        }
        return;
    }
    for (int q = 0; q < len; q++) {
        cj_s[q * 64 + t] = ccol[a + q];
        cur_s[q * 64 + t] = FILL ? gptr[a + q] : 0u;
    }
    member_entries(mptr[I], mptr[I + 1], mem, rowptr, col, agg,
                   [&](int64_t e0, int64_t e1, int32_t i, const int32_t *j, const int32_t *J) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (e0 + u >= e1) continue;
            int lo = 0, hi = (int)len - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cj_s[mid * 64 + t] < J[u]) lo = mid + 1;
                else hi = mid;
            }
            const uint32_t at = cur_s[lo * 64 + t]++;
            if (FILL) gsrc[at] = ix(n, i, j[u], e0 + u);
        }
    });
    if (!FILL)
        for (int q = 0; q < len; q++) cnt[a + q] = cur_s[q * 64 + t];
}

__global__ void k_narrow_u32(int64_t n, const int64_t *__restrict__ in, uint32_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (uint32_t)in[i];
}

// COPY: what else the value goes to: GS_F32 an FP32 copy; at the entry's place
// in aggregate order GS_ENT the FP32 cycle's pair, GS_VALF / GS_VAL its FP32 /
// FP64 value.
enum { GS_NONE = 0, GS_F32, GS_ENT, GS_VALF, GS_VAL };
// A block's entries have one contiguous stretch of sources: its threads gather
// them into LDS with coalesced list reads, all in flight at once, and each
// thread adds its entry's from there.  (A thread walking its own list waits
// for two dependent loads per four sources, and a wave for its longest list, a
// diagonal's of about 26: 1200 us for the five levels at 256^3, now 690.)
template <int COPY>
__global__ void __launch_bounds__(GS_TPB) k_gal_sum(int64_t cnnz, const uint32_t *__restrict__ gptr,
                                                    const uint32_t *__restrict__ gsrc, const double *__restrict__ val,
                                                    double *__restrict__ cval, float *__restrict__ cvalf,
                                                    const int32_t *__restrict__ place, const uint32_t *__restrict__ off,
                                                    int2 *__restrict__ ent, double *__restrict__ vval) {
    __shared__ double sv[GS_PIECE];
    const int64_t q0 = (int64_t)xcd_block() * GS_TPB, q = q0 + threadIdx.x;
    if (q0 >= cnnz) return;
    const uint32_t t0 = gptr[q0], t1 = gptr[q0 + GS_TPB < cnnz ? q0 + GS_TPB : cnnz];
    uint32_t a = t1, b = t1, of = 0;
    int32_t pl = 0;
    if (q < cnnz) {
        a = gptr[q];
        b = gptr[q + 1];
        if (COPY >= GS_ENT) pl = place[q];
        if (COPY == GS_ENT) of = off[q];
    }
    double s = 0.0;
    for (uint32_t base = t0; base < t1; base += GS_PIECE) {
        uint32_t ix[GS_PER];
        double v[GS_PER];
#pragma unroll
        for (int u = 0; u < GS_PER; u++) {
            const uint32_t t = base + threadIdx.x + GS_TPB * u;
            ix[u] = t < t1 ? __builtin_nontemporal_load(gsrc + t) : 0u;
        }
#pragma unroll
        for (int u = 0; u < GS_PER; u++) v[u] = val[ix[u]];
        if (base != t0) __syncthreads();  // the previous piece is summed
#pragma unroll
        for (int u = 0; u < GS_PER; u++) sv[threadIdx.x + GS_TPB * u] = v[u];
        __syncthreads();
        const uint32_t lo = a > base ? a - base : 0u;
        const uint32_t hi = b <= base ? 0u : b - base < GS_PIECE ? b - base : GS_PIECE;
        for (uint32_t t = lo; t < hi; t++) s += sv[t];
    }
    if (q >= cnnz) return;
    cval[q] = s;
    if (COPY == GS_F32) cvalf[q] = f32_sat(s);
    if (COPY == GS_ENT) ent[pl] = make_int2((int)of, __float_as_int(f32_sat(s)));
    if (COPY == GS_VALF) cvalf[pl] = f32_sat(s);
    if (COPY == GS_VAL) vval[pl] = s;
}

// l1 inverse diagonals 1 / sum_j |a_ij|, each row's terms added in order: a
// block's rows have one stretch of values, staged in LDS as above (a thread
// walking its own row strides across the others': five levels at 256^3 250 us,
// now 95).
// pos: place of each row in the results (null: itself).
constexpr int L1_PIECE = 2048;
__global__ void __launch_bounds__(256) k_row_l1(int64_t n, const int64_t *__restrict__ rowptr,
                                                const double *__restrict__ val, const int32_t *__restrict__ pos,
                                                double *__restrict__ invd, float *__restrict__ invdf) {
    __shared__ double sv[L1_PIECE];
    const int64_t r0 = (int64_t)blockIdx.x * 256, i = r0 + threadIdx.x;
    const int64_t t0 = rowptr[r0], t1 = rowptr[r0 + 256 < n ? r0 + 256 : n];
    int64_t a = t1, b = t1, to = i;
    if (i < n) {
        a = rowptr[i];
        b = rowptr[i + 1];
        if (pos) to = pos[i];
    }
    double s = 0.0;
    for (int64_t base = t0; base < t1; base += L1_PIECE) {
        double v[L1_PIECE / 256];
#pragma unroll
        for (int u = 0; u < L1_PIECE / 256; u++) {
            const int64_t t = base + threadIdx.x + 256 * u;
            v[u] = t < t1 ? val[t] : 0.0;
        }
        if (base != t0) __syncthreads();
#pragma unroll
        for (int u = 0; u < L1_PIECE / 256; u++) sv[threadIdx.x + 256 * u] = v[u];
        __syncthreads();
        const int lo = a > base ? (int)(a - base < L1_PIECE ? a - base : L1_PIECE) : 0;
        const int hi = b <= base ? 0 : b - base < L1_PIECE ? (int)(b - base) : L1_PIECE;
        for (int t = lo; t < hi; t++) s += fabs(sv[t]);
    }
    if (i >= n) return;
    if (invd) invd[to] = 1.0 / s;
    if (invdf) invdf[to] = f32_sat(1.0 / s);
}

__global__ void k_compose(int64_t n, int32_t *__restrict__ comp, const int32_t *__restrict__ a) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) comp[i] = a[comp[i]];
}

__global__ void k_iota(int64_t n, int32_t *__restrict__ x) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = (int32_t)i;
}

// ----------------------------------------------------- V-cycle, CSR levels
// Rows are processed by groups of G lanes (4 or 8, by the level's mean row
// length) that stride over the row's entries; the group sum is formed with
// shuffles in a fixed lane order.

// pre-smoothing from zero and residual: x0 = D^{-1} b (stored by the
// restriction that produced b), r = b - A x0
template <int G, class TB, class T>
__global__ void k_csr_pre(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                          const T *__restrict__ val, const T *__restrict__ x0, const TB *__restrict__ b,
                          T *__restrict__ r) {
    int64_t row = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) / G;
    int lane = threadIdx.x % G;
    if (row >= n) return;
    T s = 0;
    for (int64_t e = rowptr[row] + lane; e < rowptr[row + 1]; e += G) s += val[e] * x0[col[e]];
    s = group_sum<G>(s);
    if (lane == 0) r[row] = (T)b[row] - s;
}

// prolongation: xt = x0 + P xc
template <class T>
__device__ __forceinline__ void csr_prolong_at(int64_t n, const T *__restrict__ x0, const T *__restrict__ xc,
                                               const int32_t *__restrict__ agg, T *__restrict__ xt, int64_t row) {
    if (row < n) xt[row] = x0[row] + xc[agg[row]];
}
template <class T>
__global__ void k_csr_prolong(int64_t n, const T *__restrict__ x0, const T *__restrict__ xc,
                              const int32_t *__restrict__ agg, T *__restrict__ xt) {
    csr_prolong_at(n, x0, xc, agg, xt, (int64_t)xcd_block() * blockDim.x + threadIdx.x);
}

// post-smoothing: x = xt + D^{-1}(b - A xt)
template <int G, class TB, class T>
__global__ void k_csr_post(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                           const T *__restrict__ val, const T *__restrict__ invd, const TB *__restrict__ b,
                           const T *__restrict__ xt, T *__restrict__ x) {
    int64_t row = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) / G;
    int lane = threadIdx.x % G;
    if (row >= n) return;
    T s = 0;
    for (int64_t e = rowptr[row] + lane; e < rowptr[row + 1]; e += G) s += val[e] * xt[col[e]];
    s = group_sum<G>(s);
    if (lane == 0) x[row] = xt[row] + invd[row] * ((T)b[row] - s);
}

template <int G, class TB, class T>
__global__ void k_csr_sweep(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                            const T *__restrict__ val, const T *__restrict__ invd, const TB *__restrict__ b,
                            const T *__restrict__ xin, T *__restrict__ xout, int zero) {
    int64_t row = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) / G;
    int lane = threadIdx.x % G;
    if (row >= n) return;
    if (zero) {
        if (lane == 0) xout[row] = (T)b[row] * invd[row];
        return;
    }
    T s = 0;
    for (int64_t e = rowptr[row] + lane; e < rowptr[row + 1]; e += G) s += val[e] * xin[col[e]];
    s = group_sum<G>(s);
    if (lane == 0) xout[row] = xin[row] + invd[row] * ((T)b[row] - s);
}

// ------------------------------------------------ CSR-stream levels
// (hierarchies that do not run in aggregate order: smoothed prolongators, or
// aggregates too large for those kernels)
// A block takes a run of whole rows holding at most STREAM_CHUNK +
// STREAM_MAXROW - 1 entries: its threads first form the products of all the
// run's entries in entry order (coalesced loads, neighbouring gathers) into
// LDS, then one thread per row adds its row's products in order.
constexpr int STREAM_LDS = STREAM_CHUNK + STREAM_MAXROW;
// PRE: v = x0, out = b - A x0;  POST: v = xt, out = xt + D^{-1}(b - A xt).
// G lanes add up a row.
template <int G, class TB, class T, bool POST>
__device__ __forceinline__ void csr_stream_body(const int64_t *__restrict__ rb, const int64_t *__restrict__ rowptr,
                                                const int32_t *__restrict__ col, const T *__restrict__ val,
                                                const T *__restrict__ invd, const TB *__restrict__ b,
                                                const T *__restrict__ v, T *__restrict__ out, int64_t blk) {
    constexpr int PER = STREAM_LDS / 256;  // entries per thread in the product phase
    __shared__ T prod[STREAM_LDS];
    // the block's first and end rows and their first entries, read together,
    // so that the entry loads below need not wait for the row pointers
    int64_t r0 = rb[2 * blk], r1 = rb[2 * blk + 2];
    if (r0 >= r1) return;
    int64_t e0 = rb[2 * blk + 1], e1 = rb[2 * blk + 3];
    // the reduction phase's first row pointers are loaded ahead of the products
    const int lane = threadIdx.x % G;
    int64_t row0 = r0 + threadIdx.x / G;
    int64_t ra = row0 < r1 ? rowptr[row0] : 0, rbe = row0 < r1 ? rowptr[row0 + 1] : 0;
    // the row's b, D^{-1} and v of the final update, loaded with its row
    // pointers so that the write after the group sum does not wait for them
    T pb = 0, pd = 0, pv = 0;
    auto row_in = [&](int64_t row) {
        if (row < r1) {
            pb = (T)b[row];
            if (POST) {
                pd = invd[row];
                pv = v[row];
            }
        }
    };
    row_in(row0);
    // every load of the product phase is issued before the first use
    int32_t cj[PER];
    T vv[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
        int64_t e = e0 + threadIdx.x + 256 * q;
        // the matrix entries are read once per sweep: streamed past the caches
        cj[q] = e < e1 ? __builtin_nontemporal_load(col + e) : 0;
        vv[q] = e < e1 ? __builtin_nontemporal_load(val + e) : (T)0;
    }
    T xs[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) xs[q] = v[cj[q]];
#pragma unroll
    for (int q = 0; q < PER; q++) {
        int64_t e = e0 + threadIdx.x + 256 * q;
        if (e < e1) prod[e - e0] = vv[q] * xs[q];
    }
    __syncthreads();
    // every lane of a group runs the same number of row iterations (shuffles)
    for (int64_t rbase = r0; rbase < r1; rbase += blockDim.x / G) {
        int64_t row = rbase + threadIdx.x / G;
        if (rbase != r0) {
            ra = row < r1 ? rowptr[row] : 0;
            rbe = row < r1 ? rowptr[row + 1] : 0;
            row_in(row);
        }
        T s = 0;
        if (row < r1)
            for (int64_t e = ra + lane; e < rbe; e += G) s += prod[e - e0];
        s = group_sum<G>(s);
        if (lane == 0 && row < r1) {
            if (POST) out[row] = pv + pd * (pb - s);
            else out[row] = pb - s;
        }
    }
}

template <int G, class TB, class T, bool POST>
__global__ void __launch_bounds__(256) k_csr_stream(const int64_t *__restrict__ rb, const int64_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ col, const T *__restrict__ val,
                                                    const T *__restrict__ invd, const TB *__restrict__ b,
                                                    const T *__restrict__ v, T *__restrict__ out) {
    csr_stream_body<G, TB, T, POST>(rb, rowptr, col, val, invd, b, v, out, xcd_block());
}

// rb[2b] = first row whose first entry is at or past b * STREAM_CHUNK and
// rb[2b + 1] = that row's first entry; the blocks past the last chunk (grid
// padding) are empty
__global__ void k_stream_rb(int64_t n, int64_t nrb, int64_t ngrid, const int64_t *__restrict__ rowptr,
                            int64_t *__restrict__ rb) {
    int64_t blk = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blk > ngrid) return;
    int64_t lo = n;
    if (blk < nrb) {
        int64_t target = blk * (int64_t)STREAM_CHUNK, hi = n;
        lo = 0;
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if (rowptr[mid] < target) lo = mid + 1;
            else hi = mid;
        }
    }
    rb[2 * blk] = lo;
    rb[2 * blk + 1] = rowptr[lo];
}

__global__ void k_max_rowlen(int64_t n, const int64_t *__restrict__ rowptr, int *__restrict__ too_long) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && rowptr[i + 1] - rowptr[i] > STREAM_MAXROW) too_long[0] = 1;
}

// bc[I] = sum over the members of I (ascending) of r
// (and x0c[I] = D_c^{-1} bc[I], the coarse pre-smoothed iterate, when x0c is set)
// A block of RESTRICT_TPB threads takes RESTRICT_TPB consecutive coarse rows:
// their member lists are one contiguous stretch of mem, which the block reads
// with coalesced loads, gathering the r values into LDS in member order; each
// thread then adds its row's values in that order (the same sums as a thread
// walking its list alone).  A stretch longer than the LDS falls back to the
// per-thread walk.  With slot (rows in aggregate order, whose members lie in
// compact boxes of cells), the members of a staged stretch are listed in
// ascending order, so that a load's lanes run along x, and slot gives each one
// its place in the stretch (256^3: 50 us; 58 in the lists' order, and 45 on
// rows in natural order, which costs the levels below two more launches each).
template <class T>
__device__ __forceinline__ void restrict_block(int64_t nc, const int64_t *__restrict__ mptr,
                                               const int32_t *__restrict__ mem, const uint16_t *__restrict__ slot,
                                               const T *__restrict__ r,
                                               T *__restrict__ bc, const T *__restrict__ invdc,
                                               T *__restrict__ x0c, int64_t blk) {
    __shared__ T rv[RESTRICT_LDS];
    const int64_t I0 = blk * RESTRICT_TPB;
    if (I0 >= nc) return;
    const int64_t I1 = I0 + RESTRICT_TPB < nc ? I0 + RESTRICT_TPB : nc;
    const int64_t I = I0 + threadIdx.x;
    const int64_t t0 = mptr[I0], t1 = mptr[I1];
    const bool staged = t1 - t0 <= RESTRICT_LDS;
    // the thread's own row bounds are loaded before the staging, which issues
    // all its member-index loads, then all its gathers (a gather waiting for
    // its index one at a time would serialise eight round trips to memory);
    // a slot past the stretch reads member t0 and is not stored
    const int64_t a = I < nc ? mptr[I] : 0, e = I < nc ? mptr[I + 1] : 0;
    const T dI = x0c && I < nc ? invdc[I] : (T)0;  // ahead of the gather
    if (staged && t1 > t0) {
        constexpr int PER = RESTRICT_LDS / RESTRICT_TPB;
        int32_t m[PER];
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int64_t t = t0 + threadIdx.x + (int64_t)q * RESTRICT_TPB;
            // the member lists are read once per cycle: streamed past the caches
            m[q] = __builtin_nontemporal_load(mem + (t < t1 ? t : t0));
        }
        int at[PER];
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int64_t t = t0 + threadIdx.x + (int64_t)q * RESTRICT_TPB;
            at[q] = slot ? __builtin_nontemporal_load(slot + (t < t1 ? t : t0)) : (int)(t - t0);
        }
        T x[PER];
#pragma unroll
        for (int q = 0; q < PER; q++) x[q] = r[m[q]];
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int64_t t = t0 + threadIdx.x + (int64_t)q * RESTRICT_TPB;
            if (t < t1) rv[at[q]] = x[q];
        }
        __syncthreads();
    }
    if (I >= nc) return;
    T s = 0;
    if (staged)
        for (int64_t t = a; t < e; t++) s += rv[t - t0];
    else
        for (int64_t t = a; t < e; t++) s += r[mem[t]];
    bc[I] = s;
    if (x0c) x0c[I] = s * dI;
}

template <class T>
__global__ void __launch_bounds__(RESTRICT_TPB) k_restrict(int64_t nc, const int64_t *__restrict__ mptr,
                                                           const int32_t *__restrict__ mem,
                                                           const uint16_t *__restrict__ slot, const T *__restrict__ r,
                                                           T *__restrict__ bc, const T *__restrict__ invdc,
                                                           T *__restrict__ x0c) {
    restrict_block(nc, mptr, mem, slot, r, bc, invdc, x0c, xcd_block());
}

// The restriction, and the sweeps of levels that are not in aggregate order, over
// several simulations at once (same per-block code as the lone launches above).
template <class T>
__global__ void __launch_bounds__(RESTRICT_TPB) k_restrict_batch(Batch<RestrictItem<T>> B) {
    for_each_block(B, xcd_block(), [&](unsigned L) {
        const int e = batch_entry(B, L);
        const RestrictItem<T> &a = B.a[e];
        restrict_block(a.nc, a.mptr, a.mem, a.slot, a.r, a.bc, a.invdc, a.x0c, (int64_t)(L - B.begin[e]));
    });
}

template <class T>
struct StreamArgs {
    const int64_t *rb, *rowptr;
    const int32_t *col;
    const T *val, *invd, *b, *v;
    T *out;
};
template <int G, class T, bool POST>
__global__ void __launch_bounds__(256) k_csr_stream_batch(Batch<StreamArgs<T>> B) {
    for_each_block(B, xcd_block(), [&](unsigned L) {
        const int e = batch_entry(B, L);
        const StreamArgs<T> &a = B.a[e];
        csr_stream_body<G, T, T, POST>(a.rb, a.rowptr, a.col, a.val, a.invd, a.b, a.v, a.out, L - B.begin[e]);
    });
}

template <class T>
struct ProlongArgs {
    int64_t n;
    const T *x0, *xc;
    const int32_t *agg;
    T *xt;
};
template <class T>
__global__ void k_csr_prolong_batch(Batch<ProlongArgs<T>> B) {
    for_each_block(B, xcd_block(), [&](unsigned L) {
        const int e = batch_entry(B, L);
        const ProlongArgs<T> &a = B.a[e];
        csr_prolong_at(a.n, a.x0, a.xc, a.agg, a.xt, (int64_t)(L - B.begin[e]) * blockDim.x + threadIdx.x);
    });
}

__global__ void k_csr_spmv(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                           const double *__restrict__ val, const double *__restrict__ x, double *__restrict__ y) {
    int64_t row = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) / 8;
    int lane = threadIdx.x % 8;
    if (row >= n) return;
    double s = 0;
    for (int64_t e = rowptr[row] + lane; e < rowptr[row + 1]; e += 8) s += val[e] * x[col[e]];
    s = group_sum<8>(s);
    if (lane == 0) y[row] = s;
}

// ----------------------------------------------- dense coarsest inverse
__global__ void k_csr_to_dense(int64_t n, const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                               const double *__restrict__ val, double *__restrict__ D) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++) D[i * n + col[e]] = val[e];
}

// Blocked Gauss-Jordan inversion of an SPD matrix (no pivoting: every
// leading block of an SPD matrix and every Schur complement stay SPD).  For
// the pivot block K = [k0, k0+64):  P = D_KK,  R_K: = P^{-1} D_K: (with P^{-1}
// itself in the K columns),  S_:K = D_:K (old), then
//   D_ij <- R_{i-k0, j}                                  for i in K,
//   D_ij <- [j not in K] D_ij - sum_t S_it R_tj          otherwise.
// Two launches a step: a panel (S and R), then the update (the rows K, and all
// other tiles on the FP64 matrix cores); the block
// of the next pivot tile inverts it right after updating it, beside the other
// tiles' updates, so a pivot's 64 scalar steps are no launch of their own.
// Bounds: the update moves 16 n^2 bytes a step (n = 3118: 156 MB, resident in
// the last-level cache) and does 64 n^2 multiply-adds; on small n the pivot's
// serial chain (32 pairs of scalar steps: LDS, barrier, two divisions; fours,
// or single steps that hand the next row over early, take the same).  Measured a
// step: n = 3118 update 44 and panel 7 us (with the pivot and the panels as
// launches of their own: 103 + 59 + 18 + 5), n = 517 23 and 6 us (19 + 54 + 16 + 5).  The order of
// operations is part of the contract: a restarted or repeated GMRES solve in
// FP64 amplifies the last bits of the preconditioner, so sweeping only half of
// the tiles (36 us, not the same bits) is not used.
constexpr int GJB = 64;  // pivot block and tile size

// P^{-1} of the 64 x 64 block in A, one workgroup of 256 threads.  Thread
// (ti, tj) keeps the entries (ti + 16 a, tj + 16 b) in registers; the 64 scalar
// Gauss-Jordan steps go in pairs that share their two rows and columns through
// double-buffered LDS, one barrier a pair: row and column k + 1 are read as they
// are before step k, and every thread takes its part of them through that
// step itself (the same operations as their owners').  rc: 8 * 64 doubles.
__device__ __forceinline__ void invert_pivot(const double (*__restrict__ A)[GJB + 1], double *__restrict__ rc,
                                             double *__restrict__ Pinv, int *__restrict__ bad) {
    const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
    double v[4][4];
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int c = 0; c < 4; c++) v[a][c] = A[ti + 16 * a][tj + 16 * c];
    bool neg = false;
    auto inverse = [&](double p) {
        if (!(p > 0.0)) {
            neg = true;
            p = 1.0;  // keep going; the caller reports the failure
        }
        return 1.0 / p;
    };
    // row and column k are cleared where they are kept: with f_k = -1/p and
    // r_k = 1 the one update of a step serves every entry
#pragma unroll
    for (int ka = 0; ka < 4; ka++)
#pragma unroll 1
        for (int kk = 0; kk < 16; kk += 2) {
            const int k = 16 * ka + kk;
            double *row0 = rc + (kk & 2) * 2 * GJB, *row1 = row0 + GJB, *col0 = row1 + GJB, *col1 = col0 + GJB;
            if (ti == kk)
#pragma unroll
                for (int c = 0; c < 4; c++) row0[tj + 16 * c] = v[ka][c];
            if (ti == kk + 1)
#pragma unroll
                for (int c = 0; c < 4; c++) row1[tj + 16 * c] = v[ka][c];
            if (tj == kk)
#pragma unroll
                for (int a = 0; a < 4; a++) {
                    col0[ti + 16 * a] = v[a][ka];
                    v[a][ka] = 0.0;
                }
            if (tj == kk + 1)
#pragma unroll
                for (int a = 0; a < 4; a++) col1[ti + 16 * a] = v[a][ka];
            if (ti == kk)
#pragma unroll
                for (int c = 0; c < 4; c++) v[ka][c] = 0.0;
            __syncthreads();
            // step k
            double r[4], f[4], r1[4], f1[4];
            const double ip0 = inverse(row0[k]), x01 = row0[k + 1], f10 = col0[k + 1] * ip0;
#pragma unroll
            for (int c = 0; c < 4; c++) {
                r[c] = c == ka && tj == kk ? 1.0 : row0[tj + 16 * c];
                r1[c] = fma(-f10, r[c], c == ka && tj == kk ? 0.0 : row1[tj + 16 * c]);
            }
#pragma unroll
            for (int a = 0; a < 4; a++) {
                f[a] = a == ka && ti == kk ? -ip0 : col0[ti + 16 * a] * ip0;
                f1[a] = fma(-f[a], x01, a == ka && ti == kk ? 0.0 : col1[ti + 16 * a]);
            }
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 4; c++) v[a][c] = fma(-f[a], r[c], v[a][c]);
            // step k + 1
            const double ip1 = inverse(fma(-f10, x01, row1[k + 1]));
            if (ti == kk + 1)
#pragma unroll
                for (int c = 0; c < 4; c++) v[ka][c] = 0.0;
            if (tj == kk + 1)
#pragma unroll
                for (int a = 0; a < 4; a++) v[a][ka] = 0.0;
            if (tj == kk + 1) r1[ka] = 1.0;
#pragma unroll
            for (int a = 0; a < 4; a++) f1[a] = a == ka && ti == kk + 1 ? -ip1 : f1[a] * ip1;
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 4; c++) v[a][c] = fma(-f1[a], r1[c], v[a][c]);
        }
    if (neg && tid == 0) *bad = 1;
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int c = 0; c < 4; c++) Pinv[(ti + 16 * a) * GJB + tj + 16 * c] = v[a][c];
}

// The first pivot block (padded to 64 x 64 with the identity: its inverse is
// then diag(P^{-1}, I)).
__global__ void __launch_bounds__(256) k_bgj_pivot(const double *__restrict__ D, int64_t n,
                                                   double *__restrict__ Pinv, int *__restrict__ bad) {
    __shared__ double A[GJB][GJB + 1], rc[8 * GJB];
    double d[16];
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const int t = threadIdx.x + 256 * q, i = t / GJB, j = t % GJB;
        d[q] = (i < n && j < n) ? D[(int64_t)i * n + j] : (i == j ? 1.0 : 0.0);
    }
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const int t = threadIdx.x + 256 * q;
        A[t / GJB][t % GJB] = d[q];
    }
    __syncthreads();
    invert_pivot(A, rc, Pinv, bad);
}

// Panel of pivot block K, four workgroups per tile T, 16 of its rows each:
// R_T = P^{-1} D_KT (terms added in ascending t) and S_T = the old D_TK.  S
// (npad x 64) and R (64 x npad) are zero past n.  R is also the new rows K of
// D, which the update writes (here the other workgroups of T still read them).
// Bound by latency: with one workgroup a tile n = 3118 10.7 us a step and
// n = 517 9.4, now 6.9 and 5.5.
__global__ void __launch_bounds__(256) k_bgj_panel(const double *__restrict__ D, int64_t n, int64_t npad, int K,
                                                   const double *__restrict__ Pinv, double *__restrict__ S,
                                                   double *__restrict__ R) {
    __shared__ double X[GJB][GJB + 1];  // D_KT [t][j]
    __shared__ double Q[GJB][17];       // rows r0.. of Pinv, transposed [t][r]
    const int T = blockIdx.x / 4, r0 = 16 * (blockIdx.x % 4), tid = threadIdx.x;
    const int64_t t0 = (int64_t)T * GJB, k0 = (int64_t)K * GJB;
    // every load is issued before the first is stored in LDS
    double pq[4], dq[16], sq[4];
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const int t = tid + 256 * q, a = t / GJB, c = t % GJB;
        dq[q] = (k0 + a < n && t0 + c < n) ? D[(k0 + a) * n + t0 + c] : 0.0;
        if (q < 4) {
            pq[q] = Pinv[(r0 + a) * GJB + c];
            sq[q] = (t0 + r0 + a < n && k0 + c < n) ? D[(t0 + r0 + a) * n + k0 + c] : 0.0;
        }
    }
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const int t = tid + 256 * q, a = t / GJB, c = t % GJB;
        X[a][c] = dq[q];
        if (q < 4) {
            Q[c][a] = pq[q];
            // in the order of the update's A operands: column t of S at 16 (t % 4) + t / 4
            S[(t0 + r0 + a) * GJB + 16 * (c & 3) + (c >> 2)] = sq[q];
        }
    }
    __syncthreads();
    const int ti = tid >> 4, tj = tid & 15;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (T == K) {
#pragma unroll
        for (int c = 0; c < 4; c++) v[c] = Q[tj + 16 * c][ti];
    } else {
#pragma unroll 8
        for (int t = 0; t < GJB; t++) {
            const double p = Q[t][ti];
#pragma unroll
            for (int c = 0; c < 4; c++) v[c] = fma(p, X[t][tj + 16 * c], v[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < 4; c++) R[(r0 + ti) * npad + t0 + tj + 16 * c] = v[c];
}

// Update: the rows K of D are R; the other tiles D_IJ <- [J != K] D_IJ - S_I R_J.
// The four wavefronts of a block each own 16 rows of the tile and accumulate
// four 16x16 blocks with v_mfma_f64_16x16x4f64 (lane l supplies A[l%16][l/16]
// and B[l/16][l%16]; result register v of lane l is D[l/16 + 4v][l%16]).
// Block 0 takes the next pivot tile (K+1, K+1) and inverts it; the others take
// the tiles in row order.
typedef double rich_d4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256, 3) k_bgj_update(double *__restrict__ D, int64_t n, int64_t npad, int K, int tiles,
                                                    const double *__restrict__ S, const double *__restrict__ R,
                                                    double *__restrict__ Pinv, int *__restrict__ bad) {
    __shared__ double Rs[GJB][GJB + 1];  // [t][col in tile]; the next pivot's tile
    __shared__ double rc[8 * GJB];
    const bool last = K == tiles - 1, piv = blockIdx.x == 0 && !last;
    int I, J;
    if (piv) {
        I = J = K + 1;
    } else {
        const int b = (int)blockIdx.x - (last ? 0 : 1);
        I = b / tiles;
        J = b - I * tiles;
        if (!last && I == K + 1 && J == K + 1) return;  // block 0's
    }
    const int64_t i0 = (int64_t)I * GJB, j0 = (int64_t)J * GJB;
    if (I == K) {
        for (int t = threadIdx.x; t < GJB * GJB; t += 256) {
            const int64_t gi = i0 + t / GJB, gj = j0 + t % GJB;
            if (gi < n && gj < n) D[gi * n + gj] = R[(t / GJB) * npad + gj];
        }
        return;
    }
    const int tid = threadIdx.x, w = tid / 64, l = tid % 64, li = l % 16, lk = l / 16;
    // a wave's rows of S go straight into its A operands; R is shared through
    // LDS (36.5 KB: four blocks would fit a CU, the registers of the launch bounds
    // hold it at three); the tile's own entries are needed last
    typedef double d2 __attribute__((ext_vector_type(2)));
    d2 sq[8], rq[8];
    double d[4][4];
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int t = tid + 256 * q, a = t / (GJB / 2), c = t % (GJB / 2);
        rq[q] = *reinterpret_cast<const d2 *>(R + a * npad + j0 + 2 * c);
    }
    const d2 *sp = reinterpret_cast<const d2 *>(S + (i0 + 16 * w + li) * GJB + 16 * lk);
#pragma unroll
    for (int q = 0; q < 8; q++) sq[q] = sp[q];
#pragma unroll
    for (int c = 0; c < 4; c++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int64_t gi = i0 + 16 * w + lk + 4 * v, gj = j0 + 16 * c + li;
            d[c][v] = J != K && gi < n && gj < n ? D[gi * n + gj] : (piv && gi == gj ? 1.0 : 0.0);
        }
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int t = tid + 256 * q, a = t / (GJB / 2), c = t % (GJB / 2);
        Rs[a][2 * c] = rq[q].x;
        Rs[a][2 * c + 1] = rq[q].y;
    }
    __syncthreads();
    rich_d4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; c++) acc[c] = (rich_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 16; q++)
#pragma unroll
        for (int c = 0; c < 4; c++)
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(q & 1 ? sq[q / 2].y : sq[q / 2].x,
                                                          Rs[4 * q + lk][16 * c + li], acc[c], 0, 0, 0);
    if (piv) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; c++)
#pragma unroll
            for (int v = 0; v < 4; v++) Rs[16 * w + lk + 4 * v][16 * c + li] = d[c][v] - acc[c][v];
        __syncthreads();
        invert_pivot(Rs, rc, Pinv, bad);
        return;
    }
#pragma unroll
    for (int c = 0; c < 4; c++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int64_t gi = i0 + 16 * w + lk + 4 * v, gj = j0 + 16 * c + li;
            if (gi < n && gj < n) D[gi * n + gj] = d[c][v] - acc[c][v];
        }
}

}  // namespace

// ------------------------------------------------------------------ host
namespace {
size_t ws_round(size_t b) { return (b + 255) & ~(size_t)255; }
}  // namespace

size_t match_ws_bytes(int64_t n, int64_t nnz) {
    const size_t un = (size_t)(n > 0 ? n : 1);
    return ws_round(un * 8) + ws_round((size_t)(nnz > 0 ? nnz : 1) * 8) + 2 * ws_round(un * 4) +
           ws_round(un * 8) + ws_round((un + 1) * 8) + ws_round((size_t)scan_tmp_size(n) * 8) + ws_round(4);
}

MatchWs match_ws_carve(void *base, int64_t n, int64_t nnz) {
    const size_t un = (size_t)(n > 0 ? n : 1);
    char *p = static_cast<char *>(base);
    MatchWs w;
    auto take = [&](size_t b) {
        char *q = p;
        p += ws_round(b);
        return q;
    };
    w.diag = (double *)take(un * 8);
    w.wts = (double *)take((size_t)(nnz > 0 ? nnz : 1) * 8);
    w.mate = (int32_t *)take(un * 4);
    w.cand = (int32_t *)take(un * 4);
    w.flag = (int64_t *)take(un * 8);
    w.id = (int64_t *)take((un + 1) * 8);
    w.stmp = (int64_t *)take((size_t)scan_tmp_size(n) * 8);
    w.still = (int32_t *)take(4);
    return w;
}

rich_status match_sweep_ws(int64_t n, const int64_t *rowptr, const int32_t *col, const double *val, int32_t *agg,
                           int64_t *nc_out, const MatchWs &w, int *h_still, hipStream_t s) {
    if (n == 0) {
        *nc_out = 0;
        return RICH_OK;
    }
    auto sliced = [&](auto &&launch) {
        for (int64_t r0 = 0; r0 < n; r0 += ROW_SLICE) launch(r0, nblocks(std::min(ROW_SLICE, n - r0) * ROW_LANES));
    };
    sliced([&](int64_t r0, unsigned g) { k_diag<<<g, TPB, 0, s>>>(r0, n, rowptr, col, val, w.diag); });
    LAUNCH_CHECK();
    // the weights do not change between rounds: computed once
    sliced([&](int64_t r0, unsigned g) {
        k_match_weights<<<g, TPB, 0, s>>>(r0, n, rowptr, col, val, w.diag, w.wts);
    });
    LAUNCH_CHECK();
    RICH_TRY(launch_fill_i32(w.mate, -1, n, s));
    for (int64_t round = 0;; round++) {
        RICH_TRY(launch_fill_i32(w.still, 0, 1, s));
        // a few rounds per host check; extra rounds after completion are no-ops
        for (int t = 0; t < 4; t++) {
            k_candidates<<<nblocks(n), TPB, 0, s>>>(n, rowptr, col, w.wts, w.mate, w.cand);
            k_commit<<<nblocks(n), TPB, 0, s>>>(n, w.cand, w.mate, w.still);
        }
        LAUNCH_CHECK();
        HIP_TRY(hipMemcpyAsync(h_still, w.still, sizeof(int), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        if (!*h_still) break;
        if (round > 4 * n + 16) return RICH_EHIP;  // every round matches or retires at least one vertex
    }
    k_leaders<<<nblocks(n), TPB, 0, s>>>(n, w.mate, w.flag);
    LAUNCH_CHECK();
    RICH_TRY(scan_exclusive_i64(w.flag, w.id, n, w.stmp, s));
    k_number<<<nblocks(n), TPB, 0, s>>>(n, w.mate, w.id, agg);
    LAUNCH_CHECK();
    int64_t nc = 0;
    HIP_TRY(hipMemcpyAsync(&nc, w.id + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    *nc_out = nc;
    return RICH_OK;
}

rich_status match_sweep(int64_t n, const int64_t *rowptr, const int32_t *col, const double *val, int32_t *agg,
                        int64_t *nc_out, hipStream_t s) {
    if (n == 0) {
        *nc_out = 0;
        return RICH_OK;
    }
    int64_t nnz = 0;
    HIP_TRY(hipMemcpyAsync(&nnz, rowptr + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    DevAlloc tmp;
    char *base;
    RICH_TRY(tmp.get(&base, match_ws_bytes(n, nnz)));
    int *h_still = nullptr;
    HIP_TRY(hipHostMalloc((void **)&h_still, sizeof(int)));
    rich_status st = match_sweep_ws(n, rowptr, col, val, agg, nc_out, match_ws_carve(base, n, nnz), h_still, s);
    (void)hipHostFree(h_still);
    return st;
}

rich_status vmb_aggregate(const CsrDev &A, double theta, int64_t block, int32_t *agg, int64_t *nc_out,
                          hipStream_t s) {
    *nc_out = 0;
    if (A.n == 0) return RICH_OK;
    const int64_t nblk = (A.n + block - 1) / block;
    DevAlloc tmp;
    double *diag;
    int32_t *p1;
    int64_t *cnt, *off, *stmp;
    RICH_TRY(tmp.get(&diag, A.n));
    RICH_TRY(tmp.get(&p1, A.n));
    RICH_TRY(tmp.get(&cnt, nblk + 1));
    RICH_TRY(tmp.get(&off, nblk + 1));
    RICH_TRY(tmp.get(&stmp, scan_tmp_size(nblk + 1)));
    k_row_diag<<<nblocks(A.n), TPB, 0, s>>>(A.n, A.rowptr, A.col, A.val, diag);
    LAUNCH_CHECK();
    HIP_TRY(hipMemsetAsync(cnt, 0, (nblk + 1) * sizeof(int64_t), s));
    k_vmb_block<<<(unsigned)((nblk + 63) / 64), 64, 0, s>>>(A.n, block, nblk, A.rowptr, A.col, A.val, diag, theta,
                                                             agg, p1, cnt);
    LAUNCH_CHECK();
    RICH_TRY(scan_exclusive_i64(cnt, off, nblk + 1, stmp, s));  // off[nblk] = total
    k_vmb_offset<<<nblocks(A.n), TPB, 0, s>>>(A.n, block, off, agg);
    LAUNCH_CHECK();
    HIP_TRY(hipMemcpyAsync(nc_out, off + nblk, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    return RICH_OK;
}

rich_status members(const int32_t *agg, int64_t n, int64_t nc, int64_t *mptr, int32_t *mem, hipStream_t s) {
    DevAlloc tmp;
    int64_t *cnt, *stmp;
    unsigned int *cursor;
    RICH_TRY(tmp.get(&cnt, nc));
    RICH_TRY(tmp.get(&cursor, nc));
    RICH_TRY(tmp.get(&stmp, scan_tmp_size(nc)));
    HIP_TRY(hipMemsetAsync(cnt, 0, nc * sizeof(int64_t), s));
    HIP_TRY(hipMemsetAsync(cursor, 0, nc * sizeof(unsigned int), s));
    if (n > 0) {
        k_count_members<<<nblocks(n), TPB, 0, s>>>(n, agg, cnt);
        LAUNCH_CHECK();
    }
    RICH_TRY(scan_exclusive_i64(cnt, mptr, nc, stmp, s));
    if (n > 0) {
        k_place_members<<<nblocks(n), TPB, 0, s>>>(n, agg, mptr, cursor, mem);
        LAUNCH_CHECK();
    }
    if (nc > 0) {
        k_sort_members<<<nblocks(nc), TPB, 0, s>>>(nc, mptr, mem);
        LAUNCH_CHECK();
    }
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    return RICH_OK;
}

rich_status galerkin_symbolic(const CsrDev &A, const int32_t *agg, int64_t nc, const int64_t *mptr,
                              const int32_t *mem, CsrDev *C, DevAlloc &mem_out, hipStream_t s) {
    DevAlloc tmp;
    int64_t *seg, *segptr, *cnt, *stmp;
    int32_t *scratch;
    RICH_TRY(tmp.get(&seg, nc));
    RICH_TRY(tmp.get(&segptr, nc + 1));
    RICH_TRY(tmp.get(&cnt, nc));
    RICH_TRY(tmp.get(&stmp, scan_tmp_size(nc)));
    RICH_TRY(tmp.get(&scratch, A.nnz));
    C->n = nc;
    RICH_TRY(mem_out.get(&C->rowptr, nc + 1));
    if (nc > 0) {
        k_seg_len<<<nblocks(nc), TPB, 0, s>>>(nc, mptr, mem, A.rowptr, seg);
        LAUNCH_CHECK();
    }
    RICH_TRY(scan_exclusive_i64(seg, segptr, nc, stmp, s));
    if (nc > 0) {
        k_sym_collect<<<nblocks(nc, 64), 64, 0, s>>>(nc, mptr, mem, A.rowptr, A.col, agg, segptr, scratch, cnt);
        LAUNCH_CHECK();
    }
    RICH_TRY(scan_exclusive_i64(cnt, C->rowptr, nc, stmp, s));
    int64_t nnz = 0;
    HIP_TRY(hipMemcpyAsync(&nnz, C->rowptr + nc, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    C->nnz = nnz;
    RICH_TRY(mem_out.get(&C->col, nnz));
    RICH_TRY(mem_out.get(&C->val, nnz));
    if (nc > 0) {
        k_sym_write<<<nblocks(nc), TPB, 0, s>>>(nc, segptr, scratch, C->rowptr, C->col);
        LAUNCH_CHECK();
    }
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    return RICH_OK;
}

rich_status galerkin_numeric(const CsrDev &A, const int32_t *agg, const int64_t *mptr, const int32_t *mem,
                             const CsrDev &C, hipStream_t s) {
    if (C.n == 0) return RICH_OK;
    k_gal_numeric<<<nblocks(C.n, 64), 64, 0, s>>>(C.n, mptr, mem, A.rowptr, A.col, A.val, agg, C.rowptr, C.col,
                                                  C.val);
    LAUNCH_CHECK();
    return RICH_OK;
}

rich_status galerkin_sources(const CsrDev &A, const int32_t *agg, const int64_t *mptr, const int32_t *mem,
                             const CsrDev &C, const Grid3 *g, uint32_t *gptr, uint32_t *gsrc, hipStream_t s) {
    if (C.n == 0) return RICH_OK;
    DevAlloc tmp;
    int64_t *cnt, *ptr, *stmp;
    Slab scratch;
    scratch.add(&cnt, C.nnz);
    scratch.add(&ptr, C.nnz + 1);
    scratch.add(&stmp, scan_tmp_size(C.nnz));
    RICH_TRY(scratch.get(tmp));
    const StencilIndex ix{g ? g->nx : 0, g ? g->ny : 0, g ? g->nz : 0};
    const unsigned nb = nblocks(C.n, 64);
    k_gal_sources<false><<<nb, 64, 0, s>>>(C.n, A.n, ix, mptr, mem, A.rowptr, A.col, agg, C.rowptr, C.col, cnt,
                                           nullptr, nullptr);
    LAUNCH_CHECK();
    RICH_TRY(scan_exclusive_i64(cnt, ptr, C.nnz, stmp, s));
    k_narrow_u32<<<nblocks(C.nnz + 1), TPB, 0, s>>>(C.nnz + 1, ptr, gptr);
    k_gal_sources<true><<<nb, 64, 0, s>>>(C.n, A.n, ix, mptr, mem, A.rowptr, A.col, agg, C.rowptr, C.col, cnt, gptr,
                                          gsrc);
    LAUNCH_CHECK();
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    return RICH_OK;
}

rich_status galerkin_sum(const uint32_t *gptr, const uint32_t *gsrc, const double *val, Level &Lc, bool ordered,
                         bool mixed, hipStream_t s) {
    if (Lc.nnz == 0) return RICH_OK;
    const unsigned nb = xcd_grid(Lc.nnz, GS_TPB);
    const VLevel &V = Lc.V;
    if (ordered && mixed && !V.ent)
        k_gal_sum<GS_VALF><<<nb, GS_TPB, 0, s>>>(Lc.nnz, gptr, gsrc, val, Lc.val, (float *)V.val, V.place, nullptr, nullptr, nullptr);
    else if (ordered && mixed)
        k_gal_sum<GS_ENT><<<nb, GS_TPB, 0, s>>>(Lc.nnz, gptr, gsrc, val, Lc.val, nullptr, V.place, V.off, V.ent, nullptr);
    else if (ordered)
        k_gal_sum<GS_VAL><<<nb, GS_TPB, 0, s>>>(Lc.nnz, gptr, gsrc, val, Lc.val, nullptr, V.place, nullptr, nullptr, (double *)V.val);
    else if (mixed)
        k_gal_sum<GS_F32><<<nb, GS_TPB, 0, s>>>(Lc.nnz, gptr, gsrc, val, Lc.val, Lc.valf, nullptr, nullptr, nullptr, nullptr);
    else
        k_gal_sum<GS_NONE><<<nb, GS_TPB, 0, s>>>(Lc.nnz, gptr, gsrc, val, Lc.val, nullptr, nullptr, nullptr, nullptr, nullptr);
    LAUNCH_CHECK();
    return RICH_OK;
}

rich_status galerkin(const CsrDev &A, const int32_t *agg, int64_t nc, CsrDev *C, DevAlloc &mem_out,
                     hipStream_t s, bool values) {
    DevAlloc tmp;
    int64_t *mptr;
    int32_t *mem;
    RICH_TRY(tmp.get(&mptr, nc + 1));
    RICH_TRY(tmp.get(&mem, A.n));
    RICH_TRY(members(agg, A.n, nc, mptr, mem, s));
    RICH_TRY(galerkin_symbolic(A, agg, nc, mptr, mem, C, mem_out, s));
    if (values) RICH_TRY(galerkin_numeric(A, agg, mptr, mem, *C, s));
    HIP_TRY(hipStreamSynchronize(s));
    return RICH_OK;
}

rich_status stream_blocks(Level &Lv, DevAlloc &mem, hipStream_t s) {
    if (Lv.n == 0) return RICH_OK;
    DevAlloc tmp;
    int *flag;
    RICH_TRY(tmp.get(&flag, 1));
    HIP_TRY(hipMemsetAsync(flag, 0, sizeof(int), s));
    k_max_rowlen<<<nblocks(Lv.n), TPB, 0, s>>>(Lv.n, Lv.rowptr, flag);
    LAUNCH_CHECK();
    int too_long = 0;
    HIP_TRY(hipMemcpyAsync(&too_long, flag, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (too_long) return RICH_OK;
    int64_t nrb = (Lv.nnz + STREAM_CHUNK - 1) / STREAM_CHUNK;
    // lanes per row in the reduction phase, by the mean row length
    int64_t mean = Lv.nnz / Lv.n;
    Lv.sg = mean < 8 ? 1 : mean < 16 ? 2 : mean < 32 ? 4 : 8;
    // the launch grid is rounded up to a multiple of the XCD count: pad with empty blocks
    int64_t ngrid = xcd_grid(nrb, 1);
    RICH_TRY(mem.get(&Lv.rb, 2 * (ngrid + 1)));
    k_stream_rb<<<nblocks(ngrid + 1), TPB, 0, s>>>(Lv.n, nrb, ngrid, Lv.rowptr, Lv.rb);
    LAUNCH_CHECK();
    Lv.nrb = ngrid;
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    return RICH_OK;
}

rich_status csr_invd(const CsrDev &A, const int32_t *pos, double *invd, float *invdf, hipStream_t s) {
    if (A.n == 0) return RICH_OK;
    k_row_l1<<<nblocks(A.n, 256), 256, 0, s>>>(A.n, A.rowptr, A.val, pos, invd, invdf);
    LAUNCH_CHECK();
    return RICH_OK;
}

rich_status compose_agg(int32_t *comp, const int32_t *a, int64_t n, hipStream_t s) {
    if (n == 0) return RICH_OK;
    if (a == nullptr) {
        k_iota<<<nblocks(n), TPB, 0, s>>>(n, comp);
    } else {
        k_compose<<<nblocks(n), TPB, 0, s>>>(n, comp, a);
    }
    LAUNCH_CHECK();
    return RICH_OK;
}

// Inverse of an SPD CSR matrix into a dense row-major n x n buffer, using
// the workspace of dense_inverse_ws (no allocation: it runs on every refresh).
int64_t dense_inverse_ws(int64_t n) {
    const int64_t npad = (n + GJB - 1) / GJB * GJB;
    return (int64_t)GJB * GJB + 2 * (int64_t)GJB * npad + 1;
}

rich_status dense_inverse(const CsrDev &A, double *D, double *ws, hipStream_t s) {
    int64_t n = A.n;
    if (n == 0) return RICH_OK;
    const int tiles = (int)((n + GJB - 1) / GJB);
    const int64_t npad = (int64_t)tiles * GJB;
    double *Pinv = ws, *S = ws + GJB * GJB, *R = S + GJB * npad;
    int *bad = reinterpret_cast<int *>(R + GJB * npad);
    HIP_TRY(hipMemsetAsync(bad, 0, sizeof(int), s));
    HIP_TRY(hipMemsetAsync(D, 0, (size_t)n * n * sizeof(double), s));
    k_csr_to_dense<<<nblocks(n), TPB, 0, s>>>(n, A.rowptr, A.col, A.val, D);
    k_bgj_pivot<<<1, 256, 0, s>>>(D, n, Pinv, bad);
    LAUNCH_CHECK();
    for (int K = 0; K < tiles; K++) {
        k_bgj_panel<<<4 * tiles, 256, 0, s>>>(D, n, npad, K, Pinv, S, R);
        k_bgj_update<<<tiles * tiles + (K < tiles - 1 ? 1 : 0), 256, 0, s>>>(D, n, npad, K, tiles, S, R, Pinv, bad);
    }
    LAUNCH_CHECK();
    int hb = 0;
    HIP_TRY(hipMemcpyAsync(&hb, bad, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return hb ? RICH_NOT_SPD : RICH_OK;
}

// lanes per row: 4 for short rows, 8 otherwise
static inline bool short_rows(const Level &Lv) { return Lv.nnz < 16 * Lv.n; }

template <class TB, class T, bool POST>
void launch_stream(const Level &Lv, const T *val, const T *invd, const TB *b, const T *v, T *out, hipStream_t s) {
    unsigned g = (unsigned)Lv.nrb;
    switch (Lv.sg) {
    case 1: k_csr_stream<1, TB, T, POST><<<g, 256, 0, s>>>(Lv.rb, Lv.rowptr, Lv.col, val, invd, b, v, out); break;
    case 2: k_csr_stream<2, TB, T, POST><<<g, 256, 0, s>>>(Lv.rb, Lv.rowptr, Lv.col, val, invd, b, v, out); break;
    case 4: k_csr_stream<4, TB, T, POST><<<g, 256, 0, s>>>(Lv.rb, Lv.rowptr, Lv.col, val, invd, b, v, out); break;
    default: k_csr_stream<8, TB, T, POST><<<g, 256, 0, s>>>(Lv.rb, Lv.rowptr, Lv.col, val, invd, b, v, out); break;
    }
}

template <class TB, class T>
rich_status launch_csr_pre(const Level &Lv, const T *val, const T *x0, const TB *b, T *r, hipStream_t s) {
    if (Lv.n == 0) return RICH_OK;
    if (Lv.rb) {
        launch_stream<TB, T, false>(Lv, val, nullptr, b, x0, r, s);
        LAUNCH_CHECK();
        return RICH_OK;
    }
    if (short_rows(Lv))
        k_csr_pre<4, TB, T><<<xcd_grid(Lv.n * 4, TPB), TPB, 0, s>>>(Lv.n, Lv.rowptr, Lv.col, val, x0, b, r);
    else
        k_csr_pre<8, TB, T><<<xcd_grid(Lv.n * 8, TPB), TPB, 0, s>>>(Lv.n, Lv.rowptr, Lv.col, val, x0, b, r);
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class TB, class T>
rich_status launch_csr_post(const Level &Lv, const T *val, const T *invd, const TB *b, const T *x0, const T *xc,
                            T *x, hipStream_t s) {
    if (Lv.n == 0) return RICH_OK;
    T *xt = (T *)Lv.r;  // the residual of this level is dead by now
    if (Lv.prow) {
        RICH_TRY(launch_sa_prolong<TB, T>(Lv, invd, b, nullptr, x0, xc, xt, s));
    } else {
        k_csr_prolong<T><<<xcd_grid(Lv.n, TPB), TPB, 0, s>>>(Lv.n, x0, xc, Lv.agg, xt);
        LAUNCH_CHECK();
    }
    if (Lv.rb)
        launch_stream<TB, T, true>(Lv, val, invd, b, xt, x, s);
    else if (short_rows(Lv))
        k_csr_post<4, TB, T><<<xcd_grid(Lv.n * 4, TPB), TPB, 0, s>>>(Lv.n, Lv.rowptr, Lv.col, val, invd, b, xt, x);
    else
        k_csr_post<8, TB, T><<<xcd_grid(Lv.n * 8, TPB), TPB, 0, s>>>(Lv.n, Lv.rowptr, Lv.col, val, invd, b, xt, x);
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class T>
rich_status launch_restrict(const Level &Lv, const T *r, T *bc, int64_t nc, const T *invdc, T *x0c, hipStream_t s) {
    if (nc == 0) return RICH_OK;
    if (Lv.prow) return launch_sa_restrict<T>(Lv, r, bc, nc, invdc, x0c, s);
    k_restrict<T><<<xcd_grid(nc, RESTRICT_TPB), RESTRICT_TPB, 0, s>>>(nc, Lv.vmptr ? Lv.vmptr : Lv.mptr,
                                                                      Lv.vmem ? Lv.vmem : Lv.mem, Lv.vslot, r, bc,
                                                                      invdc, x0c);
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class TB, class T>
rich_status launch_csr_sweeps(const Level &Lv, const T *val, const T *invd, const TB *b, T *x, T *tmp, int sweeps,
                              hipStream_t s) {
    if (Lv.n == 0) return RICH_OK;
    T *cur = (sweeps % 2 == 1) ? x : tmp;
    unsigned g = xcd_grid(Lv.n * 8, TPB);
    k_csr_sweep<8, TB, T><<<g, TPB, 0, s>>>(Lv.n, Lv.rowptr, Lv.col, val, invd, b, nullptr, cur, 1);
    LAUNCH_CHECK();
    for (int t = 1; t < sweeps; t++) {
        T *nxt = (cur == x) ? tmp : x;
        k_csr_sweep<8, TB, T><<<g, TPB, 0, s>>>(Lv.n, Lv.rowptr, Lv.col, val, invd, b, cur, nxt, 0);
        LAUNCH_CHECK();
        cur = nxt;
    }
    return RICH_OK;
}

rich_status launch_csr_spmv(const CsrDev &A, const double *x, double *y, hipStream_t s) {
    if (A.n == 0) return RICH_OK;
    k_csr_spmv<<<xcd_grid(A.n * 8, TPB), TPB, 0, s>>>(A.n, A.rowptr, A.col, A.val, x, y);
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class T>
rich_status launch_restrict_batch(const std::vector<RestrictItem<T>> &v, hipStream_t s, WorkQueue *q) {
    std::vector<unsigned> nb;
    for (const auto &it : v) nb.push_back((unsigned)((it.nc + RESTRICT_TPB - 1) / RESTRICT_TPB));
    return launch_batches(v, nb, [&](const Batch<RestrictItem<T>> &bt, unsigned g) {
        k_restrict_batch<T><<<g, RESTRICT_TPB, 0, s>>>(bt);
    }, q);
}
template <class T, bool POST>
static rich_status stream_batch(const std::vector<CsrItem<T>> &v, hipStream_t s, WorkQueue *q) {
    for (int G : {1, 2, 4, 8}) {
        std::vector<StreamArgs<T>> a;
        std::vector<unsigned> nb;
        for (const auto &it : v) {
            const Level &Lv = *it.Lv;
            if (Lv.sg != G || Lv.n == 0) continue;
            a.push_back({Lv.rb, Lv.rowptr, Lv.col, it.val, it.invd, it.b, POST ? (const T *)Lv.r : it.x0, it.out});
            nb.push_back((unsigned)Lv.nrb);
        }
        auto launch = [&](const Batch<StreamArgs<T>> &bt, unsigned g) {
            switch (G) {
            case 1: k_csr_stream_batch<1, T, POST><<<g, 256, 0, s>>>(bt); break;
            case 2: k_csr_stream_batch<2, T, POST><<<g, 256, 0, s>>>(bt); break;
            case 4: k_csr_stream_batch<4, T, POST><<<g, 256, 0, s>>>(bt); break;
            default: k_csr_stream_batch<8, T, POST><<<g, 256, 0, s>>>(bt); break;
            }
        };
        RICH_TRY(launch_batches(a, nb, launch, q));
    }
    return RICH_OK;
}

template <class T>
rich_status launch_csr_pre_batch(const std::vector<CsrItem<T>> &v, hipStream_t s, WorkQueue *q) {
    return stream_batch<T, false>(v, s, q);
}

template <class T>
rich_status launch_csr_post_batch(const std::vector<CsrItem<T>> &v, hipStream_t s, WorkQueue *q) {
    // xt = x0 + P xc into each level's r buffer, then post-smoothing from xt
    std::vector<ProlongArgs<T>> a;
    std::vector<unsigned> nb;
    for (const auto &it : v) {
        a.push_back({it.Lv->n, it.x0, it.xc, it.Lv->agg, (T *)it.Lv->r});
        nb.push_back((unsigned)((it.Lv->n + TPB - 1) / TPB));
    }
    RICH_TRY(launch_batches(a, nb, [&](const Batch<ProlongArgs<T>> &bt, unsigned g) {
        k_csr_prolong_batch<T><<<g, TPB, 0, s>>>(bt);
    }, q));
    return stream_batch<T, true>(v, s, q);
}

#define INST_BATCH(T)                                                                                          \
    template rich_status launch_csr_pre_batch<T>(const std::vector<CsrItem<T>> &, hipStream_t, WorkQueue *);  \
    template rich_status launch_csr_post_batch<T>(const std::vector<CsrItem<T>> &, hipStream_t, WorkQueue *);
INST_BATCH(double)
INST_BATCH(float)
template rich_status launch_restrict_batch<double>(const std::vector<RestrictItem<double>> &, hipStream_t, WorkQueue *);
template rich_status launch_restrict_batch<float>(const std::vector<RestrictItem<float>> &, hipStream_t, WorkQueue *);

#define INST_CSR(TB, T)                                                                                         \
    template rich_status launch_csr_pre<TB, T>(const Level &, const T *, const T *, const TB *, T *, hipStream_t); \
    template rich_status launch_csr_post<TB, T>(const Level &, const T *, const T *, const TB *, const T *,        \
                                                const T *, T *, hipStream_t);                                     \
    template rich_status launch_csr_sweeps<TB, T>(const Level &, const T *, const T *, const TB *, T *, T *, int,  \
                                                  hipStream_t);
INST_CSR(double, double)
INST_CSR(double, float)
INST_CSR(float, float)
template rich_status launch_restrict<double>(const Level &, const double *, double *, int64_t, const double *,
                                             double *, hipStream_t);
template rich_status launch_restrict<float>(const Level &, const float *, float *, int64_t, const float *, float *,
                                            hipStream_t);

}  // namespace rich
