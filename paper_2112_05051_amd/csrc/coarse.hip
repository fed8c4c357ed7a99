// Coarse levels of the V-cycle in aggregate order.
//
// The rows of a smoothed coarse level are renumbered by the member lists of
// the next level's aggregates, so the rows of one aggregate are neighbours and
// a thread block that owns whole aggregates can finish more than its sweep:
//   down: r = b - A x0 of its rows, then P^T r of its aggregates, which goes
//         straight to the next level's right-hand side (with x0 = D^{-1} b
//         there); r is never stored;
//   up:   x = xt + D^{-1}(b - A xt) of its rows, then xt = x0 + P x of the finer
//         level's rows they stand for (one contiguous run per row).  Level 1
//         stores x in natural order, for the fine level's gather along x (in
//         aggregate order the fine post-smoother takes 153 instead of 148 us
//         at 256^3, 26 instead of 22 on the 199 x 199 x 38 grid).
// A level is two launches a cycle instead of four (sweep, restriction,
// prolongation, sweep).  The products are formed in entry order into LDS and
// added per row, in the column order of the level's matrix; members are added
// in ascending order: the sums are those of the separate kernels.
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "common.hpp"

namespace rich {

namespace {

constexpr int TPB = 256;
inline unsigned nblocks(int64_t n, int tpb = TPB) { return (unsigned)((n + tpb - 1) / tpb); }

// Entries of a level in aggregate order, read in pairs (the entry index is
// even): FP32 (byte offset of the column's value, value) pairs, FP64 offsets
// and values apart.  The offsets go into the gathers as they are loaded.
typedef int i2_t __attribute__((ext_vector_type(2)));
typedef int i4_t __attribute__((ext_vector_type(4)));
typedef double d2_t __attribute__((ext_vector_type(2)));
template <class P, bool NT>
__device__ __forceinline__ P load_as(const void *p, uint32_t off) {
    const P *q = reinterpret_cast<const P *>(reinterpret_cast<const char *>(p) + off);
    return NT ? __builtin_nontemporal_load(q) : *q;
}
template <class T>
struct Entries;
template <>
struct Entries<float> {
    const int2 *e;
    __device__ __forceinline__ void pair(int64_t base, uint32_t i, uint32_t *c, float *v) const {
        const i4_t t = load_as<i4_t, false>(e + base, i * 8);
        c[0] = t.x;
        v[0] = __int_as_float(t.y);
        c[1] = t.z;
        v[1] = __int_as_float(t.w);
    }
};
template <>
struct Entries<double> {
    const uint32_t *c_;
    const double *v_;
    __device__ __forceinline__ void pair(int64_t base, uint32_t i, uint32_t *c, double *v) const {
        const i2_t t = load_as<i2_t, false>(c_ + base, i * 4);
        const d2_t u = load_as<d2_t, false>(v_ + base, i * 8);
        c[0] = t.x;
        c[1] = t.y;
        v[0] = u.x;
        v[1] = u.y;
    }
};

// Large levels: 16-bit places in the block's column list and values, read four
// entries at a time.
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef uint16_t u16x4_t __attribute__((ext_vector_type(4)));
template <class T>
struct Locals {
    const uint16_t *i_;
    const T *v_;
    __device__ __forceinline__ void four(int64_t base, uint32_t i, u16x4_t *c, T *v) const {
        *c = load_as<u16x4_t, true>(i_ + base, i * 2);
        if constexpr (sizeof(T) == 4) {
            *reinterpret_cast<f4_t *>(v) = load_as<f4_t, true>(v_ + base, i * 4);
        } else {
            *reinterpret_cast<d2_t *>(v) = load_as<d2_t, true>(v_ + base, i * 8);
            *reinterpret_cast<d2_t *>(v + 2) = load_as<d2_t, true>(v_ + base, i * 8 + 16);
        }
    }
};

// One level's part of a cycle.  blk: first aggregate, row and entry of each
// block (x, y, z), one more than there are blocks, and (w) the columns it
// lists; lds_ent: products held.
template <class T>
struct VArgs {
    const int4 *blk;
    const int32_t *ptr;  // row starts
    Entries<T> ent;
    Locals<T> loc;
    const uint32_t *list;  // byte offsets of a block's columns, from its first entry's index
    const T *b, *v;      // right-hand side; x0 (down) or xt (up)
    // down
    const int64_t *mptr;  // rows of each aggregate
    const int32_t *pos;   // next level's place of each aggregate (null: itself)
    const T *invdc;       // next level: D^{-1} (null at the coarsest), b and x0
    T *bc, *x0c;
    // up
    const T *invd;
    T *x;               // result (level 1, in natural order: row i's at mem[i]), or
    const int32_t *mem;
    const int2 *child;  // the finer level's rows of each row,
    const T *x0f;       // their x0
    T *xtf;             // and their prolongated iterate
    int lds_ent, lds_row;
};

// The split that lists its blocks' columns, at most V_SORT entries a block.
constexpr int V_LOCAL = 4, V_SORT = 512 * V_LOCAL;

// Sum of a row's products [ra, re) as G interleaved partial sums added
// pairwise: by the G lanes of the row's group, or for G <= 2 by one lane.
template <int G, class T>
__device__ __forceinline__ T row_sum(const T *prod, int ra, int re, int lane) {
    if (G == 1) {
        T s = 0;
        for (int e = ra; e < re; e++) s += prod[e];
        return s;
    }
    if (G == 2) {
        T s0 = 0, s1 = 0;
        int e = ra;
        for (; e + 1 < re; e += 2) {
            s0 += prod[e];
            s1 += prod[e + 1];
        }
        if (e < re) s0 += prod[e];
        return s0 + s1;
    }
    T s = 0;
    for (int e = ra + lane; e < re; e += G) s += prod[e];
    return group_sum<G>(s);
}

// UP = false: down.  These kernels are bound by how their loads are issued, not
// by memory: with 8-byte loads under a bounds check each, 64-bit gather
// addresses and two lanes per row a level-1 sweep at 256^3 took about 600
// instructions a wave (82 + 78 us, then 71 + 67).  What was left was the
// gather, one L1 access per entry (30 M a sweep, about one a cycle and CU).
// NP = 4 (large levels): a block's distinct columns, about a third of its
// entries, are listed at set-up and their values staged in LDS first; entries
// are 16-bit places in that list and values (6 bytes in FP32, not 8).  Half the
// L1 accesses; level 1 at 256^3 70 + 72 us, now 62 + 57 (51 us of bytes each).
// NP <= 2: 256 NP pairs at a time, each wave a run of 128 entries per step,
// gathered from memory: one dependent load less, which is what counts where the
// blocks are few.
// Runs past a block's end are read unmasked (the next block's entries, or the
// padding behind the last) and their products not used.
template <int NP, int G, class T, bool UP>
__device__ __forceinline__ void vlevel_body(const VArgs<T> &a, T *__restrict__ prod, int blk) {
    constexpr int LPR = G <= 2 ? 1 : G;  // lanes per row
    constexpr bool LOC = NP == V_LOCAL;
    T *rr = prod + a.lds_ent;
    const int4 b0 = a.blk[blk], b1 = a.blk[blk + 1];
    const int R0 = b0.y, R1 = b1.y, E0 = b0.z & (LOC ? ~3 : ~1), E1 = b1.z;
    if (R0 >= R1) return;
    const int tid = threadIdx.x, lane = tid % LPR;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // what the row phase needs of its first row, and (up) what the last phase needs
    // of its first rows, eight lanes each, is loaded ahead of the products: on
    // small levels each of these loads is a step in the chain that a launch
    // consists of (up at 64^3 3.92, now 3.84 us; down, the same for its aggregates
    // takes longer, 4.23 for 4.08: more loads before the entries')
    int2 ch = make_int2(0, 0);
    T pc = 0;
    if (UP && a.child && R0 + tid / 8 < R1) ch = a.child[R0 + tid / 8];
    auto last_in = [&]() {
        if (UP && ch.x + tid % 8 < ch.y) pc = a.x0f[ch.x + tid % 8];
    };
    int row = R0 + tid / LPR;
    int ra = 0, re = 0;
    int32_t pm = 0;
    T pb = 0, pd = 0, pv = 0;
    auto row_in = [&]() {
        if (row < R1) {
            ra = a.ptr[row] - E0;
            re = a.ptr[row + 1] - E0;
            pb = a.b[row];
            if (UP) {
                pd = a.invd[row];
                pv = a.v[row];
                if (!a.child) pm = a.mem[row];
            }
        }
    };
    if constexpr (LOC) {
        T *xs = rr + a.lds_row;
        constexpr int QL = 4, QE = 512 * NP / 1024;
        const int nu = b0.w;
        const uint32_t *list = a.list + b0.z;
        uint32_t o[QL];
#pragma unroll
        for (int q = 0; q < QL; q++) o[q] = tid + 256 * q < nu ? list[tid + 256 * q] : 0u;
        u16x4_t c[QE];
        T v[QE][4];
#pragma unroll
        for (int q = 0; q < QE; q++) {
            c[q] = (u16x4_t){0, 0, 0, 0};
            if (E0 + 1024 * q + 256 * wave < E1) a.loc.four(E0 + 1024 * q, 4 * tid, &c[q], v[q]);
        }
#pragma unroll
        for (int q = 0; q < QL; q++)
            if (tid + 256 * q < nu) xs[tid + 256 * q] = load_as<T, false>(a.v, o[q]);
        for (int u = tid + 256 * QL; u < nu; u += 256) xs[u] = load_as<T, false>(a.v, list[u]);
        row_in();
        last_in();
        __syncthreads();
#pragma unroll
        for (int q = 0; q < QE; q++)
            if (E0 + 1024 * q + 256 * wave < E1) {
                T *to = prod + 1024 * q + 4 * tid;
                const T t0 = v[q][0] * xs[c[q].x], t1 = v[q][1] * xs[c[q].y];
                const T t2 = v[q][2] * xs[c[q].z], t3 = v[q][3] * xs[c[q].w];
                if constexpr (sizeof(T) == 4) {
                    *reinterpret_cast<f4_t *>(to) = (f4_t){t0, t1, t2, t3};
                } else {
                    *reinterpret_cast<d2_t *>(to) = (d2_t){t0, t1};
                    *reinterpret_cast<d2_t *>(to + 2) = (d2_t){t2, t3};
                }
            }
    } else {
        const int wrun = wave * 128;
        row_in();
        for (int base = E0; base < E1; base += 512 * NP) {
            uint32_t c[NP][2];
            T v[NP][2], x[NP][2];
#pragma unroll
            for (int q = 0; q < NP; q++) {
                c[q][0] = c[q][1] = 0;
                v[q][0] = v[q][1] = 0;
                if (base + 512 * q + wrun < E1) a.ent.pair(base + 512 * q, 2 * tid, c[q], v[q]);
            }
#pragma unroll
            for (int q = 0; q < NP; q++) {
                x[q][0] = load_as<T, false>(a.v, c[q][0]);
                x[q][1] = load_as<T, false>(a.v, c[q][1]);
            }
            if (base == E0) last_in();
#pragma unroll
            for (int q = 0; q < NP; q++)
                if (base + 512 * q + wrun < E1) {
                    typedef T t2 __attribute__((ext_vector_type(2)));
                    *reinterpret_cast<t2 *>(prod + (base - E0) + 512 * q + 2 * tid) =
                        (t2){v[q][0] * x[q][0], v[q][1] * x[q][1]};
                }
        }
    }
    __syncthreads();
    // every lane of a group runs the same number of row iterations (shuffles)
    for (int rb = R0; rb < R1; rb += 256 / LPR) {
        if (rb != R0) {
            row = rb + tid / LPR;
            row_in();
        }
        const T s = row_sum<G, T>(prod, ra, row < R1 ? re : ra, lane);
        if (lane == 0 && row < R1) {
            if (!UP) rr[row - R0] = pb - s;
            else if (a.child) rr[row - R0] = pv + pd * (pb - s);
            else a.x[pm] = pv + pd * (pb - s);
        }
    }
    if (UP && !a.child) return;
    __syncthreads();
    if (UP) {
        // eight lanes per row for its run on the finer level
        for (int r = R0 + tid / 8; r < R1; r += 32) {
            if (r >= R0 + 32) {
                ch = a.child[r];
                if (ch.x + tid % 8 < ch.y) pc = a.x0f[ch.x + tid % 8];
            }
            const T xr = rr[r - R0];
            if (ch.x + tid % 8 < ch.y) a.xtf[ch.x + tid % 8] = pc + xr;
            for (int t = ch.x + tid % 8 + 8; t < ch.y; t += 8) a.xtf[t] = a.x0f[t] + xr;
        }
        return;
    }
    for (int J = b0.x + tid; J < b1.x; J += 256) {
        const int m0 = (int)a.mptr[J] - R0, m1 = (int)a.mptr[J + 1] - R0;
        const int to = a.pos ? a.pos[J] : J;
        const T d = a.invdc ? a.invdc[to] : (T)0;
        T s = 0;
        for (int m = m0; m < m1; m++) s += rr[m];
        a.bc[to] = s;
        if (a.invdc) a.x0c[to] = s * d;
    }
}

extern __shared__ __align__(16) char vlevel_lds[];

template <int NP, int G, class T, bool UP>
__global__ void __launch_bounds__(256) k_vlevel(VArgs<T> a) {
    vlevel_body<NP, G, T, UP>(a, reinterpret_cast<T *>(vlevel_lds), (int)xcd_block());
}

template <int NP, int G, class T, bool UP>
__global__ void __launch_bounds__(256) k_vlevel_batch(Batch<VArgs<T>> B) {
    for_each_block(B, xcd_block(), [&](unsigned L) {
        const int e = batch_entry(B, L);
        vlevel_body<NP, G, T, UP>(B.a[e], reinterpret_cast<T *>(vlevel_lds), (int)(L - B.begin[e]));
    });
}

// x = Ainv b on the coarsest level, one wavefront per row, prolongated to the
// finer level's rows (child) or stored (one coarse level only).
template <class TB, class T>
struct GemvArgs {
    const T *Ainv;
    const TB *b;
    int64_t n;
    T *x;
    const int2 *child;
    const T *x0f;
    T *xtf;
};
template <class TB, class T>
__device__ __forceinline__ void gemv_body(const GemvArgs<TB, T> &g, int64_t blk) {
    const int64_t row = (blk * blockDim.x + threadIdx.x) / 64, n = g.n;
    const int lane = threadIdx.x % 64;
    if (row >= n) return;
    int2 c = make_int2(0, 0);
    T x0 = 0;
    if (g.child) {
        c = g.child[row];
        if (c.x + lane < c.y) x0 = g.x0f[c.x + lane];
    }
    // four independent partial sums per lane keep four row segments in flight
    const T *__restrict__ a = g.Ainv + row * n;
    const TB *__restrict__ b = g.b;
    T s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    int64_t j = lane;
    for (; j + 192 < n; j += 256) {
        s0 += a[j] * (T)b[j];
        s1 += a[j + 64] * (T)b[j + 64];
        s2 += a[j + 128] * (T)b[j + 128];
        s3 += a[j + 192] * (T)b[j + 192];
    }
    for (; j < n; j += 64) s0 += a[j] * (T)b[j];
    T s = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (g.child) {
        s = __shfl(s, 0, 64);
        if (c.x + lane < c.y) g.xtf[c.x + lane] = x0 + s;
        for (int t = c.x + lane + 64; t < c.y; t += 64) g.xtf[t] = g.x0f[t] + s;
    } else if (lane == 0) {
        g.x[row] = s;
    }
}

template <class TB, class T>
__global__ void k_dense_gemv(GemvArgs<TB, T> g) {
    gemv_body(g, blockIdx.x);
}
template <class T>
__global__ void k_dense_gemv_batch(Batch<GemvArgs<T, T>> B) {
    for_each_block(B, blockIdx.x, [&](unsigned L) {
        const int e = batch_entry(B, L);
        gemv_body(B.a[e], (int64_t)(L - B.begin[e]));
    });
}

// xt = x0 + P x on the finer level (the coarsest level without a direct solve)
template <class T>
__global__ void k_v_prolong(int64_t n, const T *__restrict__ x, const int2 *__restrict__ child,
                            const T *__restrict__ x0f, T *__restrict__ xtf) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int2 c = child[i];
    const T v = x[i];
    for (int t = c.x; t < c.y; t++) xtf[t] = x0f[t] + v;
}

// ------------------------------------------------------------------ set-up
__global__ void k_v_pos(int64_t n, const int32_t *__restrict__ mem, const int64_t *__restrict__ rowptr,
                        int32_t *__restrict__ pos, int64_t *__restrict__ len) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int32_t i = mem[p];
    pos[i] = (int32_t)p;
    len[p] = rowptr[i + 1] - rowptr[i];
}

__global__ void k_v_narrow(int64_t n, const int64_t *__restrict__ in, int32_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (int32_t)in[i];
}

// column offsets (with ent: there and by entry; otherwise in vcol, in aggregate
// order) and the place of every entry of the level's matrix
__global__ void k_v_columns(int64_t n, uint32_t tsz, const int32_t *__restrict__ mem,
                            const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                            const int32_t *__restrict__ pos, const int32_t *__restrict__ ptr,
                            int32_t *__restrict__ place, uint32_t *__restrict__ off, int2 *__restrict__ ent,
                            uint32_t *__restrict__ vcol) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int32_t i = mem[p];
    int32_t o = ptr[p];
    for (int64_t e = rowptr[i]; e < rowptr[i + 1]; e++, o++) {
        const uint32_t c = (uint32_t)pos[col[e]] * tsz;
        if (ent) ent[o].x = (int)(off[e] = c);
        else vcol[o] = c;
        place[e] = o;
    }
}

// Bitonic sort of N keys in LDS, ascending.
template <int N>
__device__ inline void sort_keys(unsigned long long *key) {
    for (int k = 2; k <= N; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < N / 2; t += 256) {
                const int lo = (t / j) * 2 * j + t % j, hi = lo + j;
                const unsigned long long x = key[lo], y = key[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    key[lo] = y;
                    key[hi] = x;
                }
            }
            __syncthreads();
        }
}

// A block's column list: its entries' offsets (vcol, from the block's first
// entry on) become the distinct ones, ascending, and idx the place of each
// entry's in that list; their number goes to blk.w, the largest and the sum to most.
static_assert(V_SORT == 2048, "11 bits of place, eight keys a thread");
__global__ void __launch_bounds__(256) k_v_local(int4 *__restrict__ blk, uint32_t *__restrict__ vcol,
                                                 uint16_t *__restrict__ idx, int *__restrict__ most) {
    __shared__ unsigned long long key[V_SORT];
    __shared__ int wsum[4];
    const int E0 = blk[blockIdx.x].z, len = blk[blockIdx.x + 1].z - E0, tid = threadIdx.x;
    for (int t = tid; t < V_SORT; t += 256)
        key[t] = t < len ? ((unsigned long long)vcol[E0 + t] << 11) | (unsigned)t : ~0ull;
    __syncthreads();
    sort_keys<V_SORT>(key);
    // a thread's eight keys: how many start a new column, and the ones before them
    auto first = [&](int t) { return t < len && (t == 0 || (key[t] >> 11) != (key[t - 1] >> 11)); };
    int mine = 0;
    for (int u = 0; u < 8; u++) mine += first(8 * tid + u);
    int incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if (tid % 64 >= o) incl += up;
    }
    if (tid % 64 == 63) wsum[tid / 64] = incl;
    __syncthreads();
    int rank = incl - mine, all = 0;
    for (int w = 0; w < 4; w++) {
        if (w < tid / 64) rank += wsum[w];
        all += wsum[w];
    }
    for (int u = 0; u < 8; u++) {
        const int t = 8 * tid + u;
        if (t >= len) break;
        if (first(t)) vcol[E0 + rank++] = (uint32_t)(key[t] >> 11);
        idx[E0 + (int)(key[t] & 2047)] = (uint16_t)(rank - 1);
    }
    if (tid == 0) {
        blk[blockIdx.x].w = all;
        atomicMax(most, all);
        atomicAdd(most + 1, all);
    }
}

// values at their places (ent: in the pairs)
template <class T>
__global__ void k_v_values(int64_t nnz, const double *__restrict__ val, const int32_t *__restrict__ place,
                           int2 *__restrict__ ent, T *__restrict__ vval) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const T v = sizeof(T) == 4 ? (T)f32_sat(val[e]) : (T)val[e];
    if (ent) ent[place[e]].y = __float_as_int((float)v);
    else vval[place[e]] = v;
}

// block b: the aggregates whose first entry lies in [b chunk, (b+1) chunk);
// the blocks past the last chunk (grid padding) are empty
__global__ void k_v_blocks(int64_t nc, int64_t nb, int64_t ngrid, int chunk, const int64_t *__restrict__ mptr,
                           const int32_t *__restrict__ ptr, int4 *__restrict__ blk) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b > ngrid) return;
    int64_t lo = nc;
    if (b < nb) {
        const int64_t target = b * (int64_t)chunk;
        int64_t hi = nc;
        lo = 0;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (ptr[mptr[mid]] < target) lo = mid + 1;
            else hi = mid;
        }
    }
    blk[b] = make_int4((int)lo, (int)mptr[lo], ptr[mptr[lo]], 0);
}

// the most entries and rows of a block
__global__ void k_v_most(int64_t ngrid, int align, const int4 *__restrict__ blk, int *__restrict__ most) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= ngrid) return;
    atomicMax(most, blk[b + 1].z - (blk[b].z & ~(align - 1)));
    atomicMax(most + 1, blk[b + 1].y - blk[b].y);
}

// the most entries of an aggregate
__global__ void k_v_most_agg(int64_t nc, const int64_t *__restrict__ mptr, const int32_t *__restrict__ ptr,
                             int *__restrict__ most) {
    const int64_t J = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int m = J < nc ? ptr[mptr[J + 1]] - ptr[mptr[J]] : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_down(m, o, 64));
    if (threadIdx.x % 64 == 0) atomicMax(most, m);
}

__global__ void k_v_child(int64_t n, const int32_t *__restrict__ mem, const int64_t *__restrict__ mptrf,
                          int2 *__restrict__ child) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t i = mem ? mem[p] : p;
    child[p] = make_int2((int)mptrf[i], (int)mptrf[i + 1]);
}

// the fine level's member lists in level 1's order, one thread per place of
// level 1 (mem1: the row there)
__global__ void k_v_count(int64_t n1, const int32_t *__restrict__ mem1, const int64_t *__restrict__ mptr,
                          int64_t *__restrict__ len) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n1) len[p] = mptr[mem1[p] + 1] - mptr[mem1[p]];
}

__global__ void k_v_members(int64_t n1, const int32_t *__restrict__ mem1, const int64_t *__restrict__ mptr,
                            const int32_t *__restrict__ mem, const int64_t *__restrict__ vmptr,
                            int32_t *__restrict__ vmem) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n1) return;
    int64_t o = vmptr[p];
    for (int64_t t = mptr[mem1[p]]; t < mptr[mem1[p] + 1]; t++) vmem[o++] = mem[t];
}

// The members of each stretch that a restriction block stages in LDS, put in
// ascending order (bitonic sort of (member, place in the stretch) keys); longer
// stretches keep the member lists' order.
static_assert(RESTRICT_LDS == 2048, "11 bits of place");
__global__ void __launch_bounds__(256) k_v_sort(int64_t n1, const int64_t *__restrict__ vmptr,
                                                int32_t *__restrict__ vmem, uint16_t *__restrict__ vslot) {
    __shared__ unsigned long long key[RESTRICT_LDS];
    const int64_t I0 = (int64_t)blockIdx.x * RESTRICT_TPB, I1 = I0 + RESTRICT_TPB < n1 ? I0 + RESTRICT_TPB : n1;
    const int64_t t0 = vmptr[I0];
    const int64_t len = vmptr[I1] - t0;
    if (len > RESTRICT_LDS) {
        for (int64_t t = threadIdx.x; t < len; t += 256) vslot[t0 + t] = 0;  // not read
        return;
    }
    for (int t = threadIdx.x; t < RESTRICT_LDS; t += 256)
        key[t] = t < len ? ((unsigned long long)(uint32_t)vmem[t0 + t] << 11) | (unsigned)t : ~0ull;
    __syncthreads();
    sort_keys<RESTRICT_LDS>(key);
    for (int t = threadIdx.x; t < len; t += 256) {
        vmem[t0 + t] = (int32_t)(key[t] >> 11);
        vslot[t0 + t] = (uint16_t)(key[t] & 2047);
    }
}

}  // namespace

// Products and row results of a block in LDS: at most this, so that two
// blocks share a CU at worst; levels with a larger aggregate keep the separate
// kernels.
constexpr size_t V_LDS_MAX = 60 << 10;
// Entries read past the last block (whole 128-entry runs from an even index;
// 256-entry ones from a multiple of four).
constexpr int64_t V_PAD = 256;

rich_status vlevel_order(Level &Lv, int64_t nc, bool mixed, DevAlloc &mem, bool *ok, hipStream_t s) {
    *ok = false;
    const size_t tsz = mixed ? sizeof(float) : sizeof(double);
    // 32-bit entry indices and byte offsets
    if (Lv.n == 0 || nc == 0 || Lv.nnz >= ((int64_t)1 << 31) - 4096 || Lv.n * (int64_t)tsz >= ((int64_t)1 << 32))
        return RICH_OK;
    VLevel &V = Lv.V;
    DevAlloc tmp;
    int64_t *len, *ptr, *stmp;
    int *most;
    int hm[4] = {0, 0, 0, 0};
    Slab scratch, rows, entries;
    scratch.add(&len, Lv.n);
    scratch.add(&ptr, Lv.n + 1);
    scratch.add(&stmp, scan_tmp_size(Lv.n));
    scratch.add(&most, 4);
    RICH_TRY(scratch.get(tmp));
    rows.add(&V.pos, Lv.n);
    rows.add(&V.ptr, Lv.n + 1);
    if (mixed) rows.add((float **)&V.invd, Lv.n);
    else rows.add((double **)&V.invd, Lv.n);
    RICH_TRY(rows.get(mem, &V.slab[0]));
    k_v_pos<<<nblocks(Lv.n), TPB, 0, s>>>(Lv.n, Lv.mem, Lv.rowptr, V.pos, len);
    LAUNCH_CHECK();
    RICH_TRY(scan_exclusive_i64(len, ptr, Lv.n, stmp, s));
    k_v_narrow<<<nblocks(Lv.n + 1), TPB, 0, s>>>(Lv.n + 1, ptr, V.ptr);
    RICH_TRY(launch_fill_i32(most, 0, 2, s));
    k_v_most_agg<<<nblocks(nc), TPB, 0, s>>>(nc, Lv.mptr, V.ptr, most);
    LAUNCH_CHECK();
    HIP_TRY(hipMemcpyAsync(hm, most, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    // A block takes whole aggregates from a stretch of `chunk` entries, so that
    // with the last one's overhang it fills 512 np.  Small levels have too few
    // blocks for more than np = 1 (a block's latency counts); the column lists of
    // np = 4 pay where the gather has outgrown the caches, in FP64 later (its
    // values' LDS doubles and leaves fewer blocks a CU).  Both sweeps of level 1, us,
    // by its entries, one np against the next:
    //   FP32  0.37 M 8.3 / 8.3, 0.56 M 9.0 / 8.9, 0.80 M 10.7 / 9.6, 1.9 M 17.2 / 14.9
    //   FP64  0.37 M 8.6 / 8.6, 0.56 M 9.3 / 9.7, 0.80 M 11.8 / 10.5, 1.9 M 19.8 / 16.9
    //   FP32 (2 / 4)  4.5 M 25.0 / 26.0, 10.3 M 44.6 / 46.4, 13.6 M 64.9 / 59.6, 36.6 M 203 / 155
    //   FP64 (2 / 4)  4.5 M 28.4 / 40.2, 15.4 M 115 / 124, 19.6 M 152 / 153, 24.5 M 193 / 187
    const int64_t local = (int64_t)(mixed ? 12 : 20) << 20, pairs2 = (int64_t)5 << 17;
    V.np = Lv.nnz >= local ? V_LOCAL : Lv.nnz >= pairs2 ? 2 : 1;
    // Where a large level's blocks would not fit the column sort, two.
    if (V.np == V_LOCAL && hm[0] + 3 > V_SORT - 256) V.np = 2;
    const int align = V.np == V_LOCAL ? 4 : 2, run = V.np == V_LOCAL ? 256 : 128;
    const int chunk = std::max(512 * V.np - hm[0] - align + 1, 256);
    const int64_t nb = (Lv.nnz + chunk - 1) / chunk, ngrid = xcd_grid(nb, 1);
    const bool pairs = mixed && V.np != V_LOCAL;
    entries.add(&V.blk, ngrid + 1);
    entries.add(&V.place, Lv.nnz);
    if (pairs) {
        entries.add(&V.ent, Lv.nnz + V_PAD);
        entries.add(&V.off, Lv.nnz);
    } else {
        entries.add(&V.col, Lv.nnz + V_PAD);
        if (mixed) entries.add((float **)&V.val, Lv.nnz + V_PAD);
        else entries.add((double **)&V.val, Lv.nnz + V_PAD);
        if (V.np == V_LOCAL) entries.add(&V.idx, Lv.nnz + V_PAD);
    }
    RICH_TRY(entries.get(mem, &V.slab[1]));
    k_v_blocks<<<nblocks(ngrid + 1), TPB, 0, s>>>(nc, nb, ngrid, chunk, Lv.mptr, V.ptr, V.blk);
    RICH_TRY(launch_fill_i32(most, 0, 4, s));
    k_v_most<<<nblocks(ngrid), TPB, 0, s>>>(ngrid, align, V.blk, most);
    LAUNCH_CHECK();
    if (pairs) {
        RICH_TRY(launch_fill_i32((int32_t *)(V.ent + Lv.nnz), 0, 2 * V_PAD, s));
    } else {
        RICH_TRY(launch_fill_i32((int32_t *)(V.col + Lv.nnz), 0, V_PAD, s));
        RICH_TRY(launch_fill_i32((int32_t *)((char *)V.val + Lv.nnz * tsz), 0, V_PAD * (int64_t)(tsz / 4), s));
    }
    k_v_columns<<<nblocks(Lv.n), TPB, 0, s>>>(Lv.n, (uint32_t)tsz, Lv.mem, Lv.rowptr, Lv.col, V.pos, V.ptr, V.place,
                                              V.off, V.ent, V.col);
    LAUNCH_CHECK();
    if (V.np == V_LOCAL) {
        RICH_TRY(launch_fill_i32((int32_t *)(V.idx + (Lv.nnz & ~(int64_t)1)), 0, V_PAD / 2, s));
        k_v_local<<<(unsigned)ngrid, 256, 0, s>>>(V.blk, V.col, V.idx, most + 2);
        LAUNCH_CHECK();
    }
    HIP_TRY(hipMemcpyAsync(hm, most, sizeof(hm), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    V.nblk = (int)ngrid;
    V.lds_ent = (hm[0] + run - 1) / run * run;
    V.lds_row = hm[1];
    V.nlist = hm[3];
    V.lds = (unsigned)(((size_t)(V.lds_ent + hm[1] + hm[2]) * tsz + 15) & ~(size_t)15);
    if (V.lds > V_LDS_MAX) return RICH_OK;
    const int64_t mean = Lv.nnz / Lv.n;
    V.g = mean < 8 ? 1 : mean < 16 ? 2 : mean < 32 ? 4 : 8;
    LAUNCH_CHECK();
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    *ok = true;
    return RICH_OK;
}

rich_status vlevel_child(Level &Lv, const Level &Lf, bool ordered, DevAlloc &mem, hipStream_t s) {
    RICH_TRY(mem.get(&Lv.V.child, Lv.n));
    k_v_child<<<nblocks(Lv.n), TPB, 0, s>>>(Lv.n, ordered ? Lv.mem : nullptr, Lf.mptr, Lv.V.child);
    LAUNCH_CHECK();
    return RICH_OK;
}

rich_status vlevel_fine(Level &L0, const Level &L1, DevAlloc &mem, hipStream_t s) {
    DevAlloc tmp;
    int64_t *len, *stmp;
    Slab scratch, lists;
    scratch.add(&len, L1.n);
    scratch.add(&stmp, scan_tmp_size(L1.n));
    RICH_TRY(scratch.get(tmp));
    lists.add(&L0.vmptr, L1.n + 1);
    lists.add(&L0.vmem, L0.n);
    lists.add(&L0.vslot, L0.n);
    RICH_TRY(lists.get(mem));
    k_v_count<<<nblocks(L1.n), TPB, 0, s>>>(L1.n, L1.mem, L0.mptr, len);
    LAUNCH_CHECK();
    RICH_TRY(scan_exclusive_i64(len, L0.vmptr, L1.n, stmp, s));
    k_v_members<<<nblocks(L1.n), TPB, 0, s>>>(L1.n, L1.mem, L0.mptr, L0.mem, L0.vmptr, L0.vmem);
    k_v_sort<<<nblocks(L1.n, RESTRICT_TPB), 256, 0, s>>>(L1.n, L0.vmptr, L0.vmem, L0.vslot);
    LAUNCH_CHECK();
    HIP_TRY(hipStreamSynchronize(s));  // tmp is freed on return
    return RICH_OK;
}

rich_status vlevel_values(Level &Lv, bool mixed, hipStream_t s) {
    const VLevel &V = Lv.V;
    if (mixed) k_v_values<float><<<nblocks(Lv.nnz), TPB, 0, s>>>(Lv.nnz, Lv.val, V.place, V.ent, (float *)V.val);
    else k_v_values<double><<<nblocks(Lv.nnz), TPB, 0, s>>>(Lv.nnz, Lv.val, V.place, nullptr, (double *)V.val);
    LAUNCH_CHECK();
    return RICH_OK;
}

// --------------------------------------------------------------- launchers
static void entries_of(const VLevel &V, VArgs<float> *a) { a->ent.e = V.ent; }
static void entries_of(const VLevel &V, VArgs<double> *a) { a->ent = {V.col, (const double *)V.val}; }
template <class T>
static void set_level(const VLevel &V, VArgs<T> *a) {
    a->blk = V.blk;
    a->ptr = V.ptr;
    entries_of(V, a);
    a->loc = {V.idx, (const T *)V.val};
    a->list = V.col;
    a->lds_ent = V.lds_ent;
    a->lds_row = V.lds_row;
}

template <class T>
static VArgs<T> down_args(const Level *L, int l, int nlev) {
    const Level &Lv = L[l], &Lc = L[l + 1];
    VArgs<T> a;
    memset(&a, 0, sizeof(a));
    set_level(Lv.V, &a);
    a.b = (const T *)Lv.b;
    a.v = (const T *)Lv.x;
    a.mptr = Lv.mptr;
    a.bc = (T *)Lc.b;
    if (l + 1 < nlev - 1) {
        a.pos = Lc.V.pos;
        a.invdc = (const T *)Lc.V.invd;
        a.x0c = (T *)Lc.x;
    }
    return a;
}

template <class T>
static VArgs<T> up_args(const Level *L, int l) {
    const Level &Lv = L[l];
    VArgs<T> a;
    memset(&a, 0, sizeof(a));
    set_level(Lv.V, &a);
    a.b = (const T *)Lv.b;
    a.v = (const T *)Lv.r;
    a.invd = (const T *)Lv.V.invd;
    if (l == 1) {
        a.x = (T *)Lv.x;
        a.mem = Lv.mem;
    } else {
        a.child = Lv.V.child;
        a.x0f = (const T *)L[l - 1].x;
        a.xtf = (T *)L[l - 1].r;
    }
    return a;
}

// f(np, g) with the level's split as compile-time constants
template <class F>
static void with_split(const VLevel &V, F &&f) {
    auto by_g = [&](auto np) {
        switch (V.g) {
        case 1: f(np, std::integral_constant<int, 1>()); break;
        case 2: f(np, std::integral_constant<int, 2>()); break;
        case 4: f(np, std::integral_constant<int, 4>()); break;
        default: f(np, std::integral_constant<int, 8>()); break;
        }
    };
    if (V.np == 4) by_g(std::integral_constant<int, 4>());
    else if (V.np == 2) by_g(std::integral_constant<int, 2>());
    else by_g(std::integral_constant<int, 1>());
}

template <class T, bool UP>
static void vlevel_launch(const VLevel &V, const VArgs<T> &a, hipStream_t s) {
    with_split(V, [&](auto np, auto g) {
        k_vlevel<np(), g(), T, UP><<<(unsigned)V.nblk, 256, V.lds, s>>>(a);
    });
}

template <class T>
rich_status launch_vdown(const Level *L, int l, int nlev, hipStream_t s) {
    vlevel_launch<T, false>(L[l].V, down_args<T>(L, l, nlev), s);
    LAUNCH_CHECK();
    return RICH_OK;
}
template <class T>
rich_status launch_vup(const Level *L, int l, hipStream_t s) {
    vlevel_launch<T, true>(L[l].V, up_args<T>(L, l), s);
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class T>
static GemvArgs<T, T> gemv_args(const Level *L, int nlev, const T *Ainv, bool prolong) {
    const Level &Lc = L[nlev - 1];
    GemvArgs<T, T> g;
    memset(&g, 0, sizeof(g));
    g.Ainv = Ainv;
    g.b = (const T *)Lc.b;
    g.n = Lc.n;
    g.x = (T *)Lc.x;
    if (prolong) {
        g.child = Lc.V.child;
        g.x0f = (const T *)L[nlev - 2].x;
        g.xtf = (T *)L[nlev - 2].r;
    }
    return g;
}

template <class TB, class T>
rich_status launch_dense_gemv(const T *Ainv, const TB *b, T *x, int64_t n, hipStream_t s) {
    if (n == 0) return RICH_OK;
    k_dense_gemv<TB, T><<<nblocks(n * 64), TPB, 0, s>>>(GemvArgs<TB, T>{Ainv, b, n, x, nullptr, nullptr, nullptr});
    LAUNCH_CHECK();
    return RICH_OK;
}
template rich_status launch_dense_gemv<double, double>(const double *, const double *, double *, int64_t, hipStream_t);
template rich_status launch_dense_gemv<double, float>(const float *, const double *, float *, int64_t, hipStream_t);
template rich_status launch_dense_gemv<float, float>(const float *, const float *, float *, int64_t, hipStream_t);

template <class T>
rich_status launch_vgemv(const Level *L, int nlev, const T *Ainv, hipStream_t s) {
    k_dense_gemv<T, T><<<nblocks(L[nlev - 1].n * 64), TPB, 0, s>>>(gemv_args<T>(L, nlev, Ainv, true));
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class T>
rich_status launch_vprolong(const Level *L, int nlev, hipStream_t s) {
    const Level &Lc = L[nlev - 1];
    k_v_prolong<T><<<nblocks(Lc.n), TPB, 0, s>>>(Lc.n, (const T *)Lc.x, Lc.V.child, (const T *)L[nlev - 2].x,
                                                 (T *)L[nlev - 2].r);
    LAUNCH_CHECK();
    return RICH_OK;
}

template <class T, bool UP>
static rich_status vlevel_batch(const std::vector<VItem<T>> &v, int l, hipStream_t s, WorkQueue *q) {
    // one launch for the simulations whose level takes the same split
    std::vector<char> done(v.size(), 0);
    for (size_t first = 0; first < v.size(); first++) {
        if (done[first] || !v[first].ordered || l >= v[first].nlev - 1) continue;
        const VLevel &V = v[first].L[l].V;
        std::vector<VArgs<T>> a;
        std::vector<unsigned> nb;
        unsigned lds = 0;
        for (size_t i = first; i < v.size(); i++) {
            if (done[i] || !v[i].ordered || l >= v[i].nlev - 1) continue;
            const VLevel &W = v[i].L[l].V;
            if (W.np != V.np || W.g != V.g) continue;
            done[i] = 1;
            if constexpr (UP) a.push_back(up_args<T>(v[i].L, l));
            else a.push_back(down_args<T>(v[i].L, l, v[i].nlev));
            nb.push_back((unsigned)W.nblk);
            lds = std::max(lds, W.lds);
        }
        rich_status st = RICH_OK;
        with_split(V, [&](auto np, auto g) {
            st = launch_batches(a, nb, [&](const Batch<VArgs<T>> &bt, unsigned grid) {
                k_vlevel_batch<np(), g(), T, UP><<<grid, 256, lds, s>>>(bt);
            }, q);
        });
        RICH_TRY(st);
    }
    return RICH_OK;
}

template <class T>
rich_status launch_vdown_batch(const std::vector<VItem<T>> &v, int l, hipStream_t s, WorkQueue *q) {
    return vlevel_batch<T, false>(v, l, s, q);
}
template <class T>
rich_status launch_vup_batch(const std::vector<VItem<T>> &v, int l, hipStream_t s, WorkQueue *q) {
    return vlevel_batch<T, true>(v, l, s, q);
}

template <class T>
rich_status launch_vgemv_batch(const std::vector<VItem<T>> &v, hipStream_t s, WorkQueue *q) {
    std::vector<GemvArgs<T, T>> a;
    std::vector<unsigned> nb;
    for (const auto &it : v) {
        a.push_back(gemv_args<T>(it.L, it.nlev, it.Ainv, it.ordered));
        nb.push_back(nblocks(it.L[it.nlev - 1].n * 64));
    }
    return launch_batches(a, nb, [&](const Batch<GemvArgs<T, T>> &bt, unsigned g) {
        k_dense_gemv_batch<T><<<g, TPB, 0, s>>>(bt);
    }, q);
}

#define INST_V(T)                                                                                      \
    template rich_status launch_vdown<T>(const Level *, int, int, hipStream_t);                        \
    template rich_status launch_vup<T>(const Level *, int, hipStream_t);                               \
    template rich_status launch_vgemv<T>(const Level *, int, const T *, hipStream_t);                  \
    template rich_status launch_vprolong<T>(const Level *, int, hipStream_t);                          \
    template rich_status launch_vdown_batch<T>(const std::vector<VItem<T>> &, int, hipStream_t, WorkQueue *); \
    template rich_status launch_vup_batch<T>(const std::vector<VItem<T>> &, int, hipStream_t, WorkQueue *);   \
    template rich_status launch_vgemv_batch<T>(const std::vector<VItem<T>> &, hipStream_t, WorkQueue *);
INST_V(double)
INST_V(float)

}  // namespace rich
