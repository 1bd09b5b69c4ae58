// Gradients of a loss L with dL/dC = G on C's stored entries, with respect to
// the stored values of A and B (sparsity patterns fixed). Both are sampled
// sparse products over the same product space as the forward pass:
//   dB(k,j) = sum over stored A(i,k), in A's storage order, of A(i,k) G(i,j)
//   dA(i,k) = sum over stored B(k,j), j ascending,          of G(i,j) B(k,j)
// Every term is rounded on its own and the terms of one entry are added in the
// stated order (no fused multiply-add), so the result is reproducible and
// matches a plain sequential loop bit for bit.
//
// Every term is one product of the forward pass: stored B entry t of column j
// times the u-th entry of A's column bri[t]. A view built once per plan
// records, in product order, the place of every product's G(i,j) among C's
// entries (gpos, by binary search of C's sorted rows); per stored B entry its
// first product (pofs) and the first of its terms of dA (woff), and the entries
// of every row of B by ascending column; per stored A entry its terms of dA.
//
// Two forms, the same sums. Two passes over the products: the first walks them
// in product order, where a column's G values lie together; it loads G once,
// adds up dB and writes the terms G(i,j) B(k,j) of dA grouped by A's column,
// entry after entry of B's row k in ascending j; the second adds up dA from
// contiguous blocks. Or one launch with a thread per stored entry, which
// gathers G for its own list: half the launches and no terms in memory, but G is
// read twice, for dA all over C, and the longest list sets the time (6.4 M
// float products, 8 per entry: 87 us, in two passes 31 + 8; 5 M double products
// of power-law columns: 324 us, in two passes 88 + 11). bw_two_passes chooses.
// Where it asks for two passes but the terms have no space, dB keeps its pass and
// dA is formed in the one launch.
#include <algorithm>
#include <cmath>

#include "devutil.h"

namespace spg {

namespace {

// largest j in [0, n) with cp[j] <= t (columns may be empty)
__device__ __forceinline__ int column_of(const int32_t *cp, int n, int t) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (cp[mid] <= t) lo = mid;
        else hi = mid;
    }
    return lo;
}

// A wavefront's 64 consecutive stored B entries and their products, which are
// consecutive too, kBwN at a time: lane l takes positions 64 r + l. Each entry
// with products in the chunk gets a rank; bit p of `bits` set means that a new
// entry starts at position p + 1, so the bits below a position count its
// entry's rank.
constexpr int kBwKpl = 8, kBwN = 64 * kBwKpl;

__device__ __forceinline__ void bw_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct Chunk {
    int lo, hi;  // the lane's entry holds positions [lo, hi) of the chunk
    int rank;    // its rank (where hi > lo)
    int n;       // products in the chunk
};

__device__ __forceinline__ Chunk chunk_of(long long c0, long long total, long long o, int z,
                                          unsigned *bits, int lane) {
    Chunk c;
    c.n = (int)max(0ll, min((long long)kBwN, total - c0));
    c.lo = (int)min(max(o - c0, 0ll), (long long)kBwN);
    c.hi = (int)min(max(o + z - c0, 0ll), (long long)kBwN);
    const unsigned long long has = ballot(c.hi > c.lo);
    c.rank = popc64(has & mask_lt());
    if (lane < kBwN / 32) bits[lane] = 0;
    bw_sync();
    if (c.hi > c.lo && c.lo > 0) atomicOr(&bits[(c.lo - 1) >> 5], 1u << ((c.lo - 1) & 31));
    bw_sync();
    return c;
}

// ranks of the lane's positions
__device__ __forceinline__ void ranks_of(const unsigned *bits, int (&rk)[kBwKpl]) {
    int cum = 0;
#pragma unroll
    for (int r = 0; r < kBwKpl; ++r) {
        const unsigned lo = __builtin_amdgcn_readfirstlane(bits[2 * r]);
        const unsigned hi = __builtin_amdgcn_readfirstlane(bits[2 * r + 1]);
        rk[r] = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, (unsigned)cum));
        cum += __builtin_popcount(lo) + __builtin_popcount(hi);
    }
}

// ---------------------------------------------------------------- first pass
// dB (if db), and the terms of dA (if w). Bound by the loads of gpos, A's
// columns and G (all contiguous per entry) and the stores of the terms; where
// long A columns meet in one wavefront (7 chunks among 1 M entries of a power
// law), by its chain of chunks, so a chunk's loads are in flight while the one
// before it is summed.
template <typename V>
__global__ __launch_bounds__(64) void k_grad_b(BwView v, int nnzb, const V *__restrict__ av,
                                               const V *__restrict__ bv,
                                               const V *__restrict__ gv, V *__restrict__ db,
                                               V *__restrict__ w, int *err) {
    __shared__ unsigned bits[2][kBwN / 32];  // of this chunk and the next
    __shared__ int s_q[2][64];
    __shared__ long long s_w[2][64];
    __shared__ V s_b[2][64];
    __shared__ V val[kBwN];
    const int lane = threadIdx.x;
    int bad = 0;
    const int t = blockIdx.x * 64 + lane;
    int2 e = make_int2(0, 0);
    long long wo = 0;
    V bval = V(0);
    const uint32_t *gpos = v.gpos + v.pofs[blockIdx.x * 64];
    if (t < nnzb) {
        e = v.E[t];
        if (w) {
            wo = v.woff[t];
            bval = bv[t];
        }
    }
    const long long inc = wave_incl_scan64(e.y), o = inc - e.y, total = wave_last64(inc);
    uint32_t gp[kBwKpl];  // the places of a chunk's products, loaded a chunk ahead
    V a[kBwKpl], g[kBwKpl];
    Chunk c;
    auto places = [&](long long c0) {
#pragma unroll
        for (int r = 0; r < kBwKpl; ++r) {
            const long long p = c0 + r * 64 + lane;
            gp[r] = p < total ? gpos[p] : 0u;
        }
    };
    auto load = [&](long long c0, int x) {
        c = chunk_of(c0, total, o, e.y, bits[x], lane);
        if (c.hi > c.lo) {
            s_q[x][c.rank] = e.x + (int)(c0 - o);
            if (w) {
                s_w[x][c.rank] = wo + (c0 - o);
                s_b[x][c.rank] = bval;
            }
        }
        bw_sync();
        int rk[kBwKpl];
        ranks_of(bits[x], rk);
#pragma unroll
        for (int r = 0; r < kBwKpl; ++r) {
            const int p = r * 64 + lane;
            const bool in = p < c.n;
            const bool ok = (long long)gp[r] < v.nnzc;
            bad |= in && !ok;
            a[r] = in && db ? av[s_q[x][rk[r]] + p] : V(0);
            g[r] = in && ok ? gv[gp[r]] : V(0);
        }
        places(c0 + kBwN);
    };
    V acc = V(0);
    places(0);
    load(0, 0);
    int x = 0;
    for (long long c0 = 0; c0 < total; c0 += kBwN, x ^= 1) {
        const Chunk d = c;
        int rk[kBwKpl];
        ranks_of(bits[x], rk);
#pragma unroll
        for (int r = 0; r < kBwKpl; ++r) {
            const int p = r * 64 + lane;
            if (p < d.n) {
                if (w) w[s_w[x][rk[r]] + p] = g[r] * s_b[x][rk[r]];
                if (db) val[p] = a[r] * g[r];
            }
        }
        if (c0 + kBwN < total) load(c0 + kBwN, x ^ 1);
        bw_sync();
        if (db) {
            // the entry's terms in order; a long list waits neither on a read
            // (the next U are in flight beside the adds) nor on masks
            constexpr int U = 8;
            int i = d.lo;
            V q[2][U];
            auto read = [&](V (&y)[U], int at) {
                const V *n = &val[min(at, kBwN - U)];
#pragma unroll
                for (int u = 0; u < U; ++u) y[u] = n[u];
            };
            auto add = [&](const V (&y)[U]) {
#pragma unroll
                for (int u = 0; u < U; ++u) acc = acc + y[u];
            };
            if (i + 2 * U <= d.hi) {
                read(q[0], i);
                read(q[1], i + U);
                for (; i + 2 * U <= d.hi; i += 2 * U) {
                    add(q[0]);
                    read(q[0], i + 2 * U);
                    add(q[1]);
                    read(q[1], i + 3 * U);
                }
            }
            for (; i < d.hi; i += U) {
                read(q[0], i);
                const int skip = i - min(i, kBwN - U);  // read at the buffer's end: shifted
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u >= skip && i + u - skip < d.hi) acc = acc + q[0][u];
            }
        }
        bw_sync();
    }
    if (db && t < nnzb) db[t] = acc;
    if (bad) atomicOr(err, ERR_CSC);
}

// ---------------------------------------------------------------- second pass
// dA: one thread per stored A entry; entries of one A column read consecutive
// terms.
template <typename V>
__global__ __launch_bounds__(kBlock) void k_grad_a(const int4 *__restrict__ aview, int nnza,
                                                   const V *__restrict__ w, V *__restrict__ da) {
    constexpr int U = 8;  // terms whose loads are issued together
    const int q = blockIdx.x * kBlock + threadIdx.x;
    if (q >= nnza) return;
    const int4 x = aview[q];
    const V *p = w + (long long)(((unsigned long long)(unsigned)x.y << 32) | (unsigned)x.x);
    const int deg = x.z, z = x.w;
    V acc = V(0);
    int r = 0;
    for (; r + U <= deg; r += U) {
        V t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = p[(long long)(r + u) * z];
#pragma unroll
        for (int u = 0; u < U; ++u) acc = acc + t[u];
    }
    if (r < deg) {
        V t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = r + u < deg ? p[(long long)(r + u) * z] : V(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (r + u < deg) acc = acc + t[u];
    }
    da[q] = acc;
}

// ---------------------------------------------------------------- one launch
// One thread per stored entry: blocks [0, nbw) dB, the others dA. Bound by the
// gathers of G and, where a list is long, by its chain of them, so kBwUnroll
// terms' loads are in flight together.
constexpr int kBwUnroll = 4;

template <typename V>
__device__ __forceinline__ V g_at(const V *__restrict__ gv, long long nnzc, uint32_t at, int &bad) {
    if ((long long)at < nnzc) return gv[at];
    bad = 1;
    return V(0);
}

template <typename V>
__global__ __launch_bounds__(kBlock) void k_grad(BwView v, int nnza, int nnzb, int nbw,
                                                 const V *__restrict__ av,
                                                 const V *__restrict__ bv,
                                                 const V *__restrict__ gv, V *__restrict__ da,
                                                 V *__restrict__ db, int *err) {
    constexpr int U = kBwUnroll;
    int bad = 0;
    V acc = V(0);
    if ((int)blockIdx.x < nbw) {
        const int t = blockIdx.x * kBlock + threadIdx.x;
        if (t >= nnzb) return;
        const int2 e = v.E[t];
        const V *__restrict__ ap = av + e.x;
        const uint32_t *__restrict__ gp = v.gpos + v.pofs[t];
        int u = 0;
        for (; u + U <= e.y; u += U) {
            V a[U], g[U];
            uint32_t at[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                a[q] = ap[u + q];
                at[q] = gp[u + q];
            }
#pragma unroll
            for (int q = 0; q < U; ++q) g[q] = g_at(gv, v.nnzc, at[q], bad);
#pragma unroll
            for (int q = 0; q < U; ++q) acc = acc + a[q] * g[q];
        }
        for (; u < e.y; ++u) acc = acc + ap[u] * g_at(gv, v.nnzc, gp[u], bad);
        db[t] = acc;
    } else {
        const int q = (blockIdx.x - nbw) * kBlock + threadIdx.x;
        if (q >= nnza) return;
        const int2 x = v.arow[q];
        const int r1 = v.rowptr[x.x + 1];
        const uint32_t *__restrict__ gp = v.gpos + x.y;
        int r = v.rowptr[x.x];
        for (; r + U <= r1; r += U) {
            int t[U];
            long long pf[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t[u] = v.rowent[r + u];
                pf[u] = v.rowpofs[r + u];
            }
            uint32_t at[U];
            V b[U], g[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                at[u] = gp[pf[u]];
                b[u] = bv[t[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) g[u] = g_at(gv, v.nnzc, at[u], bad);
#pragma unroll
            for (int u = 0; u < U; ++u) acc = acc + g[u] * b[u];
        }
        for (; r < r1; ++r)
            acc = acc + g_at(gv, v.nnzc, gp[v.rowpofs[r]], bad) * bv[v.rowent[r]];
        da[q] = acc;
    }
    if (bad) atomicOr(err, ERR_CSC);
}

// ---------------------------------------------------------------- view construction
// per stored B entry: its arrival among its row's entries; counts per row
__global__ __launch_bounds__(kBlock) void k_bv_count(Prob p, int32_t *cnt, int32_t *arrival) {
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t < p.nnzb) arrival[t] = atomicAdd(&cnt[p.bri[t]], 1);
}

// Prefix sums in two launches. Blocks [0, nbt): the lengths of the A columns
// that the stored B entries select (pofs); the others, over B's rows k: the
// entries before (rowptr) and the terms of dA before (wbase, deg_k z_k each).
// The last block also finds the longest lists of dB (z_k) and dA (deg_k), from
// the blocks' own, and publishes them. (A device-wide maximum by atomics, one a
// wavefront, took 20 us for 180,000 entries: all of them meet in one word.)
struct BvScan {
    const int2 *E;
    int nnzb, nrows, nbt;
    const int32_t *cnt, *acp;
    long long *bsum, *bsum2;  // per block: pofs or wbase sums; rowptr sums
    int2 *blong;              // per block: longest lists of dB, dA
    long long *pofs, *wbase;
    int32_t *rowptr;
};
constexpr int kBvPer = 4, kBvBlock = kBvPer * kBlock;

__device__ __forceinline__ void bv_items(const BvScan &a, int b, long long (&x)[kBvPer],
                                         long long (&y)[kBvPer], int2 &most) {
    most = make_int2(0, 0);
#pragma unroll
    for (int u = 0; u < kBvPer; ++u) {
        x[u] = y[u] = 0;
        if (b < a.nbt) {
            const int t = b * kBvBlock + threadIdx.x * kBvPer + u;
            if (t < a.nnzb) x[u] = a.E[t].y;
        } else {
            const int k = (b - a.nbt) * kBvBlock + threadIdx.x * kBvPer + u;
            if (k < a.nrows) {
                const int z = a.acp[k + 1] - a.acp[k];
                y[u] = a.cnt[k];
                x[u] = y[u] * z;
                if (y[u] > 0) most.x = max(most.x, z);
                if (y[u] > 0 && z > 0) most.y = max(most.y, (int)y[u]);
            }
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_bv_sums(BvScan a) {
    __shared__ long long s[2][kBlock / 64];
    __shared__ int2 s_most[kBlock / 64];
    long long x[kBvPer], y[kBvPer], sx = 0, sy = 0;
    int2 most;
    bv_items(a, blockIdx.x, x, y, most);
#pragma unroll
    for (int u = 0; u < kBvPer; ++u) {
        sx += x[u];
        sy += y[u];
    }
    sx = wave_sum64(sx);
    sy = wave_sum64(sy);
    most.x = wave_incl_max(most.x);
    most.y = wave_incl_max(most.y);
    if ((threadIdx.x & 63) == 63) {
        s[0][threadIdx.x >> 6] = sx;
        s[1][threadIdx.x >> 6] = sy;
        s_most[threadIdx.x >> 6] = most;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sx = sy = 0;
        most = make_int2(0, 0);
        for (int q = 0; q < kBlock / 64; ++q) {
            sx += s[0][q];
            sy += s[1][q];
            most.x = max(most.x, s_most[q].x);
            most.y = max(most.y, s_most[q].y);
        }
        a.bsum[blockIdx.x] = sx;
        a.bsum2[blockIdx.x] = sy;
        a.blong[blockIdx.x] = most;
    }
}

__global__ __launch_bounds__(kBlock) void k_bv_scan(BvScan a, PubArgs pub) {
    __shared__ long long tmp[kBlock / 64 + 1];
    const int b = blockIdx.x, first = b < a.nbt ? 0 : a.nbt;
    if (pub.dst && b == (int)gridDim.x - 1 && threadIdx.x < 64) {
        int2 most = make_int2(0, 0);
        for (int q = a.nbt + (int)threadIdx.x; q <= b; q += 64) {
            most.x = max(most.x, a.blong[q].x);
            most.y = max(most.y, a.blong[q].y);
        }
        most.x = wave_incl_max(most.x);
        most.y = wave_incl_max(most.y);
        if (threadIdx.x == 63) {
            const unsigned long long tag = (unsigned long long)pub.seq << 32;
            __hip_atomic_store(&pub.dst[0], (unsigned)most.x | tag, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&pub.dst[1], (unsigned)most.y | tag, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    long long bx = 0, by = 0;  // sums of the earlier blocks of the same list
    for (int q = first + threadIdx.x; q < b; q += kBlock) {
        bx += a.bsum[q];
        by += a.bsum2[q];
    }
    long long x[kBvPer], y[kBvPer], sx = 0, sy = 0, tx, ty;
    int2 most;
    bv_items(a, b, x, y, most);
#pragma unroll
    for (int u = 0; u < kBvPer; ++u) {
        sx += x[u];
        sy += y[u];
    }
    (void)wg_excl_scan64<kBlock>(bx, tmp, tx);
    (void)wg_excl_scan64<kBlock>(by, tmp, ty);
    long long tot;
    long long rx = tx + wg_excl_scan64<kBlock>(sx, tmp, tot);
    long long ry = ty + wg_excl_scan64<kBlock>(sy, tmp, tot);
#pragma unroll
    for (int u = 0; u < kBvPer; ++u) {
        if (b < a.nbt) {
            const int t = b * kBvBlock + threadIdx.x * kBvPer + u;
            if (t < a.nnzb) a.pofs[t] = rx;
        } else {
            const int k = (b - a.nbt) * kBvBlock + threadIdx.x * kBvPer + u;
            if (k < a.nrows) {
                a.wbase[k] = rx;
                a.rowptr[k] = (int32_t)ry;
                if (k == a.nrows - 1) a.rowptr[a.nrows] = (int32_t)(ry + y[u]);
            }
        }
        rx += x[u];
        ry += y[u];
    }
}

// each row's entries in arrival order
__global__ __launch_bounds__(kBlock) void k_bv_fill(Prob p, const int32_t *rowptr,
                                                    const int32_t *arrival, int32_t *pos) {
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t < p.nnzb) pos[rowptr[p.bri[t]] + arrival[t]] = t;
}

// Blocks [0, nbt): every B entry's rank in its row by ascending column (the
// entries before it in B's storage, counted in the row's list: by its thread,
// or for rows above kBvCount entries by the whole wavefront), the row's sorted
// entries and the entry's terms of dA. The others: every A entry's terms.
constexpr int kBvCount = 64;
__global__ __launch_bounds__(kBlock) void k_bv_rank(Prob p, const int32_t *rowptr,
                                                    const int32_t *pos, const long long *wbase,
                                                    const long long *pofs, int nbt,
                                                    int32_t *rowent, long long *rowpofs,
                                                    long long *woff, int4 *aview, int2 *arow) {
    if ((int)blockIdx.x < nbt) {
        const int t = blockIdx.x * kBlock + threadIdx.x;
        const int k = t < p.nnzb ? p.bri[t] : -1;
        const int b = k >= 0 ? rowptr[k] : 0, e = k >= 0 ? rowptr[k + 1] : 0;
        int rank = 0;
        if (e - b <= kBvCount)
            for (int r = b; r < e; ++r) rank += pos[r] < t ? 1 : 0;
        for (unsigned long long m = ballot(e - b > kBvCount); m; m &= m - 1) {
            const int src = __builtin_ctzll(m);
            const int bt = __builtin_amdgcn_readlane(t, src);
            const int bb = __builtin_amdgcn_readlane(b, src);
            const int be = __builtin_amdgcn_readlane(e, src);
            int n = 0;
            for (int r = bb + lane_id(); r < be; r += 64) n += pos[r] < bt ? 1 : 0;
            n = wave_sum(n);
            if (lane_id() == src) rank = n;
        }
        if (k < 0) return;
        rowent[b + rank] = t;
        rowpofs[b + rank] = pofs[t];
        woff[t] = wbase[k] + (long long)rank * (p.acp[k + 1] - p.acp[k]);
    } else {
        const int q = (blockIdx.x - nbt) * kBlock + threadIdx.x;
        if (q >= p.nnza) return;
        const int k = column_of(p.acp, p.k, q), u = q - p.acp[k];
        const long long base = wbase[k] + u;
        aview[q] = make_int4((int)(unsigned)base, (int)(unsigned)((unsigned long long)base >> 32),
                             rowptr[k + 1] - rowptr[k], p.acp[k + 1] - p.acp[k]);
        arow[q] = make_int2(k, u);
    }
}

// the place of every product's row among C's entries (C's columns ascend: a
// binary search), products taken as in the first pass
__global__ __launch_bounds__(64) void k_bv_gpos(Prob p, const int2 *__restrict__ E,
                                                const long long *__restrict__ pofs,
                                                const int32_t *__restrict__ cri, long long nnzc,
                                                uint32_t *__restrict__ gpos, int *err) {
    __shared__ unsigned bits[kBwN / 32];
    __shared__ int s_q[64], s_lo[64], s_hi[64];
    const int lane = threadIdx.x;
    const int t = blockIdx.x * 64 + lane;
    const long long p0 = pofs[blockIdx.x * 64];
    int2 e = make_int2(0, 0);
    int c0 = 0, c1 = 0;
    if (t < p.nnzb) {
        e = E[t];
        const int j = column_of(p.bcp, p.n, t);
        c0 = p.ccp[j];
        c1 = p.ccp[j + 1];
        if (c0 < 0 || c1 < c0 || c1 > nnzc) c0 = c1 = 0;
    }
    const long long inc = wave_incl_scan64(e.y), o = inc - e.y, total = wave_last64(inc);
    int bad = 0;
    for (long long b0 = 0; b0 < total; b0 += kBwN) {
        const Chunk c = chunk_of(b0, total, o, e.y, bits, lane);
        if (c.hi > c.lo) {
            s_q[c.rank] = e.x + (int)(b0 - o);
            s_lo[c.rank] = c0;
            s_hi[c.rank] = c1;
        }
        bw_sync();
        int rk[kBwKpl], row[kBwKpl], lo[kBwKpl], hi[kBwKpl], end[kBwKpl];
        ranks_of(bits, rk);
#pragma unroll
        for (int r = 0; r < kBwKpl; ++r) {
            const int q = r * 64 + lane;
            const bool in = q < c.n;
            row[r] = in ? p.ari[s_q[rk[r]] + q] : 0;
            lo[r] = in ? s_lo[rk[r]] : 0;
            hi[r] = end[r] = in ? s_hi[rk[r]] : 0;
        }
        for (bool more = true; more;) {  // first position whose row is not below `row`
            int mid[kBwKpl], x[kBwKpl];
#pragma unroll
            for (int r = 0; r < kBwKpl; ++r) {
                mid[r] = lo[r] + ((hi[r] - lo[r]) >> 1);
                x[r] = lo[r] < hi[r] ? cri[mid[r]] : 0;
            }
            bool any = false;
#pragma unroll
            for (int r = 0; r < kBwKpl; ++r) {
                if (lo[r] < hi[r]) {
                    if (x[r] < row[r]) lo[r] = mid[r] + 1;
                    else hi[r] = mid[r];
                }
                any |= lo[r] < hi[r];
            }
            more = ballot(any) != 0;
        }
#pragma unroll
        for (int r = 0; r < kBwKpl; ++r) {
            const int q = r * 64 + lane;
            if (q >= c.n) continue;
            const bool ok = lo[r] < end[r] && cri[lo[r]] == row[r];
            bad |= !ok;  // C does not hold the product's row
            gpos[p0 + b0 + q] = ok ? (uint32_t)lo[r] : 0u;
        }
        bw_sync();
    }
    if (bad) atomicOr(err, ERR_CSC);
}

}  // namespace

// ---------------------------------------------------------------- launchers
int bw_scan_blocks(int nnzb, int nrows) { return ceil_div(nnzb, kBvBlock) + ceil_div(nrows, kBvBlock); }

hipError_t launch_bw_view(const Prob &p, const BwView &v, const BwBuild &b, const int32_t *cri,
                          int *err, const PubArgs &pub, hipStream_t s) {
    const int nrows = p.k;  // rows of B
    hipError_t e;
    // counts and the error word lie together
    if ((e = hipMemsetAsync(b.cnt, 0, b.clear_bytes, s))) return e;
    const int gt = ceil_div(p.nnzb, kBlock), ga = ceil_div(p.nnza, kBlock);
    if (gt > 0) hipLaunchKernelGGL(k_bv_count, dim3(gt), dim3(kBlock), 0, s, p, b.cnt, b.arrival);
    BvScan sc{v.E, p.nnzb, nrows, ceil_div(p.nnzb, kBvBlock), b.cnt, p.acp,
              b.bsum, b.bsum2, b.blong, b.pofs, b.wbase, b.rowptr};
    if (const int nb = bw_scan_blocks(p.nnzb, nrows)) {
        hipLaunchKernelGGL(k_bv_sums, dim3(nb), dim3(kBlock), 0, s, sc);
        hipLaunchKernelGGL(k_bv_scan, dim3(nb), dim3(kBlock), 0, s, sc, pub);
    }
    if (gt > 0)
        hipLaunchKernelGGL(k_bv_fill, dim3(gt), dim3(kBlock), 0, s, p, (const int32_t *)b.rowptr,
                           (const int32_t *)b.arrival, b.pos);
    if (gt + ga > 0)
        hipLaunchKernelGGL(k_bv_rank, dim3(gt + ga), dim3(kBlock), 0, s, p,
                           (const int32_t *)b.rowptr, (const int32_t *)b.pos,
                           (const long long *)b.wbase, (const long long *)b.pofs, gt, b.rowent,
                           b.rowpofs, b.woff, b.aview, b.arow);
    if (p.nnzb > 0)
        hipLaunchKernelGGL(k_bv_gpos, dim3(ceil_div(p.nnzb, 64)), dim3(64), 0, s, p, v.E,
                           (const long long *)b.pofs, cri, v.nnzc, b.gpos, err);
    return hipGetLastError();
}

// The form that is faster, from the sizes and the longest lists (unknown in a
// plan's first call, which takes the two passes: they never wait on one list).
// Estimates in us, fitted to both forms' times, dA and dB together and each
// alone, in both types, on 114 products of 2 thousand to 47 million (uniform,
// power-law, banded, block, stencil and clustered patterns, columns of 2 to
// 1000 entries). With r products per entry of C and z per stored B entry:
//   one launch   products x (a + b / r^1.75): of many products on an entry of G
//                most find it in a cache, one alone reads a line for it; or the
//                longest list's chain of gathers; or a launch, 5.2.
//   two passes   what the products and entries move; or a wavefront's chain of
//                chunks (64 z products, 512 each) and half of that; or two
//                launches, 8.8.
// Both gradients took the faster form on all 114, one alone on all but 5, which
// lose 15 to 35%.
// Measured (one launch, two passes; double): 5000 columns of 8 in A and B 7.2
// and 10.0 us, 50,000 59 and 30; 500 columns of 40 12.6 and 27.1, 1500 41.8 and
// 32.3; 20,000 columns of 20 in a band (r = 10) 35.5 and 55.6; a power law of
// 20,000 columns 161 and 37.
bool bw_two_passes(const BwShape &x, bool f64, bool need_a, bool need_b) {
    if (x.longest_a < 0) return true;
    const double p = 1e-6 * (double)x.products, nb = 1e-6 * x.nnzb;
    const double z = (double)x.products / std::max(x.nnzb, 1);
    const double r = (double)x.products / (double)std::max(x.nnzc, 1ll);
    const double alone = std::pow(r, -1.75);  // of the products, those that find no line of G
    const double ga = p * (1.8 + (f64 ? 12 : 9) * alone) + 10 * nb * alone;
    // (long columns of A: a wavefront's lists pass through more lines than the
    // first cache holds, and the larger G is the less the second one does)
    const double more_g = std::max(0.0, std::log2((double)x.nnzc * (f64 ? 8 : 4) / 2e6));
    const double gb = p * ((z < 25 ? 0.7 + 0.1 * z : 3.4 + 0.6 * more_g) + (f64 ? 5 : 2.5) * alone);
    const double chain_a = 0.17 * x.longest_a, chain_b = 0.09 * x.longest_b;
    const double more = std::max(0.0, z * 64 / kBwN - 1);  // chunks after a wavefront's first
    double one, two;
    if (need_a && need_b) {
        one = std::max({1.5 + ga + gb, chain_a, chain_b, 5.2});
        two = 7.3 + std::max((f64 ? 6.2 : 4.5) * p + (f64 ? 12 : 4.5) * nb,
                             (more > 0 ? 1.5 : 0) + 4.2 * more + (f64 ? 3 : 2) * p);
        two = std::max(two, 8.8);
    } else if (need_a) {
        one = std::max({ga, chain_a, 5.2});
        two = 7.3 + std::max((f64 ? 5.1 : 3.5) * p + (f64 ? 10 : 4) * nb,
                             3 * more + (f64 ? 2.2 : 1.5) * p);
        two = std::max(two, 8.8);
    } else {  // (the first pass alone)
        one = std::max({gb, chain_b, 5.2});
        two = 5.2 + std::max((f64 ? 3 : 2) * p + (f64 ? 5 : 2.5) * nb + more,
                             2 * more + (f64 ? 2 : 1.3) * p);
        two = std::max(two, 5.8);
    }
    // (one gradient alone: the estimates part less well, and the one launch is
    // the form that needs no space)
    return (need_a && need_b ? 1.0 : 1.08) * two < one;
}

template <typename V>
static hipError_t run_backward(const Prob &p, const BwView &v, BwForm form, void *terms,
                               const V *av, const V *bv, const V *gv, V *da, V *db, int *err,
                               hipStream_t s) {
    if (p.nnzb <= 0) db = nullptr;
    if (p.nnza <= 0) da = nullptr;
    const int nb = ceil_div(p.nnzb, kBlock), na = ceil_div(p.nnza, kBlock);
    if (form != BwForm::one) {
        V *w = da && form == BwForm::two ? (V *)terms : nullptr;
        if (p.nnzb > 0 && (db || w))
            hipLaunchKernelGGL(k_grad_b<V>, dim3(ceil_div(p.nnzb, 64)), dim3(64), 0, s, v, p.nnzb,
                               av, bv, gv, db, w, err);
        db = nullptr;
        if (da && w) {
            hipLaunchKernelGGL(k_grad_a<V>, dim3(na), dim3(kBlock), 0, s, v.aview, p.nnza,
                               (const V *)w, da);
            da = nullptr;
        }
    }
    if (da || db) {
        const int nbw = db ? nb : 0, naw = da ? na : 0;
        hipLaunchKernelGGL(k_grad<V>, dim3(nbw + naw), dim3(kBlock), 0, s, v, p.nnza, p.nnzb, nbw,
                           av, bv, gv, da, db, err);
    }
    return hipGetLastError();
}

hipError_t launch_backward(const Prob &p, const BwView &v, BwForm form, void *terms, bool f64,
                           const void *av, const void *bv, const void *gv, void *da, void *db,
                           int *err, hipStream_t s) {
    if (f64)
        return run_backward<double>(p, v, form, terms, (const double *)av, (const double *)bv,
                                    (const double *)gv, (double *)da, (double *)db, err, s);
    return run_backward<float>(p, v, form, terms, (const float *)av, (const float *)bv,
                               (const float *)gv, (float *)da, (float *)db, err, s);
}

}  // namespace spg
